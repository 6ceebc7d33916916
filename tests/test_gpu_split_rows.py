"""The jump-list rows kernel (GPU) with a row's groups shared by 2, 4 or 8 parts of a workgroup (the most parts are set
by TRBL_HV_SPLIT; small spaces take them by themselves) and with one part, two 12 KB buffers."""
import os

import numpy as np
import pytest

from gpu_common import pair, say, term_bound
from workloads import SD_ORBITS, SD_SPE, random_block, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# protons, neutrons, 2M: one row, rows of one and of several wavefronts, many rows, more neutrons than number columns
CASES = [(1, 1, 0), (2, 2, 0), (1, 6, 1), (6, 1, 1), (3, 4, 1), (2, 9, 1), (4, 4, 0)]


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("most", [1, 2, 4, 8])
def test_parts_match_oracle(case, most):
    """Within the rounding bound of the oracle's terms, with the parts' sums as further additions, at widths with and
    without whole 16-byte lanes and column tiles, in FP64 and FP32; twice the same call gives the same bits."""
    z, n, twoM = case
    say("case", case, "parts", most)
    saved = {k: os.environ.get(k) for k in ("TRBL_HV_SPLIT", "TRBL_PN_TILES")}
    os.environ.update(TRBL_HV_SPLIT=str(most), TRBL_PN_TILES="0")
    try:
        g, o = pair(SD_ORBITS, z, n, twoM, random_tbme(SD_ORBITS, 5), SD_SPE, SD_SPE)
        H = o.dense() if o.dim <= 4000 else None
        rows = np.arange(o.dim) if H is not None else np.random.default_rng(1).choice(o.dim, 300, replace=False)
        for nb in (1, 3, 4, 8, 16):
            V = random_block(90 + nb, o.dim, nb)
            for dt in (np.float64, np.float32):
                x = torch.from_numpy(V.astype(dt)).cuda()
                W = g.apply(x)
                assert torch.equal(W, g.apply(x))
                v = V.astype(dt).astype(np.float64)
                if H is not None:
                    ref = H @ v
                else:
                    ptr, col, val = o.rows_generated(rows)
                    ref = np.stack([val[ptr[r]:ptr[r + 1]] @ v[col[ptr[r]:ptr[r + 1]]] for r in range(len(rows))])
                b = term_bound(o, rows, v, fp32=dt is np.float32, extra=64)
                assert np.all(np.abs(W.cpu().numpy()[rows] - ref) <= b), (nb, dt)
    finally:
        for k, x in saved.items():
            if x is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = x
