"""Pair-block products of spaces with few nucleons of one species (GPU): target rows of a few states, short runs of
cores; widths of one and of several column tiles."""
import os

import numpy as np
import pytest

from gpu_common import pair, say, term_bound
from workloads import PF_ORBITS, SD_ORBITS, random_block, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIXED_PAR = ((0, 1, 1), (0, 2, 5), (0, 1, 3))  # both parities in one proton row
SPACES = {
    "pf21": (PF_ORBITS, 2, 1, 1, 0),
    "pf41": (PF_ORBITS, 4, 1, 1, 0),
    "pf14": (PF_ORBITS, 1, 4, 1, 0),
    "pf32": (PF_ORBITS, 3, 2, 1, 0),
    "pf22": (PF_ORBITS, 2, 2, 0, 0),
    "sd61": (SD_ORBITS, 6, 1, 1, 0),
    "mixpar31": (MIXED_PAR, 3, 1, 0, 0),
    "mixpar13": (MIXED_PAR, 1, 3, 0, 0),
}
WIDTHS = (1, 3, 4, 7, 16, 17, 24, 31, 33, 48, 64)


def _model(space, env, oracle=True):
    orbits, z, n, twoM, par = SPACES[space]
    spe = [0.4 * k - 1.1 for k in range(len(orbits))]
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        return pair(orbits, z, n, twoM, random_tbme(orbits, 11), spe, spe, par, oracle)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


def _check(space, env):
    """Each row within the per-term bound of its generated terms plus the additions of the slot sum (n_prot * n_neut
    slots of blocks of at most 64 pairs); the same call twice gives the same bits."""
    g, o = _model(space, env)
    z, n = SPACES[space][1:3]
    rng = np.random.default_rng(4)
    idx = np.unique(np.concatenate([rng.choice(o.dim, min(o.dim, 300), replace=False), [0, o.dim - 1]]))
    V = random_block(70, o.dim, max(WIDTHS))
    V32 = V.astype(np.float32)
    ref, bound = o.apply_rows(V, idx), term_bound(o, idx, V, extra=z * n + 64)
    ref32, bound32 = o.apply_rows(V32.astype(np.float64), idx), term_bound(o, idx, V32, fp32=True, extra=z * n + 64)
    for nb in WIDTHS:
        say("case", space, env, "nb", nb)
        for x, r, b in ((V, ref, bound), (V32, ref32, bound32)):
            v = torch.from_numpy(x[:, :nb].copy()).cuda()
            W = g.apply(v)
            assert torch.equal(W, g.apply(v))
            assert np.all(np.abs(W.cpu().numpy()[idx].astype(np.float64) - r[:, :nb]) <= b[:, :nb])


@pytest.mark.parametrize("space", SPACES)
def test_short_rows_match_oracle(space):
    _check(space, {"TRBL_PN_TILES": "2"})


@pytest.mark.parametrize("run", ["p", "n"])
@pytest.mark.parametrize("space", SPACES)
def test_runs_over_either_species(space, run):
    """Work items that run over proton or over neutron cores, whichever the space would take."""
    _check(space, {"TRBL_PN_TILES": "2", "TRBL_PN_RUN": run})


def test_runs_over_protons_beyond_24_bit_row_steps():
    """Columns of a block with 8 MiB rows: the rows of consecutive proton states, up to 4 rows apart, are 2^25 bytes
    away (64-bit row addresses), while the whole block stays below 4 GiB. The same columns packed give the same
    products; their sums over D products differ by at most gamma_D of sum |x| |H x| each."""
    g, _ = _model("pf21", {"TRBL_PN_TILES": "2", "TRBL_PN_RUN": "p"}, oracle=False)
    ld = 1 << 20
    assert 8 * ld * g.dim < (1 << 32) - (1 << 16)
    X = torch.zeros((g.dim, ld), dtype=torch.float64, device="cuda")
    cols = [0, 1, ld // 2, ld - 1]
    V = torch.from_numpy(random_block(3, g.dim, len(cols))).cuda()
    X[:, cols] = V
    say("expect on", tuple(X.shape))
    got = g.expect(X)
    ref, HV = g.expect(V), g.apply(V)
    u = 2.0 ** -53
    bound = 2 * g.dim * u / (1 - g.dim * u) * (V.abs() * HV.abs()).sum(0).cpu().numpy()
    assert np.all(np.abs(got[cols] - ref) <= bound)
