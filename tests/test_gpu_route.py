"""Which kernels a product takes (GPU): in spaces whose jump lists are the faster side the default product has the bits of
the jump-list product, elsewhere those of the pair blocks."""
import os

import pytest

from gpu_common import say
from workloads import PF_ORBITS, SD_ORBITS, random_block, random_tbme

import paper_1902_02064_amd as trbl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# shell, protons, neutrons, {row bytes: pair blocks taken}; rows of 32, 64, 72, 128 and 256 bytes
CASES = [
    ("sd", 3, 3, ()), ("sd", 3, 4, ()), ("sd", 4, 5, ()), ("sd", 6, 6, ()), ("pf", 2, 1, ()),  # jump lists
    ("sd", 4, 4, (72, 128)), ("sd", 4, 3, (72, 128)), ("sd", 2, 5, (72, 128)), ("sd", 5, 3, (64, 72, 128)),
    ("pf", 1, 3, (72, 128)), ("pf", 2, 2, ()),
    ("pf", 3, 1, (32, 64, 72, 128, 256)), ("pf", 1, 4, (32, 64, 72, 128, 256)), ("pf", 3, 3, (32, 64, 72, 128, 256)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s%d%d" % c[:3])
def test_route_by_space_and_row(case):
    shell, z, n, tiles = case
    orbits = SD_ORBITS if shell == "sd" else PF_ORBITS
    tb, spe = random_tbme(orbits, 5), [0.3 * k for k in range(len(orbits))]
    say("case", case)
    models = {}
    for env in ("", "0", "2"):
        if env:
            os.environ["TRBL_PN_TILES"] = env
        try:
            models[env] = trbl.Model(orbits, z, n, (z + n) % 2)
            models[env].set_hamiltonian(spe, spe, tb)
        finally:
            os.environ.pop("TRBL_PN_TILES", None)
    V = random_block(3, models[""].dim, 64)
    for dt in (torch.float64, torch.float32):
        for row in (32, 64, 72, 128, 256):
            x = torch.from_numpy(V[:, :8 * row // torch.finfo(dt).bits].copy()).to("cuda", dt)
            W = {env: g.apply(x) for env, g in models.items()}
            assert not torch.equal(W["0"], W["2"])  # the two sides add in different orders
            assert torch.equal(W[""], W["2" if row in tiles else "0"]), (dt, row)


@pytest.mark.parametrize("n", [5, 6])  # sectors of up to 1,651 and 3,952 states
def test_narrow_rows_of_wide_sectors(n):
    """Several batches and sectors of more than 2,048 neutron states: jump lists for rows of up to 32 bytes at widths of
    a power of two (FP32 from 4 columns on), pair blocks beyond."""
    tb, spe = random_tbme(PF_ORBITS, 5), [0.3 * k for k in range(4)]
    models = {}
    for env in ("", "0"):
        os.environ["TRBL_PN_BATCH"] = "2000000"
        if env:
            os.environ["TRBL_PN_TILES"] = env
        try:
            models[env] = trbl.Model(PF_ORBITS, 2, n, n % 2)
            models[env].set_hamiltonian(spe, spe, tb)
        finally:
            os.environ.pop("TRBL_PN_TILES", None)
            os.environ.pop("TRBL_PN_BATCH", None)
    V = torch.randn((models[""].dim, 8), dtype=torch.float64, generator=torch.Generator().manual_seed(1))
    for dt, lists in ((torch.float64, (1, 2, 4)), (torch.float32, (4, 8))):
        for nb in (1, 2, 3, 4, 5, 8):
            say("case", dt, nb)
            x = V[:, :nb].contiguous().to("cuda", dt)
            assert torch.equal(models[""].apply(x), models["0"].apply(x)) == (n == 6 and nb in lists), (dt, nb)
