"""Pair-block products of two-species spaces (GPU) over the column widths where their tiles change and over
several batches of proton cores, against the oracle; the 64-bit row addressing of wide blocks."""
import os

import numpy as np
import pytest

from gpu_common import pair, say, term_bound
from workloads import PF_ORBITS, SD_ORBITS, random_block, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIXED_PAR = ((0, 1, 1), (0, 2, 5), (0, 1, 3))  # both parities in one proton row

SPACES = {
    "sd32": (SD_ORBITS, 3, 2, 1, 0),
    "pf22": (PF_ORBITS, 2, 2, 0, 0),
    "mixpar": (MIXED_PAR, 2, 2, 0, 0),
    "pf15": (PF_ORBITS, 1, 5, 0, 0),  # neutron sectors wider than a workgroup
}
# widths at the edges of the 16-byte pieces of a row, of the lanes per row and of the column tiles
WIDTHS = (1, 2, 3, 4, 5, 8, 9, 12, 16, 17, 31, 32, 33, 64)


def _with_env(env, make):
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        return make()
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


@pytest.mark.parametrize("batch", ["one", "several"])
@pytest.mark.parametrize("space", SPACES)
def test_widths_and_batches_match_oracle(space, batch):
    """Each row within the per-term bound of its generated terms plus the additions of the slot sum
    (n_prot * n_neut slots of blocks of at most 64 pairs), as for the other pair-block tests."""
    orbits, z, n, twoM, par = SPACES[space]
    tb = random_tbme(orbits, 11)
    spe = [0.4 * k - 1.1 for k in range(len(orbits))]
    env = {"TRBL_PN_TILES": "2"}
    if batch == "several":
        env["TRBL_PN_BATCH"] = "300"
    g, o = _with_env(env, lambda: pair(orbits, z, n, twoM, tb, spe, spe, par))
    rng = np.random.default_rng(4)
    idx = np.unique(np.concatenate([rng.choice(o.dim, min(o.dim, 400), replace=False), [0, o.dim - 1]]))
    V = random_block(70, o.dim, max(WIDTHS))
    ref, bound = o.apply_rows(V, idx), term_bound(o, idx, V, extra=z * n + 64)
    V32 = V.astype(np.float32)
    ref32 = o.apply_rows(V32.astype(np.float64), idx)
    bound32 = term_bound(o, idx, V32, fp32=True, extra=z * n + 64)
    for nb in WIDTHS:
        say("case", space, batch, "nb", nb)
        W = g.apply(torch.from_numpy(V[:, :nb].copy()).cuda()).cpu().numpy()
        assert np.all(np.abs(W[idx] - ref[:, :nb]) <= bound[:, :nb])
        W32 = g.apply(torch.from_numpy(V32[:, :nb].copy()).cuda()).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(W32[idx] - ref32[:, :nb]) <= bound32[:, :nb])
    # a second product on the same model gives the same bits
    Vt = torch.from_numpy(V[:, :16].copy()).cuda()
    assert torch.equal(g.apply(Vt), g.apply(Vt))


def test_non_finite_rows_stay_local():
    """A column with one infinite entry: rows that H does not link to that entry stay finite and equal to
    the product without it."""
    orbits, z, n, twoM, par = SPACES["pf22"]
    g, o = _with_env({"TRBL_PN_TILES": "2"},
                     lambda: pair(orbits, z, n, twoM, random_tbme(orbits, 11), [0.0] * 4, [0.0] * 4, par))
    j = o.dim // 3
    V = random_block(5, o.dim, 8)
    V[j, 3] = 0.0
    clean = g.apply(torch.from_numpy(V).cuda()).cpu().numpy()
    V[j, 3] = np.inf
    W = g.apply(torch.from_numpy(V).cuda()).cpu().numpy()
    assert np.array_equal(np.delete(W, 3, axis=1), np.delete(clean, 3, axis=1))
    # rows that share no core pair with j (two or more spectators apart in one species) and, differing
    # from it in both species, no identical-particle move either
    pj, nj = g.unrank(j)
    far = []
    for i in range(o.dim):
        p, q = g.unrank(i)
        if p != pj and q != nj and (bin(p & pj).count("1") < z - 1 or bin(q & nj).count("1") < n - 1):
            far.append(i)
    assert len(far) > 100
    assert np.array_equal(W[far, 3], clean[far, 3])


def test_rows_beyond_4_gib():
    """expect() on columns of a block whose rows span more than 4 GiB (64-bit row addresses) against the same
    columns packed: the same products, their sums over D products in another order at most
    (each within gamma_D of sum |x| |H x|)."""
    orbits, z, n, twoM, par = SPACES["pf22"]
    g, _ = _with_env({"TRBL_PN_TILES": "2"},
                     lambda: pair(orbits, z, n, twoM, random_tbme(orbits, 11), [0.0] * 4, [0.0] * 4, par, oracle=False))
    ld = (1 << 32) // (8 * g.dim) + 64
    X = torch.empty((g.dim, ld), dtype=torch.float64, device="cuda")
    say("expect on", tuple(X.shape))
    X.normal_(generator=torch.Generator(device="cuda").manual_seed(3))
    assert X.numel() * 8 > 1 << 32
    got = g.expect(X)
    cols = [0, 1, ld // 2, ld - 65, ld - 1]
    P = X[:, cols].contiguous()
    ref = g.expect(P)
    HP = g.apply(P)
    u = 2.0 ** -53
    bound = 2 * g.dim * u / (1 - g.dim * u) * (P.abs() * HP.abs()).sum(0).cpu().numpy()
    assert np.all(np.isfinite(got)) and np.all(np.abs(got[cols] - ref) <= bound)
