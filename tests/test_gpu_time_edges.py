"""Two-time records at the edges of the kernel's tiles and number formats,
exactly against plain int64 sums: one, an even and an odd number of 64-bit
chunks along L^2, Ltau around the 64-wide tiles, one and many configurations
per call (tiles shared by several workgroups, or not), both boundaries, and
sums of q2 beyond 32 bits (L = 24, Ltau = 4096, four replicas, all spins
equal: q2[d] = R L^4 Ltau)."""
import numpy as np
import pytest

from paper_2310_07486_amd import tfim
from paper_2310_07486_amd.workloads import Shape, ladder

pytestmark = pytest.mark.gpu


def _records(plan, sh, words, kidx, cfg):
    i, s = divmod(cfg, sh.n_samples)
    Lt = sh.Ltau
    c = np.zeros(Lt, dtype=np.int64)
    q2 = np.zeros(Lt, dtype=np.int64)
    t = np.arange(Lt)
    for r in range(sh.n_replicas):
        w = int(np.nonzero(kidx[r, s] == i)[0][0])
        S = tfim.unpack_lane(words[r, w, s // 64], s % 64).astype(np.int64)  # [tau][xy]
        H = S @ S.T
        for d in range(Lt):
            h = H[t, (t + d) % Lt]
            sign = np.where(t + d >= Lt, -1, 1) if sh.bc_tau else 1
            c[d] += int((sign * h).sum())
            q2[d] += int((h * h).sum())
    return np.stack([c, q2])


@pytest.mark.parametrize("L,Lt,R,nk,bc,cfg0,ncfg", [
    (2, 16, 3, 9, 0, 0, 576), (4, 64, 1, 2, 1, 5, 3), (6, 72, 6, 1, 0, 60, 4), (8, 128, 2, 10, 1, 0, 640),
    (10, 136, 5, 2, 0, 127, 1), (12, 200, 4, 1, 1, 0, 64), (14, 192, 3, 1, 0, 3, 2), (16, 264, 2, 1, 1, 1, 1),
    (18, 320, 4, 1, 0, 0, 2), (20, 456, 6, 1, 0, 63, 1), (22, 104, 3, 1, 1, 8, 1), (24, 640, 4, 1, 0, 9, 2)])
def test_time_records_at_tile_edges(L, Lt, R, nk, bc, cfg0, ncfg):
    print(f"time edges L={L} Ltau={Lt} R={R} cfg0={cfg0} ncfg={ncfg}", flush=True)
    sh = Shape(L, Lt, 1, R, ladder(0.25, 0.4, nk), bc_tau=bc)
    plan = tfim.Plan([sh], 77 * L + Lt)
    plan.init()
    plan.sweep(5)
    got = plan.measure_time(0, cfg0, ncfg)
    words = plan.export_spins(0)
    kidx, _ = plan.get_state(0)
    for c in sorted({0, ncfg // 2, ncfg - 1}):
        assert np.array_equal(got[c], _records(plan, sh, words, kidx, cfg0 + c)), c
    plan.close()


@pytest.mark.parametrize("Lt,R", [(2048, 6), (4096, 4)])
def test_time_records_of_equal_spins(Lt, R):
    """Below and above 2^32 in a bucket of q2."""
    print(f"time extremes L=24 Ltau={Lt} R={R}", flush=True)
    L = 24
    sh = Shape(L, Lt, 1, R, [0.3])
    plan = tfim.Plan([sh], 9)
    plan.init_couplings(0)
    plan.init_spins(0, np.zeros((R, 1, 1, Lt, L * L), dtype=np.uint64))
    got = plan.measure_time(0, 0, 64)
    assert np.all(got[:, 0] == R * L ** 2 * Lt)
    assert np.all(got[:, 1] == R * L ** 4 * Lt)
    plan.close()
