"""Sweeps in parts along tau (few configurations, default variant) against the
chunked kernel (variant 1), which sweeps a configuration whole: spins, k labels,
energies and counters bit for bit.  Two to the largest number of parts, a
shorter last part, lattices of one and of several waves, both boundaries,
energies counted in every sweep or only in the last; and the counters across
changes of the schedule (per-shape launches take them by value, graphs read
them on the device)."""
import numpy as np
import pytest

from paper_2310_07486_amd import tfim
from paper_2310_07486_amd.workloads import Shape, ladder

pytestmark = pytest.mark.gpu


def _state(plan):
    out = []
    for i in range(len(plan.shapes)):
        out += [plan.export_spins(i), *plan.get_state(i), np.array(plan.counters(i))]
    return out


def _same(a, b):
    return len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("L,Lt,W,R,nk,pt,bc", [
    (2, 16, 1, 1, 1, 0, 0), (4, 256, 1, 1, 2, 0, 1), (6, 136, 1, 2, 3, 1, 0), (8, 512, 1, 6, 16, 30, 0),
    (10, 104, 2, 3, 5, 1, 1), (12, 512, 1, 6, 24, 2, 0), (14, 200, 1, 4, 30, 1, 0), (16, 256, 1, 4, 32, 1, 1),
    (18, 96, 2, 4, 20, 3, 0), (20, 88, 1, 4, 40, 1, 1), (22, 168, 1, 2, 60, 1, 0), (24, 72, 1, 2, 64, 1, 1),
    (24, 64, 1, 2, 20, 5, 0)])
def test_parts_equal_whole(L, Lt, W, R, nk, pt, bc):
    print(f"parts L={L} Ltau={Lt} W={W} R={R} nk={nk} pt={pt} bc={bc}", flush=True)
    sh = Shape(L, Lt, W, R, ladder(0.2, 0.4, nk), pt_every=pt, bc_tau=bc)
    got = []
    for variant in (3, 1):
        plan = tfim.Plan([sh], 1000 * L + Lt)
        plan.set_variant(variant)
        plan.init()
        plan.sweep(1)
        plan.sweep(6)
        got.append(_state(plan))
        plan.close()
    assert _same(*got)


def test_counters_across_schedules():
    print("parts: counters across schedules", flush=True)
    shapes = [Shape(8, 64, 1, 2, ladder(0.25, 0.3, 5), pt_every=1, stream_id=0),
              Shape(12, 40, 1, 2, ladder(0.25, 0.3, 4), pt_every=3, stream_id=1),
              Shape(24, 32, 1, 2, ladder(0.25, 0.3, 3), pt_every=0, stream_id=2)]
    S = (tfim.TFIM_SCHED_PER_SHAPE, tfim.TFIM_SCHED_BATCHED, tfim.TFIM_SCHED_CONCURRENT)
    got = []
    for mixed in (False, True):
        plan = tfim.Plan(shapes, 5)
        if not mixed:
            plan.set_variant(1)
        plan.init()
        for k, n in enumerate((2, 3, 1, 4, 2, 3, 5)):
            if mixed:
                plan.set_schedule(S[k % 3])
            plan.sweep(n)
            if k % 2:
                plan.pt_swap()
        got.append(_state(plan))
        plan.close()
    assert _same(*got)


def test_callers_graph_goes_on():
    """tfim_sweep and tfim_pt_swap captured in the caller's own graph: every
    replay does the next sweeps, eager calls before and after go on likewise."""
    import torch
    shapes = [Shape(4, 32, 1, 2, ladder(0.2, 0.4, 3), pt_every=1),
              Shape(6, 40, 1, 2, ladder(0.2, 0.4, 2), pt_every=2, stream_id=1)]
    print("caller's graph", flush=True)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        plan, ref = tfim.Plan(shapes, 5, stream=st), tfim.Plan(shapes, 5, stream=st)
        for p in (plan, ref):
            p.init()
            p.sweep(2)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            plan.sweep(4)
            plan.pt_swap()
        for k in range(3):
            g.replay()
            ref.sweep(4)
            ref.pt_swap()
            torch.cuda.synchronize()
            for i in range(2):
                assert np.array_equal(plan.export_spins(i), ref.export_spins(i)), (k, i)
                assert all(np.array_equal(a, b) for a, b in zip(plan.get_state(i), ref.get_state(i))), (k, i)
        plan.sweep(4)
        ref.sweep(4)
        for i in range(2):
            assert np.array_equal(plan.export_spins(i), ref.export_spins(i))
        plan.close()
        ref.close()


@pytest.mark.parametrize("L,Lt,W,R,nk,pt", [
    (18, 256, 1, 4, 32, 1),   # six waves a workgroup: as many as fit, two parts
    (18, 1024, 1, 4, 24, 1),  # the same in two rounds of workgroups, five parts
    (4, 128, 4, 4, 64, 1),    # one wave: two to a SIMD, two parts
    (4, 128, 4, 4, 64, 0),    # four parts, two where U is counted
    (24, 16, 1, 2, 64, 1),    # whole: the join would cost more
    (8, 64, 8, 4, 60, 0),     # whole: two waves per SIMD already
])
def test_every_choice_of_parts(L, Lt, W, R, nk, pt):
    print(f"choice of parts L={L} Ltau={Lt} W={W} R={R} nk={nk} pt={pt}", flush=True)
    sh = Shape(L, Lt, W, R, ladder(0.2, 0.4, nk), pt_every=pt)
    got = []
    for variant in (3, 1):
        plan = tfim.Plan([sh], L + Lt)
        plan.set_variant(variant)
        plan.init()
        plan.sweep(3)
        got.append(_state(plan))
        plan.close()
    assert _same(*got)
