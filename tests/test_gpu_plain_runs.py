"""Plain-form sweeps: a configuration in one workgroup's LDS for a run of sweeps,
or a launch per half-sweep over the whole chip; both against the oracle at the
sizes between which the choice lies."""
import numpy as np
import pytest

from oracle import measure as om
from paper_2310_07486_amd import tfim
from paper_2310_07486_amd.workloads import Shape, ladder
from test_gpu_plain import PLAIN, _chain, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Lt,ns,nk,pt,bc", [
    (6, 30, 2, 2, 0, 1),     # one unit a thread, a part wavefront, ragged chunk of tau
    (8, 128, 2, 2, 2, 0),    # exactly 1024 units
    (8, 130, 1, 2, 3, 1),    # the first with two units a thread
    (16, 130, 1, 1, 0, 1),   # 4352 units, few configurations: half-sweep launches
    (16, 130, 1, 2, 1, 0),   # the same in runs of one sweep: LDS
    (16, 130, 3, 2, 4, 0),   # the same with 12 configurations: LDS
    (16, 236, 1, 2, 5, 0),   # the largest Ltau in LDS at this L (64512 bytes)
    (16, 238, 1, 2, 1, 0),   # one beyond it
])
def test_runs_of_sweeps(L, Lt, ns, nk, pt, bc):
    sh = Shape(L, Lt, ns, 2, ladder(0.22, 0.4, nk), pt_every=pt, stream_id=3, word_offset=1, bc_tau=bc)
    _say(f"plain runs L={L} Lt={Lt} samples={ns} nk={nk} pt={pt} bc={bc}")
    plan = tfim.Plan([sh], 77, form=PLAIN)
    plan.init()
    ch = _chain(sh, 77, list(range(ns)))
    for n in (1, 4, 2):
        plan.sweep(n)
        ch.run(n)
        kidx, U = plan.get_state(0)
        assert np.array_equal(plan.export_spins(0), ch.S), "spins differ"
        assert np.array_equal(kidx, ch.kidx), "k labels differ"
        assert np.array_equal(U, ch.U), "energies differ"
    assert plan.counters() == (7, 7 // pt if pt else 0)
    assert np.array_equal(plan.measure(0, tfim.TFIM_MEASURE_RECORDS), om.measure_chain(ch))
    plan.close()


@pytest.mark.parametrize("L,Lt,ns,nk,pt", [
    (6, 30, 2, 3, 1),        # LDS, tempering after every sweep
    (8, 32, 2, 2, 0),        # LDS, one run, tempering by tfim_pt_swap alone
    (16, 238, 1, 2, 2),      # half-sweep launches
])
def test_callers_graph_goes_on(L, Lt, ns, nk, pt):
    """tfim_sweep and tfim_pt_swap captured in the caller's own graph: every
    replay does the next sweeps, eager calls before and after go on likewise."""
    import torch
    shapes = [Shape(L, Lt, ns, 2, ladder(0.22, 0.3, nk), pt_every=pt, stream_id=3),
              Shape(4, 16, 1, 2, ladder(0.2, 0.4, 3), pt_every=2, stream_id=1)]
    _say(f"plain caller's graph L={L} Lt={Lt} samples={ns} nk={nk} pt={pt}")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        plan, ref = (tfim.Plan(shapes, 5, stream=st, form=PLAIN) for _ in range(2))
        for p in (plan, ref):
            p.init()
            p.sweep(2)
            p.pt_swap()
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
        for p in (plan, ref):
            p.sweep(3)
            p.pt_swap()
        for i in range(2):
            assert np.array_equal(plan.export_spins(i), ref.export_spins(i))
            assert all(np.array_equal(a, b) for a, b in zip(plan.get_state(i), ref.get_state(i)))
        plan.close()
        ref.close()


def test_a_long_call_in_several_runs():
    """Runs are cut at 4096 sweeps, or where they would take about 50 ms: 2048
    configurations of 6912 units at 220 sweeps."""
    _say("plain: calls longer than a run")
    for L, Lt, ns, nk, n in ((2, 8, 2, 1, 9000), (16, 216, 128, 8, 450)):
        got = []
        for parts in (1, 10):
            plan = tfim.Plan([Shape(L, Lt, ns, 2, ladder(0.22, 0.3, nk), pt_every=0)], 4, form=PLAIN)
            plan.init()
            for _ in range(parts):
                plan.sweep(n // parts)
            got.append([plan.export_spins(0), *plan.get_state(0), np.array(plan.counters())])
            plan.close()
        assert all(np.array_equal(a, b) for a, b in zip(*got))
