"""More configurations than one launch can hold (2^32 work-items): the call
goes over them in ranges.  The first and the last samples, the border between
two ranges among them, equal those of a small plan whose words are the same
ones of the random streams."""
import numpy as np
import pytest

from paper_2310_07486_amd import tfim
from paper_2310_07486_amd.workloads import Shape

pytestmark = pytest.mark.gpu

WORDS = 1 << 18  # 2^24 samples


def _plan(W, offset):
    plan = tfim.Plan([Shape(2, 16, W, 2, [0.3], word_offset=offset)], 12)
    plan.init()
    plan.sweep(2)
    return plan


def test_pair_records():
    print("pair records of 2^24 configurations", flush=True)
    plan = _plan(WORDS, 0)
    rec = plan.measure_range(0, 0, 0, 64 * WORDS)
    plan.close()
    assert np.array_equal(rec[..., :2].sum(axis=-1), rec[..., 5])  # sum_d D_x[d] = sum Q^2
    for offset, part in ((0, rec[:256]), (WORDS - 4, rec[-256:])):
        small = _plan(4, offset)
        assert np.array_equal(part, small.measure_range(0, 0, 0, 256)), offset
        small.close()


def test_two_time_records():
    import torch
    print("two-time records of 2^24 configurations", flush=True)
    plan = _plan(WORDS, 0)
    plan.measure_time(0, 0, 64 * WORDS, copy=False)
    rec = plan._tcws.view(torch.int64).reshape(64 * WORDS, 2, 16)
    assert bool((rec[:, 0, 0] == 2 * 4 * 16).all())  # c[0] = R L^2 Ltau
    ends = rec[:256].cpu().numpy(), rec[-256:].cpu().numpy()
    plan.close()
    for offset, part in zip((0, WORDS - 4), ends):
        small = _plan(4, offset)
        assert np.array_equal(part, small.measure_time(0, 0, 256)), offset
        small.close()


def test_plain_sweeps():
    """Configurations of 8 KB (1024 threads each); k labels have one value, U is a
    count over the whole trajectory."""
    print("plain sweeps of 2^22 + 64 configurations", flush=True)

    def plan(samples, offset):
        p = tfim.Plan([Shape(4, 512, samples, 1, [0.3], word_offset=offset)], 12, form=tfim.TFIM_FORM_PLAIN_I8)
        p.init()
        U0 = p.measure(0, tfim.TFIM_MEASURE_ENERGY)
        p.sweep(2)
        U = p.measure(0, tfim.TFIM_MEASURE_ENERGY)
        p.close()
        return U0[0, :, 0], U[0, :, 0]

    n = (1 << 22) + 64
    big = plan(n, 0)
    for offset in (0, n // 64 - 4):
        for got, want in zip(big, plan(256, offset)):
            assert np.array_equal(got[64 * offset:64 * offset + 256], want), offset
