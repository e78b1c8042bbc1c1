"""Full-form Retrace on the GPU where its kernel's lane layout changes: actions per step at the edges
of a lane's vector and of the lanes per step, tensors smaller than one vector, rows of several
chunks, four steps per lane, and Q and pi large enough for non-temporal loads.

The bound is the parity bound of the other tests: float32 sums of A products of magnitude up to 1
weighted by probabilities (they add to 1), then a scan whose values stay within a few units, so
1e-5 of (1 + max |result|) is some 80 roundings of the largest value."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_17641_amd as rl
import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _check(N, T, A, dtype, *, seed=0, trunc=True, shift=0, rows=None):
    ro = workloads.make_retrace_full(N, T, A, seed=seed, dtype=dtype, p_term=0.05, p_trunc=0.05 if trunc else 0.0)

    def dev(x):
        t = torch.from_numpy(np.ascontiguousarray(x))
        return (t.view(torch.bfloat16) if x.dtype == np.uint16 else t).to(DEV)

    def moved(x):  # the same values `shift` elements into a larger buffer
        t = dev(x)
        wide = torch.zeros(t.numel() + shift, dtype=t.dtype, device=DEV)
        wide[shift:] = t.reshape(-1)
        return wide[shift:].view(t.shape)

    d, q = rl.rlcs_retrace_full(moved(ro["r"]), moved(ro["q3"]), moved(ro["pi3"]), moved(ro["actions"]),
                                moved(ro["mu"]), moved(ro["term"]), moved(ro["trunc"]) if trunc else None,
                                moved(ro["bv"]) if trunc else None, dev(ro["boot"]), gamma=0.99, lam=0.95)
    take = slice(None) if rows is None else rows
    rd, rq = oracle.retrace_full(ro["r"][take], ro["q3"][take], ro["pi3"][take], ro["actions"][take],
                                 ro["mu"][take], ro["term"][take], ro["trunc"][take] if trunc else None,
                                 ro["bv"][take] if trunc else None, ro["boot"][take], gamma=0.99, lam=0.95)
    for got, ref in ((d, rd), (q, rq)):
        err = np.max(np.abs(got.double().cpu().numpy()[take] - ref))
        assert err <= 1e-5 * (1.0 + np.max(np.abs(ref))), (N, T, A, dtype, err)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("A", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 63, 65, 127, 129, 255, 256, 257, 259, 512, 515, 1025])
def test_action_counts(A, dtype):
    _check(7, 67, A, dtype, seed=A)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 2), (1, 3, 1), (1, 1, 3), (1, 2, 3), (1, 1, 7), (2, 1, 5), (1, 1, 300)])
def test_tensors_of_about_one_vector(shape, dtype):
    _check(*shape, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,T,A", [(3, 1023, 9), (3, 1024, 18), (3, 1025, 9), (2, 2500, 3), (2, 4099, 5), (1, 9000, 2), (2, 3001, 40)])
def test_rows_of_several_chunks(N, T, A, dtype):
    _check(N, T, A, dtype, seed=T)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,T,A", [(2731, 192, 3), (8193, 65, 7), (2050, 257, 1)])
def test_four_steps_per_lane(N, T, A, dtype):
    _check(N, T, A, dtype, shift=1, rows=slice(None, None, 97))


@pytest.mark.parametrize("dtype,N,T,A", [("f32", 4000, 257, 13), ("f32", 3001, 600, 7), ("bf16", 8001, 129, 33), ("f32", 1, 40000, 300)])
def test_non_temporal_loads(dtype, N, T, A):
    _check(N, T, A, dtype, trunc=False, rows=slice(None, None, 211))


@pytest.mark.parametrize("N,T,A", [(2001, 256, 41), (16001, 32, 64)])
def test_non_temporal_loads_one_step_per_lane(N, T, A):
    """bfloat16 calls of too few steps for four per lane whose Q and pi are past the cached size."""
    _check(N, T, A, "bf16", shift=1, rows=slice(None, None, 211))
