"""Masked GAE at the edges of its workgroups' waves and chunks: rows that need five to sixteen waves,
rows of two and three chunks of as few waves as hold them, and whitened calls of one pass and of
two on the same rows. Long masked runs cross waves and chunks, so that the value of the next unmasked
step is carried through all of them. Against the oracle, with the bound of the other masked tests."""
import numpy as np
import pytest

from cases import TOL, assert_parity
from test_gpu_masked import run, variant
import workloads

pytestmark = pytest.mark.gpu

ROWS = [("f32", T) for T in (1025, 1279, 1281, 2047, 2048, 2050, 2305, 3841, 4093, 4096, 4097, 4263, 8191, 8193, 9001)] + \
       [("bf16", T) for T in (2049, 2561, 4097, 4600, 8185, 8192, 8193, 12300, 16385)]


@pytest.mark.parametrize("dtype,T", ROWS)
def test_rows(dtype, T):
    N = 7
    ro = workloads.make_rollout(N, T, seed=T, dtype=dtype, p_term=0.002, p_trunc=0.002)
    mask = (np.random.default_rng(T).random((N, T)) < 0.5).astype(np.uint8)
    mask[1] = 0                      # nothing takes part
    mask[2, T // 8:T - T // 8] = 0   # one run across most of the row's waves
    mask[3] = 1
    mask[4, :-1] = 0                 # only the last step
    mask[5, 1:] = 0                  # only the first
    ro["term"][2] = 0
    ro["trunc"][2] = 0
    for norm in (False, True):
        out, ref = run(ro, mask, normalize=norm)
        assert_parity(out, ref, TOL[dtype], label=f"{T} {dtype} norm={norm}")
    with variant(1):  # whitening in two passes
        out, ref = run(ro, mask, normalize=True)
    assert_parity(out, ref, TOL[dtype], label=f"{T} {dtype} two passes")
    out, ref = run(ro, mask, trunc=False, boot=False, term=False, gamma=1.0, lam=1.0)
    assert_parity(out, ref, TOL[dtype], label=f"{T} {dtype} no flags")


@pytest.mark.parametrize("N,T", [(1024, 3000), (1000, 2049), (700, 1500), (1023, 40), (5, 3)])
def test_many_groups_whitened(N, T):
    """Moments of up to 1024 workgroups, more than workgroup 0 has lanes where rows take few waves."""
    ro = workloads.make_rollout(N, T, seed=N, p_term=0.01, p_trunc=0.01)
    mask = (np.random.default_rng(N).random((N, T)) < 0.7).astype(np.uint8)
    out, ref = run(ro, mask, normalize=True)
    assert_parity(out, ref, TOL["f32"], label=f"{N}x{T}")


@pytest.mark.parametrize("dtype,N,T", [("bf16", 7, 2049), ("bf16", 8, 2100), ("bf16", 9, 4090), ("bf16", 5, 4092),
                                       ("bf16", 4, 4093), ("bf16", 3, 4096), ("f32", 7, 1300), ("f32", 8, 1800),
                                       ("f32", 5, 2046), ("f32", 4, 2047), ("f32", 4, 2048)])
def test_several_long_rows_to_a_workgroup(dtype, N, T):
    """Rows of five to nine waves that sixteen waves hold two or three of, and the lengths beside
    them; whole workgroups and a last one of fewer rows."""
    ro = workloads.make_rollout(N, T, seed=N + T, dtype=dtype, p_term=0.002, p_trunc=0.002)
    mask = (np.random.default_rng(T).random((N, T)) < 0.5).astype(np.uint8)
    mask[1] = 0
    mask[2, T // 8:T - T // 8] = 0
    for trunc in (True, False):
        out, ref = run(ro, mask, trunc=trunc)
        assert_parity(out, ref, TOL[dtype], label=f"{N}x{T} {dtype} trunc={trunc}")
    with variant(1):
        out, ref = run(ro, mask, normalize=True)
    assert_parity(out, ref, TOL[dtype], label=f"{N}x{T} {dtype} two passes")
