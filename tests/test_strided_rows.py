"""Rows a stride apart on ragged_rows_kernel (csrc/rlcs_kernels.h, GAPS): every row takes
ceil(T / K) lanes from its own first step, the last one's vector moved back onto the row's end.

On the CPU: the geometry restated. Every step belongs to one lane, no vector leaves its row, and the
neighbour that a lane takes from the lane beside it or from memory is the adjacent step. On the GPU:
every estimator against the oracle, with NaN in the inputs' gaps and guard values in the outputs'."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_17641_amd as rl
import workloads

LENGTHS = {4: [4, 5, 7, 9, 31, 32, 63, 101, 255, 256, 257, 511, 513, 1023, 1024, 1025, 1030, 2047, 4093, 4096],
           8: [8, 9, 15, 17, 63, 64, 101, 257, 511, 513, 907, 1023, 2047, 2049, 2056, 4099, 8185, 8192]}


@pytest.mark.parametrize("back", [False, True])
@pytest.mark.parametrize("K", [4, 8])
def test_geometry(K, back):
    for T in LENGTHS[K]:
        LR = -(-T // K)
        R = max(256 // LR, 1)
        W = -(-R * LR // 64)
        assert W <= 16 and (R == 1 or W <= 4)
        magic = ((1 << 22) + LR - 1) // LR if R > 1 else 0
        for N in (1, R, R + 1, 2 * R + 1):
            owner = np.zeros((N, T), np.int32)
            for wg in range(-(-N // R)):
                for i in range(W * 64):
                    lane = 63 - i % 64 if back else i % 64
                    r = (i * magic) >> 22
                    q = i - r * LR
                    if not (r < R and wg * R + r < N and q < LR):
                        continue
                    row = wg * R + r
                    assert r == i // LR
                    t = q * K
                    k_lo = max(t + K - T, 0)
                    first = t - k_lo  # step of the vector's first element
                    assert 0 <= first and first + K <= T
                    owner[row, t:first + K] += 1
                    if back:
                        if first + K < T:  # the step after: lane l-1's first, or from memory
                            memory = lane == 0 or (T % K and q == LR - 2)
                            beside = (q + 1) * K - max((q + 2) * K - T, 0)
                            assert memory or beside == first + K
                    elif t > 0:  # the step before the lane's own first: in the vector, or lane l-1's last
                        assert k_lo > 0 or lane == 0 or (q - 1) * K + K - 1 == t - 1
            assert (owner == 1).all()


def _strided(x, ld, shift):
    """[N, T] host array as a view of wider rows on the GPU, NaN (or 1) in the gaps."""
    t = torch.from_numpy(np.ascontiguousarray(x))
    t = t.view(torch.bfloat16) if x.dtype == np.uint16 else t
    N, T = t.shape
    flat = torch.full((N * ld + shift,), float("nan") if t.is_floating_point() else 1, dtype=t.dtype, device="cuda")
    wide = flat[shift:].view(N, ld)
    wide[:, :T] = t.cuda()
    return wide[:, :T]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,T", [("f32", T) for T in LENGTHS[4]] + [("bf16", T) for T in LENGTHS[8]])
def test_against_the_oracle(dtype, T):
    K = 4 if dtype == "f32" else 8
    R = max(256 // -(-T // K), 1)
    for N, gap, shift in ((2 * R + 1, 1, 0), (R + 1, 64, 1), (2, 5, 3)):
        ld = T + gap
        ro = workloads.make_rollout(N, T, seed=T + gap, dtype=dtype, p_term=0.03, p_trunc=0.03)
        d = {k: _strided(v, ld, shift) for k, v in ro.items() if k != "boot"}
        b = torch.from_numpy(ro["boot"])
        boot = (b.view(torch.bfloat16) if dtype == "bf16" else b).cuda()
        guard = [torch.full((N * ld + shift,), 7.5, device="cuda") for _ in range(2)]
        out = [g[shift:].view(N, ld)[:, :T] for g in guard]
        x = (d["r"], d["v"], d["term"], d["trunc"], d["bv"], boot)
        a = (ro["r"], ro["v"], ro["term"], ro["trunc"], ro["bv"], ro["boot"])
        p = dict(gamma=0.99, lam=0.95)
        calls = [
            (lambda: rl.rlcs_gae_strided(*x, *out, **p), oracle.gae(*a, **p)),
            (lambda: rl.rlcs_gae_strided(x[0], x[1], None, None, None, None, *out, **p),
             oracle.gae(a[0], a[1], None, None, None, None, **p)),
            (lambda: rl.rlcs_vtrace_strided(x[0], x[1], d["log_rho"], *x[2:], *out, gamma=0.99),
             oracle.vtrace(a[0], a[1], ro["log_rho"], *a[2:], gamma=0.99)),
            (lambda: rl.rlcs_retrace_strided(x[0], d["q"], d["eq"], d["log_rho"], *x[2:], *out, **p),
             oracle.retrace(a[0], ro["q"], ro["eq"], ro["log_rho"], *a[2:], **p)),
            (lambda: rl.rlcs_td_lambda_strided(*x, out[0], **p), (oracle.td_lambda(*a, **p),)),
            (lambda: rl.rlcs_discounted_strided(x[0], *x[2:], out[0], gamma=0.99), (oracle.discounted(a[0], *a[2:], gamma=0.99),)),
            (lambda: rl.rlcs_elig_trace_strided(d["x"], x[2], x[3], out[0], **p), (oracle.elig_trace(ro["x"], a[2], a[3], **p),)),
            (lambda: rl.rlcs_elig_trace_strided(d["x"], None, x[3], out[0], **p), (oracle.elig_trace(ro["x"], None, a[3], **p),)),
            (lambda: rl.rlcs_episodic_prefix_strided(d["x"], x[2], x[3], out[0], boundary="starts_at"),
             (oracle.episodic_prefix(ro["x"], a[2], a[3], boundary="starts_at"),)),
        ]
        for i, (call, refs) in enumerate(calls):
            call()
            for o, r in zip(out, refs):
                # float32 arithmetic: the parity bound of the other tests
                err = np.max(np.abs(o.double().cpu().numpy() - r))
                assert err <= 1e-5 * (1.0 + np.max(np.abs(r))), (dtype, N, T, gap, i, err)
        for g in guard:
            assert (g[:shift] == 7.5).all() and (g[shift:].view(N, ld)[:, T:] == 7.5).all()
