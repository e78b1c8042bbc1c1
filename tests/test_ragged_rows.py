"""ragged_rows_kernel (csrc/rlcs_kernels.h; plan in csrc/rlcs_dispatch.h): dense rows of any length
of K steps and more, arrays of any element alignment.

On the CPU: its lane geometry restated, over lengths at the edges of its plan. Every step belongs to
one lane of one workgroup, whole-vector loads stay inside the array, the row of a lane's first step
is exact, a lane holds at most one row edge and it is where the kernel puts it, and the neighbour
of lane 0 lies in the range. On the GPU: every estimator against the oracle at those lengths, with
arrays on and off a vector boundary and guard values around the outputs."""
from math import gcd

import numpy as np
import pytest
import torch

import oracle
import paper_2608_17641_amd as rl
import workloads

WAVE = 64
LENGTHS = {4: [4, 5, 7, 9, 15, 63, 65, 101, 127, 129, 255, 257, 341, 511, 513, 1021, 1023, 1025, 1333, 2001,
               2047, 2049, 3071, 4063, 4065, 4067, 4093, 4095, 4096],
           8: [8, 9, 15, 17, 101, 333, 511, 513, 600, 1000, 1023, 1025, 2041, 2047, 2049, 3001, 4096, 5001,
               8127, 8129, 8183, 8185, 8191, 8192]}


def plan(T, K):
    """(R, W, grid): rows and waves of a workgroup, and what its lanes' first step is a multiple of."""
    span = WAVE * K
    R = max(4 * span // T, 1)
    most = 4 * span if R > 1 else 16 * span
    for grid in (8 * K, K, 1):
        steps = R * T + grid - gcd(R * T, grid)
        if steps <= most:
            return R, -(-steps // span), grid
    raise AssertionError((T, K))


@pytest.mark.parametrize("back", [False, True])
@pytest.mark.parametrize("K", [4, 8])
def test_geometry(K, back):
    for T in LENGTHS[K]:
        R, W, grid = plan(T, K)
        assert W <= 16
        magic = ((1 << 22) + T - 1) // T if R > 1 else 0
        for N in (1, R, R + 1, 3 * R + 2):
            total, owner = N * T, np.zeros(N * T, np.int32)
            for wg in range(-(-N // R)):
                lo, hi = wg * R * T, min(wg * R + R, N) * T
                base = lo // grid * grid
                assert base + W * WAVE * K >= hi
                for i in range(W * WAVE):
                    p0 = base + i * K
                    k_lo = min(max(lo - p0, 0), K)
                    k_hi = min(max(hi - p0, 0), K)
                    if k_lo >= k_hi:
                        continue
                    assert p0 >= 0
                    owner[p0 + k_lo:p0 + k_hi] += 1
                    o = p0 - lo + k_lo
                    assert o * magic < 1 << 32
                    r_in = (o * magic) >> 22
                    t = o - r_in * T
                    assert r_in == o // T and 0 <= t < T
                    edges = [k for k in range(k_lo, k_hi) if (p0 + k) % T == (T - 1 if back else 0)]
                    ke = k_lo + T - 1 - t if back else (k_lo if t == 0 else k_lo + T - t)
                    assert edges == ([ke] if k_lo <= ke < k_hi else [])
                    if edges:
                        row = wg * R + r_in + (1 if not back and ke > k_lo else 0)
                        assert row == (p0 + ke) // T
                    # lane 0's step past its carry-source edge, unless that edge is a row's
                    edge_step = K - 1 if back else 0
                    if k_lo <= edge_step < k_hi and edges != [edge_step]:
                        assert lo <= (p0 + K if back else p0 - 1) < hi
            assert (owner == 1).all()


def _inputs(N, T, dtype, seed, shift):
    ro = workloads.make_rollout(N, T, seed=seed, dtype=dtype, p_term=0.03, p_trunc=0.03)

    def dev(x):
        t = torch.from_numpy(np.ascontiguousarray(x))
        t = t.view(torch.bfloat16) if x.dtype == np.uint16 else t
        wide = torch.zeros(t.numel() + shift, dtype=t.dtype, device="cuda")
        wide[shift:] = t.reshape(-1).cuda()
        return wide[shift:].view(t.shape)
    return ro, {k: dev(v) for k, v in ro.items()}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,T", [("f32", T) for T in LENGTHS[4]] + [("bf16", T) for T in LENGTHS[8]])
def test_against_the_oracle(dtype, T):
    K = 4 if dtype == "f32" else 8
    R = plan(T, K)[0]
    for N, shift in ((2 * R + 1, 0), (R + 1, 1), (1, 3)):
        ro, d = _inputs(N, T, dtype, T + N, shift)
        a = (ro["r"], ro["v"], ro["term"], ro["trunc"], ro["bv"], ro["boot"])
        guard = [torch.full((N * T + 2 * 8 + shift,), 7.5, device="cuda") for _ in range(2)]
        out = [g[8 + shift:8 + shift + N * T].view(N, T) for g in guard]
        x = (d["r"], d["v"], d["term"], d["trunc"], d["bv"], d["boot"])
        # (the call, its outputs' reference, whether it writes both outputs)
        calls = [
            (lambda: rl.rlcs_gae(*x, *out, gamma=0.99, lam=0.95), oracle.gae(*a, gamma=0.99, lam=0.95), True),
            (lambda: rl.rlcs_gae(x[0], x[1], None, None, None, x[5], *out, gamma=0.99, lam=0.95),
             oracle.gae(a[0], a[1], None, None, None, a[5], gamma=0.99, lam=0.95), True),
            (lambda: rl.rlcs_vtrace(x[0], x[1], d["log_rho"], *x[2:], *out, gamma=0.99),
             oracle.vtrace(a[0], a[1], ro["log_rho"], *a[2:], gamma=0.99), True),
            (lambda: rl.rlcs_retrace(x[0], d["q"], d["eq"], d["log_rho"], *x[2:], *out, gamma=0.99, lam=0.95),
             oracle.retrace(a[0], ro["q"], ro["eq"], ro["log_rho"], *a[2:], gamma=0.99, lam=0.95), True),
            (lambda: rl.rlcs_td_lambda(*x, out[0], gamma=0.99, lam=0.95), oracle.td_lambda(*a, gamma=0.99, lam=0.95), False),
            (lambda: rl.rlcs_discounted(x[0], *x[2:], out[0], gamma=0.99), oracle.discounted(a[0], *a[2:], gamma=0.99), False),
            (lambda: rl.rlcs_elig_trace(d["x"], x[2], x[3], out[0], gamma=0.99, lam=0.95),
             oracle.elig_trace(ro["x"], a[2], a[3], gamma=0.99, lam=0.95), False),
            (lambda: rl.rlcs_elig_trace(d["x"], None, x[3], out[0], gamma=0.99, lam=0.95),
             oracle.elig_trace(ro["x"], None, a[3], gamma=0.99, lam=0.95), False),
            (lambda: rl.rlcs_episodic_prefix(d["x"], x[2], x[3], out[0], boundary="starts_at"),
             oracle.episodic_prefix(ro["x"], a[2], a[3], boundary="starts_at"), False),
            # the generic recurrence: coefficients v (as alpha) and flags turned into betas would
            # hide its carry, so alpha = r, beta = eq, forward, carry = boot
            (lambda: rl.rlcs_affine_scan(x[0], (0.25 * d["eq"]).contiguous(), x[5], out[0], reverse=False),
             None, False),
        ]
        for i, (call, ref, both) in enumerate(calls):
            call()
            if ref is None:
                wide = (lambda t: t.double().cpu().numpy())
                al, be, c = wide(x[0]), wide((0.25 * d["eq"]).contiguous()), wide(x[5])
                ref = np.empty_like(al)
                for t in range(T):
                    c = al[:, t] + be[:, t] * c
                    ref[:, t] = c
            refs = ref if both else (ref,)
            for o, r in zip(out, refs):
                # float32 arithmetic: the parity bound of the other tests
                err = np.max(np.abs(o.double().cpu().numpy() - r))
                assert err <= 1e-5 * (1.0 + np.max(np.abs(r))), (dtype, N, T, shift, i, err)
        for g in guard:
            assert (g[:8 + shift] == 7.5).all() and (g[8 + shift + N * T:] == 7.5).all()
