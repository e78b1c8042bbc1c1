"""Column walks with four columns to a lane (csrc/rlcs_colvec.h): time-major buffers of 8192 columns
and more, or of 1024 and more short ones, and vector traces, on the GPU against the oracle on sampled columns (the first and last
ones among them), at the edges of the kernel's blocks and chunks: column counts that are not a
multiple of four, rows on and off a 128-byte line, one chunk and several, strides past the last
column with the gap left alone, flags missing. One block width against another is the same
arithmetic in another association, so only the oracle's bound applies (float32 arithmetic: the
parity bound of the other tests)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_17641_amd as rl
import workloads

pytestmark = pytest.mark.gpu
GAP = 3.25


def _time_major(x, ld):
    """[N, T] host array as the [N, T] view of a [T, ld] device buffer, its gap filled."""
    t = torch.from_numpy(np.ascontiguousarray(x.T))
    t = t.view(torch.bfloat16) if x.dtype == np.uint16 else t
    wide = torch.full((t.shape[0], ld), GAP if t.is_floating_point() else 1, dtype=t.dtype, device="cuda")
    wide[:, :t.shape[1]] = t.cuda()
    return wide[:, :t.shape[1]].t()


def _close(got, ref):
    err = np.max(np.abs(got.double().cpu().numpy() - ref))
    assert err <= 1e-5 * (1.0 + np.max(np.abs(ref))), err


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,T,pad", [
    (8192, 33, 0), (8192, 257, 0), (8195, 40, 0), (8193, 129, 7), (9001, 127, 0), (9002, 130, 62),
    (16384, 65, 0), (16387, 128, 0), (24576, 193, 0), (24577, 200, 0), (24579, 260, 1), (49153, 34, 0),
    (49152, 50, 0), (1024, 33, 0), (1024, 512, 0), (1027, 256, 1), (1030, 257, 10), (2049, 31, 3),
    (4095, 255, 1), (4093, 511, 3), (4096, 512, 0), (4100, 64, 0), (8188, 16, 0)])
def test_time_major(N, T, pad, dtype):
    ro = workloads.make_rollout(N, T, seed=N + T, dtype=dtype, p_term=0.03, p_trunc=0.03)
    ld = N + pad
    d = {k: _time_major(v, ld) for k, v in ro.items() if k != "boot"}
    b = torch.from_numpy(ro["boot"])
    boot = (b.view(torch.bfloat16) if dtype == "bf16" else b).cuda()
    cols = np.unique(np.concatenate([np.arange(5), np.linspace(0, N - 1, 150).astype(int), np.arange(N - 9, N)]))
    s = {k: np.ascontiguousarray(v[cols]) for k, v in ro.items()}
    idx = torch.from_numpy(cols).cuda()
    guard = [torch.full((T, ld), GAP, device="cuda") for _ in range(2)]
    out = [g[:, :N].t() for g in guard]
    x = (d["r"], d["v"], d["term"], d["trunc"], d["bv"], boot)
    a = (s["r"], s["v"], s["term"], s["trunc"], s["bv"], s["boot"])
    p = dict(gamma=0.99, lam=0.95)
    ws = rl.make_workspace_columns(N, T, "cuda")
    calls = [
        (lambda: rl.rlcs_gae_strided(*x, *out, **p, ws=ws), oracle.gae(*a, **p)),
        (lambda: rl.rlcs_gae_strided(x[0], x[1], None, None, None, None, *out, gamma=1.0, lam=1.0),
         oracle.gae(a[0], a[1], None, None, None, None, gamma=1.0, lam=1.0)),
        (lambda: rl.rlcs_vtrace_strided(x[0], x[1], d["log_rho"], *x[2:], *out, gamma=0.99),
         oracle.vtrace(a[0], a[1], s["log_rho"], *a[2:], gamma=0.99)),
        (lambda: rl.rlcs_retrace_strided(x[0], d["q"], d["eq"], d["log_rho"], *x[2:], *out, **p),
         oracle.retrace(a[0], s["q"], s["eq"], s["log_rho"], *a[2:], **p)),
        (lambda: rl.rlcs_td_lambda_strided(*x, out[0], **p, ws=ws), (oracle.td_lambda(*a, **p),)),
        (lambda: rl.rlcs_discounted_strided(x[0], *x[2:], out[0], gamma=0.99), (oracle.discounted(a[0], *a[2:], gamma=0.99),)),
        (lambda: rl.rlcs_elig_trace_strided(d["x"], x[2], x[3], out[0], **p), (oracle.elig_trace(s["x"], a[2], a[3], **p),)),
        (lambda: rl.rlcs_elig_trace_strided(d["x"], None, x[3], out[0], **p), (oracle.elig_trace(s["x"], None, a[3], **p),)),
        (lambda: rl.rlcs_episodic_prefix_strided(d["x"], x[2], x[3], out[0], boundary="starts_at"),
         (oracle.episodic_prefix(s["x"], a[2], a[3], boundary="starts_at"),)),
        (lambda: rl.rlcs_episodic_prefix_strided(d["x"], x[2], None, out[0]), (oracle.episodic_prefix(s["x"], a[2], None),)),
    ]
    for call, refs in calls:
        for o in out:
            o.fill_(float("nan"))
        call()
        for o, r in zip(out, refs):
            _close(o[idx], r)
            assert not torch.isnan(o).any()
        for g in guard:
            assert (g[:, N:] == GAP).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,T,F", [(64, 300, 128), (64, 129, 256), (33, 257, 1024), (700, 70, 100), (331, 40, 100), (1, 100, 8192), (1, 65, 40004)])
def test_vector_traces(N, T, F, dtype):
    ro = workloads.make_vector_trace(N, T, F, seed=T + F, dtype=dtype, p_term=0.05, p_trunc=0.03)
    t = torch.from_numpy(ro["x"])
    x = (t.view(torch.bfloat16) if dtype == "bf16" else t).cuda()
    term, trunc = (torch.from_numpy(ro[k]).cuda() for k in ("term", "trunc"))
    rows = np.unique([0, N // 2, N - 1])
    for te, tr in ((term, trunc), (term, None), (None, trunc)):
        z = rl.rlcs_elig_trace_vec(x, te, tr, gamma=0.99, lam=0.95, ws=rl.make_workspace_columns(N * F, T, "cuda"))
        ref = oracle.elig_trace_vec(ro["x"][rows], None if te is None else ro["term"][rows],
                                    None if tr is None else ro["trunc"][rows], gamma=0.99, lam=0.95)
        _close(z[torch.from_numpy(rows).cuda()], ref)
        assert not torch.isnan(z).any()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,T,pad", [
    (1024, 300, 0), (1500, 80, 0), (1504, 16, 0), (8192, 128, 0), (8192, 129, 0), (8200, 513, 0), (12288, 150, 0),
    (16384, 256, 0), (16385, 272, 0), (20000, 145, 0), (40960, 260, 0), (49152, 160, 0), (65472, 64, 0),
    (65537, 80, 0), (65536, 97, 0), (90112, 49, 0), (90113, 80, 0)])
def test_choice_of_blocks(N, T, pad, dtype):
    """Both sides of the bounds between block widths and kernels, and chunks shared evenly by fewer
    than eight waves (145, 160 and 272 steps)."""
    test_time_major(N, T, pad, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,T,F", [(2731, 40, 12), (1639, 64, 20), (1639, 65, 20), (1366, 257, 24), (820, 257, 40), (330, 145, 200)])
def test_vector_traces_of_few_features(N, T, F, dtype):
    """Both sides of the bounds on features and steps from 32768 columns on."""
    test_vector_traces(N, T, F, dtype)
