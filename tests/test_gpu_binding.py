"""The native side of the Python binding (csrc/binding.cpp) against its Python side: the same calls
give the same bits, the same objects for outputs the caller passed, the same errors, and run on the
current stream; what is not a plain call is left to Python."""
import numpy as np
import pytest
import torch

import paper_2608_17641_amd as rl
import workloads

pytestmark = pytest.mark.gpu


class _Python:
    """Stands for the native functions and takes no call."""

    def __getattr__(self, name):
        return lambda *a: NotImplemented


@pytest.fixture
def sides(monkeypatch):
    """run(side, call): the call with the native functions, or without them."""
    native = rl._load_fast()
    taken = []

    class Counting:
        def __getattr__(self, name):
            f = getattr(native, name)

            def g(*a):
                r = f(*a)
                taken.append(r is not NotImplemented)
                return r
            return g

    def run(side, call):
        monkeypatch.setattr(rl, "_fast", Counting() if side == "native" else _Python())
        taken.clear()
        out = call()
        torch.cuda.synchronize()
        return out, list(taken)
    return run


def _dev(x):
    t = torch.from_numpy(np.ascontiguousarray(x))
    return (t.view(torch.bfloat16) if x.dtype == np.uint16 else t).cuda()


def _calls(dtype, layout):
    N, T = 37, 65
    d = {k: _dev(v) for k, v in workloads.make_rollout(N, T, seed=3, dtype=dtype).items()}
    f = {k: _dev(v) for k, v in workloads.make_retrace_full(N, T, 5, seed=4, dtype=dtype).items()}
    m = _dev(workloads.make_multiturn(N, T, seed=5, dtype=dtype)["mask"])
    xv = _dev(workloads.make_vector_trace(N, T, 6, seed=6, dtype=dtype)["x"])
    boot = d.pop("boot")
    p = dict(gamma=0.99, lam=0.95)
    if layout == "time_major":
        d = {k: v.t().contiguous().t() for k, v in d.items()}
    elif layout == "rows":
        pass
    else:  # the first T steps of wider rows
        d = {k: torch.nn.functional.pad(v, (0, 3)).contiguous()[:, :T] for k, v in d.items()}
    r, v, te, tr, bv = (d[k] for k in ("r", "v", "term", "trunc", "bv"))
    te_bool = te != 0
    if layout != "rows":
        return [lambda: rl.rlcs_gae_strided(r, v, te, tr, bv, boot, **p),
                lambda: rl.rlcs_gae_strided(r, v, te, want_ret=False, **p),
                lambda: rl.rlcs_vtrace_strided(r, v, d["log_rho"], te, tr, bv, boot, gamma=1, ws=rl.make_workspace_columns(N, T, "cuda")),
                lambda: rl.rlcs_retrace_strided(r, d["q"], d["eq"], d["log_rho"], te, tr, bv, boot, **p),
                lambda: rl.rlcs_td_lambda_strided(r, v, te, tr, bv, boot, **p),
                lambda: rl.rlcs_discounted_strided(r, te, tr, bv, boot, gamma=0.9),
                lambda: rl.rlcs_elig_trace_strided(d["x"], te, tr, **p),
                lambda: rl.rlcs_episodic_prefix_strided(d["x"], te, boundary="starts_at")]
    ws = torch.zeros(rl.rlcs_workspace_size_masked(N, T), dtype=torch.uint8, device="cuda")
    return [lambda: rl.rlcs_gae(r, v, te_bool, tr, bv, boot, **p),
            lambda: rl.rlcs_gae(r, v, want_ret=False, **p),
            lambda: rl.rlcs_vtrace(r, v, d["log_rho"], te, tr, bv, boot, gamma=1, rho_bar=2, c_bar=1.5),
            lambda: rl.rlcs_vtrace(r, v, d["log_rho"], gamma=0.9, want_pg=False),
            lambda: rl.rlcs_retrace(r, d["q"], d["eq"], d["log_rho"], te, tr, bv, boot, **p),
            lambda: rl.rlcs_retrace_full(f["r"], f["q3"], f["pi3"], f["actions"], f["mu"], f["term"], f["trunc"],
                                         f["bv"], f["boot"], **p),
            lambda: rl.rlcs_td_lambda(r, v, te, tr, bv, boot, ws=rl.make_workspace(N, T, "cuda"), **p),
            lambda: rl.rlcs_discounted(r, te, tr, bv, boot, gamma=0.9),
            lambda: rl.rlcs_elig_trace(d["x"], te, tr, **p),
            lambda: rl.rlcs_episodic_prefix(d["x"], te, tr),
            lambda: rl.rlcs_episodic_prefix(d["x"], te, boundary="starts_at"),
            lambda: rl.rlcs_affine_scan(r, v, boot, reverse=False),
            lambda: rl.rlcs_elig_trace_vec(xv, te, tr, **p),
            lambda: rl.rlcs_gae_masked(r, v, m, te, tr, bv, boot, **p),
            lambda: rl.rlcs_gae_masked(r, v, m, te, tr, bv, boot, normalize=True, ws=ws, **p),
            lambda: rl.rlcs_gae_masked_noalloc(r, v, m, te, normalize=True, want_ret=False, **p)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layout", ["rows", "time_major", "wider_rows"])
def test_same_results(sides, dtype, layout):
    for call in _calls(dtype, layout):
        a, taken = sides("native", call)
        assert taken == [True]
        b, _ = sides("python", call)
        a, b = (x if isinstance(x, tuple) else (x,) for x in (a, b))
        assert len(a) == len(b)
        for x, y in zip(a, b):
            assert (x is None) == (y is None)
            if x is not None:
                assert x.shape == y.shape and x.stride() == y.stride() and x.dtype == y.dtype and torch.equal(x, y)


@pytest.mark.parametrize("side", ["native", "python"])
def test_given_outputs_and_streams(sides, side):
    r, v = (torch.randn(64, 128, device="cuda") for _ in range(2))
    adv, ret = torch.empty_like(r), torch.empty_like(r)
    (a, b), _ = sides(side, lambda: rl.rlcs_gae(r, v, None, None, None, None, adv, ret, gamma=0.9, lam=0.9, want_ret=False))
    assert a is adv and b is ret
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        g = torch.cuda.CUDAGraph()
        rl.rlcs_gae(r, v, gamma=0.9, lam=0.9)
        stream.synchronize()
        with torch.cuda.graph(g, stream=stream):  # capture fails for a launch on any other stream
            x, y = rl.rlcs_gae(r, v, gamma=0.9, lam=0.9)
        for _ in range(3):
            x.zero_()
            g.replay()
            stream.synchronize()
            assert torch.equal(x, adv) and torch.equal(y, ret)


def _bad_calls():
    r = torch.randn(8, 16, device="cuda")
    f = torch.zeros(8, 16, dtype=torch.uint8, device="cuda")
    p = dict(gamma=0.9, lam=0.9)
    return {
        "shape": lambda: rl.rlcs_gae(r, r[:, :8].contiguous(), **p),
        "dtype": lambda: rl.rlcs_gae(r, r.double(), **p),
        "first_dtype": lambda: rl.rlcs_gae(r.double(), r, **p),
        "mixed": lambda: rl.rlcs_gae(r, r.bfloat16(), **p),
        "host": lambda: rl.rlcs_gae(r, r.cpu(), **p),
        "not_contiguous": lambda: rl.rlcs_gae(r, torch.randn(16, 8, device="cuda").t(), **p),
        "strides": lambda: rl.rlcs_gae_strided(r, torch.randn(16, 8, device="cuda").t(), **p),
        "flags": lambda: rl.rlcs_gae(r, r, f.int(), **p),
        "flag_shape": lambda: rl.rlcs_gae(r, r, f[:4], **p),
        "boot": lambda: rl.rlcs_gae(r, r, f, None, None, torch.randn(7, device="cuda"), **p),
        "output": lambda: rl.rlcs_gae(r, r, f, None, None, None, torch.empty(8, 16, device="cuda", dtype=torch.bfloat16), **p),
        "no_values": lambda: rl.rlcs_gae(r, None, **p),
        "no_continuation": lambda: rl.rlcs_gae(r, r, f, f, **p),
        "gamma": lambda: rl.rlcs_gae(r, r, gamma=1.5, lam=0.9),
        "nan": lambda: rl.rlcs_vtrace(r, r, r, gamma=float("nan")),
        "gamma_type": lambda: rl.rlcs_gae(r, r, gamma="1", lam=0.9),
        "boundary": lambda: rl.rlcs_episodic_prefix(r, f, boundary="middle"),
        "dims": lambda: rl.rlcs_elig_trace_vec(r, **p),
        "workspace": lambda: rl.rlcs_gae_masked(r, r, normalize=True, ws=torch.zeros(64, dtype=torch.uint8, device="cuda"), **p),
        "workspace_host": lambda: rl.rlcs_gae(r, r, ws=torch.zeros(64, dtype=torch.uint8), **p),
        "actions": lambda: rl.rlcs_retrace_full(r, r[..., None], r[..., None], f, r, **p),
    }


@pytest.mark.parametrize("name", [
    "shape", "dtype", "first_dtype", "mixed", "host", "not_contiguous", "strides", "flags", "flag_shape", "boot",
    "output", "no_values", "no_continuation", "gamma", "nan", "gamma_type", "boundary", "dims", "workspace",
    "workspace_host", "actions"])
def test_same_errors(sides, name):
    seen = []
    for side in ("native", "python"):
        with pytest.raises(Exception) as e:
            sides(side, _bad_calls()[name])
        seen.append((type(e.value), str(e.value)))
    assert seen[0] == seen[1]


def test_left_to_python(sides):
    r = torch.randn(8, 16, device="cuda")
    ref = rl.rlcs_discounted(r, gamma=0.9)

    class Sub(torch.Tensor):
        pass

    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class Dispatch(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            Dispatch.seen += 1
            return func(*args, **(kwargs or {}))

    class Function(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    out, taken = sides("native", lambda: rl.rlcs_discounted(r.as_subclass(Sub), gamma=0.9))
    assert taken == [False] and torch.equal(out, ref)
    for mode in (Dispatch, Function):
        with mode():
            out, taken = sides("native", lambda: rl.rlcs_discounted(r, gamma=0.9))
        assert taken == [False] and torch.equal(out, ref)
    assert Dispatch.seen > 0
    out, taken = sides("native", lambda: rl.rlcs_discounted(r, gamma=np.float32(0.9)))
    assert taken == [False] and torch.equal(out, ref)
    with torch.inference_mode():
        out, taken = sides("native", lambda: rl.rlcs_discounted(r, gamma=0.9))
        assert taken == [True] and out.is_inference()
    assert torch.equal(out, ref)
    # no batching rule and no autograd: as before, a batched or transformed tensor has no pointer
    for side in ("native", "python"):
        with pytest.raises(RuntimeError):
            sides(side, lambda: torch.func.vmap(lambda x: rl.rlcs_discounted(x, gamma=0.9))(r[None]))
    empty, taken = sides("native", lambda: rl.rlcs_discounted(r[:0], gamma=0.9))
    assert taken == [True] and empty.shape == (0, 16)


def test_default_device(sides):
    """torch's default device is a function mode too; it changes nothing for a call whose
    allocations all name their device, and another mode beside it still leaves the call to Python."""
    from torch.overrides import TorchFunctionMode

    class Function(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    r = torch.randn(8, 16, device="cuda")
    ref = rl.rlcs_discounted(r, gamma=0.9)
    call = lambda: rl.rlcs_discounted(r, gamma=0.9)
    for device in ("cuda", "cpu"):
        with torch.device(device):
            out, taken = sides("native", call)
            assert taken == [True] and out.is_cuda and torch.equal(out, ref)
            with Function():
                out, taken = sides("native", call)
            assert taken == [False] and torch.equal(out, ref)
    torch.set_default_device("cuda")
    try:
        out, taken = sides("native", call)
    finally:
        torch.set_default_device(None)
    assert taken == [True] and torch.equal(out, ref)
