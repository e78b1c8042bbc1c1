"""One-pass whitening when its workgroups are not all resident at once.

On the CPU, a model of the exchange between workgroup 0 and the others (csrc/rlcs_masked.h): moments,
statistics, a bounded wait, and the words that say who whitens a workgroup's advantages, run in random
order with room for some workgroups of one call or of two overlapping ones. Every
workgroup's advantages must be whitened exactly once, every workgroup must end, and a wait without
a bound must be seen to stop (so that the model can fail).

On the GPU, the kernel forced onto grids that do not fit, with workgroups that leave at once and with
the usual wait, on one stream and on two, against the oracle. Every wait in it is bounded."""
import random

import numpy as np
import pytest

LEFT, CLOSED, TAKEN = "left", "closed", "taken"


class Group:
    def __init__(self, call, g):
        self.call, self.g, self.polls = call, g, 0
        self.state = "moments"

    def step(self, wait):
        """One step; False where nothing changed but the number of polls."""
        c = self.call
        if self.state == "moments":
            c["moments"].add(self.g)
            self.state = "wait"
        elif self.g == 0 and self.state == "wait":
            if len(c["moments"]) < c["G"]:
                return False
            c["stats"] = True
            c["whitened"][0] += 1
            self.state = "closing"
        elif self.state == "closing":
            self.state, self.next = ("take" if c["leavers"] else "end"), 1
            c["closed"] = True
        elif self.state == "take":
            if self.next == c["G"]:
                self.state = "end"
                return True
            old, c["hand"][self.next] = c["hand"][self.next], CLOSED
            if old == LEFT:
                assert c["stored"][self.next]
                c["whitened"][self.next] += 1
            self.next += 1
        elif self.state == "wait":
            if c["stats"]:
                c["whitened"][self.g] += 1
                self.state = "end"
            else:
                self.polls += 1
                if wait is None or self.polls <= wait:
                    return False
                c["stored"][self.g] = True
                self.state = "leave"
        elif self.state == "leave":
            old, c["hand"][self.g] = c["hand"][self.g], LEFT
            self.state = "count"
            if old == CLOSED:
                self.whiten_own()
        elif self.state == "count":
            c["leavers"] += 1
            self.state = "take back" if c["closed"] else "end"
        elif self.state == "take back":
            old, c["hand"][self.g] = c["hand"][self.g], TAKEN
            assert old in (LEFT, CLOSED)
            self.state = "end"
            if old == LEFT:
                self.whiten_own()
        return True

    def whiten_own(self):
        assert self.call["stats"]
        self.call["whitened"][self.g] += 1
        self.state = "end"


def run_model(sizes, room, wait, rng):
    """Calls of `sizes` workgroups with `room` for workgroups at once. True if all of them ended."""
    calls = [dict(G=G, moments=set(), stats=False, closed=False, leavers=0, hand=[None] * G, stored=[False] * G, whitened=[0] * G) for G in sizes]
    waiting = [[Group(c, g) for g in range(c["G"])] for c in calls]  # each call starts its workgroups in order
    resident, quiet = [], 0
    while any(waiting) or resident:
        while len(resident) < room and any(waiting):
            resident.append(rng.choice([w for w in waiting if w]).pop(0))
        x = rng.choice(resident)
        quiet = 0 if x.step(wait) else quiet + 1
        if x.state == "end":
            resident.remove(x)
        if wait is None and quiet > 200 * room:
            return False
    assert all(n == 1 for c in calls for n in c["whitened"])
    return True


@pytest.mark.parametrize("wait", [0, 1, 5])
@pytest.mark.parametrize("sizes,room", [((1,), 1), ((8,), 8), ((9,), 4), ((40,), 7), ((6, 6), 6), ((12, 12), 12), ((7, 9, 5), 8)])
def test_model(sizes, room, wait):
    for seed in range(40):
        assert run_model(sizes, room, wait, random.Random(seed))


def test_model_without_a_bound():
    assert run_model((8,), 8, None, random.Random(0))
    assert not run_model((9,), 4, None, random.Random(0))
    assert not all(run_model((6, 6), 6, None, random.Random(s)) for s in range(20))


def _inputs(N, T, dtype):
    import workloads
    ro = workloads.make_rollout(N, T, seed=N + T, dtype=dtype, p_term=0.01, p_trunc=0.01)
    mask = (np.random.default_rng(N).random((N, T)) < 0.7).astype(np.uint8)
    return ro, mask


@pytest.fixture
def wait_polls():
    import paper_2608_17641_amd as rl

    def set_(n):
        assert rl._native.load().rlcs_testing_set_whitening_wait(n) == rl._native.RLCS_OK
    yield set_
    set_(-1)


@pytest.mark.gpu
@pytest.mark.parametrize("polls", [0, 1, 256])
@pytest.mark.parametrize("N,T,dtype", [(1, 9, "f32"), (40, 250, "f32"), (700, 2300, "f32"), (1024, 4090, "f32"),
                                       (513, 2049, "f32"), (768, 2560, "f32"), (600, 4097, "bf16"), (1023, 7001, "bf16")])
def test_grids_that_do_not_fit(wait_polls, N, T, dtype, polls):
    from cases import TOL, assert_parity
    from test_gpu_masked import run
    ro, mask = _inputs(N, T, dtype)
    wait_polls(polls)
    for tr in (True, False):
        out, ref = run(ro, mask, trunc=tr, normalize=True)
        assert_parity(out, ref, TOL[dtype], label=f"{N}x{T} {dtype} polls={polls} trunc={tr}")


@pytest.mark.gpu
@pytest.mark.parametrize("N,T", [(513, 2049), (600, 2304), (640, 2500), (768, 2560)])
def test_ten_waves_a_workgroup(N, T):
    """As dispatched: more of these rows than the GPU holds workgroups of them."""
    from cases import TOL, assert_parity
    from test_gpu_masked import run
    ro, mask = _inputs(N, T, "f32")
    out, ref = run(ro, mask, normalize=True)
    assert_parity(out, ref, TOL["f32"], label=f"{N}x{T}")


@pytest.mark.gpu
@pytest.mark.parametrize("N,T", [(512, 4096), (1024, 2048)])
def test_two_streams(N, T):
    """Whitened calls of workspaces of their own overlapping on two streams, each of a whole GPU."""
    import torch
    import paper_2608_17641_amd as rl
    ro, mask = _inputs(N, T, "f32")
    d = {k: torch.from_numpy(v).cuda() for k, v in ro.items()}
    m = torch.from_numpy(mask).cuda()
    call = lambda ws, out: rl.rlcs_gae_masked(d["r"], d["v"], m, d["term"], None, None, d["boot"], *out, gamma=1.0,  # noqa: E731
                                              lam=0.95, normalize=True, ws=ws)
    new_ws = lambda: torch.zeros(rl.rlcs_workspace_size_masked(N, T), dtype=torch.uint8, device="cuda")  # noqa: E731
    new_out = lambda: [torch.full((N, T), float("nan"), device="cuda") for _ in range(2)]  # noqa: E731
    ref = call(new_ws(), new_out())
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    sets = [(new_ws(), [new_out() for _ in range(10)]) for _ in streams]
    torch.cuda.synchronize()
    for i in range(10):
        for s, (ws, outs) in zip(streams, sets):
            with torch.cuda.stream(s):
                call(ws, outs[i])
    torch.cuda.synchronize()
    for _, outs in sets:
        for o in outs:
            assert torch.equal(o[0], ref[0]) and torch.equal(o[1], ref[1])
