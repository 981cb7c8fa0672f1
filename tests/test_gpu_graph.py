"""The step calls that enqueue kernels only - flashoptim_adamw_step_noalloc over a list, any step call on a single
tensor (the gradient-release call), and an ordinary multi-tensor call whose tables an earlier call has created and
whose descriptors have not changed since - under HIP stream capture: the captured graph is replayed several
times, with eager work and synchronisations in between, and every replay must leave the same bits as the same
calls made eagerly."""
import gc

import pytest
import torch

import paper_2602_23349_amd as fo
import workloads as W

pytestmark = pytest.mark.gpu

# An exception that a test has caught keeps the test's frame, and with it the graph that the test captured, alive in a reference cycle
# until the garbage collector runs.  If that happened within the next test's capture, the destructor of that graph would call into the
# runtime there, fail and end the process.
@pytest.fixture(autouse=True)
def nothing_left_to_collect():
    gc.collect()


B1, B2, EPS = 0.9, 0.999, 1e-8
ARRAYS = ("param", "rho", "m_q", "m_scale", "v_q", "v_scale")


def _raw(t):
    return t.view(torch.int16) if t.element_size() == 2 else t


def _twins(specs, seed):
    a_list, b_list = [], []
    for i, sp in enumerate(specs):
        rs = W.random_state(sp.numel, i, seed=seed, device="cuda")
        g = W.grad_bf16(sp, i, 1, seed=seed, device="cuda", scale=1e-3)
        pair = []
        for _ in range(2):
            b = fo.ParamBuffers(sp.numel, "adamw", with_grad=True)
            b.param.copy_(rs["thp"]); b.rho.copy_(rs["rho"]); b.m_q.copy_(rs["mq"]); b.m_scale.copy_(rs["ms"])
            b.v_q.copy_(rs["vq"]); b.v_scale.copy_(rs["vs"]); b.grad.copy_(g)
            b.lr, b.weight_decay = 1e-3, (0.01 if sp.role == "matrix" else 0.0)
            pair.append(b)
        a_list.append(pair[0]); b_list.append(pair[1])
    return a_list, b_list


def _assert_equal(ref, got, what):
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(ref, got)):
        for k in ARRAYS:
            assert torch.equal(_raw(getattr(a, k)), _raw(getattr(b, k))), (what, i, k)


def test_captured_steps_replay_like_eager_calls():
    specs = W.resnet50()[:30] + W.odd_sizes()[:8]
    ref, got = _twins(specs, seed=41)
    tl_ref, tl_got = fo.TensorList(ref), fo.TensorList(got)
    singles = [tl_got.slice(i) for i in (0, 3, 7)]
    # eager warm-up: the library's per-device set-up (the first AdamW call outside a capture puts the check of the
    # short square root on its stream; the fixed table's address is looked up once) and the tables of tl_got
    fo.adamw_step_exact(tl_ref, B1, B2, EPS, 1)
    fo.adamw_step_noalloc(tl_got, B1, B2, EPS, 1)
    fo.adamw_step_exact(tl_ref, B1, B2, EPS, 1)
    fo.adamw_step_exact(tl_got, B1, B2, EPS, 1)                # creates and uploads this list's tables
    _assert_equal(ref, got, "eager warm-up")
    assert fo.short_sqrt_state() in (1, 2)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fo.adamw_step_noalloc(tl_got, B1, B2, EPS, 2)          # multi-tensor launch, tables from kernel arguments
        for s1 in singles:                                     # single-tensor calls: table-free launches
            fo.adamw_step_exact(s1, B1, B2, EPS, 3)
        fo.adamw_step_exact(tl_got, B1, B2, EPS, 4)            # cached tables, unchanged descriptors: kernels only
    for replay in range(3):
        graph.replay()
        fo.adamw_step_exact(tl_ref, B1, B2, EPS, 2)            # the same calls, eagerly
        for i in (0, 3, 7):
            fo.adamw_step_exact(tl_ref.slice(i), B1, B2, EPS, 3)
        fo.adamw_step_exact(tl_ref, B1, B2, EPS, 4)
        _assert_equal(ref, got, f"replay {replay}")
        # eager work of the program itself between the replays
        for b in got:
            b.grad.mul_(-0.5)
        for b in ref:
            b.grad.mul_(-0.5)
        torch.cuda.synchronize()


@pytest.mark.parametrize("n_tensors", [10, 2])
def test_replays_take_the_rates_of_the_latest_call(n_tensors):
    # the captured kernels read the list's table, and every eager call leaves its rates there, also a common one that its
    # own kernels take from their arguments
    specs = W.odd_sizes()[4:4 + n_tensors] + [W.ParamSpec("big", (70_000 // n_tensors, 33), "matrix")]
    ref, got = _twins(specs, seed=43)
    tl_ref, tl_got = fo.TensorList(ref), fo.TensorList(got)

    def eager(lists, lrs, t):
        for tl in lists:
            for i in range(tl.n):
                tl.set_hyper(i, lr=lrs[i % len(lrs)])
            fo.adamw_step_exact(tl, B1, B2, EPS, t)

    common, differing = [2e-3], [1e-3, 3e-3]
    for before, captured in (([common], common), ([common, [7e-4]], [7e-4]), ([differing], differing),
                             ([differing, common], common), ([common, differing], differing)):
        for lrs in before:                                     # the last of them leaves the captured call's rates
            eager((tl_ref, tl_got), lrs, 1)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            eager((tl_got,), captured, 2)
        for replay, lrs in enumerate((captured, [5e-4], [6e-4], [4e-3, 5e-4, 6e-4], [6e-4], differing, common)):
            if replay:
                eager((tl_ref, tl_got), lrs, 3)
            for _ in range(1 + replay % 2):
                graph.replay()
                eager((tl_ref,), lrs, 2)
            _assert_equal(ref, got, f"captured at {captured}, replay {replay}")


def test_captured_pack_keeps_its_own_header():
    specs = W.odd_sizes()[:9]
    bufs, other = _twins(specs, seed=45)
    size = fo.checkpoint_size("adamw", [sp.numel for sp in specs])
    blob, want = (torch.zeros(size, dtype=torch.uint8, device="cuda") for _ in range(2))
    steps = [7, -1, 1 << 40]
    fo.checkpoint_pack("adamw", bufs, 1, blob)                 # the list's tables
    torch.cuda.synchronize()
    graphs = []
    for step in steps:
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            fo.checkpoint_pack("adamw", bufs, step, blob)
    for replay in range(3):
        for step, graph in zip(steps, graphs):
            for i in range(5):                                 # eager packs of the same list into the same blob
                fo.checkpoint_pack("adamw", bufs, 1000 + i, blob)
            torch.cuda.synchronize()
            graph.replay()
            fo.checkpoint_pack("adamw", other, step, want)
            torch.cuda.synchronize()
            assert torch.equal(blob, want), (replay, step)
            assert fo.checkpoint_unpack("adamw", blob, bufs) == step


def _list_with(bufs, grads, lrs):
    """A descriptor list over `bufs` with other gradient buffers and rates (the same list to the library)."""
    tl = fo.TensorList(bufs)
    for i in range(tl.n):
        tl.set_grad(i, grads[i])
        tl.set_hyper(i, lr=lrs[i % len(lrs)])
    return tl


def test_captured_change_of_descriptors_replays_its_own():
    # gradients of a captured step usually lie in buffers of their own, and the captured call is the first to name them
    specs = W.odd_sizes()[4:16]
    ref, got = _twins(specs, seed=46)
    sets = [[torch.randn(b.numel, device="cuda").mul_(1e-3 * (k + 1)).to(torch.bfloat16) for b in got] for k in range(8)]
    lists = {id(bufs): [_list_with(bufs, sets[k], [1e-3 * (k + 1), 2e-3]) for k in range(8)] for bufs in (ref, got)}
    tl_ref, tl_got = lists[id(ref)], lists[id(got)]
    for tl in (tl_ref[0], tl_got[0]):
        fo.adamw_step_exact(tl, B1, B2, EPS, 1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fo.adamw_step_exact(tl_got[1], B1, B2, EPS, 2)
    for replay in range(3):
        for k in (2, 3, 4, 5, 6, 7):                           # eager steps, each with gradients and rates of its own
            fo.adamw_step_exact(tl_got[k], B1, B2, EPS, 3)
            fo.adamw_step_exact(tl_ref[k], B1, B2, EPS, 3)
        torch.cuda.synchronize()
        graph.replay()
        fo.adamw_step_exact(tl_ref[1], B1, B2, EPS, 2)
        _assert_equal(ref, got, f"replay {replay}")


def test_eager_calls_around_a_captured_change_of_descriptors_use_their_own():
    # a captured call changes nothing until it is replayed, and every replay changes the list's table: an eager call with
    # the captured call's descriptors, or with those of the last eager call, finds other ones there
    specs = W.odd_sizes()[6:15]
    ref, got = _twins(specs, seed=47)
    sets = [[torch.randn(b.numel, device="cuda").mul_(1e-3 * (k + 1)).to(torch.bfloat16) for b in got] for k in range(2)]
    lists = {id(bufs): [_list_with(bufs, sets[k], [1e-3 * (k + 1), 2e-3]) for k in range(2)] for bufs in (ref, got)}
    for bufs in (ref, got):
        fo.adamw_step_exact(lists[id(bufs)][0], B1, B2, EPS, 1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fo.adamw_step_exact(lists[id(got)][1], B1, B2, EPS, 2)
    for step, k in enumerate((1, 0, None, 0, None, None, 1, 0, 0, None, 1)):         # None: a replay
        if k is None:
            graph.replay()
            fo.adamw_step_exact(lists[id(ref)][1], B1, B2, EPS, 2)
        else:
            for bufs in (ref, got):
                fo.adamw_step_exact(lists[id(bufs)][k], B1, B2, EPS, 3)
        _assert_equal(ref, got, f"step {step}")


@pytest.mark.parametrize("first_eager", [1, 0])
def test_list_whose_first_call_is_captured(first_eager):
    # a capture in relaxed mode may allocate, so a list's tables can be made by a captured call: they reach the device
    # with the replays, and an eager call in between may be the first of all to need them
    specs = W.odd_sizes()[5:13]
    ref, got = _twins(specs, seed=48)
    sets = [[torch.randn(b.numel, device="cuda").mul_(1e-3 * (k + 1)).to(torch.bfloat16) for b in got] for k in range(2)]
    lists = {id(bufs): [_list_with(bufs, sets[k], [1e-3 * (k + 1), 2e-3]) for k in range(2)] for bufs in (ref, got)}
    warm, _ = _twins(specs, seed=49)
    fo.adamw_step_exact(warm, B1, B2, EPS, 1)                  # the library's per-device set-up
    size = fo.checkpoint_size("adamw", [sp.numel for sp in specs])
    blob, want = (torch.zeros(size, dtype=torch.uint8, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        fo.adamw_step_exact(lists[id(got)][1], B1, B2, EPS, 2)
        fo.checkpoint_pack("adamw", got, 5, blob)
    for step, k in enumerate((0, None, 0, None, None, 1, None, 0)[1 - first_eager:]):         # None: a replay
        if k is None:
            graph.replay()
            fo.adamw_step_exact(lists[id(ref)][1], B1, B2, EPS, 2)
            fo.checkpoint_pack("adamw", ref, 5, want)
        else:
            for bufs, b in ((ref, want), (got, blob)):
                fo.adamw_step_exact(lists[id(bufs)][k], B1, B2, EPS, 3)
                fo.checkpoint_pack("adamw", bufs, 6, b)
        _assert_equal(ref, got, f"step {step}")
        assert torch.equal(blob, want), step


@pytest.mark.parametrize("mode", ["global", "relaxed"])
def test_calls_that_wait_for_values_refuse_a_capturing_stream_and_leave_the_capture_intact(mode):
    specs = W.odd_sizes()[5:9]
    bufs, ref = _twins(specs, seed=50)
    blob = torch.zeros(fo.checkpoint_size("adamw", [sp.numel for sp in specs]), dtype=torch.uint8, device="cuda")
    x = torch.full((4096,), 2.0, device="cuda")

    def calls():
        yield lambda: fo.quantization_nmse("momentum", False, x)
        yield lambda: fo.checkpoint_unpack("adamw", blob, bufs)
        yield lambda: fo.reconstruction_sweep(8, 0, 1 << 20)
        yield lambda: fo.selftest()

    fo.adamw_step_exact(bufs, B1, B2, EPS, 1)
    fo.adamw_step_exact(ref, B1, B2, EPS, 1)
    fo.checkpoint_pack("adamw", bufs, 3, blob)
    assert fo.quantization_nmse("momentum", False, x) == (0.0, 16384.0)        # (leaves a workspace for the next call)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        for call in calls():
            with pytest.raises(fo.FlashOptimError) as err:
                call()
            assert err.value.status == -4
        fo.adamw_step_exact(bufs, B1, B2, EPS, 2)
    for replay in range(2):
        graph.replay()
        fo.adamw_step_exact(ref, B1, B2, EPS, 2)
        _assert_equal(ref, bufs, f"replay {replay}")
    assert fo.quantization_nmse("momentum", False, x) == (0.0, 16384.0)
    assert fo.checkpoint_unpack("adamw", blob, bufs) == 3
