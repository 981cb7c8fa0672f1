"""The enqueue-only convention of the boundary: flashoptim_checkpoint_pack (header, table and sections), the
first step call on a new list (which creates and uploads its device tables) and the first AdamW call of a
process (which puts the check of the short square root on the stream) return while earlier work on the stream
is still running."""
import os
import subprocess
import sys
import threading
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2602_23349_amd as fo
import workloads as W
from helpers import bits16, compare_state, download

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _busy_stream(seconds):
    """A stream kept busy for `seconds` by the library's one-wavefront clock monitor (it ends by itself)."""
    mon = fo.ClockMonitor(n_samples=int(seconds * 1000), seconds_per_sample=1e-3)
    mon.start()
    return mon


def _stream_beside(mon):
    """A stream whose work runs while mon's stream is busy (the runtime maps streams to a few hardware queues, and two on
    the same one run in turn)."""
    for _ in range(16):
        side = torch.cuda.Stream()
        done = torch.cuda.Event()
        with torch.cuda.stream(side):
            torch.zeros(1, device="cuda")
            done.record()
        until = time.perf_counter() + 0.01
        while time.perf_counter() < until:
            if done.query():
                assert not mon.stream.query()
                return side
    raise AssertionError("no stream runs beside the busy one")


def _state(specs, seed):
    bufs, states = [], []
    for i, sp in enumerate(specs):
        rs = W.random_state(sp.numel, i, seed=seed, device="cuda")
        b = fo.ParamBuffers(sp.numel, "adamw", with_grad=True)
        b.param.copy_(rs["thp"]); b.rho.copy_(rs["rho"]); b.m_q.copy_(rs["mq"]); b.m_scale.copy_(rs["ms"])
        b.v_q.copy_(rs["vq"]); b.v_scale.copy_(rs["vs"])
        b.grad.copy_(W.grad_bf16(sp, i, 1, seed=seed, device="cuda"))
        b.lr, b.weight_decay = 1e-3, 0.01
        st = oracle.TensorState(np.zeros(1, np.float32), "adamw")
        st.n = sp.numel
        st.thp = bits16(rs["thp"]); st.rho = rs["rho"].cpu().numpy(); st.mq = rs["mq"].cpu().numpy()
        st.ms = bits16(rs["ms"]); st.vq = rs["vq"].cpu().numpy(); st.vs = bits16(rs["vs"])
        bufs.append(b); states.append(st)
    torch.cuda.synchronize()
    return bufs, states


def test_checkpoint_pack_does_not_wait_for_the_stream():
    specs = W.odd_sizes() + [W.ParamSpec("big", (3_000_000,), "matrix")]
    bufs, states = _state(specs, seed=21)
    size = fo.checkpoint_size("adamw", [s.numel for s in specs])
    blob = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    mon = _busy_stream(0.4)
    t0 = time.perf_counter()
    fo.checkpoint_pack("adamw", bufs, 5, blob, stream=mon.stream)          # first call on this list: creates its plan
    fo.checkpoint_pack("adamw", bufs, 6, blob, stream=mon.stream)          # and a second one through the cached plan
    dt = time.perf_counter() - t0
    still_busy = not mon.stream.query()
    mon.stream.synchronize()
    assert still_busy and dt < 0.3, f"pack took {dt:.3f} s on the host; stream busy afterwards: {still_busy}"
    want = oracle.checkpoint_pack("adamw", states, 6)
    assert np.array_equal(blob.cpu().numpy(), want)
    fresh = [fo.ParamBuffers(s.numel, "adamw", with_grad=False) for s in specs]
    assert fo.checkpoint_unpack("adamw", blob, fresh) == 6
    for a, b in zip(bufs, fresh):
        assert torch.equal(a.param.view(torch.int16), b.param.view(torch.int16)) and torch.equal(a.v_q, b.v_q)


def test_checkpoint_packs_in_any_number_do_not_wait_for_the_stream():
    # twelve packs behind one busy stream, each with its own step in the header; each blob is copied behind its pack
    specs = W.odd_sizes()[:12]
    bufs, states = _state(specs, seed=27)
    size = fo.checkpoint_size("adamw", [s.numel for s in specs])
    blob = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
    kept = torch.zeros((12, size), dtype=torch.uint8, device="cuda")
    fo.checkpoint_pack("adamw", bufs, 1, blob)
    kept[0].copy_(blob)
    torch.cuda.synchronize()
    mon = _busy_stream(0.4)
    t0 = time.perf_counter()
    with torch.cuda.stream(mon.stream):
        for i in range(12):
            fo.checkpoint_pack("adamw", bufs, 100 + i, blob, stream=mon.stream)
            kept[i].copy_(blob)
    dt = time.perf_counter() - t0
    still_busy = not mon.stream.query()
    mon.stream.synchronize()
    assert still_busy and dt < 0.3, f"twelve packs took {dt:.3f} s on the host; stream busy afterwards: {still_busy}"
    for i in range(12):
        assert np.array_equal(kept[i].cpu().numpy(), oracle.checkpoint_pack("adamw", states, 100 + i)), i


def test_descriptor_uploads_behind_a_busy_stream_keep_their_order():
    # every step has other learning rates: none of them may reach an earlier step that has still to run
    specs = W.odd_sizes()
    bufs, _ = _state(specs, seed=25)
    ref, _ = _state(specs, seed=25)
    tl, tl_ref = fo.TensorList(bufs), fo.TensorList(ref)
    fo.adamw_step_exact(tl_ref, 0.9, 0.999, 1e-8, 1)
    fo.adamw_step_exact(tl, 0.9, 0.999, 1e-8, 1)
    torch.cuda.synchronize()
    mon = _busy_stream(0.4)
    t0 = time.perf_counter()
    for t in range(2, 14):
        for i in range(tl.n):
            tl.set_hyper(i, lr=1e-3 * t)
        fo.adamw_step_exact(tl, 0.9, 0.999, 1e-8, t, stream=mon.stream)
        if t == 5:
            dt, still_busy = time.perf_counter() - t0, not mon.stream.query()
    mon.stream.synchronize()
    assert still_busy and dt < 0.3, f"four steps took {dt:.3f} s on the host; stream busy afterwards: {still_busy}"
    for t in range(2, 14):
        for i in range(tl_ref.n):
            tl_ref.set_hyper(i, lr=1e-3 * t)
        fo.adamw_step_exact(tl_ref, 0.9, 0.999, 1e-8, t)
        torch.cuda.synchronize()
    for a, b in zip(ref, bufs):
        assert torch.equal(a.rho, b.rho) and torch.equal(a.param.view(torch.int16), b.param.view(torch.int16))


@pytest.mark.parametrize("n_tensors", [2, 240, 241, 321, 961])
def test_changed_descriptors_in_any_number_do_not_wait_for_the_stream(n_tensors):
    # steps with other gradient buffers, differing rates and other weight decays, in every combination, behind one busy
    # stream (960 words per table update: two for the gradient, one for each of the others);
    # a second thread's multi-tensor call on an idle stream is not held up either
    specs = [W.ParamSpec(f"t{i}", (33 + i % 70,), "matrix") for i in range(n_tensors)]
    bufs, _ = _state(specs, seed=28)
    ref, _ = _state(specs, seed=28)
    idle, _ = _state(specs, seed=29)
    grads = [[torch.randn_like(b.grad, dtype=torch.float32).to(torch.bfloat16) for b in bufs] for _ in range(3)]
    tl, tl_ref, tl_idle = fo.TensorList(bufs), fo.TensorList(ref), fo.TensorList(idle)

    def prepare(t_list, step):
        for i in range(t_list.n):
            if step & 1:
                t_list.set_hyper(i, lr=1e-3 * (step + i % 5))
            if step & 2:
                t_list.set_hyper(i, weight_decay=1e-3 * (step % 7))
            if step & 4:
                t_list.set_grad(i, grads[step % 3][i])

    for t_list in (tl, tl_ref, tl_idle):
        fo.adamw_step_exact(t_list, 0.9, 0.999, 1e-8, 1)
    torch.cuda.synchronize()
    mon = _busy_stream(0.6)
    side = _stream_beside(mon)
    other = threading.Thread(target=lambda: [fo.adamw_step_exact(tl_idle, 0.9, 0.999, 1e-8, 2 + k, stream=side) for k in range(5)])
    spent = 0.0
    for step in range(1, 16):
        prepare(tl, step)
        t0 = time.perf_counter()
        fo.adamw_step_exact(tl, 0.9, 0.999, 1e-8, step, stream=mon.stream)
        spent += time.perf_counter() - t0
    other.start()
    other.join()
    side.synchronize()
    still_busy = not mon.stream.query()
    mon.stream.synchronize()
    assert still_busy and spent < 0.2, f"15 steps took {spent:.3f} s on the host; stream busy afterwards: {still_busy}"
    for step in range(1, 16):
        prepare(tl_ref, step)
        fo.adamw_step_exact(tl_ref, 0.9, 0.999, 1e-8, step)
        torch.cuda.synchronize()
    for a, b in zip(ref, bufs):
        for k in ("param", "rho", "m_q", "m_scale", "v_q", "v_scale"):
            x, y = getattr(a, k), getattr(b, k)
            assert torch.equal(x.view(torch.int16) if x.element_size() == 2 else x, y.view(torch.int16) if y.element_size() == 2 else y), k


def test_calls_that_return_values_wait_for_a_stream_that_stays_busy():
    # behind 50 ms of other work: past the time for which the host watches the kernel's flag
    bufs, _ = _state(W.odd_sizes(), seed=26)
    blob = torch.zeros(fo.checkpoint_size("adamw", [b.numel for b in bufs]), dtype=torch.uint8, device="cuda")
    fo.checkpoint_pack("adamw", bufs, 31, blob)
    x = torch.full((5000,), 2.0, device="cuda")
    torch.cuda.synchronize()
    for _ in range(2):
        mon = _busy_stream(0.05)
        assert fo.quantization_nmse("momentum", False, x, stream=mon.stream) == (0.0, 20000.0)
        fresh = [fo.ParamBuffers(b.numel, "adamw", with_grad=False) for b in bufs]
        mon = _busy_stream(0.05)
        assert fo.checkpoint_unpack("adamw", blob, fresh, stream=mon.stream) == 31
        mon.stream.synchronize()
        for a, b in zip(bufs, fresh):
            assert torch.equal(a.rho, b.rho) and torch.equal(a.v_q, b.v_q)


def test_unpack_behind_other_work_does_not_wait_for_its_copy():
    # 16 GB each way, which takes the copy some 5 ms, behind 20 ms of other work: past the time for which the host watches the
    # check's flag without a pause
    bufs = [fo.ParamBuffers(1 << 30, "sgd", with_grad=False) for _ in range(4)]
    for i, b in enumerate(bufs):
        b.rho.fill_(i + 1)
    blob = torch.empty(fo.checkpoint_size("sgd", [b.numel for b in bufs]), dtype=torch.uint8, device="cuda")
    fo.checkpoint_pack("sgd", bufs, 12, blob)
    assert fo.checkpoint_unpack("sgd", blob, bufs) == 12       # the list's tables
    for b in bufs:
        b.rho.zero_()
    torch.cuda.synchronize()
    mon = _busy_stream(0.02)
    step = fo.checkpoint_unpack("sgd", blob, bufs, stream=mon.stream)
    copying = not mon.stream.query()
    mon.stream.synchronize()
    assert step == 12 and copying
    assert all(bool((b.rho == i + 1).all()) for i, b in enumerate(bufs))


def test_refused_unpack_has_run_when_it_returns():
    # the word by which the check refuses its copy serves later calls, so the copy may not run behind them
    bufs = [fo.ParamBuffers(1 << 30, "sgd", with_grad=False) for _ in range(2)]
    blob = torch.empty(fo.checkpoint_size("sgd", [b.numel for b in bufs]), dtype=torch.uint8, device="cuda")
    fo.checkpoint_pack("sgd", bufs, 12, blob)
    blob[8] ^= 1
    for b in bufs:
        b.rho.fill_(7)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for _ in range(3):
        with pytest.raises(fo.FlashOptimError) as err:
            fo.checkpoint_unpack("sgd", blob, bufs, stream=side)
        assert side.query() and err.value.status == -5
    blob[8] ^= 1
    assert all(bool((b.rho == 7).all()) for b in bufs)
    assert fo.checkpoint_unpack("sgd", blob, bufs) == 12
    assert not any(bool(b.rho.any()) for b in bufs)


@pytest.mark.parametrize("n_tensors", [4092, 4093, 9000])
def test_unpacking_a_long_list_waits_for_its_own_stream_only(n_tensors):
    # headers and tables of 64 KB and more (4092 tensors), which one workgroup compares
    bufs = [fo.ParamBuffers(33 + i % 40, "sgd", with_grad=False) for i in range(n_tensors)]
    for i, b in enumerate(bufs):
        b.rho.fill_(i % 100)
    numels = [b.numel for b in bufs]
    blob = torch.zeros(fo.checkpoint_size("sgd", numels), dtype=torch.uint8, device="cuda")
    fo.checkpoint_pack("sgd", bufs, 77, blob)
    assert fo.checkpoint_unpack("sgd", blob, bufs) == 77       # the list's tables
    torch.cuda.synchronize()
    mon = _busy_stream(0.6)
    side = _stream_beside(mon)
    t0 = time.perf_counter()
    assert fo.checkpoint_unpack("sgd", blob, bufs, stream=side) == 77
    dt = time.perf_counter() - t0
    still_busy = not mon.stream.query()
    mon.stream.synchronize()
    assert still_busy and dt < 0.3, f"unpack took {dt:.3f} s on the host; other stream busy afterwards: {still_busy}"
    for b in bufs[::501]:
        b.rho.zero_()
    for at in (8, 64 + 16 * (n_tensors - 1), 64 + 16 * (n_tensors - 1) + 8):       # version, last tensor's size and offset
        bad = blob.clone()
        bad[at] ^= 1
        with pytest.raises(fo.FlashOptimError) as err:
            fo.checkpoint_unpack("sgd", bad, bufs)
        assert err.value.status == -5
    assert not any(b.rho.any() for b in bufs[::501])
    assert fo.checkpoint_unpack("sgd", blob, bufs) == 77
    assert all((b.rho == i * 501 % 100).all() for i, b in enumerate(bufs[::501]))


def test_packing_lists_that_differ_in_empty_tensors_only():
    # the header grows with every tensor of the list, also with those that have no element
    one = fo.ParamBuffers(64, "sgd")
    for empties in (0, 1, 40, 3):
        bufs = [one] * bool(empties % 2) + [fo.ParamBuffers(0, "sgd") for _ in range(empties)]
        numels = [b.numel for b in bufs]
        blob = torch.full((fo.checkpoint_size("sgd", numels),), 0x5A, dtype=torch.uint8, device="cuda")
        fo.checkpoint_pack("sgd", bufs, 9, blob)
        states = [oracle.TensorState(np.zeros(n, np.float32), "sgd") for n in numels]
        assert np.array_equal(blob.cpu().numpy(), oracle.checkpoint_pack("sgd", states, 9))
        assert fo.checkpoint_unpack("sgd", blob, bufs) == 9


def test_first_step_on_a_new_list_does_not_wait_for_the_stream():
    specs = W.odd_sizes()
    bufs, _ = _state(specs, seed=22)
    ref, _ = _state(specs, seed=22)
    fo.sgd_step([fo.ParamBuffers(64, "sgd")], 0.9)          # library start-up out of the way
    fo.adamw_step_exact(ref, 0.9, 0.999, 1e-8, 3)           # (also runs the once-per-device square-root check)
    torch.cuda.synchronize()
    mon = _busy_stream(0.4)
    t0 = time.perf_counter()
    fo.adamw_step_exact(bufs, 0.9, 0.999, 1e-8, 3, stream=mon.stream)      # new list: new device tables
    dt = time.perf_counter() - t0
    still_busy = not mon.stream.query()
    mon.stream.synchronize()
    assert still_busy and dt < 0.3, f"step call took {dt:.3f} s on the host; stream busy afterwards: {still_busy}"
    for a, b in zip(ref, bufs):
        assert torch.equal(a.rho, b.rho) and torch.equal(a.m_q, b.m_q) and torch.equal(a.v_q, b.v_q)
        assert torch.equal(a.param.view(torch.int16), b.param.view(torch.int16))


def test_first_adamw_call_of_a_process_does_not_wait_for_the_stream():
    # runs in a process of its own: the check of the short square root happens once per process and device
    if os.environ.get("FLASHOPTIM_TEST_FRESH_PROCESS") != "1":
        env = dict(os.environ, FLASHOPTIM_TEST_FRESH_PROCESS="1")
        env.pop("FLASHOPTIM_FORCE_GENERAL_SQRT", None)
        r = subprocess.run([sys.executable, "-u", "-m", "pytest", "-x", "-q", "-p", "no:cacheprovider", "-m", "gpu",
                            os.path.abspath(__file__), "--timeout", "200", "--timeout-method", "thread",
                            "-k", "first_adamw_call_of_a_process"],
                           cwd=ROOT, env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
        assert r.returncode == 0, r.stdout[-3000:]
        assert "1 passed" in r.stdout
        return
    specs = W.odd_sizes()
    hp = dict(beta1=0.9, beta2=0.999, eps=1e-8)
    first, first_states = _state(specs, seed=23)
    other, other_states = _state(specs, seed=24)
    fo.sgd_step([fo.ParamBuffers(64, "sgd")], 0.9)          # library start-up out of the way
    torch.cuda.synchronize()
    assert fo.short_sqrt_state() == 0
    side = torch.cuda.Stream()
    mon = _busy_stream(0.4)
    t0 = time.perf_counter()
    fo.adamw_step_exact(first, hp["beta1"], hp["beta2"], hp["eps"], 2, stream=mon.stream)      # the check goes on the busy stream, then the step
    dt = time.perf_counter() - t0
    # a second stream steps at once: its kernels run before the verdict and take the general square root
    fo.adamw_step_exact(other, hp["beta1"], hp["beta2"], hp["eps"], 2, stream=side)
    side.synchronize()
    still_busy = not mon.stream.query()
    assert still_busy and dt < 0.3, f"step call took {dt:.3f} s on the host; stream busy afterwards: {still_busy}"
    assert fo.short_sqrt_state() == 1                       # waits for the verdict
    mon.stream.synchronize()
    for bufs, states in ((first, first_states), (other, other_states)):
        for i, (b, st, sp) in enumerate(zip(bufs, states, specs)):
            oracle.adamw_step(st, bits16(b.grad), float(np.float32(b.lr)), float(np.float32(b.weight_decay)), hp["beta1"],
                              hp["beta2"], hp["eps"], 2)
            rep = compare_state(download(b), st, where=f"fresh process {sp.name}")
            assert sum(r[1] for r in rep) == 0
