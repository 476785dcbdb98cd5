"""Layers with enough work, or rows per head, for the library's auxiliary stream
(fp32: any), and a layer just below that line, which stays on the caller's
stream: the results equal those of the stage-timed calls (one stream, one
serial order) bit for bit, for back-to-back calls, for calls that two host
threads enqueue at the same time, and for calls on different inputs that share
one saved and one scratch buffer."""
import dataclasses
import threading

import pytest
import torch

import workloads as wl
from gpu_util import device_inputs, shape_of
from paper_2505_00315_amd import mosa

pytestmark = pytest.mark.gpu

CASES = {
    "bf16_two": wl.small(batch=4, seq_len=1024, d_model=1024, heads=8, d_head=64, k=32, dense_heads=4),
    "bf16_two_long_rows": wl.small(batch=1, seq_len=4500, d_model=64, heads=2, d_head=32, k=4000, dense_heads=1),
    "bf16_one": wl.small(batch=3, seq_len=1024, d_model=1024, heads=8, d_head=64, k=32, dense_heads=4),
    "f32_two": wl.small(batch=2, seq_len=96, d_model=128, heads=3, d_head=32, k=20, dense_heads=2, dtype="f32"),
}


def _step(w, dev, stream=None, timer=None):
    shape = shape_of(w)
    weights = {n: dev.get(n) for n in mosa.WEIGHT_NAMES}
    ev = (None, None) if timer is None else timer.sets
    Y, saved, scratch = mosa.forward(shape, dev["X"], weights, stream=stream, events=ev[0])
    grads = {"d" + n: torch.empty_like(dev[n]) for n in mosa.WEIGHT_NAMES if dev.get(n) is not None}
    dX = mosa.backward(shape, dev["X"], weights, dev["dY"], saved, grads, scratch=scratch, stream=stream, events=ev[1])
    return {"Y": Y, "dX": dX, **grads}, (saved, scratch)  # the buffers live until the caller has waited


def _same(a, b, what):
    for n in a:
        assert torch.equal(a[n].view(torch.uint8), b[n].view(torch.uint8)), f"{what}: {n} differs"


@pytest.mark.parametrize("name", list(CASES))
def test_same_as_one_serial_order(name):
    w = CASES[name]
    print(f"\n[case] {w}", flush=True)
    dev = device_inputs(wl.make_inputs(w, with_grad=True))
    timer = mosa.StageTimer(sets=2)
    ref, _ = _step(w, dev, timer=timer)
    torch.cuda.synchronize()
    timer.close()
    outs = [_step(w, dev) for _ in range(3)]
    torch.cuda.synchronize()
    for i, (o, _) in enumerate(outs):
        _same(o, ref, f"call {i}")

    got, errors = {}, []

    def worker(t):
        try:
            torch.cuda.set_device(0)
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                kept = [_step(w, dev, stream=s) for _ in range(2)]
            s.synchronize()
            got[t] = [o for o, _ in kept]
        except Exception as exc:  # reported by the main thread
            errors.append(repr(exc))

    threads = [threading.Thread(target=worker, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not errors, errors
    assert sorted(got) == [0, 1]
    for t, outs in got.items():
        for i, o in enumerate(outs):
            _same(o, ref, f"thread {t} call {i}")


@pytest.mark.parametrize("name", list(CASES))
def test_shared_buffers(name):
    """A program keeps one saved and one scratch buffer: the calls of a pass
    rewrite what the previous pass's kernels on either stream read.  Passes on
    two different inputs in turn, enqueued without waiting, forward and
    backward together and forwards alone, equal the one-stream calls."""
    w = CASES[name]
    print(f"\n[case] {w}", flush=True)
    shape = shape_of(w)
    devs = [device_inputs(wl.make_inputs(dataclasses.replace(w, seed=w.seed + i), with_grad=True)) for i in range(2)]
    weights = [{n: dev.get(n) for n in mosa.WEIGHT_NAMES} for dev in devs]
    timer = mosa.StageTimer(sets=2)
    refs = []
    for dev in devs:
        refs.append(_step(w, dev, timer=timer)[0])
        torch.cuda.synchronize()
    timer.close()
    assert not torch.equal(refs[0]["Y"], refs[1]["Y"])
    saved, scratch = mosa.alloc_workspace(shape)
    # every pass has outputs of its own, allocated (and poisoned) beforehand
    passes = [0, 1, 0, 1, 1, 0]
    outs = [{n: torch.full_like(t, float("nan")) for n, t in refs[i].items()} for i in passes]
    ys = [torch.full_like(refs[i]["Y"], float("nan")) for i in passes]
    torch.cuda.synchronize()
    for i, o in zip(passes, outs):
        dev = devs[i]
        mosa.forward(shape, dev["X"], weights[i], Y=o["Y"], saved=saved, scratch=scratch)
        mosa.backward(shape, dev["X"], weights[i], dev["dY"], saved, {n: t for n, t in o.items() if n.startswith("dW")},
                      dX=o["dX"], scratch=scratch)
    for i, y in zip(passes, ys):
        mosa.forward(shape, devs[i]["X"], weights[i], Y=y, saved=saved, scratch=scratch)
    torch.cuda.synchronize()
    for n, (i, o, y) in enumerate(zip(passes, outs, ys)):
        _same(o, refs[i], f"pass {n}")
        _same({"Y": y}, {"Y": refs[i]["Y"]}, f"forward {n}")
