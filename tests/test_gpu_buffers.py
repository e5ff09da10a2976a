"""Callers' buffers that are no memory of the current device (pageable and pinned host
memory; another device's takes the same route): the entry points that read and write a
caller's buffers by kernels take these by the runtime's copies, with the same results,
and the route is chosen the same way under stream capture."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_09209_amd import surrogate as S  # noqa: E402
from paper_2308_09209_amd import vstitch as V  # noqa: E402

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


def stream():
    return V._stream_handle(None)


def place(shape, where, dtype=torch.float32):
    if where == "device":
        return torch.zeros(shape, dtype=dtype, device="cuda")
    return torch.zeros(shape, dtype=dtype, pin_memory=where == "pinned")


def pair(h, w, seed):
    rng = np.random.default_rng(seed)
    T = np.clip(np.cumsum(rng.normal(size=(h, w)), axis=1) * 12 + 128, 0, 255).round().astype(np.float32)
    return torch.from_numpy(T), torch.from_numpy(np.roll(T, (1, 2), axis=(0, 1)).copy())


@pytest.mark.parametrize("entry", ["vs_flow_run", "vs_flow_run_noalloc"])
@pytest.mark.parametrize("where", [("pageable",) * 4, ("pinned",) * 4, ("device", "pageable", "pageable", "device"),
                                   ("pinned", "device", "device", "pageable")])
@pytest.mark.parametrize("w,h,levels", [(97, 61, 4), (5, 3, 1)])
def test_luma_pairs_in_any_memory(entry, where, w, h, levels):
    yt, ym = pair(h, w, w)
    pf = V.PlainFlow(w, h, lk_levels=levels)
    prm = V.default_params(lk_levels=levels)
    want = [t.cpu() for t in pf(yt.cuda(), ym.cuda())]
    bufs = [place((h, w), k) for k in where[:2]] + [place((h, w, 2), k) for k in where[2:]]
    bufs[0].copy_(yt)
    bufs[1].copy_(ym)
    torch.cuda.synchronize()
    for skip in (None, 2, 3):
        ptrs = [None if i == skip else V._p(b) for i, b in enumerate(bufs)]
        for b in bufs[2:]:
            b.fill_(-7.0)
        torch.cuda.synchronize()
        say(f"[{entry} {w}x{h}] buffers {where} without {skip}")
        if entry == "vs_flow_run":
            st = V.lib().vs_flow_run(pf.hnd, *ptrs, stream())
        else:
            st = V.lib().vs_flow_run_noalloc(w, h, C.byref(prm), *ptrs, stream())
        V.check(st, entry)
        torch.cuda.synchronize()
        for i, f in enumerate(want):
            got = bufs[2 + i].cpu()
            assert torch.equal(got, torch.full_like(f, -7.0) if skip == 2 + i else f)
    pf.close()


@pytest.mark.parametrize("where", ["device", "pageable", "pinned"])
def test_prediction_into_any_memory(where):
    sizes = [(23, 41), (16, 16)]
    P = sum(h * w for h, w in sizes)
    net = S.Net(seed=3, max_pixels=P)
    rng = np.random.default_rng(1)
    x = S.pack(*(torch.from_numpy(rng.integers(0, 256, P).astype(np.float32)).cuda() for _ in range(2)))
    imgs = V.nn_images(sizes)
    want = net.forward(x, imgs).cpu()
    assert want.abs().max() > 0
    pred = place((P, 16), where)
    torch.cuda.synchronize()
    say(f"[prediction] {where}")
    net.forward(x, imgs, pred=pred)
    torch.cuda.synchronize()
    assert torch.equal(pred.cpu(), want)
    net.close()


def test_captured_pairs_and_predictions_replay_on_new_inputs():
    w, h = 97, 61
    pf, n = V.PlainFlow(w, h), w * h
    net, imgs = S.Net(seed=4, max_pixels=n), V.nn_images([(h, w)])
    yt, ym = (torch.zeros((h, w), device="cuda") for _ in range(2))
    flows = [torch.zeros((h, w, 2), device="cuda") for _ in range(2)]
    x, pred = torch.zeros((n, 16), dtype=torch.int16, device="cuda"), torch.zeros((n, 16), device="cuda")

    def step():
        V.check(V.lib().vs_flow_run(pf.hnd, V._p(yt), V._p(ym), V._p(flows[0]), V._p(flows[1]), stream()), "vs_flow_run")
        net.forward(x, imgs, pred=pred)
    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for t in range(4):
        a, b = pair(h, w, 50 + t)
        yt.copy_(a)
        ym.copy_(b)
        x.copy_(S.pack(yt, ym))
        say(f"[capture] replay {t}")
        g.replay()
        torch.cuda.synchronize()
        got = [f.clone() for f in flows] + [pred.clone()]
        step()
        torch.cuda.synchronize()
        for r, e in zip(got, flows + [pred]):
            assert torch.equal(r, e)
    pf.close()
    net.close()
