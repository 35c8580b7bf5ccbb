"""Operands off the 16-byte grid (slices of larger buffers), which the
register-staged GEMM kernels take: linears with each operand off in turn, and
whole blocks whose biases or weights are off, unsplit, in k splits, with a split
tail and as planned.  Linears element by element within the rounding bound of
the other tile forms; blocks bit for bit against the same kernel on aligned
copies, and against the oracle."""
import numpy as np
import pytest
import torch
from _gpu import assert_close, dev, double_weights_dev, host
from test_gpu_gemm_plans import _check
from test_gpu_stages import _block_inputs

import oracle
from synth import configs as C
from synth import generator as G

pytestmark = pytest.mark.gpu


def _off(t, n):
    """A contiguous copy of t that starts n elements past a 16-byte boundary."""
    buf = torch.empty(t.numel() + n, device="cuda", dtype=t.dtype)
    v = buf[n:].view(t.shape)
    v.copy_(t)
    return v


# Fewer tiles than slots of either kernel, ragged edges, several rounds (4400 x 4872: 360 tiles of 256).
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (255, 136, 128), (513, 520, 192), (4400, 4872, 64)])
@pytest.mark.parametrize("plan", [None, "256,1", "128,1"])
@pytest.mark.parametrize("operand", ["x", "w", "bias", "out"])
def test_linear(gpu, monkeypatch, operand, plan, M, N, K):
    if plan:
        monkeypatch.setenv("AVITS_GEMM_TILE_linear", plan)
    g = torch.Generator(device="cuda").manual_seed(M * 7919 + N * 31 + K)
    x = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    w = (torch.randn(N, K, device="cuda", generator=g) * 0.05).bfloat16()
    b = (torch.randn(N, device="cuda", generator=g) * 0.05).bfloat16()
    lead = 4 if operand == "out" else 0   # 8 bytes: rows are stored eight bytes at a time
    buf = torch.full((lead + M * N + 4096,), 7.0, device="cuda", dtype=torch.bfloat16)
    out = buf[lead:lead + M * N].view(M, N)
    gpu.avits_linear(_off(x, 1) if operand == "x" else x, _off(w, 1) if operand == "w" else w,
                     _off(b, 1) if operand == "bias" else b, out)
    xs, ws, bs = x.double(), w.double(), b.double()
    ref, mag = xs @ ws.t() + bs, xs.abs() @ ws.abs().t() + bs.abs()
    rest = torch.cat([buf[:lead], buf[lead + M * N:]])
    _check(*(t.double().cpu().numpy() for t in (out, ref, mag, rest)), 2.0 ** -8, K)


PLANS = [None, "256,1,8,2", "256,2,8,2", "256,3,8,2", "256,1,8,2,2,2", "128,1,8,2", "128,3,8,2"]


@pytest.mark.parametrize("plan", PLANS)
@pytest.mark.parametrize("which", ["b_", "w_"])
@pytest.mark.parametrize("kind", ["double", "single"])
def test_block(gpu, monkeypatch, kind, which, plan):
    if plan:
        monkeypatch.setenv("AVITS_GEMM_TILE", plan)
    w = C.TINY_BF16
    n_txt, n_img = 37, 301
    x, pos = _block_inputs(w, n_txt, n_img, seed=53)
    if kind == "double":
        parts = {"txt": G.double_stream_weights(w, 0, 0), "img": G.double_stream_weights(w, 0, 1)}
        ref, _ = oracle.double_block(x, pos, n_txt, parts["txt"], parts["img"], w.H)
    else:
        parts = {"single": G.single_block_weights(w, 0)}
        ref, _ = oracle.single_block(x, pos, parts["single"], w.H)
    t_x, t_pos, outs = dev(x, w.dtype), dev(pos), []
    for off in (True, False):
        on = {s: double_weights_dev(p, w.dtype) for s, p in parts.items()}
        t = {s: {k: _off(v, 1) if off and k.startswith(which) else v for k, v in p.items()} for s, p in on.items()}
        bw = gpu.BlockWeights(gpu.BLOCK_DOUBLE if kind == "double" else gpu.BLOCK_SINGLE, **t)
        out = torch.empty_like(t_x)
        gpu.avits_block_forward(t_x, out, t_pos, n_txt, n_img, bw, w.H)
        torch.cuda.synchronize()
        outs.append(host(out))
    assert_close(outs[0] - x, ref - x, w.dtype, f"{kind} block update, {which} off the grid")
    if plan:   # aligned operands run the same kernel under these plans
        np.testing.assert_array_equal(outs[0], outs[1])
