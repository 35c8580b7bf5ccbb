"""The ping-pong GEMM (256- and 128-wide) at the edges of its rings of LDS tiles
(one to five 64-wide k-tiles: fewer tiles than slots, and the first wraps of
both rings), of its wave blocks (rows and columns that end inside one, at
one, and one past one), of its bands of row tiles (one band, two equal ones,
three of unequal size) and of its rounds (more tiles than CUs: the last round
full or not), element by element within the rounding bound of the other tile
forms; the same kernel through a whole block with an odd text length (a
transposed store that starts at an odd element) unsplit, in two and three k
splits and with a split tail; and operands off the 16-byte grid, which another
kernel takes."""
import numpy as np
import pytest
import torch
from _gpu import assert_close, dev, double_weights_dev, host
from test_gpu_gemm_plans import _check, _run
from test_gpu_stages import _block_inputs

import oracle
from synth import configs as C
from synth import generator as G

pytestmark = pytest.mark.gpu

SHAPES = [(127, 72, 64), (128, 64, 128), (129, 200, 192), (256, 256, 256), (391, 328, 320),
          (2307, 136, 64), (4096, 72, 64), (4400, 264, 128), (4100, 3976, 64)]


@pytest.mark.parametrize("plan", ["256,1", "128,1,8,1"])
@pytest.mark.parametrize("M,N,K", SHAPES, ids=[f"{m}x{n}x{k}" for m, n, k in SHAPES])
def test_linear_edges(gpu, monkeypatch, plan, M, N, K):
    got, ref, mag, tail = _run(gpu, monkeypatch, M, N, K, torch.bfloat16, plan)
    _check(got, ref, mag, tail, 2.0 ** -8, K)


@pytest.mark.parametrize("plan", ["256,1", "256,2", "256,3", "256,1,8,1,2,2", "128,1,8,1", "128,3,8,1"])
@pytest.mark.parametrize("kind", ["double", "single"])
def test_block_odd_rows(gpu, monkeypatch, kind, plan):
    monkeypatch.setenv("AVITS_GEMM_TILE", plan)
    w = C.TINY_BF16
    n_txt, n_img = 37, 301
    x, pos = _block_inputs(w, n_txt, n_img, seed=53)
    if kind == "double":
        wt, wi = G.double_stream_weights(w, 0, 0), G.double_stream_weights(w, 0, 1)
        bw = gpu.BlockWeights(gpu.BLOCK_DOUBLE, txt=double_weights_dev(wt, w.dtype), img=double_weights_dev(wi, w.dtype))
        ref, _ = oracle.double_block(x, pos, n_txt, wt, wi, w.H)
    else:
        ws = G.single_block_weights(w, 0)
        bw = gpu.BlockWeights(gpu.BLOCK_SINGLE, single=double_weights_dev(ws, w.dtype))
        ref, _ = oracle.single_block(x, pos, ws, w.H)
    t_x = dev(x, w.dtype)
    out = torch.empty_like(t_x)
    gpu.avits_block_forward(t_x, out, dev(pos), n_txt, n_img, bw, w.H)
    torch.cuda.synchronize()
    assert_close(host(out) - x, ref - x, w.dtype, f"{kind} block update")


def test_linear_off_the_16_byte_grid(gpu, monkeypatch):
    monkeypatch.setenv("AVITS_GEMM_TILE_linear", "256,1")
    M, N, K = 300, 264, 128
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    w = (torch.randn(N, K, device="cuda", generator=g) * 0.05).bfloat16()
    b = (torch.randn(N + 1, device="cuda", generator=g) * 0.05).bfloat16()[1:]   # 2 bytes off
    buf = torch.full((M * N + 4,), 7.0, device="cuda", dtype=torch.bfloat16)
    out = buf[4:].view(M, N)                                                    # 8 bytes off
    gpu.avits_linear(x, w, b, out)
    torch.cuda.synchronize()
    ref = x.double() @ w.double().t() + b.double()
    # Half an ulp of bf16 per element and the fp32 sums' rounding, as above.
    mag = x.double().abs() @ w.double().abs().t() + b.double().abs()
    bound = 2.0 ** -8 * ref.abs() + 1.01 * (K + 1) * 2.0 ** -24 * mag + 1e-30
    assert torch.all((out.double() - ref).abs() <= bound)
    assert np.all(buf[:4].float().cpu().numpy() == 7.0)
