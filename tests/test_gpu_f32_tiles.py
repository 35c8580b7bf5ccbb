"""The fp32 kernels at the edges of their tiles: avits_linear on both sides of
the rule between the 32 x 32 and the 64 x 64 tile (every element within a
rounding bound, nothing written past the output), the attention statistics with
fewer keys than waves, ragged key tiles and query tiles, and a block's whole
attention (with V) on short sequences, against 64 bits."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2608_17995_amd as avits

from test_gpu_gemm_plans import _check, _run

pytestmark = pytest.mark.gpu


# 64 x 64 tiles: 1, 2, 16 x 16 = 256 (the VALU kernel) and 16 x 15 = 240 (the matrix one).
@pytest.mark.parametrize("M,N,K", [(31, 40, 64), (33, 96, 192), (1023, 1016, 128), (1023, 952, 64)])
def test_linear_f32_tile_rule(gpu, monkeypatch, M, N, K):
    got, ref, mag, tail = _run(gpu, monkeypatch, M, N, K, torch.float32)
    _check(got, ref, mag, tail, 2.0 ** -24, K)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,nk,text", [(1, 1, 1), (15, 17, 5), (17, 127, 127), (130, 129, 0), (16, 300, 33)])
def test_stats_f32(gpu, n, nk, text, d):
    H = 3
    g = torch.Generator(device="cuda").manual_seed(n * 1000 + nk + d)
    # An odd element offset: nothing may assume more than element alignment.
    q = torch.randn(n * H * d + 1, device="cuda", generator=g)[1:].view(n, H, d)
    k = torch.randn(nk * H * d + 1, device="cuda", generator=g)[1:].view(nk, H, d)
    lse, mass = torch.empty(H, n, device="cuda"), torch.ones(H, n, device="cuda")
    gpu.avits_joint_attention_stats(q, k, text, mass, lse, accumulate=True)
    s = (q.double().permute(1, 0, 2) @ k.double().permute(1, 2, 0).contiguous()) / math.sqrt(d)
    want = torch.logsumexp(s, 2)
    share = torch.exp(s - want[..., None])[..., :text].sum(2)
    # d fp32 products per logit, each at most |q||k|: the logit's error (and, to
    # first order, the statistics') is below d 2^-24 |q||k| / sqrt(d).
    bound = d * 2.0 ** -24 * float(q.norm(dim=2).max() * k.norm(dim=2).max()) / math.sqrt(d) + 1e-6
    assert (lse.double() - want).abs().max() < bound
    assert (mass.double() - 1.0 - share).abs().max() < bound + 2.0 ** -23


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,n", [(1, 0), (0, 15), (3, 14), (16, 33), (5, 250)])
def test_single_block_f32(gpu, L, n, d):
    H, S = 2, L + n
    D, F = H * d, 4 * H * d
    r = np.random.default_rng(S * 7 + d)
    f = lambda *s, std=1.0, mean=0.0: (r.standard_normal(s) * std + mean).astype(np.float32)  # noqa: E731
    w = dict(mod=f(3, D, std=0.1), w_in=f(3 * D + F, D, std=D ** -0.5), b_in=f(3 * D + F, std=0.1), g_q=f(d, std=0.1, mean=1.0),
             g_k=f(d, std=0.1, mean=1.0), w_out=f(D, D + F, std=(D + F) ** -0.5), b_out=f(D, std=0.1))
    w["mod"][2] += 1.0
    x = f(S, D)
    pos = np.stack([np.zeros(S), np.arange(S) // 8, np.arange(S) % 8], 1).astype(np.int32)
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    bw = avits.BlockWeights(avits.BLOCK_SINGLE, single={k: cuda(v) for k, v in w.items()})
    # The workspace holds NaN beforehand: padding must not reach the result.
    ws = torch.full((avits.avits_block_workspace_bytes(bw.kind, S, H, d, F, avits.F32),), 255, dtype=torch.uint8, device="cuda")
    out = torch.empty(S, D, device="cuda")
    gpu.avits_block_forward_ex(cuda(x), out, cuda(pos), L, n, bw, H, workspace=ws)
    want, _ = oracle.single_block(x, pos, w, H)
    err = np.linalg.norm(out.double().cpu().numpy() - want) / np.linalg.norm(want)
    assert err < 3e-6, err
