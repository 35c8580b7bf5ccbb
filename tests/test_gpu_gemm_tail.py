"""The reduce of the GEMM's split tail on ragged rows and on tiles that straddle
the transposed region: a block whose QKV projection runs its tiles in k splits
against the same block unsplit.  Only the order of the fp32 sums differs, so q, k
and v differ by single roundings to bf16 (2^-9 relative, on few elements), and
the update by less than that."""
import numpy as np
import pytest
import torch

import paper_2608_17995_amd as avits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d", [(2, 128), (1, 128), (3, 64)])  # V at columns 512, 256 and 384 (half a tile)
@pytest.mark.parametrize("L,n", [(1, 0), (3, 4), (8, 1), (7, 250), (255, 258)])
@pytest.mark.parametrize("tail,tsp", [(1, 2), (100, 3)])
def test_qkv_tail_reduce(gpu, monkeypatch, H, d, L, n, tail, tsp):
    D, F, S = H * d, 4 * H * d, L + n
    g = torch.Generator(device="cuda").manual_seed(S * 31 + D)
    f = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).bfloat16()  # noqa: E731
    def stream():  # noqa: E306
        mod = f(6, D, std=0.1)
        mod[2::3] += 1.0
        return dict(mod=mod, w_qkv=f(3 * D, D, std=D ** -0.5), b_qkv=f(3 * D, std=0.1), g_q=1 + f(d, std=0.1), g_k=1 + f(d, std=0.1),
                    w_o=f(D, D, std=D ** -0.5), b_o=f(D, std=0.1), w_mlp1=f(F, D, std=D ** -0.5), b_mlp1=f(F, std=0.1),
                    w_mlp2=f(D, F, std=F ** -0.5), b_mlp2=f(D, std=0.1))
    bw = avits.BlockWeights(avits.BLOCK_DOUBLE, txt=stream(), img=stream())
    x = f(S, D)
    i = torch.arange(S, device="cuda", dtype=torch.int32)
    pos = torch.stack([torch.zeros_like(i), i // 8, i % 8], 1).contiguous()
    ws = torch.empty(avits.avits_block_workspace_bytes(bw.kind, S, H, d, F, avits.BF16), dtype=torch.uint8, device="cuda")
    out = {}
    for plan in ("256,1", f"256,1,8,1,{tail},{tsp}"):
        monkeypatch.setenv("AVITS_GEMM_TILE_gemm_qkv", plan)
        y = torch.empty_like(x)
        gpu.avits_block_forward_ex(x, y, pos, L, n, bw, H, workspace=ws)
        out[plan] = (y.double() - x.double()).cpu().numpy()
    a, b = out.values()
    assert np.isfinite(b).all()
    assert np.linalg.norm(a - b) <= 2.0 ** -8 * np.linalg.norm(a)
