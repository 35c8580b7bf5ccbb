"""avits_block_forward_batched_ex: several images through one block pass,
each with its own modulation vectors (images at different timesteps, whose
timestep reaches every block through the modulation; Section 3.2 runs each
image on its own schedule).  Image b's rows are checked against the oracle
block run with image b's modulation (each image its own joint sequence, as
Section 3.3.1 defines it); changing one image's modulation changes that
image's rows only (bit for bit elsewhere); mod_stride 0 is
avits_block_forward_batched bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from synth import configs as C
from synth import generator as G

from _gpu import assert_close, dev, double_weights_dev, host

pytestmark = pytest.mark.gpu


def _layout(txt, img):
    txt_off = np.concatenate([[0], np.cumsum(txt)]).astype(int).tolist()
    img_off = np.concatenate([[0], np.cumsum(img)]).astype(int).tolist()
    return txt_off, img_off


def _inputs(w, n_txt, n_img, seed):
    x = G.block_input(w, n_txt + n_img, seed)
    g = np.random.default_rng(3000 + seed)
    pos = np.zeros((n_txt + n_img, 3), np.int32)
    pos[n_txt:, 1] = g.integers(0, w.H_hr, n_img)
    pos[n_txt:, 2] = g.integers(0, w.W_hr, n_img)
    return x, pos


def _per_image_mods(base, B, seed, dtype, gate_std=0.0):
    """B modulation blocks [B, n_vec, D] around `base` (shifts and scales
    moved by N(0, 0.3), gates by N(0, 0.3) around theirs, and by N(0, gate_std)
    more), bf16-rounded."""
    g = np.random.default_rng(seed)
    m = np.stack([base + g.normal(0.0, 0.3, base.shape) for _ in range(B)])
    if gate_std:
        m[:, 2::3] += g.normal(0.0, gate_std, m[:, 2::3].shape)
    return np.stack([G.round_to(b, dtype) for b in m])


def _rows_of(b, txt_off, img_off):
    T = txt_off[-1]
    return np.concatenate([np.arange(txt_off[b], txt_off[b + 1]), T + np.arange(img_off[b], img_off[b + 1])])


def _setup(gpu, w, kind, B, seed, gate_std=0.0):
    if kind == "double":
        wt, wi = G.double_stream_weights(w, 0, 0), G.double_stream_weights(w, 0, 1)
        mt, mi = (_per_image_mods(t["mod"], B, seed + i, w.dtype, gate_std) for i, t in enumerate((wt, wi)))
        dt, di = double_weights_dev(wt, w.dtype), double_weights_dev(wi, w.dtype)
        dt["mod"], di["mod"] = dev(mt.reshape(-1, w.D), w.dtype), dev(mi.reshape(-1, w.D), w.dtype)
        bw = gpu.BlockWeights(gpu.BLOCK_DOUBLE, txt=dt, img=di)
        stride = 6 * w.D

        def oracle_image(x, pos, txt_off, img_off, b):
            out, lse = oracle.block_batched(x, pos, txt_off, img_off, w.H, dict(wt, mod=mt[b]), dict(wi, mod=mi[b]))
            return out, lse
        return bw, stride, oracle_image, (dt, di)
    ws_ = G.single_block_weights(w, 0)
    ms = _per_image_mods(ws_["mod"], B, seed, w.dtype, gate_std)
    ds = double_weights_dev(ws_, w.dtype)
    ds["mod"] = dev(ms.reshape(-1, w.D), w.dtype)
    bw = gpu.BlockWeights(gpu.BLOCK_SINGLE, single=ds)

    def oracle_image(x, pos, txt_off, img_off, b):
        return oracle.block_batched(x, pos, txt_off, img_off, w.H, single=dict(ws_, mod=ms[b]))
    return bw, 3 * w.D, oracle_image, (ds,)


@pytest.mark.parametrize("kind", ["double", "single"])
def test_block_batched_per_image_modulation(gpu, kind):
    w = C.TINY_BF16
    txt, img = [32, 0, 7, 129], [200, 77, 1, 64]
    txt_off, img_off = _layout(txt, img)
    B = len(txt)
    x, pos = _inputs(w, txt_off[-1], img_off[-1], seed=31)
    bw, stride, oracle_image, keep = _setup(gpu, w, kind, B, seed=41)
    t_x, t_pos = dev(x, w.dtype), dev(pos)
    out = torch.empty_like(t_x)
    lse = torch.empty(w.H, x.shape[0], device="cuda")
    gpu.avits_block_forward_batched_ex(t_x, out, t_pos, txt_off, img_off, bw, w.H, stride, lse_out=lse)
    torch.cuda.synchronize()
    got, got_lse = host(out), host(lse)
    for b in range(B):
        rows = _rows_of(b, txt_off, img_off)
        ref, ref_lse = oracle_image(x, pos, txt_off, img_off, b)
        assert_close(got[rows] - x[rows], ref[rows] - x[rows], w.dtype, f"image {b} block update ({kind})")
        assert_close(got_lse[:, rows], ref_lse[:, rows], w.dtype, f"image {b} lse ({kind})")
    # mod_stride 0: every image takes image 0's modulation, exactly the
    # shared-modulation entry point.
    o0, o1 = torch.empty_like(t_x), torch.empty_like(t_x)
    gpu.avits_block_forward_batched_ex(t_x, o0, t_pos, txt_off, img_off, bw, w.H, 0)
    gpu.avits_block_forward_batched(t_x, o1, t_pos, txt_off, img_off, bw, w.H)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(host(o0), host(o1))
    assert not np.array_equal(host(o0), got)   # the per-image modulation did change the result


# Unsplit (the gates in the GEMM's epilogue), in two and three k splits (in the
# reduce), with every tile or the last one in a split tail (in the tail's
# reduce), the 128-wide form, and the register-staged kernels.
GATED_PLANS = ["256,1", "256,2", "256,3", "256,1,8,1,100,2", "256,1,8,1,1,3", "128,1,8,1", "128,2,8,1", "256,3,8,2",
               "256,1,8,2,100,2", "128,1,8,2"]


@pytest.mark.parametrize("plan", GATED_PLANS)
@pytest.mark.parametrize("kind", ["double", "single"])
def test_per_image_gates_under_every_plan(gpu, monkeypatch, kind, plan):
    # Gates that differ by O(1) between images whose rows end inside a tile:
    # another image's gate anywhere is far outside the bar.
    for family in ("gemm_o", "gemm_mlp_out", "gemm_single_out"):
        monkeypatch.setenv(f"AVITS_GEMM_TILE_{family}", plan)
    w = C.TINY_BF16
    txt, img = [32, 0, 7, 129], [200, 77, 1, 64]
    txt_off, img_off = _layout(txt, img)
    x, pos = _inputs(w, txt_off[-1], img_off[-1], seed=31)
    bw, stride, oracle_image, keep = _setup(gpu, w, kind, len(txt), seed=41, gate_std=1.0)
    t_x = dev(x, w.dtype)
    out = torch.empty_like(t_x)
    gpu.avits_block_forward_batched_ex(t_x, out, dev(pos), txt_off, img_off, bw, w.H, stride)
    torch.cuda.synchronize()
    got = host(out)
    for b in range(len(txt)):
        rows = _rows_of(b, txt_off, img_off)
        ref, _ = oracle_image(x, pos, txt_off, img_off, b)
        assert_close(got[rows] - x[rows], ref[rows] - x[rows], w.dtype, f"image {b} update ({kind}, {plan})")


# Batches of ordinary size whose default plan splits only the tiles past the last
# full round (264 to 336 tiles of 256 x 256), against the same block unsplit: the
# order of the fp32 sums alone differs, so the update differs by single bf16
# roundings of the intermediates, far less than by any other image's gate.
@pytest.mark.parametrize("kind,B,L,n", [("double", 2, 512, 2500), ("double", 3, 512, 1400), ("single", 3, 128, 1741),
                                        ("single", 4, 512, 1229)])
def test_per_image_gates_default_tail(gpu, monkeypatch, kind, B, L, n):
    H, d = 24, 128
    D = H * d
    F = 4 * D
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + n)
    f = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).bfloat16()  # noqa: E731

    def mod(vectors):
        m = f(B, vectors, D, std=0.1)
        m[:, 2::3] = f(B, vectors // 3, D)
        return m.view(B * vectors, D)

    if kind == "double":
        def stream():
            return dict(mod=mod(6), w_qkv=f(3 * D, D, std=0.02), b_qkv=f(3 * D, std=0.02), g_q=1 + f(d, std=0.02),
                        g_k=1 + f(d, std=0.02), w_o=f(D, D, std=0.02), b_o=f(D, std=0.02), w_mlp1=f(F, D, std=0.02),
                        b_mlp1=f(F, std=0.02), w_mlp2=f(D, F, std=0.02), b_mlp2=f(D, std=0.02))
        bw, stride = gpu.BlockWeights(gpu.BLOCK_DOUBLE, txt=stream(), img=stream()), 6 * D
    else:
        one = dict(mod=mod(3), w_in=f(3 * D + F, D, std=0.02), b_in=f(3 * D + F, std=0.02), g_q=1 + f(d, std=0.02),
                   g_k=1 + f(d, std=0.02), w_out=f(D, D + F, std=0.02), b_out=f(D, std=0.02))
        bw, stride = gpu.BlockWeights(gpu.BLOCK_SINGLE, single=one), 3 * D
    txt_off, img_off = _layout([L] * B, [n] * B)
    S = txt_off[-1] + img_off[-1]
    x = f(S, D)
    i = torch.arange(S, device="cuda", dtype=torch.int32)
    pos = torch.stack([torch.zeros_like(i), i // 64 % 64, i % 64], 1).contiguous()
    ws = torch.empty(gpu.avits_block_workspace_bytes(bw.kind, S, H, d, F, gpu.BF16), dtype=torch.uint8, device="cuda")
    out = []
    for plan in (None, "256,1"):
        for family in ("gemm_o", "gemm_mlp_out", "gemm_single_out"):
            if plan:
                monkeypatch.setenv(f"AVITS_GEMM_TILE_{family}", plan)
        y = torch.empty_like(x)
        gpu.avits_block_forward_batched_ex(x, y, pos, txt_off, img_off, bw, H, stride, workspace=ws)
        out.append(y.double() - x.double())
    torch.cuda.synchronize()
    default, unsplit = out
    assert torch.isfinite(default).all()
    # Per 256-row tile, so that one wrong tile is not lost in the whole.
    worst = max(float((default[r:r + 256] - unsplit[r:r + 256]).norm() / unsplit[r:r + 256].norm())
                for r in range(0, S, 256))
    assert worst <= 2.0 ** -7, worst


@pytest.mark.parametrize("kind", ["double", "single"])
def test_per_image_modulation_touches_its_own_rows(gpu, kind):
    # Moving image 2's modulation changes image 2's rows only.
    w = C.TINY_BF16
    txt, img = [16, 9, 24], [40, 130, 3]
    txt_off, img_off = _layout(txt, img)
    B = len(txt)
    x, pos = _inputs(w, txt_off[-1], img_off[-1], seed=5)
    bw, stride, _, devw = _setup(gpu, w, kind, B, seed=7)
    t_x, t_pos = dev(x, w.dtype), dev(pos)
    o1, o2 = torch.empty_like(t_x), torch.empty_like(t_x)
    gpu.avits_block_forward_batched_ex(t_x, o1, t_pos, txt_off, img_off, bw, w.H, stride)
    for d in devw:
        blk = d["mod"].view(B, -1, w.D)
        blk[2] = (blk[2].float() * 1.5 + 0.1).to(blk.dtype)
    gpu.avits_block_forward_batched_ex(t_x, o2, t_pos, txt_off, img_off, bw, w.H, stride)
    torch.cuda.synchronize()
    a, b2 = host(o1), host(o2)
    mine = _rows_of(2, txt_off, img_off)
    others = np.setdiff1d(np.arange(x.shape[0]), mine)
    np.testing.assert_array_equal(b2[others], a[others])
    assert not np.array_equal(b2[mine], a[mine])


@pytest.mark.slow
def test_per_image_modulation_flux_pair(gpu):
    # A CFG-style pair at the FLUX 1024^2 shape, each image at its own
    # timestep's modulation; every 16th row of both images against the oracle.
    w = C.FLUX_1024
    txt, img = [w.L, w.L], [w.k, w.k]
    txt_off, img_off = _layout(txt, img)
    x, pos = _inputs(w, txt_off[-1], img_off[-1], seed=11)
    bw, stride, _, _ = _setup(gpu, w, "double", 2, seed=13)
    t_x = dev(x, w.dtype)
    out = torch.empty_like(t_x)
    gpu.avits_block_forward_batched_ex(t_x, out, dev(pos), txt_off, img_off, bw, w.H, stride)
    torch.cuda.synchronize()
    got = host(out)
    wt, wi = G.double_stream_weights(w, 0, 0), G.double_stream_weights(w, 0, 1)
    mt, mi = _per_image_mods(wt["mod"], 2, 13, w.dtype), _per_image_mods(wi["mod"], 2, 14, w.dtype)
    for b in range(2):
        rows = _rows_of(b, txt_off, img_off)
        n_txt = txt[b]
        sub = rows[::16]
        local = np.searchsorted(rows, sub)
        ref, _ = oracle.double_block(x[rows], pos[rows], n_txt, dict(wt, mod=mt[b]), dict(wi, mod=mi[b]), w.H,
                                     rows=local)
        assert_close(got[sub] - x[sub], ref - x[sub], w.dtype, f"FLUX pair image {b}")
