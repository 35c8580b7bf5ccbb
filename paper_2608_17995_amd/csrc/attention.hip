// Non-causal flash attention with log-sum-exp output (the joint attention of
// Section 3.3.1, Eqs. joint_qk and dit_attn), and its LSE-only form.
//
// bf16: one 256-thread workgroup per (128 query rows, head), 32 rows per
// wave, two workgroups per CU, the row blocks of one head on one XCD.  Key
// tiles of 64 rows and the matching V^T tiles go from memory to LDS directly,
// two tiles of each in flight or in use.  The products of a step (P(t - 1) V
// and S(t + 1) = K Q^T) do not depend on its softmax (of S(t)), so a wave
// issues them interleaved, in a fixed order: the matrix pipe runs under the
// exponentials.
// Bound by: the matrix pipe at the clock that full load leaves (S = 16896, 24 heads:
// 1.6-1.7 GHz, 62 % busy): without the softmax the same loop takes 2.43 ms there,
// without fragment reads 2.83, whole 3.15 (1110 TFLOP/s).  Measured
// before -> now (tiles staged through registers, the softmax between the two
// products): S = 16896 3.71 -> 3.15 ms, 5171 414 -> 345 us, the masked pass of
// S = 2457 119 -> 104 us.  On 16x16x32 products, which the GEMM prefers, 3.28 ms:
// twice the instructions compete with the softmax for issue.
// Both products run on v_mfma_f32_32x32x16_bf16 in transposed form:
//   S^T = K Q^T   -> each lane holds 16 keys x 1 query row (row = lane % 32),
//   O^T = V^T P^T -> each lane holds 16 head-dim values of the same row,
// so a row's online-softmax statistics live in two lanes (l, l ^ 32), and the
// probabilities produced by the first product are, register for register,
// the B operand of the second (the contraction over keys uses the same key
// permutation on both operands).  Softmax runs in the log2 domain with fp32
// statistics.
// Load balance: 128-row units of one head each take one of the two workgroup
// slots of a CU, so a grid that overruns the first slot of every CU by a few
// units leaves most CUs with one unit and some with two.  The launcher then
// splits the overrun units (or, for small grids, every unit) along the keys:
// each piece writes its unnormalised output and (max, sum) per row, and a
// combine kernel merges the pieces in key order.
// fp32: attn_f32_kernel (the exactness path).
#include <stdio.h>
#include <stdlib.h>

#include <type_traits>

#include "kernels.h"

namespace avits {
namespace {

constexpr int kRows = 128;        // query rows per workgroup (4 waves x 32)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ f32x16 mfma32(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// One workgroup's work: a head, its query rows [q_lo, q_hi) and up to two key
// ranges [ks[r], ks[r] + kn[r]).
struct AttnUnit {
  int h;
  int64_t q_lo, q_hi;
  int64_t ks[2], kn[2];
  int lead[2];  // keys at the start of each range that belong to another sequence
};

// Number of row blocks of `rows` query rows per head.
__host__ __device__ inline int64_t attn_row_blocks(const AttnArgs& a, int rows) {
  if (a.segs.n == 0) return (a.Sq + rows - 1) / rows;
  int64_t v = 0;
#pragma unroll
  for (int b = 0; b < kMaxSeqs; ++b)  // static indices: no private copy of the arguments
#pragma unroll
    for (int r = 0; r < 2; ++r) v += b < a.segs.n ? (a.segs.len[b][r] + rows - 1) / rows : 0;
  return v;
}

// Workgroup b of a class of n runs on XCD b mod 8: renumber so that each
// XCD takes a contiguous range of the class's logical ids.
__device__ __forceinline__ int64_t attn_xcd_id(int64_t b, int64_t n) {
  const int64_t x = b % 8;
  int64_t start = 0;
  for (int64_t y = 0; y < x; ++y) start += (n - y + 7) / 8;
  return start + b / 8;
}

// Unit u -> its head, query rows [q_lo, q_hi) and key ranges.  With
// sequences, the row blocks of a head enumerate each sequence's two row
// ranges in turn, and the keys are that sequence's rows.
__device__ __forceinline__ AttnUnit attn_decode(const AttnArgs& a, int rows, int64_t u) {
  const int64_t n_rb = attn_row_blocks(a, rows);
  AttnUnit w;
  w.h = int(u / n_rb);
  int64_t rb = u % n_rb;
  if (a.segs.n == 0) {
    w.q_lo = rb * rows;
    w.q_hi = std::min<int64_t>(a.Sq, w.q_lo + rows);
    w.ks[0] = 0; w.kn[0] = a.Sk;
    w.ks[1] = 0; w.kn[1] = 0;
    return w;
  }
  // Static indices throughout (a dynamically indexed argument array would be
  // copied to private memory).
  w.q_lo = w.q_hi = 0;
  w.ks[0] = w.ks[1] = 0;
  w.kn[0] = w.kn[1] = 0;
  bool found = false;
#pragma unroll
  for (int b = 0; b < kMaxSeqs; ++b) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int64_t nb = b < a.segs.n ? (a.segs.len[b][r] + rows - 1) / rows : 0;
      if (!found && rb < nb) {
        found = true;
        w.q_lo = a.segs.start[b][r] + rb * rows;
        w.q_hi = std::min<int64_t>(a.segs.start[b][r] + a.segs.len[b][r], w.q_lo + rows);
        w.ks[0] = a.segs.start[b][0];
        w.kn[0] = a.segs.len[b][0];
        w.ks[1] = a.segs.start[b][1];
        w.kn[1] = a.segs.len[b][1];
      }
      if (!found) rb -= nb;
    }
  }
  return w;  // every unit of the grid (n_rb * H of them) finds its range
}

// Workgroup -> unit, with the units of one XCD contiguous and head-major, so
// the row blocks of a head share one L2.  Split tail: units below split_from
// take workgroups 0 .. split_from - 1; each later unit runs in ksp pieces
// (workgroups split_from onwards, dispatched after the whole units), piece p
// over key tiles [T p / ksp, T (p + 1) / ksp) of the unit's T key tiles (the
// tiles of its first key range, then of its second); `piece` is the piece's
// slot in the partial buffer (-1 for a whole unit).
__device__ __forceinline__ AttnUnit attn_unit(const AttnArgs& a, int rows, int64_t& piece) {
  const int64_t U = attn_row_blocks(a, rows) * a.H;
  const int64_t bid = blockIdx.x;
  int64_t u;
  int p = 0;
  piece = -1;
  if (bid < a.split_from) {
    u = attn_xcd_id(bid, std::min<int64_t>(a.split_from, U));
  } else {
    const int64_t v = attn_xcd_id(bid - a.split_from, int64_t(gridDim.x) - a.split_from);
    u = a.split_from + v / a.ksp;
    p = int(v % a.ksp);
    piece = v;
  }
  AttnUnit w = attn_decode(a, rows, u);
  // Tiles start on 8-key boundaries, so that the 16-byte V^T loads are
  // aligned; the keys before the range are masked.
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    w.lead[r] = w.kn[r] > 0 ? int(w.ks[r] & 7) : 0;
    w.ks[r] -= w.lead[r];
    w.kn[r] += w.lead[r];
  }
  if (piece >= 0) {
    const int64_t t0 = (w.kn[0] + 63) / 64, T = t0 + (w.kn[1] + 63) / 64;
    const int64_t t_lo = T * p / a.ksp, t_hi = T * (p + 1) / a.ksp;
    // The piece's share of each range (either may be empty).
    const int64_t a0 = std::min(t_lo, t0), b0 = std::min(t_hi, t0);
    const int64_t a1 = std::max(t_lo, t0) - t0, b1 = std::max(t_hi, t0) - t0;
    const int64_t n0 = std::max<int64_t>(0, std::min<int64_t>(w.kn[0], 64 * b0) - 64 * a0);
    const int64_t n1 = std::max<int64_t>(0, std::min<int64_t>(w.kn[1], 64 * b1) - 64 * a1);
    w.ks[0] += 64 * a0;
    w.kn[0] = n0;
    w.ks[1] += 64 * a1;
    w.kn[1] = n1;
    if (a0 > 0) w.lead[0] = 0;
    if (a1 > 0) w.lead[1] = 0;
  }
  return w;
}

// Lane l of a 32x32 MFMA output tile holds row 8*(r/4) + 4*(l/32) + r%4 of
// column l%32 in register r.  With S^T = K Q^T the column is the query row
// and the row is the LDS key row.  Key rows are stored in LDS with bits 2 and
// 3 of their index within the tile swapped, so register r of lane half h
// holds key 16*(r/8) + 8h + 4*((r/4)%2) + r%4 of its 32-key sub-tile: for
// the 16-key chunk c of the P^T operand, lane half h then holds the
// contiguous keys 16c + 8h .. +7, and each V^T operand is a single 16-byte
// LDS read.
template <int DH, bool WITH_V, bool MASS>
__global__ __launch_bounds__(256, 2) void attn_bf16_kernel(const AttnArgs a) {
  constexpr int NW = kRows / 32;             // waves
  constexpr int kKT = 64;                    // keys per tile
  constexpr int kC = DH / 16;                // k steps of S
  constexpr int kDT = WITH_V ? DH / 32 : 1;  // 32-row tiles of O^T
  constexpr int kKC = DH / 8;                // 16-byte chunks per K row
  constexpr int kKR = kWave / kKC;           // K rows per load instruction
  constexpr int kKB = kKT * DH * 2, kVB = DH * kKT * 2;  // bytes of a K and a V^T tile
  constexpr int kKL = kKB / 1024 / NW, kVL = WITH_V ? kVB / 1024 / NW : 0;  // load instructions per wave and tile
  // Two K tiles, then two V^T tiles, without padding: 16-byte chunk c of K row
  // r is at c ^ (r mod 16) (128-byte rows, DH = 64: c ^ (r / 2 mod 8)), of
  // V^T row r at c ^ (r / 2 mod 8): the fragment reads are conflict-free.
  __shared__ __attribute__((aligned(16))) char smem[2 * kKB + (WITH_V ? 2 * kVB : 0)];

  int64_t piece;
  const AttnUnit un = attn_unit(a, 32 * NW, piece);
  const int h = un.h;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int l32 = lane % 32, hi = lane / 32;
  const int64_t row = un.q_lo + wave * 32 + l32;
  const bf16_t* Q = static_cast<const bf16_t*>(a.q);
  const bf16_t* K = static_cast<const bf16_t*>(a.k) + int64_t(h) * a.k_head;
  const bf16_t* VT = static_cast<const bf16_t*>(a.vt) + int64_t(h) * DH * a.ldvt;

  bf16x8 qf[kC];
  {
    const bf16_t* src = Q + std::min<int64_t>(row, un.q_hi - 1) * a.q_tok + h * a.q_head + 8 * hi;
#pragma unroll
    for (int c = 0; c < kC; ++c) qf[c] = as_bf16x8(*reinterpret_cast<const u32x4*>(src + 16 * c));
  }
  const float scale2 = kLog2e * rsqrtf(float(DH));
  float mrow = -INFINITY, lrow = 0.f, trow = 0.f;
  f32x16 oacc[kDT];
#pragma unroll
  for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;

  // Staging: a load instruction moves 1 KB straight to LDS (lane-linear, so
  // the swizzle and the key permutation are applied to each lane's source).
  auto swz_k = [](int r) { return DH == 128 ? r & 15 : (r >> 1) & 7; };
  uint32_t k_off[kKL], v_off[kVL > 0 ? kVL : 1];
#pragma unroll
  for (int j = 0; j < kKL; ++j) {
    const int r = kKR * (wave + NW * j) + lane / kKC;
    const int key = (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1);
    k_off[j] = uint32_t(key) * uint32_t(a.k_tok * 2) + uint32_t(((lane % kKC) ^ swz_k(r)) * 16);
  }
#pragma unroll
  for (int j = 0; j < kVL; ++j) {
    const int r = 8 * (wave + NW * j) + lane / 8;
    v_off[j] = uint32_t(r) * uint32_t(a.ldvt * 2) + uint32_t(((lane % 8) ^ ((r >> 1) & 7)) * 16);
  }
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(uint32_t(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) char*)(&smem[0]))));
  const uint32_t lds_w = lds0 + wave * 1024;
  const int64_t k_bytes = ((a.Sk - 1) * a.k_tok + DH) * 2, v_bytes = int64_t(DH) * a.ldvt * 2;

  // Key tiles: those of the first key range, then the second's.
  const int t0 = int((un.kn[0] + kKT - 1) / kKT);
  const int n_tiles = t0 + int((un.kn[1] + kKT - 1) / kKT);
  // First key of tile `it` and the keys [lo, up) of it that count.
  auto tile_at = [&](int it, int64_t& base, int& lo, int& up) {
    const bool first = it < t0;  // selects, not a dynamic index into un.ks / un.kn
    const int local = first ? it : it - t0;
    base = (first ? un.ks[0] : un.ks[1]) + int64_t(local) * kKT;
    lo = local == 0 ? (first ? un.lead[0] : un.lead[1]) : 0;
    up = int(std::min<int64_t>(kKT, (first ? un.kn[0] : un.kn[1]) - int64_t(local) * kKT));
  };
  // Loads past the last tile have an empty range (nothing is read); rows or
  // columns past the end of K or V^T come back as zeros.
  auto uniform = [](u32x4 r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = __builtin_amdgcn_readfirstlane(r[e]);
    return r;
  };
  auto load_k = [&](int it) {
    int64_t base;
    int lo, up;
    tile_at(it, base, lo, up);
    if (it >= n_tiles) return;
    const u32x4 r = uniform(buffer_rsrc(K + base * a.k_tok, range32(k_bytes - base * a.k_tok * 2)));
    const uint32_t dst = lds_w + (it & 1) * kKB;
#pragma unroll
    for (int j = 0; j < kKL; ++j) lds_load16(dst, k_off[j], r, 0, 1024 * NW * j);
  };
  auto load_v = [&](int it) {
    if constexpr (WITH_V) {
      int64_t base;
      int lo, up;
      tile_at(it, base, lo, up);
      const u32x4 r = uniform(buffer_rsrc(VT + base, range32(v_bytes - base * 2)));
      const uint32_t dst = lds_w + 2 * kKB + (it & 1) * kVB;
#pragma unroll
      for (int j = 0; j < kVL; ++j) lds_load16(dst, v_off[j], r, 0, 1024 * NW * j);
    }
  };
  // Key (within the tile) of accumulator register r of sub-tile t, less 8 h.
  auto key_of = [](int t, int r) { return 32 * t + 16 * (r / 8) + 4 * ((r / 4) & 1) + (r % 4); };

  const int sk = hi ^ swz_k(l32), sv = hi ^ ((l32 >> 1) & 7);
  typedef f32x16 STile[kKT / 32];
  typedef bf16x8 PTile[kKT / 16];
  constexpr int kQK = kC * (kKT / 32), kPV = WITH_V ? kDT * (kKT / 16) : 0;
  constexpr int kRd = 4;  // fragments read ahead of their product
  // Slots 0 .. kPV - 1 of a step are the V^T fragments of O^T += V^T P^T (kDT
  // independent chains), the next kQK the K fragments of S = K Q^T (two).  In
  // this order S(t + 1) and P(t) take over registers that S(t) and P(t - 1)
  // leave: 227 of the 256, where the other order needed 248.
  auto fragment = [&](int i, int kbuf, int vbuf) {
    if (i >= kPV) {
      const int c = (i - kPV) / 2, t = (i - kPV) % 2;
      return as_bf16x8(*reinterpret_cast<const u32x4*>(smem + kbuf * kKB + (l32 + 32 * t) * (DH * 2) +
                                                       ((2 * c) ^ sk) * 16));
    }
    const int c = i / kDT, dt = i % kDT;
    return as_bf16x8(*reinterpret_cast<const u32x4*>(smem + 2 * kKB + vbuf * kVB + (l32 + 32 * dt) * (kKT * 2) +
                                                     ((2 * c) ^ sv) * 16));
  };
  auto product = [&](int i, const bf16x8& f, STile& sn, const PTile& pp) {
    if (i >= kPV) {
      const int c = (i - kPV) / 2, t = (i - kPV) % 2;
      sn[t] = mfma32(f, qf[c], c == 0 ? f32x16{} : sn[t]);
    } else {
      const int c = i / kDT, dt = i % kDT;
      oacc[dt] = mfma32(f, pp[c], oacc[dt]);
    }
  };
  // Keys of tile `it` that do not count: logits to -inf.
  auto mask = [&](int it, STile& s) {
    int64_t k0;
    int lo, up;
    tile_at(it, k0, lo, up);
    if (lo == 0 && up == kKT) return;
    asm volatile("" ::: "memory");  // rare: a branch, not 32 selects on every tile
    const int l = lo - 8 * hi, u = up - 8 * hi;
#pragma unroll
    for (int t = 0; t < kKT / 32; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (key_of(t, r) < l || key_of(t, r) >= u) s[t][r] = -INFINITY;
  };
  // Logits of a tile to probabilities, without a branch, in slices
  // 0 .. n - 1 (in order): the row maximum over the first slices, then the
  // running maximum, then the exponentials and their sum.  corr is the factor
  // the output so far must be multiplied by (1 unless the maximum rose).
  float corr = 1.f, ls = 0.f, mx = -INFINITY;
  auto softmax_slice = [&](int i, int n, STile& s, PTile& p) {
    const int n_max = n / 5, e0 = n_max + 1;
    if (i < n_max) {
      if (i == 0) mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 32; ++e)
        if (e >= 32 * i / n_max && e < 32 * (i + 1) / n_max) mx = fmaxf(mx, s[e / 16][e % 16]);
    } else if (i == n_max) {
      mx = max_xor32(mx) * scale2;
      const float m_new = mx > mrow + 8.f ? mx : mrow;
      corr = __builtin_amdgcn_exp2f(mrow - m_new);
      mrow = m_new;
      ls = 0.f;
    } else {
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        if (e < 32 * (i - e0) / (n - e0) || e >= 32 * (i + 1 - e0) / (n - e0)) continue;
        const float v = __builtin_amdgcn_exp2f(fmaf(s[e / 16][e % 16], scale2, -mrow));
        s[e / 16][e % 16] = v;
        ls += v;
        if constexpr (WITH_V) {
          if (e % 2 == 1) {
            u32x4 w = __builtin_bit_cast(u32x4, p[e / 8]);
            w[(e % 8) / 2] = pack_bf2(s[e / 16][e % 16 - 1], v);
            p[e / 8] = as_bf16x8(w);
          }
        }
      }
      if (i == n - 1) lrow = lrow * corr + ls;
    }
  };
  // The rest of a step, after its products: the text mass of tile `it` and
  // the rescaled output.
  auto finish = [&](int it, const STile& s) {
    if constexpr (MASS) {
      int64_t k0;
      int lo, up;
      tile_at(it, k0, lo, up);
      float ts = k0 < a.mass_keys ? ls : 0.f;
      if (k0 < a.mass_keys && k0 + kKT > a.mass_keys) {
        asm volatile("" ::: "memory");
        ts = 0.f;
        const int lim = int(a.mass_keys - k0) - 8 * hi;
#pragma unroll
        for (int t = 0; t < kKT / 32; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) ts += key_of(t, r) < lim ? s[t][r] : 0.f;
      }
      trow = trow * corr + ts;
    }
    if constexpr (WITH_V) {
      if (__any(corr != 1.f)) {
        // Rare (the max rises by more than 8): keep it a branch, not a
        // multiply by 1 on every tile.
        asm volatile("" ::: "memory");
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) oacc[dt] *= corr;
      }
    }
  };
  // Slots [lo, up) of a step with the softmax of (s, p) spread over them
  // (SOFTMAX), in this order: the compiler, left to itself, puts the products
  // first and the softmax after them, which serialises the two units.
  auto run = [&](auto lo_tag, auto up_tag, auto soft_tag, int kbuf, int vbuf, STile& s, STile& sn, const PTile& pp,
                 PTile& p) {
    constexpr int lo = decltype(lo_tag)::value, up = decltype(up_tag)::value;
    constexpr bool soft = decltype(soft_tag)::value;
    constexpr int n = up - lo > 10 ? up - lo : 10;  // slots
    bf16x8 f[kRd];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = lo; i < up && i < lo + kRd; ++i) f[(i - lo) % kRd] = fragment(i, kbuf, vbuf);
#pragma unroll
    for (int i = lo; i < lo + n; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i < up) {
        product(i, f[(i - lo) % kRd], sn, pp);
        if (i + kRd < up) f[(i - lo) % kRd] = fragment(i + kRd, kbuf, vbuf);
      }
      if (soft) softmax_slice(i - lo, n, s, p);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;
  using Zero = std::integral_constant<int, 0>;
  using Pv = std::integral_constant<int, kPV>;
  using All = std::integral_constant<int, kQK + kPV>;
  // V^T columns of tile `it` that do not count become zeros (their
  // probabilities are 0, but the memory behind them may hold anything).
  auto clear_v = [&](int it) {
    if constexpr (WITH_V) {
      int64_t k0;
      int lo, up;
      tile_at(it, k0, lo, up);
      if (lo == 0 && up == kKT) return;
      for (int i = tid; i < DH * 8; i += 64 * NW) {
        const int r = i / 8, c = i % 8;
        u32x4* d = reinterpret_cast<u32x4*>(smem + 2 * kKB + (it & 1) * kVB + r * (kKT * 2) + (c ^ ((r >> 1) & 7)) * 16);
        if (8 * c >= lo && 8 * c + 8 <= up) continue;
        u32x4 v = *d;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = 8 * c + 2 * e;
          v[e] = (k >= lo && k < up ? v[e] & 0xffffu : 0u) | (k + 1 >= lo && k + 1 < up ? v[e] & 0xffff0000u : 0u);
        }
        *d = v;
      }
      lds_barrier();
    }
  };
  // The loads issued one step ago have landed, for every wave.
  auto step_barrier = [&]() {
    vm_wait<0>();
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  // Step t: the products that do not depend on this tile's softmax, P(t - 1)
  // V(t - 1) and S(t + 1), run on the matrix pipe while the softmax of S(t)
  // runs on the vector units.  K(t + 2) and V(t) are loaded meanwhile (into the
  // buffers of K(t) and V(t - 2), which the last step was the last to read).
  STile sa, sb;
  PTile pa, pb;
  load_k(0);
  load_k(1);
  load_v(0);
  if (n_tiles > 1) vm_wait<kKL + kVL>();
  else vm_wait<kVL>();
  lds_barrier();
  run(Pv(), All(), No(), 0, 0, sb, sa, pa, pa);
  // The step's results are made in it, not sunk to where they are used.
  auto pin = [&](STile& sn, PTile& p) {
#pragma unroll
    for (int i = 0; i < kKT / 32; ++i) asm volatile("" : "+v"(sn[i]));
    if constexpr (WITH_V) {
#pragma unroll
      for (int i = 0; i < kKT / 16; ++i) asm volatile("" : "+v"(p[i]));
#pragma unroll
      for (int i = 0; i < kDT; ++i) asm volatile("" : "+v"(oacc[i]));
    }
    asm volatile("" : "+v"(lrow));
  };
  auto middle = [&](int t, int buf, STile& s, STile& sn, PTile& pp, PTile& p) {  // buf = (t - 1) & 1
    step_barrier();
    load_k(t + 2);
    load_v(t);
    clear_v(t - 1);
    mask(t, s);
    run(Zero(), All(), Yes(), buf, buf, s, sn, pp, p);
    pin(sn, p);
    finish(t, s);
  };
  step_barrier();
  load_k(2);
  mask(0, sa);
  if (n_tiles > 1) run(Pv(), All(), No(), 1, 0, sb, sb, pa, pa);
  run(Zero(), Zero(), Yes(), 0, 0, sa, sb, pa, pa);
  finish(0, sa);
  if (n_tiles > 1) {
    int t = 1;
    for (; t + 2 < n_tiles; t += 2) {
      middle(t, 0, sb, sa, pa, pb);
      middle(t + 1, 1, sa, sb, pb, pa);
    }
    if (t + 1 < n_tiles) {
      middle(t, 0, sb, sa, pa, pb);
#pragma unroll
      for (int i = 0; i < kKT / 32; ++i) sb[i] = sa[i];
#pragma unroll
      for (int i = 0; i < kKT / 16; ++i) pa[i] = pb[i];
      ++t;
    }
    // The last tile: no tile after it to start.
    step_barrier();
    load_v(t);
    clear_v(t - 1);
    mask(t, sb);
    run(Zero(), Pv(), Yes(), 0, (t - 1) & 1, sb, sa, pa, pb);
    finish(t, sb);
#pragma unroll
    for (int i = 0; i < kKT / 16; ++i) pa[i] = pb[i];
  }
  step_barrier();
  clear_v(n_tiles - 1);
  run(Zero(), Pv(), No(), 0, (n_tiles - 1) & 1, sb, sa, pa, pb);

  float l = sum_xor32(lrow);
  const float tm = sum_xor32(trow);
  if (row >= un.q_hi) return;
  if constexpr (WITH_V) {
    if (piece >= 0) {
      // A key piece: its unnormalised output and (max, sum, text sum) per
      // row, in the output's column order, for the combine kernel.
      const int64_t lr = row - un.q_lo;
      float* po = a.part + (piece * kRows + lr) * DH + 4 * hi;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16& o = oacc[dt];
          *reinterpret_cast<float4*>(po + 32 * dt + 8 * q) = make_float4(o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]);
        }
      if (hi == 0) {
        float* pm = a.part_ml + (piece * kRows + lr) * 4;
        *reinterpret_cast<float4*>(pm) = make_float4(mrow, l, MASS ? tm : 0.f, 0.f);
      }
      return;
    }
  }
  if (a.lse && hi == 0) a.lse[int64_t(h) * a.Sq + row] = (mrow + log2f(l)) * kLn2;
  if (MASS && hi == 0) {
    float* dst = a.mass + int64_t(h) * a.Sq + row;
    *dst = (a.mass_accumulate ? *dst : 0.f) + tm / l;
  }
  if constexpr (WITH_V) {
    const float inv = 1.f / l;
    bf16_t* dst = static_cast<bf16_t*>(a.o) + row * a.ldo + int64_t(h) * DH + 4 * hi;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x16& o = oacc[dt];
        const u32x2 w = {pack_bf2(o[4 * q] * inv, o[4 * q + 1] * inv), pack_bf2(o[4 * q + 2] * inv, o[4 * q + 3] * inv)};
        *reinterpret_cast<u32x2*>(dst + 32 * dt + 8 * q) = w;
      }
  }
}

// fp32 attention on v_mfma_f32_16x16x4_f32: a workgroup of eight waves owns 16
// query rows of one head, wave w the 16-key tiles w, w + 8, ...; each wave
// keeps its own online softmax, and the eight results meet in LDS, in wave
// order.  As in the bf16 kernel the products are transposed (S^T = K Q^T,
// O^T = V^T P^T): register r of a lane (g = lane / 16) is key 4 g + r of query
// lane % 16, so the probabilities are the second product's operand as they
// stand, and its V^T operand is one 16-byte load.
// Bound by: latency at the sizes in use.  One thread per query row with the
// keys in a serial loop, which this replaces, put 20 waves on the chip at 288
// rows and 4 heads and took 214 us.
constexpr int kFRows = 16, kFWaves = 8;
template <int DH, bool WITH_V>
__global__ __launch_bounds__(64 * kFWaves) void attn_f32_kernel(const AttnArgs a) {
  constexpr int kC = DH / 16, kP = DH + 4;
  __shared__ __attribute__((aligned(16))) float so[WITH_V ? kFWaves * kFRows * kP : 4];
  __shared__ float4 sml[kFWaves][kFRows];  // max, sum, sum over the keys < mass_keys
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid % kWave, l16 = lane % 16, g = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int64_t q0 = int64_t(blockIdx.x) * kFRows;
  const float* K = static_cast<const float*>(a.k) + h * a.k_head + 4 * g;
  const float* VT = static_cast<const float*>(a.vt) + (int64_t(h) * DH + l16) * a.ldvt + 4 * g;
  f32x4 qf[kC], kf[kC], vf[kC], o[kC];
  {
    const float* Q = static_cast<const float*>(a.q) + std::min<int64_t>(q0 + l16, a.Sq - 1) * a.q_tok + h * a.q_head + 4 * g;
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      qf[j] = load4u(Q + 16 * j);
      o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  const float scale = rsqrtf(float(DH));
  float m = -INFINITY, l = 0.f, tl = 0.f;
  const int64_t n_t = (a.Sk + 15) / 16;
  // Rows past the last key repeat it; their logits are -inf.
  auto load_k = [&](int64_t t) {
    const float* src = K + std::min<int64_t>(16 * t + l16, a.Sk - 1) * a.k_tok;
#pragma unroll
    for (int j = 0; j < kC; ++j) kf[j] = load4u(src + 16 * j);
  };
  load_k(wave);
  for (int64_t t = wave; t < n_t; t += kFWaves) {
    if constexpr (WITH_V) {  // the padding of a V^T row is readable but may hold anything
#pragma unroll
      for (int j = 0; j < kC; ++j) vf[j] = load4u(VT + int64_t(16 * j) * a.ldvt + 16 * t);
    }
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < kC; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = mfma16x16x4(kf[j][e], qf[j][e], s);
    load_k(t + kFWaves);
    const int64_t key = 16 * t + 4 * g;
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = key + r < a.Sk ? s[r] * scale : -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(m, max_xor32(mx));
    const float ref = mx == -INFINITY ? 0.f : mx;  // only -inf so far: every exponential is 0
    const float corr = expf(m - ref);
    m = mx;
    l *= corr;
    tl *= corr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = expf(s[r] - ref);
      l += s[r];
      tl += key + r < a.mass_keys ? s[r] : 0.f;
    }
    if constexpr (WITH_V) {
#pragma unroll
      for (int j = 0; j < kC; ++j) {
        o[j] *= corr;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[j] = mfma16x16x4(key + r < a.Sk ? vf[j][r] : 0.f, s[r], o[j]);
      }
    }
  }
  l += __shfl_xor(l, 16);
  l = sum_xor32(l);
  tl += __shfl_xor(tl, 16);
  tl = sum_xor32(tl);
  if (g == 0) sml[wave][l16] = make_float4(m, l, tl, 0.f);
  if constexpr (WITH_V) {
#pragma unroll
    for (int j = 0; j < kC; ++j) *reinterpret_cast<f32x4*>(&so[(wave * kFRows + l16) * kP + 16 * j + 4 * g]) = o[j];
  }
  __syncthreads();
  constexpr int kQuads = WITH_V ? DH / 4 : 1;  // groups of four output columns
  if (tid >= kFRows * kQuads) return;
  const int r = tid / kQuads, c = tid % kQuads;
  const int64_t row = q0 + r;
  if (row >= a.Sq) return;
  float mt = -INFINITY, den = 0.f, tden = 0.f;
#pragma unroll
  for (int w = 0; w < kFWaves; ++w) mt = fmaxf(mt, sml[w][r].x);
  const float ref = mt == -INFINITY ? 0.f : mt;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kFWaves; ++w) {
    const float4 ml = sml[w][r];
    const float wgt = expf(ml.x - ref);
    den = fmaf(wgt, ml.y, den);
    tden = fmaf(wgt, ml.z, tden);
    if constexpr (WITH_V) v += *reinterpret_cast<const f32x4*>(&so[(w * kFRows + r) * kP + 4 * c]) * wgt;
  }
  if constexpr (WITH_V)
    *reinterpret_cast<f32x4u*>(static_cast<float*>(a.o) + row * a.ldo + int64_t(h) * DH + 4 * c) = v / den;
  if (c != 0) return;
  if (a.lse) a.lse[int64_t(h) * a.Sq + row] = mt + logf(den);
  if (a.mass) {
    float* dst = a.mass + int64_t(h) * a.Sq + row;
    *dst = (a.mass_accumulate ? *dst : 0.f) + tden / den;
  }
}

// Combine the key pieces of each split unit: 16 lanes per query row, eight
// output columns per lane (DH = 128; four for DH = 64), every piece's loads
// issued together.  With m_p, l_p the piece's running max (log2 domain) and
// sum, and O_p its unnormalised output, the row's output is
// sum_p 2^(m_p - m) O_p / sum_p 2^(m_p - m) l_p with m = max_p m_p, and its
// log-sum-exp (m + log2 of the denominator) ln 2: the single-pass result up
// to rounding.  With a text mass, the pieces' text sums t_p merge the same
// way: mass = sum_p 2^(m_p - m) t_p / sum_p 2^(m_p - m) l_p.  Pieces are
// summed in key order.
constexpr int kMaxPieces = 4;
template <int DH>
__global__ __launch_bounds__(256) void attn_combine_kernel(const AttnArgs a) {
  constexpr int kLPR = 16, kCols = DH / kLPR;  // lanes per row, columns per lane
  const int sub = threadIdx.x % kLPR;
  const int64_t n_rb = attn_row_blocks(a, kRows);
  const int64_t n_split = n_rb * a.H - a.split_from;
  const int64_t g = int64_t(blockIdx.x) * (256 / kLPR) + threadIdx.x / kLPR;  // split unit * kRows + row
  if (g >= n_split * kRows) return;
  const int64_t su = g / kRows, lr = g % kRows;
  const AttnUnit un = attn_decode(a, kRows, a.split_from + su);
  const int h = un.h;
  const int64_t row = un.q_lo + lr;
  if (row >= un.q_hi) return;
  float4 ml[kMaxPieces];
  float o[kMaxPieces][kCols];
#pragma unroll
  for (int p = 0; p < kMaxPieces; ++p) {
    if (p < a.ksp) {
      const int64_t pc = (su * a.ksp + p) * kRows + lr;
      ml[p] = *reinterpret_cast<const float4*>(a.part_ml + pc * 4);
      const float* po = a.part + pc * DH + sub * kCols;
#pragma unroll
      for (int e = 0; e < kCols; e += 4) {
        const float4 v = *reinterpret_cast<const float4*>(po + e);
        o[p][e] = v.x; o[p][e + 1] = v.y; o[p][e + 2] = v.z; o[p][e + 3] = v.w;
      }
    }
  }
  float m = -INFINITY;
#pragma unroll
  for (int p = 0; p < kMaxPieces; ++p)
    if (p < a.ksp) m = fmaxf(m, ml[p].x);
  float den = 0.f, tden = 0.f, acc[kCols];
#pragma unroll
  for (int e = 0; e < kCols; ++e) acc[e] = 0.f;
#pragma unroll
  for (int p = 0; p < kMaxPieces; ++p) {
    if (p < a.ksp) {
      const float wgt = __builtin_amdgcn_exp2f(ml[p].x - m);
      den = fmaf(wgt, ml[p].y, den);
      tden = fmaf(wgt, ml[p].z, tden);
#pragma unroll
      for (int e = 0; e < kCols; ++e) acc[e] = fmaf(wgt, o[p][e], acc[e]);
    }
  }
  const float inv = 1.f / den;
  bf16_t* dst = static_cast<bf16_t*>(a.o) + row * a.ldo + int64_t(h) * DH + sub * kCols;
  if constexpr (kCols == 8) {
    *reinterpret_cast<u32x4*>(dst) = u32x4{pack_bf2(acc[0] * inv, acc[1] * inv), pack_bf2(acc[2] * inv, acc[3] * inv),
                                           pack_bf2(acc[4] * inv, acc[5] * inv), pack_bf2(acc[6] * inv, acc[7] * inv)};
  } else {
    *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf2(acc[0] * inv, acc[1] * inv), pack_bf2(acc[2] * inv, acc[3] * inv)};
  }
  if (a.lse && sub == 0) a.lse[int64_t(h) * a.Sq + row] = (m + log2f(den)) * kLn2;
  if (a.mass && sub == 1) {
    float* dst = a.mass + int64_t(h) * a.Sq + row;
    *dst = (a.mass_accumulate ? *dst : 0.f) + tden * inv;
  }
}

// Split-tail plan for the bf16 kernel with V (one sequence or packed ones): whole units
// fill the first workgroup slot of every CU, and the units beyond it run in
// key pieces (or, with fewer units than CUs, every unit is split so that
// the CUs are busy).  Returns ksp (1: no split) and sets split_from and the
// partial pointers.
constexpr int kAttnCUs = 256;
int plan_attn_split(AttnArgs& a, int DH) {
  a.split_from = INT64_MAX;
  a.ksp = 1;
  a.part_ml = nullptr;
  if (!a.part || !a.vt) return 1;
  const int64_t U = attn_row_blocks(a, kRows) * a.H;
  // Fewest key tiles of any unit (every piece must get at least one).
  int64_t T = (a.Sk + 63) / 64;
  if (a.segs.n > 0) {
    T = INT64_MAX;
    for (int b = 0; b < a.segs.n; ++b)
      T = std::min<int64_t>(T, (a.segs.len[b][0] + 63) / 64 + (a.segs.len[b][1] + 63) / 64);
  }
  int64_t from, ksp;
  // Measured on MI355X at S = 1741 (28 key tiles): with at most 128 units,
  // pieces one per CU are fastest; up to 256 units, two per CU; for 336
  // units, 256 whole and the rest in two pieces each (finer pieces lose more
  // to the combine than they gain).
  if (2 * U <= kAttnCUs) {
    from = 0;
    ksp = std::min<int64_t>(kMaxPieces, kAttnCUs / U);
  } else if (U <= kAttnCUs) {
    from = 0;
    ksp = std::min<int64_t>(kMaxPieces, 2 * kAttnCUs / U);
  } else {
    // Both slots of every CU make a round of 2 * 256 units.  A last round of
    // at most 256 units runs in two pieces each; one of up to 384 keeps one
    // whole unit per CU and splits the rest; a fuller one is balanced enough
    // already (984 units at S = 5171: 403 us unsplit, 415 split).
    const int64_t rem = U % (2 * kAttnCUs), base = U - rem;
    if (rem == 0 || rem > kAttnCUs + kAttnCUs / 2) return 1;
    from = rem <= kAttnCUs ? base : base + kAttnCUs;
    ksp = 2;
  }
  // Tuning override "FROM,KSP" (e.g. AVITS_ATTN_SPLIT=256,3; KSP 1 disables).
  if (const char* env = getenv("AVITS_ATTN_SPLIT")) {
    long long f = 0, k = 0;
    if (sscanf(env, "%lld,%lld", &f, &k) == 2 && f >= 0 && f <= U && k >= 1 && k <= kMaxPieces) {
      from = f;
      ksp = k;
    }
  }
  if (from >= U) return 1;
  ksp = std::min<int64_t>(ksp, T);  // at least one key tile per piece
  auto need = [&](int64_t k) { return size_t((U - from) * k) * kRows * (DH + 4) * sizeof(float); };
  while (ksp >= 2 && need(ksp) > a.part_bytes) --ksp;
  if (ksp < 2) return 1;
  const int64_t pieces = (U - from) * ksp;
  a.split_from = from;
  a.ksp = int(ksp);
  a.part_ml = a.part + pieces * kRows * DH;
  return int(ksp);
}

template <int DH>
void launch_dh(AttnArgs a, int dtype, hipStream_t s) {
  const bool with_v = a.vt != nullptr;
  if (dtype == AVITS_BF16) {
    const int64_t U = attn_row_blocks(a, kRows) * a.H;
    const int ksp = plan_attn_split(a, DH);
    const dim3 grid(static_cast<unsigned>(ksp > 1 ? a.split_from + (U - a.split_from) * ksp : U));
    if (with_v) {
      if (a.mass) hipLaunchKernelGGL((attn_bf16_kernel<DH, true, true>), grid, dim3(256), 0, s, a);
      else hipLaunchKernelGGL((attn_bf16_kernel<DH, true, false>), grid, dim3(256), 0, s, a);
      if (ksp > 1) {
        const int64_t rows = (U - a.split_from) * kRows;
        hipLaunchKernelGGL((attn_combine_kernel<DH>), dim3(unsigned(ceil_div64(rows, 16))), dim3(256), 0, s, a);
      }
    } else if (a.mass) {
      hipLaunchKernelGGL((attn_bf16_kernel<DH, false, true>), grid, dim3(256), 0, s, a);
    } else {
      hipLaunchKernelGGL((attn_bf16_kernel<DH, false, false>), grid, dim3(256), 0, s, a);
    }
  } else {
    const dim3 grid(unsigned(ceil_div64(a.Sq, kFRows)), unsigned(a.H));
    if (with_v) hipLaunchKernelGGL((attn_f32_kernel<DH, true>), grid, dim3(64 * kFWaves), 0, s, a);
    else hipLaunchKernelGGL((attn_f32_kernel<DH, false>), grid, dim3(64 * kFWaves), 0, s, a);
  }
}

}  // namespace

int launch_attention(const AttnArgs& a, int dtype, hipStream_t s) {
  if (a.Sq == 0) return AVITS_OK;
  if (a.segs.n > 0 && (dtype != AVITS_BF16 || a.mass))
    return set_error(AVITS_ERR_UNSUPPORTED, "attention: packed sequences need bf16 and no text mass");
  TimedLaunch timed(a.vt ? "attention" : "joint_lse", s);
  if (a.d == 128) launch_dh<128>(a, dtype, s);
  else launch_dh<64>(a, dtype, s);
  return launch_status("attention");
}

}  // namespace avits

using namespace avits;

extern "C" int avits_joint_lse(const void* q, const void* k_all, int64_t N, int64_t Nk, int32_t H, int32_t d,
                               int dtype, float* lse, void* stream) {
  AVITS_REQUIRE(N >= 1 && Nk >= 1 && H >= 1, "joint_lse: N=%lld Nk=%lld H=%d must be >= 1", (long long)N,
                (long long)Nk, H);
  if (d != 64 && d != 128) return set_error(AVITS_ERR_UNSUPPORTED, "joint_lse: head dim %d (need 64 or 128)", d);
  if (dtype != AVITS_F32 && dtype != AVITS_BF16)
    return set_error(AVITS_ERR_UNSUPPORTED, "joint_lse: dtype %d unsupported", dtype);
  AVITS_REQUIRE(q && k_all && lse, "joint_lse: null pointer");
  AttnArgs a{};
  a.q = q;
  a.q_tok = int64_t(H) * d;
  a.q_head = d;
  a.k = k_all;
  a.k_tok = int64_t(H) * d;
  a.k_head = d;
  a.lse = lse;
  a.Sq = N;
  a.Sk = Nk;
  a.H = H;
  a.d = d;
  return launch_attention(a, dtype, static_cast<hipStream_t>(stream));
}

extern "C" int avits_joint_attention_stats(const void* q, const void* k_all, int64_t N, int64_t Nk, int64_t L,
                                           int32_t H, int32_t d, int dtype, float* lse, float* mass, int accumulate,
                                           void* stream) {
  AVITS_REQUIRE(N >= 1 && Nk >= 1 && H >= 1, "joint_attention_stats: N=%lld Nk=%lld H=%d must be >= 1",
                (long long)N, (long long)Nk, H);
  AVITS_REQUIRE(L >= 0 && L <= Nk, "joint_attention_stats: L=%lld outside [0, Nk=%lld]", (long long)L,
                (long long)Nk);
  if (d != 64 && d != 128)
    return set_error(AVITS_ERR_UNSUPPORTED, "joint_attention_stats: head dim %d (need 64 or 128)", d);
  if (dtype != AVITS_F32 && dtype != AVITS_BF16)
    return set_error(AVITS_ERR_UNSUPPORTED, "joint_attention_stats: dtype %d unsupported", dtype);
  AVITS_REQUIRE(q && k_all && mass, "joint_attention_stats: null q/k_all/mass");
  AttnArgs a{};
  a.q = q;
  a.q_tok = int64_t(H) * d;
  a.q_head = d;
  a.k = k_all;
  a.k_tok = int64_t(H) * d;
  a.k_head = d;
  a.lse = lse;
  a.mass = mass;
  a.mass_keys = L;
  a.mass_accumulate = accumulate != 0;
  a.Sq = N;
  a.Sk = Nk;
  a.H = H;
  a.d = d;
  return launch_attention(a, dtype, static_cast<hipStream_t>(stream));
}
