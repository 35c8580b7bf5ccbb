// GEMMs of the MMDiT block (QKV, output projection, MLP), with the bias,
// GELU and gated-residual epilogues fused.
//
// bf16 path (MFMA):
//  - Macro tile 256 x BN x 64, one 512-thread workgroup of 8 waves; two waves
//    per SIMD hide each other's LDS and barrier waits.  Operands on 16-byte
//    boundaries run the ping-pong form (gemm_bf16_pp_kernel, BN 256 or 128,
//    16x16x32 products): the two halves of the workgroup alternate compute and
//    memory phases.  Others run the register-staged kernels on 32x32x16 products:
//    gemm_bf16_staged_kernel (BN 256, ping-pong too) or gemm_bf16_kernel (BN 128).
//  - The MFMA computes C^T = W A^T, so each lane owns groups of four
//    consecutive output columns of one row (8-byte stores in the epilogue).
//  - k-tiles are staged global -> LDS: directly in the ping-pong kernel, through
//    registers and two LDS buffers in the register-staged ones.  LDS rows
//    are 128 bytes (64 bf16) with the 16-byte chunk index XOR-swizzled by
//    (row / 2) mod 8, which makes both the staging writes and the 16-byte
//    fragment reads of 16 consecutive rows bank-conflict free.
//  - The epilogue goes through LDS wave by wave so that every store covers
//    whole row segments (or, for the transposed store, column runs).
//  - Small-N GEMMs (the N = D projections) are split along K when the tile
//    grid would leave most of the 256 CUs idle: each split writes fp32
//    partials and a reduce kernel sums them in split order (deterministic)
//    and applies the epilogue.  When the 256-wide tiles overrun the last
//    full wave of workgroups by a few (the MLP-in projection of the FLUX
//    block: 336 tiles on 256 CUs), only those last tiles are split (the
//    split tail): they run after the whole tiles, in 2-4 k splits, and a
//    small reduce sums their partials, so the partial wave takes a fraction
//    of a tile's time instead of a whole one.
// fp32 path (the exactness path): gemm_f32_kernel on the fp32 matrix instructions, and for many tiles
// gemm_f32_valu_kernel.
#include <stdio.h>
#include <stdlib.h>

#include <type_traits>

#include "kernels.h"

namespace avits {
namespace {

constexpr int kBM = 256, kBK = 64;
constexpr int kCUs = 256;

// GELU with the tanh approximation written through the logistic function:
// 0.5 (1 + tanh(u)) = 1 / (1 + exp(-2u)), on the hardware exp2 and
// reciprocal (about 1 ulp each; the result is rounded to bf16).  Large |x|
// saturate to x and -0.
__device__ __forceinline__ float gelu_fast(float x) {
  const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
  const float e = __builtin_amdgcn_exp2f(-2.f * 1.4426950408889634f * u);
  return x * __builtin_amdgcn_rcpf(1.f + e);
}

__device__ __forceinline__ f32x16 mfma32x32x16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The fused scatter: region 0's final row m (columns from col, stored as
// the vector w) also goes to its canvas row, when the problem has one.
template <typename T, typename V>
__device__ __forceinline__ void scatter_copy(const GemmProblem& p, int64_t m, int64_t col, const V& w) {
  if (!p.scat || m < p.scat_row0) return;
  const int64_t q = p.scat_idx[m - p.scat_row0];
  if (q < 0 || q >= p.scat_n) return;
  *reinterpret_cast<V*>(static_cast<T*>(p.scat) + q * p.scat_ld + col) = w;
}

// Epilogue for four consecutive columns n..n+3 of row m of problem p (the
// four columns never straddle a region boundary: region starts are
// multiples of 4).
template <typename T>
__device__ __forceinline__ void epilogue4(const GemmArgs& a, const GemmProblem& p, int64_t m, int64_t n,
                                          float v0, float v1, float v2, float v3) {
  float v[4] = {v0, v1, v2, v3};
  if (p.bias) {
    const T* b = static_cast<const T*>(p.bias);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] += ld(b, n + r);
  }
  int mode;
  T* out;
  int64_t col, ldo;
  if (n < a.n_split) {
    mode = a.mode0; out = static_cast<T*>(p.out0); col = n; ldo = p.ld0;
  } else if (n < a.n_split2) {
    mode = a.mode1; out = static_cast<T*>(p.out1); col = n - a.n_split; ldo = p.ld1;
  } else {
    mode = a.mode2; out = static_cast<T*>(p.out2); col = n - a.n_split2; ldo = p.ld2;
  }
  if (mode == EPI_GELU) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = gelu_fast(v[r]);
  } else if (mode == EPI_RESID_GATE) {
    const T* res = static_cast<const T*>(p.resid);
    const T* gt = static_cast<const T*>(p.gate);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = ld(res, m * p.ldr + col + r) + ld(gt, n + r) * v[r];
  } else if (mode == EPI_STORE_T) {
#pragma unroll
    for (int r = 0; r < 4; ++r) st(out, (col + r) * ldo + m, v[r]);
    return;
  }
  T* dst = out + m * ldo + col;
  if constexpr (sizeof(T) == 2) {
    u32x2 w = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
    *reinterpret_cast<u32x2*>(dst) = w;
    if (n < a.n_split) scatter_copy<T>(p, m, col, w);
  } else {
    const float4 w = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(dst) = w;
    if (n < a.n_split) scatter_copy<T>(p, m, col, w);
  }
}

// Eight consecutive columns of one row (bf16 output): 16-byte loads of the
// bias, gate and residual and one 16-byte store when the eight columns share
// one output region with a row-major mode and aligned strides; otherwise two
// epilogue4 calls.  Same arithmetic, in the same order, as epilogue4.
__device__ __forceinline__ void epilogue8(const GemmArgs& a, const GemmProblem& p, int64_t m, int64_t n,
                                          const float (&v)[8]) {
  const bool r0 = n < a.n_split, r1 = n < a.n_split2;
  int mode;
  bf16_t* out;
  int64_t col, ldo;
  if (r0) { mode = a.mode0; out = static_cast<bf16_t*>(p.out0); col = n; ldo = p.ld0; }
  else if (r1) { mode = a.mode1; out = static_cast<bf16_t*>(p.out1); col = n - a.n_split; ldo = p.ld1; }
  else { mode = a.mode2; out = static_cast<bf16_t*>(p.out2); col = n - a.n_split2; ldo = p.ld2; }
  const bool same = r0 == (n + 7 < a.n_split) && r1 == (n + 7 < a.n_split2);
  const bool aligned = ((col | ldo) & 7) == 0 && (mode != EPI_RESID_GATE || (p.ldr & 7) == 0);
  if (!same || !aligned || mode == EPI_STORE_T) {
    epilogue4<bf16_t>(a, p, m, n, v[0], v[1], v[2], v[3]);
    epilogue4<bf16_t>(a, p, m, n + 4, v[4], v[5], v[6], v[7]);
    return;
  }
  float x[8];
  if (p.bias) {
    const u32x4 b = *reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.bias) + n);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[2 * e] = v[2 * e] + __uint_as_float(b[e] << 16);
      x[2 * e + 1] = v[2 * e + 1] + __uint_as_float(b[e] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = v[e];
  }
  if (mode == EPI_GELU) {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = gelu_fast(x[e]);
  } else if (mode == EPI_RESID_GATE) {
    const u32x4 r = *reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.resid) + m * p.ldr + col);
    const u32x4 g = *reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.gate) + n);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[2 * e] = __uint_as_float(r[e] << 16) + __uint_as_float(g[e] << 16) * x[2 * e];
      x[2 * e + 1] = __uint_as_float(r[e] & 0xffff0000u) + __uint_as_float(g[e] & 0xffff0000u) * x[2 * e + 1];
    }
  }
  const u32x4 w = {pack_bf2(x[0], x[1]), pack_bf2(x[2], x[3]), pack_bf2(x[4], x[5]), pack_bf2(x[6], x[7])};
  *reinterpret_cast<u32x4*>(out + m * ldo + col) = w;
  if (r0) scatter_copy<bf16_t>(p, m, col, w);
}

// Split-K reduce fused with the modulated layer norm that follows the
// output projection: one wave per output row (N = D columns, 8 per chunk,
// chunk c of lane l at columns 8 (l + 64 c)).  The row's partials are summed
// in split order, the bias and gated residual applied as epilogue4 does, the
// result rounded to bf16 and stored; the layer norm then reads those bf16
// values with the chunk layout and summation order of ln_mod_kernel, so both
// routes give the same bits.
constexpr int kRlnChunks = 8;  // rows up to 64 * 8 * 8 = 4096 columns
template <int SPLITS>
__global__ __launch_bounds__(256) void splitk_reduce_ln_kernel(const GemmArgs a, const float* __restrict__ partial,
                                                               const GemmPostLN post) {
  const int lane = threadIdx.x % kWave;
  const int64_t rows = a.p[0].M + (a.nprob > 1 ? a.p[1].M : 0);
  const int64_t grow = int64_t(blockIdx.x) * 4 + threadIdx.x / kWave;
  if (grow >= rows) return;
  const bool second = grow >= a.p[0].M;
  const int64_t m = second ? grow - a.p[0].M : grow;
  const GemmProblem& p = second ? a.p[1] : a.p[0];
  const int64_t nchunk = a.N / 8;
  // This row's image's gate and LN modulation (one set when a.mod.B == 0).
  const int64_t moff = mod_offset(a.mod, p.row0 + m);
  const bf16_t* bias = static_cast<const bf16_t*>(p.bias);
  const bf16_t* gate = static_cast<const bf16_t*>(p.gate) + moff;
  const bf16_t* res = static_cast<const bf16_t*>(p.resid) + m * p.ldr;
  bf16_t* y = static_cast<bf16_t*>(p.out0) + m * p.ld0;
  u32x4 yv[kRlnChunks];
#pragma unroll
  for (int c = 0; c < kRlnChunks; ++c) {
    const int64_t idx = lane + kWave * c;
    if (idx >= nchunk) continue;
    const int64_t n = 8 * idx;
    float v[8];
#pragma unroll
    for (int k = 0; k < SPLITS; ++k) {
      const float* src = partial + (int64_t(k) * rows + grow) * a.N + n;
      const float4 x0 = *reinterpret_cast<const float4*>(src), x1 = *reinterpret_cast<const float4*>(src + 4);
      const float t[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = k == 0 ? t[e] : v[e] + t[e];
    }
    const u32x4 rw = *reinterpret_cast<const u32x4*>(res + n);
    const u32x4 gw = *reinterpret_cast<const u32x4*>(gate + n);
    const u32x4 bw = bias ? *reinterpret_cast<const u32x4*>(bias + n) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = __uint_as_float(rw[e] << 16) +
                       __uint_as_float(gw[e] << 16) * (v[2 * e] + __uint_as_float(bw[e] << 16));
      const float hi = __uint_as_float(rw[e] & 0xffff0000u) +
                       __uint_as_float(gw[e] & 0xffff0000u) * (v[2 * e + 1] + __uint_as_float(bw[e] & 0xffff0000u));
      yv[c][e] = pack_bf2(lo, hi);
    }
    *reinterpret_cast<u32x4*>(y + n) = yv[c];
    scatter_copy<bf16_t>(p, m, n, yv[c]);
  }
  // Modulated layer norm of the bf16 row.
  const bf16_t* sc = static_cast<const bf16_t*>(post.scale[second ? 1 : 0]) + moff;
  const bf16_t* sh = static_cast<const bf16_t*>(post.shift[second ? 1 : 0]) + moff;
  bf16_t* hr = static_cast<bf16_t*>(post.out) + grow * post.ld;
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < kRlnChunks; ++c) {
    if (lane + kWave * c >= nchunk) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) s += __uint_as_float(yv[c][e] << 16) + __uint_as_float(yv[c][e] & 0xffff0000u);
  }
  const float mean = wave_sum(s) / float(a.N);
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < kRlnChunks; ++c) {
    if (lane + kWave * c >= nchunk) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x0 = __uint_as_float(yv[c][e] << 16) - mean, x1 = __uint_as_float(yv[c][e] & 0xffff0000u) - mean;
      q = fmaf(x0, x0, fmaf(x1, x1, q));
    }
  }
  const float rstd = rsqrtf(wave_sum(q) / float(a.N) + 1e-6f);
#pragma unroll
  for (int c = 0; c < kRlnChunks; ++c) {
    const int64_t idx = lane + kWave * c;
    if (idx >= nchunk) continue;
    const u32x4 g = reinterpret_cast<const u32x4*>(sc)[idx], t = reinterpret_cast<const u32x4*>(sh)[idx];
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = (__uint_as_float(yv[c][e] << 16) - mean) * rstd * (1.f + __uint_as_float(g[e] << 16)) +
                       __uint_as_float(t[e] << 16);
      const float hi = (__uint_as_float(yv[c][e] & 0xffff0000u) - mean) * rstd *
                           (1.f + __uint_as_float(g[e] & 0xffff0000u)) +
                       __uint_as_float(t[e] & 0xffff0000u);
      o[e] = pack_bf2(lo, hi);
    }
    reinterpret_cast<u32x4*>(hr)[idx] = o;
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Renumber them so that XCD x runs a contiguous range of logical ids:
// neighbouring logical tiles share weight / activation tiles in one L2.
__device__ __forceinline__ int64_t xcd_logical_id(int64_t bid, int64_t grid) {
  constexpr int kXcds = 8;
  const int64_t per = grid / kXcds, rem = grid % kXcds;
  const int64_t x = bid % kXcds, i = bid / kXcds;
  return x < rem ? x * (per + 1) + i : rem * (per + 1) + (x - rem) * per + i;
}

// Logical tile -> (problem, tile origin).  Tiles of one problem come first;
// within a problem, consecutive tiles walk down the rows of one column block
// so neighbouring workgroups share the weight tile.
__device__ __forceinline__ bool decode_tile(const GemmArgs& a, int bm, int bn, int64_t tile, int& prob, int64_t& m0,
                                            int64_t& n0) {
  const int64_t tn = (a.N + bn - 1) / bn;
  const int64_t tm0 = (a.p[0].M + bm - 1) / bm;
  const int64_t t0 = tm0 * tn;
  prob = 0;
  int64_t tm = tm0;
  if (tile >= t0) {
    tile -= t0;
    prob = 1;
    if (a.nprob < 2) return false;
    tm = (a.p[1].M + bm - 1) / bm;
  }
  if (tm == 0) return false;
  m0 = (tile % tm) * bm;
  n0 = (tile / tm) * bn;
  return m0 < a.p[prob].M && n0 < a.N;
}

// Workgroup -> (problem, tile origin, k split): the k splits of a tile are
// adjacent logical ids.
__device__ __forceinline__ bool map_tile(const GemmArgs& a, int bm, int bn, int splits, int& prob, int64_t& m0,
                                         int64_t& n0, int& ks) {
  const int64_t bid = xcd_logical_id(blockIdx.x, gridDim.x);
  ks = int(bid % splits);
  return decode_tile(a, bm, bn, bid / splits, prob, m0, n0);
}

// Epilogue through LDS, wave by wave.  The MFMA layout gives each lane four
// consecutive columns of one row, so storing straight from the accumulators
// would send every store instruction to 32 different rows.  Instead each wave
// turns its block around in its own LDS region, 32 rows at a time (no
// workgroup barrier: a wave's LDS operations complete in order): it writes
// the 32 x WN fp32 accumulators, reads them back row-major (WN / 4 lanes per
// row, four columns each) and stores whole row segments; the columns of a
// transposed region are read down the rows instead (four lanes per column,
// eight rows each), so each column's 32 rows go out as one 64-byte run.  A
// lane keeps the same columns for all rows, so its bias, gate, output region
// and mode are loaded once.  The LDS column of a value is XOR-swizzled by 8
// times its 8-row group (WN is a multiple of 32), so the down-the-rows reads
// of a half-wave hit 32 distinct banks and 4-column groups stay aligned.  Split-K
// partials take the row-major path without the epilogue.  The caller passes
// the main loop's LDS once every wave is done with it.
template <int WM, int WN, int TM, int TN>
__device__ __forceinline__ void staged_epilogue(const GemmArgs& a, const GemmProblem& p, int64_t m0, int64_t n0,
                                                bool part, float* __restrict__ pbase, int64_t pld,
                                                const f32x16 (&acc)[TM][TN], float* sm, int wave, int wm, int wn,
                                                int lane) {
  constexpr int P = WN + 4;                  // LDS row pitch (floats)
  constexpr int kLPR = WN / 4;               // lanes per row
  constexpr int kRPI = kWave / kLPR;         // rows per row-major sweep
  constexpr int kIt = 32 / kRPI;             // row-major sweeps per 32-row block
  constexpr int kTIt = WN * 4 / kWave;       // down-the-rows sweeps per 32-row block
  static_assert(32 % kRPI == 0 && (WN * 4) % kWave == 0, "epilogue lane layout");
  float* reg = sm + wave * 32 * P;
  const int l32 = lane % 32, hi = lane / 32;
  auto swz_col = [](int row, int col) { return col ^ (((row >> 3) & 3) << 3); };
  auto mode_of = [&](int64_t n) { return n < a.n_split ? a.mode0 : n < a.n_split2 ? a.mode1 : a.mode2; };

  // Row-major role of this lane: columns n .. n + 3, rows r0 + kRPI * it.
  const int c4 = lane % kLPR, r0 = lane / kLPR;
  const int64_t nb = n0 + wn * WN, n = nb + 4 * c4;
  const bool lane_ok = r0 < kRPI && n < a.N;
  const int mode = lane_ok ? mode_of(n) : EPI_STORE;
  bf16_t* out = nullptr;
  int64_t col = 0, ldo = 0;
  if (n < a.n_split) { out = static_cast<bf16_t*>(p.out0); col = n; ldo = p.ld0; }
  else if (n < a.n_split2) { out = static_cast<bf16_t*>(p.out1); col = n - a.n_split; ldo = p.ld1; }
  else { out = static_cast<bf16_t*>(p.out2); col = n - a.n_split2; ldo = p.ld2; }
  float bias[4] = {0.f, 0.f, 0.f, 0.f}, gate[4] = {0.f, 0.f, 0.f, 0.f};
  if (lane_ok && !part) {
    if (p.bias) {
#pragma unroll
      for (int r = 0; r < 4; ++r) bias[r] = ld(static_cast<const bf16_t*>(p.bias), n + r);
    }
    if (mode == EPI_RESID_GATE) {
#pragma unroll
      for (int r = 0; r < 4; ++r) gate[r] = ld(static_cast<const bf16_t*>(p.gate), n + r);
    }
  }
  const bool row_major = lane_ok && (part || mode != EPI_STORE_T);
  const bool has_t = !part && (a.mode0 == EPI_STORE_T || a.mode1 == EPI_STORE_T || a.mode2 == EPI_STORE_T);

#pragma unroll
  for (int i = 0; i < TM; ++i) {
    // acc[i][j][4q + r] = C[row 32 i + l32][col 32 j + 8 q + 4 hi + r] of this wave's block.
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x16& c = acc[i][j];
        *reinterpret_cast<float4*>(reg + l32 * P + swz_col(l32, 32 * j + 8 * q + 4 * hi)) =
            make_float4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
      }
    const int64_t mb = m0 + wm * WM + 32 * i;  // first output row of the block
    if (row_major) {
      float4 u[kIt];
#pragma unroll
      for (int it = 0; it < kIt; ++it) {
        const int rr = r0 + kRPI * it;
        u[it] = *reinterpret_cast<const float4*>(reg + rr * P + swz_col(rr, 4 * c4));
      }
      if (part) {
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
          const int64_t m = mb + r0 + kRPI * it;
          if (m < p.M) *reinterpret_cast<float4*>(pbase + (m - m0) * pld + (n - n0)) = u[it];
        }
      } else {
        float res[kIt][4];
        if (mode == EPI_RESID_GATE) {
          const bf16_t* rp = static_cast<const bf16_t*>(p.resid);
#pragma unroll
          for (int it = 0; it < kIt; ++it) {
            const int64_t m = std::min<int64_t>(mb + r0 + kRPI * it, p.M - 1);
            const u32x2 w = *reinterpret_cast<const u32x2*>(rp + m * p.ldr + col);
            res[it][0] = __uint_as_float(w[0] << 16);
            res[it][1] = __uint_as_float(w[0] & 0xffff0000u);
            res[it][2] = __uint_as_float(w[1] << 16);
            res[it][3] = __uint_as_float(w[1] & 0xffff0000u);
          }
        }
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
          const int64_t m = mb + r0 + kRPI * it;
          if (m >= p.M) continue;
          float v[4] = {u[it].x + bias[0], u[it].y + bias[1], u[it].z + bias[2], u[it].w + bias[3]};
          if (mode == EPI_GELU) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = gelu_fast(v[r]);
          } else if (mode == EPI_RESID_GATE) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = res[it][r] + gate[r] * v[r];
          }
          const u32x2 w = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
          *reinterpret_cast<u32x2*>(out + m * ldo + col) = w;
          if (n < a.n_split) scatter_copy<bf16_t>(p, m, col, w);
        }
      }
    }
    if (has_t) {
#pragma unroll
      for (int it = 0; it < kTIt; ++it) {
        const int item = it * kWave + lane;
        const int tc = item / 4, mc = item % 4;   // column of the block, 8-row group
        const int64_t nt = nb + tc, m = mb + 8 * mc;
        if (nt >= a.N || m >= p.M || mode_of(nt) != EPI_STORE_T) continue;
        const bf16_t* bp = static_cast<const bf16_t*>(p.bias);
        const float b = bp ? ld(bp, nt) : 0.f;
        bf16_t* o;
        int64_t c0, lo;
        if (nt < a.n_split) { o = static_cast<bf16_t*>(p.out0); c0 = nt; lo = p.ld0; }
        else if (nt < a.n_split2) { o = static_cast<bf16_t*>(p.out1); c0 = nt - a.n_split; lo = p.ld1; }
        else { o = static_cast<bf16_t*>(p.out2); c0 = nt - a.n_split2; lo = p.ld2; }
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = reg[(8 * mc + e) * P + swz_col(8 * mc + e, tc)] + b;
        bf16_t* dst = o + c0 * lo + m;
        if (m + 8 <= p.M) {
          const u32x4 w = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
          *reinterpret_cast<u32x4*>(dst) = w;
        } else {
          for (int e = 0; m + e < p.M; ++e) st(dst, e, v[e]);
        }
      }
    }
  }
}

// Swizzled 16-byte chunk slot of (row, chunk) in a 128-byte LDS row.
__device__ __forceinline__ int swz(int row, int chunk) { return row * 8 + (chunk ^ ((row >> 1) & 7)); }

// The 128-wide register-staged kernel: any alignment, one barrier per k-tile (while
// tile t is multiplied, tiles t + 1 and t + 2 are in flight).
__global__ __launch_bounds__(512) void gemm_bf16_kernel(const GemmArgs a, float* __restrict__ partial, int splits) {
  constexpr int BN = 128, WAVES_M = 2, WAVES_N = 4;
  constexpr int NT = 64 * WAVES_M * WAVES_N;
  constexpr int WM = kBM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 32, TN = WN / 32;  // 32x32 MFMA tiles per wave
  constexpr int CA = kBM * 8 / NT;           // 16-byte A chunks staged per thread per k-tile
  constexpr int CW = BN * 8 / NT;
  constexpr int RS = NT / 8;                 // rows between a thread's chunks
  static_assert(WM % 32 == 0 && WN % 32 == 0 && (BN * 8) % NT == 0 && RS % 16 == 0, "tile shape");
  __shared__ u32x4 lds[2][(kBM + BN) * 8];

  int prob, ks;
  int64_t m0, n0;
  if (!map_tile(a, kBM, BN, splits, prob, m0, n0, ks)) return;
  const GemmProblem p = prob ? a.p[1] : a.p[0];  // by value: a select, no indexed copy of the arguments
  const bf16_t* A = static_cast<const bf16_t*>(p.A);
  const bf16_t* W = static_cast<const bf16_t*>(p.W);
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int l32 = lane % 32, hi = lane / 32;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  const int64_t nk = a.K / kBK;
  const int64_t kt0 = nk * ks / splits, kt1 = nk * (ks + 1) / splits;

  // Staging: thread t moves 16-byte chunk (t % 8) of rows t / 8 + RS j, so all
  // of its chunks share one column offset and one swizzle (RS j / 2 = 0 mod 8).
  // Loads are raw buffer loads with loop-invariant per-thread offsets; the
  // k-advance moves the scalar resource base.  The resource covers only the
  // rows that exist, so the range check returns zeros past the end of A or W.
  constexpr int LPT = CA + CW;  // loads per thread per k-tile
  const int row_t = tid / 8, kc_t = tid % 8;
  const int slot_t = row_t * 8 + (kc_t ^ ((row_t >> 1) & 7));
  uint32_t a_off[CA], w_off[CW];
#pragma unroll
  for (int j = 0; j < CA; ++j) a_off[j] = uint32_t(((row_t + RS * j) * p.lda + kc_t * 8) * 2);
#pragma unroll
  for (int j = 0; j < CW; ++j) w_off[j] = uint32_t(((row_t + RS * j) * a.K + kc_t * 8) * 2);
  const char* a_base = reinterpret_cast<const char*>(A + m0 * p.lda);
  const char* w_base = reinterpret_cast<const char*>(W + n0 * a.K);
  const int64_t a_bytes = (p.M - m0) * p.lda * 2, w_bytes = (a.N - n0) * a.K * 2;
  struct Stage {
    u32x4 a[CA], w[CW];
  };
  auto load_tile = [&](Stage& st, int64_t kt) {
    const int64_t koff = kt * kBK * 2;
    const u32x4 ra = buffer_rsrc(a_base + koff, range32(a_bytes - koff));
    const u32x4 rw = buffer_rsrc(w_base + koff, range32(w_bytes - koff));
#pragma unroll
    for (int j = 0; j < CA; ++j) buffer_load16(st.a[j], ra, a_off[j]);
#pragma unroll
    for (int j = 0; j < CW; ++j) buffer_load16(st.w[j], rw, w_off[j]);
  };
  auto ready = [&](Stage& st) {
#pragma unroll
    for (int j = 0; j < CA; ++j) vm_ready(st.a[j]);
#pragma unroll
    for (int j = 0; j < CW; ++j) vm_ready(st.w[j]);
  };
  auto store_tile = [&](const Stage& st, int buf) {
#pragma unroll
    for (int j = 0; j < CA; ++j) lds[buf][slot_t + RS * 8 * j] = st.a[j];
#pragma unroll
    for (int j = 0; j < CW; ++j) lds[buf][kBM * 8 + slot_t + RS * 8 * j] = st.w[j];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Fragments are double-buffered across the 16-wide k steps: the LDS reads
  // of step kk + 1 are in flight while the MFMAs of step kk run, so a wave
  // rarely stalls on LDS latency.
  auto compute = [&](int buf) {
    const u32x4* L = lds[buf];
    bf16x8 af[2][TM], wf[2][TN];
    auto read = [&](int kk, int slot) {
      const int chunk = 2 * kk + hi;
#pragma unroll
      for (int i = 0; i < TM; ++i) af[slot][i] = as_bf16x8(L[swz(wm * WM + 32 * i + l32, chunk)]);
#pragma unroll
      for (int j = 0; j < TN; ++j) wf[slot][j] = as_bf16x8(L[kBM * 8 + swz(wn * WN + 32 * j + l32, chunk)]);
    };
    read(0, 0);
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      if (kk + 1 < kBK / 16) read(kk + 1, (kk + 1) & 1);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(wf[kk & 1][j], af[kk & 1][i], acc[i][j]);
    }
  };

  const int64_t n_t = kt1 - kt0;
  // Software pipeline, two register stages and two LDS buffers: while
  // k-tile t is multiplied from LDS, tile t + 1 (loaded one step earlier)
  // is stored to the other buffer and tile t + 2 is in flight.  Loads
  // complete in issue order, so "the older stage is ready" is
  // vmcnt <= LPT while the newer stage is in flight, else vmcnt == 0.
  Stage s0, s1;
  if (n_t > 0) {
    load_tile(s0, kt0);
    if (n_t > 1) {
      load_tile(s1, kt0 + 1);
      vm_wait<LPT>();
    } else {
      vm_wait<0>();
    }
    ready(s0);
    store_tile(s0, 0);
  }
  lds_barrier();
  for (int64_t t = 0; t < n_t; t += 2) {
    // even step: compute buffer 0; s1 holds tile t + 1.
    const bool next2 = t + 2 < n_t;
    if (next2) load_tile(s0, kt0 + t + 2);
    compute(0);
    if (t + 1 < n_t) {
      if (next2) vm_wait<LPT>(); else vm_wait<0>();
      ready(s1);
      store_tile(s1, 1);
    }
    lds_barrier();
    if (t + 1 >= n_t) break;
    // odd step: compute buffer 1; s0 holds tile t + 2.
    const bool next3 = t + 3 < n_t;
    if (next3) load_tile(s1, kt0 + t + 3);
    compute(1);
    if (next2) {
      if (next3) vm_wait<LPT>(); else vm_wait<0>();
      ready(s0);
      store_tile(s0, 0);
    }
    lds_barrier();
  }

  // The last barrier of the main loop has passed: LDS is free.
  const int64_t rows_all = a.p[0].M + (a.nprob > 1 ? a.p[1].M : 0);
  float* pbase = splits > 1 ? partial + (int64_t(ks) * rows_all + (prob ? a.p[0].M : 0) + m0) * a.N + n0 : nullptr;
  staged_epilogue<WM, WN, TM, TN>(a, p, m0, n0, splits > 1, pbase, a.N, acc,
                                  reinterpret_cast<float*>(&lds[0][0]), wave, wm, wn, lane);
}

// Epilogue of the ping-pong kernel: each wave turns its 128 x 64 block around
// in its own 16 KB of LDS, as bf16 results (bias, GELU and the gated residual
// are applied on the accumulators), so one 16-byte store instruction covers
// 8 rows of 128 bytes, or 4 columns of 256 bytes in a transposed region.  A
// wave's LDS operations complete in order: no barrier.  The caller passes the
// main loop's LDS once every wave is done with it.
//   acc[i][j][r] = C[row 16 i + l16][col 16 j + 4 g + r], l16 = lane % 16, g = lane / 16.
// Row-major image: 128-byte rows, 16-byte chunk c of row r at chunk
// c ^ ((r / 2) mod 8), which spreads the 8-byte accumulator writes (16 rows, two
// halves of a chunk) and the 16-byte row reads over all banks.  (Counted: none of
// the main loop's LDS instructions conflicts, the epilogue's 48 per wave lose 2.7
// cycles each.)
// Transposed image: 256-byte columns; lanes l, l ^ 1 first exchange half of
// their four columns, so each holds two rows of two columns and writes
// 4-byte row pairs; 16-byte chunk k of column c is at k ^ 2 ((c / 2) mod 8)
// (columns of 64 rows: mod 4).
// Split-K partials are stored as fp32 straight from the accumulators.
// Every global access is a buffer access whose range (or an offset past it)
// drops the rows >= M and the columns >= N: with plain accesses the bounds
// were a branch per 16 bytes, and the epilogue took 9 us of a 252-tile launch.
typedef const __attribute__((address_space(4))) GemmArgs* GemmArgsPtr;
typedef const __attribute__((address_space(4))) GemmProblem* GemmProblemPtr;
constexpr uint32_t kPast = 0x80000000u;  // a buffer offset past every range used below

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const void* base, int64_t bytes) {
  const uint32_t n = bytes <= 0 ? 0u : bytes >= int64_t(kPast) ? kPast : uint32_t(bytes);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(n), 0x00020000);
}

template <int TM, int TN>
__device__ __forceinline__ void pp_epilogue(GemmArgsPtr a, GemmProblemPtr p, int64_t m0, int64_t n0,
                                            float* __restrict__ pbase, int64_t pld, const f32x4 (&acc)[TM][TN],
                                            u32x4* sm, int wave, int wm, int wn, int lane) {
  constexpr int WM = 16 * TM, WN = 16 * TN;
  static_assert((WM == 128 || WM == 64) && WN == 64, "LDS image");
  const int l16 = lane % 16, g = lane / 16;
  const int64_t nb = n0 + wn * WN, mb = m0 + wm * WM, M = p->M, N = a->N;
  if (nb >= N || mb >= M) return;
  const int rows = int(std::min<int64_t>(WM, M - mb)), cols = int(std::min<int64_t>(WN, N - nb));
  if (pbase) {
    const __amdgpu_buffer_rsrc_t r = buf(pbase + wm * WM * pld + wn * WN, rows * pld * 4);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const uint32_t row = uint32_t(16 * i + l16) * uint32_t(pld * 4) + 16 * g;
#pragma unroll
      for (int j = 0; j < TN; ++j)  // cols is a multiple of 8 (split launches need N % 8 == 0)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), r,
                                               int(16 * j + 4 * g < cols ? row + 64 * j : kPast), 0, 0);
    }
    return;
  }
  const int64_t n_split = a->n_split, n_split2 = a->n_split2;
  const bool r0 = nb < n_split, r1 = nb < n_split2;
  const int mode = r0 ? a->mode0 : r1 ? a->mode1 : a->mode2;
  bf16_t* out = static_cast<bf16_t*>(r0 ? p->out0 : r1 ? p->out1 : p->out2);
  const int64_t ldo = r0 ? p->ld0 : r1 ? p->ld1 : p->ld2;
  const int64_t col0 = nb - (r0 ? 0 : r1 ? n_split : n_split2);
  // This lane's columns 16 j + 4 g .. + 3 of the strip (zeros past N).
  auto load4 = [&](const void* base, u32x2 (&dst)[TN]) {
    const __amdgpu_buffer_rsrc_t r = buf(static_cast<const bf16_t*>(base) + nb, base ? cols * 2 : 0);
#pragma unroll
    for (int j = 0; j < TN; ++j)
      dst[j] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, 2 * (16 * j + 4 * g), 0, 0));
  };
  auto f4 = [](const u32x2& w, int r) {
    return __uint_as_float(r & 1 ? w[r >> 1] & 0xffff0000u : w[r >> 1] << 16);
  };
  u32x2 bias[TN];
  load4(p->bias, bias);
  char* reg = reinterpret_cast<char*>(sm) + wave * (WM * WN * 2);
  if (mode == EPI_STORE_T) {
    const bool odd = lane & 1;
    auto swz_t = [](int cc) { return ((cc >> 1) & (WM / 16 - 1)) << 1; };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4& c = acc[i][j];
        const uint32_t p01 = pack_bf2(c[0] + f4(bias[j], 0), c[1] + f4(bias[j], 1));
        const uint32_t p23 = pack_bf2(c[2] + f4(bias[j], 2), c[3] + f4(bias[j], 3));
        const uint32_t got = uint32_t(
            __builtin_amdgcn_update_dpp(0, int(odd ? p01 : p23), kDppXor1, 0xf, 0xf, false));
        const uint32_t lo = odd ? got : p01, up = odd ? p23 : got;  // rows l & ~1 and l | 1
        const int cc = 16 * j + 4 * g + 2 * int(odd);               // columns cc, cc + 1
        const int chunk = (2 * i + (l16 >> 3)) ^ swz_t(cc);
        uint32_t* d = reinterpret_cast<uint32_t*>(reg + cc * (WM * 2) + chunk * 16) + ((l16 >> 1) & 3);
        d[0] = __builtin_amdgcn_perm(up, lo, 0x05040100u);
        d[WM * 2 / 4] = __builtin_amdgcn_perm(up, lo, 0x07060302u);
      }
    constexpr int kCh = WM / 8;                 // 16-byte chunks per column
    const int k = lane % kCh;
    auto column = [&](int cc) {
      return *reinterpret_cast<const u32x4*>(reg + cc * (WM * 2) + (k ^ swz_t(cc)) * 16);
    };
    // Plain stores: a transposed row may start at any element.
    bf16_t* dst = out + col0 * ldo + mb;
    const bool whole = 8 * k + 8 <= rows;
#pragma unroll
    for (int it = 0; it < WN * kCh / kWave; ++it) {
      const int cc = lane / kCh + kWave / kCh * it;
      const u32x4 w = column(cc);
      if (whole && cc < cols) *reinterpret_cast<u32x4*>(dst + cc * ldo + 8 * k) = w;
    }
    if (rows % 8 != 0 && k == rows / 8) {  // the last, partial group of eight rows
#pragma unroll 1
      for (int cc = lane / kCh; cc < cols; cc += kWave / kCh) {
        const u32x4 w = column(cc);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (8 * k + e < rows) dst[cc * ldo + 8 * k + e] = bf16_t(w[e / 2] >> (16 * (e % 2)));
      }
    }
    return;
  }
  // Row-major: lane's 16-byte role is chunk lane % 8 of rows lane / 8 + 8 it.
  const int ch = lane % 8;
  auto chunk_at = [&](int row) { return reg + row * (WN * 2) + ((ch ^ ((row >> 1) & 7)) * 16); };
  auto half_at = [&](int row, int j) {  // this lane's four columns of column tile j
    return reg + row * (WN * 2) + (((2 * j + (g >> 1)) ^ ((row >> 1) & 7)) * 16) + 8 * (g & 1);
  };
  const bool col_ok = 8 * ch < cols;
  u32x2 gate[TN] = {};
  const bool images = mode == EPI_RESID_GATE && a->mod.B > 0;
  const bf16_t* row_gate[TM];
  if (mode == EPI_RESID_GATE) {
    load4(p->gate, gate);
    if (images) {  // the segment of each of this lane's rows (see mod_offset), in a rolled loop: scalars are short
      const int B = a->mod.B;
      const int64_t row = p->row0 + mb, stride = a->mod.stride;
      int seg[TM] = {};
#pragma unroll 1
      for (int k = 0; k < 2 * B - 1; ++k) {
        const int64_t end = a->mod.end[k] - row;
#pragma unroll
        for (int i = 0; i < TM; ++i) seg[i] += std::min(16 * i + l16, rows - 1) >= end ? 1 : 0;
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
        row_gate[i] = static_cast<const bf16_t*>(p->gate) + nb + (seg[i] < B ? seg[i] : seg[i] - B) * stride;
    }
    // The residual goes through the same image, to meet the accumulators.
    const int64_t ldr = p->ldr;
    const __amdgpu_buffer_rsrc_t r = buf(static_cast<const bf16_t*>(p->resid) + mb * ldr + col0,
                                         ((rows - 1) * ldr + cols) * 2);
    const uint32_t off = uint32_t(lane / 8) * uint32_t(ldr * 2) + 16 * ch;
    u32x4 res[WM / 8];
#pragma unroll
    for (int it = 0; it < WM / 8; ++it)
      res[it] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, int(col_ok ? off + it * uint32_t(ldr * 16) : kPast), 0, 0));
#pragma unroll
    for (int it = 0; it < WM / 8; ++it) *reinterpret_cast<u32x4*>(chunk_at(lane / 8 + 8 * it)) = res[it];
  }
  auto convert = [&](auto mode_tag) {
    constexpr int kMode = decltype(mode_tag)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        u32x2* d = reinterpret_cast<u32x2*>(half_at(16 * i + l16, j));
        u32x2 rw;
        if constexpr (kMode == EPI_RESID_GATE) {
          rw = *d;
          // Per-image gates: this row's (columns past N read as another's, unused).
          if (images) gate[j] = *reinterpret_cast<const u32x2*>(row_gate[i] + std::min(16 * j + 4 * g, cols - 4));
        }
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = acc[i][j][r] + f4(bias[j], r);
          if constexpr (kMode == EPI_GELU) v[r] = gelu_fast(v[r]);
          if constexpr (kMode == EPI_RESID_GATE) v[r] = f4(rw, r) + f4(gate[j], r) * v[r];
        }
        *d = u32x2{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
      }
  };
  if (mode == EPI_GELU) convert(std::integral_constant<int, EPI_GELU>());
  else if (mode == EPI_RESID_GATE) convert(std::integral_constant<int, EPI_RESID_GATE>());
  else convert(std::integral_constant<int, EPI_STORE>());
  const __amdgpu_buffer_rsrc_t r = buf(out + mb * ldo + col0, ((rows - 1) * ldo + cols) * 2);
  const uint32_t off = uint32_t(lane / 8) * uint32_t(ldo * 2) + 16 * ch;
#pragma unroll
  for (int it = 0; it < WM / 8; ++it) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(chunk_at(lane / 8 + 8 * it));
    __builtin_amdgcn_raw_buffer_store_b128(w, r, int(col_ok ? off + it * uint32_t(ldo * 16) : kPast), 0, 0);
  }
  bf16_t* scat = static_cast<bf16_t*>(p->scat);
  if (r0 && scat) {  // the fused scatter: selected rows also go to their canvas rows
    const int64_t row0 = p->scat_row0, scat_n = p->scat_n, sld = p->scat_ld;
    const int32_t* sidx = p->scat_idx;
    int64_t at[WM / 8];
#pragma unroll
    for (int it = 0; it < WM / 8; ++it) {
      const int row = lane / 8 + 8 * it;
      const int64_t m = mb + row;
      at[it] = row < rows && m >= row0 && col_ok ? int64_t(sidx[m - row0]) : -1;
    }
#pragma unroll
    for (int it = 0; it < WM / 8; ++it) {
      const u32x4 w = *reinterpret_cast<const u32x4*>(chunk_at(lane / 8 + 8 * it));
      if (at[it] >= 0 && at[it] < scat_n) *reinterpret_cast<u32x4*>(scat + at[it] * sld + col0 + 8 * ch) = w;
    }
  }
}

// Tile order of the ping-pong kernel, in 32-bit arithmetic (the 64-bit
// divisions of the general mapping cost about 1 us at the head of every
// workgroup).  Tiles of problem 0 come first.  A problem's row tiles form
// near-equal bands of at most kBand; a band's tiles walk down its rows, then
// over the columns, so the 32 tiles that run on one XCD together share about
// kBand row tiles and 4 weight tiles in its L2 (walking down all the rows
// of a long problem re-read A once per column of tiles).
constexpr uint32_t kBand = 8;
__device__ __forceinline__ void pp_place(uint32_t id, uint32_t tn, uint32_t tm0, uint32_t tm1, int& prob, int& row,
                                         int& col) {
  prob = id >= tn * tm0;
  const uint32_t local = prob ? id - tn * tm0 : id, tm = prob ? tm1 : tm0;
  const uint32_t bands = (tm + kBand - 1) / kBand, small = tm / bands, big = tm % bands;  // `big` bands of small + 1
  const uint32_t in_big = big * (small + 1) * tn;
  const bool first = local < in_big;
  const uint32_t rows = first ? small + 1 : small, u = first ? local : local - in_big;
  const uint32_t band = u / (rows * tn), v = u % (rows * tn);
  row = int((first ? 0 : big * (small + 1)) + band * rows + v % rows);
  col = int(v / rows);
}
__device__ __forceinline__ uint32_t xcd_logical_id32(uint32_t bid, uint32_t grid) {
  const uint32_t per = grid / 8, rem = grid % 8, x = bid % 8, i = bid / 8;
  return x * per + std::min(x, rem) + i;
}
// Ping-pong form of the 256 x 256 x 64 kernel.  The 8 waves form two groups
// of four (one wave of each group per SIMD); group g owns output rows
// [128 g, 128 g + 128) and each of its waves a 128 x 64 block.  A group
// alternates a memory phase (read the fragments of a whole k-tile from LDS
// into registers, issue loads) with a compute phase (that k-tile's 64 MFMAs
// and nothing else), one workgroup barrier per phase, the groups one phase
// apart: each SIMD's matrix pipe is fed by one wave while the other does the
// memory work.
//   phase 2t:     group 0 reads k-tile t;      group 1 multiplies t - 1;
//   phase 2t + 1: group 0 multiplies k-tile t;  group 1 reads t.
// Tiles go from memory to LDS directly (buffer loads with the LDS flag), so
// no registers stage them and the fragments of a whole tile fit.  All 160 KB
// hold two A tiles and three W tiles.  Group 0 loads the second half of A
// (rows 128..255, which only group 1 reads) of tile t + 1 and the first half
// of W of tile t + 2 in phase 2t; group 1 the first half of A (read by group 0
// only, so free after phase 2t) and the second half of W of tile t + 2 in
// phase 2t + 1: every load is issued in a memory phase, each memory phase
// issues the same eight per wave, and each load has at least two phases
// (about 2000 cycles) before a barrier that waits for it.  (As built, the compiler
// also waits for the loads in flight halfway through a fragment read, because of
// registers that an epilogue path of the unit before loads; with that wait out of
// the way nothing was faster, 0.992 to 1.013 over fifteen cases.)
// Bound by: the clock under full matrix load (8192^3: 1.6-1.7 GHz from box to box,
// the matrix pipe 84 % busy; 16896 x 12288 x 3072: 1.5 GHz, 76 %; 1741 x 9216 x 3072,
// which is too short for that: 2.0 GHz, 61 %).  Hence the 16x16x32 products: alone, on all CUs, they sustain
// 2036 TFLOP/s where 32x32x16 sustain 1806 (a smaller accumulator is read and
// written per operation).  Measured (bias epilogue, TFLOP/s, before: tiles
// staged through registers, fragments read between the MFMAs; then on 32x32x16;
// now): 1741 x 9216 x 3072 1023 -> 1250 -> 1329, 16896 x 12288 x 3072 1020 ->
// 1350 -> 1446, 8192^3 1090 -> 1458 -> 1552 (the vendor library: 1150, 1352,
// 1409).  Two tiles of each operand with all loads in one phase ran 5 % slower
// at M = 1741 (the load unit needs 16 cycles per 1 KB load, a whole phase for
// a tile, and group 1's MFMAs queued behind its loads); half k-tiles per phase
// (twice the barriers) 8 % slower; without the raised priority in the compute
// phase 4-8 % slower.
template <int BN>
__global__ __launch_bounds__(512) void gemm_bf16_pp_kernel(const GemmArgs args, float* __restrict__ partial,
                                                          int units, int splits, int tail, int tsp) {
  constexpr int WM = BN / 2, WN = 64;        // a wave's block; a group's four waves cover 128 x BN
  constexpr int TM = WM / 16, TN = WN / 16, kWN = BN / WN;
  constexpr int RA = BN == 256 ? 2 : 3, RW = RA + 1;   // tiles of A and W in LDS
  constexpr int kA = kBM * 8, kW = BN * 8;   // 16-byte chunks of one operand's k-tile
  constexpr int LA = 4, LW = BN / 64;        // load instructions per wave for half an A and half a W tile
  __shared__ u32x4 lds[RA * kA + RW * kW];   // all 160 KB
  static_assert(sizeof(lds) == 160 * 1024, "LDS");

  // The arguments through the kernel-argument segment: a problem picked by a
  // uniform index stays scalar loads (a copy would live in private memory).
  const GemmArgsPtr a = (GemmArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(uint32_t(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) char*)(&lds[0]))));
  auto bar = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  // Work units in rounds of at most one per workgroup.  The units of a round
  // are renumbered so that each XCD takes a contiguous range of them; the k
  // splits of a tile are adjacent units.  Split tail: when the tiles overrun
  // the last full round by a few, the first tiles run whole and the last
  // `tail` ones in `tsp` k splits each, as units of their own in a round after
  // the whole tiles.
  const uint32_t tn_all = uint32_t((a->N + BN - 1) / BN), tm0 = uint32_t((a->p[0].M + kBM - 1) / kBM);
  const uint32_t tm1 = a->nprob > 1 ? uint32_t((a->p[1].M + kBM - 1) / kBM) : 0u;
  const uint32_t whole = tail ? tn_all * (tm0 + tm1) - uint32_t(tail) : uint32_t(units);
  for (uint32_t unit0 = 0; unit0 < uint32_t(units);) {
    const uint32_t end = std::min(unit0 < whole ? whole : uint32_t(units), unit0 + gridDim.x);
    const uint32_t here = unit0;
    unit0 = end;
    if (blockIdx.x >= end - here) continue;
    // Per-lane values are made anew for each unit (hoisted out of this loop,
    // they spilled).
    int lane = tid % kWave, wave_u = wave;
    asm volatile("" : "+v"(lane), "+s"(wave_u));
    const int l16 = lane % 16, g = lane / 16;
    const int grp = wave_u / 4, sub = wave_u % 4;
    const int wm = grp * (128 / WM) + sub / kWN, wn = sub % kWN;

    auto scalar = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const uint32_t u = here + xcd_logical_id32(blockIdx.x, end - here);
    const bool split_tail = u >= whole;
    const uint32_t nsp = split_tail ? tsp : splits, v = split_tail ? u - whole : u;
    const int ks = scalar(int(v % nsp)), tidx = split_tail ? scalar(int(v / nsp)) : -1;
    int prob, tm, tn;
    pp_place((split_tail ? whole : 0) + v / nsp, tn_all, tm0, tm1, prob, tm, tn);
    prob = scalar(prob);
    const GemmProblemPtr p = &a->p[prob];
    const int64_t m0 = int64_t(scalar(tm)) * kBM, n0 = int64_t(scalar(tn)) * BN;
    const int64_t M = p->M, N = a->N, K = a->K, lda = p->lda;
    const bf16_t* A = static_cast<const bf16_t*>(p->A);
    const bf16_t* W = static_cast<const bf16_t*>(p->W);
    const int nk = int(K / kBK);
    const int kt0 = scalar(nk * ks / int(nsp)), kt1 = scalar(nk * (ks + 1) / int(nsp));
    const int n_t = kt1 - kt0;

    // Staging: one load instruction moves 8 rows of 128 bytes; the LDS side is
    // lane-linear, so the swizzle is applied to the chunk each lane fetches.
    // Wave `sub` of a group moves rows 8 sub + 32 j of a half tile (one swizzle
    // for all j): group 0 the second half of A and the first half of W,
    // group 1 the first half of A and the second half of W.
    const int row_t = sub * 8 + lane / 8;
    const int kc_t = (lane % 8) ^ ((row_t >> 1) & 7);
    const int a_half = 128 * (1 - grp), w_half = BN / 2 * grp;
    uint32_t a_off[LA], w_off[LW];
#pragma unroll
    for (int j = 0; j < LA; ++j) a_off[j] = uint32_t(((a_half + row_t + 32 * j) * lda + kc_t * 8) * 2);
#pragma unroll
    for (int j = 0; j < LW; ++j) w_off[j] = uint32_t(((w_half + row_t + 32 * j) * K + kc_t * 8) * 2);
    auto uniform = [](u32x4 r) {
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = __builtin_amdgcn_readfirstlane(r[e]);
      return r;
    };
    const u32x4 ra = uniform(buffer_rsrc(A + m0 * lda, range32((M - m0) * lda * 2)));
    const u32x4 rw = uniform(buffer_rsrc(W + n0 * K, range32((N - n0) * K * 2)));
    const uint32_t a_dst = lds0 + a_half * 128 + sub * 1024;
    const uint32_t w_dst = lds0 + RA * kA * 16 + w_half * 128 + sub * 1024;
    // This wave's share of k-tile t of A or W, into a slot of its ring (in: t < n_t
    // for sure).  Past the last k-tile the resource's range and the scalar offset are 0: every
    // offset is out of range (also where the range is taken less the scalar
    // offset, which then may not exceed it), no memory is read, and the loads
    // still count, so every wait below is the same constant.
    using Sure = std::integral_constant<bool, true>;
    using Maybe = std::integral_constant<bool, false>;
    auto load_a = [&](int t, int slot, auto in) {
      const bool live = decltype(in)::value || t < n_t;
      const uint32_t koff = live ? uint32_t(kt0 + t) * (kBK * 2) : 0u;
      const u32x4 r = {ra[0], ra[1], live ? ra[2] : 0u, ra[3]};
#pragma unroll
      for (int j = 0; j < LA; ++j) lds_load16(a_dst + slot * (kA * 16), a_off[j], r, koff, 4096 * j);
    };
    auto load_w = [&](int t, int slot, auto in) {
      const bool live = decltype(in)::value || t < n_t;
      const uint32_t koff = live ? uint32_t(kt0 + t) * (kBK * 2) : 0u;
      const u32x4 r = {rw[0], rw[1], live ? rw[2] : 0u, rw[3]};
#pragma unroll
      for (int j = 0; j < LW; ++j) lds_load16(w_dst + slot * (kW * 16), w_off[j], r, koff, 4096 * j);
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The fragments of a whole k-tile: read in one phase, multiplied in the next.
    constexpr int KS = kBK / 32;
    bf16x8 af[KS][TM], wf[KS][TN];
    const int sw = (l16 >> 1) & 7;
    const u32x4* La = lds + (wm * WM + l16) * 8;
    const u32x4* Lw = lds + RA * kA + (wn * WN + l16) * 8;
    auto read = [&](int as, int ws) {
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const int c = (4 * k + g) ^ sw;
#pragma unroll
        for (int j = 0; j < TN; ++j) wf[k][j] = as_bf16x8(Lw[ws * kW + 128 * j + c]);
#pragma unroll
        for (int i = 0; i < TM; ++i) af[k][i] = as_bf16x8(La[as * kA + 128 * i + c]);
      }
    };
    auto mul = [&]() {
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma16x16x32(wf[k][j], af[k][i], acc[i][j]);
      __builtin_amdgcn_s_setprio(0);
    };

    // Each group runs its own straight loop; both pass the same barriers.
    // The slots of tiles t, t - 1 (= that of t + RA - 1, t + RW - 1) rotate.
    constexpr int kStep = LA + LW;
    int as = 0, ap = RA - 1, ws = 0, wp = RW - 1;
    auto next = [&]() {
      ap = as;
      wp = ws;
      as = as == RA - 1 ? 0 : as + 1;
      ws = ws == RW - 1 ? 0 : ws + 1;
    };
    if (here > 0) bar();   // every wave is done with the last unit's epilogue
    if (grp == 0) {
      load_w(0, 0, Maybe());
#pragma unroll
      for (int t = 0; t < RA - 1; ++t) {
        load_a(t, t, Maybe());
        load_w(t + 1, t + 1, Maybe());
      }
      vm_wait<(RA - 1) * kStep>();
      bar();
      auto step = [&](int t, auto in) {
        read(as, ws);
        load_a(t + RA - 1, ap, in);
        load_w(t + RW - 1, wp, in);
        vm_wait<LW + (RA - 1) * kStep>();   // the second half of A(t), which phase 2t + 1 reads
        bar();
        mul();
        vm_wait<(RA - 1) * kStep>();        // the first half of W(t + 1), which phase 2t + 2 reads
        bar();
        next();
      };
      int t = 0;
      for (; t + RW - 1 < n_t; ++t) step(t, Sure());
      for (; t < n_t; ++t) step(t, Maybe());
      vm_wait<0>();
      bar();
    } else {
#pragma unroll
      for (int t = 0; t < RA; ++t) {
        load_a(t, t, Maybe());
        load_w(t, t, Maybe());
      }
      vm_wait<(RA - 1) * kStep>();
      bar();
      if (n_t == 0) vm_wait<0>();
      bar();
      auto step = [&](int t, auto in) {
        read(as, ws);
        load_a(t + RA, as, in);
        load_w(t + RW - 1, wp, in);
        vm_wait<(RA - 1) * kStep>();        // both halves of tile t + 1, which phase 2t + 2 reads
        bar();
        mul();
        if (!decltype(in)::value && t == n_t - 1) vm_wait<0>();
        bar();
        next();
      };
      int t = 0;
      for (; t + RW - 1 < n_t; ++t) step(t, Sure());
      for (; t < n_t; ++t) step(t, Maybe());
    }

    // Split partials: a tail tile's go to its own 256 x 256 block (split-major),
    // a fully split launch's to rows of the [split][row][N] array.
    float* pbase = nullptr;
    int64_t pld = N;
    if (tidx >= 0) {
      pbase = partial + (int64_t(tidx) * tsp + ks) * (kBM * BN);
      pld = BN;
    } else if (splits > 1) {
      const int64_t M0 = a->p[0].M, rows_all = M0 + (a->nprob > 1 ? a->p[1].M : 0);
      pbase = partial + (ks * rows_all + (prob ? M0 : 0) + m0) * N + n0;
    }
    pp_epilogue<TM, TN>(a, p, m0, n0, pbase, pld, acc, lds, wave_u, wm, wn, lane);
  }
}

// Register-staged ping-pong form, 256 x 256 x 64 on 32x32x16 products, for
// operands off the 16-byte grid: loads that go to LDS directly want 16-byte
// boundaries, loads to registers and the epilogue through LDS in fp32 do not.
// The two groups of four waves (rows 0 .. 127 and 128 .. 255) alternate between
// a compute phase (the 32 MFMAs of one k-tile, fragments read from LDS) and a
// memory phase (stage half of a later k-tile into LDS and issue the loads of the
// half after it), one workgroup barrier per phase, offset by one phase:
//   phase 2t:     group 0 computes k-tile t;  group 1 stages its half of
//                 tile t + 1 and loads its half of tile t + 2;
//   phase 2t + 1: group 1 computes k-tile t;  group 0 stages / loads the same.
// Tile t lives in LDS buffer t mod 2: it is read in phases 2t and 2t + 1 and
// written in phases 2t - 2 and 2t - 1, after tile t - 2 left that buffer.
// Bound by LDS: fragment reads between the MFMAs and the staging writes.  With every
// bias one element off, against the 128-wide kernel, unsplit: 1741 x 9216 x
// 3072 127 -> 97 us, 4096 x 3072 x 12288 423 -> 287, a double block of 845 rows 568 ->
// 388, of 1741 667 -> 545, of 4608 1682 -> 1377.
__global__ __launch_bounds__(512) void gemm_bf16_staged_kernel(const GemmArgs a, float* __restrict__ partial,
                                                              int splits, int tail, int tsp) {
  constexpr int BN = 256, WM = 128, WN = 64;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int HALF = 4;                    // 16-byte chunks per thread per half-tile operand
  __shared__ u32x4 lds[2][(kBM + BN) * 8];

  // Whole tiles (or every tile's k splits) first, then the split tail's units,
  // each class renumbered for the XCDs; tiles placed as in the kernel above, which
  // the tail's reduce relies on.
  const uint32_t tn_all = uint32_t((a.N + BN - 1) / BN), tm0 = uint32_t((a.p[0].M + kBM - 1) / kBM);
  const uint32_t tm1 = a.nprob > 1 ? uint32_t((a.p[1].M + kBM - 1) / kBM) : 0u;
  const uint32_t whole = tail ? tn_all * (tm0 + tm1) - uint32_t(tail) : gridDim.x;
  const bool split_tail = blockIdx.x >= whole;
  const uint32_t v = split_tail ? xcd_logical_id32(blockIdx.x - whole, gridDim.x - whole)
                                : xcd_logical_id32(blockIdx.x, whole);
  const int nsp = split_tail ? tsp : splits, ks = int(v % uint32_t(nsp));
  const int tidx = split_tail ? int(v / uint32_t(nsp)) : -1;
  int prob, tm, tn;
  pp_place((split_tail ? whole : 0) + v / uint32_t(nsp), tn_all, tm0, tm1, prob, tm, tn);
  const int64_t m0 = int64_t(tm) * kBM, n0 = int64_t(tn) * BN;
  const GemmProblem p = prob ? a.p[1] : a.p[0];  // by value: a select, no indexed copy of the arguments
  const bf16_t* A = static_cast<const bf16_t*>(p.A);
  const bf16_t* W = static_cast<const bf16_t*>(p.W);
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int l32 = lane % 32, hi = lane / 32;
  const int grp = __builtin_amdgcn_readfirstlane(wave / 4);
  const int wm = grp, wn = wave % 4;

  const int64_t nk = a.K / kBK;
  const int64_t kt0 = nk * ks / nsp, kt1 = nk * (ks + 1) / nsp;
  const int64_t n_t = kt1 - kt0;

  // Staging of this group's half: A rows and W rows [128 grp, 128 grp + 128),
  // thread tg moves chunk tg % 8 of rows tg / 8 + 32 j (one swizzle for all j).
  const int tg = tid % 256;
  const int row_t = tg / 8, kc_t = tg % 8;
  const int slot_t = (128 * grp + row_t) * 8 + (kc_t ^ ((row_t >> 1) & 7));
  uint32_t a_off[HALF], w_off[HALF];
#pragma unroll
  for (int j = 0; j < HALF; ++j) {
    a_off[j] = uint32_t(((128 * grp + row_t + 32 * j) * p.lda + kc_t * 8) * 2);
    w_off[j] = uint32_t(((128 * grp + row_t + 32 * j) * a.K + kc_t * 8) * 2);
  }
  const char* a_base = reinterpret_cast<const char*>(A + m0 * p.lda);
  const char* w_base = reinterpret_cast<const char*>(W + n0 * a.K);
  const int64_t a_bytes = (p.M - m0) * p.lda * 2, w_bytes = (a.N - n0) * a.K * 2;
  // The staged loads stay in flight across the group's next compute phase
  // (a loop-carried value), so they are compiler-visible buffer loads: the
  // compiler places the vmcnt wait before the LDS store that consumes them.
  u32x4 sa[HALF], sw[HALF];
  auto load_half = [&](int64_t kt) {
    const int64_t koff = kt * kBK * 2;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(a_base + koff), 0, int(range32(a_bytes - koff)), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(w_base + koff), 0, int(range32(w_bytes - koff)), 0x00020000);
#pragma unroll
    for (int j = 0; j < HALF; ++j) sa[j] = __builtin_amdgcn_raw_buffer_load_b128(ra, int(a_off[j]), 0, 0);
#pragma unroll
    for (int j = 0; j < HALF; ++j) sw[j] = __builtin_amdgcn_raw_buffer_load_b128(rw, int(w_off[j]), 0, 0);
  };
  auto store_half = [&](int buf) {
#pragma unroll
    for (int j = 0; j < HALF; ++j) lds[buf][slot_t + 256 * j] = sa[j];
#pragma unroll
    for (int j = 0; j < HALF; ++j) lds[buf][kBM * 8 + slot_t + 256 * j] = sw[j];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto compute = [&](int buf) {
    const u32x4* L = lds[buf];
    bf16x8 af[2][TM], wf[2][TN];
    // Fragments are read in the order the next k step's MFMAs (i-major)
    // consume them, so the first MFMAs wait on the oldest reads.
    auto read = [&](int kk, int slot) {
      const int chunk = 2 * kk + hi;
      wf[slot][0] = as_bf16x8(L[kBM * 8 + swz(wn * WN + l32, chunk)]);
      af[slot][0] = as_bf16x8(L[swz(wm * WM + l32, chunk)]);
#pragma unroll
      for (int j = 1; j < TN; ++j) wf[slot][j] = as_bf16x8(L[kBM * 8 + swz(wn * WN + 32 * j + l32, chunk)]);
#pragma unroll
      for (int i = 1; i < TM; ++i) af[slot][i] = as_bf16x8(L[swz(wm * WM + 32 * i + l32, chunk)]);
    };
    read(0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      if (kk + 1 < kBK / 16) read(kk + 1, (kk + 1) & 1);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(wf[kk & 1][j], af[kk & 1][i], acc[i][j]);
      if (kk + 1 < kBK / 16) {
#pragma unroll
        for (int r = 0; r < TM + TN; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - (TM + TN), 0);
      } else {
        __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
      }
    }
  };

  if (n_t > 0) {
    load_half(kt0);
    store_half(0);
    if (n_t > 1) load_half(kt0 + 1);
  }
  lds_barrier();
  // Memory phase of k-tile t: stage this group's half of tile t + 1, then
  // issue its loads of tile t + 2.
  auto memory = [&](int64_t t) {
    if (t + 1 < n_t) {
      store_half(int((t + 1) & 1));
      if (t + 2 < n_t) load_half(kt0 + t + 2);
    }
  };
  // Each group runs its own straight loop; both pass the same barriers.
  if (grp == 0) {
    for (int64_t t = 0; t < n_t; ++t) {
      compute(int(t & 1));
      lds_barrier();
      memory(t);
      lds_barrier();
    }
  } else {
    for (int64_t t = 0; t < n_t; ++t) {
      memory(t);
      lds_barrier();
      compute(int(t & 1));
      lds_barrier();
    }
  }

  // Split partials, as in the kernel above.
  float* pbase = nullptr;
  int64_t pld = a.N;
  if (tidx >= 0) {
    pbase = partial + (int64_t(tidx) * tsp + ks) * (kBM * BN);
    pld = BN;
  } else if (splits > 1) {
    const int64_t rows_all = a.p[0].M + (a.nprob > 1 ? a.p[1].M : 0);
    pbase = partial + (int64_t(ks) * rows_all + (prob ? a.p[0].M : 0) + m0) * a.N + n0;
  }
  staged_epilogue<WM, WN, TM, TN>(a, p, m0, n0, pbase != nullptr, pbase, pld, acc,
                                  reinterpret_cast<float*>(&lds[0][0]), wave, wm, wn, lane);
}

// Sum the k splits of each tail tile in split order and apply the epilogue.
// Block b covers rows 8 (b mod 32) .. + 7 of tail tile b / 32, one thread per
// eight columns; in a transposed region (the last columns of the QKV
// projection, so usually all of its tail) one thread per column, whose eight
// rows are one store: as eight columns of a row they were eight 2-byte stores
// to as many lines (104 tail tiles of the QKV projection of 2457 rows: 7 us
// less).
__global__ __launch_bounds__(256) void tail_reduce_kernel(const GemmArgs a, const float* __restrict__ partial,
                                                          int64_t tail, int tsp) {
  constexpr int BN = 256;
  const int64_t t = blockIdx.x / (kBM / 8);
  const int r = int(blockIdx.x % (kBM / 8)) * 8 + int(threadIdx.x) / 32;
  const int c = (int(threadIdx.x) % 32) * 8;
  const uint32_t tn = uint32_t((a.N + BN - 1) / BN), tm0 = uint32_t((a.p[0].M + kBM - 1) / kBM);
  const uint32_t tm1 = a.nprob > 1 ? uint32_t((a.p[1].M + kBM - 1) / kBM) : 0u;
  int prob, row, col;
  pp_place(uint32_t(tn * (tm0 + tm1) - tail + t), tn, tm0, tm1, prob, row, col);
  const GemmProblem p = prob ? a.p[1] : a.p[0];
  const int64_t m = int64_t(row) * kBM + r, n = int64_t(col) * BN + c;
  const float* tile = partial + t * tsp * int64_t(kBM * BN);
  auto mode_of = [&](int64_t x) { return x < a.n_split ? a.mode0 : x < a.n_split2 ? a.mode1 : a.mode2; };
  if (m < p.M && n < a.N && mode_of(n) != EPI_STORE_T) {
    float v[8];
    for (int k = 0; k < tsp; ++k) {
      const float* q = tile + int64_t(k) * kBM * BN + r * BN + c;
      const float4 x0 = *reinterpret_cast<const float4*>(q), x1 = *reinterpret_cast<const float4*>(q + 4);
      const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = k == 0 ? x[e] : v[e] + x[e];
    }
    GemmProblem pg = p;
    if (a.mod.B) pg.gate = static_cast<const bf16_t*>(p.gate) + mod_offset(a.mod, p.row0 + m);  // this row's image
    epilogue8(a, pg, m, n, v);
  }
  const int r8 = r & ~7, tc = int(threadIdx.x);
  const int64_t mt = int64_t(row) * kBM + r8, nt = int64_t(col) * BN + tc;
  if (mt >= p.M || nt >= a.N || mode_of(nt) != EPI_STORE_T) return;
  float v[8];
  for (int k = 0; k < tsp; ++k) {
    const float* q = tile + int64_t(k) * kBM * BN + r8 * BN + tc;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = k == 0 ? q[e * BN] : v[e] + q[e * BN];
  }
  const float bias = p.bias ? ld(static_cast<const bf16_t*>(p.bias), nt) : 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] += bias;
  const bool r0 = nt < a.n_split, r1 = nt < a.n_split2;
  bf16_t* dst = static_cast<bf16_t*>(r0 ? p.out0 : r1 ? p.out1 : p.out2) +
                (nt - (r0 ? 0 : r1 ? a.n_split : a.n_split2)) * (r0 ? p.ld0 : r1 ? p.ld1 : p.ld2) + mt;
  if (mt + 8 <= p.M) {
    *reinterpret_cast<u32x4*>(dst) =
        u32x4{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (mt + e < p.M) st(dst, e, v[e]);
  }
}

// Sum the split-K partials in split order and apply the epilogue: one thread
// per eight columns of a row.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const GemmArgs a, const float* __restrict__ partial,
                                                            int splits) {
  const int64_t rows = a.p[0].M + (a.nprob > 1 ? a.p[1].M : 0);
  const int64_t groups = a.N / 8;
  const int64_t g = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (g >= rows * groups) return;
  const int64_t grow = g / groups, n = (g % groups) * 8;
  const float* src = partial + grow * a.N + n;
  float v[8];
  {
    const float4 x0 = *reinterpret_cast<const float4*>(src), x1 = *reinterpret_cast<const float4*>(src + 4);
    v[0] = x0.x; v[1] = x0.y; v[2] = x0.z; v[3] = x0.w; v[4] = x1.x; v[5] = x1.y; v[6] = x1.z; v[7] = x1.w;
  }
  for (int k = 1; k < splits; ++k) {
    const float* q = src + int64_t(k) * rows * a.N;
    const float4 x0 = *reinterpret_cast<const float4*>(q), x1 = *reinterpret_cast<const float4*>(q + 4);
    v[0] += x0.x; v[1] += x0.y; v[2] += x0.z; v[3] += x0.w; v[4] += x1.x; v[5] += x1.y; v[6] += x1.z; v[7] += x1.w;
  }
  const bool second = grow >= a.p[0].M;
  GemmProblem p = second ? a.p[1] : a.p[0];
  const int64_t m = second ? grow - a.p[0].M : grow;
  if (a.mod.B) p.gate = static_cast<const bf16_t*>(p.gate) + mod_offset(a.mod, p.row0 + m);  // this row's image
  epilogue8(a, p, m, n, v);
}

// fp32 GEMM of few tiles, on v_mfma_f32_32x32x2_f32: the eight waves of a
// workgroup share the contraction of one 32 x 32 tile, in steps of 16 (wave w
// takes steps w, w + 8, ...); their sums meet in LDS in wave order.  Operands
// go from the caches to registers: a lane holds eight consecutive k of one row
// of each, and the same k of both halves of the wave feed one product (any
// order of the contraction is as good).
// Bound by: latency.  The fp32 block of 288 rows and width 256 has 20 to 80
// tiles of 64 x 64, each a serial loop over K on one CU of 256; tiles of 32 x 32
// with K over eight waves take four times the CUs and an eighth of the chain.
// Measured against the 64 x 64 kernel: 288 x 768 x 256 18.9 -> 9.2 us, 288 x 256 x
// 1024 58.7 -> 11.9, 1024 x 384 x 1536 98 -> 30; error against 64 bits (relative,
// 2-norm) 2.9e-7 -> 1.2e-7 at K = 256, 5.7e-7 -> 2.1e-7 at 1024.
constexpr int kFT = 32, kFK = 16, kFWaves = 8;
__global__ __launch_bounds__(64 * kFWaves) void gemm_f32_kernel(const GemmArgs a) {
  constexpr int kP = kFT + 4, U = 2;
  __shared__ __attribute__((aligned(16))) float red[kFWaves][kFT * kP];
  int prob, tm, tn;  // 32-bit arithmetic: 64-bit divisions took about 1 us of the launch
  pp_place(xcd_logical_id32(blockIdx.x, gridDim.x), uint32_t((a.N + kFT - 1) / kFT),
           uint32_t((a.p[0].M + kFT - 1) / kFT), a.nprob > 1 ? uint32_t((a.p[1].M + kFT - 1) / kFT) : 0u, prob, tm, tn);
  const int64_t m0 = int64_t(tm) * kFT, n0 = int64_t(tn) * kFT;
  const GemmProblem p = prob ? a.p[1] : a.p[0];  // by value: a select, no indexed copy of the arguments
  const int tid = threadIdx.x, lane = tid % kWave, l32 = lane % 32, hi = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // Rows past the end repeat the last one; their results are not stored.
  const float* A = static_cast<const float*>(p.A) + std::min<int64_t>(m0 + l32, p.M - 1) * p.lda + 8 * hi;
  const float* W = static_cast<const float*>(p.W) + std::min<int64_t>(n0 + l32, a.N - 1) * a.K + 8 * hi;
  struct Step {
    f32x4 a[2], w[2];
  };
  const int nk = int(a.K / kFK);
  auto load = [&](Step (&st)[U], int s) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = int64_t(std::min(s + kFWaves * u, nk - 1)) * kFK;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        st[u].a[e] = load4u(A + k + 4 * e);
        st[u].w[e] = load4u(W + k + 4 * e);
      }
    }
  };
  f32x16 acc = {};
  Step cur[U], nxt[U];
  load(cur, wave);
  for (int s = wave; s < nk; s += kFWaves * U) {
    load(nxt, s + kFWaves * U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + kFWaves * u < nk) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(cur[u].w[e / 4][e % 4], cur[u].a[e / 4][e % 4], acc, 0, 0, 0);
      }
      cur[u] = nxt[u];
    }
  }
  // acc[4 q + r] = C[row l32][column 8 q + 4 hi + r] of the tile.
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<f32x4*>(&red[wave][l32 * kP + 8 * q + 4 * hi]) =
        f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
  __syncthreads();
  if (tid >= kFT * kFT / 4) return;
  const int r = tid / 8, c = tid % 8 * 4;
  f32x4 v = *reinterpret_cast<const f32x4*>(&red[0][r * kP + c]);
#pragma unroll
  for (int w = 1; w < kFWaves; ++w) v += *reinterpret_cast<const f32x4*>(&red[w][r * kP + c]);
  const int64_t m = m0 + r, n = n0 + c;
  if (m < p.M && n < a.N) epilogue4<float>(a, p, m, n, v[0], v[1], v[2], v[3]);
}


// fp32 GEMM of at least one 64 x 64 tile per CU, on the VALU: 64x64 tile, 16x16 threads, 4x4 outputs per thread.
constexpr int kFB = 64;
__global__ __launch_bounds__(256) void gemm_f32_valu_kernel(const GemmArgs a) {
  __shared__ float As[kFK][kFB + 4];
  __shared__ float Ws[kFK][kFB + 4];
  int prob, ks;
  int64_t m0, n0;
  if (!map_tile(a, kFB, kFB, 1, prob, m0, n0, ks)) return;
  const GemmProblem p = prob ? a.p[1] : a.p[0];  // by value: a select, no indexed copy of the arguments
  const float* A = static_cast<const float*>(p.A);
  const float* W = static_cast<const float*>(p.W);
  const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
  const int lrow = tid / 4, lk = (tid % 4) * 4;
  float acc[4][4] = {};
  for (int64_t k0 = 0; k0 < a.K; k0 += kFK) {
    const int64_t m = m0 + lrow, n = n0 + lrow;
    float4 va = make_float4(0.f, 0.f, 0.f, 0.f), vw = va;
    if (m < p.M) va = *reinterpret_cast<const float4*>(A + m * p.lda + k0 + lk);
    if (n < a.N) vw = *reinterpret_cast<const float4*>(W + n * a.K + k0 + lk);
    __syncthreads();
    As[lk + 0][lrow] = va.x; As[lk + 1][lrow] = va.y; As[lk + 2][lrow] = va.z; As[lk + 3][lrow] = va.w;
    Ws[lk + 0][lrow] = vw.x; Ws[lk + 1][lrow] = vw.y; Ws[lk + 2][lrow] = vw.z; Ws[lk + 3][lrow] = vw.w;
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kFK; ++kk) {
      float av[4], wv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) wv[j] = Ws[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], wv[j], acc[i][j]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t m = m0 + ty * 4 + i, n = n0 + tx * 4;
    if (m < p.M && n < a.N) epilogue4<float>(a, p, m, n, acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
  }
}

int64_t tiles_of(const GemmArgs& a, int bm, int bn) {
  int64_t t = 0;
  for (int i = 0; i < a.nprob; ++i) t += ceil_div64(a.p[i].M, bm) * ceil_div64(a.N, bn);
  return t;
}

// What the ping-pong kernel's 16-byte accesses and 64-column strips assume:
// the library's own buffers and 16-byte aligned tensors always meet it;
// anything else (a bias that is a slice at an odd element, say) takes the
// register-staged kernels.  A transposed output may start anywhere.
bool pp_layout_ok(const GemmArgs& a) {
  auto off = [](const void* ptr) { return reinterpret_cast<uintptr_t>(ptr) % 16; };
  if (a.N % 8 != 0 || (a.mod.B > 0 && a.mod.stride % 8 != 0) || (a.n_split < a.N && a.n_split % 64 != 0) || (a.n_split2 < a.N && a.n_split2 % 64 != 0))
    return false;
  for (int i = 0; i < a.nprob; ++i) {
    const GemmProblem& p = a.p[i];
    if (off(p.A) || off(p.W) || off(p.bias) || off(p.gate) || off(p.resid) || off(p.scat)) return false;
    if (p.lda % 8 || p.ldr % 8 || p.scat_ld % 8) return false;
    if (a.mode0 != EPI_STORE_T && (off(p.out0) || p.ld0 % 8)) return false;
    if (a.n_split < a.N && a.mode1 != EPI_STORE_T && (off(p.out1) || p.ld1 % 8)) return false;
    if (a.n_split2 < a.N && a.mode2 != EPI_STORE_T && (off(p.out2) || p.ld2 % 8)) return false;
  }
  return true;
}

}  // namespace

// Predicted time (us) of `units` ping-pong work units of nk k-tiles each, in
// equal rounds of at most one unit per CU.  Measured per k-tile:
//  - weights at hand (in a cache): the more CUs work the longer (the clock
//    falls with the matrix load, so 168 + 168 tiles are faster than 256 + 80):
//    256-wide 0.90 us on 84 and 120 CUs, 1.03 on 168, 1.13 on 198, 1.25 on 252;
//    128-wide 0.58 on 96, 0.67 on 168, 0.75 on 240;
//  - weights from HBM, where the loads in flight set the pace: 256-wide 1.28 on
//    168 CUs, 1.40 on 252; 128-wide 0.90.
// `cold` is the share of the tiles whose weights come from HBM: the first band
// of rows of each problem (a model's weights exceed the caches; the later
// bands find them).  4 us of prologue and epilogue per round, 7 per launch.
double pp_time(int bn, int64_t units, double nk, double cold) {
  const int64_t rounds = ceil_div64(units, kCUs);
  const double per = double(ceil_div64(units, rounds));
  const double warm = bn == 256 ? 0.90 + 0.35 * std::max(0.0, per - 130.0) / 122.0
                                : 0.58 + 0.20 * std::max(0.0, per - 96.0) / 156.0;
  const double hbm = bn == 256 ? 1.28 + 0.12 * std::max(0.0, per - 168.0) / 84.0 : 0.90;
  return double(rounds) * (nk * (cold * hbm + (1.0 - cold) * warm) + 4.0) + 7.0;
}

// Share of the row tiles that lie in the first band of their problem.
double first_band_share(const GemmArgs& a) {
  int64_t first = 0, all = 0;
  for (int i = 0; i < a.nprob; ++i) {
    const int64_t tm = ceil_div64(a.p[i].M, kBM);
    if (tm == 0) continue;
    first += ceil_div64(tm, ceil_div64(tm, kBand));
    all += tm;
  }
  return all > 0 ? double(first) / double(all) : 1.0;
}

GemmPlan plan_gemm(const GemmArgs& a, int dtype, size_t partial_bytes, const char* family, bool ln) {
  GemmPlan pl;
  if (dtype != AVITS_BF16) {
    // fp32: 64 x 64 tiles on the VALU where every CU gets one, else 32 x 32 with
    // the contraction over eight waves.  Measured, 64 against 32: 384 tiles of
    // 64 x 64 with K = 384 32.5 against 37.9 us, 96 tiles with K = 1536 98 against 30.
    pl.bn = tiles_of(a, kFB, kFB) >= kCUs ? kFB : kFT;
    pl.tiles = tiles_of(a, pl.bn, pl.bn);
    return pl;
  }
  const bool wide = pp_layout_ok(a);
  const int64_t nk = a.K / kBK;
  const int64_t rows = a.p[0].M + (a.nprob > 1 ? a.p[1].M : 0);
  pl.stages = wide ? 1 : 2;
  if (tiles_of(a, kBM, 128) == 0) return pl;
  if (!wide) {
    // Where that layout does not hold, the register-staged kernels: the largest
    // busy fraction of the last round of units on the CUs, times a factor per tile
    // (the 256-wide kernel moves less L2 data per FLOP; measured at the FLUX block
    // shapes) and one for the partials' traffic of a split.
    double best = -1.0;
    auto consider = [&](int bn, double eff, int64_t tiles, double rounds, int splits, int64_t tail, int tsp) {
      const double score = double(tiles * splits) / kCUs / rounds * eff * (splits > 1 || tail > 0 ? 0.95 : 1.0);
      if (score <= best + 1e-9) return;
      best = score;
      pl.bn = bn;
      pl.tiles = tiles;
      pl.splits = splits;
      pl.tail = tail;
      pl.tail_splits = tsp;
    };
    for (int bn : {256, 128}) {
      const double eff = bn == 256 ? 1.0 : 0.65;
      const int64_t t = tiles_of(a, kBM, bn), full = t / kCUs, rem = t % kCUs;
      for (int sp = 1; sp <= 4; ++sp) {
        if (sp > 1 && (a.N % 8 != 0 || nk / sp < 4 ||
                       size_t(sp) * size_t(rows) * size_t(a.N) * sizeof(float) > partial_bytes))
          break;
        consider(bn, eff, t, double(ceil_div64(t * sp, kCUs)), sp, 0, 1);
      }
      if (bn != 256 || full == 0 || rem == 0 || a.N % 8 != 0) continue;
      for (int tsp = 2; tsp <= 4; ++tsp) {
        if (rem * tsp > kCUs || nk / tsp < 4 || size_t(rem * tsp) * kBM * 256 * sizeof(float) > partial_bytes) break;
        consider(bn, eff, t, double(full) + 1.0 / tsp, 1, rem, tsp);
      }
    }
  } else {
    // The least predicted time over the column tile, the k splits of every
    // tile and the split tail.  A split writes fp32 partials at 4.5 TB/s beside
    // its epilogue and adds a reduce (2 us and its bytes at 4.4 TB/s); where a
    // layer norm follows, it rides on the reduce of a fully split launch and
    // is a launch of its own (3 us and its bytes) otherwise.
    const double mn = double(rows) * double(a.N) * 1e-6;  // MB per byte of an output element
    const double norm = ln ? 3.0 + 4.0 * mn / 3.5 : 0.0;
    const double cold = first_band_share(a);
    double best = 1e30;
    auto consider = [&](int bn, int64_t tiles, int splits, int64_t tail, int tsp, double us) {
      if (us >= best) return;
      best = us;
      pl.bn = bn;
      pl.stages = 1;
      pl.tiles = tiles;
      pl.splits = splits;
      pl.tail = tail;
      pl.tail_splits = tsp;
    };
    for (int bn : {256, 128}) {
      const int64_t t = tiles_of(a, kBM, bn);
      consider(bn, t, 1, 0, 1, pp_time(bn, t, double(nk), cold) + norm);
      for (int sp = 2; sp <= 4 && a.N % 8 == 0; ++sp) {
        if (nk / sp < 4 || size_t(sp) * size_t(rows) * size_t(a.N) * sizeof(float) > partial_bytes) break;
        const double part = 4.0 * sp * mn;
        consider(bn, t, sp, 0, 1, pp_time(bn, t * sp, double(nk) / sp, cold) + part / 4.5 + 2.0 +
                                      (part + (ln ? 8.0 : 6.0) * mn) / 4.4);
      }
      // Split tail (256-wide tile): only the tiles that overrun the last full
      // round run in k splits, in a round of their own.
      const int64_t full = t / kCUs, rem = t % kCUs;
      if (bn != 256 || full == 0 || rem == 0) continue;
      for (int tsp = 2; tsp <= 4; ++tsp) {
        const size_t bytes = size_t(rem * tsp) * kBM * 256 * sizeof(float);
        if (rem * tsp > kCUs || nk / tsp < 4 || bytes > partial_bytes) break;
        consider(256, t, 1, rem, tsp,
                 pp_time(256, full * kCUs, double(nk), cold) + pp_time(256, rem * tsp, double(nk) / tsp, cold) - 7.0 +
                     double(bytes) * 1e-6 * (1.0 / 4.5 + 1.0 / 4.4) + 2.0 + norm);
      }
    }
  }
  // Tuning override "BN,SPLITS[,8[,STAGES[,TAIL,TSP]]]" (e.g. AVITS_GEMM_TILE=256,3,8,1),
  // for one launch family with AVITS_GEMM_TILE_<family> (e.g. _gemm_o): BN 256 or 128,
  // STAGES 1 (the default at 256) the ping-pong kernel where its layout holds, else
  // and with 2 (the default at 128) the register-staged one of that width.  TAIL > 0
  // (256-wide tile, SPLITS 1) runs the last min(TAIL, tiles) tiles in TSP k splits.
  const char* env = nullptr;
  if (family) {
    char name[64];
    snprintf(name, sizeof(name), "AVITS_GEMM_TILE_%s", family);
    env = getenv(name);
  }
  if (!env) env = getenv("AVITS_GEMM_TILE");
  if (env) {
    int bn = 0, sp = 0, wv = 8, stg = 0, tail = 0, tsp = 1;
    const int got = sscanf(env, "%d,%d,%d,%d,%d,%d", &bn, &sp, &wv, &stg, &tail, &tsp);
    if (got < 4) stg = bn == 256 ? 1 : 2;
    if (got >= 2 && (bn == 256 || bn == 128) && sp >= 1 && sp <= 4 && wv == 8 && (stg == 1 || stg == 2)) {
      pl.bn = bn;
      pl.stages = wide ? stg : 2;
      pl.splits = sp;
      pl.tiles = tiles_of(a, kBM, pl.bn);
      pl.tail = 0;
      pl.tail_splits = 1;
      if (got == 6 && pl.bn == 256 && sp == 1 && tail > 0 && tsp >= 2 && tsp <= 4 && nk / tsp >= 1) {
        pl.tail = std::min<int64_t>(tail, pl.tiles);
        pl.tail_splits = tsp;
      }
    }
  }
  return pl;
}

size_t gemm_partial_bytes(const GemmArgs& a, const GemmPlan& pl) {
  if (pl.tail > 0) return size_t(pl.tail) * size_t(pl.tail_splits) * kBM * size_t(pl.bn) * sizeof(float);
  if (pl.splits <= 1) return 0;
  const int64_t rows = a.p[0].M + (a.nprob > 1 ? a.p[1].M : 0);
  return size_t(pl.splits) * size_t(rows) * size_t(a.N) * sizeof(float);
}

int launch_gemm(const GemmArgs& a, int dtype, hipStream_t s, const char* family, float* partial,
                size_t partial_bytes, GemmPostLN* post_ln) {
  GemmPlan pl = plan_gemm(a, dtype, partial ? partial_bytes : 0, family, post_ln != nullptr);
  if (pl.tiles == 0) return AVITS_OK;
  if (a.mod.B > 0 && a.mode0 == EPI_RESID_GATE && dtype != AVITS_BF16)
    return set_error(AVITS_ERR_UNSUPPORTED, "gemm %s: per-image gates need bf16", family ? family : "");
  // The register-staged kernels' epilogue has one gate per launch: there, per-image
  // gates are applied by the split-K reduce and such a projection runs split.
  const bool per_image_gate = a.mod.B > 0 && a.mode0 == EPI_RESID_GATE && pl.stages == 2;
  if (per_image_gate && (pl.splits < 2 || pl.tail > 0)) {
    pl.splits = 2;
    pl.tail = 0;
    pl.tail_splits = 1;
  }
  // The reduce kernels take eight columns per thread.
  if ((pl.splits > 1 || pl.tail > 0) && (!partial || partial_bytes < gemm_partial_bytes(a, pl) || a.N % 8 != 0)) {
    if (per_image_gate)
      return set_error(AVITS_ERR_UNSUPPORTED, "gemm %s: per-image gates need a split-K scratch of %zu bytes and N %% 8 == 0",
                       family ? family : "", gemm_partial_bytes(a, pl));
    pl.splits = 1;
    pl.tail = 0;
  }
  if (dtype == AVITS_BF16) {
    {
      TimedLaunch timed(family, s);  // the GEMM kernel alone; the reduce is its own family
      const int64_t units = pl.tiles * pl.splits + pl.tail * (pl.tail_splits - 1);
      // Ping-pong kernel: equal rounds (a split tail: full rounds, then its own).
      const int64_t rounds = ceil_div64(units, kCUs);
      const dim3 pgrid(unsigned(pl.tail > 0 ? std::min<int64_t>(units, kCUs) : ceil_div64(units, rounds)));
      if (pl.stages == 2 && pl.bn == 256)
        hipLaunchKernelGGL(gemm_bf16_staged_kernel, dim3(unsigned(units)), dim3(512), 0, s, a, partial, pl.splits,
                           int(pl.tail), pl.tail_splits);
      else if (pl.stages == 2)
        hipLaunchKernelGGL(gemm_bf16_kernel, dim3(unsigned(units)), dim3(512), 0, s, a, partial, pl.splits);
      else if (pl.bn == 256)
        hipLaunchKernelGGL(gemm_bf16_pp_kernel<256>, pgrid, dim3(512), 0, s, a, partial, int(units), pl.splits,
                           int(pl.tail), pl.tail_splits);
      else
        hipLaunchKernelGGL(gemm_bf16_pp_kernel<128>, pgrid, dim3(512), 0, s, a, partial, int(units), pl.splits, 0, 1);
    }
    if (post_ln) post_ln->done = false;
    if (pl.tail > 0) {
      TimedLaunch timed_reduce("splitk_reduce", s);
      hipLaunchKernelGGL(tail_reduce_kernel, dim3(unsigned(pl.tail * (kBM / 8))), dim3(256), 0, s, a,
                         (const float*)partial, pl.tail, pl.tail_splits);
    }
    const int64_t rows_all = a.p[0].M + (a.nprob > 1 ? a.p[1].M : 0);
    if (pl.splits > 1 && post_ln && a.mode0 == EPI_RESID_GATE && a.n_split >= a.N && a.N % 8 == 0 &&
        a.N <= int64_t(kWave) * 8 * kRlnChunks) {
      TimedLaunch timed_reduce("splitk_reduce", s);
      const dim3 rgrid(unsigned(ceil_div64(rows_all, 4)));
      if (pl.splits == 2) hipLaunchKernelGGL(splitk_reduce_ln_kernel<2>, rgrid, dim3(256), 0, s, a, partial, *post_ln);
      else if (pl.splits == 3) hipLaunchKernelGGL(splitk_reduce_ln_kernel<3>, rgrid, dim3(256), 0, s, a, partial, *post_ln);
      else hipLaunchKernelGGL(splitk_reduce_ln_kernel<4>, rgrid, dim3(256), 0, s, a, partial, *post_ln);
      post_ln->done = true;
    } else if (pl.splits > 1) {
      TimedLaunch timed_reduce("splitk_reduce", s);
      const int64_t rows = rows_all;
      const int64_t work = rows * (a.N / 8);
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3(unsigned(ceil_div64(work, 256))), dim3(256), 0, s, a,
                         (const float*)partial, pl.splits);
    }
  } else {
    TimedLaunch timed(family, s);
    if (pl.bn == kFB) hipLaunchKernelGGL(gemm_f32_valu_kernel, dim3(unsigned(pl.tiles)), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(gemm_f32_kernel, dim3(unsigned(pl.tiles)), dim3(64 * kFWaves), 0, s, a);
  }
  return launch_status("gemm");
}

}  // namespace avits
