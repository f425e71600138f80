// Kernels of the paper-exact layer stack (Sec. 3.1): the token-wise SwiGLU
// block of Eq. swigluffn followed by LayerNorm, on the history rows (the
// dominant cost: 6 r d^2 flop per row and layer) and the small target-side
// pieces (gate, row LayerNorm, query packing for the fused attention kernel).
//
// History transform X~ = LN(SwiGLUFFN(X)), bf16 in and out, one workgroup of
// eight waves (two per SIMD, so one wave's gate arithmetic overlaps the other's
// MFMAs) per 256 history rows, one wave per 32 rows:
//
//   U^T = W_u^T X^T, V^T = W_v^T X^T   (32 hidden columns at a time, MFMA
//                                       32x32x16 bf16, X^T held in registers)
//   G^T = U^T * V^T * sigmoid(V^T)     (registers, rounded to bf16)
//   Y^T += W_o^T G^T                   (all d rows accumulated in registers)
//   X~ = LN(Y) per row                 (the row's d values sit in one lane pair)
//
// The hidden activations never leave the registers: the result registers of
// U^T and V^T hold, for lane (row l%32, half hi), hidden columns
// 16kk + 4hi + {0..3, 8..11} (kk = 0, 1), which is a valid B operand of the
// down projection when W_o's rows are packed in that same order.  Weights are
// repacked once per call into per-chunk operand order (32 hidden columns:
// W_u^T fragments, W_v^T fragments, W_o^T fragments, contiguous) and each
// chunk is copied into LDS with direct global-to-LDS loads, double buffered,
// so the eight waves share one copy.
#include "common.h"
#include "paper.h"
#include "split.h"

namespace stca {

namespace {

__device__ __forceinline__ f32x16 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 zero8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = static_cast<__bf16>(0.f);
  return z;
}

// SiLU gate of Eq. swigluffn: u * v * sigmoid(v)
__device__ __forceinline__ float swiglu_gate(float u, float v) {
  return u * v * __builtin_amdgcn_rcpf(1.f + __expf(-v));
}

// hidden row of slot (kk, hi, i) of a packed W_o fragment: the order in which
// the up projection's result registers hold hidden columns
__device__ __forceinline__ int gate_row(int kk, int hi, int i) { return 16 * kk + 4 * hi + (i < 4 ? i : i + 4); }

__global__ void swiglu_pack_kernel(const bf16_bits* __restrict__ Wu, const bf16_bits* __restrict__ Wv,
                                   const bf16_bits* __restrict__ Wo, int D, int F, bf16_bits* __restrict__ P,
                                   int64_t groups_per_layer) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= groups_per_layer) return;
  const int layer = blockIdx.y;
  const int KS = D / 16;
  const int64_t per_chunk = (int64_t)(2 * KS + 2 * (D / 32)) * 64;
  const int c = static_cast<int>(g / per_chunk);
  int q = static_cast<int>(g % per_chunk);
  Wu += (int64_t)layer * D * F;
  Wv += (int64_t)layer * D * F;
  Wo += (int64_t)layer * F * D;
  bf16_bits* dst = P + ((int64_t)layer * groups_per_layer + g) * 8;
  const int l = q % 64, n = l % 32, hi = l / 32;
  if (q < 2 * KS * 64) {
    const bf16_bits* W = q < KS * 64 ? Wu : Wv;
    const int ks = (q / 64) % KS;
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[i] = W[(int64_t)(16 * ks + 8 * hi + i) * F + 32 * c + n];
  } else {
    q -= 2 * KS * 64;
    const int nt = q / 128, kk = (q / 64) % 2;
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[i] = Wo[(int64_t)(32 * c + gate_row(kk, hi, i)) * D + 32 * nt + n];
  }
}

// NW waves per workgroup, 32 rows each: eight (two per SIMD), or four for few
// rows (see swiglu_ln).
template <int D, int NW>
__global__ __launch_bounds__(NW * 64)
__attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void swiglu_ln_kernel(
    const bf16_bits* __restrict__ X, int64_t n_rows, const unsigned char* __restrict__ Wp, int F,
    bf16_bits* __restrict__ out16, float* __restrict__ out32) {
  constexpr int KS = D / 16;       // k-steps of the up projections
  constexpr int NT = D / 32;       // 32-row tiles of Y^T
  constexpr int UB = KS * 1024;    // bytes of one chunk's W_u^T (or W_v^T) fragments
  constexpr int CB = 2 * UB + NT * 2048;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [2][CB]
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int tcol = lane % 32, hi = lane / 32;
  const int64_t row = (int64_t)blockIdx.x * (32 * NW) + 32 * w + tcol;
  const bool live = row < n_rows;

  // X^T as B operands: lane (row, hi), k-step ks holds X[row][16ks + 8hi .. +7]
  bf16x8 xb[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    xb[ks] = live ? *reinterpret_cast<const bf16x8*>(X + row * D + 16 * ks + 8 * hi) : zero8();
  f32x16 Y[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) Y[t] = f32x16{};

  const int nch = F / 32;
  auto dma = [&](int c, int buf) {
    const unsigned char* src = Wp + (size_t)c * CB + lane * 16;
    unsigned char* dst = smem + buf * CB;
    for (int i = w; i < CB / 1024; i += NW)
      __builtin_amdgcn_global_load_lds(static_cast<const void*>(src + i * 1024),
                                       (void __attribute__((address_space(3)))*)(dst + i * 1024), 16, 0, 0);
  };
  dma(0, 0);
  for (int c = 0; c < nch; ++c) {
    const int cur = c & 1;
    // chunk c has landed (each wave waited for its own copies) and every wave
    // is done with chunk c - 1, whose buffer the next copy overwrites
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (c + 1 < nch) dma(c + 1, cur ^ 1);
    const bf16x8* Ua = reinterpret_cast<const bf16x8*>(smem + cur * CB) + lane;
    const bf16x8* Va = Ua + KS * 64;
    const bf16x8* Oa = Va + KS * 64;
    f32x16 u = {}, v = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u = mfma_bf16(Ua[ks * 64], xb[ks], u);
      v = mfma_bf16(Va[ks * 64], xb[ks], v);
    }
    bf16x8 g[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) g[i / 8][i % 8] = static_cast<__bf16>(swiglu_gate(u[i], v[i]));
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      Y[t] = mfma_bf16(Oa[(2 * t) * 64], g[0], Y[t]);
      Y[t] = mfma_bf16(Oa[(2 * t + 1) * 64], g[1], Y[t]);
    }
  }
  // LayerNorm of the row: lane (row, hi) holds Y[row][32t + 8(v/4) + 4hi + v%4]
  float s = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) s += Y[t][v];
  s += __shfl_xor(s, 32);
  const float mean = s * (1.f / D);
  float q = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = Y[t][v] - mean;
      q += e * e;
    }
  q += __shfl_xor(q, 32);
  const float rstd = rsqrtf(q * (1.f / D) + kLnEps);
  if (!live) return;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int col = 32 * t + 8 * g4 + 4 * hi;
      float o[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = (Y[t][4 * g4 + k] - mean) * rstd;
      uint2 pk;
      pk.x = (uint32_t)from_f32<bf16_bits>(o[0]) | ((uint32_t)from_f32<bf16_bits>(o[1]) << 16);
      pk.y = (uint32_t)from_f32<bf16_bits>(o[2]) | ((uint32_t)from_f32<bf16_bits>(o[3]) << 16);
      *reinterpret_cast<uint2*>(out16 + row * D + col) = pk;
      if (out32) *reinterpret_cast<float4*>(out32 + row * D + col) = make_float4(o[0], o[1], o[2], o[3]);
    }
}

template <int D>
constexpr size_t swiglu_chunk_bytes() {
  return (size_t)2 * (D / 16) * 1024 + (size_t)(D / 32) * 2048;
}

// (a parameter of the template, so that each kernel has its own record)
template <auto kernel>
hipError_t allow_lds(size_t bytes) {
  static int set_for[64] = {0};  // per device: bytes granted so far
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < 64 && set_for[dev] >= static_cast<int>(bytes)) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                          static_cast<int>(bytes));
  if (e == hipSuccess && dev >= 0 && dev < 64) set_for[dev] = static_cast<int>(bytes);
  return e;
}

// ------------------------------------------------------------ target side
__global__ void gate_kernel(float* __restrict__ u, const float* __restrict__ v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const float vv = v[i];
    u[i] = u[i] * vv / (1.f + expf(-vv));
  }
}

// one wave per row; two passes over the row (mean, then centred squares)
__global__ __launch_bounds__(256) void ln_rows_kernel(const float* __restrict__ y, int64_t rows, int d,
                                                      float* __restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
  const int lane = threadIdx.x % 64;
  if (r >= rows) return;
  const float* p = y + r * d;
  float s = 0.f;
  for (int e = lane; e < d; e += 64) s += p[e];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  const float mean = s / d;
  float q = 0.f;
  for (int e = lane; e < d; e += 64) {
    const float c = p[e] - mean;
    q += c * c;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) q += __shfl_xor(q, o);
  const float rstd = 1.f / sqrtf(q / d + kLnEps);
  for (int e = lane; e < d; e += 64) out[r * d + e] = (p[e] - mean) * rstd;
}

// One target-side stage of the bf16 path in one launch: the merge of layer i's
// attention partials into a and o^(i) = a W_O (unless `first`), the fusion
// f = [o^(1) .. o^(i) || x_t] W_C (f = x_t when `first`), the SwiGLU block
// y = ((f W_u) * silu(f W_v)) W_o, and either q = LN(y) with the next layer's
// attention queries Q = q W_Q (fp16, the attention kernel's order) or, for the
// head, z = y.  32-target tiles, one wave per 32 output columns, as the
// target update of the standard stack; every product multiplies the bf16
// weights by the fp32 activation split into three bf16 terms (exact products,
// fp32 sums).
//
// As separate GEMMs (64 x 64 tiles, the down projection on the fp32 matrix
// cores with its K split over atomics), gates, norms, merges and query
// packing, 11 launches a layer took 930 us of the 3730 us step at 2080 targets;
// here a stage streams its weights once per target group (2.3 MB at the last
// fusion of four layers, d = 256) and is bound by that stream and by the 3 x
// MFMA of the terms: 59 us a stage, 3115 us the step (two splits).  With
// `splits` > 1 workgroups (group, split) divide the hidden columns and the
// last to arrive sums their parts of y in split order (split.h), so few
// targets use more CUs.
template <int D, int NC>
__global__ __launch_bounds__(64 * (D / 32)) void paper_target_kernel(PaperTarget A) {
  constexpr int NW = D / 32;
  constexpr int H = D / 32;
  constexpr int KS = D / 16;
  constexpr int AROW = D + 8;  // padded LDS row (bf16 elements)
  constexpr int NT = 64 * NW;
  __shared__ __attribute__((aligned(16))) bf16_bits act[3][32 * AROW];
  __shared__ __attribute__((aligned(16))) bf16_bits hid[3][32 * AROW];
  __shared__ float red[NW][32];
  __shared__ int arrived;
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int tcol = lane % 32, hi = lane / 32;
  const int group = blockIdx.x / A.splits, split = blockIdx.x % A.splits;
  const int64_t tb = (int64_t)group * 32;
  const int64_t t = tb + tcol;
  const bool tok = t < A.n_tgt;

  // 4 consecutive fp32 values (row r, columns c..c+3) as three bf16 terms
  auto put4 = [&](bf16_bits (*buf)[32 * AROW], int r, int c, const float* v) {
    float x[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int term = 0; term < 3; ++term) {
      bf16_bits b[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        b[e] = from_f32<bf16_bits>(x[e]);
        x[e] -= to_f32(b[e]);
      }
      *reinterpret_cast<uint2*>(buf[term] + r * AROW + c) =
          make_uint2((uint32_t)b[0] | ((uint32_t)b[1] << 16), (uint32_t)b[2] | ((uint32_t)b[3] << 16));
    }
  };
  // a wave's result tile: lane = target tcol, elements = columns 32 w + 8 q + 4 hi + e
  auto put_tile = [&](bf16_bits (*buf)[32 * AROW], const f32x16& v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float x[4] = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      put4(buf, tcol, 32 * w + 8 * q + 4 * hi, x);
    }
  };
  auto store_tile = [&](float* dst, int64_t ld, const f32x16& v) {
    if (!tok) return;
    float* p = dst + t * ld + 32 * w + 4 * hi;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(p + 8 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
  };
  // x_t (bf16: its second and third terms are zero)
  auto put_targets = [&]() {
    for (int c = threadIdx.x; c < 32 * D / 8; c += NT) {
      const int row = c / (D / 8), col = (c % (D / 8)) * 8;
      const uint4 z = make_uint4(0, 0, 0, 0);
      *reinterpret_cast<uint4*>(act[0] + row * AROW + col) =
          tb + row < A.n_tgt ? *reinterpret_cast<const uint4*>(A.tgt + (tb + row) * D + col) : z;
      *reinterpret_cast<uint4*>(act[1] + row * AROW + col) = z;
      *reinterpret_cast<uint4*>(act[2] + row * AROW + col) = z;
    }
  };
  auto fetch = [&](bf16x8 (&r)[KS], const bf16x8* __restrict__ Wp) {
#pragma unroll
    for (int k = 0; k < KS; ++k) r[k] = Wp[k * 64 + lane];
  };
  auto operand = [&](const bf16_bits (*src)[32 * AROW], int term, int k) {
    return *reinterpret_cast<const bf16x8*>(src[term] + tcol * AROW + 8 * hi + 16 * k);
  };
  auto gemm_r = [&](const bf16x8 (&wt)[KS], const bf16_bits (*src)[32 * AROW], f32x16& acc) {
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int term = 0; term < 3; ++term) acc = mfma_bf16(wt[k], operand(src, term, k), acc);
  };
  auto gemm = [&](const bf16x8* __restrict__ Wp, const bf16_bits (*src)[32 * AROW], f32x16& acc) {
    bf16x8 wt[KS];
    fetch(wt, Wp);
    gemm_r(wt, src, acc);
  };
  const bf16x8* WoP = static_cast<const bf16x8*>(A.WoP);
  const bf16x8* WcP = static_cast<const bf16x8*>(A.WcP);
  const bf16x8* WuP = static_cast<const bf16x8*>(A.WuP);
  const bf16x8* WvP = static_cast<const bf16x8*>(A.WvP);
  const bf16x8* WdP = static_cast<const bf16x8*>(A.WdP);
  const bf16x8* WqP = static_cast<const bf16x8*>(A.WqP);
  const int KC = (A.n_cat + 1) * KS;  // k-steps of W_C
  auto wc_tile = [&](int blk) { return WcP + ((int64_t)w * KC + (int64_t)blk * KS) * 64; };

  if (A.first) {
    put_targets();
    __syncthreads();
  } else {
    bf16x8 wo[KS];
    fetch(wo, WoP + (int64_t)w * KS * 64);  // lands during the merge
    // merge the chunk partials: a wave's lanes read whole rows, four
    // dimensions a lane, eight rows a pass, four chunks a round trip; the
    // records of max_ch chunks are requested together with the target's own
    // chunk count, which only masks them
    constexpr int LPR = D / 4, CG = 4;
    const int prow = threadIdx.x / LPR, dim = 4 * (threadIdx.x % LPR), j = dim / 32;
#pragma unroll 1
    for (int p0 = 0; p0 < 32; p0 += 16) {
      float M[2], Ls[2], av[2][4];
      int nch[2];
      int64_t tt[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int64_t r = tb + p0 + 8 * i + prow;
        tt[i] = r < A.n_tgt ? r : A.n_tgt - 1;
        nch[i] = r < A.n_tgt ? A.tchunks[tt[i]] : 0;
        M[i] = -INFINITY;
        Ls[i] = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) av[i][e] = 0.f;
      }
#pragma unroll 1
      for (int cb = 0; cb < A.max_ch; cb += CG) {
        float2 ml[2][CG];
        float4 x[2][CG];
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            if (cb + c < A.max_ch) {
              ml[i][c] = static_cast<const float2*>(A.part_ml)[((int64_t)(cb + c) * A.n_tgt + tt[i]) * H + j];
              x[i][c] = *reinterpret_cast<const float4*>(A.part_acc + ((int64_t)(cb + c) * A.n_tgt + tt[i]) * D + dim);
            }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          float mn = M[i];
#pragma unroll
          for (int c = 0; c < CG; ++c)
            if (cb + c < nch[i]) mn = fmaxf(mn, ml[i][c].x);
          const float sc = M[i] == -INFINITY ? 0.f : exp2f(M[i] - mn);
          M[i] = mn;
          Ls[i] *= sc;
#pragma unroll
          for (int e = 0; e < 4; ++e) av[i][e] *= sc;
#pragma unroll
          for (int c = 0; c < CG; ++c)
            if (cb + c < nch[i]) {
              const float wgt = exp2f(ml[i][c].x - mn);
              Ls[i] += wgt * ml[i][c].y;
              av[i][0] += wgt * x[i][c].x;
              av[i][1] += wgt * x[i][c].y;
              av[i][2] += wgt * x[i][c].z;
              av[i][3] += wgt * x[i][c].w;
            }
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = p0 + 8 * i + prow;
        if (tb + row < A.n_tgt) {
          const float inv = 1.f / Ls[i];
#pragma unroll
          for (int e = 0; e < 4; ++e) av[i][e] *= inv;
          if (A.a_out && split == 0)
            *reinterpret_cast<float4*>(A.a_out + tt[i] * D + dim) =
                make_float4(av[i][0], av[i][1], av[i][2], av[i][3]);
          if (A.lse_out && split == 0 && dim % 32 == 0) A.lse_out[tt[i] * H + j] = (M[i] + log2f(Ls[i])) * kLn2;
        }
        put4(act, row, dim, av[i]);
      }
    }
    __syncthreads();
    f32x16 o = {};
    gemm_r(wo, act, o);
    if (split == 0) store_tile(A.cat + (int64_t)(A.n_cat - 1) * D, A.ldcat, o);
    // f = [o^(1) .. o^(i) || x_t] W_C: the block in registers first, then the
    // earlier layers' blocks and x_t through LDS
    f32x16 f = {};
    __syncthreads();  // every wave is done with a
    put_tile(act, o);
    __syncthreads();
    gemm(wc_tile(A.n_cat - 1), act, f);
#pragma unroll 1
    for (int blk = 0; blk + 1 < A.n_cat; ++blk) {
      __syncthreads();
      for (int c = threadIdx.x; c < 32 * D / 4; c += NT) {
        const int row = c / (D / 4), col = (c % (D / 4)) * 4;
        const float4 v = tb + row < A.n_tgt
                             ? *reinterpret_cast<const float4*>(A.cat + (tb + row) * A.ldcat + (int64_t)blk * D + col)
                             : make_float4(0.f, 0.f, 0.f, 0.f);
        const float x[4] = {v.x, v.y, v.z, v.w};
        put4(act, row, col, x);
      }
      __syncthreads();
      gemm(wc_tile(blk), act, f);
    }
    __syncthreads();
    put_targets();
    __syncthreads();
    gemm(wc_tile(A.n_cat), act, f);
    __syncthreads();
    put_tile(act, f);
    __syncthreads();
  }

  // the SwiGLU block, D hidden columns at a time (this split's)
  f32x16 y = {};
  const int nc = NC > 0 ? NC : A.F / (D * A.splits);
  const int c0 = split * nc;
#pragma unroll(NC > 0 ? NC : 1)
  for (int c = 0; c < nc; ++c) {
    const int64_t up = (int64_t)((c0 + c) * NW + w) * KS * 64;
    f32x16 u = {}, v = {};
    {
      bf16x8 wu[KS], wv[KS];
      fetch(wu, WuP + up);
      fetch(wv, WvP + up);
#pragma unroll
      for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int term = 0; term < 3; ++term) {
          const bf16x8 x = operand(act, term, k);
          u = mfma_bf16(wu[k], x, u);
          v = mfma_bf16(wv[k], x, v);
        }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) u[i] = u[i] * v[i] / (1.f + expf(-v[i]));
    if (c > 0) __syncthreads();  // hid was read by the previous chunk's down projection
    put_tile(hid, u);
    __syncthreads();
    gemm(WdP + ((int64_t)w * (A.F / 16) + (int64_t)(c0 + c) * KS) * 64, hid, y);
  }
  if (A.splits > 1 && !split_sum<NT>(y, A.spart, A.cnt + group, A.splits, A.groups, group, split, &arrived)) return;
  if (A.z_out) {
    if (tok) {
      bf16_bits* p = A.z_out + t * D + 32 * w + 4 * hi;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint2 pk;
        pk.x = (uint32_t)from_f32<bf16_bits>(y[4 * q]) | ((uint32_t)from_f32<bf16_bits>(y[4 * q + 1]) << 16);
        pk.y = (uint32_t)from_f32<bf16_bits>(y[4 * q + 2]) | ((uint32_t)from_f32<bf16_bits>(y[4 * q + 3]) << 16);
        *reinterpret_cast<uint2*>(p + 8 * q) = pk;
      }
    }
    return;
  }
  // LayerNorm over the row (all waves), mean then centred squares
  auto row_sum = [&](float s) {
    s += __shfl_xor(s, 32);
    if (hi == 0) red[w][tcol] = s;
    __syncthreads();
    float r = 0.f;
#pragma unroll
    for (int k = 0; k < NW; ++k) r += red[k][tcol];
    __syncthreads();
    return r;
  };
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) s += y[i];
  const float mean = row_sum(s) / D;
  float q2 = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    y[i] -= mean;
    q2 += y[i] * y[i];
  }
  const float rstd = 1.f / sqrtf(row_sum(q2) / D + kLnEps);
#pragma unroll
  for (int i = 0; i < 16; ++i) y[i] *= rstd;
  if (A.q_out) store_tile(A.q_out, D, y);
  put_tile(act, y);  // act was last read before the row sums' barriers
  __syncthreads();
  f32x16 q = {};
  gemm(WqP + (int64_t)w * KS * 64, act, q);
  if (tok) {
    const float qs = kLog2e * 0.17677669529663687f;  // log2(e) / sqrt(32)
    f16x8 h0, h1;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h0[i] = static_cast<_Float16>(q[i] * qs);
      h1[i] = static_cast<_Float16>(q[8 + i] * qs);
    }
    f16x8* qn = static_cast<f16x8*>(A.QN) + (t * D + 32 * w) / 8;
    qn[hi] = h0;
    qn[2 + hi] = h1;
  }
}

}  // namespace

// ------------------------------------------------------------ launchers
size_t swiglu_packed_bytes(int D, int F) { return (size_t)(F / 32) * (2 * (D / 16) * 1024 + (D / 32) * 2048); }

hipError_t swiglu_pack(const void* Wu, const void* Wv, const void* Wo, int n_layers, int D, int F, void* P,
                       hipStream_t st) {
  if (D % 32 || F % 32) return hipErrorInvalidValue;
  const int64_t groups = (int64_t)(F / 32) * (2 * (D / 16) + 2 * (D / 32)) * 64;
  hipLaunchKernelGGL(swiglu_pack_kernel, dim3(static_cast<unsigned>(ceil_div(groups, 256)), n_layers), dim3(256), 0,
                     st, (const bf16_bits*)Wu, (const bf16_bits*)Wv, (const bf16_bits*)Wo, D, F, (bf16_bits*)P,
                     groups);
  return hipGetLastError();
}

// One wave per SIMD takes 73 us for its rows' chunks and two 97-102 (d = 256,
// F = 4 d), whatever share of the rows is live, so few rows, up to 128 a CU,
// go out as four-wave workgroups (14000 rows 81 -> 73 us); more as eight-wave
// ones throughout (the rest of whole rounds as a four-wave launch: 512 + 73 us
// against 585 in one, 333397 rows).
hipError_t swiglu_ln(int D, const void* X, int64_t n_rows, const void* Wp_layer, int F, void* out16, float* out32,
                     int n_cu, hipStream_t st) {
  if (n_rows == 0) return hipSuccess;
  if (F % 32 || n_cu < 1) return hipErrorInvalidValue;
  const bool few = n_rows <= 128 * static_cast<int64_t>(n_cu);
#define STCA_SWIGLU1(DD, NW)                                                                               \
  {                                                                                                        \
    const size_t lds = 2 * swiglu_chunk_bytes<DD>();                                                       \
    hipError_t e = allow_lds<swiglu_ln_kernel<DD, NW>>(lds);                                               \
    if (e != hipSuccess) return e;                                                                         \
    hipLaunchKernelGGL((swiglu_ln_kernel<DD, NW>), dim3(static_cast<unsigned>(ceil_div(n_rows, 32 * NW))), \
                       dim3(64 * NW), lds, st, (const bf16_bits*)X, n_rows,                                \
                       (const unsigned char*)Wp_layer, F, (bf16_bits*)out16, out32);                       \
  }
#define STCA_SWIGLU(DD) \
  if (few) STCA_SWIGLU1(DD, 4) else STCA_SWIGLU1(DD, 8)
  switch (D) {
    case 64: STCA_SWIGLU(64); break;
    case 128: STCA_SWIGLU(128); break;
    case 256: STCA_SWIGLU(256); break;
    default: return hipErrorInvalidValue;
  }
#undef STCA_SWIGLU
#undef STCA_SWIGLU1
  return hipGetLastError();
}

hipError_t swiglu_gate_f32(float* u, const float* v, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(gate_kernel, dim3(static_cast<unsigned>(ceil_div(n, 256))), dim3(256), 0, st, u, v, n);
  return hipGetLastError();
}

hipError_t layer_norm_rows(const float* y, int64_t rows, int d, float* out, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(ln_rows_kernel, dim3(static_cast<unsigned>(ceil_div(rows, 4))), dim3(256), 0, st, y, rows, d,
                     out);
  return hipGetLastError();
}

hipError_t paper_target(int D, const PaperTarget& f, hipStream_t st) {
  if (f.n_tgt == 0) return hipSuccess;
  if (f.splits < 1 || f.F % (D * f.splits) || (f.splits > 1 && (!f.spart || !f.cnt)) ||
      (!f.first && (f.n_cat < 1 || f.max_ch < 1 || f.max_ch > kMaxChunks)))
    return hipErrorInvalidValue;
  PaperTarget A = f;
  A.groups = static_cast<int>(ceil_div(f.n_tgt, 32));
  const dim3 g(static_cast<unsigned>((int64_t)A.groups * A.splits));
  // hidden chunks a workgroup at F = 4 d: 1, 2 or 4, known to the compiler
  const int nc = f.F == 4 * D ? 4 / f.splits : 0;
#define STCA_PT1(DD, NC) hipLaunchKernelGGL((paper_target_kernel<DD, NC>), g, dim3(64 * (DD / 32)), 0, st, A)
#define STCA_PT(DD)                     \
  switch (nc) {                         \
    case 1: STCA_PT1(DD, 1); break;     \
    case 2: STCA_PT1(DD, 2); break;     \
    case 4: STCA_PT1(DD, 4); break;     \
    default: STCA_PT1(DD, 0); break;    \
  }
  switch (D) {
    case 64: STCA_PT(64); break;
    case 128: STCA_PT(128); break;
    case 256: STCA_PT(256); break;
    default: return hipErrorInvalidValue;
  }
#undef STCA_PT
#undef STCA_PT1
  return hipGetLastError();
}

}  // namespace stca
