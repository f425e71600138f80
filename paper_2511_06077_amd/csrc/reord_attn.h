// The reordered form's narrow attention (reordered.hip) as a device function,
// shared by its own kernel and by the kernel that runs every form of a mixed
// batch's attention side by side (fast.hip).
#pragma once

#include "common.h"
#include "ring.h"

namespace stca {
namespace reord {

constexpr int DH = 32;
constexpr float kSlack = 8.f;  // log2 units: softmax weights stay <= 256 between rescales
constexpr int kWaves = 4;      // X blocks per round of the attention workgroup (two waves each)

// X tile in LDS: the 32 rows in 1 KB segments (512 / D rows each, as one
// wave's direct global-to-LDS load fills them), segments padded by 16 bytes,
// which spreads the rows over the banks while keeping every operand address
// a per-lane base plus a compile-time offset.
constexpr int kSegPitch = 1024 + 16;
__host__ __device__ constexpr size_t tile_bytes(int D) { return (size_t)(D / 16) * kSegPitch; }
// attention kernel LDS: the pairs' double-buffered X tiles (later the merge
// area), then the unit's U rows
__host__ __device__ constexpr size_t main_lds(int D) {
  return (size_t)kWaves * 2 * tile_bytes(D) > (size_t)kWaves * 32 * (D + 2) * 4 ? (size_t)kWaves * 2 * tile_bytes(D)
                                                                                : (size_t)kWaves * 32 * (D + 2) * 4;
}
__host__ __device__ constexpr size_t attn_lds(int D) { return main_lds(D) + (size_t)32 * (D + 8) * 2; }

__device__ __forceinline__ f32x16 mfmab(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}


// v ~ hi + lo, both bf16 (round to nearest even)
__device__ __forceinline__ __bf16 bf_hi(float v) { return static_cast<__bf16>(v); }
__device__ __forceinline__ __bf16 bf_lo(float v, __bf16 hi) { return static_cast<__bf16>(v - static_cast<float>(hi)); }

__device__ __forceinline__ bf16x8 zero8b() {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = static_cast<__bf16>(0.f);
  return r;
}

// ------------------------------------------------------------ attention
// One workgroup per unit (request, target group of up to 32 / H targets,
// history chunk): its rows r = t H + j (at most 32) are the 32 columns of
// every tile.  Eight waves in four pairs; in each round the pairs take the
// next four 32-row X blocks (direct global-to-LDS loads into a per-pair
// double buffer, the next round's blocks in flight while this round's are
// used).  Both waves of a pair form
// the block's scores; each accumulates half of the d columns of Y.  Every
// pair keeps its own online-softmax state; the pairs' partials are merged at
// the end.
//   S^T (32 history rows x 32 rows (t, j)) = X U^T, K = d: A = X row operand,
//   B = U rows (staged once in LDS).
//   Y^T (d x 32) += X^T P^T, K = 32 history rows: B = P^T from the S^T
//   registers (k-step s: rows 16 s + 4 hi + {0..3, 8..11}), A = X^T gathered
//   from the LDS tile for the same history rows.
template <int D>
__device__ __forceinline__ void attn_body(unsigned char* smem, int u, const Unit* __restrict__ units,
                                          const WsHeader* __restrict__ hdr, const __bf16* __restrict__ UN,
                                          const bf16_bits* __restrict__ X, int64_t n_hist, float* __restrict__ part_y,
                                          float2* __restrict__ part_ml, int64_t n_tgt) {
  constexpr int H = D / DH;
  constexpr int KS = D / 16;
  constexpr int CPR = D / 8;          // 16-byte chunks per X row
  constexpr int NDT = D / 32;         // 32-dim tiles of Y^T
  constexpr int HALF = NDT / 2;       // tiles per wave of a pair
  constexpr int PER = 32 * CPR / 64;  // 1 KB segments per block
  constexpr int RPS = 512 / D;        // rows per segment
  constexpr int NT = 128 * kWaves;
  constexpr int TB = static_cast<int>(tile_bytes(D));
  if (u >= hdr->n_units) return;
  const Unit un = units[u];
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int pw = w % kWaves, half = w / kWaves;
  const int tcol = lane % 32, hi = lane / 32;
  const int R = un.nt * H;
  unsigned char* xb = smem + (size_t)pw * 2 * TB;
  // byte offset of element (row, col) in a tile
  auto xoff = [](int row, int col) { return (row / RPS) * kSegPitch + (row % RPS) * 2 * D + col * 2; };
  // the unit's U: hi terms in registers (B operand: row tcol, model dims
  // 16 ks + 8 hi ..), lo terms staged in LDS (padded rows) past the X tiles
  // and the merge area
  constexpr int UROW = D + 8;
  __bf16* us = reinterpret_cast<__bf16*>(smem + main_lds(D));
  for (int e = threadIdx.x; e < 32 * (D / 8); e += NT) {
    const int row = e / (D / 8), c8 = e % (D / 8);
    const bf16x8 v = row < R ? *reinterpret_cast<const bf16x8*>(UN + ((int64_t)un.t0 * H + row) * 2 * D + D + c8 * 8)
                             : zero8b();
    *reinterpret_cast<bf16x8*>(us + row * UROW + c8 * 8) = v;
  }
  const __bf16* ulo = us + tcol * UROW + 8 * hi;
  bf16x8 uhi[KS];
  {
    const __bf16* up = UN + ((int64_t)un.t0 * H + tcol) * 2 * D + 8 * hi;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) uhi[ks] = tcol < R ? *reinterpret_cast<const bf16x8*>(up + 16 * ks) : zero8b();
  }
  f32x16 Y[HALF];
#pragma unroll
  for (int dt = 0; dt < HALF; ++dt) Y[dt] = f32x16{};
  float m = -INFINITY, l = 0.f;
  const int rounds = (un.b1 - un.b0 + kWaves - 1) / kWaves;
  // this pair's block of round r: each wave of the pair loads half of it
  auto dma = [&](int r, int buf) {
    const int b = un.b0 + r * kWaves + pw;
    if (b >= un.b1) return;
#pragma unroll
    for (int i = half * (PER / 2); i < (half + 1) * (PER / 2); ++i) {
      const int p = i * 64 + lane;
      const int row = p / CPR, c = p % CPR;
      const int64_t grow = min((int64_t)b * 32 + row, n_hist - 1);
      __builtin_amdgcn_global_load_lds(static_cast<const void*>(X + grow * D + c * 8),
                                       (void __attribute__((address_space(3)))*)(xb + buf * TB + i * kSegPitch), 16,
                                       0, 0);
    }
  };
  dma(0, 0);
  for (int r = 0; r < rounds; ++r) {
    const int cur = r & 1;
    // round r's blocks have landed (every wave waited for its own loads), and
    // every wave is done with the buffers of round r - 1
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (r + 1 < rounds) dma(r + 1, cur ^ 1);
    const int b = un.b0 + r * kWaves + pw;
    if (b >= un.b1) continue;
    const unsigned char* xt = xb + cur * TB;
    f32x16 s = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 xr = *reinterpret_cast<const bf16x8*>(xt + xoff(tcol, 16 * ks + 8 * hi));
      s = mfmab(xr, uhi[ks], s);
      s = mfmab(xr, *reinterpret_cast<const bf16x8*>(ulo + 16 * ks), s);
    }
    if (b * 32 < un.l0 || b * 32 + 32 > un.l1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int tok = b * 32 + 8 * (v / 4) + 4 * hi + (v % 4);
        s[v] = (tok < un.l0 || tok >= un.l1) ? -INFINITY : s[v];
      }
    }
    float bm = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) bm = fmaxf(bm, s[v]);
    bm = fmaxf(bm, __shfl_xor(bm, 32));
    // per-lane threshold rescale: the reference max moves only when the block
    // maximum exceeds it by kSlack (every block has a valid row, so bm is finite)
    const float mn = bm > m + kSlack ? bm : m;
    const float sc = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
    m = mn;
    float ps = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[v] = __builtin_amdgcn_exp2f(s[v] - mn);
      ps += s[v];
    }
    l = l * sc + ps;
    bf16x8 ph[2], pl[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const __bf16 h = bf_hi(s[i]);
      ph[i / 8][i % 8] = h;
      pl[i / 8][i % 8] = bf_lo(s[i], h);
    }
#pragma unroll
    for (int dt = 0; dt < HALF; ++dt) {
      f32x16 acc = Y[dt] * sc;
      const int dim = 32 * (half * HALF + dt) + tcol;
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        bf16x8 a;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int row = 16 * k2 + 4 * hi + (i < 4 ? i : i + 4);
          a[i] = *reinterpret_cast<const __bf16*>(xt + xoff(row, dim));
        }
        acc = mfmab(a, ph[k2], acc);
        acc = mfmab(a, pl[k2], acc);
      }
      Y[dt] = acc;
      // two gathers in flight at a time: hoisting all of them would take
      // eight registers per element
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // merge the four pairs (the X tiles are dead: their LDS holds the partials)
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem);  // [kWaves][32][D + 2]
  const float lt = l + __shfl_xor(l, 32);
  float* rw = red + ((size_t)pw * 32 + tcol) * (D + 2);
  if (hi == 0 && half == 0) {
    rw[0] = m;
    rw[1] = lt;
  }
#pragma unroll
  for (int dt = 0; dt < HALF; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) rw[2 + 32 * (half * HALF + dt) + 8 * (v / 4) + 4 * hi + (v % 4)] = Y[dt][v];
  __syncthreads();
  for (int it = threadIdx.x; it < R * (D + 1); it += NT) {
    const int row = it / (D + 1), e = it % (D + 1);  // e == D: (max, sum)
    float M = -INFINITY;
    for (int pp = 0; pp < kWaves; ++pp) M = fmaxf(M, red[((size_t)pp * 32 + row) * (D + 2)]);
    float val = 0.f;
    for (int pp = 0; pp < kWaves; ++pp) {
      const float* rr = red + ((size_t)pp * 32 + row) * (D + 2);
      const float f = rr[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(rr[0] - M);
      val += f * (e == D ? rr[1] : rr[2 + e]);
    }
    const int t = row / H, j = row % H;
    const int64_t prow = ((int64_t)un.c * n_tgt + un.t0 + t) * H + j;
    if (e == D)
      part_ml[prow] = make_float2(M, val);
    else
      part_y[prow * D + e] = val;
  }
}

}  // namespace reord
}  // namespace stca
