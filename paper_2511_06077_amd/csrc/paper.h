// Launchers of the paper-exact layer stack's kernels (paper.hip).
#pragma once

#include "common.h"

namespace stca {

constexpr float kLnEps = 1e-5f;  // LayerNorm epsilon (scale 1, shift 0)

// Bytes of one layer's SwiGLU weights in per-chunk operand order.
size_t swiglu_packed_bytes(int D, int F);
// Repack W_u, W_v [n_layers][D][F] and W_o [n_layers][F][D] (bf16) into
// P [n_layers][swiglu_packed_bytes].
hipError_t swiglu_pack(const void* Wu, const void* Wv, const void* Wo, int n_layers, int D, int F, void* P,
                       hipStream_t st);
// out16 (bf16, required) and out32 (fp32, nullable) [n_rows][D] =
// LN(SwiGLUFFN(X)) with one layer's packed weights; D in {64, 128, 256},
// F % 32 == 0.
hipError_t swiglu_ln(int D, const void* X, int64_t n_rows, const void* Wp_layer, int F, void* out16, float* out32,
                     int n_cu, hipStream_t st);
// u = u * v * sigmoid(v), elementwise (fp32).
hipError_t swiglu_gate_f32(float* u, const float* v, int64_t n, hipStream_t st);
// out[r] = LN(y[r]) over d features (fp32; out may alias y).
hipError_t layer_norm_rows(const float* y, int64_t rows, int d, float* out, hipStream_t st);
// One target-side stage of the bf16 path (paper_target_kernel).  Packed
// weights are bf16 operand tiles (fast_pack_many with to_f16 = 0).
struct PaperTarget {
  int first;                  // f = x_t (no attention to merge)
  int n_cat;                  // else: blocks of `cat` in f, the last one formed here
  int F;
  int64_t n_tgt;
  const bf16_bits* tgt;       // [n_tgt][D]
  const int32_t* tchunks;     // attention partials of the layer merged
  const float* part_acc;
  const void* part_ml;
  int max_ch;                 // no target has more chunks
  float *a_out, *lse_out;     // nullable [n_tgt][D], [n_tgt][H]
  float* cat;                 // [n_tgt] rows of pitch ldcat, o^(k) in columns [(k-1) D, k D)
  int64_t ldcat;
  const void *WoP, *WcP;      // unused when first; W_C (or W_Z) with (n_cat + 1) D rows
  const void *WuP, *WvP, *WdP;  // the SwiGLU block
  const void* WqP;            // the next layer's W_Q (unused with z_out)
  float* q_out;               // nullable [n_tgt][D]
  void* QN;                   // fp16 queries, the fused attention kernel's layout
  bf16_bits* z_out;           // head: y goes here and nothing follows
  int splits, groups;         // workgroups per 32 targets (F / D a multiple); groups is set by the launcher
  float* spart;               // splits > 1: [splits][ceil(n_tgt / 32)][32 D]
  int32_t* cnt;               // splits > 1: [ceil(n_tgt / 32)], zero before the call
};
hipError_t paper_target(int D, const PaperTarget& f, hipStream_t st);

}  // namespace stca
