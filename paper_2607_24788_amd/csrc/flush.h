// Folding a unit's pending tokens outside a decode step: glide_state_flush and
// the start of a prefill call.
#pragma once

#include "glide_internal.h"

namespace glide {

// Fold every pending token of a unit into S and z (nf := beta = max(0, p-W)),
// leaving the state in its direct form S = sum_{j < beta} phi(k_j)^T v_j.
// Plain fp32 arithmetic: it runs once per prefill call, not per token.  Run by
// every thread of a workgroup of NTH; `lay` is the layer's sections, Wf the
// unit's feature weights.  For a linear part delayed by W > 0 only (others
// fold on every step).
template <typename T, int D, int DF, int NTH>
__device__ __forceinline__ void flush_unit(char* lay, int B, int Hkv, int W, int R, int64_t unit, const T* Wf, int phi,
                                           bool gated) {
  __shared__ float kx[kFoldPeriod][D], vx[kFoldPeriod][D], pk[kFoldPeriod][DF];
  const int tid = threadIdx.x;
  const LayerSections sec = layer_sections(B, Hkv, D, DF, R, sizeof(T));
  const int64_t p = reinterpret_cast<const int64_t*>(lay + sec.pos)[unit];
  int64_t* nf_ptr = reinterpret_cast<int64_t*>(lay + sec.nf) + unit;
  const int64_t beta = p - W > 0 ? p - W : 0;
  int64_t nf = *nf_ptr;
  nf = nf < beta ? nf : beta;
  nf = nf > beta - kFoldPeriod ? nf : beta - kFoldPeriod;
  nf = nf > 0 ? nf : 0;
  const int n = int(beta - nf);
  // gated: S, z (decayed to G_f) and the pending tokens are brought to
  // G_{p-1}, the last token consumed
  const LayerSections secg = layer_sections(B, Hkv, D, DF, R, sizeof(T), gated);
  double* gst = reinterpret_cast<double*>(lay + secg.G) + 2 * unit;
  const double* grg = reinterpret_cast<const double*>(lay + secg.GR) + unit * int64_t(R);
  const double gcur = gated ? gst[0] : 0.0;
  const bool regate = gated && nf > 0 && gst[1] != gcur;
  if (n == 0 && !regate) return;
  float* S = reinterpret_cast<float*>(lay + sec.S) + unit * DF * D;
  float* z = reinterpret_cast<float*>(lay + sec.z) + unit * DF;
  const T* Kr = reinterpret_cast<const T*>(lay + sec.K) + unit * int64_t(R) * D;
  const T* Vr = reinterpret_cast<const T*>(lay + sec.V) + unit * int64_t(R) * D;
  for (int e = tid; e < n * D; e += NTH) {
    const int i = e / D, c = e - i * D;
    const int32_t slot = int32_t((nf + i) % R);
    kx[i][c] = to_f32(Kr[kring_elem(slot, c, D)]);
    vx[i][c] = to_f32(Vr[vring_elem(slot, c, D)]);
  }
  __syncthreads();
  for (int e = tid; e < n * DF; e += NTH) {
    const int i = e / DF, f = e - i * DF;
    float acc = 0.f;
    for (int c = 0; c < D; ++c) acc = fmaf(kx[i][c], to_f32(Wf[c * DF + f]), acc);
    pk[i][f] = feat_act(acc, phi);
  }
  __syncthreads();
  if (phi == GLIDE_PHI_SOFTMAX) {
    softmax_rows_lds<DF, NTH>(&pk[0][0], DF, n);
    __syncthreads();
  }
  if (gated && n > 0) {
    for (int e = tid; e < n * DF; e += NTH) {
      const int i = e / DF, f = e - i * DF;
      pk[i][f] *= decay_exp(float(gcur - grg[(nf + i) % R]));
    }
    __syncthreads();
  }
  const bool s_nonzero = nf > 0;
  const float sd = gated && s_nonzero ? decay_exp(float(gcur - gst[1])) : 1.f;
  for (int e = tid; e < DF * D / 4; e += NTH) {
    const int f = e / (D / 4), c4 = (e - f * (D / 4)) * 4;
    float4 sv = s_nonzero ? *reinterpret_cast<const float4*>(S + f * D + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
    sv.x *= sd; sv.y *= sd; sv.z *= sd; sv.w *= sd;
    for (int i = 0; i < n; ++i) {
      const float w = pk[i][f];
      sv.x = fmaf(w, vx[i][c4], sv.x);
      sv.y = fmaf(w, vx[i][c4 + 1], sv.y);
      sv.z = fmaf(w, vx[i][c4 + 2], sv.z);
      sv.w = fmaf(w, vx[i][c4 + 3], sv.w);
    }
    *reinterpret_cast<float4*>(S + f * D + c4) = sv;
  }
  for (int f = tid; f < DF; f += NTH) {
    float zf = s_nonzero ? z[f] * sd : 0.f;
    for (int i = 0; i < n; ++i) zf += pk[i][f];
    z[f] = zf;
  }
  __syncthreads();  // every thread has read G_f
  if (tid == 0) {
    *nf_ptr = beta;
    if (gated) gst[1] = gcur;
  }
}

}  // namespace glide
