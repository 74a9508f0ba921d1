// gbla_backward.hip -- the backward pass of GBLA (the chain rule through the
// forward pass of Section 2.1), fp32 arithmetic on bf16 or fp32 inputs.
//
// For one sequence and head, with the forward quantities recomputed
// (qt = Conv1D(q), Qh = phi(qt), P = phi(kt), g = softmax(a), S, z,
// num_i = Qh_i^T S, den_i = Qh_i^T z, o_i = num_i / den_i,
// rs_i = (mean o_i^2 + eps)^(-1/2), oh_i = rs_i o_i, y = oh gamma silu(r)):
//
//   query pass  doh = dy gamma silu(r), dgamma += dy oh silu(r),
//               dr = dy oh gamma silu'(r),
//               do = rs doh - rs^3/d (doh . o) o,
//               dnum = do / den, dden = -(do . o) / den,
//               dQh = S dnum + z dden, dqt = dQh phi'(qt),
//               dS = sum_i Qh_i dnum_i^T, dz = sum_i Qh_i dden_i
//   key pass    t_j = dS vt_j + dz, dkt = g_j t_j phi'(kt), dvt = g_j dS^T P_j,
//               da_j = g_j (P_j . t_j)
//   conv pass   dx_m = sum_t w_t dxt_{m+W-1-t}, dw_t = sum_i dxt_i x_{i-W+1+t}
//
// da has no softmax centering term: o does not change when every gate of a
// sequence is scaled by the same factor (the normaliser cancels between
// numerator and denominator), so sum_l g_l dL/dg_l = 0.
//
// Every reduction (dS, dz, dgamma, the tap gradients) runs in an order fixed
// by the shape, so the results are the same bits on every call.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gbla_device.h"
#include "gbla_ext.h"
#include "gbla_plan.h"
#include "gbla_rows.h"

namespace gbla {
namespace {

template <typename T>
__device__ __forceinline__ float act(const T* p, int64_t i);
template <>
__device__ __forceinline__ float act<float>(const float* p, int64_t i) { return p[i]; }
template <>
__device__ __forceinline__ float act<uint16_t>(const uint16_t* p, int64_t i) {
  return __uint_as_float((uint32_t)p[i] << 16);
}

__device__ __forceinline__ float phi_f(float u) { return u > 0.0f ? u + 1.0f : expf(u); }

// Gate logit i, or 0 without gate logits (the no-key-gating switch: uniform
// gates, the softmax of constant logits).
template <typename T>
__device__ __forceinline__ float logit(const T* a, int64_t i) { return a ? act<T>(a, i) : 0.0f; }
// Hardware-exp forms for the matrix-core kernels (a few ulp; the gradients
// are held to fp32-sum accuracy, far above that).
__device__ __forceinline__ float phi_fast(float u) {
  const float e = __expf(u);  // formed for every u, so that no branch is
  return u > 0.0f ? u + 1.0f : e;
}
__device__ __forceinline__ float sigmoid_fast(float x) {
  return __builtin_amdgcn_rcpf(1.0f + __expf(-x));
}
// x^(-1/2): the hardware's (1 ulp) with one Newton step.
__device__ __forceinline__ float rsqrt_nr(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  return fmaf(0.5f * r, fmaf(-x * r, r, 1.0f), r);
}
__device__ __forceinline__ float dphi_f(float u) { return u > 0.0f ? 1.0f : expf(u); }

constexpr int kBwdUnit = 512;  // tokens of the channel-layout kernels' units, at most

template <int D>
struct BW {
  static constexpr int kWaves = 4;
  static constexpr int kTok = 16;                      // tokens per wave per block
  static constexpr int kBlk = kWaves * kTok;           // tokens per block of the query pass
  static constexpr int kSP = D + 1;                    // padded LDS row stride of S / dS
  static constexpr int kCPL = D > 64 ? D / 64 : 1;     // channels per lane
  static constexpr int kRS = kThreads / D;             // dS row stride between a thread's elements
  static constexpr int kEl = D / kRS;                  // dS elements per thread
};

// Channel of slot cc of a lane (may be >= D for d = 32: the lane is idle).
template <int D>
__device__ __forceinline__ int chan(int lane, int cc) { return lane + 64 * cc; }

// ---------------------------------------------------------------------------
// State recomputed in fp32: grid (units, H); a unit is the forward's chunk of
// tokens.  Writes the record [S_p | z_p | m_p | l_p] of the chunk with
//   w_j = exp(a_j - m_p), m_p = max_j a_j, l_p = sum_j w_j,
//   S_p = sum_j w_j phi(kt_j) vt_j^T, z_p = sum_j w_j phi(kt_j),
// every product in fp32 (the forward's bf16 path rounds the gated keys to
// bf16 for its MFMAs; the gradients read S and z without that rounding).
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(kThreads)
bwd_state_kernel(Plan P, const T* __restrict__ kin, const T* __restrict__ vin,
                 const T* __restrict__ ain, const float* __restrict__ conv_w,
                 const int32_t* __restrict__ cu, float* __restrict__ partials) {
  using C = BW<D>;
  constexpr int CPL = C::kCPL, kEl = C::kEl;
  __shared__ float kb[C::kBlk][D];
  __shared__ float vb[C::kBlk][D];
  __shared__ float red[C::kWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, g = blockIdx.x;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, g, &s, &chunk)) return;
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int64_t t0 = (int64_t)chunk * P.chunk;
  const int64_t t1 = min(len, t0 + (int64_t)P.chunk);

  float ml = -INFINITY;
  for (int64_t j = t0 + tid; j < t1; j += kThreads) ml = fmaxf(ml, logit<T>(ain, base_row + j));
  const float m = block_max(ml, red);

  float wk[CPL][4], wv[CPL][4];
#pragma unroll
  for (int cc = 0; cc < CPL; ++cc) {
    const int e = min(chan<D>(lane, cc), D - 1);
    load_taps4(conv_w, P.heads, h, 1, D, P.W, e, wk[cc]);
    load_taps4(conv_w, P.heads, h, 2, D, P.W, e, wv[cc]);
  }
  const int ds_e = tid % D, ds_c0 = tid / D;
  float S_acc[kEl];
#pragma unroll
  for (int i = 0; i < kEl; ++i) S_acc[i] = 0.0f;
  float z_acc = 0.0f, l_acc = 0.0f;

  for (int64_t b0 = t0; b0 < t1; b0 += C::kBlk) {
    for (int k = 0; k < C::kTok; ++k) {
      const int slot = wave * C::kTok + k;
      const int64_t j = b0 + slot;
      const bool live = j < t1;  // wave-uniform
      const float w = live ? expf(logit<T>(ain, base_row + j) - m) : 0.0f;
      if (lane == 0) l_acc += w;
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int e = chan<D>(lane, cc);
        if (e < D) {
          float ka = 0.0f, va = 0.0f;
          if (live) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int64_t src = j - 3 + t;
              if (src >= 0) {
                ka = fmaf(wk[cc][t], act<T>(kin, (base_row + src) * D + e), ka);
                va = fmaf(wv[cc][t], act<T>(vin, (base_row + src) * D + e), va);
              }
            }
          }
          kb[slot][e] = w * phi_f(ka);
          vb[slot][e] = va;
        }
      }
    }
    __syncthreads();
    // S_p += sum over the block's tokens in token order; thread tid owns
    // column e = tid % D and rows c0 + kRS * i.
#pragma unroll 2
    for (int slot = 0; slot < C::kBlk; ++slot) {
      const float vv = vb[slot][ds_e];
#pragma unroll
      for (int i = 0; i < kEl; ++i) S_acc[i] = fmaf(kb[slot][ds_c0 + C::kRS * i], vv, S_acc[i]);
    }
    if (tid < D)
      for (int slot = 0; slot < C::kBlk; ++slot) z_acc += kb[slot][tid];
    __syncthreads();
  }

  float* rec = partials + ((size_t)h * P.units + g) * P.rec_floats;
#pragma unroll
  for (int i = 0; i < kEl; ++i) rec[(ds_c0 + C::kRS * i) * D + ds_e] = S_acc[i];
  if (tid < D) rec[D * D + tid] = z_acc;
  __syncthreads();  // every wave has read red in block_max (the loop may not run)
  if (lane == 0) red[wave] = l_acc;
  __syncthreads();
  if (tid == 0) {
    float l = 0.0f;
#pragma unroll
    for (int w = 0; w < C::kWaves; ++w) l += red[w];
    rec[D * D + D] = m;
    rec[D * D + D + 1] = l;
  }
}

// ---------------------------------------------------------------------------
// Query pass: grid (units, H).
// ---------------------------------------------------------------------------
template <typename T, int D, bool kNorm>
__global__ void __launch_bounds__(kThreads)
bwd_query_kernel(Plan P, const T* __restrict__ qin, const T* __restrict__ rin,
                 const float* __restrict__ dy, const float* __restrict__ conv_w,
                 const float* __restrict__ gamma, const int32_t* __restrict__ cu,
                 const float* __restrict__ Sg, const float* __restrict__ zg,
                 float* __restrict__ dqt, float* __restrict__ dr, float* __restrict__ dsp,
                 float* __restrict__ dgp) {
  using C = BW<D>;
  constexpr int CPL = C::kCPL, kEl = C::kEl;
  __shared__ float Ss[D * C::kSP];
  __shared__ float zs[D];
  __shared__ float qh_b[C::kBlk][D];
  __shared__ float dn_b[C::kBlk][D];
  __shared__ float dd_b[C::kBlk];
  __shared__ float red[C::kWaves][D];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, g = blockIdx.x;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, g, &s, &chunk)) return;
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int64_t t0 = (int64_t)chunk * P.chunk;
  const int64_t t1 = min(len, t0 + (int64_t)P.chunk);
  const size_t sh = (size_t)s * P.heads + h;
  for (int x = tid; x < D * D; x += kThreads) Ss[(x / D) * C::kSP + x % D] = Sg[sh * D * D + x];
  if (tid < D) zs[tid] = zg[sh * D + tid];

  float wq[CPL][4], gm[CPL], dg_acc[CPL];
#pragma unroll
  for (int cc = 0; cc < CPL; ++cc) {
    const int e = min(chan<D>(lane, cc), D - 1);
    load_taps4(conv_w, P.heads, h, 0, D, P.W, e, wq[cc]);
    gm[cc] = kNorm ? gamma[(size_t)h * D + e] : 1.0f;
    dg_acc[cc] = 0.0f;
  }
  const int ds_e = tid % D, ds_c0 = tid / D;
  float dS_acc[kEl];
#pragma unroll
  for (int m = 0; m < kEl; ++m) dS_acc[m] = 0.0f;
  float dz_acc = 0.0f;
  __syncthreads();

  for (int64_t b0 = t0; b0 < t1; b0 += C::kBlk) {
    for (int k = 0; k < C::kTok; ++k) {
      const int slot = wave * C::kTok + k;
      const int64_t i = b0 + slot;  // token of the sequence
      if (i >= t1) {                // wave-uniform: contributes nothing
#pragma unroll
        for (int cc = 0; cc < CPL; ++cc) {
          const int e = chan<D>(lane, cc);
          if (e < D) {
            qh_b[slot][e] = 0.0f;
            dn_b[slot][e] = 0.0f;
          }
        }
        if (lane == 0) dd_b[slot] = 0.0f;
        continue;
      }
      const int64_t row = base_row + i;
      float qt[CPL], qh[CPL];
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int e = chan<D>(lane, cc);
        float acc = 0.0f;
        if (e < D) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int64_t src = i - 3 + t;
            if (src >= 0) acc = fmaf(wq[cc][t], act<T>(qin, (base_row + src) * D + e), acc);
          }
          qh_b[slot][e] = phi_f(acc);
        }
        qt[cc] = acc;
        qh[cc] = phi_f(acc);
      }
      wave_lds_sync();
      // num and den (z dotted with Qh over the wave)
      float num[CPL], zd = 0.0f;
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int e = chan<D>(lane, cc);
        float acc = 0.0f;
        if (e < D) {
#pragma unroll 8
          for (int c = 0; c < D; ++c) acc = fmaf(qh_b[slot][c], Ss[c * C::kSP + e], acc);
          zd = fmaf(qh[cc], zs[e], zd);
        }
        num[cc] = acc;
      }
      const float den = wave_sum(zd);
      float o[CPL], ss = 0.0f;
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        o[cc] = num[cc] / den;
        if (chan<D>(lane, cc) < D) ss = fmaf(o[cc], o[cc], ss);
      }
      float dnum[CPL], dden;
      if constexpr (kNorm) {
        const float rs = 1.0f / sqrtf(wave_sum(ss) / D + P.eps);
        float doh[CPL], s1 = 0.0f;
#pragma unroll
        for (int cc = 0; cc < CPL; ++cc) {
          const int e = chan<D>(lane, cc);
          doh[cc] = 0.0f;
          if (e < D) {
            const float rv = act<T>(rin, row * D + e), dyv = dy[row * D + e];
            const float sig = 1.0f / (1.0f + expf(-rv)), silu = rv * sig;
            const float oh = o[cc] * rs;
            doh[cc] = dyv * gm[cc] * silu;
            dg_acc[cc] = fmaf(dyv * oh, silu, dg_acc[cc]);
            dr[row * D + e] = dyv * oh * gm[cc] * sig * (1.0f + rv * (1.0f - sig));
            s1 = fmaf(doh[cc], o[cc], s1);
          }
        }
        s1 = wave_sum(s1);
#pragma unroll
        for (int cc = 0; cc < CPL; ++cc) dnum[cc] = (rs * doh[cc] - rs * rs * rs / D * s1 * o[cc]) / den;
        // do . o = eps rs^3 s1 exactly (rs^-2 = |o|^2/d + eps); see the matrix-core kernel
        dden = -P.eps * rs * rs * rs * s1 / den;
      } else {  // y = o: do = dy
        float s2 = 0.0f;
#pragma unroll
        for (int cc = 0; cc < CPL; ++cc) {
          const int e = chan<D>(lane, cc);
          const float dyv = e < D ? dy[row * D + e] : 0.0f;
          dnum[cc] = dyv / den;
          s2 = fmaf(dyv, o[cc], s2);
        }
        dden = -wave_sum(s2) / den;
      }
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int e = chan<D>(lane, cc);
        if (e < D) dn_b[slot][e] = dnum[cc];
      }
      if (lane == 0) dd_b[slot] = dden;
      wave_lds_sync();
      // dQh[c] = sum_e S[c][e] dnum[e] + z[c] dden (lane owns c)
#pragma unroll
      for (int cc = 0; cc < CPL; ++cc) {
        const int c = chan<D>(lane, cc);
        if (c < D) {
          float acc = zs[c] * dden;
#pragma unroll 8
          for (int e = 0; e < D; ++e) acc = fmaf(Ss[c * C::kSP + e], dn_b[slot][e], acc);
          dqt[row * D + c] = acc * dphi_f(qt[cc]);
        }
      }
    }
    __syncthreads();
    // dS += sum over the block's tokens (in token order) of Qh_i dnum_i^T.
    // Thread tid owns column e = tid % D and rows c0 + kRS * m of dS.
#pragma unroll 2
    for (int slot = 0; slot < C::kBlk; ++slot) {
      const float dn = dn_b[slot][ds_e];
#pragma unroll
      for (int m = 0; m < kEl; ++m) dS_acc[m] = fmaf(qh_b[slot][ds_c0 + C::kRS * m], dn, dS_acc[m]);
    }
    if (tid < D)
      for (int slot = 0; slot < C::kBlk; ++slot) dz_acc = fmaf(qh_b[slot][tid], dd_b[slot], dz_acc);
    __syncthreads();
  }

  float* rec = dsp + ((size_t)h * P.units + g) * P.rec_floats;
#pragma unroll
  for (int m = 0; m < kEl; ++m) rec[(ds_c0 + C::kRS * m) * D + ds_e] = dS_acc[m];
  if (tid < D) rec[D * D + tid] = dz_acc;
  // dgamma partial of the unit: the four waves' sums in wave order
#pragma unroll
  for (int cc = 0; cc < CPL; ++cc) {
    const int e = chan<D>(lane, cc);
    if (e < D) red[wave][e] = dg_acc[cc];
  }
  __syncthreads();
  if (tid < D) {
    float acc = 0.0f;
#pragma unroll
    for (int w = 0; w < C::kWaves; ++w) acc += red[w][tid];
    dgp[((size_t)h * P.units + g) * D + tid] = acc;
  }
}

// ---------------------------------------------------------------------------
// dS, dz of each (sequence, head): the fixed-order sum of its units' partials.
// grid (N * H, element slices of kThreads).
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_dscombine_kernel(Plan P, const int32_t* __restrict__ cu, const float* __restrict__ dsp,
                     float* __restrict__ dS) {
  constexpr int kElems = D * D + D;
  const int sh_idx = blockIdx.x;
  const int s = sh_idx / P.heads, h = sh_idx % P.heads;
  int first, count;
  if (P.ragged) {
    first = units_before(cu, s, P.chunk);
    count = units_of((int64_t)cu[s + 1] - cu[s], P.chunk);
  } else {
    first = s * P.chunks_per_seq;
    count = P.chunks_per_seq;
  }
  const int x = blockIdx.y * kThreads + threadIdx.x;
  if (x >= kElems) return;
  const float* recs = dsp + ((size_t)h * P.units + first) * P.rec_floats + x;
  const size_t rf = P.rec_floats;
  // in unit order (compensated); eight loads in flight per group
  float acc = 0.0f, cmp = 0.0f;
  int p = 0;
  for (; p + 8 <= count; p += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = recs[(size_t)(p + i) * rf];
#pragma unroll
    for (int i = 0; i < 8; ++i) kahan_add(acc, cmp, v[i]);
  }
  for (; p < count; ++p) kahan_add(acc, cmp, recs[(size_t)p * rf]);
  dS[(size_t)sh_idx * kElems + x] = acc;
}

// ---------------------------------------------------------------------------
// Key pass: grid (units, H).
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(kThreads)
bwd_key_kernel(Plan P, const T* __restrict__ kin, const T* __restrict__ vin,
               const T* __restrict__ ain, const float* __restrict__ conv_w,
               const int32_t* __restrict__ cu, const float* __restrict__ dSg,
               const float* __restrict__ mz, float* __restrict__ dkt, float* __restrict__ dvt,
               float* __restrict__ da) {
  using C = BW<D>;
  constexpr int CPL = C::kCPL;
  __shared__ float dSs[D * C::kSP];
  __shared__ float dzs[D];
  __shared__ float vb[C::kWaves][D];
  __shared__ float pb[C::kWaves][D];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, g = blockIdx.x;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, g, &s, &chunk)) return;
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int64_t t0 = (int64_t)chunk * P.chunk;
  const int64_t t1 = min(len, t0 + (int64_t)P.chunk);
  const size_t sh = (size_t)s * P.heads + h;
  const float* dsrc = dSg + sh * (D * D + D);
  for (int x = tid; x < D * D; x += kThreads) dSs[(x / D) * C::kSP + x % D] = dsrc[x];
  if (tid < D) dzs[tid] = dsrc[D * D + tid];
  const float M = mz[2 * sh], Z = mz[2 * sh + 1];
  const float invZ = Z > 0.0f ? 1.0f / Z : 0.0f;
  float wk[CPL][4], wv[CPL][4];
#pragma unroll
  for (int cc = 0; cc < CPL; ++cc) {
    const int e = min(chan<D>(lane, cc), D - 1);
    load_taps4(conv_w, P.heads, h, 1, D, P.W, e, wk[cc]);
    load_taps4(conv_w, P.heads, h, 2, D, P.W, e, wv[cc]);
  }
  __syncthreads();

  for (int64_t j = t0 + wave; j < t1; j += C::kWaves) {
    const int64_t row = base_row + j;
    wave_lds_sync();  // the previous token's reads of vb, pb are done
    float kt[CPL], pv[CPL];
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const int e = chan<D>(lane, cc);
      float ka = 0.0f, va = 0.0f;
      if (e < D) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int64_t src = j - 3 + t;
          if (src >= 0) {
            ka = fmaf(wk[cc][t], act<T>(kin, (base_row + src) * D + e), ka);
            va = fmaf(wv[cc][t], act<T>(vin, (base_row + src) * D + e), va);
          }
        }
        vb[wave][e] = va;
        pb[wave][e] = phi_f(ka);
      }
      kt[cc] = ka;
      pv[cc] = phi_f(ka);
    }
    wave_lds_sync();
    const float alog = ain ? act<T>(ain, row) : 0.0f;
    const float gj = M == -INFINITY ? 0.0f : expf(alog - M) * invZ;
    // t[c] = sum_e dS[c][e] vt[e] + dz[c]; dkt = g t phi'(kt); dg = P . t
    float dgl = 0.0f;
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const int c = chan<D>(lane, cc);
      if (c < D) {
        float acc = dzs[c];
#pragma unroll 8
        for (int e = 0; e < D; ++e) acc = fmaf(dSs[c * C::kSP + e], vb[wave][e], acc);
        dkt[row * D + c] = gj * acc * dphi_f(kt[cc]);
        dgl = fmaf(pv[cc], acc, dgl);
      }
    }
    const float dg = wave_sum(dgl);
    if (da && lane == 0) da[row] = gj * dg;
    // dvt[e] = g sum_c dS[c][e] P[c]
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const int e = chan<D>(lane, cc);
      if (e < D) {
        float acc = 0.0f;
#pragma unroll 8
        for (int c = 0; c < D; ++c) acc = fmaf(dSs[c * C::kSP + e], pb[wave][c], acc);
        dvt[row * D + e] = gj * acc;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Conv1D backward: grid (units, H, 3 tensors).  Thread (grp, e) handles
// channel e of tokens t0 + grp, t0 + grp + kThreads / D, ...; the tap
// gradients of the unit are summed over the groups in group order.
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(kThreads)
bwd_conv_kernel(Plan P, const T* __restrict__ qin, const T* __restrict__ kin,
                const T* __restrict__ vin, const float* __restrict__ dxt_all,
                const float* __restrict__ conv_w, const int32_t* __restrict__ cu,
                float* __restrict__ dq, float* __restrict__ dk, float* __restrict__ dv,
                float* __restrict__ dcp, size_t act_elems) {
  constexpr int kG = kThreads / D;
  __shared__ float red[kG][D][4];
  const int tid = threadIdx.x, e = tid % D, grp = tid / D;
  const int h = blockIdx.y, g = blockIdx.x, tensor = blockIdx.z;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, g, &s, &chunk)) return;
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int64_t t0 = (int64_t)chunk * P.chunk;
  const int64_t t1 = min(len, t0 + (int64_t)P.chunk);
  const T* x = tensor == 0 ? qin : tensor == 1 ? kin : vin;
  float* out = tensor == 0 ? dq : tensor == 1 ? dk : dv;
  const float* dxt = dxt_all + (size_t)tensor * act_elems;
  float w4[4];
  load_taps4(conv_w, P.heads, h, tensor, D, P.W, e, w4);
  float dc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int64_t i = t0 + grp; i < t1; i += kG) {
    float acc = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t m = i + 3 - t;  // the output that tap t reads token i into
      if (m < len) acc = fmaf(w4[t], dxt[(base_row + m) * D + e], acc);
    }
    out[(base_row + i) * D + e] = acc;
    const float d0 = dxt[(base_row + i) * D + e];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t src = i - 3 + t;
      if (src >= 0) dc[t] = fmaf(d0, act<T>(x, (base_row + src) * D + e), dc[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) red[grp][e][t] = dc[t];
  __syncthreads();
  if (grp == 0) {
    float* rec = dcp + (((size_t)h * P.units + g) * 3 + tensor) * D * 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float acc = 0.0f;
      for (int gg = 0; gg < kG; ++gg) acc += red[gg][e][t];
      rec[e * 4 + t] = acc;
    }
  }
}

// ---------------------------------------------------------------------------
// dgamma and the tap gradients: per head, the fixed-order sum over the head's
// units (every sequence of the batch).  grid (H, slices of 64 outputs); the
// outputs of a head are dgamma[0 .. d) then the taps in [3, d, W] order.
// Wave w sums a quarter of the units in unit order; the four quarter sums
// are added in wave order.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void bwd_params(const Plan& P, const int32_t* __restrict__ cu,
                                           const float* __restrict__ dgp,
                                           const float* __restrict__ dcp,
                                           float* __restrict__ dgamma, float* __restrict__ dconv,
                                           int h, int slice) {
  __shared__ float red[4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int total = P.ragged ? units_before(cu, P.nseq, P.chunk) : P.chunks_per_seq * P.nseq;
  const int nout = D + (dconv ? 3 * D * P.W : 0);
  const int e = slice * 64 + lane;
  const bool live = e < nout;
  size_t off = 0, stride = 0;
  if (e < D) {
    off = (size_t)h * P.units * D + e;
    stride = D;
  } else if (live) {
    const int x = e - D, tensor = x / (D * P.W), rem = x % (D * P.W);
    const int c = rem / P.W, t4 = rem % P.W + (4 - P.W);  // right-aligned slot of the tap
    off = ((size_t)h * P.units * 3 + tensor) * D * 4 + c * 4 + t4;
    stride = (size_t)3 * D * 4;
  }
  const float* src = e < D ? dgp : dcp;
  const int u0 = (int)((int64_t)total * wave / 4), u1 = (int)((int64_t)total * (wave + 1) / 4);
  float acc = 0.0f, cmp = 0.0f;  // compensated: a quarter can hold thousands of units
  if (live) {
    int u = u0;
    for (; u + 8 <= u1; u += 8) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = src[off + (size_t)(u + i) * stride];
#pragma unroll
      for (int i = 0; i < 8; ++i) kahan_add(acc, cmp, v[i]);
    }
    for (; u < u1; ++u) kahan_add(acc, cmp, src[off + (size_t)u * stride]);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (tid < 64 && live) {
    const float sum = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
    if (e < D) {
      if (dgamma) dgamma[(size_t)h * D + e] = sum;
    } else {
      const int x = e - D, tensor = x / (D * P.W), rem = x % (D * P.W);
      dconv[((size_t)tensor * P.heads + h) * D * P.W + rem] = sum;
    }
  }
}
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_param_kernel(Plan P, const int32_t* __restrict__ cu, const float* __restrict__ dgp,
                 const float* __restrict__ dcp, float* __restrict__ dgamma,
                 float* __restrict__ dconv) {
  bwd_params<D>(P, cu, dgp, dcp, dgamma, dconv, blockIdx.x, blockIdx.y);
}

// ===========================================================================
// Channel-layout path (gbla_rows.h): every head dim, slices below 2^31 bytes.
//
// Every contraction runs on v_mfma_f32_16x16x4_f32: fp32 operands, exact
// products, fp32 accumulation, so the results carry fp32 rounding only (the
// gradients cancel strongly -- dQh = S dnum + z dden, t = dS vt + dz -- and
// a two-way bf16 split of the operands would show through that cancellation).
//
// The conv's transpose is fused into the two passes.  A wave walks its
// contiguous quarter of the unit from its last tile to its first, so the three
// later tokens that a tile's dx needs are at hand: the next lane group's rows,
// or, for the last group, the first rows of the tile done before (LDS).  At
// the wave's own end those rows belong to another wave or unit: its last three
// tokens' dx are stored without them, every wave leaves the gradients of its
// first three convolved tokens in an edge buffer, and bwd_finish_kernel adds
// the missing products.  A separate conv pass over dqt, dkt, dvt in memory
// cost 1,920 bytes a token and head at d = 64, 92 of 321 us at n = 32768.
//
// Measured (query + key + conv of the kernels that these replaced, against
// query + dsum + key): n = 32768, H = 8, d = 64 bf16 280 -> 165 us; 57,511
// packed tokens, H = 8, d = 128 bf16 1810 -> 1250 us.
// ===========================================================================

// Rows of the tile's dx: dx_m = sum_t w_t dxt_{m+3-t}, and the tap sums
// dw_t += dxt_i x_{i-3+t}.  d: dxt of the tile (channel layout), x: its
// windows; stage: the wave's LDS area; later: [3][D] floats
// of LDS, dxt of the three tokens after the tile on entry, of its first three
// tokens on return.  dx of token tile + 4 g + i is stored at out row off + i.
template <typename T, int D, typename Taps>
__device__ __forceinline__ void conv_back(const float (*d)[4], const Window<T, D>& x,
                                          const Taps& taps, float* stage, float* later,
                                          __amdgpu_buffer_rsrc_t out, uint32_t off, int lane,
                                          float (*dw)[4]) {
  using C = CL<D>;
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int k = 0; k < C::NV; ++k) {
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < 3; ++i) put_vec<D>(stage + (4 * g + i) * C::kPitch + C::V * n, d, k, i);
    wave_lds_sync();
    const float* src = g < 3 ? stage + 4 * (g + 1) * C::kPitch : later + k * 16 * C::V;
    const int pitch = g < 3 ? C::kPitch : D;
    float nx[3][C::V];
#pragma unroll
    for (int i = 0; i < 3; ++i) get_vec<D>(src + i * pitch + C::V * n, nx[i]);
    wave_lds_sync();
    if (g == 0) {
#pragma unroll
      for (int i = 0; i < 3; ++i) put_vec<D>(later + i * D + k * 16 * C::V + C::V * n, d, k, i);
    }
    float y[C::V][4];
#pragma unroll
    for (int j = 0; j < C::V; ++j) {
      const int b = k * C::V + j;
      const f32x4_t w = taps(b);
      const float dd[7] = {d[b][0], d[b][1], d[b][2], d[b][3], nx[0][j], nx[1][j], nx[2][j]};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float acc = w[3] * dd[i];
        acc = fmaf(w[2], dd[i + 1], acc);
        acc = fmaf(w[1], dd[i + 2], acc);
        y[j][i] = fmaf(w[0], dd[i + 3], acc);
#pragma unroll
        for (int t = 0; t < 4; ++t) dw[b][t] = fmaf(dd[i], x.x[i + t].at(b), dw[b][t]);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t o = off + (uint32_t)(i * D * 4 + k * 16 * C::V * 4);
      if constexpr (C::V == 4) {
        const f32x4_t v = {y[0][i], y[1][i], y[2][i], y[3][i]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), out, o, 0, 0);
      } else {
        const f32x2_t v = {y[0][i], y[1][i]};
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), out, o, 0, 0);
      }
    }
  }
}

// Writes a unit's tap-gradient partial [D][4] from the lanes' sums (every
// thread calls; red: 4 x D f32x4 of LDS).
template <int D>
__device__ __forceinline__ void sum_taps(const float (*dw)[4], f32x4_t (*red)[D], float* __restrict__ dst) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int b = 0; b < CL<D>::NMB; ++b) {
    f32x4_t s;
#pragma unroll
    for (int t = 0; t < 4; ++t) s[t] = sum_groups(dw[b][t]);
    if (g == 0) red[wave][slot_chan<D>(b, n)] = s;
  }
  __syncthreads();
  if (threadIdx.x < D) {
    const int x = threadIdx.x;
    *reinterpret_cast<f32x4_t*>(dst + 4 * x) = (red[0][x] + red[1][x]) + (red[2][x] + red[3][x]);
  }
  __syncthreads();
}

// Edge rows of the wave of a unit: dxt of the wave's first three tokens.
template <int D>
__device__ __forceinline__ size_t edge_off(const Plan& P, int tensor, int h, int unit, int wave) {
  return ((((size_t)tensor * P.heads + h) * P.units + unit) * 4 + wave) * (3 * D);
}
template <int D>
__device__ __forceinline__ void store_edge(const float* later, float* __restrict__ dst, int lane) {
  for (int x = lane; x < 3 * D; x += 64) dst[x] = later[x];
}

// ---------------------------------------------------------------------------
// Query pass: grid (units, H).
// ---------------------------------------------------------------------------
// kDS: the unit's dS partial is summed here (d <= 64).  At d = 128 its 256
// accumulators leave too few registers for the rest (the compiler then moved
// and spilled some 900 of them a tile: 1207 us against 677 for this and
// bwd_dsum_rows_kernel together, 16 sequences of 57,511 tokens, H = 8), so this
// kernel writes dnum (to dnum_out, in the layout of dy) for that one.
template <typename T, int D, bool kNorm, bool kDS>
__global__ void __launch_bounds__(kThreads, D >= 128 ? 1 : 2)
bwd_query_rows_kernel(Plan P, const T* __restrict__ qin, const T* __restrict__ rin,
                      const float* __restrict__ dy, const float* __restrict__ conv_w,
                      const float* __restrict__ gamma, const int32_t* __restrict__ cu,
                      const float* __restrict__ Sg, const float* __restrict__ zg,
                      float* __restrict__ dq, float* __restrict__ dr, float* __restrict__ dsp,
                      float* __restrict__ dgp, float* __restrict__ dcp, float* __restrict__ edge,
                      float* __restrict__ dnum_out) {
  using C = CL<D>;
  constexpr int NMB = C::NMB;
  __shared__ f32x4_t f1[C::kFrag];  // num: B[c][e] = S[c][e]; later the waves' sums
  __shared__ f32x4_t f2[C::kFrag];  // dQh: B[e][c] = S'[c][e]
  __shared__ __attribute__((aligned(16))) float stg[4][C::kStage];
  __shared__ __attribute__((aligned(16))) float later[4][3 * D];
  __shared__ f32x4_t tq[D];
  __shared__ __attribute__((aligned(16))) float zs[D], gs[D], ms[D];  // by channel
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, unit = blockIdx.x;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, unit, &s, &chunk)) return;
  s = __builtin_amdgcn_readfirstlane(s);
  chunk = __builtin_amdgcn_readfirstlane(chunk);
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int t0 = chunk * P.chunk;
  const int t1 = (int)min(len, (int64_t)t0 + P.chunk);
  const uint32_t rows = (uint32_t)len * D;
  const __amdgpu_buffer_rsrc_t rq = make_rsrc(qin + base_row * D, rows * sizeof(T));
  // without the gated norm r is not read (an empty range) and dr not written
  const __amdgpu_buffer_rsrc_t rr =
      kNorm ? make_rsrc(rin + base_row * D, rows * sizeof(T)) : make_rsrc(qin, 0u);
  const __amdgpu_buffer_rsrc_t rdy = make_rsrc(dy + base_row * D, rows * 4u);
  const __amdgpu_buffer_rsrc_t rdq = make_rsrc(dq + base_row * D, rows * 4u);
  const __amdgpu_buffer_rsrc_t rdr =
      kNorm ? make_rsrc(dr + base_row * D, rows * 4u) : make_rsrc(dq, 0u);
  const __amdgpu_buffer_rsrc_t rdn =
      kDS ? make_rsrc(dq, 0u) : make_rsrc(dnum_out + base_row * D, rows * 4u);
  // the wave's quarter of the unit, in whole tiles
  const int q4 = quarter_tokens(t1 - t0);
  const int w0 = t0 + wave * q4, w1 = min(t1, w0 + q4);
  int b0 = w0 + (w1 > w0 ? (w1 - w0 - 1) / 16 * 16 : 0);  // the wave's last tile
  Window<T, D> nq;
  nq.load(rq, b0 + 4 * g, n);

  const size_t sh = (size_t)s * P.heads + h;
  const float* S = Sg + sh * D * D;
  Frags<D> fa, fb;
  fb.load_transposed(S);  // S[c][e .. e + 3]
  fa.load(S);
  stage_taps<D>(conv_w, P.heads, h, 0, P.W, tq);
  if (tid < D) {
    zs[tid] = zg[sh * D + tid];
    gs[tid] = kNorm ? gamma[(size_t)h * D + tid] : 1.0f;
  }
  for (int x = lane; x < 3 * D; x += 64) later[wave][x] = 0.0f;
  // dQh = S dnum + z dden is formed as S' dnum + z (dden + m . dnum) with
  // S' = S - z m^T, m = (sum_c S[c][.]) / (sum_c z[c]) (the gate-weighted
  // mean value row): the same quantity, but without the cancellation between
  // the two terms when the value rows share a mean (then S dnum ~ z (m . dnum)
  // and o ~ m, and the no-norm dden + m . dnum is formed as
  // -((o - m) . dy) / den directly).
  // Column sums of S from fb: a wave's vectors have the K blocks kq = wave +
  // 4 j alone (d = 32: waves w and w + 2 share block w); sixteen lanes of a
  // vector hold the block's columns c.
  constexpr int kQ = NMB > 4 ? NMB / 4 : 1, kShare = NMB < 4 ? 4 / NMB : 1;
  float* part = &stg[0][0];  // [kShare][D]
#pragma unroll
  for (int j = 0; j < kQ; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float cs = 0.0f;
#pragma unroll
      for (int u = j; u < Frags<D>::kPer; u += kQ) cs += fb.v[u][i];
      cs = sum_row16(cs);
      if (n == 0) part[(wave / NMB) * D + fb.k0(j) + i] = cs;
    }
  __syncthreads();
  if (tid < D) {
    float cs = part[tid], zsum = 0.0f;
    if constexpr (kShare == 2) cs += part[D + tid];
    for (int c = 0; c < D; ++c) zsum += zs[c];
    ms[tid] = zsum > 0.0f ? cs / zsum : 0.0f;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < Frags<D>::kPer; ++u) {
    const float z = zs[fb.col(u)];
    const f32x4_t m = *reinterpret_cast<const f32x4_t*>(&ms[fb.k0(u)]);
#pragma unroll
    for (int i = 0; i < 4; ++i) fb.v[u][i] = fmaf(-z, m[i], fb.v[u][i]);
  }
  fa.put(f1);
  fb.put(f2);
  f32x4_t acc3[kDS ? C::kBlocks : 1];
#pragma unroll
  for (int k = 0; k < (kDS ? C::kBlocks : 1); ++k) acc3[k] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  float dzacc[NMB], dgacc[NMB], dw[NMB][4];
#pragma unroll
  for (int b = 0; b < NMB; ++b) {
    dzacc[b] = dgacc[b] = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) dw[b][t] = 0.0f;
  }
  __syncthreads();

  for (; b0 >= w0 && w1 > w0; b0 -= 16) {
    float qh[NMB][4], o[NMB][4], dn[NMB][4];
    // operands and taps are re-read from LDS each tile, not held in registers
    __asm__ volatile("" ::: "memory");
    const Window<T, D> xq = nq;
    const int tb = b0 + 4 * g;
    Row<T, D> rw[4];
    Row<float, D> dyw[4];
    if constexpr (kNorm) {
#pragma unroll
      for (int i = 0; i < 4; ++i) rw[i].load(rr, row_off<T, D>(tb, n) + (uint32_t)(i * D * sizeof(T)));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) dyw[i].load(rdy, row_off<float, D>(tb, n) + (uint32_t)(i * D * 4));
    xq.conv(LdsTaps<D>{tq, n}, qh);
    nq.load(rq, b0 - 16 + 4 * g, n);  // the tile before (before the slice: reads 0, unused)
    float den[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int b = 0; b < NMB; ++b) {
      const float z = zs[slot_chan<D>(b, n)];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        qh[b][i] = phi_fast(qh[b][i]);
        den[i] = fmaf(qh[b][i], z, den[i]);
      }
    }
    // num = S^T Qh, den = z . Qh
    {
      f32x4_t acc[NMB];
#pragma unroll
      for (int b = 0; b < NMB; ++b) acc[b] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
      contract_rows<D>(qh, stg[wave], f1, lane, acc);
#pragma unroll
      for (int b = 0; b < NMB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[b][i] = acc[b][i];
    }
    float dden[4], dcen[4];  // dcen = dden + m . dnum
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float inv_den = 1.0f / sum_row16(den[i]);
      float ss = 0.0f;
#pragma unroll
      for (int b = 0; b < NMB; ++b) {
        o[b][i] *= inv_den;
        ss = fmaf(o[b][i], o[b][i], ss);
      }
      if constexpr (kNorm) {
        const float rs = rsqrt_nr(sum_row16(ss) * (1.0f / D) + P.eps);
        float s1 = 0.0f, drv[NMB][4];
#pragma unroll
        for (int b = 0; b < NMB; ++b) {
          const float r = rw[i].at(b), d = dyw[i].at(b), gm = gs[slot_chan<D>(b, n)];
          const float sig = sigmoid_fast(r), silu = r * sig;
          const float dyoh = d * (o[b][i] * rs);
          dn[b][i] = d * gm * silu;  // doh
          dgacc[b] = fmaf(dyoh, silu, dgacc[b]);
          drv[b][0] = dyoh * gm * sig * (1.0f + r * (1.0f - sig));
          s1 = fmaf(dn[b][i], o[b][i], s1);
        }
        store_row<D>(rdr, row_off<float, D>(tb, n) + (uint32_t)(i * D * 4), drv, 0);
        s1 = sum_row16(s1);
        const float c3 = rs * rs * rs / D * s1;
        // do . o = rs s1 (1 - rs^2 |o|^2 / d) = eps rs^3 s1 exactly (rs^-2 = |o|^2/d + eps):
        // the RMSNorm leaves almost nothing along o, and summing do . o would
        // return mostly the rounding of its terms.
        dden[i] = -P.eps * rs * rs * rs * s1 * inv_den;
        float md = 0.0f;
#pragma unroll
        for (int b = 0; b < NMB; ++b) {
          dn[b][i] = (rs * dn[b][i] - c3 * o[b][i]) * inv_den;
          md = fmaf(ms[slot_chan<D>(b, n)], dn[b][i], md);
        }
        dcen[i] = dden[i] + sum_row16(md);
      } else {  // y = o: do = dy
        float s2 = 0.0f, s2c = 0.0f;
#pragma unroll
        for (int b = 0; b < NMB; ++b) {
          const float d = dyw[i].at(b);
          dn[b][i] = d * inv_den;
          s2 = fmaf(d, o[b][i], s2);
          s2c = fmaf(d, o[b][i] - ms[slot_chan<D>(b, n)], s2c);
        }
        dden[i] = -sum_row16(s2) * inv_den;
        dcen[i] = -sum_row16(s2c) * inv_den;
      }
    }
    // dS += Qh dnum^T; dQh = S' dnum + z (dden + m . dnum)
    if constexpr (kDS) {
      token_product<D>(qh, dn, acc3);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        store_row<D>(rdn, row_off<float, D>(tb, n) + (uint32_t)(i * D * 4), dn, i);
    }
    {
      f32x4_t acc[NMB];
#pragma unroll
      for (int b = 0; b < NMB; ++b) acc[b] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
      contract_rows<D>(dn, stg[wave], f2, lane, acc);
#pragma unroll
      for (int b = 0; b < NMB; ++b) {
        const float z = zs[slot_chan<D>(b, n)];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // phi'(u) = 1 for u > 0 and e^u = phi(u) <= 1 otherwise: min(phi(u), 1)
          o[b][i] = fmaf(z, dcen[i], acc[b][i]) * fminf(qh[b][i], 1.0f);
          dzacc[b] = fmaf(qh[b][i], dden[i], dzacc[b]);
        }
      }
    }
    conv_back<T, D>(o, xq, LdsTaps<D>{tq, n}, stg[wave], later[wave], rdq, row_off<float, D>(tb, n), lane, dw);
  }

  wave_lds_sync();
  store_edge<D>(later[wave], edge + edge_off<D>(P, 0, h, unit, wave), lane);
  const size_t ui = (size_t)h * P.units + unit;
  float* rec = dsp + ui * P.rec_floats;
  __syncthreads();  // every wave is done with the operands
  static_assert(2 * sizeof(f1) >= 2 * D * D * sizeof(float), "f1, f2 hold the waves' sums");
  if constexpr (kDS) {
    sum_waves<D>(acc3, reinterpret_cast<float*>(f1), reinterpret_cast<float*>(f2), rec);
    __syncthreads();
  }
  sum_channels<D>(dzacc, reinterpret_cast<float(*)[D]>(f1), rec + D * D);
  sum_channels<D>(dgacc, reinterpret_cast<float(*)[D]>(f1), dgp + ui * D);
  sum_taps<D>(dw, reinterpret_cast<f32x4_t(*)[D]>(f1), dcp + (ui * 3 + 0) * D * 4);
}

// ---------------------------------------------------------------------------
// dS of a unit from the query pass's dnum (d = 128): dS_p = sum_i Qh_i dnum_i^T
// with Qh formed as the query pass forms it.  Writes the S part of the unit's
// record; the query pass wrote its dz part.
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(kThreads, D >= 128 ? 1 : 2)
bwd_dsum_rows_kernel(Plan P, const T* __restrict__ qin, const float* __restrict__ dnum,
                     const float* __restrict__ conv_w, const int32_t* __restrict__ cu,
                     float* __restrict__ dsp) {
  using C = CL<D>;
  constexpr int NMB = C::NMB;
  __shared__ __attribute__((aligned(16))) float buf[2 * D * D];  // the waves' sums
  __shared__ f32x4_t tq[D];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, unit = blockIdx.x;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, unit, &s, &chunk)) return;
  s = __builtin_amdgcn_readfirstlane(s);
  chunk = __builtin_amdgcn_readfirstlane(chunk);
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int t0 = chunk * P.chunk;
  const int t1 = (int)min(len, (int64_t)t0 + P.chunk);
  const uint32_t rows = (uint32_t)len * D;
  const __amdgpu_buffer_rsrc_t rq = make_rsrc(qin + base_row * D, rows * sizeof(T));
  // dnum past the unit's end reads 0
  const __amdgpu_buffer_rsrc_t rdn = make_rsrc(dnum + base_row * D, (uint32_t)t1 * (uint32_t)(D * 4));
  const int q4 = quarter_tokens(t1 - t0);
  const int w0 = t0 + wave * q4, w1 = min(t1, w0 + q4);
  Window<T, D> nq;
  Row<float, D> nd[4];
  auto issue = [&](int b0) {
    nq.load(rq, b0 + 4 * g, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) nd[i].load(rdn, row_off<float, D>(b0 + 4 * g, n) + (uint32_t)(i * D * 4));
  };
  issue(w0);
  stage_taps<D>(conv_w, P.heads, h, 0, P.W, tq);
  f32x4_t acc[C::kBlocks];
#pragma unroll
  for (int k = 0; k < C::kBlocks; ++k) acc[k] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  __syncthreads();
  for (int b0 = w0; b0 < w1; b0 += 16) {
    float qh[NMB][4], dn[NMB][4];
    __asm__ volatile("" ::: "memory");  // taps are re-read from LDS, not held
    nq.conv(LdsTaps<D>{tq, n}, qh);
#pragma unroll
    for (int b = 0; b < NMB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        qh[b][i] = phi_fast(qh[b][i]);
        dn[b][i] = nd[i].at(b);
      }
    issue(b0 + 16);
    token_product<D>(qh, dn, acc);
  }
  sum_waves<D>(acc, buf, buf + D * D, dsp + ((size_t)h * P.units + unit) * P.rec_floats);
}

// ---------------------------------------------------------------------------
// Key pass: grid (units, H).
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(kThreads, D >= 128 ? 1 : 2)
bwd_key_rows_kernel(Plan P, const T* __restrict__ kin, const T* __restrict__ vin,
                    const T* __restrict__ ain, const float* __restrict__ conv_w,
                    const int32_t* __restrict__ cu, const float* __restrict__ dSg,
                    const float* __restrict__ mz, float* __restrict__ dk, float* __restrict__ dv,
                    float* __restrict__ da, float* __restrict__ dcp, float* __restrict__ edge) {
  using C = CL<D>;
  constexpr int NMB = C::NMB;
  __shared__ f32x4_t f1[C::kFrag];  // t = dS vt: B[e][c] = dS[c][e]
  __shared__ f32x4_t f2[C::kFrag];  // dvt = dS^T P: B[c][e] = dS[c][e]
  __shared__ __attribute__((aligned(16))) float stg[4][C::kStage];
  __shared__ __attribute__((aligned(16))) float later[4][2][3 * D];  // dkt, dvt
  // gates of the unit's tokens, zero past the sequence end
  __shared__ __attribute__((aligned(16))) float gt[kBwdUnit];
  __shared__ float dzs[D];
  constexpr bool kRegTaps = D >= 128;  // the operand layouts fill the LDS
  __shared__ f32x4_t tk[kRegTaps ? 1 : D], tv[kRegTaps ? 1 : D];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, unit = blockIdx.x;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, unit, &s, &chunk)) return;
  s = __builtin_amdgcn_readfirstlane(s);
  chunk = __builtin_amdgcn_readfirstlane(chunk);
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int t0 = chunk * P.chunk;
  const int t1 = (int)min(len, (int64_t)t0 + P.chunk);
  const uint32_t rows = (uint32_t)len * D;
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(kin + base_row * D, rows * sizeof(T));
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(vin + base_row * D, rows * sizeof(T));
  const __amdgpu_buffer_rsrc_t rdk = make_rsrc(dk + base_row * D, rows * 4u);
  const __amdgpu_buffer_rsrc_t rdv = make_rsrc(dv + base_row * D, rows * 4u);
  // an absent da is not written (an empty range)
  const __amdgpu_buffer_rsrc_t rda =
      da ? make_rsrc(da + base_row, (uint32_t)t1 * 4u) : make_rsrc(dk, 0u);
  const int q4 = quarter_tokens(t1 - t0);
  const int w0 = t0 + wave * q4, w1 = min(t1, w0 + q4);
  int b0 = w0 + (w1 > w0 ? (w1 - w0 - 1) / 16 * 16 : 0);  // the wave's last tile
  Window<T, D> nk, nv;
  nk.load(rk, b0 + 4 * g, n);
  nv.load(rv, b0 + 4 * g, n);

  const size_t sh = (size_t)s * P.heads + h;
  const float* dS = dSg + sh * (D * D + D);
  Frags<D> fa, fb;
  fa.load_transposed(dS);
  fb.load(dS);
  using Taps = typename std::conditional<kRegTaps, RegTaps<D>, LdsTaps<D>>::type;
  Taps wk, wv;
  if constexpr (kRegTaps) {
    wk.load(conv_w, P.heads, h, 1, P.W, n);
    wv.load(conv_w, P.heads, h, 2, P.W, n);
  } else {
    stage_taps<D>(conv_w, P.heads, h, 1, P.W, tk);
    stage_taps<D>(conv_w, P.heads, h, 2, P.W, tv);
    wk = LdsTaps<D>{tk, n};
    wv = LdsTaps<D>{tv, n};
  }
  if (tid < D) dzs[tid] = dS[D * D + tid];
  const float M = mz[2 * sh], Z = mz[2 * sh + 1];
  const float invZ = Z > 0.0f ? 1.0f / Z : 0.0f;
  for (int j = tid; j < 4 * q4; j += kThreads)
    gt[j] = j < t1 - t0 ? __expf(logit<T>(ain, base_row + t0 + j) - M) * invZ : 0.0f;
  for (int x = lane; x < 6 * D; x += 64) (&later[wave][0][0])[x] = 0.0f;
  fa.put(f1);
  fb.put(f2);
  float dwk[NMB][4], dwv[NMB][4];
#pragma unroll
  for (int b = 0; b < NMB; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) dwk[b][t] = dwv[b][t] = 0.0f;
  __syncthreads();

  for (; b0 >= w0 && w1 > w0; b0 -= 16) {
    float pk[NMB][4], x[NMB][4];
    __asm__ volatile("" ::: "memory");  // operands and taps are re-read from LDS
    const Window<T, D> xk = nk, xv = nv;
    const uint32_t off = row_off<float, D>(b0 + 4 * g, n);
    xk.conv(wk, pk);
    xv.conv(wv, x);
    nk.load(rk, b0 - 16 + 4 * g, n);  // the tile before (before the slice: reads 0, unused)
    nv.load(rv, b0 - 16 + 4 * g, n);
    const f32x4_t gj = *reinterpret_cast<const f32x4_t*>(&gt[b0 - t0 + 4 * g]);
    // t = dS vt + dz; dkt = g t phi'(kt); da = g (P . t)
    {
      f32x4_t acc[NMB];
#pragma unroll
      for (int b = 0; b < NMB; ++b) acc[b] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
      contract_rows<D>(x, stg[wave], f1, lane, acc);
      float dgl[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int b = 0; b < NMB; ++b) {
        const float dz = dzs[slot_chan<D>(b, n)];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = phi_fast(pk[b][i]), t = acc[b][i] + dz;
          pk[b][i] = p;
          x[b][i] = gj[i] * t * fminf(p, 1.0f);  // phi'(u) = min(phi(u), 1)
          dgl[i] = fmaf(p, t, dgl[i]);
        }
      }
      float dg = 0.0f;  // lane n < 4 writes token 4 g + n
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = gj[i] * sum_row16(dgl[i]);
        dg = n == i ? v : dg;
      }
      if (n < 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, dg), rda,
                                              (uint32_t)(b0 + 4 * g + n) * 4u, 0, 0);
    }
    conv_back<T, D>(x, xk, wk, stg[wave], later[wave][0], rdk, off, lane, dwk);
    // dvt = g dS^T P
    {
      f32x4_t acc[NMB];
#pragma unroll
      for (int b = 0; b < NMB; ++b) acc[b] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
      contract_rows<D>(pk, stg[wave], f2, lane, acc);
#pragma unroll
      for (int b = 0; b < NMB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[b][i] = gj[i] * acc[b][i];
    }
    conv_back<T, D>(x, xv, wv, stg[wave], later[wave][1], rdv, off, lane, dwv);
  }

  wave_lds_sync();
  store_edge<D>(later[wave][0], edge + edge_off<D>(P, 1, h, unit, wave), lane);
  store_edge<D>(later[wave][1], edge + edge_off<D>(P, 2, h, unit, wave), lane);
  const size_t ui = (size_t)h * P.units + unit;
  __syncthreads();  // every wave is done with the operands
  sum_taps<D>(dwk, reinterpret_cast<f32x4_t(*)[D]>(f1), dcp + (ui * 3 + 1) * D * 4);
  sum_taps<D>(dwv, reinterpret_cast<f32x4_t(*)[D]>(f1), dcp + (ui * 3 + 2) * D * 4);
}

// ---------------------------------------------------------------------------
// What the two passes leave: block (unit, h) of the first P.units adds the
// missing products to dx of the three tokens before each wave's first token,
//   dx_{p-3+j} += sum_{t <= j} w_t dxt_{p+j-t},  p > 0 the wave's first token,
// the remaining blocks sum dgamma and the taps (bwd_params).
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_finish_kernel(Plan P, const int32_t* __restrict__ cu, const float* __restrict__ conv_w,
                  const float* __restrict__ edge, const float* __restrict__ dgp,
                  const float* __restrict__ dcp, float* __restrict__ dq, float* __restrict__ dk,
                  float* __restrict__ dv, float* __restrict__ dgamma, float* __restrict__ dconv) {
  const int h = blockIdx.y, tid = threadIdx.x;
  if ((int)blockIdx.x >= P.units) {
    bwd_params<D>(P, cu, dgp, dcp, dgamma, dconv, h, blockIdx.x - P.units);
    return;
  }
  const int unit = blockIdx.x;
  int s, chunk;
  if (!unit_of(P, cu, P.chunk, P.chunks_per_seq, unit, &s, &chunk)) return;
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int t0 = chunk * P.chunk;
  const int t1 = (int)min(len, (int64_t)t0 + P.chunk);
  const int q4 = quarter_tokens(t1 - t0);
  for (int x = tid; x < 3 * 4 * D; x += kThreads) {  // (tensor, wave, channel)
    const int c = x % D, wave = (x / D) & 3, tensor = x / (4 * D);
    const int p = t0 + wave * q4;
    if (p == 0 || p >= t1) continue;
    float w4[4], d[3];
    load_taps4(conv_w, P.heads, h, tensor, D, P.W, c, w4);
    const float* e = edge + edge_off<D>(P, tensor, h, unit, wave) + c;
#pragma unroll
    for (int j = 0; j < 3; ++j) d[j] = e[j * D];
    float* out = (tensor == 0 ? dq : tensor == 1 ? dk : dv) + (base_row + p - 3) * D + c;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      float acc = out[j * D];
#pragma unroll
      for (int t = 0; t <= j; ++t) acc = fmaf(w4[t], d[j - t], acc);
      out[j * D] = acc;
    }
  }
}

template <typename T, int D>
gbla_status run_backward(const Plan& p, const BwdLayout& L, const void* q, const void* k,
                         const void* v, const void* a, const void* r, const float* conv_w,
                         const float* gamma, const int32_t* cu, const float* dy, void* ws,
                         float* dq, float* dk, float* dv, float* da, float* dr, float* dconv,
                         float* dgamma, hipStream_t st) {
  unsigned char* base = static_cast<unsigned char*>(ws);
  float* S = reinterpret_cast<float*>(base + L.off_S);
  float* z = reinterpret_cast<float*>(base + L.off_z);
  float* mz = reinterpret_cast<float*>(base + L.off_mz);
  float* dsp = reinterpret_cast<float*>(base + L.off_dsp);
  float* dS = reinterpret_cast<float*>(base + L.off_dS);
  float* dgp = reinterpret_cast<float*>(base + L.off_dgp);
  float* dcp = reinterpret_cast<float*>(base + L.off_dcp);
  float* edge = reinterpret_cast<float*>(base + L.off_edge);
  const dim3 grid(p.units, p.heads);
  constexpr int kElems = D * D + D;
  const dim3 cgrid((unsigned)((int64_t)p.nseq * p.heads), (kElems + kThreads - 1) / kThreads);
  const int nparam = (D + 3 * D * p.W + 63) / 64;  // slices of bwd_params
  const T *qq = (const T*)q, *kk = (const T*)k, *vv = (const T*)v, *aa = (const T*)a, *rr = (const T*)r;
  if (rows_supported(p)) {
    gbla_status e = launch_state_rows(p, k, v, a, conv_w, cu, dsp, false, st);
    if (e != GBLA_OK) return e;
    e = launch_combine_f32(p, cu, dsp, S, z, mz, st);
    if (e != GBLA_OK) return e;
    // d = 128: the query pass leaves dnum in dv, which the key pass fills only
    // after bwd_dsum_rows_kernel has read it
    constexpr bool kDS = D <= 64;
    if (gamma)
      hipLaunchKernelGGL((bwd_query_rows_kernel<T, D, true, kDS>), grid, dim3(kThreads), 0, st, p, qq,
                         rr, dy, conv_w, gamma, cu, S, z, dq, dr, dsp, dgp, dcp, edge, dv);
    else
      hipLaunchKernelGGL((bwd_query_rows_kernel<T, D, false, kDS>), grid, dim3(kThreads), 0, st, p, qq,
                         rr, dy, conv_w, gamma, cu, S, z, dq, dr, dsp, dgp, dcp, edge, dv);
    if constexpr (!kDS)
      hipLaunchKernelGGL((bwd_dsum_rows_kernel<T, D>), grid, dim3(kThreads), 0, st, p, qq,
                         (const float*)dv, conv_w, cu, dsp);
    hipLaunchKernelGGL((bwd_dscombine_kernel<D>), cgrid, dim3(kThreads), 0, st, p, cu,
                       (const float*)dsp, dS);
    hipLaunchKernelGGL((bwd_key_rows_kernel<T, D>), grid, dim3(kThreads), 0, st, p, kk, vv, aa, conv_w,
                       cu, (const float*)dS, (const float*)mz, dk, dv, da, dcp, edge);
    hipLaunchKernelGGL((bwd_finish_kernel<D>), dim3(p.units + nparam, p.heads), dim3(kThreads), 0, st,
                       p, cu, conv_w, (const float*)edge, (const float*)dgp, (const float*)dcp, dq, dk,
                       dv, dgamma, dconv);
    return hipGetLastError() == hipSuccess ? GBLA_OK : GBLA_ERR_HIP;
  }
  // slices of 2^31 bytes and more: vector kernels with 64-bit indexing
  float* dxt = reinterpret_cast<float*>(base + L.off_dxt);
  const size_t act_elems = (size_t)p.tokens * p.heads * D;
  hipLaunchKernelGGL((bwd_state_kernel<T, D>), grid, dim3(kThreads), 0, st, p, kk, vv, aa, conv_w, cu, dsp);
  gbla_status e = launch_combine_f32(p, cu, dsp, S, z, mz, st);
  if (e != GBLA_OK) return e;
  if (gamma)
    hipLaunchKernelGGL((bwd_query_kernel<T, D, true>), grid, dim3(kThreads), 0, st, p, qq, rr, dy,
                       conv_w, gamma, cu, S, z, dxt, dr, dsp, dgp);
  else
    hipLaunchKernelGGL((bwd_query_kernel<T, D, false>), grid, dim3(kThreads), 0, st, p, qq, rr, dy,
                       conv_w, gamma, cu, S, z, dxt, dr, dsp, dgp);
  hipLaunchKernelGGL((bwd_dscombine_kernel<D>), cgrid, dim3(kThreads), 0, st, p, cu,
                     (const float*)dsp, dS);
  hipLaunchKernelGGL((bwd_key_kernel<T, D>), grid, dim3(kThreads), 0, st, p, kk, vv, aa, conv_w, cu,
                     (const float*)dS, (const float*)mz, dxt + act_elems, dxt + 2 * act_elems, da);
  hipLaunchKernelGGL((bwd_conv_kernel<T, D>), dim3(p.units, p.heads, 3), dim3(kThreads), 0, st, p, qq,
                     kk, vv, (const float*)dxt, conv_w, cu, dq, dk, dv, dcp, act_elems);
  hipLaunchKernelGGL((bwd_param_kernel<D>), dim3(p.heads, nparam), dim3(kThreads), 0, st, p, cu,
                     (const float*)dgp, (const float*)dcp, dgamma, dconv);
  return hipGetLastError() == hipSuccess ? GBLA_OK : GBLA_ERR_HIP;
}

}  // namespace

gbla_status launch_backward(const Plan& p, const BwdLayout& L, const void* q, const void* k,
                            const void* v, const void* a, const void* r, const float* conv_w,
                            const float* gamma, const int32_t* cu, const float* dy, void* ws,
                            float* dq, float* dk, float* dv, float* da, float* dr, float* dconv,
                            float* dgamma, hipStream_t st) {
#define GBLA_BWD(TT, DD)                                                                      \
  return run_backward<TT, DD>(p, L, q, k, v, a, r, conv_w, gamma, cu, dy, ws, dq, dk, dv, da, \
                              dr, dconv, dgamma, st)
  if (p.dtype == GBLA_BF16) {
    if (p.d == 32) GBLA_BWD(uint16_t, 32);
    if (p.d == 64) GBLA_BWD(uint16_t, 64);
    if (p.d == 128) GBLA_BWD(uint16_t, 128);
  } else {
    if (p.d == 32) GBLA_BWD(float, 32);
    if (p.d == 64) GBLA_BWD(float, 64);
    if (p.d == 128) GBLA_BWD(float, 128);
  }
#undef GBLA_BWD
  return GBLA_ERR_UNSUPPORTED;
}

}  // namespace gbla
