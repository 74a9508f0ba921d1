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
#include "gbla_split.h"

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

// Sum over the four lane groups (the lanes n, n + 16, n + 32, n + 48).
__device__ __forceinline__ float sum_groups(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
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
// x^(-1/2): the hardware's (1 ulp) with one Newton step, which has no value at
// 0 and infinity (a square sum that overflowed): there the hardware's inf and 0.
__device__ __forceinline__ float rsqrt_nr(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  const float e = fmaf(-x * r, r, 1.0f);
  return e == e ? fmaf(0.5f * r, e, r) : r;
}
__device__ __forceinline__ float dphi_f(float u) { return u > 0.0f ? 1.0f : expf(u); }

constexpr int kBwdUnit = 512;  // tokens of the split-product kernels' units, at most

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
      wave_fence();
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
      wave_fence();
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
  float acc = 0.0f, cmp = 0.0f;
  sum_records(count, [&](int p) { return recs[(size_t)p * rf]; }, [](int, float x) { return x; }, acc, cmp);
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
    wave_fence();  // the previous token's reads of vb, pb are done
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
    wave_fence();
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
// Split-product path (gbla_split.h): every head dim, slices below 2^31 bytes.
//
// The gradients cancel strongly (dQh = S dnum + z dden, t = dS vt + dz), so the
// products carry fp32 operands to fp32 accuracy: a two-way bf16 split of the
// operands would show through that cancellation, the three-way one does not.
//
// The conv's transpose is fused into the two passes: a unit is walked from its
// last tile to its first, so the three later tokens that a tile's dx needs are
// at hand.  At the unit's end those belong to the next unit: its last three
// tokens' dx are stored without them, every unit leaves the gradients of its
// first three convolved tokens in an edge buffer, and bwd_finish_kernel adds
// the missing products.
//
// Bound: the waves of a workgroup meet at each tile's barriers, so the tile's
// LDS reads (every wave reads all channels' planes), products and vector work
// follow one another with two waves on a SIMD.  Measured, state / query / key,
// against the fp32-product kernels with a conv pass of their own that these
// replaced (n = 32768, H = 8, d = 64 bf16: 52 / 107 / 71 + conv 92 us; 57,511
// packed tokens, H = 8, d = 128: 405 / 681 + 330 for dS / 440 + conv 345): 33 /
// 84 / 57 and 125 / 440 / 281 us.
// ===========================================================================

// State of a unit with fp32-accurate products: the record [S_p | z_p | m_p |
// l_p].  Grid (units, H).
template <typename T, int D>
__global__ void __launch_bounds__(SP<D>::NT, 2)
bwd_state_split_kernel(Plan P, const T* __restrict__ kin, const T* __restrict__ vin,
                       const T* __restrict__ ain, const float* __restrict__ conv_w,
                       const int32_t* __restrict__ cu, float* __restrict__ partials) {
  using C = SP<D>;
  constexpr int NW = C::NW, NT = C::NT;
  // value planes of two steps, token 8 g + j at position 8 g + j
  __shared__ __attribute__((aligned(16))) unsigned char pv[2][C::kOperand];
  __shared__ __attribute__((aligned(16))) float wts[kBwdUnit];  // gate weights
  __shared__ float red[NW];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, unit = blockIdx.x;
  int s, chunk;
  if (!unit_of<NT>(P, cu, P.chunk, P.chunks_per_seq, unit, &s, &chunk)) return;
  s = __builtin_amdgcn_readfirstlane(s);
  chunk = __builtin_amdgcn_readfirstlane(chunk);
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int t0 = chunk * P.chunk;
  const int t1 = (int)min(len, (int64_t)t0 + P.chunk);
  const uint32_t bytes = (uint32_t)len * (uint32_t)(D * sizeof(T));
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(kin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(vin + base_row * D, bytes);
  const int c = 16 * wave + n;
  Column<T, D> nk, nv;
  nk.load(rk, t0 + 8 * g, c);
  nv.load(rv, t0 + 8 * g, c);
  float wk[4], wv[4];
  load_taps4(conv_w, P.heads, h, 1, D, P.W, c, wk);
  load_taps4(conv_w, P.heads, h, 2, D, P.W, c, wv);
  float ml = -INFINITY;
  for (int j = tid; j < t1 - t0; j += NT) {
    const float a = logit<T>(ain, base_row + t0 + j);
    wts[j] = a;
    ml = fmaxf(ml, a);
  }
  const float m = block_max<NT>(ml, red);
  float lacc = 0.0f;
  for (int j = tid; j < (t1 - t0 + 31) / 32 * 32; j += NT) {
    float w = 0.0f;
    if (j < t1 - t0) w = m == -INFINITY ? 0.0f : __expf(wts[j] - m);
    wts[j] = j & 32 ? -w : w;  // every second tile negated
    lacc += w;
  }
  __syncthreads();
  f32x4_t acc[NW];
#pragma unroll
  for (int b = 0; b < NW; ++b) acc[b] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  float z = 0.0f;
  int par = 0;
  float sign = 1.0f;
  auto tile = [&](auto tail, int b0) {
    float kt[8], vt[8];
    nv.conv(wv, vt);
    nk.conv(wk, kt);
    nk.load(rk, b0 + 32 + 8 * g, c);  // past the slice they read 0; unused
    nv.load(rv, b0 + 32 + 8 * g, c);
    zero_past(tail, t1 - b0 - 8 * g, vt);
    u32x4_t A[3];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t x0, x1, x2;
      split3(vt[2 * p], vt[2 * p + 1], x0, x1, x2);
      A[0][p] = x0;
      A[1][p] = x1;
      A[2][p] = x2;
    }
#pragma unroll
    for (int x = 0; x < 3; ++x)
      *reinterpret_cast<u32x4_t*>(pv[par] + x * C::kPlane + plane_unit(c, g)) = A[x];
    zero_past(tail, t1 - b0 - 8 * g, kt);  // phi of a zero: the weights do the rest
    const f32x4_t wa = *reinterpret_cast<const f32x4_t*>(&wts[b0 - t0 + 8 * g]);
    const f32x4_t wb = *reinterpret_cast<const f32x4_t*>(&wts[b0 - t0 + 8 * g + 4]);
    float zt = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      kt[j] = (j < 4 ? wa[j & 3] : wb[j & 3]) * phi_fast(kt[j]);
      zt += kt[j];
    }
    z = fmaf(sign, zt, z);  // a tile at a time, as all sums over a unit
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t x0, x1, x2;
      split3(kt[2 * p], kt[2 * p + 1], x0, x1, x2);
      A[0][p] = x0;
      A[1][p] = x1;
      A[2][p] = x2;
    }
    __syncthreads();  // the planes are whole (and the step before's are read)
#pragma unroll
    for (int b = 0; b < NW; ++b) {
      u32x4_t B[3];
      row_operand<D>(pv[par], 16 * b + n, g, B);
      const f32x4_t y = step_product(A, B);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[b][i] = fmaf(sign, y[i], acc[b][i]);
    }
    par ^= 1;
    sign = -sign;
  };
  int b0 = t0;
  for (; b0 + 32 <= t1; b0 += 32) tile(std::false_type{}, b0);
  if (b0 < t1) tile(std::true_type{}, b0);
  float* rec = partials + ((size_t)h * P.units + unit) * P.rec_floats;
#pragma unroll
  for (int b = 0; b < NW; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) rec[(16 * wave + 4 * g + i) * D + 16 * b + n] = acc[b][i];
  z = sum_groups(z);
  if (g == 0) rec[D * D + c] = z;
  lacc = wave_sum(lacc);
  __syncthreads();  // red's maxima are read
  if (lane == 0) red[wave] = lacc;
  __syncthreads();
  if (tid == 0) {
    float l = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) l += red[w];
    rec[D * D + D] = m;
    rec[D * D + D + 1] = l;
  }
}

// Edge rows of a unit: dxt of its first three tokens.
template <int D>
__device__ __forceinline__ size_t edge_off(const Plan& P, int tensor, int h, int unit) {
  return (((size_t)tensor * P.heads + h) * P.units + unit) * (3 * D);
}

// ---------------------------------------------------------------------------
// Query pass: grid (units, H).  Three barriers a tile: the planes of Qh and the
// denominators' parts; the norm's sums; the planes of dnum.
// ---------------------------------------------------------------------------
template <typename T, int D, bool kNorm>
__global__ void __launch_bounds__(SP<D>::NT, 2)
bwd_query_split_kernel(Plan P, const T* __restrict__ qin, const T* __restrict__ rin,
                       const float* __restrict__ dy, const float* __restrict__ conv_w,
                       const float* __restrict__ gamma, const int32_t* __restrict__ cu,
                       const float* __restrict__ Sg, const float* __restrict__ zg,
                       float* __restrict__ dq, float* __restrict__ dr, float* __restrict__ dsp,
                       float* __restrict__ dgp, float* __restrict__ dcp, float* __restrict__ edge) {
  using C = SP<D>;
  constexpr int NW = C::NW, NT = C::NT, KS = C::KS;
  __shared__ __attribute__((aligned(16))) unsigned char pq[C::kOperand];  // Qh
  __shared__ __attribute__((aligned(16))) unsigned char pd[C::kOperand];  // dnum
  __shared__ __attribute__((aligned(16))) float part[4][NW][32];  // the waves' channel sums
  __shared__ __attribute__((aligned(16))) float dist[NW][5][32];  // a wave's token values
  __shared__ __attribute__((aligned(16))) float ms[D];
  // at d = 128 two parts of one operand's columns leave the registers
  constexpr bool kLdsCols = D >= 128;
  __shared__ u32x4_t cols[kLdsCols ? 2 * KS * NT : 1];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, unit = blockIdx.x;
  int s, chunk;
  if (!unit_of<NT>(P, cu, P.chunk, P.chunks_per_seq, unit, &s, &chunk)) return;
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
  const int c = 16 * wave + n;
  int b0 = t0 + (t1 > t0 ? (t1 - t0 - 1) / 32 * 32 : 0);  // the last tile
  Column<T, D> nq;
  uint32_t nr[8], ndy[8];
  nq.load(rq, b0 + 8 * g, c);
  auto issue_rdy = [&](int tok) {
    const uint32_t e = (uint32_t)(tok * D + c);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if constexpr (kNorm) nr[j] = load_elem<T>(rr, (e + (uint32_t)(j * D)) * (uint32_t)sizeof(T));
      ndy[j] = load_elem<float>(rdy, (e + (uint32_t)(j * D)) * 4u);
    }
  };
  issue_rdy(b0 + 8 * g);

  const size_t sh = (size_t)s * P.heads + h;
  const float* S = Sg + sh * D * D;
  const float* zrow = zg + sh * D;
  float w4[4];
  load_taps4(conv_w, P.heads, h, 0, D, P.W, c, w4);
  const float z = zrow[c], gm = kNorm ? gamma[(size_t)h * D + c] : 1.0f;
  // The wave's columns: f1 of num (X[k][e] = S[k][e]), f2 of dQh (X[k][c] =
  // S'[c][k]).  dQh = S dnum + z dden is formed as S' dnum + z (dden + m . dnum)
  // with S' = S - z m^T, m = (sum_c S[c][.]) / (sum_c z[c]) (the gate-weighted
  // mean value row): the same quantity, but without the cancellation between
  // the two terms when the value rows share a mean (then S dnum ~ z (m . dnum)
  // and o ~ m, and the no-norm dden + m . dnum is formed as
  // -((o - m) . dy) / den directly).
  Columns<D> f1;
  typename std::conditional<kLdsCols, ColumnsLds<D>, Columns<D>>::type f2;
  if constexpr (kLdsCols) f2.lds = cols;
  float m;
  {
    float x[KS][8], y[KS][8], cs = 0.0f, zs = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int i = 0; i < 8; ++i) x[ks][i] = S[(size_t)(32 * ks + 8 * g + i) * D + c];
      const f32x4_t y0 = *reinterpret_cast<const f32x4_t*>(S + (size_t)c * D + 32 * ks + 8 * g);
      const f32x4_t y1 = *reinterpret_cast<const f32x4_t*>(S + (size_t)c * D + 32 * ks + 8 * g + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        y[ks][i] = y0[i];
        y[ks][4 + i] = y1[i];
      }
    }
    for (int k = lane; k < D; k += 64) zs += zrow[k];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < 8; ++i) cs += x[ks][i];
    cs = sum_groups(cs);
    zs = wave_sum(zs);
    m = zs > 0.0f ? cs / zs : 0.0f;
    if (g == 0) ms[c] = m;
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int i = 0; i < 8; ++i) y[ks][i] = fmaf(-z, ms[32 * ks + 8 * g + i], y[ks][i]);
      f1.set(ks, x[ks]);
      f2.set(ks, y[ks]);
    }
  }
  f32x4_t acc[NW];  // dS rows 16 wave + 4 g + i, columns 16 b + n
#pragma unroll
  for (int b = 0; b < NW; ++b) acc[b] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  float dzacc = 0.0f, dgacc = 0.0f, dw[4] = {0.0f, 0.0f, 0.0f, 0.0f}, prev[3] = {0.0f, 0.0f, 0.0f};
  const int tok32 = lane & 31;  // the token of a lane in the channel sums
  // the waves' sums of one quantity for the lane's token
  auto total = [&](int q) {
    float x = part[q][0][tok32];
#pragma unroll
    for (int w = 1; w < NW; ++w) x += part[q][w][tok32];
    return x;
  };
  auto get8 = [&](int q, float* v) {
    const f32x4_t a = *reinterpret_cast<const f32x4_t*>(&dist[wave][q][8 * g]);
    const f32x4_t b = *reinterpret_cast<const f32x4_t*>(&dist[wave][q][8 * g + 4]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = a[j];
      v[4 + j] = b[j];
    }
  };
  const int slot = 8 * g + (n >> 1);  // the token whose sum scatter_sum8 leaves here
  auto put_part = [&](int q, const float* v) {
    const float x = scatter_sum8(v, n);
    if (!(n & 1)) part[q][wave][slot] = x;
  };

  float sign = 1.0f;
  auto tile = [&](auto tail) {
    const Column<T, D> xq = nq;
    nq.load(rq, b0 - 32 + 8 * g, c);  // the tile before (before the slice: reads 0, unused)
    float qh[8], o[8], v[8];
    xq.conv(w4, qh);
    // Tokens past the sequence take no part, whatever their windows hold of it:
    // zeros for Qh, o and dQh, and 1 / den and rs by the token's lanes.
    const int live = t1 - b0 - 8 * g;
    const bool past = decltype(tail)::value && b0 + tok32 >= t1;
#pragma unroll
    for (int j = 0; j < 8; ++j) qh[j] = phi_fast(qh[j]);
    zero_past(tail, live, qh);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = qh[j] * z;
    }
    put_part(0, v);
    put_planes<D>(pq, c, g, qh);
    __syncthreads();
    // num = S^T Qh, den = z . Qh
    const float inv = past ? 0.0f : 1.0f / total(0);
    if (lane < 32) dist[wave][0][tok32] = inv;
    contract_planes<D>(pq, f1, lane, o);
    float dn[8], dd = 0.0f;  // dd: dden of token tok32
    float t1v[8], t2v[8];  // dr and dgamma's terms but for the factor oh
    if constexpr (kNorm) {  // what the products do not enter, beside them
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float r = widen<T>(nr[j]), d = __uint_as_float(ndy[j]), sig = sigmoid_fast(r);
        t1v[j] = d * (r * sig);
        dn[j] = t1v[j] * gm;  // doh
        t2v[j] = d * gm * sig * (1.0f + r * (1.0f - sig));
      }
      issue_rdy(b0 - 32 + 8 * g);
    }
    wave_fence();
    get8(0, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] *= v[j];
    zero_past(tail, live, o);
    const uint32_t off = (uint32_t)((b0 + 8 * g) * D + c) * 4u;
    if constexpr (kNorm) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = o[j] * o[j];
      put_part(1, v);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = dn[j] * o[j];
      put_part(2, v);
      __syncthreads();
      // |o|^2 in the lower lanes, doh . o in the upper, then both in both
      const float x = total(lane < 32 ? 1 : 2), y = __shfl_xor(x, 32);
      const float s2 = lane < 32 ? x : y, s1 = lane < 32 ? y : x;
      const float rs = past ? 0.0f : rsqrt_nr(s2 * (1.0f / D) + P.eps);
      // do . o = rs s1 (1 - rs^2 |o|^2 / d) = eps rs^3 s1 exactly (rs^-2 = |o|^2/d + eps):
      // the RMSNorm leaves almost nothing along o, and summing do . o would
      // return mostly the rounding of its terms.
      dd = -P.eps * rs * rs * rs * s1 * inv;
      dist[wave][lane < 32 ? 0 : 1][tok32] = lane < 32 ? rs : rs * inv;
      dist[wave][lane < 32 ? 2 : 3][tok32] = lane < 32 ? rs * rs * rs * (1.0f / D) * s1 * inv : dd;
      wave_fence();
      get8(0, v);
      float dgt = 0.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float oh = v[j] * o[j];
        dgt = fmaf(oh, t1v[j], dgt);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(oh * t2v[j]), rdr, off + (uint32_t)(j * D * 4), 0, 0);
      }
      dgacc += dgt;
      get8(1, v);
#pragma unroll
      for (int j = 0; j < 8; ++j) dn[j] *= v[j];
      get8(2, v);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        dn[j] = fmaf(-v[j], o[j], dn[j]);
        v[j] = m * dn[j];
      }
      put_part(3, v);
    } else {  // y = o: do = dy
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float d = __uint_as_float(ndy[j]);
        dn[j] = d * v[j];
        v[j] = d * o[j];
        o[j] = d * (o[j] - m);
      }
      issue_rdy(b0 - 32 + 8 * g);
      put_part(1, v);
      put_part(2, o);
      __syncthreads();
      const float x = -total(lane < 32 ? 1 : 2);
      dist[wave][lane < 32 ? 3 : 4][tok32] = x * inv;
      wave_fence();
    }
    get8(3, v);  // dden
    float dzt = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) dzt = fmaf(qh[j], v[j], dzt);
    dzacc += dzt;
    put_planes<D>(pd, c, g, dn);
    __syncthreads();
    // dQh = S' dnum + z (dden + m . dnum); dS += Qh dnum^T
    contract_planes<D>(pd, f2, lane, o);
    // dden + m . dnum, the second from the products that dnum itself enters: m is
    // close to o, dnum nearly orthogonal to it, and m . dnum as a difference of
    // the sums m . doh and m . o left 1.4 times the error in dq
    if constexpr (kNorm) {
      if (lane < 32) dist[wave][4][tok32] = dd + total(3);
      wave_fence();
    }
    get8(4, v);
    // phi'(u) = 1 for u > 0 and e^u = phi(u) <= 1 otherwise: min(phi(u), 1)
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = fmaf(z, v[j], o[j]) * fminf(qh[j], 1.0f);
    zero_past(tail, live, o);
    conv_back8<T, D>(o, xq, w4, prev, lane, tail, live, rdq, off, dw);
    u32x4_t A[3];
    row_operand<D>(pq, c, g, A);
    const uint32_t flip = sign < 0.0f ? 0x80008000u : 0u;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int p = 0; p < 4; ++p) A[x][p] ^= flip;
#pragma unroll
    for (int b = 0; b < NW; ++b) {
      u32x4_t B[3];
      row_operand<D>(pd, 16 * b + n, g, B);
      const f32x4_t y = step_product(A, B);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[b][i] = fmaf(sign, y[i], acc[b][i]);
    }
    b0 -= 32;
    sign = -sign;
  };
  if (b0 + 32 > t1 && t1 > t0) tile(std::true_type{});
  while (b0 >= t0 && t1 > t0) tile(std::false_type{});

  const size_t ui = (size_t)h * P.units + unit;
  float* rec = dsp + ui * P.rec_floats;
#pragma unroll
  for (int b = 0; b < NW; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) rec[(16 * wave + 4 * g + i) * D + 16 * b + n] = acc[b][i];
  dzacc = sum_groups(dzacc);
  dgacc = sum_groups(dgacc);
#pragma unroll
  for (int t = 0; t < 4; ++t) dw[t] = sum_groups(dw[t]);
  if (g == 0) {
    rec[D * D + c] = dzacc;
    dgp[ui * D + c] = dgacc;
    *reinterpret_cast<f32x4_t*>(dcp + (ui * 3 + 0) * D * 4 + 4 * c) = (f32x4_t){dw[0], dw[1], dw[2], dw[3]};
    float* e = edge + edge_off<D>(P, 0, h, unit) + c;
#pragma unroll
    for (int i = 0; i < 3; ++i) e[i * D] = prev[i];
  }
}

// ---------------------------------------------------------------------------
// Key pass: grid (units, H).  Two barriers a tile.
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(SP<D>::NT, 2)
bwd_key_split_kernel(Plan P, const T* __restrict__ kin, const T* __restrict__ vin,
                     const T* __restrict__ ain, const float* __restrict__ conv_w,
                     const int32_t* __restrict__ cu, const float* __restrict__ dSg,
                     const float* __restrict__ mz, float* __restrict__ dk, float* __restrict__ dv,
                     float* __restrict__ da, float* __restrict__ dcp, float* __restrict__ edge) {
  using C = SP<D>;
  constexpr int NW = C::NW, NT = C::NT, KS = C::KS;
  __shared__ __attribute__((aligned(16))) unsigned char pv[C::kOperand];  // vt
  __shared__ __attribute__((aligned(16))) unsigned char pk[C::kOperand];  // P = phi(kt)
  __shared__ __attribute__((aligned(16))) float gt[kBwdUnit];  // gates, zero past the sequence end
  __shared__ float part[NW][32];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, unit = blockIdx.x;
  int s, chunk;
  if (!unit_of<NT>(P, cu, P.chunk, P.chunks_per_seq, unit, &s, &chunk)) return;
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
  const int c = 16 * wave + n;
  int b0 = t0 + (t1 > t0 ? (t1 - t0 - 1) / 32 * 32 : 0);  // the last tile
  Column<T, D> nk, nv;
  nk.load(rk, b0 + 8 * g, c);
  nv.load(rv, b0 + 8 * g, c);
  const size_t sh = (size_t)s * P.heads + h;
  const float* dS = dSg + sh * (D * D + D);
  float wk[4], wv[4];
  load_taps4(conv_w, P.heads, h, 1, D, P.W, c, wk);
  load_taps4(conv_w, P.heads, h, 2, D, P.W, c, wv);
  const float dz = dS[D * D + c];
  Columns<D> f1, f2;  // t: X[e][c] = dS[c][e]; dvt: X[c][e] = dS[c][e]
  {
    float x[KS][8], y[KS][8];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int i = 0; i < 8; ++i) x[ks][i] = dS[(size_t)(32 * ks + 8 * g + i) * D + c];
      const f32x4_t y0 = *reinterpret_cast<const f32x4_t*>(dS + (size_t)c * D + 32 * ks + 8 * g);
      const f32x4_t y1 = *reinterpret_cast<const f32x4_t*>(dS + (size_t)c * D + 32 * ks + 8 * g + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        y[ks][i] = y0[i];
        y[ks][4 + i] = y1[i];
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      f1.set(ks, y[ks]);
      f2.set(ks, x[ks]);
    }
  }
  const float M = mz[2 * sh], Z = mz[2 * sh + 1];
  const float invZ = Z > 0.0f ? 1.0f / Z : 0.0f;
  for (int j = tid; j < (t1 - t0 + 31) / 32 * 32; j += NT)
    gt[j] = j < t1 - t0 ? __expf(logit<T>(ain, base_row + t0 + j) - M) * invZ : 0.0f;
  float dwk[4] = {0.0f, 0.0f, 0.0f, 0.0f}, dwv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  float pvk[3] = {0.0f, 0.0f, 0.0f}, pvv[3] = {0.0f, 0.0f, 0.0f};
  int turn = 0;  // the wave that writes the tile's da

  auto tile = [&](auto tail) {
    const Column<T, D> xk = nk, xv = nv;
    nk.load(rk, b0 - 32 + 8 * g, c);  // the tile before (before the slice: reads 0, unused)
    nv.load(rv, b0 - 32 + 8 * g, c);
    float p[8], t[8];
    xv.conv(wv, t);
    put_planes<D>(pv, c, g, t);
    xk.conv(wk, p);
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = phi_fast(p[j]);
    put_planes<D>(pk, c, g, p);
    __syncthreads();  // the planes (and, the first time, the gates)
    const f32x4_t ga = *reinterpret_cast<const f32x4_t*>(&gt[b0 - t0 + 8 * g]);
    const f32x4_t gb = *reinterpret_cast<const f32x4_t*>(&gt[b0 - t0 + 8 * g + 4]);
    const float gj[8] = {ga[0], ga[1], ga[2], ga[3], gb[0], gb[1], gb[2], gb[3]};
    const uint32_t off = (uint32_t)((b0 + 8 * g) * D + c) * 4u;
    // t = dS vt + dz; dkt = g t phi'(kt); da = g (P . t)
    contract_planes<D>(pv, f1, lane, t);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      t[j] += dz;
      v[j] = p[j] * t[j];
    }
    const float dg = scatter_sum8(v, n);
    if (!(n & 1)) part[wave][8 * g + (n >> 1)] = dg;
    // dvt = g dS^T P
    contract_planes<D>(pk, f2, lane, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      t[j] = gj[j] * t[j] * fminf(p[j], 1.0f);  // phi'(u) = min(phi(u), 1)
      v[j] *= gj[j];
    }
    // tokens past the sequence take no part, whatever their windows hold of it
    const int live = t1 - b0 - 8 * g;
    zero_past(tail, live, t);
    zero_past(tail, live, v);
    __syncthreads();  // the planes are read, the sums of da whole
    if (wave == turn && lane < 32) {
      float x = part[0][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) x += part[w][lane];
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(gt[b0 - t0 + lane] * x), rda,
                                            (uint32_t)(b0 + lane) * 4u, 0, 0);
    }
    turn = turn + 1 == NW ? 0 : turn + 1;
    conv_back8<T, D>(t, xk, wk, pvk, lane, tail, live, rdk, off, dwk);
    conv_back8<T, D>(v, xv, wv, pvv, lane, tail, live, rdv, off, dwv);
    b0 -= 32;
  };
  if (b0 + 32 > t1 && t1 > t0) tile(std::true_type{});
  while (b0 >= t0 && t1 > t0) tile(std::false_type{});

  const size_t ui = (size_t)h * P.units + unit;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    dwk[t] = sum_groups(dwk[t]);
    dwv[t] = sum_groups(dwv[t]);
  }
  if (g == 0) {
    *reinterpret_cast<f32x4_t*>(dcp + (ui * 3 + 1) * D * 4 + 4 * c) = (f32x4_t){dwk[0], dwk[1], dwk[2], dwk[3]};
    *reinterpret_cast<f32x4_t*>(dcp + (ui * 3 + 2) * D * 4 + 4 * c) = (f32x4_t){dwv[0], dwv[1], dwv[2], dwv[3]};
    float* ek = edge + edge_off<D>(P, 1, h, unit) + c;
    float* ev = edge + edge_off<D>(P, 2, h, unit) + c;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      ek[i * D] = pvk[i];
      ev[i * D] = pvv[i];
    }
  }
}

// ---------------------------------------------------------------------------
// What the two passes leave: block (unit, h) of the first P.units adds the
// missing products to dx of the three tokens before the unit's first token,
//   dx_{p-3+j} += sum_{t <= j} w_t dxt_{p+j-t},  p > 0 the unit's first token,
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
  const int p = chunk * P.chunk;
  if (p == 0) return;
  for (int x = tid; x < 3 * D; x += kThreads) {  // (tensor, channel)
    const int c = x % D, tensor = x / D;
    float w4[4], d[3];
    load_taps4(conv_w, P.heads, h, tensor, D, P.W, c, w4);
    const float* e = edge + edge_off<D>(P, tensor, h, unit) + c;
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
    const dim3 block(SP<D>::NT);
    hipLaunchKernelGGL((bwd_state_split_kernel<T, D>), grid, block, 0, st, p, kk, vv, aa, conv_w, cu, dsp);
    gbla_status e = launch_combine_f32(p, cu, dsp, S, z, mz, st);
    if (e != GBLA_OK) return e;
    if (gamma)
      hipLaunchKernelGGL((bwd_query_split_kernel<T, D, true>), grid, block, 0, st, p, qq, rr, dy, conv_w,
                         gamma, cu, S, z, dq, dr, dsp, dgp, dcp, edge);
    else
      hipLaunchKernelGGL((bwd_query_split_kernel<T, D, false>), grid, block, 0, st, p, qq, rr, dy, conv_w,
                         gamma, cu, S, z, dq, dr, dsp, dgp, dcp, edge);
    hipLaunchKernelGGL((bwd_dscombine_kernel<D>), cgrid, dim3(kThreads), 0, st, p, cu,
                       (const float*)dsp, dS);
    hipLaunchKernelGGL((bwd_key_split_kernel<T, D>), grid, block, 0, st, p, kk, vv, aa, conv_w, cu,
                       (const float*)dS, (const float*)mz, dk, dv, da, dcp, edge);
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
