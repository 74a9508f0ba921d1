// gbla_rows.hip -- the state reduction and the readout with fp32 products
// (channel layout, gbla_rows.h): the whole fp32 forward, and the state that
// the backward recomputes.  Slices below 2^31 bytes.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gbla_ext.h"
#include "gbla_rows.h"

namespace gbla {
namespace {


// phi(u) = elu(u) + 1 without a branch.  kFwd: as the fp32 forward has it, with
// the library's expf; otherwise as the backward's other passes have it (the
// hardware exponential, a few ulp).
template <bool kFwd>
__device__ __forceinline__ float phi(float u) {
  if constexpr (kFwd) {
    return fmaxf(u, 0.0f) + expf(fminf(u, 0.0f));
  } else {
    const float e = __expf(u);
    return u > 0.0f ? u + 1.0f : e;
  }
}
template <bool kFwd>
__device__ __forceinline__ float gate(float x) {
  if constexpr (kFwd) return expf(x);
  else return __expf(x);
}

template <typename T>
__device__ __forceinline__ float load_logit(__amdgpu_buffer_rsrc_t r, int tok) {
  if constexpr (sizeof(T) == 4)
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (uint32_t)tok * 4u, 0, 0));
  else
    return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, (uint32_t)tok * 2u, 0, 0) << 16);
}

// ---------------------------------------------------------------------------
// State: grid (units, H).  A unit of at most P.chunk tokens is reduced to the
// record [S_p | z_p | m_p | l_p],
//   w_j = exp(a_j - m_p), m_p = max_j a_j, l_p = sum_j w_j,
//   S_p = sum_j w_j phi(kt_j) vt_j^T, z_p = sum_j w_j phi(kt_j).
// Each wave takes a contiguous quarter of the unit's tokens, 16 at a time, and
// keeps its own D x D sum, so the waves never meet inside the loop; the
// quarters are added as (w0 + w1) + (w2 + w3).  Measured against the kernels
// that this replaced: fp32 forward, B = 2, n = 8191, H = 8, d = 64 52 -> 29 us;
// the backward's bf16 state at n = 32768, H = 8, d = 64 52 -> 39 us, on 57,511
// packed tokens, H = 8, d = 128 407 -> 275 us (256 products a tile are 107 us).
// ---------------------------------------------------------------------------
template <typename T, int D, bool kFwd>
__global__ void __launch_bounds__(kThreads, D >= 128 ? 1 : 2)
state_rows_kernel(Plan P, const T* __restrict__ kin, const T* __restrict__ vin,
                  const T* __restrict__ ain, const float* __restrict__ conv_w,
                  const int32_t* __restrict__ cu, float* __restrict__ partials) {
  using C = CL<D>;
  constexpr int NMB = C::NMB;
  __shared__ __attribute__((aligned(16))) float buf[2 * D * D];  // the waves' sums
  __shared__ __attribute__((aligned(16))) float wts[kMaxChunk];   // gate weights
  __shared__ f32x4_t tk[D], tv[D];
  __shared__ float red[4][D];
  __shared__ float red4[4];
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
  const uint32_t bytes = (uint32_t)len * (uint32_t)(D * sizeof(T));
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(kin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(vin + base_row * D, bytes);
  // no gate logits: an empty range, so every logit reads as 0
  const __amdgpu_buffer_rsrc_t ra =
      ain ? make_rsrc(ain + base_row, (uint32_t)len * (uint32_t)sizeof(T)) : make_rsrc(kin, 0u);

  // the wave's quarter of the unit, in whole tiles
  const int q4 = quarter_tokens(t1 - t0);
  const int w0 = t0 + wave * q4, w1 = min(t1, w0 + q4);
  Window<T, D> nk, nv;
  nk.load(rk, w0 + 4 * g, n);
  nv.load(rv, w0 + 4 * g, n);
  stage_taps<D>(conv_w, P.heads, h, 1, P.W, tk);
  stage_taps<D>(conv_w, P.heads, h, 2, P.W, tv);

  // gate weights of the unit, zero past its end
  float ml = -INFINITY;
  for (int j = t0 + tid; j < t1; j += kThreads) {
    const float a = load_logit<T>(ra, j);
    wts[j - t0] = a;
    ml = fmaxf(ml, a);
  }
  const float m = block_max(ml, red4);  // its barriers also publish the taps
  float lacc = 0.0f;
  for (int j = tid; j < 4 * q4; j += kThreads) {
    float w = 0.0f;
    if (j < t1 - t0) w = m == -INFINITY ? 0.0f : gate<kFwd>(wts[j] - m);
    wts[j] = w;
    lacc += w;
  }
  __syncthreads();

  f32x4_t acc[C::kBlocks];
#pragma unroll
  for (int k = 0; k < C::kBlocks; ++k) acc[k] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  float z[NMB];
#pragma unroll
  for (int b = 0; b < NMB; ++b) z[b] = 0.0f;

  for (int b0 = w0; b0 < w1; b0 += 16) {
    float kt[NMB][4], vt[NMB][4];
    __asm__ volatile("" ::: "memory");  // taps are re-read from LDS, not held
    nk.conv(LdsTaps<D>{tk, n}, kt);
    nv.conv(LdsTaps<D>{tv, n}, vt);
    // the next tile's rows (past the slice they read 0; unused)
    nk.load(rk, b0 + 16 + 4 * g, n);
    nv.load(rv, b0 + 16 + 4 * g, n);
    const f32x4_t w = *reinterpret_cast<const f32x4_t*>(&wts[b0 - t0 + 4 * g]);
#pragma unroll
    for (int b = 0; b < NMB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        kt[b][i] = w[i] * phi<kFwd>(kt[b][i]);
        z[b] += kt[b][i];
      }
    token_product<D>(kt, vt, acc);
  }

  float* rec = partials + ((size_t)h * P.units + unit) * P.rec_floats;
  sum_waves<D>(acc, buf, buf + D * D, rec);
  sum_channels<D>(z, red, rec + D * D);
  lacc = wave_sum(lacc);
  if (lane == 0) red4[wave] = lacc;
  __syncthreads();
  if (tid == 0) {
    rec[D * D + D] = m;
    rec[D * D + D + 1] = (red4[0] + red4[1]) + (red4[2] + red4[3]);
  }
}

// ---------------------------------------------------------------------------
// Readout of the fp32 forward: grid (readout units, H).
//   o_i = phi(qt_i)^T S / phi(qt_i)^T z,  y_i = o_i rs_i gamma silu(r_i).
// The operands [S; z] are the combine's fp32 readout fragments, laid out again
// in LDS for contract_rows.  Measured against the kernel that this replaced: B =
// 2, n = 8191, H = 8, d = 64 49 -> 32 us (100 MB: 20 us of plain copy).
// ---------------------------------------------------------------------------
template <int D, bool kNorm>
__global__ void __launch_bounds__(kThreads, D >= 128 ? 1 : 2)
readout_rows_kernel(Plan P, const float* __restrict__ qin, const float* __restrict__ rin,
                    const float* __restrict__ conv_w, const float* __restrict__ gamma,
                    const int32_t* __restrict__ cu, const unsigned char* __restrict__ frags,
                    float* __restrict__ out) {
  using C = CL<D>;
  constexpr int NMB = C::NMB;
  __shared__ f32x4_t fs[C::kFrag];  // B[c][e] = S[c][e]
  __shared__ __attribute__((aligned(16))) float stg[4][C::kStage];
  __shared__ f32x4_t tq[D];
  __shared__ float zs[D], gs[D];  // slot order 16 b + n
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, unit = blockIdx.x;
  int s, tile;
  if (!unit_of(P, cu, P.rtile, P.rtiles_per_seq, unit, &s, &tile)) return;
  s = __builtin_amdgcn_readfirstlane(s);
  tile = __builtin_amdgcn_readfirstlane(tile);
  int64_t len, base_row;
  seq_geometry(P, cu, s, h, &len, &base_row);
  const int t0 = tile * P.rtile;
  const int t1 = (int)min(len, (int64_t)t0 + P.rtile);
  if (t1 <= t0) return;
  const uint32_t bytes = (uint32_t)len * (uint32_t)(D * 4);
  const __amdgpu_buffer_rsrc_t rq = make_rsrc(qin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rr = kNorm ? make_rsrc(rin + base_row * D, bytes) : make_rsrc(qin, 0u);
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out + base_row * D, (uint32_t)t1 * (uint32_t)(D * 4));
  const int q4 = quarter_tokens(t1 - t0);
  const int w0 = t0 + wave * q4, w1 = min(t1, w0 + q4);
  Window<float, D> nq;
  Row<float, D> nr[4];
  auto issue_r = [&](int tok) {
    const uint32_t off = row_off<float, D>(tok, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) nr[i].load(rr, off + (uint32_t)(i * D * 4));
  };
  nq.load(rq, w0 + 4 * g, n);
  if constexpr (kNorm) issue_r(w0 + 4 * g);
  stage_taps<D>(conv_w, P.heads, h, 0, P.W, tq);
  // fragment of S[c .. c + 3][e] / z[c] in the combine's layout (eight values
  // per 32-byte lane slot)
  const float* fr = reinterpret_cast<const float*>(frags + ((size_t)s * P.heads + h) * P.frag_bytes);
  constexpr int NKB = D / 32;
  Frags<D> f;
#pragma unroll
  for (int u = 0; u < Frags<D>::kPer; ++u) {
    const int c = f.k0(u), e = f.col(u);
    const int mb = 2 * (e / 32) + (e % 8) / 4, m = 4 * ((e % 32) / 8) + e % 4;
    f.v[u] = *reinterpret_cast<const f32x4_t*>(
        fr + ((mb * NKB + c / 32) * 64 + 16 * ((c % 32) / 8) + m) * 8 + c % 8);
  }
  if (tid < D) {
    const int c = slot_chan<D>(tid >> 4, tid & 15);
    zs[tid] = fr[((D / 16) * NKB + c / 32) * 512 + 16 * ((c % 32) / 8) * 8 + c % 8];
    gs[tid] = kNorm ? gamma[(size_t)h * D + c] : 1.0f;
  }
  f.put(fs);
  __syncthreads();

  for (int b0 = w0; b0 < w1; b0 += 16) {
    float x[NMB][4], rv[NMB][4];
    __asm__ volatile("" ::: "memory");  // operands are re-read from LDS, not held
    nq.conv(LdsTaps<D>{tq, n}, x);
    nq.load(rq, b0 + 16 + 4 * g, n);
    float den[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int b = 0; b < NMB; ++b) {
      const float z = zs[16 * b + n];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[b][i] = phi<true>(x[b][i]);
        den[i] = fmaf(x[b][i], z, den[i]);
      }
    }
    f32x4_t o[NMB];
#pragma unroll
    for (int b = 0; b < NMB; ++b) o[b] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
    contract_rows<D>(x, stg[wave], fs, lane, o);
    if constexpr (kNorm) {
#pragma unroll
      for (int b = 0; b < NMB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) rv[b][i] = nr[i].at(b);
      issue_r(b0 + 16 + 4 * g);
    }
    const uint32_t off = row_off<float, D>(b0 + 4 * g, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float inv_den = 1.0f / sum_row16(den[i]);
      float ss = 0.0f;
#pragma unroll
      for (int b = 0; b < NMB; ++b) {
        x[b][i] = o[b][i] * inv_den;
        ss = fmaf(x[b][i], x[b][i], ss);
      }
      if constexpr (kNorm) {
        const float scale = __builtin_amdgcn_rsqf(sum_row16(ss) * (1.0f / D) + P.eps);
#pragma unroll
        for (int b = 0; b < NMB; ++b) {
          const float r = rv[b][i];
          x[b][i] = x[b][i] * scale * gs[16 * b + n] * (r * __builtin_amdgcn_rcpf(1.0f + expf(-r)));
        }
      }
      store_row<D>(ro, off + (uint32_t)(i * D * 4), x, i);
    }
  }
}

template <typename T, bool kFwd>
gbla_status run_state(const Plan& p, const void* k, const void* v, const void* a,
                      const float* conv_w, const int32_t* cu, float* partials, hipStream_t st) {
  const dim3 grid(p.units, p.heads);
#define GBLA_STATE_ROWS(DD)                                                                       \
  hipLaunchKernelGGL((state_rows_kernel<T, DD, kFwd>), grid, dim3(kThreads), 0, st, p, (const T*)k, \
                     (const T*)v, (const T*)a, conv_w, cu, partials)
  if (p.d == 128) GBLA_STATE_ROWS(128);
  else if (p.d == 64) GBLA_STATE_ROWS(64);
  else GBLA_STATE_ROWS(32);
#undef GBLA_STATE_ROWS
  return hipGetLastError() == hipSuccess ? GBLA_OK : GBLA_ERR_HIP;
}

}  // namespace

gbla_status launch_state_rows(const Plan& p, const void* k, const void* v, const void* a,
                              const float* conv_w, const int32_t* cu, float* partials,
                              bool forward, hipStream_t st) {
  if (p.dtype == GBLA_BF16) return run_state<uint16_t, false>(p, k, v, a, conv_w, cu, partials, st);
  if (forward) return run_state<float, true>(p, k, v, a, conv_w, cu, partials, st);
  return run_state<float, false>(p, k, v, a, conv_w, cu, partials, st);
}

gbla_status launch_readout_rows(const Plan& p, const void* q, const void* r, const float* conv_w,
                                const float* gamma, const int32_t* cu, const unsigned char* frags,
                                float* out, hipStream_t st, KernelEvents ev) {
  const dim3 grid(p.runits, p.heads);
  const float *qq = (const float*)q, *rr = (const float*)r;
#define GBLA_READOUT_ROWS(DD, NORM)                                                             \
  do {                                                                                          \
    if (ev.any())                                                                               \
      hipExtLaunchKernelGGL((readout_rows_kernel<DD, NORM>), grid, dim3(kThreads), 0, st,       \
                            ev.start, ev.stop, 0, p, qq, rr, conv_w, gamma, cu, frags, out);    \
    else                                                                                        \
      hipLaunchKernelGGL((readout_rows_kernel<DD, NORM>), grid, dim3(kThreads), 0, st, p, qq,   \
                         rr, conv_w, gamma, cu, frags, out);                                    \
  } while (0)
  const bool norm = gamma != nullptr;  // NULL gamma: the no-gated-norm switch
  if (p.d == 128) {
    if (norm) GBLA_READOUT_ROWS(128, true); else GBLA_READOUT_ROWS(128, false);
  } else if (p.d == 64) {
    if (norm) GBLA_READOUT_ROWS(64, true); else GBLA_READOUT_ROWS(64, false);
  } else {
    if (norm) GBLA_READOUT_ROWS(32, true); else GBLA_READOUT_ROWS(32, false);
  }
#undef GBLA_READOUT_ROWS
  return hipGetLastError() == hipSuccess ? GBLA_OK : GBLA_ERR_HIP;
}

}  // namespace gbla
