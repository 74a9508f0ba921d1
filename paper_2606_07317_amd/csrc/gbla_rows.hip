// gbla_rows.hip -- the fp32 forward (state reduction and readout with fp32
// products) and the one-launch forward of short sequences, in the channel
// layout of gbla_rows.h.  Slices below 2^31 bytes.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gbla_ext.h"
#include "gbla_rows.h"

namespace gbla {
namespace {

// kFull: the library's expf (the fp32 forward); otherwise the hardware
// exponential, a few ulp.
template <bool kFull>
__device__ __forceinline__ float gate(float x) {
  if constexpr (kFull) return expf(x);
  else return __expf(x);
}
// phi(u) = elu(u) + 1 without a branch.
template <bool kFull>
__device__ __forceinline__ float phi(float u) {
  return fmaxf(u, 0.0f) + gate<kFull>(fminf(u, 0.0f));
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
// quarters are added as (w0 + w1) + (w2 + w3).  Measured against the kernel
// that this replaced: B = 2, n = 8191, H = 8, d = 64 52 -> 29 us.  At d = 128 a
// wave's sum takes 256 accumulators, so one wave runs on a SIMD and 57 registers
// spill; the whole forward there took 397 us with the kernels before these and
// takes 178, n = 1000, H = 4 206 and 58.
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(kThreads, D >= 128 ? 1 : 2)
state_rows_kernel(Plan P, const float* __restrict__ kin, const float* __restrict__ vin,
                  const float* __restrict__ ain, const float* __restrict__ conv_w,
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
  const uint32_t bytes = (uint32_t)len * (uint32_t)(D * 4);
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(kin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(vin + base_row * D, bytes);
  // no gate logits: an empty range, so every logit reads as 0
  const __amdgpu_buffer_rsrc_t ra =
      ain ? make_rsrc(ain + base_row, (uint32_t)len * 4u) : make_rsrc(kin, 0u);

  // the wave's quarter of the unit, in whole tiles
  const int q4 = quarter_tokens(t1 - t0);
  const int w0 = t0 + wave * q4, w1 = min(t1, w0 + q4);
  Window<float, D> nk, nv;
  nk.load(rk, w0 + 4 * g, n);
  nv.load(rv, w0 + 4 * g, n);
  stage_taps<D>(conv_w, P.heads, h, 1, P.W, tk);
  stage_taps<D>(conv_w, P.heads, h, 2, P.W, tv);

  // gate weights of the unit, zero past its end
  float ml = -INFINITY;
  for (int j = t0 + tid; j < t1; j += kThreads) {
    const float a = load_logit<float>(ra, j);
    wts[j - t0] = a;
    ml = fmaxf(ml, a);
  }
  const float m = block_max(ml, red4);  // its barriers also publish the taps
  float lacc = 0.0f;
  for (int j = tid; j < 4 * q4; j += kThreads) {
    float w = 0.0f;
    if (j < t1 - t0) w = m == -INFINITY ? 0.0f : gate<true>(wts[j] - m);
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
        kt[b][i] = w[i] * phi<true>(kt[b][i]);
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

// Ragged batches of short sequences are taken longest first, in four classes by
// length against the batch's mean (over 4, 2, 1 times, the rest) and in
// sequence order inside a class: with lognormal lengths sequence order left the
// grid ending on long sequences that started last (256 sequences, T = 39,470, H =
// 8, d = 64: 117 us against 75).  The sequence of rank r; every
// thread of the block calls.
__device__ __forceinline__ int long_first(const int32_t* cu, int nseq, int tokens, int r) {
  __shared__ int cnt[4][4];
  __shared__ int found;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int mean = tokens / nseq + 1;
  auto cls = [&](int s) {
    if (s >= nseq) return -1;
    const int len = cu[s + 1] - cu[s];
    return len > 4 * mean ? 0 : len > 2 * mean ? 1 : len > mean ? 2 : 3;
  };
  int mine[4] = {0, 0, 0, 0};  // wave-uniform
  int first = 0;
  for (int base = 0; base < nseq; base += kThreads) {
    const int c = cls(base + tid);
    if (base == 0) first = c;
#pragma unroll
    for (int k = 0; k < 4; ++k) mine[k] += __popcll(__ballot(c == k));
  }
  if (lane < 4) cnt[wave][lane] = lane == 0 ? mine[0] : lane == 1 ? mine[1] : lane == 2 ? mine[2] : mine[3];
  __syncthreads();
  int q = r, want = 3;
#pragma unroll
  for (int k = 2; k >= 0; --k) {
    // ranks before class k + 1
    int before = 0;
#pragma unroll
    for (int j = 0; j <= k; ++j) before += (cnt[0][j] + cnt[1][j]) + (cnt[2][j] + cnt[3][j]);
    if (r < before) want = k;
  }
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (j < want) q -= (cnt[0][j] + cnt[1][j]) + (cnt[2][j] + cnt[3][j]);
  for (int base = 0; base < nseq; base += kThreads) {
    const bool is = (base == 0 ? first : cls(base + tid)) == want;
    const uint64_t mask = __ballot(is);
    __syncthreads();  // cnt's earlier values are read
    if (lane == 0) cnt[wave][0] = __popcll(mask);
    __syncthreads();
    int at = __popcll(mask & ((1ull << lane) - 1)), all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      at += w < wave ? cnt[w][0] : 0;
      all += cnt[w][0];
    }
    if (is && at == q) found = base + tid;
    if (q >= 0 && q < all) break;
    q -= all;
  }
  __syncthreads();
  return found;
}

// Sequence and head of a workgroup of the one-launch forward, grid (N * H): the
// heads of a sequence next to each other.
__device__ __forceinline__ void short_unit(const Plan& P, const int32_t* cu, int* s, int* h) {
  const int r = (int)blockIdx.x / P.heads;
  *h = (int)blockIdx.x - r * P.heads;
  *s = __builtin_amdgcn_readfirstlane(P.ragged ? long_first(cu, P.nseq, P.rows, r) : r);
}

// ---------------------------------------------------------------------------
// The whole fp32 forward of short sequences in one launch: grid (N * H).  A workgroup
// reduces its (sequence, head) to [S; z] as the state kernel does, keeps it in
// LDS as the readout's operands and reads the sequence out as the readout
// kernel does.  The gates are not normalised (the factor cancels in o).
// ---------------------------------------------------------------------------
template <int D, bool kNorm>
__global__ void __launch_bounds__(kThreads, 2)
short_forward_kernel(Plan P, const float* __restrict__ qin, const float* __restrict__ kin,
                     const float* __restrict__ vin, const float* __restrict__ ain, const float* __restrict__ rin,
                     const float* __restrict__ conv_w, const float* __restrict__ gamma,
                     const int32_t* __restrict__ cu, float* __restrict__ out) {
  using C = CL<D>;
  constexpr int NMB = C::NMB;
  // the waves' sums, then the operands B[c][e] = S[c][e]
  __shared__ __attribute__((aligned(16))) float buf[2 * D * D];
  __shared__ __attribute__((aligned(16))) float stg[4][C::kStage];
  __shared__ f32x4_t tk[D], tv[D], tq[D];
  __shared__ float zs[D], gs[D];  // by channel
  __shared__ float red4[4];
  f32x4_t* fs = reinterpret_cast<f32x4_t*>(buf);
  float (*red)[D] = reinterpret_cast<float(*)[D]>(&stg[0][0]);  // before the readout
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int s, h;
  short_unit(P, cu, &s, &h);
  int64_t len64, base_row;
  seq_geometry(P, cu, s, h, &len64, &base_row);
  const int len = (int)len64;
  if (len <= 0) return;
  const uint32_t bytes = (uint32_t)len * (uint32_t)(D * 4);
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(kin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(vin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rq = make_rsrc(qin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rr = kNorm ? make_rsrc(rin + base_row * D, bytes) : make_rsrc(qin, 0u);
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out + base_row * D, (uint32_t)len * (uint32_t)(D * 4));
  // no gate logits: an empty range, so every logit reads as 0
  const __amdgpu_buffer_rsrc_t ra =
      ain ? make_rsrc(ain + base_row, (uint32_t)len * 4u) : make_rsrc(kin, 0u);
  const int q4 = quarter_tokens(len);
  const int w0 = wave * q4, w1 = min(len, w0 + q4);
  Window<float, D> nk, nv;
  float na[4];
  auto issue_kv = [&](int tok) {
    nk.load(rk, tok, n);
    nv.load(rv, tok, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) na[i] = load_logit<float>(ra, tok + i);
  };
  issue_kv(w0 + 4 * g);
  stage_taps<D>(conv_w, P.heads, h, 0, P.W, tq);
  stage_taps<D>(conv_w, P.heads, h, 1, P.W, tk);
  stage_taps<D>(conv_w, P.heads, h, 2, P.W, tv);
  if (tid < D) gs[tid] = kNorm ? gamma[(size_t)h * D + tid] : 1.0f;
  float ml = -INFINITY;
  for (int j = tid; j < len; j += kThreads) ml = fmaxf(ml, load_logit<float>(ra, j));
  const float m = block_max(ml, red4);  // its barriers also publish the taps

  {
    f32x4_t acc[C::kBlocks];
#pragma unroll
    for (int k = 0; k < C::kBlocks; ++k) acc[k] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
    float z[NMB];
#pragma unroll
    for (int b = 0; b < NMB; ++b) z[b] = 0.0f;
    for (int b0 = w0; b0 < w1; b0 += 16) {
      float kt[NMB][4], vt[NMB][4], w[4];
      __asm__ volatile("" ::: "memory");  // taps are re-read from LDS, not held
      nk.conv(LdsTaps<D>{tk, n}, kt);
      nv.conv(LdsTaps<D>{tv, n}, vt);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = b0 + 4 * g + i < len && m != -INFINITY ? gate<true>(na[i] - m) : 0.0f;
      issue_kv(b0 + 16 + 4 * g);  // past the sequence they read 0; unused
#pragma unroll
      for (int b = 0; b < NMB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          kt[b][i] = w[i] * phi<true>(kt[b][i]);
          z[b] += kt[b][i];
        }
      token_product<D>(kt, vt, acc);
    }
    // S = (w0 + w1) + (w2 + w3), as in sum_waves, laid out as operands
    put_waves<D>(acc, buf, buf + D * D);
#pragma unroll
    for (int b = 0; b < NMB; ++b) {
      const float zsum = sum_groups(z[b]);
      if (g == 0) red[wave][slot_chan<D>(b, n)] = zsum;
    }
  }
  // the readout's first rows, in flight over the sums
  Window<float, D> nq;
  Row<float, D> nr[4];
  auto issue_r = [&](int tok) {
    const uint32_t off = row_off<float, D>(tok, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) nr[i].load(rr, off + (uint32_t)(i * D * 4));
  };
  nq.load(rq, w0 + 4 * g, n);
  if constexpr (kNorm) issue_r(w0 + 4 * g);
  __syncthreads();
  if (tid < D) zs[tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
  Frags<D> f;
#pragma unroll
  for (int u = 0; u < Frags<D>::kPer; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int x = (f.k0(u) + i) * D + f.col(u);
      f.v[u][i] = buf[x] + buf[D * D + x];
    }
  __syncthreads();
  f.put(fs);
  __syncthreads();

  for (int b0 = w0; b0 < w1; b0 += 16) {
    float x[NMB][4], rv4[NMB][4];
    __asm__ volatile("" ::: "memory");  // operands are re-read from LDS, not held
    nq.conv(LdsTaps<D>{tq, n}, x);
    nq.load(rq, b0 + 16 + 4 * g, n);
    float den[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int b = 0; b < NMB; ++b) {
      const float z = zs[slot_chan<D>(b, n)];
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
        for (int i = 0; i < 4; ++i) rv4[b][i] = nr[i].at(b);
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
          const float r = rv4[b][i];
          x[b][i] = x[b][i] * scale * gs[slot_chan<D>(b, n)] *
                    (r * __builtin_amdgcn_rcpf(1.0f + gate<true>(-r)));
        }
      }
      store_row<D>(ro, off + (uint32_t)(i * D * 4), x, i);
    }
  }
}

// ---------------------------------------------------------------------------
// The same in one launch for bf16 inputs: tiles of 32 tokens, a lane holding
// eight consecutive tokens 8 g + j, products on v_mfma_f32_16x16x32_bf16 (which,
// unlike the fp32 one, runs beside the vector unit).  As in the other bf16
// kernels the gated keys, phi(qt) and the readout's S are rounded to bf16 and
// the values enter without rounding error (here as bf16 + bf16 residue).  Without
// the norm the denominators take the rounded z and phi(qt), as the readout kernel's
// products do: the roundings then cancel in part in o (sequences of 1 to 10 tokens
// 5.2e-4 from 64 bits, 5.7e-4 with both in fp32); the norm takes the
// denominators out, and z stays in fp32.  S is normalised by the sum of the gates before it is rounded, as the
// combine does, so that both forms round the same values: rounded as summed, the
// output was 4.2e-4 (2-norm) from the three launches' on these sequences, as far
// as either is from the exact result.  256 packed sequences, T = 39,470 (5 to
// 1,019 tokens), H = 8, d = 64: 72 us against 164 us for the three launches,
// whose partial records and operands (70 MB) and one workgroup per CU this
// avoids; 243 MB of inputs and outputs are 48 us of plain copy.  117 us in
// sequence order (long_first), 216 us with fp32 products.
// ---------------------------------------------------------------------------
template <int D, bool kNorm>
__global__ void __launch_bounds__(kThreads, 3)
short_forward_bf16_kernel(Plan P, const uint16_t* __restrict__ qin, const uint16_t* __restrict__ kin,
                          const uint16_t* __restrict__ vin, const uint16_t* __restrict__ ain,
                          const uint16_t* __restrict__ rin, const float* __restrict__ conv_w,
                          const float* __restrict__ gamma, const int32_t* __restrict__ cu,
                          float* __restrict__ out) {
  using C = CL<D>;
  using T = uint16_t;
  constexpr int NMB = C::NMB, KS = D / 32, V = C::V;
  constexpr int kOps = NMB * KS * 64;      // operand vectors of S (16 bytes)
  constexpr int kPitch = 2 * D + 16;       // bytes of a staged token row
  constexpr int kBuf = 2 * D * D * 4;      // the waves' sums; then operands and stages
  constexpr int kLds = kOps * 16 + 4 * 32 * kPitch;
  __shared__ __attribute__((aligned(16))) unsigned char lds[kBuf > kLds ? kBuf : kLds];
  __shared__ f32x4_t tk[D], tv[D], tq[D];
  __shared__ float red[4][D];
  __shared__ float zs[D], gs[D];  // by channel
  __shared__ float red4[4];
  float* buf = reinterpret_cast<float*>(lds);
  u32x4_t* ops = reinterpret_cast<u32x4_t*>(lds);
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int s, h;
  short_unit(P, cu, &s, &h);
  int64_t len64, base_row;
  seq_geometry(P, cu, s, h, &len64, &base_row);
  const int len = (int)len64;
  if (len <= 0) return;
  const uint32_t bytes = (uint32_t)len * (uint32_t)(D * 2);
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(kin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(vin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rq = make_rsrc(qin + base_row * D, bytes);
  const __amdgpu_buffer_rsrc_t rr = kNorm ? make_rsrc(rin + base_row * D, bytes) : make_rsrc(qin, 0u);
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(out + base_row * D, (uint32_t)len * (uint32_t)(D * 4));
  // no gate logits: an empty range, so every logit reads as 0
  const __amdgpu_buffer_rsrc_t ra = ain ? make_rsrc(ain + base_row, (uint32_t)len * 2u) : make_rsrc(kin, 0u);
  // the wave's tiles: every fourth one
  const int w0 = 32 * wave, w1 = len;
  auto load_rows = [&](__amdgpu_buffer_rsrc_t r, int tok, Row<T, D>(&x)[11]) {
    const uint32_t off = row_off<T, D>(tok, n);
#pragma unroll
    for (int j = 0; j < 11; ++j) x[j].load(r, off + (uint32_t)((j - 3) * D * 2));
  };
  Row<T, D> xk[11], xv[11];
  float na[8];
  auto issue_kv = [&](int tok) {
    load_rows(rk, tok, xk);
    load_rows(rv, tok, xv);
#pragma unroll
    for (int j = 0; j < 8; ++j) na[j] = load_logit<T>(ra, tok + j);
  };
  if (w0 < w1) issue_kv(w0 + 8 * g);
  stage_taps<D>(conv_w, P.heads, h, 0, P.W, tq);
  stage_taps<D>(conv_w, P.heads, h, 1, P.W, tk);
  stage_taps<D>(conv_w, P.heads, h, 2, P.W, tv);
  if (tid < D) gs[tid] = kNorm ? gamma[(size_t)h * D + tid] : 1.0f;
  float ml = -INFINITY;
  for (int j = tid; j < len; j += kThreads) ml = fmaxf(ml, load_logit<T>(ra, j));
  const float m = block_max(ml, red4);  // its barriers also publish the taps

  {
    f32x4_t acc[C::kBlocks];
#pragma unroll
    for (int k = 0; k < C::kBlocks; ++k) acc[k] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
    float z[NMB];
#pragma unroll
    for (int b = 0; b < NMB; ++b) z[b] = 0.0f;
    float lacc = 0.0f;
    for (int b0 = w0; b0 < w1; b0 += 128) {
      __asm__ volatile("" ::: "memory");  // taps are re-read from LDS, not held
      if (b0 > w0) issue_kv(b0 + 8 * g);
      float w[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        w[j] = b0 + 8 * g + j < len && m != -INFINITY ? __expf(na[j] - m) : 0.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) lacc += w[j];
      u32x4_t A[NMB];
#pragma unroll
      for (int b = 0; b < NMB; ++b) {
        const f32x4_t t4 = tk[16 * b + n];
        float kw[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          float a = t4[0] * xk[j].at(b);
#pragma unroll
          for (int t = 1; t < 4; ++t) a = fmaf(t4[t], xk[j + t].at(b), a);
          kw[j] = w[j] * phi<false>(a);
          z[b] += kw[j];
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) A[b][p] = pack_bf16x2(kw[2 * p], kw[2 * p + 1]);
      }
#pragma unroll
      for (int nb = 0; nb < NMB; ++nb) {
        const f32x4_t t4 = tv[16 * nb + n];
        float vt[8];
        u32x4_t hi, lo;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          float a = t4[0] * xv[j].at(nb);
#pragma unroll
          for (int t = 1; t < 4; ++t) a = fmaf(t4[t], xv[j + t].at(nb), a);
          vt[j] = a;
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          hi[p] = pack_bf16x2(vt[2 * p], vt[2 * p + 1]);
          // no residue is below -2^120; that of an infinite value is NaN, which
          // fmaxf replaces: its products stay infinite
          lo[p] = pack_bf16x2(fmaxf(vt[2 * p] - bf16_lo(hi[p]), -0x1p120f),
                              fmaxf(vt[2 * p + 1] - bf16_hi(hi[p]), -0x1p120f));
        }
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) {
          f32x4_t& c = acc[mb * NMB + nb];
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A[mb]),
                                                      __builtin_bit_cast(bf16x8_t, hi), c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A[mb]),
                                                      __builtin_bit_cast(bf16x8_t, lo), c, 0, 0, 0);
        }
      }
    }
    put_waves<D>(acc, buf, buf + D * D);
#pragma unroll
    for (int b = 0; b < NMB; ++b) {
      const float zsum = sum_groups(z[b]);
      if (g == 0) red[wave][slot_chan<D>(b, n)] = zsum;
    }
    lacc = sum_groups(lacc);
    if (lane == 0) red4[wave] = lacc;
  }
  // the readout's first rows, in flight over the sums
  Row<T, D>(&xq)[11] = xk;
  Row<T, D> xr[8];
  auto issue_qr = [&](int tok) {
    load_rows(rq, tok, xq);
    if constexpr (kNorm) {
      const uint32_t off = row_off<T, D>(tok, n);
#pragma unroll
      for (int j = 0; j < 8; ++j) xr[j].load(rr, off + (uint32_t)(j * D * 2));
    }
  };
  if (w0 < w1) issue_qr(w0 + 8 * g);
  __syncthreads();
  const float l = (red4[0] + red4[1]) + (red4[2] + red4[3]);
  const float inv_l = l > 0.0f ? 1.0f / l : 0.0f;
  if (tid < D) {
    const float z = ((red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid])) * inv_l;
    zs[tid] = kNorm ? z : bf16_lo(pack_bf16x2(z, 0.0f));
  }
  // B operands of S: vector (nb * KS + ks) * 64 + lane holds S[32 ks + 8 g + i]
  // [slot_chan(nb, n)], i < 8
  constexpr int kPer = (kOps + kThreads - 1) / kThreads;
  u32x4_t f[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int idx = (tid + u * kThreads) & (kOps - 1);
    const int l = idx & 63, x0 = (32 * ((idx >> 6) % KS) + 8 * (l >> 4)) * D + slot_chan<D>((idx >> 6) / KS, l & 15);
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (buf[x0 + i * D] + buf[D * D + x0 + i * D]) * inv_l;
#pragma unroll
    for (int p = 0; p < 4; ++p) f[u][p] = pack_bf16x2(v[2 * p], v[2 * p + 1]);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    if (tid + u * kThreads < kOps) ops[tid + u * kThreads] = f[u];
  __syncthreads();
  unsigned char* stage = lds + kOps * 16 + wave * 32 * kPitch;

  for (int b0 = w0; b0 < w1; b0 += 128) {
    __asm__ volatile("" ::: "memory");  // operands are re-read from LDS, not held
    if (b0 > w0) issue_qr(b0 + 8 * g);
    float x[NMB][8], den[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) den[j] = 0.0f;
#pragma unroll
    for (int b = 0; b < NMB; ++b) {
      const f32x4_t t4 = tq[16 * b + n];
      const float z = zs[slot_chan<D>(b, n)];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float a = t4[0] * xq[j].at(b);
#pragma unroll
        for (int t = 1; t < 4; ++t) a = fmaf(t4[t], xq[j + t].at(b), a);
        x[b][j] = phi<false>(a);
        if constexpr (!kNorm) x[b][j] = bf16_lo(pack_bf16x2(x[b][j], 0.0f));
        den[j] = fmaf(x[b][j], z, den[j]);
      }
    }
    wave_lds_sync();  // the tile before is read
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int k = 0; k < C::NV; ++k) {
        unsigned char* p = stage + (8 * g + j) * kPitch + (k * 16 * V + V * n) * 2;
        if constexpr (V == 4)
          *reinterpret_cast<u32x2_t*>(p) = (u32x2_t){pack_bf16x2(x[4 * k][j], x[4 * k + 1][j]),
                                                     pack_bf16x2(x[4 * k + 2][j], x[4 * k + 3][j])};
        else
          *reinterpret_cast<uint32_t*>(p) = pack_bf16x2(x[0][j], x[1][j]);
      }
    wave_lds_sync();
    // o[t]: tokens 8 g + 4 t + i
    f32x4_t o[2][NMB];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int nb = 0; nb < NMB; ++nb) o[t][nb] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const u32x4_t a = *reinterpret_cast<const u32x4_t*>(
            stage + (8 * (n >> 2) + 4 * t + (n & 3)) * kPitch + (32 * ks + 8 * g) * 2);
#pragma unroll
        for (int nb = 0; nb < NMB; ++nb)
          o[t][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, ops[(nb * KS + ks) * 64 + lane]),
              o[t][nb], 0, 0, 0);
      }
    }
    const uint32_t off = row_off<float, D>(b0 + 8 * g, n);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float inv_den = __builtin_amdgcn_rcpf(sum_row16(den[j]));
      float y[NMB][4], ss = 0.0f;  // y[b][0]
#pragma unroll
      for (int b = 0; b < NMB; ++b) {
        y[b][0] = o[j >> 2][b][j & 3] * inv_den;
        ss = fmaf(y[b][0], y[b][0], ss);
      }
      if constexpr (kNorm) {
        const float scale = __builtin_amdgcn_rsqf(sum_row16(ss) * (1.0f / D) + P.eps);
#pragma unroll
        for (int b = 0; b < NMB; ++b) {
          const float r = xr[j].at(b);
          y[b][0] = y[b][0] * scale * gs[slot_chan<D>(b, n)] *
                    (r * __builtin_amdgcn_rcpf(1.0f + __expf(-r)));
        }
      }
      store_row<D>(ro, off + (uint32_t)(j * D * 4), y, 0);
    }
  }
}

}  // namespace

gbla_status launch_state_rows(const Plan& p, const void* k, const void* v, const void* a,
                              const float* conv_w, const int32_t* cu, float* partials,
                              hipStream_t st) {
  const dim3 grid(p.units, p.heads);
#define GBLA_STATE_ROWS(DD)                                                                     \
  hipLaunchKernelGGL((state_rows_kernel<DD>), grid, dim3(kThreads), 0, st, p, (const float*)k,  \
                     (const float*)v, (const float*)a, conv_w, cu, partials)
  if (p.d == 128) GBLA_STATE_ROWS(128);
  else if (p.d == 64) GBLA_STATE_ROWS(64);
  else GBLA_STATE_ROWS(32);
#undef GBLA_STATE_ROWS
  return hipGetLastError() == hipSuccess ? GBLA_OK : GBLA_ERR_HIP;
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

gbla_status launch_short_forward(const Plan& p, const void* q, const KeyInputs& in, const void* r,
                                 const float* conv_w, const float* gamma, const int32_t* cu,
                                 float* out, hipStream_t st, KernelEvents ev) {
  const dim3 grid((unsigned)((int64_t)p.nseq * p.heads));
#define GBLA_SHORT(TT, KERNEL)                                                                       \
  do {                                                                                               \
    const TT *qq = (const TT*)q, *kk = (const TT*)in.k, *vv = (const TT*)in.v, *aa = (const TT*)in.a, \
             *rr = (const TT*)r;                                                                     \
    if (ev.any())                                                                                    \
      hipExtLaunchKernelGGL(KERNEL, grid, dim3(kThreads), 0, st, ev.start, ev.stop, 0, p, qq, kk,    \
                            vv, aa, rr, conv_w, gamma, cu, out);                                     \
    else                                                                                             \
      hipLaunchKernelGGL(KERNEL, grid, dim3(kThreads), 0, st, p, qq, kk, vv, aa, rr, conv_w, gamma,  \
                         cu, out);                                                                   \
  } while (0)
  const bool norm = gamma != nullptr;  // NULL gamma: the no-gated-norm switch
  if (p.dtype == GBLA_BF16) {
    if (p.d == 64) { if (norm) GBLA_SHORT(uint16_t, (short_forward_bf16_kernel<64, true>)); else GBLA_SHORT(uint16_t, (short_forward_bf16_kernel<64, false>)); }
    else { if (norm) GBLA_SHORT(uint16_t, (short_forward_bf16_kernel<32, true>)); else GBLA_SHORT(uint16_t, (short_forward_bf16_kernel<32, false>)); }
  } else {
    if (p.d == 64) { if (norm) GBLA_SHORT(float, (short_forward_kernel<64, true>)); else GBLA_SHORT(float, (short_forward_kernel<64, false>)); }
    else { if (norm) GBLA_SHORT(float, (short_forward_kernel<32, true>)); else GBLA_SHORT(float, (short_forward_kernel<32, false>)); }
  }
#undef GBLA_SHORT
  return hipGetLastError() == hipSuccess ? GBLA_OK : GBLA_ERR_HIP;
}

}  // namespace gbla
