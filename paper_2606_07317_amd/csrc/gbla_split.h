// gbla_split.h -- device helpers of the backward's kernels: products of fp32
// operands on the bf16 matrix instructions, each operand split into three bf16
// parts.
//
// x = h + m + l with h, m, l bf16 (8 + 8 + 8 significant bits, rounded to
// nearest, so the remainders are signed and the third part is exact).  Of the
// nine products of two operands m l, l m and l l are left out: m l and l m are
// up to 2^-25 of the product each, 2^-24 together, about the rounding of one
// fp32 product.
// The split is exact from about 2^-109 to bf16's largest value, 3.39e38.  Below,
// the smaller parts leave bf16's normal range and the operand keeps fewer bits.
// An infinite operand, or one that rounds to bf16's infinity, has NaN for its
// remainders (inf - inf), so every product that it enters is NaN where fp32
// products are infinite (or NaN, with a zero); sequences and heads other than its
// own are not touched.
// v_mfma_f32_16x16x32_bf16 takes 7.9 ns a SIMD and runs beside the vector unit
// (two vector instructions hide under each), v_mfma_f32_16x16x4_f32 takes 15 ns
// and does not: 32 K steps cost 47 ns as six bf16 products and 120 ns in fp32.
//
// Work layout.  A workgroup has D/16 waves and goes through its unit 32 tokens
// at a time, all waves on the same tokens; wave w owns channels 16 w .. 16 w +
// 15, lane (n, g) = (lane & 15, lane >> 4) channel 16 w + n of the eight
// consecutive tokens 8 g + j.  So a wave's part of a constant D x D operand is
// 16 columns and stays in its registers (a whole operand in three parts would
// not fit the LDS), the D x D sums over tokens take D/4 accumulators a lane, and
// the convs slide through registers.  What every wave needs of the others'
// channels goes through LDS in planes:
//   plane p of an operand: [channel][32 tokens] bf16 token
//   8 g + 4 t + i at position 16 t + 4 g + i.
// A product over channels reads the planes transposed (ds_read_b64_tr_b16, one
// token per lane); its two 16-row results are tokens 8 g + 4 t + i of a lane,
// its own eight.
#pragma once

#include <type_traits>

#include "gbla_device.h"

namespace gbla {

template <int D>
struct SP {
  static constexpr int NW = D / 16;           // waves
  static constexpr int NT = 64 * NW;
  static constexpr int KS = D / 32;           // K steps of a product over channels
  // Rows of 64 bytes, their 16-byte units at unit ^ (row / 4 % 4), so that the
  // four rows of a transposed read and the four that the lane groups beside it
  // read lie on distinct banks.  The 16-byte accesses still meet: conflict cycles
  // per LDS instruction at d = 64 are 3.5 in the state kernel, which has no
  // others, 1.0 in the query kernel and 0.7 in the key kernel.  (Rows 80 bytes
  // apart without the swizzle: two cycles of conflict to three of access in the
  // query kernel, and 61 KB instead of 49 for two operands at d = 128.)
  static constexpr int kPitch = 64;
  static constexpr int kPlane = D * kPitch;
  static constexpr int kOperand = 3 * kPlane;  // bytes of the three planes
};

// Byte offset in a plane of the 16-byte unit u of row r.
__device__ __forceinline__ int plane_unit(int r, int u) { return r * 64 + ((u ^ ((r >> 2) & 3)) << 4); }

// Two fp32 values as packed bf16 parts.
__device__ __forceinline__ void split3(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = pack_bf16x2(a, b);
  const float ra = a - bf16_lo(h), rb = b - bf16_hi(h);
  m = pack_bf16x2(ra, rb);
  l = pack_bf16x2(ra - bf16_lo(m), rb - bf16_hi(m));
}

__device__ __forceinline__ f32x4_t mfma_bf16(u32x4_t a, u32x4_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// hi += A_h B_h, lo += the five smaller products.
__device__ __forceinline__ void mfma_split(const u32x4_t* a, const u32x4_t* b, f32x4_t& hi, f32x4_t& lo) {
  lo = mfma_bf16(a[2], b[0], lo);
  hi = mfma_bf16(a[0], b[0], hi);
  lo = mfma_bf16(a[0], b[2], lo);
  lo = mfma_bf16(a[1], b[1], lo);
  lo = mfma_bf16(a[1], b[0], lo);
  lo = mfma_bf16(a[0], b[1], lo);
}

// A B of one K step, formed from zero (the smaller products first).  Sums over
// many steps add this to their accumulator, one rounding a step: six products
// chained onto the accumulator doubled the error of 512-token sums.  The matrix
// unit's own sums of 32 products are not rounded to nearest, so such a sum also
// takes the sign of its first operand the other way round every second step
// (acc -= (-A) B), which lets those errors cancel: without it the gradients'
// error at n = 32768 was 1.3 to 2.3 times that of fp32 products.
__device__ __forceinline__ f32x4_t step_product(const u32x4_t* a, const u32x4_t* b) {
  f32x4_t c = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  c = mfma_bf16(a[2], b[0], c);
  c = mfma_bf16(a[0], b[2], c);
  c = mfma_bf16(a[1], b[1], c);
  c = mfma_bf16(a[1], b[0], c);
  c = mfma_bf16(a[0], b[1], c);
  return mfma_bf16(a[0], b[0], c);
}

__device__ __forceinline__ u32x2_t tr_read16(const unsigned char* p) {
  typedef short v4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(
      u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4*)(p)));
}

// Splits the lane's eight values and writes them to row `row` of the planes.
template <int D>
__device__ __forceinline__ void put_planes(unsigned char* planes, int row, int g, const float* v) {
  u32x4_t q[3];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    uint32_t h, m, l;
    split3(v[2 * p], v[2 * p + 1], h, m, l);
    q[0][p] = h;
    q[1][p] = m;
    q[2][p] = l;
  }
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    unsigned char* d = planes + x * SP<D>::kPlane + 8 * (g & 1);
    *reinterpret_cast<u32x2_t*>(d + plane_unit(row, g >> 1)) = (u32x2_t){q[x][0], q[x][1]};
    *reinterpret_cast<u32x2_t*>(d + plane_unit(row, 2 + (g >> 1))) = (u32x2_t){q[x][2], q[x][3]};
  }
}

// A wave's 16 columns of a constant operand: part x, K step ks: eight values
// X[32 ks + 8 g + i][column n].
template <int D>
struct Columns {
  u32x4_t v[SP<D>::KS][3];
  __device__ __forceinline__ void get(int ks, u32x4_t* b) const {
#pragma unroll
    for (int x = 0; x < 3; ++x) b[x] = v[ks][x];
  }
  __device__ __forceinline__ void set(int ks, const float* x8) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t h, m, l;
      split3(x8[2 * p], x8[2 * p + 1], h, m, l);
      v[ks][0][p] = h;
      v[ks][1][p] = m;
      v[ks][2][p] = l;
    }
  }
};

// The same with the two smaller parts in LDS, where the registers are full.
template <int D>
struct ColumnsLds {
  u32x4_t h[SP<D>::KS];
  u32x4_t* lds;  // [2][KS][NT], the lane's slots at threadIdx.x
  __device__ __forceinline__ void set(int ks, const float* x8) {
    u32x4_t m, l;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t a, b, c;
      split3(x8[2 * p], x8[2 * p + 1], a, b, c);
      h[ks][p] = a;
      m[p] = b;
      l[p] = c;
    }
    lds[ks * SP<D>::NT + threadIdx.x] = m;
    lds[(SP<D>::KS + ks) * SP<D>::NT + threadIdx.x] = l;
  }
  __device__ __forceinline__ void get(int ks, u32x4_t* b) const {
    b[0] = h[ks];
    b[1] = lds[ks * SP<D>::NT + threadIdx.x];
    b[2] = lds[(SP<D>::KS + ks) * SP<D>::NT + threadIdx.x];
  }
};

// out[4 t + i] = sum_k planes(token 8 g + 4 t + i)[k] X[k][n].
template <int D, typename Cols>
__device__ __forceinline__ void contract_planes(const unsigned char* planes, const Cols& X, int lane,
                                                float* out) {
  using C = SP<D>;
  const int g = lane >> 4, j = lane & 15;
  // rows 32 ks + 8 g + j / 4 and four on, units 2 t + j / 2 % 2
  const int u = (j >> 1) & 1, r = 8 * g + (j >> 2), o = 8 * (j & 1);
  const unsigned char* base[2][2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int q = 0; q < 2; ++q) base[t][q] = planes + plane_unit(r + 4 * q, 2 * t + u) + o;
  f32x4_t hi[2], lo[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) hi[t] = lo[t] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int ks = 0; ks < C::KS; ++ks) {
    u32x4_t b[3];
    X.get(ks, b);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      u32x4_t a[3];
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        const int at = x * C::kPlane + 32 * ks * C::kPitch;
        const u32x2_t u0 = tr_read16(base[t][0] + at), u1 = tr_read16(base[t][1] + at);
        a[x] = (u32x4_t){u0[0], u0[1], u1[0], u1[1]};
      }
      mfma_split(a, b, hi[t], lo[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) out[4 * t + i] = hi[t][i] + lo[t][i];
}

// The eight token values of row `row` that K step positions 8 g .. 8 g + 7 hold.
template <int D>
__device__ __forceinline__ void row_operand(const unsigned char* planes, int row, int g, u32x4_t* v) {
#pragma unroll
  for (int x = 0; x < 3; ++x)
    v[x] = *reinterpret_cast<const u32x4_t*>(planes + x * SP<D>::kPlane + plane_unit(row, g));
}

// One channel of one token as loaded.
template <typename T>
__device__ __forceinline__ uint32_t load_elem(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(T) == 4) return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
  else return (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
}
template <typename T>
__device__ __forceinline__ float widen(uint32_t w) {
  if constexpr (sizeof(T) == 4) return __uint_as_float(w);
  else return __uint_as_float(w << 16);
}

// The conv windows of a lane's eight tokens tok .. tok + 7 of its channel: rows
// tok - 3 .. tok + 7 (rows outside the slice read 0).
template <typename T, int D>
struct Column {
  uint32_t x[11];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int tok, int c) {
    const uint32_t off = (uint32_t)(tok * D + c) * (uint32_t)sizeof(T);
#pragma unroll
    for (int k = 0; k < 11; ++k) x[k] = load_elem<T>(r, off + (uint32_t)((k - 3) * D * (int)sizeof(T)));
  }
  __device__ __forceinline__ float at(int k) const { return widen<T>(x[k]); }
  // out[j] = sum_t w[t] x_{tok + j - 3 + t}
  __device__ __forceinline__ void conv(const float* w, float* out) const {
    float f[11];
#pragma unroll
    for (int k = 0; k < 11; ++k) f[k] = at(k);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float a = w[0] * f[j];
#pragma unroll
      for (int t = 1; t < 4; ++t) a = fmaf(w[t], f[j + t], a);
      out[j] = a;
    }
  }
};

// Sums over the sixteen lanes of a group of eight values: lane n receives the
// total of value n >> 1.  Halving exchanges (8 + 4 + 2 values) and one last
// pair: 22 instructions, where eight full sums by rotation take 32.
template <int kCtrl>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, true));
}
__device__ __forceinline__ float scatter_sum8(const float* v, int n) {
  float a[4], b[2];
  const bool h8 = n & 8, h4 = n & 4, h2 = n & 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = (h8 ? v[4 + i] : v[i]) + dpp<0x128>(h8 ? v[i] : v[4 + i]);  // lane n ^ 8
#pragma unroll
  for (int i = 0; i < 2; ++i) b[i] = (h4 ? a[2 + i] : a[i]) + dpp<0x141>(h4 ? a[i] : a[2 + i]);  // lane n ^ 7
  const float s = (h2 ? b[1] : b[0]) + dpp<0x4E>(h2 ? b[0] : b[1]);                              // lane n ^ 2
  return s + dpp<0xB1>(s);                                                                       // lane n ^ 1
}

// In a sequence's last tile (`Tail` true) zeros for a lane's tokens from the
// live-th on (live may be negative or over 8).  The kernels walk that tile in a
// copy of its own: with branches around these selects in one loop the backward
// took 2.4% longer (n = 32768, H = 8, d = 64 176 us, 180).
template <typename Tail>
__device__ __forceinline__ void zero_past(Tail, int live, float* v) {
  if constexpr (Tail::value) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = j < live ? v[j] : 0.0f;
  }
}

// The conv's transpose for a lane's eight tokens: dx_j = sum_t w_t d_{j+3-t}, and
// the tap sums dw_t += d_j x_{j-3+t}.  Units are walked from their last tile to
// their first: `prev` holds the first three values of the tile done before
// (lanes of group 0), which are the three tokens after this tile.  In a
// sequence's last tile the tap sums take the lane's first `live` tokens: d is
// zero past them, but x may be infinite.
template <typename T, int D, typename Tail>
__device__ __forceinline__ void conv_back8(const float* d, const Column<T, D>& x, const float* w, float* prev,
                                           int lane, Tail, int live, __amdgpu_buffer_rsrc_t out, uint32_t off, float* dw) {
  float e[11];
#pragma unroll
  for (int j = 0; j < 8; ++j) e[j] = d[j];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float give = lane < 16 ? prev[i] : d[i];
    e[8 + i] = __shfl(give, (lane + 16) & 63);
    prev[i] = d[i];
  }
  float t4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float y = w[3] * e[j];
    y = fmaf(w[2], e[j + 1], y);
    y = fmaf(w[1], e[j + 2], y);
    y = fmaf(w[0], e[j + 3], y);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y), out, off + (uint32_t)(j * D * 4), 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) t4[t] = fmaf(d[j], !Tail::value || j < live ? x.at(j + t) : 0.0f, t4[t]);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) dw[t] += t4[t];  // a tile at a time, as all sums over a unit
}

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace gbla
