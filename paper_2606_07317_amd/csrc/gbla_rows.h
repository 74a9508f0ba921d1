// gbla_rows.h -- device helpers of the fp32 forward and of the one-launch
// forward: rows of a tensor held channel-major in registers, so that every
// product of the fp32 kernels runs on v_mfma_f32_16x16x4_f32 with fp32 operands.
//
// Channel layout.  A wave works on a tile of 16 consecutive tokens.  Lane (n,
// g) = (lane & 15, lane >> 4) holds the D/16 channels slot_chan(b, n), b < D/16, of
// the four consecutive tokens 4 g + i, i < 4.
//   - The conv window of its tokens is the lane's own seven rows (three of
//     them loaded again from L1), so the conv slides through
//     registers with no cross-lane traffic.  A layout with one token per lane
//     needed two DPP moves per tap and channel: 12 vector instructions per
//     element against 6.
//   - Per-channel sums over tokens (z) take one accumulator per channel slot:
//     D/16 a lane instead of D/4.
//   - Token sums (S) take the values as MFMA operands directly: in K step
//     i, lane group g supplies token 4 g + i.
//   - Channel sums need one token per lane: the tile goes through the wave's
//     own LDS stage (contract_rows), whose product comes out in the channel
//     layout again, because the tokens are the M index.
// slot_chan gives a lane V consecutive channels, so a tile's rows are read and
// written with 4- to 16-byte accesses, sixteen lanes to a row.
// What bounds these kernels: v_mfma_f32_16x16x4_f32 and the vector unit share
// a SIMD without overlapping (measured, per SIMD: 15 ns a product and 2.1 ns a
// vector instruction with one wave, 14.3 and 1.2-1.5 ns with two; a wave of
// products beside a wave of vector work takes the sum), so a tile costs the sum
// of both and vector instructions are what a layout can save.
#pragma once

#include "gbla_device.h"

namespace gbla {

template <int D>
struct CL {
  static constexpr int NMB = D / 16;            // channels per lane
  static constexpr int V = D == 32 ? 2 : 4;     // consecutive channels
  static constexpr int NV = NMB / V;            // vectors per row
  static constexpr int SH = D > 64 ? 64 : D;    // channels staged at a time
  static constexpr int NH = D / SH;
  // row pitch of the stage: rows start four banks apart, so the sixteen rows
  // of a 16-byte read cover the 64 banks
  static constexpr int kPitch = SH + 4;
  static constexpr int kStage = 16 * kPitch;    // floats, per wave
  static constexpr int kBlocks = NMB * NMB;     // 16x16 blocks of a D x D result
  static constexpr int kFrag = kBlocks * 64;    // f32x4 operand vectors of a D x D matrix
};

template <int D>
__device__ __forceinline__ constexpr int slot_chan(int b, int n) {
  constexpr int V = CL<D>::V;
  return (b / V) * (16 * V) + V * n + b % V;
}

// Tokens of a wave's quarter of a unit of `tokens` tokens, in whole tiles.
__device__ __forceinline__ int quarter_tokens(int tokens) { return ((tokens + 3) / 4 + 15) / 16 * 16; }

// Orders a wave's LDS stores before its later LDS loads of other lanes'
// slots (one wave's LDS operations complete in order; this keeps the
// compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ f32x4_t mfma4(float a, float b, f32x4_t acc) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
}

// One row's channels of a lane as loaded (bf16 pairs or fp32), widened where
// they are used.
template <typename T, int D>
struct Row {
  static constexpr int kBytes = CL<D>::V * (int)sizeof(T);  // of one vector
  static constexpr int kW = kBytes / 4;
  uint32_t w[CL<D>::NV * kW];
  // off: byte offset of the lane's first channel of the row
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
#pragma unroll
    for (int v = 0; v < CL<D>::NV; ++v) {
      const uint32_t o = off + (uint32_t)(v * 16 * kBytes);
      if constexpr (kW == 1) {
        w[v] = __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
      } else if constexpr (kW == 2) {
        const u32x2_t x = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
        w[2 * v] = x[0];
        w[2 * v + 1] = x[1];
      } else {
        const u32x4_t x = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
#pragma unroll
        for (int k = 0; k < 4; ++k) w[4 * v + k] = x[k];
      }
    }
  }
  __device__ __forceinline__ float at(int b) const {
    if constexpr (sizeof(T) == 4) return __uint_as_float(w[b]);
    else return b & 1 ? bf16_hi(w[b >> 1]) : bf16_lo(w[b >> 1]);
  }
};

// Byte offset of the lane's first channel of token `tok` of a slice.
template <typename T, int D>
__device__ __forceinline__ uint32_t row_off(int tok, int n) {
  return (uint32_t)(tok * D + CL<D>::V * n) * (uint32_t)sizeof(T);
}

// The conv windows of a lane's four tokens tok .. tok + 3: rows tok - 3 ..
// tok + 3 (rows outside the slice read 0).
template <typename T, int D>
struct Window {
  Row<T, D> x[7];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int tok, int n) {
    const uint32_t off = row_off<T, D>(tok, n);
#pragma unroll
    for (int k = 0; k < 7; ++k) x[k].load(r, off + (uint32_t)((k - 3) * D * (int)sizeof(T)));
  }
  // out[b][i] = sum_t taps(b)[t] x_{tok + i - 3 + t}[slot_chan(b, n)]
  template <typename Taps>
  __device__ __forceinline__ void conv(const Taps& taps, float (*out)[4]) const {
#pragma unroll
    for (int b = 0; b < CL<D>::NMB; ++b) {
      const f32x4_t w = taps(b);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float acc = w[0] * x[i].at(b);
#pragma unroll
        for (int t = 1; t < 4; ++t) acc = fmaf(w[t], x[i + t].at(b), acc);
        out[b][i] = acc;
      }
    }
  }
};

// Stores v[.][i] as row `off` of an fp32 tensor.
template <int D>
__device__ __forceinline__ void store_row(__amdgpu_buffer_rsrc_t r, uint32_t off, const float (*v)[4],
                                          int i) {
  constexpr int V = CL<D>::V;
#pragma unroll
  for (int k = 0; k < CL<D>::NV; ++k) {
    const uint32_t o = off + (uint32_t)(k * 16 * V * 4);
    if constexpr (V == 4) {
      const f32x4_t x = {v[4 * k][i], v[4 * k + 1][i], v[4 * k + 2][i], v[4 * k + 3][i]};
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, x), r, o, 0, 0);
    } else {
      const f32x2_t x = {v[2 * k][i], v[2 * k + 1][i]};
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, x), r, o, 0, 0);
    }
  }
}

// Puts / gets vector k (channels V n .. of the k-th run of 16 V) of v[.][i]
// at p.
template <int D>
__device__ __forceinline__ void put_vec(float* p, const float (*v)[4], int k, int i) {
  if constexpr (CL<D>::V == 4)
    *reinterpret_cast<f32x4_t*>(p) = (f32x4_t){v[4 * k][i], v[4 * k + 1][i], v[4 * k + 2][i], v[4 * k + 3][i]};
  else
    *reinterpret_cast<f32x2_t*>(p) = (f32x2_t){v[2 * k][i], v[2 * k + 1][i]};
}
template <int D>
__device__ __forceinline__ void get_vec(const float* p, float* v) {
  if constexpr (CL<D>::V == 4) {
    const f32x4_t x = *reinterpret_cast<const f32x4_t*>(p);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = x[j];
  } else {
    const f32x2_t x = *reinterpret_cast<const f32x2_t*>(p);
    v[0] = x[0];
    v[1] = x[1];
  }
}

// Sum over the sixteen lanes of a lane group (the channels of a token), in
// every lane; the same bits in each (the rotations pair the same sums).
__device__ __forceinline__ float sum_row16(float x) {
#define GBLA_ROR_ADD(N) \
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xF, 0xF, true))
  GBLA_ROR_ADD(8);
  GBLA_ROR_ADD(4);
  GBLA_ROR_ADD(2);
  GBLA_ROR_ADD(1);
#undef GBLA_ROR_ADD
  return x;
}

// Sum over the four lane groups.
__device__ __forceinline__ float sum_groups(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// B operand vectors of a D x D matrix X[k][col] for contract_rows: vector
// (nb * NMB + kq) * 64 + lane holds X[16 kq + 4 g + i][slot_chan(nb, n)],
// i < 4.  A thread has kPer of them, number u at index threadIdx.x + u
// kThreads.
template <int D>
struct Frags {
  static constexpr int kPer = CL<D>::kFrag / kThreads;
  f32x4_t v[kPer];
  static __device__ __forceinline__ int k0(int u) {
    const int idx = threadIdx.x + u * kThreads;
    return 16 * ((idx >> 6) % CL<D>::NMB) + 4 * ((idx >> 4) & 3);
  }
  static __device__ __forceinline__ int col(int u) {
    const int idx = threadIdx.x + u * kThreads;
    return slot_chan<D>((idx >> 6) / CL<D>::NMB, idx & 15);
  }
  __device__ __forceinline__ void put(f32x4_t* frag) const {
#pragma unroll
    for (int u = 0; u < kPer; ++u) frag[threadIdx.x + u * kThreads] = v[u];
  }
};

// acc[nb][i] += sum_k v(token 4 g + i)[k] X[k][slot_chan(nb, n)]: the channel sum
// of a tile, v in the channel layout.  The tile is staged in the wave's own
// LDS area (64 channels at a time) and read back with one token per lane as
// the A operand.
template <int D>
__device__ __forceinline__ void contract_rows(const float (*v)[4], float* stage, const f32x4_t* frag,
                                              int lane, f32x4_t* acc) {
  using C = CL<D>;
  constexpr int NMB = C::NMB, KQ = C::SH / 16;
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int hf = 0; hf < C::NH; ++hf) {
    wave_lds_sync();  // earlier reads of the stage are done
#pragma unroll
    for (int i = 0; i < 4; ++i) put_vec<D>(stage + (4 * g + i) * C::kPitch + C::V * n, v, hf, i);
    wave_lds_sync();
// at d = 128 the K steps are not unrolled, so that their operand reads are
// not all hoisted into registers at once
#pragma unroll D >= 128 ? 1 : KQ
    for (int kq = 0; kq < KQ; ++kq) {
      const f32x4_t a = *reinterpret_cast<const f32x4_t*>(stage + n * C::kPitch + 16 * kq + 4 * g);
      f32x4_t b[NMB];
#pragma unroll
      for (int nb = 0; nb < NMB; ++nb) b[nb] = frag[(nb * NMB + hf * KQ + kq) * 64 + lane];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int nb = 0; nb < NMB; ++nb) acc[nb] = mfma4(a[i], b[nb][i], acc[nb]);
    }
  }
}

// acc[mb * NMB + nb] += sum over the tile's tokens of x[slot_chan(mb, .)] y[slot_chan(nb, .)].
template <int D>
__device__ __forceinline__ void token_product(const float (*x)[4], const float (*y)[4], f32x4_t* acc) {
  constexpr int NMB = CL<D>::NMB;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NMB; ++nb)
        acc[mb * NMB + nb] = mfma4(x[mb][i], y[nb][i], acc[mb * NMB + nb]);
}

// buf0[c * D + e] = w0 + w1, buf1[c * D + e] = w2 + w3 of the four waves' token
// products.  buf0, buf1: D^2 floats of LDS each, free to use.  Every thread
// calls; the last step is a barrier.
template <int D>
__device__ __forceinline__ void put_waves(const f32x4_t* acc, float* buf0, float* buf1) {
  using C = CL<D>;
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  float* half = wave >> 1 ? buf1 : buf0;
  // slot (mb, i, k): row slot_chan(mb, 4 g + i), columns of vector k
#pragma unroll
  for (int phase = 0; phase < 2; ++phase) {
    if ((wave & 1) != phase) {
#pragma unroll
      for (int mb = 0; mb < C::NMB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int k = 0; k < C::NV; ++k) {
            float* p = half + slot_chan<D>(mb, 4 * g + i) * D + k * 16 * C::V + C::V * n;
            float x[C::V];
            if (phase == 1) get_vec<D>(p, x);
#pragma unroll
            for (int j = 0; j < C::V; ++j) {
              const float v = acc[mb * C::NMB + k * C::V + j][i];
              x[j] = phase == 1 ? v + x[j] : v;
            }
            if constexpr (C::V == 4)
              *reinterpret_cast<f32x4_t*>(p) = (f32x4_t){x[0], x[1], x[2], x[3]};
            else
              *reinterpret_cast<f32x2_t*>(p) = (f32x2_t){x[0], x[1]};
          }
    }
    __syncthreads();
  }
}
// dst[c * D + e] = (w0 + w1) + (w2 + w3).
template <int D>
__device__ __forceinline__ void sum_waves(const f32x4_t* acc, float* buf0, float* buf1,
                                          float* __restrict__ dst) {
  put_waves<D>(acc, buf0, buf1);
  for (int x = 4 * threadIdx.x; x < D * D; x += 4 * kThreads)
    *reinterpret_cast<f32x4_t*>(dst + x) = *reinterpret_cast<const f32x4_t*>(buf0 + x) +
                                           *reinterpret_cast<const f32x4_t*>(buf1 + x);
}

// Sums per-lane channel accumulators over the lane groups and the waves in a
// fixed order and writes the D sums to dst.  red: 4 x D floats of LDS.  Every
// thread calls.
template <int D>
__device__ __forceinline__ void sum_channels(const float* v, float (*red)[D], float* __restrict__ dst) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int b = 0; b < CL<D>::NMB; ++b) {
    const float s = sum_groups(v[b]);
    if (g == 0) red[wave][slot_chan<D>(b, n)] = s;
  }
  __syncthreads();
  if (threadIdx.x < D) {
    const int x = threadIdx.x;
    dst[x] = (red[0][x] + red[1][x]) + (red[2][x] + red[3][x]);
  }
  __syncthreads();
}

// Taps of a lane's channel slot b, read from LDS where they are used.
template <int D>
struct LdsTaps {
  const f32x4_t* t;  // slot order: slot 16 b + n holds channel slot_chan(b, n)
  int n;
  __device__ __forceinline__ f32x4_t operator()(int b) const { return t[16 * b + n]; }
};

// Taps of one tensor into LDS in LdsTaps' order.
template <int D>
__device__ __forceinline__ void stage_taps(const float* conv_w, int H, int h, int tensor, int W,
                                           f32x4_t* taps) {
  const int t = threadIdx.x;
  if (t < D) {
    float w4[4];
    load_taps4(conv_w, H, h, tensor, D, W, slot_chan<D>(t >> 4, t & 15), w4);
    taps[t] = (f32x4_t){w4[0], w4[1], w4[2], w4[3]};
  }
}

}  // namespace gbla
