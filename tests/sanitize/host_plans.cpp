// Host-only driver for the sanitizer test: the plans and the argument checks
// of libgbla.so (gbla_plan.cpp, gbla_ext_plan.cpp, gbla_api.cpp), built with
// -fsanitize=address,undefined and the kernel launchers replaced by stubs
// that only count their calls.  Every shape below goes through the plan and
// workspace arithmetic; an overflow, out-of-bounds access or other undefined
// behaviour aborts the run.  Prints "host plans ok" at the end.
#include <limits.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include "gbla.h"
#include "gbla_ext.h"
#include "gbla_plan.h"

#define REQUIRE(cond)                                                          \
  do {                                                                         \
    if (!(cond)) {                                                             \
      fprintf(stderr, "host_plans: %s failed at line %d\n", #cond, __LINE__); \
      abort();                                                                 \
    }                                                                          \
  } while (0)

namespace gbla {
static int g_launches = 0;
gbla_status launch_conv(const Plan&, const void*, const void*, const void*, const float*,
                        const int32_t*, float*, float*, float*, hipStream_t) { ++g_launches; return GBLA_OK; }
gbla_status launch_state(const Plan& p, const void*, const void*, const void*, const float*,
                         const int32_t*, void*, float*, float*, float*, hipStream_t) {
  // the state and combine grids the real launcher builds
  REQUIRE(p.units >= 1 && p.heads >= 1 && (int64_t)p.nseq * p.heads <= INT32_MAX);
  ++g_launches;
  return GBLA_OK;
}
gbla_status launch_readout(const Plan& p, const void*, const void*, const float*, const float*,
                           const int32_t*, const void*, float*, hipStream_t, KernelEvents) {
  REQUIRE(p.runits >= 1 && p.heads >= 1);
  ++g_launches;
  return GBLA_OK;
}
gbla_status launch_backward(const Plan&, const BwdLayout&, const void*, const void*, const void*,
                            const void*, const void*, const float*, const float*, const int32_t*,
                            const float*, void*, float*, float*, float*, float*, float*, float*,
                            float*, hipStream_t) { ++g_launches; return GBLA_OK; }
gbla_status launch_project(const LayerPlan&, const void*, const float*, const void*,
                           const int32_t*, void*, void*, void*, void*, void*, void*, hipStream_t) {
  ++g_launches;
  return GBLA_OK;
}
}  // namespace gbla

extern "C" hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }

namespace {

// Stand-in device pointers: aligned, never dereferenced by host code.
alignas(256) unsigned char g_buf[1024];
void* A() { return g_buf; }
const float* F() { return reinterpret_cast<const float*>(g_buf); }
float* FO() { return reinterpret_cast<float*>(g_buf); }
const int32_t* CU() { return reinterpret_cast<const int32_t*>(g_buf); }

gbla_shape shape(int32_t B, int32_t H, int32_t n, int32_t d, int32_t W = 4, int32_t msl = 0,
                 int32_t dtype = GBLA_BF16, uint32_t flags = 0) {
  gbla_shape s;
  s.batch = B;
  s.heads = H;
  s.seqlen = n;
  s.head_dim = d;
  s.conv_width = W;
  s.max_seqlen = msl;
  s.dtype = dtype;
  s.eps = 1e-6f;
  s.flags = flags;
  return s;
}

void drive(const gbla_shape& s) {
  fprintf(stderr, "shape B=%d H=%d n=%d d=%d W=%d max=%d dtype=%d flags=%u\n", s.batch, s.heads,
          s.seqlen, s.head_dim, s.conv_width, s.max_seqlen, s.dtype, s.flags);
  const size_t fwd = gbla_workspace_bytes(&s);
  const size_t bwd = gbla_backward_workspace_bytes(&s);
  for (int ragged = 0; ragged < 2; ++ragged) {
    gbla::Plan p;
    if (gbla::make_plan(&s, ragged != 0, &p) == GBLA_OK) {
      REQUIRE(p.total_bytes <= fwd);  // the workspace size covers both readings
      gbla::Plan b;
      if (gbla::backward_plan(p, &b) == GBLA_OK) {
        const gbla::BwdLayout L = gbla::make_bwd_layout(b);
        REQUIRE(L.total_bytes <= bwd);
      }
    }
  }
  // The entry points check everything and then call the (stubbed) launchers;
  // a workspace size of SIZE_MAX passes the size check, so the arithmetic
  // behind each launch runs too.
  const int32_t* cu_opts[2] = {nullptr, CU()};
  for (const int32_t* cu : cu_opts) {
    (void)gbla_forward(&s, A(), A(), A(), A(), A(), F(), F(), cu, A(), SIZE_MAX, FO(), nullptr);
    (void)gbla_state(&s, A(), A(), A(), F(), cu, A(), SIZE_MAX, FO(), FO(), nullptr);
    (void)gbla_readout(&s, A(), A(), F(), F(), cu, A(), SIZE_MAX, FO(), nullptr);
    (void)gbla_conv1d(&s, A(), A(), A(), F(), cu, FO(), FO(), FO(), nullptr);
    (void)gbla_backward(&s, A(), A(), A(), A(), A(), F(), F(), cu, F(), A(), SIZE_MAX, FO(), FO(),
                        FO(), FO(), FO(), FO(), FO(), nullptr);
  }
}

void drive_layer(int32_t B, int32_t L, int32_t dm, int32_t H, int32_t d, int32_t msl = 0) {
  gbla_layer_shape s;
  s.batch = B;
  s.seqlen = L;
  s.d_model = dm;
  s.heads = H;
  s.head_dim = d;
  s.conv_width = 4;
  s.max_seqlen = msl;
  s.dtype = GBLA_BF16;
  s.eps = 1e-6f;
  (void)gbla_layer_workspace_bytes(&s);
  const int32_t* cu_opts[2] = {nullptr, CU()};
  for (const int32_t* cu : cu_opts) {
    (void)gbla_layer_project(&s, A(), F(), A(), cu, A(), SIZE_MAX, A(), A(), A(), A(), A(), nullptr);
    (void)gbla_layer_forward(&s, A(), F(), A(), F(), cu, A(), SIZE_MAX, FO(), nullptr);
  }
}

// Whether the forward of B sequences of n tokens takes one launch (dense), or
// does with max_seqlen = n over B * n packed tokens (ragged).
bool one_launch(bool ragged, int32_t B, int32_t H, int32_t n, int32_t d, int32_t dtype) {
  const gbla_shape s = shape(B, H, ragged ? B * n : n, d, 4, ragged ? n : 0, dtype);
  gbla::Plan p;
  REQUIRE(gbla::make_plan(&s, ragged, &p) == GBLA_OK);
  return gbla::short_forward(p);
}

void choices() {
  for (int r = 0; r < 2; ++r) {
    // short sequences, whatever their number
    REQUIRE(one_launch(r, 1, 1, 512, 64, GBLA_BF16) && one_launch(r, 3, 2, 1, 32, GBLA_BF16));
    REQUIRE(one_launch(r, 2, 2, 128, 64, GBLA_F32) && one_launch(r, 2, 2, 256, 32, GBLA_F32));
    REQUIRE(!one_launch(r, 1, 1, 513, 64, GBLA_BF16) && !one_launch(r, 2, 2, 129, 64, GBLA_F32));
    REQUIRE(!one_launch(r, 2, 2, 64, 128, GBLA_BF16) && !one_launch(r, 2, 2, 64, 128, GBLA_F32));
    // longer ones where the pairs are many
    REQUIRE(one_launch(r, 75, 4, 2048, 64, GBLA_BF16) && !one_launch(r, 74, 4, 2048, 64, GBLA_BF16));
    REQUIRE(one_launch(r, 75, 4, 1536, 32, GBLA_BF16) && !one_launch(r, 75, 4, 1537, 32, GBLA_BF16));
    REQUIRE(one_launch(r, 64, 4, 2048, 64, GBLA_F32) && !one_launch(r, 63, 4, 2048, 64, GBLA_F32));
    // and no sums over more tokens than the precision allows
    for (int32_t d = 32; d <= 64; d += 32) {
      REQUIRE(one_launch(r, 600, 4, 8192, d, GBLA_BF16) && !one_launch(r, 600, 4, 8193, d, GBLA_BF16));
      REQUIRE(one_launch(r, 600, 4, 2048, d, GBLA_F32) && !one_launch(r, 600, 4, 2049, d, GBLA_F32));
    }
  }
  // state units of the fp32 forward and units of the backward, by tokens x heads
  // (2691 x 24: records of 128-token units past the fixed scratch)
  const struct { int32_t T, H, d, fwd, bwd; } units[] = {
      {2691, 1, 64, 64, 64},      {2691, 13, 64, 128, 128},   {2691, 24, 64, 256, 128},  {2691, 49, 64, 1024, 512},
      {16383, 1, 64, 64, 64},     {32767, 1, 64, 64, 64},     {32768, 1, 64, 64, 128},   {65535, 1, 64, 128, 128},
      {65536, 1, 64, 128, 256},   {131072, 1, 64, 256, 512},  {16579, 5, 64, 256, 256},  {16579, 10, 64, 512, 512},
      {16579, 20, 64, 1024, 512}, {16579, 34, 64, 2048, 512}, {1 << 20, 8, 64, 2048, 512},
      {65536, 1, 32, 128, 128},   {2691, 98, 32, 1024, 512},  {65535, 4, 32, 512, 256},  {65536, 4, 32, 512, 512},
      {2691, 25, 128, 512, 512},  {65535, 1, 128, 256, 256},  {16383, 1, 128, 256, 64}};
  for (const auto& u : units) {
    const gbla_shape s = shape(13, u.H, u.T, u.d, 4, 2048, GBLA_F32);
    gbla::Plan p, b;
    REQUIRE(gbla::make_plan(&s, true, &p) == GBLA_OK && gbla::backward_plan(p, &b) == GBLA_OK);
    if (p.chunk != u.fwd || b.chunk != u.bwd) fprintf(stderr, "T %d H %d d %d: units %d, %d\n", u.T, u.H, u.d, p.chunk, b.chunk);
    REQUIRE(p.chunk == u.fwd && b.chunk == u.bwd);
  }
  // bf16 readout tiles at d = 128: no second round of 256 workgroups for shorter
  // tiles, where a batch of few tokens does not need one (shape: B, n, H; B packed
  // sequences of B * n tokens where n is negative)
  const struct { int32_t B, n, H, tile; } tiles[] = {
      {9, 971, 8, 512},  {1, 16000, 8, 512}, {1, 5000, 8, 256}, {8, 1000, 8, 256}, {4, 971, 8, 128}, {1, 4000, 8, 128},
      {24, 300, 8, 512}, {32, 200, 8, 512},  {1, 20000, 1, 128}, {24, -1027, 4, 256}, {30, -520, 3, 128},
      {1, 32768, 8, 512}};
  for (const auto& u : tiles) {
    const gbla_shape s = shape(u.B, u.H, u.n < 0 ? -u.n * u.B : u.n, 128);
    gbla::Plan p;
    REQUIRE(gbla::make_plan(&s, u.n < 0, &p) == GBLA_OK);
    if (p.rtile != u.tile) fprintf(stderr, "B %d n %d H %d: readout tile %d\n", u.B, u.n, u.H, p.rtile);
    REQUIRE(p.rtile == u.tile);
  }
  // longer units where one long sequence would have too many records
  const struct { int32_t T, longest, bwd; } long_units[] = {
      {10922, 10922, 64},  {10923, 10923, 128},  {30000, 0, 64},      {30000, 30000, 128},
      {43691, 43691, 256}, {60000, 2048, 64},    {60000, 60000, 256}, {60000, INT32_MAX, 256}};
  for (const auto& u : long_units) {
    const gbla_shape s = shape(u.longest == u.T ? 1 : 13, 1, u.T, 32, 4, u.longest);
    for (int r = u.longest == u.T ? 0 : 1; r < 2; ++r) {
      gbla::Plan p, b;
      REQUIRE(gbla::make_plan(&s, r != 0, &p) == GBLA_OK && gbla::backward_plan(p, &b) == GBLA_OK);
      if (b.chunk != u.bwd) fprintf(stderr, "T %d longest %d: units of %d\n", u.T, u.longest, b.chunk);
      REQUIRE(b.chunk == u.bwd);
    }
  }
}

}  // namespace

int main() {
  choices();
  const int32_t dims[3] = {32, 64, 128};
  for (int32_t d : dims) {
    for (int32_t W = 1; W <= 4; ++W) drive(shape(1, 8, 32768, d, W));
    drive(shape(1, 1, INT32_MAX, d));           // the longest sequence an int32 can name
    drive(shape(1, 1, INT32_MAX - 1, d, 4, INT32_MAX));
    drive(shape(INT32_MAX, 1, 1, d));           // the most sequences
    drive(shape(1, 65535, 32768, d));           // the most heads
    drive(shape(2, 65535, INT32_MAX, d));
    drive(shape(64, 8, 0, d, 4, 0));            // ragged batch of empty sequences
    drive(shape(64, 8, 1, d, 4, 1));            // ragged batch with a single token
    drive(shape(1, 1, 1, d, 1, 1, GBLA_F32));
    drive(shape(8, 8, 2048, d, 4, 0, GBLA_F32, GBLA_BLA));
    drive(shape(8, 8, 2048, d, 4, 0, GBLA_BF16, GBLA_NO_GATE | GBLA_NO_NORM));
  }
  // invalid shapes are refused before any arithmetic
  drive(shape(0, 8, 1, 64));
  drive(shape(1, 0, 1, 64));
  drive(shape(1, 8, -1, 64));
  drive(shape(1, 65536, 1, 64));
  drive(shape(1, 8, 1, 48));
  drive(shape(1, 8, 1, 64, 5));
  drive(shape(1, 8, 1, 64, 4, -1));
  // layers: widest embeddings, most heads, longest sequences the 32-bit offsets allow
  drive_layer(8, 32768, 1024, 16, 64);
  drive_layer(1, 1, 16384, 1, 128);
  drive_layer(1, 65536, 16384, 4, 64);
  drive_layer(1, INT32_MAX, 64, 1, 32);
  drive_layer(64, 4096, 64, 65535, 32);
  drive_layer(3, 0, 1024, 16, 64, 0);
  drive_layer(3, 1, 1024, 16, 64, 1);
  drive_layer(1, 8, 16448, 4, 64);  // d_model beyond the supported range: refused
  printf("host plans ok (%d stub launches)\n", gbla::g_launches);
  return 0;
}
