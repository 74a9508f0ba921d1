// gbla_plan.cpp -- the launch plan of the attention pass: split sizes and the
// workspace layout, a function of the shape alone.
#include <math.h>
#include <stdint.h>

#include "gbla.h"
#include "gbla_plan.h"

namespace gbla {
namespace {

constexpr int kMaxGridY = 65535;
constexpr int64_t kMaxGridX = 2147483647LL;
constexpr int kReadoutTile = 512;

int64_t next_pow2(int64_t x) {
  int64_t p = 1;
  while (p < x) p <<= 1;
  return p;
}

// Offsets and size of the workspace for `units` partial records per head.
void set_workspace(Plan* q, int64_t units) {
  const size_t part_bytes = (size_t)units * q->heads * q->rec_floats * sizeof(float);
  q->off_frags = align_up(q->off_partials + part_bytes, 256);
  q->total_bytes = align_up(q->off_frags + (size_t)q->nseq * q->heads * q->frag_bytes, 256);
}

// Shorter readout tiles, down to `least` tokens, while the work would not fill
// 256 workgroups; never so many that the grid would refuse the batch.
void halve_rtile(Plan* q, int32_t least) {
  while (q->rtile > least && q->tokens * q->heads < (int64_t)q->rtile * 256 &&
         q->tokens / (q->rtile / 2) + q->nseq <= kMaxGridX)
    q->rtile /= 2;
}

// Readout tile of the bf16 kernel at d = 128, where one workgroup runs on a CU:
// of the tiles that halve_rtile would go through, the one whose rounds of 256
// workgroups take least.  A round is its longest tile and about 105 tokens of
// set-up (4 us; 0.038 us a token).  Whole forward in us, tiles of 512 / 256 / 128,
// H = 8: B = 9, n = 971 57 / 61 / -; B = 1, n = 16000 67 / 74 / -; B = 1, n = 5000 48
// / 38 / 42; B = 4, n = 971 48 / 39 / 34; B = 24, n = 300 62 / 71 / 69; packed, 24
// sequences, T = 24,659, H = 4 103 / 88 / -; 30, T = 15,617, H = 3 71 / 74 / 66.
void rtile_by_rounds(Plan* q) {
  int64_t best = -1;
  int32_t tile = q->rtile;
  for (int32_t t = q->rtile; t >= 128; t /= 2) {
    if (q->tokens / t + q->nseq > kMaxGridX) break;  // the grid would refuse the batch
    const int64_t units = q->ragged ? q->tokens / t + q->nseq : (int64_t)q->nseq * (((int64_t)q->rows + t - 1) / t);
    const int64_t longest = !q->ragged && q->rows < t ? q->rows : t;
    const int64_t cost = (units * q->heads + 255) / 256 * (longest + 105);
    if (best < 0 || cost < best) {
      best = cost;
      tile = t;
    }
    if (q->tokens * q->heads >= (int64_t)t * 256) break;
  }
  q->rtile = tile;
}

// Split of the fp32 kernels, whose workgroups are smaller (four waves, two
// workgroups per CU up to d = 64).  Small batches are cut finer: state units
// of down to 64 tokens, readout tiles of down to 64 (whole forward, chunk 256 /
// tile 512 against this rule: n = 256, H = 2, d = 32 19.4 against 15.1 us;
// n = 1000, H = 4, d = 64 43.7 / 21.7; B = 2, n = 8191, H = 8, d = 64 66.8 /
// 64.6).  At d = 128 a record is 66 KB and the units stay as they are (B = 8,
// n = 2048, H = 8: 176 us, 201 with twice as many).  More records than the
// fixed scratch of gbla_forward_noalloc holds are not taken for this, so that
// the call accepts every shape that it does with the coarser split.
void fp32_split(Plan* q) {
  const int64_t work = q->tokens * q->heads;
  halve_rtile(q, 64);
  if (q->d == 128) return;
  int64_t chunk = next_pow2((work + 511) / 512);
  if (chunk < 64) chunk = 64;
  if (chunk >= q->chunk) return;
  Plan t = *q;
  set_workspace(&t, t.tokens / chunk + t.nseq);
  if (t.total_bytes <= GBLA_NOALLOC_SCRATCH_BYTES) q->chunk = (int32_t)chunk;
}

}  // namespace

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

bool rows_supported(const Plan& p) {
  // 32-bit buffer offsets: every fp32 (sequence, head) slice below 2^31 bytes
  return p.chunk <= kMaxChunk && p.chunk % 64 == 0 && p.rtile % 64 == 0 &&
         (int64_t)p.rows * p.d * 4 < (int64_t(1) << 31);
}

// The one-launch forward gives each (sequence, head) one workgroup, so its time
// is at least the longest sequence's (bf16 d = 64: 5 us + 0.037 us a token, half
// of that at d = 32; fp32 about twice), while three launches spread long
// sequences over the chip but take 14 to 25 us for any batch.  So: lengths up to
// a first bound, or batches of so many pairs that the longest sequence is a small
// part of the chip's work.  Whole forward in us, one launch / three:
//   first bound, H = 8: bf16 d = 64 B = 1 n = 256 15 / 24, B = 2 n = 512 24 / 26,
//   B = 1 n = 1024 42 / 26; fp32 d = 64 n = 128 16 / 18, n = 256 26 / 19; d = 32
//   n = 256 14 / 14, n = 512 23 / 15.
//   bf16 d = 64: 256 pairs n = 1024 56 / 41; 304 n = 1024 66 / 79, n = 2048 138 /
//   143, n = 3000 202 / 199; 384 n = 3000 214 / 229, n = 4096 281 / 292, n = 8192
//   567 / 537; 512 n = 8192 664 / 710.
//   bf16 d = 32: 304 n = 1400 49 / 53, n = 2048 68 / 63; 352 n = 2048 80 / 82; 384
//   n = 4096 155 / 157, n = 8192 301 / 272; 512 n = 8192 340 / 356.
//   fp32 d = 64: 128 pairs n = 512 49 / 47; 256 n = 1024 107 / 130, n = 2048 203 /
//   230, n = 4096 391 / 344; d = 32: 256 n = 2048 98 / 90, n = 4096 192 / 163.
// A wave sums a quarter of its sequence into one fp32 accumulator, so the error
// of the sums grows with the length, which that of the three launches'
// compensated units does not: against 64 bits, fp32 d = 32, 1.67e-7 / 1.55e-7 at
// n = 2048, 2.5e-7 / 1.8e-7 at 8192, 3.3e-7 / 1.9e-7 at 16384.  So at most 2048
// tokens (a unit's) in fp32; in bf16, where roundings of the operands are 4.5e-4,
// 8192, which keeps a wave's sum to a unit's tokens.  max_seqlen only chooses.
bool short_forward(const Plan& p) {
  if (!rows_supported(p) || p.d == 128) return false;
  const bool bf16 = p.dtype == GBLA_BF16;
  const int64_t longest = p.ragged ? p.max_seqlen : p.rows;
  if ((int64_t)p.nseq * p.heads > kMaxGridX) return false;
  if (longest <= (bf16 ? 512 : p.d == 64 ? 128 : 256)) return true;
  if (longest > (bf16 ? 4 * kMaxChunk : kMaxChunk)) return false;
  int64_t pairs = 256;
  if (bf16) pairs = p.d == 32 && longest > 1536 ? 352 : 300;
  if (longest > kMaxChunk) pairs += (longest - kMaxChunk) / 32;
  return longest * pairs <= p.tokens * p.heads;
}

gbla_status make_plan(const gbla_shape* s, bool ragged, Plan* p) {
  if (!s || !p) return GBLA_ERR_INVALID_ARGUMENT;
  if (s->batch < 1 || s->heads < 1 || s->seqlen < 0) return GBLA_ERR_INVALID_ARGUMENT;
  if (s->head_dim != 32 && s->head_dim != 64 && s->head_dim != 128) return GBLA_ERR_UNSUPPORTED;
  if (s->conv_width < 1 || s->conv_width > 4) return GBLA_ERR_UNSUPPORTED;
  if (s->dtype != GBLA_F32 && s->dtype != GBLA_BF16) return GBLA_ERR_UNSUPPORTED;
  if (!(s->eps >= 0.0f) || !isfinite(s->eps)) return GBLA_ERR_INVALID_ARGUMENT;
  if (ragged && s->max_seqlen < 0) return GBLA_ERR_INVALID_ARGUMENT;
  if (s->heads > kMaxGridY) return GBLA_ERR_UNSUPPORTED;
  if (s->flags & ~(uint32_t)GBLA_BLA) return GBLA_ERR_INVALID_ARGUMENT;

  Plan q{};
  q.nseq = s->batch;
  q.heads = s->heads;
  q.rows = s->seqlen;
  q.d = s->head_dim;
  q.W = s->conv_width;
  q.dtype = s->dtype;
  q.ragged = ragged ? 1 : 0;
  q.max_seqlen = ragged ? s->max_seqlen : 0;
  q.eps = s->eps;
  q.flags = s->flags;
  q.tokens = ragged ? (int64_t)s->seqlen : (int64_t)s->batch * s->seqlen;

  // Chunk of the state reduction: about one workgroup per CU over all heads,
  // a power of two between 256 and 2048 tokens.  Depends on the shape only.
  const int64_t work = q.tokens * q.heads;
  int64_t chunk = next_pow2((work + 255) / 256);
  if (chunk < 256) chunk = 256;
  if (chunk > kMaxChunk) chunk = kMaxChunk;
  q.chunk = (int32_t)chunk;
  q.rtile = kReadoutTile;
  q.rec_floats = (int32_t)align_up((size_t)q.d * q.d + q.d + 2, 64);
  const size_t nmb = q.d / 16 + 1, nkb = q.d / 32;
  const size_t lane_bytes = q.dtype == GBLA_BF16 ? 16 : 32;
  q.frag_bytes = align_up(nmb * nkb * 64 * lane_bytes, 256);
  // bf16 readout tiles: 512 tokens, of a small batch down to 128 (four waves of
  // 32), for a workgroup per CU where the batch has the tokens for it (9662
  // tokens, H = 4, d = 64: readout 10 us, 15 with 512; twice as many workgroups
  // 10, and B = 1, n = 32768, H = 8 then takes 29 us against 28).  Up to d = 64
  // several workgroups run on a CU and a few past 256 cost nothing (whole forward,
  // n = 16000, H = 8, d = 64 35.7 us with 256, 35.8 with 512).
  if (q.dtype == GBLA_F32) fp32_split(&q);
  else if (q.d == 128) rtile_by_rounds(&q);
  else halve_rtile(&q, 128);

  // Upper bounds valid for both layouts: sum_s max(1, ceil(len_s / u)) <=
  // tokens / u + N.  The partial records are sized with this bound so the
  // workspace layout is the same for the dense and the ragged call.
  const int64_t units_cap = q.tokens / q.chunk + q.nseq;
  const int64_t runits_cap = q.tokens / q.rtile + q.nseq;
  if (units_cap > kMaxGridX || runits_cap > kMaxGridX) return GBLA_ERR_UNSUPPORTED;
  if (ragged) {
    q.chunks_per_seq = 0;
    q.rtiles_per_seq = 0;
    q.units = (int32_t)units_cap;
    q.runits = (int32_t)runits_cap;
  } else {
    int64_t cps = ((int64_t)q.rows + q.chunk - 1) / q.chunk;
    int64_t rps = ((int64_t)q.rows + q.rtile - 1) / q.rtile;
    if (cps < 1) cps = 1;
    if (rps < 1) rps = 1;
    q.chunks_per_seq = (int32_t)cps;
    q.rtiles_per_seq = (int32_t)rps;
    q.units = (int32_t)(cps * q.nseq);
    q.runits = (int32_t)(rps * q.nseq);
  }

  q.off_partials = 0;
  set_workspace(&q, units_cap);
  *p = q;
  return GBLA_OK;
}

}  // namespace gbla
