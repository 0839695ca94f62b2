// Internal helpers shared by the HIP translation units of libbass (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bass.h"
#include "attn_plan.h"
#include "bass_layout.h"

namespace bass {

constexpr int kWave = 64;          // CDNA wavefront
// The registers of the streaming kernel allow one wavefront per SIMD (256 CUs x 4 SIMDs = 1024
// resident wavefronts).  Measured on the paper-shaped batches, three quarters of that is fastest:
// the memory system is saturated either way, and fewer wavefronts mean fewer partials to merge.
constexpr int kDefaultWaves = 768;

// Quantizer of the INT8 caches (see bass.h, BASS_DTYPE_INT8KV): every step is one fp32 operation.
#ifdef __HIPCC__
__device__ inline float bf16_bits_to_float(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// codes of 8 bf16 values (in a uint4) for the row scale 127 / amax; returns them packed in 8 bytes
__device__ inline uint2 quantize8(const uint4& v, float inv) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t out[2] = {0u, 0u};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float x = bf16_bits_to_float((w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
    const int code = (int)__builtin_rintf(x * inv);  // one fp32 product, round half to even
    out[e >> 2] |= ((uint32_t)code & 0xFFu) << (8 * (e & 3));
  }
  return make_uint2(out[0], out[1]);
}

__device__ inline float amax8(const uint4& v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  float m = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(bf16_bits_to_float((w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu)));
  return m;
}
#endif

// 64-bit inclusive prefix sum and total over a wavefront.  Shifts inside rows of 16 lanes are DPP moves of
// the two halves (a generic shuffle of a 64-bit value is two trips through the LDS crossbar per step); the
// three row totals are then added from scalar registers.  Integer sums: the order is irrelevant.
#ifdef __HIPCC__
template <int N>
__device__ inline uint64_t row_shift_right_u64(uint64_t v) {  // lane i of a row gets lane i - N of the row, 0 for i < N
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0x110 + N, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), 0x110 + N, 0xF, 0xF, true);
  return ((uint64_t)hi << 32) | lo;
}

__device__ inline uint64_t read_lane_u64(uint64_t v, int src) {  // src: wave-uniform
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

__device__ inline uint64_t wave_incl_scan_u64(uint64_t v, int lane) {
  v += row_shift_right_u64<1>(v);
  v += row_shift_right_u64<2>(v);
  v += row_shift_right_u64<4>(v);
  v += row_shift_right_u64<8>(v);
  const uint64_t t0 = read_lane_u64(v, 15), t1 = read_lane_u64(v, 31), t2 = read_lane_u64(v, 47);
  const int row = lane >> 4;
  return v + (row > 0 ? t0 : 0) + (row > 1 ? t1 : 0) + (row > 2 ? t2 : 0);
}

template <int N>
__device__ inline float row_shift_right_keep(float v) {  // lane i of a row gets lane i - N of the row, its own value for i < N
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x110 + N, 0xF, 0xF, false));
}

__device__ inline float wave_max_f32(float v) {  // the same maximum in every lane
  v = fmaxf(v, row_shift_right_keep<1>(v));
  v = fmaxf(v, row_shift_right_keep<2>(v));
  v = fmaxf(v, row_shift_right_keep<4>(v));
  v = fmaxf(v, row_shift_right_keep<8>(v));
  const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 15));
  const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 31));
  const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 47));
  const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

__device__ inline uint64_t wave_sum_u64(uint64_t v) {  // the same total in every lane
  v += row_shift_right_u64<1>(v);
  v += row_shift_right_u64<2>(v);
  v += row_shift_right_u64<4>(v);
  v += row_shift_right_u64<8>(v);
  return read_lane_u64(v, 15) + read_lane_u64(v, 31) + read_lane_u64(v, 47) + read_lane_u64(v, 63);
}
#endif

inline int check_desc(const bass_attn_desc* d) {
  if (!d) return BASS_ERR_INVALID_ARG;
  if (d->B <= 0 || d->kmax <= 0 || d->Hq <= 0 || d->Hkv <= 0 || d->D <= 0 || d->Lcap <= 0)
    return BASS_ERR_INVALID_ARG;
  if (d->Hq % d->Hkv != 0) return BASS_ERR_INVALID_ARG;
  if (d->dtype == BASS_DTYPE_BF16 || d->dtype == BASS_DTYPE_INT8KV) {
    if (d->D != 64 && d->D != 128) return BASS_ERR_UNSUPPORTED;
  } else if (d->dtype == BASS_DTYPE_FP32) {
    if (d->D % 4 != 0 || d->D > 256) return BASS_ERR_UNSUPPORTED;
  } else {
    return BASS_ERR_UNSUPPORTED;
  }
  // index arithmetic inside the kernels is 32-bit for block counts and 64-bit for bytes
  // (the flattened block list counts up to kMaxPad virtual blocks per unit on top of the real ones)
  if ((int64_t)d->B * d->Hkv * ((int64_t)num_blocks(d->Lcap) + kMaxPad) >= (1ll << 30)) return BASS_ERR_UNSUPPORTED;
  return BASS_OK;
}

// ---------------------------------------------------------------------------------------
// Shape of an attention launch: which kernel serves the descriptor, over how many shares the block
// list is divided, and the virtual blocks of a unit.  The plan of a step and the launches that
// consume it derive it from the same inputs.
// ---------------------------------------------------------------------------------------
constexpr int kWavesPerWorkgroup = 4;  // also the grain of a launch's wavefront count
constexpr int kComputeUnits = 256;     // MI355X
// Wavefronts per workgroup of a launch whose wavefronts each fill a SIMD's registers (one workgroup per
// compute unit at a time).  Four, except where three put exactly one workgroup on every compute unit: 768
// wavefronts as 256 x 3 measured 2 % shorter attention launches than as 192 x 4 with 64 units idle (two per
// workgroup, 384 workgroups: 7 % longer; one: 1 % shorter).
inline int waves_per_workgroup(int nwaves) { return nwaves == 3 * kComputeUnits ? 3 : kWavesPerWorkgroup; }
constexpr int kAppendPad = 3;     // virtual blocks per unit when the append is fused (measured best: 3)
constexpr int kPlainPad = 2;      // ... and when it is not (the unit's last blocks are the masked, slower ones)
constexpr int kAppendBefore = 1;  // how many of those sit in front of the unit's last real block (one-tile matrix-core
constexpr int kPlainBefore = 0;   // kernel; measured: +0.5 % with the fused append, slightly slower without)
// More than 16 query rows per kv head: the workgroup-level kernels.  verify_attn_wide (a wavefront has all rows of its own blocks)
// takes whatever has at most 32 rows.  With more rows there is a choice.  The kernels that share a block's rows between wavefronts have the
// shorter way from the first block to the last store, verify_attn_wide the shorter time per block; which counts depends on the lengths,
// which are known on the device only.  So by what the host knows:
// - Caches of at most kShortCache blocks per sequence share rows: 48 and 64 rows, 8 kv heads of 128, 4 / 8 / 32 sequences, sharing rows ->
//   wide: bf16, at most 150 tokens 10.4 / 13.4 / 20.2 -> 12.4 / 15.0 / 23.6 us, 400 tokens 15.3 / 15.2 / 23.1 -> 16.3 / 16.6 / 25.6, 700 tokens
//   15.0 / 18.9 / 30.2 -> 16.4 / 17.8 / 30.9, 1200 tokens 19.5 / 21.8 / 42.0 -> 18.9 / 21.6 / 40.5; INT8, 700 tokens 19.7 / 19.9 / 30.7 -> 17.6 / 18.2 /
//   31.2, 1200 tokens 21.4 / 21.7 / 39.4 -> 19.4 / 23.8 / 35.8.
// - So do few units in caches of any size, where a short list loses most: units of 128, 48 rows, 60 / 150 / 400 / 1000 / 1500 / 2500 / 4000
//   tokens, sharing rows -> wide: bf16, 8 units 9.8 / 9.3 / 9.8 / 11.9 / 13.0 / 15.3 / 16.6 -> 12.6 / 12.7 / 12.5 / 13.3 / 13.6 / 14.9 / 16.6, 16 units 10.1 / 9.6 /
//   10.9 / 14.3 / 15.5 / 19.8 / 21.0 -> 12.7 / 12.8 / 13.2 / 14.4 / 15.3 / 16.9 / 18.6, 32 units 10.6 / 11.0 / 13.2 / 17.5 / 20.1 / 22.3 / 26.2 -> 13.1 / 13.8 / 14.5 /
//   17.1 / 17.4 / 21.4 / 24.9, 64 units 12.8 / 13.5 / 15.3 / 22.3 / 25.0 -> 15.0 / 15.5 / 16.5 / 19.5 / 23.9; INT8, 8 units 10.9 / 10.6 / 10.7 / 12.2 / 13.8 / 13.8 /
//   17.0 -> 14.1 / 14.1 / 14.0 / 14.2 / 14.4 / 15.3 / 16.2, 16 units 11.1 / 10.9 / 11.6 / 13.0 / 15.9 / 18.5 / 19.8 -> 14.1 / 14.3 / 14.2 / 14.8 / 15.2 / 16.8 / 17.8, 32 units
//   11.4 / 11.5 / 14.4 / 18.4 / 19.9 / 24.1 / 26.8 -> 14.5 / 14.5 / 14.7 / 16.2 / 17.3 / 22.5 / 24.9.  Units of 64 turn at half as many: INT8, 16 units 9.9 / 11.1 / 10.0 / 12.6 /
//   13.7 / 16.7 / 18.6 -> 11.0 / 11.1 / 11.1 / 11.4 / 12.0 / 13.0 / 14.2; bf16, 32 units 8.9 / 10.1 / 11.2 / 13.4 / 16.5 / 17.7 / 19.9 -> 10.2 / 10.4 / 10.7 / 13.2 / 13.5 / 15.8 /
//   17.6.  So up to a quarter of the head size over bf16 caches, an eighth over INT8 ones.
//   There shares get 2, over INT8 caches 4 entries at least where the units are long enough (kRowGrow), because each is a partial result to
//   be merged: 8 units of 128, 48 rows, at least 1 / 2 / 4 entries, INT8 60 tokens 10.6 / 10.9 / 12.5, 700 12.5 / 11.5 / 12.8, 1000 14.9 / 12.3 / 12.1, 2500
//   19.6 / 16.8 / 13.9 (6 entries 16.2); bf16 9.1 / 9.8 / 10.6, 11.7 / 10.7 / 11.1, 12.9 / 11.9 / 11.5, 15.2 / 15.3 / 13.6, but with 4 a wavefront has two
//   blocks, and precision is lost as below.
constexpr int kShortCache = 24;
constexpr int kFewUnitsDiv = 4, kFewUnitsDivInt8 = 8;  // ... of the head size
constexpr int kRowEntries = 2, kRowEntriesInt8 = 4, kRowGrow = 17;
// verify_attn_wide: one workgroup per compute unit.  The end of a unit inside a stretch -- four states merged, the next unit's first
// blocks waited for -- costs its workgroup about as much as 7 blocks: 16 layers of 16 sequences of 1024 - 4096 tokens, 64/8 heads, with 3 / 5 /
// 7 virtual blocks per unit 769 / 758 / 758 us, 8 sequences, 32 heads, 32 rows 765 / 751 / 745.  Short lists go to fewer workgroups so that
// every wavefront has a block (a target: a unit always gets a share of its own): 1 sequence of 1000 tokens, 64 rows, 8 kv heads, with at least
// 1 / 4 / 8 / 12 entries per share 26.5 / 17.8 / 18.0 / 20.8 us (few_units takes this shape to the kernels that share rows now); from 8 on a wavefront's state spans several blocks, fewer probabilities are exactly 1 and precision is lost.
// Two where two fit (at most 32 rows of 64 elements) and the units are many: 256 units of 32 rows, 512 - 2048 tokens, INT8 23.6 -> 20.7, bf16
// 25.7 -> 25.6; of 24 rows, 100 - 400 tokens, 15.9 -> 12.6 and 14.7 -> 13.2; 64 - 128 units 0 - 8 % longer.  Up to 1024 units: more
// stretches need more scratch memory, and bass_verify_attention_noalloc has only so much of it.  (INT8 heads of 128 held to the registers of
// two: short lists of 512 units 33.9 -> 29.7, but one workgroup alone 5 - 8 % longer.)
constexpr int kTileShares = 256, kTwoUnits = 256;
constexpr int kWidePad = 7, kWideEntries = 4;
// Stretches of whole units (PlanShape::whole): a block for each of the four wavefronts, or two.  Even division -> whole stretches, head size
// 128: 1 sequence of 960 tokens, 32 heads, 8 rows (30 blocks a unit) 11.9 -> 11.0 us; 8 kv heads, 32 rows, 1 / 16 sequences of 60 tokens
// 9.7 / 11.4 -> 7.6 / 9.5; 48 rows, 16 sequences of 400 tokens 21.0 -> 17.9, 32 of 60 / 150 24.9 / 24.6 -> 19.7 / 20.8.
constexpr int kWidePerStep = 4;
// At most 16 query rows: up to this many units (sequence, kv head) take verify_attn_wide too, with a tile of 16 rows; more of them stay with a
// wavefront per share (verify_attn_bf16), where a unit's merge costs no workgroup barrier.  8 query rows, a wavefront per share -> a
// workgroup, us per layer, 32 / 64 / 96 / 128 / 192 units, even division over the stretches: head size 128, 200 - 500 tokens 12.6 / 14.2 / 14.6 / 14.3 /
// 16.6 -> 10.4 / 11.7 / 12.9 / 15.4 / 18.0, 700 - 1500 tokens 17.2 / 19.2 / 20.6 / 21.3 / 28.4 -> 13.0 / 16.6 / 18.5 / 21.8 / 28.9, 2000 - 5000 tokens
// 20.8 / 30.1 / 36.8 / 44.4 / 65.1 -> 18.2 / 28.2 / 36.9 / 44.5 / 67.3; head size 64, 2000 - 5000 tokens 15.4 / 20.4 / 22.1 -> 14.8 / 18.7 / 22.9.
// At 96 units heads of 128 are still level or up to 12 % shorter, heads of 64 4 % longer, at 128 all are longer: one line for both.
// With whole stretches, 32 / 64 units: head size 128, 200 - 500 tokens 13.2 / 14.4 -> 10.1 / 11.6, 600 - 1500 14.8 / 19.6 -> 11.6 / 17.9, 2000 - 5000
// 24.9 / 34.8 -> 20.9 / 32.4, INT8 13.6 / 14.7 -> 10.1 / 10.7, 16.1 / 19.0 -> 10.8 / 16.0, 25.5 / 26.8 -> 18.5 / 23.0; head size 64 10.0 / 10.9 -> 8.2 /
// 8.9, 11.6 / 13.8 -> 8.8 / 13.0, 17.5 / 21.2 -> 15.2 / 20.1.  1 sequence of 2000 tokens, 32/8 heads: 21.3 -> 11.0, 32 heads of 960: 14.7 -> 11.8.
// There all 24 bits of the probabilities are multiplied (wide_softmax): with few shares per unit few probabilities are exactly 1, and the
// error against 64 bits would rise from 1.3e-3 to 1.6e-3.
// A share is at least 5 entries where the list is divided evenly: a target, since a unit always gets a share of its own.
constexpr int kNarrowUnits = 80;
constexpr int kNarrowPad = 7, kNarrowEntries = 5, kNarrowShares = 256;  // (8 entries: short lists a third longer)
// The kernels that share rows.  bf16: one workgroup per compute unit; INT8: two, because a step's conversions and softmax leave issue slots
// to fill.  INT8 plans have room for twice the stretches.
constexpr int kRowShares = 256, kRowSharesInt8 = 512;
constexpr int kMaxStagedElems = 2048;  // kmax * D up to which the one-tile kernels stage the step's rows in LDS

int attention_waves_setting();  // bass_set_attention_waves (0 = defaults); verify_attention.hip

struct LaunchShape {
  bool mfma;        // bf16 or INT8 caches: the matrix-core kernels
  bool tiles;       // more than one 16-row query tile per kv head: the workgroup-level kernels
  bool narrow;      // at most 16 query rows and few units: verify_attn_wide with one tile of 16
  bool wide;        // verify_attn_wide, narrow or with one or two tiles of 32
  bool fused_append;  // the step's rows are appended inside the attention launch, and its plan says so
  bool tiles_append;  // longer drafts, workgroup-level kernels: those that share rows patch a block at a time and stage nothing,
                      // verify_attn_wide has LDS for all rows that it takes, so planned launches may append there too; the
                      // plan is the one of a launch that does not append
  int rows_max, nwaves, nshares, used_shares, target, pad, pad_before, min_entries, whole, grow;
};

// One query tile per kv head: 768 wavefronts, over INT8 caches too -- as 256 workgroups of three they measured level with 1024 on
// the long-context shape and 2 - 3 % shorter on the benchmark shape (a fourth wavefront on a compute unit costs the others
// issue slots).  An explicit setting is clamped and rounded here.
inline int attention_waves(int setting) {
  int w = setting > 0 ? setting : kDefaultWaves;
  if (w < 64) w = 64;
  if (w > kMaxWaves) w = kMaxWaves;
  return w - w % kWavesPerWorkgroup;
}

inline LaunchShape launch_shape(const bass_attn_desc* d, bool append) {
  LaunchShape s;
  const int setting = attention_waves_setting();
  s.rows_max = d->kmax * (d->Hq / d->Hkv);
  s.mfma = d->dtype != BASS_DTYPE_FP32;
  const bool int8 = d->dtype == BASS_DTYPE_INT8KV;
  s.tiles = s.mfma && s.rows_max > 16;
  s.fused_append = append && (d->dtype == BASS_DTYPE_FP32 || (int64_t)d->kmax * d->D <= kMaxStagedElems);
  // (a launch wider than the shares it aims at, with all shares equally long -- plan_split -- was measured
  // 1 - 2 % slower than the even division on the benchmark shapes: more wavefronts, more partials to merge)
  s.nwaves = attention_waves(setting);
  s.narrow = s.mfma && !s.tiles && setting <= 0 && d->B * d->Hkv <= kNarrowUnits;
  const bool few_units = d->B * d->Hkv <= d->D / (int8 ? kFewUnitsDivInt8 : kFewUnitsDiv);
  s.wide = s.narrow || (s.tiles && (s.rows_max <= 32 || (num_blocks(d->Lcap) > kShortCache && !few_units)));
  // Longer drafts than the wavefronts stage: a patch costs a workgroup 1 - 3 us, one after the other for each of its units; an append by
  // itself goes by cache blocks from kBlockTokens slots on, which takes a 32-slot call 5 - 10 us.  Before the launch / inside it, us,
  // 32 rows, 32 heads of 128, 16 sequences of 100 / 450 / 1200 tokens, 32 of 450, 12 of 2000: verify_attn_wide, bf16 30.4 / 45.9 / 79.8 / 75.1 /
  // 90.6 -> 29.9 / 42.9 / 77.7 / 73.6 / 89.1: inside; INT8 29.8 / 37.6 / 54.9 / 57.9 / 59.0 -> 30.3 / 39.0 / 54.2 / 60.1 / 56.6: only up to 256
  // units, as in the kernels that share rows (64 rows, 8 sequences of 500, 34.7 / 34.7, 32 sequences 121.3 / 106.7).
  s.tiles_append = append && s.tiles && !s.fused_append && (d->kmax < kBlockTokens || d->B * d->Hkv <= kTileShares || (s.wide && !int8));
  // the workgroup-level kernels take one stretch per workgroup: half as many as an explicit setting has wavefronts
  const int stretches = setting > 0 ? s.nwaves / 2 : (int8 ? kRowSharesInt8 : kRowShares);
  const bool two = s.rows_max <= 32 && d->D == 64 && d->B * d->Hkv >= kTwoUnits && d->B * d->Hkv <= 4 * kTwoUnits;
  s.used_shares = s.narrow ? kNarrowShares : !s.tiles ? s.nwaves : s.wide && setting <= 0 ? (two ? 2 * kTileShares : kTileShares) : stretches;
  s.nshares = !s.tiles ? s.nwaves : int8 ? 2 * stretches : s.wide && two && setting <= 0 ? s.used_shares : stretches;
  s.target = s.nshares;
  s.pad = s.narrow ? kNarrowPad : s.wide ? kWidePad : s.fused_append ? kAppendPad : kPlainPad;
  s.min_entries = setting > 0 ? 0 : s.narrow ? kNarrowEntries : s.wide ? kWideEntries : s.tiles && few_units ? (int8 ? kRowEntriesInt8 : kRowEntries) : 0;
  s.grow = !s.wide && s.min_entries > 0 ? kRowGrow : 0;
  s.whole = s.wide && s.min_entries > 0 ? kWidePerStep : 0;
  s.pad_before = 0;
  if (s.mfma && !s.tiles && !s.wide) s.pad_before = s.fused_append ? kAppendBefore : kPlainBefore;
  return s;
}

// Peek, so that the caller can still fetch the HIP error code after a BASS_ERR_HIP return.
inline int launch_status() { return hipPeekAtLastError() == hipSuccess ? BASS_OK : BASS_ERR_HIP; }

}  // namespace bass
