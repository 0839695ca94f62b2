// Ragged verify attention of libbass: bass_verify_attention, bass_append_verify_attention (the
// step's K/V rows appended inside the same launch), bass_verify_attention_pad / _split (the paper's
// BASS-PAD and BASS-SPLIT as launch variants), for bf16, INT8 and fp32 caches.
//
// BASS paper, Section 3.2 (attention flow): scores of the current tokens' queries against
// the keys of all tokens processed so far, P = softmax(Q^T K / c), then P times V, with
// ragged K, V, P because every sequence has its own length.  Section 2.2: the draft tokens
// are processed as incremental context encoding, i.e. causally among themselves.  BASS-PAD
// gives padded positions probability zero, BASS-SPLIT computes every sequence at its true
// length with one launch per sequence; here ONE launch covers all sequences at their true
// lengths, and nothing outside a sequence's valid range is read.
//
// Work decomposition.  Attention shares no reads between sequences (Section 3.2), so the
// cost is streaming every valid K and V row once.  All (sequence, kv-head) units are cut
// into 32-token cache blocks and laid end to end; that flattened list is divided evenly
// over a fixed number of wavefronts.  A wavefront streams its contiguous share of blocks
// (registers are filled by 1 KiB-contiguous loads of MFMA-ordered cache blocks, next block
// in flight while the current one is computed), keeps an online softmax (running max and
// sum per query row) and, for every unit it touches, writes one partial (max, sum,
// unnormalised output).  The wavefront that delivers the LAST partial of a unit (found with
// one atomic counter per unit) merges the unit's partials -- the split-context reduction --
// and writes O and the log-sum-exp, so the whole call is a single launch.  (More than 16 query
// rows per kv head -- grouped-query attention, long drafts -- have kernels of their own, and with
// more than 32 the merge is a second, chip-wide launch: reduce_wide.)
//
// Matrix-core mapping (v_mfma_f32_16x16x32_bf16, wave64).  Tokens sit on the M side:
//   S^T[16 tokens x 16 query rows] = K[16 x D] * Q^T[D x 16]          (D/32 MFMAs per tile)
//   O^T[D x 16 query rows]        += V^T[D x 32 tokens] * P^T[32 x 16] (D/16 MFMAs per block)
// The result layout of the first (a lane owns 4 consecutive tokens of one query row) is,
// for two 16-token tiles, exactly the operand layout of the second once the V block is
// stored in that token order, so P goes from accumulator to operand with a bf16 pack only.
// Query rows of one kv head are (draft i, head-in-group) pairs, up to 64 rows = 4 tiles.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "bass_common.h"

namespace bass {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;

// Tuning knob of bass_set_attention_waves: process wide, read once per call.
static std::atomic<int> g_attention_waves{0};  // 0 = defaults
int attention_waves_setting() { return g_attention_waves.load(std::memory_order_relaxed); }

struct AttnParams {
  int B, kmax, Hq, Hkv, D, Lcap, nblk_cap, g, rows_max, nwaves;
  unsigned g_magic;  // ceil(2^20 / g) if g <= 64 and rows_max <= 2048 (then r / g == (r * g_magic) >> 20 for every row r), else 0
  int wpw;  // wavefronts per workgroup of the attention launch (nwaves is a multiple)
  float scale_log2;  // scale * log2(e): scores are kept in the log2 domain
  const void* Q;
  const void* Kc;
  const void* Vc;
  const void* Knew;  // [B,kmax,Hkv,D] rows of this step to append first, or null
  const void* Vnew;
  // the step's plan (attn_plan.h): header, one record per share, the further segments, per-sequence
  // query counts, per-unit contributors
  int32_t signature;  // plan_signature() of the plan this launch expects
  const ShareRecord* records;
  const Segment* overflow;
  const int32_t* seq_L;
  const int32_t* seq_nq;
  const int32_t* unit_owners;
  float* O;
  float* lse;
  float* part_acc;  // [slots][rows_max][D]
  float* part_ml;   // [slots][rows_max][2]  (running max in log2 units, running sum)
  int32_t* counters;  // [B*Hkv] partials delivered per unit; zero between calls
  int32_t* status;
};

// Query row r of a kv head is query token r / g, head r % g of the group.  The division by the run-time
// group size is a multiplication by a constant the host prepared (a generic integer division is some 35
// instructions, and these sit on the way out).
__device__ inline int row_token(const AttnParams& p, int r) {
  return p.g_magic ? (int)(((unsigned)r * p.g_magic) >> 20) : r / p.g;
}

__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// ---------------------------------------------------------------------------------------
// The share of a wavefront (or workgroup), read from the step's plan.
// ---------------------------------------------------------------------------------------
// A segment whose address is the same in every lane, as wave-uniform values.
__device__ inline Segment load_segment(const Segment* src) {
  const i32x4 a = *(const i32x4*)src, b = *((const i32x4*)src + 1);
  Segment g;
  g.b = uniform(a[0]); g.kvh = uniform(a[1]); g.L = uniform(a[2]); g.nq = uniform(a[3]);
  g.first = uniform(b[0]); g.n = uniform(b[1]); g.owners = uniform(b[2]); g.flags = uniform(b[3]);
  return g;
}

// Segment si >= 1 of a share
__device__ inline const Segment* later_segment_address(const AttnParams& p, const ShareRecord* rec, int overflow, int si) {
  return si == 1 ? &rec->seg[1] : p.overflow + overflow + (si - 2);
}
__device__ inline Segment later_segment(const AttnParams& p, const ShareRecord* rec, int overflow, int si) {
  return load_segment(later_segment_address(p, rec, overflow, si));
}

// A segment requested early and used late (its address is the same in every lane): the request travels while
// the wavefront streams, so that going on to the next units of a long share costs no round trip.
struct SegmentInFlight {
  i32x4 a, b;
};
__device__ inline SegmentInFlight request_segment(const Segment* src) {
  return SegmentInFlight{*(const i32x4*)src, *((const i32x4*)src + 1)};
}
__device__ inline Segment arrived_segment(const SegmentInFlight& f) {
  Segment g;
  g.b = uniform(f.a[0]); g.kvh = uniform(f.a[1]); g.L = uniform(f.a[2]); g.nq = uniform(f.a[3]);
  g.first = uniform(f.b[0]); g.n = uniform(f.b[1]); g.owners = uniform(f.b[2]); g.flags = uniform(f.b[3]);
  return g;
}

// The plan must have been made for this launch: same batch shape, same number of shares, and for a launch
// that appends or does not; every record carries a signature of these.  Anything else (also a buffer that
// holds no plan) stops the wavefront before it stores anything, with BASS_STATUS_PLAN_MISMATCH.
__device__ inline bool record_matches(const AttnParams& p, const ShareRecord* rec) {
  int sig = uniform(rec->signature);
  asm volatile("" : "+s"(sig));  // keeps the comparison (and with it the wait for the record) where it is written
  return sig == p.signature;
}

__device__ inline void report_mismatch(const AttnParams& p, bool first_lane) {
  if (first_lane && p.status) atomicOr(p.status, BASS_STATUS_PLAN_MISMATCH);
}

struct Unit {
  int b, kvh, L, nq;
};
__device__ inline Unit unit_of(const Segment& g) { return Unit{g.b, g.kvh, g.L, g.nq}; }

// Partials travel between wavefronts that may sit on different XCDs, whose L2 caches are not
// coherent with each other for ordinary accesses.  Instead of device-scope fences (which write
// back and invalidate a whole L2 and cost far more than the data is worth), every partial is
// written and read with device-scope relaxed atomic 64-bit accesses, which go through to the
// device-coherent level; "wait for my stores, then bump the counter" orders them.
__device__ inline void store_dev(float* dst, float a, float b) {
  unsigned long long v = ((unsigned long long)__float_as_uint(b) << 32) | __float_as_uint(a);
  __hip_atomic_store((unsigned long long*)dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 128-bit variants through raw buffer accesses with the device-scope cache policy (sc1); the
// buffer descriptor also bounds the access: offsets beyond `bytes` read zero / are dropped.
constexpr int kAuxDeviceScope = 16;  // sc1

// base and bytes are wave-uniform by construction; saying so keeps the descriptor in scalar
// registers (otherwise every access is wrapped in a loop over distinct descriptors).
__device__ inline __amdgpu_buffer_rsrc_t dev_buffer(const float* base, unsigned bytes) {
  const unsigned long long a = (unsigned long long)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  float* ub = (float*)(((unsigned long long)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, 0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

__device__ inline void store_dev4(__amdgpu_buffer_rsrc_t rs, unsigned byte_off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, (int)byte_off, 0, kAuxDeviceScope);
}

__device__ inline f32x4 load_dev4(__amdgpu_buffer_rsrc_t rs, unsigned byte_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)byte_off, 0, kAuxDeviceScope));
}

// ---------------------------------------------------------------------------------------
// Split-context reduction, done by the wavefront that completes a unit:
//   M = max_s m_s ;  l = sum_s l_s 2^(m_s - M) ;  O = sum_s acc_s 2^(m_s - M) / l
// over the partials of wavefronts w_lo..w_hi, then zeros for the unit's unused query slots.
// ---------------------------------------------------------------------------------------
// DC: the head size when it is known at compile time (the divisions below then cost nothing; this code
// runs before a wavefront's first K/V load), 0: read it from the descriptor.
template <int DC>
__device__ inline void zero_rows(const AttnParams& p, int b, int kvh, int row_from, int lane, int row_to = 1 << 30) {
  const int D = DC ? DC : p.D, lpr = D / 4, rpi = 64 / lpr;
  const int rows_all = min(p.kmax * p.g, row_to);
  for (int r0 = row_from; r0 < rows_all; r0 += rpi) {
    const int r = r0 + lane / lpr;
    if (lane < rpi * lpr && r < rows_all) {
      const int i = row_token(p, r), hg = r - i * p.g;
      const size_t orow = ((size_t)b * p.kmax + i) * p.Hq + kvh * p.g + hg;
      *(float4*)(p.O + orow * D + (lane % lpr) * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p.lse && lane % lpr == 0) p.lse[orow] = 0.f;
    }
  }
}

// Split-context reduction of a unit, 64 / LPR query rows per sweep: LPR lanes per row, each lane owning
// KC float4 chunks of its row.  A round takes eight partials, in two phases, so that the requests of two
// rounds (of two sweeps, or of one sweep with more than eight partials) can be in flight together:
//   issue : requests, for the round's partials, the row's (max, sum) pairs (every lane of a row
//           asks for all of them, so no cross-lane traffic is needed later) and the lane's
//           output chunks -- one round trip to memory;
//   fold  : weights 2^(m_s - M) and the weighted sum, all lane-local; a later round rescales what is there
//           by the change of the running maximum.
// combine_finish then divides and writes O and lse.
// Few units leave many partials each (one sequence of 32 heads over 768 wavefronts: 24 per unit).  They used to be
// fetched two per round trip after the first eight, behind a pass of their own over the maxima: ten round
// trips to memory in a row instead of two for 24 partials.
// Device-scope requests cost a trip to memory each: partials that do not exist are skipped by
// wave-uniform branches, and idle row slots get an offset beyond the buffer descriptor's size,
// which the hardware answers with zeros without touching memory.
constexpr int kRound = 8;  // partials per round

template <int KC>
struct CombineRegs {
  bool rok;
  int r;
  float2 ml[kRound];
  f32x4 a[kRound][KC];
};

// What a sweep has merged so far: running maximum, sum of weights, weighted output chunks
template <int KC>
struct MergeState {
  float M, L;
  f32x4 acc[KC];
};

struct CombineJob {
  Unit u;
  int w_lo, w_hi;
};

// 2 GiB: larger than any descriptor, and adding a partial's offset, which the host keeps below
// 2 GiB, cannot wrap around.
constexpr unsigned kNoSuchOffset = 0x80000000u;

typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

__device__ inline float2 load_dev2(__amdgpu_buffer_rsrc_t rs, unsigned byte_off) {
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)byte_off, 0, kAuxDeviceScope);
  return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}

// A sweep merges 64 / LPR rows: LPR lanes share a row, lane dl of them holds the 16-byte chunks dl + LPR k
// (k < KC) of it.  Requests partials j0 .. j0 + 7 of the job (those that exist).
template <int KC, int DC, int LPR = 16>
__device__ inline void combine_issue(const AttnParams& p, const CombineJob& job, int r0, int j0, int lane, CombineRegs<KC>& c) {
  const Unit& u = job.u;
  const int D = DC > 0 ? DC : p.D;
  const int rr = lane / LPR, dl = lane % LPR;
  const int rows = uniform(u.nq * p.g);
  const int n = min(uniform(job.w_hi - job.w_lo + 1 - j0), kRound);
  const size_t slot0 = (size_t)uniform(job.w_lo + j0 + u.b * p.Hkv + u.kvh);
  const unsigned slot_bytes = (unsigned)p.rows_max * D * 4, ml_bytes = (unsigned)p.rows_max * 8;
  const __amdgpu_buffer_rsrc_t rs = dev_buffer(p.part_acc + slot0 * p.rows_max * D, (unsigned)n * slot_bytes);
  const __amdgpu_buffer_rsrc_t rs_ml = dev_buffer(p.part_ml + slot0 * p.rows_max * 2, (unsigned)n * ml_bytes);
  c.rok = r0 + rr < rows;
  c.r = r0 + rr;
  const unsigned ml_off = c.rok ? (unsigned)c.r * 8 : kNoSuchOffset;
#pragma unroll
  for (int j = 0; j < kRound; ++j) {
    if (j >= n) break;  // wave-uniform: no such partial (combine_fold never looks at it)
    c.ml[j] = load_dev2(rs_ml, (unsigned)j * ml_bytes + ml_off);
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const int d = 4 * (dl + LPR * k);
      const unsigned row_off = (c.rok && d < D) ? (unsigned)(c.r * D + d) * 4 : kNoSuchOffset;
      c.a[j][k] = load_dev4(rs, (unsigned)j * slot_bytes + row_off);
    }
  }
}

// Adds partials j0 .. j0 + 7 (issued into c) to what the sweep has merged; j0 = 0 starts it.
template <int KC>
__device__ inline void combine_fold(const CombineJob& job, int j0, const CombineRegs<KC>& c, MergeState<KC>& t) {
  const int n = uniform(job.w_hi - job.w_lo + 1 - j0);
  // M = max_s m_s, L = sum_s l_s 2^(m_s - M).  A valid row has at least one partial with a
  // visible token (token 0, which the first partial holds), so M is finite from the first round on; a partial
  // that saw none has m = -inf, weight 0.  (Idle row slots were answered with zeros.)
  float M = j0 == 0 ? -INFINITY : t.M;
#pragma unroll
  for (int j = 0; j < kRound; ++j)
    if (j < n) M = fmaxf(M, c.ml[j].x);  // wave-uniform guards: partials beyond n were never requested
  const float Mf = (M == -INFINITY) ? 0.f : M;
  if (j0 == 0) {
    t.L = 0.f;
#pragma unroll
    for (int k = 0; k < KC; ++k) t.acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
    const float alpha = __builtin_amdgcn_exp2f(t.M - Mf);
    t.L *= alpha;
#pragma unroll
    for (int k = 0; k < KC; ++k) t.acc[k] *= alpha;
  }
  t.M = M;
#pragma unroll
  for (int j = 0; j < kRound; ++j) {
    if (j < n) {
      const float wgt = __builtin_amdgcn_exp2f(c.ml[j].x - Mf);
      t.L = fmaf(c.ml[j].y, wgt, t.L);
#pragma unroll
      for (int k = 0; k < KC; ++k) t.acc[k] += c.a[j][k] * wgt;
    }
  }
}

template <int KC, int DC, int LPR = 16>
__device__ inline void combine_finish(const AttnParams& p, const CombineJob& job, int lane, const CombineRegs<KC>& c,
                                      const MergeState<KC>& t) {
  const Unit& u = job.u;
  const int D = DC > 0 ? DC : p.D;
  const int dl = lane % LPR, r = c.r;
  if (c.rok) {
    const float invL = __builtin_amdgcn_rcpf(t.L);  // 1 ulp: far inside both tolerances, and a fraction of the instructions of a division
    const int i = row_token(p, r), hg = r - i * p.g;
    const size_t orow = ((size_t)u.b * p.kmax + i) * p.Hq + u.kvh * p.g + hg;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const int d = 4 * (dl + LPR * k);
      if (d < D) *(f32x4*)(p.O + orow * D + d) = t.acc[k] * invL;
    }
    if (p.lse && dl == 0) p.lse[orow] = (t.M + __builtin_amdgcn_logf(t.L)) * 0.6931471805599453f;
  }
}

// One sweep with any number of partials; kTwo: two rounds in flight at a time.
template <int KC, int DC, int LPR, bool kTwo>
__device__ inline void combine_sweep(const AttnParams& p, const CombineJob& job, int r0, int lane) {
  const int S = uniform(job.w_hi - job.w_lo + 1);
  MergeState<KC> t;
  CombineRegs<KC> cx, cy;
#pragma unroll 1
  for (int j0 = 0; j0 < S; j0 += kTwo ? 2 * kRound : kRound) {
    combine_issue<KC, DC, LPR>(p, job, r0, j0, lane, cx);
    if constexpr (kTwo) {
      const bool more = j0 + kRound < S;  // wave-uniform
      if (more) combine_issue<KC, DC, LPR>(p, job, r0, j0 + kRound, lane, cy);
      combine_fold<KC>(job, j0, cx, t);
      if (more) combine_fold<KC>(job, j0 + kRound, cy, t);
    } else {
      combine_fold<KC>(job, j0, cx, t);
    }
  }
  combine_finish<KC, DC, LPR>(p, job, lane, cx, t);
}

// Reduction of the one or two units this wavefront completed.  The sweeps of both jobs are laid end to
// end and handled two at a time, so that two sweeps share one round trip.  With a compile-time head size
// a sweep takes 8 rows (8 lanes per row): a wavefront's merge is bound by its own instruction stream, and
// the kv heads of this path have at most 16 query rows, mostly 8 or fewer -- one sweep per unit.
template <int DC>
__device__ inline void combine_jobs(const AttnParams& p, const CombineJob& ja, bool do_a, const CombineJob& jb, bool do_b,
                                    int lane) {
  constexpr bool kOverlap = DC > 0;  // the run-time-D (fp32) variant has too many chunk registers for two sweeps
  constexpr int LPR = DC > 0 ? 8 : 16, RPS = 64 / LPR;  // lanes per row, rows per sweep
  constexpr int KC = DC > 0 ? DC / 4 / LPR : 4;         // 16-byte chunks per lane (fp32: head sizes up to 256)
  const CombineJob& j0 = do_a ? ja : jb;  // first (or only) job
  const bool two = do_a && do_b;
  const int n0 = (j0.u.nq * p.g + RPS - 1) / RPS;
  const int n1 = two ? (jb.u.nq * p.g + RPS - 1) / RPS : 0;
  const bool many = uniform(j0.w_hi - j0.w_lo) >= kRound || (two && uniform(jb.w_hi - jb.w_lo) >= kRound);
  if (!kOverlap || many) {
#pragma unroll 1
    for (int t = 0; t < n0 + n1; ++t) {
      const CombineJob jx = (t < n0) ? j0 : jb;
      combine_sweep<KC, DC, LPR, kOverlap>(p, jx, (t < n0) ? RPS * t : RPS * (t - n0), lane);
    }
    return;
  }
#pragma unroll 1
  for (int t = 0; t < n0 + n1; t += 2) {
    const bool has_y = t + 1 < n0 + n1;
    const CombineJob jx = (t < n0) ? j0 : jb;
    const int rx = (t < n0) ? RPS * t : RPS * (t - n0);
    const CombineJob jy = (t + 1 < n0) ? j0 : jb;
    const int ry = (t + 1 < n0) ? RPS * (t + 1) : RPS * (t + 1 - n0);
    CombineRegs<KC> cx, cy;
    MergeState<KC> tx, ty;
    combine_issue<KC, DC, LPR>(p, jx, rx, 0, lane, cx);
    if (has_y) combine_issue<KC, DC, LPR>(p, jy, ry, 0, lane, cy);
    combine_fold<KC>(jx, 0, cx, tx);
    combine_finish<KC, DC, LPR>(p, jx, lane, cx, tx);
    if (has_y) {
      combine_fold<KC>(jy, 0, cy, ty);
      combine_finish<KC, DC, LPR>(p, jy, lane, cy, ty);
    }
  }
}

// All of this wavefront's partial stores have reached the device-coherent level once their
// acknowledgements are back (the sc1 stores are written through; the vector-memory counter of this
// wavefront falls to zero only when every one of them has been acknowledged); only then may its
// arrival be counted.  The wait is spelled out: a workgroup-scope fence is lowered without it.
__device__ inline void partial_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Counts this wavefront's arrival at one or two units (after partial_stores_done).  A job's
// `last` result is true if this wavefront delivered the unit's last partial: it then owns the
// reduction over wavefronts w_lo..w_hi.  Both counters are bumped before either result is awaited.
__device__ inline CombineJob job_of(const Segment& g) { return CombineJob{unit_of(g), seg_w_lo(g), seg_w_hi(g)}; }

__device__ inline int32_t* arrival_counter(const AttnParams& p, CombineJob& j, int& nparts) {
  nparts = j.w_hi - j.w_lo + 1;
  return p.counters + (size_t)j.u.b * p.Hkv + j.u.kvh;
}

__device__ inline void arrive(const AttnParams& p, int lane, CombineJob& ja, bool& last_a, bool has_b, CombineJob& jb,
                              bool& last_b) {
  int na, nb = 1, old_a = 0, old_b = 0;
  int32_t* ctr_a = arrival_counter(p, ja, na);
  int32_t* ctr_b = ctr_a;
  if (has_b) ctr_b = arrival_counter(p, jb, nb);
  if (na > 1 && lane == 0) old_a = __hip_atomic_fetch_add(ctr_a, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (has_b && nb > 1 && lane == 0) old_b = __hip_atomic_fetch_add(ctr_b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  last_a = na == 1 || __builtin_amdgcn_readfirstlane(old_a) == na - 1;
  last_b = has_b && (nb == 1 || __builtin_amdgcn_readfirstlane(old_b) == nb - 1);
  // every contributor has arrived: leave the counter clean for the next call
  if (last_a && na > 1 && lane == 0) __hip_atomic_store(ctr_a, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (last_b && nb > 1 && lane == 0) __hip_atomic_store(ctr_b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Query slots beyond draft_len (all of them for an inactive sequence) are zero in O and lse.
// Wavefront w clears them for the units w, w + nw, ...
// kInactiveOnly: only the units of sequences without query tokens (they have no blocks, hence no
// wavefront of their own); the caller then clears the unused rows of the other units elsewhere (the
// one-tile matrix-core kernel: by the wavefront that holds the unit's last block).
template <int DC, bool kInactiveOnly = false>
__device__ inline void zero_unused_rows(const AttnParams& p, int w, int nw, int lane) {
  for (int unit = w; unit < p.B * p.Hkv; unit += nw) {
    const int b = unit / p.Hkv;
    const int nq = uniform(p.seq_nq[b]);
    if (!kInactiveOnly || nq == 0) zero_rows<DC>(p, b, unit - b * p.Hkv, nq * p.g, lane);
  }
}

// ---------------------------------------------------------------------------------------
// bf16 streaming kernel
// ---------------------------------------------------------------------------------------
template <int D>
struct KvRegs {
  uint4 k[2 * (D / 32)];
  uint4 v[D / 16];
};

// kb, vb already include the lane offset
template <int D>
__device__ inline void load_block(KvRegs<D>& r, const uint4* kb, const uint4* vb) {
  // every K/V byte is read once per launch: non-temporal loads keep the stream from displacing
  // other data in the caches (measured: 10 % shorter launches than with ordinary loads)
#pragma unroll
  for (int i = 0; i < 2 * (D / 32); ++i) r.k[i] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4*)(kb + i * 64)));
#pragma unroll
  for (int i = 0; i < D / 16; ++i) r.v[i] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4*)(vb + i * 64)));
}

// Scales of the eight tokens whose scores / probabilities a lane holds (INT8 caches): slot j is token
// 4 grp + j (j < 4) or 16 + 4 grp + j - 4 of the block.
struct TokenScales {
  float k[8], v[8];
};

// Reductions over the four lanes l, l + 16, l + 32, l + 48 (the lanes that share a query row in the
// matrix-core result layout) with gfx950's lane-swap instructions: v_permlane32_swap of a value with
// itself leaves (low half, low half) and (high half, high half), v_permlane16_swap (rows 0 and 2 twice)
// and (rows 1 and 3 twice) -- two VALU operations per step instead of two trips through the LDS crossbar.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ inline float rows4_max(float v) {
  const u32x2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const u32x2 b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ inline float rows4_sum(float v) {
  const u32x2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const u32x2 b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// INT8 caches: a block's codes and the scales of this lane's tokens.  k[tt * (D/64) + ks]: the 16 codes of
// token 16 tt + lane % 16, head elements 64 ks + 16 grp ..; v[m]: V fragments 2m and 2m + 1 (8 codes each).
template <int D>
struct KvRegsI8 {
  u32x4 k[D / 32], v[D / 32];
  f32x4 ks[2], vs[2];  // tokens 4 grp .. 4 grp + 3 and 16 + 4 grp .. 16 + 4 grp + 3
};

// kb, vb: the block's first uint4; lane16 / grp16 are this lane's offsets (0 for a dummy fetch)
template <int D>
__device__ inline void load_block_i8(KvRegsI8<D>& r, const uint4* kb, const uint4* vb, int lane16, int grp16) {
#pragma unroll
  for (int i = 0; i < D / 32; ++i) r.k[i] = __builtin_nontemporal_load((const u32x4*)(kb + i * 64 + lane16));
#pragma unroll
  for (int i = 0; i < D / 32; ++i) r.v[i] = __builtin_nontemporal_load((const u32x4*)(vb + i * 64 + lane16));
  const f32x4* ks = (const f32x4*)(kb + 2 * D);  // the codes take 32 D bytes = 2 D uint4
  const f32x4* vs = (const f32x4*)(vb + 2 * D);
  r.ks[0] = ks[grp16];
  r.ks[1] = ks[4 + grp16];
  r.vs[0] = vs[grp16];
  r.vs[1] = vs[4 + grp16];
}

// eight INT8 codes (two words) -> eight bf16 (exact: |code| <= 127)
__device__ inline uint4 codes_to_bf16(uint32_t lo, uint32_t hi) {
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (__bf16)(float)(int)(int8_t)((e < 4 ? lo : hi) >> (8 * (e & 3)));
  return __builtin_bit_cast(uint4, o);
}

// V codes -> bf16 fragments (the K codes go to the INT8 matrix instruction as they are) and the scales
template <int D>
__device__ inline void dequant_block(const KvRegsI8<D>& q, KvRegs<D>& r, TokenScales& sc) {
#pragma unroll
  for (int f = 0; f < D / 16; ++f) r.v[f] = codes_to_bf16(q.v[f >> 1][2 * (f & 1)], q.v[f >> 1][2 * (f & 1) + 1]);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sc.k[j] = q.ks[0][j];
    sc.k[4 + j] = q.ks[1][j];
    sc.v[j] = q.vs[0][j];
    sc.v[4 + j] = q.vs[1][j];
  }
}

// Fused append: the step's own K/V rows of one unit (rows i < nq of K_new, V_new for sequence b,
// kv head kvh).  The wavefront whose share holds the unit's last blocks copies those rows into its
// own slice of LDS before it starts streaming; when it reaches the (masked) blocks the new tokens
// belong to, it patches the fetched K and V fragments from LDS and writes the patched 16-byte
// chunks back into the cache (plain stores that nobody waits for: no other wavefront reads those
// blocks in this launch).  The patch needs no global load, so the ring of outstanding K/V fetches
// is never drained for it.
extern __shared__ __align__(16) unsigned char new_rows_lds[];

struct NewRows {
  unsigned k_off, v_off;    // byte offsets of the unit's K and V rows in new_rows_lds: [row][D] bf16, or INT8 codes
  unsigned ks_off, vs_off;  // INT8 caches: the rows' fp32 scales
  int L, nq;
};

// A pass copies 128 16-byte chunks (2 per lane and tensor): 8 rows of 128 head elements.  The first
// pass overlaps the first K/V fetches; longer drafts take further passes, one after the other.
// The host keeps kmax * D <= kMaxStagedElems so that a workgroup's slices fit in 64 KiB of LDS.
constexpr int kStageLoads = 2;
constexpr int kStagePass = kStageLoads * 64;

struct StageRegs {
  u32x4 k[kStageLoads], v[kStageLoads];
};

// Loads of a unit's nq new rows, chunk c = c0 + 64 i + lane: row c / (D/8), head elements 8 (c % (D/8)) ..
template <int D>
__device__ inline void stage_issue(const AttnParams& p, const Unit& u, int c0, int lane, StageRegs& sr) {
  constexpr int CPR = D / 8;
  const size_t row_stride = (size_t)p.Hkv * D;
  const size_t first = ((size_t)u.b * p.kmax * p.Hkv + u.kvh) * D;
  const uint16_t* kn = (const uint16_t*)p.Knew + first;
  const uint16_t* vn = (const uint16_t*)p.Vnew + first;
  const int nchunks = u.nq * CPR;
  const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i) {
    sr.k[i] = zero;
    sr.v[i] = zero;
    if (c0 + i * 64 < nchunks) {  // wave-uniform
      const int c = min(c0 + i * 64 + lane, nchunks - 1);  // lanes past the end repeat the last chunk
      const size_t e = (size_t)(c / CPR) * row_stride + 8 * (c % CPR);
      sr.k[i] = *(const u32x4*)(kn + e);
      sr.v[i] = *(const u32x4*)(vn + e);
    }
  }
}

template <int D>
__device__ inline void stage_commit(const Unit& u, int c0, int lane, const StageRegs& sr, const NewRows& nr) {
  const int nchunks = u.nq * (D / 8);
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i) {
    const int c = c0 + i * 64 + lane;
    if (c < nchunks) {
      *(u32x4*)&new_rows_lds[nr.k_off + 16 * c] = sr.k[i];
      *(u32x4*)&new_rows_lds[nr.v_off + 16 * c] = sr.v[i];
    }
  }
}

// INT8 caches: the staged rows are quantized on the way into LDS (codes [row][D] bytes, one fp32 scale
// per row), exactly as the append kernel does; a row's D/8 chunks sit in consecutive lanes.
template <int D>
__device__ inline void stage_commit_i8(const Unit& u, int c0, int lane, const StageRegs& sr, const NewRows nr) {
  constexpr int CPR = D / 8;
  const int nchunks = u.nq * CPR;
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i) {
    if (c0 + i * 64 < nchunks) {  // wave-uniform
      const int c = c0 + i * 64 + lane;
      const uint4 kv = __builtin_bit_cast(uint4, sr.k[i]), vv = __builtin_bit_cast(uint4, sr.v[i]);
      float ka = amax8(kv), va = amax8(vv);
#pragma unroll
      for (int o = CPR >> 1; o >= 1; o >>= 1) {
        ka = fmaxf(ka, __shfl_xor(ka, o));
        va = fmaxf(va, __shfl_xor(va, o));
      }
      if (c < nchunks) {
        const float kinv = ka > 0.f ? 127.0f / ka : 0.f;
        const float vinv = va > 0.f ? 127.0f / va : 0.f;
        *(uint2*)&new_rows_lds[nr.k_off + 8 * c] = quantize8(kv, kinv);
        *(uint2*)&new_rows_lds[nr.v_off + 8 * c] = quantize8(vv, vinv);
        if (c % CPR == 0) {
          *(float*)&new_rows_lds[nr.ks_off + 4 * (c / CPR)] = ka / 127.0f;
          *(float*)&new_rows_lds[nr.vs_off + 4 * (c / CPR)] = va / 127.0f;
        }
      }
    }
  }
}

// INT8 caches, fused append: put the new tokens' codes and scales into the fetched block (before it is
// widened) and write them into the cache block at kblk / vblk (first byte of the block).
template <int D>
__device__ inline void patch_block_i8(KvRegsI8<D>& q, int tok0, const NewRows nr, int lane, uint8_t* kblk, uint8_t* vblk) {
  constexpr int KS = D / 64, MT = D / 16;
  const int dr = lane & 15, grp = lane >> 4;
  // K: chunk tl * KS + ks of a lane is token 16 tl + lane % 16, head elements 64 ks + 16 grp .. + 15
#pragma unroll
  for (int tl = 0; tl < 2; ++tl) {
    const int i = tok0 + 16 * tl + dr - nr.L;
    if (i >= 0 && i < nr.nq) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const u32x4 c = *(const u32x4*)&new_rows_lds[nr.k_off + i * D + 64 * ks + 16 * grp];
        q.k[tl * KS + ks] = c;
        *(u32x4*)(kblk + ((tl * KS + ks) * 64 + lane) * 16) = c;
      }
    }
  }
  // V codes and both scales: slot j of a lane is token 4 grp + j (j < 4) or 16 + 4 grp + j - 4
  bool v_new = false;
  float* kscale = (float*)(kblk + kBlockTokens * D);
  float* vscale = (float*)(vblk + kBlockTokens * D);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int w = j < 4 ? 4 * grp + j : 16 + 4 * grp + (j - 4);
    const int i = tok0 + w - nr.L;
    if (i >= 0 && i < nr.nq) {
      v_new = true;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const uint32_t code = new_rows_lds[nr.v_off + i * D + 16 * mt + dr];
        const uint32_t word = q.v[mt >> 1][2 * (mt & 1) + (j >> 2)];
        q.v[mt >> 1][2 * (mt & 1) + (j >> 2)] = (word & ~(0xFFu << (8 * (j & 3)))) | (code << (8 * (j & 3)));
      }
      const float ks = *(const float*)&new_rows_lds[nr.ks_off + 4 * i];
      const float vs = *(const float*)&new_rows_lds[nr.vs_off + 4 * i];
      q.ks[j >> 2][j & 3] = ks;
      q.vs[j >> 2][j & 3] = vs;
      if (dr == 0) {  // one lane per token group writes the scales
        kscale[w] = ks;
        vscale[w] = vs;
      }
    }
  }
  if (v_new) {
#pragma unroll
    for (int m = 0; m < D / 32; ++m) *(u32x4*)(vblk + (m * 64 + lane) * 16) = q.v[m];
  }
}

constexpr float kMaxSlack = 8.f;  // see block_step

template <int D>
struct RowState {
  f32x4 acc[D / 16];
  float m;  // running max (log2 units), identical in the 4 lanes that share a query row
  float l;  // this lane's share of the running sum
};

// One 32-token block against all query tiles.  kMasked: the block reaches beyond ctx_len, so
// causal limits and the valid-token bound apply (wave-uniform choice).
// INT8 caches: what the block step needs besides the widened V fragments -- the block's K codes, the
// quantized queries and all the scales.
template <int D>
struct I8Operands {
  const u32x4* k;                 // KvRegsI8::k of the block
  const u32x4* q;                 // query codes, B operand of the INT8 matrix instruction
  float q_scale_log2;             // this lane's query-row scale * softmax scale * log2(e)
  const TokenScales* sc;
};

template <int D, bool kMasked, bool kI8 = false>
__device__ inline void block_step(KvRegs<D>& r, const bf16x8* qf, RowState<D>& st, int tok0,
                                  int n_valid, int lim, float scale_log2, int lane,
                                  bool fused = false, const NewRows& nr = NewRows{}, uint4* kdst = nullptr,
                                  uint4* vdst = nullptr, const I8Operands<D>* i8 = nullptr) {
  constexpr int KS = D / 32, MT = D / 16;
  const int grp = lane >> 4;
  // INT8 caches: a score is the integer product (q codes . k codes) * q-scale * k-scale, a value is
  // code * v-scale, the latter folded into the probabilities that multiply V (r.v holds the codes as
  // bf16).  Stale tokens may carry any scale.
  float vsl[8];
  if (kI8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      vsl[j] = i8->sc->v[j];
      if (kMasked && tok0 + (j < 4 ? 4 * grp + j : 16 + 4 * grp + (j - 4)) >= n_valid) vsl[j] = 0.f;
    }
  }
  bool v_new = false;  // this lane's V chunks hold a new token
  if (kMasked && fused) {
    const int dr = lane & 15;
    // K: fragment tl * KS + t of a lane is token 16 tl + lane % 16, head elements 32 t + 8 grp .. + 7:
    // one 16-byte chunk of the new row
#pragma unroll
    for (int tl = 0; tl < 2; ++tl) {
      const int i = tok0 + 16 * tl + dr - nr.L;
      if (i >= 0 && i < nr.nq) {
#pragma unroll
        for (int t = 0; t < KS; ++t) {
          const u32x4 kv = *(const u32x4*)&new_rows_lds[nr.k_off + 2 * (i * D + 32 * t + 8 * grp)];
          r.k[tl * KS + t] = __builtin_bit_cast(uint4, kv);
          *(u32x4*)(kdst + (tl * KS + t) * 64) = kv;
        }
      }
    }
    // V: slot j of a lane is token 4 grp + j (j < 4) or 16 + 4 grp + j - 4, head element 16 mt + lane % 16
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = tok0 + (j < 4 ? 4 * grp + j : 16 + 4 * grp + (j - 4)) - nr.L;
      if (i >= 0 && i < nr.nq) {
        v_new = true;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const uint32_t v = *(const uint16_t*)&new_rows_lds[nr.v_off + 2 * (i * D + 16 * mt + dr)];
          uint32_t* wv = (uint32_t*)&r.v[mt];
          wv[j >> 1] = (j & 1) ? (wv[j >> 1] & 0x0000FFFFu) | (v << 16) : (wv[j >> 1] & 0xFFFF0000u) | v;
        }
      }
    }
  }
  if (kMasked) {
    // stale cache rows (token >= n_valid) may hold anything, NaN included: zero them in V so
    // that 0 * garbage cannot reach the accumulator.  Word w of a lane holds slots 2w, 2w+1.
    const int tA = tok0 + 4 * grp, tB = tok0 + 16 + 4 * grp;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      uint32_t* wv = (uint32_t*)&r.v[mt];
#pragma unroll
      for (int wd = 0; wd < 4; ++wd) {
        const int t_lo = (wd < 2 ? tA : tB) + 2 * (wd & 1);
        uint32_t keep = 0;
        if (t_lo < n_valid) keep |= 0x0000FFFFu;
        if (t_lo + 1 < n_valid) keep |= 0xFFFF0000u;
        wv[wd] &= keep;
      }
    }
    if (v_new) {  // the patched chunks go back into the cache (stale slots zeroed: they may hold anything)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) *(u32x4*)(vdst + mt * 64) = __builtin_bit_cast(u32x4, r.v[mt]);
    }
  }
  float s[8];
  if constexpr (kI8) {
    i32x4 a0 = {0, 0, 0, 0}, a1 = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < D / 64; ++ks) {
      a0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, i8->k[ks]), __builtin_bit_cast(i32x4, i8->q[ks]), a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, i8->k[D / 64 + ks]), __builtin_bit_cast(i32x4, i8->q[ks]), a1, 0, 0, 0);
    }
    const float qs = i8->q_scale_log2;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s[j] = (float)a0[j] * (i8->sc->k[j] * qs);
      s[4 + j] = (float)a1[j] * (i8->sc->k[4 + j] * qs);
    }
  } else {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.k[t]), qf[t], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.k[KS + t]), qf[t], s1, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s[j] = s0[j] * scale_log2;
      s[4 + j] = s1[j] * scale_log2;
    }
  }
  if (kMasked) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (tok0 + 4 * grp + j > lim) s[j] = -INFINITY;
      if (tok0 + 16 + 4 * grp + j > lim) s[4 + j] = -INFINITY;
    }
  }
  float mx = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
  mx = rows4_max(mx);
  // The reference maximum of a row moves only when a block exceeds it by more than kMaxSlack (log2 units).
  // The probabilities are then at most 2^kMaxSlack -- harmless in the fp32 sums and in the bf16 operand --
  // and the rescale of the running sum and of the accumulator (a third of a block step's instructions at
  // one wavefront per SIMD, where every instruction is paid for) runs in a unit's first block and hardly
  // ever again.  Wave-uniform branch; a row that does not move has alpha = 1.
  const float m_old = st.m;
  const bool grow = mx > m_old + kMaxSlack;
  if (__any(grow)) {
    const float m_new = grow ? mx : m_old;
    const float m_to = (kMasked && m_new == -INFINITY) ? 0.f : m_new;  // rows without a visible token yet
    const float alpha = __builtin_amdgcn_exp2f(m_old - m_to);
    st.l *= alpha;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) st.acc[mt] *= alpha;
    st.m = m_new;
  }
  // a row that has seen no visible token yet keeps m = -inf; subtract 0 instead so that
  // exp2(-inf - 0) = 0 and no inf - inf appears
  const float m_use = (kMasked && st.m == -INFINITY) ? 0.f : st.m;
  float psum = 0.f;
  bf16x8 pf;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float pj = __builtin_amdgcn_exp2f(s[j] - m_use);
    psum += pj;
    pf[j] = (__bf16)(kI8 ? pj * vsl[j] : pj);
  }
  st.l += psum;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    st.acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.v[mt]), pf, st.acc[mt], 0, 0, 0);
}

template <int D, bool kI8 = false>
__device__ inline void block_dispatch(KvRegs<D>& r, const bf16x8* qf, RowState<D>& st, int blk,
                                      int L, int n_valid, int lim, float scale_log2, int lane,
                                      bool fused, const NewRows& nr, uint4* kdst, uint4* vdst,
                                      const I8Operands<D>* i8 = nullptr) {
  const int tok0 = blk * kBlockTokens;
  // plain step: every token of the block is visible to every query (tokens <= L) and, with a fused
  // append, none of them is new (tokens < L)
  if (tok0 + kBlockTokens - 1 < L + (fused ? 0 : 1))
    block_step<D, false, kI8>(r, qf, st, tok0, n_valid, lim, scale_log2, lane, false, NewRows{}, nullptr, nullptr, i8);
  else
    block_step<D, true, kI8>(r, qf, st, tok0, n_valid, lim, scale_log2, lane, fused, nr, kdst, vdst, i8);
}

template <int D>
struct QFrag {
  bf16x8 q[D / 32];  // B operand: lane (col, grp) holds query row col of the tile, elements 32 t + 8 grp .. +7
  int lim;           // last token visible to that row
};

template <int D>
__device__ inline void load_queries(const AttnParams& p, const Unit& u, bool enable, int col, int grp, QFrag<D>& f,
                                    int row0 = 0) {
  const int rows = u.nq * p.g;
  const int rrow = row0 + col;  // row0: first query row of this wavefront (tile kernel)
  const bool ok = enable && rrow < rows;
  const int i = ok ? row_token(p, rrow) : 0, hg = ok ? rrow - i * p.g : 0;
  f.lim = u.L + i;
  const uint4* qrow = (const uint4*)((const uint16_t*)p.Q + (((size_t)u.b * p.kmax + i) * p.Hq + u.kvh * p.g + hg) * D);
#pragma unroll
  for (int t = 0; t < D / 32; ++t) {
    uint4 qv = make_uint4(0, 0, 0, 0);
    if (ok) qv = qrow[t * 4 + grp];
    f.q[t] = __builtin_bit_cast(bf16x8, qv);
  }
}

// INT8 caches: the queries are quantized like the cache rows (one scale per token and query head, codes
// rint(x * 127 / amax)) so that QK^T runs on the INT8 matrix cores.  B operand of the 16x16x64
// instruction: lane (col, grp) holds query row col of the tile, head elements 64 ks + 16 grp .. + 15.
template <int D>
struct QFragI8 {
  u32x4 q[D / 64];
  float q_scale_log2;  // row scale (amax / 127) * softmax scale * log2(e)
  int lim;
};

template <int D>
__device__ inline void load_queries_i8(const AttnParams& p, const Unit& u, bool enable, int col, int grp, QFragI8<D>& f,
                                       int row0 = 0) {
  const int rows = u.nq * p.g;
  const int rrow = row0 + col;
  const bool ok = enable && rrow < rows;
  const int i = ok ? row_token(p, rrow) : 0, hg = ok ? rrow - i * p.g : 0;
  f.lim = u.L + i;
  const uint4* qrow = (const uint4*)((const uint16_t*)p.Q + (((size_t)u.b * p.kmax + i) * p.Hq + u.kvh * p.g + hg) * D);
  uint4 raw[D / 64][2];
  float amax = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 64; ++ks)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      raw[ks][h] = ok ? qrow[ks * 8 + grp * 2 + h] : make_uint4(0, 0, 0, 0);
      amax = fmaxf(amax, amax8(raw[ks][h]));
    }
  amax = rows4_max(amax);  // the four lanes of a row hold a quarter of it each
  const float inv = amax > 0.f ? 127.0f / amax : 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 64; ++ks) {
    const uint2 lo = quantize8(raw[ks][0], inv), hi = quantize8(raw[ks][1], inv);
    f.q[ks] = u32x4{lo.x, lo.y, hi.x, hi.y};
  }
  f.q_scale_log2 = amax / 127.0f * p.scale_log2;
}

template <int D>
__device__ inline void clear_state(RowState<D>& st) {
  st.m = -INFINITY;
  st.l = 0.f;
#pragma unroll
  for (int mt = 0; mt < D / 16; ++mt) st.acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Partial of (wavefront w, unit u): slot ids w + unit are unique because both grow monotonically
// along the flattened list.
template <int D>
__device__ inline void store_partial(const AttnParams& p, const Unit& u, int w, const RowState<D>& st, int col, int grp,
                                     int row0 = 0) {
  const int rows = u.nq * p.g;
  const size_t slot = (size_t)w + (size_t)u.b * p.Hkv + u.kvh;
  const __amdgpu_buffer_rsrc_t rs = dev_buffer(p.part_acc + slot * p.rows_max * D, (unsigned)p.rows_max * D * 4);
  float l = st.l;
  l = rows4_sum(l);
  const int rrow = row0 + col;
  if (rrow < rows) {
    const unsigned off = (unsigned)(rrow * D + 4 * grp) * 4;
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) store_dev4(rs, off + 64 * mt, st.acc[mt]);
    if (grp == 0) store_dev(p.part_ml + (slot * p.rows_max + rrow) * 2, st.m, l);
  }
}

// A unit that this wavefront streamed alone needs no exchange: its output rows are written straight from the
// registers.  The arithmetic is that of the merge of a single partial (weight 2^0 = 1, the same reciprocal and
// logarithm), so a unit's result does not depend on which of the two ways it took.
template <int D>
__device__ inline void finalize_single(const AttnParams& p, const Unit& u, const RowState<D>& st, int col, int grp,
                                       int row0 = 0) {
  const int rows = u.nq * p.g;
  const float L = fmaf(rows4_sum(st.l), 1.0f, 0.f);
  const int rrow = row0 + col;
  if (rrow < rows) {
    const float M = st.m;
    const float invL = __builtin_amdgcn_rcpf(L);
    const int i = row_token(p, rrow), hg = rrow - i * p.g;
    const size_t orow = ((size_t)u.b * p.kmax + i) * p.Hq + u.kvh * p.g + hg;
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) *(f32x4*)(p.O + orow * D + 16 * mt + 4 * grp) = st.acc[mt] * invL;
    if (p.lse && grp == 0) p.lse[orow] = (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
  }
}

template <int D, bool kI8>
__global__ __launch_bounds__(256) void verify_attn_bf16(AttnParams p) {
  // uint4 per block: 32 tokens of D bf16, or of D INT8 codes followed by 32 fp32 scales
  constexpr ptrdiff_t kBlkVec = kI8 ? 2 * D + 8 : (ptrdiff_t)kBlockTokens * D * 2 / 16;
  using Regs = typename std::conditional<kI8, KvRegsI8<D>, KvRegs<D>>::type;
  // There are registers to spare for a second unit's state, so a wavefront
  // whose share of blocks crosses a unit boundary keeps streaming: it parks the first unit's
  // accumulators, carries on with the second unit, and delivers both partials at the end.
  // (Storing the first partial at the boundary instead costs about 1 us per launch: the stores
  // sit in the ring's wait counts.)
  const int lane = threadIdx.x & 63;
  const int w = uniform(blockIdx.x * p.wpw + (threadIdx.x >> 6));
  const int col = lane & 15, grp = lane >> 4;

  // This wavefront's share: the first two segments come with the record, in one round trip; the plan's
  // header travels at the same time.  Nothing waits for either before the first K/V fetch needs its
  // address: what the loop below sets up once (constants, lane offsets) runs under that round trip.
  const ShareRecord* rec = p.records + w;
  Segment sa = load_segment(&rec->seg[0]);
  Segment sb = load_segment(&rec->seg[1]);
  int nseg_plan = uniform(rec->nseg), overflow = uniform(rec->overflow);
  const int rec_flags = uniform(rec->flags);
  __builtin_amdgcn_sched_barrier(0);  // the loads above are issued here, whatever is scheduled below
  bool ok;
  int nseg;
  int si = 0;
  do {
    // The first fetch is issued before the plan has been checked, so its address is forced into the
    // cache whatever the record holds (a buffer without a plan must not turn into a wild read); stores
    // and everything else wait for the check.
    const int firstA = min(max(sa.first, 0), p.nblk_cap - 1);
    const ptrdiff_t unitA = (ptrdiff_t)min(max(sa.b, 0), p.B - 1) * p.Hkv + min(max(sa.kvh, 0), p.Hkv - 1);
    const ptrdiff_t vecA = (unitA * p.nblk_cap + firstA) * kBlkVec;
    const uint4* kc = (const uint4*)p.Kc;
    const uint4* vc = (const uint4*)p.Vc;
    Regs r0;
    if constexpr (kI8) load_block_i8<D>(r0, kc + vecA, vc + vecA, lane, grp);
    else load_block<D>(r0, kc + vecA + lane, vc + vecA + lane);
    ok = record_matches(p, rec);
    asm volatile("" : "+s"(nseg_plan), "+s"(overflow));  // as in record_matches: no use of the record ahead of the loop
    nseg = ok ? nseg_plan : 0;
    if (si >= nseg) break;  // an idle wavefront, or no plan for this launch
    const Unit uA = unit_of(sa);
    const int nA = sa.n;  // our real blocks of unit A: firstA .. firstA + nA - 1
    const bool hasB = si + 1 < nseg;
    // the segments after these (shares that touch more units than the record holds) are requested now and
    // looked at when this pair is done; without any, the request re-reads the record (loads stay outside
    // branches: the wait counts of the K/V ring must stay exact)
    const int si_next = si + (hasB ? 2 : 1);
    const SegmentInFlight nextA = request_segment(si_next < nseg ? later_segment_address(p, rec, overflow, si_next) : &rec->seg[0]);
    const SegmentInFlight nextB =
        request_segment(si_next + 1 < nseg ? later_segment_address(p, rec, overflow, si_next + 1) : &rec->seg[1]);
    const Unit uB = hasB ? unit_of(sb) : uA;
    const int firstB = hasB ? sb.first : 0, nB = hasB ? sb.n : 0;
    const bool lastA = (sa.flags & kSegLast) != 0, lastB = hasB && (sb.flags & kSegLast) != 0;  // we hold the unit's last block
    const int n = nA + nB;

    typename std::conditional<kI8, QFragI8<D>, QFrag<D>>::type qc, qB;
    if constexpr (kI8) {
      load_queries_i8<D>(p, uA, true, col, grp, qc);
      load_queries_i8<D>(p, uB, hasB, col, grp, qB);
    } else {
      load_queries<D>(p, uA, true, col, grp, qc);
      load_queries<D>(p, uB, hasB, col, grp, qB);
    }
    RowState<D> st, parked;
    clear_state<D>(st);
    CombineJob ja = job_of(sa), jb = ja;  // who else contributes to our units
    if (hasB) jb = job_of(sb);
    int cur_L = uA.L, cur_valid = uA.L + uA.nq, cur_blk = firstA;  // block index = cur_blk + s

    // fused append: the units whose new tokens lie in our blocks get their rows staged in LDS
    const bool fused = p.Knew != nullptr;
    // one unit's slice: K rows, V rows (bf16, or INT8 codes), then for INT8 the rows' K and V scales
    const unsigned lds_rows = (unsigned)p.kmax * D * (kI8 ? 1 : 2);
    const unsigned lds_unit = 2 * lds_rows + (kI8 ? 8 * (unsigned)p.kmax : 0);
    const unsigned lds_base = (threadIdx.x >> 6) * 2 * lds_unit;
    const NewRows newA{lds_base, lds_base + lds_rows, lds_base + 2 * lds_rows, lds_base + 2 * lds_rows + 4 * (unsigned)p.kmax,
                       uA.L, uA.nq};
    const NewRows newB{newA.k_off + lds_unit, newA.v_off + lds_unit, newA.ks_off + lds_unit, newA.vs_off + lds_unit,
                       uB.L, uB.nq};
    NewRows cur_new = newA;
    const bool stageA = fused && uA.nq > 0 && (firstA + nA) * kBlockTokens > uA.L;
    const bool stageB = fused && hasB && uB.nq > 0 && (firstB + nB) * kBlockTokens > uB.L;
    // one set of staging registers: a share that holds the new tokens of both its units is rare (the
    // second unit then lies wholly inside the share) and stages the second unit's rows afterwards
    const bool stage1 = stageA || stageB;
    const Unit& u1 = stageA ? uA : uB;
    const NewRows new1 = stageA ? newA : newB;  // a copy: a reference would put both structs in memory
    StageRegs sr;
    if (stage1) stage_issue<D>(p, u1, 0, lane, sr);
    auto commit = [&](const Unit& u, int c0, const StageRegs& regs, const NewRows nr) {
      if constexpr (kI8) stage_commit_i8<D>(u, c0, lane, regs, nr);
      else stage_commit<D>(u, c0, lane, regs, nr);
    };
    // what is left after the overlapped pass (drafts of more than 8 rows, a second unit): rare
    auto stage_rest = [&]() {
      for (int c0 = kStagePass; c0 < u1.nq * (D / 8); c0 += kStagePass) {
        StageRegs sr2;
        stage_issue<D>(p, u1, c0, lane, sr2);
        commit(u1, c0, sr2, new1);
      }
      if (stageA && stageB)
        for (int c0 = 0; c0 < uB.nq * (D / 8); c0 += kStagePass) {
          StageRegs sr2;
          stage_issue<D>(p, uB, c0, lane, sr2);
          commit(uB, c0, sr2, newB);
        }
    };

    // element offsets (in uint4) of step s inside the K and V caches
    const ptrdiff_t vecB = (((ptrdiff_t)uB.b * p.Hkv + uB.kvh) * p.nblk_cap + firstB - nA) * kBlkVec;

    // Every fetch is issued unconditionally so that the wait counts before each compute step are
    // exact (a fetch under a branch would force a wait for ALL outstanding loads at the join and
    // serialise load and compute).  A fetch past the end of the share reads 16 bytes of the
    // share's first block with every lane instead: valid memory, one cache line, never used.
    auto fetch = [&](Regs& r, int s) {
      if constexpr (kI8) {
        const bool real = s < n;
        const ptrdiff_t off = real ? (s < nA ? vecA : vecB) + (ptrdiff_t)s * kBlkVec : vecA;
        load_block_i8<D>(r, kc + off, vc + off, real ? lane : 0, real ? grp : 0);
      } else {
        ptrdiff_t off = vecA;
        if (s < n) off = (s < nA ? vecA : vecB) + (ptrdiff_t)s * kBlkVec + lane;
        load_block<D>(r, kc + off, vc + off);
      }
    };
    auto step = [&](Regs& r, int s) {
      if (s == nA) {  // first block of unit B: park A's state (register moves only)
        parked = st;
        clear_state<D>(st);
        qc = qB;
        cur_L = uB.L;
        cur_valid = uB.L + uB.nq;
        cur_blk = firstB - nA;
        cur_new = newB;
      }
      const ptrdiff_t own = (s < nA ? vecA : vecB) + (ptrdiff_t)s * kBlkVec + lane;  // this lane's chunks of block s
      uint4* kdst = (uint4*)const_cast<void*>(p.Kc) + own;
      uint4* vdst = (uint4*)const_cast<void*>(p.Vc) + own;
      if constexpr (kI8) {
        if (fused && (cur_blk + s) * kBlockTokens + kBlockTokens - 1 >= cur_L) {  // the block holds new tokens
          const ptrdiff_t blk_vec = (s < nA ? vecA : vecB) + (ptrdiff_t)s * kBlkVec;
          patch_block_i8<D>(r, (cur_blk + s) * kBlockTokens, cur_new, lane,
                            (uint8_t*)const_cast<void*>(p.Kc) + blk_vec * 16, (uint8_t*)const_cast<void*>(p.Vc) + blk_vec * 16);
        }
        KvRegs<D> t;
        TokenScales sc;
        dequant_block<D>(r, t, sc);
        const I8Operands<D> i8{r.k, qc.q, qc.q_scale_log2, &sc};
        block_dispatch<D, true>(t, nullptr, st, cur_blk + s, cur_L, cur_valid, qc.lim, p.scale_log2, lane, false,
                                    cur_new, nullptr, nullptr, &i8);  // the codes are patched already: no fused work inside
      } else {
        block_dispatch<D>(r, qc.q, st, cur_blk + s, cur_L, cur_valid, qc.lim, p.scale_log2, lane, fused, cur_new, kdst, vdst);
      }
    };
    // Unused query rows of a unit are cleared by the wavefront that holds the unit's last block (it is handed
    // fewer real blocks), while its first fetches are under way: the stores are acknowledged long before the
    // wavefront waits for its partial stores at the end, and nothing waits for them here.
    auto clear_unused = [&]() {
      if (lastA) zero_rows<D>(p, uA.b, uA.kvh, uA.nq * p.g, lane);
      if (lastB) zero_rows<D>(p, uB.b, uB.kvh, uB.nq * p.g, lane);
    };
    // The next segments were requested right behind the first block and are here with it; kept as scalars
    // from here on, they do not take vector registers away from the ring.
    Segment next_sa, next_sb;
    auto next_arrived = [&]() {
      next_sa = arrived_segment(nextA);
      next_sb = arrived_segment(nextB);
    };
    // three-deep register ring: two blocks (32 KiB per wavefront) in flight while one is computed
    Regs r1, r2;  // r0 is on its way already
    fetch(r1, 1);
    if (stage1) {
      commit(u1, 0, sr, new1);  // these loads were issued before the fetches
      stage_rest();
    }
    clear_unused();
    next_arrived();
    for (int s = 0; s < n; s += 3) {
      fetch(r2, s + 2);
      step(r0, s);
      fetch(r0, s + 3);
      if (s + 1 < n) step(r1, s + 1);
      fetch(r1, s + 4);
      if (s + 2 < n) step(r2, s + 2);
    }
    // A unit that lies wholly inside this share (common with many short sequences) is finished from the
    // registers; the others leave a partial, and the wavefront that delivers a unit's last partial merges.
    const bool soloA = ja.w_lo == ja.w_hi;
    const bool soloB = hasB && jb.w_lo == jb.w_hi;
    if (hasB) {
      if (soloA) finalize_single<D>(p, uA, parked, col, grp);
      else store_partial<D>(p, uA, w, parked, col, grp);
      if (soloB) finalize_single<D>(p, uB, st, col, grp);
      else store_partial<D>(p, uB, w, st, col, grp);
    } else {
      if (soloA) finalize_single<D>(p, uA, st, col, grp);
      else store_partial<D>(p, uA, w, st, col, grp);
    }
    const bool exchA = !soloA, exchB = hasB && !soloB;
    if (exchA || exchB) {
      partial_stores_done();
      bool mergeA = false, mergeB = false, unused;
      if (exchA) arrive(p, lane, ja, mergeA, exchB, jb, mergeB);
      else arrive(p, lane, jb, mergeB, false, jb, unused);
      if (mergeA || mergeB) combine_jobs<D>(p, ja, mergeA, jb, mergeB, lane);
    }
    si = si_next;
    sa = next_sa;
    sb = next_sb;
  } while (si < nseg);
  if (!ok) {
    report_mismatch(p, w == 0 && lane == 0);
    return;
  }
  // Unused query rows of inactive sequences (those of an active one: clear_unused above)
  if (rec_flags & kRecAnyInactive) zero_unused_rows<D, true>(p, w, p.nwaves, lane);
}

// ---------------------------------------------------------------------------------------
// Workgroup-level kernel for kv heads with more than 16 query rows (grouped-query attention, long drafts): NT tiles of 32 rows,
// bf16 and INT8 caches.  A workgroup of four wavefronts takes a stretch of the block list together and its wavefronts take the
// blocks in turn, each with the state of ALL query rows: a block is fetched once, straight into the operand registers of the one
// wavefront that needs it, nothing but the scales of INT8 blocks passes through LDS and nobody waits for anybody until the unit ends.  There the four
// states are merged through LDS (each wavefront collects a quarter of the accumulators) and one partial is stored.  What this is
// built around: a step of 32 x 32 tiles (v_mfma_f32_32x32x16_bf16) has half the matrix and cross-lane instructions per row
// of one of 16 x 16, and with two tiles two independent chains, so that one wavefront per SIMD keeps up with its share of the
// memory.  Attention with its merge per layer, against 16-row tiles of one wavefront each that read the blocks from a ring in LDS behind a
// barrier per phase: 16 sequences of 1024 - 4096 tokens, 64/8 heads of 128, bf16 with 48 rows (181 MB) 42.7 -> 41.7 us, INT8 with 64 rows
// (94 MB) 46.3 -> 36.0; 8 sequences of 512 - 2048, 32 heads, 32 rows, bf16 (182 MB) 51.8 -> 44.0, INT8 40.1 -> 33.3; rounding the scores
// (wide_scores) has cost 0.3 / 0.4 / 0.1 us of the first three since.  What is left over the
// memory's time is the way in (3 us to the first block), the merges and stretches that end 22 - 33 us after the start.  Counters, 48 rows:
// bf16 executes in 33 % of its wavefronts' cycles, waits for loads and LDS in 30 %, for an instruction to issue in 38 %; INT8 57 / 33 / 10 %, bound by
// its 615 vector instructions per block (bf16: 395).  Both tiles are computed for every unit, also where all rows are in the first.
//
// Matrix-core mapping (32 x 32, c = lane % 32, h = lane / 32):
//   S^T[32 tokens x 32 rows] = K Q^T: row c of operand A is token wide_token(c) of the block (bits 3 and 4 of c exchanged), step ks
//     takes head elements 8 (2 ks + h) .. + 7 (INT8: 16 (2 ks + h) .. + 15); a lane then holds, for query row c, the tokens
//     16 ((i >> 2) & 1) + 8 (i >> 3) + 4 h + (i & 3), i = 0 .. 15,
//   which is, eight by eight, the token order of the cache's V chunks, so that the probabilities are operand B of
//   O^T[32 head elements x 32 rows] += V^T P^T as they are.
// ---------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(16))) int i32x16;

constexpr int kWideWaves = 4;
constexpr int kAuxNonTemporal = 2;  // nt

// NT tiles of 32 query rows, or (NT = 0) one of 16.  A lane belongs to row lane % kRows of a tile; h = lane / kRows.
template <int D, bool kI8, int NT>
struct Wide {
  static constexpr bool kSmall = NT == 0;
  static constexpr int kTiles = kSmall ? 1 : NT, kRows = kSmall ? 16 : 32, kLanes = 64 / kRows;  // lanes of a row
  static constexpr int kAllRows = kRows * kTiles;
  static constexpr int kBlkVec = kI8 ? 2 * D + 8 : 4 * D;   // uint4 per block and tensor
  static constexpr int kChunks = D / (kI8 ? 32 : 16);       // 16-byte chunks per lane, block and tensor
  static constexpr int kQuerySteps = D / (kLanes * (kI8 ? 16 : 8));  // operands of a score tile's queries
  static constexpr int kScores = kSmall ? 8 : 16;           // scores of a lane per block and tile
  static constexpr int kProbs = kScores / 8;                // operands of the V product
  static constexpr int kAcc = D / kRows;                    // accumulators per tile ...
  static constexpr int kQuads = kSmall ? 1 : 4;             // ... of this many quads of head elements each
  typedef typename std::conditional<kSmall, f32x4, f32x16>::type Acc;

  // Token of the block that a lane's score i belongs to; eight by eight these are the tokens of the cache's V chunks.
  __device__ static int token(int i, int h) {
    return kSmall ? 16 * (i >> 2) + 4 * h + (i & 3) : 16 * ((i >> 2) & 1) + 8 * (i >> 3) + 4 * h + (i & 3);
  }
  // Chunk x of K: this lane's token and which 16 bytes of its row.  (32 rows: bits 3 and 4 of the row exchanged.)
  __device__ static int k_token(int x, int c) {
    return kSmall ? 16 * (x / (kChunks / 2)) + c : (c & 7) | ((c & 8) << 1) | ((c & 16) >> 1);
  }
  __device__ static int k_part(int x, int h) { return kSmall ? 4 * (x % (kChunks / 2)) + h : 2 * x + h; }
  // First head element of a lane's fragment f of V chunk x (INT8 chunks hold two fragments)
  __device__ static int v_elem(int x, int f, int c) {
    return kSmall ? (kI8 ? 32 * x + 16 * f + c : 16 * x + c) : kI8 ? 64 * (x >> 1) + 32 * (c >> 4) + 16 * f + (c & 15) : 32 * (x >> 1) + c;
  }
  // First of the four head elements of quad q of accumulator a
  __device__ static int elem(int a, int q, int h) {
    return kSmall ? 16 * a + 4 * h : kI8 ? 64 * (a >> 1) + 32 * (q >> 1) + 16 * (a & 1) + 8 * (q & 1) + 4 * h : 32 * a + 8 * q + 4 * h;
  }
  // Where a lane's chunks lie in a block (uint4): a lane offset and a step per chunk.
  __device__ static int k_lane(int lane) {
    const int c = lane & 31, t = k_token(0, c);
    return kSmall ? lane : (t >> 4) * (32 * kChunks) + (lane >> 5) * 16 + (t & 15);
  }
  __device__ static int v_lane(int lane) { return kSmall ? lane : ((lane >> 4) & 1) * 64 + (lane >> 5) * 16 + (lane & 15); }
  __device__ static constexpr int k_step(int x) { return kSmall ? 64 * x : (x >> 1) * 64 + (x & 1) * 32; }
  __device__ static constexpr int v_step(int x) { return kSmall ? 64 * x : (x >> 1) * 128 + (x & 1) * 32; }

  __device__ static float row_max(float v) {  // over the lanes of a row
    if constexpr (kSmall) return rows4_max(v);
    const u32x2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  }
  __device__ static float row_sum(float v) {
    if constexpr (kSmall) return rows4_sum(v);
    const u32x2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
  }
};

// Place of a quad of head elements in a partial.  Slots lie 32 KB apart at 64 rows of 128: without the rotation all workgroups would
// write to the same few memory channels at a time.
template <int D>
__device__ inline int wide_quad(int quad, int slot) { return (quad + slot) & (D / 4 - 1); }

// A block on its way to its wavefront, and (INT8) one scale: lane l < 32 the K scale of token l, lane l >= 32 the V scale of
// token l - 32.
template <int D, bool kI8>
struct WideBlock {
  static constexpr int kChunks = D / (kI8 ? 32 : 16);
  u32x4 k[kChunks], v[kChunks];
  float scale;
};

template <int D, bool kI8, int NT>
struct WideQueries {
  using G = Wide<D, kI8, NT>;
  u32x4 q[G::kTiles][G::kQuerySteps];  // operand B of the score tiles
  float row_scale[G::kTiles];          // INT8: row scale * |softmax scale| * log2(e)
  int lim[G::kTiles];                  // last token visible to the row
};

// The queries go through LDS, because an operand's rows lie far apart: fetched by the wavefronts themselves, each would touch 32
// cache lines with every load.  The workgroup fetches them row by row (8 elements per lane: kLoads per thread), INT8 caches quantize them
// there like cache rows (a row's D / 8 lanes agree on its largest magnitude), and every wavefront reads its operands from LDS.
template <int D, bool kI8, int NT>
struct WideQueryRows {
  static constexpr int kRows = Wide<D, kI8, NT>::kAllRows;
  static constexpr int kRowBytes = D * (kI8 ? 1 : 2) + 16;  // 16 bytes apart in the banks
  static constexpr int kPieces = kRows * (D / 8), kLoads = (kPieces + 64 * kWideWaves - 1) / (64 * kWideWaves);
  __align__(16) unsigned char q[kRows * kRowBytes];
  float row_scale[kI8 ? kRows : 1];
};

// A negative softmax scale is moved into the queries (exact) and so is a zero, so that the factor that is left is positive: the
// largest product is the largest score, and masked ones stay -inf.
template <int D, bool kI8, int NT>
__device__ inline void commit_wide_queries(const AttnParams& p, const Unit& u, int tid, const u32x4 (&raw)[WideQueryRows<D, kI8, NT>::kLoads],
                                           WideQueryRows<D, kI8, NT>& lds) {
  const uint32_t flip = p.scale_log2 < 0.f ? 0x80008000u : 0u;
#pragma unroll
  for (int x = 0; x < lds.kLoads; ++x) {
    const int at = x * 64 * kWideWaves + tid, row = at / (D / 8), ck = at % (D / 8);
    const u32x4 v = (raw[x] ^ flip) & (row < u.nq * p.g && p.scale_log2 != 0.f ? 0xFFFFFFFFu : 0u);
    if constexpr (kI8) {
      const uint4 w = __builtin_bit_cast(uint4, v);
      float amax = amax8(w);
#pragma unroll
      for (int o = D / 16; o >= 1; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
      const float scale = amax / 127.0f * fabsf(p.scale_log2);
      const float inv = amax > 0.f && scale != 0.f ? 127.0f / amax : 0.f;
      if (row < lds.kRows) {
        *(uint2*)&lds.q[row * lds.kRowBytes + 8 * ck] = quantize8(w, inv);
        if (ck == 0) lds.row_scale[row] = scale != 0.f ? scale : 1.f;
      }
    } else if (row < lds.kRows) {
      *(u32x4*)&lds.q[row * lds.kRowBytes + 16 * ck] = v;
    }
  }
}

template <int D, bool kI8, int NT>
__device__ inline void read_wide_queries(const AttnParams& p, const Unit& u, int c, int h, const WideQueryRows<D, kI8, NT>& lds,
                                         WideQueries<D, kI8, NT>& q) {
  using G = Wide<D, kI8, NT>;
#pragma unroll
  for (int nt = 0; nt < G::kTiles; ++nt) {
    const int row = G::kRows * nt + c;
    q.lim[nt] = u.L + (row < u.nq * p.g ? row_token(p, row) : 0);
#pragma unroll
    for (int x = 0; x < G::kQuerySteps; ++x) q.q[nt][x] = *(const u32x4*)&lds.q[row * lds.kRowBytes + 16 * (G::kLanes * x + h)];
    if constexpr (kI8) q.row_scale[nt] = lds.row_scale[row];
  }
}

template <int D, bool kI8, int NT>
struct WideState {
  using G = Wide<D, kI8, NT>;
  typename G::Acc acc[G::kTiles][G::kAcc];
  float m[G::kTiles], l[G::kTiles];  // running maximum (log2 units; the same in all lanes of a row), this lane's share of the sum
};

// The step's own rows of a unit in LDS ([row][D] bf16, or codes and one scale per row), as in the one-tile kernel.
template <int D, bool kI8, int NT>
struct WideNewRows {
  static constexpr int kRows = Wide<D, kI8, NT>::kAllRows, kElem = kI8 ? 1 : 2;
  __align__(16) unsigned char k[kRows * D * kElem], v[kRows * D * kElem];
  float k_scale[kI8 ? kRows : 1], v_scale[kI8 ? kRows : 1];
};

// New tokens into a fetched block's registers.
template <int D, bool kI8, int NT>
__device__ inline void patch_wide(WideBlock<D, kI8>& r, int tok0, int L, int nq, int lane, const WideNewRows<D, kI8, NT>& nr) {
  using G = Wide<D, kI8, NT>;
  const int c = lane % G::kRows, h = lane / G::kRows;
#pragma unroll
  for (int x = 0; x < G::kChunks; ++x) {
    const int i = tok0 + G::k_token(x, c) - L;
    if (i >= 0 && i < nq) r.k[x] = *(const u32x4*)&nr.k[(size_t)i * D * nr.kElem + 16 * G::k_part(x, h)];
  }
  if constexpr (kI8) {
    const int i = tok0 + lane % 32 - L;
    if (i >= 0 && i < nq) r.scale = lane < 32 ? nr.k_scale[i] : nr.v_scale[i];
  }
#pragma unroll
  for (int s = 0; s < G::kProbs; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = tok0 + G::token(8 * s + j, h) - L;
      if (i >= 0 && i < nq) {
#pragma unroll
        for (int x = s; x < G::kChunks; x += G::kProbs) {  // the chunks of these tokens
          if constexpr (kI8) {
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              const uint32_t code = nr.v[i * D + G::v_elem(x, f, c)];
              const int word = 2 * f + (j >> 2), sh = 8 * (j & 3);
              r.v[x][word] = (r.v[x][word] & ~(0xFFu << sh)) | (code << sh);
            }
          } else {
            const uint32_t val = *(const uint16_t*)&nr.v[2 * (i * D + G::v_elem(x, 0, c))];
            r.v[x][j >> 1] = (j & 1) ? (r.v[x][j >> 1] & 0x0000FFFFu) | (val << 16) : (r.v[x][j >> 1] & 0xFFFF0000u) | val;
          }
        }
      }
    }
}

// Scores of a block in log2 units.  INT8: integer products times the product of the token's and the row's scale, which is in range
// where the scales and the integers one after the other need not be.
template <int D, bool kI8, int NT>
__device__ inline void wide_scores(const WideBlock<D, kI8>& r, const WideQueries<D, kI8, NT>& q, float abs_scale_log2, int h, const float* scales,
                                   float (&s)[Wide<D, kI8, NT>::kTiles][Wide<D, kI8, NT>::kScores]) {
  using G = Wide<D, kI8, NT>;
  constexpr int n = G::kQuerySteps;
#pragma unroll
  for (int nt = 0; nt < G::kTiles; ++nt) {
    if constexpr (G::kSmall) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if constexpr (kI8) {
          i32x4 z = {0, 0, 0, 0};
#pragma unroll
          for (int x = 0; x < n; ++x)
            z = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, r.k[t * n + x]), __builtin_bit_cast(i32x4, q.q[nt][x]), z, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) s[nt][4 * t + i] = (float)z[i];
        } else {
          f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int x = 0; x < n; ++x)
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.k[t * n + x]), __builtin_bit_cast(bf16x8, q.q[nt][x]), z, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) s[nt][4 * t + i] = z[i];
        }
      }
    } else if constexpr (kI8) {
      i32x16 z = {0};
#pragma unroll
      for (int x = 0; x < n; ++x)
        z = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(i32x4, r.k[x]), __builtin_bit_cast(i32x4, q.q[nt][x]), z, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) s[nt][i] = (float)z[i];
    } else {
      f32x16 z = {0.f};
#pragma unroll
      for (int x = 0; x < n; ++x)
        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, r.k[x]), __builtin_bit_cast(bf16x8, q.q[nt][x]), z, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) s[nt][i] = z[i];
    }
    // A rounded product, as the maximum is: fused with the subtraction of the maximum, the largest probability would not be 1 but 2 to
    // the power of what the rounding took from the maximum, which costs precision from 2^10 on and is not finite from 2^31 on.
#pragma unroll
    for (int y = 0; y < G::kScores / 4; ++y) {
#pragma clang fp contract(off)
      f32x4 scale = {abs_scale_log2, abs_scale_log2, abs_scale_log2, abs_scale_log2};
      if constexpr (kI8) scale = *(const f32x4*)&scales[G::token(4 * y, h)] * q.row_scale[nt];
#pragma unroll
      for (int e = 0; e < 4; ++e) s[nt][4 * y + e] *= scale[e];
    }
  }
}

// A block that reaches beyond ctx_len: causal limits; and stale cache rows may hold anything, NaN included: they are zero in V
// (bf16), so that 0 * garbage cannot reach the accumulator.  In place and apart from the step itself: two instances of the step,
// with and without masks, would make the compiler merge their register tuples and spill hundreds of them.
template <int D, bool kI8, int NT>
__device__ inline void mask_wide(WideBlock<D, kI8>& r, float (&s)[Wide<D, kI8, NT>::kTiles][Wide<D, kI8, NT>::kScores],
                                 const WideQueries<D, kI8, NT>& q, int tok0, int n_valid, int h) {
  using G = Wide<D, kI8, NT>;
#pragma unroll
  for (int nt = 0; nt < G::kTiles; ++nt)
#pragma unroll
    for (int i = 0; i < G::kScores; ++i)
      if (tok0 + G::token(i, h) > q.lim[nt]) s[nt][i] = -INFINITY;
  if constexpr (!kI8) {
#pragma unroll
    for (int y = 0; y < G::kProbs; ++y)
#pragma unroll
      for (int wd = 0; wd < 4; ++wd) {
        const int t_lo = tok0 + G::token(8 * y + 2 * wd, h);
        const uint32_t keep = (t_lo < n_valid ? 0x0000FFFFu : 0u) | (t_lo + 1 < n_valid ? 0xFFFF0000u : 0u);
#pragma unroll
        for (int x = y; x < G::kChunks; x += G::kProbs) r.v[x][wd] &= keep;
      }
  }
}

// Online softmax of a block: scores -> probabilities as operand B of the V product (INT8: times the tokens' V scales), running
// maximum and sum.  16 rows: with few shares per unit the rounding of the probabilities to bf16 would cost precision (kNarrowUnits); their
// 24 bits are cut into three operands of 8 and all multiplied.  No part is negative, and none is
// zero where the probability is not, so that an infinite element of V stays infinite in every product: the second and third are at
// least 2^-133, the smallest bf16, which the matrix instruction takes as it is (a probability is 0 or at least 2^-126; together they are
// off by at most 2^-132, 2^-22 of a probability of 2^-110).  (Two parts leave 2^-17: 3.6e-6 instead of 2.3e-6 with a rounded first part,
// whose remainder may be negative.)
template <int D, bool kI8, int NT>
__device__ inline void wide_softmax(const float (&s)[Wide<D, kI8, NT>::kTiles][Wide<D, kI8, NT>::kScores], WideState<D, kI8, NT>& st, int h, const float* scales,
                                    bf16x8 (&pf)[Wide<D, kI8, NT>::kTiles][Wide<D, kI8, NT>::kProbs],
                                    bf16x8 (&pr)[2][Wide<D, kI8, NT>::kTiles][Wide<D, kI8, NT>::kProbs]) {
  using G = Wide<D, kI8, NT>;
  auto cut = [](float z) { return __uint_as_float(__float_as_uint(z) & 0xFFFF0000u); };
#pragma unroll
  for (int nt = 0; nt < G::kTiles; ++nt) {
    float mx = s[nt][0];
#pragma unroll
    for (int i = 1; i < G::kScores; ++i) mx = fmaxf(mx, s[nt][i]);
    mx = G::row_max(mx);
    // The reference maximum of a row moves only when a block exceeds it by more than kMaxSlack (log2 units).
    const float m_old = st.m[nt];
    const bool grow = mx > m_old + kMaxSlack;
    if (__any(grow)) {
      const float m_new = grow ? mx : m_old;
      const float alpha = __builtin_amdgcn_exp2f(m_old - (m_new == -INFINITY ? 0.f : m_new));
      st.l[nt] *= alpha;
#pragma unroll
      for (int a = 0; a < G::kAcc; ++a) st.acc[nt][a] *= alpha;
      st.m[nt] = m_new;
    }
    const float m_use = st.m[nt] == -INFINITY ? 0.f : st.m[nt];  // rows without a visible token yet
    float psum = 0.f;
#pragma unroll
    for (int y = 0; y < G::kScores / 4; ++y) {
      f32x4 vs = {1.f, 1.f, 1.f, 1.f};
      if constexpr (kI8) vs = *(const f32x4*)&scales[32 + G::token(4 * y, h)];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 4 * y + e;
        const float pj = __builtin_amdgcn_exp2f(s[nt][i] - m_use);
        psum += pj;
        const float z = kI8 ? pj * vs[e] : pj;
        if constexpr (G::kSmall) {
          const float a = cut(z), b = cut(z - a), least = fminf(z, 0x1p-133f);
          pf[nt][i >> 3][i & 7] = (__bf16)a;
          pr[0][nt][i >> 3][i & 7] = (__bf16)fmaxf(b, least);
          pr[1][nt][i >> 3][i & 7] = (__bf16)fmaxf(z - a - b, least);
        } else {
          pf[nt][i >> 3][i & 7] = (__bf16)z;
        }
      }
    }
    st.l[nt] += psum;
  }
}

template <int D, bool kI8, int NT>
__device__ inline void wide_values(const WideBlock<D, kI8>& r, const bf16x8 (&pf)[Wide<D, kI8, NT>::kTiles][Wide<D, kI8, NT>::kProbs],
                                   const bf16x8 (&pr)[2][Wide<D, kI8, NT>::kTiles][Wide<D, kI8, NT>::kProbs], WideState<D, kI8, NT>& st) {
  using G = Wide<D, kI8, NT>;
  constexpr int kFrags = kI8 ? 2 : 1;  // V fragments of a chunk
#pragma unroll
  for (int x = 0; x < G::kChunks; ++x)
#pragma unroll
    for (int f = 0; f < kFrags; ++f) {
      bf16x8 v;
      if constexpr (kI8) v = __builtin_bit_cast(bf16x8, codes_to_bf16(r.v[x][2 * f], r.v[x][2 * f + 1]));
      else v = __builtin_bit_cast(bf16x8, r.v[x]);
#pragma unroll
      for (int nt = 0; nt < G::kTiles; ++nt) {
        typename G::Acc& acc = st.acc[nt][kFrags * (x / G::kProbs) + f];
        if constexpr (G::kSmall) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pr[1][nt][0], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pr[0][nt][0], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pf[nt][0], acc, 0, 0, 0);
        } else {
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pf[nt][x & 1], acc, 0, 0, 0);
        }
      }
    }
}

// Merge of a unit's partials, in their order, by the workgroup that delivered the last of them: its O and lse.  Every thread has one
// row of a tile and some quads of head elements; up to four partials (16 rows: eight) are on their way at a time.
struct WideJob {
  int b, kvh, nq, w_lo, n;
};

template <int D, bool kI8, int NT>
__device__ inline void merge_wide(const AttnParams& p, const WideJob& j, int wv, int lane) {
  using G = Wide<D, kI8, NT>;
  constexpr int kTiles = G::kTiles, kQuads = D / 4 / (kWideWaves * G::kLanes), kRoundW = G::kSmall ? 8 : 4;
  const int c = lane % G::kRows, h = lane / G::kRows, rows = j.nq * p.g;
  const int slot0 = j.w_lo + j.b * p.Hkv + j.kvh;
  const unsigned slot_bytes = (unsigned)p.rows_max * D * 4, ml_bytes = (unsigned)p.rows_max * 8;
  float M[kTiles], L[kTiles];
  f32x4 o[kTiles][kQuads];
#pragma unroll
  for (int nt = 0; nt < kTiles; ++nt) {
    M[nt] = -INFINITY;
    L[nt] = 0.f;
#pragma unroll
    for (int k = 0; k < kQuads; ++k) o[nt][k] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto quad_of = [&](int k) { return G::kLanes * (wv + kWideWaves * k) + h; };
  for (int j0 = 0; j0 < j.n; j0 += kRoundW) {
    const int n = min(j.n - j0, kRoundW);
    // partials that do not exist and idle rows: beyond the buffers, answered with zeros
    const __amdgpu_buffer_rsrc_t rs = dev_buffer(p.part_acc + (size_t)(slot0 + j0) * p.rows_max * D, (unsigned)n * slot_bytes);
    const __amdgpu_buffer_rsrc_t rs_ml = dev_buffer(p.part_ml + (size_t)(slot0 + j0) * p.rows_max * 2, (unsigned)n * ml_bytes);
    float2 s[kTiles][kRoundW];
    f32x4 a[kTiles][kRoundW][kQuads];
#pragma unroll
    for (int x = 0; x < kRoundW; ++x)
#pragma unroll
      for (int nt = 0; nt < kTiles; ++nt) {
        const int row = G::kRows * nt + c;
        s[nt][x] = load_dev2(rs_ml, row < rows ? x * ml_bytes + 8u * row : kNoSuchOffset);
#pragma unroll
        for (int k = 0; k < kQuads; ++k)
          a[nt][x][k] = load_dev4(rs, row < rows ? x * slot_bytes + 16u * (wide_quad<D>(quad_of(k), slot0 + j0 + x) * p.rows_max + row) : kNoSuchOffset);
      }
#pragma unroll
    for (int nt = 0; nt < kTiles; ++nt) {
      // a valid row has a visible token (token 0) in the first partial, so M is finite from there on
      const float M_old = M[nt];
#pragma unroll
      for (int x = 0; x < kRoundW; ++x)
        if (x < n) M[nt] = fmaxf(M[nt], s[nt][x].x);
      const float Mf = M[nt] == -INFINITY ? 0.f : M[nt], alpha = __builtin_amdgcn_exp2f(M_old - Mf);
      L[nt] *= alpha;
#pragma unroll
      for (int k = 0; k < kQuads; ++k) o[nt][k] *= alpha;
#pragma unroll
      for (int x = 0; x < kRoundW; ++x)
        if (x < n) {
          const float wgt = __builtin_amdgcn_exp2f(s[nt][x].x - Mf);
          L[nt] = fmaf(s[nt][x].y, wgt, L[nt]);
#pragma unroll
          for (int k = 0; k < kQuads; ++k) o[nt][k] += a[nt][x][k] * wgt;
        }
    }
  }
#pragma unroll
  for (int nt = 0; nt < kTiles; ++nt) {
    const int row = G::kRows * nt + c;
    if (row < rows) {
      const int i = row_token(p, row), hg = row - i * p.g;
      const size_t orow = ((size_t)j.b * p.kmax + i) * p.Hq + j.kvh * p.g + hg;
      const float inv = __builtin_amdgcn_rcpf(L[nt]);
#pragma unroll
      for (int k = 0; k < kQuads; ++k) *(f32x4*)(p.O + orow * D + 4 * quad_of(k)) = o[nt][k] * inv;
      if (p.lse && wv == 0 && h == 0) p.lse[orow] = (M[nt] + __builtin_amdgcn_logf(L[nt])) * 0.6931471805599453f;
    }
  }
}

template <int D, bool kI8, int NT>
__global__ __launch_bounds__(64 * kWideWaves, 1) void verify_attn_wide(AttnParams p) {
  using G = Wide<D, kI8, NT>;
  constexpr int W = kWideWaves, kTiles = G::kTiles, kRows = G::kRows, kQuads = G::kQuads;
  constexpr int kAccs = kTiles * G::kAcc;  // accumulators; wavefront x % W collects number x
  constexpr bool kMerge = NT <= 1;  // units that several workgroups share are merged here, not by reduce_wide
  constexpr int kBlkVec = G::kBlkVec;
  constexpr int R = 2;  // blocks a wavefront has in its registers or on the way there (three: 1 - 2 us longer)
  using Block = WideBlock<D, kI8>;
  __shared__ f32x4 exchange[kAccs][W - 1][kQuads][64];
  __shared__ float wave_m[W][kTiles][kRows], wave_l[W][kTiles][kRows];
  __shared__ __align__(16) float scales[W][kI8 ? 64 : 1];
  static_assert(__alignof__(scales) % 16 == 0, "read four at a time (wide_scores, wide_softmax)");
  __shared__ int arrived_last[2];
  __shared__ WideQueryRows<D, kI8, NT> q_lds;
  __shared__ WideNewRows<D, kI8, NT> rows_lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6);
  const int c = lane % kRows, h = lane / kRows;
  const int wg = blockIdx.x;  // the stretch of this workgroup
  const bool fused = p.Knew != nullptr;

  const ShareRecord* rec = p.records + wg;
  Segment seg = load_segment(&rec->seg[0]);
  const int nseg = uniform(rec->nseg), overflow = uniform(rec->overflow), rec_flags = uniform(rec->flags);
  if (!record_matches(p, rec)) {
    report_mismatch(p, wg == 0 && tid == 0);
    return;
  }
  if (kMerge && (rec_flags & kRecAnyInactive)) zero_unused_rows<D, true>(p, wg * W + wv, gridDim.x * W, lane);
  if (nseg == 0) return;

  const uint4* kc = (const uint4*)p.Kc;
  const uint4* vc = (const uint4*)p.Vc;
  const float abs_scale = p.scale_log2 == 0.f ? 1.f : fabsf(p.scale_log2);
  const int k_lane = 16 * G::k_lane(lane), v_lane = 16 * G::v_lane(lane);
  // The wavefronts take the stretch's blocks in turn: this one's t-th block of the segment at hand is block turn + W t.  All fetches
  // are unconditional (exact wait counts); one past the end goes through a buffer descriptor of size zero and touches nothing.
  int turn = wv;
  auto block_buffer = [&](const uint4* cache, const Segment& g, int t) {
    const int x = turn + W * t;
    const uint4* at = cache + (((ptrdiff_t)g.b * p.Hkv + g.kvh) * p.nblk_cap + g.first + x) * kBlkVec;
    return dev_buffer((const float*)at, x < g.n ? 16u * kBlkVec : 0u);
  };
  auto fetch_k = [&](Block& r, const Segment& g, int t) {
    const __amdgpu_buffer_rsrc_t at = block_buffer(kc, g, t);
#pragma unroll
    for (int x = 0; x < Block::kChunks; ++x) r.k[x] = __builtin_amdgcn_raw_buffer_load_b128(at, k_lane, 16 * G::k_step(x), kAuxNonTemporal);
    if constexpr (kI8) {
      const int x = turn + W * t;
      const ptrdiff_t off = (((ptrdiff_t)g.b * p.Hkv + g.kvh) * p.nblk_cap + g.first + (x < g.n ? x : 0)) * kBlkVec;
      r.scale = ((const float*)((lane < 32 ? kc : vc) + off + 2 * D))[lane % 32];
    }
  };
  auto fetch_v = [&](Block& r, const Segment& g, int t) {
    const __amdgpu_buffer_rsrc_t at = block_buffer(vc, g, t);
#pragma unroll
    for (int x = 0; x < Block::kChunks; ++x) r.v[x] = __builtin_amdgcn_raw_buffer_load_b128(at, v_lane, 16 * G::v_step(x), kAuxNonTemporal);
  };

  // Fused append: the new rows whose blocks are ours go into LDS and into the cache (nothing but the new rows is written: other
  // appends may write other tokens of the same blocks), 8 elements of a row per lane.  The first pass is requested ahead of the
  // first blocks; all conditions are workgroup-uniform.
  auto first_new_row = [&](const Segment& g) { return max(0, g.first * kBlockTokens - g.L); };
  auto new_rows_of = [&](const Segment& g) { return min(g.nq, (g.first + g.n) * kBlockTokens - g.L) - first_new_row(g); };
  u32x4 new_k = {0u, 0u, 0u, 0u}, new_v = new_k;
  auto request_rows = [&](const Segment& g, int c0) {
    const int x = min(c0 + tid, new_rows_of(g) * (D / 8) - 1);  // whole rows, also past the end
    const int i = first_new_row(g) + x / (D / 8);
    const size_t src = (((size_t)g.b * p.kmax + i) * p.Hkv + g.kvh) * D + 8 * (tid % (D / 8));
    new_k = *(const u32x4*)((const uint16_t*)p.Knew + src);
    new_v = *(const u32x4*)((const uint16_t*)p.Vnew + src);
  };
  auto commit_rows = [&](const Segment& g, int c0) {
    WideNewRows<D, kI8, NT>& nr = rows_lds;
    const int n_ck = new_rows_of(g) * (D / 8), x = min(c0 + tid, n_ck - 1);
    const int ck = tid % (D / 8), i = first_new_row(g) + x / (D / 8);
    const int blk = (g.L + i) / kBlockTokens, tw = (g.L + i) % kBlockTokens;
    const uint4 kv = __builtin_bit_cast(uint4, new_k), vv = __builtin_bit_cast(uint4, new_v);
    const size_t at = (((size_t)g.b * p.Hkv + g.kvh) * p.nblk_cap + blk) * (size_t)kBlkVec * 16;
    uint8_t* kblk = (uint8_t*)const_cast<void*>(p.Kc) + at;
    uint8_t* vblk = (uint8_t*)const_cast<void*>(p.Vc) + at;
    if constexpr (kI8) {  // quantized as the append kernel does: a row's D / 8 lanes agree on its largest magnitude
      float ka = amax8(kv), va = amax8(vv);
#pragma unroll
      for (int o = D / 16; o >= 1; o >>= 1) {
        ka = fmaxf(ka, __shfl_xor(ka, o));
        va = fmaxf(va, __shfl_xor(va, o));
      }
      const float kinv = ka > 0.f ? 127.0f / ka : 0.f;
      const float vinv = va > 0.f ? 127.0f / va : 0.f;
      if (c0 + tid < n_ck) {
        const uint2 kq = quantize8(kv, kinv), vq = quantize8(vv, vinv);
        *(uint2*)&nr.k[i * D + 8 * ck] = kq;
        *(uint2*)&nr.v[i * D + 8 * ck] = vq;
        *(uint2*)(kblk + i8_k_offset(D, tw, 8 * ck)) = kq;
#pragma unroll
        for (int e = 0; e < 8; ++e) vblk[i8_v_offset(D, tw, 8 * ck + e)] = (uint8_t)((e < 4 ? vq.x : vq.y) >> (8 * (e & 3)));
        if (ck == 0) {
          const float ks = ka / 127.0f, vs = va / 127.0f;
          nr.k_scale[i] = ks;
          nr.v_scale[i] = vs;
          ((float*)(kblk + kBlockTokens * D))[tw] = ks;
          ((float*)(vblk + kBlockTokens * D))[tw] = vs;
        }
      }
    } else if (c0 + tid < n_ck) {
      *(uint4*)&nr.k[2 * (i * D + 8 * ck)] = kv;
      *(uint4*)&nr.v[2 * (i * D + 8 * ck)] = vv;
      *(uint4*)(kblk + 2 * k_elem_offset(D, tw, 8 * ck)) = kv;
      const uint32_t vw[4] = {vv.x, vv.y, vv.z, vv.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) ((uint16_t*)vblk)[v_elem_offset(D, tw, 8 * ck + e)] = (uint16_t)(vw[e >> 1] >> (16 * (e & 1)));
    }
  };

  Block ring[R];
  u32x4 raw_q[WideQueryRows<D, kI8, NT>::kLoads];
  auto request_queries = [&](const Segment& g) {  // rows that do not exist read row 0
    const int rows = g.nq * p.g;
#pragma unroll
    for (int x = 0; x < WideQueryRows<D, kI8, NT>::kLoads; ++x) {
      const int at = x * 64 * W + tid, row = at / (D / 8) < rows ? at / (D / 8) : 0, ck = at % (D / 8);
      const int i = row_token(p, row), hg = row - i * p.g;
      raw_q[x] = ((const u32x4*)((const uint16_t*)p.Q + (((size_t)g.b * p.kmax + i) * p.Hq + g.kvh * p.g + hg) * D))[ck];
    }
  };
  auto begin = [&](const Segment& g) {
    fetch_k(ring[0], g, 0);
    request_queries(g);
    if (fused && new_rows_of(g) > 0) request_rows(g, 0);
    fetch_v(ring[0], g, 0);
#pragma unroll
    for (int x = 1; x < R; ++x) {
      fetch_k(ring[x], g, x);
      fetch_v(ring[x], g, x);
    }
  };
  WideJob job_a{}, job_b{};  // units that others contribute to
  int shared = 0;
  begin(seg);
  for (int si = 0;; ++si) {
    const Unit u = unit_of(seg);
    const int rows = u.nq * p.g, tiles = (rows + kRows - 1) / kRows;
    const int first_mine = turn, n_mine = (seg.n - turn + W - 1) / W;  // 0 for n <= turn
    commit_wide_queries<D, kI8, NT>(p, u, tid, raw_q, q_lds);
    if (fused && new_rows_of(seg) > 0) {
      commit_rows(seg, 0);
      for (int c0 = 64 * W; c0 < new_rows_of(seg) * (D / 8); c0 += 64 * W) {
        request_rows(seg, c0);
        commit_rows(seg, c0);
      }
    }
    __syncthreads();
    WideQueries<D, kI8, NT> q;
    read_wide_queries<D, kI8, NT>(p, u, c, h, q_lds, q);
    WideState<D, kI8, NT> st;
#pragma unroll
    for (int nt = 0; nt < kTiles; ++nt) {
      st.m[nt] = -INFINITY;
      st.l[nt] = 0.f;
#pragma unroll
      for (int a = 0; a < G::kAcc; ++a)
#pragma unroll
        for (int i = 0; i < 4 * kQuads; ++i) st.acc[nt][a][i] = 0.f;
    }
    auto step = [&](Block& r, int t) {
      const int tok0 = (seg.first + first_mine + W * t) * kBlockTokens;
      // every token of the block is visible to every query and, with a fused append, none of them is new
      const bool plain = tok0 + kBlockTokens - 1 < u.L + (fused ? 0 : 1);
      if (fused && !plain) patch_wide<D, kI8, NT>(r, tok0, u.L, u.nq, lane, rows_lds);
      float* sc = scales[wv];
      if constexpr (kI8) {
        sc[lane] = (lane >= 32 && tok0 + lane - 32 >= u.L + u.nq) ? 0.f : r.scale;  // stale tokens may carry any V scale
        __builtin_amdgcn_wave_barrier();  // a wavefront's LDS accesses stay in order
      }
      float s[kTiles][G::kScores];
      wide_scores<D, kI8, NT>(r, q, abs_scale, h, sc, s);
      fetch_k(r, seg, t + R);
      if (!plain) mask_wide<D, kI8, NT>(r, s, q, tok0, u.L + u.nq, h);
      bf16x8 pf[kTiles][G::kProbs], pr[2][kTiles][G::kProbs];
      wide_softmax<D, kI8, NT>(s, st, h, sc, pf, pr);
      if constexpr (kI8) __builtin_amdgcn_wave_barrier();
      wide_values<D, kI8, NT>(r, pf, pr, st);
      fetch_v(r, seg, t + R);
    };
    for (int t = 0; t < n_mine; t += R) {
#pragma unroll
      for (int x = 0; x < R; ++x) {
        if (x > 0 && t + x >= n_mine) break;
        step(ring[x], t + x);
      }
    }

    // the next segment's queries and first blocks travel while this one's states are merged
    const bool more = si + 1 < nseg;
    const Segment done = seg;
    if (more) {
      turn = (first_mine - seg.n) & (W - 1);
      seg = later_segment(p, rec, overflow, si + 1);
      begin(seg);
    }

    // merge of the four wavefronts' states: M = max m_w, weights 2^(m_w - M) (a wavefront that saw no visible token has m = -inf
    // and weight 0)
#pragma unroll
    for (int nt = 0; nt < kTiles; ++nt) {
      const float l = G::row_sum(st.l[nt]);
      if (h == 0) {
        wave_m[wv][nt][c] = st.m[nt];
        wave_l[wv][nt][c] = l;
      }
    }
    __syncthreads();
    float M[kTiles], sum[kTiles], mine[kTiles];
#pragma unroll
    for (int nt = 0; nt < kTiles; ++nt) {
      M[nt] = -INFINITY;
      sum[nt] = 0.f;
#pragma unroll
      for (int w = 0; w < W; ++w) M[nt] = fmaxf(M[nt], wave_m[w][nt][c]);
      const float Mf = M[nt] == -INFINITY ? 0.f : M[nt];
#pragma unroll
      for (int w = 0; w < W; ++w) sum[nt] += wave_l[w][nt][c] * __builtin_amdgcn_exp2f(wave_m[w][nt][c] - Mf);
      mine[nt] = __builtin_amdgcn_exp2f(st.m[nt] - Mf);
    }
    auto quad = [&](int x, int y) {
      const typename G::Acc& t = st.acc[x / G::kAcc][x % G::kAcc];
      return f32x4{t[4 * y], t[4 * y + 1], t[4 * y + 2], t[4 * y + 3]};
    };
#pragma unroll
    for (int x = 0; x < kAccs; ++x) {
      const int nt = x / G::kAcc, owner = x % W;
      if (nt > 0 && nt >= tiles) break;
      st.acc[nt][x % G::kAcc] *= mine[nt];
      if (wv != owner) {
#pragma unroll
        for (int y = 0; y < kQuads; ++y) exchange[x][wv < owner ? wv : wv - 1][y][lane] = quad(x, y);
      }
    }
    __syncthreads();
    const bool solo = kMerge && seg_w_lo(done) == seg_w_hi(done);
    const size_t slot = (size_t)wg + (size_t)done.b * p.Hkv + done.kvh;
    const __amdgpu_buffer_rsrc_t rs = dev_buffer(p.part_acc + slot * p.rows_max * D, (unsigned)p.rows_max * D * 4);
#pragma unroll
    for (int x = 0; x < kAccs; ++x) {
      const int nt = x / G::kAcc, a = x % G::kAcc;
      if (wv != x % W) continue;
      if (nt > 0 && nt >= tiles) break;
      const int rrow = kRows * nt + c, i = row_token(p, rrow), hg = rrow - i * p.g;
      const size_t orow = ((size_t)done.b * p.kmax + i) * p.Hq + done.kvh * p.g + hg;
      f32x4 v[kQuads];
#pragma unroll
      for (int y = 0; y < kQuads; ++y) {
        v[y] = quad(x, y);
#pragma unroll
        for (int w = 0; w < W - 1; ++w) v[y] += exchange[x][w][y][lane];
      }
      if (rrow < rows) {
        if (solo) {
          const float inv = __builtin_amdgcn_rcpf(sum[nt]);
#pragma unroll
          for (int y = 0; y < kQuads; ++y) *(f32x4*)(p.O + orow * D + G::elem(a, y, h)) = v[y] * inv;
        } else {
#pragma unroll
          for (int y = 0; y < kQuads; ++y) store_dev4(rs, (unsigned)(wide_quad<D>(G::elem(a, y, h) / 4, (int)slot) * p.rows_max + rrow) * 16, v[y]);
        }
        if (a == 0 && h == 0) {
          if (!solo) store_dev(p.part_ml + (slot * p.rows_max + rrow) * 2, M[nt], sum[nt]);
          else if (p.lse) p.lse[orow] = (M[nt] + __builtin_amdgcn_logf(sum[nt])) * 0.6931471805599453f;
        }
      }
    }
    if (kMerge && (done.flags & kSegLast)) {  // query slots beyond draft_len are zero in O and lse
      for (int x = tid; x < (p.rows_max - rows) * (D / 4); x += 64 * W) {
        const int row = rows + x / (D / 4), i = row_token(p, row), hg = row - i * p.g;
        const size_t orow = ((size_t)done.b * p.kmax + i) * p.Hq + done.kvh * p.g + hg;
        *(f32x4*)(p.O + orow * D + 4 * (x % (D / 4))) = f32x4{0.f, 0.f, 0.f, 0.f};
        if (p.lse && x % (D / 4) == 0) p.lse[orow] = 0.f;
      }
    }
    if (kMerge && !solo) {  // a stretch's first and last unit at most
      const WideJob job{done.b, done.kvh, done.nq, seg_w_lo(done), seg_w_hi(done) - seg_w_lo(done) + 1};
      if (shared == 0) job_a = job;
      job_b = job;
      ++shared;
    }
    if (!more) break;
  }

  // Delivery: this workgroup's partials have reached the device-coherent level once every wavefront's stores are acknowledged; only
  // then is its arrival counted, and who counts last merges (the ordering of the one-tile kernel's partials).
  if (!kMerge || shared == 0) return;
  partial_stores_done();
  __syncthreads();
  if (tid < shared) {
    int32_t* counter = p.counters + (tid == 0 ? job_a.b * p.Hkv + job_a.kvh : job_b.b * p.Hkv + job_b.kvh);
    const bool last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (tid == 0 ? job_a.n : job_b.n) - 1;
    if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // clean for the next call
    arrived_last[tid] = last;
  }
  __syncthreads();
  if (uniform(arrived_last[0])) merge_wide<D, kI8, NT>(p, job_a, wv, lane);
  if (shared > 1 && uniform(arrived_last[1])) merge_wide<D, kI8, NT>(p, job_b, wv, lane);
}

// ---------------------------------------------------------------------------------------
// Short caches or few units (launch_shape), more than 32 query rows: a workgroup with a wavefront (bf16: two) per 16-row tile.  With few blocks per
// unit what counts is the time of one block and of the way out: four wavefronts share a block's rows here, and no states of several
// tiles have to be merged at the end.
// bf16: every K/V block is fetched from memory once (each wavefront a part of it), put into a ring in LDS, two blocks per phase, and
// read from there by the wavefronts that own a query tile (rows 16 t .. 16 t + 15), one for the even and one for the odd blocks,
// whose states are merged through LDS at the end of the unit.  One barrier per phase: a slot is rewritten only after the barrier that
// follows the last step that read it.  Every barrier sits in workgroup-uniform control flow (the stretch, the units and the block
// counts depend on the workgroup index and the lengths only).
// ---------------------------------------------------------------------------------------
// Partial of a 16-row tile in the layout of reduce_wide.
template <int D>
__device__ inline void store_partial_quads(const AttnParams& p, const Unit& u, int w, const RowState<D>& st, int col, int grp, int row0) {
  const int rrow = row0 + col;
  const size_t slot = (size_t)w + (size_t)u.b * p.Hkv + u.kvh;
  const __amdgpu_buffer_rsrc_t rs = dev_buffer(p.part_acc + slot * p.rows_max * D, (unsigned)p.rows_max * D * 4);
  const float l = rows4_sum(st.l);
  if (rrow < u.nq * p.g) {
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) store_dev4(rs, (unsigned)(wide_quad<D>(4 * mt + grp, (int)slot) * p.rows_max + rrow) * 16, st.acc[mt]);
    if (grp == 0) store_dev(p.part_ml + (slot * p.rows_max + rrow) * 2, st.m, l);
  }
}

// Two wavefronts per tile: the state of the odd blocks joins that of the even ones (one that saw no visible token has
// m = -inf and no weight).  All wavefronts call; a stretch of one block has nothing to join.  acc: LDS for TW tiles' accumulators.
template <int D, int TW>
__device__ inline void merge_halves(RowState<D>& st, int n, int half, int tile, bool active, int lane, f32x4* acc,
                                    float (&other_m)[TW][64], float (&other_l)[TW][64]) {
  if (n <= 1) return;  // workgroup-uniform
  __syncthreads();     // the last steps have left the ring
  f32x4* other_acc = acc + tile * (D / 16) * 64 + lane;
  if (half == 1 && active) {
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) other_acc[mt * 64] = st.acc[mt];
    other_m[tile][lane] = st.m;
    other_l[tile][lane] = st.l;
  }
  __syncthreads();
  if (half == 0 && active) {
    const float m1 = other_m[tile][lane], M = fmaxf(st.m, m1), Mf = M == -INFINITY ? 0.f : M;
    const float w0 = __builtin_amdgcn_exp2f(st.m - Mf), w1 = __builtin_amdgcn_exp2f(m1 - Mf);
    st.m = M;
    st.l = st.l * w0 + other_l[tile][lane] * w1;
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) st.acc[mt] = st.acc[mt] * w0 + other_acc[mt * 64] * w1;
  }
}

template <int D, bool kFused>
__global__ __launch_bounds__(512, 2) void verify_attn_tiles_bf16(AttnParams p) {
  constexpr int TW = 4, H = 2, kThreads = 64 * TW * H;
  constexpr int kTileAhead = 2;                       // phases a workgroup has in flight from memory
  constexpr int kBlkVec = kBlockTokens * D * 2 / 16;  // uint4 per block and tensor
  constexpr int kPhase = H * kBlkVec;                  // ... and per phase (a unit's blocks lie one after the other)
  constexpr int kLoads = kPhase / kThreads;            // 16-byte loads per lane, phase and tensor
  __shared__ uint4 ring_k[2][kPhase];
  __shared__ uint4 ring_v[2][kPhase];
  __shared__ float other_m[TW][64], other_l[TW][64];  // states of the odd blocks' wavefronts (accumulators: in ring_k)
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int tile = wv % TW, half = wv / TW;
  const int col = lane & 15, grp = lane >> 4;
  const int wg = blockIdx.x;  // the stretch of this workgroup
  const int row0 = 16 * tile;

  const ShareRecord* rec = p.records + wg;
  const int nseg = uniform(rec->nseg), overflow = uniform(rec->overflow);
  if (!record_matches(p, rec)) {
    report_mismatch(p, wg == 0 && tid == 0);
    return;
  }
  // (the unused query rows are cleared by the merge launch, which visits every row of every unit anyway)

  const uint4* kc = (const uint4*)p.Kc;
  const uint4* vc = (const uint4*)p.Vc;
  struct Stage {
    uint4 k[kLoads], v[kLoads];
  };

  for (int si = 0; si < nseg; ++si) {
    const Segment seg = si == 0 ? load_segment(&rec->seg[0]) : later_segment(p, rec, overflow, si);
    const Unit u = unit_of(seg);
    const int n = seg.n;  // real blocks seg.first .. seg.first + n - 1 of the unit
    const bool active = uniform(row0 < u.nq * p.g);  // this wavefront owns a query tile of the unit
    QFrag<D> q;
    load_queries<D>(p, u, active, col, grp, q, row0);
    const uint32_t flip = p.scale_log2 < 0.f ? 0x80008000u : 0u;  // a negative scale is moved into the queries, as in verify_attn_wide
#pragma unroll
    for (int t = 0; t < D / 32; ++t) q.q[t] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, q.q[t]) ^ flip);
    RowState<D> st;
    clear_state<D>(st);
    const int blk0 = seg.first;
    const ptrdiff_t vec0 = (((ptrdiff_t)u.b * p.Hkv + u.kvh) * p.nblk_cap + blk0) * kBlkVec;

    // all fetches unconditional (exact wait counts); a block past the end re-reads the stretch's first block
    auto fetch = [&](Stage& g, int ph) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        const int c = i * kThreads + tid, h = i * kThreads / kBlkVec + (tid >= kBlkVec ? 1 : 0);
        const ptrdiff_t off = vec0 + (H * ph + h < n ? (ptrdiff_t)ph * kPhase + c : (ptrdiff_t)(c - h * kBlkVec));
        g.k[i] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4*)(kc + off)));
        g.v[i] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4*)(vc + off)));
      }
    };
    // phase ph (blocks 2 ph and 2 ph + 1): own part into LDS, next fetch, barrier -- for every phase, also past the
    // end (the loads and the barrier stay outside all branches: a load under a branch costs a full wait at the
    // join) -- then, for real blocks, the one-tile step from LDS
    auto phase = [&](Stage& g, int ph) {
      const int slot = ph & 1;
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        ring_k[slot][i * kThreads + tid] = g.k[i];
        ring_v[slot][i * kThreads + tid] = g.v[i];
      }
      fetch(g, ph + kTileAhead);
      // Fused append: blocks that hold new tokens are patched in LDS once they are complete there (K: the
      // 16-byte chunks of the new rows; V: their elements, 2 bytes each), and the same bytes go into the cache: nothing
      // but the new rows is written, other appends may write other tokens of the block.  The test is
      // workgroup-uniform; the loads of the new rows sit under this branch and cost a full wait, in these one or
      // two phases per unit only.
      const int tok0 = (blk0 + H * ph) * kBlockTokens;                     // the phase's tokens that are ours:
      const int tok1 = (blk0 + min(H * ph + H, n)) * kBlockTokens;         // tok0 .. tok1 - 1
      if (kFused && u.nq > 0 && tok0 < min(u.L + u.nq, tok1) && tok1 > u.L) {
        __syncthreads();  // the blocks are complete in LDS
        const int i_lo = max(0, tok0 - u.L), i_hi = min(u.nq, tok1 - u.L);
        uint4* kdst = (uint4*)const_cast<void*>(p.Kc) + vec0 + (ptrdiff_t)ph * kPhase;
        uint4* vdst = (uint4*)const_cast<void*>(p.Vc) + vec0 + (ptrdiff_t)ph * kPhase;
        for (int c = tid; c < (i_hi - i_lo) * (D / 8); c += kThreads) {  // the new rows by 16-byte chunks
          const int i = i_lo + c / (D / 8), ck = c % (D / 8);
          const int t = u.L + i - tok0, h = t / kBlockTokens, tw = t % kBlockTokens;  // its token slot in the phase's blocks
          const size_t src = (((size_t)u.b * p.kmax + i) * p.Hkv + u.kvh) * D + 8 * ck;
          const uint4 kv = *(const uint4*)((const uint16_t*)p.Knew + src);
          const uint4 vv = *(const uint4*)((const uint16_t*)p.Vnew + src);
          const size_t ko = h * kBlkVec + k_elem_offset(D, tw, 8 * ck) / 8;  // in 16-byte chunks
          ring_k[slot][ko] = kv;
          kdst[ko] = kv;
          const uint32_t vw[4] = {vv.x, vv.y, vv.z, vv.w};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint16_t v = (uint16_t)(vw[e >> 1] >> (16 * (e & 1)));
            const size_t vo = h * kBlkVec * 8 + v_elem_offset(D, tw, 8 * ck + e);
            ((uint16_t*)&ring_v[slot][0])[vo] = v;
            ((uint16_t*)vdst)[vo] = v;
          }
        }
        __syncthreads();  // the patches are visible
      } else {
        __syncthreads();
      }
      if (active && H * ph + half < n) {
        KvRegs<D> r;
        const uint4* lk = &ring_k[slot][half * kBlkVec + lane];
        const uint4* lv = &ring_v[slot][half * kBlkVec + lane];
#pragma unroll
        for (int i = 0; i < 2 * (D / 32); ++i) r.k[i] = lk[i * 64];
#pragma unroll
        for (int i = 0; i < D / 16; ++i) r.v[i] = lv[i * 64];
        block_dispatch<D>(r, q.q, st, blk0 + H * ph + half, u.L, u.L + u.nq, q.lim, fabsf(p.scale_log2), lane, false, NewRows{}, nullptr, nullptr);
      }
    };
    __syncthreads();  // the previous unit's merge has left the ring
    Stage g[kTileAhead];
#pragma unroll
    for (int j = 0; j < kTileAhead; ++j) fetch(g[j], j);
    for (int ph = 0; H * ph < n; ph += kTileAhead) {  // workgroup-uniform trip count
#pragma unroll
      for (int j = 0; j < kTileAhead; ++j) phase(g[j], ph + j);
    }
    merge_halves<D, TW>(st, n, half, tile, active, lane, (f32x4*)&ring_k[0][0], other_m, other_l);
    if (half == 0 && active) store_partial_quads<D>(p, u, wg, st, col, grp, row0);
  }
}

// The same for INT8 caches, one block per phase: the wavefront that fetched a V chunk widens it to bf16 on its way into LDS, so that
// every code is widened once per block.
template <int D, bool kFused>
__global__ __launch_bounds__(256, 2) void verify_attn_tiles_i8(AttnParams p) {
  constexpr int kAhead = 4;                   // blocks a workgroup has in flight from memory
  constexpr int kCodeVec = 2 * D;             // uint4 of codes per block and tensor
  constexpr int kBlkVec = kCodeVec + 8;       // ... and its 32 scales
  constexpr int kChunks = D / 32;             // 64-lane chunks of codes per tensor
  constexpr int kMoves = 2 * kChunks / 4;     // chunks a wavefront moves per block: numbers wv, wv + 4, ... of K's, then V's
    __shared__ uint4 ring_k[2][kCodeVec];      // codes
  __shared__ uint4 ring_v[2][2 * kCodeVec];  // the codes as bf16, fragments as in a bf16 cache
  __shared__ __align__(16) float ring_s[2][2 * kBlockTokens];  // K scales, V scales of each block
  const int lane = threadIdx.x & 63, wv = uniform(threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int wg = blockIdx.x;
  const int row0 = 16 * wv;  // the query tile of this wavefront

  const ShareRecord* rec = p.records + wg;
  const int nseg = uniform(rec->nseg), overflow = uniform(rec->overflow);
  if (!record_matches(p, rec)) {
    report_mismatch(p, wg == 0 && threadIdx.x == 0);
    return;
  }

  const uint4* kc = (const uint4*)p.Kc;
  const uint4* vc = (const uint4*)p.Vc;
  struct Stage {
    u32x4 c[kMoves];
    float scale;
  };

  for (int si = 0; si < nseg; ++si) {
    const Segment seg = si == 0 ? load_segment(&rec->seg[0]) : later_segment(p, rec, overflow, si);
    const Unit u = unit_of(seg);
    const int n = seg.n;
    const bool active = row0 < u.nq * p.g;  // this wavefront owns a query tile of the unit
    QFragI8<D> q;
    load_queries_i8<D>(p, u, active, col, grp, q, row0);
    RowState<D> st;
    clear_state<D>(st);
    const int blk0 = seg.first;
    const ptrdiff_t vec0 = (((ptrdiff_t)u.b * p.Hkv + u.kvh) * p.nblk_cap + blk0) * kBlkVec;

    // all fetches unconditional (exact wait counts); a block past the end re-reads the stretch's first block
    auto block_at = [&](int s) { return vec0 + (s < n ? (ptrdiff_t)s * kBlkVec : 0); };
    auto fetch = [&](Stage& g, int ph) {
#pragma unroll
      for (int i = 0; i < kMoves; ++i) {
        const ptrdiff_t off = block_at(ph);
        const int c = wv + 4 * i;
        const uint4* src = (c < kChunks ? kc + off + c * 64 : vc + off + (c - kChunks) * 64) + lane;
        g.c[i] = __builtin_nontemporal_load((const u32x4*)src);
      }
      const ptrdiff_t at = block_at(ph);
      g.scale = ((const float*)((lane < kBlockTokens ? kc : vc) + at + kCodeVec))[lane % kBlockTokens];
    };
    auto phase = [&](Stage& g, int ph) {
      const int slot = ph & 1;
#pragma unroll
      for (int i = 0; i < kMoves; ++i) {
        const int c = wv + 4 * i;
        if (c < kChunks) {
          ring_k[slot][c * 64 + lane] = __builtin_bit_cast(uint4, g.c[i]);
        } else {
          const int m = c - kChunks;
          ring_v[slot][(2 * m) * 64 + lane] = codes_to_bf16(g.c[i][0], g.c[i][1]);
          ring_v[slot][(2 * m + 1) * 64 + lane] = codes_to_bf16(g.c[i][2], g.c[i][3]);
        }
      }
      if (wv == 0) ring_s[slot][lane] = g.scale;
      fetch(g, ph + kAhead);
      // Fused append: as in the bf16 kernel; the rows are quantized as the append kernel does (a row's D / 8 lanes agree
      // on its largest magnitude), codes and scales go into LDS and into the cache.
      const int tok0 = (blk0 + ph) * kBlockTokens, tok1 = (blk0 + min(ph + 1, n)) * kBlockTokens;
      if (kFused && u.nq > 0 && tok0 < min(u.L + u.nq, tok1) && tok1 > u.L) {
        __syncthreads();  // the blocks are complete in LDS
        const int i_lo = max(0, tok0 - u.L), n_ck = (min(u.nq, tok1 - u.L) - i_lo) * (D / 8);
        for (int c0 = 0; c0 < n_ck; c0 += 256) {  // the new rows of this block, 8 elements per lane
          const int c = min(c0 + (int)threadIdx.x, n_ck - 1);  // whole rows: a row's lanes stay together past the end too
          const int ck = threadIdx.x % (D / 8), i = i_lo + c / (D / 8);
          const int tw = u.L + i - tok0;  // its token slot in the block
          const size_t src = (((size_t)u.b * p.kmax + i) * p.Hkv + u.kvh) * D + 8 * ck;
          const uint4 kv = *(const uint4*)((const uint16_t*)p.Knew + src);
          const uint4 vv = *(const uint4*)((const uint16_t*)p.Vnew + src);
          float ka = amax8(kv), va = amax8(vv);
#pragma unroll
          for (int o = D / 16; o >= 1; o >>= 1) {
            ka = fmaxf(ka, __shfl_xor(ka, o));
            va = fmaxf(va, __shfl_xor(va, o));
          }
          const float kinv = ka > 0.f ? 127.0f / ka : 0.f;
          const float vinv = va > 0.f ? 127.0f / va : 0.f;
          if (c0 + (int)threadIdx.x < n_ck) {
            const uint2 kq = quantize8(kv, kinv), vq = quantize8(vv, vinv);
            uint8_t* kblk = (uint8_t*)((uint4*)const_cast<void*>(p.Kc) + vec0 + (ptrdiff_t)ph * kBlkVec);
            uint8_t* vblk = (uint8_t*)((uint4*)const_cast<void*>(p.Vc) + vec0 + (ptrdiff_t)ph * kBlkVec);
            const size_t ko = i8_k_offset(D, tw, 8 * ck);
            *(uint2*)((uint8_t*)&ring_k[slot][0] + ko) = kq;
            *(uint2*)(kblk + ko) = kq;
            const uint4 vb = codes_to_bf16(vq.x, vq.y);
            const uint32_t vw[4] = {vb.x, vb.y, vb.z, vb.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              ((uint16_t*)&ring_v[slot][0])[v_elem_offset(D, tw, 8 * ck + e)] = (uint16_t)(vw[e >> 1] >> (16 * (e & 1)));
              vblk[i8_v_offset(D, tw, 8 * ck + e)] = (uint8_t)((e < 4 ? vq.x : vq.y) >> (8 * (e & 3)));
            }
            if (ck == 0) {
              const float ks = ka / 127.0f, vs = va / 127.0f;
              ring_s[slot][tw] = ks;
              ring_s[slot][kBlockTokens + tw] = vs;
              ((float*)(kblk + kBlockTokens * D))[tw] = ks;
              ((float*)(vblk + kBlockTokens * D))[tw] = vs;
            }
          }
        }
        __syncthreads();  // the patches are visible
      } else {
        __syncthreads();
      }
      if (active && ph < n) {
        KvRegs<D> r;
        u32x4 k[kChunks];
        TokenScales sc;
#pragma unroll
        for (int i = 0; i < kChunks; ++i) k[i] = __builtin_bit_cast(u32x4, ring_k[slot][i * 64 + lane]);
#pragma unroll
        for (int i = 0; i < D / 16; ++i) r.v[i] = ring_v[slot][i * 64 + lane];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 ks = *(const f32x4*)&ring_s[slot][16 * h + 4 * grp];
          const f32x4 vs = *(const f32x4*)&ring_s[slot][kBlockTokens + 16 * h + 4 * grp];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            sc.k[4 * h + j] = ks[j];
            sc.v[4 * h + j] = vs[j];
          }
        }
        const I8Operands<D> i8{k, q.q, q.q_scale_log2, &sc};
        block_dispatch<D, true>(r, nullptr, st, blk0 + ph, u.L, u.L + u.nq, q.lim, p.scale_log2, lane, false, NewRows{}, nullptr,
                                   nullptr, &i8);
      }
    };
    __syncthreads();  // the previous unit's last step has left the ring
    Stage g[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) fetch(g[j], j);
    for (int ph = 0; ph < n; ph += kAhead) {  // workgroup-uniform trip count
#pragma unroll
      for (int j = 0; j < kAhead; ++j) phase(g[j], ph + j);
    }
    if (active) store_partial_quads<D>(p, u, wg, st, col, grp, row0);
  }
}

// ---------------------------------------------------------------------------------------
// Split-context reduction as a launch of its own, used with more than 32 query rows: a unit's partials are then tens of KiB per
// contributor, too much for the one workgroup that happens to arrive last, so they are spread over the whole chip.  A partial's
// accumulators lie as [head element / 4, rotated][row][4].  A wavefront takes 16 rows: of four quads (kParts = 1), or of one, lanes l, l + 16,
// l + 32 and l + 48 every fourth of its partials, so that up to sixteen are on their way at a time.  The latter with few units, which
// have many partials and leave the chip empty otherwise: attention and reduction, 48 rows of 128, 16 / 64 / 128 / 256 units, kParts = 1 -> 4: 27.4
// -> 23.2, 21.4 -> 21.2, 41.5 -> 43.3, 40.3 -> 45.7 us.
// ---------------------------------------------------------------------------------------
constexpr int kReduceSplitUnits = 64;

template <int D, int kParts>
__global__ __launch_bounds__(256) void reduce_wide(AttnParams p) {
  constexpr int kQuads = 4 / kParts, kSub = D / 4 / kQuads;  // quads of a wavefront, wavefronts per 16 rows
  const int lane = threadIdx.x & 63;
  const int tiles = (p.rows_max + 15) / 16;
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int per_unit = tiles * kSub;
  if (item >= (long)p.B * p.Hkv * per_unit) return;
  const int unit = (int)(item / per_unit), sub = (int)(item - (long)unit * per_unit);
  const int b = unit / p.Hkv, kvh = unit - b * p.Hkv;
  const int rows = uniform(p.seq_nq[b]) * p.g, owners = uniform(p.unit_owners[unit]);  // requested together with the record
  __builtin_amdgcn_sched_barrier(0);
  if (!record_matches(p, p.records)) return;  // reported by the attention launch
  const int row0 = 16 * (sub / kSub), row = row0 + lane % 16;
  const int quad = kQuads * (sub % kSub) + (kParts == 1 ? lane / 16 : 0), part = kParts == 1 ? 0 : lane / 16;
  const int i = row_token(p, row), hg = row - i * p.g;
  const size_t orow = ((size_t)b * p.kmax + i) * p.Hq + kvh * p.g + hg;
  const bool writes = part == 0 && row < p.rows_max;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  float lse = 0.f;
  if (row0 < rows) {  // wave-uniform; rows beyond draft_len (all of an inactive sequence) are zero in O and lse
    const int w_lo = owners & 0xFFFF, n = ((owners >> 16) & 0xFFFF) - w_lo + 1;
    const size_t slot0 = (size_t)w_lo + unit, stride = (size_t)p.rows_max * D;
    const int at = min(row, p.rows_max - 1);
    const float* acc = p.part_acc + slot0 * stride + 4 * at;
    const float2* ml = (const float2*)p.part_ml + slot0 * p.rows_max + at;
    float M = -INFINITY, L = 0.f;
    for (int j0 = 0; j0 < n; j0 += 4 * kParts) {  // partials that do not exist repeat the last one, with no weight
      float2 s[4];
      f32x4 a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j0 + kParts * j >= n) break;  // wave-uniform
        const int x = min(j0 + kParts * j + part, n - 1);
        s[j] = ml[(size_t)x * p.rows_max];
        a[j] = *(const f32x4*)(acc + x * stride + 4 * wide_quad<D>(quad, (int)slot0 + x) * p.rows_max);
      }
      const float M_old = M;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j0 + kParts * j < n) M = fmaxf(M, j0 + kParts * j + part < n ? s[j].x : -INFINITY);
      const float Mf = M == -INFINITY ? 0.f : M, alpha = __builtin_amdgcn_exp2f(M_old - Mf);
      L *= alpha;
      o *= alpha;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j0 + kParts * j < n) {
          const float wgt = j0 + kParts * j + part < n ? __builtin_amdgcn_exp2f(s[j].x - Mf) : 0.f;
          L = fmaf(s[j].y, wgt, L);
          if (wgt != 0.f) o += a[j] * wgt;
        }
    }
    // a valid row has a visible token (token 0) in the unit's first partial
    float top = M;
    if constexpr (kParts > 1) {
      top = rows4_max(M);
      const float wgt = __builtin_amdgcn_exp2f(M - (top == -INFINITY ? 0.f : top));
      L = rows4_sum(L * wgt);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = rows4_sum(wgt != 0.f ? o[e] * wgt : 0.f);
    }
    o *= __builtin_amdgcn_rcpf(L);
    lse = (top + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
  }
  if (!writes) return;
  if (row >= rows) {
    o = f32x4{0.f, 0.f, 0.f, 0.f};
    lse = 0.f;
  }
  *(f32x4*)(p.O + orow * D + 4 * quad) = o;
  if (p.lse && quad == 0) p.lse[orow] = lse;
}

// ---------------------------------------------------------------------------------------
// fp32 kernel: same schedule and partial format; the products run on the fp32 matrix instruction (16x16x4, fp32 operands and sums),
// probabilities stay fp32.  Cache is token-major [B][Hkv][Lcap][D].  What bounds the short lists it serves is the chain of
// dependent steps of one 32-token block: with a lane per token it was D / 4 strided loads per query row, twelve shuffles for each maximum
// and sum, and a walk over the tokens for P V.  As below the rows of a tile are done together:
//   S^T[16 tokens x 16 rows] += K Q^T: step (u, j) takes head element 16 u + 4 grp + j of both, so that operands are 16-byte loads,
//   O^T[16 head elements x 16 rows] += V^T P^T: step i takes tokens 4 grp + i, which is where the scores of that lane lie.
// New rows of a fused append are read where the model left them, and copied into the cache on the way.  2 sequences, 4 heads of 64, 37 and 90
// tokens: 24.8 -> 8.2 us.
// DT: the head has at most 16 DT elements; DC: its size where the merge is compiled for it, else 0.
// ---------------------------------------------------------------------------------------
__device__ inline void append_own_rows_fp32(const AttnParams& p, const Unit& u, int tok_lo, int tok_hi, int lane) {
  float* kc = (float*)const_cast<void*>(p.Kc);
  float* vc = (float*)const_cast<void*>(p.Vc);
  for (int t = max(u.L, tok_lo); t < tok_hi; ++t) {
    const size_t row = (((size_t)u.b * p.kmax + (t - u.L)) * p.Hkv + u.kvh) * p.D;
    const size_t dst = (((size_t)u.b * p.Hkv + u.kvh) * p.Lcap + t) * p.D;
    for (int d = 4 * lane; d < p.D; d += 256) {
      *(float4*)(kc + dst + d) = *(const float4*)((const float*)p.Knew + row + d);
      *(float4*)(vc + dst + d) = *(const float4*)((const float*)p.Vnew + row + d);
    }
  }
}

template <int DT, int DC>
__global__ __launch_bounds__(256) void verify_attn_fp32(AttnParams p) {
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  const int w = uniform(blockIdx.x * p.wpw + (threadIdx.x >> 6));
  const int D = DC > 0 ? DC : p.D;

  const ShareRecord* rec = p.records + w;
  Segment seg = load_segment(&rec->seg[0]);
  const int nseg = uniform(rec->nseg), overflow = uniform(rec->overflow), rec_flags = uniform(rec->flags);
  if (!record_matches(p, rec)) {
    report_mismatch(p, w == 0 && lane == 0);
    return;
  }

  for (int si = 0; si < nseg; ++si) {
    if (si > 0) seg = later_segment(p, rec, overflow, si);
    const Unit u = unit_of(seg);
    const int rows = u.nq * p.g;
    const int tok_lo = seg.first * kBlockTokens;
    const int tok_hi = min(u.L + u.nq, (seg.first + seg.n) * kBlockTokens);
    // tokens from `fresh` on are this step's own
    const int fresh = p.Knew ? u.L : 0x7FFFFFFF;
    const size_t cached = ((size_t)u.b * p.Hkv + u.kvh) * p.Lcap * D, given = ((size_t)u.b * p.kmax * p.Hkv + u.kvh) * D;
    auto token_row = [&](const void* cache, const void* now, int tok) {
      const int t = min(tok, tok_hi - 1);  // tokens past the end repeat the last one and are masked
      return t < fresh ? (const float*)cache + cached + (size_t)t * D : (const float*)now + given + (size_t)(t - u.L) * p.Hkv * D;
    };
    const size_t slot = (size_t)w + (size_t)u.b * p.Hkv + u.kvh;

    for (int r0 = 0; r0 < rows; r0 += 16) {
      const int rrow = r0 + col;
      const bool row_ok = rrow < rows;
      const int i = row_ok ? row_token(p, rrow) : 0, hg = row_ok ? rrow - i * p.g : 0;
      const float* qrow = (const float*)p.Q + (((size_t)u.b * p.kmax + i) * p.Hq + u.kvh * p.g + hg) * D;
      const int lim = min(u.L + i, tok_hi - 1);  // last token visible to the row
      f32x4 q[DT], acc[DT];
#pragma unroll
      for (int x = 0; x < DT; ++x) {
        const int d = 16 * x + 4 * grp;
        q[x] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (row_ok && d < D) q[x] = *(const f32x4*)(qrow + d);
        acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      float m = -INFINITY, l = 0.f;
#pragma unroll 1
      for (int t0 = tok_lo; t0 < tok_hi; t0 += 16) {
        f32x4 k[DT];
        float v[4][DT];
        const float* krow = token_row(p.Kc, p.Knew, t0 + col);
#pragma unroll
        for (int x = 0; x < DT; ++x) {
          const int d = 16 * x + 4 * grp;
          k[x] = *(const f32x4*)(krow + (d < D ? d : 0));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float* vrow = token_row(p.Vc, p.Vnew, t0 + 4 * grp + e);
#pragma unroll
          for (int x = 0; x < DT; ++x) {
            v[e][x] = vrow[16 * x + col < D ? 16 * x + col : 0];
            if (t0 + 4 * grp + e >= tok_hi) v[e][x] = 0.f;  // the last token again: it may be infinite
          }
        }
        f32x4 z[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};  // two chains
#pragma unroll
        for (int x = 0; x < DT; ++x)
#pragma unroll
          for (int j = 0; j < 4; ++j) z[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(16 * x + 4 * grp < D ? k[x][j] : 0.f, q[x][j], z[j & 1], 0, 0, 0);
        float s[4], mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[e] = t0 + 4 * grp + e <= lim ? (z[0][e] + z[1][e]) * p.scale_log2 : -INFINITY;
          mx = fmaxf(mx, s[e]);
        }
        const float m_new = fmaxf(m, rows4_max(mx)), m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = exp2f(m - m_use);
        l *= alpha;
        m = m_new;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[e] = exp2f(s[e] - m_use);
          l += s[e];
        }
#pragma unroll
        for (int x = 0; x < DT; ++x) {
          acc[x] *= alpha;
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e][x], s[e], acc[x], 0, 0, 0);
        }
      }
      const float sum = rows4_sum(l);
      if (row_ok) {
        const __amdgpu_buffer_rsrc_t rs = dev_buffer(p.part_acc + slot * p.rows_max * D, (unsigned)p.rows_max * D * 4);
#pragma unroll
        for (int x = 0; x < DT; ++x)
          if (16 * x + 4 * grp < D) store_dev4(rs, (unsigned)(rrow * D + 16 * x + 4 * grp) * 4, acc[x]);
        if (grp == 0) store_dev(p.part_ml + (slot * p.rows_max + rrow) * 2, m, sum);
      }
    }
    partial_stores_done();
    CombineJob job = job_of(seg);
    bool last, unused;
    arrive(p, lane, job, last, false, job, unused);
    if (last) combine_jobs<DC>(p, job, true, job, false, lane);
    // what nobody waits for
    if (seg.flags & kSegLast) zero_rows<DC>(p, u.b, u.kvh, rows, lane);
    if (p.Knew) append_own_rows_fp32(p, u, tok_lo, tok_hi, lane);
  }
  if (rec_flags & kRecAnyInactive) zero_unused_rows<DC, true>(p, w, p.nwaves, lane);
}

// Workspace = [unit counters, padded to 256 B][the plan of calls that bring none][partial outputs]
// [partial (max, sum) pairs], laid out for `shares` stretches.
struct Workspace {
  size_t plan, part_acc, part_ml, bytes;
};

static Workspace workspace_layout(const bass_attn_desc* d, int shares) {
  Workspace w;
  const size_t slots = (size_t)shares + (size_t)d->B * d->Hkv;
  const size_t rows = (size_t)d->kmax * (d->Hq / d->Hkv);
  w.plan = (((size_t)d->B * d->Hkv * sizeof(int32_t)) + 255) & ~(size_t)255;
  w.part_acc = w.plan + plan_layout(d->B, d->Hkv, shares).bytes;
  w.part_ml = w.part_acc + slots * rows * (size_t)d->D * sizeof(float);
  w.bytes = w.part_ml + slots * rows * 2 * sizeof(float);
  return w;
}

PlanShape plan_shape(const bass_attn_desc* d, const LaunchShape& ls, int span);
int launch_plan(const bass_attn_desc* d, const LaunchShape& ls, int span, const int32_t* ctx_len, const int32_t* draft_len,
                void* plan, int32_t* dev_status, void* stream, int32_t* clear_counters);
// bass_kv_append for a planned launch; writes nothing if the word at `signature` is not `expected`  (kv_cache.hip)
int append_planned(const bass_attn_desc* d, void* Kcache, void* Vcache, const void* K_new, const void* V_new, const int32_t* L,
                   const int32_t* nq, const int32_t* signature, int32_t expected, int32_t* dev_status, void* stream);

}  // namespace bass

extern "C" int bass_set_attention_waves(int waves) {
  bass::g_attention_waves.store(waves > 0 ? waves : 0, std::memory_order_relaxed);
  return bass::attention_waves(bass::attention_waves_setting());
}

extern "C" size_t bass_verify_attention_workspace_bytes(const bass_attn_desc* d) {
  if (bass::check_desc(d) != BASS_OK) return 0;
  return bass::workspace_layout(d, bass::kMaxWaves).bytes;
}

namespace bass {

static int check_attention_args(const bass_attn_desc* d, const LaunchShape& ls, const void* Q, const void* K_new,
                                const void* V_new, const void* Kcache, const void* Vcache, const float* O,
                                const void* workspace) {
  if (!Q || !Kcache || !Vcache || !O || !workspace) return BASS_ERR_INVALID_ARG;
  if ((K_new == nullptr) != (V_new == nullptr)) return BASS_ERR_INVALID_ARG;
  if (((uintptr_t)workspace & 15) != 0) return BASS_ERR_INVALID_ARG;
  if (ls.mfma && ls.rows_max > 64) return BASS_ERR_UNSUPPORTED;
  // partials of one unit are addressed with 32-bit byte offsets
  if ((int64_t)ls.rows_max * d->D * 4 * kMaxWaves >= (1ll << 31)) return BASS_ERR_UNSUPPORTED;
  return BASS_OK;
}

// The workgroup-level kernels.
template <int D, bool kI8>
static void launch_wide(dim3 grid, hipStream_t s, const AttnParams& p) {
  const dim3 block(64 * kWideWaves);
  if (p.rows_max > 32) hipLaunchKernelGGL((verify_attn_wide<D, kI8, 2>), grid, block, 0, s, p);
  else if (p.rows_max > 16) hipLaunchKernelGGL((verify_attn_wide<D, kI8, 1>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((verify_attn_wide<D, kI8, 0>), grid, block, 0, s, p);
}

template <bool kFused>
static void launch_tiles(const bass_attn_desc* d, dim3 grid, hipStream_t s, const AttnParams& p) {
  const bool big = d->D == 128;
  if (d->dtype == BASS_DTYPE_INT8KV) {
    if (big) hipLaunchKernelGGL((verify_attn_tiles_i8<128, kFused>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((verify_attn_tiles_i8<64, kFused>), grid, dim3(256), 0, s, p);
  } else {
    if (big) hipLaunchKernelGGL((verify_attn_tiles_bf16<128, kFused>), grid, dim3(512), 0, s, p);
    else hipLaunchKernelGGL((verify_attn_tiles_bf16<64, kFused>), grid, dim3(512), 0, s, p);
  }
}

// The attention launch (and, with many query rows per kv head, the merge launch) for a plan that lies at
// `plan`, made for the shape `ls`; K_new / V_new: the rows a fused append puts into the caches, or null.
static int launch_attention(const bass_attn_desc* d, const LaunchShape& ls, const void* Q, const void* K_new,
                            const void* V_new, const void* Kcache, const void* Vcache, const void* plan, float* O,
                            float* lse, const Workspace& wl, void* workspace, int32_t* dev_status, void* stream) {
  const int g = d->Hq / d->Hkv;
  const int rows_max = ls.rows_max;
  AttnParams p;
  p.B = d->B; p.kmax = d->kmax; p.Hq = d->Hq; p.Hkv = d->Hkv; p.D = d->D; p.Lcap = d->Lcap;
  p.nblk_cap = num_blocks(d->Lcap); p.g = g; p.rows_max = rows_max;
  p.g_magic = (g <= 64 && rows_max <= 2048) ? ((1u << 20) + (unsigned)g - 1u) / (unsigned)g : 0u;  // exact there: checked exhaustively
  p.nwaves = ls.nwaves;
  p.scale_log2 = d->scale * 1.4426950408889634f;
  p.Q = Q; p.Kc = Kcache; p.Vc = Vcache; p.Knew = K_new; p.Vnew = V_new;
  const PlanLayout pl = plan_layout(d->B, d->Hkv, ls.nshares);
  const char* pb = (const char*)plan;
  p.signature = plan_signature(plan_shape(d, ls, 0), K_new && ls.fused_append ? kPlanAppend : 0);
  p.records = (const ShareRecord*)(pb + pl.records);
  p.overflow = (const Segment*)(pb + pl.overflow);
  p.seq_L = (const int32_t*)(pb + pl.seq_L);
  p.seq_nq = (const int32_t*)(pb + pl.seq_nq);
  p.unit_owners = (const int32_t*)(pb + pl.unit_owners);
  p.O = O; p.lse = lse; p.status = dev_status;
  p.counters = (int32_t*)workspace;
  p.part_acc = (float*)((char*)workspace + wl.part_acc);
  p.part_ml = (float*)((char*)workspace + wl.part_ml);

  hipStream_t s = (hipStream_t)stream;
  p.wpw = waves_per_workgroup(p.nwaves);
  const dim3 grid(p.nwaves / p.wpw), block(64 * p.wpw);
  if (d->dtype == BASS_DTYPE_FP32) {
    if (d->D == 32) hipLaunchKernelGGL((verify_attn_fp32<2, 32>), grid, block, 0, s, p);
    else if (d->D == 64) hipLaunchKernelGGL((verify_attn_fp32<4, 64>), grid, block, 0, s, p);
    else if (d->D == 128) hipLaunchKernelGGL((verify_attn_fp32<8, 128>), grid, block, 0, s, p);
    else if (d->D <= 128) hipLaunchKernelGGL((verify_attn_fp32<8, 0>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((verify_attn_fp32<16, 0>), grid, block, 0, s, p);
  } else if (ls.wide) {
    const dim3 wgrid((unsigned)ls.used_shares);
    if (d->dtype == BASS_DTYPE_INT8KV) {
      if (d->D == 128) launch_wide<128, true>(wgrid, s, p);
      else launch_wide<64, true>(wgrid, s, p);
    } else {
      if (d->D == 128) launch_wide<128, false>(wgrid, s, p);
      else launch_wide<64, false>(wgrid, s, p);
    }
  } else if (ls.tiles) {
    const dim3 tgrid((unsigned)ls.used_shares);
    if (K_new) launch_tiles<true>(d, tgrid, s, p);
    else launch_tiles<false>(d, tgrid, s, p);
  } else {  // one query tile
    // LDS slice per wavefront of a fused append: K and V rows of two units (bf16, or INT8 codes + scales)
    const size_t unit_lds = d->dtype == BASS_DTYPE_INT8KV ? (size_t)2 * d->kmax * d->D + 8 * d->kmax
                                                          : (size_t)2 * d->kmax * d->D * 2;
    const size_t lds = K_new ? (size_t)p.wpw * 2 * unit_lds : 0;
    if (d->dtype == BASS_DTYPE_INT8KV) {
      if (d->D == 128) hipLaunchKernelGGL((verify_attn_bf16<128, true>), grid, block, lds, s, p);
      else hipLaunchKernelGGL((verify_attn_bf16<64, true>), grid, block, lds, s, p);
    } else {
      if (d->D == 128) hipLaunchKernelGGL((verify_attn_bf16<128, false>), grid, block, lds, s, p);
      else hipLaunchKernelGGL((verify_attn_bf16<64, false>), grid, block, lds, s, p);
    }
  }
  if (launch_status() != BASS_OK) return BASS_ERR_HIP;
  if (ls.tiles && rows_max > 32) {
    const bool split = d->B * d->Hkv <= kReduceSplitUnits;
    const long items = (long)d->B * d->Hkv * ((rows_max + 15) / 16) * (d->D / (split ? 4 : 16));
    const dim3 rgrid((unsigned)((items + 3) / 4)), rblock(256);
    if (d->D == 128 && split) hipLaunchKernelGGL((reduce_wide<128, 4>), rgrid, rblock, 0, s, p);
    else if (d->D == 128) hipLaunchKernelGGL((reduce_wide<128, 1>), rgrid, rblock, 0, s, p);
    else if (split) hipLaunchKernelGGL((reduce_wide<64, 4>), rgrid, rblock, 0, s, p);
    else hipLaunchKernelGGL((reduce_wide<64, 1>), rgrid, rblock, 0, s, p);
  }
  return launch_status();
}

// Plan (into the workspace) and attention in one call.
static int plan_and_launch(const bass_attn_desc* d, const void* Q, const void* K_new, const void* V_new,
                           const void* Kcache, const void* Vcache, const int32_t* ctx_len, const int32_t* draft_len,
                           float* O, float* lse, void* workspace, size_t workspace_bytes, int32_t* dev_status,
                           void* stream, int span = 0) {
  int rc = check_desc(d);
  if (rc != BASS_OK) return rc;
  if (!ctx_len || !draft_len) return BASS_ERR_INVALID_ARG;
  const LaunchShape ls = launch_shape(d, K_new != nullptr);
  rc = check_attention_args(d, ls, Q, K_new, V_new, Kcache, Vcache, O, workspace);
  if (rc != BASS_OK) return rc;
  const Workspace wl = workspace_layout(d, kMaxWaves);
  if (workspace_bytes < wl.bytes) return BASS_ERR_WORKSPACE_TOO_SMALL;
  void* plan = (char*)workspace + wl.plan;
  rc = launch_plan(d, ls, span, ctx_len, draft_len, plan, dev_status, stream, nullptr);
  if (rc != BASS_OK) return rc;
  return launch_attention(d, ls, Q, K_new, V_new, Kcache, Vcache, plan, O, lse, wl, workspace, dev_status, stream);
}

}  // namespace bass

extern "C" int bass_verify_attention(const bass_attn_desc* d, const void* Q, const void* Kcache, const void* Vcache,
                                     const int32_t* ctx_len, const int32_t* draft_len, float* O, float* lse,
                                     void* workspace, size_t workspace_bytes, int32_t* dev_status, void* stream) {
  return bass::plan_and_launch(d, Q, nullptr, nullptr, Kcache, Vcache, ctx_len, draft_len, O, lse, workspace,
                               workspace_bytes, dev_status, stream);
}

extern "C" int bass_verify_attention_pad(const bass_attn_desc* d, const void* Q, const void* Kcache,
                                         const void* Vcache, const int32_t* ctx_len, const int32_t* draft_len,
                                         int32_t padded_len, float* O, float* lse, void* workspace,
                                         size_t workspace_bytes, int32_t* dev_status, void* stream) {
  if (padded_len < 0) return BASS_ERR_INVALID_ARG;
  return bass::plan_and_launch(d, Q, nullptr, nullptr, Kcache, Vcache, ctx_len, draft_len, O, lse, workspace,
                               workspace_bytes, dev_status, stream, padded_len);
}

extern "C" int bass_verify_attention_split(const bass_attn_desc* d, const void* Q, const void* Kcache,
                                           const void* Vcache, const int32_t* ctx_len, const int32_t* draft_len,
                                           float* O, float* lse, void* workspace, size_t workspace_bytes,
                                           int32_t* dev_status, void* stream) {
  const int rc = bass::check_desc(d);
  if (rc != BASS_OK) return rc;
  if (!Q || !Kcache || !Vcache || !ctx_len || !draft_len || !O || !workspace) return BASS_ERR_INVALID_ARG;
  if (workspace_bytes < bass::workspace_layout(d, bass::kMaxWaves).bytes) return BASS_ERR_WORKSPACE_TOO_SMALL;
  bass_attn_desc one = *d;
  one.B = 1;
  const size_t elt = d->dtype == BASS_DTYPE_FP32 ? 4 : 2;  // Q is bf16 with bf16 and with INT8 caches
  const size_t q_seq = (size_t)d->kmax * d->Hq * d->D;  // elements of Q (and O) per sequence
  const size_t cache_seq = bass_kv_cache_bytes(&one);
  for (int b = 0; b < d->B; ++b) {  // one plan and one launch per sequence; they share the workspace in stream order
    const int r = bass::plan_and_launch(&one, (const char*)Q + b * q_seq * elt, nullptr, nullptr,
                                        (const char*)Kcache + b * cache_seq, (const char*)Vcache + b * cache_seq,
                                        ctx_len + b, draft_len + b, O + b * q_seq,
                                        lse ? lse + (size_t)b * d->kmax * d->Hq : nullptr, workspace, workspace_bytes,
                                        dev_status, stream);
    if (r != BASS_OK) return r;
  }
  return BASS_OK;
}

extern "C" int bass_append_verify_attention(const bass_attn_desc* d, const void* Q, const void* K_new,
                                            const void* V_new, void* Kcache, void* Vcache, const int32_t* ctx_len,
                                            const int32_t* draft_len, float* O, float* lse, void* workspace,
                                            size_t workspace_bytes, int32_t* dev_status, void* stream) {
  if (!K_new || !V_new) return BASS_ERR_INVALID_ARG;
  if (d && d->dtype != BASS_DTYPE_FP32 && (int64_t)d->kmax * d->D > bass::kMaxStagedElems) {
    // more new rows than a wavefront stages in LDS: append with a launch of its own (the workgroup-level kernels could
    // take them, as planned launches do; this way is what those are tested against)
    const int rc = bass_kv_append(d, Kcache, Vcache, K_new, V_new, ctx_len, draft_len, dev_status, stream);
    if (rc != BASS_OK) return rc;
    return bass::plan_and_launch(d, Q, nullptr, nullptr, Kcache, Vcache, ctx_len, draft_len, O, lse, workspace,
                                 workspace_bytes, dev_status, stream);
  }
  return bass::plan_and_launch(d, Q, K_new, V_new, Kcache, Vcache, ctx_len, draft_len, O, lse, workspace,
                               workspace_bytes, dev_status, stream);
}

// A verification step's attention with a plan made once for all of its layers (bass_attention_plan).
extern "C" int bass_verify_attention_planned(const bass_attn_desc* d, const void* Q, const void* K_new, const void* V_new,
                                             void* Kcache, void* Vcache, const void* plan, float* O, float* lse,
                                             void* workspace, size_t workspace_bytes, int32_t* dev_status,
                                             void* stream) {
  int rc = bass::check_desc(d);
  if (rc != BASS_OK) return rc;
  if (!plan || ((uintptr_t)plan & 15) != 0) return BASS_ERR_INVALID_ARG;
  const bass::LaunchShape ls = bass::launch_shape(d, K_new != nullptr);
  rc = bass::check_attention_args(d, ls, Q, K_new, V_new, Kcache, Vcache, O, workspace);
  if (rc != BASS_OK) return rc;
  const bass::Workspace wl = bass::workspace_layout(d, bass::kMaxWaves);
  if (workspace_bytes < wl.bytes) return BASS_ERR_WORKSPACE_TOO_SMALL;
  if (K_new && !ls.fused_append && !ls.tiles_append) {  // a launch of its own, at the (clamped) lengths the plan holds
    const bass::PlanLayout pl = bass::plan_layout(d->B, d->Hkv, ls.nshares);
    const char* at = (const char*)plan;
    rc = bass::append_planned(d, Kcache, Vcache, K_new, V_new, (const int32_t*)(at + pl.seq_L), (const int32_t*)(at + pl.seq_nq),
                              &((const bass::ShareRecord*)(at + pl.records))->signature,
                              bass::plan_signature(bass::plan_shape(d, ls, 0), 0), dev_status, stream);
    if (rc != BASS_OK) return rc;
    return bass::launch_attention(d, ls, Q, nullptr, nullptr, Kcache, Vcache, plan, O, lse, wl, workspace, dev_status,
                                  stream);
  }
  return bass::launch_attention(d, ls, Q, K_new, V_new, Kcache, Vcache, plan, O, lse, wl, workspace, dev_status, stream);
}

// ---------------------------------------------------------------------------------------
// bass_verify_attention_noalloc: for callers that cannot allocate or own a workspace.  The arrival
// counters, the plan and the partial results live in a file-scope device array.  In host code the array's
// name is only a stand-in: its device address is asked for once per device (hipGetSymbolAddress, with that
// device current) and that pointer, never the name, is what launches receive.
// ---------------------------------------------------------------------------------------
constexpr size_t kScratchBytes = BASS_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace bass {

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];  // per device: each GPU holds its own copy of the array
static std::mutex g_scratch_mutex;

static int scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BASS_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return BASS_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return BASS_OK;
}

}  // namespace bass

extern "C" int bass_verify_attention_noalloc(const bass_attn_desc* d, const void* Q, const void* Kcache,
                                             const void* Vcache, const int32_t* ctx_len, const int32_t* draft_len,
                                             float* O, float* lse, int32_t* dev_status, void* stream) {
  int rc = bass::check_desc(d);
  if (rc != BASS_OK) return rc;
  if (!ctx_len || !draft_len) return BASS_ERR_INVALID_ARG;
  const bass::LaunchShape ls = bass::launch_shape(d, false);
  // laid out for the shares this launch really uses, not for the largest spread the tuning knob allows
  const bass::Workspace wl = bass::workspace_layout(d, ls.nshares);
  if (wl.bytes > kScratchBytes) return BASS_ERR_WORKSPACE_TOO_SMALL;
  void* ptr = nullptr;
  rc = bass::scratch_address(&ptr);
  if (rc != BASS_OK) return rc;
  rc = bass::check_attention_args(d, ls, Q, nullptr, nullptr, Kcache, Vcache, O, ptr);
  if (rc != BASS_OK) return rc;
  void* plan = (char*)ptr + wl.plan;
  // the array keeps the last call's contents: the planning launch also clears the arrival counters
  rc = bass::launch_plan(d, ls, 0, ctx_len, draft_len, plan, dev_status, stream, (int32_t*)ptr);
  if (rc != BASS_OK) return rc;
  return bass::launch_attention(d, ls, Q, nullptr, nullptr, Kcache, Vcache, plan, O, lse, wl, ptr, dev_status, stream);
}
