// Planning of a verification step's attention launches: bass_attention_plan (one small launch),
// bass_attention_plan_host (the same arithmetic on the host), bass_attention_plan_bytes.
//
// BASS paper, Section 3.2: every sequence of the batch has its own length and proceeds at its own pace;
// the lengths are the same for all attention layers of a verification step.  The division of the ragged
// work over the wavefronts of the attention launch (attn_plan.h) is therefore computed once per step, here,
// and each layer's launch reads its share from a record instead of recomputing it.
#include <cstring>

#include "bass_common.h"

namespace bass {

// Planning kernel.  Phase 0, where it is asked for: whether every unit gets stretches of its own.  Phase 1: clamp the lengths,
// count blocks, inclusive prefix over the sequences.  Phase 2: one
// thread per share walks its stretch of the block list and writes the record.  Phase 3: the contributors of
// every unit, for the merge launch.  Batches of up to kPlanSeqs sequences keep phase 1's results in LDS, every
// workgroup computes them for itself (a few hundred instructions) and the shares are spread over several
// workgroups, i.e. compute units: the walk is serial integer arithmetic with divisions, and one compute unit
// needs 10 us for 768 shares.  Larger batches are planned by a single workgroup through global memory.
constexpr int kPlanThreads = 256;
constexpr int kPlanSeqs = 1024;

// Inclusive prefix sum over the workgroup's kPlanThreads values and their total; all threads call.
__device__ inline int block_incl_scan(int v, int* lds, int tid, int& total) {
  const int lane = tid & 63, wv = tid >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(x, o);
    if (lane >= o) x += t;
  }
  if (lane == 63) lds[wv] = x;
  __syncthreads();
  int base = 0;
  total = 0;
  for (int i = 0; i < kPlanThreads / 64; ++i) {
    const int t = lds[i];
    if (i < wv) base += t;
    total += t;
  }
  __syncthreads();  // lds may be written again
  return x + base;
}

// Writes the segments of share w: the first two into its record, the others into the overflow list from entry
// w + (unit of the third segment) on.  These runs cannot overlap: the units of a share are distinct and
// increasing, and the next share starts at a unit that is not smaller than this share's last one.
struct RecordWriter {
  ShareRecord* rec;
  Segment* overflow;
  int w, Hkv, n, base;
  BASS_HD void operator()(const Segment& g) {
    if (n < 2) {
      rec->seg[n] = g;
    } else {
      if (n == 2) base = w + g.b * Hkv + g.kvh;
      overflow[base + n - 2] = g;
    }
    ++n;
  }
};

BASS_HD inline void clear_record(ShareRecord* r) {
  int32_t* w = (int32_t*)r;
  for (size_t i = 0; i < sizeof(ShareRecord) / 4; ++i) w[i] = 0;
}

BASS_HD inline void write_record(const PlanShape& s, const int32_t* seq_L, const int32_t* seq_nq, const int32_t* inc, int total,
                                 int w, int32_t signature, bool any_inactive, ShareRecord* records, Segment* overflow) {
  clear_record(&records[w]);
  RecordWriter wr{&records[w], overflow, w, s.Hkv, 0, 0};
  if (total > 0) plan_share(s, seq_L, seq_nq, inc, w, wr);
  records[w].nseg = wr.n;
  records[w].overflow = wr.base;
  records[w].signature = signature;
  records[w].flags = any_inactive ? kRecAnyInactive : 0;
}

BASS_HD inline int32_t owners_of_unit(const PlanShape& s, const Split& sp, int pb, const int32_t* seq_L, const int32_t* seq_nq,
                                      const int32_t* inc, int unit) {
  const int b = unit / s.Hkv, kvh = unit - b * s.Hkv;
  const int npad = inc[b] - (b > 0 ? inc[b - 1] : 0);
  const int nblk = s.whole > 0 ? seq_blocks(s, seq_L[b], seq_nq[b]) : npad - s.pad;
  return npad > 0 ? unit_owners(sp, (inc[b] - npad) * s.Hkv + kvh * npad, nblk, pb) : 0;
}

BASS_HD inline PlanHeader make_header(const PlanShape& s, int flags, int total, bool any_inactive, bool any_clamped) {
  PlanHeader h;
  h.magic = kPlanMagic;
  h.B = s.B; h.kmax = s.kmax; h.Hkv = s.Hkv; h.Lcap = s.Lcap;
  h.nshares = s.nshares; h.pad = s.pad; h.pad_before = s.pad_before; h.span = s.span;
  h.flags = flags;
  h.total = total;
  h.any_inactive = any_inactive ? 1 : 0;
  h.any_clamped = any_clamped ? 1 : 0;
  h.reserved[0] = h.reserved[1] = h.reserved[2] = 0;
  return h;
}

// clear_counters (optional): the arrival counters of the attention launch that follows, B * Hkv words,
// cleared here for callers whose workspace is not known to be clean.
// kWhole: real blocks of the stretches of whole units that the launch asks for (PlanShape::whole), or 0.  Phase 0 takes 0.6 - 1.2 us of a
// launch of 7 - 8 (16 sequences); with LDS atomics in place of the wave sums, which go lane by lane, 2 us.
template <int kWhole>
__global__ __launch_bounds__(kPlanThreads) void attention_plan_kernel(PlanShape asked, int flags, const int32_t* ctx_len,
                                                                      const int32_t* draft_len, char* plan, int32_t* status,
                                                                      int32_t* clear_counters) {
  PlanShape s = asked;
  s.whole = kWhole;
  __shared__ int lds[kPlanThreads / 64];
  __shared__ uint64_t sums[2][kPlanThreads / 64];
  __shared__ int32_t lds_L[kPlanSeqs], lds_nq[kPlanSeqs], lds_inc[kPlanSeqs];
  const int tid = threadIdx.x;
  const int gtid = blockIdx.x * kPlanThreads + tid, gthreads = gridDim.x * kPlanThreads;
  const bool first = blockIdx.x == 0;
  const bool in_lds = s.B <= kPlanSeqs;  // else: one workgroup (the host launches it so), results through global memory
  const PlanLayout lay = plan_layout(s.B, s.Hkv, s.nshares);
  int32_t* seq_L = (int32_t*)(plan + lay.seq_L);
  int32_t* seq_nq = (int32_t*)(plan + lay.seq_nq);
  int32_t* inc = (int32_t*)(plan + lay.seq_inc);
  ShareRecord* records = (ShareRecord*)(plan + lay.records);
  Segment* overflow = (Segment*)(plan + lay.overflow);
  int32_t* owners = (int32_t*)(plan + lay.unit_owners);

  if (clear_counters)
    for (int i = gtid; i < s.B * s.Hkv; i += gthreads) clear_counters[i] = 0;

  // the lengths of sequence b (every workgroup for itself; the first one also writes the plan's copy)
  bool bad = false, inactive = false;
  auto read_lengths = [&](int b, int& L, int& nq) {
    L = ctx_len[b];
    nq = draft_len[b];
    bad |= clamp_lengths(L, nq, s.kmax, s.Lcap);
    inactive |= nq == 0;
    if (first) {
      seq_L[b] = L;
      seq_nq[b] = nq;
    }
    if (in_lds) {
      lds_L[b] = L;
      lds_nq[b] = nq;
    }
  };

  // phase 0: whether every unit gets stretches of its own
  int entries = 0;
  if constexpr (kWhole > 0) {
    uint64_t mine = 0, mine_twice = 0;  // entries with their pads, stretches of kWhole blocks above
    for (int b = tid; b < s.B; b += kPlanThreads) {
      int L, nq;
      read_lengths(b, L, nq);
      const int nblk = seq_blocks(s, L, nq);
      mine += (uint64_t)padded_blocks(s.pad, nblk) | (uint64_t)stretches_of(kWhole, nblk) << 32;
      mine_twice += stretches_of(2 * kWhole, nblk);
    }
    mine = wave_sum_u64(mine);
    mine_twice = wave_sum_u64(mine_twice);
    if (tid % 64 == 0) {
      sums[0][tid / 64] = mine;
      sums[1][tid / 64] = mine_twice;
    }
    __syncthreads();
    uint64_t all = 0, twice = 0;
    for (int i = 0; i < kPlanThreads / 64; ++i) {
      all += sums[0][i];
      twice += sums[1][i];
    }
    entries = __builtin_amdgcn_readfirstlane((int)(uint32_t)all) * s.Hkv;
    const int once = __builtin_amdgcn_readfirstlane((int)(all >> 32));
    s = settle_whole(s, entries, (int64_t)once * s.Hkv, (int64_t)__builtin_amdgcn_readfirstlane((int)twice) * s.Hkv);
  }

  // phase 1
  int carry = 0;
  for (int c0 = 0; c0 < s.B; c0 += kPlanThreads) {
    const int b = c0 + tid;
    int nb = 0;
    if (b < s.B) {
      int L, nq;
      if constexpr (kWhole > 0) {  // what this thread wrote
        L = in_lds ? lds_L[b] : seq_L[b];
        nq = in_lds ? lds_nq[b] : seq_nq[b];
        const int nblk = seq_blocks(s, L, nq);
        nb = s.whole == 0 ? padded_blocks(s.pad, nblk)
             : s.whole == kWhole ? stretches_of(kWhole, nblk) * kWhole : stretches_of(2 * kWhole, nblk) * 2 * kWhole;
      } else {
        read_lengths(b, L, nq);
        nb = padded_blocks(s.pad, seq_blocks(s, L, nq));
      }
    }
    int chunk_total;
    const int incl = carry + block_incl_scan(nb, lds, tid, chunk_total);
    if (b < s.B) {
      if (first) inc[b] = incl;
      if (in_lds) lds_inc[b] = incl;
    }
    carry += chunk_total;
  }
  const int any_bad = __syncthreads_or(bad ? 1 : 0);
  const int any_inactive = __syncthreads_or(inactive ? 1 : 0);  // also orders the writes above before the reads below
  const int total = carry * s.Hkv;
  if (first && tid == 0) {
    *(PlanHeader*)plan = make_header(s, flags, kWhole > 0 ? entries : total, any_inactive != 0, any_bad != 0);
    if (any_bad && status) atomicOr(status, BASS_STATUS_LEN_CLAMPED);
  }
  const int32_t* rd_L = in_lds ? lds_L : seq_L;
  const int32_t* rd_nq = in_lds ? lds_nq : seq_nq;
  const int32_t* rd_inc = in_lds ? lds_inc : inc;

  // phase 2
  const int32_t signature = plan_signature(asked, flags);
  for (int w = gtid; w < s.nshares; w += gthreads)
    write_record(s, rd_L, rd_nq, rd_inc, total, w, signature, any_inactive != 0, records, overflow);

  // phase 3
  const Split sp = plan_split(s, total);
  const int pb = pad_before_in_effect(s, sp);
  for (int unit = gtid; unit < s.B * s.Hkv; unit += gthreads)
    owners[unit] = total > 0 ? owners_of_unit(s, sp, pb, rd_L, rd_nq, rd_inc, unit) : 0;
}

// The same plan, byte for byte, written by the host into host memory.
static bool plan_on_host(const PlanShape& asked, int flags, const int32_t* ctx_len, const int32_t* draft_len, char* plan) {
  PlanShape s = asked;
  const PlanLayout lay = plan_layout(s.B, s.Hkv, s.nshares);
  int32_t* seq_L = (int32_t*)(plan + lay.seq_L);
  int32_t* seq_nq = (int32_t*)(plan + lay.seq_nq);
  int32_t* inc = (int32_t*)(plan + lay.seq_inc);
  ShareRecord* records = (ShareRecord*)(plan + lay.records);
  Segment* overflow = (Segment*)(plan + lay.overflow);
  int32_t* owners = (int32_t*)(plan + lay.unit_owners);
  bool bad = false, any_inactive = false;
  int entries = 0, carry = 0;
  int64_t once = 0, twice = 0;
  for (int b = 0; b < s.B; ++b) {
    int L = ctx_len[b], nq = draft_len[b];
    bad |= clamp_lengths(L, nq, s.kmax, s.Lcap);
    any_inactive |= nq == 0;
    seq_L[b] = L;
    seq_nq[b] = nq;
    entries += padded_blocks(s.pad, seq_blocks(s, L, nq));
    once += stretches_of(imax(s.whole, 1), seq_blocks(s, L, nq));
    twice += stretches_of(imax(2 * s.whole, 1), seq_blocks(s, L, nq));
  }
  entries *= s.Hkv;
  s = settle_whole(s, entries, once * s.Hkv, twice * s.Hkv);
  for (int b = 0; b < s.B; ++b) {
    carry += unit_entries(s, seq_blocks(s, seq_L[b], seq_nq[b]));
    inc[b] = carry;
  }
  const int total = carry * s.Hkv;
  *(PlanHeader*)plan = make_header(s, flags, entries, any_inactive, bad);
  const int32_t signature = plan_signature(asked, flags);
  for (int w = 0; w < s.nshares; ++w) write_record(s, seq_L, seq_nq, inc, total, w, signature, any_inactive, records, overflow);
  const Split sp = plan_split(s, total);
  const int pb = pad_before_in_effect(s, sp);
  for (int unit = 0; unit < s.B * s.Hkv; ++unit)
    owners[unit] = total > 0 ? owners_of_unit(s, sp, pb, seq_L, seq_nq, inc, unit) : 0;
  return bad;
}

PlanShape plan_shape(const bass_attn_desc* d, const LaunchShape& ls, int span) {
  PlanShape s;
  s.B = d->B; s.kmax = d->kmax; s.Hkv = d->Hkv; s.Lcap = d->Lcap;
  s.nshares = ls.nshares; s.target = ls.target; s.pad = ls.pad; s.pad_before = ls.pad_before; s.span = span;
  s.min_entries = ls.min_entries; s.used = ls.used_shares; s.whole = ls.whole; s.grow = ls.grow;
  return s;
}

size_t plan_bytes_max(const bass_attn_desc* d) { return plan_layout(d->B, d->Hkv, kMaxWaves).bytes; }

int launch_plan(const bass_attn_desc* d, const LaunchShape& ls, int span, const int32_t* ctx_len, const int32_t* draft_len,
                void* plan, int32_t* dev_status, void* stream, int32_t* clear_counters) {
  const PlanShape s = plan_shape(d, ls, span);
  const unsigned groups = s.B <= kPlanSeqs ? (unsigned)((s.nshares + kPlanThreads - 1) / kPlanThreads) : 1u;
  const dim3 grid(groups), block(kPlanThreads);
  const int flags = ls.fused_append ? kPlanAppend : 0;
  hipStream_t st = (hipStream_t)stream;
  if (s.whole == kWidePerStep) hipLaunchKernelGGL(attention_plan_kernel<kWidePerStep>, grid, block, 0, st, s, flags, ctx_len, draft_len, (char*)plan, dev_status, clear_counters);
  else hipLaunchKernelGGL(attention_plan_kernel<0>, grid, block, 0, st, s, flags, ctx_len, draft_len, (char*)plan, dev_status, clear_counters);
  return launch_status();
}

}  // namespace bass

extern "C" size_t bass_attention_plan_bytes(const bass_attn_desc* d) {
  if (bass::check_desc(d) != BASS_OK) return 0;
  return bass::plan_bytes_max(d);
}

static int check_plan_args(const bass_attn_desc* d, const void* ctx_len, const void* draft_len, int32_t flags,
                           int32_t padded_len, const void* plan, size_t plan_bytes) {
  const int rc = bass::check_desc(d);
  if (rc != BASS_OK) return rc;
  if (!ctx_len || !draft_len || !plan || padded_len < 0 || (flags & ~BASS_PLAN_APPEND) != 0) return BASS_ERR_INVALID_ARG;
  if (((uintptr_t)plan & 15) != 0) return BASS_ERR_INVALID_ARG;
  if ((flags & BASS_PLAN_APPEND) && padded_len > 0) return BASS_ERR_INVALID_ARG;
  if (plan_bytes < bass::plan_bytes_max(d)) return BASS_ERR_WORKSPACE_TOO_SMALL;
  return BASS_OK;
}

extern "C" int bass_attention_plan(const bass_attn_desc* d, const int32_t* ctx_len, const int32_t* draft_len, int32_t flags,
                                   int32_t padded_len, void* plan, size_t plan_bytes, int32_t* dev_status, void* stream) {
  const int rc = check_plan_args(d, ctx_len, draft_len, flags, padded_len, plan, plan_bytes);
  if (rc != BASS_OK) return rc;
  const bass::LaunchShape ls = bass::launch_shape(d, (flags & BASS_PLAN_APPEND) != 0);
  return bass::launch_plan(d, ls, padded_len, ctx_len, draft_len, plan, dev_status, stream, nullptr);
}

extern "C" int bass_attention_plan_host(const bass_attn_desc* d, const int32_t* ctx_len, const int32_t* draft_len,
                                        int32_t flags, int32_t padded_len, void* plan, size_t plan_bytes,
                                        int32_t* host_status) {
  const int rc = check_plan_args(d, ctx_len, draft_len, flags, padded_len, plan, plan_bytes);
  if (rc != BASS_OK) return rc;
  const bass::LaunchShape ls = bass::launch_shape(d, (flags & BASS_PLAN_APPEND) != 0);
  const bass::PlanShape s = bass::plan_shape(d, ls, padded_len);
  memset(plan, 0, bass::plan_layout(s.B, s.Hkv, s.nshares).bytes);
  const bool bad = bass::plan_on_host(s, ls.fused_append ? bass::kPlanAppend : 0, ctx_len, draft_len, (char*)plan);
  if (bad && host_status) *host_status |= BASS_STATUS_LEN_CLAMPED;
  return BASS_OK;
}
