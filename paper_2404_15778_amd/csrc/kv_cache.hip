// KV-cache writer / reader of libbass: bass_kv_append, bass_kv_gather, bass_kv_cache_bytes.
//
// Section 2.1 of the BASS paper: keys and values of processed tokens are cached.  Section
// 3.2: sequences advance at their own pace, so every sequence has its own write offset and
// the rows of rejected drafts are discarded by overwriting them in the next step.
//
// The library owns the cache layout: bf16 caches are kept in MFMA fragment order (see
// bass_common.h) so the attention kernel's loads are 1 KiB-contiguous per wavefront and
// need no transposition; fp32 caches are token-major [B][Hkv][Lcap][D]; INT8 caches (the paper's
// appendix: keys and values quantized dynamically per head and per token) hold codes in the same
// fragment order plus one fp32 scale per token and kv head.
#include "bass_common.h"

namespace bass {

struct KvParams {
  int B, kmax, Hkv, D, Lcap, nblk;
  void* Kc;
  void* Vc;
  void* Kr;  // rows [B,kmax,Hkv,D] (source for append, destination for gather)
  void* Vr;
  const int32_t* off;  // [B] first cache token
  const int32_t* cnt;  // [B] number of rows
  int32_t* status;
  float* Ks;  // INT8 gather only: scales out [B,kmax,Hkv]
  float* Vs;
  const int32_t* signature;  // appends for a planned launch: nothing is written unless this word of its plan is `expected`
  int32_t expected;
};

// One thread per (sequence b, row slot i, kv head, 16-byte chunk of the row): everything a thread
// needs is two length words and one 16-byte load per tensor, so the whole launch is one short
// dependent chain (lengths -> row loads -> stores) however few rows there are.
// Cache token of row slot i of sequence b; false if the slot is unused or falls outside the
// cache.  The thread that handles the first chunk of the row (report = true) raises the status bit
// for a row count outside [0, kmax] (once, from slot 0) and for a used row outside the cache.
__device__ inline bool row_target(const KvParams& p, int b, int i, bool report, long& tok) {
  int n = p.cnt[b];
  bool bad = false;
  if (n < 0) { n = 0; bad = (i == 0); }
  if (n > p.kmax) { n = p.kmax; bad = (i == 0); }
  tok = (long)p.off[b] + i;
  const bool active = i < n;
  const bool inside = tok >= 0 && tok < p.Lcap;
  if (active && !inside) bad = true;
  if (bad && report && p.status) atomicOr(p.status, BASS_STATUS_LEN_CLAMPED);
  return active && inside;
}

template <bool kGather>
__global__ __launch_bounds__(256) void kv_rows_bf16(KvParams p) {
  const int chunks = p.D / 8;
  const long item = (long)blockIdx.x * 256 + threadIdx.x;  // over [B][kmax][Hkv][chunks]
  if (item >= (long)p.B * p.kmax * p.Hkv * chunks) return;
  const int ck = (int)(item % chunks);
  const int kvh = (int)((item / chunks) % p.Hkv);
  const int i = (int)((item / ((long)chunks * p.Hkv)) % p.kmax);
  const int b = (int)(item / ((long)chunks * p.Hkv * p.kmax));
  long tok;
  if (!row_target(p, b, i, ck == 0 && kvh == 0, tok)) return;
  const int blk = (int)(tok / kBlockTokens), w = (int)(tok % kBlockTokens);
  const int d0 = ck * 8;
  const size_t row = (size_t)item * 8;  // [B][kmax][Hkv][D] element offset of this chunk
  const size_t base = (((size_t)b * p.Hkv + kvh) * p.nblk + blk) * ((size_t)kBlockTokens * p.D);
  uint16_t* kc = (uint16_t*)p.Kc + base;
  uint16_t* vc = (uint16_t*)p.Vc + base;
  if (!kGather) {
    const uint4 kv = *(const uint4*)((const uint16_t*)p.Kr + row);
    const uint4 vv = *(const uint4*)((const uint16_t*)p.Vr + row);
    *(uint4*)(kc + k_elem_offset(p.D, w, d0)) = kv;  // 8 consecutive d share one 16-byte slot
    const uint16_t* ve = (const uint16_t*)&vv;
#pragma unroll
    for (int e = 0; e < 8; ++e) vc[v_elem_offset(p.D, w, d0 + e)] = ve[e];
  } else {
    *(uint4*)((uint16_t*)p.Kr + row) = *(const uint4*)(kc + k_elem_offset(p.D, w, d0));
    uint4 vv;
    uint16_t* ve = (uint16_t*)&vv;
#pragma unroll
    for (int e = 0; e < 8; ++e) ve[e] = vc[v_elem_offset(p.D, w, d0 + e)];
    *(uint4*)((uint16_t*)p.Vr + row) = vv;
  }
}

// ---------------------------------------------------------------------------------------
// Many rows at once (a prompt, a moved sequence): one workgroup per (sequence, kv head, 32-token cache block),
// in either direction and for bf16 and INT8 caches.  Bound by memory; what matters is that both sides are whole
// 16-byte chunks of consecutive addresses.  A cache block mixes its 32 tokens (and V turns them: eight tokens of
// one head element per chunk), so the block is turned in LDS instead of by 1- or 2-byte accesses to memory.
// Of a block that the rows cover only partly nothing but their own bytes is written, element by element in V: appends
// to other tokens of the block may run at the same time.
// Measured, 8 prompts of up to 2048 tokens, 32 heads of 128, one layer: INT8 append 162 -> 52 us (4.7 TB/s), bf16
// append and gather together 209 -> 131 us (4.9 TB/s); before: one thread per 16 bytes of a row, V by single bytes
// (INT8) or halfwords (bf16 gather).
// ---------------------------------------------------------------------------------------
constexpr int kXcds = 8;  // workgroups are dealt to the XCDs in turn

// The block a workgroup handles, and the tokens t0 .. t1 - 1 of it that take part (row slot = token - off).
struct BlockJob {
  int b, kvh, blk;
  long off, t0, t1;
  bool whole;
};

// kGrouped: all kv heads of a block of tokens go to the same XCD, one after the other: a token's rows of all heads lie
// side by side in the row tensors, and so do its scales there (4 bytes per head), which then leave that XCD's
// L2 as whole cache lines.  A sequence has an odd number of places in that order, so that every XCD is loaded alike both by a
// call that uses a few row slots of every sequence and by one with sequences of different lengths.  (1 of 200 slots, 32
// sequences, 32 heads of 128, INT8 append: 28.6 us with 8 places, of which one XCD held all the first ones.  8 prompts of 512 -
// 2048 tokens by first, second ... blocks of all sequences: a sequence to an XCD, 252 instead of 205 us for 4 layers.)
// Otherwise in the order of the caches: appends to bf16 caches, which read and write whole cache lines anyway, are 3 - 10 %
// quicker so, 32 sequences of up to 2048 tokens, 8 heads of 128: 100 -> 97 us.
// False (for the whole workgroup): nothing to do.
template <bool kGrouped>
__device__ inline bool block_job(const KvParams& p, int blocks_per_seq, BlockJob& o) {
  int j;
  if (kGrouped) {
    const int xcd = (int)(blockIdx.x % kXcds), local = (int)(blockIdx.x / kXcds);
    const int group = local / p.Hkv * kXcds + xcd, places = blocks_per_seq | 1;  // over [B][places]
    o.b = group / places;
    j = group - o.b * places;
    if (o.b >= p.B || j >= blocks_per_seq) return false;
    o.kvh = local % p.Hkv;
  } else {
    const int unit = (int)(blockIdx.x / blocks_per_seq);  // over [B][Hkv]; the grid may be rounded up
    j = (int)(blockIdx.x % blocks_per_seq);
    o.b = unit / p.Hkv;
    o.kvh = unit % p.Hkv;
    if (o.b >= p.B) return false;
  }
  int n = p.cnt[o.b];
  bool bad = false;
  if (n < 0) { n = 0; bad = true; }
  if (n > p.kmax) { n = p.kmax; bad = true; }
  o.off = p.off[o.b];
  const long lo = max(o.off, 0l), hi = min(o.off + n, (long)p.Lcap);  // tokens that exist in the cache
  if (n > 0 && (o.off < 0 || o.off + n > p.Lcap)) bad = true;
  if (bad && j == 0 && o.kvh == 0 && threadIdx.x == 0 && p.status) atomicOr(p.status, BASS_STATUS_LEN_CLAMPED);
  if (hi <= lo) return false;
  o.blk = (int)(lo / kBlockTokens) + j;
  const long first = (long)o.blk * kBlockTokens;
  o.t0 = max(lo, first);
  o.t1 = min(hi, first + kBlockTokens);
  o.whole = o.t1 - o.t0 == kBlockTokens;
  return o.t1 > o.t0;
}

// First element of token slot w's row in a row tensor [B][kmax][Hkv][D]
__device__ inline size_t row_element(const KvParams& p, const BlockJob& o, int w, int D) {
  return (((size_t)o.b * p.kmax + (size_t)((long)o.blk * kBlockTokens + w - o.off)) * p.Hkv + o.kvh) * D;
}
__device__ inline bool takes_part(const BlockJob& o, int w) {
  const long tok = (long)o.blk * kBlockTokens + w;
  return tok >= o.t0 && tok < o.t1;
}

// Token slot j (0 .. 7) of a V chunk of lane group grp
__device__ inline int v_token(int grp, int j) { return j < 4 ? 4 * grp + j : 16 + 4 * grp + (j - 4); }

template <int D, bool kPlanned>
__global__ __launch_bounds__(256) void kv_blocks_bf16_append(KvParams p, int blocks_per_seq) {
  __shared__ __align__(16) uint16_t vt[kBlockTokens][D + 8];
  const int tid = threadIdx.x;
  BlockJob o;
  if (kPlanned && *p.signature != p.expected) return;
  if (!block_job<false>(p, blocks_per_seq, o)) return;
  const size_t base = (((size_t)o.b * p.Hkv + o.kvh) * p.nblk + o.blk) * ((size_t)kBlockTokens * D);
  uint16_t* kc = (uint16_t*)p.Kc + base;
  uint16_t* vc = (uint16_t*)p.Vc + base;
  constexpr int CPR = D / 8;  // 16-byte chunks per row
  for (int c = tid; c < kBlockTokens * CPR; c += 256) {
    const int w = c / CPR, ck = c % CPR;
    if (takes_part(o, w)) {
      const size_t src = row_element(p, o, w, D) + ck * 8;
      *(uint4*)(kc + k_elem_offset(D, w, ck * 8)) = *(const uint4*)((const uint16_t*)p.Kr + src);
      *(uint4*)&vt[w][ck * 8] = *(const uint4*)((const uint16_t*)p.Vr + src);
    }
  }
  __syncthreads();
  for (int c = tid; c < (D / 16) * 64; c += 256) {
    const int mt = c / 64, l = c % 64, grp = l >> 4, dr = l & 15;
    uint16_t* dst = vc + (size_t)c * 8;
    if (o.whole) {
      uint4 chunk;
      uint16_t* e = (uint16_t*)&chunk;
#pragma unroll
      for (int jj = 0; jj < 8; ++jj) e[jj] = vt[v_token(grp, jj)][16 * mt + dr];
      *(uint4*)dst = chunk;
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {  // four consecutive tokens, or single ones
        const int w = v_token(grp, 4 * q);
        const bool first = takes_part(o, w), last = takes_part(o, w + 3);
        uint16_t e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = vt[w + i][16 * mt + dr];
        if (first && last) {
          *(uint2*)(dst + 4 * q) = make_uint2(e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (takes_part(o, w + i)) dst[4 * q + i] = e[i];
        }
      }
    }
  }
}

// Rows read back from a bf16 cache.  Both tensors pass through LDS, so that a row leaves as D / 8 consecutive
// chunks; rows are 8 elements longer there than in memory, which keeps the 2-byte writes of a V chunk (lanes:
// 16 head elements of 4 token groups) off each other's banks.
template <int D>
__global__ __launch_bounds__(256) void kv_blocks_bf16_gather(KvParams p, int blocks_per_seq) {
  __shared__ __align__(16) uint16_t kt[kBlockTokens][D + 8], vt[kBlockTokens][D + 8];
  const int tid = threadIdx.x;
  BlockJob o;
  if (!block_job<true>(p, blocks_per_seq, o)) return;
  const size_t base = (((size_t)o.b * p.Hkv + o.kvh) * p.nblk + o.blk) * ((size_t)kBlockTokens * D);
  const uint4* kc = (const uint4*)((const uint16_t*)p.Kc + base);
  const uint4* vc = (const uint4*)((const uint16_t*)p.Vc + base);
  constexpr int CPR = D / 8, kTurns = kBlockTokens * CPR / 256;  // 16-byte chunks per row; chunks per thread and tensor
  uint4 k[kTurns], v[kTurns];
#pragma unroll
  for (int i = 0; i < kTurns; ++i) {
    k[i] = kc[tid + 256 * i];
    v[i] = vc[tid + 256 * i];
  }
#pragma unroll
  for (int i = 0; i < kTurns; ++i) {
    const int c = tid + 256 * i, l = c % 64, grp = l >> 4, r = l & 15;
    const int tile = c / 64 / (D / 32), t = c / 64 % (D / 32);  // K: token 16 tile + r, head elements 32 t + 8 grp ..
    *(uint4*)&kt[16 * tile + r][32 * t + 8 * grp] = k[i];
    const uint32_t e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};     // V: head element 16 (c / 64) + r of eight tokens
#pragma unroll
    for (int j = 0; j < 8; ++j) vt[v_token(grp, j)][16 * (c / 64) + r] = (uint16_t)(e[j >> 1] >> (16 * (j & 1)));
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kTurns; ++i) {
    const int c = tid + 256 * i, w = c / CPR, ck = c % CPR;
    if (takes_part(o, w)) {
      const size_t dst = row_element(p, o, w, D) + ck * 8;
      *(uint4*)((uint16_t*)p.Kr + dst) = *(const uint4*)&kt[w][ck * 8];
      *(uint4*)((uint16_t*)p.Vr + dst) = *(const uint4*)&vt[w][ck * 8];
    }
  }
}

// Rows quantized into an INT8 cache: codes and scales as in kv_rows_i8_append below (the same operations on the
// same row).  The codes are laid down row by row in LDS (rows 16 bytes longer than in memory: chunks of
// different tokens start at different banks); the block's chunks are put together from there -- K: 16 codes of
// one row, V: one byte of 16 rows each -- and stored in consecutive order.
template <int D, bool kPlanned>
__global__ __launch_bounds__(256) void kv_blocks_i8_append(KvParams p, int blocks_per_seq) {
  __shared__ __align__(16) uint8_t kt[kBlockTokens][D + 16], vt[kBlockTokens][D + 16];
  __shared__ float kscale[kBlockTokens], vscale[kBlockTokens];
  const int tid = threadIdx.x;
  BlockJob o;
  if (kPlanned && *p.signature != p.expected) return;
  if (!block_job<true>(p, blocks_per_seq, o)) return;
  constexpr int CPR = D / 8, kTurns = kBlockTokens * CPR / 256;  // chunks of 8 elements per row; per thread and tensor
  uint4 k[kTurns], v[kTurns];
#pragma unroll
  for (int i = 0; i < kTurns; ++i) {
    const int c = tid + 256 * i, w = c / CPR, ck = c % CPR;
    k[i] = v[i] = make_uint4(0, 0, 0, 0);
    if (takes_part(o, w)) {
      const size_t src = row_element(p, o, w, D) + ck * 8;
      k[i] = *(const uint4*)((const uint16_t*)p.Kr + src);
      v[i] = *(const uint4*)((const uint16_t*)p.Vr + src);
    }
  }
#pragma unroll
  for (int i = 0; i < kTurns; ++i) {
    const int c = tid + 256 * i, w = c / CPR, ck = c % CPR;
    float ka = amax8(k[i]), va = amax8(v[i]);
#pragma unroll
    for (int s = CPR >> 1; s >= 1; s >>= 1) {  // the threads of a row are consecutive lanes
      ka = fmaxf(ka, __shfl_xor(ka, s));
      va = fmaxf(va, __shfl_xor(va, s));
    }
    const float kinv = ka > 0.f ? 127.0f / ka : 0.f;
    const float vinv = va > 0.f ? 127.0f / va : 0.f;
    *(uint2*)&kt[w][ck * 8] = quantize8(k[i], kinv);
    *(uint2*)&vt[w][ck * 8] = quantize8(v[i], vinv);
    if (ck == 0) {
      kscale[w] = ka / 127.0f;
      vscale[w] = va / 127.0f;
    }
  }
  __syncthreads();
  const size_t base = (((size_t)o.b * p.Hkv + o.kvh) * p.nblk + o.blk) * i8_block_bytes(D);
  uint8_t* kc = (uint8_t*)p.Kc + base;
  uint8_t* vc = (uint8_t*)p.Vc + base;
  for (int c = tid; c < 2 * D; c += 256) {  // the block's 16-byte chunks of codes
    const int l = c % 64, grp = l >> 4, r = l & 15;
    const int tile = c / 64 / (D / 64), ks = c / 64 % (D / 64);  // K: token 16 tile + r, head elements 64 ks + 16 grp ..
    if (takes_part(o, 16 * tile + r)) *(uint4*)(kc + 16 * c) = *(const uint4*)&kt[16 * tile + r][64 * ks + 16 * grp];
    const int d = 32 * (c / 64) + r;  // V: head elements d and d + 16 of eight tokens
    uint8_t* dst = vc + 16 * c;
    if (o.whole) {
      uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < 16; ++e) word[e >> 2] |= (uint32_t)vt[v_token(grp, e & 7)][d + 16 * (e >> 3)] << (8 * (e & 3));
      *(uint4*)dst = make_uint4(word[0], word[1], word[2], word[3]);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {  // four consecutive tokens of a head element, or single ones
        const int w = v_token(grp, 4 * (q & 1));
        const bool first = takes_part(o, w), last = takes_part(o, w + 3);
        uint8_t e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = vt[w + i][d + 16 * (q >> 1)];
        if (first && last) {
          *(uint32_t*)(dst + 4 * q) = e[0] | (uint32_t)e[1] << 8 | (uint32_t)e[2] << 16 | (uint32_t)e[3] << 24;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (takes_part(o, w + i)) dst[4 * q + i] = e[i];
        }
      }
    }
  }
  if (tid < kBlockTokens && takes_part(o, tid)) {
    ((float*)(kc + (size_t)kBlockTokens * D))[tid] = kscale[tid];
    ((float*)(vc + (size_t)kBlockTokens * D))[tid] = vscale[tid];
  }
}

// Codes and scales read back from an INT8 cache: the inverse of the turn above.
template <int D>
__global__ __launch_bounds__(256) void kv_blocks_i8_gather(KvParams p, int blocks_per_seq) {
  __shared__ __align__(16) uint8_t kt[kBlockTokens][D + 16], vt[kBlockTokens][D + 16];
  const int tid = threadIdx.x;
  BlockJob o;
  if (!block_job<true>(p, blocks_per_seq, o)) return;
  const size_t base = (((size_t)o.b * p.Hkv + o.kvh) * p.nblk + o.blk) * i8_block_bytes(D);
  const uint8_t* kc = (const uint8_t*)p.Kc + base;
  const uint8_t* vc = (const uint8_t*)p.Vc + base;
  for (int c = tid; c < 2 * D; c += 256) {
    const uint4 k = *(const uint4*)(kc + 16 * c), v = *(const uint4*)(vc + 16 * c);
    const int l = c % 64, grp = l >> 4, r = l & 15;
    const int tile = c / 64 / (D / 64), ks = c / 64 % (D / 64);
    *(uint4*)&kt[16 * tile + r][64 * ks + 16 * grp] = k;
    const uint32_t word[4] = {v.x, v.y, v.z, v.w};
    const int d = 32 * (c / 64) + r;
#pragma unroll
    for (int e = 0; e < 16; ++e) vt[v_token(grp, e & 7)][d + 16 * (e >> 3)] = (uint8_t)(word[e >> 2] >> (8 * (e & 3)));
  }
  __syncthreads();
  constexpr int CPR = D / 8;
  for (int c = tid; c < kBlockTokens * CPR; c += 256) {
    const int w = c / CPR, ck = c % CPR;
    if (takes_part(o, w)) {
      const size_t dst = row_element(p, o, w, D) + ck * 8;
      *(uint2*)((uint8_t*)p.Kr + dst) = *(const uint2*)&kt[w][ck * 8];
      *(uint2*)((uint8_t*)p.Vr + dst) = *(const uint2*)&vt[w][ck * 8];
    }
  }
  if (tid < kBlockTokens && takes_part(o, tid)) {
    const size_t row = row_element(p, o, tid, 1);  // [B][kmax][Hkv]
    p.Ks[row] = ((const float*)(kc + (size_t)kBlockTokens * D))[tid];
    p.Vs[row] = ((const float*)(vc + (size_t)kBlockTokens * D))[tid];
  }
}

template <int D>
static void launch_blocks(bool gather, bool int8, dim3 grid, hipStream_t s, const KvParams& p, int blocks_per_seq) {
  const dim3 block(256);
  if (int8) {
    if (gather) hipLaunchKernelGGL(kv_blocks_i8_gather<D>, grid, block, 0, s, p, blocks_per_seq);
    else if (p.signature) hipLaunchKernelGGL((kv_blocks_i8_append<D, true>), grid, block, 0, s, p, blocks_per_seq);
    else hipLaunchKernelGGL((kv_blocks_i8_append<D, false>), grid, block, 0, s, p, blocks_per_seq);
  } else {
    if (gather) hipLaunchKernelGGL(kv_blocks_bf16_gather<D>, grid, block, 0, s, p, blocks_per_seq);
    else if (p.signature) hipLaunchKernelGGL((kv_blocks_bf16_append<D, true>), grid, block, 0, s, p, blocks_per_seq);
    else hipLaunchKernelGGL((kv_blocks_bf16_append<D, false>), grid, block, 0, s, p, blocks_per_seq);
  }
}

template <bool kGather>
__global__ __launch_bounds__(256) void kv_rows_fp32(KvParams p) {
  const int chunks = p.D / 4;
  const long item = (long)blockIdx.x * 256 + threadIdx.x;  // over [B][kmax][Hkv][chunks]
  if (item >= (long)p.B * p.kmax * p.Hkv * chunks) return;
  const int ck = (int)(item % chunks);
  const int kvh = (int)((item / chunks) % p.Hkv);
  const int i = (int)((item / ((long)chunks * p.Hkv)) % p.kmax);
  const int b = (int)(item / ((long)chunks * p.Hkv * p.kmax));
  long tok;
  if (!row_target(p, b, i, ck == 0 && kvh == 0, tok)) return;
  const size_t row = (size_t)item * 4;
  const size_t dst = (((size_t)b * p.Hkv + kvh) * p.Lcap + tok) * p.D + ck * 4;
  if (!kGather) {
    *(float4*)((float*)p.Kc + dst) = *(const float4*)((const float*)p.Kr + row);
    *(float4*)((float*)p.Vc + dst) = *(const float4*)((const float*)p.Vr + row);
  } else {
    *(float4*)((float*)p.Kr + row) = *(const float4*)((const float*)p.Kc + dst);
    *(float4*)((float*)p.Vr + row) = *(const float4*)((const float*)p.Vc + dst);
  }
}

// ---------------------------------------------------------------------------------------
// INT8 caches.  One thread per (sequence, row slot, kv head, chunk of 8 head elements); the D/8
// threads of a row are consecutive lanes of one wavefront and agree on the row's largest
// magnitude through shuffles, so no thread may leave before them.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void kv_rows_i8_append(KvParams p) {
  const int chunks = p.D / 8;  // 8 or 16: a row's threads share an aligned group of lanes
  const long total = (long)p.B * p.kmax * p.Hkv * chunks;
  const long item_raw = (long)blockIdx.x * 256 + threadIdx.x;  // over [B][kmax][Hkv][chunks]
  const bool in_range = item_raw < total;
  const long item = in_range ? item_raw : total - 1;
  const int ck = (int)(item % chunks);
  const int kvh = (int)((item / chunks) % p.Hkv);
  const int i = (int)((item / ((long)chunks * p.Hkv)) % p.kmax);
  const int b = (int)(item / ((long)chunks * p.Hkv * p.kmax));
  long tok = 0;
  const bool ok = in_range && row_target(p, b, i, ck == 0 && kvh == 0, tok);
  uint4 kv = make_uint4(0, 0, 0, 0), vv = kv;
  if (ok) {
    kv = *(const uint4*)((const uint16_t*)p.Kr + (size_t)item * 8);
    vv = *(const uint4*)((const uint16_t*)p.Vr + (size_t)item * 8);
  }
  float ka = amax8(kv), va = amax8(vv);
  for (int o = chunks >> 1; o >= 1; o >>= 1) {
    ka = fmaxf(ka, __shfl_xor(ka, o));
    va = fmaxf(va, __shfl_xor(va, o));
  }
  if (!ok) return;
  const float kinv = ka > 0.f ? 127.0f / ka : 0.f;  // one fp32 division each
  const float vinv = va > 0.f ? 127.0f / va : 0.f;
  const int blk = (int)(tok / kBlockTokens), w = (int)(tok % kBlockTokens);
  const size_t base = (((size_t)b * p.Hkv + kvh) * p.nblk + blk) * i8_block_bytes(p.D);
  uint8_t* kc = (uint8_t*)p.Kc + base;
  uint8_t* vc = (uint8_t*)p.Vc + base;
  *(uint2*)(kc + i8_k_offset(p.D, w, ck * 8)) = quantize8(kv, kinv);  // 8 consecutive d share 8 bytes
  const uint2 vq = quantize8(vv, vinv);
#pragma unroll
  for (int e = 0; e < 8; ++e) vc[i8_v_offset(p.D, w, ck * 8 + e)] = (uint8_t)((e < 4 ? vq.x : vq.y) >> (8 * (e & 3)));
  if (ck == 0) {
    ((float*)(kc + (size_t)kBlockTokens * p.D))[w] = ka / 127.0f;
    ((float*)(vc + (size_t)kBlockTokens * p.D))[w] = va / 127.0f;
  }
}

__global__ __launch_bounds__(256) void kv_rows_i8_gather(KvParams p) {
  const int chunks = p.D / 8;
  const long item = (long)blockIdx.x * 256 + threadIdx.x;  // over [B][kmax][Hkv][chunks]
  if (item >= (long)p.B * p.kmax * p.Hkv * chunks) return;
  const int ck = (int)(item % chunks);
  const int kvh = (int)((item / chunks) % p.Hkv);
  const int i = (int)((item / ((long)chunks * p.Hkv)) % p.kmax);
  const int b = (int)(item / ((long)chunks * p.Hkv * p.kmax));
  long tok;
  if (!row_target(p, b, i, ck == 0 && kvh == 0, tok)) return;
  const int blk = (int)(tok / kBlockTokens), w = (int)(tok % kBlockTokens);
  const size_t base = (((size_t)b * p.Hkv + kvh) * p.nblk + blk) * i8_block_bytes(p.D);
  const uint8_t* kc = (const uint8_t*)p.Kc + base;
  const uint8_t* vc = (const uint8_t*)p.Vc + base;
  *(uint2*)((uint8_t*)p.Kr + (size_t)item * 8) = *(const uint2*)(kc + i8_k_offset(p.D, w, ck * 8));
  uint32_t out[2] = {0u, 0u};
#pragma unroll
  for (int e = 0; e < 8; ++e) out[e >> 2] |= (uint32_t)vc[i8_v_offset(p.D, w, ck * 8 + e)] << (8 * (e & 3));
  *(uint2*)((uint8_t*)p.Vr + (size_t)item * 8) = make_uint2(out[0], out[1]);
  if (ck == 0) {
    const size_t row = item / chunks;  // [B][kmax][Hkv]
    p.Ks[row] = ((const float*)(kc + (size_t)kBlockTokens * p.D))[w];
    p.Vs[row] = ((const float*)(vc + (size_t)kBlockTokens * p.D))[w];
  }
}

template <bool kGather>
static int launch_rows(const bass_attn_desc* d, void* Kc, void* Vc, void* Kr, void* Vr, const int32_t* off,
                       const int32_t* cnt, int32_t* status, void* stream, float* Ks = nullptr, float* Vs = nullptr,
                       const int32_t* signature = nullptr, int32_t expected = 0) {
  int rc = check_desc(d);
  if (rc != BASS_OK) return rc;
  if (!Kc || !Vc || !Kr || !Vr || !off || !cnt) return BASS_ERR_INVALID_ARG;
  if (d->dtype == BASS_DTYPE_INT8KV && (kGather != (Ks != nullptr) || kGather != (Vs != nullptr)))
    return BASS_ERR_UNSUPPORTED;  // INT8 caches are read back with bass_kv_gather_int8
  if (d->dtype != BASS_DTYPE_INT8KV && Ks) return BASS_ERR_UNSUPPORTED;
  const int chunk = d->dtype == BASS_DTYPE_FP32 ? 4 : 8;
  const int64_t items = (int64_t)d->B * d->kmax * d->Hkv * (d->D / chunk);
  if ((items + 255) / 256 > 0x7fffffff) return BASS_ERR_UNSUPPORTED;
  KvParams p{d->B, d->kmax, d->Hkv, d->D, d->Lcap, num_blocks(d->Lcap), Kc, Vc, Kr, Vr, off, cnt, status, Ks, Vs, signature, expected};
  dim3 grid((unsigned)((items + 255) / 256));
  hipStream_t s = (hipStream_t)stream;
  // From one block of row slots on, by blocks; fewer (a step's drafts) by single rows, whose launch is one short
  // dependent chain.  So are appends to INT8 caches that fill less than 192 workgroups by rows: the turn in LDS costs
  // 0.3 - 0.8 us, and there is a fraction of a wave of workgroups to gain.  Against blocks, calls of up to 192 such
  // workgroups: 4 - 5 us, up to 20 % shorter with few rows in many slots, 0 - 5 % longer with all slots used; of 192 - 256 and
  // more: blocks 16 % and more shorter with all slots used.
  const int64_t per_seq = (d->kmax + kBlockTokens - 1) / kBlockTokens + 1;  // blocks the rows of a sequence can touch
  const int64_t wgs = ((int64_t)d->B * (per_seq | 1) + kXcds - 1) / kXcds * kXcds * d->Hkv;
  const bool int8 = d->dtype == BASS_DTYPE_INT8KV;
  const bool few_rows = int8 && !kGather && !signature && items <= 192 * 256;
  if (d->dtype != BASS_DTYPE_FP32 && d->kmax >= kBlockTokens && !few_rows && wgs <= 0x7fffffff) {
    if (d->D == 128) launch_blocks<128>(kGather, int8, dim3((unsigned)wgs), s, p, (int)per_seq);
    else launch_blocks<64>(kGather, int8, dim3((unsigned)wgs), s, p, (int)per_seq);
  } else if (signature) {
    return BASS_ERR_UNSUPPORTED;  // not reached: appends for a planned launch bring at least a block of row slots
  } else if (int8) {
    if (kGather) hipLaunchKernelGGL(kv_rows_i8_gather, grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL(kv_rows_i8_append, grid, dim3(256), 0, s, p);
  } else if (d->dtype == BASS_DTYPE_BF16) {
    hipLaunchKernelGGL(kv_rows_bf16<kGather>, grid, dim3(256), 0, s, p);
  } else
    hipLaunchKernelGGL(kv_rows_fp32<kGather>, grid, dim3(256), 0, s, p);
  return launch_status();
}

int append_planned(const bass_attn_desc* d, void* Kcache, void* Vcache, const void* K_new, const void* V_new, const int32_t* L,
                   const int32_t* nq, const int32_t* signature, int32_t expected, int32_t* dev_status, void* stream) {
  return launch_rows<false>(d, Kcache, Vcache, (void*)K_new, (void*)V_new, L, nq, dev_status, stream, nullptr, nullptr,
                            signature, expected);
}

}  // namespace bass

extern "C" size_t bass_kv_cache_bytes(const bass_attn_desc* d) {
  if (bass::check_desc(d) != BASS_OK) return 0;
  if (d->dtype == BASS_DTYPE_INT8KV)
    return (size_t)d->B * d->Hkv * bass::num_blocks(d->Lcap) * bass::i8_block_bytes(d->D);
  if (d->dtype == BASS_DTYPE_BF16)
    return (size_t)d->B * d->Hkv * bass::num_blocks(d->Lcap) * bass::kBlockTokens * d->D * 2;
  return (size_t)d->B * d->Hkv * d->Lcap * d->D * 4;
}

extern "C" int bass_kv_append(const bass_attn_desc* desc, void* Kcache, void* Vcache, const void* K_new,
                              const void* V_new, const int32_t* ctx_len, const int32_t* n_new,
                              int32_t* dev_status, void* stream) {
  return bass::launch_rows<false>(desc, Kcache, Vcache, (void*)K_new, (void*)V_new, ctx_len, n_new,
                                  dev_status, stream);
}

extern "C" int bass_kv_gather(const bass_attn_desc* desc, const void* Kcache, const void* Vcache, void* K_out,
                              void* V_out, const int32_t* start, const int32_t* n, int32_t* dev_status,
                              void* stream) {
  return bass::launch_rows<true>(desc, (void*)Kcache, (void*)Vcache, K_out, V_out, start, n, dev_status,
                                 stream);
}

extern "C" int bass_kv_gather_int8(const bass_attn_desc* desc, const void* Kcache, const void* Vcache,
                                   int8_t* K_codes, int8_t* V_codes, float* K_scales, float* V_scales,
                                   const int32_t* start, const int32_t* n, int32_t* dev_status, void* stream) {
  if (!desc || desc->dtype != BASS_DTYPE_INT8KV) return desc ? BASS_ERR_UNSUPPORTED : BASS_ERR_INVALID_ARG;
  if (!K_scales || !V_scales) return BASS_ERR_INVALID_ARG;
  return bass::launch_rows<true>(desc, (void*)Kcache, (void*)Vcache, K_codes, V_codes, start, n, dev_status, stream,
                                 K_scales, V_scales);
}
