// lcq_compress.hip -- the quantizer and the lossless packing stage fused,
// for gfx950.
//
// lcq_compress writes the bytes lcq_pack(lcq_quantize(x)) would, without
// the int32 codes ever reaching memory; lcq_decompress decodes a packed
// stream straight to values, as lcq_dequantize(lcq_unpack(p)) would.  Both
// directions are bound by HBM bandwidth, and the codes are the bulky
// intermediate (4 bytes per value against about 1.4 packed): not storing
// and re-reading them is what fusing buys.  The price on the compress side
// is reading the input twice, once to size the records and once to write
// them: the second pass takes the outliers from the first pass's flags and
// recomputes only the bins, with the same operations as the encoder, so
// both passes see the same codes.  (One pass with a decoupled look-back over
// the record sizes measured 453 us and more against 227 on the 512^3 float32
// field: the waiting workgroups' polls across XCDs are the cost.)
//
// Kernels (one wavefront per 1024-value chunk, the chunk kernels' lane
// layout, lcq_chunk.hpp):
//   k_cmp_stage   pass 1: classify / bin / reconstruct / verify (sections
//                 2.2, 3.1-3.3) of each value; the chunk's outlier flags and
//                 count, its record's width, mode and size; per workgroup its
//                 totals, or (large fields) atomic adds into its group's sums
//   k_cmp_scan    large fields only, one workgroup per group: chunk table and
//                 record offsets (two exclusive scans), and (last group)
//                 header, padding and size
//   k_cmp_write   pass 3: each chunk's codes again from the input -- the
//                 outliers as pass 1 flagged them, the other values' bins
//                 recomputed -- and its record (header, outlier bitmap,
//                 packed bits assembled in LDS) written at its offset, its
//                 outliers from registers behind the payload; up to
//                 kMaxCmpDirect workgroups, also the offsets themselves
//   k_decompress  per chunk: record checks, codes from the record's bits,
//                 then the dequantize path's decode and outlier gather
//                 (section 3) and one store of the values
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>

#include "lcq.h"
#include "lcq_chunk.hpp"
#include "lcq_host.hpp"
#include "lcq_math.hpp"
#include "lcq_packfmt.hpp"
#include "lcq_range.hpp"
#include "lcq_tile.hpp"

#pragma clang fp contract(off)

using namespace lcq;

namespace {

// Up to this many workgroups (of kWaves chunks) pass 3 finds its own offsets
// from pass 1's totals, 8 KiB read from L2 by each: no clear kernel before
// and no scan kernel between (31.2 to 24.9 us for a 5 M value float64 field).
// Above it the scan is worth its launch (at 4096 workgroups 38.0 us with it,
// 39.5 without).
constexpr unsigned kMaxCmpDirect = 2048;

struct CmpArgs {
  const void *in;
  uint64_t n;
  uint8_t *out;                // packed stream
  uint64_t *out_bytes;
  uint16_t *counts;            // outliers per chunk
  uint32_t *meta;              // w | mode << 8 | hb << 16 per chunk
  uint32_t *sizes;             // record bytes per chunk
  uint16_t *flags;             // per lane of a chunk with outliers: its outlier flags
  uint32_t *totals;            // per workgroup: record bytes / 16 << 16 | outliers, or null:
  unsigned long long *group;   // outliers per group of workgroups
  unsigned long long *rgroup;  // record bytes per group
  uint64_t ntiles;
  uint64_t tiles_per_group, chunks_per_group, ngroups;
  DevParams *noa;              // NOA: parameters computed on the device
  const void *partials;        // NOA, nparts > 0: range pairs pass 1 still has to reduce
  unsigned nparts;
  uint64_t eb_down;
  uint64_t step, inv, bound, low;  // ABS / REL parameters (raw bits)
  uint64_t hdr[8];                 // header of the packed stream
};
static_assert(kWaves * kChunk < 65536 && kWaves * kMaxRecord / 16 < 65536, "totals fit 16 bits each");

template <typename T, int Q>
__device__ __forceinline__ FieldParams<T> cmp_params(const CmpArgs &a) {
  using U = typename FT<T>::U;
  if constexpr (Q == kNOA) return params_from<T>(*a.noa);
  FieldParams<T> p;
  p.step = from_bits((U)a.step);
  p.inv = from_bits((U)a.inv);
  p.bound = from_bits((U)a.bound);
  p.low = from_bits((U)a.low);
  p.lossless_all = 0;
  return p;
}

// Codes of a chunk (values x in the chunk lane layout) as c' values -- the
// code, or 0 for an outlier -- and the outlier flags (bit W j + e: the lane's
// position j, e, below len).  FULL: the chunk has 1024 values.  Returns the
// chunk's outlier count.
template <typename T, int Q, bool FULL>
__device__ __forceinline__ unsigned encode_keep(
    const T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W], const FieldParams<T> &p,
    const EncK<T> &k, unsigned len, int lane,
    uint32_t (&cv)[ChunkShape<T>::NSUB][ChunkShape<T>::W], unsigned &flags) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  unsigned cnt = 0;
  flags = 0;
#pragma unroll
  for (int j = 0; j < NSUB; j++) {
    const unsigned pos = chunk_pos<W>(j, lane);
#pragma unroll
    for (int e = 0; e < W; e++) {
      // (pinned in the ragged copy: see encode_chunk_at)
      const int32_t code = encode<T, Q>(FULL ? x[j][e] : pin_v(x[j][e]), p, k);
      const bool s = code == kSent;
      const bool fs = FULL ? s : (s && pos + e < len);
      cnt += (unsigned)__popcll(__ballot(fs));
      cv[j][e] = s ? 0u : (uint32_t)code;
      flags |= (fs ? 1u : 0u) << (W * j + e);
    }
  }
  return cnt;
}

// Pass 1 for one chunk: its outlier flags and count, width, mode and record
// size (all lanes get the count and the record size).
template <typename T, int Q, bool FULL>
__device__ __forceinline__ void stage_chunk(const CmpArgs &a, const FieldParams<T> &p,
                                            const EncK<T> &k, uint64_t c, unsigned len, int lane,
                                            const T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W],
                                            unsigned &cnt, unsigned &rb) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  uint32_t cv[NSUB][W];
  unsigned flags;
  cnt = encode_keep<T, Q, FULL>(x, p, k, len, lane, cv, flags);
  unsigned w, mode;
  chunk_width<FULL, W, NSUB>(cv, len, lane, w, mode);
  const unsigned hb = cnt ? 1u : 0u;
  rb = (unsigned)record_bytes(len, w, hb);
  if (hb) a.flags[c * 64 + lane] = (uint16_t)flags;
  if (lane == 0) {
    a.counts[c] = (uint16_t)cnt;
    a.meta[c] = w | (mode << 8) | (hb << 16);
    a.sizes[c] = rb;
  }
}

// The 16 values per lane of chunk c, with ordinary (cache-allocating)
// loads when the chunk is full: the read-only first pass measured faster
// with them than with streaming loads (6 us ABS, 12-18 us REL on the 512^3
// float32 field).
template <typename T>
__device__ __forceinline__ void load_chunk_cached(const T *in, uint64_t n, uint64_t c, int lane,
                                                  T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W]) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  if (n - c * kChunk >= kChunk) {
#pragma unroll
    for (int j = 0; j < NSUB; j++) {
      const uint64_t i0 = chunk_value<W>(c, j, lane);
      if constexpr (sizeof(T) == 4) {
        const nt_f4 v = *reinterpret_cast<const nt_f4 *>(in + i0);
        x[j][0] = v.x; x[j][1] = v.y; x[j][2] = v.z; x[j][3] = v.w;
      } else {
        const nt_d2 v = *reinterpret_cast<const nt_d2 *>(in + i0);
        x[j][0] = v.x; x[j][1] = v.y;
      }
    }
  } else {
    load_chunk<T>(in, n, c, lane, x);
  }
}

// Pass 1, one chunk per wavefront.  (2 and 4 measured slower on the 512^3
// float32 field: compress 263-272 us against 253 us for ABS; their registers
// cost more occupancy than the extra loads in flight gain.  float32 is held to
// 64 registers, 8 wavefronts per SIMD: 227 to 221 us; float64 at 7 or 8 per
// SIMD spills, 196 to 216 us REL, and is left to the compiler.)
template <typename T, int Q>
__global__ __launch_bounds__(kBlock, sizeof(T) == 4 ? 8 : 1) void k_cmp_stage(CmpArgs a) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  __shared__ unsigned s_cnt[kWaves], s_rb[kWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: chunk logic is scalar
  const uint64_t n = a.n, nch = n_chunks(n);
  FieldParams<T> p;
  if (Q == kNOA && a.nparts)  // (uniform)
    p = params_from<T>(fold_params<T>(static_cast<const T *>(a.partials), a.nparts,
                                      from_bits((typename FT<T>::U)a.eb_down), a.noa));
  else
    p = cmp_params<T, Q>(a);
  const EncK<T> k = enc_consts_pinned<T, Q>(p);
  unsigned cnt = 0, rb = 0;
  const uint64_t c = (uint64_t)blockIdx.x * kWaves + wave;
  if (c < nch) {  // uniform over the wavefront
    T x[NSUB][W];
    load_chunk_cached<T>(static_cast<const T *>(a.in), n, c, lane, x);
    const unsigned len = chunk_len(n, c);
    if (len == kChunk) stage_chunk<T, Q, true>(a, p, k, c, len, lane, x, cnt, rb);
    else stage_chunk<T, Q, false>(a, p, k, c, len, lane, x, cnt, rb);
  }
  if (lane == 0) {
    s_cnt[wave] = cnt;
    s_rb[wave] = rb;
  }
  __syncthreads();
  if (tid == 0) {
    unsigned t = 0, r = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
      t += s_cnt[w];
      r += s_rb[w];
    }
    if (a.totals) {
      a.totals[blockIdx.x] = (r / 16) << 16 | t;
    } else {
      const uint64_t g = blockIdx.x / a.tiles_per_group;
      if (t) atomicAdd(a.group + g, (unsigned long long)t);
      if (r) atomicAdd(a.rgroup + g, (unsigned long long)r);
    }
  }
}

// Header (k outliers), padding and size of the packed stream, by one thread.
template <typename T, int Q>
__device__ __forceinline__ void finish_packed(const CmpArgs &a, uint64_t payload, uint64_t k) {
  const uint64_t nch = n_chunks(a.n);
  const uint64_t ot = packed_table_offset(nch), pl = packed_payload_offset(nch);
  const uint64_t oo = align16(pl + payload);
  uint64_t h[8];
#pragma unroll
  for (int i = 0; i < 8; i++) h[i] = a.hdr[i];
  h[2] = k;
  if constexpr (Q == kNOA) {
    h[4] = a.noa->step;
    h[5] = a.noa->bound;
    h[6] = a.noa->lo;
    h[7] = a.noa->hi;
  }
  uint64_t *hd = reinterpret_cast<uint64_t *>(a.out);
#pragma unroll
  for (int i = 0; i < 8; i++) hd[i] = h[i];
  reinterpret_cast<uint64_t *>(a.out + ot)[nch] = payload;
  for (uint64_t x = 64 + 8 * nch; x < ot; x++) a.out[x] = 0;
  for (uint64_t x = ot + 8 * (nch + 1); x < pl; x++) a.out[x] = 0;
  for (uint64_t x = pl + payload; x < oo; x++) a.out[x] = 0;
  *a.out_bytes = oo + k * sizeof(T);
}

// Pass 2 for group g: chunk table and record offsets.
template <typename T, int Q>
__global__ __launch_bounds__(kBlock) void k_cmp_scan(CmpArgs a) {
  __shared__ unsigned long long s_red[2][kWaves];
  __shared__ unsigned s_wt[2][kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t g = blockIdx.x;
  const uint64_t nch = n_chunks(a.n);
  const uint64_t c0 = g * a.chunks_per_group;
  const uint64_t c1 = min(c0 + a.chunks_per_group, nch);
  // the first batch's counts and sizes are loaded before the group sums are
  // reduced
  unsigned cnt_next = c0 + tid < c1 ? a.counts[c0 + tid] : 0u;
  unsigned sz_next = c0 + tid < c1 ? a.sizes[c0 + tid] : 0u;
  // outliers and record bytes of the earlier groups (unconditional loads at
  // a clamped index, masked after)
  static_assert(kMaxGroups % kBlock == 0, "whole rounds of group sums");
  unsigned long long bo = 0, br = 0;
#pragma unroll
  for (int r = 0; r < (int)(kMaxGroups / kBlock); r++) {
    const uint64_t i = (uint64_t)tid + (uint64_t)r * kBlock;
    const unsigned long long vo = a.group[i < g ? i : 0];
    const unsigned long long vr = a.rgroup[i < g ? i : 0];
    bo += i < g ? vo : 0ull;
    br += i < g ? vr : 0ull;
  }
  bo = wave_sum(bo);
  br = wave_sum(br);
  if (lane == 0) {
    s_red[0][wave] = bo;
    s_red[1][wave] = br;
  }
  __syncthreads();
  uint64_t run = 0, rrun = 0;
#pragma unroll
  for (int w = 0; w < kWaves; w++) {
    run += s_red[0][w];
    rrun += s_red[1][w];
  }
  uint64_t *chunk_tab = reinterpret_cast<uint64_t *>(a.out + 64);
  uint64_t *offs = reinterpret_cast<uint64_t *>(a.out + packed_table_offset(nch));
  for (uint64_t cb = c0; cb < c1; cb += kBlock) {
    const uint64_t c = cb + tid;
    const unsigned cnt = cnt_next, sz = sz_next;
    cnt_next = cb + kBlock + tid < c1 ? a.counts[cb + kBlock + tid] : 0u;
    sz_next = cb + kBlock + tid < c1 ? a.sizes[cb + kBlock + tid] : 0u;
    // (a batch's record bytes fit 32 bits)
    const unsigned incl = wave_incl_add(cnt), sincl = wave_incl_add(sz);
    if (lane == 63) {
      s_wt[0][wave] = incl;
      s_wt[1][wave] = sincl;
    }
    __syncthreads();
    uint64_t before = 0, total = 0, sbefore = 0, stotal = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
      if (w < wave) {
        before += s_wt[0][w];
        sbefore += s_wt[1][w];
      }
      total += s_wt[0][w];
      stotal += s_wt[1][w];
    }
    if (c < c1) {
      chunk_tab[c] = run + before + (incl - cnt);
      offs[c] = rrun + sbefore + (sincl - sz);
    }
    run += total;
    rrun += stotal;
    __syncthreads();  // s_wt is rewritten by the next batch
  }
  if (g == a.ngroups - 1 && tid == 0) finish_packed<T, Q>(a, rrun, run);
}

// c' of x: 0 for an outlier, else x's code -- its bin computed by the
// same operations as in encode (section 3.3 for REL), in the same order;
// the classification, reconstruction and check that decided which values
// are outliers were made by the first pass, whose flags say so.
template <typename T, int Q>
__device__ __forceinline__ uint32_t bin_code(T x, const FieldParams<T> &p, bool outlier) {
  if constexpr (is_rel_q<Q>()) {
    const T q = rel_bin(x, p.inv);
    const int32_t b = (int32_t)(outlier ? (T)0 : q);  // in range when not an outlier
    const uint32_t hi = (uint32_t)(to_bits(x) >> (sizeof(T) * 8 - 32));
    const uint32_t code = __builtin_amdgcn_alignbit((uint32_t)b, hi, 31);
    return outlier ? 0u : code;
  } else {
    const T q = rint_t(x * p.inv);
    return (uint32_t)(int32_t)(outlier ? (T)0 : q);  // in range when not an outlier
  }
}

// The chunk's outliers (flags: bit W j + e of each lane) to outl, in input
// order, from the registers that hold its values: gathered in the
// wavefront's LDS row (before its bits are packed there) and stored in
// contiguous runs; what does not fit the row (float64, more than 512) goes
// directly.
template <typename T>
__device__ __forceinline__ void put_outliers(const T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W],
                                             unsigned flags, int lane, uint32_t *row,
                                             typename FT<T>::U *outl) {
  using U = typename FT<T>::U;
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  constexpr unsigned kFit = 4 * kChunk / sizeof(U);
  U *srow = reinterpret_cast<U *>(row);
  unsigned at = 0;
#pragma unroll
  for (int j = 0; j < NSUB; j++) {
    uint64_t b[W], any = 0;
#pragma unroll
    for (int e = 0; e < W; e++) {
      b[e] = __ballot((flags >> (W * j + e)) & 1u);
      any |= b[e];
    }
    if (!any) continue;  // uniform
    unsigned r = at;
#pragma unroll
    for (int e = 0; e < W; e++) {
      r = lanes_below(b[e], r);
      at += (unsigned)__popcll(b[e]);
    }
#pragma unroll
    for (int e = 0; e < W; e++)
      if ((flags >> (W * j + e)) & 1u) {
        if (kFit >= kChunk || r < kFit) srow[r] = to_bits(x[j][e]);
        else outl[r] = to_bits(x[j][e]);
        r++;
      }
  }
  // (LDS accesses of one wavefront complete in issue order)
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const unsigned fit = min(at, kFit);  // uniform
  for (unsigned i = (unsigned)lane; i < fit; i += 64) outl[i] = srow[i];
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Pass 3 for one chunk: its c' values again (the first pass's outlier
// flags, the bins recomputed), its record written at rec, its outliers (by
// rank) at outl.
template <typename T, int Q, bool FULL>
__device__ __forceinline__ void write_chunk(const CmpArgs &a, const FieldParams<T> &p, uint64_t c,
                                            uint32_t m, unsigned len, int lane,
                                            const T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W],
                                            uint32_t *row, uint8_t *rec, typename FT<T>::U *outl) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  const unsigned w = m & 0xFF, mode = (m >> 8) & 1, hb = (m >> 16) & 1;
  const unsigned flags = hb ? (unsigned)a.flags[c * 64 + lane] : 0u;
  if (hb) put_outliers<T>(x, flags, lane, row, outl);
  uint32_t cv[NSUB][W];
#pragma unroll
  for (int j = 0; j < NSUB; j++) {
    const unsigned pos = chunk_pos<W>(j, lane);
#pragma unroll
    for (int e = 0; e < W; e++) {
      // positions past the end count as outliers: c' 0, no bin computed
      const bool out = ((flags >> (W * j + e)) & 1u) != 0 || (!FULL && pos + e >= len);
      cv[j][e] = bin_code<T, Q>(FULL ? x[j][e] : pin_v(x[j][e]), p, out);
    }
  }
  uint32_t z[NSUB][W];
  if (mode) chunk_z<true, W, NSUB, FULL>(cv, len, lane, z);
  else chunk_z<false, W, NSUB, FULL>(cv, len, lane, z);
  pack_bits<W, NSUB>(z, len, w, row, lane);
  write_record_head<W, NSUB>(rec, w, mode, hb, flags, lane);
  copy_words(row, packed_words(len, w), reinterpret_cast<uint32_t *>(rec + 16 + (hb ? 128 : 0)),
             lane);
}

// Record bytes / 16 and outliers of the workgroups before `tile`, and of all
// (a.totals), to every thread of the workgroup.
struct CmpSums {
  uint32_t bytes16, outliers, all_bytes16, all_outliers;
};
__device__ __forceinline__ CmpSums sum_totals(const CmpArgs &a, unsigned tile) {
  __shared__ uint32_t s_sum[4][kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  static_assert(kMaxCmpDirect == 8 * kBlock, "two loads of four per thread");
  const nt_i4 *tot = reinterpret_cast<const nt_i4 *>(a.totals);
  const unsigned nt = (unsigned)a.ntiles;
  uint32_t v[4] = {0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < 2; k++) {
    const unsigned i = (unsigned)(tid + k * kBlock);
    if (4u * (unsigned)(k * kBlock) < nt) {  // uniform
      const nt_i4 q = tot[4 * i < nt ? i : 0];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const unsigned t = 4 * i + u;
        const uint32_t w = t < nt ? (uint32_t)q[u] : 0u;  // (words past the last are garbage)
        v[0] += t < tile ? w >> 16 : 0u;
        v[1] += t < tile ? w & 0xFFFFu : 0u;
        v[2] += w >> 16;
        v[3] += w & 0xFFFFu;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const uint32_t t = lane63(wave_incl_add(v[q]));
    if (lane == 0) s_sum[q][wave] = t;
  }
  __syncthreads();
  uint32_t r[4] = {0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 4; q++)
#pragma unroll
    for (int w = 0; w < kWaves; w++) r[q] += s_sum[q][w];
  return CmpSums{r[0], r[1], r[2], r[3]};
}

// DIRECT: offsets from the totals (no scan kernel ran).  (float32 spills at 8
// wavefronts per SIMD: 512^3 ABS compress 217.4 us, REL 270; with 7, 215.9
// and 269.)
template <typename T, int Q, bool DIRECT>
__global__ __launch_bounds__(kBlock, sizeof(T) == 8 ? 1 : 7) void k_cmp_write(CmpArgs a) {
  using U = typename FT<T>::U;
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  __shared__ __align__(16) uint32_t s_w[kWaves][kChunk];  // each wavefront's packed words
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t n = a.n, nch = n_chunks(n);
  const uint64_t c = (uint64_t)blockIdx.x * kWaves + wave;
  const bool act = c < nch;  // uniform over the wavefront
  const uint64_t ot = packed_table_offset(nch), pl = packed_payload_offset(nch);
  uint64_t *chunk_tab = reinterpret_cast<uint64_t *>(a.out + 64);
  uint64_t *offs = reinterpret_cast<uint64_t *>(a.out + ot);
  T x[NSUB][W];
  if (act) load_chunk<T>(static_cast<const T *>(a.in), n, c, lane, x);
  uint64_t off, first, payload;
  if constexpr (DIRECT) {
    const CmpSums s = sum_totals(a, blockIdx.x);
    off = 16ull * s.bytes16;
    first = s.outliers;
    payload = 16ull * s.all_bytes16;
    for (int i = 0; i < wave; i++) {  // this workgroup's earlier chunks
      off += a.sizes[(uint64_t)blockIdx.x * kWaves + i];
      first += a.counts[(uint64_t)blockIdx.x * kWaves + i];
    }
    if (act && lane == 0) {
      offs[c] = off;
      chunk_tab[c] = first;
    }
    if (blockIdx.x == a.ntiles - 1 && threadIdx.x == kBlock - 1)
      finish_packed<T, Q>(a, payload, s.all_outliers);
    if (!act) return;  // no barrier follows
  } else {
    if (!act) return;  // no barrier at all
    off = offs[c];
    first = chunk_tab[c];
    payload = offs[nch];
  }
  const FieldParams<T> p = cmp_params<T, Q>(a);
  const uint32_t m = a.meta[c];
  const unsigned len = chunk_len(n, c);
  uint8_t *rec = a.out + pl + off;
  U *outl = reinterpret_cast<U *>(a.out + align16(pl + payload)) + first;
  if (len == kChunk) write_chunk<T, Q, true>(a, p, c, m, len, lane, x, s_w[wave], rec, outl);
  else write_chunk<T, Q, false>(a, p, c, m, len, lane, x, s_w[wave], rec, outl);
}

struct DcmpArgs {
  const uint8_t *in;  // packed stream
  uint64_t in_bytes;
  uint64_t n;
  void *out;
  unsigned long long *status;
  uint64_t epoch;
  int dtype;
};

// LDS of one k_decompress workgroup (each wavefront's whole record).
constexpr unsigned kDecompressLds = kWaves * (kMaxRecord + 4 * kRowPad);

template <typename T>
__global__ __launch_bounds__(kBlock) void k_decompress(DcmpArgs a) {
  using U = typename FT<T>::U;
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  __shared__ uint32_t s_rec[kWaves][kMaxRecord / 4 + kRowPad];  // each wavefront's whole record
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t n = a.n, nch = n_chunks(n);
  const uint64_t ot = packed_table_offset(nch), pl = packed_payload_offset(nch);
  const unsigned long long tag = (unsigned long long)(a.epoch << 16);
  // header and table bounds (the host checked in_bytes >= pl)
  const uint64_t *hd = reinterpret_cast<const uint64_t *>(a.in);
  const uint64_t h0 = hd[0], k = hd[2];
  const int q = (int)((h0 >> 48) & 0xFF);
  const uint64_t *offs = reinterpret_cast<const uint64_t *>(a.in + ot);
  const uint64_t payload = offs[nch];
  const bool bad = (h0 & ~(0xFFull << 48)) != packed_word0(a.dtype) || q > 2 || hd[1] != n ||
                   k > n || payload > a.in_bytes - pl ||
                   align16(pl + payload) + k * sizeof(T) > a.in_bytes;
  if (blockIdx.x == 0 && threadIdx.x == 0)
    report_status(a.status, tag, bad ? LCQ_ERR_STREAM : LCQ_OK);
  if (bad || n == 0) return;
  const uint64_t c = (uint64_t)blockIdx.x * kWaves + wave;
  if (c >= nch) return;  // uniform over the wavefront; no barrier follows
  // the record's extent from the offset table: whole 16-byte units inside
  // the payload, at most the largest record
  const uint64_t off = offs[c], nxt = offs[c + 1];
  // the chunk-table entries the decode checks, loaded with the offsets
  const uint64_t *chunk_tab = reinterpret_cast<const uint64_t *>(a.in + 64);
  const uint64_t ct_cur = chunk_tab[c], ct_nxt = c + 1 < nch ? chunk_tab[c + 1] : k;
  const unsigned len = chunk_len(n, c);
  bool ok = record_extent_ok(off, nxt, payload);
  if (!ok) {
    if (lane == 0) report_status(a.status, tag, LCQ_ERR_STREAM);
    return;
  }
  // the whole record (header, bitmap, bits) staged in LDS with 128-bit
  // loads, one round trip; then its header decides the rest
  uint32_t *row = s_rec[wave];
  stage_words(a.in + pl + off, (unsigned)((nxt - off) / 4), row, lane);
  const uint32_t h = row[0];
  const unsigned w = h & 0xFF, mode = (h >> 8) & 0xFF, hb = (h >> 16) & 0xFF;
  ok = w <= 32 && mode <= 1 && hb <= 1 && nxt - off == record_bytes(len, w, hb);
  if (!ok) {
    if (lane == 0) report_status(a.status, tag, LCQ_ERR_STREAM);
    return;
  }
  int32_t cc[NSUB][W];
  record_codes<W, NSUB>(row + (hb ? 36 : 4), hb ? reinterpret_cast<const uint8_t *>(row + 4) : nullptr,
                        w, mode, lane, cc);
  DField<T> f;
  f.stream = a.in;
  f.n = n;
  f.k = k;
  f.step = from_bits((U)hd[4]);
  f.rel = q == kREL;
  f.out = static_cast<T *>(a.out);
  f.status = a.status;
  f.tag = tag;
  const U *outl = reinterpret_cast<const U *>(a.in + align16(pl + payload));
  decode_chunk_any<T, false>(f, ct_cur, ct_nxt, outl, c, lane, cc);
}

__global__ void k_clear_cmp(uint64_t *p, uint64_t count) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// ------------------------------------------------------------ workspace ---
// [0,8)       status word of the last decompress that used it
// [64,128)    NOA parameters (DevParams)
// [256, ...)  outliers per group, then record bytes per group (kMaxGroups
//             each), cleared by every compress
// then        counts, meta and record sizes (4 bytes per chunk each), the
//             outlier flags (2 bytes per lane of a chunk), NOA's range pairs.
//             Counts take 2 of their 4 bytes per chunk; the totals follow
//             them there.
constexpr uint64_t kCwParams = 64, kCwGroups = 256;
uint64_t al256(uint64_t v) { return (v + 255) & ~255ull; }
uint64_t cw_counts_off() { return al256(kCwGroups + 16 * kMaxGroups); }
uint64_t cw_meta_off(uint64_t C) { return cw_counts_off() + counts_area(C); }
uint64_t cw_sizes_off(uint64_t C) { return al256(cw_meta_off(C) + 4 * C); }
uint64_t cw_flags_off(uint64_t C) { return al256(cw_sizes_off(C) + 4 * C); }
uint64_t cw_partials_off(uint64_t C) { return al256(cw_flags_off(C) + 128 * C); }
uint64_t cw_need(lcq_quantizer q, uint64_t n) {
  return cw_partials_off(n_chunks(n)) + (q == LCQ_NOA ? 16ull * kMinmaxBlocks : 0);
}

lcq_status check_launch_cmp() { return hipGetLastError() == hipSuccess ? LCQ_OK : LCQ_ERR_HIP; }

// Decode-call epochs tag the status word (as for the other decoders);
// seeded from the clock so a workspace left over from another process
// cannot match.
std::atomic<uint64_t> g_cmp_epoch{
    ((uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^ 0x3C3C3C3C3ull) &
    0xFFFFFFFFFFFull};

template <typename T, int Q>
lcq_status run_compress(double eb, const void *d_in, uint64_t n, void *d_out, uint64_t *d_bytes,
                        void *d_ws, hipStream_t s) {
  const int dt = sizeof(T) == 8 ? LCQ_F64 : LCQ_F32;
  const HostParams hp = host_params<T>(Q, eb);
  uint8_t *ws = static_cast<uint8_t *>(d_ws);
  const uint64_t C = n_chunks(n);
  const uint64_t ntiles = (C + kWaves - 1) / kWaves;
  CmpArgs a{};
  a.in = d_in;
  a.n = n;
  a.out = static_cast<uint8_t *>(d_out);
  a.out_bytes = d_bytes;
  a.counts = reinterpret_cast<uint16_t *>(ws + cw_counts_off());
  a.meta = reinterpret_cast<uint32_t *>(ws + cw_meta_off(C));
  a.sizes = reinterpret_cast<uint32_t *>(ws + cw_sizes_off(C));
  a.flags = reinterpret_cast<uint16_t *>(ws + cw_flags_off(C));
  a.group = reinterpret_cast<unsigned long long *>(ws + kCwGroups);
  a.rgroup = a.group + kMaxGroups;
  a.ntiles = ntiles;
  if (ntiles && ntiles <= kMaxCmpDirect)
    a.totals = reinterpret_cast<uint32_t *>(ws + cw_counts_off() + totals_at(C));
  a.tiles_per_group = tiles_per_group(ntiles, kWaves);
  a.chunks_per_group = a.tiles_per_group * kWaves;
  a.ngroups = std::max<uint64_t>(1, (ntiles + a.tiles_per_group - 1) / a.tiles_per_group);
  a.noa = reinterpret_cast<DevParams *>(ws + kCwParams);
  a.step = hp.step;
  a.inv = hp.inv;
  a.bound = hp.bound;
  a.low = hp.low;
  a.hdr[0] = (header_word0(dt, Q) & ~0xFFFFFFFFull) | kMagicPacked;
  a.hdr[1] = n;
  a.hdr[2] = 0;
  a.hdr[3] = __builtin_bit_cast(uint64_t, eb);
  a.hdr[4] = hp.step;
  a.hdr[5] = hp.bound;
  a.hdr[6] = hp.aux0;
  a.hdr[7] = hp.aux1;
  uint64_t *clear_ptr = reinterpret_cast<uint64_t *>(a.group);
  const uint64_t clear_count = a.totals ? 0 : 2 * kMaxGroups;
  if (Q == kNOA) {
    T *partials = reinterpret_cast<T *>(ws + cw_partials_off(C));
    a.partials = partials;
    a.eb_down = hp.eb_down;
    a.nparts = launch_noa_range<T>(static_cast<const T *>(d_in), n, partials, clear_ptr,
                                   clear_count, from_bits((typename FT<T>::U)hp.eb_down), a.noa, s,
                                   n != 0);
  } else if (clear_count) {
    hipLaunchKernelGGL(k_clear_cmp, dim3((unsigned)(clear_count / kBlock)), dim3(kBlock), 0, s,
                       clear_ptr, clear_count);
  }
  if (ntiles)
    hipLaunchKernelGGL((k_cmp_stage<T, Q>), dim3((unsigned)ntiles), dim3(kBlock), 0, s, a);
  if (a.totals) {
    hipLaunchKernelGGL((k_cmp_write<T, Q, true>), dim3((unsigned)ntiles), dim3(kBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL((k_cmp_scan<T, Q>), dim3((unsigned)a.ngroups), dim3(kBlock), 0, s, a);
    if (ntiles)
      hipLaunchKernelGGL((k_cmp_write<T, Q, false>), dim3((unsigned)ntiles), dim3(kBlock), 0, s, a);
  }
  return check_launch_cmp();
}

}  // namespace

extern "C" {

uint64_t lcq_compress_workspace_bytes(lcq_quantizer q, lcq_dtype t, uint64_t n) {
  if ((t != LCQ_F32 && t != LCQ_F64) || (q != LCQ_ABS && q != LCQ_REL && q != LCQ_NOA) ||
      n > LCQ_MAX_N)
    return 0;
  return cw_need(q, n);
}

lcq_status lcq_compress(lcq_quantizer q, lcq_dtype t, double eb, const void *d_in, uint64_t n,
                        void *d_packed, uint64_t packed_cap, uint64_t *d_packed_bytes, void *d_ws,
                        uint64_t ws_bytes, hipStream_t stream) {
  if (q != LCQ_ABS && q != LCQ_REL && q != LCQ_NOA) return LCQ_ERR_ARG;
  if (t != LCQ_F32 && t != LCQ_F64) return LCQ_ERR_ARG;
  if (!(eb > 0.0) || !std::isfinite(eb) || (q == LCQ_REL && !(eb < 1.0))) return LCQ_ERR_ARG;
  if (n > LCQ_MAX_N) return LCQ_ERR_ARG;
  if ((n && !d_in) || !d_packed || !d_packed_bytes || !d_ws) return LCQ_ERR_ARG;
  if ((n && !aligned16(d_in)) || !aligned16(d_packed) || !aligned16(d_ws) ||
      ((uintptr_t)d_packed_bytes & 7u))
    return LCQ_ERR_ARG;
  if (packed_cap < lcq_pack_max_bytes(t, n)) return LCQ_ERR_CAPACITY;
  if (ws_bytes < cw_need(q, n)) return LCQ_ERR_CAPACITY;
  if (t == LCQ_F32) {
    switch (q) {
      case LCQ_ABS: return run_compress<float, kABS>(eb, d_in, n, d_packed, d_packed_bytes, d_ws, stream);
      case LCQ_REL: return run_compress<float, kREL>(eb, d_in, n, d_packed, d_packed_bytes, d_ws, stream);
      default: return run_compress<float, kNOA>(eb, d_in, n, d_packed, d_packed_bytes, d_ws, stream);
    }
  }
  switch (q) {
    case LCQ_ABS: return run_compress<double, kABS>(eb, d_in, n, d_packed, d_packed_bytes, d_ws, stream);
    case LCQ_REL: return run_compress<double, kREL>(eb, d_in, n, d_packed, d_packed_bytes, d_ws, stream);
    default: return run_compress<double, kNOA>(eb, d_in, n, d_packed, d_packed_bytes, d_ws, stream);
  }
}

lcq_status lcq_decompress(lcq_dtype t, const void *d_packed, uint64_t packed_bytes, void *d_out,
                          uint64_t n, void *d_ws, uint64_t ws_bytes, hipStream_t stream) {
  if (t != LCQ_F32 && t != LCQ_F64) return LCQ_ERR_ARG;
  if (n > LCQ_MAX_N) return LCQ_ERR_ARG;
  if (!d_packed || (n && !d_out) || !d_ws) return LCQ_ERR_ARG;
  if (!aligned16(d_packed) || (n && !aligned16(d_out)) || !aligned16(d_ws)) return LCQ_ERR_ARG;
  if (ws_bytes < 8) return LCQ_ERR_CAPACITY;
  const uint64_t C = n_chunks(n);
  if (packed_bytes < packed_payload_offset(C)) return LCQ_ERR_STREAM;
  DcmpArgs a{};
  a.in = static_cast<const uint8_t *>(d_packed);
  a.in_bytes = packed_bytes;
  a.n = n;
  a.out = d_out;
  a.status = static_cast<unsigned long long *>(d_ws);
  a.epoch = g_cmp_epoch.fetch_add(1) + 1;
  a.dtype = (int)t;
  const uint64_t ntiles = std::max<uint64_t>(1, (C + kWaves - 1) / kWaves);
  if (t == LCQ_F32)
    hipLaunchKernelGGL(k_decompress<float>, dim3((unsigned)ntiles), dim3(kBlock), 0, stream, a);
  else
    hipLaunchKernelGGL(k_decompress<double>, dim3((unsigned)ntiles), dim3(kBlock),
                       lds_for_waves(24, kDecompressLds), stream, a);
  return check_launch_cmp();
}

}  // extern "C"
