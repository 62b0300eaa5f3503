// lcq_chunk.hpp -- chunk-per-wavefront quantize / dequantize for gfx950.
//
// One 64-lane wavefront owns one 1024-value chunk of the stream format (the
// granularity of its chunk table).  With W = 16 / sizeof(T), lane l holds
// values 64 W j + W l + e of the chunk (e < W): each sub-block j is one
// contiguous run of 64 W values, so every load and store instruction of a
// wavefront covers one contiguous 1 KiB (values) or 1 KiB / 512 B (codes,
// float32 / float64) range.  Ranks of outliers inside a chunk follow from
// ballots alone; no LDS and no barrier is needed for them.
//
// Quantize runs as two passes instead of one pass with a decoupled
// look-back:
//   pass 1  per value classify / bin / reconstruct / verify (sections 2.2,
//           3.1-3.3), int32 code stores, the chunk's outlier count, and the
//           first stage_cap<T>() outliers' raw bits staged per chunk; one
//           count per workgroup (very large fields: one atomic add into the
//           sum of its group of workgroups).
//   pass 2  one workgroup per group: exclusive scan of the chunk counts
//           (the chunk table), copy of staged outliers to their final,
//           input-ordered place, header and size.  A chunk with more than
//           stage_cap<T>() outliers has its codes rescanned and its raw bits
//           read from the input, by a workgroup chosen so that runs of
//           such chunks spread over all of them.
// Dequantize gathers each outlier's bits before the single store of its
// values and checks every chunk-table entry against the counted sentinels.
#pragma once
#include <hip/hip_runtime.h>

#include "lcq_math.hpp"
#include "lcq_tile.hpp"

#pragma clang fp contract(off)

namespace lcq {

// Streamed data is touched once: its loads and stores are non-temporal
// (clang's nontemporal builtins need native vector types).
typedef float nt_f4 __attribute__((ext_vector_type(4)));
typedef double nt_d2 __attribute__((ext_vector_type(2)));
typedef int nt_i4 __attribute__((ext_vector_type(4)));
typedef int nt_i2 __attribute__((ext_vector_type(2)));

// Outliers staged per chunk in pass 1: 512 bytes (float32) or 2 KiB
// (float64) per 1024-value chunk.  Hard stretches of data put tens to
// hundreds of outliers into a chunk (float32 REL at bounds near 1e-5: up to
// about 100; float64 values placed on bin borders: about 200); a chunk over
// the cap is rescanned from its codes and input in pass 2, at the cost of
// reading both again.
template <typename T> constexpr int stage_cap() { return sizeof(T) == 4 ? 128 : 256; }
constexpr uint64_t kMaxGroups = 1024;  // pass-2 workgroups (groups) at most
constexpr uint64_t kGroupChunks = 64;  // chunks per group at least (many fields at once)
// The same for one field alone, which has no other field's groups to fill
// the GPU with: a 3 M value float32 REL field at 1e-5, whose chunks mostly
// exceed the stage cap, kept 46 workgroups of 64 rescans each busy for 18 us.
constexpr uint64_t kGroupChunksAlone = 16;
// Up to this many pass-1 workgroups each stores its own outlier count and
// pass 2 sums those of the earlier groups itself (16 KiB at most, four loads
// per thread); above it the counts go to one atomic sum per group, which a
// kernel of its own has to clear first.  The launch saved is a third of a
// small field's, and 1 us of a 16.7 M value one (4096 workgroups, ABS 31.7 to
// 30.6 us); a large one does not show it (the clear runs in the shadow of the
// operation before), and 16,384 totals summed by each of 1024 pass-2
// workgroups cost more than the clear (512^3 float32 ABS 195 us against 191).
constexpr uint64_t kMaxDirectTiles = 4096;
// There, a group is four pass-1 workgroups (16 or 32 chunks).
constexpr uint64_t kDirectTilesPerGroup = kMaxDirectTiles / kMaxGroups;
static_assert(4 * kDirectTilesPerGroup >= kGroupChunksAlone, "groups of kGroupChunksAlone chunks");

// The chunk counts (2 bytes each) and the totals (4 bytes per pass-1 workgroup
// of at least kWaves chunks, read four at a time) share an area of 4 bytes per
// chunk, aligned to 256: the totals' place from its start, and where they end.
// Pass 2's write addresses come from the totals, so nothing else may lie there.
// (Checked for 256 consecutive numbers of chunks, and that 256 chunks more never
// take more than the area grows: so for all.)
constexpr uint64_t counts_area(uint64_t chunks) { return (4 * chunks + 255) / 256 * 256; }
constexpr uint64_t totals_at(uint64_t chunks) { return (2 * chunks + 15) / 16 * 16; }
constexpr uint64_t totals_end(uint64_t chunks) {
  const uint64_t tiles = (chunks + kWaves - 1) / kWaves;
  return totals_at(chunks) + (4 * tiles + 15) / 16 * 16;
}
constexpr bool totals_fit() {
  for (uint64_t c = 0; c < 256; c++) {
    if (totals_end(c) > counts_area(c) || totals_at(c) < 2 * c) return false;
    if (totals_end(c + 256) - totals_end(c) > counts_area(c + 256) - counts_area(c)) return false;
  }
  return true;
}
static_assert(totals_fit(), "the totals lie between the chunk counts and the next area");

// Pass-1 workgroups per pass-2 group for a field of `ntiles` pass-1
// workgroups of `chunks_per_tile` chunks each: at least min_chunks chunks
// per group (fewer, fuller pass-2 workgroups for many small fields), at
// most kMaxGroups groups.
__host__ __device__ inline uint64_t tiles_per_group(uint64_t ntiles, uint64_t chunks_per_tile,
                                                    uint64_t min_chunks = kGroupChunks) {
  const uint64_t by_size = (min_chunks + chunks_per_tile - 1) / chunks_per_tile;
  const uint64_t by_count = (ntiles + kMaxGroups - 1) / kMaxGroups;
  return by_size > by_count ? by_size : by_count;
}

// A lane holds W = 16 / sizeof(T) consecutive values of each sub-block (one
// 128-bit access), so a chunk is NSUB = 1024 / (64 W) sub-blocks and every
// lane holds 16 values of it: 4 x 4 (float32) or 8 x 2 (float64).
template <typename T> struct ChunkShape {
  static constexpr int W = 16 / (int)sizeof(T);
  static constexpr int NSUB = (int)kChunk / (64 * W);
  static_assert(W * NSUB == 16, "16 values per lane per chunk");
};

// W consecutive values at i0 (zeros past n).
template <typename T, int W>
__device__ __forceinline__ void load_vals(const T *in, uint64_t i0, uint64_t n, T (&x)[W]) {
  if (i0 + W <= n) {
    if constexpr (sizeof(T) == 4) {
      const nt_f4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f4 *>(in + i0));
      x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else {
      const nt_d2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_d2 *>(in + i0));
      x[0] = v.x; x[1] = v.y;
    }
  } else {
#pragma unroll
    for (int e = 0; e < W; e++) x[e] = (i0 + e < n) ? in[i0 + e] : (T)0;
  }
}

// (FULL: the caller knows all W lie below n)
template <typename T, int W, bool FULL = false>
__device__ __forceinline__ void store_vals(T *out, uint64_t i0, uint64_t n, const T (&y)[W]) {
  if (FULL || i0 + W <= n) {
    if constexpr (sizeof(T) == 4) {
      const nt_f4 o = {y[0], y[1], y[2], y[3]};
      __builtin_nontemporal_store(o, reinterpret_cast<nt_f4 *>(out + i0));
    } else {
      const nt_d2 o = {y[0], y[1]};
      __builtin_nontemporal_store(o, reinterpret_cast<nt_d2 *>(out + i0));
    }
  } else {
#pragma unroll
    for (int e = 0; e < W; e++)
      if (i0 + e < n) out[i0 + e] = y[e];
  }
}

template <int W>
__device__ __forceinline__ void load_codes(const int32_t *codes, uint64_t i0, uint64_t n,
                                           int32_t (&c)[W]) {
  if (i0 + W <= n) {
    if constexpr (W == 4) {
      const nt_i4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_i4 *>(codes + i0));
      c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
    } else {
      const nt_i2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_i2 *>(codes + i0));
      c[0] = v.x; c[1] = v.y;
    }
  } else {
#pragma unroll
    for (int e = 0; e < W; e++) c[e] = (i0 + e < n) ? codes[i0 + e] : 0;
  }
}

// (FULL: the caller knows all W lie below n)
template <int W, bool FULL = false>
__device__ __forceinline__ void store_codes(int32_t *codes, uint64_t i0, uint64_t n,
                                            const int32_t (&c)[W]) {
  if (FULL || i0 + W <= n) {
    if constexpr (W == 4) {
      const nt_i4 o = {c[0], c[1], c[2], c[3]};
      __builtin_nontemporal_store(o, reinterpret_cast<nt_i4 *>(codes + i0));
    } else {
      const nt_i2 o = {c[0], c[1]};
      __builtin_nontemporal_store(o, reinterpret_cast<nt_i2 *>(codes + i0));
    }
  } else {
#pragma unroll
    for (int e = 0; e < W; e++)
      if (i0 + e < n) codes[i0 + e] = c[e];
  }
}

// Sub-block j of chunk c, lane's first value.
template <int W>
__device__ __forceinline__ uint64_t chunk_value(uint64_t c, int j, int lane) {
  return c * kChunk + (uint64_t)(64 * W) * (unsigned)j + (uint64_t)W * (unsigned)lane;
}

// ------------------------------------------------------------- pass 1 ---
template <typename T> struct StageField {
  const T *in;
  uint64_t n;
  int32_t *codes;                 // stream + 64
  uint16_t *counts;               // one per chunk (at most 1024)
  typename FT<T>::U *stage;       // stage_cap<T>() per chunk
  uint32_t *totals;               // one count per workgroup, or null:
  unsigned long long *group;      // one sum per group of workgroups
  uint64_t tiles_per_group;
  FieldParams<T> p;
};

// The 16 values per lane of chunk c (c uniform; zeros past n).  A full
// float64 chunk is read from a scalar base with one 32-bit lane offset and
// constant sub-block offsets: its eight 64-bit addresses and bounds tests
// cost the registers of a wavefront per SIMD.  float32 has four, keeps all
// wavefronts either way, and measured faster with the test between its
// loads (512^3 ABS quantize 189.0 us against 191.9 us).
template <typename T>
__device__ __forceinline__ void load_chunk(const T *in, uint64_t n, uint64_t c, int lane,
                                           T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W]) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  const T *base = in + c * kChunk;
  const uint64_t left = n - c * kChunk;
  if (sizeof(T) == 8 && left >= kChunk) {
    typedef T nv __attribute__((ext_vector_type(16 / sizeof(T))));
#pragma unroll
    for (int j = 0; j < NSUB; j++) {
      const nv v = __builtin_nontemporal_load(
          reinterpret_cast<const nv *>(base + (unsigned)(64 * W * j) + (unsigned)(W * lane)));
#pragma unroll
      for (int e = 0; e < W; e++) x[j][e] = v[e];
    }
  } else {
#pragma unroll
    for (int j = 0; j < NSUB; j++)
      load_vals<T, W>(base, (unsigned)(64 * W * j) + (unsigned)(W * lane), left, x[j]);
  }
}

// Number of set bits of the wavefront mask b in lanes below this one, plus
// acc.
__device__ __forceinline__ unsigned lanes_below(uint64_t b, unsigned acc) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, acc));
}

// Wavefront mask of the lanes whose value e of sub-block j lies below n,
// for a chunk with `left` values from its first one on (all lanes when the
// chunk is full).  Uniform: scalar arithmetic only.
template <int W>
__device__ __forceinline__ uint64_t valid_lanes(uint64_t left, int j, int e) {
  if (left >= kChunk) return ~0ull;
  const int64_t t = (int64_t)left - (int64_t)(64 * W * j + e);  // values from lane 0's
  if (t <= 0) return 0;
  const uint64_t lanes = ((uint64_t)t + W - 1) / W;
  return lanes >= 64 ? ~0ull : ((1ull << lanes) - 1);
}

// Pass 1 for chunk c held in x (c is uniform over the wavefront): codes,
// staged outliers and the chunk's count; returns the count.  Sub-block by
// sub-block: each value's outlier flag is one wavefront mask, and a
// sub-block with outliers puts them into the wavefront's LDS row `srow` at
// their ranks (running rank = outliers of earlier sub-blocks + set bits of
// lower lanes); the first stage_cap<T>() then leave in contiguous stores.
// k: the encoder's operands (enc_consts_pinned: held in vector registers).
// FULL: the chunk has 1024 values (scalar base, no bounds test).
template <typename T, int Q, bool FULL>
__device__ __forceinline__ unsigned encode_chunk_at(const StageField<T> &f, uint64_t c, int lane,
                                                    const T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W],
                                                    typename FT<T>::U *srow, const EncK<T> &k) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  constexpr unsigned kCap = (unsigned)stage_cap<T>();
  const uint64_t left = FULL ? (uint64_t)kChunk : f.n - c * kChunk;
  int32_t *codes = f.codes + c * kChunk;
  unsigned cnt = 0;
#pragma unroll
  for (int j = 0; j < NSUB; j++) {
    const unsigned pos = (unsigned)(64 * W * j) + (unsigned)(W * lane);
    int32_t code[W];
    uint64_t b[W], any = 0;
#pragma unroll
    for (int e = 0; e < W; e++) {
      // (pinned in the ragged copy: the compiler would otherwise find the two
      // copies' arithmetic alike and hoist all of it above their branch, every
      // bin of the chunk live at once: 100 vector registers for float64 REL)
      code[e] = encode<T, Q>(FULL ? x[j][e] : pin_v(x[j][e]), f.p, k);
      b[e] = __ballot(code[e] == kSent) & valid_lanes<W>(left, j, e);
      any |= b[e];
    }
    store_codes<W, FULL>(codes, pos, left, code);
    if (any) {  // uniform
      unsigned r = cnt;
#pragma unroll
      for (int e = 0; e < W; e++) {
        r = lanes_below(b[e], r);
        cnt += (unsigned)__popcll(b[e]);
      }
#pragma unroll
      for (int e = 0; e < W; e++) {
        const bool mine = FULL ? code[e] == kSent : ((b[e] >> lane) & 1u) != 0;
        if (mine) {
          if (r < kCap) srow[r] = to_bits(x[j][e]);
          r++;
        }
      }
    }
  }
  // other lanes' LDS writes above, then this lane's read: a wavefront-scope
  // fence orders them (LDS accesses of one wavefront complete in issue
  // order, so it costs no wait)
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const unsigned staged = min(cnt, kCap);  // uniform
  for (unsigned b = 0; b < staged; b += 64)
    if (b + (unsigned)lane < staged) f.stage[c * kCap + b + lane] = srow[b + lane];
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // before the next chunk's writes
  if (lane == 0) f.counts[c] = (uint16_t)cnt;
  return cnt;
}

template <typename T, int Q>
__device__ __forceinline__ unsigned encode_chunk(const StageField<T> &f, uint64_t c, int lane,
                                                 const T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W],
                                                 typename FT<T>::U *srow, const EncK<T> &k) {
  return f.n - c * kChunk >= kChunk ? encode_chunk_at<T, Q, true>(f, c, lane, x, srow, k)
                                    : encode_chunk_at<T, Q, false>(f, c, lane, x, srow, k);
}

// Pass 1 for the CPW * stage_waves<T, Q>() chunks of workgroup `tile`, PF chunks per
// wavefront loaded before any is encoded.
template <typename T, int Q, int CPW, int PF>
__device__ void quant_chunks(const StageField<T> &f, uint64_t tile) {
  static_assert(PF > 0 && CPW % PF == 0, "whole prefetch groups");
  constexpr int kSW = stage_waves<T, Q>();
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  __shared__ unsigned s_cnt[kSW];
  __shared__ typename FT<T>::U s_stage[kSW][stage_cap<T>()];  // one row per wavefront
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: chunk logic is scalar
  const uint64_t nch = n_chunks(f.n);
  const EncK<T> k = enc_consts_pinned<T, Q>(f.p);
  unsigned wsum = 0;
#pragma unroll
  for (int r0 = 0; r0 < CPW; r0 += PF) {
    T x[PF][NSUB][W];
#pragma unroll
    for (int p = 0; p < PF; p++) {
      const uint64_t c = (tile * CPW + r0 + p) * kSW + wave;
      if (c < nch) load_chunk<T>(f.in, f.n, c, lane, x[p]);
    }
#pragma unroll
    for (int p = 0; p < PF; p++) {
      const uint64_t c = (tile * CPW + r0 + p) * kSW + wave;
      if (c < nch) wsum += encode_chunk<T, Q>(f, c, lane, x[p], s_stage[wave], k);  // uniform
    }
  }
  if (lane == 0) s_cnt[wave] = wsum;
  __syncthreads();
  if (tid == 0) {
    unsigned t = 0;
#pragma unroll
    for (int w = 0; w < kSW; w++) t += s_cnt[w];
    if (f.totals) f.totals[tile] = t;
    else if (t) atomicAdd(f.group + tile / f.tiles_per_group, (unsigned long long)t);
  }
}

// Pass 1 for the cpw * kWaves chunks of workgroup `tile`, cpw given at run
// time (the batched form, where every workgroup item first loads its
// field's descriptor): one chunk per wavefront at a time, chunk (tile cpw +
// r) kWaves + wave in round r.  The LDS (a stage row per wavefront, and its
// count) is the caller's: the batched kernel inlines this function once per
// dtype and quantizer, and arrays declared here would be allocated once for
// each of those six copies (31 KiB per workgroup: 5 workgroups per CU
// instead of 8).
template <typename T, int Q>
__device__ void quant_chunks_n(const StageField<T> &f, uint64_t tile, unsigned cpw,
                               typename FT<T>::U (*s_stage)[stage_cap<T>()], unsigned *s_cnt) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: chunk logic is scalar
  const uint64_t nch = n_chunks(f.n);
  const EncK<T> k = enc_consts_pinned<T, Q>(f.p);
  unsigned wsum = 0;
#pragma nounroll
  for (unsigned r = 0; r < cpw; r++) {
    const uint64_t c = (tile * cpw + r) * kWaves + wave;
    if (c >= nch) break;  // uniform
    // (the lane's positions recomputed in every round: hoisted out of the
    // loop they took the kernel from 36 to 95 vector registers for float32)
    const int ln = pin_v(lane);
    T x[NSUB][W];
    load_chunk<T>(f.in, f.n, c, ln, x);
    wsum += encode_chunk<T, Q>(f, c, ln, x, s_stage[wave], k);
  }
  if (lane == 0) s_cnt[wave] = wsum;
  __syncthreads();
  if (tid == 0) {
    unsigned long long t = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) t += s_cnt[w];
    if (t) atomicAdd(f.group + tile / f.tiles_per_group, t);
  }
}

// Header (outlier count k; NOA: the device's parameters), padding and size
// of an LCQ1 stream, by one thread.
template <typename T>
__device__ __forceinline__ void finish_stream(uint8_t *stream, uint64_t *stream_bytes, uint64_t n,
                                              const uint64_t (&hdr)[8], uint64_t k,
                                              const DevParams *noa) {
  const uint64_t nch = n_chunks(n);
  const uint64_t ct = chunk_table_offset(n);
  const uint64_t ce = ct + 8 * nch;
  const uint64_t oo = outlier_offset(n);
  for (uint64_t x = 64 + 4 * n; x < ct; x++) stream[x] = 0;
  for (uint64_t x = ce; x < oo; x++) stream[x] = 0;
  uint64_t h[8];
#pragma unroll
  for (int i = 0; i < 8; i++) h[i] = hdr[i];
  h[2] = k;
  if (noa) {
    h[4] = noa->step;
    h[5] = noa->bound;
    h[6] = noa->lo;
    h[7] = noa->hi;
  }
  uint64_t *hd = reinterpret_cast<uint64_t *>(stream);
#pragma unroll
  for (int i = 0; i < 8; i++) hd[i] = h[i];
  *stream_bytes = oo + k * sizeof(T);
}

// ------------------------------------------------------------- pass 2 ---
template <typename T> struct FinishField {
  const T *in;
  uint64_t n;
  uint8_t *stream;
  uint64_t *stream_bytes;
  const uint16_t *counts;
  const typename FT<T>::U *stage;
  const uint32_t *totals;  // pass-1 workgroups' counts, or null:
  const unsigned long long *group;
  uint64_t ntiles;  // (with totals)
  uint64_t chunks_per_group;
  uint64_t ngroups;
  const DevParams *noa;  // NOA: header words 4-7 come from here
  uint64_t hdr[8];
};

// Outliers of chunk c from its codes and the input (a chunk with more
// outliers than were staged), written to outl from index P on.  One wavefront; all
// code and value loads of the chunk are issued before the first rank.
template <typename T>
__device__ void rescan_chunk(const FinishField<T> &f, typename FT<T>::U *outl, uint64_t c,
                             uint64_t P, int lane) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  const int32_t *codes = reinterpret_cast<const int32_t *>(f.stream + 64);
  int32_t cc[NSUB][W];
  T x[NSUB][W];
#pragma unroll
  for (int j = 0; j < NSUB; j++) load_codes<W>(codes, chunk_value<W>(c, j, lane), f.n, cc[j]);
  load_chunk<T>(f.in, f.n, c, lane, x);
  const uint64_t left = f.n - c * kChunk;
  uint64_t run = P;
#pragma unroll
  for (int j = 0; j < NSUB; j++) {
    uint64_t b[W];
    uint64_t r = run;
#pragma unroll
    for (int e = 0; e < W; e++) {
      b[e] = __ballot(cc[j][e] == kSent) & valid_lanes<W>(left, j, e);
      r = lanes_below(b[e], (unsigned)0) + r;
      run += (uint64_t)__popcll(b[e]);
    }
#pragma unroll
    for (int e = 0; e < W; e++)
      if ((b[e] >> lane) & 1u) outl[r++] = to_bits(x[j][e]);
  }
}

// The staged rows that a pass-2 workgroup moves for its own chunks to their
// places, one outlier per thread, kCopyWindow outliers at a time: each thread
// writes the number of its chunk into LDS for its share [own0, own1) of the
// chunk's outliers, as far as they lie in the window; then outlier t (of the
// batch's `total`) of chunk i = s_own[t] is entry t - s_S[i] of its row and goes
// s_L[i] places further than t (the outliers of earlier chunks that are
// finished elsewhere, which the ranks t leave out).  Reads
// follow the rows, writes are contiguous, a batch without outliers costs
// nothing, and the work is spread evenly whatever the counts: chunk by chunk,
// with rows of more than 32 taken by one wavefront after another, this took
// 24 of the 29 us of pass 2 for a 3 M value float32 REL field at 1e-5 (about
// 100 outliers in every chunk).  (Chunk numbers found by bisection of the
// prefixes instead, up to seven dependent LDS reads: pass 2 of the 512^3
// float32 fields 6.8 us ABS and 10.0 REL against 6.5 and 8.7.)  Short loops on
// purpose: unrolled over 16 rows the kernel's instruction fetch cost more than
// the loads it overlapped.
constexpr unsigned kCopyWindow = 2048;
template <typename T>
__device__ __forceinline__ void copy_rows(const typename FT<T>::U *stage, typename FT<T>::U *out,
                                          const unsigned *s_S, const unsigned *s_L, uint8_t *s_own,
                                          unsigned chunk, unsigned own0, unsigned own1,
                                          unsigned total) {
  using U = typename FT<T>::U;
  constexpr unsigned kCap = (unsigned)stage_cap<T>();
  constexpr int kRound = 4;  // outliers per thread in flight
  static_assert(kBlock <= 256, "a batch's chunk numbers fit a byte");
#pragma nounroll
  for (unsigned w0 = 0; w0 < total; w0 += kCopyWindow) {  // uniform
    const unsigned wend = min(total, w0 + kCopyWindow);
    const unsigned end = min(own1, wend);
#pragma nounroll
    for (unsigned t = max(own0, w0); t < end; t++) s_own[t - w0] = (uint8_t)chunk;
    __syncthreads();
#pragma nounroll
    for (unsigned t0 = w0 + threadIdx.x; t0 < wend; t0 += kBlock * kRound) {
      unsigned i[kRound], t[kRound];
#pragma unroll
      for (int u = 0; u < kRound; u++) {
        t[u] = min(t0 + (unsigned)(u * kBlock), wend - 1);
        i[u] = s_own[t[u] - w0];
      }
      U v[kRound];
#pragma unroll
      for (int u = 0; u < kRound; u++) {
        v[u] = stage[i[u] * kCap + (t[u] - s_S[i[u]])];
        i[u] = s_L[i[u]];
      }
#pragma unroll
      for (int u = 0; u < kRound; u++)
        if (t0 + (unsigned)(u * kBlock) < wend) out[t[u] + i[u]] = v[u];
    }
    if (wend < total) __syncthreads();  // (uniform) s_own is rewritten
  }
}

// The staged row of chunk c (cnt <= stage cap outliers) to outl from index
// P on.  One wavefront; every load is issued before the first store.
template <typename T>
__device__ __forceinline__ void copy_staged(const FinishField<T> &f, typename FT<T>::U *outl,
                                            uint64_t c, uint64_t P, unsigned cnt, int lane) {
  using U = typename FT<T>::U;
  constexpr unsigned kCap = (unsigned)stage_cap<T>();
  constexpr int kR = (int)kCap / 64;
  U v[kR];
#pragma unroll
  for (int r = 0; r < kR; r++) {
    const unsigned i = (unsigned)lane + 64u * r;
    v[r] = f.stage[c * kCap + min(i, cnt - 1)];
  }
#pragma unroll
  for (int r = 0; r < kR; r++) {
    const unsigned i = (unsigned)lane + 64u * r;
    if (i < cnt) outl[P + i] = v[r];
  }
}

static_assert(LCQ_MAX_N / kChunk <= 0xFFFFFFFFull, "chunk indices fit 32 bits");

// Exclusive prefix of the groups' outlier counts, in LDS: every workgroup sums
// them for itself, once, and then has the first outlier and the count of any
// group without another load.  (Summed anew for each row that is not its own
// group's, and the sums of such rows' groups loaded for the hot test, pass 2
// took 2 us longer on a 384^3 float64 field with 1024 consecutive chunks of
// 200 outliers, and 2.7 us of 11 on one of 8 M values.)
constexpr int kGroupsPerThread = (int)(kMaxGroups / kBlock);  // consecutive ones
static_assert(kMaxGroups % kBlock == 0, "whole rounds of group sums");
struct GroupPrefix {
  uint64_t at[kGroupsPerThread][kBlock];  // within the wavefront that summed it
  uint64_t wave[kWaves];                  // the wavefronts' sums
};

// Fills g but for the barrier after.  Every load is issued before the first
// add (unconditional loads at a clamped index, masked afterwards).
template <typename T>
__device__ __forceinline__ void sum_groups(const FinishField<T> &f, GroupPrefix &g) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t v[kGroupsPerThread];  // (a group's count fits 32 bits: n <= 2^38)
  if (f.totals) {  // uniform
    const nt_i4 *tot = reinterpret_cast<const nt_i4 *>(f.totals);
    const unsigned nt = (unsigned)f.ntiles;
    static_assert(kDirectTilesPerGroup == 4, "a group's totals are one load");
#pragma unroll
    for (int k = 0; k < kGroupsPerThread; k++) {
      const unsigned i = (unsigned)(tid * kGroupsPerThread + k);
      const nt_i4 q = tot[4 * i < nt ? i : 0];
      v[k] = 0;
#pragma unroll
      for (int u = 0; u < 4; u++)  // (words past the last workgroup's are garbage)
        v[k] += 4 * i + u < nt ? (uint32_t)q[u] : 0u;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kGroupsPerThread; k++) {
      const unsigned i = (unsigned)(tid * kGroupsPerThread + k);
      const uint32_t w = (uint32_t)f.group[i < f.ngroups ? i : 0];
      v[k] = i < f.ngroups ? w : 0u;
    }
  }
  uint32_t sum = 0;  // (below 2^31)
#pragma unroll
  for (int k = 0; k < kGroupsPerThread; k++) sum += v[k];
  // a wavefront's sum may take more than 32 bits: its two halves apart
  const uint64_t incl = ((uint64_t)wave_incl_add(sum >> 16) << 16) + wave_incl_add(sum & 0xFFFFu);
  uint64_t at = incl - sum;
#pragma unroll
  for (int k = 0; k < kGroupsPerThread; k++) {
    g.at[k][tid] = at;
    at += v[k];
  }
  if (lane == 63) g.wave[wave] = incl;
}

// First outlier of group G (G < ngroups); outliers of all groups.
__device__ __forceinline__ uint64_t group_first(const GroupPrefix &g, uint32_t G) {
  const uint32_t t = G / kGroupsPerThread;  // the thread that holds it
  uint64_t s = g.at[G % kGroupsPerThread][t];
#pragma unroll
  for (int w = 0; w < kWaves - 1; w++) s += t >= (uint32_t)(64 * (w + 1)) ? g.wave[w] : 0ull;
  return s;
}
__device__ __forceinline__ uint64_t all_outliers(const GroupPrefix &g) {
  uint64_t s = 0;
#pragma unroll
  for (int w = 0; w < kWaves; w++) s += g.wave[w];
  return s;
}

// Index of chunk c's first outlier, from the groups' prefix and the chunk
// counts alone (so any workgroup can find it before the chunk table is
// written).  One wavefront; uniform result.
template <typename T>
__device__ uint64_t chunk_first_outlier(const FinishField<T> &f, uint64_t c, int lane,
                                        const GroupPrefix &g) {
  // chunk and group indices fit 32 bits (n <= LCQ_MAX_N = 2^38)
  const uint32_t gc = (uint32_t)c / (uint32_t)f.chunks_per_group;
  uint32_t s = 0;
  // eight loads per lane in flight per round (unconditional loads at a
  // clamped index, masked afterwards)
  for (uint64_t i0 = gc * f.chunks_per_group + (uint64_t)lane; i0 < c; i0 += 64 * 8) {
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const uint64_t i = i0 + 64 * (uint64_t)k;
      const unsigned v = f.counts[i < c ? i : 0];
      s += i < c ? v : 0u;
    }
  }
  s = wave_sum32(s);
  return group_first(g, gc) + s;
}

// A group with far more outliers than the average one (a stretch of hard
// data in an otherwise smooth field) is hot: its chunks with more than
// kDirect outliers are left to all workgroups.  Fields that are hard
// everywhere have no hot group: there each workgroup's own batch is an even
// share already.
// Pass 2 of a float64 ABS field with 1024 consecutive chunks of 200 outliers:
// of 8 M values 6.4 us with the margin 1024, one turn of copy_rows, 6.4 with 512,
// 8.0 with 2048, 8.3 with 6144 (384^3: 8.7 and 10.3 with 1024 and 6144); of 2 M
// values 6.1 with 4 times the average, 6.3 with 2, 7.7 with 8.  Fields whose
// density of outliers rises and falls over their length do not tell them apart.
constexpr unsigned kDirect = 32;
constexpr unsigned kHotMargin = 1024;
// Group G is hot: its outliers > 4 all / ngroups + kHotMargin, without the 64-bit
// division, which is built on fused multiply-adds (all: the field's outliers).
__device__ __forceinline__ bool hot_group(const GroupPrefix &g, uint32_t G, uint64_t all,
                                          uint64_t ngroups) {
  const uint64_t own = (G + 1 < ngroups ? group_first(g, G + 1) : all) - group_first(g, G);
  return own > kHotMargin && (own - kHotMargin) * ngroups > 4 * all;
}

// log2 of the threads per chunk of a pass-2 workgroup with `chunks` left.
__device__ __forceinline__ unsigned batch_shift(uint64_t chunks) {
  static_assert(kBlock == 256, "8 bits of threads");
  const unsigned m = (unsigned)min<uint64_t>((uint64_t)kBlock, chunks);
  return 8u - (m > 1 ? 32u - (unsigned)__builtin_clz(m - 1) : 0u);
}

// Pass 2 for group g: chunk-table entries of its chunks, their outliers,
// and (last group) header, padding and stream size.
template <typename T>
__device__ void quant_finish(const FinishField<T> &f, uint64_t g) {
  using U = typename FT<T>::U;
  __shared__ unsigned s_wt[kWaves];
  __shared__ unsigned s_P[kBlock];
  __shared__ unsigned s_c[kBlock];
  __shared__ uint8_t s_own[kCopyWindow];
  __shared__ GroupPrefix s_grp;
  constexpr unsigned kCap = (unsigned)stage_cap<T>();
  constexpr unsigned kScanBits = 17, kScanMask = (1u << kScanBits) - 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t n = f.n;
  const uint64_t nch = n_chunks(n);
  uint64_t *chunk_tab = reinterpret_cast<uint64_t *>(f.stream + chunk_table_offset(n));
  U *outl = reinterpret_cast<U *>(f.stream + outlier_offset(n));

  const uint64_t c0 = g * f.chunks_per_group;
  const uint64_t c1 = min(c0 + f.chunks_per_group, nch);
  // A batch of chunks: up to kBlock of them, the 1 << shift threads of each chunk
  // in a row (all of them know its count; the first one adds it to the scan).
  unsigned shift = batch_shift(c1 - c0);
  // the first batch's count (and the first count of the rescan duty below)
  // is loaded before the earlier groups are summed
  const uint64_t ca = c0 + ((unsigned)tid >> shift);
  unsigned cnt_next = ca < c1 ? f.counts[ca] : 0u;
  const uint64_t cd0 = g + (uint64_t)tid * f.ngroups;
  const unsigned duty0 = cd0 < nch ? f.counts[cd0] : 0u;

  sum_groups<T>(f, s_grp);
  __syncthreads();
  const uint64_t all = all_outliers(s_grp);
  uint64_t run = group_first(s_grp, (uint32_t)g);
  const bool hot = hot_group(s_grp, (uint32_t)g, all, f.ngroups);  // uniform

  for (uint64_t cb = c0; cb < c1; cb += kBlock) {
    const unsigned i = (unsigned)tid >> shift, part = (unsigned)tid & ((1u << shift) - 1);
    const unsigned cnt = cnt_next;
    // two prefixes from one scan: all outliers, and those moved here (chunks
    // left to other workgroups, below, would only be searched and dropped: for
    // a 512^3 float32 field with every value lossless pass 2 took 556 us with
    // them, 397 without)
    const unsigned mine = cnt <= (hot ? kDirect : kCap) ? cnt : 0u;
    const unsigned share = (mine + (1u << shift) - 1) >> shift;  // of the chunk's threads
    if (cb + kBlock < c1) {  // uniform
      shift = batch_shift(c1 - cb - kBlock);
      const uint64_t cn = cb + kBlock + ((unsigned)tid >> shift);
      cnt_next = cn < c1 ? f.counts[cn] : 0u;
    }
    static_assert(64 * kChunk < 1u << kScanBits && 64ull * kCap < 1ull << (32 - kScanBits),
                  "a wavefront's two sums fit one word");
    const unsigned incl = wave_incl_add(part == 0 ? cnt | mine << kScanBits : 0u);
    if (lane == 63) s_wt[wave] = incl;
    __syncthreads();
    unsigned before = 0, total = 0, mbefore = 0, mtotal = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
      const unsigned t = s_wt[w] & kScanMask, m = s_wt[w] >> kScanBits;
      if (w < wave) {
        before += t;
        mbefore += m;
      }
      total += t;
      mtotal += m;
    }
    before += (incl & kScanMask) - cnt;
    mbefore += (incl >> kScanBits) - mine;
    if (part == 0 && cb + i < c1) chunk_tab[cb + i] = run + before;
    s_P[i] = mbefore;
    s_c[i] = before - mbefore;
    copy_rows<T>(f.stage + cb * kCap, outl + run, s_P, s_c, s_own, i, mbefore + min(part * share, mine),
                 mbefore + min((part + 1) * share, mine), mtotal);
    run += total;
    __syncthreads();  // s_wt, s_P, s_c are rewritten by the next batch
  }

  // Chunks with more outliers than were staged, and those with more than
  // kDirect of a hot group, are finished not by their own group: workgroup g
  // takes chunks g, g + ngroups, g + 2 ngroups, ... so that runs of such chunks
  // (a stretch of hard data) spread over every workgroup instead of queueing
  // behind one.  One wavefront
  // per such chunk copies its staged row or, past the stage cap, finds its
  // outliers again from its codes and input.
  for (uint64_t t0 = 0; g + t0 * f.ngroups < nch; t0 += kBlock) {
    const uint64_t c = g + (t0 + (uint64_t)tid) * f.ngroups;
    const unsigned cn = t0 == 0 ? duty0 : (c < nch ? f.counts[c] : 0u);
    // (chunk indices fit 32 bits)
    const bool ov = cn > kCap ||
                    (cn > kDirect &&
                     hot_group(s_grp, (uint32_t)c / (uint32_t)f.chunks_per_group, all, f.ngroups));
    if (!__syncthreads_or(ov)) continue;
    const uint64_t wb = __ballot(ov);
    if (lane == 0) s_wt[wave] = (unsigned)__popcll(wb);
    __syncthreads();
    unsigned base = 0, nov = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
      if (w < wave) base += s_wt[w];
      nov += s_wt[w];
    }
    if (ov) {  // compact list of this batch's chunks and their counts
      s_P[base + lanes_below(wb, 0u)] = (unsigned)c;
      s_c[base + lanes_below(wb, 0u)] = cn;
    }
    __syncthreads();
    for (unsigned i = (unsigned)wave; i < nov; i += kWaves) {
      const uint64_t cv = s_P[i];
      const int ln = pin_v(lane);  // (positions recomputed, not held for the whole kernel)
      const uint64_t P = chunk_first_outlier<T>(f, cv, ln, s_grp);
      const unsigned cc = __builtin_amdgcn_readfirstlane(s_c[i]);
      if (cc <= kCap) copy_staged<T>(f, outl, cv, P, cc, ln);
      else rescan_chunk<T>(f, outl, cv, P, ln);
    }
    __syncthreads();  // s_wt, s_P and s_c are rewritten by the next batch
  }

  if (g == f.ngroups - 1 && tid == 0)
    finish_stream<T>(f.stream, f.stream_bytes, n, f.hdr, all, f.noa);
}

// ------------------------------------------------- small fields ---
// A field of at most small_chunks<T, Q>() chunks is quantized by one workgroup of
// kSmallWaves wavefronts in one launch: range (NOA), codes, chunk table,
// outliers and header.  At these sizes the launches are the cost, not the
// bytes: three (NOA: four) dependent launches took 14-16 us of host time
// for a field one workgroup streams in a few.  Every value stays in
// registers from its load to the outlier store (K chunks per wavefront;
// float64 NOA with two holds 127 and spills one 64-bit operand), so
// nothing is staged and the input is read once, NOA's too.
constexpr int kSmallWaves = 16;
constexpr int kSmallK = 2;  // chunks per wavefront at most
// Chunks up to which one workgroup is the faster way (kernel durations: the
// two passes take 9-10 us together at these sizes, float64 REL 10.4, NOA's
// four kernels 15.3; one workgroup takes, at 16 and 32 chunks, 5.0 and 8.3 us
// for float32 ABS, 6.4 and 11.2 REL, 7.2 and 11.6 NOA; float64 5.8 and 10.0
// ABS, 8.2 and 15.1 REL, 8.2 and 13.5 NOA).  An ablation goes where its
// counterpart goes.
template <typename T, int Q> constexpr uint64_t small_chunks() {
  if (Q == kNOA) return 32;
  return is_rel_q<Q>() ? (sizeof(T) == 4 ? 24 : 18) : (sizeof(T) == 4 ? 32 : 24);
}

// Finite minimum and maximum of the chunk's values below len (section 2.1.3;
// -0 counts as +0).
template <typename T>
__device__ __forceinline__ void chunk_range(const T (&x)[ChunkShape<T>::NSUB][ChunkShape<T>::W],
                                            unsigned len, int lane, T &lo, T &hi) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  using F = FT<T>;
#pragma unroll
  for (int j = 0; j < NSUB; j++)
#pragma unroll
    for (int e = 0; e < W; e++) {
      const T v = x[j][e];
      const bool in = (unsigned)(64 * W * j + W * lane + e) < len &&
                      ((to_bits(v) >> F::kMant) & F::kExpMask) != F::kExpMask;
      const T y = (v == (T)0) ? (T)0 : v;
      lo = in ? fmin(lo, y) : lo;
      hi = in ? fmax(hi, y) : hi;
    }
}

// Minimum and maximum over a workgroup of WAVES wavefronts, to every thread
// (s_lo, s_hi: one entry per wavefront).
template <typename T, int WAVES>
__device__ __forceinline__ void block_range(T &lo, T &hi, T *s_lo, T *s_hi) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, 64));
    hi = fmax(hi, __shfl_xor(hi, o, 64));
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_lo[wave] = lo;
    s_hi[wave] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; w++) {
    lo = fmin(lo, s_lo[w]);
    hi = fmax(hi, s_hi[w]);
  }
}

template <typename T> struct SmallField {
  const T *in;
  uint64_t n;  // 0 < n <= kSmallWaves * K * kChunk
  uint8_t *stream;
  uint64_t *stream_bytes;
  FieldParams<T> p;  // ABS / REL
  T eb_down;         // NOA
  uint64_t hdr[8];
};

template <typename T, int Q, int K>
__device__ __forceinline__ void quant_small(const SmallField<T> &f) {
  using U = typename FT<T>::U;
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  __shared__ T s_lo[kSmallWaves], s_hi[kSmallWaves];
  __shared__ unsigned s_cnt[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t n = f.n;
  const unsigned nch = (unsigned)n_chunks(n);
  if (tid < 64) s_cnt[tid] = 0;
  T x[K][NSUB][W];
#pragma unroll
  for (int r = 0; r < K; r++) {
    const unsigned c = (unsigned)(r * kSmallWaves + wave);
    if (c < nch) load_chunk<T>(f.in, n, c, lane, x[r]);
  }
  FieldParams<T> p = f.p;
  DevParams d;
  if constexpr (Q == kNOA) {
    T lo = (T)INFINITY, hi = (T)-INFINITY;
#pragma unroll
    for (int r = 0; r < K; r++) {
      const unsigned c = (unsigned)(r * kSmallWaves + wave);
      if (c < nch) {
        const uint64_t left = n - (uint64_t)c * kChunk;
        chunk_range<T>(x[r], left < kChunk ? (unsigned)left : kChunk, lane, lo, hi);
      }
    }
    block_range<T, kSmallWaves>(lo, hi, s_lo, s_hi);
    d = noa_params<T, false>(uniform(lo), uniform(hi), f.eb_down);
    p = params_from<T>(d);
  } else {
    __syncthreads();  // s_cnt is zero
  }
  const EncK<T> k = enc_consts_pinned<T, Q>(p);
  int32_t *codes = reinterpret_cast<int32_t *>(f.stream + 64);
  unsigned flags[K];  // bit W j + e: the lane's value of sub-block j is an outlier
#pragma unroll
  for (int r = 0; r < K; r++) {
    const unsigned c = (unsigned)(r * kSmallWaves + wave);
    flags[r] = 0;
    if (c >= nch) continue;  // uniform
    const uint64_t left = n - (uint64_t)c * kChunk;
    unsigned cnt = 0;
#pragma unroll
    for (int j = 0; j < NSUB; j++) {
      int32_t code[W];
#pragma unroll
      for (int e = 0; e < W; e++) {
        code[e] = encode<T, Q>(x[r][j][e], p, k);
        const uint64_t b = __ballot(code[e] == kSent) & valid_lanes<W>(left, j, e);
        cnt += (unsigned)__popcll(b);
        flags[r] |= ((unsigned)(b >> lane) & 1u) << (W * j + e);
      }
      store_codes<W>(codes + (uint64_t)c * kChunk, (unsigned)(64 * W * j + W * lane), left, code);
    }
    if (lane == 0) s_cnt[c] = cnt;
  }
  __syncthreads();
  // every wavefront scans the counts for itself
  const unsigned cc = s_cnt[lane];
  const unsigned incl = wave_incl_add(cc);
  const unsigned total = lane63(incl);
  if (wave == 0 && (unsigned)lane < nch)
    reinterpret_cast<uint64_t *>(f.stream + chunk_table_offset(n))[lane] = incl - cc;
  U *outl = reinterpret_cast<U *>(f.stream + outlier_offset(n));
#pragma unroll
  for (int r = 0; r < K; r++) {
    const unsigned c = (unsigned)(r * kSmallWaves + wave);
    if (!__ballot(flags[r] != 0)) continue;  // uniform; also past the end
    unsigned at = (unsigned)__builtin_amdgcn_readlane((int)(incl - cc), (int)c);
#pragma unroll
    for (int j = 0; j < NSUB; j++) {
      unsigned q = at;
#pragma unroll
      for (int e = 0; e < W; e++) {
        const uint64_t b = __ballot((flags[r] >> (W * j + e)) & 1u);
        q = lanes_below(b, q);
        at += (unsigned)__popcll(b);
      }
#pragma unroll
      for (int e = 0; e < W; e++)
        if ((flags[r] >> (W * j + e)) & 1u) outl[q++] = to_bits(x[r][j][e]);
    }
  }
  if (tid == (kSmallWaves - 1) * 64)  // (the wavefront with the fewest chunks)
    finish_stream<T>(f.stream, f.stream_bytes, n, f.hdr, total, Q == kNOA ? &d : nullptr);
}

// ---------------------------------------------------------- dequantize ---
// The 16 codes per lane of chunk c (c uniform; zeros past n), from a scalar
// base (as load_chunk).
template <int W, int NSUB>
__device__ __forceinline__ void load_chunk_codes(const int32_t *codes, uint64_t n, uint64_t c,
                                                 int lane, int32_t (&cc)[NSUB][W]) {
  const int32_t *base = codes + c * kChunk;
  const uint64_t left = n - c * kChunk;
  if (left >= kChunk) {
    typedef int nv __attribute__((ext_vector_type(W)));
#pragma unroll
    for (int j = 0; j < NSUB; j++) {
      const nv v = __builtin_nontemporal_load(
          reinterpret_cast<const nv *>(base + (unsigned)(64 * W * j) + (unsigned)(W * lane)));
#pragma unroll
      for (int e = 0; e < W; e++) cc[j][e] = v[e];
    }
  } else {
#pragma unroll
    for (int j = 0; j < NSUB; j++)
      load_codes<W>(base, (unsigned)(64 * W * j) + (unsigned)(W * lane), left, cc[j]);
  }
}

// The chunk-table entry of chunk c must count exactly the sentinels before it
// (cnt: those of the chunk).
template <typename T>
__device__ __forceinline__ void check_chunk(const DField<T> &f, uint64_t cur, uint64_t nxt,
                                            unsigned cnt, uint64_t c, int lane) {
  if (lane == 0 && (cur > f.k || nxt - cur != cnt || (c == 0 && cur != 0)))
    report_status(f.status, f.tag, LCQ_ERR_STREAM);
}

// v of lane `src` (mod 64), 32 or 64 bits, through the LDS permute network
// (no LDS storage).
__device__ __forceinline__ uint32_t lane_read(uint32_t v, unsigned src) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)v);
}
__device__ __forceinline__ uint64_t lane_read(uint64_t v, unsigned src) {
  return (uint64_t)lane_read((uint32_t)v, src) |
         ((uint64_t)lane_read((uint32_t)(v >> 32), src) << 32);
}

// The chunk's outliers as one row over the wavefront: lane l holds outlier l
// of the first 64 (their index range [cur, nxt) comes from the chunk table,
// so the row is loaded while the codes are decoded, in one instruction, and
// costs two registers at most; gathering each value by its rank held the
// whole chunk's values, 32 registers for float64, across a second round
// trip).  Never past the outlier count k.
template <typename T> struct OutlierRow {
  const typename FT<T>::U *outl;
  uint64_t cur, k;
  unsigned have;  // outliers in the row (uniform)
  typename FT<T>::U row;
};
template <typename T>
__device__ __forceinline__ OutlierRow<T> load_outlier_row(const typename FT<T>::U *outl,
                                                          uint64_t cur, uint64_t nxt, uint64_t k,
                                                          int lane) {
  OutlierRow<T> o;
  o.outl = outl;
  o.cur = cur;
  o.k = k;
  const uint64_t d = nxt - cur;
  o.have = d < 64 ? (unsigned)d : 64u;
  const uint64_t r = cur + (unsigned)lane;
  o.row = 0;
  if ((unsigned)lane < o.have && r < k) o.row = outl[r];
  return o;
}

// Sub-block j of a chunk: the lane's W codes decoded, sentinels replaced by
// their outliers (by rank: from the row, or past it from memory), stored.
// cnt: sentinels of the chunk before this sub-block, advanced.  FULL: the
// chunk has 1024 values; else `left`.  LIBM: the library-exp2 REL ablation.
template <typename T, bool LIBM, bool REL, bool FULL>
__device__ __forceinline__ void decode_sub(const OutlierRow<T> &o, T step, T *out, uint64_t left,
                                           int j, int lane,
                                           const int32_t (&cc)[ChunkShape<T>::W], unsigned &cnt) {
  using U = typename FT<T>::U;
  constexpr int W = ChunkShape<T>::W;
  const unsigned pos = (unsigned)(64 * W * j) + (unsigned)(W * lane);
  T y[W];
  uint64_t b[W], any = 0;
#pragma unroll
  for (int e = 0; e < W; e++) {
    y[e] = decode<T, LIBM>(cc[e], step, REL);  // (harmless for a sentinel)
    b[e] = __ballot(cc[e] == kSent) & valid_lanes<W>(FULL ? (uint64_t)kChunk : left, j, e);
    any |= b[e];
  }
  if (any) {  // uniform
    unsigned r = cnt;
#pragma unroll
    for (int e = 0; e < W; e++) {
      r = lanes_below(b[e], r);
      cnt += (unsigned)__popcll(b[e]);
    }
    const bool past = cnt > o.have;  // uniform
#pragma unroll
    for (int e = 0; e < W; e++) {
      U v = lane_read(o.row, r);
      const bool mine = ((b[e] >> lane) & 1u) != 0;
      if (past && mine && r >= o.have) {
        const uint64_t i = o.cur + r;  // checked against the outlier count
        v = i < o.k ? o.outl[i] : (U)0;
      }
      y[e] = mine ? from_bits(v) : y[e];
      r += mine ? 1u : 0u;
    }
  }
  store_vals<T, W, FULL>(out, pos, left, y);
}

// A chunk with more outliers than one row holds, by the chunk table: the
// outliers of half its sub-blocks are loaded by rank before the first of these
// sub-blocks is put together, so that one round trip serves them all.
// (Sub-block by sub-block, a trip each: 384^3 float64 fields decompressed in
// 167 us with every value lossless and 137 with 200 outliers per chunk, 154 and
// 126 this way; all sub-blocks at once, their values held: 157 and 142.)
// lim: outliers from o.cur on that may be read, at least one.
template <typename T, bool LIBM, bool REL, bool FULL>
__device__ __forceinline__ unsigned decode_dense(const OutlierRow<T> &o, unsigned lim, T step,
                                                 T *out, uint64_t left, int lane,
                                                 const int32_t (&cc)[ChunkShape<T>::NSUB][ChunkShape<T>::W]) {
  using U = typename FT<T>::U;
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB, kHalf = NSUB / 2;
  const U *outl = o.outl + o.cur;
  unsigned cnt = 0;
#pragma unroll
  for (int j0 = 0; j0 < NSUB; j0 += kHalf) {
    U v[kHalf][W];
    unsigned mine = 0;
#pragma unroll
    for (int j = 0; j < kHalf; j++) {
      unsigned r = cnt;
#pragma unroll
      for (int e = 0; e < W; e++) {
        const uint64_t b = __ballot(cc[j0 + j][e] == kSent) &
                           valid_lanes<W>(FULL ? (uint64_t)kChunk : left, j0 + j, e);
        r = lanes_below(b, r);
        cnt += (unsigned)__popcll(b);
        mine |= ((unsigned)(b >> lane) & 1u) << (W * j + e);
      }
#pragma unroll
      for (int e = 0; e < W; e++) {
        const U w = outl[min(r, lim - 1)];
        v[j][e] = r < lim ? w : (U)0;
        r += (mine >> (W * j + e)) & 1u;
      }
    }
#pragma unroll
    for (int j = 0; j < kHalf; j++) {
      T y[W];
#pragma unroll
      for (int e = 0; e < W; e++) {
        const T d = decode<T, LIBM>(cc[j0 + j][e], step, REL);
        y[e] = (mine >> (W * j + e)) & 1u ? from_bits(v[j][e]) : d;
      }
      store_vals<T, W, FULL>(out, (unsigned)(64 * W * (j0 + j)) + (unsigned)(W * lane), left, y);
    }
  }
  return cnt;
}

// Decode chunk c from its codes cc: its outliers put in, its chunk-table
// entry checked, its values stored.  cur and nxt: the chunk's chunk-table
// entry and the next one (the outlier count after the last chunk), loaded
// by the caller; the outliers are at outl.  REL: the stream's quantizer is
// REL (a template parameter, so each value's decode is straight-line code).
template <typename T, bool LIBM, bool REL, bool FULL>
__device__ __forceinline__ void decode_chunk_at(const DField<T> &f, const OutlierRow<T> &o,
                                                uint64_t nxt, uint64_t c, int lane,
                                                const int32_t (&cc)[ChunkShape<T>::NSUB][ChunkShape<T>::W]) {
  constexpr int W = ChunkShape<T>::W, NSUB = ChunkShape<T>::NSUB;
  const uint64_t left = FULL ? (uint64_t)kChunk : f.n - c * kChunk;
  T *out = f.out + c * kChunk;
  unsigned cnt = 0;
  // (float64 alone: the second path costs float32, with half the sub-blocks, more
  // on ordinary fields, 512^3 REL dequantize 172.0 us to 173.1, than it gives dense
  // ones, 175.7 to 172.5 with 100 outliers per chunk)
  if (sizeof(T) == 8 && __builtin_amdgcn_readfirstlane(nxt - o.cur > 64 && o.cur < o.k)) {
    const unsigned lim = (unsigned)min<uint64_t>(o.k - o.cur, (uint64_t)kChunk);
    cnt = decode_dense<T, LIBM, REL, FULL>(o, lim, f.step, out, left, lane, cc);
    check_chunk(f, o.cur, nxt, cnt, c, lane);
    return;
  }
#pragma unroll
  for (int j = 0; j < NSUB; j++) {
    // (pinned in the ragged copy: see encode_chunk_at)
    int32_t code[W];
#pragma unroll
    for (int e = 0; e < W; e++) code[e] = FULL ? cc[j][e] : pin_v(cc[j][e]);
    decode_sub<T, LIBM, REL, FULL>(o, f.step, out, left, j, lane, code, cnt);
  }
  check_chunk(f, o.cur, nxt, cnt, c, lane);
}

// decode_chunk_at with the quantizer kind and the chunk's fullness (both
// uniform) made template parameters.
template <typename T, bool LIBM>
__device__ __forceinline__ void decode_chunk_any(const DField<T> &f, uint64_t cur, uint64_t nxt,
                                                 const typename FT<T>::U *outl, uint64_t c,
                                                 int lane,
                                                 const int32_t (&cc)[ChunkShape<T>::NSUB][ChunkShape<T>::W]) {
  const bool full = f.n - c * kChunk >= kChunk;
  const OutlierRow<T> o = load_outlier_row<T>(outl, cur, nxt, f.k, lane);
  if (f.rel) {
    if (full) decode_chunk_at<T, LIBM, true, true>(f, o, nxt, c, lane, cc);
    else decode_chunk_at<T, LIBM, true, false>(f, o, nxt, c, lane, cc);
  } else {
    if (full) decode_chunk_at<T, LIBM, false, true>(f, o, nxt, c, lane, cc);
    else decode_chunk_at<T, LIBM, false, false>(f, o, nxt, c, lane, cc);
  }
}

// What one wavefront reads of an LCQ1 stream before anything depends on
// the header: the codes of its chunk and the two chunk-table entries
// (nxt of the last chunk is the header's outlier count, set by the caller).
// All of it lies below outlier_offset(n), which the host checked against
// the stream's size, so it may be read whatever the header says: the
// header's round trip overlaps with these loads instead of preceding them.
template <typename T> struct DecodeIn {
  int32_t cc[ChunkShape<T>::NSUB][ChunkShape<T>::W];
  uint64_t cur, nxt;
};
template <typename T>
__device__ __forceinline__ void load_decode(const uint8_t *stream, uint64_t n, uint64_t c, int lane,
                                            DecodeIn<T> &d) {
  const uint64_t *chunk_tab = reinterpret_cast<const uint64_t *>(stream + chunk_table_offset(n));
  load_chunk_codes<ChunkShape<T>::W, ChunkShape<T>::NSUB>(
      reinterpret_cast<const int32_t *>(stream + 64), n, c, lane, d.cc);
  d.cur = chunk_tab[c];
  d.nxt = chunk_tab[c + 1 < n_chunks(n) ? c + 1 : c];
}
template <typename T, bool LIBM = false>
__device__ __forceinline__ void decode_loaded(const DField<T> &f, uint64_t c, int lane,
                                              const DecodeIn<T> &d) {
  using U = typename FT<T>::U;
  const U *outl = reinterpret_cast<const U *>(f.stream + outlier_offset(f.n));
  const uint64_t nxt = c + 1 < n_chunks(f.n) ? d.nxt : f.k;
  decode_chunk_any<T, LIBM>(f, d.cur, nxt, outl, c, lane, d.cc);
}

}  // namespace lcq
