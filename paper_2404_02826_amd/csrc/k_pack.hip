// k_pack.hip -- leaf bit offsets and bit packing (Sec. 4.2, storage layout),
// for every set of a batch.
//
//   k_scan_reduce / k_scan_top / k_scan_down
//        exclusive prefix sum of the per-leaf payload bits over the whole
//        batch (depth-first leaf order inside each set); a set's offsets are
//        differences against its first leaf's offset
//        (k_scan_down adds up the block totals before its own by itself up to
//        kScanFold of them; k_scan_sizes does it all in one block for up to
//        kScanOne leaves, and k_set_sizes's work with it: a small set's leaves
//        are scanned faster than a launch starts)
//   k_set_sizes     per set: payload and meta bits, stream size, capacity
//                   check, the 128-byte header, and the size and status
//   k_pack_meta, k_pack_payload, k_pack (both in one launch, for small sets):
//   pack_meta       one thread per 64-bit meta word: gathers the fixed-stride
//                   leaf records (widths, reference codes) that overlap it
//   pack_payload    leaf-aligned blocks: each block owns the payload words
//                   that start inside its leaves, ORs every member code
//                   q - q_ref + 2^(m-1) into an LDS copy of those words (LDS
//                   atomics; a run of 8 or 4 consecutive members of one leaf
//                   per thread, 16 bytes an axis, codes of up to 32 bits put
//                   together in registers and ORed a word at a time),
//                   completes its last word from the next leaves (a member
//                   per lane), then writes every owned word once with a
//                   coalesced plain store (no global atomics, no zeroing of
//                   the output)
#include <type_traits>

#include "bbx_internal.h"

namespace bbx {

typedef unsigned __int128 u128;

constexpr int kScanPer = 16;
constexpr uint64_t kScanChunk = (uint64_t)kBlock * kScanPer;

uint64_t scan_blocks(uint64_t count) { return (count + kScanChunk - 1) / kScanChunk; }

__device__ inline uint64_t bexscan(uint64_t v, uint64_t* total) {
  __shared__ uint64_t wsum[kBlock / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint64_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    uint64_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wv] = x;
  __syncthreads();
  uint64_t off = 0, tot = 0;
  for (int k = 0; k < kBlock / 64; ++k) {
    if (k < wv) off += wsum[k];
    tot += wsum[k];
  }
  __syncthreads();
  *total = tot;
  return off + x - v;
}

// P (optional): skip when its status is not OK
__global__ void __launch_bounds__(kBlock) k_scan_reduce(uint64_t count, const uint64_t* bits,
                                                        uint64_t* part, const DevParams* P) {
  if (P && P->status != BBX_OK) return;
  const uint64_t base = blockIdx.x * kScanChunk + (uint64_t)threadIdx.x * kScanPer;
  uint64_t s = 0;
  for (int k = 0; k < kScanPer; ++k)
    if (base + k < count) s += bits[base + k];
  uint64_t tot;
  (void)bexscan(s, &tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Exclusive scan of the block partials; the grand total goes to *total.
// With P: the total must equal expect (decoding) or the status turns ECORRUPT.
__global__ void __launch_bounds__(kBlock) k_scan_top(uint64_t nparts, uint64_t* part,
                                                     uint64_t* total, DevParams* P,
                                                     uint64_t expect) {
  if (P && P->status != BBX_OK) return;
  const uint64_t per = (nparts + kBlock - 1) / kBlock;
  const uint64_t b0 = threadIdx.x * per;
  uint64_t s = 0;
  for (uint64_t k = 0; k < per; ++k)
    if (b0 + k < nparts) s += part[b0 + k];
  uint64_t tot;
  uint64_t run = bexscan(s, &tot);
  for (uint64_t k = 0; k < per; ++k)
    if (b0 + k < nparts) {
      const uint64_t v = part[b0 + k];
      part[b0 + k] = run;
      run += v;
    }
  if (threadIdx.x == 0) {
    if (total) *total = tot;
    if (P) {
      if (tot != expect) P->status = BBX_ECORRUPT;
      P->payload_bits = tot;
    }
  }
}

// fold: part holds the block totals themselves (no k_scan_top before): each
// block sums those before its own, and the last one also reports the total as
// k_scan_top does.  (It may set the status while other blocks start: what they
// then do is of no use, but stays within bits, which every later launch of the
// call leaves alone.)
constexpr uint64_t kScanFold = 1024;
__global__ void __launch_bounds__(kBlock) k_scan_down(uint64_t count, uint64_t* bits,
                                                      const uint64_t* part, uint32_t fold, uint64_t* total,
                                                      DevParams* P, uint64_t expect) {
  if (P && P->status != BBX_OK) return;
  uint64_t before = fold ? 0 : part[blockIdx.x];
  if (fold) {
    uint64_t mine = 0;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kBlock) mine += part[b];
    (void)bexscan(mine, &before);
  }
  const uint64_t base = blockIdx.x * kScanChunk + (uint64_t)threadIdx.x * kScanPer;
  uint64_t v[kScanPer];
  uint64_t s = 0;
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = base + k < count ? bits[base + k] : 0;
    s += v[k];
  }
  uint64_t tot;
  uint64_t run = bexscan(s, &tot) + before;
  for (int k = 0; k < kScanPer; ++k)
    if (base + k < count) {
      bits[base + k] = run;
      run += v[k];
    }
  if (fold && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    if (total) *total = before + tot;
    if (P) {
      if (before + tot != expect) P->status = BBX_ECORRUPT;
      P->payload_bits = before + tot;
    }
  }
}

static hipError_t scan_launch(uint64_t count, uint64_t* bits, uint64_t* part, uint64_t* total,
                              DevParams* P, uint64_t expect, hipStream_t s) {
  const uint64_t nb = scan_blocks(count);
  const uint32_t fold = nb > 0 && nb <= kScanFold;
  if (nb > 0) BBX_LAUNCH("scan_reduce", k_scan_reduce, nb, kBlock, 0, s, count, bits, part, P);
  if (!fold) BBX_LAUNCH("scan_top", k_scan_top, 1, kBlock, 0, s, nb, part, total, P, expect);
  if (nb > 0)
    BBX_LAUNCH("scan_down", k_scan_down, nb, kBlock, 0, s, count, bits, part, fold, total, P, expect);
  return hipGetLastError();
}

hipError_t launch_dec_scan(uint64_t count, uint64_t* bits, uint64_t* part, DevParams* params,
                           uint64_t expect_payload, hipStream_t s) {
  return scan_launch(count, bits, part, nullptr, params, expect_payload, s);
}

// The 128-byte header of a set whose stream is written.
__device__ void write_header(const SetDesc& S, const DevParams* P) {
  const bool lossless = P->status == kStatusLossless;
  const uint32_t dims = S.dims;
  uint64_t h[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) h[k] = 0;
  const uint64_t ver = lossless ? 3 : (seq_stream(S) ? 2 : 1);
  h[0] = (uint64_t)kMagic | (ver << 32) | ((uint64_t)S.dtype << 48) | ((uint64_t)dims << 56);
  h[1] = S.n;
  h[3] = __double_as_longlong(P->eb_user);
  h[4] = __double_as_longlong(P->eb_abs);
  h[14] = P->payload_bits;
  if (lossless) {  // no grid, no leaves, no meta section; no reference field
    h[2] = (uint64_t)S.r | ((uint64_t)S.eb_mode << 32) | ((uint64_t)S.mbits << 56);
  } else {
    h[2] = (uint64_t)S.r | ((uint64_t)S.eb_mode << 32) | ((uint64_t)S.split << 40) |
           ((uint64_t)S.ref_mode << 48) | ((uint64_t)S.mbits << 56);
    h[5] = __double_as_longlong(P->eb_eff);
    h[6] = __double_as_longlong(P->w);
    h[7] = __double_as_longlong(P->inv_w);
#pragma unroll
    for (uint32_t d = 0; d < 3; ++d) h[8 + d] = d < dims ? __double_as_longlong(P->lo[d]) : 0;
    h[11] = (uint64_t)P->G[0] | ((uint64_t)(dims > 1 ? P->G[1] : 0) << 8) |
            ((uint64_t)(dims > 2 ? P->G[2] : 0) << 16);
    h[12] = S.split ? P->nleaves : S.n_leaves;  // a split-rule partition's count is the device's
    h[13] = P->meta_bits;
    h[15] = seq_stream(S) ? P->nseq : 0;  // version 2: the sequence count
  }
  uint64_t* o = (uint64_t*)S.out;
#pragma unroll
  for (int k = 0; k < 16; ++k) o[k] = h[k];
}

// One set (one thread): payload/meta bits, stream size, capacity check, then
// the header and the caller's size and status (nothing later can fail).
__device__ void set_sizes(uint32_t s, const SetDesc* sets, DevParams* params, const uint64_t* off,
                          uint64_t total_leaves, uint64_t total, uint32_t* lossless) {
  const SetDesc& S = sets[s];
  DevParams* P = params + s;
  if (P->status == kStatusLossless) {  // every coordinate as its bits, no meta section
    P->payload_base = 0;
    P->meta_bits = 0;
    P->payload_bits = S.n * S.dims * coord_bits(S.dtype);
    P->total_bytes = kHeaderBytes + ((P->payload_bits + 63) / 64) * 8;
    if (P->total_bytes > S.out_cap)
      P->status = BBX_ENOSPC;
    else
      lossless[1 + atomicAdd(lossless, 1u)] = s;  // its coordinates are copied by k_pack
  } else if (P->status == BBX_OK) {
    const uint64_t b = S.leaf_off, e = S.leaf_off + S.n_leaves;
    const uint64_t base = S.n_leaves ? off[b] : 0;
    const uint64_t endv = S.n_leaves ? (e < total_leaves ? off[e] : total) : 0;
    uint32_t sumG = 0;  // reference field: codes, or original coordinates with ref_mode 1
    for (uint32_t d = 0; d < S.dims; ++d) sumG += S.ref_mode ? coord_bits(S.dtype) : P->G[d];
    // one record per leaf; with the bit box reduction one per sequence, with
    // a 32-bit particle count
    const uint64_t meta = seq_stream(S) ? P->nseq * (uint64_t)(S.dims * S.mbits + sumG + 32)
                                        : S.n_leaves * (uint64_t)(S.dims * S.mbits + sumG);
    P->payload_base = base;
    P->meta_bits = meta;
    P->payload_bits = endv - base;
    P->total_bytes = kHeaderBytes + ((meta + 63) / 64) * 8 + ((P->payload_bits + 63) / 64) * 8;
    if (P->total_bytes > S.out_cap) P->status = BBX_ENOSPC;
  }
  const uint32_t st = P->status == kStatusLossless ? (uint32_t)BBX_OK : P->status;
  if (st == BBX_OK) write_header(S, P);
  if (S.d_size) *S.d_size = st == BBX_OK ? P->total_bytes : ~0ull;
  if (S.d_status) *S.d_status = st;
}

__global__ void k_set_sizes(uint32_t nsets, const SetDesc* sets, DevParams* params,
                            const uint64_t* off, uint64_t total_leaves, const uint64_t* total,
                            uint32_t* lossless) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nsets) set_sizes(s, sets, params, off, total_leaves, *total, lossless);
}

// The scan and the set sizes of a batch of few leaves in one block.
constexpr uint64_t kScanOne = 8192;
constexpr uint32_t kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads) k_scan_sizes(uint32_t nsets, const SetDesc* sets,
                                                             DevParams* params, uint64_t count, uint64_t* bits,
                                                             uint32_t* lossless) {
  constexpr uint32_t W = kScanThreads / 64, kPer = kScanOne / kScanThreads;
  __shared__ uint64_t wsum[W];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t base = (uint64_t)threadIdx.x * kPer;
  uint64_t v[kPer], sum = 0;
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    v[k] = base + k < count ? bits[base + k] : 0;
    sum += v[k];
  }
  uint64_t x = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o);
    if ((int)lane >= o) x += y;
  }
  if (lane == 63) wsum[wv] = x;
  __syncthreads();
  uint64_t run = x - sum, total = 0;
#pragma unroll
  for (uint32_t k = 0; k < W; ++k) {
    run += k < wv ? wsum[k] : 0ull;
    total += wsum[k];
  }
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k)
    if (base + k < count) {
      bits[base + k] = run;
      run += v[k];
    }
  __syncthreads();
  for (uint32_t s = threadIdx.x; s < nsets; s += kScanThreads)
    set_sizes(s, sets, params, bits, count, total, lossless);
}

// ---------------------------------------------------------------- packing

// OR the bits of `val` (len bits, whose bit 0 sits at absolute bit `at`) into
// the 64-bit word whose bit 0 sits at absolute bit `w0`.
__device__ inline void or_into(uint64_t& word, uint64_t w0, u128 val, uint64_t at, uint32_t len) {
  if (len == 0) return;
  const int64_t rel = (int64_t)(at - w0);
  if (rel >= 64 || rel + (int64_t)len <= 0) return;
  if (len < 128) val &= (((u128)1) << len) - 1;
  if (rel >= 0)
    word |= (uint64_t)(val << rel);
  else
    word |= (uint64_t)(val >> (-rel));
}

// Bits of the reference's original coordinate on axis d (ref_mode 1): the
// caller's value at the reference's source index.
__device__ inline uint64_t ref_coord_bits(const SetDesc& S, uint32_t src, uint32_t d) {
  const uint64_t k = S.layout == BBX_AOS ? (uint64_t)src * S.dims + d : (uint64_t)d * S.n + src;
  if (S.dtype == BBX_F32) return ((const uint32_t*)S.pos)[k];
  return ((const uint64_t*)S.pos)[k];
}

// (forced inline: a function that two kernels call is otherwise outlined, with
// its uniform values in vector registers)
__device__ __forceinline__ void pack_meta(uint32_t nsets, const uint64_t* pre, uint64_t vb, const SetDesc* sets,
                          const DevParams* params, const LeafRec* leaves0) {
  const uint32_t s = wave_find_set(pre, nsets, vb);
  const SetDesc& S = sets[s];
  const DevParams* P = params + s;
  if (P->status != BBX_OK) return;
  const uint64_t lb = vb - pre[s], nblk = pre[s + 1] - pre[s];
  const uint32_t dims = S.dims, mbits = S.mbits;
  const uint32_t G[3] = {P->G[0], P->G[1], P->G[2]};
  const uint64_t nwords = (P->meta_bits + 63) / 64;
  const LeafRec* leaves = leaves0 + S.leaf_off;
  uint64_t* meta = (uint64_t*)(S.out + kHeaderBytes);
  if (S.ref_mode) {  // records of dims * (mbits + M) bits, written field by field
    const uint32_t M = coord_bits(S.dtype);
    const uint32_t Sb = dims * (mbits + M);
    for (uint64_t w = lb * blockDim.x + threadIdx.x; w < nwords; w += nblk * blockDim.x) {
      const uint64_t b0 = w * 64;
      const uint64_t i0 = b0 / Sb;
      uint64_t i1 = (b0 + 63) / Sb;
      if (i1 >= S.n_leaves) i1 = S.n_leaves - 1;
      uint64_t word = 0;
      for (uint64_t i = i0; i <= i1; ++i) {
        const LeafRec rec = leaves[i];
        uint64_t at = i * Sb;
#pragma unroll
        for (uint32_t d = 0; d < 3; ++d) {
          if (d >= dims) break;
          or_into(word, b0, (rec.m >> (8 * d)) & 0xffu, at, mbits);
          at += mbits;
        }
#pragma unroll
        for (uint32_t d = 0; d < 3; ++d) {
          if (d >= dims) break;
          or_into(word, b0, ref_coord_bits(S, rec.ref_src, d), at, M);
          at += M;
        }
      }
      meta[w] = word;
    }
    return;
  }
  uint32_t Sb = dims * mbits + G[0] + (dims > 1 ? G[1] : 0u) + (dims > 2 ? G[2] : 0u);
  for (uint64_t w = lb * blockDim.x + threadIdx.x; w < nwords; w += nblk * blockDim.x) {
    const uint64_t b0 = w * 64;
    const uint64_t i0 = b0 / Sb;
    uint64_t i1 = (b0 + 63) / Sb;
    if (i1 >= S.n_leaves) i1 = S.n_leaves - 1;
    uint64_t word = 0;
    for (uint64_t i = i0; i <= i1; ++i) {
      const LeafRec rec = leaves[i];
      u128 v = 0;
      uint32_t at = 0;
#pragma unroll
      for (uint32_t d = 0; d < 3; ++d) {
        if (d >= dims) break;
        v |= (u128)((rec.m >> (8 * d)) & 0xffu) << at;
        at += mbits;
      }
#pragma unroll
      for (uint32_t d = 0; d < 3; ++d) {
        if (d >= dims) break;
        v |= (u128)rec.qref[d] << at;
        at += G[d];
      }
      or_into(word, b0, v, i * Sb, Sb);
    }
    meta[w] = word;
  }
}

template <typename KT>
__device__ inline u128 member_code(const KT* keys, uint64_t stride, uint32_t dims, const LeafRec& rec,
                                   uint64_t slot) {
  u128 v = 0;
  uint32_t at = 0;
#pragma unroll
  for (uint32_t d = 0; d < 3; ++d) {
    if (d >= dims) break;
    const uint32_t m = (rec.m >> (8 * d)) & 0xffu;
    if (m == 0) continue;
    const uint32_t q = keys[(uint64_t)d * stride + slot];
    const uint64_t u = (uint64_t)((int64_t)q - (int64_t)rec.qref[d] + ((int64_t)1 << (m - 1)));
    v |= (u128)u << at;
    at += m;
  }
  return v;
}

__device__ inline uint32_t sum_m(uint32_t m) { return (m & 0xffu) + ((m >> 8) & 0xffu) + ((m >> 16) & 0xffu); }

constexpr uint32_t kLeafStage = 256;   // leaves per block (leaves_per_block)

// 16 bytes of consecutive codes, of any element alignment
template <typename KT>
struct PackRun {
  struct __attribute__((packed, aligned(2))) Raw {
    uint32_t w[4];
  } v;
  __device__ __forceinline__ void load(const KT* p) { v = *(const Raw*)p; }
  __device__ __forceinline__ uint32_t operator[](int i) const {
    return sizeof(KT) == 4 ? v.w[i & 3] : ((i & 1) ? v.w[i >> 1] >> 16 : v.w[i >> 1] & 0xffffu);
  }
};

constexpr uint32_t kPackLdsWords = 3072;  // payload words of one block's members (24 KB)

// Leaf-aligned packing: a block takes leaves_per_block(r) consecutive leaves
// and stages their records and bit offsets.  Every thread ORs the codes
// of a run of a leaf's members into an LDS copy of the payload words the
// leaves' bits touch (LDS atomics), and the block stores the words whose first
// bit lies in its leaves' bit range with coalesced plain stores.  The last such
// word can also hold the first bits of the next block's leaves: one wavefront
// adds those few members from global memory, or one thread when they come from
// several leaves.  Blocks whose bits exceed the LDS copy (very large leaves)
// assemble each word from global memory instead.
template <typename KT>
__device__ __forceinline__ void pack_payload_body(const SetDesc& S, const DevParams* P, uint64_t blk,
                                  const LeafRec* leaves, const uint64_t* off, const KT* keys,
                                  LeafRec* s_rec, uint64_t* s_off, unsigned long long* s_w) {
  const uint64_t kst = S.kst, nl = S.n_leaves, base = P->payload_base, pbits = P->payload_bits;
  const uint32_t dims = S.dims;
  const uint32_t lpb = leaves_per_block(S.r);
  const uint64_t L0 = blk * lpb;
  if (L0 >= nl) return;
  const uint32_t nlb = (uint32_t)(nl - L0 < lpb ? nl - L0 : lpb);
  for (uint32_t t = threadIdx.x; t < nlb; t += kBlock) {
    s_rec[t] = leaves[L0 + t];
    s_off[t] = off[L0 + t] - base;
  }
  const uint64_t bo1 = L0 + nlb < nl ? off[L0 + nlb] - base : pbits;
  __syncthreads();
  const uint64_t bo0 = s_off[0];
  if (bo1 <= bo0) return;  // no payload bits in these leaves (uniform)
  uint64_t* pay = (uint64_t*)(S.out + kHeaderBytes + ((P->meta_bits + 63) / 64) * 8);
  const uint64_t w_first = (bo0 + 63) / 64, w_end = (bo1 + 63) / 64;  // owned words
  const uint64_t wlo = bo0 / 64;
  const uint64_t nwb = w_end - wlo;
  const uint64_t Lend = L0 + nlb;
  if (nwb > kPackLdsWords) {  // large leaves: each owned word from global memory
    for (uint64_t w = w_first + threadIdx.x; w < w_end; w += kBlock) {
      const uint64_t b0 = w * 64;
      uint32_t a = 0, z = nlb - 1;
      while (a < z) {
        const uint32_t mid = (a + z + 1) >> 1;
        if (s_off[mid] <= b0)
          a = mid;
        else
          z = mid - 1;
      }
      uint64_t i = L0 + a;
      LeafRec rec = s_rec[a];
      uint32_t sm = sum_m(rec.m);
      const uint64_t oi = s_off[a];
      uint64_t jm = sm ? (b0 - oi) / sm : 0;
      uint64_t at = oi + jm * sm;
      uint64_t word = 0;
      while (at < b0 + 64) {
        if (sm > 0 && jm + 1 < rec.size) {
          const u128 c = member_code(keys, kst, dims, rec, (uint64_t)rec.start + 1 + jm);
          or_into(word, b0, c, at, sm);
          at += sm;
          ++jm;
        } else {
          ++i;
          if (i >= nl) break;
          rec = i < Lend ? s_rec[i - L0] : leaves[i];
          sm = sum_m(rec.m);
          jm = 0;
        }
      }
      pay[w] = word;
    }
    return;
  }
  for (uint32_t t = threadIdx.x; t < (uint32_t)nwb; t += kBlock) s_w[t] = 0;
  __syncthreads();
  // a thread takes V consecutive members of one leaf (one 16-byte load an axis,
  // of any element alignment; what lies past the leaf is in the workspace and
  // not used), a leaf of at most r members by `runs` threads.  Runs aligned in
  // the arrays needed a search for their leaf, and in sets with ragged leaves
  // every wavefront took the code for a run over two leaves as well: 13.1
  // million members in leaves of 24 and 25 84 us, 51 now; 33.6 million of 16 to
  // 32 178 and 105; 256 sets 300 and 198; 2^27 in whole leaves 480 and 434.
  // (r may be any 32-bit number, far above the set, but no leaf has more than
  // n.  With a count of runs from the block's leaf sizes, which are not in
  // scalar registers, 2^27 took 467 us)
  constexpr uint32_t V = 16 / sizeof(KT);
  const uint32_t runs = (uint32_t)(((S.r < S.n ? S.r : S.n) + V - 1) / V);
  for (uint32_t u = threadIdx.x; u < nlb * runs; u += kBlock) {
    const uint32_t a = u / runs;
    const LeafRec ra = s_rec[a];
    const uint32_t sma = sum_m(ra.m), at0 = (uint32_t)(s_off[a] - wlo * 64);
    const uint32_t j0 = V * (u - a * runs);  // (one run: a leaf has at most r members, and at most n)
    if (sma == 0 || j0 >= ra.size) continue;
    const uint32_t num = ra.size - j0 < V ? ra.size - j0 : V;
    PackRun<KT> kk[3];
#pragma unroll
    for (uint32_t d = 0; d < 3; ++d)
      if (d < dims) kk[d].load(keys + (uint64_t)d * kst + ra.start + j0);
    uint32_t hm[3], sh3[3] = {0, 0, 0};
#pragma unroll
    for (uint32_t d = 0; d < 3; ++d) {
      const uint32_t m = d < dims ? (ra.m >> (8 * d)) & 0xffu : 0u;
      hm[d] = (uint32_t)((1ull << m) >> 1) - (d < dims ? ra.qref[d] : 0u);
      if (d + 1 < 3) sh3[d + 1] = sh3[d] + m;
    }
    // (u_d = q_d - q_ref,d + 2^(m_d - 1) lies in [0, 2^m_d), m_d <= 32, so 32-bit
    // wrap-around arithmetic gives it; an axis with m_d = 0 adds nothing.  Bits
    // in the LDS copy lie below kPackLdsWords * 64: 32-bit arithmetic)
    uint32_t at = at0 + (j0 ? j0 - 1 : 0u) * sma;
    if (sma <= 32) {
      // codes of at most 32 bits: consecutive bits, assembled in registers and
      // ORed into LDS one 64-bit word at a time
      uint32_t w = at >> 6, pos = at & 63;
      uint64_t lo = 0, hi = 0;
      auto put = [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t k = 0; k < V; ++k) {
          if (j0 + k == 0 || (!whole && k >= num)) continue;  // the reference carries no payload
          uint64_t c = 0;
#pragma unroll
          for (uint32_t d = 0; d < 3; ++d)
            if (d < dims) c |= (uint64_t)(kk[d][k] + hm[d]) << sh3[d];
          lo |= c << pos;
          hi |= pos ? c >> (64 - pos) : 0ull;
          pos += sma;
          if (pos >= 64) {
            atomicOr(&s_w[w], (unsigned long long)lo);
            ++w;
            lo = hi;
            hi = 0;
            pos -= 64;
          }
        }
      };
      if (__builtin_amdgcn_ballot_w64(num < V) == 0)
        put(std::true_type());
      else
        put(std::false_type());
      if (pos > 0) atomicOr(&s_w[w], (unsigned long long)lo);
      continue;
    }
#pragma unroll
    for (uint32_t k = 0; k < V; ++k) {
      if (j0 + k == 0 || k >= num) continue;
      const uint32_t w = at >> 6, sh = at & 63;
      at += sma;
      if (sma <= 64) {
        uint64_t c = 0;
#pragma unroll
        for (uint32_t d = 0; d < 3; ++d)
          if (d < dims) c |= (uint64_t)(kk[d][k] + hm[d]) << (sh3[d] & 63);  // (64: an axis of no bits)
        atomicOr(&s_w[w], (unsigned long long)(c << sh));
        if (sh + sma > 64) atomicOr(&s_w[w + 1], (unsigned long long)(c >> (64 - sh)));
      } else {
        const u128 m = member_code(keys, kst, dims, ra, (uint64_t)ra.start + j0 + k);
        const u128 c = m << sh;
        atomicOr(&s_w[w], (unsigned long long)(uint64_t)c);
        atomicOr(&s_w[w + 1], (unsigned long long)(uint64_t)(c >> 64));
        if (sh + sma > 128) atomicOr(&s_w[w + 2], (unsigned long long)(uint64_t)(m >> (128 - sh)));
      }
    }
  }
  __syncthreads();
  if ((bo1 & 63) != 0 && bo1 < pbits && threadIdx.x < 64) {
    // bits [bo1, w_end * 64) of the last owned word come from the next leaves
    // (bo1 < pbits: leaf Lend exists).  When leaf Lend alone holds them, the
    // first wavefront adds one member per lane; otherwise one thread walks
    // the following leaves.
    const uint64_t b0 = (w_end - 1) * 64, need = w_end * 64 - bo1;
    const LeafRec rn = leaves[Lend];
    const uint32_t smn = sum_m(rn.m);
    if (smn > 0 && (uint64_t)(rn.size - 1) * smn >= need) {
      const uint32_t t = threadIdx.x;
      const uint64_t at = bo1 + (uint64_t)t * smn;
      if (t + 1 < rn.size && at < w_end * 64) {
        uint64_t part = 0;
        or_into(part, b0, member_code(keys, kst, dims, rn, (uint64_t)rn.start + 1 + t), at, smn);
        atomicOr(&s_w[w_end - 1 - wlo], (unsigned long long)part);
      }
    } else if (threadIdx.x == 0) {
      uint64_t word = s_w[w_end - 1 - wlo];
      uint64_t i = Lend;
      uint64_t at = bo1;
      while (i < nl && at < w_end * 64) {
        const LeafRec rec = leaves[i];
        const uint32_t sm = sum_m(rec.m);
        for (uint64_t jm = 0; sm > 0 && jm + 1 < rec.size && at < w_end * 64; ++jm) {
          const u128 c = member_code(keys, kst, dims, rec, (uint64_t)rec.start + 1 + jm);
          or_into(word, b0, c, at, sm);
          at += sm;
        }
        ++i;
      }
      s_w[w_end - 1 - wlo] = word;
    }
  }
  __syncthreads();
  for (uint64_t w = w_first + threadIdx.x; w < w_end; w += kBlock) pay[w] = s_w[w - wlo];
}

__device__ __forceinline__ void pack_payload(uint32_t nsets, const uint64_t* pre, uint64_t vb, const SetDesc* sets,
                             const DevParams* params, const LeafRec* leaves0, const uint64_t* off0,
                             const uint8_t* keys0, const uint8_t* keys1, LeafRec* s_rec, uint64_t* s_off,
                             unsigned long long* s_w) {
  const uint32_t s = wave_find_set(pre, nsets, vb);
  const SetDesc& S = sets[s];
  const DevParams* P = params + s;
  if (P->status != BBX_OK) return;
  if (P->payload_bits == 0) return;
  const uint64_t blk = vb - pre[s];
  const uint8_t* keys = (S.final_buf ? keys1 : keys0) + S.key_off;
  const LeafRec* leaves = leaves0 + S.leaf_off;
  const uint64_t* off = off0 + S.leaf_off;
  if (P->key16)
    pack_payload_body<uint16_t>(S, P, blk, leaves, off, (const uint16_t*)keys, s_rec, s_off, s_w);
  else
    pack_payload_body<uint32_t>(S, P, blk, leaves, off, (const uint32_t*)keys, s_rec, s_off, s_w);
}

__device__ void lossless_copy(const SetDesc& S, uint64_t lb, uint64_t nblk) {
  const uint64_t nv = S.n * S.dims, step = nblk * kBlock;
  uint8_t* pay = S.out + kHeaderBytes;
  if (S.dtype == BBX_F32) {
    const uint32_t* in = (const uint32_t*)S.pos;
    uint32_t* out = (uint32_t*)pay;
    for (uint64_t k = lb * kBlock + threadIdx.x; k < nv; k += step) {
      const uint64_t i = k / S.dims, d = k - i * S.dims;
      out[k] = S.layout == BBX_AOS ? in[k] : in[d * S.n + i];
    }
    if (lb == 0 && threadIdx.x == 0 && (nv & 1)) out[nv] = 0;  // zero padding to 8 bytes
  } else {
    const uint64_t* in = (const uint64_t*)S.pos;
    uint64_t* out = (uint64_t*)pay;
    for (uint64_t k = lb * kBlock + threadIdx.x; k < nv; k += step) {
      const uint64_t i = k / S.dims, d = k - i * S.dims;
      out[k] = S.layout == BBX_AOS ? in[k] : in[d * S.n + i];
    }
  }
  uint32_t* perm = seq_stream(S) ? S.user_perm : S.perm;
  if (perm)
    for (uint64_t i = lb * kBlock + threadIdx.x; i < S.n; i += step) perm[i] = (uint32_t)i;
}

// The sets stored losslessly (listed by set_sizes): their coordinates'
// bits, particle by particle in input order (x, y, z), M bits each,
// zero-padded to 8 bytes; perm is the identity.  A fixed number of blocks
// shares each listed set's copy; with no such set every one exits at once.
constexpr uint32_t kLosslessBlocks = 256;

__device__ inline void pack_lossless(uint64_t lb, const SetDesc* sets, const uint32_t* list) {
  const uint32_t count = list[0];
  for (uint32_t li = 0; li < count; ++li) lossless_copy(sets[list[1 + li]], lb, kLosslessBlocks);
}

// The meta words (g_pm blocks), and the lossless sets behind them.
__global__ void __launch_bounds__(kBlock) k_pack_meta(uint32_t nsets, const uint64_t* pre, uint64_t g_pm,
                                                      const SetDesc* sets, const DevParams* params,
                                                      const LeafRec* leaves0, const uint32_t* list) {
  if (blockIdx.x < g_pm)
    pack_meta(nsets, pre, blockIdx.x, sets, params, leaves0);
  else
    pack_lossless(blockIdx.x - g_pm, sets, list);
}

__global__ void __launch_bounds__(kBlock) k_pack_payload(uint32_t nsets, const uint64_t* pre,
                                                         const SetDesc* sets, const DevParams* params,
                                                         const LeafRec* leaves0, const uint64_t* off0,
                                                         const uint8_t* keys0, const uint8_t* keys1) {
  __shared__ LeafRec s_rec[kLeafStage];
  __shared__ uint64_t s_off[kLeafStage];
  __shared__ unsigned long long s_w[kPackLdsWords];
  pack_payload(nsets, pre, blockIdx.x, sets, params, leaves0, off0, keys0, keys1, s_rec, s_off, s_w);
}

// Both in one launch, for few payload blocks (up to kPackOnce): a launch
// costs such sets more than the payload's LDS takes from the meta words'
// occupancy.  With more blocks that is the other way round (fluid 2^27: 633
// us in one launch for 478 + 77 in two, which are 434 + 58 now).
constexpr uint64_t kPackOnce = 2048;
__global__ void __launch_bounds__(kBlock) k_pack(uint32_t nsets, const uint64_t* pre_pp, uint64_t g_pp,
                                                 const uint64_t* pre_pm, uint64_t g_pm, const SetDesc* sets,
                                                 const DevParams* params, const LeafRec* leaves0,
                                                 const uint64_t* off0, const uint8_t* keys0,
                                                 const uint8_t* keys1, const uint32_t* list) {
  __shared__ LeafRec s_rec[kLeafStage];
  __shared__ uint64_t s_off[kLeafStage];
  __shared__ unsigned long long s_w[kPackLdsWords];
  const uint64_t b = blockIdx.x;
  if (b < g_pp)
    pack_payload(nsets, pre_pp, b, sets, params, leaves0, off0, keys0, keys1, s_rec, s_off, s_w);
  else if (b < g_pp + g_pm)
    pack_meta(nsets, pre_pm, b - g_pp, sets, params, leaves0);
  else
    pack_lossless(b - g_pp - g_pm, sets, list);
}

hipError_t launch_pack(const BatchPlan& bp, const Ws& w, hipStream_t s) {
  if (bp.total_leaves <= kScanOne) {
    BBX_LAUNCH("scan_sizes", k_scan_sizes, 1, kScanThreads, 0, s, bp.nsets, w.sets, w.params, bp.total_leaves,
               w.leaf_bits, w.lossless);
  } else {
    const hipError_t e = scan_launch(bp.total_leaves, w.leaf_bits, w.scan_part, w.scan_total, nullptr, 0, s);
    if (e != hipSuccess) return e;
    BBX_LAUNCH("set_sizes", k_set_sizes, (bp.nsets + 63) / 64, 64, 0, s, bp.nsets, w.sets, w.params,
               w.leaf_bits, bp.total_leaves, w.scan_total, w.lossless);
  }
  if (bp.g_pp <= kPackOnce) {
    BBX_LAUNCH("pack_payload", k_pack, bp.g_pp + bp.g_pm + kLosslessBlocks, kBlock, 0, s, bp.nsets,
               w.pre + bp.o_pp, bp.g_pp, w.pre + bp.o_pm, bp.g_pm, w.sets, w.params, w.leaves, w.leaf_bits,
               w.keys[0], w.keys[1], w.lossless);
  } else {
    BBX_LAUNCH("pack_meta", k_pack_meta, bp.g_pm + kLosslessBlocks, kBlock, 0, s, bp.nsets, w.pre + bp.o_pm,
               bp.g_pm, w.sets, w.params, w.leaves, w.lossless);
    BBX_LAUNCH("pack_payload", k_pack_payload, bp.g_pp, kBlock, 0, s, bp.nsets, w.pre + bp.o_pp, w.sets,
               w.params, w.leaves, w.leaf_bits, w.keys[0], w.keys[1]);
  }
  return launch_reduce_pack(bp, w, s);
}

}  // namespace bbx
