// k_reorder.hip -- the two reorderings of Sec. 4.2 applied to the sequence
// layout (bbx_export_sequences) before entropy coding: sequences in
// ascending sum of widths (stable: equal sums keep leaf order), and in each
// sequence the members in ascending R-index, the members' codes concatenated
// with the axes in ascending entropy of their width distributions (first
// axis most significant), equal R-indices in stored order.  A sequence keeps
// its centre, widths and end mark; its members keep their codes.
//
// From the stream itself (every leaf's record and payload offset are in the
// decompression workspace by then):
//   k_ro_hist    per leaf: its widths into per-axis histograms, its key
//                (the sum of widths) and its counts per block of leaves
//   (host: the axis order from the width histograms)
//   k_ro_scan    one block: exclusive scan of the (key, block) counts, key
//                major, so that a key's leaves follow the smaller keys' in
//                block order
//   k_ro_place   per leaf: its place in the new order (its key's base for its
//                block plus the leaves of the block before it with its key);
//                the leaf at each place and that leaf's payload bits there
//   (scan of the placed payload bits: each sequence's new offset)
//   k_ro_write   SUB lanes per sequence of at most SUB other members: centre
//                and widths copied, members ranked by (R-index, stored
//                position), their codes written in that order, the end mark
//   k_ro_long    a wavefront per sequence, for larger leaves
//   Both OR the words into the zeroed output (sequences share boundary words).
#include "bbx_internal.h"

namespace bbx {

typedef unsigned __int128 u128;

constexpr uint32_t kRoKeys = 94;        // sums of widths 0 .. 3 * 31
// counts per key: one per block of leaves, an even number (94 keys: a multiple of
// four entries in all)
__host__ __device__ inline uint64_t ro_stride(uint64_t blocks) { return (blocks + 1) & ~1ull; }
constexpr uint32_t kRoLocal = 256;      // members ranked from LDS (more: from the stream)
constexpr uint32_t kRoStage = 64;       // words of a sequence staged in LDS (longer: written in place)

__device__ inline uint64_t ro_read(const uint64_t* sec, uint64_t nwords, uint64_t at, uint32_t len) {
  if (len == 0) return 0;
  const uint64_t w = at >> 6;
  const uint32_t s = (uint32_t)(at & 63);
  uint64_t v = w < nwords ? sec[w] >> s : 0ull;
  if (s && s + len > 64 && w + 1 < nwords) v |= sec[w + 1] << (64 - s);
  return len < 64 ? v & ((1ull << len) - 1) : v;
}

__device__ inline void ro_write(unsigned long long* sec, uint64_t at, uint64_t v, uint32_t len) {
  if (len == 0) return;
  if (len < 64) v &= (1ull << len) - 1;
  const uint64_t w = at >> 6;
  const uint32_t s = (uint32_t)(at & 63);
  if (v == 0) return;
  atomicOr(&sec[w], (unsigned long long)(v << s));
  if (s && s + len > 64) atomicOr(&sec[w + 1], (unsigned long long)(v >> (64 - s)));
}

__global__ void __launch_bounds__(kBlock) k_ro_hist(uint64_t n_leaves, uint32_t dims,
                                                    const LeafRec* leaves, uint32_t* whist,
                                                    uint8_t* key, uint32_t* bcount,
                                                    const DevParams* P) {
  if (P->status != BBX_OK) return;
  __shared__ uint32_t kc[kRoKeys];
  __shared__ uint32_t wh[3 * 64];  // the block's width counts, added to the device's once
  for (uint32_t k = threadIdx.x; k < kRoKeys; k += kBlock) kc[k] = 0;
  for (uint32_t k = threadIdx.x; k < 3 * 64; k += kBlock) wh[k] = 0;
  __syncthreads();
  const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n_leaves) {
    const uint32_t m = leaves[i].m;
    uint32_t sm = 0;
    for (uint32_t d = 0; d < dims; ++d) {
      const uint32_t md = (m >> (8 * d)) & 0xffu;
      atomicAdd(&wh[d * 64 + (md & 63)], 1u);
      sm += md;
    }
    key[i] = (uint8_t)sm;
    atomicAdd(&kc[sm < kRoKeys ? sm : kRoKeys - 1], 1u);
  }
  __syncthreads();
  for (uint32_t k = threadIdx.x; k < 3 * 64; k += kBlock)
    if (wh[k]) atomicAdd(&whist[k], wh[k]);
  const uint64_t nblk = ro_stride(gridDim.x);
  for (uint32_t k = threadIdx.x; k < kRoKeys; k += kBlock) {
    bcount[(uint64_t)k * nblk + blockIdx.x] = kc[k];
    if (blockIdx.x == gridDim.x - 1)  // the blocks that are not there
      for (uint64_t b = gridDim.x; b < nblk; ++b) bcount[(uint64_t)k * nblk + b] = 0;
  }
}

// one block: exclusive scan of counts[key][block], key major; 16 entries per
// thread and round (entries is a multiple of 4, c of 16 bytes: one entry per
// thread and round took 178 us for the 192,512 entries of 524,288 leaves, this
// takes 46)
__global__ void __launch_bounds__(1024) k_ro_scan(uint32_t* c, uint64_t entries, const DevParams* P) {
  if (P->status != BBX_OK) return;
  __shared__ uint32_t ws[2][16];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint4* const c4 = (uint4*)c;
  const uint64_t quads = entries / 4;
  uint32_t run = 0, buf = 0;
  for (uint64_t q0 = 0; q0 < quads; q0 += 4 * 1024, buf ^= 1) {
    const uint64_t q = q0 + 4 * threadIdx.x;
    uint4 v[4];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = q + k < quads ? c4[q + k] : make_uint4(0, 0, 0, 0);
      sum += v[k].x + v[k].y + v[k].z + v[k].w;
    }
    const uint32_t incl = wave_incl(sum);
    if (lane == 63) ws[buf][wv] = incl;
    __syncthreads();
    uint32_t at = run + incl - sum, tot = 0;
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k) {
      at += k < wv ? ws[buf][k] : 0u;
      tot += ws[buf][k];
    }
    run += tot;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint4 o;
      o.x = at, o.y = o.x + v[k].x, o.z = o.y + v[k].y, o.w = o.z + v[k].z;
      at = o.w + v[k].w;
      if (q + k < quads) c4[q + k] = o;
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_ro_place(uint64_t n_leaves, const uint8_t* key,
                                                     const uint32_t* base, const LeafRec* leaves,
                                                     uint32_t* order, uint64_t* sbits,
                                                     const DevParams* P) {
  if (P->status != BBX_OK) return;
  __shared__ uint8_t kl[kBlock];
  const uint64_t i0 = (uint64_t)blockIdx.x * kBlock, i = i0 + threadIdx.x;
  const bool ok = i < n_leaves;
  kl[threadIdx.x] = ok ? key[i] : 0xffu;
  __syncthreads();
  if (!ok) return;
  const uint32_t k = kl[threadIdx.x];
  uint32_t before = 0;
  for (uint32_t t = 0; t < threadIdx.x; ++t) before += kl[t] == k ? 1u : 0u;
  const uint64_t q = base[(uint64_t)k * ro_stride(gridDim.x) + blockIdx.x] + before;
  const uint32_t m = leaves[i].m;
  const uint32_t sm = (m & 0xffu) + ((m >> 8) & 0xffu) + ((m >> 16) & 0xffu);
  order[q] = (uint32_t)i;
  sbits[q] = (uint64_t)(leaves[i].size - 1) * sm;
}

__global__ void __launch_bounds__(kBlock) k_ro_zero(uint64_t* p, uint64_t words, const DevParams* P) {
  if (P->status != BBX_OK) return;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < words;
       i += (uint64_t)gridDim.x * kBlock)
    p[i] = 0;
}

// value t of a 3-array held in registers (no dynamic indexing)
template <typename T>
__device__ inline T ro_pick(const T (&v)[3], uint32_t t) {
  return t == 0 ? v[0] : (t == 1 ? v[1] : v[2]);
}

// What the writing kernels read and write.
struct RoView {
  uint64_t n_leaves;
  const LeafRec* leaves;
  const uint64_t* poff;   // a leaf's first payload bit
  const uint32_t* order;  // leaf of each sequence
  const uint64_t* soff;   // code bits before each sequence
  const uint64_t* meta;
  const uint64_t* pay;
  uint64_t mwords, pwords;
  unsigned long long* out;
  uint32_t dims, M, mbits, ord[3];
};

// A member's code bits: its axes' codes in axis order, sm of them (at most 93).
__device__ inline u128 ro_code(const RoView& v, uint64_t at, uint32_t sm) {
  u128 c = ro_read(v.pay, v.pwords, at, sm < 64 ? sm : 64);
  if (sm > 64) c |= (u128)ro_read(v.pay, v.pwords, at + 64, sm - 64) << 64;
  return c;
}
// Its R-index: the axes' codes with ord[0] most significant.
template <typename T>
__device__ inline T ro_rindex(const RoView& v, T c, const uint32_t (&m)[3]) {
  const T f[3] = {c & (((T)1 << m[0]) - 1), (c >> m[0]) & (((T)1 << m[1]) - 1),
                  (c >> (m[0] + m[1])) & (((T)1 << m[2]) - 1)};
  T r = 0;
#pragma unroll
  for (uint32_t k = 0; k < 3; ++k)
    if (k < v.dims) r = (r << ro_pick(m, v.ord[k])) | ro_pick(f, v.ord[k]);
  return r;
}
__device__ inline void ro_write128(unsigned long long* sec, uint64_t at, u128 c, uint32_t len) {
  ro_write(sec, at, (uint64_t)c, len < 64 ? len : 64);
  if (len > 64) ro_write(sec, at + 64, (uint64_t)(c >> 64), len - 64);
}

// Centre and widths of leaf i at bit `at` of dst: lane k of at least 8 takes
// 32 bits of the centre, the lane after the last of them the widths.
__device__ inline void ro_header(const RoView& v, uint64_t i, unsigned long long* dst, uint64_t at, uint32_t k) {
  const uint32_t cw = v.dims * v.M / 32, rec = v.dims * (v.mbits + v.M), wb = v.dims * v.mbits;
  if (k < cw)
    ro_write(dst, at + 32 * k, ro_read(v.meta, v.mwords, i * rec + wb + 32 * k, 32), 32);
  else if (k == cw)
    ro_write(dst, at + 32 * cw, ro_read(v.meta, v.mwords, i * rec, wb), wb);
}

// SUB lanes per sequence, one per member besides the reference (at most SUB).
// A member's codes are read once, as one bit string; its rank is the number
// of smaller (R-index, position) keys among the sequence's, which all fit one
// word with the position (R-indices of up to 58 bits; longer ones compare as
// two words).  The sequence is put together in LDS, so that only its two
// boundary words need atomics.  A wavefront per sequence with 128-bit keys
// read from a plain layout written before took 929 us (and that layout 140)
// for the cosmology 2^24 set's 524,288 sequences; this takes 296.  Bound
// by instruction issue (SUB comparisons per lane).
template <int SUB>
__global__ void __launch_bounds__(kBlock) k_ro_write(RoView v, const DevParams* P) {
  if (P->status != BBX_OK) return;
  constexpr uint32_t NS = 64 / SUB;                             // sequences per wavefront
  constexpr uint32_t WORDS = (63 + 242 + 93 * SUB + 63) / 64;   // words of a sequence at most
  __shared__ __align__(16) uint64_t keys[kBlock / 64][64];
  __shared__ uint64_t high[kBlock / 64][64];
  __shared__ unsigned long long stage[kBlock / 64][NS][WORDS];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t sub = lane / SUB, k = lane % SUB;
  const uint32_t F = v.dims * (v.M + v.mbits) + 32, hdr = F - 32;  // bits besides the codes
  const uint64_t q = ((uint64_t)blockIdx.x * (kBlock / 64) + wv) * NS + sub;
  const bool valid = q < v.n_leaves;
  uint64_t i = 0, op = 0, at = 0;
  uint32_t m[3] = {0, 0, 0}, sm = 0, cnt = 0, nwd = 0;
  unsigned long long* const st = stage[wv][sub];
  if (valid) {
    i = v.order[q];
    const uint32_t mp = v.leaves[i].m;
    m[0] = mp & 0xffu, m[1] = (mp >> 8) & 0xffu, m[2] = (mp >> 16) & 0xffu;
    sm = m[0] + m[1] + m[2];
    cnt = v.leaves[i].size - 1;
    op = q * F + v.soff[q];
    at = v.poff[i];
    nwd = (uint32_t)(((op & 63) + F + (uint64_t)cnt * sm + 63) >> 6);
    if (cnt > SUB) cnt = SUB;  // (never: the launch is chosen by the leaf size)
    if (nwd > WORDS) nwd = WORDS;
  }
  for (uint32_t x = k; x < nwd; x += SUB) st[x] = 0;
  const bool mine = k < cnt && sm > 0;
  const uint64_t o0 = op & 63, c0 = o0 + hdr;  // the sequence's first bit, and its first code's, in the stage
  uint32_t rank = 0;
  if (__ballot(sm > 58) == 0) {
    const uint64_t code = mine ? ro_read(v.pay, v.pwords, at + (uint64_t)k * sm, sm) : 0ull;
    const uint64_t own = mine ? ro_rindex<uint64_t>(v, code, m) << 6 | k : ~0ull;
    keys[wv][lane] = own;
    wave_sync();
    const ulonglong2* o = (const ulonglong2*)&keys[wv][sub * SUB];
#pragma unroll 4
    for (uint32_t t = 0; t < SUB / 2; ++t) {
      const ulonglong2 x = o[t];
      rank += (x.x < own ? 1u : 0u) + (x.y < own ? 1u : 0u);
    }
    if (mine) ro_write(st, c0 + (uint64_t)rank * sm, code, sm);
  } else {
    const u128 code = mine ? ro_code(v, at + (uint64_t)k * sm, sm) : (u128)0;
    const u128 r = mine ? ro_rindex<u128>(v, code, m) : ~(u128)0;
    keys[wv][lane] = (uint64_t)r;
    high[wv][lane] = (uint64_t)(r >> 64);
    wave_sync();
    for (uint32_t t = 0; t < SUB; ++t) {
      const u128 x = (u128)high[wv][sub * SUB + t] << 64 | keys[wv][sub * SUB + t];
      rank += x < r || (x == r && t < k) ? 1u : 0u;
    }
    if (mine) ro_write128(st, c0 + (uint64_t)rank * sm, code, sm);
  }
  if (valid) {
    ro_header(v, i, st, o0, k);
    if (k == 0) ro_write(st, c0 + (uint64_t)cnt * sm, 0xffffffffull, 32);  // end mark
  }
  wave_sync();
  for (uint32_t x = k; x < nwd; x += SUB) {
    unsigned long long* const d = v.out + (op >> 6) + x;
    if (x == 0 || x + 1 == nwd)
      atomicOr(d, st[x]);
    else
      *d = st[x];
  }
}

// A wavefront per sequence of any size: up to 256 other members are ranked by
// keys in LDS, of one word up to R-indices of 56 bits (a position takes 8);
// longer sequences read their codes again for every comparison.  Bound by the
// comparisons: 30,000,001 particles in 2-D, 262,144 leaves of 114 and 115, 617
// us (2,291 with two-word keys whatever the R-index); 13,000,001 in 3-D, 32,768
// leaves of 396 and 397, 19.9 ms.
__global__ void __launch_bounds__(kBlock) k_ro_long(RoView v, const DevParams* P) {
  if (P->status != BBX_OK) return;
  __shared__ u128 rk[kBlock / 64][kRoLocal];
  __shared__ unsigned long long stg[kBlock / 64][kRoStage];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t hdr = v.dims * (v.M + v.mbits);
  const uint64_t F = (uint64_t)hdr + 32;  // a sequence's bits besides its codes
  const uint64_t gw = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
  const uint64_t nw = ((uint64_t)gridDim.x * kBlock) >> 6;
  for (uint64_t q = gw; q < v.n_leaves; q += nw) {
    const uint32_t i = v.order[q];
    const LeafRec L = v.leaves[i];
    const uint64_t cin = v.poff[i], op = q * F + v.soff[q];
    const uint32_t m[3] = {L.m & 0xffu, (L.m >> 8) & 0xffu, (L.m >> 16) & 0xffu};
    const uint32_t sm = m[0] + m[1] + m[2];
    const uint32_t cnt = L.size - 1;
    // the sequence's words: staged in LDS when few (then only the two
    // boundary words, shared with the neighbours, need atomics), else ORed
    // into the output in place
    const uint64_t w0 = op >> 6, nwd = ((op + F + (uint64_t)cnt * sm - 1) >> 6) - w0 + 1;
    const bool staged = nwd <= kRoStage;
    unsigned long long* dst = staged ? stg[wv] : v.out;
    const uint64_t dbase = staged ? w0 * 64 : 0;  // bit offset of dst[0] in the output
    if (staged) {
      for (uint32_t k = lane; k < kRoStage; k += 64) stg[wv][k] = 0;
      wave_sync();
    }
    ro_header(v, i, dst, op - dbase, lane);
    const uint64_t cout = op + hdr - dbase;
    if (sm > 0 && cnt > 0) {
      auto rindex = [&](uint32_t j) { return ro_rindex<u128>(v, ro_code(v, cin + (uint64_t)j * sm, sm), m); };
      // the members' codes, in axis order, at their ranks by key(j)
      auto place = [&](auto&& key) {
        for (uint32_t j = lane; j < cnt; j += 64) {
          const u128 kj = key(j);
          uint32_t rank = 0;
          for (uint32_t t = 0; t < cnt; ++t) {
            const u128 kt = key(t);
            rank += (kt < kj || (kt == kj && t < j)) ? 1u : 0u;
          }
          ro_write128(dst, cout + (uint64_t)rank * sm, ro_code(v, cin + (uint64_t)j * sm, sm), sm);
        }
      };
      if (cnt <= kRoLocal && sm <= 56) {  // (R-index, position) in one word
        uint64_t* const keys = (uint64_t*)rk[wv];
        for (uint32_t j = lane; j < ((cnt + 1) & ~1u); j += 64)
          keys[j] = j < cnt ? ro_rindex<uint64_t>(v, ro_read(v.pay, v.pwords, cin + (uint64_t)j * sm, sm), m) << 8 | j
                            : ~0ull;
        wave_sync();
        const ulonglong2* const o = (const ulonglong2*)keys;
        for (uint32_t j = lane; j < cnt; j += 64) {
          const uint64_t own = keys[j];
          uint32_t rank = 0;
#pragma unroll 4
          for (uint32_t t = 0; t < (cnt + 1) / 2; ++t) {
            const ulonglong2 x = o[t];
            rank += (x.x < own ? 1u : 0u) + (x.y < own ? 1u : 0u);
          }
          ro_write(dst, cout + (uint64_t)rank * sm, ro_read(v.pay, v.pwords, cin + (uint64_t)j * sm, sm), sm);
        }
      } else if (cnt <= kRoLocal) {
        for (uint32_t j = lane; j < cnt; j += 64) rk[wv][j] = rindex(j);
        wave_sync();
        place([&](uint32_t j) { return rk[wv][j]; });
      } else {
        place(rindex);
      }
      wave_sync();  // rk is rewritten by the wavefront's next sequence
    }
    if (lane == 0) ro_write(dst, cout + (uint64_t)cnt * sm, 0xffffffffull, 32);  // end mark
    if (staged) {
      wave_sync();
      for (uint32_t k = lane; k < nwd; k += 64) {
        const unsigned long long x = stg[wv][k];
        if (k == 0 || k + 1 == nwd)
          atomicOr(&v.out[w0 + k], x);
        else
          v.out[w0 + k] = x;
      }
      wave_sync();  // stg is rewritten by the wavefront's next sequence
    }
  }
}

hipError_t launch_reorder_hist(uint64_t n_leaves, uint32_t dims, const DecompressWs& w,
                               uint32_t* whist, uint8_t* key, uint32_t* bcount, hipStream_t s) {
  const uint64_t nblk = (n_leaves + kBlock - 1) / kBlock;
  if (nblk > 0)
    BBX_LAUNCH("reorder_hist", k_ro_hist, nblk, kBlock, 0, s, n_leaves, dims, w.leaves, whist, key,
               bcount, w.params);
  return hipGetLastError();
}

template <int SUB>
static void launch_ro_write(const RoView& v, const DevParams* P, hipStream_t s) {
  constexpr uint32_t per = kBlock / SUB;  // sequences per block
  BBX_LAUNCH("reorder_write", k_ro_write<SUB>, (uint32_t)((v.n_leaves + per - 1) / per), kBlock, 0, s, v, P);
}

hipError_t launch_reorder_write(const DecompressPlan& p, const DecompressWs& w, const uint32_t ord[3],
                                const uint8_t* stream, uint8_t* out, uint64_t out_words, uint8_t* key,
                                uint32_t* bcount, uint32_t* order, uint64_t* sbits, hipStream_t s) {
  const uint64_t nl = p.n_leaves, nblk = (nl + kBlock - 1) / kBlock;
  if (nl == 0) return hipGetLastError();
  BBX_LAUNCH("reorder_scan", k_ro_scan, 1, 1024, 0, s, bcount, (uint64_t)kRoKeys * ro_stride(nblk), w.params);
  BBX_LAUNCH("reorder_place", k_ro_place, nblk, kBlock, 0, s, nl, key, bcount, w.leaves, order, sbits,
             w.params);
  hipError_t e = launch_dec_scan(nl, sbits, w.scan_part, w.params, p.payload_bits, s);
  if (e != hipSuccess) return e;
  BBX_LAUNCH("reorder_zero", k_ro_zero, (uint32_t)std::min<uint64_t>(out_words / kBlock + 1, 4096), kBlock, 0,
             s, (uint64_t*)out, out_words, w.params);
  RoView v;
  v.n_leaves = nl;
  v.leaves = w.leaves;
  v.poff = w.leaf_bits;
  v.order = order;
  v.soff = sbits;
  v.mwords = (p.meta_bits + 63) / 64;
  v.pwords = (p.payload_bits + 63) / 64;
  v.meta = (const uint64_t*)(stream + kHeaderBytes);
  v.pay = v.meta + v.mwords;
  v.out = (unsigned long long*)out;
  v.dims = p.dims;
  v.M = coord_bits(p.dtype);
  v.mbits = p.mbits;
  for (int d = 0; d < 3; ++d) v.ord[d] = ord[d];
  // as many lanes per sequence as a leaf can have members besides its
  // reference, at least the header's 8
  if (p.r <= 9)
    launch_ro_write<8>(v, w.params, s);
  else if (p.r <= 17)
    launch_ro_write<16>(v, w.params, s);
  else if (p.r <= 33)
    launch_ro_write<32>(v, w.params, s);
  else if (p.r <= 65)
    launch_ro_write<64>(v, w.params, s);
  else
    BBX_LAUNCH("reorder_write", k_ro_long, (uint32_t)std::min<uint64_t>((nl + 3) / 4, 65536), kBlock, 0, s, v,
               w.params);
  return hipGetLastError();
}

}  // namespace bbx
