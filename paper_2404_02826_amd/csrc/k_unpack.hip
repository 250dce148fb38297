// k_unpack.hip -- unpack and dequantize (Sec. 3: reconstruction at the bin
// centre origin + q*w, FP64 multiply then add, then rounding to the type).
//
//   k_dec_sums   payload bits of each unpack block: a thread per leaf reads
//                and checks its record (widths, with ref_mode 1 the reference's
//                coordinates); its span follows from (n, r) alone (the tree's
//                leaf sizes depend on n and r only)
//   k_dec_top    (up to kDecTop blocks, else k_dec_init and the scan kernels)
//                their exclusive scan, total checked against the header
//   k_unpack     a block takes leaves_per_block(r) leaves: their records, a
//                scan of their payload bits, the payload words into LDS, then
//                every thread decodes slots (reference -> its code; member j
//                -> payload code j-1); with ref_mode 1 the reference's code
//                comes from its stored coordinate by the quantization of
//                Sec. 3, and its slot gets the coordinate itself
//   k_dec_meta   one thread per leaf: its record, span and payload bits, for
//                the export of the sequence layout
//   k_export     the Sec. 4.2 sequence layout of a ref_mode 1 stream (with
//                k_dec_meta and the scan for the leaves' code offsets)
#include <type_traits>

#include "bbx_internal.h"

namespace bbx {

typedef unsigned __int128 u128;

__device__ inline u128 read_bits(const uint64_t* sec, uint64_t nwords, uint64_t at, uint32_t len) {
  if (len == 0) return 0;
  const uint64_t w0 = at >> 6;
  const uint32_t s = (uint32_t)(at & 63);
  u128 v = (u128)sec[w0];
  if (w0 + 1 < nwords) v |= (u128)sec[w0 + 1] << 64;
  v >>= s;
  if (s + len > 128 && w0 + 2 < nwords) v |= (u128)sec[w0 + 2] << (128 - s);
  if (len < 128) v &= (((u128)1) << len) - 1;
  return v;
}

// Reference field of a ref_mode 1 record: the stored coordinate of axis d
// (M bits at absolute bit `at`), and the code the encoder's quantization gave
// it: floor((x - origin) * inv_w + 1/2) in FP64, the same separately rounded
// operations as the quantize pass (no contraction).  Returns false when the
// value is not finite or its code lies outside [0, 2^G).
__device__ inline bool ref_code_from_coord(const uint64_t* meta, uint64_t nwords, uint64_t at,
                                           uint32_t dtype, double origin, double inv_w,
                                           uint32_t G, uint32_t* q) {
  const uint64_t raw = (uint64_t)read_bits(meta, nwords, at, coord_bits(dtype));
  const double x = dtype == BBX_F32 ? (double)__uint_as_float((uint32_t)raw) : __longlong_as_double((long long)raw);
  if (!isfinite(x)) return false;
  const double t = floor((x - origin) * inv_w + 0.5);
  if (!(t >= 0.0 && t < (double)(1ull << G))) return false;
  *q = (uint32_t)t;
  return true;
}

__global__ void __launch_bounds__(kBlock) k_dec_meta(uint64_t n_leaves, uint32_t dims,
                                                     uint32_t mbits, uint32_t G0, uint32_t G1,
                                                     uint32_t G2, uint64_t meta_bits, TreeGeom g,
                                                     const uint8_t* stream, LeafRec* leaves,
                                                     uint64_t* bits, DevParams* P,
                                                     uint32_t ref_mode, uint32_t dtype, double o0,
                                                     double o1, double o2, double inv_w) {
  const uint32_t G[3] = {G0, G1, G2};
  const double origin[3] = {o0, o1, o2};
  uint32_t S = dims * mbits;
  for (uint32_t d = 0; d < dims; ++d) S += ref_mode ? coord_bits(dtype) : G[d];
  const uint64_t* meta = (const uint64_t*)(stream + kHeaderBytes);
  const uint64_t nwords = (meta_bits + 63) / 64;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_leaves;
       i += (uint64_t)gridDim.x * blockDim.x) {
    // widths (and with ref_mode 0 the reference codes) in one read: at most
    // 3 * (6 + 30) bits
    u128 v = read_bits(meta, nwords, i * S, ref_mode ? dims * mbits : S);
    LeafRec rec;
    uint32_t m = 0, summ = 0;
    bool bad = false;
    for (uint32_t d = 0; d < dims; ++d) {
      uint32_t md = (uint32_t)(v & ((1u << mbits) - 1));
      v >>= mbits;
      if (md == 1 || md > 31 || md > G[d] + 1) bad = true;
      m |= md << (8 * d);
      summ += md;
    }
    for (uint32_t d = 0; d < 3; ++d) {
      rec.qref[d] = 0;
      if (d < dims && ref_mode) {
        const uint64_t at = i * S + dims * mbits + d * coord_bits(dtype);
        if (!ref_code_from_coord(meta, nwords, at, dtype, origin[d], inv_w, G[d], &rec.qref[d]))
          bad = true;
      } else if (d < dims) {
        rec.qref[d] = (uint32_t)(v & ((((u128)1) << G[d]) - 1));
        v >>= G[d];
      }
    }
    rec.ref_src = 0;
    uint64_t st, sz;
    leaf_span(g, i, &st, &sz);
    rec.start = (uint32_t)st;
    rec.size = (uint32_t)sz;
    rec.m = m;
    leaves[i] = rec;
    bits[i] = bad ? 0 : (sz - 1) * (uint64_t)summ;
    if (bad) P->status = BBX_ECORRUPT;
  }
}

constexpr uint32_t kLeafStage = 256;     // leaves per block (leaves_per_block)
constexpr uint32_t kUnpackWords = 1534;  // staged payload words per block (+2 zero words: 12 KB)
constexpr uint32_t kMapGroups = 520;     // 4-slot groups of a block's leaf map (2,048 slots and the ends)

// What the decoding kernels need of a stream's meta section and tree.
struct MetaView {
  uint64_t n_leaves, meta_bits;
  TreeGeom g;
  double origin[3], w, inv_w;
  uint32_t G[3], dims, mbits, dtype, ref_mode, r;
  uint32_t even;  // particles per leaf when there are 2^k leaves that all hold as many (0: not so)
};

__device__ inline uint32_t record_bits(const MetaView& v) {
  const uint32_t M = coord_bits(v.dtype);
  uint32_t S = 0;
#pragma unroll
  for (uint32_t d = 0; d < 3; ++d)
    if (d < v.dims) S += v.mbits + (v.ref_mode ? M : v.G[d]);
  return S;
}
__device__ inline void view_span(const MetaView& v, uint64_t i, uint64_t* st, uint64_t* sz) {
  if (v.even) {
    *st = i * v.even;
    *sz = v.even;
  } else {
    leaf_span(v.g, i, st, sz);
  }
}
// The widths of record i (packed m_x | m_y << 8 | m_z << 16); false when one
// cannot be a width.
__device__ inline bool record_widths(const MetaView& v, u128 bits, uint32_t* m, uint32_t* sum) {
  bool ok = true;
  *m = *sum = 0;
#pragma unroll
  for (uint32_t d = 0; d < 3; ++d) {
    if (d >= v.dims) break;
    const uint32_t md = (uint32_t)bits & ((1u << v.mbits) - 1);
    bits >>= v.mbits;
    if (md == 1 || md > 31 || md > v.G[d] + 1) ok = false;
    *m |= md << (8 * d);
    *sum += md;
  }
  return ok;
}

// Payload bits of each unpack block (leaves_per_block leaves), a thread per
// leaf.  A record with a bad width or a reference coordinate outside the grid
// makes the stream corrupt before anything is decoded: reported in P,
// or (P null) as a total of all ones for k_dec_top.  starts: each leaf's first
// slot, when the leaves are not all equal.  (Where the threads of k_unpack
// walked the tree for their leaves' spans, some twenty levels each, their
// blocks waited for them: 67,108,941 particles at r = 128 470 us a decode and
// 385 with the starts from here, 100,000,007 in 2-D 614 and 441.)
__global__ void __launch_bounds__(kBlock) k_dec_sums(MetaView v, const uint8_t* stream, uint64_t blocks,
                                                     uint64_t* part, uint32_t* starts, DevParams* P) {
  __shared__ unsigned long long sum[kBlock];
  __shared__ uint32_t bad[kBlock];
  const uint32_t lpb = leaves_per_block(v.r), nbk = kBlock / lpb;  // unpack blocks per block
  sum[threadIdx.x] = 0;
  bad[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t i = (uint64_t)blockIdx.x * nbk * lpb + threadIdx.x;
  const uint32_t x = threadIdx.x / lpb;
  if (x < nbk && i < v.n_leaves) {
    const uint64_t* meta = (const uint64_t*)(stream + kHeaderBytes);
    const u128 bits = read_bits(meta, (v.meta_bits + 63) / 64, i * record_bits(v), v.dims * v.mbits);
    uint32_t m, summ;
    bool ok = record_widths(v, bits, &m, &summ);
    if (v.ref_mode) {
#pragma unroll
      for (uint32_t d = 0; d < 3; ++d) {
        if (d >= v.dims) break;
        const uint64_t at = i * record_bits(v) + v.dims * v.mbits + d * coord_bits(v.dtype);
        uint32_t q;
        ok &= ref_code_from_coord(meta, (v.meta_bits + 63) / 64, at, v.dtype, v.origin[d], v.inv_w, v.G[d], &q);
      }
    }
    uint64_t st, sz;
    view_span(v, i, &st, &sz);
    if (!v.even) starts[i] = (uint32_t)st;
    if (ok)
      atomicAdd(&sum[x], (unsigned long long)((sz - 1) * summ));
    else
      bad[x] = 1;
  }
  __syncthreads();
  const uint64_t b = (uint64_t)blockIdx.x * nbk + threadIdx.x;
  if (threadIdx.x < nbk && b < blocks) {
    part[b] = bad[threadIdx.x] && !P ? ~0ull : (uint64_t)sum[threadIdx.x];
    if (bad[threadIdx.x] && P) P->status = BBX_ECORRUPT;
  }
}

// For up to kDecTop unpack blocks: the start of a decode (the stream's own
// header against the one the launch was planned from), the exclusive scan of
// the blocks' payload bits, and its total against the header's, in one block.
constexpr uint64_t kDecTop = 16384;
__global__ void __launch_bounds__(1024) k_dec_top(uint64_t blocks, uint64_t* part, DevParams* P,
                                                  const uint8_t* stream, HeaderCopy h, uint64_t expect) {
  constexpr uint32_t W = 16;
  __shared__ uint64_t wsum[W];
  __shared__ uint32_t bad;
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  if (threadIdx.x < kHeaderBytes / 8 && ((const uint64_t*)stream)[threadIdx.x] != h.w[threadIdx.x]) bad = 1;
  const uint64_t per = (blocks + 1023) / 1024, b0 = threadIdx.x * per;
  uint64_t sum = 0;
  for (uint64_t k = b0; k < b0 + per && k < blocks; ++k) {
    const uint64_t x = part[k];
    if (x == ~0ull) bad = 1;
    sum += x;
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
  for (uint64_t k = b0; k < b0 + per && k < blocks; ++k) {
    const uint64_t c = part[k];
    part[k] = run;
    run += c;
  }
  if (threadIdx.x == 0) {
    P->status = bad || total != expect ? BBX_ECORRUPT : BBX_OK;
    P->damage = 0;
    P->payload_bits = total;
  }
}

// up to 64 bits at absolute bit `at` of a word array (the words exist)
__device__ inline uint64_t read64(const uint64_t* sec, uint64_t at, uint32_t len) {
  const uint64_t w = at >> 6;
  const uint32_t s = (uint32_t)(at & 63);
  uint64_t v = sec[w] >> s;
  if (s + len > 64) v |= sec[w + 1] << (64 - s);
  return len < 64 ? v & ((1ull << len) - 1) : v;
}

// The staged leaves of an unpack block.
struct UnpackStage {
  uint32_t start[kLeafStage + 1];  // first slot of each leaf (+ the end)
  uint32_t m[kLeafStage];          // widths
  uint32_t q[3][kLeafStage];       // reference codes
  uint64_t off[kLeafStage];        // first payload bit
  uint64_t pay[kUnpackWords + 2];
  uint64_t wsum[kBlock / 64];
  uint16_t map[kMapGroups];
};

// Leaf-aligned decoding: a block takes leaves_per_block(r) consecutive
// leaves, reads their meta records, scans their payload bits from the block's
// first one, stages the payload words with coalesced loads, and decodes the
// slots (reference -> its code; member j -> payload code j-1) from LDS.  The
// records are read here and not from a table that an earlier kernel wrote:
// 36 bytes per leaf written and read twice took the 2^27-particle set 160 us.
// Bound by instruction issue (about half of its time) beside the 14 bytes per
// particle it reads and writes: 2^27 particles in 575 us, the whole decode 764
// -> 638 us.  Non-temporal stores (594 for 602 then) and storing through LDS in
// lane order (615) change little.
template <typename T, int DIMS>
__device__ __forceinline__ void unpack_body(const MetaView& V, uint64_t n, uint32_t layout, const uint64_t* meta,
                                            const uint64_t* pay, uint64_t pbits, const uint64_t* part,
                                            const uint32_t* starts, T* out, DevParams* P, UnpackStage& sm) {
  constexpr uint32_t dims = DIMS;
  const uint32_t lpb = leaves_per_block(V.r);
  const uint64_t nl = V.n_leaves;
  const uint64_t L0 = (uint64_t)blockIdx.x * lpb;
  if (L0 >= nl) return;
  const uint32_t nlb = (uint32_t)(nl - L0 < lpb ? nl - L0 : lpb);
  const uint64_t mwords = (V.meta_bits + 63) / 64, pay_words = (pbits + 63) / 64;
  const uint64_t bo0 = part[blockIdx.x], bo1 = L0 + nlb < nl ? part[blockIdx.x + 1] : pbits;
  const uint32_t rb = record_bits(V);
  bool corrupt = false;
  {
    const uint32_t t = threadIdx.x;
    uint64_t bits = 0;
    if (t < nlb) {
      const uint64_t i = L0 + t;
      u128 v = read_bits(meta, mwords, i * rb, V.ref_mode ? dims * V.mbits : rb);
      uint32_t m, summ;
      if (!record_widths(V, v, &m, &summ)) m = summ = 0;  // (found before: not reached)
      v >>= dims * V.mbits;
#pragma unroll
      for (uint32_t d = 0; d < DIMS; ++d) {
        uint32_t q = 0;
        if (V.ref_mode) {
          const uint64_t at = i * rb + dims * V.mbits + d * coord_bits(V.dtype);
          (void)ref_code_from_coord(meta, mwords, at, V.dtype, V.origin[d], V.inv_w, V.G[d], &q);
        } else {
          q = (uint32_t)v & ((1u << V.G[d]) - 1);
          v >>= V.G[d];
        }
        sm.q[d][t] = q;
      }
      const uint32_t st = V.even ? (uint32_t)i * V.even : starts[i];
      const uint32_t en = V.even ? st + V.even : i + 1 < nl ? starts[i + 1] : (uint32_t)n;
      sm.start[t] = st;
      if (t == nlb - 1) sm.start[nlb] = en;
      sm.m[t] = m;
      bits = (uint64_t)(en - st - 1) * summ;
    }
    // exclusive scan over the block's leaves
    const uint32_t lane = t & 63, wv = t >> 6;
    uint64_t x = bits;
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t y = __shfl_up(x, o);
      if ((int)lane >= o) x += y;
    }
    if (lane == 63) sm.wsum[wv] = x;
    __syncthreads();
    uint64_t before = bo0;
#pragma unroll
    for (uint32_t k = 0; k < kBlock / 64; ++k) before += k < wv ? sm.wsum[k] : 0ull;
    if (t < nlb) sm.off[t] = before + x - bits;
  }
  // leaf map: the leaf holding the first slot of each 4-aligned group of
  // slots (each leaf writes the groups that start inside it), when the
  // block's slots fit the map
  const uint32_t slot0 = sm.start[0], slot1 = sm.start[nlb];
  const uint32_t mbase = slot0 & ~3u;
  const bool mapped = slot1 - mbase <= 4u * kMapGroups;
  if (mapped)
    for (uint32_t t = threadIdx.x; t < nlb; t += kBlock) {
      const uint32_t st = sm.start[t] - mbase, en = sm.start[t + 1] - mbase;
      for (uint32_t g = (st + 3) >> 2; 4 * g < en; ++g) sm.map[g] = (uint16_t)t;
    }
  const uint64_t w0 = bo0 / 64, w1 = bo1 > bo0 ? (bo1 + 63) / 64 : w0;
  const bool staged = w1 - w0 <= kUnpackWords;
  const uint32_t nw = staged ? (uint32_t)(w1 - w0) : 0u;
  for (uint32_t t = threadIdx.x; t < nw; t += kBlock) sm.pay[t] = w0 + t < pay_words ? pay[w0 + t] : 0;
  if (threadIdx.x < 2) sm.pay[nw + threadIdx.x] = 0;  // read past the end, then unused
  __syncthreads();
  // each thread decodes 4 consecutive slots (4-aligned slot indices); with an
  // aligned array-of-structures output the 4 particles go out as whole
  // 16-byte stores
  const bool vec = layout == BBX_AOS && ((uintptr_t)out & 15) == 0;
  // staged payload, 16-byte AoS stores, and every member within 64 code bits
  // (m_d <= G_d + 1, so sum_d (G_d + 1) <= 64 bounds every leaf): the four
  // slots of a thread decode without branches (below)
  uint32_t gsum = 0, top[3];
#pragma unroll
  for (uint32_t d = 0; d < DIMS; ++d) gsum += V.G[d] + 1, top[d] = 1u << V.G[d];
  const bool simple = staged && vec && gsum <= 64;
  const uint64_t bit0 = w0 * 64;  // staged bit offsets from here fit 32 bits
  // a code in the bin centre; q = q_ref + u - 2^(m-1), whose 32-bit value is
  // below 2^G exactly when q is in range (q_ref < 2^30, u < 2^31, 2^(m-1) <=
  // 2^30: a negative q wraps to 2^31 or more)
  auto centre = [&](uint32_t d, uint32_t q) {
    if (q >= top[d]) corrupt = true, q = 0;
    return (T)(V.origin[d] + (double)q * V.w);
  };
  const uint64_t end = slot1;
  for (uint64_t gs = mbase + 4ull * threadIdx.x; gs < end; gs += 4ull * kBlock) {
    const bool full = vec && gs >= slot0 && gs + 4 <= end;
    union {
      T e[4 * DIMS];
      uint4 v[4 * DIMS * sizeof(T) / 16];
    } o;
    const uint32_t pfirst = (uint32_t)(gs > slot0 ? gs : slot0);
    uint32_t a = 0;  // last staged leaf starting at or before pfirst
    if (mapped && gs >= slot0) {
      a = sm.map[((uint32_t)gs - mbase) >> 2];
    } else {
      uint32_t z = nlb - 1;
      while (a < z) {
        const uint32_t mid = (a + z + 1) >> 1;
        if (sm.start[mid] <= pfirst)
          a = mid;
        else
          z = mid - 1;
      }
    }
    if (simple && full) {
      // one slot of leaf (m, codes q, first bit `off` in the staged words): member j
      auto slot = [&](uint32_t k, uint32_t j, uint32_t off, const uint32_t (&mm)[3], uint32_t summ,
                      const uint32_t (&q)[3]) {
        // member j > 0 holds payload code j - 1; the reference reads a code
        // it does not use
        const uint32_t at = off + (j ? j - 1 : 0u) * summ;
        const uint32_t wi = at >> 6, sh = at & 63u;
        const uint64_t lo = sm.pay[wi], hi = sm.pay[wi + 1];
        uint64_t v = sh ? (lo >> sh) | (hi << (64 - sh)) : lo;
#pragma unroll
        for (uint32_t d = 0; d < DIMS; ++d) {
          const uint32_t u = (uint32_t)v & ((1u << mm[d]) - 1u);
          v >>= mm[d];
          if (j && mm[d] && !u) corrupt = true;
          o.e[k * DIMS + d] = centre(d, q[d] + (j ? u - ((1u << mm[d]) >> 1) : 0u));
        }
      };
      const uint32_t g0 = (uint32_t)gs;
      uint32_t mm[3], q[3] = {0, 0, 0}, summ = 0, off = 0, st = 0, en = 0;
      auto leaf = [&]() {
        const uint32_t m = sm.m[a];
#pragma unroll
        for (uint32_t d = 0; d < 3; ++d) mm[d] = d < DIMS ? (m >> (8 * d)) & 0xffu : 0u;
#pragma unroll
        for (uint32_t d = 0; d < DIMS; ++d) q[d] = sm.q[d][a];
        summ = mm[0] + mm[1] + mm[2];
        off = (uint32_t)(sm.off[a] - bit0);
        st = sm.start[a];
        en = sm.start[a + 1];
      };
      leaf();
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        if (k && g0 + k >= en) {  // the group runs into the next leaf (not in sets of equal leaves)
          while (g0 + k >= sm.start[a + 1]) ++a;
          leaf();
        }
        slot(k, g0 + k - st, off, mm, summ, q);
      }
    } else {
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint64_t p = gs + k;
        if (p < slot0 || p >= end) continue;
        while (a + 1 < nlb && sm.start[a + 1] <= p) ++a;
        const uint32_t j = (uint32_t)(p - sm.start[a]), m = sm.m[a];
        // widths (m_d <= 31: the meta check rejects wider); m_d = 0 gives a
        // zero mask and a zero offset, so such an axis keeps the reference code
        const uint32_t m0 = m & 0xffu, m1 = dims > 1 ? (m >> 8) & 0xffu : 0u,
                       m2 = dims > 2 ? (m >> 16) & 0xffu : 0u;
        const uint32_t summ = m0 + m1 + m2;
        uint32_t u[3] = {0, 0, 0};
        const uint32_t mm[3] = {m0, m1, m2};
        if (j > 0) {
          const uint64_t at = sm.off[a] + (uint64_t)(j - 1) * summ;
          if (summ <= 64) {
            const uint64_t v = staged ? read64(sm.pay, at - bit0, summ) : read64(pay, at, summ);
            u[0] = (uint32_t)v & ((1u << m0) - 1);
            u[1] = (uint32_t)(v >> m0) & ((1u << m1) - 1);
            u[2] = (uint32_t)(v >> (m0 + m1)) & ((1u << m2) - 1);
          } else {
            u128 v = staged ? read_bits(sm.pay, nw, at - bit0, summ) : read_bits(pay, pay_words, at, summ);
#pragma unroll
            for (uint32_t d = 0; d < 3; ++d) {
              u[d] = (uint32_t)(v & ((((u128)1) << mm[d]) - 1));
              v >>= mm[d];
            }
          }
#pragma unroll
          for (uint32_t d = 0; d < 3; ++d)
            if (d < dims && mm[d] != 0 && u[d] == 0) corrupt = true;
        }
#pragma unroll
        for (uint32_t d = 0; d < DIMS; ++d) {
          const T t = centre(d, sm.q[d][a] + (j > 0 ? u[d] - ((1u << mm[d]) >> 1) : 0u));
          if (full)
            o.e[k * dims + d] = t;
          else if (layout == BBX_AOS)
            out[p * dims + d] = t;
          else
            out[(uint64_t)d * n + p] = t;
        }
      }
    }
    if (full) {
      uint4* dst = (uint4*)(out + gs * dims);
#pragma unroll
      for (uint32_t i = 0; i < 4 * DIMS * sizeof(T) / 16; ++i) dst[i] = o.v[i];
    }
  }
  // not P->status: every wavefront reads that when it starts, and one that
  // left alone would leave its leaves' spans unwritten, by which the others
  // of its block store (a barrier in front of that read takes the
  // 2^27-particle decode from 637 us to 663)
  if (corrupt) P->damage = 1;
  // ref_mode 1: each leaf's first slot (its reference, where its code's bin
  // centre was written) receives the stored original coordinates, bit for bit
  if (V.ref_mode) {
    __syncthreads();
    typedef typename std::conditional<sizeof(T) == 4, uint32_t, uint64_t>::type U;
    constexpr uint32_t M = 8 * sizeof(T);
    for (uint32_t t = threadIdx.x; t < nlb * dims; t += kBlock) {
      const uint32_t l = t / dims, d = t - l * dims;
      const uint64_t st = sm.start[l];
      ((U*)out)[layout == BBX_AOS ? st * dims + d : (uint64_t)d * n + st] =
          (U)read_bits(meta, mwords, (L0 + l) * rb + dims * V.mbits + d * M, M);
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(kBlock) k_unpack(MetaView V, uint64_t n, uint32_t layout, const uint64_t* part,
                                                   const uint32_t* starts, const uint8_t* stream,
                                                   uint64_t pay_bits, T* out, DevParams* P) {
  if (P->status != BBX_OK) return;  // (set by earlier kernels only)
  __shared__ UnpackStage sm;
  const uint64_t* meta = (const uint64_t*)(stream + kHeaderBytes);
  const uint64_t* pay = meta + (V.meta_bits + 63) / 64;
  if (V.dims == 3)
    unpack_body<T, 3>(V, n, layout, meta, pay, pay_bits, part, starts, out, P, sm);
  else
    unpack_body<T, 2>(V, n, layout, meta, pay, pay_bits, part, starts, out, P, sm);
}

// Starts a decode: clears the status and checks that the stream's own
// header is the one the launch was planned from (one 8-byte word per lane).
__global__ void k_dec_init(DevParams* P, const uint8_t* stream, HeaderCopy h) {
  const uint32_t lane = threadIdx.x;
  const bool diff = lane < kHeaderBytes / 8 && ((const uint64_t*)stream)[lane] != h.w[lane];
  const uint64_t any = __ballot(diff);
  if (lane == 0) {
    P->status = any ? BBX_ECORRUPT : BBX_OK;
    P->damage = 0;
    P->payload_bits = 0;
  }
}

__global__ void k_dec_finish(const DevParams* P, uint32_t* d_status) {
  if (threadIdx.x == 0 && d_status) *d_status = P->damage ? (uint32_t)BBX_ECORRUPT : P->status;
}

// A lossless stream: the stored bits of every coordinate, in input order.
__global__ void __launch_bounds__(kBlock) k_unpack_lossless(uint64_t n, uint32_t dims, uint32_t dtype,
                                                            uint32_t layout, const uint8_t* stream,
                                                            void* pos, const DevParams* P) {
  if (P->status != BBX_OK) return;
  const uint64_t nv = n * dims;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nv;
       k += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t i = k / dims, d = k - i * dims;
    const uint64_t o = layout == BBX_AOS ? k : d * n + i;
    if (dtype == BBX_F32)
      ((uint32_t*)pos)[o] = ((const uint32_t*)(stream + kHeaderBytes))[k];
    else
      ((uint64_t*)pos)[o] = ((const uint64_t*)(stream + kHeaderBytes))[k];
  }
}

hipError_t launch_decompress(const DecompressPlan& p, const DecompressWs& w, const uint8_t* stream,
                             void* pos, uint32_t* d_status, hipStream_t s) {
  const uint64_t lpb = leaves_per_block(p.r), blocks = (p.n_leaves + lpb - 1) / lpb;
  const bool leaves = p.n > 0 && p.version == 1, top = leaves && blocks <= kDecTop;
  if (!top) BBX_LAUNCH("dec_init", k_dec_init, 1, 64, 0, s, w.params, stream, p.header);
  if (p.n > 0 && p.version == 3) {
    uint64_t g = (p.n * p.dims + kBlock - 1) / kBlock;
    if (g > 16384) g = 16384;
    BBX_LAUNCH("unpack_lossless", k_unpack_lossless, g, kBlock, 0, s, p.n, p.dims, p.dtype,
               p.layout, stream, pos, w.params);
  } else if (p.n > 0 && p.version == 2) {
    hipError_t e = launch_decompress2(p, w, stream, pos, s);
    if (e != hipSuccess) return e;
  } else if (leaves) {
    MetaView v;
    v.n_leaves = p.n_leaves;
    v.meta_bits = p.meta_bits;
    v.g = p.geom;
    v.w = p.w;
    v.inv_w = p.inv_w;
    for (int d = 0; d < 3; ++d) v.origin[d] = p.origin[d], v.G[d] = p.G[d];
    v.dims = p.dims;
    v.mbits = p.mbits;
    v.dtype = p.dtype;
    v.ref_mode = p.ref_mode;
    v.r = p.r;
    // every node of the halving tree splits evenly: leaf i starts at i * even
    v.even = (p.n_leaves & (p.n_leaves - 1)) == 0 && p.n % p.n_leaves == 0 ? (uint32_t)(p.n / p.n_leaves) : 0u;
    const uint64_t per = (kBlock / lpb);  // unpack blocks per block of k_dec_sums
    uint64_t* part = w.leaf_bits;         // the unpack blocks' payload bits, then their first ones
    uint32_t* starts = (uint32_t*)w.leaves;
    BBX_LAUNCH("dec_meta", k_dec_sums, (blocks + per - 1) / per, kBlock, 0, s, v, stream, blocks, part,
               starts, top ? (DevParams*)nullptr : w.params);
    if (top) {
      BBX_LAUNCH("dec_top", k_dec_top, 1, 1024, 0, s, blocks, part, w.params, stream, p.header, p.payload_bits);
    } else {
      hipError_t e = launch_dec_scan(blocks, part, w.scan_part, w.params, p.payload_bits, s);
      if (e != hipSuccess) return e;
    }
    if (p.dtype == BBX_F32)
      BBX_LAUNCH("unpack", k_unpack<float>, blocks, kBlock, 0, s, v, p.n, p.layout, part, starts, stream,
                 p.payload_bits, (float*)pos, w.params);
    else
      BBX_LAUNCH("unpack", k_unpack<double>, blocks, kBlock, 0, s, v, p.n, p.layout, part, starts, stream,
                 p.payload_bits, (double*)pos, w.params);
  }
  if (d_status) BBX_LAUNCH("dec_finish", k_dec_finish, 1, 64, 0, s, w.params, d_status);
  return hipGetLastError();
}

// ---------------------------------------------------------------- sequence export

constexpr uint32_t kExportLeaves = 256;  // leaves per block of k_export

// ORs the low `len` (<= 64) bits of v, whose bit 0 sits at absolute bit
// `at`, into the word whose bit 0 sits at absolute bit w0.
__device__ inline void or_bits(uint64_t& word, uint64_t w0, uint64_t v, uint64_t at, uint32_t len) {
  if (len == 0 || at >= w0 + 64 || at + len <= w0) return;
  if (len < 64) v &= (1ull << len) - 1;
  if (at >= w0)
    word |= v << (at - w0);
  else
    word |= v >> (w0 - at);
}

// Zeroes the output words that two blocks of k_export share (the word
// holding the first bit of every block's first sequence but the first).
// After a failed validation (the offsets may then run past the layout)
// nothing is written.
__global__ void k_export_edges(uint64_t n_leaves, uint64_t F, const uint64_t* off, uint64_t* out,
                               uint64_t out_words, const DevParams* P) {
  if (P->status != BBX_OK) return;
  const uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x + 1;
  const uint64_t L0 = b * kExportLeaves;
  if (L0 >= n_leaves) return;
  const uint64_t at = L0 * F + off[L0];
  if ((at & 63) && (at >> 6) < out_words) out[at >> 6] = 0;
}

// The Sec. 4.2 sequence layout of a ref_mode 1 stream: per leaf, in stored
// order, the centre's coordinate bits (M per axis), the widths (mbits each),
// the member codes (the leaf's payload segment, `off` its exclusive bit
// offsets) and a 32-bit end mark of all ones.  A block takes kExportLeaves
// leaves and writes the output words their sequences cover, one thread per
// word; the words it shares with a neighbouring block (zeroed before) take
// an atomic OR, every other word a plain store.
__global__ void __launch_bounds__(kBlock) k_export(uint64_t n_leaves, uint32_t dims, uint32_t mbits,
                                                   uint32_t M, uint64_t meta_bits,
                                                   uint64_t payload_bits, const uint64_t* off,
                                                   const uint8_t* stream, uint64_t* out,
                                                   const DevParams* P) {
  if (P->status != BBX_OK) return;
  __shared__ uint64_t so[kExportLeaves + 1];  // first output bit of each sequence (+ the end)
  const uint64_t F = (uint64_t)dims * (M + mbits) + 32;  // bits of a sequence besides its codes
  const uint64_t L0 = (uint64_t)blockIdx.x * kExportLeaves;
  const uint32_t cnt = (uint32_t)(n_leaves - L0 < kExportLeaves ? n_leaves - L0 : kExportLeaves);
  for (uint32_t t = threadIdx.x; t <= cnt; t += blockDim.x) {
    const uint64_t L = L0 + t;
    so[t] = L * F + (L < n_leaves ? off[L] : payload_bits);
  }
  __syncthreads();
  const uint64_t* meta = (const uint64_t*)(stream + kHeaderBytes);
  const uint64_t mwords = (meta_bits + 63) / 64;
  const uint64_t* pay = meta + mwords;
  const uint64_t pwords = (payload_bits + 63) / 64;
  const uint64_t S = (uint64_t)dims * (mbits + M);
  const uint64_t b_beg = so[0], b_end = so[cnt];  // b_end - b_beg >= F > 0
  const uint64_t w_first = b_beg >> 6, w_last = (b_end - 1) >> 6;
  for (uint64_t w = w_first + threadIdx.x; w <= w_last; w += blockDim.x) {
    const uint64_t b0 = w << 6;
    // the last sequence starting at or before the word (or the block's first)
    const uint64_t x = b0 > b_beg ? b0 : b_beg;
    uint32_t lo = 0, hi = cnt;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (so[mid] <= x)
        lo = mid;
      else
        hi = mid;
    }
    uint64_t word = 0;
    for (uint32_t i = lo; i < cnt && so[i] < b0 + 64; ++i) {
      const uint64_t L = L0 + i, at = so[i], rec = L * S;
      const uint64_t p0 = at + dims * (M + mbits), plen = so[i + 1] - at - F;
      if (at < b0 + 64 && p0 > b0) {  // centre and widths reach into the word
        for (uint32_t d = 0; d < dims; ++d) {
          or_bits(word, b0, (uint64_t)read_bits(meta, mwords, rec + dims * mbits + d * M, M),
                  at + d * M, M);
          or_bits(word, b0, (uint64_t)read_bits(meta, mwords, rec + d * mbits, mbits),
                  at + dims * M + d * mbits, mbits);
        }
      }
      if (plen && p0 < b0 + 64 && p0 + plen > b0) {  // the part of the codes inside the word
        const uint64_t s0 = p0 > b0 ? p0 : b0;
        const uint64_t e0 = p0 + plen < b0 + 64 ? p0 + plen : b0 + 64;
        const uint32_t len = (uint32_t)(e0 - s0);
        or_bits(word, b0, (uint64_t)read_bits(pay, pwords, off[L] + (s0 - p0), len), s0, len);
      }
      or_bits(word, b0, 0xffffffffull, p0 + plen, 32);  // end mark
    }
    const bool shared = (w == w_first && (b_beg & 63) && L0 > 0) ||
                        (w == w_last && (b_end & 63) && L0 + cnt < n_leaves);
    if (shared)
      atomicOr((unsigned long long*)&out[w], (unsigned long long)word);
    else
      out[w] = word;
  }
}

// Every leaf's record (w.leaves) and first payload bit (w.leaf_bits).
hipError_t launch_records(const DecompressPlan& p, const DecompressWs& w, const uint8_t* stream, hipStream_t s) {
  BBX_LAUNCH("dec_init", k_dec_init, 1, 64, 0, s, w.params, stream, p.header);
  if (p.n == 0) return hipGetLastError();
  uint64_t g = (p.n_leaves + kBlock - 1) / kBlock;
  if (g > 65536) g = 65536;
  BBX_LAUNCH("dec_meta", k_dec_meta, g, kBlock, 0, s, p.n_leaves, p.dims, p.mbits, p.G[0],
             p.G[1], p.G[2], p.meta_bits, p.geom, stream, w.leaves, w.leaf_bits, w.params,
             p.ref_mode, p.dtype, p.origin[0], p.origin[1], p.origin[2], p.inv_w);
  return launch_dec_scan(p.n_leaves, w.leaf_bits, w.scan_part, w.params, p.payload_bits, s);
}

hipError_t launch_export(const DecompressPlan& p, const DecompressWs& w, const uint8_t* stream,
                         void* out, uint32_t* d_status, hipStream_t s) {
  const hipError_t e = launch_records(p, w, stream, s);
  if (e != hipSuccess) return e;
  if (p.n > 0) {
    const uint32_t M = coord_bits(p.dtype);
    const uint64_t F = (uint64_t)p.dims * (M + p.mbits) + 32;
    const uint64_t blocks = (p.n_leaves + kExportLeaves - 1) / kExportLeaves;
    const uint64_t out_words = (p.n_leaves * F + p.payload_bits + 63) / 64;
    if (blocks > 1)
      BBX_LAUNCH("export_edges", k_export_edges, (blocks - 1 + kBlock - 1) / kBlock, kBlock, 0, s,
                 p.n_leaves, F, w.leaf_bits, (uint64_t*)out, out_words, w.params);
    BBX_LAUNCH("export", k_export, blocks, kBlock, 0, s, p.n_leaves, p.dims, p.mbits, M,
               p.meta_bits, p.payload_bits, w.leaf_bits, stream, (uint64_t*)out, w.params);
  }
  if (d_status) BBX_LAUNCH("dec_finish", k_dec_finish, 1, 64, 0, s, w.params, d_status);
  return hipGetLastError();
}

}  // namespace bbx
