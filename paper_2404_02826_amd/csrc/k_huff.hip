// k_huff.hip -- Huffman coding of a byte buffer: the encoding phase of
// Sec. 3, which the paper applies to its sequence layout (Sec. 4.2).
//
// Symbols are bytes.  Code lengths come from Huffman's construction, the two
// lightest nodes merging first (on equal weights the node created earlier:
// leaves, in symbol order, before merged nodes, in creation order); a tree
// deeper than kHufMaxLen is rebuilt from the weights halved (rounded up)
// until it fits.  Codes are canonical in (length, symbol) order.  The input
// is cut into chunks of kHufChunk bytes whose first bit offsets are stored,
// so that the chunks decode independently.
//
// Stream: [0,4) 'BBXH' | [4,6) version 1 | [6] kHufMaxLen | [7] 0 |
// [8,16) n | [16,20) kHufChunk | [20,24) 0 | [24,32) chunks |
// [32,40) payload bits | [40,48) 0 | [48,176) code lengths, a nibble per
// symbol (low nibble: even symbol) | chunk bit offsets, u64 each, from the
// payload start | payload: the codes in input order, each code's most
// significant bit first, bit i = bit i mod 64 of u64 word i / 64, zero
// padded to 8 bytes.
//
// Encode (the call waits twice: for the histogram, from which the host builds
// the code, and for the total size):
//   k_huf_hist    byte histogram (LDS bins per block, then global atomics)
//   k_huf_count   bits of every chunk (a block per chunk)
//   k_huf_offsets one block: exclusive scan of the chunk bits into the
//                 stream's offset table, and the payload's total bits
//   k_huf_write   a block per chunk: each thread's 16 bytes of codes at its
//                 offset (block scan) in an LDS copy of the chunk's words
// Decode:
//   k_huf_table   one block: checks the header against the host's copy, the
//                 lengths (at most kHufMaxLen, Kraft sum at most 1), and builds
//                 the 4,096-entry table from a 12-bit window to (symbol, length)
//   k_huf_decode  a wavefront per chunk, the table and the chunk's bits in LDS
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "bbx_internal.h"

namespace bbx {

typedef unsigned __int128 u128;

constexpr uint32_t kHufMagic = 0x48584242u;  // bytes 'B','B','X','H'
constexpr uint32_t kHufMaxLen = 12;
constexpr uint32_t kHufChunk = 4096;
constexpr uint32_t kHufHeader = 176;
constexpr uint32_t kHufPer = kHufChunk / kBlock;  // bytes per thread of a chunk block

// The host's copy of a stream header, for the device to compare.
struct HufHeaderCopy {
  uint64_t w[kHufHeader / 8];
};

__host__ __device__ inline uint64_t huf_chunks(uint64_t n) { return (n + kHufChunk - 1) / kHufChunk; }
__host__ __device__ inline uint64_t huf_words(uint64_t bits) { return (bits + 63) / 64; }

// ---------------------------------------------------------------- host: the code

// Code lengths by the two-queue form of Huffman's construction: leaves sorted
// by (weight, symbol) in one queue, merged nodes in creation order in the
// other (their weights never decrease); the lighter front merges first, the
// leaf on equal weights (every leaf was created before every merged node).
static void huf_build_lengths(const uint64_t* counts, uint32_t* len) {
  std::vector<uint64_t> w(counts, counts + 256);
  for (int s = 0; s < 256; ++s) len[s] = 0;
  for (;;) {
    std::vector<int> leaves;
    for (int s = 0; s < 256; ++s)
      if (w[s]) leaves.push_back(s);
    const size_t k = leaves.size();
    if (k == 0) return;
    if (k == 1) {
      len[leaves[0]] = 1;
      return;
    }
    std::stable_sort(leaves.begin(), leaves.end(), [&](int a, int b) { return w[a] < w[b]; });
    // node ids: leaves 0..k-1 (in symbol order), merged k..; parent links
    std::vector<int> leaf_id(256, -1), parent(2 * k - 1, -1);
    {
      int id = 0;
      for (int s = 0; s < 256; ++s)
        if (w[s]) leaf_id[s] = id++;
    }
    std::vector<uint64_t> mw;  // merged nodes' weights, in creation order
    size_t li = 0, mi = 0;
    auto take = [&]() -> std::pair<int, uint64_t> {
      const bool leaf = mi >= mw.size() || (li < k && w[leaves[li]] <= mw[mi]);
      if (leaf) {
        const int s = leaves[li++];
        return {leaf_id[s], w[s]};
      }
      const int id = (int)(k + mi);
      return {id, mw[mi++]};
    };
    for (size_t m = 0; m + 1 < k; ++m) {
      const auto a = take(), b = take();
      const int id = (int)(k + mw.size());
      parent[a.first] = parent[b.first] = id;
      mw.push_back(a.second + b.second);
    }
    uint32_t deepest = 0;
    std::vector<uint32_t> depth(256, 0);
    for (int s = 0; s < 256; ++s) {
      if (!w[s]) continue;
      uint32_t dpt = 0;
      for (int p = parent[leaf_id[s]]; p >= 0; p = parent[p]) ++dpt;
      depth[s] = dpt;
      deepest = std::max(deepest, dpt);
    }
    if (deepest <= kHufMaxLen) {
      for (int s = 0; s < 256; ++s) len[s] = depth[s];
      return;
    }
    for (int s = 0; s < 256; ++s)
      if (w[s]) w[s] = (w[s] + 1) / 2;
  }
}

// Canonical codes, each reversed into the stream's bit order (the code's
// first bit at bit 0), packed with the length: rev | len << 16.
static void huf_build_table(const uint32_t* len, uint32_t* tab) {
  uint32_t code = 0, prev = 0;
  bool first = true;
  for (uint32_t L = 1; L <= kHufMaxLen; ++L)
    for (int s = 0; s < 256; ++s) {
      if (len[s] != L) continue;
      if (!first) code = (code + 1) << (L - prev);
      first = false;
      prev = L;
      uint32_t rev = 0;
      for (uint32_t b = 0; b < L; ++b) rev |= ((code >> (L - 1 - b)) & 1u) << b;
      tab[s] = rev | (L << 16);
    }
  for (int s = 0; s < 256; ++s)
    if (!len[s]) tab[s] = 0;
}

// ---------------------------------------------------------------- kernels

// Every block adds its 256 bins to the same addresses at its end, one after
// another: 40 MB take 50 us with 2,048 blocks, 24 with 512.
constexpr uint64_t kHistBlocks = 512;
__global__ void __launch_bounds__(kBlock) k_huf_hist(const uint8_t* in, uint64_t n,
                                                     unsigned long long* counts) {
  __shared__ uint32_t h[4][257];  // four copies, staggered across banks
  for (uint32_t i = threadIdx.x; i < 4 * 257; i += kBlock) (&h[0][0])[i] = 0;
  __syncthreads();
  const uint32_t cp = threadIdx.x & 3;
  const uint64_t nv = n / 16;
  const uint4* in4 = (const uint4*)in;
  for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v < nv;
       v += (uint64_t)gridDim.x * kBlock) {
    const uint4 q = in4[v];
    const uint32_t wv[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int b = 0; b < 4; ++b) atomicAdd(&h[cp][(wv[k] >> (8 * b)) & 255u], 1u);
  }
  if (blockIdx.x == 0)
    for (uint64_t i = nv * 16 + threadIdx.x; i < n; i += kBlock) atomicAdd(&h[cp][in[i]], 1u);
  __syncthreads();
  const uint32_t c = h[0][threadIdx.x] + h[1][threadIdx.x] + h[2][threadIdx.x] + h[3][threadIdx.x];
  if (c) atomicAdd(&counts[threadIdx.x], (unsigned long long)c);
}

__device__ inline uint64_t huf_block_exscan(uint64_t v, uint64_t* total) {
  __shared__ uint64_t ws[16];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  uint64_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o);
    if ((int)lane >= o) x += y;
  }
  if (lane == 63) ws[wv] = x;
  __syncthreads();
  uint64_t off = 0, tot = 0;
  for (uint32_t k = 0; k < nw; ++k) {
    off += k < wv ? ws[k] : 0ull;
    tot += ws[k];
  }
  __syncthreads();
  *total = tot;
  return off + x - v;
}

// The thread's kHufPer bytes of a chunk (in + a, 16-byte aligned; those from n
// on are not there), one load for all.
struct HufBytes {
  uint32_t w[kHufPer / 4];
  uint32_t count;
};
static_assert(kHufPer == 16, "one 16-byte load per thread");
__device__ __forceinline__ HufBytes huf_bytes(const uint8_t* in, uint64_t n, uint64_t a) {
  HufBytes b;
  if (a + kHufPer <= n) {
    const uint4 q = *(const uint4*)(in + a);
    b.w[0] = q.x, b.w[1] = q.y, b.w[2] = q.z, b.w[3] = q.w;
    b.count = kHufPer;
  } else {
#pragma unroll
    for (uint32_t k = 0; k < kHufPer / 4; ++k) b.w[k] = 0;
    b.count = a < n ? (uint32_t)(n - a) : 0u;
#pragma unroll
    for (uint32_t k = 0; k < kHufPer; ++k)
      if (k < b.count) b.w[k / 4] |= (uint32_t)in[a + k] << (8 * (k & 3));
  }
  return b;
}
__device__ __forceinline__ uint32_t huf_byte(const HufBytes& b, uint32_t k) {
  return (b.w[k / 4] >> (8 * (k & 3))) & 255u;
}

// code bits of the thread's bytes
__device__ __forceinline__ uint32_t huf_thread_bits(const HufBytes& b, const uint32_t* tab) {
  uint32_t bits = 0;
#pragma unroll
  for (uint32_t k = 0; k < kHufPer; ++k)
    if (k < b.count) bits += tab[huf_byte(b, k)] >> 16;
  return bits;
}

// Exclusive scan over the block of a value per thread (totals below 2^32).
__device__ inline uint32_t huf_scan32(uint32_t x, uint32_t* total) {
  __shared__ uint32_t ws[kBlock / 64];
  const uint32_t incl = wave_incl(x), wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) ws[wv] = incl;
  __syncthreads();
  uint32_t off = incl - x, tot = 0;
#pragma unroll
  for (uint32_t k = 0; k < kBlock / 64; ++k) {
    off += k < wv ? ws[k] : 0u;
    tot += ws[k];
  }
  *total = tot;
  return off;
}

__global__ void __launch_bounds__(kBlock) k_huf_count(const uint8_t* in, uint64_t n,
                                                      const uint32_t* tab0, uint64_t* chunk_bits) {
  __shared__ uint32_t tab[256];
  const HufBytes b = huf_bytes(in, n, (uint64_t)blockIdx.x * kHufChunk + (uint64_t)threadIdx.x * kHufPer);
  tab[threadIdx.x] = tab0[threadIdx.x];
  __syncthreads();
  uint32_t tot;
  (void)huf_scan32(huf_thread_bits(b, tab), &tot);
  if (threadIdx.x == 0) chunk_bits[blockIdx.x] = tot;
}

// One block: chunk offsets into the stream (after the header) and the total;
// kOffPer chunks per thread and round.
constexpr uint32_t kOffPer = 8;
__global__ void __launch_bounds__(1024) k_huf_offsets(const uint64_t* chunk_bits, uint64_t chunks,
                                                      uint8_t* out, uint64_t* total_out) {
  uint64_t* offs = (uint64_t*)(out + kHufHeader);
  uint64_t run = 0;
  for (uint64_t c0 = 0; c0 < chunks; c0 += kOffPer * 1024) {
    const uint64_t c = c0 + kOffPer * threadIdx.x;
    uint64_t v[kOffPer], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kOffPer; ++k) {
      v[k] = c + k < chunks ? chunk_bits[c + k] : 0ull;
      sum += v[k];
    }
    uint64_t tot;
    uint64_t at = run + huf_block_exscan(sum, &tot);
#pragma unroll
    for (uint32_t k = 0; k < kOffPer; ++k) {
      if (c + k < chunks) offs[c + k] = at;
      at += v[k];
    }
    run += tot;
  }
  if (threadIdx.x == 0) {
    *total_out = run;
    *(uint64_t*)(out + 32) = run;  // payload bits
  }
}

// A block per chunk: each thread's 16 codes go to its offset (block scan) in
// an LDS copy of the chunk's words.  The block owns the words that begin in
// its chunk; the last of them is completed with the first codes of the next
// chunk by one wavefront (64 bytes of input hold at least 64 bits of codes,
// or reach the input's end), so every word is written once, coalesced, and
// nothing has to be zeroed before.  (ORing each thread's words into a zeroed
// payload with global atomics took 150 us for 40 MB and the zeroing 8, this
// takes 34.)
constexpr uint32_t kHufOutWords = kHufChunk * kHufMaxLen / 64 + 2;
__global__ void __launch_bounds__(kBlock) k_huf_write(const uint8_t* in, uint64_t n,
                                                      const uint32_t* tab0, uint8_t* out,
                                                      uint64_t chunks, uint64_t bits) {
  __shared__ uint32_t tab[256];
  __shared__ unsigned long long wd[kHufOutWords];
  const uint64_t c = blockIdx.x;
  const uint64_t* offs = (const uint64_t*)(out + kHufHeader);
  unsigned long long* pay = (unsigned long long*)(out + kHufHeader + 8 * chunks);
  const HufBytes b = huf_bytes(in, n, c * kHufChunk + (uint64_t)threadIdx.x * kHufPer);
  const uint64_t pos = offs[c], end = c + 1 < chunks ? offs[c + 1] : bits;
  const uint64_t next = (c + 1) * kHufChunk + threadIdx.x;  // the byte that the first wavefront adds
  const uint32_t after = threadIdx.x < 64 && next < n ? in[next] : 0u;
  tab[threadIdx.x] = tab0[threadIdx.x];
  for (uint32_t k = threadIdx.x; k < kHufOutWords; k += kBlock) wd[k] = 0;
  __syncthreads();
  uint32_t tot;
  const uint32_t at0 = (uint32_t)(pos & 63) + huf_scan32(huf_thread_bits(b, tab), &tot);
  auto put = [&](uint32_t word, uint64_t v) {
    if (word < kHufOutWords) atomicOr(&wd[word], (unsigned long long)v);
  };
  {
    // the thread's codes gathered in a 64-bit window
    uint64_t win = 0;
    uint32_t fill = at0 & 63, word = at0 >> 6;
#pragma unroll
    for (uint32_t k = 0; k < kHufPer; ++k) {
      const uint32_t e = k < b.count ? tab[huf_byte(b, k)] : 0u;
      const uint32_t L = e >> 16;
      const uint64_t rev = e & 0xffffu;
      win |= rev << fill;
      fill += L;
      if (fill >= 64) {
        put(word, win);
        ++word;
        fill -= 64;
        win = fill ? rev >> (L - fill) : 0ull;  // (L <= 12)
      }
    }
    if (win) put(word, win);
  }
  // the owned words [w0, w1): those whose first bit is in [pos, end)
  const uint64_t base = pos >> 6, w0 = (pos + 63) >> 6, w1 = (end + 63) >> 6;
  if (threadIdx.x < 64 && (end & 63) && end < bits) {
    const uint32_t e = next < n ? tab[after] : 0u, L = e >> 16;
    const uint32_t from = (uint32_t)(end & 63) + wave_incl(L) - L;  // in the last word
    if (L && from < 64) put((uint32_t)((end >> 6) - base), (uint64_t)(e & 0xffffu) << from);
  }
  __syncthreads();
  for (uint64_t w = w0 + threadIdx.x; w < w1; w += kBlock) pay[w] = wd[w - base];
}

// Decode table: 12-bit window (the code's first bit at bit 0) -> symbol |
// length << 8, 0 where no code matches.  Also checks the stream's header
// against the host's copy and the lengths, and sets *status.  A thread per
// symbol: canonical codes from the lengths' counts and the symbol's rank
// among the symbols of its length, then a wavefront per symbol fills the
// windows that begin with its code (one thread doing it all took 340 us, this
// takes 11).
__global__ void __launch_bounds__(kBlock) k_huf_table(const uint8_t* s, HufHeaderCopy h,
                                                      uint16_t* table, uint32_t* status) {
  constexpr uint32_t kW = kBlock / 64;
  __shared__ uint32_t cnt[kW][kHufMaxLen + 1];  // per wavefront: symbols of each length
  __shared__ uint32_t tab[256];
  __shared__ uint32_t bad;
  static_assert(kBlock == 256, "a thread per symbol");
  const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
  if (t == 0) bad = 0;
  __syncthreads();
  if (t < kHufHeader / 8 && ((const uint64_t*)s)[t] != h.w[t]) atomicOr(&bad, 1u);
  const uint32_t len = (s[48 + t / 2] >> ((t & 1) ? 4 : 0)) & 15u;
  if (len > kHufMaxLen) atomicOr(&bad, 1u);
  uint32_t rank = 0;
#pragma unroll
  for (uint32_t L = 1; L <= kHufMaxLen; ++L) {
    const uint64_t m = __ballot(len == L);
    if (len == L) rank = lanes_below(m);
    if (lane == 0) cnt[wv][L] = (uint32_t)__popcll(m);
  }
  __syncthreads();
  // first code of each length: (first code of the one before + its count) * 2
  uint32_t code = 0, kraft = 0, mine = 0;
#pragma unroll
  for (uint32_t L = 1; L <= kHufMaxLen; ++L) {
    uint32_t before = 0, all = 0;
#pragma unroll
    for (uint32_t w = 0; w < kW; ++w) {
      before += w < wv ? cnt[w][L] : 0u;
      all += cnt[w][L];
    }
    code <<= 1;
    if (len == L) mine = code + before + rank;
    code += all;
    kraft += all << (kHufMaxLen - L);
  }
  if (kraft > (1u << kHufMaxLen) && t == 0) bad = 1;
  // the code's first bit at bit 0
  tab[t] = len >= 1 && len <= kHufMaxLen ? (__brev(mine) >> (32 - len)) | (len << 16) : 0u;
  __syncthreads();
  if (t == 0) *status = bad ? BBX_ECORRUPT : BBX_OK;
  if (bad) return;
  for (uint32_t x = t; x < (1u << kHufMaxLen); x += kBlock) table[x] = 0;
  __syncthreads();
  for (uint32_t y = wv; y < 256; y += kW) {
    const uint32_t e = tab[y], L = e >> 16;
    if (!L) continue;
    const uint32_t rev = e & 0xffffu;
    for (uint32_t hi = lane; hi < (1u << (kHufMaxLen - L)); hi += 64)
      table[rev | (hi << L)] = (uint16_t)(y | (L << 8));
  }
}

// A wavefront per chunk.  The chunk's bits are cut into 64 runs of whole
// 32-bit words, one per lane; where a lane's first code starts depends on
// all codes before it, but as a code is at most 12 bits long it is one of
// the first 12 bits of the run.  So:
//   1. every lane walks its run's bit positions backwards and keeps, for the
//      12 positions after the current one, how far past the run's end the
//      codes that start there lead (a nibble each, 15: no code); at the run's
//      first bit that is a map from entry offset to exit offset,
//   2. the 64 maps are followed from the chunk's first bit, which gives every
//      lane its first code,
//   3. every lane decodes its run, first counting its symbols (a scan gives
//      its place in the output), then storing them four at a time.
// The walk looks at every bit position, about eight per symbol, but in 64
// lanes at once and with independent table reads; the thread per chunk that
// this replaces was one chain of 4,096 dependent reads.  Bound by the walk
// (instruction issue and table reads): 40 MB in 198 us, before in 2,195.
constexpr uint32_t kHufWords = (kHufChunk * kHufMaxLen + 31) / 32 + 3;  // a chunk's 32-bit words at most, two of look-ahead
constexpr uint32_t kHufPad = kHufWords + kHufWords / 16 + 1;  // one word in 17 unused: runs of 16 words start in different banks
__device__ __forceinline__ uint32_t huf_at(uint32_t w) { return w + (w >> 4); }

__global__ void __launch_bounds__(kBlock) k_huf_decode(const uint8_t* s, uint64_t n, uint64_t chunks,
                                                       uint64_t bits, const uint16_t* table0,
                                                       uint8_t* out, uint32_t* status) {
  constexpr uint32_t kW = kBlock / 64;
  __shared__ uint16_t table[1u << kHufMaxLen];
  __shared__ uint32_t stage[kW][kHufPad];
  // every thread of the block takes the same way at the barrier, also when
  // another block sets the status meanwhile
  if (__syncthreads_or(*(volatile uint32_t*)status != BBX_OK)) return;
  for (uint32_t x = threadIdx.x; x < (1u << kHufMaxLen) / 2; x += kBlock)
    ((uint32_t*)table)[x] = ((const uint32_t*)table0)[x];
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint64_t c = (uint64_t)blockIdx.x * kW + wv;
  if (c >= chunks) return;
  const uint64_t* offs = (const uint64_t*)(s + kHufHeader);
  const uint64_t nwords = 2 * huf_words(bits);  // 32-bit words of the payload
  const uint32_t* pay = (const uint32_t*)(offs + chunks);
  const uint64_t pos = offs[c];
  const uint64_t end = c + 1 < chunks ? offs[c + 1] : bits;
  const uint32_t syms = (uint32_t)(c * kHufChunk + kHufChunk < n ? kHufChunk : n - c * kHufChunk);
  if (pos > end || end > bits || end - pos > (uint64_t)syms * kHufMaxLen) {
    if (lane == 0) atomicExch(status, (uint32_t)BBX_ECORRUPT);
    return;
  }
  // bit positions from here on count from the chunk's first word
  const uint64_t w0 = pos >> 5;
  const uint32_t first = (uint32_t)(pos & 31), last = first + (uint32_t)(end - pos);
  const uint32_t words = (last + 31) / 32;  // <= kHufWords - 2
  uint32_t* const wd = stage[wv];
  for (uint32_t x = lane; x < words + 2; x += 64) wd[huf_at(x)] = w0 + x < nwords ? pay[w0 + x] : 0u;
  wave_sync();
  const uint32_t per = (words + 63) / 64;  // words per run
  const uint32_t a = lane * per * 32 < first ? first : lane * per * 32;  // the run's bits [a, b)
  const uint32_t b = (lane + 1) * per * 32 < last ? (lane + 1) * per * 32 : last;

  // ---- 1: entry offset -> exit offset
  uint64_t E = 0xffffba9876543210ull;
  for (uint32_t k = per; k-- > 0;) {
    const uint32_t x = lane * per + k;
    const bool some = x * 32 < b;  // a run past the chunk's end keeps the identity
    const uint32_t lo = some ? wd[huf_at(x)] : 0u, hi = some ? wd[huf_at(x + 1)] : 0u;
    if (__ballot(!some || (x * 32 >= a && x * 32 + 32 <= b)) == ~0ull) {
      if (some) {
#pragma unroll
        for (int j = 31; j >= 0; --j) {
          const uint32_t L = table[__builtin_amdgcn_alignbit(hi, lo, j) & ((1u << kHufMaxLen) - 1)] >> 8;
          const uint32_t o = L ? (uint32_t)(E >> (4 * (L - 1) & 63)) & 15u : 15u;
          E = (E << 4) | o;
        }
      }
    } else {  // the words of the chunk's first and last bit
      for (int j = 31; j >= 0; --j) {
        const uint32_t p = x * 32 + (uint32_t)j;
        const uint32_t L = table[__builtin_amdgcn_alignbit(hi, lo, j) & ((1u << kHufMaxLen) - 1)] >> 8;
        const uint32_t o = L ? (uint32_t)(E >> (4 * (L - 1) & 63)) & 15u : 15u;
        if (p >= a && p < b) E = (E << 4) | o;
      }
    }
  }
  E |= 0xffffull << 48;  // 15 leads to 15

  // ---- 2: the maps in lane order from the first bit
  uint32_t e = 0, in = 0;
#pragma unroll
  for (int i = 0; i < 64; ++i) {
    const uint64_t Ei = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(E >> 32), i) << 32 |
                        (uint32_t)__builtin_amdgcn_readlane((int)E, i);
    if ((int)lane == i) in = e;
    e = (uint32_t)(Ei >> (4 * e)) & 15u;
  }
  if (e != 0) {  // no code somewhere, or the last one does not end with the chunk
    if (lane == 0) atomicExch(status, (uint32_t)BBX_ECORRUPT);
    return;
  }

  // ---- 3: every lane decodes the codes that start in [a + in, b)
  auto decode = [&](auto&& emit) {
    uint32_t p = a + in;
    if (p >= b) return;
    uint32_t x = p >> 5;
    uint64_t acc = ((uint64_t)wd[huf_at(x + 1)] << 32 | wd[huf_at(x)]) >> (p & 31);
    uint32_t have = 64 - (p & 31);
    x += 2;
    while (p < b) {
      const uint32_t t = table[(uint32_t)acc & ((1u << kHufMaxLen) - 1)];
      const uint32_t L = t >> 8;
      emit(t & 0xffu);
      acc >>= L;
      have -= L;
      p += L;
      if (have <= 32) {  // (a word past the chunk's look-ahead holds no bit that is used)
        acc |= (uint64_t)wd[huf_at(x < words + 2 ? x : words + 1)] << have;
        have += 32;
        ++x;
      }
    }
  };
  uint32_t count = 0;
  decode([&](uint32_t) { ++count; });
  uint32_t total;
  {
    const uint32_t incl = wave_incl(count);
    total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    count = incl - count;  // the lane's first symbol
  }
  if (total != syms) {
    if (lane == 0) atomicExch(status, (uint32_t)BBX_ECORRUPT);
    return;
  }
  uint8_t* const o = out + c * kHufChunk;  // 8-byte aligned
  uint32_t i = count, i0 = count, pk = 0;
  decode([&](uint32_t sym) {
    pk |= sym << (8 * (i & 3));
    if ((i & 3) == 3) {
      if (i - i0 >= 3) {
        *(uint32_t*)(o + (i & ~3u)) = pk;
      } else {  // a word begun by the lane before
        for (uint32_t t = i0; t <= i; ++t) o[t] = (uint8_t)(pk >> (8 * (t & 3)));
      }
      pk = 0;
    }
    ++i;
  });
  for (uint32_t t = (i & ~3u) > i0 ? (i & ~3u) : i0; t < i; ++t) o[t] = (uint8_t)(pk >> (8 * (t & 3)));
}

}  // namespace bbx

using namespace bbx;

namespace {

struct HufHead {
  uint64_t n, chunks, bits;
};

bbx_status huf_parse(const uint8_t* h, size_t bytes, HufHead* o) {
  if (!h || bytes < kHufHeader) return set_error(BBX_ECORRUPT, "Huffman stream shorter than its header");
  uint32_t magic, chunk;
  uint16_t ver;
  memcpy(&magic, h, 4);
  memcpy(&ver, h + 4, 2);
  memcpy(&chunk, h + 16, 4);
  memcpy(&o->n, h + 8, 8);
  memcpy(&o->chunks, h + 24, 8);
  memcpy(&o->bits, h + 32, 8);
  uint64_t z0, z1 = 0;
  memcpy(&z0, h + 40, 8);
  memcpy(&z1, h + 20, 4);
  if (magic != kHufMagic || ver != 1 || h[6] != kHufMaxLen || h[7] != 0 || chunk != kHufChunk ||
      z0 != 0 || z1 != 0)
    return set_error(BBX_ECORRUPT, "not a Huffman stream of this version");
  if (o->chunks != huf_chunks(o->n) || o->bits > o->n * kHufMaxLen)
    return set_error(BBX_ECORRUPT, "Huffman chunk count or payload size out of range");
  return BBX_OK;
}

size_t huf_decode_ws(uint64_t chunks) {
  (void)chunks;
  return 256 + 2 * (1u << kHufMaxLen);
}

}  // namespace

extern "C" {

size_t bbx_huffman_bound(uint64_t n) {
  return kHufHeader + 8 * huf_chunks(n) + 8 * huf_words(n * kHufMaxLen);
}

size_t bbx_huffman_workspace_size(uint64_t n) {
  // counts (256 u64), code table (256 u32), chunk bits (u64 each), the total,
  // or when decoding: status and the 4,096-entry table
  const size_t enc = 2048 + 1024 + 8 * huf_chunks(n) + 8 + 256;
  return std::max(enc, huf_decode_ws(huf_chunks(n)));
}

bbx_status bbx_huffman_encode(const void* d_in, uint64_t n, void* d_out, size_t out_cap,
                              size_t* h_out_size, void* d_ws, size_t ws_size, hipStream_t stream) {
  if (!h_out_size) return set_error(BBX_EINVAL, "h_out_size is NULL");
  if (n > 0 && !d_in) return set_error(BBX_EINVAL, "input pointer is NULL");
  if (!d_out || ((uintptr_t)d_out & 7)) return set_error(BBX_EINVAL, "output must be 8-byte aligned");
  if (((uintptr_t)d_in & 15) && n >= 16) return set_error(BBX_EINVAL, "input must be 16-byte aligned");
  if (!d_ws || ((uintptr_t)d_ws & 255) || ws_size < bbx_huffman_workspace_size(n))
    return set_error(BBX_ENOMEM, "workspace too small or not 256-byte aligned");
  const uint64_t chunks = huf_chunks(n);
  uint8_t* ws = (uint8_t*)d_ws;
  unsigned long long* counts = (unsigned long long*)ws;
  uint32_t* tab = (uint32_t*)(ws + 2048);
  uint64_t* cbits = (uint64_t*)(ws + 3072);
  uint64_t* total = cbits + chunks;
  const uint8_t* in = (const uint8_t*)d_in;
  uint8_t* out = (uint8_t*)d_out;
  hipError_t e = hipMemsetAsync(counts, 0, 2048, stream);
  if (e == hipSuccess && n > 0)
    BBX_LAUNCH("huf_hist", k_huf_hist, (uint32_t)std::min<uint64_t>((n / 16 + kBlock - 1) / kBlock + 1, kHistBlocks),
               kBlock, 0, stream, in, n, counts);
  uint64_t hc[256];
  if (e == hipSuccess) e = hipMemcpyAsync(hc, counts, sizeof(hc), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return set_error(BBX_EHIP, hipGetErrorString(e));
  uint32_t len[256], htab[256];
  huf_build_lengths(hc, len);
  huf_build_table(len, htab);
  uint64_t bits = 0;
  for (int s = 0; s < 256; ++s) bits += hc[s] * len[s];
  const size_t size = kHufHeader + 8 * chunks + 8 * huf_words(bits);
  *h_out_size = size;
  if (size > out_cap) return set_error(BBX_ENOSPC, "output capacity below the Huffman stream");
  uint8_t head[kHufHeader];
  memset(head, 0, sizeof(head));
  const uint32_t magic = kHufMagic, chunk = kHufChunk;
  const uint16_t ver = 1;
  memcpy(head, &magic, 4);
  memcpy(head + 4, &ver, 2);
  head[6] = (uint8_t)kHufMaxLen;
  memcpy(head + 8, &n, 8);
  memcpy(head + 16, &chunk, 4);
  memcpy(head + 24, &chunks, 8);
  memcpy(head + 32, &bits, 8);
  for (int s = 0; s < 256; ++s) head[48 + s / 2] |= (uint8_t)(len[s] << ((s & 1) ? 4 : 0));
  e = hipMemcpyAsync(out, head, kHufHeader, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipMemcpyAsync(tab, htab, sizeof(htab), hipMemcpyHostToDevice, stream);
  if (e == hipSuccess && chunks > 0) {
    BBX_LAUNCH("huf_count", k_huf_count, (uint32_t)chunks, kBlock, 0, stream, in, n, tab, cbits);
    BBX_LAUNCH("huf_offsets", k_huf_offsets, 1, 1024, 0, stream, cbits, chunks, out, total);
    BBX_LAUNCH("huf_write", k_huf_write, (uint32_t)chunks, kBlock, 0, stream, in, n, tab, out, chunks, bits);
    e = hipGetLastError();
  }
  uint64_t dev_bits = bits;
  if (e == hipSuccess && chunks > 0)
    e = hipMemcpyAsync(&dev_bits, total, 8, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return set_error(BBX_EHIP, hipGetErrorString(e));
  if (dev_bits != bits) return set_error(BBX_EHIP, "chunk bit counts disagree with the histogram");
  return BBX_OK;
}

bbx_status bbx_huffman_decode(const void* d_stream, size_t stream_size, const void* h_header,
                              void* d_out, size_t out_cap, uint32_t* d_status, void* d_ws,
                              size_t ws_size, hipStream_t stream) {
  HufHead h;
  bbx_status st = huf_parse((const uint8_t*)h_header, h_header ? kHufHeader : 0, &h);
  if (st != BBX_OK) return st;
  if (!d_stream || stream_size < kHufHeader + 8 * h.chunks + 8 * huf_words(h.bits))
    return set_error(BBX_ECORRUPT, "Huffman stream shorter than its sections");
  if (h.n > out_cap) return set_error(BBX_ENOSPC, "output capacity below the decoded size");
  if (h.n > 0 && (!d_out || ((uintptr_t)d_out & 7))) return set_error(BBX_EINVAL, "output must be 8-byte aligned");
  if (!d_ws || ((uintptr_t)d_ws & 255) || ws_size < huf_decode_ws(h.chunks))
    return set_error(BBX_ENOMEM, "workspace too small or not 256-byte aligned");
  uint8_t* ws = (uint8_t*)d_ws;
  uint32_t* status = d_status ? d_status : (uint32_t*)ws;
  uint16_t* table = (uint16_t*)(ws + 256);
  HufHeaderCopy hc;
  memcpy(hc.w, h_header, kHufHeader);
  BBX_LAUNCH("huf_table", k_huf_table, 1, kBlock, 0, stream, (const uint8_t*)d_stream, hc, table,
             status);
  if (h.chunks > 0)
    BBX_LAUNCH("huf_decode", k_huf_decode, (uint32_t)((h.chunks + kBlock / 64 - 1) / (kBlock / 64)),
               kBlock, 0, stream, (const uint8_t*)d_stream, h.n, h.chunks, h.bits, table,
               (uint8_t*)d_out, status);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(BBX_EHIP, hipGetErrorString(e));
  if (d_status) return BBX_OK;
  uint32_t hs = 0;
  e = hipMemcpyAsync(&hs, status, 4, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return set_error(BBX_EHIP, hipGetErrorString(e));
  if (hs != BBX_OK) return set_error((bbx_status)hs, "the Huffman stream fails validation");
  return BBX_OK;
}

}  // extern "C"
