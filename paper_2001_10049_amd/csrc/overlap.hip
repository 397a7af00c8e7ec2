// overlap.hip - candidate read pairs on one GPU (paper: section 4 stages 1-3,
// sections 6, 7 and 8): every pair of reads sharing a retained k-mer, with the
// positions of all the retained k-mers it shares, as the seed lists that
// xd_align_pairs consumes.
//
// Pass 1 streams every k-mer through a blocked Bloom filter A (one 64-bit word
// and three bits per k-mer; neighbours that share a word set theirs with one
// atomic OR).  An occurrence that finds
// all its bits already set is a repeat (or a false positive) and marks the
// k-mer in a second, smaller filter B, so every k-mer occurring twice or more
// is in B while most singletons never reach it (section 6).  Pass 2 streams
// the k-mers again and inserts those in B into an open-addressing hash table
// (linear probing over 64-bit keys) that counts every occurrence and keeps the
// first m (read, position) locations (section 7).  Retained k-mers, those with
// 2 <= count <= m, expand into all pairs of their locations in different reads
// (Alg. 1, without the rank-placement rule that only matters across ranks),
// and an LSD radix sort by (read a, read b, pos a, pos b) groups the seeds per
// read pair.
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include <algorithm>
#include <mutex>
#include <utility>
#include <vector>

#include "scan.h"
#include "store_view.h"
#include "xdrop.h"

namespace {

using xscan::Arena;
using xscan::block_excl_scan;
using xscan::grid_for;

constexpr int kThreads = 256;
constexpr int kChunk = 64;                   // k-mer starts per thread in the passes
constexpr int kScanPer = xscan::kPer;         // slots per thread in the table scans
constexpr int kScanTile = xscan::kTile;
constexpr int kSortPer = 16;                 // items per thread in the radix sort
constexpr int kSortTile = kThreads * kSortPer;
constexpr uint64_t kMaxProbe = 1024;       // longest linear probe before the table regrows
constexpr uint64_t kSaltB = 0x9e3779b97f4a7c15ull;
constexpr uint64_t kSaltT = 0xd1b54a32d192ed03ull;

// ---- hashing ------------------------------------------------------------------

// MurmurHash3's 64-bit finalizer (a bijection with full avalanche)
__device__ __forceinline__ uint64_t fmix64(uint64_t x) {
  x ^= x >> 33;
  x *= 0xff51afd7ed558ccdull;
  x ^= x >> 33;
  x *= 0xc4ceb9fe1a85ec53ull;
  x ^= x >> 33;
  return x;
}

// three bit positions from the low 18 bits of h (two may coincide)
__device__ __forceinline__ uint64_t bloom_bits(uint64_t h) {
  return (1ull << (h & 63)) | (1ull << ((h >> 6) & 63)) | (1ull << ((h >> 12) & 63));
}

// word index in [0, W) from the high 32 bits of h (W < 2^32)
__device__ __forceinline__ uint64_t bloom_word(uint64_t h, uint64_t W) {
  return ((h >> 32) * W) >> 32;
}

// Neighbouring k-mers share the smallest hash `mh` of their m-mers, three of them
// or so, and the filters are laid out by it (RUNS), up to 2^27 words of filter A.
//
// Filter A: all k-mers of one mh lie in one word, so that a run of them in a
// thread takes one atomic.  Atomics are what bounds pass 1: the counters show
// every one carried out at the memory, 26 G a second, whatever line it lies in
// (138 Mbp, k = 17: 149 M -> 78 M of them, 5.7 -> 3.7 ms).  Words fill less
// evenly than by the k-mer's own hash: the m-mers have to outnumber the
// words by eight, which keeps false repeats to 1 % of the k-mers (0.25 % by the
// k-mer's own hash; 2.8 % with four to a word, 18 % with half a one to a word),
// and filters of more than 2^27 words (1 GB) are too many for a 32-bit mh.  Those,
// and their filter B, go by the k-mer's own hash, a k-mer at a time: without runs
// the m-mers and eight k-mers in flight only cost (0.7 Gbp, both strands, k = 31:
// 105 ms before the runs, 116 with B in lines and eight in flight, 104 so; one
// strand, k = 17: 217, 197, 184).
__device__ __forceinline__ uint64_t run_word(uint32_t mh, uint64_t W) {
  return ((uint64_t)(mh * 0x9e3779b1u) * W) >> 32;
}
constexpr uint64_t kRunWords = 1ull << 27;

// Filter B is lines of kLine words (128 bytes, what a memory access moves): the
// line comes from mh, the word in the line from four bits of h that bloom_bits
// leaves.  Pass 2 looks four k-mers up at once and so waits for fewer lines
// (2.73 -> 2.1 ms; 2.63 with a line for every k-mer).
constexpr uint64_t kLine = 16;

template <bool RUNS>
__device__ __forceinline__ uint64_t line_word(uint32_t mh, uint64_t h, uint64_t W) {
  if (!RUNS) return bloom_word(h, W);
  const uint32_t lines = (uint32_t)(W / kLine);
  return (uint64_t)__umulhi(mh * 0x9e3779b1u, lines) * kLine + ((h >> 18) & (kLine - 1));
}

// ---- k-mer enumeration --------------------------------------------------------

struct KmerScan {
  const uint32_t* words;
  const uint64_t* word_off;
  const uint32_t* len;
  const uint64_t* chunk_off;  // [n_reads + 1]: read r owns chunks [chunk_off[r], chunk_off[r+1])
  uint64_t n_chunks;
  uint32_t n_reads;
  int32_t k;
  uint64_t kmask;             // 2k low bits
  int32_t both;               // 1: canonical k-mers (both strands)
  int32_t m;                  // length of the m-mers that choose a k-mer's words
  uint64_t mmask;             // 2m low bits
};

constexpr int kWindow = 6;  // the m-mers of a k-mer, at most

// a k-mer: its code and strand, and the smallest hash of its m-mers
struct Kmer {
  uint64_t code;
  uint32_t strand;
  uint32_t mh;
};

// Calls f(read, pos, kmers, n) for the k-mer starts of chunk c in increasing
// pos, AHEAD of them at a time (n <= AHEAD in the last call); code packs the k
// bases 2 bits each, the first base highest.  Forward strand only: the k-mer's
// code, strand 0.  Both strands: the smaller of the code and its reverse
// complement's code (the complement 3 - b of each base, in reverse order),
// strand 1 when the reverse complement is the smaller; the m-mers likewise.
// MERS: find mh (else 0).
template <int AHEAD, bool MERS, class F>
__device__ __forceinline__ void for_kmers(const KmerScan& s, uint64_t c, F&& f) {
  uint32_t lo = 0, hi = s.n_reads - 1;  // the last read whose first chunk is <= c
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo + 1) / 2;
    if (s.chunk_off[mid] <= c) lo = mid;
    else hi = mid - 1;
  }
  const uint32_t r = lo;
  const uint32_t n_starts = s.len[r] - (uint32_t)s.k + 1;  // >= 1: read r owns a chunk
  const uint32_t p0 = (uint32_t)(c - s.chunk_off[r]) * kChunk;
  const uint32_t p1 = min(p0 + (uint32_t)kChunk, n_starts);
  const uint32_t* w = s.words + s.word_off[r];
  uint32_t cur_w = 0xffffffffu, wv = 0;
  auto base = [&](uint32_t q) -> uint64_t {
    if ((q >> 4) != cur_w) {
      cur_w = q >> 4;
      wv = w[cur_w];
    }
    return (wv >> ((q & 15) * 2)) & 3u;
  };
  const uint32_t top = 2u * (uint32_t)(s.k - 1);  // bit of a reverse-complement k-mer's last base
  const uint32_t mtop = 2u * (uint32_t)(s.k - s.m);
  const int window = s.k - s.m + 1;
  uint64_t code = 0, rcode = 0;
  uint32_t h[kWindow];  // hashes of the last m-mers, the newest first
  for (int i = 0; i < kWindow; ++i) h[i] = 0xffffffffu;
  auto add = [&](uint64_t b) {
    code = ((code << 2) | b) & s.kmask;
    rcode = (rcode >> 2) | ((3ull - b) << top);
  };
  auto add_hash = [&]() {
    if (!MERS) return;
    uint64_t v = code & s.mmask;
    if (s.both) v = min(v, rcode >> mtop);
    for (int i = kWindow - 1; i > 0; --i) h[i] = h[i - 1];
    h[0] = (uint32_t)((v * 0x9e3779b97f4a7c15ull) >> 32);
  };
  for (uint32_t q = 0; q + 1 < (uint32_t)s.k; ++q) {
    add(base(p0 + q));
    if (q + 1 >= (uint32_t)s.m) add_hash();
  }
  for (uint32_t p = p0; p < p1; p += AHEAD) {
    Kmer km[AHEAD];
    const int n = (int)min((uint32_t)AHEAD, p1 - p);
    for (int i = 0; i < AHEAD; ++i) {
      if (i < n) {
        add(base(p + i + (uint32_t)s.k - 1));
        add_hash();
      }
      const bool flip = s.both && rcode < code;
      uint32_t mh = MERS ? h[0] : 0u;
      for (int q = 1; MERS && q < kWindow; ++q) mh = q < window ? min(mh, h[q]) : mh;
      km[i] = Kmer{flip ? rcode : code, flip ? 1u : 0u, mh};
    }
    f(r, p, km, n);
  }
}

__device__ __forceinline__ void block_add(unsigned long long* dst, uint64_t v) {
  __shared__ unsigned long long acc;
  if (threadIdx.x == 0) acc = 0;
  __syncthreads();
  if (v) atomicAdd(&acc, (unsigned long long)v);
  __syncthreads();
  if (threadIdx.x == 0 && acc) atomicAdd(dst, acc);
}

// pass 1: filter A, repeats into filter B; ctr[0] += repeats, ctr[3] += the
// repeats that set new bits in B (about one per distinct repeated k-mer).
// RUNS: A's words by mh, the k-mers of a run with one atomic (eight at a time).
template <bool RUNS>
__global__ __launch_bounds__(kThreads) void k_bloom(KmerScan s, unsigned long long* A,
                                                    uint64_t WA, unsigned long long* B,
                                                    uint64_t WB, unsigned long long* ctr) {
  constexpr int kAhead = RUNS ? 8 : 1;
  const uint64_t c = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  uint32_t rep = 0, fresh = 0;
  if (c < s.n_chunks) {
    for_kmers<kAhead, RUNS>(s, c, [&](uint32_t, uint32_t, const Kmer* km, int n) {
      // each k-mer's bits, with those of the run's k-mers after it, and what the
      // word held before it
      unsigned long long bits[kAhead], all[kAhead], old[kAhead];
      uint64_t word[kAhead];
      for (int q = 0; q < kAhead; ++q) {
        const uint64_t h = fmix64(km[q].code);
        bits[q] = q < n ? bloom_bits(h) : 0ull;
        word[q] = RUNS ? run_word(km[q].mh, WA) : bloom_word(h, WA);
      }
      auto first = [&](int q) { return !RUNS || q == 0 || km[q].mh != km[q - 1].mh; };
      for (int q = kAhead - 1; q >= 0; --q)
        all[q] = bits[q] | (q + 1 < kAhead && !first(q + 1) ? all[q + 1] : 0ull);
      for (int q = 0; q < kAhead; ++q)
        if (q < n && first(q)) old[q] = atomicOr(&A[word[q]], all[q]);
      for (int q = 0; q < kAhead; ++q) {
        if (q >= n) break;
        if (!first(q)) old[q] = old[q - 1] | bits[q - 1];
        if ((old[q] & bits[q]) == bits[q]) {
          const uint64_t h2 = fmix64(km[q].code ^ kSaltB);
          const unsigned long long b2 = bloom_bits(h2);
          const unsigned long long old2 = atomicOr(&B[line_word<RUNS>(km[q].mh, h2, WB)], b2);
          ++rep;
          fresh += (old2 & b2) != b2;
        }
      }
    });
  }
  block_add(&ctr[0], rep);
  block_add(&ctr[3], fresh);
}

// ctr[1] += set bits of B
__global__ __launch_bounds__(kThreads) void k_popcount(const unsigned long long* B, uint64_t WB,
                                                       unsigned long long* ctr) {
  uint64_t n = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < WB;
       i += (uint64_t)gridDim.x * kThreads)
    n += __popcll(B[i]);
  block_add(&ctr[1], n);
}

struct Table {
  unsigned long long* keys;  // code + 1; 0 = empty
  uint32_t* cnt;             // occurrences
  uint2* loc;                // [cap * m]: the first m (read, pos) of each key, in no order
  uint64_t cap;              // power of two
  uint32_t m;
};

// pass 2: the k-mers in B into the table; ctr[2] = 1 when a key found no slot
// within kMaxProbe probes (the host then doubles the table and reruns the pass)
template <bool RUNS>
__global__ __launch_bounds__(kThreads) void k_table(KmerScan s, const unsigned long long* B,
                                                    uint64_t WB, Table t,
                                                    unsigned long long* ctr) {
  const uint64_t c = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (c >= s.n_chunks) return;
  constexpr int kAhead = 4;
  for_kmers<kAhead, RUNS>(s, c, [&](uint32_t r, uint32_t p, const Kmer* km, int n) {
    unsigned long long bits[kAhead], have[kAhead];
    for (int q = 0; q < kAhead; ++q) {
      const uint64_t h2 = fmix64(km[q].code ^ kSaltB);
      bits[q] = bloom_bits(h2);
      have[q] = B[line_word<RUNS>(km[q].mh, h2, WB)];
    }
    for (int q = 0; q < kAhead; ++q) {
      if (q >= n || (have[q] & bits[q]) != bits[q]) continue;
      const unsigned long long key = km[q].code + 1;
      uint64_t slot = fmix64(km[q].code ^ kSaltT) & (t.cap - 1);
      for (uint64_t probe = 0;; ++probe) {
        if (probe == t.cap || probe == kMaxProbe) {  // full or crowded: the host regrows it
          atomicOr(&ctr[2], 1ull);
          return;
        }
        unsigned long long cur = t.keys[slot];
        if (cur == 0) {
          cur = atomicCAS(&t.keys[slot], 0ull, key);
          if (cur == 0) cur = key;
        }
        if (cur == key) break;
        slot = (slot + 1) & (t.cap - 1);
      }
      const uint32_t i = atomicAdd(&t.cnt[slot], 1u);
      if (i < t.m) t.loc[slot * t.m + i] = make_uint2(r, (p + q) | km[q].strand << 31);
    }
  });
}

// ---- retention and pair expansion ---------------------------------------------

struct RetainCtr {
  unsigned long long keys, non_singletons, retained, occurrences;
};

// per tile of slots: retained count into blk[tile]; statistics into rc
__global__ __launch_bounds__(kThreads) void k_retain_count(Table t, uint64_t* blk,
                                                           RetainCtr* rc) {
  const uint64_t b0 = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanPer;
  uint64_t keys = 0, multi = 0, kept = 0, occ = 0;
  for (int u = 0; u < kScanPer; ++u) {
    const uint64_t s = b0 + u;
    if (s >= t.cap) break;
    const uint32_t c = t.cnt[s];
    keys += c >= 1;
    multi += c >= 2;
    if (c >= 2 && c <= t.m) {
      ++kept;
      occ += c;
    }
  }
  uint64_t total;
  block_excl_scan(kept, total);
  if (threadIdx.x == 0) blk[blockIdx.x] = total;
  block_add(&rc->keys, keys);
  block_add(&rc->non_singletons, multi);
  block_add(&rc->retained, kept);
  block_add(&rc->occurrences, occ);
}

// retained slots in slot order into ret[]; npair[i] = pairs of ret[i]'s
// locations that lie in different reads
__global__ __launch_bounds__(kThreads) void k_retain_write(Table t, const uint64_t* blk_off,
                                                           uint32_t* ret, uint64_t* npair) {
  const uint64_t b0 = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanPer;
  uint64_t kept = 0;
  for (int u = 0; u < kScanPer; ++u) {
    const uint64_t s = b0 + u;
    if (s < t.cap) {
      const uint32_t c = t.cnt[s];
      kept += c >= 2 && c <= t.m;
    }
  }
  uint64_t total;
  uint64_t idx = block_excl_scan(kept, total) + blk_off[blockIdx.x];
  for (int u = 0; u < kScanPer; ++u) {
    const uint64_t s = b0 + u;
    if (s >= t.cap) break;
    const uint32_t c = t.cnt[s];
    if (c < 2 || c > t.m) continue;
    const uint2* L = t.loc + s * t.m;
    uint64_t np = 0;
    for (uint32_t x = 0; x < c; ++x) {
      const uint32_t rx = L[x].x;
      for (uint32_t y = x + 1; y < c; ++y) np += L[y].x != rx;
    }
    ret[idx] = (uint32_t)s;
    npair[idx] = np;
    ++idx;
  }
}

// How the sort holds a seed (ra, rb, rc, pa, pb), most significant part first.
// In 64 bits when the read set's ids and positions leave room (138 Mbp: 60
// bits): half the bytes a pass (17.4 M seeds, eight passes: 1.93 -> 1.07 ms).
struct Narrow {
  using Item = uint64_t;
  uint32_t bits_r, bits_s, bits_p;  // of a read id, the strand flag (0 or 1), a position
  __device__ Item pack(uint32_t ra, uint32_t rb, uint32_t rc, uint32_t pa, uint32_t pb) const {
    const uint64_t pair = ((uint64_t)ra << bits_r | rb) << bits_s | rc;
    return (pair << bits_p | pa) << bits_p | pb;
  }
  __device__ uint64_t pair_of(Item v) const { return v >> (2 * bits_p); }
  __device__ bool same_pair(Item a, Item b) const { return pair_of(a) == pair_of(b); }
  __device__ uint32_t rc(Item v) const { return (uint32_t)pair_of(v) & ((1u << bits_s) - 1u); }
  __device__ uint2 reads(Item v) const {
    const uint64_t q = pair_of(v) >> bits_s;
    return make_uint2((uint32_t)(q >> bits_r), (uint32_t)(q & ((1ull << bits_r) - 1ull)));
  }
  __device__ uint2 seed(Item v) const {
    const uint32_t m = (1u << bits_p) - 1u;
    return make_uint2((uint32_t)(v >> bits_p) & m, (uint32_t)v & m);
  }
  __device__ static uint32_t digit(Item v, int, int shift) { return (uint32_t)(v >> shift) & 255u; }
};

// In four words otherwise: ra, rb, rc << sbit | pa, pb (sbit is above every position).
struct Wide {
  using Item = uint4;
  uint32_t sbit;
  __device__ Item pack(uint32_t ra, uint32_t rb, uint32_t rc, uint32_t pa, uint32_t pb) const {
    return make_uint4(ra, rb, rc << sbit | pa, pb);
  }
  __device__ bool same_pair(Item a, Item b) const {
    return a.x == b.x && a.y == b.y && a.z >> sbit == b.z >> sbit;
  }
  __device__ uint32_t rc(Item v) const { return v.z >> sbit; }
  __device__ uint2 reads(Item v) const { return make_uint2(v.x, v.y); }
  __device__ uint2 seed(Item v) const { return make_uint2(v.z & ((1u << sbit) - 1u), v.w); }
  __device__ static uint32_t digit(const Item& v, int field, int shift) {
    const uint32_t f = field == 0 ? v.x : field == 1 ? v.y : field == 2 ? v.z : v.w;
    return (f >> shift) & 255u;
  }
};

// one thread per retained k-mer: its seeds with ra < rb.  rc = the two
// occurrences' strand bits differ: read rb matches the reverse complement of
// read ra there, and pb counts in that reverse complement (len[rb] - k - its
// position in rb).  The flag is above every position, so the sort orders a
// pair's forward seeds before its reverse ones.
template <class F>
__global__ __launch_bounds__(kThreads) void k_emit(Table t, const uint32_t* ret, uint64_t n_ret,
                                                   const uint64_t* pair_off, const uint32_t* len,
                                                   int32_t k, F form, typename F::Item* items) {
  const uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n_ret) return;
  const uint64_t s = ret[i];
  const uint32_t c = t.cnt[s];
  const uint2* L = t.loc + s * t.m;
  uint64_t o = pair_off[i];
  for (uint32_t x = 0; x < c; ++x) {
    const uint2 a = L[x];
    for (uint32_t y = x + 1; y < c; ++y) {
      const uint2 b = L[y];
      if (a.x == b.x) continue;
      const uint2 lo = a.x < b.x ? a : b, hi = a.x < b.x ? b : a;
      const uint32_t rc = (lo.y ^ hi.y) >> 31;
      const uint32_t pa = lo.y & 0x7fffffffu, p_hi = hi.y & 0x7fffffffu;
      const uint32_t pb = rc ? len[hi.x] - (uint32_t)k - p_hi : p_hi;
      items[o++] = form.pack(lo.x, hi.x, rc, pa, pb);
    }
  }
}

// ---- LSD radix sort of (ra, rb, rc, pa, pb) ---------------------------------------

// hist[d * n_tiles + tile] = items of the tile with digit d
template <class F>
__global__ __launch_bounds__(kThreads) void k_sort_hist(const typename F::Item* in, uint64_t n,
                                                        int field, int shift, uint32_t* hist) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t b0 = (uint64_t)blockIdx.x * kSortTile;
  for (int u = 0; u < kSortPer; ++u) {
    const uint64_t i = b0 + (uint64_t)u * kThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[F::digit(in[i], field, shift)], 1u);
  }
  __syncthreads();
  hist[(uint64_t)threadIdx.x * gridDim.x + blockIdx.x] = h[threadIdx.x];
}

// stable scatter: the tile's items with digit d go to out[off[d * n_tiles +
// tile] ...] in their input order.  Each round ranks 256 items: within a wave
// by matching digits over eight ballots, across the block's four waves by
// per-wave digit counts in LDS.
template <class F>
__global__ __launch_bounds__(kThreads) void k_sort_scatter(const typename F::Item* in,
                                                           typename F::Item* out, uint64_t n,
                                                           int field, int shift,
                                                           const uint32_t* off) {
  constexpr int kWaves = kThreads / 64;
  __shared__ uint32_t run[256];
  __shared__ uint32_t wcnt[kWaves][256];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  run[t] = off[(uint64_t)t * gridDim.x + blockIdx.x];
  for (int w = 0; w < kWaves; ++w) wcnt[w][t] = 0;
  __syncthreads();
  const uint64_t b0 = (uint64_t)blockIdx.x * kSortTile;
  for (int u = 0; u < kSortPer; ++u) {
    const uint64_t i = b0 + (uint64_t)u * kThreads + t;
    const bool valid = i < n;
    const typename F::Item v = valid ? in[i] : typename F::Item{};
    const uint32_t d = valid ? F::digit(v, field, shift) : 0;
    uint64_t peers = __builtin_amdgcn_ballot_w64(valid);
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __builtin_amdgcn_ballot_w64(bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
    (void)lane;
    if (valid && below == 0) wcnt[wave][d] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t pos = run[d] + below;
      for (int w = 0; w < wave; ++w) pos += wcnt[w][d];
      out[pos] = v;
    }
    __syncthreads();
    uint32_t sum = 0;
    for (int w = 0; w < kWaves; ++w) {
      sum += wcnt[w][t];
      wcnt[w][t] = 0;
    }
    run[t] += sum;
    __syncthreads();
  }
}

// ---- output -------------------------------------------------------------------

// a new pair starts where (ra, rb, rc) changes
template <class F>
__global__ __launch_bounds__(kThreads) void k_heads(const typename F::Item* items, uint64_t n,
                                                    F form, uint32_t* flag) {
  const uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  flag[i] = i == 0 || !form.same_pair(items[i], items[i - 1]);
}

// head[] is the exclusive scan of the head flags (n + 1 entries); rc may be
// null (forward strand only)
template <class F>
__global__ __launch_bounds__(kThreads) void k_csr(const typename F::Item* items, uint64_t n,
                                                  const uint32_t* head, F form,
                                                  uint32_t* pairs, uint8_t* rc,
                                                  uint64_t* seed_off, uint32_t* seeds) {
  const uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const typename F::Item v = items[i];
  const uint32_t p = head[i];
  if (head[i + 1] != p) {
    const uint2 r = form.reads(v);
    pairs[2 * (uint64_t)p] = r.x;
    pairs[2 * (uint64_t)p + 1] = r.y;
    if (rc) rc[p] = (uint8_t)form.rc(v);
    seed_off[p] = i;
  }
  const uint2 q = form.seed(v);
  seeds[2 * i] = q.x;
  seeds[2 * i + 1] = q.y;
  if (i == 0) seed_off[head[n]] = n;
}

// ---- host ---------------------------------------------------------------------

// the stage's device buffers, kept between calls (xd_release_memory frees them)
constexpr int kMaxDevices = 64;
std::mutex g_cache_mu[kMaxDevices];
xscan::BlockCache g_cache[kMaxDevices];

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  return xd_internal_fail(code, buf);
}

int hip_fail(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? XD_ENOMEM : XD_EDEVICE, "xd_find_overlaps: %s: %s",
              what, hipGetErrorString(e));
}

#define OV_TRY(call)                                  \
  do {                                                \
    hipError_t e_ = (call);                           \
    if (e_ != hipSuccess) return hip_fail(e_, #call); \
  } while (0)

template <typename T>
int fetch(hipStream_t st, const T* dev, T* host, uint64_t count = 1) {
  OV_TRY(hipMemcpyAsync(host, dev, count * sizeof(T), hipMemcpyDeviceToHost, st));
  OV_TRY(hipStreamSynchronize(st));
  return XD_OK;
}

uint32_t bit_length(uint64_t v) { return v ? 64u - (uint32_t)__builtin_clzll(v) : 0u; }

}  // namespace

namespace {

// the retained k-mers and their seeds' places
struct Seeds {
  Table t;
  const uint32_t* ret;
  const uint64_t* npair;
  uint64_t retained, seeds;
  const uint32_t* len;
  int32_t k;
};

// the sort's fields, least significant first, and their bits
struct Digits {
  int n;
  int field[4];
  uint32_t bits[4];
};

// where the pairs go, when they fit (pairs null: nowhere)
struct Csr {
  uint64_t max_pairs, max_seeds;
  uint32_t* pairs;
  uint8_t* rc;
  uint64_t* seed_off;
  uint32_t* seeds;
};

// lists the seeds, sorts them, counts the pairs and writes them out
template <class F>
int sort_seeds(Arena& ar, hipStream_t st, const Seeds& in, F form, const Digits& dg,
               const Csr& out, uint64_t* n_pairs) {
  using Item = typename F::Item;
  const uint64_t S = in.seeds;
  Item *cur = nullptr, *alt = nullptr;
  OV_TRY(ar.get(&cur, S));
  OV_TRY(ar.get(&alt, S));
  hipLaunchKernelGGL(k_emit<F>, dim3(grid_for(in.retained, kThreads)), dim3(kThreads), 0, st, in.t,
                     in.ret, in.retained, in.npair, in.len, in.k, form, cur);
  const uint32_t nt = grid_for(S, kSortTile);
  uint32_t* hist = nullptr;
  OV_TRY(ar.get(&hist, (uint64_t)nt * 256 + 1));
  for (int fi = 0; fi < dg.n; ++fi)
    for (uint32_t sh = 0; sh < dg.bits[fi]; sh += 8) {
      hipLaunchKernelGGL(k_sort_hist<F>, dim3(nt), dim3(kThreads), 0, st, cur, S, dg.field[fi],
                         (int)sh, hist);
      OV_TRY(xscan::exclusive_scan<uint32_t>(ar, hist, hist, (uint64_t)nt * 256));
      hipLaunchKernelGGL(k_sort_scatter<F>, dim3(nt), dim3(kThreads), 0, st, cur, alt, S,
                         dg.field[fi], (int)sh, hist);
      std::swap(cur, alt);
    }
  uint32_t* head = nullptr;
  OV_TRY(ar.get(&head, S + 1));
  hipLaunchKernelGGL(k_heads<F>, dim3(grid_for(S, kThreads)), dim3(kThreads), 0, st, cur, S, form,
                     head);
  OV_TRY(xscan::exclusive_scan<uint32_t>(ar, head, head, S));
  uint32_t P = 0;
  if (int rc = fetch(st, head + S, &P)) return rc;
  *n_pairs = P;
  if (out.pairs && P <= out.max_pairs && S <= out.max_seeds)
    hipLaunchKernelGGL(k_csr<F>, dim3(grid_for(S, kThreads)), dim3(kThreads), 0, st, cur, S, head,
                       form, out.pairs, out.rc, out.seed_off, out.seeds);
  return XD_OK;
}

int find_overlaps(const xd_store* store, int32_t k, uint32_t m, uint32_t bloom_bits,
                  uint64_t table_slots, int32_t strands, uint64_t max_pairs, uint32_t* pairs,
                  uint8_t* rc_out, uint64_t* seed_off, uint64_t max_seeds, uint32_t* seeds,
                  xd_overlap_counts* counts, void* hip_stream) {
  if (strands != 1 && strands != 2)
    return fail(XD_EINVAL, "xd_find_overlaps: strands must be 1 or 2 (got %d)", strands);
  StoreView sv;
  int rc = xd_internal_store_view(store, &sv);
  if (rc) return rc;
  if (k < 1 || k > XD_OVERLAP_K_MAX)
    return fail(XD_EINVAL, "xd_find_overlaps: k must be in [1, %d] (got %d)", XD_OVERLAP_K_MAX, k);
  if (m < 1 || m > XD_OVERLAP_M_MAX)
    return fail(XD_EINVAL, "xd_find_overlaps: m must be in [1, %d] (got %u)", XD_OVERLAP_M_MAX, m);
  if (bloom_bits == 0) bloom_bits = 16;
  if (bloom_bits < 4 || bloom_bits > 64)
    return fail(XD_EINVAL, "xd_find_overlaps: bloom_bits must be 0 or in [4, 64] (got %u)",
                bloom_bits);
  const bool write = pairs || seed_off || seeds;
  if (write && !(pairs && seed_off && seeds))
    return fail(XD_EINVAL, "xd_find_overlaps: pairs, seed_off and seeds must all be given or "
                           "all be NULL");
  if (write && strands == 2 && !rc_out)
    return fail(XD_EINVAL, "xd_find_overlaps: both strands need the rc output");
  if (strands == 1) rc_out = nullptr;
  hipStream_t st = (hipStream_t)hip_stream;
  xd_overlap_counts cn = {};
  // one call at a time per device: its buffers come from the device's cache
  int dev = 0;
  OV_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(XD_EINVAL, "xd_find_overlaps: device %d", dev);
  std::lock_guard<std::mutex> call_lock(g_cache_mu[dev]);

  // chunks of kChunk k-mer starts, per read
  std::vector<uint64_t> chunk_off((size_t)sv.n_reads + 1);
  uint64_t n_chunks = 0;
  for (uint32_t r = 0; r < sv.n_reads; ++r) {
    chunk_off[r] = n_chunks;
    const uint32_t L = sv.host_len[r];
    if (L >= (uint32_t)k) {
      cn.kmers += L - (uint32_t)k + 1;
      n_chunks += (L - (uint32_t)k + 1 + kChunk - 1) / kChunk;
    }
  }
  chunk_off[sv.n_reads] = n_chunks;
  if (cn.kmers >= 0xffffffffull)
    return fail(XD_EINVAL, "xd_find_overlaps: %llu k-mers (limit 2^32 - 2)",
                (unsigned long long)cn.kmers);

  Arena ar(st, &g_cache[dev]);
  if (cn.kmers > 0) {
    const uint64_t WA = (cn.kmers * bloom_bits + 63) / 64;
    const uint64_t WB = (WA / 16 + 64 + kLine - 1) & ~(kLine - 1);
    uint64_t* d_chunk = nullptr;
    unsigned long long *A = nullptr, *B = nullptr, *ctr = nullptr;
    OV_TRY(ar.get(&d_chunk, chunk_off.size()));
    OV_TRY(ar.get(&A, WA));
    OV_TRY(ar.get(&B, WB));
    OV_TRY(ar.get(&ctr, 4));
    OV_TRY(hipMemcpyAsync(d_chunk, chunk_off.data(), chunk_off.size() * 8, hipMemcpyHostToDevice,
                          st));
    OV_TRY(hipMemsetAsync(A, 0, WA * 8, st));
    OV_TRY(hipMemsetAsync(B, 0, WB * 8, st));
    OV_TRY(hipMemsetAsync(ctr, 0, 4 * 8, st));
    // up to kWindow m-mers to a k-mer, and eight to a word
    const bool runs = WA <= kRunWords;
    int32_t mm = 1;
    while (mm < 16 && (1ull << (2 * mm)) < 8 * WA) ++mm;
    mm = std::min(k, std::max(k - kWindow + 1, mm));
    KmerScan ks{sv.words, sv.word_off, sv.len, d_chunk, n_chunks, sv.n_reads, k,
                k == 32 ? ~0ull : (1ull << (2 * k)) - 1, strands == 2 ? 1 : 0, mm,
                mm == 32 ? ~0ull : (1ull << (2 * mm)) - 1};
    hipLaunchKernelGGL(runs ? k_bloom<true> : k_bloom<false>,
                       dim3(grid_for(n_chunks, kThreads)), dim3(kThreads), 0, st, ks, A, WA, B, WB,
                       ctr);
    hipLaunchKernelGGL(k_popcount, dim3(grid_for(WB, kThreads * 16)), dim3(kThreads), 0, st, B,
                       WB, ctr);
    unsigned long long h_ctr[4];
    if ((rc = fetch(st, ctr, h_ctr, 4))) return rc;
    cn.bloom_repeats = h_ctr[0];
    ar.drop(A);

    // table size: the repeats that set new bits in B count the k-mers
    // occurring twice or more (fewer only where B's bits collide); the
    // singletons passing B are estimated from B's fill (three bits per key);
    // 1.5 times that keeps the expected load near 2/3, and a table that
    // still fills up is regrown
    const double f = (double)h_ctr[1] / (64.0 * (double)WB);
    const double expect = (double)h_ctr[3] + 2.0 * f * f * f * (double)cn.kmers;
    uint64_t cap = 4096;
    if (table_slots) {
      while (cap < table_slots && cap < (1ull << 32)) cap <<= 1;
    } else {
      while ((double)cap < 1.5 * expect + 1024.0) cap <<= 1;
    }

    Table t{};
    t.m = m;
    for (;;) {
      t.cap = cap;
      OV_TRY(ar.get(&t.keys, cap));
      OV_TRY(ar.get(&t.cnt, cap));
      OV_TRY(ar.get(&t.loc, cap * m));
      OV_TRY(hipMemsetAsync(t.keys, 0, cap * 8, st));
      OV_TRY(hipMemsetAsync(t.cnt, 0, cap * 4, st));
      OV_TRY(hipMemsetAsync(ctr + 2, 0, 8, st));
      hipLaunchKernelGGL(runs ? k_table<true> : k_table<false>,
                         dim3(grid_for(n_chunks, kThreads)), dim3(kThreads), 0, st, ks, B, WB, t,
                         ctr);
      unsigned long long full = 0;
      if ((rc = fetch(st, ctr + 2, &full))) return rc;
      if (!full) break;
      ar.drop(t.keys);  // a key found no free slot: double the table and rerun
      ar.drop(t.cnt);
      ar.drop(t.loc);
      if (cap >= (1ull << 32)) return fail(XD_ENOMEM, "xd_find_overlaps: hash table overflow");
      cap <<= 1;
    }
    ar.drop(B);
    cn.table_slots = cap;

    // retention
    const uint32_t nb = grid_for(cap, kScanTile);
    uint64_t* blk = nullptr;
    RetainCtr* d_rc = nullptr;
    OV_TRY(ar.get(&blk, (uint64_t)nb + 1));
    OV_TRY(ar.get(&d_rc, 1));
    OV_TRY(hipMemsetAsync(d_rc, 0, sizeof(RetainCtr), st));
    hipLaunchKernelGGL(k_retain_count, dim3(nb), dim3(kThreads), 0, st, t, blk, d_rc);
    OV_TRY(xscan::exclusive_scan<uint64_t>(ar, blk, blk, nb));
    RetainCtr h_rc;
    if ((rc = fetch(st, d_rc, &h_rc))) return rc;
    cn.table_keys = h_rc.keys;
    cn.non_singletons = h_rc.non_singletons;
    cn.retained = h_rc.retained;
    cn.occurrences = h_rc.occurrences;

    uint32_t* ret = nullptr;     // retained slots
    uint64_t* npair = nullptr;   // per retained k-mer: seed count, then first seed
    if (cn.retained > 0) {
      OV_TRY(ar.get(&ret, cn.retained));
      OV_TRY(ar.get(&npair, cn.retained + 1));
      hipLaunchKernelGGL(k_retain_write, dim3(nb), dim3(kThreads), 0, st, t, blk, ret, npair);
      OV_TRY(xscan::exclusive_scan<uint64_t>(ar, npair, npair, cn.retained));
      if ((rc = fetch(st, npair + cn.retained, &cn.seeds))) return rc;
      if (cn.seeds >= 0xffffffffull)
        return fail(XD_EINVAL, "xd_find_overlaps: %llu seeds (limit 2^32 - 2); lower m",
                    (unsigned long long)cn.seeds);
    }

    if (cn.seeds > 0) {
      // read ids take bits_r bits, positions bits_p, the strand flag one
      const uint32_t bits_r = bit_length(sv.n_reads ? sv.n_reads - 1 : 0);
      const uint32_t bits_p = bit_length(sv.max_len);
      const uint32_t bits_s = strands == 2 ? 1u : 0u;
      const uint32_t bits = 2 * bits_r + bits_s + 2 * bits_p;
      const Seeds in{t, ret, npair, cn.retained, cn.seeds, sv.len, k};
      const Csr out{write ? max_pairs : 0, write ? max_seeds : 0, pairs, rc_out, seed_off, seeds};
      if (bits <= 64) {
        const Digits d{1, {0}, {bits}};
        rc = sort_seeds(ar, st, in, Narrow{bits_r, bits_s, bits_p}, d, out, &cn.pairs);
      } else {  // least significant field first
        const Digits d{4, {3, 2, 1, 0}, {bits_p, bits_p + bits_s, bits_r, bits_r}};
        rc = sort_seeds(ar, st, in, Wide{bits_p}, d, out, &cn.pairs);
      }
      if (rc) return rc;
    }
  }
  if (counts) *counts = cn;
  if (write && (cn.pairs > max_pairs || cn.seeds > max_seeds))
    return fail(XD_EAGAIN, "xd_find_overlaps: outputs hold %llu pairs / %llu seeds, need %llu / %llu",
                (unsigned long long)max_pairs, (unsigned long long)max_seeds,
                (unsigned long long)cn.pairs, (unsigned long long)cn.seeds);
  if (write && cn.seeds == 0) OV_TRY(hipMemsetAsync(seed_off, 0, 8, st));
  hipError_t le = hipGetLastError();
  if (le != hipSuccess) return hip_fail(le, "kernel launch");
  OV_TRY(hipStreamSynchronize(st));
  return XD_OK;
}

}  // namespace

extern "C" int xd_find_overlaps(const xd_store* store, int32_t k, uint32_t m, uint32_t bloom_bits,
                                uint64_t table_slots, uint64_t max_pairs, uint32_t* pairs,
                                uint64_t* seed_off, uint64_t max_seeds, uint32_t* seeds,
                                xd_overlap_counts* counts, void* hip_stream) {
  return find_overlaps(store, k, m, bloom_bits, table_slots, 1, max_pairs, pairs, nullptr,
                       seed_off, max_seeds, seeds, counts, hip_stream);
}

extern "C" int xd_find_overlaps_strands(const xd_store* store, int32_t k, uint32_t m,
                                        uint32_t bloom_bits, uint64_t table_slots,
                                        int32_t strands, uint64_t max_pairs, uint32_t* pairs,
                                        uint8_t* rc, uint64_t* seed_off, uint64_t max_seeds,
                                        uint32_t* seeds, xd_overlap_counts* counts,
                                        void* hip_stream) {
  return find_overlaps(store, k, m, bloom_bits, table_slots, strands, max_pairs, pairs, rc,
                       seed_off, max_seeds, seeds, counts, hip_stream);
}

// frees the stage's kept buffers on every device (for xd_release_memory)
__attribute__((visibility("hidden"))) void xd_internal_overlap_release() {
  for (int d = 0; d < kMaxDevices; ++d) {
    std::lock_guard<std::mutex> lk(g_cache_mu[d]);
    if (g_cache[d].blocks.empty()) continue;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(d);
    g_cache[d].release();
    (void)hipSetDevice(cur);
  }
}
