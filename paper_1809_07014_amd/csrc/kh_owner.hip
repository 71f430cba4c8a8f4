// Owner-partitioned counting: the k-mer analysis of Section II-B laid out the
// way the paper distributes it.  There, every k-mer is sent to the process
// that owns it, and each owner runs the two-pass Bloom screen and the
// hash-table count over its own k-mers in local memory.  Here an owner is a
// range of key prefixes small enough for one workgroup, and the owner's local
// memory is that workgroup's LDS.
//
// Routing (the all-to-all exchange of the paper) is two streaming radix
// partitions over the key prefix: the windows' records go to 2^p1 level-1
// buckets (the top p1 key bits), then each bucket is split by its next p2_b
// bits into owners of a few thousand records (p2_b chosen per bucket from its
// size).  Every pass writes contiguous runs at offsets from a scanned
// histogram matrix, so no device-scope atomic touches a random address.  An
// owner workgroup then counts its records in LDS, where the keys seen once are
// told apart exactly (the few owners of too many records for that run Bloom
// pass A and count pass B), and classifies the kept k-mers; the copy of the
// owners' rows into the table sorts each owner's rows, and the owners'
// prefixes are disjoint and in key order, so sorting within owners orders the
// whole table.
//
// A record is one window: its canonical key without the level-1 digit (the
// bucket implies those bits), shifted left by 6 bits with the extension byte
// (left valid, left base, right valid, right base) below it, as
// R = own_record_words(k) words, most significant first.  Owners count these
// partial keys (they share the digit) and put the digit back when
// they write their rows.
#include <algorithm>

#include "kh_internal.hpp"

namespace kh {

// ------------------------------------------------------------ helpers ----

// Bits [pos, pos + len) (MSB-first, 0 <= len <= 32) of an N-word value held
// in registers, most significant word first.  Indexes are static.
template <int N>
__device__ __forceinline__ uint32_t top_bits(const uint64_t (&v)[N], int pos, int len) {
  if (len <= 0) return 0u;
  const int q = pos >> 6, r = pos & 63;
  uint64_t hi = 0;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i == q) hi = v[i] << r;
  if (r + len > 64) {
#pragma unroll
    for (int i = 0; i + 1 < N; ++i)
      if (i == q) hi |= v[i + 1] >> (64 - r);
  }
  return (uint32_t)(hi >> (64 - len));
}

// (key << 6) | e6 as R words (R = W or W + 1).
template <int W, int R>
__device__ __forceinline__ void make_record(const uint64_t (&f)[W], uint32_t e6,
                                            uint64_t (&v)[R]) {
#pragma unroll
  for (int j = 0; j < R; ++j) {  // j counts words from the least significant
    const uint64_t cur = j < W ? f[W - 1 - j] : 0ull;
    const uint64_t low = j == 0 ? (uint64_t)e6 : (j - 1 < W ? f[W - j] >> 58 : 0ull);
    v[R - 1 - j] = (cur << 6) | low;
  }
}

// The key of a record (record >> 6) as R words, most significant first.
template <int R>
__device__ __forceinline__ void record_key(const uint64_t (&v)[R], uint64_t (&key)[R]) {
#pragma unroll
  for (int j = 0; j < R; ++j)
    key[j] = (v[j] >> 6) | (j > 0 ? v[j - 1] << 58 : 0ull);
}

template <int R>
__device__ __forceinline__ void load_record(const uint64_t* __restrict__ rec, uint64_t r,
                                            uint64_t (&v)[R]) {
  if (R == 2) {
    const uint4 x = reinterpret_cast<const uint4*>(rec)[r];
    v[0] = (uint64_t)x.x | ((uint64_t)x.y << 32);
    v[R - 1] = (uint64_t)x.z | ((uint64_t)x.w << 32);
  } else {
#pragma unroll
    for (int w = 0; w < R; ++w) v[w] = rec[r * R + w];
  }
}

// The next window's words: base b enters at the right of the forward words
// and, complemented, at the left of the reverse complement (k-base values,
// W words most significant first, the top word holding 2k - 64 (W - 1) bits).
template <int W>
__device__ __forceinline__ void roll_words(uint64_t (&f)[W], uint64_t (&r)[W], uint32_t b,
                                           uint32_t k) {
  const int tb = 2 * (int)k - 64 * (W - 1);  // 2 .. 64
  const uint64_t tmask = tb >= 64 ? ~0ull : (1ull << tb) - 1ull;
#pragma unroll
  for (int j = 0; j < W; ++j) f[j] = (f[j] << 2) | (j + 1 < W ? f[j + 1] >> 62 : (uint64_t)b);
  f[0] &= tmask;
#pragma unroll
  for (int j = W - 1; j > 0; --j) r[j] = (r[j] >> 2) | (r[j - 1] << 62);
  r[0] = (r[0] >> 2) | ((uint64_t)(3u - b) << (tb - 2));
}

// Records of a batch starting at record b0 that lane `tid` holds (records
// b0 + q x kOwnThreads + tid for q < the result, at most NB) when the
// owner's records end at r1.
template <int NB>
__device__ __forceinline__ int lane_records(uint64_t b0, uint64_t r1, int tid) {
  const uint64_t first = b0 + (uint64_t)tid;
  if (first >= r1) return 0;
  const uint64_t n = (r1 - first + kOwnThreads - 1) / kOwnThreads;
  return n < (uint64_t)NB ? (int)n : NB;
}

// Hash of a key held as stored chunks, for the LDS table and the Bloom
// filter of one owner (whose keys share their prefix; only the other bits
// vary): a multiply-add over the chunks and one xor-shift.  Slot index: its
// top 32 bits scaled to the table; Bloom word and four pattern bits: two
// 32-bit multiply-xorshift steps on its low half.
template <int C>
__device__ __forceinline__ uint64_t owner_hash(const uint64_t (&ch)[C], int ws) {
  const uint64_t K[5] = {0x9e3779b97f4a7c15ull, 0xc2b2ae3d27d4eb4full, 0x165667b19e3779f9ull,
                         0xd6e8feb86659fd93ull, 0xff51afd7ed558ccdull};
  uint64_t h = 0;
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (c < ws) h += ch[c] * K[c];
  return h ^ (h >> 29);
}

__device__ __forceinline__ void owner_bloom(uint64_t h, uint32_t& bi, uint32_t& pat) {
  uint32_t t = (uint32_t)h * 0x85ebca6bu;
  t ^= t >> 13;
  bi = t >> (32 - kOwnBloomBits);
  const uint32_t u = (t ^ (t >> 16)) * 0xc2b2ae35u;
  pat = (1u << (u & 31)) | (1u << ((u >> 5) & 31)) | (1u << ((u >> 10) & 31)) |
        (1u << ((u >> 15) & 31));
}

// Barrier for LDS exchange only: it waits for this wave's LDS operations but
// not for its outstanding global loads and stores, which the fence in
// __syncthreads would wait for (a full memory round trip at every barrier).
// Used where the waves of a block share data through LDS alone.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Exclusive scan of one value per thread over the block (blockDim.x a
// multiple of 64, at most 1024); returns the block total.  s_w holds one
// word per wave.  Every thread calls it.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t& excl,
                                                    uint32_t* s_w) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nw = (int)(blockDim.x >> 6);
  uint32_t incl = x;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  lds_barrier();
  if (lane == 63) s_w[wave] = incl;
  lds_barrier();
  uint32_t off = 0, total = 0;
  for (int w = 0; w < nw; ++w) {
    const uint32_t s = s_w[w];
    if (w < wave) off += s;
    total += s;
  }
  excl = off + incl - x;
  return total;
}

// ------------------------------------------------------ level 1 route ----

// x << s over three words, most significant first, 0 <= s < 64.
__device__ __forceinline__ void shl3(const uint64_t (&x)[3], int s, uint64_t (&y)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
    y[i] = s == 0 ? x[i] : (x[i] << s) | (i < 2 ? x[i + 1] >> (64 - s) : 0ull);
}

// The windows of one k as three bit planes indexed by window start, 64 starts
// per thread: win (it is a k-mer: no non-base in [p, p + k), no read start in
// (p, p + k)), lx (its left neighbour is an extension: p starts no read and
// base p - 1 is of high quality) and rx (likewise base p + k).  A run of k - 1
// set-or-not bits is a shifted OR doubled log2(k) times, so 64 windows cost
// what one costs when each looks at its own k bits; the routing passes then
// read one bit per window and plane.  Positions from n on are marked as
// non-bases, so windows that end past n are none.
//
// Bound by the planes: 3/8 byte in and 3/8 out per base; 1.5e9 bases 0.30 ms.
__global__ __launch_bounds__(kBlock) void k_own_planes(OwnRouteArgs a) {
  const int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (w >= (a.n + 63) / 64) return;
  const int k = (int)a.k;
  uint64_t c[3], t[3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
    c[i] = w + i < a.plane_words ? a.bad[w + i] | a.st[w + i] : ~0ull;
  uint64_t x[3] = {0, 0, 0};
  if (k > 1) {  // any of the next k - 1 positions
    shl3(c, 1, x);
    int m = 1;
    while (2 * m <= k - 1) {
      shl3(x, m, t);
#pragma unroll
      for (int i = 0; i < 3; ++i) x[i] |= t[i];
      m *= 2;
    }
    shl3(x, k - 1 - m, t);
    x[0] |= t[0];
  }
  a.win[w] = ~(a.bad[w] | x[0]);
  a.lx[w] = ((a.hq[w] >> 1) | (w > 0 ? a.hq[w - 1] << 63 : 0ull)) & ~a.st[w];
  uint64_t y[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t g = w + (k >> 6) + i;
    y[i] = g < a.plane_words ? a.hq[g] & ~a.st[g] : 0ull;
  }
  const int s = k & 63;  // k is odd: 1 .. 63
  a.rx[w] = (y[0] << s) | (y[1] >> (64 - s));
}

// h mod d with inv = floor((2^64 - 1) / d): the estimate of the quotient is
// at most one (two for the inverse's own rounding) short.
__device__ __forceinline__ uint32_t mod_u32(uint64_t h, uint32_t d, uint64_t inv) {
  uint64_t r = h - __umul64hi(h, inv) * d;
  if (r >= d) r -= d;
  if (r >= d) r -= d;
  return (uint32_t)r;
}

// A key-space part (owner of shards): the windows of other parts leave the
// win plane, four consecutive windows a thread, so that the histogram and the
// emit route only the part's own and no key is hashed twice.
//
// Bound by forming and hashing every window's key (VALU).  5.6e8 windows of
// k = 77, part 0 of 8: 2.4 ms, and histogram and emit 0.3 and 2.8 ms; when
// both formed and hashed every key (with a 64-bit division) they took 7.0 and
// 7.9 ms.
template <int W>
__global__ __launch_bounds__(kBlock) void k_own_part_filter(OwnRouteArgs a, uint64_t inv) {
  const int64_t words = (a.n + 63) / 64;
  for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < 16 * words;
       g += (int64_t)gridDim.x * kBlock) {
    const int64_t p0 = 4 * g, w = p0 >> 6;
    const uint32_t v4 = (uint32_t)(a.win[w] >> (60 - (p0 & 63))) & 15u;
    uint32_t keep = 0;
    if (v4) {
      uint64_t fw[W], rw[W];
      window_words<W>(a.bases + (p0 >> 5), 2 * (uint32_t)(p0 & 31), a.k, fw);
      revcomp_words<W>(fw, a.k, rw);
      const int64_t q0 = p0 + a.k;
      const uint32_t rb = (uint32_t)get_bits(a.bases + (q0 >> 5), 2 * (uint32_t)(q0 & 31), 8);
#pragma unroll
      for (int pw = 0; pw < 4; ++pw) {
        if (pw > 0) roll_words<W>(fw, rw, (rb >> (8 - 2 * pw)) & 3u, a.k);
        if (!((v4 >> (3 - pw)) & 1u)) continue;
        const bool use_rc = words_less<W>(rw, fw);
        uint64_t h = 0;
#pragma unroll
        for (int j = 0; j < W; ++j) h = splitmix_out(h ^ (use_rc ? rw[j] : fw[j]));
        if (mod_u32(h, a.shards, inv) == a.owner) keep |= 8u >> pw;
      }
    }
    uint64_t m = (uint64_t)keep << (60 - (p0 & 63));  // 16 lanes hold a word
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) m |= __shfl_xor((unsigned long long)m, o);
    if ((threadIdx.x & 15) == 0) a.win[w] = m;
  }
}

// Routing tiles: kOwnTile consecutive window starts, four of them per lane.
constexpr int kOwnLane = 4;
constexpr int kOwnTile = kOwnRouteThreads * kOwnLane;

// Level-1 histogram: block b counts the buckets of the windows of routing
// tiles b, b + grid, ... (the tiles the emit kernel gives the same block)
// into column b of the bucket-major matrix h1[bucket * grid + b].  The top p1
// bits of a canonical key are the smaller of the window's first p1 / 2 bases
// and the reverse complement of its last p1 / 2 (when the two are equal, the
// key starts with them whichever strand it is read on), so no key is formed:
// a thread walks 32 consecutive windows and shifts one base into each of the
// two digits.
//
// Bound by the LDS histogram's atomics and the base stream (3/8 byte per
// window).  1.3e9 windows of k = 21: 0.85 ms (5.4 ms with every window's
// digits and validity bits read from a staged tile).
constexpr int kHistTile = kOwnTile / 32;                     // threads per routing tile
constexpr int kHistTiles = kOwnRouteThreads / kHistTile;     // tiles a block takes at once

__global__ __launch_bounds__(kOwnRouteThreads) void k_own_hist(OwnRouteArgs a) {
  __shared__ uint32_t s_h[kOwnL1Max];
  __shared__ uint64_t s_red[kOwnRouteThreads / 64];
  const int tid = threadIdx.x;
  const int nbins = 1 << a.p1;
  for (int i = tid; i < nbins; i += kOwnRouteThreads) s_h[i] = 0;
  lds_barrier();
  const int64_t n_tiles = (a.n + kOwnTile - 1) / kOwnTile;
  const uint32_t p1 = a.p1, nb = p1 >> 1, dmask = (1u << p1) - 1u;
  uint64_t nwin = 0;
  for (int64_t t = blockIdx.x + (int64_t)(tid / kHistTile) * gridDim.x; t < n_tiles;
       t += (int64_t)kHistTiles * gridDim.x) {
    const int64_t p0 = t * kOwnTile + 32 * (tid % kHistTile);
    if (p0 >= a.n) continue;
    const uint32_t v = (uint32_t)(a.win[p0 >> 6] >> (32 - (p0 & 63)));
    if (!v) continue;
    nwin += __popc(v);
    // fx: the bases that enter the first digit, tx: those that enter the last
    const int64_t q0 = p0 + nb - 1, e0 = p0 + a.k - 1;
    const uint64_t* fb = a.bases + (q0 >> 5);
    const uint64_t* tb = a.bases + (e0 >> 5);
    const uint64_t fx = get_bits(fb, 2 * (uint32_t)(q0 & 31), 64);
    const uint64_t tx = get_bits(tb, 2 * (uint32_t)(e0 & 31), 64);
    uint32_t f = 0, r = 0;
    if (nb > 1) {  // the first window's other nb - 1 bases
      f = (uint32_t)(a.bases[p0 >> 5] >> (64 - 2 * (nb - 1)));
      const int64_t l0 = e0 - (nb - 1);
      const uint32_t l = (uint32_t)get_bits(a.bases + (l0 >> 5), 2 * (uint32_t)(l0 & 31),
                                            2 * (nb - 1));
      for (uint32_t j = 0; j < nb - 1; ++j)  // base j of l: place j + 1 from the low end
        r |= (3u - ((l >> (2 * (nb - 2 - j))) & 3u)) << (2 * (j + 1));
    }
#pragma unroll 8
    for (int i = 0; i < 32; ++i) {
      f = ((f << 2) | ((uint32_t)(fx >> (62 - 2 * i)) & 3u)) & dmask;
      r = (r >> 2) | ((3u - ((uint32_t)(tx >> (62 - 2 * i)) & 3u)) << (p1 - 2));
      if ((v >> (31 - i)) & 1u) atomicAdd(&s_h[f < r ? f : r], 1u);
    }
  }
  lds_barrier();
  for (int i = tid; i < nbins; i += kOwnRouteThreads)
    a.h1[(uint64_t)i * gridDim.x + blockIdx.x] = s_h[i];
  if (blockIdx.x == 0 && tid == 0) a.h1[(uint64_t)nbins * gridDim.x] = 0;  // the total, scanned
  block_add(&a.ctr[kCtrWindows], nwin, s_red);
}

// Level-1 emit: the same routing tiles as k_own_hist, taken in batches (three
// tiles for one-word records, two for two words, else one: what the LDS
// holds).  A lane forms four consecutive
// windows of a tile, the first one's words read from the staged bases, each
// next one's by shifting one base in, and keeps their records; the bucket
// counts' atomics return each record's rank in its bucket, so after a scan of
// the counts the records go to LDS in bucket order and leave as one
// contiguous run per bucket at the block's cursors (the scanned matrix
// column): HBM sees whole lines rather than scattered 8-byte stores.
//
// One-word records are bound by the LDS exchange and its barriers at one block
// per CU, longer ones more and more by their stores.  10M reads of 150 bases:
// k = 21, 33, 55, 77, 99 take 7.3, 7.5, 9.3, 12.4 and 10.9 ms, from 14.1,
// 15.7, 17.4, 19.0 and 19.4 ms when each window looked up its own validity and
// extension bits and a record's bucket place was found by a second atomic.
template <int R>
struct EmitBatch {
  static constexpr int kTiles = R == 1 ? 3 : R == 2 ? 2 : 1;  // routing tiles
  static constexpr int kCap = kTiles * kOwnTile;      // records per batch
};

// Words staged per tile: its bases from 32 before it (the left neighbour of
// its first window) to the right neighbour of its last (k <= 127), then 64
// words of each plane.  One word per thread, loaded a tile ahead.
constexpr int kOwnBaseWords = (32 + kOwnTile + 127 + kOwnLane + 31) / 32 + 1;
constexpr int kOwnPlaneWords = kOwnTile / 64;
constexpr int kOwnWin = kOwnBaseWords, kOwnLx = kOwnWin + kOwnPlaneWords,
              kOwnRx = kOwnLx + kOwnPlaneWords, kOwnStaged = kOwnRx + kOwnPlaneWords;
static_assert(kOwnStaged <= kOwnRouteThreads, "one staged word per thread");

__device__ __forceinline__ uint64_t tile_word(const OwnRouteArgs& a, int64_t P0, int tid) {
  if (tid < kOwnWin) {
    const int64_t g = P0 / 32 - 1 + tid;
    return g >= 0 && g < a.base_words ? a.bases[g] : 0ull;
  }
  if (tid >= kOwnStaged) return 0ull;
  const uint64_t* plane = tid < kOwnLx ? a.win : tid < kOwnRx ? a.lx : a.rx;
  const int64_t g = P0 / 64 + (tid - kOwnWin) % kOwnPlaneWords;
  return g < (a.n + 63) / 64 ? plane[g] : 0ull;
}

template <int W, int R>
__global__ __launch_bounds__(kOwnRouteThreads) void k_own_emit_staged(OwnRouteArgs a) {
  constexpr int BT = EmitBatch<R>::kTiles;
  constexpr int PT = kOwnLane;
  constexpr int CAP = EmitBatch<R>::kCap;
  __shared__ uint64_t s_tile[kOwnStaged];
  __shared__ uint64_t s_rec[CAP * R];  // the batch's records in bucket order
  __shared__ uint16_t s_bin[CAP];      // and their buckets
  __shared__ uint32_t s_cnt[kOwnL1Max];
  __shared__ uint32_t s_start[kOwnL1Max];
  __shared__ uint32_t s_dst[kOwnL1Max];  // cursor minus place in the batch
  __shared__ uint32_t s_w[kOwnRouteThreads / 64];
  static_assert(kOwnL1Max <= kOwnRouteThreads, "one bucket per lane in the scan");
  const int tid = threadIdx.x;
  const int nbins = 1 << a.p1;
  const int top_bits_kept = own_rest_bits(a.k) + 6 - 64 * (R - 1);  // 1..64
  const uint64_t top_mask = top_bits_kept >= 64 ? ~0ull : (1ull << top_bits_kept) - 1ull;
  const int tb = 2 * (int)a.k - 64 * (W - 1);  // bits of the top word
  const int64_t G = gridDim.x, blk = blockIdx.x;
  uint32_t cur = tid < nbins ? a.h1[(uint64_t)tid * G + blk] : 0u;  // this lane's bucket's
  if (tid < nbins) s_cnt[tid] = 0;
  const int64_t n_tiles = (a.n + kOwnTile - 1) / kOwnTile;
  const int64_t mine = n_tiles > blk ? (n_tiles - blk + G - 1) / G : 0;  // tiles blk + j G
  if (mine > 0 && tid < kOwnStaged) s_tile[tid] = tile_word(a, blk * kOwnTile, tid);
  lds_barrier();
  for (int64_t j0 = 0; j0 < mine; j0 += BT) {
    uint64_t v[BT * PT][R];
    uint32_t br[BT * PT];  // bucket << 16 | rank, ~0 for no record
#pragma unroll
    for (int bt = 0; bt < BT; ++bt) {
      // the next tile's word: in flight while this one's windows are formed
      const int64_t jn = j0 + bt + 1;
      const uint64_t next = jn < mine ? tile_word(a, (blk + jn * G) * kOwnTile, tid) : 0ull;
      const uint32_t at = 4 * (uint32_t)tid;  // the lane's first window in the tile
      const int sh = 60 - (int)(at & 63);
      const uint32_t v4 =
          j0 + bt < mine ? (uint32_t)(s_tile[kOwnWin + (at >> 6)] >> sh) & 15u : 0u;
      const uint32_t l4 = (uint32_t)(s_tile[kOwnLx + (at >> 6)] >> sh) & 15u;
      const uint32_t r4 = (uint32_t)(s_tile[kOwnRx + (at >> 6)] >> sh) & 15u;
      const uint32_t lp = 32 + at;  // staged base of that window
      uint64_t fw[W], rw[W];
      window_words<W>(s_tile, 2 * lp, a.k, fw);
      revcomp_words<W>(fw, a.k, rw);
      const uint32_t rb = (uint32_t)get_bits(s_tile, 2 * (lp + a.k), 8);  // right neighbours
      uint32_t left = get_base(s_tile, lp - 1);
#pragma unroll
      for (int pw = 0; pw < PT; ++pw) {
        const int q = bt * PT + pw;
        if (pw > 0) {
          left = (uint32_t)(fw[0] >> (tb - 2)) & 3u;  // the base leaving the window
          roll_words<W>(fw, rw, (rb >> (8 - 2 * pw)) & 3u, a.k);
        }
        const uint32_t right = (rb >> (6 - 2 * pw)) & 3u;
        const uint32_t lb = (l4 >> (3 - pw)) & 1u, xb = (r4 >> (3 - pw)) & 1u;
        const bool use_rc = words_less<W>(rw, fw);
        // extension byte: valid bit and base per side; on the reverse strand
        // the sides swap and complement
        const uint32_t e_l = lb ? 4u | left : 0u, e_r = xb ? 4u | right : 0u;
        const uint32_t c_l = xb ? 7u - right : 0u, c_r = lb ? 7u - left : 0u;
        const uint32_t e6 = use_rc ? (c_l << 3) | c_r : (e_l << 3) | e_r;
        uint64_t key[W], f[W + 1];
#pragma unroll
        for (int w = 0; w < W; ++w) key[w] = use_rc ? rw[w] : fw[w];
        const int p1 = (int)a.p1;
        const uint32_t b =
            tb >= p1 ? (uint32_t)(key[0] >> (tb - p1))
                     : (uint32_t)((key[0] << (p1 - tb)) | (key[W > 1 ? 1 : 0] >> (64 - p1 + tb)));
        make_record<W, W + 1>(key, e6, f);
        // the low R words, without the digit's bits
#pragma unroll
        for (int w = 0; w < R; ++w) v[q][w] = w == 0 ? f[W + 1 - R] & top_mask : f[W + 1 - R + w];
        br[q] = ~0u;
        if ((v4 >> (3 - pw)) & 1u) br[q] = (b << 16) | atomicAdd(&s_cnt[b], 1u);
      }
      lds_barrier();  // every window of the staged tile is formed
      if (tid < kOwnStaged) s_tile[tid] = next;
      if (bt + 1 < BT) lds_barrier();  // the batch's next tile is formed next
    }
    uint32_t excl = 0;
    const uint32_t c = tid < nbins ? s_cnt[tid] : 0u;
    const uint32_t total = block_excl_scan(c, excl, s_w);
    if (tid < nbins) {
      s_start[tid] = excl;
      s_dst[tid] = cur - excl;
      s_cnt[tid] = 0;
      cur += c;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < BT * PT; ++q) {
      if (br[q] == ~0u) continue;
      const uint32_t b = br[q] >> 16, pos = s_start[b] + (br[q] & 0xffffu);
#pragma unroll
      for (int w = 0; w < R; ++w) s_rec[pos * R + w] = v[q][w];
      s_bin[pos] = (uint16_t)b;
    }
    lds_barrier();
    for (uint32_t i = tid; i < total * R; i += kOwnRouteThreads) {
      const uint32_t rr = i / R;
      a.rec[(uint64_t)(s_dst[s_bin[rr]] + rr) * R + (i - rr * R)] = s_rec[i];
    }
    // the next batch writes these arrays only behind its own barriers, which
    // this wave reaches after its write-out
  }
}

// ------------------------------------------------------ level 2 route ----

// Records per level-2 chunk (one block): 12,288 record words, as many as one
// block's share of the LDS holds beside the digits' tables.  Longer chunks mean
// longer runs: 10M reads, k = 21 (450 owners per bucket) 8.4 ms with 12,288
// words, 9.8 with 8,192, before neighbouring chunks shared an XCD.
template <int R>
struct PartShape {
  static constexpr int kChunk = 12288 / R / kOwnPartThreads * kOwnPartThreads;
  static constexpr int kPerThread = kChunk / kOwnPartThreads;
};

int own_chunk_records(uint32_t k) {
  switch (own_record_words(k)) {
    case 1: return PartShape<1>::kChunk;
    case 2: return PartShape<2>::kChunk;
    case 3: return PartShape<3>::kChunk;
    default: return PartShape<4>::kChunk;
  }
}

// The bucket of every owner and of every level-2 chunk (one block per
// bucket), so that later kernels find theirs with one load.
__global__ void k_own_maps(OwnPartArgs a) {
  const OwnBucket bk = a.buckets[blockIdx.x];
  const uint32_t n_own = 1u << bk.p2;
  for (uint32_t i = threadIdx.x; i < n_own; i += blockDim.x) {
    a.owner_bucket[bk.sbbase + i] = (uint16_t)blockIdx.x;
    a.owner_pfx[bk.sbbase + i] = (uint8_t)(a.p1 + bk.p2);
  }
  for (uint32_t i = threadIdx.x; i < bk.chunks; i += blockDim.x)
    a.chunk_bucket[bk.cbase + i] = (uint16_t)blockIdx.x;
}

// Level-2 histogram: chunk c of bucket b counts its records' next p2_b key
// bits into its row of the bucket's chunk-major matrix,
// m[b.mbase + c * 2^p2_b + digit].
template <int R>
__global__ __launch_bounds__(kOwnPartThreads) void k_own_hist2(OwnPartArgs a) {
  __shared__ uint32_t s_h[1 << kOwnL2Max];
  constexpr int CH = PartShape<R>::kChunk;
  const int tid = threadIdx.x;
  const int b = a.chunk_bucket[blockIdx.x];
  const OwnBucket bk = a.buckets[b];
  const uint32_t c = blockIdx.x - bk.cbase;
  const int nbins = 1 << bk.p2;
  for (int i = tid; i < nbins; i += kOwnPartThreads) s_h[i] = 0;
  lds_barrier();
  const uint64_t r0 = bk.start + (uint64_t)c * CH;
  const uint64_t r1 = r0 + (uint64_t)CH < bk.start + bk.n ? r0 + (uint64_t)CH : bk.start + bk.n;
  const int roff = 64 * R - 2 * (int)a.k - 6 + (int)a.p1;
  for (uint64_t r = r0 + tid; r < r1; r += kOwnPartThreads) {
    uint64_t v[R];
    load_record<R>(a.rec_in, r, v);
    atomicAdd(&s_h[top_bits<R>(v, roff, (int)bk.p2)], 1u);
  }
  lds_barrier();
  for (int i = tid; i < nbins; i += kOwnPartThreads)
    a.m[bk.mbase + (uint64_t)c * nbins + i] = s_h[i];
}

// Level-2 scatter: the same chunks, ranked by digit in LDS and written as
// one run per owner at the chunk's cursors (owner start + the column prefix
// of the matrix).
template <int R>
__global__ __launch_bounds__(kOwnPartThreads) void k_own_scatter2(OwnPartArgs a) {
  constexpr int CH = PartShape<R>::kChunk;
  constexpr int PT = PartShape<R>::kPerThread;
  __shared__ uint64_t s_rec[CH * R];
  __shared__ uint16_t s_bin[CH];
  __shared__ uint32_t s_cnt[1 << kOwnL2Max];  // counts, then places in the chunk
  __shared__ uint32_t s_dst[1 << kOwnL2Max];  // cursor minus place
  __shared__ uint32_t s_w[kOwnPartThreads / 64];
  const int tid = threadIdx.x;
  // consecutive chunks to one XCD (blocks go round robin over 8): the runs of
  // neighbouring chunks adjoin, and the line they share is completed in one L2
  // instead of leaving two in parts.  k = 21, 55, 77, 99 of 10M reads: 4.6,
  // 6.4, 7.6 and 6.7 ms (4.5 TB/s), from 8.4, 11.5, 15.8 and 11.4 ms.
  const uint32_t id = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (id >= a.n_chunks) return;
  const int b = a.chunk_bucket[id];
  const OwnBucket bk = a.buckets[b];
  const uint32_t c = id - bk.cbase;
  const int nbins = 1 << bk.p2;
  const uint64_t r0 = bk.start + (uint64_t)c * CH;
  const uint64_t r1 = r0 + (uint64_t)CH < bk.start + bk.n ? r0 + (uint64_t)CH : bk.start + bk.n;
  const uint32_t n = (uint32_t)(r1 - r0);
  uint64_t v[PT][R];
#pragma unroll
  for (int q = 0; q < PT; ++q) {
    const uint32_t r = (uint32_t)q * kOwnPartThreads + tid;
#pragma unroll
    for (int w = 0; w < R; ++w) v[q][w] = 0;
    if (r < n) load_record<R>(a.rec_in, r0 + r, v[q]);
  }
  // the two digits of this thread (nbins <= 2 x kOwnPartThreads) and their
  // cursors
  uint32_t cur[2] = {0, 0};
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int d = 2 * tid + e;
    if (d < nbins) {
      cur[e] = a.start2[bk.sbbase + d] + a.m[bk.mbase + (uint64_t)c * nbins + d];
      s_cnt[d] = 0;
    }
  }
  lds_barrier();
  const int roff = 64 * R - 2 * (int)a.k - 6 + (int)a.p1;
  uint32_t br[PT];  // digit << 16 | rank among the chunk's records of that digit
#pragma unroll
  for (int q = 0; q < PT; ++q) {
    br[q] = ~0u;
    if ((uint32_t)q * kOwnPartThreads + tid < n) {
      const uint32_t d = top_bits<R>(v[q], roff, (int)bk.p2);
      br[q] = (d << 16) | atomicAdd(&s_cnt[d], 1u);
    }
  }
  lds_barrier();
  const uint32_t c0 = 2 * tid < nbins ? s_cnt[2 * tid] : 0u;
  const uint32_t c1 = 2 * tid + 1 < nbins ? s_cnt[2 * tid + 1] : 0u;
  uint32_t excl = 0;
  block_excl_scan(c0 + c1, excl, s_w);
  if (2 * tid < nbins) {
    s_cnt[2 * tid] = excl;
    s_dst[2 * tid] = cur[0] - excl;
  }
  if (2 * tid + 1 < nbins) {
    s_cnt[2 * tid + 1] = excl + c0;
    s_dst[2 * tid + 1] = cur[1] - excl - c0;
  }
  lds_barrier();
#pragma unroll
  for (int q = 0; q < PT; ++q) {
    if (br[q] == ~0u) continue;
    const uint32_t d = br[q] >> 16, pos = s_cnt[d] + (br[q] & 0xffffu);
#pragma unroll
    for (int w = 0; w < R; ++w) s_rec[pos * R + w] = v[q][w];
    s_bin[pos] = (uint16_t)d;
  }
  lds_barrier();
  for (uint32_t i = tid; i < n * R; i += kOwnPartThreads) {
    const uint32_t rr = i / R;
    a.rec_out[(uint64_t)(s_dst[s_bin[rr]] + rr) * R + (i - rr * R)] = s_rec[i];
  }
}

// Column scan of the level-2 matrix: one thread per owner (bucket b, digit
// d) turns its column (chunks 0, 1, ... of b) into exclusive prefixes and
// leaves the owner's record count in tot[owner]; thread n_owners writes 0, so
// that an exclusive scan of tot[0 .. n_owners] gives every owner's first
// record and the total after the last.  Owners of more than n_small records
// are listed in big.
__global__ void k_own_colscan(OwnPartArgs a, uint32_t n_owners) {
  const uint32_t sb = blockIdx.x * blockDim.x + threadIdx.x;
  if (sb > n_owners) return;
  if (sb == n_owners) {
    a.start2[sb] = 0;
    return;
  }
  const int b = a.owner_bucket[sb];
  const OwnBucket bk = a.buckets[b];
  const uint32_t d = sb - bk.sbbase, nbins = 1u << bk.p2;
  uint32_t run = 0;
  for (uint32_t c = 0; c < bk.chunks; ++c) {
    const uint64_t i = bk.mbase + (uint64_t)c * nbins + d;
    const uint32_t v = a.m[i];
    a.m[i] = run;
    run += v;
  }
  a.start2[sb] = run;
  if (run > a.n_small) a.big[atomicAdd(a.n_big, 1u)] = sb;
}

// ------------------------------------------------------------- owners ----

// LDS table slots per owner: as many as fit (a multiple of 64) beside the
// Bloom filter in one owner block's share of the CU's
// 160 KiB (kOwnBlocksPerCU blocks share a CU), and at most kRecLanes x
// threads / 2, so that an owner's 2T records are kRecLanes per lane: more
// records per lane spill registers at four waves per SIMD.
template <int C>
struct OwnerShape {
  static constexpr int kPerSlot = 8 * C + 4 + 32 + 2;  // chunks, count, tallies, row list
  static constexpr int kFixed = kOwnBloomWords * 8 + 16 + 8 + (kOwnThreads / 64) * 4 * 5 + 256;
  static constexpr int kFit = (kOwnLdsBytes - kFixed) / kPerSlot / 64 * 64;
  static constexpr int kRecLanes = C == 1 ? 5 : (C <= 3 ? 4 : 3);
  static constexpr int kCap = kRecLanes * kOwnThreads / 2;
  static constexpr int kSlots = kFit < kCap ? kFit : kCap;
  static_assert(kFixed + kSlots * kPerSlot <= kOwnLdsBytes, "owner LDS");
};


int own_slots(uint32_t k) {
  switch (own_chunks(k)) {
    case 1: return OwnerShape<1>::kSlots;
    case 2: return OwnerShape<2>::kSlots;
    case 3: return OwnerShape<3>::kSlots;
    case 4: return OwnerShape<4>::kSlots;
    default: return OwnerShape<5>::kSlots;
  }
}

// Staging.  Blocks take chunks of staging rows from a shared cursor (one atomic
// per chunk, not per owner) and fill them owner after owner; an owner past the
// end of staging is flagged and the pass runs again with every owner's rows at
// its scanned offset.
//
// A chunk is a block's share of an eighth of staging, or of a quarter of what
// was left behind the block's chunk before (or one owner's rows): large while
// there is room, so that few owners fall between two chunks, and exact towards
// the end, so that no block holds a chunk others lack.  Rows that take up to
// 79 % of staging fit (0.2 to 1.5 million reads, k = 21 and 55); with chunks of
// one size, a sixteenth of a block's share but 64 rows at least, sets of 200,000
// reads ran out at 67 % and sets of under 2,000 always.
// seen: the end of the block's last chunk (no more than the cursor).
__device__ __forceinline__ uint64_t staging_want(const OwnCountArgs& a, uint64_t rows,
                                                 uint64_t seen, uint32_t blocks) {
  const int share = 32 - __clz((int)(blocks - 1));  // log2 of the blocks, rounded up
  const uint64_t left = a.st_cap > seen ? a.st_cap - seen : 0;
  const uint64_t eighth = a.st_cap >> (share + 3), quarter = left >> (share + 2);
  const uint64_t chunk = eighth < quarter ? eighth : quarter;
  return rows > chunk ? rows : chunk;
}

// The owners with more records than k_own_count holds at once (a.big: key
// prefixes shared by very many windows, down to the finest split): Bloom pass
// A and count pass B over the records in batches, 32-bit tallies in an
// open-addressing table of the keys that pass the screen, then classify
// (count >= min_count, extension codes) and write the rows to staging.
//
// Without the screen every key takes a slot, and an owner of more records than
// slots may hold too many: its keys are then counted in parts by their hash,
// pass B and the rows once per part, each part expected to fill the table to
// 0.86 at most if no key repeats.  (One owner of too many keys had every owner
// split finer and counted again: 2M reads of 150 bases with 1 % errors, k = 29,
// 3,544 owners of too many keys, 83.7 ms a call, 11.8 ms in parts.)
//
// Few keys many times need no parts, and every part reads all records again:
// an owner is tried whole first where the block's last one would have fitted
// whole, or where it has more records than its parts are sure to hold.  A try
// that fails is cut short (kTryProbes).  500,000 reads of 150 bases, a fifth of
// them of period 1 or 3, unscreened, k = 21: 47.9 ms a call in parts alone,
// 13.4 with tries; 100,000 reads with 3 % errors, whose keys fill the parts, 0.49
// either way.
constexpr uint32_t kTryProbes = 64;

template <int R, int C>
__global__ __launch_bounds__(kOwnThreads, kOwnThreads * kOwnBlocksPerCU / 256) void k_own_count_big(OwnCountArgs a) {
  constexpr int T = OwnerShape<C>::kSlots;
  // records per lane per batch: an owner of the usual size (up to 2 T
  // records) is one batch
  constexpr int NB = (2 * T + kOwnThreads - 1) / kOwnThreads;
  constexpr uint64_t kBatch = (uint64_t)NB * kOwnThreads;
  __shared__ uint64_t s_bloom[kOwnBloomWords];
  __shared__ uint64_t s_ch[C][T];
  __shared__ uint32_t s_cnt[T];  // occurrences without a left extension
  __shared__ uint32_t s_tal[8][T];
  __shared__ uint16_t s_list[T];  // the owner's kept slots, in slot order
  __shared__ uint32_t s_misc[4];
  __shared__ uint64_t s_chunk;
  __shared__ uint32_t s_w[kOwnThreads / 64];
  __shared__ uint32_t s_acc[4];  // the owner's first sightings, second, passed, claimed
  const int tid = threadIdx.x;
  const uint32_t k = a.k;
  constexpr int ws = C;  // the launcher picks C = own_chunks(k)
  const int W = (int)(k + 31) / 32;
  const uint32_t tcap = a.slots < (uint32_t)T ? a.slots : (uint32_t)T;
  const uint32_t N = *a.n_big, G = gridDim.x;
  // optional phase clocks (thread 0, summed over the block's owners)
  uint64_t prof_acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  uint64_t prof_t = 0;
#define PROF_MARK(e)                                         \
  if (a.prof && tid == 0) {                                  \
    const uint64_t now_ = wall_clock64();                    \
    if ((e) > 0) prof_acc[(e) > 8 ? 7 : ((e) > 0 ? (e) - 1 : 0)] += now_ - prof_t; \
    prof_t = now_;                                           \
  }

  // Persistent blocks: the listed owners blockIdx.x, + G, ...
  bool whole = false;  // the block's last unscreened owner would have fitted whole
  // the block's staging chunk (uniform): empty, behind the small owners' ones
  if (tid == 0)
    s_chunk = __hip_atomic_load(a.st_cursor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  lds_barrier();
  uint64_t st_cur = s_chunk, st_end = st_cur;
  for (uint32_t x = blockIdx.x; x < N; x += G) {
  const uint32_t sb = a.big[x];
  const uint64_t r0 = a.start2[sb], r1 = a.start2[sb + 1];
  // an owner of at most NB records per lane is loaded once for both passes
  const bool one_batch = r1 - r0 <= kBatch;
  uint64_t vb[NB][R];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const uint64_t r = r0 + (uint64_t)q * kOwnThreads + tid;
#pragma unroll
    for (int w = 0; w < R; ++w) vb[q][w] = 0;
    if (one_batch && r < r1) load_record<R>(a.rec, r, vb[q]);
  }

  PROF_MARK(0);
  for (int i = tid; i < kOwnBloomWords; i += kOwnThreads) s_bloom[i] = 0;
  for (int i = tid; i < T; i += kOwnThreads) {
#pragma unroll
    for (int c = 0; c < C; ++c) s_ch[c][i] = 0;
    s_cnt[i] = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) s_tal[e][i] = 0;
  }
  if (tid == 0) {
    s_misc[0] = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) s_acc[e] = 0;
  }
  lds_barrier();
  PROF_MARK(1);

  uint32_t l1 = 0, l2 = 0, passed = 0, claimed = 0;
  const uint32_t per_part = tcap - tcap / 7;
  const uint32_t most_parts =
      a.use_bloom || tcap < (uint32_t)T || r1 - r0 <= tcap
          ? 1u
          : (uint32_t)(r1 - r0 < 8ull * per_part ? (r1 - r0 + per_part - 1) / per_part : 8);
  uint32_t parts = whole || r1 - r0 > 8ull * per_part ? 1u : most_parts;
  // Both passes take a lane's records of a batch together, one memory step
  // at a time for all of them (hashes, then every LDS load, then every
  // atomic), so a lane has several LDS round trips in flight instead of one.
  // ---- pass A (Bloom): every sighting sets the key's level-1 pattern; a
  // sighting of a key whose level-1 pattern was complete completes level 2
  if (a.use_bloom) {
    for (uint64_t b0 = r0; b0 < r1; b0 += kBatch) {
      // this lane's records of the batch are its first nq
      const int nq = lane_records<NB>(b0, r1, tid);
      uint32_t bi[NB], pat[NB];
      uint64_t cur[NB];
      if (!one_batch) {
#pragma unroll
        for (int q = 0; q < NB; ++q) {  // every load of the batch in flight at once
#pragma unroll
          for (int w = 0; w < R; ++w) vb[q][w] = 0;
          if (q < nq) load_record<R>(a.rec, b0 + (uint64_t)q * kOwnThreads + tid, vb[q]);
        }
      }
      // hashes of every slot (a slot past the owner's records holds zeros):
      // no branch per record
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        uint64_t key[R], ch[C];
        record_key<R>(vb[q], key);
        to_chunks<R, C>(key, ws, ch);
        owner_bloom(owner_hash<C>(ch, ws), bi[q], pat[q]);
      }
#pragma unroll
      for (int q = 0; q < NB; ++q) cur[q] = s_bloom[bi[q]];
      bool set1[NB], set2[NB];
      uint64_t old[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        set1[q] = q < nq && ((uint32_t)cur[q] & pat[q]) != pat[q];
        set2[q] = q < nq && !set1[q] && ((uint32_t)(cur[q] >> 32) & pat[q]) != pat[q];
        old[q] = 0;
        if (set1[q] || set2[q])
          old[q] = atomicOr(reinterpret_cast<unsigned long long*>(&s_bloom[bi[q]]),
                            set1[q] ? (unsigned long long)pat[q]
                                    : (unsigned long long)pat[q] << 32);
      }
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        if (set1[q]) {
          if (((uint32_t)old[q] & pat[q]) != pat[q]) {
            ++l1;  // first sighting (up to false positives)
          } else {  // seen meanwhile: complete the level-2 pattern
            const uint64_t o2 = atomicOr(reinterpret_cast<unsigned long long*>(&s_bloom[bi[q]]),
                                         (unsigned long long)pat[q] << 32);
            if (((uint32_t)(o2 >> 32) & pat[q]) != pat[q]) ++l2;
          }
        } else if (set2[q] && ((uint32_t)(old[q] >> 32) & pat[q]) != pat[q]) {
          ++l2;
        }
      }
    }
    lds_barrier();
  }
  PROF_MARK(2);
  uint64_t base = 0;          // the owner's first staging row
  uint32_t done = 0;          // rows of the parts before
  bool fits = true, unfit = false;  // uniform
  bool again = false;  // the owner did not fit whole
  for (uint32_t part = 0; part < parts; ++part) {
  if (part > 0 || again) {
    lds_barrier();  // the last part's rows have left LDS (or every lane has read the flag)
    if (tid == 0) {
      s_misc[0] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) s_acc[e] = 0;
    }
    for (int i = tid; i < T; i += kOwnThreads) {
#pragma unroll
      for (int c = 0; c < C; ++c) s_ch[c][i] = 0;
      s_cnt[i] = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) s_tal[e][i] = 0;
    }
    lds_barrier();
  }
  // ---- pass B: count the records whose key completed level 2 (all records
  // without the Bloom screen) in the open-addressing LDS table.  Each stored
  // chunk is written once by CAS from 0 (chunks never are 0), so a slot's
  // chunks always spell one key and equal keys meet in one slot (a word
  // read as 0 may have been written since, which the CAS then reports; a
  // non-zero word is final).  An occurrence adds 1 to its left tally (or to the no-left-extension count)
  // and 1 to its right tally if it has one: the count is the sum of the
  // first five, so it needs no add of its own.
  const bool trying = parts < most_parts;
  const uint32_t probes = trying ? kTryProbes : tcap;
  for (uint64_t b0 = r0; b0 < r1; b0 += kBatch) {
    if (trying && *static_cast<volatile uint32_t*>(&s_misc[0])) break;  // no barrier inside
    const int nq = lane_records<NB>(b0, r1, tid);
    uint32_t okm = (1u << nq) - 1u;  // bit q: record q is counted
    uint64_t ch[NB][C], w0[NB], h[NB];
    uint32_t i0[NB];
    if (!one_batch) {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
#pragma unroll
        for (int w = 0; w < R; ++w) vb[q][w] = 0;
        if (q < nq) load_record<R>(a.rec, b0 + (uint64_t)q * kOwnThreads + tid, vb[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      uint64_t key[R];
      record_key<R>(vb[q], key);
      to_chunks<R, C>(key, ws, ch[q]);
      h[q] = owner_hash<C>(ch[q], ws);
    }
    if (a.use_bloom) {
      uint32_t bi[NB], pat[NB];
      uint64_t bw[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) owner_bloom(h[q], bi[q], pat[q]);
#pragma unroll
      for (int q = 0; q < NB; ++q) bw[q] = s_bloom[bi[q]];
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (((uint32_t)(bw[q] >> 32) & pat[q]) != pat[q]) okm &= ~(1u << q);
    }
    if (parts > 1) {
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (__umulhi((uint32_t)h[q] * 0x85ebca6bu, parts) != part) okm &= ~(1u << q);
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {  // first word of every record's first probe at once
      i0[q] = __umulhi((uint32_t)(h[q] >> 32), tcap);
      w0[q] = s_ch[0][i0[q]];
    }
    int slot[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      slot[q] = -1;
      if (!((okm >> q) & 1u)) continue;
      ++passed;
      uint32_t i = i0[q];
      for (uint32_t probe = 0; probe < probes; ++probe) {
        bool match = true;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          if (c < ws && match) {
            uint64_t w = (probe == 0 && c == 0) ? w0[q] : s_ch[c][i];
            if (w == 0) {
              const uint64_t o = atomicCAS(reinterpret_cast<unsigned long long*>(&s_ch[c][i]),
                                           0ull, (unsigned long long)ch[q][c]);
              w = o == 0 ? ch[q][c] : o;
              if (o == 0 && c == 0) ++claimed;
            }
            match = w == ch[q][c];
          }
        }
        if (match) {
          slot[q] = (int)i;
          break;
        }
        if (++i == tcap) i = 0;
      }
      if (slot[q] < 0) s_misc[0] = 1;  // the owner's keys do not fit
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (slot[q] < 0) continue;
      const uint32_t e6 = (uint32_t)(vb[q][R - 1] & 63u);
      atomicAdd((e6 & 32u) ? &s_tal[(e6 >> 3) & 3u][slot[q]] : &s_cnt[slot[q]], 1u);
      if (e6 & 4u) atomicAdd(&s_tal[4 + (e6 & 3u)][slot[q]], 1u);
    }
  }
  // ---- statistics, added once per owner to one of kOwnStripes copies of
  // the counters (the host sums them): each wave adds its sums into LDS, and
  // the barrier that completes the table also completes them
  PROF_MARK(3);
  unsigned long long* sc = a.ctr + (uint64_t)(sb % kOwnStripes) * kCtrCount;
  if (part + 1 == parts) {
    uint32_t v[4] = {l1, l2, passed, claimed};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      for (int o = 32; o > 0; o >>= 1) v[e] += __shfl_down(v[e], o);
    if ((tid & 63) == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v[e]) atomicAdd(&s_acc[e], v[e]);
    }
  }
  lds_barrier();
  // s_misc[0] and s_acc change only in the next clear, after a barrier every
  // lane passes after reading them
  unfit = s_misc[0] != 0;
  if (unfit && trying) {
    unfit = whole = false;
    again = true;
    parts = most_parts;
    passed = claimed = 0;
    part = ~0u;  // from part 0
    continue;
  }
  if (most_parts > 1 && part + 1 == parts) whole = s_acc[3] <= tcap / 4 * 3;
  if (tid == 0 && part + 1 == parts) {
    const uint32_t t0 = s_acc[0], t1 = s_acc[1], t2 = s_acc[2], t3 = s_acc[3];
    if (t0) atomicAdd(&sc[kCtrL1New], (unsigned long long)t0);
    if (t1) atomicAdd(&sc[kCtrL2New], (unsigned long long)t1);
    if (t2) atomicAdd(&sc[kCtrPassed], (unsigned long long)t2);
    if (t3) atomicAdd(&sc[kCtrClaimed], (unsigned long long)t3);
    // keys of the fullest owner, and the owners whose keys did not fit
    atomicMax(&sc[kCtrWindows], (unsigned long long)t3);
  }
  if (unfit) break;  // the flag is stable until the next owner's clear

  PROF_MARK(4);
  // ---- classify: a slot is a row when its count reaches min_count.  Rows
  // leave in slot order, each thread's at its place from one block scan;
  // the copy to the table puts every owner's rows in key order.
  // Rows are ranked in slot order (slot i = tid + m x kOwnThreads): one scan
  // of the kept flags of every m at once, packed in 11-bit fields (each m's
  // count is at most kOwnThreads); the kept slots are then listed in LDS so
  // that every lane writes the same number of rows.
  constexpr int SP = (T + kOwnThreads - 1) / kOwnThreads;  // slots per thread
  static_assert(SP <= 3 && (SP < 3 || T - 2 * kOwnThreads < 1024), "packed rank fields");
  uint32_t keep = 0, packed = 0;
#pragma unroll
  for (int m = 0; m < SP; ++m) {
    const uint32_t i = tid + m * kOwnThreads;
    if (i < tcap && s_ch[0][i] != 0 &&
        s_cnt[i] + s_tal[0][i] + s_tal[1][i] + s_tal[2][i] + s_tal[3][i] >= a.min_count) {
      keep |= 1u << m;
      packed += 1u << (11 * m);
    }
  }
  PROF_MARK(5);
  uint32_t excl_p = 0;
  const uint32_t total_p = block_excl_scan(packed, excl_p, s_w);
  uint32_t first[SP];  // first row of slot column m
  uint32_t rows = 0;
#pragma unroll
  for (int m = 0; m < SP; ++m) {
    first[m] = rows + ((excl_p >> (11 * m)) & 0x7ffu);
    rows += (total_p >> (11 * m)) & 0x7ffu;
  }
#pragma unroll
  for (int m = 0; m < SP; ++m)  // the kept slots in slot order
    if ((keep >> m) & 1u) s_list[first[m]] = (uint16_t)(tid + m * kOwnThreads);
  // more rows than one owner of the copy may have
  unfit = done + rows > (uint32_t)T;
  if (unfit) break;
  lds_barrier();
  PROF_MARK(6);
  PROF_MARK(7);
  // ---- rows to staging (staging_want).  An owner of several parts takes room
  // for all of them at its first: as many rows each, and a quarter more.
  if (part == 0) {
    if (a.st_fixed) {
      base = a.st_fixed[sb];
    } else {
      const uint32_t all = rows * parts;
      const uint64_t most = parts == 1 ? all : min(all + all / 4 + 64u, (uint32_t)T);
      if (st_cur + most > st_end) {  // uniform
        const uint64_t want = staging_want(a, most, st_end, G);
        if (tid == 0) s_chunk = atomicAdd(a.st_cursor, (unsigned long long)want);
        lds_barrier();
        st_cur = s_chunk;
        st_end = st_cur + want;
      }
      base = st_cur;
    }
  }
  const uint64_t row0 = base + done;
  if (!a.st_fixed) {
    fits = row0 + rows <= (st_end < a.st_cap ? st_end : a.st_cap);
    st_cur += rows;
  }
  done += rows;
  // the key's level-1 digit goes back above its rest bits
  const uint64_t digit = a.owner_bucket[sb];
  const int rest_bits = own_rest_bits(k), dw = rest_bits >> 6, doff = rest_bits & 63;
  for (uint32_t j = tid; j < (fits ? rows : 0u); j += kOwnThreads) {
    const uint32_t i = s_list[j];
    uint64_t cv[C], f[R];
#pragma unroll
    for (int c = 0; c < C; ++c) cv[c] = s_ch[c][i];
    from_chunks<R>(cv, ws, f);
    const uint64_t row = row0 + j;
    uint64_t lw[R + 1];  // the whole key (W <= R + 1 words), least significant first
#pragma unroll
    for (int q = 0; q <= R; ++q) {
      lw[q] = q < R ? f[R - 1 - q] : 0ull;
      if (q == dw) lw[q] |= digit << doff;
      if (q == dw + 1 && doff > 0) lw[q] |= digit >> (64 - doff);
    }
#pragma unroll
    for (int q = 0; q <= R; ++q)
      if (q < W) a.st_keys[row * W + (W - 1 - q)] = lw[q];
    uint32_t l[4], rr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      l[e] = s_tal[e][i];
      rr[e] = s_tal[4 + e][i];
    }
    const uint32_t cnt = s_cnt[i] + l[0] + l[1] + l[2] + l[3];
    a.st_counts[row] = cnt;
    uint4* ep = reinterpret_cast<uint4*>(a.st_ext + row * 8);
    ep[0] = make_uint4(l[0], l[1], l[2], l[3]);
    ep[1] = make_uint4(rr[0], rr[1], rr[2], rr[3]);
    reinterpret_cast<uint16_t*>(a.st_codes)[row] =
        (uint16_t)((uint32_t)side_code(l, cnt, a.t_min_ext, a.t_base, a.err_ppm) |
                   ((uint32_t)side_code(rr, cnt, a.t_min_ext, a.t_base, a.err_ppm) << 8));
  }
  if (!fits && tid == 0) atomicOr(&sc[kCtrStatus], (unsigned long long)kStatusStaging);
  }  // parts
  if (tid == 0) {
    unsigned long long* sc = a.ctr + (uint64_t)(sb % kOwnStripes) * kCtrCount;
    const uint32_t rows = unfit ? 0u : done;
    a.rows_sb[sb] = rows;
    a.row_off[sb] = rows;
    a.st_off[sb] = base;
    if (rows) atomicAdd(&sc[kCtrRows], (unsigned long long)rows);
    if (unfit) {
      atomicAdd(&sc[kCtrHeavy], 1ull);
      atomicOr(&sc[kCtrStatus], (unsigned long long)kStatusProbeLimit);
    }
  }
  lds_barrier();  // the rows have left LDS: the next owner may clear it
  PROF_MARK(8);
  }
  if (a.prof && tid == 0)
    for (int e = 0; e < 8; ++e) atomicAdd(&a.prof[e], (unsigned long long)prof_acc[e]);
#undef PROF_MARK
}

// Owners of up to kRecs records, counted without a filter and without key
// slots: the records lie in LDS, a hash table of kSlots 32-bit words names for
// every key its first record (index + 1 in the low half, 0: free) and counts
// its occurrences (high half), and only the keys that become rows get tallies,
// once their number is known, over the records' space.  An owner always fits:
// there are more slots than records, and room for half as many rows (rows of
// one record, min_count 1, come from owners of half the records).
//
// The tallies are 16 bits wide (an owner has under 2^16 records), two to a
// word: 16 bytes a row.
//
// Two blocks of 512 threads share a CU's LDS, so that one block's barriers and
// loads hide behind the other's work; as many records as that leaves room for
// keep the level-2 runs long.
//
// Bound by instruction issue (about 140 vector instructions per 64 records),
// then by the records and rows: 10M reads of 150 bases at k = 21, 33, 55, 77,
// 99 take 8.9, 8.9, 8.8, 9.0 and 7.7 ms and the big owners (3 % of them) 1.1
// ms each, from 18.8, 18.8, 18.6, 17.6 and 15.6 ms with a Bloom filter, key
// slots and 32-bit tallies in one block's LDS per CU.  Probing for a group of
// a lane's records at once instead of one after another is slower (11.0 ms at
// k = 21): it issues more instructions.
template <int R>
struct SmallShape {
  static constexpr int kThreads = 512;
  static constexpr int kRecs = R == 1 ? 4608 : R == 2 ? 3584 : R == 3 ? 2560 : 2048;
  static constexpr int kSlots = kRecs / 2 * 3;
  static constexpr int kLane = kRecs / kThreads;  // records per lane
  static constexpr int kRows = kRecs / 2;
  // row list (first record, count): beside the records for one-word records,
  // whose space the tallies fill, else behind the tallies
  static constexpr int kList = R == 1 ? kRows : 1;
  static_assert(kRecs * 8 * R >= kRows * (R == 1 ? 16 : 20), "tallies over the records");
  static_assert(kRecs * 8 * R + kSlots * 4 + kList * 4 <= 79 * 1024, "small owner LDS");
  static_assert(kRecs % kThreads == 0 && kSlots % 4 == 0 && kRows % 4 == 0, "even shares");
  static_assert(kLane * (kThreads / 64) <= 128, "two counts per lane in the row scan");
};

int own_small_records(uint32_t k) {
  switch (own_record_words(k)) {
    case 1: return SmallShape<1>::kRecs;
    case 2: return SmallShape<2>::kRecs;
    case 3: return SmallShape<3>::kRecs;
    default: return SmallShape<4>::kRecs;
  }
}

// Do two records hold the same key (all bits but the extension byte)?
template <int R>
__device__ __forceinline__ bool same_key(const uint64_t (&a)[R], const uint64_t* b) {
  uint64_t d = (a[R - 1] ^ b[R - 1]) >> 6;
#pragma unroll
  for (int w = 0; w + 1 < R; ++w) d |= a[w] ^ b[w];
  return d == 0;
}

template <int R>
__global__ __launch_bounds__(SmallShape<R>::kThreads, 4) void k_own_count(OwnCountArgs a) {
  using Shape = SmallShape<R>;
  constexpr int NT = Shape::kThreads, NB = Shape::kLane, S = Shape::kSlots, NW = NT / 64;
  constexpr int NE = (NB + 3) / 4;  // words of extension bytes
  constexpr int kGroup = 3;  // records of a lane whose hashes and claims are issued together
  __shared__ __align__(16) uint64_t s_rec[Shape::kRecs * R];  // records, then tallies
  __shared__ __align__(16) uint32_t s_slot[S];
  __shared__ uint32_t s_c[128];    // rows of each (record column, wave)
  __shared__ uint32_t s_keys[2];   // keys of this owner, of the next
  __shared__ uint64_t s_chunk;
  __shared__ uint64_t s_red[NW];
  __shared__ uint64_t s_clock;
  // over the records: the rows' tallies (left A C, G T, right A C, G T)
  uint4* s_tal = reinterpret_cast<uint4*>(s_rec);
  uint32_t* s_tal32 = reinterpret_cast<uint32_t*>(s_rec);
  __shared__ uint32_t s_list1[Shape::kList];
  uint32_t* s_list = R == 1 ? s_list1 : s_tal32 + 4 * Shape::kRows;
  int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const uint32_t k = a.k;
  const int W = (int)(k + 31) / 32;
  const int rest_bits = own_rest_bits(k), dw = rest_bits >> 6, doff = rest_bits & 63;
  uint64_t st_cur = 0, st_end = 0;  // the block's staging chunk (uniform)
  uint32_t n_first = 0, n_pass = 0;              // per lane (windows number under 2^32)
  uint32_t n_keys = 0, n_rows = 0;               // per wave, per block
  uint32_t fullest = 0, par = 0;
  bool spilt = false;  // staging ran out (uniform)
  if (tid < 128) s_c[tid] = 0;
  // optional phase clocks of thread 0
#define PROF_MARK(e)                                                                \
  if (a.prof && tid_ == 0) {                                                        \
    const uint64_t now_ = wall_clock64();                                           \
    if ((e) > 0) atomicAdd(&a.prof[(e) - 1], (unsigned long long)(now_ - s_clock)); \
    s_clock = now_;                                                                 \
  }
  const int tid_ = threadIdx.x;
  if (tid < 2) s_keys[tid] = 0;
  for (uint32_t sb = blockIdx.x; sb < a.n_owners; sb += gridDim.x) {
    // keeps the addresses that depend on tid alone from being held in
    // registers across owners
    asm volatile("" : "+v"(tid));
    const uint64_t r0 = a.start2[sb];
    const uint64_t n64 = a.start2[sb + 1] - r0;
    if (n64 > a.n_small) continue;
    const uint32_t n = (uint32_t)n64;
    if (n == 0) {
      if (tid == 0) {
        a.rows_sb[sb] = 0;
        a.row_off[sb] = 0;
      }
      continue;
    }
    const uint64_t digit = a.owner_bucket ? a.owner_bucket[sb] : sb;
    const int nq = (int)((n + NT - 1) / NT);  // record columns in use (uniform)
    PROF_MARK(0);
    // ---- the records, and free slots
    uint64_t v[NB][R];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const uint32_t r = q * NT + tid;
#pragma unroll
      for (int w = 0; w < R; ++w) v[q][w] = 0;
      if (q < nq && r < n) load_record<R>(a.rec, r0 + r, v[q]);
    }
    for (int i = tid; i < S / 4; i += NT) reinterpret_cast<uint4*>(s_slot)[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const uint32_t r = q * NT + tid;
      if (q < nq && r < n) {
#pragma unroll
        for (int w = 0; w < R; ++w) s_rec[r * R + w] = v[q][w];
      }
    }
    lds_barrier();
    PROF_MARK(1);
    // ---- every record finds its key's slot or claims a free one; each step
    // is issued for a group of a lane's records before the next
    uint32_t at[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) at[q] = 0;
    uint32_t first = 0;  // bit q: record q is its key's first
#pragma unroll
    for (int q0 = 0; q0 < NB; q0 += kGroup) {
      if (q0 >= nq) continue;
      uint32_t old[kGroup];
#pragma unroll
      for (int g = 0; g < kGroup; ++g) {
        const int q = q0 + g;
        if (q >= NB || q >= nq) continue;
        uint64_t key[R], h = 0;
        const uint64_t K[4] = {0x9e3779b97f4a7c15ull, 0xc2b2ae3d27d4eb4full, 0x165667b19e3779f9ull,
                               0xd6e8feb86659fd93ull};
        record_key<R>(v[q], key);
#pragma unroll
        for (int w = 0; w < R; ++w) h += key[w] * K[w];
        h ^= h >> 29;
        at[q] = __umulhi((uint32_t)(h >> 32), (uint32_t)S);
        const uint32_t r = q * NT + tid;
        old[g] = r < n ? atomicCAS(&s_slot[at[q]], 0u, (r + 1) | 0x10000u) : 0u;
      }
#pragma unroll
      for (int g = 0; g < kGroup; ++g) {
        const int q = q0 + g;
        if (q >= NB || q >= nq) continue;
        const uint32_t r = q * NT + tid;
        if (r >= n) continue;
        uint32_t o = old[g], i = at[q];
        // free slots outnumber the records: every search ends
        while (o != 0 && !same_key<R>(v[q], s_rec + ((o & 0xffffu) - 1) * R)) {
          if (++i == (uint32_t)S) i = 0;
          o = atomicCAS(&s_slot[i], 0u, (r + 1) | 0x10000u);
        }
        at[q] = i;
        if (o == 0)
          first |= 1u << q;
        else
          atomicAdd(&s_slot[i], 0x10000u);
      }
      __builtin_amdgcn_sched_barrier(0);  // one group's registers at a time
    }
    uint32_t ext[NE];  // the records' extension bytes (their keys are not needed again)
#pragma unroll
    for (int e = 0; e < NE; ++e) ext[e] = 0;
#pragma unroll
    for (int q = 0; q < NB; ++q) ext[q / 4] |= (uint32_t)(v[q][R - 1] & 63u) << (8 * (q % 4));
    PROF_MARK(2);
    lds_barrier();
    PROF_MARK(3);
    // ---- rows: keys with min_count occurrences, numbered in the order of
    // their first records (columns of 64 records, one per wave and q), so
    // that neighbouring lanes write neighbouring rows
    uint32_t keep = 0, nkeys = 0;
    const uint32_t thr = a.use_bloom ? 2u : 1u;  // the screen's: keys seen twice
    n_first += __popc(first);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (q >= nq) continue;
      const uint32_t c = (first >> q) & 1u ? s_slot[at[q]] >> 16 : 0u;
      const bool row = c >= max(a.min_count, 1u);
      keep |= row ? 1u << q : 0u;
      const uint64_t m = __ballot(row);
      if (lane == 0) s_c[q * NW + wave] = (uint32_t)__popcll(m);
      n_pass += c >= thr ? c : 0u;
      nkeys += (uint32_t)__popcll(__ballot(c >= thr));
    }
    n_keys += nkeys;
    if (lane == 0) atomicAdd(&s_keys[par], nkeys);
    lds_barrier();
    PROF_MARK(4);
    const bool used = 2 * lane < nq * NW;  // NW is even
    const uint32_t x0 = used ? s_c[2 * lane] : 0u, x1 = used ? s_c[2 * lane + 1] : 0u;
    uint32_t incl = x0 + x1;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    const uint32_t rows = __shfl(incl, 63);  // uniform over the block
    // first row of column (q, wave): NW is even, so a wave's columns are all
    // even or all odd
    const uint32_t mine = incl - x0 - x1 + ((wave & 1) ? x0 : 0u);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (q >= nq) continue;
      const uint32_t base = __shfl(mine, (q * NW + wave) >> 1);
      const uint64_t m = __ballot((keep >> q) & 1u);
      if (!((first >> q) & 1u)) continue;
      const uint32_t w = s_slot[at[q]];
      const uint32_t j = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
      const bool row = (keep >> q) & 1u;
      // the word now holds the key's row + 1 (0: no row), its count stays
      s_slot[at[q]] = (w & 0xffff0000u) | (row ? j + 1 : 0u);
      if (row && j < (uint32_t)Shape::kRows) {
        s_list[j] = (w & 0xffff0000u) | (uint32_t)(q * NT + tid);
        s_tal[j] = make_uint4(0, 0, 0, 0);
      }
    }
    if (tid == 0) {
      fullest = max(fullest, s_keys[par]);
      s_keys[par ^ 1] = 0;
    }
    par ^= 1;
    // staging rows (staging_want)
    uint64_t base_row;
    bool fits = true;
    const bool fresh = !a.st_fixed && st_cur + rows > st_end;  // uniform
    const uint64_t want = staging_want(a, rows, st_end, gridDim.x);
    if (fresh && tid == 0) s_chunk = atomicAdd(a.st_cursor, (unsigned long long)want);
    lds_barrier();
    PROF_MARK(5);
    uint64_t u[R];
#pragma unroll
    for (int w = 0; w < R; ++w) u[w] = 0;
    if ((uint32_t)tid < rows) load_record<R>(a.rec, r0 + (s_list[tid] & 0xffffu), u);
    if (a.st_fixed) {
      base_row = a.st_fixed[sb];
    } else {
      if (fresh) {
        st_cur = s_chunk;
        st_end = st_cur + want;
      }
      base_row = st_cur;
      fits = base_row + rows <= a.st_cap;
      st_cur += rows;
    }
    spilt |= !fits;
    n_rows += rows;
    // ---- tallies, then the rows
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (q >= nq || (uint32_t)(q * NT + tid) >= n) continue;
      const uint32_t j = (s_slot[at[q]] & 0xffffu) - 1;
      if (j >= (uint32_t)Shape::kRows) continue;  // no row (wrapped)
      const uint32_t e6 = ext[q / 4] >> (8 * (q % 4));
      if (e6 & 32u) atomicAdd(&s_tal32[4 * j + ((e6 >> 4) & 1u)], (e6 & 8u) ? 0x10000u : 1u);
      if (e6 & 4u) atomicAdd(&s_tal32[4 * j + 2 + ((e6 >> 1) & 1u)], (e6 & 1u) ? 0x10000u : 1u);
    }
    lds_barrier();
    PROF_MARK(6);
    for (uint32_t j = tid; j < (fits ? rows : 0u); j += NT) {
      const uint32_t cnt = s_list[j] >> 16;
      uint64_t f[R];
      if (j >= (uint32_t)NT) load_record<R>(a.rec, r0 + (s_list[j] & 0xffffu), u);
      record_key<R>(u, f);
      const uint4 t = s_tal[j];
      const uint64_t row = base_row + j;
#pragma unroll
      for (int w = 0; w <= R; ++w) {  // the whole key, least significant word first
        uint64_t x = w < R ? f[R - 1 - w] : 0ull;
        if (w == dw) x |= digit << doff;
        if (w == dw + 1 && doff > 0) x |= digit >> (64 - doff);
        if (w < W) a.st_keys[row * W + (W - 1 - w)] = x;
      }
      const uint32_t l[4] = {t.x & 0xffffu, t.x >> 16, t.y & 0xffffu, t.y >> 16};
      const uint32_t rr[4] = {t.z & 0xffffu, t.z >> 16, t.w & 0xffffu, t.w >> 16};
      a.st_counts[row] = cnt;
      uint4* ep = reinterpret_cast<uint4*>(a.st_ext + row * 8);
      ep[0] = make_uint4(l[0], l[1], l[2], l[3]);
      ep[1] = make_uint4(rr[0], rr[1], rr[2], rr[3]);
      reinterpret_cast<uint16_t*>(a.st_codes)[row] =
          (uint16_t)((uint32_t)side_code(l, cnt, a.t_min_ext, a.t_base, a.err_ppm) |
                     ((uint32_t)side_code(rr, cnt, a.t_min_ext, a.t_base, a.err_ppm) << 8));
    }
    PROF_MARK(7);
    if (tid == 0) {
      a.rows_sb[sb] = rows;
      a.row_off[sb] = rows;
      a.st_off[sb] = base_row;
    }
    lds_barrier();  // the rows have left LDS: the next owner may use it
    PROF_MARK(8);
  }
#undef PROF_MARK
  // ---- statistics of the block's owners: first and second sightings (as an
  // exact Bloom screen would see them), records counted, keys, rows
  unsigned long long* sc = a.ctr + (uint64_t)(blockIdx.x % kOwnStripes) * kCtrCount;
  __syncthreads();
  if (a.use_bloom) block_add(&sc[kCtrL1New], n_first, s_red);
  __syncthreads();
  block_add(&sc[kCtrPassed], n_pass, s_red);
  if (lane == 0 && n_keys) {
    atomicAdd(&sc[kCtrClaimed], (unsigned long long)n_keys);
    if (a.use_bloom) atomicAdd(&sc[kCtrL2New], (unsigned long long)n_keys);
  }
  if (tid == 0) {
    if (n_rows) atomicAdd(&sc[kCtrRows], (unsigned long long)n_rows);
    atomicMax(&sc[kCtrWindows], (unsigned long long)fullest);
    if (spilt) atomicOr(&sc[kCtrStatus], (unsigned long long)kStatusStaging);
  }
}

// Owners' rows from staging to the table at the scanned row offsets, in key
// order (one block per owner; the owner pass leaves them in slot order).
// The owner's keys share its prefix, so each row's sort key is the next
// (at most) 32 key bits: rows are bucketed by the top kOwnSortBits of them,
// each bucket (almost always 0-2 rows) is ordered by them (by the whole key,
// read again, when two are equal), and every row is copied to its place.
// NR: rows of an owner at most for W-word keys.
template <int W, int NR>
__global__ __launch_bounds__(kOwnCopyThreads) void k_own_copy(OwnCopyArgs a) {
  constexpr int NSB = 1 << kOwnSortBits;
  __shared__ uint32_t s_k32[NR];
  __shared__ uint16_t s_rank[NR];
  __shared__ uint16_t s_ord[NR];
  __shared__ uint32_t s_bc[NSB];
  __shared__ uint32_t s_bs[NSB];
  __shared__ uint32_t s_w[kOwnCopyThreads / 64];
  const int tid = threadIdx.x;
  const uint32_t sb = blockIdx.x;
  const uint32_t n = a.rows_sb[sb];
  if (n == 0) return;  // the whole block
  const uint64_t src0 = a.st_off[sb], dst0 = a.row_off[sb];
  const int pfx = a.owner_pfx ? (int)a.owner_pfx[sb] : (int)a.p1;
  const int rest = 2 * (int)a.k - pfx;
  const int len = rest < 32 ? (rest > 0 ? rest : 0) : 32;  // sort-key bits
  const int nb = len < kOwnSortBits ? len : kOwnSortBits;
  const int nbins = 1 << nb;
  const int koff = 64 * W - 2 * (int)a.k + pfx;
  for (int i = tid; i < nbins; i += kOwnCopyThreads) s_bc[i] = 0;
  lds_barrier();
  for (uint32_t r = tid; r < n; r += kOwnCopyThreads) {
    uint64_t v[W];
#pragma unroll
    for (int w = 0; w < W; ++w) v[w] = a.st_keys[(src0 + r) * W + w];
    const uint32_t x = top_bits<W>(v, koff, len);
    s_k32[r] = x;
    s_rank[r] = (uint16_t)atomicAdd(&s_bc[x >> (len - nb)], 1u);
  }
  lds_barrier();
  // bucket starts: NSB / kOwnCopyThreads consecutive buckets per thread
  constexpr int BPT = NSB / kOwnCopyThreads;
  uint32_t mine = 0;
#pragma unroll
  for (int q = 0; q < BPT; ++q) {
    const int d = tid * BPT + q;
    mine += d < nbins ? s_bc[d] : 0u;
  }
  uint32_t excl = 0;
  block_excl_scan(mine, excl, s_w);
#pragma unroll
  for (int q = 0; q < BPT; ++q) {
    const int d = tid * BPT + q;
    if (d < nbins) {
      s_bs[d] = excl;
      excl += s_bc[d];
    }
  }
  lds_barrier();
  for (uint32_t r = tid; r < n; r += kOwnCopyThreads)
    s_ord[s_bs[s_k32[r] >> (len - nb)] + s_rank[r]] = (uint16_t)r;
  lds_barrier();
  for (int d = tid; d < nbins; d += kOwnCopyThreads) {  // insertion sort of each bucket
    const uint32_t cnt = s_bc[d], st = s_bs[d];
    for (uint32_t x = st + 1; x < st + cnt; ++x) {
      const uint16_t cur = s_ord[x];
      const uint32_t kc = s_k32[cur];
      int y = (int)x - 1;
      while (y >= (int)st) {
        const uint16_t o = s_ord[y];
        const uint32_t ko = s_k32[o];
        bool less = kc < ko;
        if (kc == ko) {  // the next bits decide (most significant word first)
          for (int w = 0; w < W; ++w) {
            const uint64_t p = a.st_keys[(src0 + cur) * W + w];
            const uint64_t q = a.st_keys[(src0 + o) * W + w];
            if (p != q) {
              less = p < q;
              break;
            }
          }
        }
        if (!less) break;
        s_ord[y + 1] = o;
        --y;
      }
      s_ord[y + 1] = cur;
    }
  }
  lds_barrier();
  for (uint32_t j = tid; j < n; j += kOwnCopyThreads) {
    const uint64_t s = src0 + s_ord[j], d = dst0 + j;
#pragma unroll
    for (int w = 0; w < W; ++w) a.keys[d * W + w] = a.st_keys[s * W + w];
    a.counts[d] = a.st_counts[s];
    const uint4* se = reinterpret_cast<const uint4*>(a.st_ext + s * 8);
    uint4* de = reinterpret_cast<uint4*>(a.ext + d * 8);
    de[0] = se[0];
    de[1] = se[1];
    reinterpret_cast<uint16_t*>(a.codes)[d] = reinterpret_cast<const uint16_t*>(a.st_codes)[s];
  }
}

// dst[i] = src[i * stride], i < n (the first column of a histogram matrix).
__global__ void k_gather_strided(const uint32_t* __restrict__ src, uint64_t stride, uint32_t n,
                                 uint32_t* __restrict__ dst) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[(uint64_t)i * stride];
}

// ---------------------------------------------------------- launchers ----

void launch_gather_strided(const uint32_t* src, uint64_t stride, uint32_t n, uint32_t* dst,
                           hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_gather_strided, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                     src, stride, n, dst);
}

void launch_own_planes(const OwnRouteArgs& a, hipStream_t s) {
  const int64_t words = (a.n + 63) / 64;
  hipLaunchKernelGGL(k_own_planes, dim3((unsigned)((words + kBlock - 1) / kBlock)), dim3(kBlock),
                     0, s, a);
  if (a.shards <= 1) return;
  // a launch holds under 2^32 threads, which 4 windows a thread would pass
  const dim3 g((unsigned)std::min<int64_t>((words * 16 + kBlock - 1) / kBlock, 1 << 20)),
      t(kBlock);
  const uint64_t inv = ~0ull / a.shards;
  switch ((a.k + 31) / 32) {
    case 1: hipLaunchKernelGGL(k_own_part_filter<1>, g, t, 0, s, a, inv); break;
    case 2: hipLaunchKernelGGL(k_own_part_filter<2>, g, t, 0, s, a, inv); break;
    case 3: hipLaunchKernelGGL(k_own_part_filter<3>, g, t, 0, s, a, inv); break;
    default: hipLaunchKernelGGL(k_own_part_filter<4>, g, t, 0, s, a, inv); break;
  }
}

void launch_own_hist(const OwnRouteArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_own_hist, dim3(grid), dim3(kOwnRouteThreads), 0, s, a);
}

void launch_own_emit(const OwnRouteArgs& a, int grid, hipStream_t s) {
  const int W = (int)(a.k + 31) / 32;
  const int R = own_record_words(a.k);  // W - 1 .. W words
  const dim3 g(grid), t(kOwnRouteThreads);
  if (W == 1) hipLaunchKernelGGL((k_own_emit_staged<1, 1>), g, t, 0, s, a);
  else if (W == 2 && R == 1) hipLaunchKernelGGL((k_own_emit_staged<2, 1>), g, t, 0, s, a);
  else if (W == 2) hipLaunchKernelGGL((k_own_emit_staged<2, 2>), g, t, 0, s, a);
  else if (W == 3 && R == 2) hipLaunchKernelGGL((k_own_emit_staged<3, 2>), g, t, 0, s, a);
  else if (W == 3) hipLaunchKernelGGL((k_own_emit_staged<3, 3>), g, t, 0, s, a);
  else if (R == 3) hipLaunchKernelGGL((k_own_emit_staged<4, 3>), g, t, 0, s, a);
  else hipLaunchKernelGGL((k_own_emit_staged<4, 4>), g, t, 0, s, a);
}

void launch_own_part(const OwnPartArgs& a, uint32_t n_chunks, int scatter, hipStream_t s) {
  if (n_chunks == 0) return;
  const int R = own_record_words(a.k);  // 1 .. 4
  const dim3 g(n_chunks), t(kOwnPartThreads);
  if (!scatter) {
    switch (R) {
      case 1: hipLaunchKernelGGL(k_own_hist2<1>, g, t, 0, s, a); break;
      case 2: hipLaunchKernelGGL(k_own_hist2<2>, g, t, 0, s, a); break;
      case 3: hipLaunchKernelGGL(k_own_hist2<3>, g, t, 0, s, a); break;
      default: hipLaunchKernelGGL(k_own_hist2<4>, g, t, 0, s, a); break;
    }
  } else {
    const dim3 g8((n_chunks + 7) / 8 * 8);
    switch (R) {
      case 1: hipLaunchKernelGGL(k_own_scatter2<1>, g8, t, 0, s, a); break;
      case 2: hipLaunchKernelGGL(k_own_scatter2<2>, g8, t, 0, s, a); break;
      case 3: hipLaunchKernelGGL(k_own_scatter2<3>, g8, t, 0, s, a); break;
      default: hipLaunchKernelGGL(k_own_scatter2<4>, g8, t, 0, s, a); break;
    }
  }
}

void launch_own_maps(const OwnPartArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_own_maps, dim3(a.n_buckets), dim3(kBlock), 0, s, a);
}

void launch_own_colscan(const OwnPartArgs& a, uint32_t n_owners, hipStream_t s) {
  const uint32_t n = n_owners + 1;
  hipLaunchKernelGGL(k_own_colscan, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a,
                     n_owners);
}

void launch_own_count(const OwnCountArgs& a, uint32_t cus, bool any_big, hipStream_t s) {
  if (a.n_owners == 0) return;
  const int R = own_record_words(a.k);
  const int C = own_chunks(a.k);  // R - 1 .. R chunks (rest bits + 6 over 64, rest over 62)
  {
    const dim3 g(2 * cus < a.n_owners ? 2 * cus : a.n_owners), t(SmallShape<1>::kThreads);
    switch (R) {
      case 1: hipLaunchKernelGGL(k_own_count<1>, g, t, 0, s, a); break;
      case 2: hipLaunchKernelGGL(k_own_count<2>, g, t, 0, s, a); break;
      case 3: hipLaunchKernelGGL(k_own_count<3>, g, t, 0, s, a); break;
      default: hipLaunchKernelGGL(k_own_count<4>, g, t, 0, s, a); break;
    }
  }
  if (!any_big) return;
  const dim3 g(cus < a.n_owners ? cus : a.n_owners), t(kOwnThreads);
  if (R == 1) hipLaunchKernelGGL((k_own_count_big<1, 1>), g, t, 0, s, a);
  else if (R == 2 && C == 1) hipLaunchKernelGGL((k_own_count_big<2, 1>), g, t, 0, s, a);
  else if (R == 2) hipLaunchKernelGGL((k_own_count_big<2, 2>), g, t, 0, s, a);
  else if (R == 3 && C == 2) hipLaunchKernelGGL((k_own_count_big<3, 2>), g, t, 0, s, a);
  else if (R == 3) hipLaunchKernelGGL((k_own_count_big<3, 3>), g, t, 0, s, a);
  else hipLaunchKernelGGL((k_own_count_big<4, 4>), g, t, 0, s, a);
}

constexpr int cmax(int a, int b) { return a > b ? a : b; }

void launch_own_copy(const OwnCopyArgs& a, uint32_t n_owners, hipStream_t s) {
  if (n_owners == 0) return;
  // rows of an owner at most: a small one's or the slots of a big one, for
  // the fewest record words (W = 1, 2: one; 3: two; 4: three) and key chunks
  // (one, two, three) a W-word key can have
  const dim3 g(n_owners), t(kOwnCopyThreads);
  constexpr int n1 = cmax(SmallShape<1>::kRows, OwnerShape<1>::kSlots);
  constexpr int n2 = cmax(SmallShape<2>::kRows, OwnerShape<2>::kSlots);
  constexpr int n3 = cmax(SmallShape<3>::kRows, OwnerShape<3>::kSlots);
  switch (a.W) {
    case 1: hipLaunchKernelGGL((k_own_copy<1, n1>), g, t, 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_own_copy<2, n1>), g, t, 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_own_copy<3, n2>), g, t, 0, s, a); break;
    default: hipLaunchKernelGGL((k_own_copy<4, n3>), g, t, 0, s, a); break;
  }
}

}  // namespace kh
