// De Bruijn graph traversal on the device (paper Section II-C): the kept
// k-mers of a table are the vertices, each with its two-letter extension
// code, and a contig is a maximal path of k-mers joined by unique
// high-quality extensions.
//
// Definition (the same as the contig oracle's):
//  * k-mer S joins S' = S[1..k) + b when S's right code is b, S' is a kept
//    k-mer and S''s left code is S[0] (the edge is mutual); codes of a k-mer
//    read on its reverse strand swap sides and complement; an edge from a
//    k-mer to itself or to its reverse complement is dropped;
//  * every k-mer is in exactly one contig, a maximal path or a cycle;
//  * a path is written in the orientation that is lexicographically smaller
//    than its reverse complement; a cycle is opened at its smallest k-mer in
//    canonical orientation and written walking right (k + n - 1 bases);
//  * contigs are listed by their smallest k-mer, with their number of
//    k-mers and the sum of their counts.
//
// Method.  A k-mer read in orientation o (0 canonical, 1 reverse
// complement) and walked to the right is a *state* 2i + o.  Every state has
// at most one successor, so the states form 2 directed chains per path
// (one per reading direction; succ[t ^ 1] = s ^ 1 whenever succ[s] = t) and
// 2 directed cycles per cycle.
//
// Ranking every state by pointer jumping moves all of them through memory
// once per doubling round.  Here a sample of the k-mers (one in 16 to 64 by
// a hash of the row, and every chain's ends) are *splitters*: a walker per
// splitter state follows the successors to the next splitter, telling every
// k-mer it passes its splitter and its place behind it, so each state is read
// once; only the splitter states (a few per cent) are then ranked by pointer
// jumping (distance to the chain's end, its last state, the smallest k-mer
// behind).  1.6e8 rows (k = 21, 1.2e6 contigs): 39 ms, from 192 ms with every
// state ranked (16 rounds over 32-byte records took 128 ms of it) over a
// hashed index of the rows (10 ms to build; 0.5 ms now).  The chains' heads choose each contig's reading, contigs are
// numbered by their smallest k-mer (a bit per row and a popcount rank), and a
// streaming pass over the rows writes every k-mer's base and contig.
//
// Cycles show as splitter states still moving after enough rounds to cover
// any path, or, without a splitter, as k-mers no walker passed: each cycle is
// cut in front of its smallest k-mer's canonical state and everything after
// the links is done again.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "kh_device.hpp"
#include "kh_host.hpp"
#include "kh_rows.hpp"

using namespace kh;

namespace {

constexpr int kTB = 256;

__device__ __forceinline__ int base_of(uint8_t c) {
  switch (c) {
    case 'A': return 0;
    case 'C': return 1;
    case 'G': return 2;
    case 'T': return 3;
    default: return -1;
  }
}

__device__ __forceinline__ uint8_t comp_code(uint8_t c) {
  switch (c) {
    case 'A': return 'T';
    case 'C': return 'G';
    case 'G': return 'C';
    case 'T': return 'A';
    default: return c;
  }
}

template <int W>
__device__ __forceinline__ void load_row(const uint64_t* keys, int64_t i, uint64_t (&w)[W]) {
#pragma unroll
  for (int j = 0; j < W; ++j) w[j] = keys[i * W + j];
}

// A k-mer's successors (of states 2i and 2i + 1) and count, one 16-byte
// record so that a walker's step is one access.  S: 32-bit states for tables
// under 2^31 rows, 64-bit ones beyond.
template <typename S>
struct Node;
template <>
struct alignas(16) Node<uint32_t> {
  uint32_t succ[2];
  uint32_t count, pad;
};
template <>
struct alignas(32) Node<uint64_t> {
  uint64_t succ[2];
  uint32_t count, pad;
};

// A k-mer's place: `off` states behind splitter state `sid` in the chain that
// holds state 2i.
template <typename S>
struct alignas(2 * sizeof(S)) Seg {
  S sid, off;
};

// Pointer-jumping record of a splitter state.
template <typename S>
struct alignas(sizeof(S) == 4 ? 16 : 8) Rec {
  S nxt;          // splitter state reached so far (kEnd: the chain's end is behind)
  S last;         // last splitter state of the chain reached so far
  uint32_t dist;  // k-mers from here to `last`
  uint32_t mn;    // smallest k-mer from here to `last` (inclusive)
};

// Where a splitter state's segment is written: its k-mer lies at k-mer place
// `start` of all contigs laid out one after another (as base offsets), the
// ones behind it at start +- off.
struct alignas(16) Place {
  uint64_t start;
  uint32_t contig;
  int32_t dir;  // +1: written in this chain's direction, -1: in the mirror's
};

template <typename S>
__host__ __device__ constexpr S end_of() { return ~S(0); }

// Is row i a sampled splitter?  (mask + 1 a power of two: one in mask + 1)
__device__ __forceinline__ bool sampled(uint64_t i, uint32_t mask) {
  return ((((uint32_t)i ^ (uint32_t)(i >> 32)) * 0x9e3779b1u) >> 20 & mask) == 0;
}

template <typename S>
__device__ __forceinline__ bool is_splitter(uint64_t i, const Node<S>& nd, uint32_t mask) {
  return nd.succ[0] == end_of<S>() || nd.succ[1] == end_of<S>() || sampled(i, mask);
}

// Set bits of a bit-per-row mask before row i (cnt: scanned popcounts of its
// words).
__device__ __forceinline__ uint32_t bit_rank(const uint64_t* bits, const uint32_t* cnt,
                                             uint64_t i) {
  const uint64_t w = bits[i >> 6];
  return cnt[i >> 6] + (uint32_t)__popcll(w & ((1ull << (i & 63)) - 1ull));
}

template <typename S>
__global__ __launch_bounds__(kTB) void k_nodes(const uint32_t* counts, int64_t n,
                                               Node<S>* nodes) {
  const int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x;
  if (i >= n) return;
  Node<S> nd;
  nd.succ[0] = nd.succ[1] = end_of<S>();
  nd.count = counts[i];
  nd.pad = 0;
  nodes[i] = nd;
}

// Successors.  An edge and its mirror are one (k+1)-mer read on its two
// strands, and only the end that reads the smaller of the two looks the other
// one up and writes both successors: with X the state's reading and Y the
// next one, it is X + b against rc(Y) + comp(X[0]), which X < rc(Y) decides
// (X = rc(Y) is an edge to the k-mer itself).  Half the lookups (index entry,
// row, code: three random lines) for one scattered store.
//
// Bound by random lines: n x (3 reads + 1 store) where every k-mer has both
// neighbours; 1.6e8 rows: 12 ms, 5.5e10 lines/s (16.7 ms with both ends
// looking the other up through a hashed index).
template <int W, typename S>
__global__ __launch_bounds__(kTB) void k_link(const uint64_t* keys, const uint8_t* codes,
                                              int64_t n, uint32_t k, RowIndex ix,
                                              Node<S>* nodes) {
  const int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x;
  if (i >= n) return;
  const int top = 2 * (int)k - 64 * (W - 1);
  uint64_t s[W], rs[W];
  load_row<W>(keys, i, s);
  const uint32_t cc = reinterpret_cast<const uint16_t*>(codes)[i];
  revcomp_words<W>(s, k, rs);
  const int first = (int)((s[0] >> (top - 2)) & 3), last = (int)(s[W - 1] & 3);
  const uint8_t letters[4] = {'A', 'C', 'G', 'T'};
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    // o = 0: canonical reading, step right; o = 1: reverse-complement
    // reading, step right = canonical step left
    const int b = base_of((uint8_t)(o == 0 ? cc >> 8 : cc & 0xffu));
    if (b < 0) continue;
    uint64_t t[W], r[W];
    if (o == 0)
      push_right<W>(s, b, top, t);
    else
      push_left<W>(s, b, top, t);
    revcomp_words<W>(t, k, r);
    // the reading X against rc(Y): s against r (o = 0), rs against t (o = 1)
    if (o == 0 ? !words_less<W>(s, r) : !words_less<W>(rs, t)) continue;
    const bool fwd = !words_less<W>(r, t);
#pragma unroll
    for (int j = 0; j < W; ++j) r[j] = fwd ? t[j] : r[j];
    const int64_t j = find_row<W>(keys, ix, top, r);
    if (j < 0 || j == i) continue;
    // the code of j on the side it is entered from, read in the contig's
    // direction, must name the base the step leaves behind
    const uint8_t c = codes[2 * j + ((o == 0) == fwd ? 0 : 1)];
    const uint8_t back = fwd ? c : comp_code(c);
    if (back != letters[o == 0 ? first : last]) continue;
    const S from = (S)(2 * i + o), to = (S)(2 * j + (fwd ? o : o ^ 1));
    nodes[i].succ[o] = to;
    nodes[to >> 1].succ[(to & 1) ^ 1] = from ^ 1;
  }
}

// One bit per row: splitter; and the popcount of every word (cnt[words]: 0).
template <typename S>
__global__ __launch_bounds__(kTB) void k_split_mark(const Node<S>* nodes, int64_t n,
                                                    uint32_t mask, uint64_t* bits,
                                                    uint32_t* cnt) {
  const int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x;
  const bool on = i < n && is_splitter<S>((uint64_t)i, nodes[i], mask);
  const uint64_t w = __ballot(on);
  const int64_t words = (n + 63) / 64;
  if ((threadIdx.x & 63) == 0) {
    if (i / 64 < words) {
      bits[i / 64] = w;
      cnt[i / 64] = (uint32_t)__popcll(w);
    } else if (i / 64 == words) {
      cnt[words] = 0;
    }
  }
}

// The splitters' rows in row order, and their own places.
template <typename S>
__global__ __launch_bounds__(kTB) void k_split_list(const uint64_t* bits, const uint32_t* cnt,
                                                    int64_t n, uint32_t* spl, Seg<S>* seg) {
  const int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x;
  if (i >= n || !((bits[i >> 6] >> (i & 63)) & 1)) return;
  const uint32_t q = bit_rank(bits, cnt, (uint64_t)i);
  spl[q] = (uint32_t)i;
  seg[i] = Seg<S>{(S)2 * q, (S)0};
}

// Raise *moving if any state of the block is still moving (a plain store of
// 1 per block; only "any" is needed, so no counting atomics).
__device__ __forceinline__ void flag_moving(unsigned int* moving, bool on) {
  if (__syncthreads_or(on) && threadIdx.x == 0) *moving = 1u;
}

// Walkers: each splitter state is followed to the next splitter (or the
// chain's end, which is itself a splitter).  Every other k-mer of a path is
// passed twice, once in each reading; the walk that passes its canonical
// state writes its place.  visited collects the k-mers with a place.
// rec[q].nxt is left as the state reached (k_walk_ends numbers it).
//
// Bound by dependent random reads (one 16-byte node per state, 2n in all).
// Lanes step in lockstep, one node each per turn, and a lane whose walk has
// ended takes its next splitter state (already loaded) in the same turn: with
// one walk per lane, a wave waited for its longest walk (about five times the
// mean) with most lanes idle.  1.6e8 rows: 15.3 ms for 3.2e8 reads and 1.6e8
// scattered stores; 1.5e6 rows: 128 us, from 281 us.
template <typename S>
__global__ __launch_bounds__(kTB) void k_walk(const Node<S>* nodes, int64_t n,
                                              const uint32_t* spl, uint64_t nq, uint32_t mask,
                                              Seg<S>* seg, Rec<S>* rec,
                                              unsigned long long* depth,
                                              unsigned long long* visited,
                                              unsigned int* moving) {
  __shared__ uint64_t red[kTB / 64];
  const uint64_t stride = (uint64_t)gridDim.x * kTB;
  uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x;
  uint64_t seen = 0;
  bool on = false;
  if (q < nq) {
    uint64_t j = spl[q >> 1];
    uint32_t ahead = q + stride < nq ? spl[(q + stride) >> 1] : 0;
    uint32_t mn = 0, len = 0;
    unsigned long long sum = 0;
    S t = (S)(q & 1);
    for (;;) {
      const Node<S> nd = nodes[j];
      // a walk ends at a splitter (its own start at the latest): within n steps
      bool done = len > 0 && (is_splitter<S>(j, nd, mask) || (int64_t)len >= n);
      if (!done) {
        if (!(t & 1)) {
          ++seen;
          if (len > 0) seg[j] = Seg<S>{(S)q, (S)len};
        }
        mn = len > 0 ? min(mn, (uint32_t)j) : (uint32_t)j;
        sum += nd.count;
        ++len;
        t = nd.succ[t & 1];
        done = t == end_of<S>();
        j = (uint64_t)(t >> 1);
      }
      if (done) {
        Rec<S> r;
        const bool open = t != end_of<S>();
        on |= open;
        r.nxt = t;
        r.last = (S)q;
        r.dist = open ? len : 0;
        r.mn = mn;
        rec[q] = r;
        depth[q] = sum;
        q += stride;
        if (q >= nq) break;
        j = ahead;
        ahead = q + stride < nq ? spl[(q + stride) >> 1] : 0;
        t = (S)(q & 1);
        len = 0;
        sum = 0;
      }
    }
  }
  flag_moving(moving, on);
  block_add(visited, seen, red);
}

// The states the walks reached, as splitter states.
template <typename S>
__global__ __launch_bounds__(kTB) void k_walk_ends(const uint64_t* bits, const uint32_t* cnt,
                                                   Rec<S>* rec, uint64_t nq) {
  const uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x;
  if (q >= nq) return;
  const S t = rec[q].nxt;
  if (t == end_of<S>()) return;
  const S to = (S)(2 * (uint64_t)bit_rank(bits, cnt, (uint64_t)(t >> 1)) + (t & 1));
  rec[q].nxt = to;
  rec[q].last = to;
}

// One round of pointer jumping: a state's stretch [q, nxt) absorbs those of
// the next three states it leads to, so stretches grow fourfold (a launch
// costs a small table as much as the jump itself).  moving[0]: the round
// before left states moving (else there is nothing to do and the records stay
// where they are), moving[1]: this one.
template <typename S>
__global__ __launch_bounds__(kTB) void k_jump(const Rec<S>* a, Rec<S>* b, uint64_t nq,
                                              unsigned int* moving) {
  if (moving[0] == 0) return;
  bool on = false;
  for (uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x; q < nq;
       q += (uint64_t)gridDim.x * kTB) {
    Rec<S> r = a[q];
#pragma unroll 1
    for (int hop = 0; hop < 3 && r.nxt != end_of<S>(); ++hop) {
      const Rec<S> u = a[r.nxt];
      r.nxt = u.nxt;
      r.last = u.last;
      r.dist += u.dist;
      r.mn = min(r.mn, u.mn);
    }
    on |= r.nxt != end_of<S>();
    b[q] = r;
  }
  flag_moving(moving + 1, on);
}

// Open a cycle in front of the canonical state of its smallest k-mer m (and
// end its reverse reading at that k-mer's other state).
template <typename S>
__device__ __forceinline__ void cut_at(Node<S>* nodes, uint32_t m, uint64_t* on_cycle) {
  const S x = nodes[m].succ[1];  // the state before 2m is x ^ 1
  if (x != end_of<S>()) {
    nodes[m].succ[1] = end_of<S>();
    nodes[x >> 1].succ[(x & 1) ^ 1] = end_of<S>();
  }
  atomicOr(reinterpret_cast<unsigned long long*>(&on_cycle[m >> 6]), 1ull << (m & 63));
}

// Splitter states still moving lie on cycles (every path has ended), and
// their smallest k-mer is that of the whole cycle.
template <typename S>
__global__ __launch_bounds__(kTB) void k_cut_cycles(const Rec<S>* a, uint64_t nq, Node<S>* nodes,
                                                    uint64_t* on_cycle) {
  const uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x;
  if (q >= nq || a[q].nxt == end_of<S>()) return;
  cut_at<S>(nodes, a[q].mn, on_cycle);
}

// K-mers no walker passed (their place still holds kEnd) lie on cycles
// without a splitter; the smallest k-mer of each is the one whose walk comes
// back to it without meeting a smaller one.
template <typename S>
__global__ __launch_bounds__(kTB) void k_find_leaders(const Seg<S>* seg, int64_t n,
                                                      const Node<S>* nodes, uint8_t* leader) {
  const int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x;
  if (i >= n) return;
  bool lead = false;
  if (seg[i].sid == end_of<S>()) {
    S t = nodes[i].succ[0];
    lead = true;
    for (int64_t step = 0; step < n && t != end_of<S>(); ++step) {
      if ((int64_t)(t >> 1) <= i) break;
      t = nodes[t >> 1].succ[t & 1];
    }
    lead = t == (S)(2 * i);
  }
  leader[i] = lead ? 1 : 0;
}

template <typename S>
__global__ __launch_bounds__(kTB) void k_cut_leaders(const uint8_t* leader, int64_t n,
                                                     Node<S>* nodes, uint64_t* on_cycle) {
  const int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x;
  if (i >= n || !leader[i]) return;
  cut_at<S>(nodes, (uint32_t)i, on_cycle);
}

__device__ __forceinline__ bool bit_of(const uint64_t* bits, uint64_t i) {
  return (bits[i >> 6] >> (i & 63)) & 1;
}

// The reading of state (row i, orientation o).
template <int W>
__device__ __forceinline__ void reading(const uint64_t* keys, uint64_t i, uint32_t o, uint32_t k,
                                        uint64_t (&x)[W]) {
  load_row<W>(keys, (int64_t)i, x);
  if (!o) return;
  uint64_t r[W];
  revcomp_words<W>(x, k, r);
#pragma unroll
  for (int j = 0; j < W; ++j) x[j] = r[j];
}

// At every chain's head: is the contig written in this chain's direction?  A
// path is if its first k-mer's reading is the smaller of the two (the two
// chains' first readings are never equal), a cycle where it opens at the
// canonical state.  The smallest k-mer of each written chain gets a bit.
template <int W, typename S>
__global__ __launch_bounds__(kTB) void k_heads(const uint64_t* keys, uint32_t k,
                                               const Node<S>* nodes, const uint32_t* spl,
                                               uint64_t nq, const Rec<S>* a,
                                               const uint64_t* on_cycle, uint8_t* written,
                                               uint64_t* rep) {
  const uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x;
  if (q >= nq) return;
  const uint64_t i = spl[q >> 1];
  if (nodes[i].succ[(q & 1) ^ 1] != end_of<S>()) return;  // not a head
  const uint32_t mn = a[q].mn;
  bool w;
  if (bit_of(on_cycle, mn)) {
    w = i == mn && !(q & 1);
  } else {
    const uint64_t other = (uint64_t)a[q].last ^ 1;  // head of the mirror chain
    uint64_t x[W], y[W];
    reading<W>(keys, i, (uint32_t)(q & 1), k, x);
    reading<W>(keys, spl[other >> 1], (uint32_t)(other & 1), k, y);
    w = !words_less<W>(y, x);
  }
  written[q] = w ? 1 : 0;
  if (w) atomicOr(reinterpret_cast<unsigned long long*>(&rep[mn >> 6]), 1ull << (mn & 63));
}

__global__ __launch_bounds__(kTB) void k_bit_counts(const uint64_t* bits, int64_t words,
                                                    uint32_t* cnt) {
  const int64_t w = (int64_t)blockIdx.x * kTB + threadIdx.x;
  if (w <= words) cnt[w] = w < words ? (uint32_t)__popcll(bits[w]) : 0u;
}

// The contigs' sizes in contig order.  totals[0] collects the k-mers on
// cycles.
template <typename S>
__global__ __launch_bounds__(kTB) void k_contig_sizes(
    uint32_t k, const Node<S>* nodes, const uint32_t* spl, uint64_t nq, const Rec<S>* a,
    const uint64_t* on_cycle, const uint8_t* written, const uint64_t* rep, const uint32_t* rcnt,
    uint64_t n_contigs, uint64_t* lens, int64_t* n_kmers, unsigned long long* depth,
    uint8_t* cycle, unsigned long long* totals, unsigned int* bad) {
  const uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x;
  if (q >= nq) return;
  if (nodes[spl[q >> 1]].succ[(q & 1) ^ 1] != end_of<S>() || !written[q]) return;
  const Rec<S> r = a[q];
  const uint64_t c = bit_rank(rep, rcnt, r.mn);
  if (c >= n_contigs) {
    atomicOr(bad, 1u);
    return;
  }
  const bool cyc = bit_of(on_cycle, r.mn);
  n_kmers[c] = (int64_t)r.dist + 1;
  lens[c] = (uint64_t)k + r.dist;
  depth[c] = 0;
  cycle[c] = cyc ? 1 : 0;
  if (cyc) atomicAdd(&totals[0], (unsigned long long)r.dist + 1ull);
}

// Every splitter state's place in its contig; the written chains add up their
// stretches' counts, and their heads write the contig's first k - 1 bases.
template <int W, typename S>
__global__ __launch_bounds__(kTB) void k_place(const uint64_t* keys, uint32_t k,
                                               const uint32_t* spl, uint64_t nq, const Rec<S>* a,
                                               const uint8_t* written, const uint64_t* rep,
                                               const uint32_t* rcnt, const uint64_t* offs,
                                               uint64_t n_contigs,
                                               const unsigned long long* seg_depth, char* seq,
                                               unsigned long long* depth, Place* place,
                                               unsigned int* bad) {
  const uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x;
  if (q >= nq) return;
  const uint64_t h = (uint64_t)a[q ^ 1].last ^ 1;  // head of the chain through q
  const Rec<S> rh = a[h];
  const uint64_t c = bit_rank(rep, rcnt, rh.mn);
  const uint32_t mine = a[q].dist;
  Place p{0, 0xffffffffu, 1};
  if (c >= n_contigs || mine > rh.dist) {  // inconsistent chains: refuse to place
    atomicOr(bad, 2u);
    place[q] = p;
    return;
  }
  const bool w = written[h] != 0;
  p.start = offs[c] + (w ? rh.dist - mine : mine);
  p.contig = (uint32_t)c;
  p.dir = w ? 1 : -1;
  place[q] = p;
  if (!w) return;
  atomicAdd(&depth[c], seg_depth[q]);
  if (h != q) return;
  uint64_t x[W];
  reading<W>(keys, spl[q >> 1], (uint32_t)(q & 1), k, x);
  const int up = 64 * W - 2 * (int)k;  // base 0 to the top of word 0 (2 .. 62)
#pragma unroll
  for (int j = 0; j < W; ++j) x[j] = (x[j] << up) | (j + 1 < W ? x[j + 1] >> (64 - up) : 0ull);
  char* to = seq + offs[c];
  for (uint32_t b = 0; b + 1 < k; b += 8) {  // eight bases, the top 16 bits
    uint64_t eight = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      eight |= (uint64_t)((0x54474341u >> (8 * (uint32_t)((x[0] >> (62 - 2 * e)) & 3))) & 0xffu)
               << (8 * e);
    if (b + 8 < k) {  // not past the k - 1 bases
      __builtin_memcpy(to + b, &eight, 8);
    } else {
      for (uint32_t e = 0; b + e + 1 < k; ++e) to[b + e] = (char)(eight >> (8 * e));
    }
#pragma unroll
    for (int j = 0; j < W; ++j) x[j] = (x[j] << 16) | (j + 1 < W ? x[j + 1] >> 48 : 0ull);
  }
}

// Every k-mer's last base in its contig's reading, and its contig.
//
// Bound by one scattered byte store and one random place record per row (the
// records are a few per cent of the rows); the rows themselves stream.  1.6e8
// rows: 5.0 ms, from 12.1 ms with an atomic on the contig's depth per row.
template <int W, typename S>
__global__ __launch_bounds__(kTB) void k_emit(const uint64_t* keys, int64_t n, uint32_t k,
                                              const Seg<S>* seg, const Place* place, uint64_t nq,
                                              uint64_t total, char* seq, uint32_t* row_contig,
                                              unsigned int* bad) {
  const int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x;
  if (i >= n) return;
  const Seg<S> sg = seg[i];
  if ((uint64_t)sg.sid >= nq) {
    atomicOr(bad, 4u);
    return;
  }
  const Place p = place[sg.sid];
  const uint64_t at = p.start + (p.dir > 0 ? (uint64_t)sg.off : 0 - (uint64_t)sg.off) + k - 1;
  if (p.contig == 0xffffffffu || at >= total) {
    atomicOr(bad, 8u);
    return;
  }
  const int top = 2 * (int)k - 64 * (W - 1);
  const uint32_t last = (uint32_t)(keys[i * W + W - 1] & 3);
  const uint32_t first = (uint32_t)((keys[i * W] >> (top - 2)) & 3);
  const char letters[4] = {'A', 'C', 'G', 'T'};
  // sg is the canonical state's place: the mirror reads the reverse complement
  seq[at] = letters[p.dir > 0 ? last : 3 - first];
  row_contig[i] = p.contig;
}

// ---- exclusive prefix sum over uint64 (block scan + recursion on block sums)

constexpr int kScanItems = 4;
constexpr int kScanTile = kTB * kScanItems;

__global__ __launch_bounds__(kTB) void k_scan_tile(const uint64_t* in, uint64_t* out,
                                                   int64_t n, uint64_t* sums) {
  __shared__ uint64_t wsum[kTB / 64];
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint64_t v[kScanItems], run = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    v[j] = (t0 + j < n) ? in[t0 + j] : 0;
    run += v[j];
  }
  unsigned long long inc = run;  // inclusive scan of the thread totals in the wave
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint64_t before = inc - run;
  for (int q = 0; q < wave; ++q) before += wsum[q];
  uint64_t acc = before;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    if (t0 + j < n) out[t0 + j] = acc;
    acc += v[j];
  }
  if (threadIdx.x == kTB - 1) sums[blockIdx.x] = acc;
}

__global__ __launch_bounds__(kTB) void k_scan_add(uint64_t* out, int64_t n,
                                                  const uint64_t* offs) {
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  const uint64_t add = offs[blockIdx.x];
#pragma unroll
  for (int j = 0; j < kScanItems; ++j)
    if (t0 + j < n) out[t0 + j] += add;
}

// out[i] = in[0] + ... + in[i-1]; *total (device) = the sum of all.
int scan_exclusive(Pool* pool, const uint64_t* in, uint64_t* out, int64_t n, uint64_t* total,
                   hipStream_t s) {
  const int64_t blocks = (n + kScanTile - 1) / kScanTile;
  if (n == 0) {
    launch_fill_u64(total, 1, 0ull, s);
    return KH_OK;
  }
  Buf<uint64_t> sums(pool), offs(pool);
  KH_TRY(sums.alloc(blocks));
  KH_TRY(offs.alloc(blocks));
  hipLaunchKernelGGL(k_scan_tile, dim3((unsigned)blocks), dim3(kTB), 0, s, in, out, n, sums.p);
  HIP_TRY(hipGetLastError());
  if (blocks == 1) {
    HIP_TRY(hipMemcpyAsync(total, sums.p, 8, hipMemcpyDeviceToDevice, s));
    launch_fill_u64(offs.p, 1, 0ull, s);
  } else {
    KH_TRY(scan_exclusive(pool, sums.p, offs.p, blocks, total, s));
  }
  hipLaunchKernelGGL(k_scan_add, dim3((unsigned)blocks), dim3(kTB), 0, s, out, n, offs.p);
  HIP_TRY(hipGetLastError());
  return KH_OK;
}

unsigned grid(int64_t n) { return (unsigned)((n + kTB - 1) / kTB); }

// One k-mer in mask + 1 is a splitter.  Longer stretches mean fewer records to
// rank and place; shorter ones more walkers in flight and a shorter longest
// walk (about log(walkers) times the mean), which is what a small table waits
// for.  The call at one in 16 / 32 / 64 (k = 21): 5.9e5 rows 0.39 / 0.44 / 0.52
// ms, 2.0e6 0.64 / 0.62 / 0.71, 1.1e7 2.20 / 2.09 / 2.11, 1.6e7 3.14 / 2.89 /
// 2.93, 2.1e7 4.34 / 3.98 / 3.92, 6.8e7 17.4 / 16.0 / 15.4, 1.6e8 46.1 / 41.3 /
// 39.2 (one in 8 is slower throughout, one in 128 up to 6.8e7 rows).
uint32_t sample_mask(int64_t n) { return n < (3 << 19) ? 15u : n < (1 << 24) ? 31u : 63u; }

template <int W, typename S>
int traverse_ws(kh_ctx* ctx, const kh_table* t, hipStream_t s, kh_contigs* out) {
  Pool* pool = &ctx->pool;
  const int64_t n = t->n_rows;
  const uint32_t k = t->k;
  const int64_t words = (n + 63) / 64;
  const uint32_t mask = sample_mask(n);
  // ---- successors of every state
  Buf<Node<S>> nodes(pool);
  KH_TRY(nodes.alloc(n));
  {
    Buf<uint32_t> start(pool);
    RowIndex ix{};
    KH_TRY(row_index_build(pool, t->keys, n, k, start, &ix, s));
    hipLaunchKernelGGL((k_nodes<S>), dim3(grid(n)), dim3(kTB), 0, s, t->counts, n, nodes.p);
    hipLaunchKernelGGL((k_link<W, S>), dim3(grid(n)), dim3(kTB), 0, s, t->keys, t->codes, n, k,
                       ix, nodes.p);
    HIP_TRY(hipGetLastError());
  }
  // ---- splitters, walks, ranks; once more after opening cycles
  Buf<uint64_t> bits(pool), on_cycle(pool), scal(pool);
  Buf<uint32_t> cnt(pool), part(pool), spl(pool), flags(pool);
  Buf<Seg<S>> seg(pool);
  Buf<Rec<S>> recs[2] = {Buf<Rec<S>>(pool), Buf<Rec<S>>(pool)};
  Buf<unsigned long long> seg_depth(pool);
  constexpr int kMaxRounds = 20;  // 4^18 > 2^33 states
  KH_TRY(bits.alloc(words));
  KH_TRY(on_cycle.alloc(words));
  KH_TRY(cnt.alloc(words + 1));
  KH_TRY(part.alloc(scan_tmp_words(words + 1)));
  KH_TRY(seg.alloc(n));
  // scal: [0] k-mers placed, [1] contig bases, [2] k-mers on cycles, [3] bad;
  // flags: one word per round
  KH_TRY(scal.alloc(4));
  KH_TRY(flags.alloc(kMaxRounds + 2));
  launch_fill_u64(on_cycle.p, words, 0ull, s);
  uint64_t nq = 0;  // splitter states
  int cur = 0;
  for (int attempt = 0;; ++attempt) {
    hipLaunchKernelGGL((k_split_mark<S>), dim3(grid((words + 1) * 64)), dim3(kTB), 0, s, nodes.p,
                       n, mask, bits.p, cnt.p);
    HIP_TRY(hipGetLastError());
    exclusive_scan_u32(cnt.p, words + 1, part.p, s);
    uint32_t n_split = 0;
    KH_TRY(fetch(ctx, s, {&n_split, cnt.p + words, 4}));
    nq = 2 * (uint64_t)n_split;
    launch_fill_u64(scal.p, 4, 0ull, s);
    launch_fill_u64(reinterpret_cast<uint64_t*>(flags.p), (kMaxRounds + 2) / 2, 0ull, s);
    KH_TRY(spl.alloc(n_split));
    KH_TRY(recs[0].alloc(nq));
    KH_TRY(recs[1].alloc(nq));
    KH_TRY(seg_depth.alloc(nq));
    auto walk = [&](Rec<S>* rec) -> int {
      hipLaunchKernelGGL((k_split_list<S>), dim3(grid(n)), dim3(kTB), 0, s, bits.p, cnt.p, n,
                         spl.p, seg.p);
      if (nq > 0) {
        // as many walkers as the chip holds
        const unsigned blocks = std::min(grid((int64_t)nq), (unsigned)ctx->cus * 8u);
        hipLaunchKernelGGL((k_walk<S>), dim3(blocks), dim3(kTB), 0, s, nodes.p, n, spl.p, nq,
                           mask, seg.p, rec, seg_depth.p,
                           reinterpret_cast<unsigned long long*>(scal.p), flags.p);
        hipLaunchKernelGGL((k_walk_ends<S>), dim3(grid((int64_t)nq)), dim3(kTB), 0, s, bits.p,
                           cnt.p, rec, nq);
      }
      HIP_TRY(hipGetLastError());
      return KH_OK;
    };
    KH_TRY(walk(recs[0].p));
    // enough rounds for any path: 4^rounds >= splitter states.  Every launch
    // looks at the flag of the round before, so the host need not wait after
    // each; those past the last moving state return at once.
    int rounds = 1;
    while ((1ull << 2 * rounds) < nq) ++rounds;
    rounds = std::min(rounds + 1, kMaxRounds);
    for (int r = 0; r < rounds && nq > 0; ++r)
      hipLaunchKernelGGL((k_jump<S>), dim3(std::min(grid((int64_t)nq), (unsigned)ctx->cus * 8u)),
                         dim3(kTB), 0, s, recs[r & 1].p,
                         recs[(r & 1) ^ 1].p, nq, flags.p + r);
    HIP_TRY(hipGetLastError());
    uint32_t moved[kMaxRounds + 2];
    uint64_t placed = 0;
    KH_TRY(fetch(ctx, s, {moved, flags.p, sizeof moved}, {&placed, scal.p, 8}));
    int ran = 0;
    while (ran < rounds && moved[ran]) ++ran;
    out->rounds += ran;
    cur = ran & 1;
    const bool ringed = ran == rounds && moved[rounds];  // cycles with a splitter
    const bool missed = placed != (uint64_t)n;           // cycles without one
    if (!ringed && !missed) break;
    if (attempt > 0) return fail(KH_EDEVICE, "contig chains did not end after opening cycles");
    if (missed) {
      // the walks again over cleared places, to see which k-mers have none
      // (recs[cur] keeps the ranks)
      Buf<uint8_t> leader(pool);
      KH_TRY(leader.alloc(n));
      launch_fill_u64(reinterpret_cast<uint64_t*>(seg.p), (uint64_t)n * sizeof(Seg<S>) / 8,
                      ~0ull, s);
      KH_TRY(walk(recs[cur ^ 1].p));
      hipLaunchKernelGGL((k_find_leaders<S>), dim3(grid(n)), dim3(kTB), 0, s, seg.p, n, nodes.p,
                         leader.p);
      hipLaunchKernelGGL((k_cut_leaders<S>), dim3(grid(n)), dim3(kTB), 0, s, leader.p, n,
                         nodes.p, on_cycle.p);
      HIP_TRY(hipGetLastError());
    }
    if (ringed) {
      hipLaunchKernelGGL((k_cut_cycles<S>), dim3(grid((int64_t)nq)), dim3(kTB), 0, s,
                         recs[cur].p, nq, nodes.p, on_cycle.p);
      HIP_TRY(hipGetLastError());
    }
  }
  recs[cur ^ 1].reset();
  const Rec<S>* A = recs[cur].p;
  // ---- written chains, contig numbering and offsets
  Buf<uint8_t> written(pool);
  Buf<uint64_t> rep(pool);
  KH_TRY(written.alloc(nq));
  KH_TRY(rep.alloc(words));
  launch_fill_u64(rep.p, words, 0ull, s);
  hipLaunchKernelGGL((k_heads<W, S>), dim3(grid((int64_t)nq)), dim3(kTB), 0, s, t->keys, k,
                     nodes.p, spl.p, nq, A, on_cycle.p, written.p, rep.p);
  Buf<uint32_t> rcnt(pool);
  KH_TRY(rcnt.alloc(words + 1));
  hipLaunchKernelGGL(k_bit_counts, dim3(grid(words + 1)), dim3(kTB), 0, s, rep.p, words, rcnt.p);
  HIP_TRY(hipGetLastError());
  exclusive_scan_u32(rcnt.p, words + 1, part.p, s);
  uint32_t n_contigs = 0;
  KH_TRY(fetch(ctx, s, {&n_contigs, rcnt.p + words, 4}));
  const uint64_t nc = n_contigs;
  Buf<uint64_t> lens(pool), offs(pool), depth(pool);
  Buf<int64_t> nk(pool);
  Buf<uint8_t> cyc(pool);
  KH_TRY(lens.alloc(nc + 1));
  KH_TRY(offs.alloc(nc + 1));
  KH_TRY(nk.alloc(nc));
  KH_TRY(depth.alloc(nc));
  KH_TRY(cyc.alloc(nc));
  unsigned int* bad = reinterpret_cast<unsigned int*>(scal.p + 3);
  unsigned long long* dep = reinterpret_cast<unsigned long long*>(depth.p);
  hipLaunchKernelGGL((k_contig_sizes<S>), dim3(grid((int64_t)nq)), dim3(kTB), 0, s, k, nodes.p,
                     spl.p, nq, A, on_cycle.p, written.p, rep.p, rcnt.p, nc, lens.p, nk.p, dep,
                     cyc.p, reinterpret_cast<unsigned long long*>(scal.p + 2), bad);
  HIP_TRY(hipGetLastError());
  KH_TRY(scan_exclusive(pool, lens.p, offs.p, (int64_t)nc, scal.p + 1, s));
  HIP_TRY(hipMemcpyAsync(offs.p + nc, scal.p + 1, 8, hipMemcpyDeviceToDevice, s));
  uint64_t h[4];
  KH_TRY(fetch(ctx, s, {h, scal.p, 32}));
  if (h[3]) return fail(KH_EDEVICE, "inconsistent contig chains (code %u)", (unsigned)h[3]);
  const uint64_t total = h[1];
  nodes.reset();
  // ---- emission
  Buf<char> seq(pool);
  Buf<uint32_t> rowc(pool);
  Buf<Place> place(pool);
  KH_TRY(seq.alloc(total));
  KH_TRY(rowc.alloc(n));
  KH_TRY(place.alloc(nq));
  hipLaunchKernelGGL((k_place<W, S>), dim3(grid((int64_t)nq)), dim3(kTB), 0, s, t->keys, k,
                     spl.p, nq, A, written.p, rep.p, rcnt.p, offs.p, nc, seg_depth.p, seq.p, dep,
                     place.p, bad);
  hipLaunchKernelGGL((k_emit<W, S>), dim3(grid(n)), dim3(kTB), 0, s, t->keys, n, k, seg.p,
                     place.p, nq, total, seq.p, rowc.p, bad);
  HIP_TRY(hipGetLastError());
  unsigned int hbad = 0;
  KH_TRY(fetch(ctx, s, {&hbad, bad, 4}));
  if (hbad) return fail(KH_EDEVICE, "inconsistent contig chains (code %u)", hbad);
  out->cycle_kmers = (int64_t)h[2];
  out->n_contigs = (int64_t)nc;
  out->total_bases = (int64_t)total;
  out->seq = seq.release();
  out->offsets = reinterpret_cast<int64_t*>(offs.release());
  out->n_kmers = nk.release();
  out->depth = depth.release();
  out->cycle = cyc.release();
  out->row_contig = rowc.release();
  out->n_rows = n;
  return KH_OK;
}

// 32-bit states wherever they can number two readings of every row.
// KMERHIP_TRAVERSE_WIDE (a testing hook) takes the 64-bit ones.
template <int W>
int traverse_w(kh_ctx* ctx, const kh_table* t, hipStream_t s, kh_contigs* out) {
  if (t->n_rows < (1ll << 31) && !std::getenv("KMERHIP_TRAVERSE_WIDE"))
    return traverse_ws<W, uint32_t>(ctx, t, s, out);
  return traverse_ws<W, uint64_t>(ctx, t, s, out);
}

}  // namespace

int kh_scan_exclusive_u64(Pool* pool, const uint64_t* in, uint64_t* out, int64_t n,
                          uint64_t* total, hipStream_t s) {
  return scan_exclusive(pool, in, out, n, total, s);
}

static void release_contigs(kh_contigs* c) {
  if (!c->ctx) return;
  Pool& pl = c->ctx->pool;
  std::lock_guard<std::recursive_mutex> lk(pl.mu);
  pl.put(c->seq);
  pl.put(c->offsets);
  pl.put(c->n_kmers);
  pl.put(c->depth);
  pl.put(c->cycle);
  pl.put(c->row_contig);
  c->row_contig = nullptr;
  c->seq = nullptr;
  c->offsets = nullptr;
  c->n_kmers = nullptr;
  c->depth = nullptr;
  c->cycle = nullptr;
}

extern "C" int kh_traverse(kh_ctx* ctx, const kh_table* t, void* hip_stream,
                           kh_contigs** out) {
  if (!ctx || !t || !out) return fail(KH_EINVAL, "NULL argument");
  *out = nullptr;
  if (!t->ctx) return fail(KH_EINVAL, "the table's context was destroyed");
  if (t->ctx->device != ctx->device)
    return fail(KH_EINVAL, "the table lives on device %d, the context on %d", t->ctx->device,
                ctx->device);
  if (t->n_rows > (int64_t)0xfffffffe) return fail(KH_EINVAL, "too many rows");
  HIP_TRY(hipSetDevice(ctx->device));
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  kh_contigs* c = new (std::nothrow) kh_contigs();
  if (!c) return fail(KH_ENOMEM, "host allocation failed");
  c->ctx = ctx;
  c->k = t->k;
  c->source = t->serial;
  int rc = KH_OK;
  if (t->n_rows == 0) {
    Buf<int64_t> off(&ctx->pool);
    rc = off.alloc(1);
    if (rc == KH_OK) {
      launch_fill_u64(reinterpret_cast<uint64_t*>(off.p), 1, 0ull, s);
      rc = hipStreamSynchronize(s) == hipSuccess ? KH_OK : fail(KH_EDEVICE, "sync failed");
      c->offsets = off.release();
    }
  } else {
    switch ((t->k + 31) / 32) {
      case 1: rc = traverse_w<1>(ctx, t, s, c); break;
      case 2: rc = traverse_w<2>(ctx, t, s, c); break;
      case 3: rc = traverse_w<3>(ctx, t, s, c); break;
      default: rc = traverse_w<4>(ctx, t, s, c); break;
    }
  }
  if (rc != KH_OK) {
    release_contigs(c);
    delete c;
    return rc;
  }
  {
    std::lock_guard<std::recursive_mutex> lk(ctx->pool.mu);
    ctx->live_contigs.insert(c);
  }
  *out = c;
  return KH_OK;
}

extern "C" int kh_contigs_info(const kh_contigs* c, uint32_t* k, int64_t* n_contigs,
                               int64_t* total_bases, int64_t* cycle_kmers, int* rounds) {
  if (!c) return fail(KH_EINVAL, "contigs is NULL");
  if (k) *k = c->k;
  if (n_contigs) *n_contigs = c->n_contigs;
  if (total_bases) *total_bases = c->total_bases;
  if (cycle_kmers) *cycle_kmers = c->cycle_kmers;
  if (rounds) *rounds = c->rounds;
  return KH_OK;
}

extern "C" int kh_contigs_export(const kh_contigs* c, char* seq, int64_t* offsets,
                                 int64_t* n_kmers, uint64_t* depth, uint8_t* cycle,
                                 int dst_on_device) {
  if (!c) return fail(KH_EINVAL, "contigs is NULL");
  if (!c->ctx && c->n_contigs > 0) return fail(KH_EINVAL, "the contigs' context was destroyed");
  if (!c->ctx) return KH_OK;
  HIP_TRY(hipSetDevice(c->ctx->device));
  const hipMemcpyKind kind = dst_on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  const size_t m = (size_t)c->n_contigs;
  if (seq && c->total_bases) HIP_TRY(hipMemcpy(seq, c->seq, (size_t)c->total_bases, kind));
  if (offsets) HIP_TRY(hipMemcpy(offsets, c->offsets, (m + 1) * 8, kind));
  if (m) {
    if (n_kmers) HIP_TRY(hipMemcpy(n_kmers, c->n_kmers, m * 8, kind));
    if (depth) HIP_TRY(hipMemcpy(depth, c->depth, m * 8, kind));
    if (cycle) HIP_TRY(hipMemcpy(cycle, c->cycle, m, kind));
  }
  return KH_OK;
}

extern "C" int kh_contigs_device(const kh_contigs* c, const char** seq,
                                 const int64_t** offsets) {
  if (!c) return fail(KH_EINVAL, "contigs is NULL");
  if (seq) *seq = c->seq;
  if (offsets) *offsets = c->offsets;
  return KH_OK;
}

extern "C" int kh_contigs_free(kh_contigs* c) {
  if (!c) return KH_OK;
  if (c->ctx) {
    std::lock_guard<std::recursive_mutex> lk(c->ctx->pool.mu);
    c->ctx->live_contigs.erase(c);
    release_contigs(c);
  }
  delete c;
  return KH_OK;
}

// Called by kh_destroy: the contigs' device memory goes with the context.
void kh_orphan_contigs(kh_ctx* ctx) {
  for (kh_contigs* c : ctx->live_contigs) {
    c->ctx = nullptr;
    c->n_contigs = 0;
    c->total_bases = 0;
    c->seq = nullptr;
    c->offsets = nullptr;
    c->n_kmers = nullptr;
    c->depth = nullptr;
    c->cycle = nullptr;
    c->row_contig = nullptr;
  }
  ctx->live_contigs.clear();
}
