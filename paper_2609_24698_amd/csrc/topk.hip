// CSA top-k: per (row, node), keep the topk candidates with the largest
// indexer score, ties to the lower logical index, and list them ascending.
//
// Candidates of node i are the committed entries (scores from the score
// kernel) and the entries closed on i's own root path (scored here from their
// scratch indexer keys): a node never sees an entry compressed on another
// branch (Sec. 3.1, Sec. 4.1).
//
// Selection is an exact radix select on order-preserving 32-bit keys held in
// registers (committed candidate e of an NT-thread workgroup in slot e / NT of
// thread e % NT, the path entries in a slot of their own after them; NT is
// 512 for a segment and 1024 for a merge).  A key is the complement of the
// usual order-preserving bits, so the best candidates have the smallest keys
// and padding is all ones.  Up to three passes count the keys that share the
// digits found so far, each in histogram words of its own (all cleared while
// the first loads are in flight), until the bin holding the topk-th key holds
// exactly the keys still needed or every bit is fixed.  An ordered compaction
// then lists the keys below the threshold and the lowest-index keys equal to
// it.
//
// What bounds it: with few candidates a chain of dependent steps (round trips
// to memory, barriers, LDS round trips), with many the vector instructions per
// key, sixteen wavefronts sharing a compute unit.  Hence one round trip to
// memory before the selection (score slots and path entries are loaded before
// the length and the masks say which count); one barrier per pass, every
// wavefront scanning the whole histogram itself (eight conflict-free 16-byte
// reads a lane and two wavefront prefix sums), which also keeps the digits in
// scalar registers; and as few sweeps over the keys as possible, each a few
// instructions a key.  A selection among 2,048 candidates took 12.1 us in its
// workgroup with two round trips and four barriers a pass, and takes 6.1; among
// 8,192 (256 workgroups) 15.9 -> 12.0; of a ragged batch of 512 with up to
// 16,384 21.4 -> 17.0; a merge launch of 16 x 2,048 survivors 21.0 -> 16.9, with
// distances of more than 26 bits 22.2 -> 22.5.
//
// A node with up to kTopkSeg committed entries is selected by one workgroup.
// A longer node is cut into segments of kTopkSeg entries: each segment's
// workgroup keeps its own topk (a superset of its share of the node's topk),
// and a merge kernel selects the node's topk among the survivors of all its
// segments, which are already in index order.
//
// The selecting workgroup also writes its node's key list (one latent-row
// pointer per key, in attention order) so that the attention kernel starts
// from a table instead of re-deriving it; the table and a copy of the key
// count are kept by (row rank, node), the attention's own order.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "compress_body.h"
#include "node_keys.h"
#include "tv_common.h"
#include "tv_internal.h"

namespace tv {

constexpr int kMaxScratch = 64;
constexpr int kTkNT = 512;  // threads of a selecting workgroup
constexpr int kMergeNT = 1024;  // threads of a merging workgroup (one per node: the more, the fewer keys each)
constexpr int kTkNW = kTkNT / 64;
constexpr int kTkKPT = kTopkSeg / kTkNT;  // committed keys per thread of a full segment
constexpr int kTkSpec = 4;       // score slots loaded before the row's length is known
constexpr int kTkMaxK = 8192;    // largest topk: the output list below
constexpr uint32_t kPadKey = 0xFFFFFFFFu;
constexpr int kMergeWideBits = 26;  // a merge whose distances have more bits takes the wide first digit
static_assert(kTkNT * kTkKPT == kTopkSeg, "a segment fills whole slots");
static_assert(kMaxScratch <= 64, "the path entries fit the first wavefront's path slot");
static_assert(kTkMaxK < kTopkSeg, "a full segment has more candidates than a node keeps");

// Histogram words of the three passes: 13, 11 and 8 bits (a digit of up to 11 bits spreads over 2048 words), or
// 11, 11 and 10 bits in the same words.
constexpr int kHistWords = 8192 + 2048 + 2048;

template <int NT>
struct __align__(16) SelShared {
  union {
    uint32_t hist[kHistWords];  // cleared once; every pass counts in words of its own
    int32_t list[kTkMaxK];      // then the taken elements, in element order
  };
  union {
    uint32_t cnt[64][NT / 64];      // taken counts by (slot, wavefront)
    uint64_t bits[2][36 * NT / 64];  // or ballots by (slot, wavefront): below the threshold, equal to it
  };
  uint32_t wsum[NT / 64];
};

// Barrier for shared-memory hand-offs only: global loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ float dot8_bf16(uint4 a, uint4 b) {
  float s = bf2f_lo(a.x) * bf2f_lo(b.x);
  s = fmaf(bf2f_hi(a.x), bf2f_hi(b.x), s);
  s = fmaf(bf2f_lo(a.y), bf2f_lo(b.y), s);
  s = fmaf(bf2f_hi(a.y), bf2f_hi(b.y), s);
  s = fmaf(bf2f_lo(a.z), bf2f_lo(b.z), s);
  s = fmaf(bf2f_hi(a.z), bf2f_hi(b.z), s);
  s = fmaf(bf2f_lo(a.w), bf2f_lo(b.w), s);
  s = fmaf(bf2f_hi(a.w), bf2f_hi(b.w), s);
  return s;
}

template <int NT>
__device__ __forceinline__ void clear_hist(SelShared<NT> &sh) {
  uint4 *h = reinterpret_cast<uint4 *>(&sh.hist[0]);
  for (int t = threadIdx.x; t < kHistWords / 4; t += NT) h[t] = make_uint4(0u, 0u, 0u, 0u);
}

// Counter of digit d of a pass of up to BITS bits.  A lane scans PER
// consecutive digits (32 of 2048, 16 of each 1024-digit block otherwise): the
// low bits of a digit select one of PER / 4 blocks of words and the rest the
// word there, so that the lane's digits lie in one 16-byte piece of each block
// and the lanes' reads of a block are contiguous.
template <int BITS>
__device__ __forceinline__ uint32_t *hist_at(uint32_t *h, uint32_t d) {
  if constexpr (BITS == 13)
    return h + ((d & ~1023u) | ((d >> 2) & 255u) | ((d & 3u) << 8));  // eight blocks of 1024 digits
  else
    return h + ((d >> 3) | ((d & 7u) << 8));
}

// Keys a pass counts and the digits it finds, the same in every wavefront.
struct Threshold {
  uint32_t prefix, pmask;  // the k smallest keys: (key & pmask) < prefix, and
  int remaining;           // the `remaining` lowest elements with (key & pmask) == prefix
  bool all_eq;             // every key equal to the prefix is taken
};

// Threshold of the k smallest of the keys the workgroup holds: key[j], j < nr
// (padding among them), and pk where pk_live; only the low `bits` bits of a
// key may be set.  At least k keys are real.  The histograms are clear on
// entry and visible.  WIDE: digits of 13, 11 and 8 bits, else 11, 11 and 10.
// Many keys want the wide first digit (the scores crowd into few exponents: it
// leaves fewer keys in the threshold bin, usually one pass less, and fewer
// lanes on one counter); it costs a second barrier, since the scan of 8192
// counters is shared out over the wavefronts.  Padding never enters an early
// end: a bin that ends the search early holds exactly the real keys still
// needed, and after the last digit padding has a bin of its own behind every
// real key.
template <bool WIDE, int NS, int KPT, int NT>
__device__ __forceinline__ Threshold radix_threshold(const uint32_t (&key)[KPT], int nr, uint32_t pk, bool pk_live,
                                                     int k, int bits, SelShared<NT> &sh) {
  static_assert(NS <= KPT && NT >= 512, "slots; eight wavefronts share the wide scan");
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Threshold t{0u, 0u, k, false};
  int left = bits;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    constexpr int kW[2][3] = {{11, 11, 10}, {13, 11, 8}};
    constexpr int kAt[2][3] = {{0, 2048, 4096}, {0, 8192, 8192 + 2048}};
    const bool wide = WIDE && p == 0;
    const int nb = std::min(kW[WIDE][p], left);
    const int sft = left - nb;
    const uint32_t dmask = (1u << nb) - 1u;
    uint32_t *h = sh.hist + kAt[WIDE][p];
    auto at = [&](uint32_t d) { return wide ? hist_at<13>(h, d) : hist_at<11>(h, d); };
    // The slot bound, laundered through a scalar move each pass: a bound known
    // across passes becomes one lane mask per slot, kept for every pass.
    int nr_p;
    asm volatile("s_mov_b32 %0, %1" : "=s"(nr_p) : "s"(nr));
#pragma unroll
    for (int j = 0; j < NS; ++j)
      if (j < nr_p && (key[j] & t.pmask) == t.prefix) atomicAdd(at((key[j] >> sft) & dmask), 1u);
    if (pk_live && (pk & t.pmask) == t.prefix) atomicAdd(at((pk >> sft) & dmask), 1u);
    lds_barrier();
    uint32_t below = 0u;  // counts below the scanned block
    int d0 = 0;           // its first digit
    const uint4 *h4 = reinterpret_cast<const uint4 *>(h);
    uint32_t local = 0u;
    if (wide) {  // wavefront w sums block w, then every wavefront scans the block that holds the threshold
      if (NT == 512 || wv < 8) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint4 x = h4[256 * wv + 64 * u + lane];
          local += (x.x + x.y) + (x.z + x.w);
        }
      }
      const uint32_t sum = wave_total(local);
      if (lane == 0) sh.wsum[wv] = sum;
      lds_barrier();
      const uint32_t ws = lane < NT / 64 ? sh.wsum[lane] : 0u;
      const uint32_t wi = wave_prefix_sum(ws);
      const int wb = __ffsll((unsigned long long)__builtin_amdgcn_ballot_w64(wi >= (uint32_t)t.remaining)) - 1;
      below = (uint32_t)__builtin_amdgcn_readlane((int)(wi - ws), wb);
      d0 = 1024 * wb;
      h4 += 256 * wb;
      local = 0u;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint4 x = h4[64 * u + lane];
        local += (x.x + x.y) + (x.z + x.w);
      }
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint4 x = h4[64 * u + lane];
        local += (x.x + x.y) + (x.z + x.w);
      }
    }
    // the first lane whose running sum reaches `remaining` holds the digit,
    // found by a second scan over its `per` digits
    const int per = wide ? 16 : 32;
    const uint32_t incl = wave_prefix_sum(local) + below;
    const int f = __ffsll((unsigned long long)__builtin_amdgcn_ballot_w64(incl >= (uint32_t)t.remaining)) - 1;
    const uint32_t above_f = (uint32_t)__builtin_amdgcn_readlane((int)(incl - local), f);
    const uint32_t c = lane < per ? *at((uint32_t)(d0 + per * f + lane)) : 0u;
    const uint32_t incl2 = wave_prefix_sum(c) + above_f;
    const int g = __ffsll((unsigned long long)__builtin_amdgcn_ballot_w64(lane < per && incl2 >= (uint32_t)t.remaining)) - 1;
    const int c_g = __builtin_amdgcn_readlane((int)c, g);
    const int above = __builtin_amdgcn_readlane((int)incl2, g) - c_g;
    t.prefix |= (uint32_t)(d0 + per * f + g) << sft;
    t.pmask |= dmask << sft;
    t.remaining -= above;
    t.all_eq = c_g == t.remaining;
    if (t.all_eq) break;
    left = sft;
    if (left == 0) break;
  }
  return t;
}

// The lanes whose key the threshold takes for certain (g), and those equal to
// it (q): with kAll every equal key is taken and g holds both.
template <bool kAll>
__device__ __forceinline__ void taken_ballots(uint32_t kv, bool live, const Threshold &t, uint32_t pad, uint64_t &g,
                                              uint64_t &q) {
  const uint32_t km = kv & t.pmask;
  if constexpr (kAll) {
    g = __builtin_amdgcn_ballot_w64(live && km <= t.prefix);
    q = 0ull;
  } else {
    g = __builtin_amdgcn_ballot_w64(live && km < t.prefix);
    q = __builtin_amdgcn_ballot_w64(live && km == t.prefix && kv != pad);
  }
}

// The compiler's lane write: v with lane `lane` replaced by the wavefront-uniform
// x.  (Not inline assembly: the wait states a lane write needs after a compare
// has written its scalar source are the compiler's to insert.)
extern "C" __device__ uint32_t tv_writelane(uint32_t x, uint32_t lane, uint32_t v) __asm("llvm.amdgcn.writelane.i32");
template <int J>
__device__ __forceinline__ void put_lane(uint32_t &v, uint32_t x) {
  v = tv_writelane(x, J, v);
}
template <int... J, typename F>
__device__ __forceinline__ void for_slots(std::integer_sequence<int, J...>, F &&f) {
  (f(std::integral_constant<int, J>{}), ...);
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Ordered compaction of the keys the threshold takes: the element index of the
// pos-th taken key (in element order: slot j < nr, then the path slot with pk
// where pk_live, whose elements are n0 + thread) goes to sh.list[pos].  The
// list is complete after the caller's next barrier.
//
// Few slots: a count per (slot, wavefront) through LDS, one barrier, a prefix
// sum over the slots in every wavefront (lane j: slot j), then every thread
// writes its own taken elements.
template <bool kAll, int NS, int KPT, int NT>
__device__ __forceinline__ void compact_slots(const uint32_t (&key)[KPT], int nr, uint32_t pk, bool pk_live, int n0,
                                              Threshold t, SelShared<NT> &sh) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t mine = 0u;  // lane j: counts of slot j, taken for certain | equal << 16 (each below 2^16)
  auto count = [&](int j, uint32_t kv, bool live) {
    uint64_t g, q;
    taken_ballots<kAll>(kv, live, t, kPadKey, g, q);
    const uint32_t n = (uint32_t)__popcll(g) | ((uint32_t)__popcll(q) << 16);
    if (lane == j) mine = n;
  };
#pragma unroll
  for (int j = 0; j < NS; ++j)
    if (j < nr) count(j, key[j], true);
  count(nr, pk, pk_live);
  sh.cnt[lane][wv] = mine;
  lds_barrier();
  asm volatile("" : "+s"(t.prefix));  // the ballots are formed again, not kept across the barrier
  uint32_t total = 0u, before = 0u;
#pragma unroll
  for (int w4 = 0; w4 < NW / 4; ++w4) {
    const uint4 c = reinterpret_cast<const uint4 *>(&sh.cnt[lane][0])[w4];
    const uint32_t cw[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      total += cw[e];
      before += 4 * w4 + e < wv ? cw[e] : 0u;
    }
  }
  const uint32_t base = wave_prefix_sum(total) - total + before;  // lane j: counts before this wavefront's slot j
  auto emit = [&](int j, uint32_t kv, bool live, int e) {
    uint64_t g, q;
    taken_ballots<kAll>(kv, live, t, kPadKey, g, q);
    const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)base, j);
    const int gr = (int)((b0 & 0xFFFFu) + lanes_below(g));
    if constexpr (kAll) {
      if ((g >> lane) & 1ull) sh.list[gr] = e;
    } else {
      const int qr = (int)((b0 >> 16) + lanes_below(q));
      if (((g >> lane) & 1ull) || (((q >> lane) & 1ull) && qr < t.remaining))
        sh.list[gr + std::min(qr, t.remaining)] = e;
    }
  };
#pragma unroll
  for (int j = 0; j < NS; ++j)
    if (j < nr) emit(j, key[j], true, tid + NT * j);
  emit(nr, pk, pk_live, n0 + tid);
}

// Many slots, few of them taken: each wavefront's ballots (lane j keeps slot
// j's) go to LDS as a bitmap in element order; thread w then takes 64-bit word
// w, finds the taken elements before it by a prefix sum, and writes its own.
template <bool kAll, int NS, int KPT, int NT>
__device__ __forceinline__ void compact_words(const uint32_t (&key)[KPT], int nr, uint32_t pk, bool pk_live, int n0,
                                              const Threshold &t, uint32_t pad, SelShared<NT> &sh) {
  constexpr int NW = NT / 64;
  static_assert(NS + 1 <= 36 && (NS + 1) * NW <= NT, "the bitmap fits, a thread per word");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t glo = 0u, ghi = 0u, qlo = 0u, qhi = 0u;
  for_slots(std::make_integer_sequence<int, NS>{}, [&](auto j) {
    if (j < nr) {
      uint64_t g, q;
      taken_ballots<kAll>(key[j], true, t, pad, g, q);
      put_lane<j>(glo, (uint32_t)g);
      put_lane<j>(ghi, (uint32_t)(g >> 32));
      if constexpr (!kAll) {
        put_lane<j>(qlo, (uint32_t)q);
        put_lane<j>(qhi, (uint32_t)(q >> 32));
      }
    }
  });
  {
    uint64_t g, q;
    taken_ballots<kAll>(pk, pk_live, t, pad, g, q);
    if (lane == nr) {
      glo = (uint32_t)g;
      ghi = (uint32_t)(g >> 32);
      qlo = (uint32_t)q;
      qhi = (uint32_t)(q >> 32);
    }
  }
  if (lane <= nr) {
    sh.bits[0][lane * NW + wv] = ((uint64_t)ghi << 32) | glo;
    if constexpr (!kAll) sh.bits[1][lane * NW + wv] = ((uint64_t)qhi << 32) | qlo;
  }
  lds_barrier();
  const int nw = (nr + 1) * NW;
  if (64 * wv >= nw) return;
  auto word = [&](int k, int w) { return w < nw ? sh.bits[k][w] : 0ull; };
  auto counts = [&](uint64_t g, uint64_t q) { return (uint32_t)__popcll(g) | ((uint32_t)__popcll(q) << 16); };
  uint32_t before = 0u;
  for (int v = 0; v < wv; ++v)
    before += counts(word(0, 64 * v + lane), kAll ? 0ull : word(1, 64 * v + lane));
  before = wave_total(before);
  const uint64_t g = word(0, tid), q = kAll ? 0ull : word(1, tid);
  const uint32_t mine = counts(g, q);
  before += wave_prefix_sum(mine) - mine;
  const int qb = (int)(before >> 16);
  uint64_t take = g;
  if constexpr (!kAll) {  // the lowest equal keys still needed
    const int nq = __popcll(q), r = std::min(std::max(t.remaining - qb, 0), nq);
    uint64_t y = q;
    if (r < nq)
      for (int c = 0; c < r; ++c) y &= y - 1ull;
    take |= r == nq ? q : q ^ y;
  }
  int pos = (int)(before & 0xFFFFu) + (kAll ? 0 : std::min(qb, t.remaining));
  const int j = tid / NW;
  const int e0 = j == nr ? n0 + 64 * (tid % NW) : NT * j + 64 * (tid % NW);
  while (take) {
    sh.list[pos++] = e0 + (__ffsll((unsigned long long)take) - 1);
    take &= take - 1ull;
  }
}

// Latent row of CSA entry s of node (b, i): committed entries from the pool,
// path entries from the scratch slot of the path node that closed them.
__device__ __forceinline__ const uint16_t *csa_row(const tv_dims &d, const NodeKeys &nk, int b, int s,
                                                   const int32_t *path, const uint16_t *c4, int64_t c4b,
                                                   const int32_t *page_table,
                                                   const uint16_t *scr_c4) {
  if (s < nk.n4) return c4 + committed_slot(d, page_table, c4b, b, s, d.ratio_csa) * d.d_row;
  int64_t dd = (int64_t)(s + 1) * d.ratio_csa - 1 - nk.L;
  if (dd < 0 || dd > nk.p - nk.L) dd = 0;  // defensive: stay on the node's own path
  return scr_c4 + ((int64_t)b * d.D + path[dd]) * (d.d_row + d.d_idx);
}

// Key of a real candidate: the complement of the order-preserving bits of its
// score (a larger score has a smaller key, -0 equals +0), below kPadKey (only
// the two all-ones negative NaN patterns share the last key).
__device__ __forceinline__ uint32_t live_key(float s) {
  const uint32_t u = __float_as_uint(s + 0.0f);
  return min((int32_t)u < 0 ? u : u ^ 0x7FFFFFFFu, kPadKey - 1u);
}

__device__ __forceinline__ int topk_segments(int n4) { return n4 <= kTopkSeg ? 1 : (n4 + kTopkSeg - 1) / kTopkSeg; }

// One workgroup per (node, segment).  Segment 0 of node 0 of a row also ranks
// the row by length for the attention's row order, and segment 0 of every
// node writes the node's non-CSA keys into its key table.
struct TopkSmem {
  SelShared<kTkNT> sh;
  float scr_score[kMaxScratch];
  int wcnt[kTkNW];
  int32_t path[64], hca_nd[64];
};

__device__ __forceinline__ void topk_node(const tv_dims &d, const CacheView &c, const uint16_t *__restrict__ tree_u,
                                          const uint64_t *__restrict__ anc, const int32_t *__restrict__ depth,
                                          const uint16_t *__restrict__ scr_c4, const uint16_t *__restrict__ scr_c128,
                                          const uint16_t *__restrict__ q_idx, const uint16_t *__restrict__ w_idx,
                                          const float *__restrict__ scores, int score_stride,
                                          int32_t *__restrict__ sel, int32_t *__restrict__ row_status,
                                          int32_t *__restrict__ row_order, int32_t *__restrict__ row_rank,
                                          const uint16_t **__restrict__ keytab, int keytab_stride,
                                          int32_t *__restrict__ nkeys_tab, int32_t *__restrict__ nkeys_rank,
                                          int max_seg, int32_t *__restrict__ surv_idx,
                                          uint32_t *__restrict__ surv_key, uint32_t *__restrict__ surv_worst, int blk,
                                          TopkSmem &sm) {
  SelShared<kTkNT> &sh = sm.sh;
  float *scr_score = sm.scr_score;
  int *wcnt = sm.wcnt;
  int32_t *path = sm.path, *hca_nd = sm.hca_nd;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t node = blk / max_seg;
  const int seg = blk - (int)node * max_seg;
  const int b = (int)(node / d.D);
  const int i = (int)(node - (int64_t)b * d.D);
  const int d_u = d.d_row + d.d_idx;
  // One round trip: everything whose address is known from (row, node, lane).
  // That includes the segment's first kTkSpec score slots, loaded before the
  // row's length says how many exist (clamped to the node's score area; what
  // lies past the length is dropped), and, for wavefront w, the indexer key of
  // node w's scratch entry, which counts only if w closes an entry on the path.
  const int32_t status = row_status[b];
  const int32_t L = c.len[b];
  const uint64_t m = anc[node];
  const bool flat = d.page_size == 0;
  const int64_t c4b = flat ? c.c4_base[b] : 0, c128b = flat ? c.c128_base[b] : 0;
  const int dl = lane < d.D ? depth[(int64_t)b * d.D + lane] : 0;  // depth of the row's node `lane`
  const int c0 = seg * kTopkSeg;
  const float *sc = scores + node * score_stride + c0;
  const int area = std::max(score_stride - c0, 1);  // a segment below max_seg starts inside the area
  float raw[kTkSpec];
#pragma unroll
  for (int j = 0; j < kTkSpec; ++j) raw[j] = sc[std::min(tid + kTkNT * j, area - 1)];
  const int hl = lane >> 3, cc = lane & 7;  // path-entry scoring: head h0 + hl, channels 8cc..8cc+7
  uint4 qv0 = make_uint4(0, 0, 0, 0);
  float wh0 = 0.f;
  if (hl < d.H_idx) {
    qv0 = *reinterpret_cast<const uint4 *>(q_idx + (node * d.H_idx + hl) * 64 + 8 * cc);
    wh0 = bf2f(w_idx[node * d.H_idx + hl]);
  }
  auto scr_key = [&](int nd) {
    return *reinterpret_cast<const uint4 *>(scr_c4 + ((int64_t)b * d.D + nd) * d_u + d.d_row + 8 * cc);
  };
  const uint4 kv0 = scr_key(std::min(wv, d.D - 1));
  clear_hist<kTkNT>(sh);
  // Rank of row b by (committed length descending, row ascending), for every
  // row whatever its status: row_order[rank] = b, row_rank[b] = rank.  The
  // key table and a copy of the key count are kept by (rank, node), so the
  // attention reads them from its workgroup index without the row first.
  // Each wave's count goes to LDS now; the rank is summed after the next
  // barrier the workgroup passes anyway.
  int nb = 0;
  for (int r = tid; r < d.B; r += kTkNT) {
    const int32_t Lr = c.len[r];
    nb += (Lr > L || (Lr == L && r < b)) ? 1 : 0;
  }
  nb = (int)wave_total((uint32_t)nb);
  if (lane == 0) wcnt[wv] = nb;
  auto rank_of_row = [&]() {  // after a barrier
    int rk = 0;
#pragma unroll
    for (int w = 0; w < kTkNW; ++w) rk += wcnt[w];
    if (i == 0 && seg == 0 && tid == 0) {
      row_order[rk] = b;
      row_rank[b] = rk;
    }
    return rk;
  };
  const bool bad_len = !len_ok(L, d.max_len);
  if (status != TV_ROW_OK || bad_len) {  // the attention skips the node
    __syncthreads();
    const int rk = rank_of_row();
    if (seg == 0 && tid == 0) nkeys_rank[(int64_t)rk * d.D + i] = 0;
    if (status == TV_ROW_OK && i == 0 && seg == 0 && tid == 0) row_status[b] = TV_ROW_BAD_LEN;
    return;
  }
  const int n4 = L / d.ratio_csa;
  const int nseg = topk_segments(n4);
  if (seg >= nseg) return;
  const bool last = seg == nseg - 1;
  const int cn = std::min(n4, c0 + kTopkSeg) - c0;  // committed candidates of this segment

  // The node's root path (its key layout) from the ancestor mask, no barrier.
  uint64_t csa_mask;
  const NodeKeys nk = path_keys(d, L, i, m, dl, path, hca_nd, csa_mask);

  // Entries closed on the root path take the consecutive logical indices
  // n4, n4+1, ... in depth (= node index) order; the last segment scores them.
  const int nscr = last ? __popcll(csa_mask) : 0;
  if (last) {
    // Wave w takes the entries of nodes w, w + 8, ...; lane (h8, c) holds
    // channels 8c..8c+7 of head h0 + h8, for head groups h0.
    for (int nd = wv; nd < d.D; nd += kTkNW) {
      if (!((csa_mask >> nd) & 1ull)) continue;
      const uint4 kv = nd == wv ? kv0 : scr_key(nd);
      float sum = 0.f;
      for (int h0 = 0; h0 < d.H_idx; h0 += 8) {
        const int h = h0 + hl;
        float part = 0.f, wh = 0.f;
        if (h < d.H_idx) {
          const uint4 qv =
              h0 == 0 ? qv0 : *reinterpret_cast<const uint4 *>(q_idx + (node * d.H_idx + h) * 64 + 8 * cc);
          part = dot8_bf16(qv, kv);
          wh = h0 == 0 ? wh0 : bf2f(w_idx[node * d.H_idx + h]);
        }
        part += __shfl_xor(part, 1, 64);
        part += __shfl_xor(part, 2, 64);
        part += __shfl_xor(part, 4, 64);
        float term = wh * fmaxf(part, 0.f);
        term += __shfl_xor(term, 8, 64);
        term += __shfl_xor(term, 16, 64);
        term += __shfl_xor(term, 32, 64);
        sum += term;
      }
      if (lane == 0) scr_score[__popcll(csa_mask & ((1ull << nd) - 1ull))] = sum;
    }
  }
  lds_barrier();  // path, hca_nd, the path-entry scores, the clear histograms and the rank's wave counts are visible
  const int64_t rnode = (int64_t)rank_of_row() * d.D + i;
  const int seg_n = cn + nscr;  // path entries follow the committed ones of the last segment

  // The node's key table: non-CSA keys here, selected CSA entries below.
  const uint16_t **tab = keytab + rnode * keytab_stride;
  if (seg == 0) {
    for (int t = nk.nsel + tid; t < nk.n_keys; t += kTkNT)
      tab[t] = key_row(d, nk, b, t, nullptr, path, hca_nd, c.ring, c.c4, c4b, c.c128, c128b, scr_c4, scr_c128,
                       tree_u, c.page_table);
    if (tid == 0) {
      nkeys_tab[node] = nk.n_keys;
      nkeys_rank[rnode] = nk.n_keys;
    }
  }

  const int k = d.topk;
  int32_t *out = sel + node * k;  // single segment: the node's selection (ascending, -1 padded)
  const int64_t sv = ((int64_t)node * max_seg + seg) * k;  // segmented: survivors in index order, then padding
  const int nr = (cn + kTkNT - 1) / kTkNT;  // slots that hold committed candidates
  const bool pk_live = tid < nscr;
  const uint32_t pk = pk_live ? live_key(scr_score[tid]) : kPadKey;

  // The selection with the committed candidates in up to NS slots a thread:
  // the taken elements in element order in sh.list, and the threshold.
  uint32_t worst = kPadKey - 1u;  // no taken key is larger
  auto select = [&](auto ns_tag) {
    constexpr int NS = decltype(ns_tag)::value;
    constexpr bool kFew = NS <= kTkSpec;
    uint32_t key[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j)  // slots past the segment re-read its last entry
      key[j] = __float_as_uint(
          j < kTkSpec ? raw[j < kTkSpec ? j : 0] : sc[std::max(std::min(tid + kTkNT * j, cn - 1), 0)]);
    const int whole = cn / kTkNT;  // slots without padding
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      key[j] = live_key(__uint_as_float(key[j]));
      if (j >= whole) key[j] = tid + kTkNT * j < cn ? key[j] : kPadKey;
    }
    const Threshold t = radix_threshold<!kFew, NS>(key, nr, pk, pk_live, k, 32, sh);
    worst = std::min(t.prefix | ~t.pmask, kPadKey - 1u);
    if constexpr (kFew) {
      if (t.all_eq)
        compact_slots<true, NS>(key, nr, pk, pk_live, cn, t, sh);
      else
        compact_slots<false, NS>(key, nr, pk, pk_live, cn, t, sh);
    } else {
      if (t.all_eq)
        compact_words<true, NS>(key, nr, pk, pk_live, cn, t, kPadKey, sh);
      else
        compact_words<false, NS>(key, nr, pk, pk_live, cn, t, kPadKey, sh);
    }
    lds_barrier();  // the list is complete
  };
  const bool all = seg_n <= k;  // every candidate is taken
  if (!all) {
    // the smallest body that holds the segment: fewer slots to step over, and
    // up to kTkSpec of them need no load beyond the first round trip
    if (nr <= kTkSpec)
      select(std::integral_constant<int, kTkSpec>{});
    else if (nr <= 16)
      select(std::integral_constant<int, 16>{});
    else
      select(std::integral_constant<int, kTkKPT>{});
  }
  // element t of the taken ones, -1 past them (a list entry stays inside the segment whatever it holds)
  auto taken = [&](int t) {
    return all ? (t < seg_n ? t : -1) : std::min(std::max(sh.list[t], 0), seg_n - 1);
  };
  if (nseg == 1) {  // element index = logical index
    for (int t = tid; t < k; t += kTkNT) {
      const int s = taken(t);
      out[t] = s;
      if (s >= 0) tab[t] = csa_row(d, nk, b, s, path, c.c4, c4b, c.page_table, scr_c4);
    }
  } else {
    for (int t = tid; t < k; t += kTkNT) {
      const int e = taken(t);
      surv_idx[sv + t] = e < 0 ? -1 : (e < cn ? c0 + e : n4 + (e - cn));
      surv_key[sv + t] = e < 0 ? kPadKey : live_key(e < cn ? sc[e] : scr_score[e - cn]);
    }
    // a key none of the segment's k best exceeds (no bound when it has fewer)
    if (tid == 0) surv_worst[node * max_seg + seg] = all ? kPadKey - 1u : worst;
  }
}

__global__ void __launch_bounds__(kTkNT) __attribute__((amdgpu_waves_per_eu(4))) topk_kernel(
    tv_dims d, CacheView c, const uint16_t *__restrict__ tree_u, const uint64_t *__restrict__ anc,
    const int32_t *__restrict__ depth, const uint16_t *__restrict__ scr_c4, const uint16_t *__restrict__ scr_c128,
    const uint16_t *__restrict__ q_idx, const uint16_t *__restrict__ w_idx, const float *__restrict__ scores,
    int score_stride, int32_t *__restrict__ sel, int32_t *__restrict__ row_status, int32_t *__restrict__ row_order,
    int32_t *__restrict__ row_rank, const uint16_t **__restrict__ keytab, int keytab_stride,
    int32_t *__restrict__ nkeys_tab, int32_t *__restrict__ nkeys_rank, int max_seg, int32_t *__restrict__ surv_idx,
    uint32_t *__restrict__ surv_key, uint32_t *__restrict__ surv_worst) {
  __shared__ TopkSmem sm;
  topk_node(d, c, tree_u, anc, depth, scr_c4, scr_c128, q_idx, w_idx, scores, score_stride, sel, row_status,
            row_order, row_rank, keytab, keytab_stride, nkeys_tab, nkeys_rank, max_seg, surv_idx, surv_key, surv_worst,
            blockIdx.x, sm);
}

// The top-k and, in the same grid after its workgroups, the HCA entries of
// the split compression (one workgroup per node; nodes that close no HCA
// block exit at once).  The top-k reads no HCA scratch entry (it only lists
// their addresses), so the two are independent; the HCA workgroups start as
// the short nodes' selections finish.
__global__ void __launch_bounds__(kTkNT) __attribute__((amdgpu_waves_per_eu(4))) topk_hca_kernel(
    tv_dims d, CacheView c, const uint16_t *__restrict__ tree_u, const uint64_t *__restrict__ anc,
    const int32_t *__restrict__ depth, const uint16_t *__restrict__ scr_c4, uint16_t *__restrict__ scr_c128,
    const uint16_t *__restrict__ q_idx, const uint16_t *__restrict__ w_idx, const float *__restrict__ scores,
    int score_stride, int32_t *__restrict__ sel, int32_t *__restrict__ row_status, int32_t *__restrict__ row_order,
    int32_t *__restrict__ row_rank, const uint16_t **__restrict__ keytab, int keytab_stride,
    int32_t *__restrict__ nkeys_tab, int32_t *__restrict__ nkeys_rank, int max_seg, int32_t *__restrict__ surv_idx,
    uint32_t *__restrict__ surv_key, uint32_t *__restrict__ surv_worst, const uint16_t *__restrict__ gate_w) {
  static_assert(kTkNT == kHcaNT, "one workgroup size for both roles");
  __shared__ union {
    TopkSmem t;
    HcaSmem h;
  } sm;
  const int ntk = d.B * d.D * max_seg;
  if ((int)blockIdx.x < ntk)
    topk_node(d, c, tree_u, anc, depth, scr_c4, scr_c128, q_idx, w_idx, scores, score_stride, sel, row_status,
              row_order, row_rank, keytab, keytab_stride, nkeys_tab, nkeys_rank, max_seg, surv_idx, surv_key,
              surv_worst, blockIdx.x, sm.t);
  else
    hca_node(d, c, tree_u, anc, depth, gate_w, scr_c128, row_status, false, blockIdx.x - ntk, sm.h);
}

// Merge of a segmented node: the topk of the survivors of all its segments.
// Segment s holds k slots (survivors in index order, then padding kPadKey), so
// the slots of all segments in order list the survivors in index order.  Every
// segment but the last is full and fills its k slots, and the last has a
// candidate, so there are always more than k survivors.
template <int NT>
__global__ void __launch_bounds__(NT, 1) topk_merge_kernel(tv_dims d, CacheView c, const uint64_t *__restrict__ anc,
                                                           const int32_t *__restrict__ depth,
                                                           const uint16_t *__restrict__ scr_c4,
                                                           int32_t *__restrict__ sel,
                                                           const int32_t *__restrict__ row_status,
                                                           const int32_t *__restrict__ row_rank,
                                                           const uint16_t **__restrict__ keytab, int keytab_stride,
                                                           int max_seg, const int32_t *__restrict__ surv_idx,
                                                           const uint32_t *__restrict__ surv_key,
                                                           const uint32_t *__restrict__ surv_worst) {
  __shared__ SelShared<NT> sh;
  __shared__ uint32_t worst_key;
  __shared__ int32_t path[64], hca_node[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t node = blockIdx.x;
  const int b = (int)(node / d.D);
  const int i = (int)(node - (int64_t)b * d.D);
  const int k = d.topk;
  // One round trip for everything whose address is known from (row, node,
  // lane): the row's state, the node's path, and all of the node's survivor
  // slots and bounds (those of segments the row does not have are dropped
  // once its length is known).
  const int32_t status = row_status[b];
  const int32_t L = c.len[b];
  const int32_t rank = row_rank[b];
  const int64_t c4b = d.page_size == 0 ? c.c4_base[b] : 0;
  const uint64_t m = anc[node];
  const int dl = lane < d.D ? depth[(int64_t)b * d.D + lane] : 0;
  const int64_t sv = (int64_t)node * max_seg * k;
  const uint32_t seg_worst = tid < max_seg ? surv_worst[node * max_seg + tid] : kPadKey - 1u;  // max_seg <= 64: wave 0
  const int all_slots = max_seg * k;
  constexpr int KPT = kTopkMergeCap / NT;
  static_assert(KPT * NT == kTopkMergeCap, "merge capacity");
  static_assert(KPT < 64, "a lane per slot");
  const int nr_all = (all_slots + NT - 1) / NT;
  uint32_t key[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    key[j] = j < nr_all ? surv_key[sv + std::min(tid + NT * j, all_slots - 1)] : kPadKey;
  clear_hist<NT>(sh);
  if (status != TV_ROW_OK || !len_ok(L, d.max_len)) return;
  const int n4 = L / d.ratio_csa;
  const int nseg = topk_segments(n4);
  if (nseg <= 1) return;
  const int slots = nseg * k;
  uint32_t best = kPadKey;
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    if (tid + NT * j >= slots) key[j] = kPadKey;
    best = min(best, key[j]);
  }
  best = ~wave_max_u32(~best);
  if (lane == 0) sh.wsum[tid >> 6] = best;
  if (tid < 64) {
    const uint32_t w = ~wave_max_u32(~(tid < nseg ? seg_worst : kPadKey - 1u));
    if (tid == 0) worst_key = w;
  }
  uint64_t csa_mask;
  const NodeKeys nk = path_keys(d, L, i, m, dl, path, hca_node, csa_mask);
  __syncthreads();  // the survivors' bounds, the clear histograms and the node's path are visible
  const uint16_t **tab = keytab + ((int64_t)rank * d.D + i) * keytab_stride;  // kept by (rank, node)
  int32_t *out = sel + node * k;
  const int nr = (slots + NT - 1) / NT;
  // The survivors' keys crowd into a few exponents, where a digit of leading
  // bits would put thousands of them on one counter.  The digits are therefore
  // taken from the distance to the best key, and a survivor beyond the worst
  // key of a segment that filled its k slots cannot be among the node's k best
  // and becomes padding: the distance then has fewer bits.
  best = ~wave_max_u32(~sh.wsum[lane & (NT / 64 - 1)]);
  const uint32_t worst = std::max((uint32_t)__builtin_amdgcn_readfirstlane((int)worst_key), best);
  const int bits = 32 - __clz((int)(worst - best + 1u));
  const uint32_t pad = bits == 32 ? kPadKey : (1u << bits) - 1u;  // above every distance
#pragma unroll
  for (int j = 0; j < KPT; ++j) key[j] = key[j] <= worst ? key[j] - best : pad;
  Threshold t;
  // Survivors of both signs span most of the 32 bits (few keys lie far from
  // zero): 11 bits of that put thousands on one counter (6,324 of 30,828 on a
  // 1M-token node, the merge 27 us), so such nodes take the wide first digit
  // (22.5 us).
  if (bits > kMergeWideBits)
    t = radix_threshold<true, KPT>(key, nr, pad, false, k, bits, sh);
  else
    t = radix_threshold<false, KPT>(key, nr, pad, false, k, bits, sh);
  if (t.all_eq)
    compact_words<true, KPT>(key, nr, pad, false, 0, t, pad, sh);
  else
    compact_words<false, KPT>(key, nr, pad, false, 0, t, pad, sh);
  lds_barrier();  // the list is complete
  for (int t = tid; t < k; t += NT) {
    const int s = surv_idx[sv + std::min(std::max(sh.list[t], 0), slots - 1)];
    out[t] = s;
    if (s >= 0) tab[t] = csa_row(d, nk, b, s, path, c.c4, c4b, c.page_table, scr_c4);
  }
}

int topk_max_segments(const tv_dims &d) {
  const int64_t n4 = (int64_t)d.max_len / d.ratio_csa;
  return n4 <= kTopkSeg ? 1 : (int)((n4 + kTopkSeg - 1) / kTopkSeg);
}

bool topk_supported(const tv_dims &d) {
  const int s = topk_max_segments(d);
  return d.topk <= kTkMaxK && (s == 1 || (s <= kTopkMaxSeg && (int64_t)s * d.topk <= kTopkMergeCap));
}

hipError_t launch_topk(const tv_dims &d, const CacheView &c, const uint16_t *tree_u, const uint64_t *anc,
                       const int32_t *depth, const uint16_t *scr_c4, const uint16_t *scr_c128, const uint16_t *q_idx,
                       const uint16_t *w_idx, const float *scores, int32_t score_stride, int32_t *sel,
                       int32_t *row_status, int32_t *row_order, int32_t *row_rank, const uint16_t **keytab,
                       int32_t keytab_stride, int32_t *nkeys, int32_t *nkeys_rank, int32_t *surv_idx,
                       uint32_t *surv_key, uint32_t *surv_worst, const uint16_t *hca_gate_w, uint16_t *hca_out,
                       hipStream_t s) {
  if (d.D > kMaxScratch || !topk_supported(d)) return hipErrorInvalidValue;
  const int max_seg = topk_max_segments(d);
  const int64_t ntk = (int64_t)d.B * d.D * max_seg;
  if (hca_gate_w) {  // with the HCA entries of the split compression, into hca_out (the scr_c128 buffer)
    if (!compress_split(d) || d.d_row + d.d_idx > kMaxDu || hca_out != scr_c128 ||
        ntk + (int64_t)d.B * d.D > 0x7FFFFFFF)
      return hipErrorInvalidValue;
    topk_hca_kernel<<<(unsigned)(ntk + (int64_t)d.B * d.D), kTkNT, 0, s>>>(
        d, c, tree_u, anc, depth, scr_c4, hca_out, q_idx, w_idx, scores, score_stride, sel,
        row_status, row_order, row_rank, keytab, keytab_stride, nkeys, nkeys_rank, max_seg, surv_idx, surv_key,
        surv_worst, hca_gate_w);
    return hipGetLastError();
  }
  topk_kernel<<<(unsigned)ntk, kTkNT, 0, s>>>(
      d, c, tree_u, anc, depth, scr_c4, scr_c128, q_idx, w_idx, scores, score_stride, sel, row_status, row_order,
      row_rank, keytab, keytab_stride, nkeys, nkeys_rank, max_seg, surv_idx, surv_key, surv_worst);
  return hipGetLastError();
}

hipError_t launch_topk_merge(const tv_dims &d, const CacheView &c, const uint64_t *anc, const int32_t *depth,
                             const uint16_t *scr_c4, int32_t *sel, const int32_t *row_status,
                             const int32_t *row_rank, const uint16_t **keytab, int32_t keytab_stride,
                             const int32_t *surv_idx, const uint32_t *surv_key, const uint32_t *surv_worst,
                             hipStream_t s) {
  const int max_seg = topk_max_segments(d);
  if (max_seg <= 1) return hipSuccess;
  topk_merge_kernel<kMergeNT><<<(unsigned)((int64_t)d.B * d.D), kMergeNT, 0, s>>>(d, c, anc, depth, scr_c4, sel,
                                                                                 row_status,
                                                                     row_rank, keytab, keytab_stride, max_seg,
                                                                     surv_idx, surv_key, surv_worst);
  return hipGetLastError();
}

}  // namespace tv
