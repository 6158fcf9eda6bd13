// Accepted-path refresh of the committed state.
//
// After verification only the accepted root path survives (Sec. 3.2, Sec. 4.2):
// its raw rows enter the window ring, every block it closed becomes a committed
// CSA / HCA entry (copied from the path node's scratch slot), and the committed
// length advances.  Entries compressed on rejected branches are never copied,
// so they leave no trace in the persistent state.
//
// One workgroup per row.  All checks run before the first write, so a failing
// row is left exactly as it was.  Destinations follow the cache layout: the
// ring and per-row pools, or with a paged pool the raw, CSA and HCA layers
// through the row's page table (a page it does not allocate fails the row).
// The row's loads go out together; the copies (ring rows, CSA and HCA
// entries) form one list of 16-byte chunks whose loads a thread issues
// before its stores.
//
// With FP8 indexer keys a CSA entry's indexer channels (E4M3 values held
// in bfloat16 in scratch) are narrowed, exactly, to E4M3 codes in the pool.
//
// Refresh schedule (Sec. 4.3): with a designated chain (the root path of
// primary_last[b]), whose CSA entries the compression already wrote into the
// pool, the CSA copies of accepted nodes on that chain are skipped: a single
// chain, or an accepted path that is the cached chain, needs no CSA refresh.
// HCA entries are always written here, once the path is known, all of a
// round's in one pass.
#include "pool_addr.h"

namespace tv {

struct CommitSmem {
  int32_t path[64];
  int32_t ent[2][64];  // closing path depths: CSA entries to copy, HCA entries
  int nent[2];
  int64_t raw_at[64], slot_at[2][64];  // by path depth: raw-row index, CSA / HCA pool slot
};

// The part of a row's commit that one layer's cache decides: destinations
// (flat: ring slot, base + index below the capacity; paged: through the page
// table), all resolved before any write, then the copies and the new length.
// The accepted path (a nodes, path[] in LDS by depth) and the designated
// chain are the row's.  Returns TV_ROW_OK, or TV_ROW_CAPACITY (written to
// row_status[b]) when a destination is missing.  Uniform over the workgroup;
// ends with the entry lists and slots read out.
__device__ __forceinline__ int32_t commit_layer(const tv_dims &d, const tv_cache &c,
                                                const uint16_t *__restrict__ tree_u,
                                                const uint16_t *__restrict__ scr_c4,
                                                const uint16_t *__restrict__ scr_c128,
                                                int32_t *__restrict__ row_status, int b, int32_t L, int a,
                                                uint64_t chain, int32_t cap4, int32_t cap128, int64_t base4,
                                                int64_t base128, CommitSmem &sm) {
  int32_t *path = sm.path;
  int32_t(*ent)[64] = sm.ent;
  int *nent = sm.nent;
  int64_t *raw_at = sm.raw_at;
  int64_t(*slot_at)[64] = sm.slot_at;
  const int tid = threadIdx.x;
  const int64_t rb = (int64_t)b * d.D;
  const bool flat = d.page_size == 0;
  if (tid < 2) nent[tid] = 0;
  bool bad = false;
  if (tid < a) {
    const int64_t p = (int64_t)L + tid;  // path node at depth tid stands at L + tid
    const int64_t ri = raw_index(d, c.page_table, b, p);
    raw_at[tid] = ri;
    bad |= ri < 0;
    if ((p + 1) % d.ratio_csa == 0) {
      const int64_t s4 = (p + 1) / d.ratio_csa - 1;
      const int64_t sl = flat ? (s4 < cap4 ? base4 + s4 : -1)
                              : pool_slot(d, c.page_table, nullptr, nullptr, b, s4, d.ratio_csa);
      slot_at[0][tid] = sl;
      bad |= sl < 0;
    }
    if ((p + 1) % d.ratio_hca == 0) {
      const int64_t s128 = (p + 1) / d.ratio_hca - 1;
      const int64_t sl = flat ? (s128 < cap128 ? base128 + s128 : -1)
                              : pool_slot(d, c.page_table, nullptr, nullptr, b, s128, d.ratio_hca);
      slot_at[1][tid] = sl;
      bad |= sl < 0;
    }
  }
  if (__syncthreads_or(bad)) {
    if (tid == 0) row_status[b] = TV_ROW_CAPACITY;
    return TV_ROW_CAPACITY;
  }
  // the closing path depths, in depth order (wave 0: ballots over lanes t < a)
  if (tid < 64) {
    const int64_t p = (int64_t)L + tid;
    const bool c4 = tid < a && (p + 1) % d.ratio_csa == 0 && !((chain >> path[tid < a ? tid : 0]) & 1ull);
    const bool c128 = tid < a && (p + 1) % d.ratio_hca == 0;
    const uint64_t b4 = __ballot(c4), b128 = __ballot(c128);
    const uint64_t below = (1ull << tid) - 1ull;  // lanes below this one
    if (c4) ent[0][__popcll(b4 & below)] = tid;
    if (c128) ent[1][__popcll(b128 & below)] = tid;
    if (tid == 0) {
      nent[0] = __popcll(b4);
      nent[1] = __popcll(b128);
    }
  }
  __syncthreads();
  // Copies as one list of 16-byte chunks: raw rows of the path into the ring,
  // CSA entries (latent row, then indexer key) and HCA entries into their
  // pool slots.  A thread's loads all go out before its stores.
  const int d_u = d.d_row + d.d_idx;
  const int cpr = d_u / 8, c4c = d_u / 8, c128c = d.d_row / 8;
  const int n_ring = a * cpr, n4 = nent[0] * c4c, n128 = nent[1] * c128c;
  const int total = n_ring + n4 + n128;
  constexpr int kBatch = 4;
  for (int e0 = 0; e0 < total; e0 += kBatch * (int)blockDim.x) {
    uint4 v[kBatch];
    uint16_t *dst[kBatch];
    uint8_t *dst8[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int e = e0 + u * (int)blockDim.x + tid;
      dst[u] = nullptr;
      dst8[u] = nullptr;
      v[u] = make_uint4(0, 0, 0, 0);
      if (e < n_ring) {
        const int t = e / cpr, cc = (e - t * cpr) * 8;
        v[u] = *reinterpret_cast<const uint4 *>(tree_u + (rb + path[t]) * d_u + cc);
        dst[u] = c.ring + raw_at[t] * d_u + cc;
      } else if (e < n_ring + n4) {
        const int x = e - n_ring, k = x / c4c, ch = (x - k * c4c) * 8;
        const int t = ent[0][k];
        const int64_t slot = slot_at[0][t];
        v[u] = *reinterpret_cast<const uint4 *>(scr_c4 + (rb + path[t]) * d_u + ch);
        dst[u] = ch < d.d_row ? c.c4 + slot * d.d_row + ch : c.c4_idx + slot * d.d_idx + (ch - d.d_row);
        if (ch >= d.d_row && d.idx_fmt == TV_IDX_E4M3) {  // eight E4M3 codes: 8 bytes at byte offset slot*d_idx + ...
          dst8[u] = reinterpret_cast<uint8_t *>(c.c4_idx) + slot * d.d_idx + (ch - d.d_row);
          dst[u] = nullptr;
        }
      } else if (e < total) {
        const int x = e - n_ring - n4, k = x / c128c, ch = (x - k * c128c) * 8;
        const int t = ent[1][k];
        const int64_t slot = slot_at[1][t];
        v[u] = *reinterpret_cast<const uint4 *>(scr_c128 + (rb + path[t]) * d.d_row + ch);
        dst[u] = c.c128 + slot * d.d_row + ch;
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (dst[u]) *reinterpret_cast<uint4 *>(dst[u]) = v[u];
      if (dst8[u]) {  // the scratch holds E4M3 values in bfloat16: narrow them exactly
        uint2 w;
        w.x = bf16_to_e4m3(v[u].x & 0xFFFF) | (bf16_to_e4m3(v[u].x >> 16) << 8) |
              (bf16_to_e4m3(v[u].y & 0xFFFF) << 16) | (bf16_to_e4m3(v[u].y >> 16) << 24);
        w.y = bf16_to_e4m3(v[u].z & 0xFFFF) | (bf16_to_e4m3(v[u].z >> 16) << 8) |
              (bf16_to_e4m3(v[u].w & 0xFFFF) << 16) | (bf16_to_e4m3(v[u].w >> 16) << 24);
        *reinterpret_cast<uint2 *>(dst8[u]) = w;
      }
    }
  }
  if (tid == 0) c.len[b] = L + a;
  __syncthreads();  // the entry lists and slots are read out
  return TV_ROW_OK;
}

// The commit of row b of one layer's cache, by the whole workgroup.  `status`
// is the row's status before it (TV_ROW_OK to commit); returns the row's status
// after it, having written row_status[b] where it changed.  Uniform over the
// workgroup; ends with the workgroup's LDS free for the next call.
__device__ __forceinline__ int32_t commit_row(const tv_dims &d, const tv_cache &c, const uint16_t *__restrict__ tree_u,
                                              const uint64_t *__restrict__ anc, const int32_t *__restrict__ depth,
                                              const uint16_t *__restrict__ scr_c4,
                                              const uint16_t *__restrict__ scr_c128,
                                              const int32_t *__restrict__ accepted_last,
                                              int32_t *__restrict__ accept_nodes, int32_t *__restrict__ accept_len,
                                              int32_t *__restrict__ row_status,
                                              const int32_t *__restrict__ primary_last, int b, int32_t status,
                                              CommitSmem &sm) {
  const int tid = threadIdx.x;
  const int64_t rb = (int64_t)b * d.D;
  // every independent load first, one wait for all of them
  const int32_t L = c.len[b];
  const int32_t last = accepted_last[b];
  const int32_t P = primary_last ? primary_last[b] : -1;
  const int32_t dt = tid < d.D ? depth[rb + tid] : 0;
  const bool flat = d.page_size == 0;
  const int32_t cap4 = flat ? c.c4_cap[b] : 0, cap128 = flat ? c.c128_cap[b] : 0;
  const int64_t base4 = flat ? c.c4_base[b] : 0, base128 = flat ? c.c128_base[b] : 0;
  if (status != TV_ROW_OK) return status;
  if (!len_ok(L, d.max_len)) {
    if (tid == 0) row_status[b] = TV_ROW_BAD_LEN;
    return TV_ROW_BAD_LEN;
  }
  if (last < 0 || last >= d.D) {
    if (tid == 0) row_status[b] = TV_ROW_BAD_ACCEPT;
    return TV_ROW_BAD_ACCEPT;
  }
  const uint64_t m = anc[rb + last];
  const uint64_t chain = (P >= 0 && P < d.D) ? anc[rb + P] : 0ull;
  const int a = depth[rb + last] + 1;
  if (tid < d.D && ((m >> tid) & 1ull)) sm.path[dt] = tid;
  const int32_t st = commit_layer(d, c, tree_u, scr_c4, scr_c128, row_status, b, L, a, chain, cap4, cap128, base4,
                                  base128, sm);
  if (st != TV_ROW_OK) return st;
  if (tid < d.D) accept_nodes[rb + tid] = tid < a ? sm.path[tid] : -1;
  if (tid == 0) accept_len[b] = a;
  __syncthreads();  // the path is read out
  return TV_ROW_OK;
}

__global__ void __launch_bounds__(256) commit_kernel(tv_dims d, tv_cache c, const uint16_t *__restrict__ tree_u,
                                                     const uint64_t *__restrict__ anc,
                                                     const int32_t *__restrict__ depth,
                                                     const uint16_t *__restrict__ scr_c4,
                                                     const uint16_t *__restrict__ scr_c128,
                                                     const int32_t *__restrict__ accepted_last,
                                                     int32_t *__restrict__ accept_nodes,
                                                     int32_t *__restrict__ accept_len,
                                                     int32_t *__restrict__ row_status,
                                                     const int32_t *__restrict__ primary_last) {
  __shared__ CommitSmem sm;
  const int b = blockIdx.x;
  const int32_t status = row_status[b];
  (void)commit_row(d, c, tree_u, anc, depth, scr_c4, scr_c128, accepted_last, accept_nodes, accept_len, row_status,
                   primary_last, b, status, sm);
}

// The commits of several layers that share a tree, one workgroup per row: one
// launch replaces a launch per layer (the graph round's commits).  The
// accepted path is the row's and is resolved once.  As with one call per layer
// in order, a row stops at the first layer that fails it: the layers before it
// are committed, it and the later ones are left as they were.
//
// What bounds it: dependent round trips and barriers (a row's copies are tens
// of kilobytes a layer).  The layers therefore share out the workgroup's
// sixteen wavefronts instead of following each other: every team of
// wavefronts checks and resolves its own layers, one barrier publishes the
// verdicts, and each team copies its layers with no further barrier.  Sixteen
// rows of six layers took 25.7 us layer after layer and take 8.9.
constexpr int kCommitNW = 16;

struct CommitLayersSmem {
  int32_t verdict[kCommitMaxLayers];
  int32_t path[64];
  // per wavefront, the tables of the layer it copies: by path depth (raw-row
  // index), and by entry (pool slot and path node of CSA, HCA entries)
  int64_t raw_at[kCommitNW][64], slot_at[2][kCommitNW][64];
  int32_t ent[2][kCommitNW][64];
};
static_assert(kCommitMaxLayers <= 2 * kCommitNW, "a team takes at most two layers");

__global__ void __launch_bounds__(kCommitNW * 64) commit_layers_kernel(
    tv_dims d, CommitLayers ls, const uint64_t *__restrict__ anc, const int32_t *__restrict__ depth,
    const int32_t *__restrict__ accepted_last, int32_t *__restrict__ accept_nodes, int32_t *__restrict__ accept_len,
    int32_t *__restrict__ row_status, const int32_t *__restrict__ primary_last) {
  __shared__ CommitLayersSmem sm;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t rb = (int64_t)b * d.D;
  const bool flat = d.page_size == 0;
  // Teams of `waves` wavefronts, a layer each while there are enough; team t
  // takes layers t and t + teams.
  const int waves = std::max(1, kCommitNW / ls.n);
  const int teams = std::min(ls.n, kCommitNW);
  const int team = wv / waves;
  const bool active = team < teams;
  const int32_t status = row_status[b];
  const int32_t last = accepted_last[b];
  const int32_t P = primary_last ? primary_last[b] : -1;
  const int32_t dl = lane < d.D ? depth[rb + lane] : 0;
  struct Layer {  // lane t: the destinations of the path node at depth t
    int32_t L;
    int32_t cap4, cap128;
    int64_t base4, base128;
    int64_t raw, s4, s128;
  } st[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int l = team + u * teams;
    if (active && l < ls.n) {
      const tv_cache &c = ls.l[l].cache;
      st[u].L = c.len[b];
      st[u].cap4 = flat ? c.c4_cap[b] : 0;
      st[u].cap128 = flat ? c.c128_cap[b] : 0;
      st[u].base4 = flat ? c.c4_base[b] : 0;
      st[u].base128 = flat ? c.c128_base[b] : 0;
    }
  }
  if (status != TV_ROW_OK) return;
  const bool last_ok = last >= 0 && last < d.D;
  const uint64_t m = last_ok ? anc[rb + last] : 0ull;
  const uint64_t chain = (P >= 0 && P < d.D) ? anc[rb + P] : 0ull;
  const int a = last_ok ? depth[rb + last] + 1 : 0;
  if (wv == 0 && lane < d.D && ((m >> lane) & 1ull)) sm.path[dl] = lane;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int l = team + u * teams;
    if (!active || l >= ls.n) continue;
    const tv_cache &c = ls.l[l].cache;
    Layer &x = st[u];
    x.raw = x.s4 = x.s128 = -1;
    int32_t v = !len_ok(x.L, d.max_len) ? TV_ROW_BAD_LEN : !last_ok ? TV_ROW_BAD_ACCEPT : TV_ROW_OK;
    if (v == TV_ROW_OK) {
      bool bad = false;
      if (lane < a) {
        const int64_t p = (int64_t)x.L + lane;  // path node at depth `lane` stands at L + lane
        x.raw = raw_index(d, c.page_table, b, p);
        bad |= x.raw < 0;
        if ((p + 1) % d.ratio_csa == 0) {
          const int64_t e = (p + 1) / d.ratio_csa - 1;
          x.s4 = flat ? (e < x.cap4 ? x.base4 + e : -1)
                      : pool_slot(d, c.page_table, nullptr, nullptr, b, e, d.ratio_csa);
          bad |= x.s4 < 0;
        }
        if ((p + 1) % d.ratio_hca == 0) {
          const int64_t e = (p + 1) / d.ratio_hca - 1;
          x.s128 = flat ? (e < x.cap128 ? x.base128 + e : -1)
                        : pool_slot(d, c.page_table, nullptr, nullptr, b, e, d.ratio_hca);
          bad |= x.s128 < 0;
        }
      }
      if (__any(bad)) v = TV_ROW_CAPACITY;
    }
    if (lane == 0 && wv == team * waves) sm.verdict[l] = v;
  }
  __syncthreads();  // verdicts and path are visible, and every layer's length is read
  const int32_t vl = lane < ls.n ? sm.verdict[lane] : TV_ROW_OK;
  const uint64_t failed = __ballot(vl != TV_ROW_OK);
  const int n_ok = failed ? __ffsll((unsigned long long)failed) - 1 : ls.n;
  if (failed && tid == 0) row_status[b] = sm.verdict[n_ok];
  if (n_ok > 0 && wv == 0) {  // every layer's commit writes the same path
    if (lane < d.D) accept_nodes[rb + lane] = lane < a ? sm.path[lane] : -1;
    if (lane == 0) accept_len[b] = a;
  }
  // Copies of a layer as one list of 16-byte chunks: raw rows of the path into
  // the ring, CSA entries (latent row, then indexer key) and HCA entries into
  // their pool slots.  A lane's loads all go out before its stores.
  const int d_u = d.d_row + d.d_idx;
  const int cpr = d_u / 8, c128c = d.d_row / 8;
  int64_t *raw_at = sm.raw_at[wv];
  int64_t *slot4 = sm.slot_at[0][wv], *slot128 = sm.slot_at[1][wv];
  int32_t *node4 = sm.ent[0][wv], *node128 = sm.ent[1][wv];
  const int my_node = lane < a ? sm.path[lane] : 0;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int l = team + u * teams;
    if (!active || l >= n_ok) continue;
    const CommitLayer &cl = ls.l[l];
    const tv_cache &c = cl.cache;
    const Layer &x = st[u];
    const bool e4 = x.s4 >= 0 && !((chain >> my_node) & 1ull), e128 = x.s128 >= 0;
    const uint64_t b4 = __ballot(e4), b128 = __ballot(e128);
    const uint64_t below = (1ull << lane) - 1ull;
    // this wavefront's own tables: its LDS operations stay in order
    raw_at[lane] = x.raw;
    if (e4) {
      slot4[__popcll(b4 & below)] = x.s4;
      node4[__popcll(b4 & below)] = my_node;
    }
    if (e128) {
      slot128[__popcll(b128 & below)] = x.s128;
      node128[__popcll(b128 & below)] = my_node;
    }
    __builtin_amdgcn_wave_barrier();
    const int n_ring = a * cpr, n4 = __popcll(b4) * cpr, total = n_ring + n4 + __popcll(b128) * c128c;
    constexpr int kBatch = 8;
    for (int e0 = (wv - team * waves) * 64; e0 < total; e0 += kBatch * 64 * waves) {
      uint4 v[kBatch];
      uint16_t *dst[kBatch];
      uint32_t narrow = 0u;  // chunks stored as E4M3 codes: 8 bytes
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int e = e0 + k * 64 * waves + lane;
        dst[k] = nullptr;
        v[k] = make_uint4(0, 0, 0, 0);
        if (e < n_ring) {
          const int t = e / cpr, ch = (e - t * cpr) * 8;
          v[k] = *reinterpret_cast<const uint4 *>(cl.tree_u + (rb + sm.path[t]) * d_u + ch);
          dst[k] = c.ring + raw_at[t] * d_u + ch;
        } else if (e < n_ring + n4) {
          const int y = e - n_ring, t = y / cpr, ch = (y - t * cpr) * 8;
          const int64_t slot = slot4[t];
          v[k] = *reinterpret_cast<const uint4 *>(cl.scr_c4 + (rb + node4[t]) * d_u + ch);
          if (ch < d.d_row) {
            dst[k] = c.c4 + slot * d.d_row + ch;
          } else if (d.idx_fmt == TV_IDX_E4M3) {
            dst[k] = reinterpret_cast<uint16_t *>(reinterpret_cast<uint8_t *>(c.c4_idx) + slot * d.d_idx +
                                                  (ch - d.d_row));
            narrow |= 1u << k;
          } else {
            dst[k] = c.c4_idx + slot * d.d_idx + (ch - d.d_row);
          }
        } else if (e < total) {
          const int y = e - n_ring - n4, t = y / c128c, ch = (y - t * c128c) * 8;
          v[k] = *reinterpret_cast<const uint4 *>(cl.scr_c128 + (rb + node128[t]) * d.d_row + ch);
          dst[k] = c.c128 + slot128[t] * d.d_row + ch;
        }
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        if (!dst[k]) continue;
        if ((narrow >> k) & 1u) {  // the scratch holds E4M3 values in bfloat16: narrow them exactly
          uint2 w;
          w.x = bf16_to_e4m3(v[k].x & 0xFFFF) | (bf16_to_e4m3(v[k].x >> 16) << 8) |
                (bf16_to_e4m3(v[k].y & 0xFFFF) << 16) | (bf16_to_e4m3(v[k].y >> 16) << 24);
          w.y = bf16_to_e4m3(v[k].z & 0xFFFF) | (bf16_to_e4m3(v[k].z >> 16) << 8) |
                (bf16_to_e4m3(v[k].w & 0xFFFF) << 16) | (bf16_to_e4m3(v[k].w >> 16) << 24);
          *reinterpret_cast<uint2 *>(dst[k]) = w;
        } else {
          *reinterpret_cast<uint4 *>(dst[k]) = v[k];
        }
      }
    }
    if (lane == 0 && wv == team * waves) c.len[b] = x.L + a;
    __builtin_amdgcn_wave_barrier();  // the tables are read out
  }
}

hipError_t launch_commit_layers(const tv_dims &d, const CommitLayers &ls, const uint64_t *anc, const int32_t *depth,
                                const int32_t *accepted_last, int32_t *accept_nodes, int32_t *accept_len,
                                int32_t *row_status, const int32_t *primary_last, hipStream_t s) {
  if (ls.n < 1 || ls.n > kCommitMaxLayers) return hipErrorInvalidValue;
  commit_layers_kernel<<<d.B, kCommitNW * 64, 0, s>>>(d, ls, anc, depth, accepted_last, accept_nodes, accept_len, row_status,
                                           primary_last);
  return hipGetLastError();
}

hipError_t launch_commit(const tv_dims &d, const tv_cache &c, const uint16_t *tree_u, const uint64_t *anc,
                         const int32_t *depth, const uint16_t *scr_c4, const uint16_t *scr_c128,
                         const int32_t *accepted_last, int32_t *accept_nodes, int32_t *accept_len,
                         int32_t *row_status, const int32_t *primary_last, hipStream_t s) {
  commit_kernel<<<d.B, 256, 0, s>>>(d, c, tree_u, anc, depth, scr_c4, scr_c128, accepted_last, accept_nodes,
                                    accept_len, row_status, primary_last);
  return hipGetLastError();
}

}  // namespace tv
