// Host-side work lists of the attention kernels.
//
// One item = one workgroup: a (segment, tile, head) triple.  In the forward and dQ passes the
// workgroups that read the same K / V rows (the query tiles and the query heads of one (segment, kv
// head)) are put on the SAME XCD, next to one another in time, so that the rows they share are
// fetched into that XCD's L2 once and not once per workgroup: left to the default order they spread
// over all eight XCDs and over time and every workgroup streams its rows from the memory side (measured
// on 16 samples of 2048 tokens, 32 / 8 heads of 128: 4.5 GB fetched per forward launch against 0.4 GB of
// q, k, v; with this order 0.41 GB and the kernel 5-12 % faster).
//
// The hardware deals workgroups to the XCDs round-robin by linear id, so workgroup `pid` runs on
// XCD pid % 8 as that XCD's workgroup number pid / 8.  The list is the eight XCDs' sub-lists
// interleaved: entry pid is item pid / 8 of XCD pid % 8, so a workgroup finds its item with one
// load; sub-lists shorter than the longest end in empty items (seg_len = 0: the workgroup exits).
// The grid is 8 * the longest sub-list.
//
// Groups of items that belong together are formed per (segment, kv head) and cut into runs of
// consecutive tiles of about one XCD's resident workgroups; the groups go to the XCDs heaviest
// first, each to the least loaded XCD (the LPT rule of the paper's Online Microbatch Scheduler
// applied to tiles), and every XCD works through its groups heaviest first.  The dK/dV pass keeps
// one global heaviest-first list (see below).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "../../include/mllm_stage.h"
#include "kernels.h"

namespace mllm {

constexpr int ATTN_XCDS = 8;

inline int64_t attn_count_tiles(const mllm_pack_t& p, int tile) {
  int64_t n = 0;
  for (int s = 0; s < p.n_segments; s++) n += (p.cu_seqlens_host[s + 1] - p.cu_seqlens_host[s] + tile - 1) / tile;
  return n;
}
// Upper bound of the bytes of a list over `heads` heads (query heads for the forward / dQ list, kv
// heads for dK/dV): no sub-list is longer than all items together.
inline size_t attn_list_bytes(const mllm_pack_t& p, int tile, int heads) {
  return (size_t)ATTN_XCDS * (size_t)attn_count_tiles(p, tile) * (size_t)heads * sizeof(AttnItem);
}

// Parts of the dK/dV pass over this token space (attn_kv_parts).
inline int attn_kv_parts_of(const mllm_pack_t& p, int n_kv_heads, int heads_per_kv, int head_dim) {
  int64_t heaviest = 0, total = 0;
  for (int s = 0; s < p.n_segments; s++) {
    const int len = p.cu_seqlens_host[s + 1] - p.cu_seqlens_host[s];
    for (int t0 = 0; t0 < len; t0 += ATTN_BWD_KV_TILE) {
      const int64_t its = (int64_t)heads_per_kv * (((p.mask_kind_host[s] == MLLM_MASK_CAUSAL ? len - t0 : len) + 63) / 64);
      heaviest = std::max(heaviest, its);
      total += its * n_kv_heads;
    }
  }
  return attn_kv_parts(heaviest, total, (int64_t)p.total_tokens * n_kv_heads, head_dim);
}

// Writes the list to dst (at most attn_list_bytes(...) bytes, grid * sizeof(AttnItem) of them used) and
// returns the grid size, 8 * the longest sub-list.
//   kv_major: items are key tiles (dK/dV pass) and `head` is the kv head; otherwise items are query
//   tiles and `head` runs over the heads_per_kv query heads of every kv head.
inline int build_attn_list(const mllm_pack_t& p, int tile, bool kv_major, int n_kv_heads, int heads_per_kv,
                           int resident_per_xcd, char* dst) {
  if (kv_major) {
    // dK/dV pass: one list for the whole chip, heaviest key tile first, the kv heads of a tile next to one
    // another (with eight kv heads each lands on an XCD of its own).  Its workgroups differ a lot in
    // length (the first key tile of a causal sample meets every query tile, the last one a single one),
    // so the fine-grained heaviest-first order matters more here than keeping a sample on one XCD:
    // measured 6 % faster than the grouped order on 16 samples of 2048 tokens, equal on the seeded mixes.
    struct It { int start, len, t0, causal; int64_t work; };
    std::vector<It> its;
    for (int s = 0; s < p.n_segments; s++) {
      const int start = p.cu_seqlens_host[s], len = p.cu_seqlens_host[s + 1] - start;
      const int causal = p.mask_kind_host[s] == MLLM_MASK_CAUSAL;
      for (int t0 = 0; t0 < len; t0 += tile) its.push_back({start, len, t0, causal, causal ? len - t0 : len});
    }
    std::stable_sort(its.begin(), its.end(), [](const It& a, const It& b) { return a.work > b.work; });
    AttnItem* items = reinterpret_cast<AttnItem*>(dst);
    int64_t n = 0;
    for (const It& it : its)
      for (int hh = 0; hh < n_kv_heads; hh++) items[n++] = {it.start, it.len, it.t0, it.causal, hh};
    return (int)n;
  }
  struct Group { int seg, kvh, first, count; int64_t work; };
  const int hpg = heads_per_kv;
  auto tile_work = [&](int len, bool causal, int t0) -> int64_t {
    if (!causal) return len;
    return kv_major ? len - t0 : std::min(len, t0 + tile);
  };
  // position k of a segment's tiles in heaviest-first order -> first row of the tile
  auto tile0_of = [&](int ntiles, bool causal, int k) { return (causal && !kv_major ? ntiles - 1 - k : k) * tile; };
  int64_t total_tiles = attn_count_tiles(p, tile);
  int chunk = std::max(1, resident_per_xcd / hpg);
  auto count_groups = [&](int c) {
    int64_t n = 0;
    for (int s = 0; s < p.n_segments; s++) {
      const int nt = (p.cu_seqlens_host[s + 1] - p.cu_seqlens_host[s] + tile - 1) / tile;
      n += (int64_t)((nt + c - 1) / c) * n_kv_heads;
    }
    return n;
  };
  while (chunk > 1 && count_groups(chunk) < 4 * ATTN_XCDS) chunk = (chunk + 1) / 2;   // small problems: still use every XCD
  std::vector<Group> groups;
  for (int s = 0; s < p.n_segments; s++) {
    const int len = p.cu_seqlens_host[s + 1] - p.cu_seqlens_host[s];
    const bool causal = p.mask_kind_host[s] == MLLM_MASK_CAUSAL;
    const int nt = (len + tile - 1) / tile;
    for (int first = 0; first < nt; first += chunk) {
      const int count = std::min(chunk, nt - first);
      int64_t w = 0;
      for (int k = first; k < first + count; k++) w += tile_work(len, causal, tile0_of(nt, causal, k));
      for (int g = 0; g < n_kv_heads; g++) groups.push_back({s, g, first, count, w * hpg});
    }
  }
  std::stable_sort(groups.begin(), groups.end(), [](const Group& a, const Group& b) { return a.work > b.work; });
  std::vector<int> per_xcd[ATTN_XCDS];
  int64_t load[ATTN_XCDS] = {0};
  int64_t n_items[ATTN_XCDS] = {0};
  for (size_t gi = 0; gi < groups.size(); gi++) {
    int best = 0;
    for (int x = 1; x < ATTN_XCDS; x++)
      if (load[x] < load[best]) best = x;
    per_xcd[best].push_back((int)gi);
    load[best] += groups[gi].work;
    n_items[best] += (int64_t)groups[gi].count * hpg;
  }
  int64_t longest = 0;
  for (int x = 0; x < ATTN_XCDS; x++) longest = std::max(longest, n_items[x]);
  AttnItem* items = reinterpret_cast<AttnItem*>(dst);
  memset(dst, 0, (size_t)(ATTN_XCDS * longest) * sizeof(AttnItem));
  for (int x = 0; x < ATTN_XCDS; x++) {
    int64_t local = 0;
    for (int gi : per_xcd[x]) {
      const Group& G = groups[gi];
      const int start = p.cu_seqlens_host[G.seg], len = p.cu_seqlens_host[G.seg + 1] - start;
      const bool causal = p.mask_kind_host[G.seg] == MLLM_MASK_CAUSAL;
      const int nt = (len + tile - 1) / tile;
      for (int k = G.first; k < G.first + G.count; k++)
        for (int j = 0; j < hpg; j++)
          items[(local++) * ATTN_XCDS + x] = {start, len, tile0_of(nt, causal, k), causal ? 1 : 0, G.kvh * hpg + j};
    }
  }
  (void)total_tiles;
  return (int)(ATTN_XCDS * longest);
}

}  // namespace mllm
