// Host-side launchers of the library's HIP kernels.  All take a stream and
// enqueue only; none allocates or synchronises.
#pragma once

#include <cstddef>

#include "og_internal.h"

namespace og {

// Tile of the scans (node ranks, active targets); scan_partial_words(n) tile
// sums each.
constexpr uint32_t kScanTile = 4096;

// LSD radix sort of (key, val) pairs, 8-bit digits.  Key passes
// [pass_lo, pass_hi) on the 64-bit key, then `box_passes` passes on the box
// of each value (global particle index).  Ping-pongs between a and b;
// returns true when the result ends in b.  `tile`: keys per workgroup, kSortTile
// or a quarter of it; `hist` holds radix_hist_words(n, tile) words.
constexpr uint32_t kSortTile = 4096;
bool radix_sort(uint64_t *keys_a, uint32_t *vals_a, uint64_t *keys_b, uint32_t *vals_b,
                uint32_t n, int pass_lo, int pass_hi, int box_passes, const BoxDev *boxes,
                int B, uint32_t *hist, uint32_t *digit_tot, hipStream_t s, uint32_t tile = kSortTile);
size_t radix_hist_words(uint32_t n, uint32_t tile = kSortTile);

// Tile of the merge sort that small boxes and target lists take.
constexpr uint32_t kMergeTile = 1024;

struct BuildArrays {
  BoxDev *boxes;
  int B;
  uint32_t n;                 // total particles
  uint32_t node_cap;          // node capacity
  uint32_t max_n, n_tiles;    // particles of the largest box; sort tiles of all boxes (kMergeTile each)
  uint64_t *minmax;           // [B][6] ordered-bits min/max for open boxes
  uint64_t *keys_a, *keys_b;
  uint32_t *vals_a, *vals_b;
  uint32_t *hist, *digit_tot;
  uint32_t *perm, *inv;
  double4 *part64;
  float4 *part32;
  int8_t *lcp;
  uint8_t *depth;
  uint32_t *nstart, *S, *scan_partial;
  Topo *topo;
  Mom64 *mom64;
  WNode *wnode;
  double4 *cen64;  // per node: FP64 cube centre (x, y, z) and side (w), for the FP64 walks
  uint32_t *first, *skip, *parent;
  uint32_t *kid, *sib;        // per node: its child slots (k_links); the slots (one array of 2 node_cap)
  uint32_t *top_cnt;          // [0] top nodes [1] child slots taken [2] deepest top level
  uint32_t *top_buf;          // TopArrays' lists, kTopWords per top node (top_cap)
  uint32_t *top_id;           // per node: index of a top node in the top list
  uint32_t top_cap;           // bound on the top nodes (top_node_bound)
  uint32_t *scalars;          // [0] status [3] n_nodes [4] n [5] deepest level (stats)
  int any_open;               // some box has periodic = 0
  int leaf_max;               // largest leaf_max of the boxes
  double *seps;               // sorted per-particle softening lengths (null: none given)
  double *semax, *semin;      // per node: largest and smallest of its particles' lengths
};

// The moment kernels sum subtrees of up to kSegNodes nodes per workgroup;
// the nodes with larger subtrees ("top" nodes) are summed by one workgroup.
// Top nodes of one level have disjoint subtrees of more than kSegNodes
// nodes each, so there are fewer than node_cap / kSegNodes + 1 per level.
constexpr uint32_t kSegNodes = 768;
inline uint32_t top_node_bound(uint32_t node_cap) { return 2 * (((kLevels + 1) * (node_cap / kSegNodes + 1) + 1) / 2); }

// The top-node list the moment kernels pass to the top-node kernel.
struct TopArrays {
  uint32_t *cnt;    // [0] top nodes [2] deepest level of a top node
  uint4 *list;      // top nodes (cap): node, level, cube corner (low, high word)
  uint64_t *slot;   // per top node: eight child slots by octant (8 cap)
  uint32_t *id;     // per node (node_cap): its class (a top node: with its index in `list`)
  uint32_t cap;
};
// Walk group queues: one per XCD (see k_walk.hip), each counter on a cache
// line of its own.  A tree's and a target list's stand in their digit_tot, which
// is free once the sort is done (and which launch_walk resets), so that they
// take no memory of their own.
constexpr uint32_t kQueues = 8, kQueueStride = 32;
constexpr uint32_t kQueueWords = kQueues * kQueueStride;
static_assert(kQueueWords <= 256, "the counters fit digit_tot");

constexpr size_t kTopWords = 20;  // words of top_buf per top node

void launch_build(BuildArrays &A, hipStream_t s);
void launch_max_level(const BuildArrays &A, uint32_t *out, hipStream_t s);

// Targets given as caller-order indices (box 0 only): the target list
// sorted by tree position (so that consecutive targets are neighbours).
struct TargetArrays {
  const int64_t *idx;
  uint32_t M;
  uint64_t *tkey_a, *tkey_b;
  uint32_t *tval_a, *tval_b;
  uint32_t *hist, *digit_tot;
  uint32_t *scalars;          // [0] status
  const uint64_t *tkey;       // result (points at a or b)
  const uint32_t *tval;
};
void launch_targets(const BuildArrays &A, TargetArrays &T, hipStream_t s);

// Active targets of one tree: the particles whose time-step level bin[i]
// (caller order) is <= level, in curve order, compacted on the device.
// counts[0] = number of active targets, counts[1] = walk groups of `chunk`;
// n_active (optional) receives counts[0] as int64.
struct ActiveArrays {
  const int8_t *bin;
  int32_t level;
  uint8_t *flags;
  uint32_t *partial;
  uint64_t *tkey;
  uint32_t *tval;
  uint32_t *counts;           // [0] active, [1] groups, [32..] walk queues (kQueueWords)
  int64_t *n_active;
};
void launch_active(const BuildArrays &A, ActiveArrays &T, uint32_t chunk, hipStream_t s);
size_t scan_partial_words(uint32_t n);

struct WalkArgs {
  const BoxDev *boxes;
  const Topo *topo;
  // Smallest theta of the boxes, for the host's choice of walk.  It stands here
  // for the place of the pointers after it: with wnode at byte 16 of the
  // arguments instead of 24 the screened FP64 walk is 1.1 to 2 % slower (2M
  // particles 13.01 | 12.85 ms, 700k 5.50 | 5.39).
  double theta;
  const WNode *wnode;
  const double4 *cen64;
  const Mom64 *mom64;
  const float4 *part32;
  const double4 *part64;
  const uint32_t *perm;
  const uint64_t *skeys;      // sorted Morton keys
  const uint32_t *kid, *sib;  // child slots of the nodes (see k_links)
  uint32_t n_groups;          // walk groups (chunks of `chunk` targets)
  uint32_t chunk;             // targets per group, <= 64
  int list_cap;               // mixed walk list entries per lane (0 = default)
  uint32_t n_targets;         // targets: length of the list (tkey != null; a bound with dev_count), or all particles
  int B;                      // boxes
  int box_kind;               // shared by all boxes: 1 cutoff+open, 2 cutoff+periodic,
                              // 3 Newtonian+open; 0 mixed
  uint32_t *counter;          // kQueues group counters, kQueueStride words apart
  const uint64_t *tkey;       // sorted target positions, or null: all particles
  const uint32_t *tval;       // target slots
  double *acc;                // non-null: outputs by slot; null: per-box acc/pot
  double *pot;
  int64_t *nint;
  int pot_override;           // 1: use `pot` (possibly null) instead of the box's
  int ext;                    // some box uses spline softening or the relative criterion
  const uint32_t *dev_count;  // non-null: n_targets = [0], n_groups = [1], read on the device
  const double *seps, *semax, *semin;  // per-particle softening (null: the boxes' eps)
  int group_lists;            // 1: group-shared interaction lists, 0: per-target walk
  const double *a_old;        // relative criterion: previous accelerations [n][3], caller order
  uint32_t n_particles;       // particles of the forest
  uint32_t small_max;         // walks of up to this many targets are eight-lane walks (set by launch_walk)
  int few;                    // 1: every array within 4 GiB, so the eight-lane walk may run
  int leaf_max, relative;     // smallest leaf_max of the boxes; a box with the relative criterion
  double alpha;               // smallest of the boxes (relative criterion)
  int negative;               // some box's G carries a minus sign
  int wide_nodes;             // the node records span more than 4 GiB (64-bit record offsets)
  int no_interior;            // mixed walk: reduce every periodic offset (no raw form for interior groups)
  int erfc_tail;              // FP64 walks: some box has r_cut / (2 r_s) >= 3 (library erfc past the polynomial)
};
static_assert(offsetof(WalkArgs, wnode) == 24, "the place of the walks' pointers (see theta)");
void launch_walk(const WalkArgs &W, int precision, hipStream_t s);
void launch_reset(uint32_t *word, hipStream_t s);
void launch_reset_queues(uint32_t *counter, hipStream_t s);

int device_cu_count();

}  // namespace og
