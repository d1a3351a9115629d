// What the extend planner decides for one sequence and one work item, as plain
// functions of the arguments: plan_extend_kernel calls them from the threads
// of one workgroup, plan_extend_on_host (a check of the sizing and of the list)
// in order.
#pragma once

#include "kernels.hpp"

namespace rl {

constexpr int kSortMax = 1024;          // sequences sorted by key count up to this batch size
constexpr int kXcds = 8;                // workgroups go to the 8 XCDs round-robin by index
constexpr bool kXcdGroups = true;       // keep each (sequence, KV head)'s units on one XCD

struct SeqRange {
  int q0, n, kv;
};

// Chunk rows and keys of sequence b, clamped into the call's buffers (*bad records it).
inline __host__ __device__ SeqRange seq_range(const ExtendArgs& a, int b, int* bad) {
  const int max_tokens = a.kv.max_pages * a.kv.page_size;
  if (a.decode_rows) {
    // decode: sequence b owns rows b * n .. b * n + n - 1, its last n keys
    const int n = a.decode_rows;
    int kv = a.kv_lens[(int64_t)b * a.kv_lens_s];
    if (kv < 0 || kv > max_tokens) {
      *bad |= kErrLen;
      kv = kv < 0 ? 0 : max_tokens;
    }
    if (kv == 0) return {b * n, 0, 0};
    if (kv < n) {
      *bad |= kErrKvShort;
      kv = n <= max_tokens ? n : max_tokens;
    }
    return {b * n, n, kv};
  }
  int q0 = a.qo_indptr[(int64_t)b * a.indptr_s];
  int q1 = a.qo_indptr[(int64_t)(b + 1) * a.indptr_s];
  if (q0 < 0 || q0 > a.total_q || q1 < q0 || q1 > a.total_q) {
    *bad |= kErrIndptr;
    q0 = q0 < 0 ? 0 : (q0 > a.total_q ? a.total_q : q0);
    q1 = q1 < q0 ? q0 : (q1 > a.total_q ? a.total_q : q1);
  }
  int n = q1 - q0;
  int kv = a.kv_lens[(int64_t)b * a.kv_lens_s];
  if (kv < 0 || kv > max_tokens) {
    *bad |= kErrLen;
    kv = kv < 0 ? 0 : max_tokens;
  }
  if (n > kv) {           // the chunk must be inside the cache
    *bad |= kErrKvShort;
    if (n > max_tokens) n = max_tokens;
    kv = n;
  }
  return {q0, n, kv};
}

inline __host__ __device__ int unit_tiles(int n, int tt) { return (int)(((int64_t)n + tt - 1) / tt); }

// Tiles of tt chunk rows (nt in all; chunk of n rows behind `prefix` keys)
// whose keys reach into segment s: all but the first tiles, which end before it.
inline __host__ __device__ int segment_tiles(int s, int prefix, int n, int nt, int tt) {
  const int t = segment_start(s);
  if (t >= prefix + n) return 0;
  return t <= prefix ? nt : nt - (t - prefix) / tt;
}
// (tile, segment) pairs of one head group of a sequence
inline __host__ __device__ long long unit_segments(const SeqRange& r, int tt) {
  const int nt = unit_tiles(r.n, tt);
  long long c = 0;
  for (int s = segment_count(r.kv) - 1; s >= 0; --s) c += segment_tiles(s, r.kv - r.n, r.n, nt, tt);
  return c;
}

// Slots that splitting sequence r takes, 0 if it is not to be split
// (max_slots + 1: more than there are). all_keys and all_units: keys and number
// of all the call's units. None is split when the units alone do not fit the
// list (chunks that overlap, an invalid qo_indptr): items fall off its end then,
// and a split unit must not be finished without all of its parts.
// Split are the sequences with a unit longer than half a workgroup's share of
// the call's keys. Below that, whole units in longest-first order fill the
// chip: six sequences of 15-24K keys, 57K a workgroup, took 1.735 ms whole and
// 1.771 ms split; one of 23.8K, 8.2K a workgroup, 527 and 314 us (segments
// from 4096).
inline __host__ __device__ int split_need(const ExtendArgs& a, const SeqRange& r, unsigned long long all_keys,
                                          unsigned long long all_units) {
  if (all_units > (unsigned long long)(a.max_items - a.max_slots)) return 0;
  if (r.n <= 0 || r.kv <= kSegKeys || (unsigned long long)r.kv * (2 * a.workers) <= all_keys) return 0;
  const long long n = (long long)a.Hkv * a.head_blocks * unit_segments(r, a.tile_tokens);
  return n > a.max_slots ? a.max_slots + 1 : (int)n;
}

// A sequence in the list: its items start at `first`, `per` for each head
// group; its slots start at `slot` (-1: its units are whole).
struct SeqPlan {
  int b, n, prefix, slot;
  int first, per;
};

// Entries of the list (a call that splits no unit has one for each).
inline __host__ __device__ int list_room(const ExtendArgs& a, bool parts) {
  return parts ? a.max_items : a.max_items - a.max_slots;
}

// Writes item i of a sequence (its part too, if the call splits any). With a multiple of 8 head groups (xcd), group gh
// of a sequence runs on XCD gh % 8: its units share their keys through that
// XCD's L2 instead of every XCD streaming every group's keys. Each XCD's units
// stay in list order (longest first), and every XCD gets the same number of units.
inline __host__ __device__ int place_item(const ExtendArgs& a, const SeqPlan& s, int i, bool xcd, bool parts) {
  const int tt = a.tile_tokens, nt = unit_tiles(s.n, tt);
  // (the tests spare a decode's items, one a head group, the divisions)
  const int gh = s.per == 1 ? i : i / s.per, u = i - gh * s.per;
  const int g = a.head_blocks == 1 ? gh : gh / a.head_blocks, hb = gh - g * a.head_blocks;
  // last tile first: it has the longest key range of the sequence; a
  // split sequence's items go segment by segment, so that the tiles
  // that read the same keys are neighbours, the last (longest) first
  int j = u, seg = -1;
  if (s.slot >= 0) {
    seg = segment_count(s.prefix + s.n) - 1;
    for (int c = segment_tiles(seg, s.prefix, s.n, nt, tt); j >= c; c = segment_tiles(seg, s.prefix, s.n, nt, tt)) {
      j -= c;
      --seg;
    }
  }
  int idx = s.first + i;
  if (xcd)   // position in the XCD's own list, behind its items of the earlier sequences and groups
    idx = (s.first / kXcds + (gh / kXcds) * s.per + u) * kXcds + gh % kXcds;
  const int i0 = (nt - 1 - j) * tt;
  const int4 unit = make_int4(s.b, i0, tt < s.n - i0 ? tt : s.n - i0, g | (hb << 16));
  // beyond the list (chunks that overlap, so only with an invalid qo_indptr; their
  // count may even pass 31 bits): reported, never dropped silently
  if ((unsigned)idx >= (unsigned)list_room(a, parts)) return kErrCapacity;
  a.ws.items[idx] = unit;
  if (parts) {
    a.ws.segs[idx] = make_int2(seg, seg < 0 ? -1 : s.slot + i);
    if (seg == 0) a.ws.arrived[s.slot + i] = 0;    // (every tile reaches into segment 0)
  }
  return 0;
}

// Slot of a split unit's segment s - 1, given that of its segment s.
inline __host__ __device__ int slot_before(int slot, int s, int prefix, int n, int tt) {
  return slot + segment_tiles(s, prefix, n, unit_tiles(n, tt), tt);
}

// The planner on host arrays (a.ws, a.qo_indptr and a.kv_lens in host memory):
// fills the list and returns the error bits. split_seqs: sequences that were split.
int plan_extend_on_host(const ExtendArgs& a, int* split_seqs);

}  // namespace rl
