// Causal extend over a paged cache: appended chunk rows attend to the cached
// prefix plus, causally, to the chunk itself (bottom-right mask).
//
// A unit of work is (sequence b, KV head g, block of query heads, run of
// chunk tokens): up to 256 query rows, token-major (row r -> token r / RB,
// head r % RB), all reading the same keys; one workgroup computes it with the
// MFMA tile of tile_attn.hpp. Keys [0, prefix + first token) are visible to
// every row of a unit, so only the last steps of a unit apply the mask.
//
// The planner orders units longest key range first and keeps the units of one
// (sequence, KV head) together on one XCD (workgroups go to the XCDs
// round-robin by index), so they run at the same time and stream the same
// keys through that XCD's L2.
//
// A row over more than kSegKeys keys is the in-order merge of one partial per
// key segment. The planner splits a sequence's units at the segments where
// whole units would leave CUs idle: then every (unit, segment) is an item that
// leaves its partial in a slot, and the workgroup that brings a unit's last one
// finishes its rows; otherwise one workgroup takes all of a unit's keys, segment
// after segment. Both give the same bits. One 333-token turn behind 23.5K keys
// (64/8 heads: 88 units for 256 CUs): 483 us a call with whole units, 355 split;
// deterministic decode of 24 sequences of 1-32K keys (192 units): 603 and 332 us.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "extend_plan.hpp"
#include "kernels.hpp"
#include "tile_attn.hpp"

namespace rl {

namespace {

__global__ __launch_bounds__(1024) void plan_extend_kernel(ExtendArgs a) {
  __shared__ int order[kSortMax];
  __shared__ int keys[kSortMax];
  __shared__ int slot_of[kSortMax];
  // of the sequences being emitted: (sequence, chunk rows, prefix, first slot or -1), (first item, items of one
  // head group)
  __shared__ int4 seq_a[1024];
  __shared__ int2 seq_b[1024];
  __shared__ unsigned long long all_keys, all_units;
  __shared__ int wave_tot[16];
  const int tid = threadIdx.x;
  int bad = 0;
  if (a.gate && *a.gate != 0) {          // the split decode passes compute the rows
    if (tid < 2) a.ws.hdr[tid] = 0;
    if (tid < kXcds) a.ws.hdr[8 + tid] = 0;
    return;
  }
  if (a.decode_rows) {
    // decode rows of empty sequences have no work unit: out = 0, lse = -inf.
    // The empty sequences of each pass of blockDim sequences are listed first
    // (one length load per thread), then their rows are written by all threads.
    __shared__ int empties[1024];
    __shared__ int n_empty;
    const int per_seq = a.decode_rows * a.Hq;
    for (int b0 = 0; b0 < a.B; b0 += blockDim.x) {
      if (tid == 0) n_empty = 0;
      __syncthreads();
      const int b = b0 + tid;
      int dummy = 0;
      if (b < a.B && seq_range(a, b, &dummy).n == 0) empties[atomicAdd(&n_empty, 1)] = b;
      __syncthreads();
      const int rows = n_empty * per_seq;
      for (int i = tid; i < rows; i += blockDim.x) {
        const int e = empties[i / per_seq], rest = i % per_seq;
        const int64_t row = (int64_t)e * a.decode_rows + rest / a.Hq;
        const int h = rest % a.Hq;
        if (a.out_f32) {
          float4* op = reinterpret_cast<float4*>((float*)a.out + row * a.out_st + (int64_t)h * a.out_sh);
          for (int c = 0; c < kHeadDim / 4; ++c) op[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
          uint4* op = reinterpret_cast<uint4*>((__bf16*)a.out + row * a.out_st + (int64_t)h * a.out_sh);
          for (int c = 0; c < kHeadDim / 8; ++c) op[c] = make_uint4(0u, 0u, 0u, 0u);
        }
        if (a.lse) a.lse[row * a.lse_st + (int64_t)h * a.lse_sh] = kNegInf;
      }
      __syncthreads();                   // the list is rebuilt for the next pass
    }
  }
  const bool sorted = a.B <= kSortMax;
  const int heads = a.Hkv * a.head_blocks, tt = a.tile_tokens;
  auto tiles = [&](int n) { return unit_tiles(n, tt); };
  // rows over several segments (then a workgroup per CU runs the list), and units split at them
  bool any_long = false, any_split = false;
  if (sorted) {
    SeqRange r{0, 0, 0};
    if (tid < a.B) {
      r = seq_range(a, tid, &bad);
      keys[tid] = r.kv;
      slot_of[tid] = -1;
    }
    any_long = __syncthreads_or(a.segmented && r.n > 0 && r.kv > kSegKeys);
    if (any_long && a.max_slots > 0) {
      if (tid == 0) all_keys = all_units = 0;
      __syncthreads();
      if (r.n > 0) {
        const unsigned long long units = (unsigned long long)tiles(r.n) * (unsigned long long)heads;
        atomicAdd(&all_units, units);
        atomicAdd(&all_keys, units * r.kv);
      }
      __syncthreads();
      const int need = tid < a.B ? split_need(a, r, all_keys, all_units) : 0;
      int tot;
      const int first = block_exclusive_scan(need, &tot, wave_tot);
      const bool split = need > 0 && first + need <= a.max_slots;
      if (split) {
        slot_of[tid] = first;
        keys[tid] = max(kSegKeys, r.kv / 2);   // about its longest item
      }
      any_split = __syncthreads_or(split);
    }
    for (int b = tid; b < a.B; b += blockDim.x) {
      const int kb = keys[b];
      int rank = 0;
      for (int j = 0; j < a.B; ++j) rank += (keys[j] > kb) || (keys[j] == kb && j < b);
      order[rank] = b;
    }
    __syncthreads();
  }
  const bool xcd = kXcdGroups && heads % kXcds == 0;
  int offset = 0;
  for (int p0 = 0; p0 < a.B; p0 += blockDim.x) {
    const int p = p0 + tid;
    int per = 0, b = 0, slot = -1;
    SeqRange r{0, 0, 0};
    if (p < a.B) {
      b = sorted ? order[p] : p;
      int dummy = 0;
      r = seq_range(a, b, sorted ? &dummy : &bad);
      slot = sorted ? slot_of[b] : -1;
      per = slot >= 0 ? (int)unit_segments(r, tt) : tiles(r.n);
    }
    if (!sorted && a.segmented) any_long |= __syncthreads_or(r.n > 0 && r.kv > kSegKeys) != 0;
    int tot;
    const int excl = block_exclusive_scan(per * heads, &tot, wave_tot);
    seq_a[tid] = make_int4(b, r.n, r.kv - r.n, slot);
    seq_b[tid] = make_int2(offset + excl, per);
    __syncthreads();
    // the items of a sequence are written by as many threads as the batch leaves
    // it (a wave each instead: draft batch of 96 x 8 units, 851 against 847 us a call)
    const int n_seq = min((int)blockDim.x, a.B - p0);
    const int lps_log = 10 - (n_seq > 1 ? 32 - __builtin_clz((unsigned)(n_seq - 1)) : 0);
    const int lps = 1 << lps_log, s = tid >> lps_log;
    if (s < n_seq) {
      const int4 sa = seq_a[s];
      const int2 sb = seq_b[s];
      const SeqPlan plan{sa.x, sa.y, sa.z, sa.w, sb.x, sb.y};
      for (int i = tid & (lps - 1); i < sb.y * heads; i += lps) bad |= place_item(a, plan, i, xcd, any_split);
    }
    offset += tot;
    if (p0 + (int)blockDim.x < a.B) __syncthreads();   // the lists are rebuilt for the next pass
  }
  if (tid == 0) a.ws.hdr[0] = min(offset, list_room(a, any_split));
  if (tid == 1) a.ws.hdr[1] = any_split ? kSplit : any_long ? kSegments : kOneSegment;
  if (tid < kXcds) a.ws.hdr[8 + tid] = (a.workers + kXcds - 1 - tid) / kXcds;
  if (bad) atomicOr(a.ws.err, bad);
}

constexpr int kExtWaves = 8;            // waves per extend workgroup: 256 query rows per unit

// Page lookups of the tile routine, chosen on the host: one scalar id per
// step (pages of at least 64 keys), one per wave and 32-row set (smaller
// pages), or one per row (in-page offsets past 31 bits). Each is its own
// kernel, so the common case keeps its register allocation. bf16 pages of at
// least 64 keys take 128-key steps with rows loaded straight into LDS
// (kDirectPages).
constexpr int kStepPages = 0, kSetPages = 1, kRowPages = 2, kDirectPages = 3;

// The next unit of a worker: the head of its XCD's list (entries i with
// i % 8 == the workgroup's index % 8), or of another list once that is empty;
// n or more when all are. (The XCDs do not end together: with its own list only,
// twelve FP8 turns behind 20-30K keys took 6618 against 6154 us.)
__device__ __forceinline__ int take_unit(int* taken, int n) {
  for (int d = 0; d < kXcds; ++d) {
    const int q = (blockIdx.x + d) & (kXcds - 1);
    const int idx = atomicAdd(&taken[q], 1) * kXcds + q;
    if (idx < n) return idx;
  }
  return n;
}

// A lane's query row (MFMA column r) of a unit.
struct UnitRow {
  bool ok;
  int ti, head;
};
__device__ __forceinline__ UnitRow unit_row(const ExtendArgs& a, int r, int cnt, int g, int hb) {
  const int RB = a.rows_head;
  const int ti = r / RB, hi = r - ti * RB;
  const bool ok = ti < cnt && hb * RB + hi < a.R;
  return {ok, ti, g * a.R + hb * RB + (ok ? hi : 0)};
}

// Joins a split unit's partials in key order, as a workgroup that has all of the
// unit's segments does (row block `wave` of the unit). slot0: the slot of segment 0.
// (The slots follow from the lengths, which are read again here: a caller that
// changes them under a running call gets wrong rows, but no slot outside the buffer.)
__device__ __forceinline__ void join_parts(const ExtendArgs& a, int slot0, int n_seg, int prefix, int n, int wave,
                                           f32x16 (&o)[4], float& m, float& l) {
  int slot = slot0;
  for (int s = 0; s < n_seg; ++s) {
    const StateWord* p = (const StateWord*)a.ws.part + ((size_t)slot * a.slot_waves + wave) * kSegWaveFloats;
    if (s == 0)
      seg_load(p, o, m, l);
    else
      seg_join(p, o, m, l);
    if (s + 1 < n_seg) slot = max(0, slot - segment_tiles(s + 1, prefix, n, unit_tiles(n, a.tile_tokens), a.tile_tokens));
  }
}

// The kernel's arguments, read again (the empty asm hides that they are the same).
__device__ __forceinline__ ExtendArgs reread_args() {
  typedef __attribute__((address_space(4))) const ExtendArgs ConstArgs;
  ConstArgs* ap = (ConstArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(ap));
  return *(const ExtendArgs*)ap;
}

// The LDS of a workgroup. The K and V buffers of the 128-key steps are arrays of
// their own (see tile_attn.hpp).
struct DirectLds {
  char *kl0, *kl1, *vl0, *vl1;
};

// One list entry `it` (its place: unit): attention of the unit's rows over all
// of its keys, or over one segment of a split unit. kSeg: the call has rows over
// several segments (mode: kSegments or kSplit) and the next unit of this
// workgroup is left in *next_unit. kSeg = false is the plain run over the keys.
template <bool kFp8, int kPages, bool kNt, bool kSeg, typename Lds>
__device__ __forceinline__ void extend_unit(const ExtendArgs& a, int unit, const int4 it, int mode, int n_units,
                                            const Lds& lds, int* next_unit, int* parts_here) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int swave = __builtin_amdgcn_readfirstlane(wave);
  const int2 part = kSeg && mode == kSplit ? a.ws.segs[unit] : make_int2(-1, -1);
  const int b = it.x, i0 = it.y, cnt = it.z, g = it.w & 0xffff, hb = it.w >> 16;
  int bad_seq = 0, bad = 0;               // sequence errors are reported by the planner
  const SeqRange sr = seq_range(a, b, &bad_seq);
  const int prefix = sr.kv - sr.n;
  const int t_unit = prefix + i0 + cnt;    // keys [0, t_unit) are visible to some row
  const int t_full = prefix + i0;          // keys [0, t_full) are visible to every row
  // segments of the unit's n_seg: one of a split unit, else all in turn
  const int n_seg = kSeg ? segment_count(t_unit) : 1;
  int seg = part.x >= 0 ? part.x : 0;

  const UnitRow row = unit_row(a, wave * kWaveRows + (lane & 31), cnt, g, hb);
  const int limit = row.ok ? prefix + i0 + row.ti : t_unit - 1;
  const int64_t qrow = sr.q0 + i0 + (row.ok ? row.ti : 0);

  bf16x8 qv[8];
  load_q_operand((const __bf16*)a.q + qrow * a.q_st + (int64_t)row.head * a.q_sh, row.ok, qv);
  int bad_scale = 0;
  // the K dequantisation scale joins the softmax scale, the V scale the output
  const KvScales dq = kv_scales<kFp8>(a.kv, g, &bad_scale);
  const float scale = a.scale * dq.k;
  const int* bt_row = a.kv.bt + (int64_t)b * a.kv.bt_sb;
  // a wave whose 32 rows are all past the unit's tokens (a short chunk, or
  // the one token of a deterministic decode) only stages
  const bool active = __builtin_amdgcn_ballot_w64(row.ok) != 0;
  f32x16 o[4];
  float m_run = kNegInf, l_run = 0.f;
  const bool whole = kSeg && part.x < 0 && n_seg > 1;   // this workgroup merges the unit's segments
  for (;;) {
    const int t_lo = segment_start(seg);
    const int t_end = seg + 1 < n_seg ? segment_start(seg + 1) : t_unit;
    // the segment before joins the running merge while this one's first rows are
    // on their way (its address is hidden from the compiler, which would otherwise
    // form it before the segments and spill: 133 instead of 115 us for 128 x 1K rows)
    auto begin = [&]() {
      if (kSeg && whole && seg > 0) {
        const ExtendArgs e = reread_args();
        StateWord* stash = (StateWord*)e.ws.stash + ((size_t)blockIdx.x * e.slot_waves + swave) * kSegWaveFloats;
        asm volatile("" : "+s"(stash));
        if (seg > 1) seg_merge(stash, o, m_run, l_run);
        seg_store(stash, o, m_run, l_run);
      }
#pragma unroll
      for (int jd = 0; jd < 4; ++jd)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[jd][e] = 0.f;
      m_run = kSeg && seg > 0 ? kNoKey : kNegInf;
      l_run = 0.f;
    };
    auto attend = [&](auto compute_tag, auto&& start) {
      constexpr bool kC = decltype(compute_tag)::value;
      if constexpr (kPages == kDirectPages) {
        static_assert(!kFp8, "rows go to LDS as stored: bf16 pages only");
        tile_attend_dl<kC, kNt>(a.kv, scale, bt_row, g, t_lo, t_end, t_full, limit, qv, lds.kl0, lds.kl1, lds.vl0,
                                lds.vl1, o, m_run, l_run, bad, start);
      } else {
        tile_attend_pp<kExtWaves, kPages != kRowPages, kFp8, kC, kPages == kSetPages, kNt>(
            a.kv, scale, bt_row, g, t_lo, t_end, t_full, limit, qv, *lds, o, m_run, l_run, bad, start);
      }
    };
    // (pages of fewer than 64 keys: before the rows, 6344 against 6442 us for twelve
    // turns of 512-1024 tokens behind 20-30K keys)
    constexpr bool kBefore = kPages == kSetPages;
    if (kBefore && active) begin();
    if (active)
      attend(std::true_type{}, [&] {
        if constexpr (!kBefore) begin();
      });
    else
      attend(std::false_type{}, [] {});
    if constexpr (!kSeg) break;
    if (!whole || ++seg == n_seg) break;
    __syncthreads();                       // the LDS tiles are free
  }
  // (as for the next unit, so that the step loop carries nothing of what follows it)
  const ExtendArgs e = kSeg ? reread_args() : a;
  if (kSeg && whole && active) {
    StateWord* stash = (StateWord*)e.ws.stash + ((size_t)blockIdx.x * e.slot_waves + swave) * kSegWaveFloats;
    asm volatile("" : "+s"(stash));
    seg_merge(stash, o, m_run, l_run);
  }
  // the next unit is taken only now, so that no worker holds one it cannot start
  if (kSeg && threadIdx.x == 0) *next_unit = take_unit(e.ws.hdr + 8, n_units);

  bool finish = true;
  if (kSeg && part.x >= 0) {
    // A part of a split unit goes to its slot, and the workgroup that brings
    // the last one finishes the rows; none waits, and a unit that lacks a part
    // is left unwritten. Every wave waits for its stores before the barrier;
    // behind it one thread makes them visible to the device, counts, and for
    // the last part takes in the others' (a release by each wave cost 7% on the
    // ragged deterministic decode: it writes the XCD's L2 back).
    int slot0 = part.y;
    for (int s = 1; s <= part.x; ++s) slot0 = slot_before(slot0, s, prefix, sr.n, e.tile_tokens);
    slot0 = min(slot0, e.max_slots - 1);
    StateWord* mine = (StateWord*)e.ws.part + ((size_t)part.y * e.slot_waves + swave) * kSegWaveFloats;
    asm volatile("" : "+s"(mine));         // (as the stash's)
    if (active) seg_store(mine, o, m_run, l_run);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      const int n = __hip_atomic_fetch_add(&e.ws.arrived[slot0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
      if (n == n_seg) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      *parts_here = n;
    }
    __syncthreads();
    finish = __builtin_amdgcn_readfirstlane(*parts_here) == n_seg;
    if (finish && active) join_parts(e, slot0, n_seg, prefix, sr.n, swave, o, m_run, l_run);
  }
  if (finish) {
    const float l_tot = sum_l32(l_run);
    if (row.ok) {
      const float inv = l_tot > 0.f ? dq.v / l_tot : 0.f;
      if (e.out_f32)
        store_o_row((float*)e.out + qrow * e.out_st + (int64_t)row.head * e.out_sh, o, inv);
      else
        store_o_row((__bf16*)e.out + qrow * e.out_st + (int64_t)row.head * e.out_sh, o, inv);
      if (e.lse && lane < 32)
        e.lse[qrow * e.lse_st + (int64_t)row.head * e.lse_sh] =
            l_tot > 0.f ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : kNegInf;
    }
  }
  if (bad) atomicOr(e.ws.err, kErrPage);
  if (bad_scale) atomicOr(e.ws.err, kErrScale);
}

// Units run in list order (longest key range first). Workgroups are handed
// to the XCDs round-robin, so each XCD takes every eighth entry; the planner
// lays the list out so those are the units of the (sequence, KV head) groups
// assigned to that XCD, which then share their keys through its L2.
//
// The planner, which knows the lengths, decides how the list is run. With no row
// over more than a segment: a workgroup per unit and the plain routine, whatever
// the block table's width (with the segments' routine for both, calls of short
// rows took 1-3% longer: 115.0 against 113.5 us for a deterministic decode of 128
// x 1K keys, 34.9 and 34.1 for two 64-token chunks). With such rows: a workgroup
// per CU, each with one running merge, takes units until the list is empty
// (multi-turn batch 40.2 ms against 42.0 with a workgroup per unit and no
// segments); the rest of the grid ends at once.
template <bool kFp8, int kPages, bool kNt>
__global__ __launch_bounds__(kExtWaves * 64, 2) void extend_mfma_kernel(ExtendArgs args) {
  __shared__ int next_unit, parts_here;
  // (read beside the header: the grid is no larger than the list's room)
  int4 it = args.ws.items[blockIdx.x];
  const int n_units = args.ws.hdr[0], mode = args.ws.hdr[1];
  int unit = blockIdx.x;    // (a worker's first unit needs no counter: the planner starts them behind these)
  auto run = [&](const auto& lds) {
    // (this branch first: laid out behind the other, the 64-key step loops of
    // long rows ran 1-2% slower)
    if (__builtin_expect(mode != kOneSegment, 1)) {
      if (unit >= args.workers) return;
      // every pass takes a new entry of a finite list, so the loop ends
      while (unit < n_units) {
        // The arguments are read again for each unit: kept over the loop they would
        // not fit the scalar registers beside a unit's own values.
        const ExtendArgs a = reread_args();
        extend_unit<kFp8, kPages, kNt, true>(a, unit, it, mode, n_units, lds, &next_unit, &parts_here);
        // the LDS tiles are free and next_unit is written; it is read before the
        // next unit's barriers, which every wave passes before the next write
        __syncthreads();
        unit = __builtin_amdgcn_readfirstlane(next_unit);
        if (unit < n_units) it = a.ws.items[unit];
      }
    } else if (unit < n_units) {
      extend_unit<kFp8, kPages, kNt, false>(args, unit, it, mode, n_units, lds, &next_unit, &parts_here);
    }
  };
  if constexpr (kPages == kDirectPages) {
    __shared__ __attribute__((aligned(16))) char kl0[kDlKBytes], kl1[kDlKBytes], vl0[kDlVBytes], vl1[kDlVBytes];
    run(DirectLds{kl0, kl1, vl0, vl1});
  } else {
    __shared__ TileLds lds;
    run(&lds);
  }
}

}  // namespace

int plan_extend_on_host(const ExtendArgs& a, int* split_seqs) {
  const int heads = a.Hkv * a.head_blocks;
  int bad = 0;
  std::vector<SeqRange> r(a.B);
  std::vector<int> order(a.B), keys(a.B), slot_of(a.B, -1);
  unsigned long long all_keys = 0, all_units = 0;
  for (int b = 0; b < a.B; ++b) {
    r[b] = seq_range(a, b, &bad);
    order[b] = b;
    keys[b] = r[b].kv;
    const unsigned long long units = (unsigned long long)unit_tiles(r[b].n, a.tile_tokens) * heads;
    all_units += units;
    all_keys += units * r[b].kv;
  }
  *split_seqs = 0;
  if (a.B <= kSortMax) {
    long long first = 0;
    for (int b = 0; b < a.B && a.max_slots > 0; ++b) {
      const int need = split_need(a, r[b], all_keys, all_units);
      if (need > 0 && first + need <= a.max_slots) {
        slot_of[b] = (int)first;
        keys[b] = std::max(kSegKeys, r[b].kv / 2);
        ++*split_seqs;
      }
      first += need;
    }
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return keys[x] > keys[y]; });
  }
  bool any_long = false;
  for (const SeqRange& x : r) any_long = any_long || (a.segmented && x.n > 0 && x.kv > kSegKeys);
  int offset = 0;
  for (int p = 0; p < a.B; ++p) {
    const SeqRange& s = r[order[p]];
    const int slot = slot_of[order[p]];
    const int per = slot >= 0 ? (int)unit_segments(s, a.tile_tokens) : unit_tiles(s.n, a.tile_tokens);
    const SeqPlan plan{order[p], s.n, s.kv - s.n, slot, offset, per};
    for (int i = 0; i < per * heads; ++i)
      bad |= place_item(a, plan, i, kXcdGroups && heads % kXcds == 0, *split_seqs > 0);
    offset += per * heads;
  }
  a.ws.hdr[0] = std::min(offset, list_room(a, *split_seqs > 0));
  a.ws.hdr[1] = *split_seqs > 0 ? kSplit : any_long ? kSegments : kOneSegment;
  return bad;
}

hipError_t launch_extend(const ExtendArgs& a, hipStream_t stream, KernelTimer* timer) {
  plan_extend_kernel<<<1, 1024, 0, stream>>>(a);
  // a workgroup per unit, or per worker (the device decides; both at most max_items)
  const unsigned grid = (unsigned)std::max(a.max_items - a.max_slots, a.workers);
  if (timer) (void)hipEventRecord(timer->start, stream);
  const bool scalar_ids = scalar_page_offsets(a.kv);
  const int pages = !scalar_ids ? kRowPages : (a.kv.page_size >= kKeys ? kStepPages : kSetPages);
  // decode through the extend kernel with one unit per (sequence, KV head):
  // every key row is read once, so the rows are loaded non-temporally (pages
  // of at least a step only)
  const bool once = a.decode_rows > 0 && a.head_blocks == 1 && a.decode_rows <= a.tile_tokens;
  auto go = [&](auto fp8_tag) {
    constexpr bool kF = decltype(fp8_tag)::value;
    auto launch = [&](auto pages_tag, auto nt_tag) {
      extend_mfma_kernel<kF, decltype(pages_tag)::value, decltype(nt_tag)::value>
          <<<grid, kExtWaves * 64, 0, stream>>>(a);
    };
    const std::true_type nt{};
    const std::false_type cached{};
    if constexpr (!kF) {
      if (pages == kStepPages && !a.staged) {
        const std::integral_constant<int, kDirectPages> direct{};
        if (once)
          launch(direct, nt);
        else
          launch(direct, cached);
        return;
      }
    }
    const std::integral_constant<int, kStepPages> step{};
    if (pages == kStepPages && once)
      launch(step, nt);
    else if (pages == kStepPages)
      launch(step, cached);
    else if (pages == kSetPages)
      launch(std::integral_constant<int, kSetPages>{}, cached);
    else
      launch(std::integral_constant<int, kRowPages>{}, cached);
  };
  if (a.kv.k_scale)
    go(std::true_type{});
  else
    go(std::false_type{});
  if (timer) (void)hipEventRecord(timer->stop, stream);
  return hipGetLastError();
}

}  // namespace rl
