// Internal: the plan blob shared by the host planner and the kernels.
//
// The blob is position independent (offsets, no pointers) so the caller can copy
// it to the device byte for byte.  It holds the result of Alg. 1's prefill loop
// (which chunk goes to which bitwidth class, in which order) plus the derived
// block layout of the packed cache and the work split of the decode kernel.
#pragma once
#include <stdint.h>

#include "../../include/cocktail.h"

namespace cocktail {

constexpr uint32_t kPlanMagic = 0x434b544cu;  // "CKTL"
constexpr uint32_t kPlanVersion = 16;
// (15 keeps its ticket counters a line apart in plans without pools too, where no kernel looks at them)
constexpr bool known_version(uint32_t version) { return version == 15 || version == kPlanVersion; }
constexpr int kTB = 64;                        // tokens per block
constexpr int kNumClasses = 4;                 // INT2, INT4, INT8, FP16: the order of the concatenation
constexpr int kFp16Class = kNumClasses - 1;
constexpr int kClassBits[kNumClasses] = {2, 4, 8, 16};
constexpr int kPartialFloats = 4;              // (m, l, tokens covered as int32, unused) in front of the D output values
// Units one wave consumes per loop iteration in class INT2, INT4, INT8, FP16: the grain of the shared pools.
#ifndef COCKTAIL_J2
#define COCKTAIL_J2 4
#endif
#ifndef COCKTAIL_J4
#define COCKTAIL_J4 2
#endif
#ifndef COCKTAIL_J8
#define COCKTAIL_J8 1
#endif
#ifndef COCKTAIL_J16
#define COCKTAIL_J16 1
#endif
constexpr int kIterUnits[kNumClasses] = {COCKTAIL_J2, COCKTAIL_J4, COCKTAIL_J8, COCKTAIL_J16};
constexpr int kMaxPoolSegments = 32;           // segments one pool may touch (a worker tracks them in a bit mask)
// The appended tokens of a (sequence, kv head) are attended to by one extra wave per this many 64-token
// blocks of append capacity (one partial state each), so a long generation does not hang on a single wave.
constexpr int kAppendSliceBlocks = 8;
// Packed K+V bytes of a call from which its loads are non-temporal (decode_common.h).
constexpr int64_t kNonTemporalMinBytes = int64_t(64) << 20;
// The chip: 256 compute units of four SIMDs; the decode kernels run two waves per SIMD.
constexpr int kCuWaves = 8, kChipWorkers = 256 * kCuWaves, kSimds = kChipWorkers / 2;
// Waves per workgroup of a decode launch: a compute unit's where the workers fill the chip exactly once, else one.  With twice or three
// times as many workers the next workgroup of a unit waits for the slowest of eight waves, where a single wave starts as soon as one
// ends.  One by one | by unit (us per call, caches in turn): one head per wave, 4096 workers, 32K 32 heads 36.6 | 38.4, 128K 40 heads 117.7 |
// 121.8, 6144 workers 40.1 | 42.6 and 122 | 132; eight heads, 4 x 32K 44.8 | 46.7 and 48.9 | 56.0.  (4 x 64K with four heads 76.3 | 74.4 and
// 84 | 80.4, 4 x 128K with eight 148 | 138.5; but 2048 workers take 67 and 126 there.)  A call with append slices in its grid: launch_workers.
__host__ __device__ inline int workgroup_waves(int num_workers, int append_slices) {
  return num_workers == kChipWorkers && append_slices == 0 ? kCuWaves : 1;
}
// uint32 slots between two ticket counters: a 128-byte line each where there are pools (half a line each: ragged contexts up to 130K, four heads
// per kv head, 205.1 -> 205.25 us per call; 128K, 40 heads 102.4 -> 102.5).  In plans without pools nobody draws a ticket, and a line each would be an
// eighth of what a request uploads (2 contexts up to 32K, 8 kv heads: 485 -> 428 KB).
constexpr int kPoolCounterStride = 32, kCounterStride = 4;
inline int counter_stride(int num_pool_segs) { return num_pool_segs > 0 ? kPoolCounterStride : kCounterStride; }
// Query heads per kv head for which one wave serves all of them with matrix instructions and V is stored in token quads.
constexpr int kQuadMinRep = 2, kQuadMaxRep = 8;
__host__ __device__ inline bool uses_token_quads(int rep) { return rep >= kQuadMinRep && rep <= kQuadMaxRep; }
// Of these, 5 to 8 heads run on the kernel with eight heads per wave (16x16x32 instructions), 2 to 4 on the one with four.
__host__ __device__ inline bool uses_tiles(int rep) { return rep > 4 && rep <= kQuadMaxRep; }
// Query heads one wave serves when rep = Hq / Hkv heads share a kv head: all of them up to kQuadMaxRep; beyond
// that the heads of a kv head are cut into equal sets (the largest divisor of rep that the matrix kernel takes),
// each walking the kv head's blocks by itself; 1 (a wave per query head, vector ALU) if there is no such divisor
// or the plan asks for it.
__host__ __device__ inline int work_rep_of(int rep, bool vector_alu_only) {
  if (vector_alu_only || rep <= 1) return 1;
  if (rep <= kQuadMaxRep) return rep;
  for (int d = kQuadMaxRep; d >= kQuadMinRep; --d)
    if (rep % d == 0) return d;
  return 1;
}

// What a plan may need of the built-in workspace.  The common limit holds the plans of the kernels with up to four heads per wave; two
// kinds of plans have more partial states and may go as much beyond it: with eight heads per wave there are twice the workers of the
// former kernel, whose workgroups of two waves were a worker each (up to 1024 more states of 8 x 132 floats, 4.3 MB), and where the sets
// of a kv head are planned as twins every set is cut where the others are (up to 4.6 MB more over some 400,000 random plans).
inline int64_t static_workspace_limit(int v_layout, int work_rep, int rep) {
  return v_layout == COCKTAIL_V_TOKEN_QUADS && (uses_tiles(work_rep) || work_rep < rep) ? COCKTAIL_STATIC_WORKSPACE_BYTES_TILES
                                                                                        : COCKTAIL_STATIC_WORKSPACE_BYTES;
}

// One contiguous run of blocks of one (sequence, kv head, class): the part of it that one group works on.
struct Segment {
  int32_t b, h, cls, ntok;   // ntok: valid tokens from the first block of this piece to the end of the
                             // (sequence, kv head, class) run; may exceed nblk * 64
  int32_t blk0;              // first block, index into the class buffer
  int32_t nblk;
  int32_t gblk0;             // first block in the global order
  int32_t pid0;              // partial id of the first worker whose own range touches this segment
};

// Everything a decode worker (wave) needs to start streaming, in one 64-byte record.
struct WorkerRec {
  int32_t g0, g1;            // its own block range [g0, g1) of the global order
  int32_t seg0;              // index of the segment holding g0
  int32_t pid0;              // partial id of its piece of segment seg0 (in later segments it is the first visitor)
  Segment first;             // copy of segments[seg0]
  int32_t group;             // index of its GroupRec and of the group's ticket counter
  int32_t rank_nps;          // position inside the group | (GroupRec::nps << 16)
  int32_t ngran, pseg0;      // copies of the GroupRec fields, so that a worker starts from one record
};
static_assert(sizeof(WorkerRec) == 64, "WorkerRec is one 64-byte line");

// A group of consecutive workers shares a pool: the tail of the group's block range, handed out one
// loop iteration at a time through an atomic ticket counter, so that workers that finish their own
// range early take over work from slower ones.
struct GroupRec {
  int32_t ngran;             // tickets 0 .. ngran-1 are valid; 0 = the group has no pool
  int32_t pseg0;             // index of its first PoolSeg
  int32_t nps;               // number of PoolSegs (<= kMaxPoolSegments)
  int32_t nworkers;
  int32_t counter;           // index of its ticket counter (times counter_stride)
  int32_t pad[3];
};
static_assert(sizeof(GroupRec) == 32, "GroupRec layout");

// Short contexts have a second split of the work, which leaves the merge to the workgroups themselves: a workgroup of kCuWaves waves works on one
// row (sequence, work head), every wave on a range of units of one class, or of the row's appended tokens.
struct ShortGroup {          // a workgroup
  int32_t b, qrow;           // its row: sequence, index of the first query head
  int32_t context;           // tokens of the sequence
  uint32_t place;            // index among the workgroups of the row | their number << 8 | the row's counter << 20
};
struct ShortRec {            // one of its waves
  int32_t cls;               // class, or kNumClasses: the appended tokens
  uint32_t range;            // units u0 | u1 << 16 of the run (appended tokens: part u0 of u1 equal parts); u0 == u1: no work
  int32_t ntok, blk0;        // tokens and first block of the run (appended tokens: 2^32 / u1 + 1, first block in the append buffers)
};
static_assert(sizeof(ShortGroup) == 16 && sizeof(ShortRec) == 16, "layout of the split for short contexts");
constexpr int kShortCounterStride = 16;        // uint32 slots between two counters
// States (of one query head each) of a row that the last of its workgroups may find: they are merged in shared memory.
constexpr int kShortThreads = 64 * kCuWaves, kShortStates = 128;

// The part of a pool that lies inside one segment.  Ticket t with gran0 <= t < gran0 + ceil(nunits / J)
// stands for units [unit0 + (t - gran0) * J, + J) of the segment, J = kIterUnits[class].
struct PoolSeg {
  int32_t seg;               // segment index
  int32_t unit0;             // first unit, counted from the start of the segment (a unit = what a wave handles at a
                             // time: 32 tokens at head_dim 128, 64 at head_dim 64)
  int32_t nunits;
  int32_t gran0;             // first ticket of this part
  int32_t slot0;             // partial id of rank 0; rank r < nslots of the group writes slot0 + r
  int32_t nslots;            // ranks that can start a partial state here: those whose own range ends in an
                             // earlier segment (the others arrive with the state of this segment)
  int32_t pad[2];
};
static_assert(sizeof(PoolSeg) == 32, "PoolSeg layout");

// One 64-token block of the packed cache as the reorder+quantize kernel sees it (one record per
// block, class by class in (b, h, block) order, i.e. in the order of the class buffers).
struct RQItem {
  int64_t ragged_row;        // row index of the block's first token in the ragged source layout
  int32_t b, h;
  int32_t t0;                // source token of row 0 if the block's rows are consecutive source tokens, else -1
  int32_t cls_nvalid;        // class | valid rows << 8
  int32_t j;                 // block index inside its (b, h, class) run
  int32_t pad;
};
static_assert(sizeof(RQItem) == 32, "RQItem layout");

struct PlanHeader {
  uint32_t magic, version;
  int32_t batch, num_q_heads, num_kv_heads, head_dim, chunk_size, group_size;
  int32_t rep;               // Hq / Hkv
  int32_t work_heads;        // heads of the decode work split: Hkv, or Hq where every query head is served by a wave
                             // of its own (vector-ALU-only plans, and Hq / Hkv beyond what the matrix kernel takes):
                             // Segment::h and the (sequence, head) ranges of partial ids count in these
  int32_t work_rep;          // query heads one wave serves: Hq / work_heads
  int32_t num_workers, num_segments, num_partials;
  int32_t total_gblocks;
  int32_t v_layout;          // 0: V blocks hold token rows like K; 1: token quads (2 to 8 query heads per kv head)
  int64_t total_chunks;
  int64_t total_tokens;
  int64_t class_blocks[kNumClasses];
  int64_t class_bytes[kNumClasses];
  int32_t block_bytes[kNumClasses];
  int32_t row_bytes[kNumClasses];     // code bytes per token row
  int64_t workspace_bytes;
  int64_t plan_bytes;
  int64_t packed_bytes;
  // byte offsets of the arrays inside the blob (each 16-byte aligned)
  int32_t off_seq_len;        // int32 [B]
  int32_t off_cum_tokens;     // int64 [B+1]
  int32_t off_chunk_off;      // int32 [B+1]   prefix of N_b
  int32_t off_perm;           // int32 [total_chunks]  per-sequence chunk indices, gather form
  int32_t off_class_tokens;   // int32 [B][4]
  int32_t off_class_chunk0;   // int32 [B][4]  first position in perm_b of class c
  int32_t off_blk_base;       // int32 [B+1][4] first block of sequence b in class buffer c
  int32_t off_nblk;           // int32 [B][4]  blocks per head that hold tokens
  int32_t off_run_blocks;     // int32 [B][4]  blocks per head the run is laid out with (>= the above: FP16 runs with
                              //               room for tokens that are folded in later)
  int32_t off_segments;       // Segment [num_segments]
  int32_t append_capacity;    // tokens per sequence the append buffers hold (0 = none)
  int32_t off_worker_rec;     // WorkerRec [num_workers]
  int32_t off_group_rec;      // GroupRec [num_groups]
  int32_t off_pool_seg;       // PoolSeg [num_pool_segs]
  int32_t off_counters;       // uint32 [num_groups * counter_stride], zero; the only part kernels write
  int32_t num_groups, num_pool_segs;
  int32_t append_blocks;      // blocks per (sequence, kv head) in the append buffers
  int32_t off_bh_off;         // int32 [B*Hkv + 1] prefix: (b, kv head) owns partial ids bh_off[bh] .. bh_off[bh+1]-1;
                              // with append buffers the last append_slices ids of each range are those of the appended tokens
  int32_t off_rq_items;       // RQItem [sum of class_blocks]
  int32_t append_slices;      // waves (and partial ids) per (sequence, kv head) for the appended tokens
  int64_t ws_status_off;      // byte offset, inside the decode workspace, of int32 [B * Hq]: per (sequence, query
                              // head) tokens covered by the last call's partial states minus tokens of the sequence
                              // (0 = every token was attended to exactly once)
  int16_t short_groups;       // workgroups of the split for short contexts (ShortRec), 0 = the plan has none
  int16_t short_units;        // 1: a loop iteration of its waves is one unit (or staged block) of any class; 0: kIterUnits
  int32_t off_short;          // ShortRec [short_groups * kCuWaves], ShortGroup [short_groups], then (128-byte aligned) a counter per row, zero
                              // between calls
};
static_assert(sizeof(PlanHeader) == 304, "the arrays start behind 304 bytes; the last two fields are zero in plans that were written before they existed");

inline int64_t short_group_offset(const PlanHeader& hd) { return hd.off_short + int64_t(sizeof(ShortRec)) * kCuWaves * hd.short_groups; }
inline int64_t short_counters_offset(const PlanHeader& hd) { return (short_group_offset(hd) + int64_t(sizeof(ShortGroup)) * hd.short_groups + 127) & ~int64_t(127); }

// Token-quad form of a V block: byte offset, inside the block, of the half-word that holds token i
// (0..63) of lane j's channels e .. e + per - 1 in the 64-channel half h, where per = 16 / bits values
// fill a half-word and ph = pieces of 16 bytes per 64-channel half of a row (bits / 2).  Channel of (h, j, e):
// 64 h + 32 (e / 8) + 8 j + e % 8.
__host__ __device__ inline uint32_t quad_halfword_offset(int ph, int per, int i, int h, int j, int e) {
  const int w = 2 * (e / per) + ((i & 3) >> 1);
  return uint32_t(((ph * h + (w >> 2)) * kTB + ((i & ~3) | j)) * 16 + (w & 3) * 4 + 2 * (i & 1));
}

template <typename T>
__host__ __device__ inline const T* plan_array(const void* blob, int32_t off) {
  return reinterpret_cast<const T*>(static_cast<const char*>(blob) + off);
}

}  // namespace cocktail
