// Host planner: Alg. 1 prefill loop (stable partition of chunks by bitwidth),
// block layout of the packed cache, and the static split of the decode work.
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <cstring>
#include <unistd.h>
#include <queue>
#include <utility>
#include <vector>

#include "../../include/cocktail.h"
#include "common.h"
#include "plan.h"

namespace cocktail {

static thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

int check_shape(const cocktail_shape* s) {
  if (!s) return fail(COCKTAIL_EINVAL, "shape is NULL");
  if (s->batch < 1 || s->num_q_heads < 1 || s->num_kv_heads < 1 || s->chunk_size < 1)
    return fail(COCKTAIL_EINVAL, "batch, head counts and chunk_size must be >= 1");
  if (s->num_q_heads % s->num_kv_heads != 0)
    return fail(COCKTAIL_EINVAL, "num_q_heads %d is not a multiple of num_kv_heads %d", s->num_q_heads,
                s->num_kv_heads);
  if (s->head_dim < 64 || s->head_dim % 64 != 0 || s->head_dim > 512)
    return fail(COCKTAIL_EINVAL, "head_dim %d must be a multiple of 64 in [64, 512]", s->head_dim);
  if (s->group_size != 32 && s->group_size != 64 && s->group_size != 128)
    return fail(COCKTAIL_EINVAL, "group_size %d must be 32, 64 or 128", s->group_size);
  if (s->head_dim % s->group_size != 0)
    return fail(COCKTAIL_EINVAL, "group_size %d does not divide head_dim %d", s->group_size, s->head_dim);
  return COCKTAIL_OK;
}

constexpr int64_t kCostWeight[kNumClasses] = {1150, 1300, 1100, 530};
// The same for the kernels on the matrix unit: two to four query heads per wave.
constexpr int64_t kQuadCostWeight[kNumClasses] = {1300, 1250, 950, 450};
// Five to eight heads per wave: the split is static, so nothing absorbs an error, and a byte of an INT2 or INT4 block carries twice the
// vector work of the kernel above while one of an FP16 block only waits for memory.  FP16 at 450 | 420 | 400 | 380 | 360 (us):
// 4 x 128K at 8 heads 134.6 | 131.4 | 130.5 | 129.8 | 132.3; one of 64K 30.7 | 30.0 | 29.7 | 29.8 | 30.7; 2 x 64K at 5 heads 41.1 | 40.4 | 40.3 |
// 39.9 | 39.8; INT2 and INT4 5 % to either side of these figures differ by no more than two runs do.
constexpr int64_t kTileCostWeight[kNumClasses] = {1300, 1250, 950, 390};
// With the sets of heads of a kv head as twins all but the first read the blocks from the L2, so FP16 bytes are cheaper still.  FP16 at
// 450 | 400 | 360 | 340 | 320 | 300 (us): 8 ragged contexts, 16 heads 52.8 | 51.4 | 50.8 | 50.5 | 50.1 | 50.9; 2 x 40K at 12 heads 42.7 | 40.6 | 40.7 |
// 40.1 | 39.9 | 40.1; one of 128K at 16 60.5 | 60.7 | 58.3 | 58.4 | 57.9 | 58.3.
constexpr int64_t kTwinCostWeight[kNumClasses] = {1300, 1250, 950, 330};
// Workers per group.  Measured on MI355X: with one query head per kv head 4 to 8 are equal on long
// ranges (8 a hair ahead at 128K), 5 to 6 clearly best on short ones (32K: 33.2 against 35.9 us); the
// grouped-query kernel likes 4.
constexpr int kGroupWorkers = 8, kGroupWorkersShort = 6, kQuadGroupWorkers = 4;
constexpr int kXcds = 8;   // workgroups (of one wave or a unit's eight, workgroup_waves) are handed to the XCDs round robin
constexpr int kLongRangeBlocks = 24;   // average blocks per worker from which a range counts as long
// The share of a group's cost that goes into its shared pool.
constexpr int kPoolPercent = 25;
constexpr int kPairMode = 0;
constexpr int kLayout = 0;
// The split for short contexts is taken while no wave has more loop iterations than this: of one unit of any class (five heads and more: a staged block),
// else of kIterUnits.  Calls on prepared arguments, as two launches -> one (us).  One unit, one to four heads: 8 heads 2K (1 unit) 9.6 -> 7.5, 32 heads
// 5.3K (2) 12.9 -> 9.7, 4 ragged up to 7K at head_dim 64 (4) 12.5 -> 9.7, 3 x 32 heads 2.3K (6) 14.2 -> 11.3, 4 ragged up to 4.4K at 64 q / 32 kv heads
// (8) 18.6 -> 16.4.  kIterUnits: the same up to 5K (3 iterations) 22.4 -> 20.2, 4 ragged at 80 q / 40 kv heads, 3.2K and 205 appended (6) 25.7 ->
// 25.0.  With kIterUnits for all of them a wave with one unit runs the code of four: 10.3 instead of 8.9 on the first of these shapes.  Five heads and more,
// where what is written and read per state is five to eight times as much: 3 x 1.4K at five heads (1 block) 10.3 -> 9.9, 4 x 1.4K at seven
// (1) 10.9 -> 9.8, seven at head_dim 64 with appended tokens (3) 15.4 -> 13.0; 3 ragged up to 17K at five heads, 476 appended (4) 27.2 -> 22.4, 8 x
// 7.3K at seven (4) 22.1 -> 19.5, 3 x 13.4K at six (4) 20.3 -> 19.8; with longer ranges 24.8K at six (6) 15.7 -> 18.9.  At head_dim 64, where a
// block has half the bytes: 8 x 6.4K at eight heads (4) 16.6 -> 13.4, 3 x 23.4K at five (5) 21.0 -> 16.5, 3 ragged up to 49K (6) 18.8 -> 18.3.  Sets
// of heads, which as twins find each other's blocks in the L2: 3 blocks, as four and more gain and lose (3 x 7K at sixteen heads 16.3 -> 16.5, 25K
// 19.8 -> 22.2, 8 x 7.3K at ten (5) 19.0 -> 20.3, but 2 x 14K at twelve 17.9 -> 17.1).
constexpr int kShortUnits = 8, kShortIterations = 6, kShortUnitsSets = 3, kShortUnitsTiles = 4, kShortUnitsTilesD64 = 6;
// A row that one workgroup finishes is done 2 us after its waves, one of several after 3: worth this many iterations.
constexpr int kShortMergeIterations = 1;
// Sets of heads at head_dim 128 keep two launches where a wave has two staged blocks and more and a row more workgroups than this, unless they
// fill the chip: the last of a row merges as many states of five to eight heads, and in the two launches twins find each other's blocks in the L2.
// Without appended tokens.  Two launches -> one (us): 16 heads per kv head 15.6K 15.6 -> 16.7, 0.9K and 14.3K 16.2 -> 18.3, 10 heads 8 ragged up to 11.5K
// 14.5 -> 15.8, 12 heads 11.1K 12.5 -> 13.8; of 29 shapes one gains, 10 heads 19.3K 16.7 -> 15.8.  Taken: 3 x 6.8K at ten heads (5 workgroups) 18.9 -> 16.9,
// 8 x 12.8K at sixteen (16, a full chip) 15.2 -> 14.3, 14.6K and 362 appended at sixteen 21.4 -> 20.6.
constexpr int kShortGroupsSets = 8;
// Relative speed of a worker of class [self] whose SIMD mate works on class [mate] (INT2, INT4, INT8, FP16), traced
// on MI355X at equal weighted cost: two bandwidth-bound or two ALU-bound waves on a SIMD get in each other's way,
// an INT4 wave next to an FP16 wave runs well ahead.  (INT8 was not traced: neutral.)
constexpr double kPairSpeed[kNumClasses][kNumClasses] = {
    {0.87, 1.0, 1.0, 1.0}, {1.0, 1.17, 1.0, 1.27}, {1.0, 1.0, 1.0, 1.0}, {0.97, 1.06, 1.0, 0.9}};
// A group only gets a pool if its range holds at least this many blocks per worker.
constexpr int kMinBlocksPerWorkerForPool = 4;
// Groups with short ranges (below this many blocks per worker) put a larger share into the pool: there the
// differences between compute units weigh more than the cost of the tickets.
constexpr int kShortRangeBlocks = 16;
constexpr int kShortRangePoolPercent = 40;

// Plans without pools whose ranges end where runs end (aligned_ranges).  A worker whose range crosses from one run into the next starts a second
// partial state: another query, another flush, and across classes a pipeline that runs empty; and where a worker has few blocks, ranges cut
// by cost to the nearest block differ by a block, i.e. by a whole iteration.  With up to this many blocks per worker on average that
// costs more than the pools bring in; five to eight heads per wave never have pools.  By cost and with pools -> aligned (us; MIX 10 % FP16,
// 30 % INT4, 60 % INT2): one head, 8 kv heads, 16K 16.1 -> 15.0, 24K 17.7 -> 16.4, 64K (4 blocks per worker) 25.5 -> 23.2, 32 x 32K (8)
// 35.3 -> 34.4, 4 x 45K (11) 44.3 -> 43.7, but 40.2 -> 42.4 with 5 / 25 / 70 %, 40 x 128K (40) 104 -> 117; four heads, 24K 20.5 -> 18.5, 64K
// 29.4 -> 25.2, 4 x 45K 48.6 -> 45.6, 4 x 64K (16) 68.5 -> 67.3, ragged up to 128K (36) 206 -> 210; eight heads, 24K 20.8 -> 18.3, 64K 28.8 ->
// 25.0, 4 x 128K 130 -> 126.7, 8 x 16K with 300 appended 49.8 -> 47.6; sixteen, ragged up to 64K 50.3 -> 47.3.
// With kInt2Stretch as well, one head, 10 and 12 blocks per worker: 42.8 -> 41.0 and 48.4 -> 45.9 at 5 / 25 / 70 %, 46.6 -> 45.6 and 52.0 ->
// 51.4 at MIX; at 16 blocks 58.4 -> 57.0, but 64.7 -> 65.0.
// (One cache again and again.  With distinct caches in turn, as a model's layers are, 173 shapes of 8 to 20 blocks, six mixes, G 32 to 128: 4.1 % in the
// mean; 4 x 64K, four heads, 5 % FP16, 15 % INT8, 30 % INT4, 50 % INT2 65.2 -> 63.6 at G 32 and 60.2 -> 59.1 at G 64, 32 heads 32K at MIX 35.1 ->
// 34.4; losses of up to 3 % at 14 blocks and more, e.g. 4 x 64K at 15 / 35 / 50 %, G 64 63.7 -> 65.3, against 68.0 -> 66.6 at G 32.)
constexpr int kAlignedBlocks = 8, kAlignedBlocksHeads = 12, kAlignedBlocksQuads = 20;
// One head per wave and more than kAlignedBlocks: not where INT2 has more than one worker per SIMD but fewer than kFewInt2Pairs (kInt2Stretch could
// not hold it) and the runs are few (kFewRuns): some SIMDs have two INT2 workers, and without pools the call waits for those.  10 to 12 blocks
// per worker, caches in turn, by cost and with pools -> aligned: 80 % INT2 37.6 -> 38.9, 41.4 -> 44.2, 36.1 -> 37.6, 85 % 38.6 -> 40.1, 41.5 -> 43.2,
// 2.1 % in the mean of 28 such shapes (-8 to +10 %).  With more pairs they are the rule, not the exception: 90 % 36.9 -> 35.6, all INT2 33.1 -> 30.3;
// with more runs pools need a partial state for each: 34 shapes -1.9 % in the mean (-17 to +7 %).  (Waves launched one by one meet by chance:
// 75 % INT2 and 300 tokens appended 41.5 -> 39.9, 39.5 -> 39.9.)
constexpr double kFewInt2Pairs = 1.4;
constexpr int kFewRuns = 256;
// (the larger two with a full chip.  With one worker per SIMD the longest range decides: 1024 workers, behind another kernel, 4 x 40K with four
// heads at 5 / 25 / 70 % (20 blocks) 61.5 -> 64.7; 1536, 32 heads 32K (11) 41.1 -> 43.5, but 4 x 40K with four heads (13) 51.1 -> 48.4.)
// Workers w and w + kSimds share a SIMD, and two INT2 ranges side by side, both bound by the vector ALU, take 1.4 times as long as one next to
// another class (5 / 25 / 70 %, 2 x 60K, 12 heads: workers next to INT4 or FP16 end at 34 us, the later one of two INT2 workers at 47).
// So INT2 gets no more than kSimds workers where its ranges need not become longer than this for it; those of the other classes become
// shorter.  Without -> with (us, behind another kernel of 6): 32 heads 32K 39.6 -> 35.3, 4 x 64K at 8 heads 65.8 -> 61.9, 2 x 40K at 9 56.3 ->
// 48.0, at 16 45.2 -> 37.1, 4 x 45K at 4 48.6 -> 46.9.  A limit of 1.15 misses some (2 x 64K at 5 heads 37.4 -> 35.3), 1.7 brings nothing more;
// the same for INT4 (10 / 60 / 30 %, needs 1.4) 44.1 -> 48.
// Only where the launch goes by compute unit (workgroup_waves), which is what makes w and w + kSimds mates whatever ran before: one by one the
// longer INT2 ranges still meet each other on some SIMDs.  Without -> with, 300 tokens appended, behind another kernel: 4 x 64K, four heads
// 62.7 -> 69.9, eight 67.4 -> 75.9; 2 x 40K, nine 55.1 -> 58.7 (by cost 63.0, 66.8 and 56.2); 3072 workers, 32 heads 32K 35.6 -> 37.6.
constexpr double kInt2Stretch = 1.25;
// Such ranges are taken where the longest is at most this many times the mean plus this many blocks of the dearest class.  Beyond, the runs are
// too many for the workers: the longest ones cannot be cut further, and the whole call waits for them (32 heads, 128K and 79 contexts of 1K:
// 9.2 times the mean).  By cost -> aligned (us; longest range over mean, blocks per worker): five heads and more, 48 x 16K 183 -> 207 (1.8, 48),
// 40 x 16K 163 -> 179 (1.4, 40), 64 of up to 13K 68 -> 153 (6.7, 11), but 64 x 4K 87.1 -> 82.2 (1.5, 16).  Up to four, where the pools
// need a partial state per run and rank, more: 32K and 79 x 2K 71 -> 78 (2.3, 12), 64 of up to 24K 98 -> 221 (8.6, 14), but 32K and 48 x 2K
// 51.9 -> 44.5 (1.5, 8), at 70 % INT2 32K and 79 x 2K 59.8 -> 53.6 (1.75, 12).  Of 1324 random shapes (up to four heads | more) these keep 1090 | 181
// with 24 | 4 that lose more than 4 %, at most 11, and leave out 17 | 3 that would have gained 3 % and more (1.25 for all: 68).
constexpr double kLongestRange = 1.8, kLongestRangeTiles = 1.25;
constexpr int kLongestRangeBlocks = 2;
// Fewer blocks per worker than this are rounded to whole iterations (INT2: four units): 24K, eight heads 20.2 -> 18.7.
constexpr int kWholeIterationBlocks = 8;

// The split parameters.  The defaults are what was measured best on MI355X; the environment variables
// are tuning aids for experiments and are read once per cocktail_plan call.
struct Tuning {
  int64_t weight[kNumClasses] = {kCostWeight[0], kCostWeight[1], kCostWeight[2], kCostWeight[3]};   // COCKTAIL_COST_WEIGHTS="int2,int4,int8,fp16" or "int2,int4,fp16"
  bool weight_set = false;
  int pool_percent = kPoolPercent;      // COCKTAIL_POOL_PERCENT   0..100
  bool pool_percent_set = false;        // the environment fixed the share for every group
  int group_workers = 0;                // COCKTAIL_GROUP_WORKERS  1..1024; 0 = the default for the kernel that will run
  bool pair_speed = true;               // COCKTAIL_PAIR_SPEED     0 | 1
  int layout = kLayout;                 // COCKTAIL_LAYOUT         0 | 1
  int pair_mode = kPairMode;            // COCKTAIL_PAIR_MODE      0 | 2 | 3
  int min_pool_blocks = kMinBlocksPerWorkerForPool;   // COCKTAIL_MIN_POOL_BLOCKS  1..4096
  double pair_table[kNumClasses][kNumClasses];        // COCKTAIL_PAIR_TABLE="16 numbers, row = own class": replaces
  bool pair_table_set = false;                        // kPairSpeed, and switches the correction on for the matrix kernel too
  bool changed = false;                 // any of these is set to a value it takes: no split for short contexts, which knows none of them
};

static Tuning read_tuning() {
  Tuning t;
  for (int a = 0; a < kNumClasses; ++a)
    for (int b = 0; b < kNumClasses; ++b) t.pair_table[a][b] = kPairSpeed[a][b];
  // (one look for all of them: sixteen searches of the environment took 3 us of a short context's 11)
  bool any = false;
  for (char** e = environ; e && *e; ++e)
    if (std::strncmp(*e, "COCKTAIL_", 9) == 0)
      for (const char* name : {"COST_WEIGHTS=", "POOL_PERCENT=", "GROUP_WORKERS=", "PAIR_SPEED=", "LAYOUT=", "PAIR_MODE=", "MIN_POOL_BLOCKS=", "PAIR_TABLE="})
        any = any || std::strncmp(*e + 9, name, std::strlen(name)) == 0;
  if (!any) return t;
  if (const char* e = std::getenv("COCKTAIL_COST_WEIGHTS")) {
    long a = 0, b = 0, c = 0, d = 0;
    const int n = std::sscanf(e, "%ld,%ld,%ld,%ld", &a, &b, &c, &d);
    if (n == 4 && a > 0 && b > 0 && c > 0 && d > 0)
      t.weight[0] = a, t.weight[1] = b, t.weight[2] = c, t.weight[3] = d, t.weight_set = true;
    else if (n == 3 && a > 0 && b > 0 && c > 0)
      t.weight[0] = a, t.weight[1] = b, t.weight[3] = c, t.weight_set = true;
    t.changed = t.weight_set;
  }
  auto int_knob = [&](const char* name, int lo, int hi, int& out) {
    if (const char* e = std::getenv(name)) {
      const int v = std::atoi(e);
      if (v >= lo && v <= hi) out = v, t.changed = true;
    }
  };
  if (const char* e = std::getenv("COCKTAIL_PAIR_TABLE")) {
    double v[16];
    int n = 0;
    const char* q = e;
    while (n < 16) {
      char* end = nullptr;
      const double x = std::strtod(q, &end);
      if (end == q) break;
      v[n++] = x;
      q = end;
      while (*q == ',' || *q == ' ') ++q;
    }
    bool ok = n == 16;
    for (int i = 0; ok && i < 16; ++i) ok = v[i] > 0.25 && v[i] < 4.0;
    if (ok) {
      for (int i = 0; i < 16; ++i) t.pair_table[i / 4][i % 4] = v[i];
      t.pair_table_set = t.changed = true;
    }
  }
  int ps = 1;
  int_knob("COCKTAIL_POOL_PERCENT", 0, 100, t.pool_percent);
  t.pool_percent_set = std::getenv("COCKTAIL_POOL_PERCENT") != nullptr;
  int_knob("COCKTAIL_GROUP_WORKERS", 1, 1024, t.group_workers);
  int_knob("COCKTAIL_PAIR_SPEED", 0, 1, ps);
  int_knob("COCKTAIL_LAYOUT", 0, 1, t.layout);
  int_knob("COCKTAIL_PAIR_MODE", 0, 3, t.pair_mode);
  int_knob("COCKTAIL_MIN_POOL_BLOCKS", 1, 4096, t.min_pool_blocks);
  t.pair_speed = ps != 0;
  return t;
}

// Ranges that end where runs end.  `nblk` [kNumClasses][B] as [NC * b + c]: blocks of a run, the same for all `heads` heads; cost[c]: of a
// block; `most_int2`: workers INT2 may have (kInt2Stretch); `longest_range`: kLongestRange; `too_long`: whether it
// is exceeded, which `any_length` allows.  Finds the smallest cost a worker may be given such that `slots` workers are enough, cuts every run into equal parts of at most
// that, and lets workers that are left over (beyond 1 in 40: they would bring nothing) cut the dearest parts once more.  Returns the first block of every worker's range
// in class, sequence, head order (slots + 1 entries), or nothing if there are more runs than workers or the longest range is too long
// (kLongestRange).
static std::vector<int32_t> aligned_ranges(const std::vector<int32_t>& nblk, int B, int heads, int slots, const double (&cost)[kNumClasses],
                                           int units_per_block, int64_t most_int2, double longest_range,
                                           bool any_length, bool* too_long) {
  constexpr int NC = kNumClasses;
  int64_t int2_range = 0;   // blocks of a range of INT2, if not by cost
  auto per_worker = [&](int c, double budget) {
    if (c == 0 && int2_range) return int2_range;
    int64_t n = static_cast<int64_t>(budget / cost[c]);
    const int whole = std::max(1, kIterUnits[c] / units_per_block);
    if (n < kWholeIterationBlocks) n = n / whole * whole;
    return std::max<int64_t>(n, 1);
  };
  auto parts_of = [&](int c, int64_t per) {
    int64_t n = 0;
    for (int b = 0; b < B; ++b) n += (nblk[NC * b + c] + per - 1) / per;
    return n * heads;
  };
  auto workers_for = [&](double budget) {
    int64_t n = 0;
    for (int c = 0; c < NC; ++c) n += parts_of(c, per_worker(c, budget));
    return n;
  };
  double total = 0;
  for (int b = 0; b < B; ++b)
    for (int c = 0; c < NC; ++c) total += cost[c] * heads * nblk[NC * b + c];
  std::vector<int32_t> bound;
  if (total == 0 || workers_for(2 * total) > slots) return bound;
  auto smallest_budget = [&] {
    double lo = 0, hi = total / slots;
    while (workers_for(hi) > slots) lo = hi, hi *= 2;
    for (int i = 0; i < 20; ++i) {
      const double mid = 0.5 * (lo + hi);
      (workers_for(mid) <= slots ? hi : lo) = mid;
    }
    return hi;
  };
  double hi = smallest_budget();
  if (most_int2 < slots && parts_of(0, per_worker(0, hi)) > most_int2) {
    const int whole = std::max(1, kIterUnits[0] / units_per_block);
    int64_t per = per_worker(0, hi);
    while (per * cost[0] <= kInt2Stretch * hi && parts_of(0, per) > most_int2) per += per < kWholeIterationBlocks ? whole : 1;
    if (per * cost[0] <= kInt2Stretch * hi) int2_range = per, hi = smallest_budget();
  }
  std::vector<int32_t> parts(NC * B), extra(NC * B, 0);   // parts per run; in addition one more for the first `extra` heads
  int64_t left = slots - slots / 40;
  for (int c = 0; c < NC; ++c) {
    const int64_t per = per_worker(c, hi);
    for (int b = 0; b < B; ++b) {
      parts[NC * b + c] = static_cast<int32_t>((nblk[NC * b + c] + per - 1) / per);
      left -= int64_t(heads) * parts[NC * b + c];
    }
  }
  std::priority_queue<std::pair<double, int>> dearest;   // cost of the largest part, run
  auto offer = [&](int i) {
    if (parts[i] > 0 && parts[i] < nblk[i] && !(i % NC == 0 && int2_range)) dearest.push({(nblk[i] + parts[i] - 1) / parts[i] * cost[i % NC], i});
  };
  if (left > 0)
    for (int i = 0; i < NC * B; ++i) offer(i);
  while (left > 0 && !dearest.empty()) {
    const int i = dearest.top().second;
    dearest.pop();
    if (left < heads) extra[i] = static_cast<int32_t>(left);
    else ++parts[i], offer(i);
    left -= heads;
  }
  double longest = 0, dearest_block = 0;
  for (int i = 0; i < NC * B; ++i)
    if (parts[i] > 0) {
      longest = std::max(longest, (nblk[i] + parts[i] - 1) / parts[i] * cost[i % NC]);
      dearest_block = std::max(dearest_block, cost[i % NC]);
    }
  if (longest > longest_range * total / slots + kLongestRangeBlocks * dearest_block) {
    if (too_long) *too_long = true;
    if (!any_length) return bound;
  }
  bound.reserve(slots + 1);
  int32_t at = 0;
  for (int c = 0; c < NC; ++c)
    for (int b = 0; b < B; ++b)
      for (int h = 0; h < heads; ++h) {
        const int i = NC * b + c, m = parts[i] + (h < extra[i]);
        for (int k = 0; k < m; ++k) bound.push_back(at), at += nblk[i] / m + (k < nblk[i] % m);
      }
  bound.resize(slots + 1, at);   // the rest has no work
  return bound;
}

// The split for short contexts (decode_short_impl.h).  Every row gets as many workgroups as it takes for no wave to have more than some number of loop
// iterations, the smallest for which the chip's workgroups are enough; a run is cut into equal parts, one per wave.
struct ShortSplit {
  struct Run {
    int cls, units, step, iters, parts;   // step: units a range is a multiple of
  };
  struct Sequence {
    Run runs[kNumClasses + 1];            // the last one: appended tokens
    int n = 0, groups = 0;                // runs, workgroups of a row
  };
  std::vector<Sequence> sequences;
  int groups = 0, rows = 0;               // 0: no such split
  bool one = false;                       // an iteration is one unit (or staged block)
  bool shared = false;                    // some row has several workgroups
};
static ShortSplit short_split(const std::vector<int32_t>& ntok, int B, int heads, int head_dim, int append_capacity, int rep, int share, bool one,
                              int most_groups) {
  constexpr int NC = kNumClasses, W = kCuWaves;
  const bool tiles = uses_tiles(rep);   // which stage whole blocks of INT2 and INT4
  const int most_iterations = tiles ? share > 1 ? kShortUnitsSets : head_dim == 64 ? kShortUnitsTilesD64 : kShortUnitsTiles : one ? kShortUnits : kShortIterations;
  const int units_per_block = head_dim == 64 ? 1 : 2, unit_tokens = kTB / units_per_block;
  ShortSplit s;
  const int64_t rows = int64_t(B) * heads;
  if (rows > most_groups) return s;
  s.sequences.resize(B);
  for (int b = 0; b < B; ++b) {
    ShortSplit::Sequence& q = s.sequences[b];
    for (int cls = 0; cls <= NC; ++cls) {
      const int64_t tokens = cls == NC ? append_capacity : ntok[NC * b + cls];
      if (tokens <= 0) continue;
      const int c = std::min(cls, kFp16Class), step = tiles && c < 2 ? units_per_block : 1, iteration = one ? step : kIterUnits[c];
      const int64_t units = (tokens + unit_tokens * step - 1) / (unit_tokens * step) * step;
      if (units > 0xffff && cls < NC) return s;   // (units are 16-bit fields)
      q.runs[q.n++] = {cls, int(units), step, int((units + iteration - 1) / iteration), 0};
    }
  }
  auto waves_for = [&](int b, int most) {
    const ShortSplit::Sequence& q = s.sequences[b];
    int64_t n = 0;
    for (int i = 0; i < q.n; ++i) n += (q.runs[i].iters + most - 1) / most;
    return n;
  };
  const int64_t most_of_row = kShortStates / rep / W * W;
  auto groups_for = [&](int most, bool limit) {
    int64_t n = 0;
    for (int b = 0; b < B; ++b) {
      const int64_t row = std::max<int64_t>((waves_for(b, most) + W - 1) / W, 1);
      n += limit && row > most_of_row ? most_groups + 1 : row * heads;
    }
    return n;
  };
  if (groups_for(most_iterations, true) > most_groups) return s;
  auto fewest = [&](bool limit) {
    int lo = 0, hi = most_iterations;
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      (groups_for(mid, limit) <= most_groups ? hi : lo) = mid;
    }
    return hi;
  };
  int hi = fewest(true);
  // few rows: too many workgroups of one for a merge in shared memory, and those it may have leave a part of the chip idle
  if (hi > fewest(false) + (tiles ? 0 : 1)) return s;
  // rows that one workgroup finishes need no second merge
  int whole = 1;
  while (whole <= hi + kShortMergeIterations && whole <= most_iterations && groups_for(whole, true) > rows) ++whole;
  if (whole <= hi + kShortMergeIterations && whole <= most_iterations) hi = whole;
  if (share > 1 && tiles && head_dim == 128 && hi > 1 && append_capacity == 0 && groups_for(hi, true) < most_groups)
    for (int b = 0; b < B; ++b)
      if (waves_for(b, hi) > int64_t(kShortGroupsSets) * W) return s;
  s.one = one, s.groups = int(groups_for(hi, true)), s.rows = int(rows);
  for (int b = 0; b < B; ++b) {
    ShortSplit::Sequence& q = s.sequences[b];
    q.groups = int(std::max<int64_t>((waves_for(b, hi) + W - 1) / W, 1));
    s.shared = s.shared || q.groups > 1;
    int left = q.groups * W;
    for (int i = 0; i < q.n; ++i) q.runs[i].parts = (q.runs[i].iters + hi - 1) / hi, left -= q.runs[i].parts;
    // spare waves go to the run whose ranges are longest
    for (; left > 0; --left) {
      int best = -1;
      for (int i = 0; i < q.n; ++i) {
        const ShortSplit::Run &r = q.runs[i], *p = best < 0 ? nullptr : &q.runs[best];
        if (r.iters > r.parts && (!p || int64_t(r.iters) * p->parts > int64_t(p->iters) * r.parts)) best = i;
      }
      if (best < 0) break;
      ++q.runs[best].parts;
    }
  }
  return s;
}

// Its records (by copies, as everything in the blob: the caller's buffer need not be aligned).
static void write_short_split(const ShortSplit& s, const std::vector<int32_t>& ntok, const std::vector<int32_t>& blk_base, const std::vector<int32_t>& cap,
                              const int32_t* seq_lens, int heads, int share, int rep, int append_blocks, char* recs, char* place) {
  constexpr int NC = kNumClasses, W = kCuWaves;
  for (int b = 0; b < int(s.sequences.size()); ++b) {
    const ShortSplit::Sequence& q = s.sequences[b];
    for (int h = 0; h < heads; ++h, recs += sizeof(ShortRec) * W * q.groups) {
      for (int g = 0; g < q.groups; ++g, place += sizeof(ShortGroup)) {
        const ShortGroup p = {b, (b * heads + h) * rep, seq_lens[b], uint32_t(g) | uint32_t(q.groups) << 8 | uint32_t(b * heads + h) << 20};
        std::memcpy(place, &p, sizeof(p));
      }
      if (h > 0) {   // the same ranges of the next head's runs
        const size_t bytes = sizeof(ShortRec) * W * q.groups;
        std::memcpy(recs, recs - bytes, bytes);
        if (h % share == 0)
          for (int i = 0; i < q.groups * W; ++i) {
            ShortRec r;
            std::memcpy(&r, recs + i * sizeof(r), sizeof(r));
            r.blk0 += r.cls == NC ? append_blocks : cap[NC * b + r.cls];
            std::memcpy(recs + i * sizeof(r), &r, sizeof(r));
          }
        continue;
      }
      // range after range, each on another workgroup: the waves of one work on all classes, and SIMD mates (four waves apart) on different ones
      int g = 0, w = 0;
      auto put = [&](const ShortRec& r) {
        std::memcpy(recs + (g * W + w) * sizeof(r), &r, sizeof(r));
        if (++g == q.groups) g = 0, ++w;
      };
      for (int i = 0; i < q.n; ++i) {
        const ShortSplit::Run& r = q.runs[i];
        if (r.cls == NC) {
          const int32_t inverse = int32_t((uint64_t(1) << 32) / r.parts + 1), blk0 = b * (heads / share) * append_blocks;
          for (int k = 0; k < r.parts; ++k) put({r.cls, uint32_t(k) | uint32_t(r.parts) << 16, inverse, blk0});
          continue;
        }
        const int each = r.units / r.step / r.parts, more = r.units / r.step % r.parts;   // (the first `more` ranges have one more)
        const int32_t tokens = ntok[NC * b + r.cls], blk0 = blk_base[NC * b + r.cls];
        uint32_t at = 0;
        for (int k = 0; k < r.parts; ++k) {
          const uint32_t end = at + (each + (k < more)) * r.step;
          put({r.cls, at | end << 16, tokens, blk0});
          at = end;
        }
      }
      while (w < W) put({0, 0, 0, 0});   // no work
    }
  }
}

static inline int64_t align16(int64_t x) { return (x + 15) & ~int64_t(15); }

}  // namespace cocktail

using namespace cocktail;

extern "C" const char* cocktail_last_error(void) { return g_err; }
extern "C" int cocktail_version(void) { return (0 << 16) | 5; }

// Reads one field of the plan header by name, so that tools and tests that look inside a plan follow the
// header's real layout instead of a copy of it.
extern "C" int cocktail_plan_field(const void* plan_host, const char* name, int32_t index, int64_t* value) {
  if (!plan_host || !name || !value) return fail(COCKTAIL_EINVAL, "plan_host, name and value must not be NULL");
  const PlanHeader* hd = static_cast<const PlanHeader*>(plan_host);
  if (hd->magic != kPlanMagic || !known_version(hd->version))
    return fail(COCKTAIL_EINVAL, "plan_host is not a plan written by this library version");
#define COCKTAIL_FIELD(f)                                                                            \
  if (std::strcmp(name, #f) == 0) {                                                                  \
    if (index != 0) return fail(COCKTAIL_EINVAL, "plan field %s is not an array", name);             \
    *value = static_cast<int64_t>(hd->f);                                                            \
    return COCKTAIL_OK;                                                                              \
  }
#define COCKTAIL_ARRAY(f)                                                                            \
  if (std::strcmp(name, #f) == 0) {                                                                  \
    if (index < 0 || index >= kNumClasses) return fail(COCKTAIL_EINVAL, "index %d of plan field %s", index, name); \
    *value = static_cast<int64_t>(hd->f[index]);                                                     \
    return COCKTAIL_OK;                                                                              \
  }
  COCKTAIL_FIELD(magic) COCKTAIL_FIELD(version) COCKTAIL_FIELD(batch) COCKTAIL_FIELD(num_q_heads)
  COCKTAIL_FIELD(num_kv_heads) COCKTAIL_FIELD(head_dim) COCKTAIL_FIELD(chunk_size) COCKTAIL_FIELD(group_size)
  COCKTAIL_FIELD(rep) COCKTAIL_FIELD(work_heads) COCKTAIL_FIELD(work_rep) COCKTAIL_FIELD(num_workers) COCKTAIL_FIELD(num_segments) COCKTAIL_FIELD(num_partials)
  COCKTAIL_FIELD(total_gblocks) COCKTAIL_FIELD(v_layout) COCKTAIL_FIELD(total_chunks) COCKTAIL_FIELD(total_tokens)
  COCKTAIL_ARRAY(class_blocks) COCKTAIL_ARRAY(class_bytes) COCKTAIL_ARRAY(block_bytes) COCKTAIL_ARRAY(row_bytes)
  COCKTAIL_FIELD(workspace_bytes) COCKTAIL_FIELD(plan_bytes) COCKTAIL_FIELD(packed_bytes)
  COCKTAIL_FIELD(off_seq_len) COCKTAIL_FIELD(off_cum_tokens) COCKTAIL_FIELD(off_chunk_off) COCKTAIL_FIELD(off_perm)
  COCKTAIL_FIELD(off_class_tokens) COCKTAIL_FIELD(off_class_chunk0) COCKTAIL_FIELD(off_blk_base)
  COCKTAIL_FIELD(off_nblk) COCKTAIL_FIELD(off_run_blocks) COCKTAIL_FIELD(off_segments) COCKTAIL_FIELD(append_capacity)
  COCKTAIL_FIELD(off_worker_rec) COCKTAIL_FIELD(off_group_rec) COCKTAIL_FIELD(off_pool_seg)
  COCKTAIL_FIELD(off_counters) COCKTAIL_FIELD(num_groups) COCKTAIL_FIELD(num_pool_segs)
  COCKTAIL_FIELD(append_blocks) COCKTAIL_FIELD(append_slices) COCKTAIL_FIELD(off_bh_off) COCKTAIL_FIELD(off_rq_items)
  COCKTAIL_FIELD(ws_status_off) COCKTAIL_FIELD(short_groups) COCKTAIL_FIELD(short_units) COCKTAIL_FIELD(off_short)
#undef COCKTAIL_FIELD
#undef COCKTAIL_ARRAY
  // constants of the layout that are not stored in the header
  if (std::strcmp(name, "counter_stride_bytes") == 0) return *value = 4 * counter_stride(hd->num_pool_segs), COCKTAIL_OK;
  if (std::strcmp(name, "partial_header_floats") == 0) return *value = kPartialFloats, COCKTAIL_OK;
  if (std::strcmp(name, "iter_units") == 0 && index >= 0 && index < kNumClasses) return *value = kIterUnits[index], COCKTAIL_OK;
  if (std::strcmp(name, "workgroup_waves") == 0) return *value = workgroup_waves(hd->num_workers, hd->append_slices), COCKTAIL_OK;
  if (std::strcmp(name, "sizeof_segment") == 0) return *value = sizeof(Segment), COCKTAIL_OK;
  if (std::strcmp(name, "sizeof_worker_rec") == 0) return *value = sizeof(WorkerRec), COCKTAIL_OK;
  if (std::strcmp(name, "sizeof_group_rec") == 0) return *value = sizeof(GroupRec), COCKTAIL_OK;
  if (std::strcmp(name, "sizeof_pool_seg") == 0) return *value = sizeof(PoolSeg), COCKTAIL_OK;
  if (hd->short_groups > 0 && std::strcmp(name, "off_short_place") == 0) return *value = short_group_offset(*hd), COCKTAIL_OK;
  if (hd->short_groups > 0 && std::strcmp(name, "off_short_counters") == 0) return *value = short_counters_offset(*hd), COCKTAIL_OK;
  if (std::strcmp(name, "short_counter_stride_bytes") == 0) return *value = 4 * kShortCounterStride, COCKTAIL_OK;
  if (std::strcmp(name, "sizeof_rq_item") == 0) return *value = sizeof(RQItem), COCKTAIL_OK;
  return fail(COCKTAIL_EINVAL, "unknown plan field %s[%d]", name, index);
}

extern "C" int cocktail_plan(const cocktail_shape* shape, const int32_t* seq_lens, const uint8_t* chunk_bits,
                             int32_t num_workers, cocktail_sizes* sizes, void* plan_host, size_t plan_capacity,
                             int32_t* class_tokens, int32_t* perm) {
  return cocktail_plan_ex(shape, seq_lens, chunk_bits, num_workers, nullptr, sizes, plan_host, plan_capacity,
                          class_tokens, perm);
}

// cocktail_plan_ex with one of the two splits of the work where the longest range would be too long (kLongestRange); says in `too_long`
// whether it would.
static int make_plan(const cocktail_shape* shape, const int32_t* seq_lens, const uint8_t* chunk_bits, int32_t num_workers,
                     const cocktail_plan_options* options, cocktail_sizes* sizes, void* plan_host, size_t plan_capacity,
                     int32_t* class_tokens, int32_t* perm, bool any_length, bool* too_long) {
  if (int rc = check_shape(shape)) return rc;
  const int32_t append_capacity = options ? options->append_capacity : 0;
  const bool reproducible = options && options->reproducible != 0;
  const bool vector_alu_only = options && options->vector_alu_only != 0;
  const int32_t* max_seq_lens = options ? options->max_seq_lens : nullptr;
  if (options) {
    if (options->reserved0 != 0) return fail(COCKTAIL_EINVAL, "cocktail_plan_options::reserved must be zero");
    for (int32_t v : options->reserved)
      if (v != 0) return fail(COCKTAIL_EINVAL, "cocktail_plan_options::reserved must be zero");
  }
  if (append_capacity < 0 || append_capacity > (1 << 24) - kTB)   // an append run stays below 4 GiB, like a context run
    return fail(COCKTAIL_EINVAL, "append_capacity %d out of range [0, 2^24 - 64]", append_capacity);
  if (!seq_lens || !sizes) return fail(COCKTAIL_EINVAL, "seq_lens and sizes must not be NULL");
  if (num_workers < 1 || num_workers > (1 << 20))
    return fail(COCKTAIL_EINVAL, "num_workers %d out of range [1, 2^20]", num_workers);
  const int B = shape->batch, Hkv = shape->num_kv_heads, D = shape->head_dim, C = shape->chunk_size,
            G = shape->group_size;
  // a wave handles 64 tokens at a time at head_dim 64 and 32 at head_dim 128 (a lane works on 64 channels):
  // the units the pool tickets count in
  const int units_per_block = D == 64 ? 1 : 2;

  int64_t total_chunks = 0, total_tokens = 0;
  for (int b = 0; b < B; ++b) {
    if (seq_lens[b] < 0) return fail(COCKTAIL_EINVAL, "seq_lens[%d] = %d is negative", b, seq_lens[b]);
    if (max_seq_lens && max_seq_lens[b] < seq_lens[b])
      return fail(COCKTAIL_EINVAL, "max_seq_lens[%d] = %d is below seq_lens[%d] = %d", b, max_seq_lens[b], b, seq_lens[b]);
    // the kernels address the blocks of one (b, h, class) run with 32-bit byte offsets and describe it by a
    // buffer resource with a 32-bit size: an all-FP16 run of T tokens has ceil(T / 64) * 64 * 2 D bytes
    const int32_t longest = max_seq_lens ? max_seq_lens[b] : seq_lens[b];   // what the sequence may grow to
    if ((int64_t(longest) + kTB - 1) / kTB * kTB * 2 * D >= (int64_t(1) << 32))
      return fail(COCKTAIL_EUNSUPPORTED, "sequence %d with %d tokens: one (sequence, kv head) run in FP16 would reach 4 GiB "
                  "(at most %lld tokens per sequence at head_dim %d)", b, longest,
                  (long long)(((int64_t(1) << 32) / (2 * D) - 1) / kTB * kTB), D);
    total_chunks += seq_lens[b] / C;
    total_tokens += seq_lens[b];
  }
  if (total_chunks > 0 && !chunk_bits) return fail(COCKTAIL_EINVAL, "chunk_bits is NULL");
  if (total_tokens >= (int64_t(1) << 31)) return fail(COCKTAIL_EINVAL, "more than 2^31 tokens in one call");
  for (int64_t i = 0; i < total_chunks; ++i) {
    const uint8_t v = chunk_bits[i];
    if (v != 2 && v != 4 && v != 8 && v != 16)
      return fail(COCKTAIL_EINVAL, "chunk_bits[%lld] = %d is not one of 2, 4, 8, 16", (long long)i, int(v));
  }

  constexpr int NC = kNumClasses;
  const int* bits_of = kClassBits;
  int32_t row_bytes[NC], block_bytes[NC], algo_row[NC];
  for (int c = 0; c < NC; ++c) {
    const int meta = (c == kFp16Class) ? 0 : 4 * (D / G);
    row_bytes[c] = D * bits_of[c] / 8;
    block_bytes[c] = kTB * (row_bytes[c] + meta);
    algo_row[c] = row_bytes[c] + meta;
  }

  // ---- Alg. 1 prefill loop: class lists in loop order, concatenated INT2 | INT4 | INT8 | FP16 ----
  // v_nblk: blocks per head that hold tokens; v_cap: blocks per head the run is laid out with (more than v_nblk
  // only for FP16 runs with room to grow, cocktail_plan_options::max_seq_lens)
  std::vector<int32_t> v_perm(total_chunks), v_chunk_off(B + 1, 0), v_ct(NC * B), v_cc0(NC * B), v_nblk(NC * B),
      v_cap(NC * B), v_blk_base(NC * (B + 1), 0);
  std::vector<int64_t> v_cum(B + 1, 0);
  int64_t class_tokens_tot[NC] = {};
  int64_t packed = 0;
  for (int b = 0; b < B; ++b) {
    const int n = seq_lens[b] / C;
    const uint8_t* bits = chunk_bits ? chunk_bits + v_chunk_off[b] : nullptr;
    int32_t* pb = v_perm.data() + v_chunk_off[b];
    int pos = 0;
    for (int c = 0; c < NC; ++c) {
      v_cc0[NC * b + c] = pos;
      for (int i = 0; i < n; ++i)
        if (bits[i] == bits_of[c]) pb[pos++] = i;
      int64_t ntok = int64_t(pos - v_cc0[NC * b + c]) * C;
      if (c == kFp16Class) ntok += seq_lens[b] - n * C;  // Sec. III-A: the remainder stays FP16
      v_ct[NC * b + c] = static_cast<int32_t>(ntok);
      v_nblk[NC * b + c] = static_cast<int32_t>((ntok + kTB - 1) / kTB);
      const int64_t room = (c == kFp16Class && max_seq_lens) ? int64_t(max_seq_lens[b]) - seq_lens[b] : 0;
      v_cap[NC * b + c] = static_cast<int32_t>((ntok + room + kTB - 1) / kTB);
      class_tokens_tot[c] += ntok;
      packed += 2 * int64_t(Hkv) * ntok * algo_row[c];
      const int64_t nb = int64_t(v_blk_base[NC * b + c]) + int64_t(Hkv) * v_cap[NC * b + c];
      if (nb >= (int64_t(1) << 31)) return fail(COCKTAIL_EINVAL, "class %d needs more than 2^31 blocks", c);
      v_blk_base[NC * (b + 1) + c] = static_cast<int32_t>(nb);
    }
    v_chunk_off[b + 1] = v_chunk_off[b] + n;
    v_cum[b + 1] = v_cum[b] + seq_lens[b];
  }

  // Relative time per byte of the three classes in the decode kernel (1/64 units).  The FP16 class is
  // a pure stream; the quantised classes also keep the vector ALU busy, so a byte of them takes longer.
  // Measured on MI355X with all three classes running side by side.
  Tuning tune = read_tuning();
  int pool_percent = tune.pool_percent;
  const int rep = shape->num_q_heads / Hkv;
  // Waves of five to eight query heads keep the purely static split: their calls are reproducible bit for bit.
  // Up to eight query heads of a kv head are served by one wave.  Where more of them share a kv head they are
  // cut into equal sets, and with one wave per query head (the vector-ALU kernel, on request) every head is a set
  // of its own: each set walks the blocks of its kv head as if they were its own.
  const int wrep = work_rep_of(rep, vector_alu_only);   // query heads a wave serves
  const int Hw = shape->num_q_heads / wrep;             // heads of the decode work split
  const int share = rep / wrep;                         // work heads that walk the blocks of one kv head
  const bool quads = uses_token_quads(wrep);
  if ((wrep > 1 && !(quads && !uses_tiles(wrep))) || reproducible) pool_percent = 0;

  // ---- physical runs of the class buffers: (class, b, h) order, each a contiguous run of blocks ----
  struct Run {
    int b, h, cls, nb, ntok, blk0;
  };
  std::vector<Run> runs;
  int64_t class_nblk[NC] = {};
  for (int c = 0; c < NC; ++c)
    for (int b = 0; b < B; ++b)
      for (int h = 0; h < Hw; ++h) {
        const int nb = v_nblk[NC * b + c];
        if (nb == 0) continue;
        runs.push_back({b, h, c, nb, v_ct[NC * b + c], v_blk_base[NC * b + c] + (h / share) * v_cap[NC * b + c]});
        class_nblk[c] += nb;
      }
  int64_t tot_blocks = 0;
  for (int c = 0; c < NC; ++c) tot_blocks += class_nblk[c];
  if (tot_blocks >= (int64_t(1) << 31)) return fail(COCKTAIL_EINVAL, "more than 2^31 blocks in one call");
  // `num_workers` is an upper bound: a short context has fewer units of work than the chip has wave slots, and
  // waves without work only lengthen the launch (8 heads x 2048 tokens on MI355X: 12.4 us per call with 2048
  // of them, 11.5 us with 512).  At most one worker per unit, in multiples of 64.
  const int64_t unit_workers = (tot_blocks * units_per_block + 63) / 64 * 64;
  const int P = static_cast<int>(std::min<int64_t>(num_workers, std::max<int64_t>(unit_workers, 64)));
  const int group_workers = tune.group_workers > 0 ? tune.group_workers
                            : quads                ? kQuadGroupWorkers
                            : tot_blocks >= int64_t(kLongRangeBlocks) * P ? kGroupWorkers : kGroupWorkersShort;
  // Where a kv head has several sets of query heads (ratios above eight on the matrix kernels), each set walks the same
  // blocks.  `sets` consecutive groups take the same stripe of blocks, one set each, worker by worker, and the workers
  // of a stripe get worker ids that differ by multiples of kXcds: they run on one XCD, start together, and all but the first find
  // the blocks in its L2.  (In run order the sets lay half a class apart and every byte was fetched once per set:
  // 8 ragged contexts up to 64K, 64 q / 4 kv heads, 61 -> 52 us per call;
  // 4 x 128K, 128 q / 8 kv heads, 235 -> 167.)  Workers beyond whole units of kXcds * share stay without work: taken where
  // they are at most 1/32 of all.
  const int unit = kXcds * share;
  const bool twins = quads && share > 1 && !tune.layout && tune.pair_mode < 2 && kXcds % group_workers == 0 &&
                     P >= unit && int64_t(P % unit) * 32 <= P;
  const int sets = twins ? share : 1;
  if (quads && !tune.weight_set)   // (sets that are not twins fetch their blocks from memory each)
    for (int c = 0; c < NC; ++c)
      tune.weight[c] = !uses_tiles(wrep) ? kQuadCostWeight[c] : twins ? kTwinCostWeight[c] : kTileCostWeight[c];
  const int64_t* weight = tune.weight;

  // ---- global order and segments ----
  // The workers form groups of `group_workers`; group j works on one stripe [cut[c][j], cut[c][j+1]) of
  // the blocks of every class c (blocks in (b, h, block) order).  A segment is the intersection of a
  // stripe with a run; the global order lists the groups one after the other.
  //   layout 0: the class-major order INT2 | INT4 | INT8 | FP16 is cut into NGR parts of equal cost, so a
  //             group works on one class (two where it straddles a class boundary);
  //   layout 1: every group receives the same share of every class (FP16 stripe, then INT2, INT4, INT8).
  const int NGR = (P + group_workers - 1) / group_workers, NST = twins ? P / unit * (kXcds / group_workers) : NGR;   // groups, stripes
  if (twins)
    for (int c = 0; c < NC; ++c) class_nblk[c] /= sets;   // blocks of one set
  const bool pair_speed_on = tune.pair_speed;
  const int layout = tune.layout;
  const int class_order[NC] = {layout ? 3 : 0, layout ? 0 : 1, layout ? 1 : 2, layout ? 2 : 3};
  std::vector<int64_t> cut[NC];
  std::vector<int32_t> bound;   // aligned ranges of one set's workers
  const bool tiles = quads && uses_tiles(wrep);
  const int slots = twins ? NST * group_workers : P;
  const int aligned_blocks = P < kChipWorkers ? kAlignedBlocks : quads ? kAlignedBlocksQuads : kAlignedBlocksHeads;
  if (!layout && !tune.pair_table_set && (tiles || (!tune.pool_percent_set && tot_blocks <= int64_t(aligned_blocks) * P))) {
    double block_cost[NC];
    for (int c = 0; c < NC; ++c) block_cost[c] = double(block_bytes[c]) * double(weight[c]);
    const bool mates = workgroup_waves(P, append_capacity) > 1;   // SIMD mates are known
    bound = aligned_ranges(v_nblk, B, Hw / sets, slots, block_cost, units_per_block, mates ? kSimds / sets : slots,
                           tiles ? kLongestRangeTiles : kLongestRange, any_length, too_long);
    if (!bound.empty() && wrep == 1 && mates && runs.size() <= kFewRuns && tot_blocks > int64_t(kAlignedBlocks) * P) {
      const int64_t int2_workers = std::lower_bound(bound.begin(), bound.end(), class_nblk[0]) - bound.begin();
      if (int2_workers > kSimds && int2_workers < kFewInt2Pairs * kSimds) bound.clear();
    }
    if (!bound.empty()) pool_percent = 0;
  }
  {
    int64_t per[NC], tot = 0, start[NC];
    for (int c = 0; c < NC; ++c) {
      per[c] = 2 * int64_t(block_bytes[c]) * weight[c];
      start[c] = tot;
      tot += class_nblk[c] * per[c];
      cut[c].assign(NGR + 1, 0);
    }
    if (!bound.empty()) {
      for (int j = 0; j <= NST; ++j) {
        int64_t at = bound[std::min(j * group_workers, slots)];
        for (int c = 0; c < NC; ++c) cut[c][j] = std::min(std::max<int64_t>(at, 0), class_nblk[c]), at -= class_nblk[c];
      }
    } else {
      // Share of the total cost in front of every group.  Equal shares per worker to begin with; then,
      // if the workers fill the chip with two waves per SIMD (worker i and i + P/2 share a SIMD), a few rounds that
      // scale every worker's share by the measured relative speed of its class next to its mate's class.
      std::vector<double> wcap(P, 1.0), gfrac(NGR + 1, 0.0);
      const bool pair_speed = pair_speed_on && !layout && P % 2 == 0 && P >= 2 * group_workers &&
                              (wrep == 1 || (tune.pair_table_set && quads && !twins));
      for (int round = 0; round < (pair_speed ? 4 : 1); ++round) {
        double total_cap = 0.0;
        for (int w = 0; w < P; ++w) total_cap += wcap[w];
        double acc = 0.0;
        for (int j = 0; j < NGR; ++j) {
          gfrac[j] = acc / total_cap;
          for (int w = j * group_workers; w < P && w < (j + 1) * group_workers; ++w) acc += wcap[w];
        }
        gfrac[NGR] = 1.0;
        if (twins)
          for (int j = 0; j <= NST; ++j) gfrac[j] = double(j) / NST;
        if (!pair_speed || round == 3) break;
        std::vector<int> wclass(P);
        for (int w = 0; w < P; ++w) {
          const int j = w / group_workers, k = (j + 1) * group_workers <= P ? group_workers : P - j * group_workers;
          const double x = double(tot) * (gfrac[j] + (w - j * group_workers + 0.5) / k * (gfrac[j + 1] - gfrac[j]));
          wclass[w] = x < double(start[1]) ? 0 : x < double(start[2]) ? 1 : x < double(start[3]) ? 2 : 3;
        }
        for (int w = 0; w < P; ++w) wcap[w] = tune.pair_table[wclass[w]][wclass[(w + P / 2) % P]];
      }
      for (int j = 0; j <= NST; ++j) {
        for (int c = 0; c < NC; ++c) {
          if (layout) {
            const int w_lo = j * group_workers < P ? j * group_workers : P;
            cut[c][j] = class_nblk[c] * w_lo / P;
          } else {
            const int64_t target = static_cast<int64_t>(double(tot) * gfrac[j]);
            int64_t v = (target - start[c] + per[c] / 2) / per[c];
            cut[c][j] = v < 0 ? 0 : (v > class_nblk[c] ? class_nblk[c] : v);
          }
        }
      }
    }
    for (int c = 0; c < NC; ++c) cut[c][0] = 0, cut[c][NST] = class_nblk[c];
  }
  std::vector<Segment> segs;
  std::vector<int64_t> seg_cost0;   // cumulative cost (weighted bytes of K+V) at the start of each segment
  std::vector<int32_t> group_g0(NGR + 1, 0), group_s0(NGR + 1, 0);
  segs.reserve(runs.size() + NC * NGR), seg_cost0.reserve(runs.size() + NC * NGR + 1);   // every cut ends a segment, and every run
  int64_t gblk = 0, cost = 0;
  {
    struct Walk {
      std::vector<Run> by_class[NC];
      size_t cur_run[NC] = {};      // run holding the next block of each class
      int64_t run_first[NC] = {};   // index of that run's first block among the set's blocks of the class
    };
    std::vector<Walk> walks(sets);
    for (const Run& r : runs) walks[r.h % sets].by_class[r.cls].push_back(r);
    for (int j = 0; j < NGR; ++j) {
      auto& [by_class, cur_run, run_first] = walks[j % sets];
      group_g0[j] = static_cast<int32_t>(gblk), group_s0[j] = static_cast<int32_t>(segs.size());
      for (int ci = 0; ci < NC; ++ci) {
        const int c = class_order[ci];
        int64_t lo = j < NST * sets ? cut[c][j / sets] : 0;
        const int64_t hi = j < NST * sets ? cut[c][j / sets + 1] : 0;
        while (lo < hi) {
          while (run_first[c] + by_class[c][cur_run[c]].nb <= lo) run_first[c] += by_class[c][cur_run[c]++].nb;
          const Run& r = by_class[c][cur_run[c]];
          const int off = static_cast<int>(lo - run_first[c]);
          const int n = static_cast<int>((hi < run_first[c] + r.nb ? hi : run_first[c] + r.nb) - lo);
          Segment sgm;
          sgm.b = r.b, sgm.h = r.h, sgm.cls = c, sgm.ntok = r.ntok - off * kTB;
          sgm.blk0 = r.blk0 + off, sgm.nblk = n;
          sgm.gblk0 = static_cast<int32_t>(gblk);
          sgm.pid0 = 0;
          segs.push_back(sgm);
          seg_cost0.push_back(cost);
          gblk += n;
          cost += int64_t(n) * 2 * block_bytes[c] * weight[c];
          lo += n;
        }
      }
    }
    group_g0[NGR] = static_cast<int32_t>(gblk), group_s0[NGR] = static_cast<int32_t>(segs.size());
  }
  seg_cost0.push_back(cost);
  const int S = static_cast<int>(segs.size());
  const int32_t g_end = static_cast<int32_t>(gblk);
  auto blk_cost = [&](int s) { return 2 * int64_t(block_bytes[segs[s].cls]) * weight[segs[s].cls]; };
  // cumulative cost in front of global block g, which lies in segment s (or g == end of segment s)
  auto cost_at = [&](int32_t g, int s) { return s >= S ? cost : seg_cost0[s] + int64_t(g - segs[s].gblk0) * blk_cost(s); };
  // block boundary whose cumulative cost is nearest to `target`; `s` is a monotone search cursor and
  // returns the segment that holds the boundary block (S at the very end)
  auto block_at = [&](int64_t target, int& s) -> int32_t {
    while (s < S && seg_cost0[s + 1] <= target) ++s;
    if (s >= S) return g_end;
    const int64_t per = blk_cost(s);
    int64_t j = (target - seg_cost0[s] + per / 2) / per;
    if (j < 0) j = 0;
    if (j >= segs[s].nblk) {
      j = 0;
      ++s;
      if (s >= S) return g_end;
    }
    return segs[s].gblk0 + static_cast<int32_t>(j);
  };
  auto seg_of = [&](int32_t g, int s) {   // segment holding block g, searching forward from s
    while (s < S && segs[s].gblk0 + segs[s].nblk <= g) ++s;
    return s;
  };

  // ---- groups of consecutive workers: an equal-cost range each; its tail becomes the shared pool,
  //      the rest is split into one own range per worker ----
  struct Item {
    int32_t g0, g1, seg0, pid0, group, rank;
  };
  std::vector<Item> items(P);
  std::vector<GroupRec> groups;
  std::vector<PoolSeg> psegs;
  {
    groups.reserve((P + group_workers - 1) / group_workers), psegs.reserve(2 * groups.capacity());
    for (int w0 = 0, j = 0; w0 < P; w0 += group_workers, ++j) {
      const int w1 = w0 + group_workers < P ? w0 + group_workers : P;
      const int k = w1 - w0;
      const int32_t G0 = group_g0[j], G1 = group_g0[j + 1];
      const int sG0 = group_s0[j], sG1 = group_s0[j + 1];
      GroupRec gr;
      std::memset(&gr, 0, sizeof(gr));
      gr.nworkers = k;
      gr.counter = static_cast<int32_t>(groups.size());
      gr.pseg0 = static_cast<int32_t>(psegs.size());
      if (!bound.empty()) {
        const int w = std::min(j / sets * group_workers, slots - k);
        int32_t prev = G0;
        int sprev = sG0;
        for (int r = 0; r < k; ++r) {
          const int32_t nb = r < k - 1 && j < NST * sets ? G0 + (bound[w + r + 1] - bound[w]) : G1;
          sprev = seg_of(prev, sprev);
          items[w0 + r] = {prev, nb, sprev, 0, gr.counter, r};
          prev = nb;
        }
        groups.push_back(gr);
        continue;
      }
      const int64_t c0 = cost_at(G0, sG0), c1 = cost_at(G1, sG1);
      int32_t Gp = G1;
      int sGp = sG1;
      if (pool_percent > 0 && int64_t(G1 - G0) >= int64_t(tune.min_pool_blocks) * k) {
        int sc = sG0;
        const int share = int64_t(G1 - G0) < int64_t(kShortRangeBlocks) * k && !tune.pool_percent_set
                              ? kShortRangePoolPercent : pool_percent;
        Gp = block_at(c1 - (c1 - c0) * share / 100, sc);
        sGp = sc;
        if (Gp < G0) Gp = G0, sGp = sG0;
        if (Gp > G1) Gp = G1, sGp = sG1;
        // a pool touches at most kMaxPoolSegments segments: move its start forward if it has to
        int first = seg_of(Gp, sGp);
        const int last = G1 > Gp ? seg_of(G1 - 1, first) : first;
        if (last - first + 1 > kMaxPoolSegments) {
          first = last - kMaxPoolSegments + 1;
          Gp = segs[first].gblk0, sGp = first;
        }
        int32_t gran = 0;
        for (int s = first; s < S && segs[s].gblk0 < G1 && Gp < G1; ++s) {
          const int32_t lo = Gp > segs[s].gblk0 ? Gp : segs[s].gblk0;
          const int32_t hi = G1 < segs[s].gblk0 + segs[s].nblk ? G1 : segs[s].gblk0 + segs[s].nblk;
          if (hi <= lo) continue;
          PoolSeg ps;
          std::memset(&ps, 0, sizeof(ps));
          ps.seg = s;
          ps.unit0 = units_per_block * (lo - segs[s].gblk0);
          ps.nunits = units_per_block * (hi - lo);
          ps.gran0 = gran;
          const int J = kIterUnits[segs[s].cls];
          gran += (ps.nunits + J - 1) / J;
          psegs.push_back(ps);
        }
        gr.ngran = gran;
        gr.nps = static_cast<int32_t>(psegs.size()) - gr.pseg0;
      }
      // own ranges: [G0, Gp) in k parts of equal cost
      const int64_t cp = cost_at(Gp, sGp);
      const int64_t own_q = (cp - c0) / k, own_r = (cp - c0) % k;
      int sc = sG0;
      int32_t prev = G0;
      int sprev = sG0;
      for (int r = 0; r < k; ++r) {
        int32_t nb;
        int snb;
        if (r == k - 1) {
          nb = Gp, snb = sGp;
        } else {
          nb = block_at(c0 + own_q * (r + 1) + int32_t(own_r) * (r + 1) / k, sc);   // c0 + (cp - c0) (r + 1) / k without 128-bit arithmetic
          snb = sc;
          if (nb > Gp) nb = Gp, snb = sGp;
          if (nb < prev) nb = prev, snb = sprev;
        }
        items[w0 + r] = {prev, nb, seg_of(prev, sprev), 0, gr.counter, r};
        prev = nb, sprev = snb;
      }
      groups.push_back(gr);
    }
  }
  const int NG = static_cast<int>(groups.size());
  const int NPS = static_cast<int>(psegs.size());

  // partial ids.  One per (worker, segment its own range touches) and one per (pool part, rank).  The
  // ids of a (b, kv head) are contiguous, so the merge reads one dense block of the workspace.  A worker
  // enters every segment but its first one at the segment's start, i.e. as its first visitor; so the
  // id of its first piece is stored with the worker and the id of the first visitor with the segment.
  const int BH = B * Hw;
  auto bh_of = [&](const Segment& sg) { return sg.b * Hw + sg.h; };
  std::vector<int32_t> own_cnt(S, 0), bh_off(BH + 1, 0);
  for (int w = 0; w < P; ++w) {
    int sidx = items[w].seg0;
    for (int32_t g = items[w].g0; g < items[w].g1; ++sidx) {
      ++own_cnt[sidx];
      const int32_t end = segs[sidx].gblk0 + segs[sidx].nblk;
      g = end < items[w].g1 ? end : items[w].g1;
    }
  }
  for (int sidx = 0; sidx < S; ++sidx) bh_off[bh_of(segs[sidx]) + 1] += own_cnt[sidx];
  // A pool part needs a partial slot for every rank that can enter its segment from another one.  Own
  // ranges and pool parts both ascend, so these are the leading ranks: those whose own range is empty or
  // ends in an earlier segment.
  for (int g = 0, w0 = 0; g < NG; w0 += groups[g].nworkers, ++g)
    for (int i = 0; i < groups[g].nps; ++i) {
      PoolSeg& ps = psegs[groups[g].pseg0 + i];
      int n = 0;
      for (int r = 0; r < groups[g].nworkers; ++r) {
        const Item& it = items[w0 + r];
        const bool ends_here = it.g0 < it.g1 && seg_of(it.g1 - 1, it.seg0) == ps.seg;
        if (!ends_here) n = r + 1;
      }
      ps.nslots = n;
      bh_off[bh_of(segs[ps.seg]) + 1] += n;
    }
  // the appended tokens: one more partial per slice of the append buffer of a (b, kv head), at the end of its range
  const int append_blocks = (append_capacity + kTB - 1) / kTB;
  const int append_slices = (append_blocks + kAppendSliceBlocks - 1) / kAppendSliceBlocks;
  for (int i = 0; i < BH; ++i) bh_off[i + 1] += append_slices;
  for (int i = 0; i < BH; ++i) bh_off[i + 1] += bh_off[i];
  const int32_t npart = bh_off[BH];
  {
    std::vector<int32_t> cursor(bh_off.begin(), bh_off.end() - 1);
    for (int sidx = 0; sidx < S; ++sidx) {
      segs[sidx].pid0 = cursor[bh_of(segs[sidx])];
      cursor[bh_of(segs[sidx])] += own_cnt[sidx];
    }
    for (int g = 0; g < NG; ++g)
      for (int i = 0; i < groups[g].nps; ++i) {
        PoolSeg& ps = psegs[groups[g].pseg0 + i];
        ps.slot0 = cursor[bh_of(segs[ps.seg])];
        cursor[bh_of(segs[ps.seg])] += ps.nslots;
      }
    std::vector<int32_t> visitors(S, 0);
    for (int w = 0; w < P; ++w) {
      int sidx = items[w].seg0;
      items[w].pid0 = items[w].g0 < items[w].g1 ? segs[sidx].pid0 + visitors[sidx] : 0;
      for (int32_t g = items[w].g0; g < items[w].g1; ++sidx) {
        ++visitors[sidx];
        const int32_t end = segs[sidx].gblk0 + segs[sidx].nblk;
        g = end < items[w].g1 ? end : items[w].g1;
      }
    }
  }

  // reorder+quantize records, one per block of the class buffers: the largest array of a plan by far (2.6 MB for 40 heads of
  // 128K tokens), so they are written straight into the blob, and not at all when only the sizes are asked for
  const int64_t num_items = int64_t(v_blk_base[NC * B + 0]) + v_blk_base[NC * B + 1] + v_blk_base[NC * B + 2] + v_blk_base[NC * B + 3];
  // (blocks of an FP16 run that are only room to grow get a record without valid rows: they are written as zeros)
  // (by copies, as everything in the blob: the caller's buffer need not be aligned)
  auto write_items = [&](char* out) {
    for (int c = 0; c < NC; ++c)
      for (int b = 0; b < B; ++b) {
        const int nb = v_cap[NC * b + c], ntok = v_ct[NC * b + c];
        if (nb == 0) continue;
        const int n = seq_lens[b] / C;
        const int32_t* pb = v_perm.data() + v_chunk_off[b];
        const int cc0 = v_cc0[NC * b + c];
        const int tail = seq_lens[b] - n * C;
        const int chunk_tokens = c == kFp16Class ? ntok - tail : ntok;
        auto src_token = [&](int r) {   // source token of row r of the class (Alg. 1 order; tail after the FP16 chunks)
          if (r < chunk_tokens) return pb[cc0 + r / C] * C + r % C;
          return n * C + (r - chunk_tokens);
        };
        const int64_t row0 = v_cum[b] * Hkv;   // first source row of the sequence in the ragged layout
        for (int j = 0; j < nb; ++j) {
          RQItem it;
          std::memset(&it, 0, sizeof(it));
          const int r0 = j * kTB;
          const int nvalid = ntok - r0 < kTB ? (ntok > r0 ? ntok - r0 : 0) : kTB;
          it.b = b, it.j = j;
          it.cls_nvalid = c | (nvalid << 8);
          if (nvalid > 0) {   // else room to grow: t0 = 0, nothing is read
            const int t0 = src_token(r0);
            // rows are consecutive tokens iff the last one is (chunks keep their order, so tokens in between are too)
            it.t0 = src_token(r0 + nvalid - 1) == t0 + nvalid - 1 ? t0 : -1;
          }
          it.ragged_row = row0 + (it.t0 >= 0 ? it.t0 : 0);
          std::memcpy(out + int64_t(j) * sizeof(it), &it, sizeof(it));
        }
        for (int h = 1; h < Hkv; ++h)   // the other heads: the same rows, seq_lens[b] further on each
          for (int j = 0; j < nb; ++j) {
            RQItem it;
            std::memcpy(&it, out + int64_t(j) * sizeof(it), sizeof(it));
            it.h = h;
            it.ragged_row += int64_t(h) * seq_lens[b];
            std::memcpy(out + (int64_t(h) * nb + j) * sizeof(it), &it, sizeof(it));
          }
        out += int64_t(Hkv) * nb * sizeof(RQItem);
      }
  };

  // ---- the split for short contexts ----
  ShortSplit quick;
  // (from kNonTemporalMinBytes on the two launches read past the caches; up to twice that 47 random shapes of up to four heads in one, with up to ten
  // iterations per wave, took 2.3 % longer in the mean, 6 % behind another kernel, from -11 to +18 %)
  if (!tune.changed && packed < kNonTemporalMinBytes)
    for (const bool one : {true, false}) {
      if (quick.groups > 0 || (tiles && !one)) break;
      quick = short_split(v_ct, B, Hw, D, append_capacity, wrep, share, one, std::min(num_workers, kChipWorkers) / kCuWaves);
    }
  if (quick.shared && quick.groups > npart) quick = ShortSplit();   // (their states share the workspace with those of the other split)

  // ---- sizes and blob layout ----
  PlanHeader hd;
  std::memset(&hd, 0, sizeof(hd));
  hd.magic = kPlanMagic, hd.version = kPlanVersion;
  hd.batch = B, hd.num_q_heads = shape->num_q_heads, hd.num_kv_heads = Hkv, hd.head_dim = D;
  hd.chunk_size = C, hd.group_size = G, hd.rep = rep, hd.work_heads = Hw, hd.work_rep = wrep;
  hd.num_workers = P, hd.num_segments = S, hd.num_partials = npart;
  hd.num_groups = NG, hd.num_pool_segs = NPS;
  hd.append_capacity = append_capacity, hd.append_blocks = append_blocks, hd.append_slices = append_slices;
  hd.total_gblocks = static_cast<int32_t>(gblk);
  hd.v_layout = quads ? 1 : 0;
  hd.total_chunks = total_chunks, hd.total_tokens = total_tokens, hd.packed_bytes = packed;
  for (int c = 0; c < NC; ++c) {
    hd.class_blocks[c] = v_blk_base[NC * B + c];
    hd.class_bytes[c] = hd.class_blocks[c] * block_bytes[c];
    hd.block_bytes[c] = block_bytes[c];
    hd.row_bytes[c] = row_bytes[c];
  }
  // decode workspace: the partial states, then one status word per (sequence, query head)
  hd.ws_status_off = align16(int64_t(npart > 0 ? npart : 1) * wrep * (D + kPartialFloats) * int64_t(sizeof(float)));
  hd.workspace_bytes = hd.ws_status_off + align16(int64_t(sizeof(int32_t)) * B * shape->num_q_heads);
  int64_t off = align16(sizeof(PlanHeader));
  bool too_large = false;
  auto place = [&](int32_t& field, int64_t bytes) {
    if (off + bytes >= (int64_t(1) << 31)) too_large = true;   // the offsets are 32-bit fields
    field = static_cast<int32_t>(too_large ? 0 : off);
    off = align16(off + bytes);
  };
  place(hd.off_seq_len, 4 * int64_t(B));
  place(hd.off_cum_tokens, 8 * int64_t(B + 1));
  place(hd.off_chunk_off, 4 * int64_t(B + 1));
  place(hd.off_perm, 4 * total_chunks);
  place(hd.off_class_tokens, 4 * NC * int64_t(B));
  place(hd.off_class_chunk0, 4 * NC * int64_t(B));
  place(hd.off_blk_base, 4 * NC * int64_t(B + 1));
  place(hd.off_nblk, 4 * NC * int64_t(B));
  place(hd.off_run_blocks, 4 * NC * int64_t(B));
  place(hd.off_segments, int64_t(sizeof(Segment)) * S);
  place(hd.off_bh_off, 4 * int64_t(BH + 1));
  place(hd.off_worker_rec, int64_t(sizeof(WorkerRec)) * P);
  place(hd.off_group_rec, int64_t(sizeof(GroupRec)) * NG);
  place(hd.off_pool_seg, int64_t(sizeof(PoolSeg)) * NPS);
  place(hd.off_rq_items, int64_t(sizeof(RQItem)) * num_items);
  off = (off + 127) & ~int64_t(127);
  place(hd.off_counters, int64_t(4 * counter_stride(NPS)) * NG);
  if (quick.groups > 0) {
    place(hd.off_short, int64_t(sizeof(ShortRec) * kCuWaves + sizeof(ShortGroup)) * quick.groups);
    hd.short_groups = int16_t(quick.groups), hd.short_units = quick.one;
    int32_t counters;
    off = short_counters_offset(hd);
    place(counters, int64_t(4 * kShortCounterStride) * quick.rows);
  }
  if (too_large || off >= (int64_t(1) << 31)) return fail(COCKTAIL_EUNSUPPORTED, "plan larger than 2 GiB");
  hd.plan_bytes = off;

  std::memset(sizes, 0, sizeof(*sizes));
  sizes->total_chunks = total_chunks;
  for (int c = 0; c < NC; ++c) {
    sizes->class_tokens[c] = class_tokens_tot[c];
    sizes->class_blocks[c] = hd.class_blocks[c];
    sizes->class_bytes[c] = hd.class_bytes[c];
  }
  sizes->plan_bytes = hd.plan_bytes;
  sizes->workspace_bytes = hd.workspace_bytes;
  sizes->packed_bytes = packed;
  sizes->num_workers = P, sizes->num_partials = npart, sizes->num_segments = S;
  sizes->append_capacity = append_capacity;
  sizes->v_layout = hd.v_layout, sizes->reserved = 0;
  sizes->append_bytes = int64_t(B) * Hkv * hd.append_blocks * kTB * 2 * D;

  if (class_tokens) std::memcpy(class_tokens, v_ct.data(), sizeof(int32_t) * v_ct.size());
  if (perm && total_chunks) std::memcpy(perm, v_perm.data(), sizeof(int32_t) * v_perm.size());

  if (plan_host) {
    if (plan_capacity < static_cast<size_t>(hd.plan_bytes))
      return fail(COCKTAIL_ENOSPACE, "plan buffer holds %zu bytes, %lld needed", plan_capacity,
                  (long long)hd.plan_bytes);
    char* p = static_cast<char*>(plan_host);
    std::memset(p, 0, hd.off_rq_items);   // the records fill their part themselves
    const int64_t items_end = hd.off_rq_items + int64_t(sizeof(RQItem)) * num_items;
    const int64_t zeros_end = quick.groups > 0 ? hd.off_short : hd.plan_bytes;
    std::memset(p + items_end, 0, zeros_end - items_end);
    if (quick.groups > 0) {   // (whose records are written below)
      const int64_t end = short_group_offset(hd) + int64_t(sizeof(ShortGroup)) * quick.groups;
      std::memset(p + end, 0, hd.plan_bytes - end);
    }
    std::memcpy(p, &hd, sizeof(hd));
    auto put = [&](int32_t o, const void* src, size_t bytes) {
      if (bytes) std::memcpy(p + o, src, bytes);
    };
    put(hd.off_seq_len, seq_lens, 4 * size_t(B));
    put(hd.off_cum_tokens, v_cum.data(), 8 * size_t(B + 1));
    put(hd.off_chunk_off, v_chunk_off.data(), 4 * size_t(B + 1));
    put(hd.off_perm, v_perm.data(), 4 * size_t(total_chunks));
    put(hd.off_class_tokens, v_ct.data(), 4 * NC * size_t(B));
    put(hd.off_class_chunk0, v_cc0.data(), 4 * NC * size_t(B));
    put(hd.off_blk_base, v_blk_base.data(), 4 * NC * size_t(B + 1));
    put(hd.off_nblk, v_nblk.data(), 4 * NC * size_t(B));
    put(hd.off_run_blocks, v_cap.data(), 4 * NC * size_t(B));
    put(hd.off_segments, segs.data(), sizeof(Segment) * size_t(S));
    put(hd.off_bh_off, bh_off.data(), 4 * bh_off.size());
    if (quick.groups > 0)
      write_short_split(quick, v_ct, v_blk_base, v_cap, seq_lens, Hw, share, wrep, append_blocks, p + hd.off_short, p + short_group_offset(hd));
    // Which worker id runs which range.  Worker ids are handed to the compute units in order
    // (round-robin over the XCDs), and when P fills the chip twice, worker i shares a SIMD with
    // worker i + P/2, which was dispatched later and loses every issue arbitration against it.
    //   mode 0 (default): range w runs as worker w.  With the class-major layout the INT2 ranges
    //           get INT4 / FP16 ranges as SIMD mates, the mix that keeps both the vector ALU and the
    //           memory pipeline busy.
    //   mode 2: rank r of group j becomes worker (r odd ? P/2 : 0) + j*k/2 + (r/2 + j) mod (k/2):
    //           SIMD mates are neighbouring ranks of one group.  Mode 3: mates are ranks r and r + k/2.
    // With twins the groups of a unit are dealt out so that the workers of a stripe are kXcds apart.
    // Where a class has more than half of the workers, some have a mate of their own class, and of those the one dispatched first gets ahead
    // of the other by a third of the call (128K tokens, 40 heads: INT2 next to INT2 ends at 77 and 105 us, every other worker
    // between 88 and 97).  Every other rank of such groups trades places with its mate: each group then has both
    // kinds, and its pool evens them out (107.5 -> 103.9 us per call).  One head per wave only: with four, a cache of FP16 alone got
    // slower by it (32 q / 8 kv heads, 64K tokens: 51.4 -> 52.6 us; INT2 alone and INT4 alone the same).
    const int pair_mode = tune.pair_mode;
    const bool spread = pair_mode >= 2 && group_workers % 2 == 0 && P % group_workers == 0;
    const bool trade = wrep == 1 && pool_percent > 0 && pair_mode == 0 && P % 2 == 0;
    auto class_of = [&](int w) { return items[w].g0 < items[w].g1 ? segs[items[w].seg0].cls : -1; };
    for (int w = 0; w < P; ++w) {
      int id = w;
      const int mate = (w + P / 2) % P;
      if (trade && items[std::min(w, mate)].rank % 2 == 1 && class_of(w) == class_of(mate)) id = mate;
      if (spread) {
        const int hk = group_workers / 2, j = items[w].group, r = items[w].rank;
        id = pair_mode == 2 ? (r & 1) * (P / 2) + j * hk + ((r >> 1) + j) % hk
                            : (r / hk) * (P / 2) + j * hk + (r % hk + j) % hk;
      }
      if (twins && w < P - P % unit) {   // group g of a unit: set g % sets of stripe g / sets
        const int r = w % unit, g = r / group_workers;
        id = w - r + g % sets * kXcds + g / sets * group_workers + r % group_workers;
      }
      WorkerRec rc = {};
      rc.g0 = items[w].g0, rc.g1 = items[w].g1;
      rc.seg0 = items[w].seg0, rc.pid0 = items[w].pid0;
      rc.group = items[w].group;
      rc.rank_nps = items[w].rank | (groups[items[w].group].nps << 16);
      rc.ngran = groups[items[w].group].ngran, rc.pseg0 = groups[items[w].group].pseg0;
      if (items[w].g0 < items[w].g1) rc.first = segs[items[w].seg0];
      std::memcpy(p + hd.off_worker_rec + int64_t(id) * sizeof(rc), &rc, sizeof(rc));
    }
    put(hd.off_group_rec, groups.data(), sizeof(GroupRec) * groups.size());
    put(hd.off_pool_seg, psegs.data(), sizeof(PoolSeg) * psegs.size());
    write_items(p + hd.off_rq_items);
  }
  g_err[0] = 0;
  return COCKTAIL_OK;
}

extern "C" int cocktail_plan_ex(const cocktail_shape* shape, const int32_t* seq_lens, const uint8_t* chunk_bits,
                                int32_t num_workers, const cocktail_plan_options* options, cocktail_sizes* sizes,
                                void* plan_host, size_t plan_capacity, int32_t* class_tokens, int32_t* perm) {
  auto plan = [&](cocktail_sizes* to, bool write, bool any_length, bool* too_long) {
    return make_plan(shape, seq_lens, chunk_bits, num_workers, options, to, write ? plan_host : nullptr, write ? plan_capacity : 0,
                     class_tokens, perm, any_length, too_long);
  };
  bool too_long = false;
  const int rc = plan(sizes, true, false, &too_long);
  if (!too_long || (rc != COCKTAIL_OK && rc != COCKTAIL_ENOSPACE)) return rc;
  // The split by cost of that many runs has a partial state for nearly each worker and run.  With more workers than the chip holds they
  // may outgrow the built-in workspace where one state per worker does not: a slow plan that cocktail_decode_attention_static takes,
  // rather than one it refuses.
  const int rep = shape->num_q_heads / shape->num_kv_heads;
  const int64_t limit = static_workspace_limit(sizes->v_layout, work_rep_of(rep, options && options->vector_alu_only != 0), rep);
  if (sizes->workspace_bytes <= limit) return rc;
  cocktail_sizes other;
  const bool fits = plan(&other, false, true, nullptr) == COCKTAIL_OK && other.workspace_bytes <= limit;
  return plan(sizes, true, fits, nullptr);
}
