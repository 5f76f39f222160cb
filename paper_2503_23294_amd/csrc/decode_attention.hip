// Decode side of Alg. 1 (Sec. III-C): single-query attention over the INT2, INT4,
// INT8 and FP16 classes of the packed cache.
//
// This file holds the exact merge of the partial softmax states and the host side of the decode entry points; short contexts run on kernels
// that merge by themselves (decode_short_impl.h);
// the partial-state kernels are templates (decode_heads_impl.h: one query head per kv head, vector ALU;
// decode_quads_impl.h: two to four query heads per wave, 4x4x4 matrix instructions; decode_tiles_impl.h: five to eight,
// 16x16x32 matrix instructions) instantiated per head_dim in their own translation units.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <mutex>
#include <vector>

#include "decode_heads_impl.h"

namespace cocktail {

typedef float f4 __attribute__((ext_vector_type(4)));

template hipError_t launch_decode_heads<128>(const DecodeParams&, int, bool, bool, int, hipStream_t);

// Exact merge of the partial states of one (sequence, query head):
//   M = max m_i,  L = sum l_i 2^(m_i - M),  out = sum o_i 2^(m_i - M) / L,  lse = ln2 (M + log2 L).
// The partials of a (sequence, kv head) are a dense block of the workspace.  A thread holds four channels of every SLICES-th of them, up to
// eight at a time (usually the whole block in one round); the slices of a wave are summed up in registers, those of the eight waves
// through shared memory.  A (sequence, query head) without any partial (empty sequence) gets zeros and lse = -inf.
//
// Bound by a chain of latencies: range of partials -> partials -> out.  The arguments of the first links are in scalar registers from
// the start, and what the rest needs (context length, appended tokens, pointers) is fetched beside the partials; as the compiler ordered it,
// these four dependent reads came first.  With that the calls of small layers went from 11.3 to 10.3 us (30 blocks), 13.8 to 12.8
// (32 heads, 5K tokens), 34.3 to 33.3 (32 heads, 32K).
// PARTS: the channels of a row on several workgroups.  Few rows have many partials each (2048 workers on four rows: 500), 264 KB
// for one compute unit: 4 ragged contexts up to 51K, 5 query heads on one kv head 18.8 -> 15.2 us per call (21.2 as one workgroup folded
// them before); 32 rows 33.25 -> 33.0, 128 rows the same; 256 rows and more lose up to 6 % (22.3 -> 23.6 us), since every part reads
// the states' headers: kSplitMergeRows.
// Every partial also says how many tokens it covers.  Their sum has to be the token count of the
// sequence: the softmax over the concatenation of Alg. 1 attends to every token exactly once.  If it is
// not (ticket counters that were not zero when the call started, calls overlapping on one cache, a
// damaged plan), the row is not a result: out and lse are set to NaN and the difference goes to the
// status array.
constexpr int kSplitMergeRows = 128;
constexpr int kMergeThreads = 512, kMergeWaves = kMergeThreads / 64;
#define COCKTAIL_MERGE_ARGS const int32_t *bh_off, const float *ws, const int32_t *seq_len, int32_t rep, int32_t num_kv_heads, DecodeParams
typedef void (*merge_kernel)(COCKTAIL_MERGE_ARGS);
constexpr int kMergeParamsOffset = LastArgument<merge_kernel>::offset();   // of the DecodeParams in the merge's kernel argument segment
template <int D, int PARTS>
__global__ __launch_bounds__(kMergeThreads) void decode_merge_kernel(COCKTAIL_MERGE_ARGS) {
  constexpr int CH = D / PARTS, QUADS = CH / 4, SLICES = kMergeThreads / QUADS;
  static_assert(QUADS >= 8 && QUADS <= 32, "the slices of a wave are 8, 16 or 32 lanes apart");
  constexpr int STRIDE = D + kPartialFloats;
  constexpr int U = 8;   // partials in flight per thread
  __shared__ float sm_m[kMergeWaves];
  __shared__ float sm_l[kMergeWaves];
  __shared__ int sm_c[kMergeWaves];
  __shared__ __attribute__((aligned(16))) float sm_o[kMergeWaves][CH];
  const int bh = blockIdx.x, r = blockIdx.y, part = blockIdx.z;
  const int lo = load_record(bh_off + bh);
  const int n = load_record(bh_off + bh + 1) - lo;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int quad = tid % QUADS, slice = tid / QUADS;
  // the row's partials as a buffer (below 4 GiB: a partial per worker and pool part at most): reads past them return zeros
  const uint32_t step = rep * (STRIDE * 4);   // bytes
  const rsrc_t rows = make_rsrc(reinterpret_cast<const char*>(ws) + int64_t(lo) * step, uint32_t(n) * step);
  const uint32_t head = slice * step + r * (STRIDE * 4), body = head + (kPartialFloats + part * CH + quad * 4) * 4;
  f4 hd[U], va[U];
  auto fetch = [&](int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && i0 + SLICES * u >= n) break;
      const uint32_t at = (i0 + SLICES * u) * step;
      hd[u] = __builtin_bit_cast(f4, load16<kAuxDefault>(rows, head, at));   // m, l, tokens, unused
      va[u] = __builtin_bit_cast(f4, load16<kAuxDefault>(rows, body, at));
    }
  };
  if (n > 0) fetch(0);
  // What the rest of the kernel needs is fetched together with the partial states, not in front of them.
  sched_fence();
  typedef const __attribute__((address_space(4))) DecodeParams* params_t;
  uint64_t pp = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr()) + kMergeParamsOffset;
  asm volatile("" : "+s"(pp) : "s"(lo));
  const params_t prm = reinterpret_cast<params_t>(pp);
  const int b = bh / num_kv_heads;
  const int context = load_record(seq_len + b);
  _Float16* const out = prm->out;
  float* const lse = prm->lse;
  int32_t* const status = prm->status;
  int appended = prm->num_appended;
  const int32_t* const counts = prm->appended;
  const int capacity = prm->app_capacity;
  if (counts) appended = load_record(counts + b);
  const int expected = context + min(max(appended, 0), capacity);
  // every worker has drawn its last ticket: put the counters back to zero for the next call
  if (bh == 0 && r == 0 && part == 0)
    for (int i = tid; i < prm->num_groups; i += kMergeThreads) prm->counters[i * kPoolCounterStride] = 0u;
  sched_fence();
  float m = -INFINITY, l = 0.f;
  f4 o = {0.f, 0.f, 0.f, 0.f};
  int covered = 0;
  // 2^(x - reference); a state without tokens (reference and x are -inf) has weight 0
  auto weight = [](float x, float reference) { return x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x - reference); };
  for (int i0 = 0; i0 < n; i0 += SLICES * U) {
    if (i0 > 0) fetch(i0);
    float top = m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && i0 + SLICES * u >= n) break;
      if (i0 + slice + SLICES * u >= n) hd[u].x = -INFINITY, hd[u].z = 0.f;
      top = fmaxf(top, hd[u].x);
    }
    const float a = weight(m, top);
    m = top, l *= a, o *= a;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && i0 + SLICES * u >= n) break;
      const float w = weight(hd[u].x, top);
      l += hd[u].y * w, o += va[u] * w;
      covered += __float_as_int(hd[u].z);
    }
  }
  // the slices of the wave, QUADS lanes apart, then those of the waves
  float top = m;
  if constexpr (QUADS <= 8) top = fmaxf(top, row_ror<8>(top));
  if constexpr (QUADS <= 16) {
    float x, y;
    swap_rows(top, top, x, y);
    top = fmaxf(x, y);
  }
  top = both_halves(top, true);
  const float a = weight(m, top);
  l *= a, o *= a;
  auto slice_sum = [](float x) {
    if constexpr (QUADS <= 8) x += row_ror<8>(x);
    if constexpr (QUADS <= 16) {
      float p, q;
      swap_rows(x, x, p, q);
      x = p + q;
    }
    return both_halves(x, false);
  };
  l = slice_sum(l);
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = slice_sum(o[i]);
#pragma unroll
  for (int s = QUADS; s < 64; s *= 2) covered += __shfl_xor(covered, s);
  if (lane < QUADS) *reinterpret_cast<f4*>(&sm_o[wave][quad * 4]) = o;
  if (lane == 0) sm_m[wave] = top, sm_l[wave] = l, sm_c[wave] = covered;
  __syncthreads();
  if (tid < CH) {
    float mx = sm_m[0];
    int total = sm_c[0];
#pragma unroll
    for (int w = 1; w < kMergeWaves; ++w) mx = fmaxf(mx, sm_m[w]), total += sm_c[w];
    float big_l = 0.f, sum = 0.f;
#pragma unroll
    for (int w = 0; w < kMergeWaves; ++w) {
      const float x = weight(sm_m[w], mx);
      big_l += sm_l[w] * x;
      sum += sm_o[w][tid] * x;
    }
    const bool empty = !(big_l > 0.f);
    const bool sound = total == expected;
    const float res = empty ? 0.f : sum / big_l;
    const int bhq = bh * rep + r;
    out[int64_t(bhq) * D + part * CH + tid] = static_cast<_Float16>(sound ? res : __builtin_nanf(""));
    if (tid == 0 && part == 0) {
      status[bhq] = total - expected;
      if (lse) lse[bhq] = !sound ? __builtin_nanf("") : empty ? -INFINITY : (mx + log2f(big_l)) * 0.6931471805599453f;
    }
  }
}

}  // namespace cocktail

using namespace cocktail;

extern "C" int cocktail_default_workers(const cocktail_shape* shape, int32_t* num_workers) {
  if (int rc = check_shape(shape)) return rc;
  if (!num_workers) return fail(COCKTAIL_EINVAL, "num_workers is NULL");
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
    (void)hipGetLastError();
    return fail(COCKTAIL_EHIP, "no HIP device available");
  }
  *num_workers = prop.multiProcessorCount * 8;   // two waves per SIMD at <= 256 VGPRs
  return COCKTAIL_OK;
}

// Scratch of the entry point that allocates nothing: the partial softmax states and the status words of one
// decode call.  In host code this name is only a handle; the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[COCKTAIL_STATIC_WORKSPACE_BYTES_TILES];
size_t static_workspace_limit(const PlanHeader* hd) {
  return static_cast<size_t>(static_workspace_limit(hd->v_layout, hd->work_rep, hd->rep));
}

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};   // per device: address of `scratch` there

// Address of the static workspace on the current device (looked up once per device).
int static_workspace(void** ptr) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return fail(COCKTAIL_EHIP, "no current HIP device (or its index is not below %d)", kMaxDevices);
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      return fail(COCKTAIL_EHIP, "hipGetSymbolAddress(static workspace) failed on device %d: %s", dev, hipGetErrorString(e));
    }
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return COCKTAIL_OK;
}

int check_plan_matches(const cocktail_shape* shape, const cocktail_cache* cache, const PlanHeader** out) {
  if (int rc = check_shape(shape)) return rc;
  if (!cache || !cache->plan_host || !cache->plan_dev) return fail(COCKTAIL_EINVAL, "cache or its plan is NULL");
  const PlanHeader* hd = static_cast<const PlanHeader*>(cache->plan_host);
  if (hd->magic != kPlanMagic || !known_version(hd->version))
    return fail(COCKTAIL_EINVAL, "plan_host is not a plan written by this library version");
  if (hd->batch != shape->batch || hd->num_kv_heads != shape->num_kv_heads || hd->head_dim != shape->head_dim ||
      hd->chunk_size != shape->chunk_size || hd->group_size != shape->group_size ||
      hd->num_q_heads != shape->num_q_heads)
    return fail(COCKTAIL_EINVAL, "plan was made for a different shape");
  *out = hd;
  return COCKTAIL_OK;
}

// Validates the arguments and enqueues the kernels; `workspace` holds at least hd->workspace_bytes.
int decode_enqueue(const cocktail_shape* shape, const PlanHeader* hd, const void* q, const cocktail_cache* cache,
                   float sm_scale, void* out, float* lse, void* workspace, void* stream, void* event_between = nullptr) {
  if (shape->head_dim != 64 && shape->head_dim != 128)
    return fail(COCKTAIL_EUNSUPPORTED, "kernels are built for head_dim 64 and 128, got %d", shape->head_dim);
  if (hd->rep > COCKTAIL_MAX_Q_PER_KV)
    return fail(COCKTAIL_EUNSUPPORTED, "Hq/Hkv = %d exceeds %d", hd->rep, COCKTAIL_MAX_Q_PER_KV);
  if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(workspace) |
       reinterpret_cast<uintptr_t>(cache->plan_dev)) & 15)
    return fail(COCKTAIL_EALIGN, "q, out, workspace and plan_dev must be 16-byte aligned");
  if (lse && (reinterpret_cast<uintptr_t>(lse) & 3)) return fail(COCKTAIL_EALIGN, "lse must be 4-byte aligned");
  DecodeParams p;
  char* pd = static_cast<char*>(cache->plan_dev);
  p.recs = reinterpret_cast<const WorkerRec*>(pd + hd->off_worker_rec);
  p.segs = reinterpret_cast<const Segment*>(pd + hd->off_segments);
  p.psegs = reinterpret_cast<const PoolSeg*>(pd + hd->off_pool_seg);
  p.counters = reinterpret_cast<uint32_t*>(pd + hd->off_counters);
  p.seq_len = reinterpret_cast<const int32_t*>(pd + hd->off_seq_len);
  p.num_groups = hd->num_pool_segs > 0 ? hd->num_groups : 0;   // whose counters the merge puts back
  p.num_workers = hd->num_workers;
  p.k_app = p.v_app = nullptr;
  p.num_appended = 0, p.app_blocks = hd->append_blocks;
  p.appended = nullptr, p.app_capacity = hd->append_capacity, p.app_slices = hd->append_slices;
  if (hd->append_capacity > 0) {
    if (!cache->k_app || !cache->v_app) return fail(COCKTAIL_EINVAL, "the plan has append buffers but k_app or v_app is NULL");
    if ((reinterpret_cast<uintptr_t>(cache->k_app) | reinterpret_cast<uintptr_t>(cache->v_app)) & 15)
      return fail(COCKTAIL_EALIGN, "append buffers must be 16-byte aligned");
    if (cache->num_appended < 0 || cache->num_appended > hd->append_capacity)
      return fail(COCKTAIL_EINVAL, "num_appended %d outside [0, %d]", cache->num_appended, hd->append_capacity);
    if (cache->appended_dev && (reinterpret_cast<uintptr_t>(cache->appended_dev) & 3))
      return fail(COCKTAIL_EALIGN, "appended_dev must be 4-byte aligned");
    if (cache->appended_dev && cache->num_appended != 0)
      return fail(COCKTAIL_EINVAL, "num_appended must be 0 when appended_dev holds the per-sequence counts");
    p.k_app = static_cast<const char*>(cache->k_app), p.v_app = static_cast<const char*>(cache->v_app);
    p.num_appended = cache->num_appended;
    p.appended = cache->appended_dev;
  } else if (cache->num_appended != 0 || cache->appended_dev) {
    return fail(COCKTAIL_EINVAL, "num_appended / appended_dev are set but the plan was made without append buffers");
  }
  p.bh_off = reinterpret_cast<const int32_t*>(pd + hd->off_bh_off);
  p.q = static_cast<const uint32_t*>(q);
  for (int c = 0; c < kNumClasses; ++c) {
    if (hd->class_bytes[c] > 0 && (!cache->k[c] || !cache->v[c]))
      return fail(COCKTAIL_EINVAL, "cache buffer of class %d is NULL", c);
    if ((reinterpret_cast<uintptr_t>(cache->k[c]) | reinterpret_cast<uintptr_t>(cache->v[c])) & 15)
      return fail(COCKTAIL_EALIGN, "cache buffers must be 16-byte aligned");
    p.k[c] = static_cast<const char*>(cache->k[c]);
    p.v[c] = static_cast<const char*>(cache->v[c]);
  }
  p.ws = static_cast<float*>(workspace);
  p.status = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + hd->ws_status_off);
  p.out = static_cast<_Float16*>(out);
  p.lse = lse;
  if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt(static_cast<float>(shape->head_dim));
  p.scale_log2 = sm_scale * 1.4426950408889634f;
  p.rep = hd->work_rep, p.num_q_heads = hd->num_q_heads, p.num_kv_heads = hd->work_heads;
  p.kv_share = hd->work_heads / hd->num_kv_heads;
#ifdef COCKTAIL_TRACE
  // debugging builds only: the caller provides 32 bytes per worker behind the regular workspace
  p.trace = reinterpret_cast<uint64_t*>(static_cast<char*>(workspace) + ((hd->workspace_bytes + 255) & ~int64_t(255)));
#endif
  hipStream_t st = static_cast<hipStream_t>(stream);
#ifdef COCKTAIL_TRACE
  const bool one_launch = false;   // (the workers' records are what is traced)
#else
  // (between the two kernels: an event there wants two)
  const bool one_launch = hd->short_groups > 0 && !event_between;
#endif
  if (one_launch) {
    const ShortRec* recs = reinterpret_cast<const ShortRec*>(pd + hd->off_short);
    const ShortGroup* place = reinterpret_cast<const ShortGroup*>(pd + short_group_offset(*hd));
    const int counters = static_cast<int>(short_counters_offset(*hd) - short_group_offset(*hd));
    const bool quads = hd->v_layout == COCKTAIL_V_TOKEN_QUADS, int8 = hd->class_blocks[2] > 0;
    const hipError_t e = shape->head_dim == 64 ? launch_decode_short<64>(p, recs, place, counters, quads, shape->group_size, int8, hd->short_units == 1, hd->short_groups, st)
                                               : launch_decode_short<128>(p, recs, place, counters, quads, shape->group_size, int8, hd->short_units == 1, hd->short_groups, st);
    return e == hipSuccess ? COCKTAIL_OK : fail(COCKTAIL_EHIP, "decode launch failed: %s", hipGetErrorString(e));
  }
  const int app_groups = hd->batch * hd->work_heads * hd->append_slices;   // 0 without append buffers
  if (hd->total_gblocks > 0 || app_groups > 0) {
    const bool quads = hd->v_layout == COCKTAIL_V_TOKEN_QUADS;
    const dim3 grid(hd->num_workers + app_groups, 1, 1);
    // non-temporal K/V loads when nothing is read twice (one wave per kv head's blocks: the vector-ALU kernel
    // with one query head per kv head, the matrix kernel with all query heads of a kv head in one wave) and the
    // cache is large enough that it cannot stay in the memory-side cache from one call to the next
    static const int nt_override = [] {   // tuning aid, read once: COCKTAIL_NON_TEMPORAL=0 | 1
      const char* e = std::getenv("COCKTAIL_NON_TEMPORAL");
      return e ? (std::atoi(e) != 0 ? 1 : 0) : -1;
    }();
    // (several work heads per kv head - one wave per query head of a grouped-query shape, or sets of eight at
    // ratios above eight - read the same lines from different waves: default policy, the L2 serves the repeats)
    const bool nt = nt_override >= 0 ? nt_override == 1
                                     : (hd->work_rep == hd->rep && hd->packed_bytes >= kNonTemporalMinBytes);
    const bool int8 = hd->class_blocks[2] > 0;
    const bool d64 = shape->head_dim == 64;
    const bool tiles = quads && uses_tiles(p.rep);
    const hipError_t e = tiles ? (d64 ? launch_decode_tiles<64>(p, shape->group_size, nt, int8, int(grid.x), st)
                                      : launch_decode_tiles<128>(p, shape->group_size, nt, int8, int(grid.x), st))
                       : quads ? (d64 ? launch_decode_quads<64>(p, shape->group_size, nt, int8, int(grid.x), st)
                                      : launch_decode_quads<128>(p, shape->group_size, nt, int8, int(grid.x), st))
                               : (d64 ? launch_decode_heads<64>(p, shape->group_size, nt, int8, int(grid.x), st)
                                      : launch_decode_heads<128>(p, shape->group_size, nt, int8, int(grid.x), st));
    if (e != hipSuccess) return fail(COCKTAIL_EHIP, "decode launch failed: %s", hipGetErrorString(e));
  }
  if (event_between) {   // measurement aid: when the partial-state kernel is done
    const hipError_t ev = hipEventRecord(static_cast<hipEvent_t>(event_between), st);
    if (ev != hipSuccess) return fail(COCKTAIL_EHIP, "recording the event between the two kernels failed: %s", hipGetErrorString(ev));
  }
  const bool split = int64_t(hd->batch) * hd->num_q_heads <= kSplitMergeRows;
  auto merge = [&](merge_kernel kernel, int parts) {
    return launch(kernel, dim3(hd->batch * hd->work_heads, hd->work_rep, parts), dim3(kMergeThreads), st, p.bh_off, p.ws, p.seq_len, p.rep, p.num_kv_heads, p);
  };
  const hipError_t e = shape->head_dim == 64 ? split ? merge(decode_merge_kernel<64, 2>, 2) : merge(decode_merge_kernel<64, 1>, 1)
                                             : split ? merge(decode_merge_kernel<128, 4>, 4) : merge(decode_merge_kernel<128, 1>, 1);
  if (e != hipSuccess)
    return fail(COCKTAIL_EHIP, "decode_merge launch failed: %s (the ticket counters in plan_dev were not reset: upload the plan again)",
                hipGetErrorString(e));
  return COCKTAIL_OK;
}

}  // namespace

extern "C" int cocktail_decode_attention(const cocktail_shape* shape, const void* q, const cocktail_cache* cache,
                                         float sm_scale, void* out, float* lse, void* workspace,
                                         size_t workspace_bytes, void* stream) {
  const PlanHeader* hd = nullptr;
  if (int rc = check_plan_matches(shape, cache, &hd)) return rc;
  if (!q || !out || !workspace) return fail(COCKTAIL_EINVAL, "q, out and workspace must not be NULL");
  if (workspace_bytes < static_cast<size_t>(hd->workspace_bytes))
    return fail(COCKTAIL_ENOSPACE, "workspace holds %zu bytes, %lld needed", workspace_bytes,
                (long long)hd->workspace_bytes);
  return decode_enqueue(shape, hd, q, cache, sm_scale, out, lse, workspace, stream);
}

extern "C" int cocktail_decode_attention_marked(const cocktail_shape* shape, const void* q, const cocktail_cache* cache,
                                                float sm_scale, void* out, float* lse, void* workspace,
                                                size_t workspace_bytes, void* stream, void* event_between) {
  const PlanHeader* hd = nullptr;
  if (int rc = check_plan_matches(shape, cache, &hd)) return rc;
  if (!q || !out || !workspace || !event_between) return fail(COCKTAIL_EINVAL, "q, out, workspace and event_between must not be NULL");
  if (workspace_bytes < static_cast<size_t>(hd->workspace_bytes))
    return fail(COCKTAIL_ENOSPACE, "workspace holds %zu bytes, %lld needed", workspace_bytes,
                (long long)hd->workspace_bytes);
  return decode_enqueue(shape, hd, q, cache, sm_scale, out, lse, workspace, stream, event_between);
}

extern "C" int cocktail_decode_attention_static(const cocktail_shape* shape, const void* q, const cocktail_cache* cache,
                                                float sm_scale, void* out, float* lse, void* stream) {
  const PlanHeader* hd = nullptr;
  if (int rc = check_plan_matches(shape, cache, &hd)) return rc;
  if (!q || !out) return fail(COCKTAIL_EINVAL, "q and out must not be NULL");
  if (static_cast<size_t>(hd->workspace_bytes) > static_workspace_limit(hd))
    return fail(COCKTAIL_ENOSPACE, "this plan needs a workspace of %lld bytes, the built-in one holds %zu: use "
                "cocktail_decode_attention with a caller-supplied workspace", (long long)hd->workspace_bytes,
                static_workspace_limit(hd));
  void* ws = nullptr;
  if (int rc = static_workspace(&ws)) return rc;
  return decode_enqueue(shape, hd, q, cache, sm_scale, out, lse, ws, stream);
}

extern "C" int cocktail_decode_check(const cocktail_shape* shape, const cocktail_cache* cache, const void* workspace,
                                     void* stream) {
  const PlanHeader* hd = nullptr;
  if (int rc = check_plan_matches(shape, cache, &hd)) return rc;
  void* ws = const_cast<void*>(workspace);
  if (!ws) {
    if (static_cast<size_t>(hd->workspace_bytes) > static_workspace_limit(hd))
      return fail(COCKTAIL_ENOSPACE, "this plan does not fit the built-in workspace");
    if (int rc = static_workspace(&ws)) return rc;
  }
  const int rows = hd->batch * hd->num_q_heads;
  std::vector<int32_t> status(rows);
  hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
  if (e == hipSuccess)
    e = hipMemcpy(status.data(), static_cast<const char*>(ws) + hd->ws_status_off, sizeof(int32_t) * rows, hipMemcpyDeviceToHost);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(COCKTAIL_EHIP, "reading the status of the last decode call failed: %s", hipGetErrorString(e));
  }
  int bad = 0, first = -1;
  for (int i = 0; i < rows; ++i)
    if (status[i] != 0) {
      if (first < 0) first = i;
      ++bad;
    }
  if (bad)
    return fail(COCKTAIL_ESTATE, "the last decode call covered %d tokens too %s for sequence %d, query head %d (%d of %d rows "
                "affected; their out and lse are NaN): the counters in plan_dev were not zero when the call "
                "started, calls on this cache overlapped, or plan_dev was modified; upload the plan again",
                status[first] < 0 ? -status[first] : status[first], status[first] < 0 ? "few" : "many",
                first / hd->num_q_heads, first % hd->num_q_heads, bad, rows);
  return COCKTAIL_OK;
}
