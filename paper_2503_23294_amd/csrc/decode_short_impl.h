// Internal: the decode kernels for short contexts, as templates over head_dim; the translation units of the kernel families instantiate them.
//
// Where every wave has a few loop iterations of work at most, a call is bound by chains of latencies: launch, record, blocks, flush, a
// second launch, and its own chain over the partial states of the first.  Here a workgroup of eight waves works on one row (sequence,
// work head) and merges its eight states in shared memory; a row that one workgroup holds is finished there, and otherwise
// the last workgroup of a row merges what the others have written through to memory (a state per workgroup, counted by one
// atomic each: short_count.h).  One launch instead of two.
//
// Measured (us, two launches -> one; calls back to back, device time alone in brackets): 8 heads 2K 10.0 -> 7.5 [9.6 -> 7.5], 32 heads 5.3K
// [12.9 -> 9.7], appended tokens at 1 to 2K [16.4 -> 9.4, 15.9 -> 11.0]; 60 random short shapes 0.81 in the geometric mean.  Of the 7.5: launch, record
// and blocks 4, fold in shared memory 0.7, write-through store, count and the last workgroup's fold 1.5.  A plan grows by 144 bytes per workgroup and 64
// per row for it (8 heads 2K by 9.7 KB, the largest by 37 to 53).
// What one launch for all contexts costs where the chip is full (a worker's states written through, the merge by the last wave of a row): 4 x
// 64K at four heads 66 -> 68, 4 x 128K at eight 126 -> 128.5, 8 x 32K at 40 heads 73.7 -> 76.6; those keep two.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "decode_heads_impl.h"
#include "decode_tiles_impl.h"
#include "short_count.h"

namespace cocktail {

constexpr int kAuxWriteThrough = 16;   // sc1: device scope

// The arguments are laid out like those of the other decode kernels (kparams).
#define COCKTAIL_SHORT_ARGS const ShortRec *recs, const ShortGroup *place, int32_t rep, int32_t counters_offset, DecodeParams
typedef void (*short_kernel)(COCKTAIL_SHORT_ARGS);
static_assert(LastArgument<short_kernel>::offset() == kParamsOffset, "kparams finds them where the other kernels have them");

// Shared memory for the states of a row (in whole batches of the fold), those of the slices they are folded in where they are more than
// kShortDirect, and a flag.
constexpr int kShortDirect = 16;
template <int HD>
constexpr int kShortBytes = (kShortStates + 8 * kCuWaves) * (HD + kPartialFloats) * 4 + 16;

struct ShortWave {
  int wave, lane;
  ShortRec rec;
  ShortGroup group;
};
__device__ __forceinline__ ShortWave short_wave(const ShortRec* recs, const ShortGroup* place) {
  ShortWave w;
  w.wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), w.lane = int(threadIdx.x) & 63;
  w.rec = load_record(recs + int(blockIdx.x) * kCuWaves + w.wave);
  w.group = load_record(place + int(blockIdx.x));
  touch_params(w.rec.cls);
  return w;
}

__device__ __forceinline__ uint32_t* counters_of(const ShortGroup* place, int offset) {
  return reinterpret_cast<uint32_t*>(reinterpret_cast<uint64_t>(place) + offset);
}

// The wave's range as a stream of pieces (Stream without segments to enter and without pools).
template <int HD, bool ONE, bool STAGED>
struct ShortStream {
  static constexpr int UT = Geo<HD>::UT;
  int u, u1, cls, ntok, blk0, nblk, qrow;

  __device__ __forceinline__ explicit ShortStream(const ShortWave& w) {
    u = w.rec.range & 0xffff, u1 = w.rec.range >> 16, cls = w.rec.cls, ntok = w.rec.ntok, blk0 = w.rec.blk0, qrow = w.group.qrow;
    nblk = (ntok + kTB - 1) / kTB;
    if (cls == kNumClasses) {
      const uint32_t inverse = uint32_t(ntok);
      ntok = appended_count(w.group.b), nblk = kparams()->app_blocks, cls = kFp16Class;
      const int units = (ntok + UT - 1) / UT, parts = u1;
      const int each = parts == 1 ? units : int(uint64_t(uint32_t(units + parts - 1)) * inverse >> 32);   // (divided as scalars)
      u1 = min(u * each + each, units), u = min(u * each, units);
    }
  }
  __device__ __forceinline__ Piece next(int) {
    Piece d;
    d.nu = min(!ONE ? iter_units(cls) : STAGED && cls < 2 ? Geo<HD>::UPB : 1, u1 - u), d.us = u;
    d.valid = max(0, min(ntok - u * UT, d.nu * UT));
    d.cls = cls, d.fresh = 0, d.pid = 0;
    u += d.nu;
    return d;
  }
};

// Other XCDs see the store, and no L2 holds it back to write it later.
template <class T>
__device__ __forceinline__ void write_through(T* p, T x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Counts this workgroup of a row (short_count.h); true if it is the one that merges.  For one lane.
__device__ __forceinline__ bool short_arrives(__attribute__((address_space(1))) uint64_t* word, uint64_t step, uint32_t groups) {
  auto add = [&] { return __hip_atomic_fetch_add(word, step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto to_zero = [&](uint64_t& from) { return __hip_atomic_compare_exchange_strong(word, &from, uint64_t(0), __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  uint64_t all = groups * step, old = add();
  if (__builtin_expect(old + step != all && !short_own(old, step), 0)) {
    uint64_t now = old + step;
    for (int i = 0; i < kShortHealTries && !short_own(now, step) && !to_zero(now); ++i);
    old = add();
  }
  if (old + step != all) return false;
  to_zero(all);
  return true;
}

// A state without tokens.
template <int HD>
__device__ __forceinline__ void short_empty(char* slot, int rep, int lane) {
  constexpr int STRIDE = (HD + kPartialFloats) * 4;
  for (int i = lane; i < rep * (STRIDE / 16); i += 64) {
    const float m = i % (STRIDE / 16) == 0 ? -INFINITY : 0.f;
    *reinterpret_cast<float4*>(slot + i * 16) = float4{m, 0.f, 0.f, 0.f};
  }
}

// The waves' states are in shared memory: the workgroup's state, then the row's.  The instructions of a part that runs once are fetched at the
// speed of a read from memory (caches start cold with every launch), so the last workgroup of a row copies the states of the others to where those
// of its waves were and runs the same fold again: with a fold of its own for them, unrolled, it took 2.2 us instead of 0.7.
template <int HD>
__device__ __forceinline__ void short_finish(char* states, const ShortWave& w, uint32_t* counters, int rep) {
  constexpr int QUADS = HD / 4, STRIDE = (HD + kPartialFloats) * 4, U = kCuWaves;
  const int tid = threadIdx.x, head = tid / QUADS, quad = tid % QUADS;   // a thread folds four channels of a head
  const bool mine = head < rep;
  const int group = int(blockIdx.x), index = w.group.place & 0xff, groups = w.group.place >> 8 & 0xfff, counter = w.group.place >> 20;
  const int expected = w.group.context + appended_count(w.group.b);
  const rsrc_t rs = make_rsrc(reinterpret_cast<const char*>(kparams()->ws) + int64_t(group - index) * rep * STRIDE, uint32_t(groups * rep * STRIDE));
  // 2^(x - reference); a state without tokens (reference and x are -inf) has weight 0
  auto weight = [](float x, float reference) { return x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x - reference); };
  const char* from = states;
  int count = kCuWaves;
  bool last = groups == 1;
  const uint64_t step = short_step(reinterpret_cast<uint64_t>(__builtin_amdgcn_dispatch_ptr()));
  auto* const word = reinterpret_cast<__attribute__((address_space(1))) uint64_t*>(reinterpret_cast<uint64_t>(counters + counter * kShortCounterStride));
#pragma unroll 1
  while (true) {
    __syncthreads();
    float m = -INFINITY, l = 0.f;
    f4 o = splat(0.f);
    int covered = 0;
    if (mine) {
#pragma unroll 1
      for (int i0 = 0; i0 < count; i0 += U) {   // (slots behind the last state of a batch hold zeros)
        f4 hd[U], va[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const char* const at = from + ((i0 + u) * rep + head) * STRIDE;
          hd[u] = *reinterpret_cast<const f4*>(at), va[u] = *reinterpret_cast<const f4*>(at + 16 + quad * 16);
        }
        float top = m;
#pragma unroll
        for (int u = 0; u < U; ++u) hd[u].x = i0 + u < count ? hd[u].x : -INFINITY, top = fmaxf(top, hd[u].x);
        const float a = weight(m, top);
        m = top, l *= a, o *= a;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float x = weight(hd[u].x, top);
          l += hd[u].y * x, o += va[u] * x;
          covered += __float_as_int(hd[u].z);
        }
      }
    }
    if (last) {
      if (!mine) return;
      kparams_t kp = kparams();
      const bool empty = !(l > 0.f), sound = covered == expected;
      const int row = w.group.qrow + head;
      typedef _Float16 h4 __attribute__((ext_vector_type(4)));
      h4 res;
#pragma unroll
      for (int i = 0; i < 4; ++i) res[i] = static_cast<_Float16>(!sound ? __builtin_nanf("") : empty ? 0.f : o[i] / l);
      *reinterpret_cast<h4*>(kp->out + int64_t(row) * HD + quad * 4) = res;
      if (quad == 0) {
        kp->status[row] = covered - expected;
        if (kp->lse) kp->lse[row] = !sound ? __builtin_nanf("") : empty ? -INFINITY : (m + log2f(l)) * 0.6931471805599453f;
      }
      return;
    }
    if (mine) {
      const uint32_t at = (index * rep + head) * STRIDE;
      const f4 hd = {m, l, __int_as_float(covered), 0.f};
      if (quad == 0) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hd), rs, at, 0, kAuxWriteThrough);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rs, at + 16 + quad * 16, 0, kAuxWriteThrough);
      if (index == 0) {   // until the row is merged
        kparams_t kp = kparams();
        const int row = w.group.qrow + head;
        write_through(reinterpret_cast<uint64_t*>(kp->out + int64_t(row) * HD + quad * 4), uint64_t(0x7e007e007e007e00));
        if (quad == 0) {
          write_through(kp->status + row, short_pending(expected));
          if (kp->lse) write_through(kp->lse + row, __builtin_nanf(""));
        }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // written through: other XCDs see it
    if (rep * QUADS > 64) __syncthreads();             // by more than the first wave
    int* const flag = reinterpret_cast<int*>(states + kShortBytes<HD>) - 4;
    if (tid == 0) *flag = short_arrives(word, step, groups);
    __syncthreads();
    if (!uni(*flag)) return;
    asm volatile("" ::: "memory");
    count = groups, last = true;
    const int bytes = (groups + U - 1) / U * U * rep * STRIDE;   // (past the last state: zeros)
#pragma unroll 2
    for (int at = tid * 16; at < bytes; at += kShortThreads * 16)
      *reinterpret_cast<u32x4*>(states + at) = load16<kAuxWriteThrough>(rs, at, 0);
    if (__builtin_expect(groups > kShortDirect, 0)) {
      // many: every thread of the workgroup folds some of them first
      const int shift = rep <= 1 ? 0 : rep <= 2 ? 1 : rep <= 4 ? 2 : 3;
      const int h = head & ((1 << shift) - 1), slice = head >> shift, slices = kShortThreads / QUADS >> shift;
      char* const to = states + kShortStates * STRIDE;
      __syncthreads();
      if (h < rep) {
        f4 s = splat(0.f), t = {-INFINITY, 0.f, 0.f, 0.f};
        int c = 0;
#pragma unroll 1
        for (int i = slice; i < groups; i += slices) t.x = fmaxf(t.x, *reinterpret_cast<const float*>(states + (i * rep + h) * STRIDE));
#pragma unroll 2
        for (int i = slice; i < groups; i += slices) {
          const char* const at = states + (i * rep + h) * STRIDE;
          const f4 hd = *reinterpret_cast<const f4*>(at);
          const float x = weight(hd.x, t.x);
          t.y += hd.y * x, s += *reinterpret_cast<const f4*>(at + 16 + quad * 16) * x;
          c += __float_as_int(hd.z);
        }
        t.z = __int_as_float(c);
        for (int i = slice; i < U; i += slices) {   // (zeros behind the last slice)
          char* const at = to + (i * rep + h) * STRIDE;
          if (quad == 0) *reinterpret_cast<f4*>(at) = t;
          *reinterpret_cast<f4*>(at + 16 + quad * 16) = s;
          t = s = splat(0.f);
        }
        if (slice >= U) {
          char* const at = to + (slice * rep + h) * STRIDE;
          if (quad == 0) *reinterpret_cast<f4*>(at) = t;
          *reinterpret_cast<f4*>(at + 16 + quad * 16) = s;
        }
      }
      from = to, count = slices;
    }
  }
}

#define COCKTAIL_SHORT_BEGIN(STAGED)                                                        \
  extern __shared__ __attribute__((aligned(16))) char shared[];                       \
  const ShortWave w = short_wave(recs, place);                                        \
  int slot = w.wave * rep * ((HD + kPartialFloats) * 4);                              \
  asm("" : "+v"(slot)); /* not one value with the scalar addresses of the staged blocks */ \
  const SharedStates<ONE> dest = {shared + slot};                                     \
  ShortStream<HD, ONE, STAGED> sm(w);                                                 \
  Piece cur = sm.next(w.lane);                                                        \
  const bool app = w.rec.cls == kNumClasses;

// one query head per wave
template <int HD, int G, bool INT8, bool ONE>
__global__ __launch_bounds__(kShortThreads) __attribute__((amdgpu_waves_per_eu(2))) void decode_short_heads_kernel(COCKTAIL_SHORT_ARGS) {
  COCKTAIL_SHORT_BEGIN(false)
  if (cur.nu <= 0) short_empty<HD>(dest.p, rep, w.lane);
  else if (cur.cls == 0) run_class<HD, QuantClass<HD, 2, G>, 0, G, kAuxDefault>(sm, cur, 0, w.lane, false, dest);
  else if (cur.cls == 1) run_class<HD, QuantClass<HD, 4, G>, 1, G, kAuxDefault>(sm, cur, 0, w.lane, false, dest);
  else if (INT8 && cur.cls == 2) {
    if constexpr (INT8) run_class<HD, QuantClass<HD, 8, G>, 2, G, kAuxDefault>(sm, cur, 0, w.lane, false, dest);
  } else run_class<HD, HalfClass<HD, G>, kFp16Class, G, kAuxDefault>(sm, cur, 0, w.lane, app, dest);
  short_finish<HD>(shared, w, counters_of(place, counters_offset), rep);
}

// two to four
template <int HD, int G, bool INT8, bool ONE>
__global__ __launch_bounds__(kShortThreads) __attribute__((amdgpu_waves_per_eu(2))) void decode_short_quads_kernel(COCKTAIL_SHORT_ARGS) {
  COCKTAIL_SHORT_BEGIN(false)
  if (cur.nu <= 0) short_empty<HD>(dest.p, rep, w.lane);
  else if (cur.cls == 0) run_quads<HD, QuadQuant<HD, 2, G>, 0, G, kAuxDefault>(sm, cur, w.lane, false, dest);
  else if (cur.cls == 1) run_quads<HD, QuadQuant<HD, 4, G>, 1, G, kAuxDefault>(sm, cur, w.lane, false, dest);
  else if (INT8 && cur.cls == 2) {
    if constexpr (INT8) run_quads<HD, QuadQuant<HD, 8, G>, 2, G, kAuxDefault>(sm, cur, w.lane, false, dest);
  } else run_quads<HD, QuadHalf<HD, G>, kFp16Class, G, kAuxDefault>(sm, cur, w.lane, app, dest);
  short_finish<HD>(shared, w, counters_of(place, counters_offset), rep);
}

// five to eight: a staged block per iteration only
template <int HD, int G, bool INT8>
__global__ __launch_bounds__(kShortThreads) __attribute__((amdgpu_waves_per_eu(2))) void decode_short_tiles_kernel(COCKTAIL_SHORT_ARGS) {
  constexpr bool ONE = true;
  COCKTAIL_SHORT_BEGIN(true)
  char* const lds = shared + kCuWaves * rep * ((HD + kPartialFloats) * 4) + w.wave * kTileLds;   // (free when the states of a row come in)
  if (cur.nu <= 0) short_empty<HD>(dest.p, rep, w.lane);
  else if (cur.cls == 0) run_tiles_lds<HD, 2, 0, G, kAuxDefault>(sm, cur, lds, w.lane, dest);
  else if (cur.cls == 1) run_tiles_lds<HD, 4, 1, G, kAuxDefault>(sm, cur, lds, w.lane, dest);
  else if (INT8 && cur.cls == 2) {
    if constexpr (INT8) run_tiles<HD, 8, 2, G, kAuxDefault>(sm, cur, w.lane, false, dest);
  } else run_tiles<HD, 16, kFp16Class, G, kAuxDefault>(sm, cur, w.lane, app, dest);
  short_finish<HD>(shared, w, counters_of(place, counters_offset), rep);
}
#undef COCKTAIL_SHORT_BEGIN

template <int HD>
hipError_t launch_decode_short(const DecodeParams& p, const ShortRec* recs, const ShortGroup* place, int counters_offset, bool quads, int group_size, bool int8, bool one,
                               int groups, hipStream_t st) {
  short_kernel kern = nullptr;
  const bool tiles = quads && uses_tiles(p.rep);
  if (tiles && !one) return hipErrorInvalidValue;   // not a split the planner makes
#define COCKTAIL_PICK3(G, I8, ONE)                                       \
  kern = tiles ? decode_short_tiles_kernel<HD, G, I8>                    \
         : quads ? decode_short_quads_kernel<HD, G, I8, ONE> : decode_short_heads_kernel<HD, G, I8, ONE>
#define COCKTAIL_PICK2(G, I8)            \
  if (one) COCKTAIL_PICK3(G, I8, true);  \
  else COCKTAIL_PICK3(G, I8, false)
#define COCKTAIL_PICK(G)             \
  if (int8) { COCKTAIL_PICK2(G, true); } \
  else { COCKTAIL_PICK2(G, false); }
  if (group_size == 32) {
    COCKTAIL_PICK(32);
  } else if (group_size == 64) {
    COCKTAIL_PICK(64);
  } else if constexpr (HD >= 128) {
    COCKTAIL_PICK(128);
  }
#undef COCKTAIL_PICK
#undef COCKTAIL_PICK2
#undef COCKTAIL_PICK3
  if (!kern) return hipErrorInvalidValue;   // a group size larger than head_dim: refused by the shape check before
  const size_t lds = tiles ? std::max<size_t>(kShortBytes<HD>, kCuWaves * (p.rep * ((HD + kPartialFloats) * 4) + kTileLds)) : kShortBytes<HD>;
  return launch_lds(kern, dim3(groups), dim3(kShortThreads), lds, st, recs, place, p.rep, counters_offset, p);
}

}  // namespace cocktail
