// Internal: the decode kernel for one query head per kv head (Hq = Hkv), as templates over head_dim; one
// translation unit per head_dim instantiates launch_decode_heads<HD>.
//
// Design (gfx950, wave64):
//  * The host planner puts all 64-token blocks of a layer into one global order and cuts it into
//    groups of a few workers.  A worker (wave) streams its own block range and then takes
//    pieces of the group's shared pool through an atomic ticket counter, so that the workers of a
//    group finish together; it emits one partial softmax state per (sequence, kv head) segment it
//    touches.
//  * Inside a wave a token is owned by a PAIR of lanes: lane l works on token
//    l % 32 of a 32-token unit and on channels [64*(l/32), 64*(l/32)+64).  The block
//    layout stores the j-th 16-byte piece of all 64 tokens contiguously, so each
//    half-wave reads one contiguous 512-byte run per load instruction, and the q.k
//    dot product needs a single cross-lane add per token.  A lane keeps 64 output
//    accumulators and its half of the query in registers; the kernel stays below
//    256 VGPRs so that two waves share every SIMD and one wave's loads hide behind
//    the other's arithmetic.
//  * Codes are expanded without any conversion: a code field masked out of a
//    half-word IS an fp16 subnormal of value code * 2^(pos-24), which v_dot2_f32_f16
//    and v_fma_mix_f32 consume exactly; the power of two is folded into per-group
//    factors.  Dequantisation is folded too:
//      q.k^      = sum_g scale_g * (q.code)_g + zero_g * sum(q_g)
//      sum p v^  = sum_t (p_t scale_tg) code_t + sum_t p_t zero_tg
//  * Loads go through buffer resources (one VGPR of address per lane) and are
//    software pipelined by hand: J register stages of K units and J of V units are
//    refilled one loop iteration ahead of the arithmetic, with the units of whatever
//    piece comes next (same segment, next segment, or a pool piece).
//  * Softmax is online per lane pair: logits of J units, one lazy rescale when the
//    reference maximum grows by more than 2^8, then the V pass.  (m, l, o[D])
//    partials go to the workspace and a second small kernel merges them exactly
//    (the softmax-weighted sum does not depend on how tokens are grouped, Eq. 4-5).
//  * This kernel serves one query head per wave (one query head per kv head; ratios above eight without a divisor from
//    2 to 8; plans for the vector ALU only); the other grouped-query shapes run on the kernels of decode_quads_impl.h and
//    decode_tiles_impl.h, which share the pieces and the buffer loads with this one, the former its pools too.
#pragma once
#include <hip/hip_runtime.h>

#include "decode_common.h"

namespace cocktail {

// One lazy-rescale step of a lane's online softmax followed by p_j = 2^(s_j - m).
template <int NGH, int J>
__device__ __forceinline__ void softmax_step(const float (&s)[J], float (&p)[J], LaneState<NGH>& st) {
  float smax = s[0];
#pragma unroll
  for (int jj = 1; jj < J; ++jj) smax = fmaxf(smax, s[jj]);
  // the reference maximum only moves when it is exceeded by more than 2^8, and then for the whole
  // wave at once (to the largest logit any lane has seen): the lanes share one reference, so the
  // number of rescales per state is that of one running maximum, not of 64 independent ones
  const bool grow = smax > st.m + kRescaleThreshold;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(grow) != 0, 0)) {
    const float mnew = wave_max(fmaxf(smax, st.m));
    const float alpha = __builtin_amdgcn_exp2f(st.m - mnew);
    st.m = mnew;
    st.l *= alpha;
#pragma unroll
    for (int d = 0; d < DH; ++d) st.acc[d] *= alpha;
#pragma unroll
    for (int g = 0; g < NGH; ++g) st.zacc[g] *= alpha;
  }
#pragma unroll
  for (int jj = 0; jj < J; ++jj) {
    p[jj] = __builtin_amdgcn_exp2f(s[jj] - st.m);
    st.l += p[jj];
  }
}

// Writes this wave's partial state: (m, l, o[HD]) summed over its lanes, and the number of tokens it covers.
// The lanes share one reference m, so nothing is rescaled.  The sums over the token lanes halve the number of values a
// lane holds step by step: 130 instructions in registers.  Through a shared-memory tile, sixteen channels at a time, a
// flush took 1.5 us of a worker's 6 on a 2K-token layer (32K tokens, 32 heads: 36.3 -> 35.4 us per call; 128K, 40 heads:
// 107.4 -> 106.3; four heads per wave, INT8 mix, 4 x 64K tokens: 62.2 -> 60.6, its other mixes gain 0.5 %).
template <int HD, int NGH, int GL, class SLOT>
__device__ __forceinline__ void flush_partial(const LaneState<NGH>& st, SLOT out, int r, int lane, int tokens) {
  constexpr int UT = Geo<HD>::UT;       // lanes that hold different tokens
  const float lw = token_sum<UT>(st.l);
  float z[NGH];
#pragma unroll
  for (int g = 0; g < NGH; ++g) z[g] = token_sum<UT>(st.zacc[g]);
  const int at = r * ((HD + kPartialFloats) * 4);
  if (lane == 0) put_header(out, at, st.m, lw, tokens);
  // after the folds lane (bits b5 .. b0) holds channels 32 b4 + 16 b3 + 8 b2 + 4 b1 + 2 b0 + {0, 1} of its half (head_dim
  // 64: one channel, 32 b5 + 16 b4 + 8 b3 + 4 b2 + 2 b1 + b0); a channel's group is bit 4 (b4; b5) of 64 channels at G 32
  float v[32];
  if constexpr (HD == 64) {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = fold32(st.acc[i], st.acc[i + 32]);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = fold16(v[i], v[i + 16]);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fold8(v[i], v[i + 8]);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fold7(v[i], v[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = fold2(v[i], v[i + 2], lane & 2);
    v[0] = fold1(v[0], v[1], lane & 1);
    const float zz = NGH == 2 ? (lane & 32 ? z[NGH - 1] : z[0]) : z[0];
    put(out, at + (kPartialFloats + lane) * 4, v[0] + zz);
  } else {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = fold16(st.acc[i], st.acc[i + 32]);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = fold8(v[i], v[i + 16]);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fold7(v[i], v[i + 8]);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fold2(v[i], v[i + 4], lane & 2);
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = fold1(v[i], v[i + 2], lane & 1);
    const float zz = NGH == 2 ? (lane & 16 ? z[NGH - 1] : z[0]) : z[0];
    put(out, at + (kPartialFloats + 2 * lane) * 4, float2{v[0] + zz, v[1] + zz});
  }
}

// Zeroes the partial state and loads this lane's half of the query row `qrow`.
template <int HD, int NGH, int GL>
__device__ __forceinline__ void begin_state(int qrow, int h, LaneState<NGH>& st, uint32_t (&q)[DH / 2],
                                            float (&qsum)[NGH]) {
#pragma unroll
  for (int i = 0; i < DH; ++i) st.acc[i] = 0.f;
#pragma unroll
  for (int gq = 0; gq < NGH; ++gq) st.zacc[gq] = 0.f;
  st.m = kNegBig;
  st.l = 0.f;
  const u32x4* qp = reinterpret_cast<const u32x4*>(kparams()->q + int64_t(qrow) * (HD / 2) + h * (DH / 2));
#pragma unroll
  for (int i = 0; i < DH / 8; ++i) {
    const u32x4 v = qp[i];
    q[4 * i] = v.x, q[4 * i + 1] = v.y, q[4 * i + 2] = v.z, q[4 * i + 3] = v.w;
  }
#pragma unroll
  for (int gq = 0; gq < NGH; ++gq) {
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < GL / 2; ++i) a = dot2(q[gq * (GL / 2) + i], 0x3C003C00u, a);   // (1.0, 1.0)
    qsum[gq] = a;
  }
}

// Consumes the stream while its pieces belong to class CID, starting with `cur` (whose loads have
// not been issued yet); returns with `cur` = the first piece of another class, or the end piece.
//
// J register stages hold the K units and J the V units of the piece being worked on; each stage is
// refilled with the corresponding unit of the NEXT piece as soon as it has been consumed, so the
// loads of a piece are in flight during the arithmetic of the piece before it, across segment and
// pool boundaries alike.  A piece with fewer than J units leaves stages unused, and after the last
// piece of the class nothing is left to fetch: those refills address the first unit past the segment,
// which the buffer resource answers with zeros without touching memory, so the loop body has no
// branches around the loads (the zeros are masked like padding).  The accumulators live and die inside this function, one
// instance per class.
template <int HD, class CLS, int CID, int G, int AUX, class DEST = Workspace<HD>, class STREAM = Stream<HD>>
__device__ __forceinline__ void run_class(STREAM& sm, Piece& cur, int r, int lane, bool app = false, DEST dest = {}) {
  constexpr int NGH = CLS::NGH;
  constexpr int GL = G < DH ? G : DH;
  constexpr int J = DEST::kOne ? 1 : CLS::J;
  constexpr int UT = Geo<HD>::UT, UPB = Geo<HD>::UPB;
  static_assert(DEST::kOne || J == kIterUnits[CID], "the planner cuts pool pieces to the kernel's iteration size");
  const int t = lane % UT, h = lane / UT;
  const uint32_t vc = CLS::code_voff(t, h), vm = CLS::meta_voff(t, h);
  const char* const kbase = uni(app ? kparams()->k_app : kparams()->k[CID]);   // app: the append buffers
  const char* const vbase = uni(app ? kparams()->v_app : kparams()->v[CID]);
  const float scale_log2 = kparams()->scale_log2;
  LaneState<NGH> st;
  uint32_t q[DH / 2];
  float qsum[NGH];
  typename CLS::Stage ks[J], vs[J];
  int pid = cur.pid;
  // `cur` is the piece the stream produced last, so the stream's segment fields describe it
  rsrc_t krs = make_rsrc(kbase + int64_t(sm.blk0) * CLS::BLOCKB, uint32_t(sm.nblk) * CLS::BLOCKB);
  rsrc_t vrs = make_rsrc(vbase + int64_t(sm.blk0) * CLS::BLOCKB, uint32_t(sm.nblk) * CLS::BLOCKB);
  int ru = cur.us, rn = cur.nu;   // the piece the stages are (re)filled with
  int roob = UPB * sm.nblk;       // first unit past its segment: a load from there is out of range and costs nothing
#pragma unroll
  for (int jj = 0; jj < J; ++jj) CLS::template load<AUX>(ks[jj], krs, jj < rn ? ru + jj : roob, vc, vm);
#pragma unroll
  for (int jj = 0; jj < J; ++jj) CLS::template load<AUX>(vs[jj], vrs, jj < rn ? ru + jj : roob, vc, vm);
  sched_fence();
  begin_state<HD, NGH, GL>(sm.qrow + r, h, st, q, qsum);   // the query arrives while the first units are on their way
  int valid = cur.valid;
  int covered = 0;   // tokens the current partial state covers (the merge checks the total per sequence)
  Piece nxt = sm.next(lane);
#pragma unroll 1
  while (true) {
    const bool more = nxt.nu > 0 && nxt.cls == CID;
    if (more) {
      krs = make_rsrc(kbase + int64_t(sm.blk0) * CLS::BLOCKB, uint32_t(sm.nblk) * CLS::BLOCKB);
      vrs = make_rsrc(vbase + int64_t(sm.blk0) * CLS::BLOCKB, uint32_t(sm.nblk) * CLS::BLOCKB);
      ru = nxt.us, rn = nxt.nu, roob = UPB * sm.nblk;
    } else {
      rn = 0;   // nothing follows in this class: every refill goes out of range
    }
    covered += valid;
    float s[J], p[J];
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
      s[jj] = CLS::half_logit(ks[jj], q, qsum);
      sched_fence();
      CLS::template load<AUX>(ks[jj], krs, jj < rn ? ru + jj : roob, vc, vm);
      sched_fence();
    }
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
      float full = s[jj];
      if constexpr (HD == 128) full = both_halves(full, false);   // both halves of the token
      full *= scale_log2;
      s[jj] = (jj * UT + t < valid) ? full : -INFINITY;
    }
    softmax_step<NGH, J>(s, p, st);
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
      CLS::accumulate(vs[jj], p[jj], st);
      sched_fence();
      CLS::template load<AUX>(vs[jj], vrs, jj < rn ? ru + jj : roob, vc, vm);
      sched_fence();
    }
    if (!more || nxt.fresh) flush_partial<HD, NGH, GL>(st, dest.slot(pid), r, lane, covered);
    if (!more) break;
    if (nxt.fresh) {
      pid = nxt.pid;
      covered = 0;
      begin_state<HD, NGH, GL>(sm.qrow + r, h, st, q, qsum);
    }
    valid = nxt.valid;
    nxt = sm.next(lane);
  }
  cur = nxt;
}

// Workgroups behind the regular workers attend to the tokens appended during decoding (Sec. III-A): FP16 runs in
// the append buffers, one wave per slice of a (sequence, kv head)'s run, each writing one of the last
// partials of that head's range.
template <int HD, int G, int AUX>
__device__ __forceinline__ void appended_tokens(int idx, int r, int lane) {
  const AppendSlice a = append_slice(idx);
  if (a.tokens <= 0) {
    write_neutral<HD>(a.pid, r, lane);
    return;
  }
  Stream<HD> sm;
  sm.init_run(kFp16Class, a.tokens, a.first_block, a.blocks, a.qrow, a.pid);
  Piece cur = sm.next(lane);
  if (cur.nu > 0) run_class<HD, HalfClass<HD, G>, kFp16Class, G, AUX>(sm, cur, r, lane, true);
}

// One wave per worker (Hq = Hkv: the query head of a kv head is that head).  INT8: the cache
// has an INT8 class; caches without one run a kernel without that code (a third less of it to fetch and
// to allocate registers for, worth 1.5 us on a 32K-token layer).
template <int HD, int G, int AUX, bool INT8>
__global__ __launch_bounds__(64 * kCuWaves) __attribute__((amdgpu_waves_per_eu(2))) void decode_attention_kernel(COCKTAIL_WORKER_ARGS) {
  constexpr int r = 0;             // query head inside the kv head's group
#ifdef COCKTAIL_TRACE
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
#endif
  const FirstParams fp = {recs, num_workers, num_q_heads, rep};
  const Place me = place(fp);
  const int lane = me.lane;
  if (me.worker >= fp.num_workers) {
    appended_tokens<HD, G, AUX>(me.worker - fp.num_workers, r, lane);
    return;
  }
  Stream<HD> sm;
  WorkerRec rec = load_record(fp.recs + me.worker);
  touch_params(rec.g0);
  sm.init(rec, fp);
  Piece cur = sm.next(lane);
  while (cur.nu > 0) {
    if (cur.cls == 0) {
      run_class<HD, QuantClass<HD, 2, G>, 0, G, AUX>(sm, cur, r, lane);
    } else if (cur.cls == 1) {
      run_class<HD, QuantClass<HD, 4, G>, 1, G, AUX>(sm, cur, r, lane);
    } else if (INT8 && cur.cls == 2) {
      if constexpr (INT8) run_class<HD, QuantClass<HD, 8, G>, 2, G, AUX>(sm, cur, r, lane);
    } else {
      run_class<HD, HalfClass<HD, G>, kFp16Class, G, AUX>(sm, cur, r, lane);
    }
  }
  // pool parts this worker never entered still own a partial slot: fill it with the neutral state
  for (int i = 0; i < sm.nps; ++i) {
    if ((sm.used >> i) & 1u) continue;
    const PoolSeg ps = load_record(kparams()->psegs + sm.pseg0 + i);
    if (sm.rank < ps.nslots) write_neutral<HD>(ps.slot0 + sm.rank, r, lane);
  }
#ifdef COCKTAIL_TRACE
  if (lane == 0) {
    uint64_t* tr = kparams()->trace + me.worker * 4;
    tr[0] = t_start;
    tr[1] = __builtin_amdgcn_s_memrealtime();
    tr[2] = __builtin_amdgcn_s_getreg((4) | (0 << 6) | (31 << 11));    // HW_ID
    tr[3] = __builtin_amdgcn_s_getreg((20) | (0 << 6) | (31 << 11));   // XCC_ID
  }
#endif
}

// Picks the instance for the group size, the cache policy and the classes present, and launches it.
template <int HD>
hipError_t launch_decode_heads(const DecodeParams& p, int group_size, bool nt, bool int8, int grid, hipStream_t st) {
  worker_kernel kern = nullptr;
#define COCKTAIL_PICK(G)                                                                                                      \
  kern = int8 ? (nt ? decode_attention_kernel<HD, G, kAuxNonTemporal, true> : decode_attention_kernel<HD, G, kAuxDefault, true>) \
              : (nt ? decode_attention_kernel<HD, G, kAuxNonTemporal, false> : decode_attention_kernel<HD, G, kAuxDefault, false>)
  if (group_size == 32) {
    COCKTAIL_PICK(32);
  } else if (group_size == 64) {
    COCKTAIL_PICK(64);
  } else if constexpr (HD >= 128) {
    COCKTAIL_PICK(128);
  }
#undef COCKTAIL_PICK
  if (!kern) return hipErrorInvalidValue;   // a group size larger than head_dim: refused by the shape check before
  return launch_workers(kern, p, grid, 0, st);
}

}  // namespace cocktail
