// Internal: the decode kernel for five to eight query heads per wave, as templates over head_dim; one
// translation unit per head_dim instantiates launch_decode_tiles<HD>.
//
// Decode side of Alg. 1 (Sec. III-C).  One wave serves all (up to eight) query heads of a set, so every K/V byte is
// fetched and unpacked once.  The contractions run on the 16x16x32 fp16 matrix instruction,
//     D[i][j] += sum_k A[i][k] B[k][j],   lane 16 g + c: A row c and B column c for k = 8 g .. 8 g + 7;
//                                         D column c, rows 4 g .. 4 g + 3.
// Sixteen rows for eight heads: row 8 par + head.  The two halves par = 0, 1 are two channel groups, each with
// its own scale, so that one instruction makes the sums of two groups at once and half of what it computes is not
// thrown away:
//  * q.k:  A = query, row (head, par) holding the head's channels of the half par of a token's row and zero for the
//          other half's; B = sixteen tokens, lane (g, c) holding 8 channels of token c out of half g >> 1.  Column =
//          token, so a lane has the sums of its own token for four heads and one half: it applies the scale and zero
//          of its token and group (the first load of a lane's scale/zero pairs), and two sets of sixteen tokens
//          trade halves (v_permlane32_swap) so that one addition leaves 32 tokens x 8 heads in four registers per
//          lane, none of them twice: the softmax does no work for copies.
//  * p.V:  A = p_t scale_tg, row (head, par), k = 32 tokens; B = V in token quads: a lane holds 8 tokens (two quads)
//          of one channel per instruction.  The columns belong to two groups, one per half; the rows of half par are
//          meant for the columns of the same half, the other quarter blocks of D are dropped at the flush.
//          p is made with "lane = token, register = head"; one product with a 0/1 matrix per sixteen tokens turns it
//          into "lane = (head, half), register = token".
// The reductions over tokens happen inside the matrix unit, so a flush writes the accumulators as they are.
// Codes, scales, the reference m and the fp16 rounding of p * scale are treated as in decode_quads_impl.h: codes go in as
// fp16 subnormals (exact), scale and zero are applied to 32-bit sums, and what the rounding of p * scale loses is fed
// back around the middle of the code range (sum of the rounded weights: a product with a column of ones).
//
// Bound by memory and, for the INT2 class, by the vector ALU (busy 90 % of a call on INT2 blocks of G 32): 190 vector and 22
// matrix instructions per 32 INT2 tokens and eight heads at G 32 (151 and 19 at G 64; the loop of the built kernel without its
// rescale), where a pair of waves with four heads each took 280 + 64.
// 4 x 128K tokens, 64 query / 8 kv heads (759 MB): 182.5 -> 126.5 us per call; 8 ragged sequences, 64 q / 4 kv heads (two
// sets per kv head): 92 -> 60 us, 47.5 with the sets as twins and ranges that end where runs end (plan.hip); 8 x 16K tokens and 300 appended, 64 q / 8 kv heads:
// 66.5 -> 47.2 us.
#pragma once
#include <hip/hip_runtime.h>

#include "decode_common.h"
#include "decode_quads_impl.h"

namespace cocktail {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f4 mfma16(u32x4 a, u32x4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// N dwords at a lane's offset, in the widest loads that fit; more than 16 bytes continue in the next piece of the row
template <int N>
struct Words {
  static_assert(N == 1 || N == 2 || N % 4 == 0, "a piece is 16 bytes");
  static constexpr int V = N < 4 ? N : 4;
  typedef uint32_t vec __attribute__((ext_vector_type(V)));
  vec v[N / V];
  __device__ __forceinline__ uint32_t operator[](int i) const {
    if constexpr (N == 1) return v[0][0];
    else return v[i / V][i % V];
  }
  template <int AUX>
  __device__ __forceinline__ void load(rsrc_t rs, uint32_t voff, uint32_t soff) {
    if constexpr (N == 1) {
      v[0][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, AUX);
    } else if constexpr (N == 2) {
      v[0] = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, AUX);
    } else {
#pragma unroll
      for (int p = 0; p < N / 4; ++p) v[p] = load16<AUX>(rs, voff, soff + p * (kTB * 16));
    }
  }
  __device__ __forceinline__ void read(const char* lds) {
    if constexpr (N == 1) {
      v[0][0] = *reinterpret_cast<const uint32_t*>(lds);
    } else {
#pragma unroll
      for (int p = 0; p < N / V; ++p) v[p] = *reinterpret_cast<const vec*>(lds + p * (kTB * 16));
    }
  }
};

// How a wave holds one class.  A unit (Geo<HD>::UT tokens) is GR granules of 32 tokens, a granule two sets of 16.
template <int HD, int BITS, int G>
struct TileClass {
  static constexpr bool QUANT = BITS < 16;
  static constexpr int UT = Geo<HD>::UT, UPB = Geo<HD>::UPB, GR = UT / 32;
  static constexpr int NG = HD / G;                        // scale/zero pairs per token
  static constexpr bool FOUR = QUANT && NG == 4;           // four groups: two per half, one after the other
  static constexpr int NR = FOUR ? 2 : 1;                  // chains of K sums with scales of their own
  static constexpr int M = HD / 32;                        // matrix instructions per sixteen tokens
  static constexpr int CPL = M / NR;                       // of them per chain: 8 channels of the lane's token each
  static constexpr int NA = FOUR ? 2 : 1;                  // A operands of the V side: (head, half) x tokens
  static constexpr int ES = HD == 128 && !FOUR ? 8 : 4;    // channels a lane has per A operand
  static constexpr int NPOS = QUANT ? 8 / BITS : 1;
  static constexpr int PER = 16 / BITS;                    // values per half-word of a token-quad word
  static constexpr int ROWB = HD * BITS / 8;
  static constexpr int BLOCKB = kTB * (ROWB + (QUANT ? 4 * NG : 0));
  static constexpr int J = BITS == 2 ? J2 : BITS == 4 ? J4 : BITS == 8 ? J8 : J16;
  static constexpr int KD = CPL * BITS / 4;                // dwords of K codes per lane, set and chain
  static constexpr int VD = ES * BITS / 8 < 2 ? 2 : ES * BITS / 8;   // dwords of V codes per lane, quad and A operand
  static constexpr int NM = QUANT ? NG : 1;
  // Where the lowest field of a byte is put before it is masked.  The matrix unit aligns the 32 products of an
  // instruction to the largest by their nominal exponents, in which a subnormal counts as 2^-14 however many leading zeros
  // it has, and cuts off below: fields at bit 2 instead of 0 keep two more bits of every product.  (Error of `out` against
  // 64 bits, 64 query / 8 kv heads, 128K tokens, INT4, G 32, worse of two seeds: 3.6e-4 at bit 0, 2.3e-4 at bit 2; 2.8e-4 for
  // instructions over 4 products with the fields at bit 0.)
  static constexpr int POS0 = BITS <= 4 ? 2 : 0;
  static constexpr uint32_t MASK0 = BITS == 2 ? 0x000C000Cu : BITS == 4 ? 0x003C003Cu : 0x00FF00FFu;
  static constexpr float UNIT = QUANT ? float(1 << (24 - POS0)) : 1.0f;   // what a product with such a field has to be scaled by
  // the low (hi = 0) or high byte of both half-words, its fields from bit POS0 on (the rest is for the mask to remove)
  __device__ static __forceinline__ uint32_t byte_at(uint32_t w, int hi) {
    return hi ? w >> (8 - POS0) : POS0 ? w << POS0 : w;
  }

  // INT2 and INT4 blocks are staged through shared memory (run_tiles_lds), as they lie in the cache
  static constexpr bool LDS = BITS <= 4;
  static constexpr int NI = BLOCKB / 1024 + BLOCKB % 1024 / 256;   // load instructions per block

  struct KStage {
    Words<KD> c[GR][2][NR];   // codes of the lane's token in set 0 and 1
    Words<NR> meta[GR][2];
  };
  struct VStage {
    Words<VD> c[GR][2][NA];   // two quads of tokens: set 0 and 1
    Words<NM> meta[GR];       // all scale/zero pairs of the token the lane makes p for
  };
  struct Lane {                  // byte offsets and the shift that brings the lane's fields to the bottom
    uint32_t kc, km, vc, vm, shift;
  };

  // first 8-channel chunk of chain r for the lane group g
  __device__ static constexpr int chunk0(int r, int g) { return (HD / 16) * (g >> 1) + r * 2 * CPL + CPL * (g & 1); }
  // first of the lane's channels e (0..15) of a 64-channel half, and which half (A operand a adds to it where FOUR)
  __device__ static constexpr int e_first(int c) { return HD == 128 && !FOUR ? 8 * ((c >> 2) & 1) : 8 * (c >> 3) + 4 * ((c >> 2) & 1); }
  __device__ static constexpr int half_of(int c) { return HD == 128 && !FOUR ? c >> 3 : 0; }

  __device__ static __forceinline__ Lane lane_offsets(int lane) {
    const int g = lane >> 4, c = lane & 15, par = lane >> 5;
    Lane o;
    const int kb = chunk0(0, g) * BITS;   // bytes into the row
    o.kc = uint32_t((kb >> 4) * (kTB * 16) + c * 16 + (kb & 15));
    o.km = uint32_t(c * 4 * NG + (FOUR ? 8 * par : NG == 2 ? 4 * par : 0));
    const int wp = e_first(c) / PER;      // pair of words inside the half row
    o.vc = uint32_t(((BITS / 2) * half_of(c) + (wp >> 1)) * (kTB * 16) + (wp & 1) * 8 + (4 * g + (c & 3)) * 16);
    o.vm = uint32_t((16 * par + c) * 4 * NG);
    o.shift = (c >> 2) & 1 ? 8 - POS0 : 32 - POS0;   // rotation that brings byte (c >> 2) & 1 where byte_at puts it
    return o;
  }

  template <int AUX>
  __device__ static __forceinline__ void load_k(KStage& s, rsrc_t rs, int u, const Lane& o) {
    const uint32_t boff = uint32_t(u / UPB) * BLOCKB, sub = uint32_t(u % UPB);
#pragma unroll
    for (int gr = 0; gr < GR; ++gr)
#pragma unroll
      for (int set = 0; set < 2; ++set) {
        const uint32_t tok = sub * UT + gr * 32 + set * 16;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          // a chain's codes start 2 CPL BITS bytes behind those of the chain before: inside the piece (INT2) or pieces on
          constexpr int step = 2 * CPL * BITS;
          const uint32_t roff = step < 16 ? r * step : r * (step / 16) * (kTB * 16);
          s.c[gr][set][r].template load<AUX>(rs, o.kc, boff + tok * 16 + roff);
        }
        if constexpr (QUANT) s.meta[gr][set].template load<AUX>(rs, o.km, boff + kTB * ROWB + tok * (4 * NG));
      }
  }

  // the same 32 tokens (granule gr, 0 or 1, of a block) out of a block's image in shared memory
  __device__ static __forceinline__ void read_k(KStage& s, const char* image, int gr, const Lane& o) {
#pragma unroll
    for (int set = 0; set < 2; ++set) {
      const int tok = gr * 32 + set * 16;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        constexpr int step = 2 * CPL * BITS;
        const int roff = step < 16 ? r * step : r * (step / 16) * (kTB * 16);
        s.c[0][set][r].read(image + o.kc + tok * 16 + roff);
      }
      s.meta[0][set].read(image + o.km + kTB * ROWB + tok * (4 * NG));
    }
  }
  __device__ static __forceinline__ void read_v(VStage& s, const char* image, int gr, const Lane& o) {
#pragma unroll
    for (int set = 0; set < 2; ++set)
#pragma unroll
      for (int a = 0; a < NA; ++a)
        s.c[0][set][a].read(image + o.vc + (gr * 32 + set * 16) * 16 + a * (BITS / 2) * (kTB * 16));
  }
  __device__ static __forceinline__ void read_v_meta(VStage& s, const char* image, int gr, const Lane& o) {
    s.meta[0].read(image + o.vm + kTB * ROWB + gr * 32 * (4 * NG));
  }

  template <int AUX>
  __device__ static __forceinline__ void load_v(VStage& s, rsrc_t rs, int u, const Lane& o) {
    const uint32_t boff = uint32_t(u / UPB) * BLOCKB, sub = uint32_t(u % UPB);
#pragma unroll
    for (int gr = 0; gr < GR; ++gr) {
      const uint32_t tok = sub * UT + gr * 32;
#pragma unroll
      for (int set = 0; set < 2; ++set)
#pragma unroll
        for (int a = 0; a < NA; ++a)
          s.c[gr][set][a].template load<AUX>(rs, o.vc, boff + (tok + set * 16) * 16 + a * (BITS / 2) * (kTB * 16));
      if constexpr (QUANT) s.meta[gr].template load<AUX>(rs, o.vm, boff + kTB * ROWB + tok * (4 * NG));
    }
  }

  // B operand of the K side: 8 channels of a token, in channel order; the pair jd comes out as code * 2^(BITS kpos(jd)) / UNIT
  __device__ static constexpr int kpos(int jd) { return BITS == 2 ? jd : BITS == 4 ? jd & 1 : 0; }
  __device__ static __forceinline__ u32x4 k_operand(const Words<KD>& c, int m) {
    u32x4 b;
    if constexpr (BITS == 2) {
      const uint32_t w = byte_at(c[m / 2], m & 1);
      b.x = w & MASK0, b.y = w & (MASK0 << 2), b.z = w & (MASK0 << 4), b.w = w & (MASK0 << 6);
    } else if constexpr (BITS == 4) {
      const uint32_t w = byte_at(c[m], 0), v = byte_at(c[m], 1);
      b.x = w & MASK0, b.y = w & (MASK0 << 4), b.z = v & MASK0, b.w = v & (MASK0 << 4);
    } else if constexpr (BITS == 8) {
      const uint32_t w = c[2 * m], v = c[2 * m + 1];
      b.x = byte_at(w, 0) & MASK0, b.y = byte_at(w, 1) & MASK0, b.z = byte_at(v, 0) & MASK0, b.w = byte_at(v, 1) & MASK0;
    } else {
      b.x = c[4 * m], b.y = c[4 * m + 1], b.z = c[4 * m + 2], b.w = c[4 * m + 3];
    }
    return b;
  }
  // four tokens (one quad) of the lane's channel `st`: two dwords of the V side's B operand
  __device__ static __forceinline__ void v_operand(const Words<VD>& c, uint32_t shift, int st, uint32_t& x, uint32_t& y) {
    if constexpr (BITS == 16) {
      x = c[2 * st], y = c[2 * st + 1];
    } else if constexpr (BITS == 2 && ES == 4) {
      x = __builtin_amdgcn_alignbit(c[0], c[0], shift) & (MASK0 << (2 * st));
      y = __builtin_amdgcn_alignbit(c[1], c[1], shift) & (MASK0 << (2 * st));
    } else {
      const int p = st / PER, f = st % PER, hi = f / NPOS, k = f % NPOS;
      x = byte_at(c[2 * p], hi) & (MASK0 << (BITS * k)), y = byte_at(c[2 * p + 1], hi) & (MASK0 << (BITS * k));
    }
  }
  // what the sums of the lane's channel `st` have to be multiplied with at the end
  __device__ static constexpr float fac(int st) { return QUANT ? UNIT / float(1 << (BITS * ((st % PER) % NPOS))) : 1.0f; }
};

template <class T>
struct TileState {
  f4 acc[T::NA][T::ES];   // D: rows (half, head), column = channel
  f4 ones[T::NA];         // sum of the rounded weights p_t scale_tg of row (half, head)
  f4 zacc[T::NM];         // per group: sum over the lane's tokens of (zero + c0 scale) p, one component per head
  f4 l, m;                // sum over the lane's tokens of p; reference (the same in all lanes of a head)
};

// The lane's four heads are 4 ((lane >> 4) & 1) .. + 3 everywhere: in the logits, in p and (rows 4 g .. 4 g + 3 of D are
// row 8 (g >> 1) + 4 (g & 1) + i) in the accumulators.
template <int HD, class T>
__device__ __forceinline__ void begin_tiles(int qrow, int lane, TileState<T>& st, u32x4 (&qa)[T::M], f4 (&qs)[T::NR]) {
#pragma unroll
  for (int a = 0; a < T::NA; ++a) {
    st.ones[a] = splat(0.f);
#pragma unroll
    for (int e = 0; e < T::ES; ++e) st.acc[a][e] = splat(0.f);
  }
#pragma unroll
  for (int g = 0; g < T::NM; ++g) st.zacc[g] = splat(0.f);
  st.m = splat(0.f);
  const int g = lane >> 4, head = lane & 7;
  const bool real = head < kparams()->rep;                  // rows of heads that do not exist are zero
  const bool mine = real && ((lane >> 3) & 1) == (g >> 1);  // the row's half and the half the lane group's channels lie in
  const u32x4* qp = reinterpret_cast<const u32x4*>(kparams()->q + int64_t(qrow + (real ? head : 0)) * (HD / 2));
  // A head whose query is not finite must not reach the others, which share the products of tile_accumulate with it (0 times
  // a NaN weight): its row becomes zero, and its l NaN, which no weight changes any more.  (0.1 to 0.25 us of the calls named
  // at the top; by the sums of the matrix unit and a branch it was 0.4 to 0.6.)
  typedef uint16_t us2 __attribute__((ext_vector_type(2)));
  us2 top = {0, 0};
#pragma unroll
  for (int r = 0; r < T::NR; ++r)
#pragma unroll
    for (int m = 0; m < T::CPL; ++m) {
      const u32x4 v = qp[T::chunk0(r, g) + m];
      qa[r * T::CPL + m] = v;
#pragma unroll
      for (int w = 0; w < 4; ++w) top = __builtin_elementwise_max(top, __builtin_bit_cast(us2, v[w] & 0x7FFF7FFFu));
    }
  uint64_t bad = __builtin_amdgcn_ballot_w64(mine && max(top.x, top.y) >= 0x7C00);
  bad |= bad >> 32, bad |= bad >> 16, bad |= bad >> 8;      // one bit per head
  const bool keep = mine && !(uint32_t(bad) >> head & 1u);
#pragma unroll
  for (int i = 0; i < 4; ++i) st.l[i] = uint32_t(bad) >> (4 * (g & 1) + i) & 1u ? __builtin_nanf("") : 0.f;
  u32x4 ones;
  ones.x = ones.y = ones.z = ones.w = 0x3C003C00u;
#pragma unroll
  for (int r = 0; r < T::NR; ++r) {
    qs[r] = splat(0.f);
#pragma unroll
    for (int m = 0; m < T::CPL; ++m) {
      u32x4 v = qa[r * T::CPL + m];
      v.x = keep ? v.x : 0u, v.y = keep ? v.y : 0u, v.z = keep ? v.z : 0u, v.w = keep ? v.w : 0u;
      if constexpr (T::QUANT) {
        // the sum of the query channels of the half, which the zero is multiplied with
        qs[r] = mfma16(v, ones, qs[r]);
        constexpr int B = T::QUANT ? 16 / T::PER : 0;   // bits
        auto fac = [](int k) { const uint32_t h = uint32_t(15 - B * k) << 10; return h | (h << 16); };
        v.x = pk_mul(v.x, fac(T::kpos(0))), v.y = pk_mul(v.y, fac(T::kpos(1)));
        v.z = pk_mul(v.z, fac(T::kpos(2))), v.w = pk_mul(v.w, fac(T::kpos(3)));
      }
      qa[r * T::CPL + m] = v;
    }
    if constexpr (T::QUANT) qs[r] *= 1.0f / T::UNIT;
  }
}

// q.k^ (in units of 1 / UNIT) of the granule's token 16 (lane / 32) + lane % 16 for the lane's four heads
template <class T>
__device__ __forceinline__ f4 tile_logits(const typename T::KStage& s, int gr, const u32x4 (&qa)[T::M], const f4 (&qs)[T::NR]) {
  f4 part[2];
#pragma unroll
  for (int set = 0; set < 2; ++set) {
    f4 ga[T::NR];
#pragma unroll
    for (int r = 0; r < T::NR; ++r) {
      ga[r] = splat(0.f);
#pragma unroll
      for (int m = 0; m < T::CPL; ++m) ga[r] = mfma16(qa[r * T::CPL + m], T::k_operand(s.c[gr][set][r], m), ga[r]);
    }
    if constexpr (T::QUANT) {
      f4 sum = splat(0.f);
#pragma unroll
      for (int r = 0; r < T::NR; ++r) {
        const h2 mz = as_h2(s.meta[gr][set][r]);
        const float sc = static_cast<float>(mz.x), ze = static_cast<float>(mz.y);
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] = sum[i] + ze * qs[r][i] + sc * ga[r][i];
      }
      part[set] = sum;
    } else {
      part[set] = ga[0];
    }
  }
  f4 full;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float lo, hi;
    swap_halves(part[0][i], part[1][i], lo, hi);
    full[i] = lo + hi;
  }
  return full;
}

// binary exponent of the lane's V scales: every scale is below 2^e
template <class T>
__device__ __forceinline__ float tile_exponent(const typename T::VStage& s, int gr) {
  if constexpr (!T::QUANT) return 0.f;
  h2 top = as_h2(s.meta[gr][0]);   // (scale, zero): the maximum of the low halves is the one that counts
#pragma unroll
  for (int g = 1; g < T::NM; ++g) top = __builtin_elementwise_max(top, as_h2(s.meta[gr][g]));
  return static_cast<float>(__builtin_amdgcn_frexp_expf(static_cast<float>(top.x)));
}

// fp16(scale * p) of four heads, rounded once (v_fma_mixlo/hi_f16; a plain product would become a product and a
// conversion): scale = low half of a scale/zero pair
__device__ __forceinline__ u32x2 scaled_h4(uint32_t meta, f4 p) {
  const float sc = static_cast<float>(as_h2(meta).x);
  h4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = static_cast<_Float16>(__builtin_fmaf(sc, p[i], 0.0f));
  return __builtin_bit_cast(u32x2, r);
}

// p: softmax weights of the lane's token for its four heads
template <class T>
__device__ __forceinline__ void tile_accumulate(const typename T::VStage& s, int gr, f4 p, TileState<T>& st, const u32x4 (&sel)[2],
                                                uint32_t shift) {
  constexpr float c0 = T::QUANT ? 0.5f * float((1 << (16 / T::PER)) - 1) : 0.f;   // the middle of the code range
  u32x2 x16[T::NM];
#pragma unroll
  for (int g = 0; g < T::NM; ++g) {
    if constexpr (T::QUANT) {
      const h2 mz = as_h2(s.meta[gr][g]);
      const float mid = static_cast<float>(mz.y) + c0 * static_cast<float>(mz.x);
      x16[g] = scaled_h4(s.meta[gr][g], p);
      st.zacc[g] += mid * p;
    } else {
      x16[g] = to_h4(p);
    }
  }
  u32x4 one;
  one.x = one.y = one.z = one.w = 0x3C003C00u;
#pragma unroll
  for (int a = 0; a < T::NA; ++a) {
    const u32x2 x0 = x16[T::FOUR ? 2 * a : 0], x1 = x16[T::FOUR ? 2 * a + 1 : T::NM - 1];
    u32x4 x;
    x.x = x0.x, x.y = x0.y, x.z = x1.x, x.w = x1.y;
    const u32x2 p0 = to_h4(mfma16(x, sel[0], splat(0.f))), p1 = to_h4(mfma16(x, sel[1], splat(0.f)));
    u32x4 pa;
    pa.x = p0.x, pa.y = p0.y, pa.z = p1.x, pa.w = p1.y;
    if constexpr (T::QUANT) st.ones[a] = mfma16(pa, one, st.ones[a]);
#pragma unroll
    for (int e = 0; e < T::ES; ++e) {
      uint32_t b0, b1, b2, b3;
      T::v_operand(s.c[gr][0][a], shift, e, b0, b1);
      T::v_operand(s.c[gr][1][a], shift, e, b2, b3);
      u32x4 b;
      b.x = b0, b.y = b1, b.z = b2, b.w = b3;
      st.acc[a][e] = mfma16(pa, b, st.acc[a][e]);
    }
  }
}

// Another reference for the lane's head i: what has been summed up is multiplied with alpha = 2^(old - new).
template <class T>
__device__ __forceinline__ void tile_rescale(TileState<T>& st, int i, float m, float alpha) {
  st.m[i] = m;
  st.l[i] *= alpha;
#pragma unroll
  for (int g = 0; g < T::NM; ++g) st.zacc[g][i] *= alpha;
#pragma unroll
  for (int a = 0; a < T::NA; ++a) {
    st.ones[a][i] *= alpha;
#pragma unroll
    for (int e = 0; e < T::ES; ++e) st.acc[a][e][i] *= alpha;
  }
}

// Online softmax over N granules: p holds q.k^ (in units of 1 / UNIT) and becomes the weights; c turns it into
// log2 units, ev = exponents of the V scales.  `first`: the state is empty, its reference comes from these granules.
//
// `far`: some reference of the state is 2^24 or more, where binary32 holds no fractions.  p c - m of the unrounded product is then
// off by up to half a unit of m, which at 2^31 is more than the weights' whole range: all of them may vanish, and equal logits of
// different pieces get different weights.  So the logits are rounded first there, and the reference is one of the rounded values,
// without headroom (it could not be held): the largest weight is 1, and with it the largest product a V scale.  Decided once
// per state and when a reference is raised; the common path pays for a branch (4 x 128K at eight heads 129.65 -> 129.5 us, sixteen
// heads 52.15 -> 52.3; the unrounded logits kept for a second pass instead took 48 bytes of scratch: 145 us).
template <class T, int N>
__device__ __forceinline__ void tile_softmax(f4 (&p)[N], const float (&ev)[N], float c, bool first, bool& far, TileState<T>& st) {
  constexpr float kRoom = kTopExp - kHeadroom;
  if (first) {
    bool any = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float tmax = kNegBig;
#pragma unroll
      for (int n = 0; n < N; ++n) tmax = fmaxf(tmax, __builtin_fmaf(p[n][i], c, ev[n]));
      tmax = both_halves(row_max(tmax), true);
      any |= !(__builtin_fabsf(tmax) < kFar);
      st.m[i] = tmax - kRoom;
    }
    far = __builtin_amdgcn_ballot_w64(any) != 0;
  }
  if (__builtin_expect(far, 0)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float tmax = kNegBig;
#pragma unroll
      for (int n = 0; n < N; ++n) {
        float s = p[n][i] * c;
        pin(s);   // rounded: no product inside the subtraction below
        p[n][i] = s;
        tmax = fmaxf(tmax, s + ev[n]);
      }
      tmax = both_halves(row_max(tmax), true);
      const float m = first || tmax > st.m[i] + kTopExp ? tmax : st.m[i];
      tile_rescale(st, i, m, first ? 1.f : __builtin_amdgcn_exp2f(st.m[i] - m));
    }
    c = 1.f;
  }
  float top = -INFINITY;
#pragma unroll
  for (int n = 0; n < N; ++n) {
#pragma unroll
    for (int i = 0; i < 4; ++i) p[n][i] = __builtin_fmaf(p[n][i], c, -st.m[i]);   // log2 of the weight
    top = fmaxf(top, fmaxf(fmaxf(p[n][0], p[n][1]), fmaxf(p[n][2], p[n][3])) + ev[n]);
  }
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(top > kTopExp) != 0, 0)) {
    f4 up;
    bool any = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float tmax = -INFINITY;
#pragma unroll
      for (int n = 0; n < N; ++n) tmax = fmaxf(tmax, p[n][i] + ev[n]);
      up[i] = both_halves(row_max(tmax), true);
      any |= up[i] > kTopExp && !(__builtin_fabsf(st.m[i] + up[i]) < kFar);
    }
    far = far || __builtin_amdgcn_ballot_w64(any) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // the reference as binary32 holds it, and the step that was really made
      const float m = up[i] > kTopExp ? st.m[i] + (up[i] - (far ? 0.f : kRoom)) : st.m[i];
      const float step = m - st.m[i];
      tile_rescale(st, i, m, __builtin_amdgcn_exp2f(-step));
#pragma unroll
      for (int n = 0; n < N; ++n) p[n][i] -= step;
    }
  }
#pragma unroll
  for (int n = 0; n < N; ++n) {
#pragma unroll
    for (int i = 0; i < 4; ++i) p[n][i] = __builtin_amdgcn_exp2f(p[n][i]);
    st.l += p[n];
  }
}

// Writes the partial states of the set's query heads: (m, l, tokens, o[HD]) per head.
template <int HD, class T, class SLOT>
__device__ __forceinline__ void flush_tiles(const TileState<T>& st, SLOT out, int lane, int tokens) {
  constexpr int STRIDE = HD + kPartialFloats;
  constexpr float c0 = T::QUANT ? 0.5f * float((1 << (16 / T::PER)) - 1) : 0.f;
  const int rep = kparams()->rep;
  const int c = lane & 15, par = lane >> 5, head0 = 4 * ((lane >> 4) & 1);
  f4 l, z[T::NM];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    l[i] = both_halves(row_sum(st.l[i]), false);
#pragma unroll
    for (int g = 0; g < T::NM; ++g) z[g][i] = T::QUANT ? both_halves(row_sum(st.zacc[g][i]), false) : 0.f;
  }
  if (lane < 32 && c < 4 && head0 + c < rep) put_header(out, (head0 + c) * (STRIDE * 4), pick(st.m, c), pick(l, c), tokens);
  const bool mine = (c >> 3) == par;   // not the columns of the other half
#pragma unroll
  for (int a = 0; a < T::NA; ++a) {
    const int ch = 64 * (T::FOUR ? a : T::half_of(c)) + 32 * (T::e_first(c) >> 3) + 8 * (c & 3) + (T::e_first(c) & 7);
    const f4 za = T::FOUR ? (par ? z[2 * a + 1] : z[2 * a]) : par ? z[T::NM - 1] : z[0];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float base = T::QUANT ? za[i] - c0 * st.ones[a][i] : 0.f;
#pragma unroll
      for (int e = 0; e < T::ES; e += 4) {
        f4 o;
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = st.acc[a][e + x][i] * T::fac(e + x) + base;
        if (mine && head0 + i < rep) put(out, ((head0 + i) * STRIDE + kPartialFloats + ch + e) * 4, o);
      }
    }
  }
}

// sel[set]: B operand that moves set `set` of x[half][4 heads] (A: row = token % 16, k = 8 (lane group) + 4 half + head) to
// column 8 half + head.
__device__ __forceinline__ void tile_select(int lane, u32x4 (&sel)[2]) {
  const int col = lane & 15, g = lane >> 4;
  const uint32_t bit = (col & 1) ? 0x3C000000u : 0x00003C00u;
  const int word = 2 * (col >> 3) + ((col >> 1) & 1);
#pragma unroll
  for (int set = 0; set < 2; ++set) {
    const bool here = g == 2 * set + ((col >> 2) & 1);
#pragma unroll
    for (int w = 0; w < 4; ++w) sel[set][w] = here && w == word ? bit : 0u;
  }
}

// The eight-head version of run_class (decode_heads_impl.h): the same pipeline over the stream's pieces.
template <int HD, int BITS, int CID, int G, int AUX, class DEST = Workspace<HD>, class STREAM = Stream<HD>>
__device__ __forceinline__ void run_tiles(STREAM& sm, Piece& cur, int lane, bool app = false, DEST dest = {}) {
  typedef TileClass<HD, BITS, G> T;
  constexpr int J = DEST::kOne ? 1 : T::J, GR = T::GR, UT = T::UT, UPB = T::UPB;
  static_assert(DEST::kOne || J == kIterUnits[CID], "the stream hands out pieces of the kernel's iteration size");
  const typename T::Lane off = T::lane_offsets(lane);
  const char* const kbase = uni(app ? kparams()->k_app : kparams()->k[CID]);
  const char* const vbase = uni(app ? kparams()->v_app : kparams()->v[CID]);
  const float c = kparams()->scale_log2 * T::UNIT;
  u32x4 sel[2];
  tile_select(lane, sel);
  TileState<T> st;
  u32x4 qa[T::M];
  f4 qs[T::NR];
  typename T::KStage ks[J];
  typename T::VStage vs[J];
  int pid = cur.pid;
  rsrc_t krs = make_rsrc(kbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
  rsrc_t vrs = make_rsrc(vbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
  int ru = cur.us, rn = cur.nu;
  int roob = UPB * sm.nblk;
#pragma unroll
  for (int jj = 0; jj < J; ++jj) T::template load_k<AUX>(ks[jj], krs, jj < rn ? ru + jj : roob, off);
#pragma unroll
  for (int jj = 0; jj < J; ++jj) T::template load_v<AUX>(vs[jj], vrs, jj < rn ? ru + jj : roob, off);
  sched_fence();
  begin_tiles<HD, T>(sm.qrow, lane, st, qa, qs);
  int valid = cur.valid;
  int covered = 0;
  bool first = true, far = false;                    // the partial state is empty; see tile_softmax
  const int tpos = 16 * (lane >> 5) + (lane & 15);   // the token of a granule the lane makes p for
  Piece nxt = sm.next(lane);
#pragma unroll 1
  while (true) {
    const bool more = nxt.nu > 0 && nxt.cls == CID;
    if (more) {
      krs = make_rsrc(kbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
      vrs = make_rsrc(vbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
      ru = nxt.us, rn = nxt.nu, roob = UPB * sm.nblk;
    } else {
      rn = 0;
    }
    covered += valid;
    f4 p[J * GR];
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
#pragma unroll
      for (int gr = 0; gr < GR; ++gr) p[jj * GR + gr] = tile_logits<T>(ks[jj], gr, qa, qs);
      sched_fence();
      T::template load_k<AUX>(ks[jj], krs, jj < rn ? ru + jj : roob, off);
      sched_fence();
    }
    if (valid < J * UT) {
#pragma unroll
      for (int n = 0; n < J * GR; ++n)
        p[n] = n * 32 + tpos < valid ? p[n] : splat(-INFINITY);
    }
    float ev[J * GR];
#pragma unroll
    for (int n = 0; n < J * GR; ++n) ev[n] = tile_exponent<T>(vs[n / GR], n % GR);
    tile_softmax<T, J * GR>(p, ev, c, first, far, st);
    first = false;
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
#pragma unroll
      for (int gr = 0; gr < GR; ++gr) tile_accumulate<T>(vs[jj], gr, p[jj * GR + gr], st, sel, off.shift);
      sched_fence();
      T::template load_v<AUX>(vs[jj], vrs, jj < rn ? ru + jj : roob, off);
      sched_fence();
    }
    if (!more || nxt.fresh) flush_tiles<HD, T>(st, dest.slot(pid), lane, covered);
    if (!more) break;
    if (nxt.fresh) {
      pid = nxt.pid;
      covered = 0;
      first = true;
      begin_tiles<HD, T>(sm.qrow, lane, st, qa, qs);
    }
    valid = nxt.valid;
    nxt = sm.next(lane);
  }
  cur = nxt;
}

// ---------------------------------------------------------------- INT2 and INT4: staged through shared memory
// Loads that write shared memory: 16 (4) bytes per lane from `rs` at voff + soff, to lds + 16 (4) * lane.  Written as
// assembly because the compiler would otherwise wait for all of them before any read of shared memory; the caller waits
// (wait_newest) for the ones it needs.  No register but m0 is written (the compiler warns that m0 is reserved: it is named so that
// nothing is kept there); the address registers are read when the load issues.  The compiler does not see a load inside and so does
// not keep the five wait states a vector-memory instruction needs after a vector instruction wrote one of its scalar operands (a
// read of a lane, also the reload of a spilled scalar): fetch_block takes them once for the loads of a block, and a test looks in
// the built library for such a write between them.  (One wait for a block costs up to 0.3 %, one per load up to 1.6 %.  All loads of
// a block in one statement with the offset of the instruction: 4 x 128K 129.5 -> 127.5 us, but append 49.0 -> 50.0 and sixteen
// heads 52.0 -> 52.6.)
struct LdsRsrc {
  u32x4 w;
};
__device__ __forceinline__ LdsRsrc lds_rsrc(const char* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  LdsRsrc r;
  r.w.x = uint32_t(b), r.w.y = uint32_t(b >> 32) & 0xffffu, r.w.z = bytes, r.w.w = 0x00020000u;
  return r;
}
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int AUX, bool WIDE>
__device__ __forceinline__ void load_to_lds(uint32_t lds, const LdsRsrc& rs, uint32_t voff, uint32_t soff) {
  // (one wait state between the write of m0 and the load that reads it)
  if constexpr (WIDE && AUX == kAuxNonTemporal)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(lds), "v"(voff), "s"(rs.w), "s"(soff) : "memory", "m0");
  else if constexpr (WIDE)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rs.w), "s"(soff) : "memory", "m0");
  else if constexpr (AUX == kAuxNonTemporal)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen nt lds" ::"s"(lds), "v"(voff), "s"(rs.w), "s"(soff) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rs.w), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop
// Until all but the newest N vector-memory operations of this wave are complete (they complete in order; operations the
// caller has not counted only make the wait longer).
template <int N>
__device__ __forceinline__ void wait_newest() {
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Block `blk` of a run (out of range: zeros) to an image in shared memory.
template <class T, int AUX>
__device__ __forceinline__ void fetch_block(uint32_t lds, const LdsRsrc& rs, int blk, int lane) {
  uint32_t off = uint32_t(blk) * T::BLOCKB;
  // What is still being read out of the image has been read; the wait states of the loads.  The offsets are changed as far as the compiler
  // knows, so that it adds the constants behind this, with scalar instructions, and brings no sum back from a spill (v_readlane).
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 4" : "+s"(off), "+s"(lds) : "s"(rs.w) : "memory");
#pragma unroll
  for (int i = 0; i < T::BLOCKB / 1024; ++i) load_to_lds<AUX, true>(lds + i * 1024, rs, lane * 16, off + i * 1024);
#pragma unroll
  for (int i = 0; i < T::BLOCKB % 1024 / 256; ++i) {
    const uint32_t o = T::BLOCKB / 1024 * 1024 + i * 256;
    load_to_lds<AUX, false>(lds + o, rs, lane * 4, off + o);
  }
}

// run_tiles for the classes staged through shared memory: an iteration takes JB whole blocks (ranges are cut at blocks and
// these shapes have no pools), each in an image of its own for K and V, refilled with the block of the next iteration as
// soon as it has been read.  Reading the fragments of the matrix operands straight from memory took 240 cycles of a
// compute unit's load path per 32 INT2 tokens (4-byte loads 16 bytes apart cost 32 cycles, 8-byte loads as much as
// 16-byte ones: 16); contiguous 16-byte loads take 48.
constexpr int kTileLds = 12 * 1024;
template <int HD, int BITS, int CID, int G, int AUX, class DEST = Workspace<HD>, class STREAM = Stream<HD>>
__device__ __forceinline__ void run_tiles_lds(STREAM& sm, Piece& cur, char* lds, int lane, DEST dest = {}) {
  typedef TileClass<HD, BITS, G> T;
  constexpr int UPB = T::UPB, J = DEST::kOne ? UPB : T::J, JB = J / UPB, NG = 2 * JB;   // blocks, granules per iteration
  static_assert(DEST::kOne || J == kIterUnits[CID], "the stream hands out pieces of the kernel's iteration size");
  static_assert(2 * JB * T::BLOCKB <= kTileLds, "the images of an iteration fit");
  const typename T::Lane off = T::lane_offsets(lane);
  const char* const kbase = uni(kparams()->k[CID]);
  const char* const vbase = uni(kparams()->v[CID]);
  const float c = kparams()->scale_log2 * T::UNIT;
  u32x4 sel[2];
  tile_select(lane, sel);
  TileState<T> st;
  u32x4 qa[T::M];
  f4 qs[T::NR];
  int pid = cur.pid;
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lds));
  auto kimg = [&](int j) { return j * T::BLOCKB; };
  auto vimg = [&](int j) { return (JB + j) * T::BLOCKB; };
  LdsRsrc krs = lds_rsrc(kbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
  LdsRsrc vrs = lds_rsrc(vbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
  int rb = cur.us / UPB, rn = cur.nu / UPB;   // blocks to fetch: first, count
  int oob = sm.nblk;                          // first block past the run: costs nothing
#pragma unroll
  for (int j = 0; j < JB; ++j) fetch_block<T, AUX>(lds0 + kimg(j), krs, j < rn ? rb + j : oob, lane);
#pragma unroll
  for (int j = 0; j < JB; ++j) fetch_block<T, AUX>(lds0 + vimg(j), vrs, j < rn ? rb + j : oob, lane);
  begin_tiles<HD, T>(sm.qrow, lane, st, qa, qs);
  int valid = cur.valid;
  int covered = 0;
  bool first = true, far = false;
  const int tpos = 16 * (lane >> 5) + (lane & 15);
  Piece nxt = sm.next(lane);
#pragma unroll 1
  while (true) {
    const bool more = nxt.nu > 0 && nxt.cls == CID;
    if (more) {
      krs = lds_rsrc(kbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
      vrs = lds_rsrc(vbase + int64_t(sm.blk0) * T::BLOCKB, uint32_t(sm.nblk) * T::BLOCKB);
      rb = nxt.us / UPB, rn = nxt.nu / UPB, oob = sm.nblk;
    } else {
      rn = 0;
    }
    covered += valid;
    f4 p[NG];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      wait_newest<(JB - 1) * T::NI + JB * T::NI>();   // K image j is complete: newer are the other K images and all V images
#pragma unroll
      for (int gr = 0; gr < 2; ++gr) {
        typename T::KStage ks;
        T::read_k(ks, lds + kimg(j), gr, off);
        p[2 * j + gr] = tile_logits<T>(ks, 0, qa, qs);
      }
      sched_fence();
      fetch_block<T, AUX>(lds0 + kimg(j), krs, j < rn ? rb + j : oob, lane);
      sched_fence();
    }
    if (valid < J * T::UT) {
#pragma unroll
      for (int n = 0; n < NG; ++n) p[n] = n * 32 + tpos < valid ? p[n] : splat(-INFINITY);
    }
    wait_newest<JB * T::NI>();   // all V images are complete: newer are the K images of the next iteration
    typename T::VStage vs[NG];
    float ev[NG];
#pragma unroll
    for (int n = 0; n < NG; ++n) {
      T::read_v_meta(vs[n], lds + vimg(n / 2), n % 2, off);
      ev[n] = tile_exponent<T>(vs[n], 0);
    }
    tile_softmax<T, NG>(p, ev, c, first, far, st);
    first = false;
#pragma unroll
    for (int j = 0; j < JB; ++j) {
#pragma unroll
      for (int gr = 0; gr < 2; ++gr) {
        T::read_v(vs[2 * j + gr], lds + vimg(j), gr, off);
        tile_accumulate<T>(vs[2 * j + gr], 0, p[2 * j + gr], st, sel, off.shift);
      }
      sched_fence();
      fetch_block<T, AUX>(lds0 + vimg(j), vrs, j < rn ? rb + j : oob, lane);
      sched_fence();
    }
    if (!more || nxt.fresh) flush_tiles<HD, T>(st, dest.slot(pid), lane, covered);
    if (!more) break;
    if (nxt.fresh) {
      pid = nxt.pid;
      covered = 0;
      first = true;
      begin_tiles<HD, T>(sm.qrow, lane, st, qa, qs);
    }
    valid = nxt.valid;
    nxt = sm.next(lane);
  }
  wait_newest<0>();   // nothing of this class lands in shared memory any more
  cur = nxt;
}

template <int HD>
__device__ __forceinline__ void write_neutral_set(int slot, int lane) {
  const int rep = kparams()->rep;
  for (int i = 0; i < rep; ++i) write_neutral<HD>(slot, i, lane);
}

// One wave per worker, then one per slice of the appended tokens.  The plans of these shapes have no
// pools (a plan that had one would lose tokens, which the merge reports).
template <int HD, int G, int AUX, bool INT8>
__global__ __launch_bounds__(64 * kCuWaves) __attribute__((amdgpu_waves_per_eu(2))) void decode_tiles_kernel(COCKTAIL_WORKER_ARGS) {
  extern __shared__ __attribute__((aligned(16))) char all_lds[];   // kTileLds for every wave
#ifdef COCKTAIL_TRACE
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
#endif
  const FirstParams fp = {recs, num_workers, num_q_heads, rep};
  const Place me = place(fp);
  const int lane = me.lane;
  char* const lds = all_lds + me.wave * kTileLds;
  if (me.worker >= fp.num_workers) {
    const AppendSlice a = append_slice(me.worker - fp.num_workers);
    if (a.tokens <= 0) {
      write_neutral_set<HD>(a.pid, lane);
      return;
    }
    Stream<HD> sm;
    sm.init_run(kFp16Class, a.tokens, a.first_block, a.blocks, a.qrow, a.pid);
    Piece cur = sm.next(lane);
    if (cur.nu > 0) run_tiles<HD, 16, kFp16Class, G, AUX>(sm, cur, lane, true);
    return;
  }
  Stream<HD> sm;
  WorkerRec rec = load_record(fp.recs + me.worker);
  touch_params(rec.g0);
  sm.init(rec, fp);
  sm.ngran = 0, sm.nps = 0;
  Piece cur = sm.next(lane);
  while (cur.nu > 0) {
    if (cur.cls == 0) {
      run_tiles_lds<HD, 2, 0, G, AUX>(sm, cur, lds, lane);
    } else if (cur.cls == 1) {
      run_tiles_lds<HD, 4, 1, G, AUX>(sm, cur, lds, lane);
    } else if (INT8 && cur.cls == 2) {
      if constexpr (INT8) run_tiles<HD, 8, 2, G, AUX>(sm, cur, lane);
    } else {
      run_tiles<HD, 16, kFp16Class, G, AUX>(sm, cur, lane);
    }
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

template <int HD>
hipError_t launch_decode_tiles(const DecodeParams& p, int group_size, bool non_temporal, bool int8, int grid, hipStream_t st) {
  worker_kernel kern = nullptr;
#define COCKTAIL_PICK2(G, I8) \
  kern = non_temporal ? decode_tiles_kernel<HD, G, kAuxNonTemporal, I8> : decode_tiles_kernel<HD, G, kAuxDefault, I8>
#define COCKTAIL_PICK(G)             \
  if (int8) COCKTAIL_PICK2(G, true); \
  else COCKTAIL_PICK2(G, false)
  if (group_size == 32) {
    COCKTAIL_PICK(32);
  } else if (group_size == 64) {
    COCKTAIL_PICK(64);
  } else if constexpr (HD >= 128) {
    COCKTAIL_PICK(128);
  }
#undef COCKTAIL_PICK
#undef COCKTAIL_PICK2
  if (!kern) return hipErrorInvalidValue;   // a group size larger than head_dim: refused by the shape check before
  return launch_workers(kern, p, grid, kTileLds, st);
}

}  // namespace cocktail
