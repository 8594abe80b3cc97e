// Fused decode attention for gfx950 (Eq. 2 with Eq. 6's 1/sqrt(d), one softmax over
// the original-precision rows and the quantized rows, Sec. 2.4).  The quantized rows
// (2-bit codes, or 4-bit: Sec. 3.2.1) are never dequantized in memory:
//
//   logits   q.k_hat_t = sum_c q_c z_c + sum_c (q_c s_c) code_tc
//            -> per key group (G tokens) the products q_c s_c are formed once, split
//               into three fp16 pieces (the top six bits of the rounded product, its
//               other five bits, the rounding residual: together exact for 11-bit or
//               8-bit factors) and become three rows of the A operand of a 16x16x32
//               matrix instruction: row 4*head + piece (piece 3 is zero).
//               The code tile is the B operand, 16 tokens per instruction.  Lane
//               (row group q4, column n16) of the result then holds, for head q4 and
//               token n16, the pieces in three registers: two adds give the logit.
//               sum_c q_c z_c is a per-group bias.  (A single fp16 rounding of
//               q_c s_c is not enough: with outlier channels its error alone moves
//               the logits by ~1e-2.)
//   output   sum_t p_t v_hat_tc = sum_t p_t vz_t + sum_t (p_t vs_t) code_tc
//            -> p_t vs_t (row 4*channel group + head) is the A operand, the code
//               tile the B operand; sum_t p_t vz_t is kept per channel group.  The
//               probabilities go from the softmax lanes (head x token) to the lanes
//               of the output step (token octets) through LDS as fp16.
//
// Codes as operands.  An fp16 lane whose only set bits are mantissa bits 2v+2, 2v+3 is
// the subnormal number code * 2^(2v-22); gfx950's matrix cores take subnormal
// operands exactly.  The packed layout puts the eight 2-bit codes a lane feeds to
// one matrix instruction into one byte of the low and one byte of the high half of
// a 32-bit word, so one shift and four ANDs
// produce the four operand registers: 10 VALU instructions per 16 codes, no
// integer-to-float conversion.  The factor 2^(2v) that depends on the position v
// of a code inside its byte is cancelled in the other operand: q is pre-multiplied
// by 2^(3-2v) per channel, and the probabilities by the same factor per token slot
// (folded into the exponent of exp2, so it costs nothing).  4-bit codes work the
// same way with two nibble positions (see codes4).
//
// Work split: a workgroup has eight (or four, or twelve) independent wavefronts; the
// wavefronts of all workgroups of one (batch row, kv head, head group) share its fp rows
// in units of 32 and its quantized rows in tiles of 64 (lq_schedule.h).
// Partial (max, sum, output) triples are merged in LDS per workgroup and written
// to the workspace.  Every workgroup then takes a ticket from a counter of its
// (batch row, kv head, head group); the one that draws the last ticket merges all
// splits of that group and writes the output, so no second launch is needed and
// the merge of one group overlaps the tail of the others.  Nobody waits on anybody.
// The partials and the counter are accessed with device-scope relaxed atomics
// (write-through stores, cache-bypassing loads): a device-scope fence would write
// back and invalidate a whole L2 per workgroup, which costs more than the kernel.
#pragma once
#include "lq_device.h"
#include "lq_internal.h"
#include "lq_schedule.h"

namespace lq {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

struct AttnParams {
  const uint16_t* q;
  const uint32_t* k_codes;
  const uint32_t* v_codes;
  const uint16_t* k_scale;
  const uint16_t* k_zero;
  const uint16_t* v_scale;
  const uint16_t* v_zero;
  float* ws;          // partials
  int* counters;      // CTR_LINES lines per group (ticket, tile pools), zero between launches
  uint16_t* out;
  // fused append (null k_new: none): the new row of every (b, kv head), [B][Hkv][d],
  // becomes fp slot n_fp - 1 (n_fp already counts it)
  const uint16_t* k_new;
  const uint16_t* v_new;
  uint16_t* k_fp[2];      // [0]: the live fp buffer (the same for every sequence), or, with
  uint16_t* v_fp[2];      // per-sequence state, the two buffers, chosen by the sequence's `cur`
  int32_t* pos_fp[2];
  const SeqState* seq;    // device array of per-sequence state (seq_mode 2)
  int seq_mode;           // 0: counts below hold for every sequence; 1: state in the kernel arguments
  int Hkv;
  int cap, qcap, n_fp, n_q, gh, hb, splits, nwf;
  int across;         // groups side by side in the grid (its first dimension)
  Divisor div_subgroups, div_kv_heads;   // by the head groups of a kv head (gh / hb), by the kv heads
  int cus;            // workgroups of 4 from this index on are the younger of a pair (the compute units planned for)
  int W, Wq;          // of every Wq quantized slots (one filtering event) the first W hold tokens
  int n_tok_q;        // tokens in the n_q quantized slots
  int tiles;          // tiles_of(n_q)
  LiveTiles live;     // key groups of 64 and 128: the tiles that hold tokens
  uint32_t dead_bit;  // an offset past the end of every array of a slice (0: none; padding is then read)
  int dynamic;        // 0: static tile schedule only
  float c;  // softmax scale * log2(e)
};

constexpr int PSHIFT = 5;   // probabilities are kept relative to 2^(max - PSHIFT)
constexpr float MAX_SLACK = 4.f;
constexpr int FP_LEAD = 30;     // the fp rows' reference is lowered by this much when their sums pass to the quantized rows
constexpr float DEAD_LOGIT = -1e30f;   // logit of a padding slot; exp2(DEAD_LOGIT - anything finite) == 0

__device__ __forceinline__ floatx4 mfma_f16(uint4 a, uint4 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a),
                                                __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma_bf16(uint4 a, uint4 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
template <bool BF16>
__device__ __forceinline__ floatx4 mfma_T(uint4 a, uint4 b, floatx4 c) {
  if constexpr (BF16) return mfma_bf16(a, b, c); else return mfma_f16(a, b, c);
}

// The eight codes of one operand live in byte 0 and byte 2 of `w` (even operand of
// the word) or in byte 1 and byte 3 (odd operand).  Register v gets the code at
// bits 2v+2, 2v+3 of each fp16 lane: value code * 2^(2v-22).  (As high as a subnormal
// number allows: the matrix unit aligns the addends of a dot product by exponent fields,
// and every place the bits lie below the nominal exponent costs one of the sum.  Left at
// bits 2v, 2v+1, one instruction less for even operands, the noise of fp16 outputs was
// about twice as large - 16.6 instead of 9.9% not the nearest value - and the time 1% shorter.)
__device__ __forceinline__ uint4 codes_of(uint32_t w, int odd) {
  const uint32_t x = odd ? w >> 6 : w << 2;
  return make_uint4(x & 0x000C000Cu, x & 0x00300030u, x & 0x00C000C0u, x & 0x03000300u);
}
// 4-bit codes: a word holds the eight codes of one operand, element i = 2v + h in
// nibble v of half h.  Registers 0 and 2 keep their codes at mantissa bits 0..3
// (code * 2^-24), registers 1 and 3 at bits 4..7 (code * 2^-20); two of the four
// nibbles of a half would reach into the exponent and are shifted down first.
__device__ __forceinline__ uint4 codes4(uint32_t w) {
  const uint32_t h = w >> 8;
  return make_uint4(w & 0x000F000Fu, w & 0x00F000F0u, h & 0x000F000Fu, h & 0x00F000F0u);
}
// Operand o (of the 2 * NKC a lane holds for one 32-slot block) of a code tile, and
// the power of two by which the other operand's register v has to be scaled so that
// every product carries the common factor 2^-CODE_SHIFT.
template <int BITS, int N>
__device__ __forceinline__ uint4 operand_codes(const uint32_t (&w)[N], int o) {
  if constexpr (BITS == 2) return codes_of(w[o >> 1], o & 1);
  else return codes4(w[o]);
}
template <int BITS>
__device__ __forceinline__ constexpr int pos_exp(int v) {   // log2 of the scale of register v's partner
  return BITS == 2 ? 3 - 2 * v : 2 - 4 * (v & 1);
}
template <int BITS>
constexpr float CODE_SCALE = BITS == 2 ? 524288.f : 4194304.f;   // 2^19, 2^22

__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  half2_t h = {(_Float16)a, (_Float16)b};
  return __builtin_bit_cast(uint32_t, h);
}
template <bool BF16>
__device__ __forceinline__ uint32_t pack_T(float a, float b) {
  if constexpr (BF16) return (uint32_t)f2t<true>(a) | ((uint32_t)f2t<true>(b) << 16);
  else return pack_f16(a, b);
}
template <bool BF16>
__device__ __forceinline__ float lo_T(uint32_t w) {
  if constexpr (BF16) return __uint_as_float(w << 16);
  else return (float)__builtin_bit_cast(half2_t, w)[0];
}
template <bool BF16>
__device__ __forceinline__ float hi_T(uint32_t w) {
  if constexpr (BF16) return __uint_as_float(w & 0xFFFF0000u);
  else return (float)__builtin_bit_cast(half2_t, w)[1];
}
template <bool BF16>
__device__ __forceinline__ void unpack8_T(uint4 v, float* f) {
  f[0] = lo_T<BF16>(v.x); f[1] = hi_T<BF16>(v.x); f[2] = lo_T<BF16>(v.y); f[3] = hi_T<BF16>(v.y);
  f[4] = lo_T<BF16>(v.z); f[5] = hi_T<BF16>(v.z); f[6] = lo_T<BF16>(v.w); f[7] = hi_T<BF16>(v.w);
}
// a pair of T values -> a pair of fp16 values (exact for normal-range bf16 inputs)
template <bool BF16>
__device__ __forceinline__ half2_t pair_to_f16(uint32_t w) {
  if constexpr (BF16) return half2_t{(_Float16)lo_T<true>(w), (_Float16)hi_T<true>(w)};
  else return __builtin_bit_cast(half2_t, w);
}
// Scales and zero-points are stored as fp16 whatever the cache type (for a bf16 cache
// converting them here cost a sixth of the tile loop's instructions): a stored pair is
// an operand as it is.
__device__ __forceinline__ half2_t meta_pair(uint32_t w) { return __builtin_bit_cast(half2_t, w); }
// fp32 accumulate of a two-element dot product of fp16 pairs (exact products)
__device__ __forceinline__ float dot2_h(half2_t a, half2_t b, float c) {
  return __builtin_amdgcn_fdot2(a, b, c, false);
}

// v of lane `src` (__shfl adds the lane's wavefront to the index, one more register that lives through the kernel)
__device__ __forceinline__ float from_lane(float v, int src) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * src, __float_as_int(v)));
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
// lane i <-> lane i^16 and lane i <-> lane i^32 exchanges without the LDS crossbar:
// the swap instructions trade rows (halves) between two registers, so swapping a
// register with a copy of itself leaves one holding the even rows (low half) twice
// and the other the odd rows (high half) twice.
__device__ __forceinline__ void xor16_pair(float v, float* a, float* b) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  *a = __uint_as_float(r[0]); *b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void xor32_pair(float v, float* a, float* b) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  *a = __uint_as_float(r[0]); *b = __uint_as_float(r[1]);
}
// all-reduce over the 16 lanes that share lane & 3 (one query head): two rotations
// inside the row of 16 lanes, two exchanges across rows
__device__ __forceinline__ float head_max(float v) {
  float a, b;
  v = fmaxf(v, dpp_f<0x124>(v));   // row_ror:4
  v = fmaxf(v, dpp_f<0x128>(v));   // row_ror:8
  xor16_pair(v, &a, &b); v = fmaxf(a, b);
  xor32_pair(v, &a, &b); v = fmaxf(a, b);
  return v;
}
__device__ __forceinline__ float head_sum(float v) {
  float a, b;
  v += dpp_f<0x124>(v);
  v += dpp_f<0x128>(v);
  xor16_pair(v, &a, &b); v = a + b;
  xor32_pair(v, &a, &b); v = a + b;
  return v;
}
// all-reduce over the 16 lanes of a lane row (lanes that share lane >> 4)
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_f<0x128>(v);   // row_ror:8
  v += dpp_f<0x124>(v);
  v += dpp_f<0x122>(v);
  v += dpp_f<0x121>(v);
  return v;
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_f<0x128>(v));
  v = fmaxf(v, dpp_f<0x124>(v));
  v = fmaxf(v, dpp_f<0x122>(v));
  v = fmaxf(v, dpp_f<0x121>(v));
  return v;
}
// sum over the four lanes that differ in lane >> 4
__device__ __forceinline__ float rows_sum(float v) {
  float a, b;
  xor16_pair(v, &a, &b); v = a + b;
  xor32_pair(v, &a, &b); v = a + b;
  return v;
}

// maximum over the four lanes that differ in lane >> 4
__device__ __forceinline__ float rows_max(float v) {
  float a, b;
  xor16_pair(v, &a, &b); v = fmaxf(a, b);
  xor32_pair(v, &a, &b); v = fmaxf(a, b);
  return v;
}

// LDS-visible ordering inside one wavefront (no workgroup barrier needed: DS
// instructions of a wavefront execute in order).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// device-coherent accesses to the partial results (see the ticket merge below)
__device__ __forceinline__ void st_dev(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_dev(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void buffer_store16(uint4 x, __amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  __builtin_amdgcn_raw_buffer_store_b128(u32x4{x.x, x.y, x.z, x.w}, rs, voff, soff, 0);
}

template <int N>
struct Words { uint32_t w[N]; };

// Running softmax state of one wavefront.  m and l belong to head (lane & 3);
// acc[nt][j] is output row 4*(lane>>4)+j, column lane&15 of channel tile nt.
// Everything is relative to 2^(m - PSHIFT); l[j] additionally carries the factor
// 2^offs[j] of its token slot.
template <int NNT>
struct State {
  floatx4 acc[NNT];
  float m;
  float l[4];
  float zacc[4];   // per code position v (token slots 2v, 2v+1 of a lane)
};

// s[0..3]: log2-domain logits (slot offsets included) of this lane's four tokens
// -> p[0..3] = 2^(s - m + PSHIFT); updates the state.
template <int NNT, bool ZACC>
__device__ __forceinline__ void online_softmax(State<NNT>& st, const float* s, float* p) {
  // the running maximum only has to bound every logit seen so far: the cross-lane
  // reduction runs only when some lane's tile maximum exceeds it
  // (a logit may exceed the reference by up to MAX_SLACK before that happens:
  // probabilities then reach 2^(PSHIFT + MAX_SLACK), still far inside fp16 range)
  float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
  if (__any(mx > st.m + MAX_SLACK)) {
    mx = head_max(mx);
    const float m_new = fmaxf(st.m, mx);
    const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);   // 0 on the first tile (m = -inf)
#pragma unroll
    for (int j = 0; j < 4; ++j) st.l[j] *= alpha;
    if constexpr (ZACC) {
#pragma unroll
      for (int i = 0; i < 4; ++i) st.zacc[i] *= alpha;
    }
    float a4[4];
#pragma unroll
    for (int gg = 0; gg < 4; ++gg) a4[gg] = from_lane(alpha, (threadIdx.x & 60) | gg);
#pragma unroll
    for (int nt = 0; nt < NNT; ++nt) {
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) st.acc[nt][gg] *= a4[gg];
    }
    st.m = m_new;
  }
  const float mref = st.m - (float)PSHIFT;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    p[j] = __builtin_amdgcn_exp2f(s[j] - mref);
    st.l[j] += p[j];
  }
}

// Quantized-row variant: lane row q4 = lane >> 4 is a query head, the 16 lanes of a
// row hold different tokens; s[u], u = 0..3, are this lane's tokens.  The output
// accumulators and zacc are laid out by the output step: acc[nt][j] belongs to head
// j, zacc to head g = lane & 3.
// ROUND_P: the probabilities come back already rounded to fp16, the form in which the
// output step uses them, and the denominator sums these rounded values.  Numerator and
// denominator then describe the same (slightly perturbed) weights, so that the rounding
// cancels where one token dominates instead of scaling the whole output.
// slack: by how much a logit may exceed the reference before that moves.  The token that moved it last has the probability
// 2^PSHIFT, which rounds without error.
template <int NNT, bool ROUND_P>
__device__ __forceinline__ void online_softmax_rows(State<NNT>& st, const float* s, float* p, int g, float slack) {
  float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
  if (__any(mx > st.m + slack)) {
    mx = row_max(mx);
    const float m_new = fmaxf(st.m, mx);
    const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);   // 0 on the first tile (m = -inf)
#pragma unroll
    for (int u = 0; u < 4; ++u) st.l[u] *= alpha;
    float a4[4];
#pragma unroll
    for (int gg = 0; gg < 4; ++gg)
      a4[gg] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha), 16 * gg));
    const float ag = g == 0 ? a4[0] : g == 1 ? a4[1] : g == 2 ? a4[2] : a4[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) st.zacc[i] *= ag;
#pragma unroll
    for (int nt = 0; nt < NNT; ++nt) {
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) st.acc[nt][gg] *= a4[gg];
    }
    st.m = m_new;
  }
  const float mref = st.m - (float)PSHIFT;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    p[u] = __builtin_amdgcn_exp2f(s[u] - mref);
    if constexpr (ROUND_P) p[u] = (float)(_Float16)p[u];
    st.l[u] += p[u];
  }
}

// NWB: wavefronts per workgroup: 8; 4 when there are enough (b, kv head) groups to put
// two workgroups on every compute unit; 12 (three wavefronts per SIMD, at most 168
// registers) for long contexts, where the extra wavefront hides more than the tighter
// register budget costs.
// KIND: EQUAL: rows of one length, no padding; PER_ROW: counts per row (per-sequence lengths); PADDED: padding slots in
// the quantized region (group size not dividing the window), with either.  Each carries no more than it needs: as one
// variant, the search for the tiles that hold tokens cost rows without padding 3% (scalar registers spill).
enum { EQUAL, PER_ROW, PADDED };
// per-sequence state in the kernel arguments
template <int KIND> struct SeqArgs { SeqState e[SEQ_CHUNK]; };
template <> struct SeqArgs<EQUAL> {};

// PROG: how fp rows and tiles are dealt to the wavefronts, see lq_schedule.h.
// NH: sets of four query heads that a workgroup works on side by side, P.hb heads in all.  Two sets share the loads of a
// tile and the codes once they are unpacked; each has its own q*s, probabilities and sums (250 registers for d = 128, none
// spilled but 4 to 5 with padding, 4 bits and G = 32).  Eight heads per kv head in two workgroups of four were bound by
// unpacking and by reading every byte twice: 8 kv heads x 9 rows x 49079 tokens, d = 96, 104 -> 83 us a launch, 64 x 8192,
// d = 128, 24.8 -> 20.5 (heads_per_group says when).
template <bool BF16, int D, int G, int NWB, int BITS, int KIND, int PROG, int NH>
__global__ void __launch_bounds__(64 * NWB, NWB == 12 ? 3 : 2)
attn_mfma_kernel(const AttnParams P, const SeqArgs<KIND> S) {
  constexpr bool ONE = PROG == ONE_SPLIT, DRAW = PROG == DRAWN;
  constexpr int NKC = D / 32, NNT = D / 16, NGC = (D + G - 1) / G;
  constexpr int WPL = NKC * (BITS / 2);           // code words per lane and 32-slot block
  constexpr int NGRP = G < 64 ? 64 / G : 1;     // key groups per 64-token tile
  // fp16 pieces of q*s per wave, one row per (piece, head).  The 16 lanes of a
  // lane row read 16 bytes each from thirteen different rows at the same column; a row
  // pitch that is an odd number of 16-byte units puts those on different banks.
  constexpr int QS_ROW = D + 8;
  static_assert((QS_ROW * 2 / 16) % 2 == 1, "q*s row pitch");
  constexpr int QS_ROWS = 12 * NH + 1;
  __shared__ __attribute__((aligned(16))) uint16_t qs_lds[NWB][NGRP][QS_ROWS][QS_ROW];   // rows 12*set+4*piece+head (three pieces), the last row = zeros
  __shared__ __attribute__((aligned(16))) uint16_t p_lds[NWB][NH][2][9][32];        // [wave][set][32-token step][row][token]: rows 0-3 p of head, 4 zeros, 5-8 p's fp16 rounding residual
  __shared__ __attribute__((aligned(16))) float o_lds[NWB][4 * NH][D];                   // (the split merge stores 16 bytes at a time)
  __shared__ float ml_lds[NWB][4 * NH][2];
  __shared__ float zs_lds[NWB][4][4 * NH];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroups are handed to the eight XCDs in turn (linear index mod 8).  When the number of groups is a multiple of 8
  // the grid is (8, splits, groups / 8): all splits of one group are placed on one XCD, so that the partials they
  // exchange at the end meet in that XCD's L2.  Else it is (1, splits, groups).
  const int split = ONE ? 0 : blockIdx.y, group = blockIdx.z * P.across + blockIdx.x;
  int bh = P.div_subgroups.quotient(group);
  const int hsub = group - bh * P.div_subgroups.n;
  if constexpr (KIND != EQUAL) {
    // per-sequence lengths: workgroups are dispatched in index order, so the rows are
    // taken longest first (seq[i].order = the row with the i-th most tokens)
    if (P.seq_mode) {
      const int i = P.div_kv_heads.quotient(bh);
      bh = (P.seq_mode == 1 ? seq_in_args(args_offset_after(sizeof(AttnParams)))[i].order : P.seq[i].order) * P.Hkv +
           bh - i * P.Hkv;   // (the argument block is P, then S)
    }
  }
  const int q4 = lane >> 4, n16 = lane & 15, up = n16 >> 2, g = lane & 3;
  const int64_t head0 = (int64_t)bh * P.gh + hsub * P.hb;   // this workgroup's first query head
  constexpr uint32_t OUT_OF_RANGE = 0x40000000u;            // an offset past the end of its heads' q
  const auto rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(P.q) + head0 * D, 0, P.hb * (D * 2), 0x00020000);

  // counts and live fp buffer: the same for every sequence, or (per-sequence lengths)
  // read from the sequence's entry of the state array
  int n_fp = P.n_fp, n_q = P.n_q, nwf = P.nwf, n_tok_q = P.n_tok_q, cur = 0;
  int TQ = P.tiles;
  if constexpr (KIND != EQUAL) {
    if (P.seq_mode) {
      const int b = P.div_kv_heads.quotient(bh);
      const SeqState sq = P.seq_mode == 1 ? seq_load(seq_in_args(args_offset_after(sizeof(AttnParams))), b) : P.seq[b];
      n_fp = sq.n_fp; n_q = sq.n_q; nwf = sq.nwf; n_tok_q = sq.n_tok_q; cur = sq.cur; TQ = sq.item;
    }
  }
  // (a select between two kernel arguments, not a load that depends on `cur`)
  uint16_t* k_fp_w = cur ? P.k_fp[1] : P.k_fp[0];
  uint16_t* v_fp_w = cur ? P.v_fp[1] : P.v_fp[0];
  int32_t* pos_fp = cur ? P.pos_fp[1] : P.pos_fp[0];
  const int TF = (n_fp + 31) >> 5;
  const Deal<PROG, NWB> deal(P.splits, split, wave, nwf, TF);
  const bool one_split = ONE || (!DRAW && P.splits == 1);
  // Of wavefronts that share a SIMD the older one wins the issue slots: with two to a SIMD and a static schedule the
  // younger ones ended 25% later (165 against 212 us at 16 rows x 32 kv heads x 32768 tokens), the last part with the
  // SIMD to themselves and too few loads in flight.  So the younger ones - the upper four of a workgroup of 8; of
  // workgroups of 4, those dispatched when every compute unit already has one - take precedence for the first half
  // of their tiles, which lets both end together (206 -> 199 us; a batch of 64 x 4096 tokens 47.6 -> 46.6 us a step,
  // with rows of different lengths 46.4 -> 45.0; three and five eighths of the tiles measured up to 1% slower).
  // (Not where the younger of a pair of workgroups has the shorter row: see pairs_workgroups.)
  const bool young = ONE && (NWB == 8 ? wave >= 4 : NWB == 4 && group >= P.cus);
  const int own_half = young ? (deal.first + TQ) / 2 : 0;
  if (young) __builtin_amdgcn_s_setprio(1);
  const int64_t part_base = (((int64_t)bh * P.splits + split) * P.gh + hsub * P.hb) * (D + 4);
  State<NNT> st[NH];
#pragma unroll
  for (int hs = 0; hs < NH; ++hs) {
#pragma unroll
    for (int nt = 0; nt < NNT; ++nt) st[hs].acc[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    st[hs].m = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) st[hs].l[j] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) st[hs].zacc[i] = 0.f;
  }

  // ------------------------- original-precision rows -------------------------
  auto fp_rows = [&](const int unit0, const int unit_step) __attribute__((always_inline)) {
    const int64_t fp_slice = (int64_t)bh * P.cap * D;
    const int lane16 = lane * 16;
    const uint16_t* kb = k_fp_w + fp_slice + lane * 8;
    const uint16_t* vb = v_fp_w + fp_slice + lane * 8;
    // q is loaded out of range (zeros, nothing read) for absent heads: as a choice after the load it became a branch, and
    // with fewer heads than four a wait for each of these loads before the next was issued.
    uint4 qreg[NH][NKC];
#pragma unroll
    for (int hs = 0; hs < NH; ++hs) {
      const uint32_t q_off = 4 * hs + g < P.hb ? (uint32_t)((4 * hs + g) * D + 8 * q4) * 2 : OUT_OF_RANGE;
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) qreg[hs][kc] = buffer_load16(rs_q, (int)q_off, 64 * kc);
    }
    // Fused append: the wavefront that owns the unit receiving the new row fetches the row
    // first.  (The compiler waits for it before it issues the unit's own loads: one more
    // latency for this wavefront.  As loads of all wavefronts, out of range for the others, without that wait: 1 to 1.5% slower
    // steps at 8 rows of 8192 and 64 of 4096 tokens.)
    const int new_unit = (n_fp - 1) >> 5, new_sx = (n_fp - 1) & 31, new_kx = kperm(new_sx);
    const bool owner = P.k_new && new_unit % unit_step == unit0;
    uint4 kn_r[NKC];
    uint32_t vn_r[NNT];
    if (owner) {
      const char* kn = (const char*)(P.k_new + (int64_t)bh * D);
      const char* vn = (const char*)(P.v_new + (int64_t)bh * D);
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) kn_r[kc] = *reinterpret_cast<const uint4*>(kn + 64 * kc + (uint32_t)(16 * q4));
#pragma unroll
      for (int nt = 0; nt < NNT; ++nt) vn_r[nt] = *reinterpret_cast<const uint16_t*>(vn + 32 * nt + (uint32_t)(2 * n16));
    }
    for (int unit = unit0; unit < TF; unit += unit_step) {
      // The stores of the new row, and with 12 wavefronts the loads, are buffer accesses, one descriptor for the keys of a
      // unit and one for its values: with 64-bit lane addresses for all of them 12 wavefronts spilled up to 20 registers
      // for d = 128, and a kernel with scratch memory starts later (29 rows x 8 kv heads x 1548 tokens, one launch
      // 21.9 -> 18.1 us, 26 of 4206, one head per kv head 32.5 -> 26.8, 15 of 21020 51.4 -> 48.3, one of 131072
      // 24.0 -> 23.5).  With 4 and 8, which have the registers, lane addresses are 1% faster (8 rows of 8192, four layers,
      // 65.5 against 64.8 us).
      const auto rs_kf = __builtin_amdgcn_make_buffer_rsrc(k_fp_w + fp_slice + (int64_t)unit * (32 * D), 0, 32 * D * 2, 0x00020000);
      const auto rs_vf = __builtin_amdgcn_make_buffer_rsrc(v_fp_w + fp_slice + (int64_t)unit * (32 * D), 0, 32 * D * 2, 0x00020000);
      uint4 ka[2][NKC], va[NNT];
#pragma unroll
      for (int uu = 0; uu < 2; ++uu)
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc)
          ka[uu][kc] = NWB == 12 ? buffer_load16(rs_kf, lane16, (uu * NKC + kc) * 1024)
                                 : *reinterpret_cast<const uint4*>(kb + ((int64_t)(2 * unit + uu) * NKC + kc) * 512);
#pragma unroll
      for (int nt = 0; nt < NNT; ++nt)
        va[nt] = NWB == 12 ? buffer_load16(rs_vf, lane16, nt * 1024) : *reinterpret_cast<const uint4*>(vb + ((int64_t)unit * NNT + nt) * 512);

      if (owner && unit == new_unit) {
        // Fused append.  This wavefront is the only reader of the unit that receives
        // the new row: it takes the row from the caller's buffers instead of the cache
        // (whatever the loads above found in that slot is replaced) and stores it into
        // the cache for the steps to come (once per (b, kv head): head group 0).
        const int sx = new_sx, uu_ = sx >> 4;
        if (n16 == (sx & 15)) {
#pragma unroll
          for (int kc = 0; kc < NKC; ++kc) {
            const uint4 x = kn_r[kc];
            if (uu_ == 0) ka[0][kc] = x; else ka[1][kc] = x;
            if (hsub == 0)
              buffer_store16(x, rs_kf, lane16 + kc * 1024, uu_ * (NKC * 1024));
          }
        }
        const int kx = new_kx;         // element kx & 7 of the lanes of token octet kx >> 3
        if (q4 == (kx >> 3)) {
          const int sh = 16 * (kx & 1), wi = (kx & 7) >> 1;
#pragma unroll
          for (int nt = 0; nt < NNT; ++nt) {
            const uint32_t e = vn_r[nt];
            uint32_t w[4] = {va[nt].x, va[nt].y, va[nt].z, va[nt].w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (i == wi) w[i] = (w[i] & ~(0xFFFFu << sh)) | (e << sh);
            va[nt] = make_uint4(w[0], w[1], w[2], w[3]);
            if (hsub == 0)
              __builtin_amdgcn_raw_buffer_store_b16((uint16_t)e, rs_vf, lane16 + nt * 1024, 2 * (kx & 7), 0);
          }
        }
        if (hsub == 0 && bh % P.Hkv == 0 && lane == 0)
          pos_fp[(bh / P.Hkv) * P.cap + n_fp - 1] = n_fp - 1 + n_tok_q;
      }

#pragma unroll
      for (int hs = 0; hs < NH; ++hs) {
        floatx4 Du[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) {
          Du[0] = mfma_T<BF16>(ka[0][kc], qreg[hs][kc], Du[0]);
          Du[1] = mfma_T<BF16>(ka[1][kc], qreg[hs][kc], Du[1]);
        }
        float s[4], p[4];
        {
          const floatx4 d = up == 0 ? Du[0] : Du[1];
          const int tok0 = 32 * unit + 16 * up + 4 * q4;
#pragma unroll
          for (int j = 0; j < 4; ++j) s[j] = (up < 2 && tok0 + j < n_fp) ? d[j] * P.c : -INFINITY;
        }
        online_softmax<NNT, false>(st[hs], s, p);

        float pv[8];
        const int src0 = (lane & 0x33), src1 = (lane & 0x33) | 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          pv[j] = from_lane(p[j], src0);
          pv[4 + j] = from_lane(p[j], src1);
        }
        // rows 0..3: p rounded to T; rows 4..7: the rounding residual, again in T (masks: as a choice between the two
        // the compiler made eight branches of it; 512 tokens, 8 kv heads 10.2 instead of 9.9 us)
        const uint32_t hi_row = up == 0 ? 0xFFFFFFFFu : 0u, lo_row = up == 1 ? 0xFFFFFFFFu : 0u;
        uint32_t aw[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const uint32_t hi = pack_T<BF16>(pv[2 * r], pv[2 * r + 1]);
          const uint32_t lo = pack_T<BF16>(pv[2 * r] - lo_T<BF16>(hi), pv[2 * r + 1] - hi_T<BF16>(hi));
          aw[r] = (hi & hi_row) | (lo & lo_row);
        }
        const uint4 a = make_uint4(aw[0], aw[1], aw[2], aw[3]);
        if (hs == 0 && 32 * unit + 32 > n_fp) {   // slots beyond n_fp hold unspecified bits
          uint32_t keep[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i0 = 2 * r, i1 = 2 * r + 1;
            const int x0 = 16 * ((i0 >> 2) & 1) + 4 * q4 + (i0 & 3), x1 = 16 * ((i1 >> 2) & 1) + 4 * q4 + (i1 & 3);
            keep[r] = (32 * unit + x0 < n_fp ? 0x0000FFFFu : 0u) | (32 * unit + x1 < n_fp ? 0xFFFF0000u : 0u);
          }
#pragma unroll
          for (int nt = 0; nt < NNT; ++nt) {
            va[nt].x &= keep[0]; va[nt].y &= keep[1]; va[nt].z &= keep[2]; va[nt].w &= keep[3];
          }
        }
#pragma unroll
        for (int nt = 0; nt < NNT; ++nt) st[hs].acc[nt] = mfma_T<BF16>(a, va[nt], st[hs].acc[nt]);
      }
    }
  };
  auto hand_over = [&]() __attribute__((always_inline)) {
    // Hand-over to the quantized rows, whose state is laid out differently: m and l by lane row (l as one addend,
    // of a lane whose token slot carries the factor 2^pos_exp(0)), and the sum of head and residual rows of a
    // channel tile in the lane row of its channel group, in units of a code.
    // The reference m goes down by FP_LEAD, the sums up by 2^FP_LEAD (exact): the first tile then raises it to its own
    // maximum, unless that lies more than FP_LEAD below the fp rows'.  The tiles' probabilities are fp16 operands and
    // must not shrink beside heavy fp rows; the fp32 sums do not mind (at most 2^9 |v| per row, times 2^30).  Tiles
    // further below weigh under 2^-30 a token, 2^17 tokens under 2^-13 of the output, and down to 2^-40 their operands
    // are still normal numbers.  (With the fp rows' maximum as the reference, 16384 tokens 2^14 below 10 heavy rows,
    // value scales of 2^-8.5, were off by 1.3e-2 of the output; now within the output's own rounding.)
#pragma unroll
    for (int hs = 0; hs < NH; ++hs) {
      const float l_tot = head_sum((st[hs].l[0] + st[hs].l[1]) + (st[hs].l[2] + st[hs].l[3]));
      const float m_g = st[hs].m;
      st[hs].m = from_lane(m_g, q4) - (float)FP_LEAD;
      const float l_q = from_lane(l_tot, q4) * __builtin_ldexpf(1.f, FP_LEAD + pos_exp<BITS>(0));
      st[hs].l[0] = n16 == 0 ? l_q : 0.f;
      st[hs].l[1] = st[hs].l[2] = st[hs].l[3] = 0.f;
#pragma unroll
      for (int nt = 0; nt < NNT; ++nt) {
        const int gc = (16 * nt) / G;
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
          float x, y;
          xor16_pair(st[hs].acc[nt][gg], &x, &y);
          float tot = x + y;
          if (gc >= 2) { xor32_pair(tot, &x, &y); tot = x + y; }
          st[hs].acc[nt][gg] = q4 == gc ? tot * (__builtin_ldexpf(1.f, FP_LEAD) / CODE_SCALE<BITS>) : 0.f;
        }
      }
    }
  };

  // ------------------------- quantized rows -------------------------
  auto quantized_rows = [&]() __attribute__((always_inline)) {
    const char* kcb = (const char*)(P.k_codes + (int64_t)bh * (P.qcap >> 5) * 64 * WPL);
    const char* vcb = (const char*)(P.v_codes + (int64_t)bh * (P.qcap >> 5) * 64 * WPL);
    const char* ksb = (const char*)(P.k_scale + (int64_t)bh * (P.qcap / G) * D);
    const char* kzb = (const char*)(P.k_zero + (int64_t)bh * (P.qcap / G) * D);
    const char* vsb = (const char*)(P.v_scale + (int64_t)bh * (P.qcap >> 5) * NGC * 32);
    const char* vzb = (const char*)(P.v_zero + (int64_t)bh * (P.qcap >> 5) * NGC * 32);
    // Rows of the probability operand of the output step: row 4*up + g.  With at most
    // two channel groups there are rows to spare, and the probabilities enter in two
    // pieces: a head piece (p rounded to fp16; for bf16 caches cut to three significant
    // bits, see where it is written) and what that leaves out (rows up = piece * NGC +
    // channel group), so that only the rounding of the product p * vs remains.
    // With three or four groups there is one piece (up = channel group); the softmax
    // denominator then sums the rounded probabilities, so that the rounding does not
    // bias the normalised weights.
    constexpr int VPIECES = NGC <= 2 ? 2 : 1;
    // The operand p * vs is rounded to fp16.  Where the cache type is fp16 (whose output
    // tolerance that rounding alone can use up when one token carries most of the weight
    // and its code is large) the part the rounding drops is carried as well: in the
    // residual rows when there are two pieces, in a second product otherwise.
    constexpr bool PROD_LO = !BF16;
    // With one piece the rounding of p is the largest error before the output's own.  A wavefront's heaviest token has none
    // of it if it is the one that the reference was taken from, so that a row with half the wavefronts, each with twice the
    // tiles, is further off: 64 rows of up to 4096 tokens, fp16, against 64 bits and without the output's rounding
    // 1.29e-4 (2-norm) with 8 wavefronts, 1.39e-4 with 4.  Rows of different lengths take workgroups of 4 where equal rows
    // take 8 or 12: there the reference follows the maximum more closely (at a scale of 2 / sqrt(d), squares off 64 bits, the
    // output's rounding included, as a multiple of those with 8: 1.034 with the usual slack, 1.004 with a slack of 2,
    // 0.991 with 1; 64 rows of up to 4096 tokens, 16 steps 662 -> 667 us, ten shapes 1.2% on average).
    constexpr float SLACK = VPIECES == 1 && NWB == 4 && KIND != EQUAL ? 1.f : MAX_SLACK;
    const bool row_live = up < VPIECES * NGC;
    const int upc = row_live ? up % NGC : 0;          // channel group of this lane's row
    const bool tail_row = VPIECES == 2 && up >= NGC;  // this lane feeds the residual piece
    const uint32_t code_off = lane * WPL * 4;                 // byte offsets of this lane
    const uint32_t vm_off = (upc * 32 + 8 * q4) * 2;
    // Lane roles.  Logits and softmax: lane row q4 is query head q4, lane column n16
    // is a token of each of the four 16-token tiles.  q*s preparation: head q4,
    // channel octet n16.  Output step: row n16 = (channel group up, head g) of the
    // probability operand, token octet q4.
    const int c8 = n16;
    const bool prep = 8 * c8 < D;
    const uint32_t km_off = (prep ? 8 * c8 : 0) * 2;

    struct Tile {
      Words<WPL> kc[2], vc[2];
      uint4 vs[2], vz[2];
      uint4 ks8[NGRP], kz8[NGRP];
    };
    // A tile's registers are refilled piecewise with the next tile's data as soon as
    // their content has been consumed (key scales right after the q*s preparation,
    // key codes after the logits, value codes and scales after each output step), so
    // only one tile's worth of registers is live and every piece still has most of a
    // tile's processing time to arrive.
    // The tile loads are buffer loads: one descriptor per array over this slice, the
    // lane's offset in a register, the tile's offset in a scalar register, so that the
    // per-tile address arithmetic runs on the scalar unit (and a load past the slice
    // would return zeros instead of faulting).
    const uint32_t code_bytes = (uint32_t)(P.qcap >> 5) * 64 * WPL * 4;
    const auto rs_kc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(kcb), 0, code_bytes, 0x00020000);
    const auto rs_vc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(vcb), 0, code_bytes, 0x00020000);
    const uint32_t kmeta_bytes = (uint32_t)(P.qcap / G) * D * 2, vmeta_bytes = (uint32_t)(P.qcap >> 5) * NGC * 32 * 2;
    const auto rs_ks = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(ksb), 0, kmeta_bytes, 0x00020000);
    const auto rs_kz = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(kzb), 0, kmeta_bytes, 0x00020000);
    const auto rs_vs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(vsb), 0, vmeta_bytes, 0x00020000);
    const auto rs_vz = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(vzb), 0, vmeta_bytes, 0x00020000);
    auto load_words = [&](__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff) {
      Words<WPL> r;
#pragma unroll
      for (int i = 0; i + 4 <= WPL; i += 4) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff + 4 * i, (int)soff, 0);
        r.w[i] = v[0]; r.w[i + 1] = v[1]; r.w[i + 2] = v[2]; r.w[i + 3] = v[3];
      }
      if constexpr (WPL % 4 == 3) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b96(rs, (int)voff + 4 * (WPL - 3), (int)soff, 0);
        r.w[WPL - 3] = v[0]; r.w[WPL - 2] = v[1]; r.w[WPL - 1] = v[2];
      } else if constexpr (WPL % 4 == 2) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff + 4 * (WPL - 2), (int)soff, 0);
        r.w[WPL - 2] = v[0]; r.w[WPL - 1] = v[1];
      }
      return r;
    };
    // Where tile t lies; dead: the bit that takes the loads of its second half out of range (they then return zeros and
    // read nothing) when that half is padding.
    struct Place { int t; uint32_t dead; int slot0; };
    auto place = [&](int t) {
      if constexpr (KIND == PADDED && G >= 64) {
        const LiveTiles::Place p = P.live.place(t);
        return Place{p.tile, p.slot0 + 32 >= P.W ? P.dead_bit : 0u, p.slot0};
      } else {
        return Place{t, 0u, 0};
      }
    };
    // Events of one tile (W <= 64) all end at the same slot of its second half, so that the lanes whose slots lie behind it
    // are known from the start: they read nothing either (W = 42, four layers of 131072 tokens 126.2 -> 122.1 us, two rows
    // of 60000, 4 bits, 172 -> 158).  With longer events, where the lanes would have to be found for every tile, that cost
    // as much as it gave (W = 85: 0.96 to 1 times as fast).
    uint32_t k_off2 = code_off, v_off2 = code_off, vm_off2 = vm_off;
    if constexpr (KIND == PADDED && G >= 64) {
      if (P.live.per_event == 1) {
        if (32 + n16 >= P.W) k_off2 |= P.dead_bit;      // key codes: slots n16 and 16 + n16 of the half
        if (32 + 4 * q4 >= P.W) { v_off2 |= P.dead_bit; vm_off2 |= P.dead_bit; }   // values: slots 4 * q4 .. +3 and 16 + 4 * q4 .. +3
      }
    }
    auto load_kmeta = [&](Tile& T, int t) {
#pragma unroll
      for (int e = 0; e < NGRP; ++e) {
        const int grp = t * NGRP / (G <= 64 ? 1 : G / 64) + e;
        T.ks8[e] = buffer_load16(rs_ks, (int)km_off, (int)((uint32_t)grp * (D * 2)));
        T.kz8[e] = buffer_load16(rs_kz, (int)km_off, (int)((uint32_t)grp * (D * 2)));
      }
    };
    auto load_kcodes = [&](Tile& T, const Place& pl) {
      const int t = pl.t;
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2)
        T.kc[b2] = load_words(rs_kc, b2 ? k_off2 | pl.dead : code_off, (uint32_t)t * (2 * 64 * WPL * 4) + b2 * (64 * WPL * 4));
    };
    auto load_v = [&](Tile& T, const Place& pl, int b2) {
      const int t = pl.t;
      const uint32_t c_off = b2 ? v_off2 | pl.dead : code_off, m_off = b2 ? vm_off2 | pl.dead : vm_off;
      T.vc[b2] = load_words(rs_vc, c_off, (uint32_t)t * (2 * 64 * WPL * 4) + b2 * (64 * WPL * 4));
      T.vs[b2] = buffer_load16(rs_vs, (int)m_off, (int)((uint32_t)t * (2 * NGC * 32 * 2) + b2 * (NGC * 32 * 2)));
      T.vz[b2] = buffer_load16(rs_vz, (int)m_off, (int)((uint32_t)t * (2 * NGC * 32 * 2) + b2 * (NGC * 32 * 2)));
    };
    // Tiles that are drawn.  The first two of a wavefront without units are fixed, and the loads of the first go out
    // before anything else touches memory.  The later tiles are dealt out dynamically, so that wavefronts that start
    // late or see slower memory take fewer of them.
    // A draw is issued a whole tile ahead of its use and before that tile's loads: loads
    // and atomics return in issue order, so waiting for the drawn index does not wait
    // for the loads behind it.  The draw is a buffer atomic over a 4-byte buffer: only
    // lane 0 is in range, the other lanes are dropped by the bounds check, and no
    // branch is needed (the join of a branch would make the compiler wait for every
    // outstanding load).
    // With few tiles per wavefront, or no more wavefronts than pools, there is nothing
    // to balance: the deal is then static, and where only the row's counts decide
    // (per-sequence lengths) the atomic is aimed out of range.
    // A single split has no last workgroup that could re-arm the pool counters for the
    // next launch (it returns before the ticket): static as well.
    // q goes out ahead of the first tile: loads return in order, so that its operands are ready when the key scales arrive,
    // and not when the whole tile has (Q_FIRST).  Not with 12 wavefronts, whose registers are short.  (8 rows of 2048 tokens,
    // four layers, 41.5 -> 40.5 us, 4 of 8192 44.4 -> 43.3; 54 shapes 0.985 to 1.026 times as fast, 1.002 on average, those
    // with 4-bit codes among them.)
    constexpr bool Q_FIRST = NWB != 12;
    constexpr bool MAY_DRAW = DRAW || (KIND != EQUAL && !ONE);
    const bool dyn = DRAW || (MAY_DRAW && P.seq_mode && !one_split && draws_tiles(P.dynamic, P.splits * NWB, nwf, TF, TQ));
    const __amdgpu_buffer_rsrc_t pool = __builtin_amdgcn_make_buffer_rsrc(
        P.counters + (group * CTR_LINES + 1 + (MAY_DRAW ? deal.pool() : 0)) * CTR_LINE, 0, 4, 0x00020000);
    auto draw = [&]() {   // raw counter value in lane 0
      if constexpr (!MAY_DRAW) return 0;
      else return __builtin_amdgcn_raw_ptr_buffer_atomic_add_i32(1, pool, dyn ? lane * 4 : 4, 0, 0);
    };
    auto drawn_tile = [&](int k) { return deal.drawn(__builtin_amdgcn_readfirstlane(k)); };
    int ta = deal.first, tb = deal.second();
    if (DRAW && deal.takes_units(TF)) {   // done with its units: joins in
      const int ka = draw(), kb = draw();
      ta = drawn_tile(ka);
      tb = drawn_tile(kb);
    }
    uint4 raw[NH];   // zeros for absent heads and past the last channel
    auto load_q = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int hs = 0; hs < NH; ++hs)
        raw[hs] = buffer_load16(rs_q, (int)(prep && 4 * hs + q4 < P.hb ? (uint32_t)((4 * hs + q4) * D + 8 * c8) * 2 : OUT_OF_RANGE), 0);
    };
    if constexpr (Q_FIRST) load_q();
    Tile A;
    Place pa = place(ta);
    if (ta < TQ) {
      load_kmeta(A, pa.t);
      load_kcodes(A, pa);
      load_v(A, pa, 0);
      load_v(A, pa, 1);
    }
    // q of (head q4, channels 8*c8..+7): fp16 pairs for the bias dot products, and
    // fp16 pairs pre-multiplied by 2^(3-2v) (v = pair index) for the q*s operands
    half2_t qz[NH][4], qh[NH][4];
    if constexpr (!Q_FIRST) load_q();
#pragma unroll
    for (int hs = 0; hs < NH; ++hs) {
      const uint32_t qraw[4] = {raw[hs].x, raw[hs].y, raw[hs].z, raw[hs].w};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float f = __builtin_ldexpf(1.f, pos_exp<BITS>(v));
        qh[hs][v] = half2_t{(_Float16)(lo_T<BF16>(qraw[v]) * f), (_Float16)(hi_T<BF16>(qraw[v]) * f)};
        qz[hs][v] = pair_to_f16<BF16>(qraw[v]);
      }
    }
    const float c_codes = P.c * CODE_SCALE<BITS>;   // codes and the pre-scaled q*s together carry 1 / CODE_SCALE
    // slot offsets: this lane's token of tile u is token x = 16*(u&1) + n16 of its
    // 32-token output step, element i = 4*(x/16) + x%4 of its lane group there, whose
    // codes sit at position v = i >> 1
    float offs[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int v = 2 * (u & 1) + ((n16 & 3) >> 1);
      offs[u] = (float)pos_exp<BITS>(v);
    }

    // rows of the q*s operand: matrix row n16 = 4*head + piece, piece 3 is zero
    const uint16_t* qs_rd[NH];
#pragma unroll
    for (int hs = 0; hs < NH; ++hs) qs_rd[hs] = &qs_lds[wave][0][(n16 & 3) < 3 ? 12 * hs + 4 * (n16 & 3) + (n16 >> 2) : QS_ROWS - 1][8 * q4];
    uint16_t* qs_wr = &qs_lds[wave][0][q4][8 * c8];
    // probabilities: written per (head q4, token), read per (head g, token octet q4);
    // lanes of absent channel groups read the zero row
    const uint16_t* p_rd = &p_lds[wave][0][0][!row_live ? 4 : tail_row ? 5 + g : g][4 * q4];
    const uint16_t* p_hd = &p_lds[wave][0][0][!row_live ? 4 : g][4 * q4];
    uint16_t* p_wr = &p_lds[wave][0][0][q4][n16];
    {
#pragma unroll
      for (int e = 0; e < NGRP; ++e)
        if (lane < QS_ROW / 8) *reinterpret_cast<uint4*>(&qs_lds[wave][e][QS_ROWS - 1][8 * lane]) = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int hs = 0; hs < NH; ++hs)
        if (lane < 32) { p_lds[wave][hs][0][4][lane] = 0; p_lds[wave][hs][1][4][lane] = 0; }
    }

    auto process = [&](Tile& cur, const Place& pl, const Place& tn) {   // tn: the tile to refill the registers with
      const int t = pl.t;
      // ---- q*s (fp16 head and tail) and bias = sum_c q_c z_c for each key group
      float bo[NH][4];
      {
        float bias[NH][NGRP];
#pragma unroll
        for (int e = 0; e < NGRP; ++e) {
          const uint32_t sw[4] = {cur.ks8[e].x, cur.ks8[e].y, cur.ks8[e].z, cur.ks8[e].w};
          const uint32_t zw[4] = {cur.kz8[e].x, cur.kz8[e].y, cur.kz8[e].z, cur.kz8[e].w};
          // q*s in three pieces whose sum is the exact product: the top six significant
          // bits of the rounded product, its other five bits, and what the rounding dropped.
          // The code operands are fp16 subnormals; the matrix unit aligns the addends of a
          // dot product by the exponent fields of their operands and keeps about 24 bits
          // below the largest, while a code's bits lie up to 9 bits below its nominal
          // exponent: measured, an 11-bit operand loses its low bits as soon as another
          // channel of the block has a q*s a few times larger.  A six-bit piece has 5 bits
          // of room more, and the two small pieces lose nothing that matters (they may be
          // subnormal themselves: single products of two subnormals were measured exact).
#pragma unroll
          for (int hs = 0; hs < NH; ++hs) {
            float bp = 0.f;
            uint32_t h[4], r[4], l[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma clang fp contract(off)   // hi - top must subtract from the ROUNDED product: fused into fma(q, s, -top) it would hold lo as well
              bp = dot2_h(qz[hs][v], meta_pair(zw[v]), bp);
              const half2_t sh = meta_pair(sw[v]);
              const half2_t hi = qh[hs][v] * sh;
              const half2_t lo = __builtin_elementwise_fma(qh[hs][v], sh, -hi);
              h[v] = __builtin_bit_cast(uint32_t, hi) & 0xFFE0FFE0u;
              r[v] = __builtin_bit_cast(uint32_t, hi - __builtin_bit_cast(half2_t, h[v]));
              l[v] = __builtin_bit_cast(uint32_t, lo);
            }
            if (prep) {
              uint16_t* wr = qs_wr + (e * QS_ROWS + 12 * hs) * QS_ROW;
              *reinterpret_cast<uint4*>(wr) = make_uint4(h[0], h[1], h[2], h[3]);
              *reinterpret_cast<uint4*>(wr + 4 * QS_ROW) = make_uint4(r[0], r[1], r[2], r[3]);
              *reinterpret_cast<uint4*>(wr + 8 * QS_ROW) = make_uint4(l[0], l[1], l[2], l[3]);
            }
            bias[hs][e] = row_sum(bp) * P.c;
          }
        }
        load_kmeta(cur, tn.t);
#pragma unroll
        for (int hs = 0; hs < NH; ++hs)
#pragma unroll
          for (int u = 0; u < 4; ++u) bo[hs][u] = bias[hs][(u * NGRP) >> 2] + offs[u];
      }
      wave_lds_sync();

      // ---- logits: rows (head, piece) x four 16-token tiles, NKC channel chunks each
      floatx4 Du[NH][4];
#pragma unroll
      for (int hs = 0; hs < NH; ++hs)
#pragma unroll
        for (int u = 0; u < 4; ++u) Du[hs][u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < NGRP; ++e) {
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) {
          uint4 qa[NH];
#pragma unroll
          for (int hs = 0; hs < NH; ++hs) qa[hs] = *reinterpret_cast<const uint4*>(qs_rd[hs] + e * (QS_ROWS * QS_ROW) + 32 * kc);
#pragma unroll
          for (int u = e * (4 / NGRP); u < (e + 1) * (4 / NGRP); ++u) {
            const int o = (u & 1) * NKC + kc;
            const uint4 b = operand_codes<BITS>(cur.kc[u >> 1].w, o);
#pragma unroll
            for (int hs = 0; hs < NH; ++hs) Du[hs][u] = mfma_f16(qa[hs], b, Du[hs][u]);
          }
        }
      }

      load_kcodes(cur, tn);

      // this lane: head q4 of each set, token 16*u + n16 of the tile; the three pieces are rows j = 0, 1, 2
      const bool partial = 64 * t + 64 > n_q;
#pragma unroll
      for (int hs = 0; hs < NH; ++hs) {
        float s[4], p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) s[u] = fmaf(Du[hs][u][0] + (Du[hs][u][1] + Du[hs][u][2]), c_codes, bo[hs][u]);
        if (partial) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (64 * t + 16 * u + n16 >= n_q) s[u] = -INFINITY;
        }
        if constexpr (KIND == PADDED) {
          // padding slots behind a short key group (zero codes, zero value scales and
          // zero-points): a finite sentinel, so that a tile made of padding only leaves
          // a state whose weight in every later merge is exactly 0
          const int r0 = G >= 64 ? pl.slot0 : (64 * t) % P.Wq;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            int r = r0 + 16 * u + n16;
            r = r >= P.Wq ? r - P.Wq : r;
            if (r >= P.W) s[u] = DEAD_LOGIT;
          }
        }
        online_softmax_rows<NNT, VPIECES == 1>(st[hs], s, p, g, SLACK);

        // ---- hand the probabilities (fp16) to the lanes that feed the output step
        uint16_t* wr = p_wr + hs * (2 * 9 * 32);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          _Float16 ph16 = (_Float16)p[u];
          // Two pieces and no carried product residual (bf16 caches): the head piece keeps only the three
          // leading significant bits of p, so that its product with a value scale - a bf16 number, 8
          // significant bits - is exact in fp16; the rounding of the product then hits the second piece
          // only, which is at most a quarter of p.
          if constexpr (VPIECES == 2 && !PROD_LO)
            ph16 = __builtin_bit_cast(_Float16, (uint16_t)(__builtin_bit_cast(uint16_t, ph16) & 0xFF00u));
          wr[(u >> 1) * (9 * 32) + 16 * (u & 1)] = __builtin_bit_cast(uint16_t, ph16);
          if constexpr (VPIECES == 2)   // what the head piece leaves out, for the residual rows
            wr[(u >> 1) * (9 * 32) + 16 * (u & 1) + 5 * 32] = __builtin_bit_cast(uint16_t, (_Float16)(p[u] - (float)ph16));
        }
      }
      wave_lds_sync();

      // ---- output: two 32-token steps x NNT channel tiles
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        // (the probabilities are on their way from LDS before the branch)
        uint32_t ph[NH][4], hd[NH][4];   // slots (0,1) (2,3) (4,5) (6,7); the head piece of the same slots
#pragma unroll
        for (int hs = 0; hs < NH; ++hs) {
          const int at = hs * (2 * 9 * 32) + ks * (9 * 32);
          const uint2 pa = *reinterpret_cast<const uint2*>(p_rd + at);        // tokens 4*q4 .. +3
          const uint2 pb = *reinterpret_cast<const uint2*>(p_rd + at + 16);   // tokens 16 + 4*q4 .. +3
          ph[hs][0] = pa.x; ph[hs][1] = pa.y; ph[hs][2] = pb.x; ph[hs][3] = pb.y;
          if constexpr (PROD_LO && VPIECES == 2) {
            const uint2 ha = *reinterpret_cast<const uint2*>(p_hd + at);
            const uint2 hb = *reinterpret_cast<const uint2*>(p_hd + at + 16);
            hd[hs][0] = ha.x; hd[hs][1] = ha.y; hd[hs][2] = hb.x; hd[hs][3] = hb.y;
          }
        }
        uint4 vsr = cur.vs[ks], vzr = cur.vz[ks];
        if (partial) {   // slots beyond n_q hold unspecified bits: keep them out of the sums
          uint32_t keep[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i0 = 2 * r, i1 = 2 * r + 1;
            const int x0 = 16 * ((i0 >> 2) & 1) + 4 * q4 + (i0 & 3), x1 = 16 * ((i1 >> 2) & 1) + 4 * q4 + (i1 & 3);
            keep[r] = (64 * t + 32 * ks + x0 < n_q ? 0x0000FFFFu : 0u) |
                      (64 * t + 32 * ks + x1 < n_q ? 0xFFFF0000u : 0u);
          }
          vsr.x &= keep[0]; vsr.y &= keep[1]; vsr.z &= keep[2]; vsr.w &= keep[3];
          vzr.x &= keep[0]; vzr.y &= keep[1]; vzr.z &= keep[2]; vzr.w &= keep[3];
        }
        const uint32_t vsw[4] = {vsr.x, vsr.y, vsr.z, vsr.w}, vzw[4] = {vzr.x, vzr.y, vzr.z, vzr.w};
        uint4 a[NH], al[NH];
#pragma unroll
        for (int hs = 0; hs < NH; ++hs) {
          uint32_t aw[4], lw[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const half2_t pp = __builtin_bit_cast(half2_t, ph[hs][v]);
            const half2_t sv = meta_pair(vsw[v]);
            if constexpr (!PROD_LO) {
              aw[v] = __builtin_bit_cast(uint32_t, pp * sv);
            } else if constexpr (VPIECES == 2) {
              // head rows: p_hi * vs rounded; residual rows: what that rounding dropped plus p_lo * vs
              const half2_t hh = __builtin_bit_cast(half2_t, hd[hs][v]);
              const half2_t hi = hh * sv;
              const half2_t lo = __builtin_elementwise_fma(pp, sv, __builtin_elementwise_fma(hh, sv, -hi));
              aw[v] = __builtin_bit_cast(uint32_t, tail_row ? lo : hi);
            } else {
              const half2_t hi = pp * sv;
              aw[v] = __builtin_bit_cast(uint32_t, hi);
              lw[v] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(pp, sv, -hi));
            }
            st[hs].zacc[v] = __builtin_amdgcn_fdot2(pp, meta_pair(vzw[v]), st[hs].zacc[v], false);
          }
          a[hs] = make_uint4(aw[0], aw[1], aw[2], aw[3]);
          if constexpr (PROD_LO && VPIECES == 1) al[hs] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
        }
#pragma unroll
        for (int nt = 0; nt < NNT; ++nt) {
          const uint4 b = operand_codes<BITS>(cur.vc[ks].w, nt);
#pragma unroll
          for (int hs = 0; hs < NH; ++hs) {
            st[hs].acc[nt] = mfma_f16(a[hs], b, st[hs].acc[nt]);
            if constexpr (PROD_LO && VPIECES == 1)   // no spare rows: the dropped part takes a product of its own
              st[hs].acc[nt] = mfma_f16(al[hs], b, st[hs].acc[nt]);
          }
        }
        load_v(cur, tn, ks);
      }
      wave_lds_sync();   // p_lds and qs_lds are rewritten by the next tile
    };

    if (ta < TQ) {
      while (true) {
        const bool more = tb < TQ;
        const int kd = draw();                 // for the tile after tb
        const Place pb = place(more ? tb : ta);
        process(A, pa, pb);
        if (ONE && NWB != 12 && ta >= own_half) __builtin_amdgcn_s_setprio(0);
        if (!more) break;
        ta = tb; pa = pb;
        tb = dyn ? drawn_tile(kd) : deal.after(tb);
      }
    }
    // canonical partial of this wavefront: o[g][c], m[g], l[g]
#pragma unroll
    for (int hs = 0; hs < NH; ++hs) {
      float lsum = 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u) lsum += st[hs].l[u] * __builtin_amdgcn_exp2f(-offs[u]);
      const float l_tot = row_sum(lsum);
      float zs = 0.f;
      {
#pragma unroll
        for (int v = 0; v < 4; ++v) zs += st[hs].zacc[v] * __builtin_ldexpf(1.f, -pos_exp<BITS>(v));
      }
      zs = rows_sum(zs);
      if (q4 == 0) zs_lds[wave][up][4 * hs + g] = zs;       // the residual rows hold the residual's share of sum_t p_t vz_t
      if (n16 == 0) { ml_lds[wave][4 * hs + q4][0] = st[hs].m; ml_lds[wave][4 * hs + q4][1] = l_tot; }
    }
    wave_lds_sync();
#pragma unroll
    for (int hs = 0; hs < NH; ++hs) {
      // the accumulators of lane group q4 are the rows of channel group q4 (and of its
      // residual piece, q4 + NGC): sum_t p_t vz_t of that group, both pieces, per head
      if constexpr (VPIECES == 2 && NGC == 2) {
        // Two channel groups, two pieces: lane groups 0 and 2 hold the two pieces of
        // channel group 0, lane groups 1 and 3 those of channel group 1.  One swap of
        // the 32-lane halves of two registers sums the pieces of FOUR channel tiles at
        // once - lane group 0 ends up with the total of tile a, 2 with that of tile b
        // (both of channel group 0), 1 and 3 with tiles c and d of channel group 1 - and
        // every lane group writes its own.
        constexpr int T0 = G / 16;                 // channel tiles of group 0 (group 1: the rest, at most as many)
        const int grp = q4 & 1;
        float zsv[4];
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) zsv[gg] = zs_lds[wave][grp][4 * hs + gg] + zs_lds[wave][grp + NGC][4 * hs + gg];
#pragma unroll
        for (int k = 0; k < (T0 + 1) / 2; ++k) {
          constexpr int NONE = -1;
          const int ta = 2 * k, tb = 2 * k + 1 < T0 ? 2 * k + 1 : NONE;
          const int tc = T0 + 2 * k < NNT ? T0 + 2 * k : NONE, td = T0 + 2 * k + 1 < NNT ? T0 + 2 * k + 1 : NONE;
          const int mine = grp ? (q4 >> 1 ? td : tc) : (q4 >> 1 ? tb : ta);
#pragma unroll
          for (int gg = 0; gg < 4; ++gg) {
            const float xa = st[hs].acc[ta][gg], xb = st[hs].acc[tb == NONE ? ta : tb][gg];
            const float xc = st[hs].acc[tc == NONE ? ta : tc][gg], xd = st[hs].acc[td == NONE ? ta : td][gg];
            const unsigned X = __float_as_uint(grp ? xc : xa), Y = __float_as_uint(grp ? xd : xb);
            const auto r = __builtin_amdgcn_permlane32_swap(X, Y, false, false);
            const float tot = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            if (mine != NONE) o_lds[wave][4 * hs + gg][16 * mine + n16] = tot * CODE_SCALE<BITS> + zsv[gg];
          }
        }
      } else {
        const int gq = q4 < NGC ? q4 : 0;
        float zsv[4];
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
          zsv[gg] = zs_lds[wave][gq][4 * hs + gg];
          if constexpr (VPIECES == 2) zsv[gg] += zs_lds[wave][gq + NGC][4 * hs + gg];
        }
#pragma unroll
        for (int nt = 0; nt < NNT; ++nt) {
          const int gc = (16 * nt) / G;
          if constexpr (VPIECES == 2) {   // add the residual piece's row: lane group q4 + NGC
            float a[4];
#pragma unroll
            for (int gg = 0; gg < 4; ++gg) {
              float x, y;
              xor16_pair(st[hs].acc[nt][gg], &x, &y);   // (NGC == 1)
              a[gg] = x + y;
            }
            if (q4 == gc) {
#pragma unroll
              for (int gg = 0; gg < 4; ++gg) o_lds[wave][4 * hs + gg][16 * nt + n16] = a[gg] * CODE_SCALE<BITS> + zsv[gg];
            }
          } else {
#pragma unroll
            for (int gg = 0; gg < 4; ++gg)
              if (q4 == gc) o_lds[wave][4 * hs + gg][16 * nt + n16] = st[hs].acc[nt][gg] * CODE_SCALE<BITS> + zsv[gg];
          }
        }
      }
    }
  };

  if constexpr (ONE || DRAW) {
    if (deal.takes_units(TF)) { fp_rows(deal.unit0, deal.unit_step); hand_over(); }
    quantized_rows();
  } else if (deal.takes_tiles()) {
    quantized_rows();
  } else {
    fp_rows(deal.unit0, deal.unit_step);
#pragma unroll
    for (int hs = 0; hs < NH; ++hs) {
      const float l_tot = head_sum((st[hs].l[0] + st[hs].l[1]) + (st[hs].l[2] + st[hs].l[3]));
      if (lane < 4) { ml_lds[wave][4 * hs + g][0] = st[hs].m; ml_lds[wave][4 * hs + g][1] = l_tot; }
#pragma unroll
      for (int nt = 0; nt < NNT; ++nt) {
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {   // the sum of head and residual rows
          const float v = st[hs].acc[nt][gg] + __shfl_xor(st[hs].acc[nt][gg], 16);
          if (q4 == 0) o_lds[wave][4 * hs + gg][16 * nt + n16] = v;
        }
      }
    }
  }
  __syncthreads();
  // merge the wavefronts; write this split's partial: per head D floats, then m, l
  for (int idx = threadIdx.x; idx < P.hb * D; idx += 64 * NWB) {
    const int gg = idx / D, c = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NWB; ++w) M = fmaxf(M, ml_lds[w][gg][0]);
    float acc = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < NWB; ++w) {
      const float mw = ml_lds[w][gg][0];
      const float a = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - M);
      acc += a * o_lds[w][gg][c];
      L += a * ml_lds[w][gg][1];
    }
    if (one_split) {   // nothing to merge across workgroups: this is the result
      P.out[(head0 + gg) * D + c] = f2t<BF16>(acc / L);
      continue;
    }
    const int64_t base = part_base + gg * (D + 4);
    st_dev(P.ws + base + c, acc);
    if (c == 0) { st_dev(P.ws + base + D, M); st_dev(P.ws + base + D + 1, L); }
  }
  if (one_split) return;

  // ---- ticket: the last workgroup of this (b, kv head, head group) merges the splits.
  // The barrier waits for this workgroup's stores to be acknowledged before thread 0
  // draws; a workgroup that draws the last ticket therefore finds every partial.
  __shared__ int is_last;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);   // vmcnt(0): the write-through stores above have been acknowledged
  __syncthreads();
  if (threadIdx.x == 0) {
    int* ctr = P.counters + group * (CTR_LINES * CTR_LINE);
    const int old = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    is_last = old == P.splits - 1;
    if (is_last) {   // every other workgroup is past its tile loop and its ticket: re-arm for the next launch
#pragma unroll
      for (int i = 0; i < CTR_LINES; ++i)
        __hip_atomic_store(ctr + i * CTR_LINE, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  if (!is_last) return;
  // Up to NI * RPI splits one wavefront merges a head (several in turn where there are fewer wavefronts).  With more of them
  // NWB / hb wavefronts share the rows (splits) of a head, the others idle, and their sums meet in LDS: 0.8 us less from the ticket to the end at 32 splits,
  // but 0.6 us more at few (3 splits of 512 tokens 9.7 instead of 9.0 us a launch, 8 splits of 2048 tokens at d = 64
  // 8.7 instead of 8.0).  The partials are read past the caches (device-coherent loads), 16 bytes per lane so that the
  // address unit sees few, wide instructions, and the loads of a batch are issued before anything is consumed: the merge
  // then costs about one memory round trip.
  constexpr int PR = D + 4;                    // floats per partial row
  constexpr int C4 = D / 4;                    // 16-byte chunks per row
  constexpr int RPI = 64 / C4;                 // rows covered by one wave-level load
  constexpr int NI = 8;                        // loads in flight
  const int rows = P.splits;
  // one wavefront per head, no sum over wavefronts: where one batch of loads will do, or there are no more wavefronts
  const bool alone = rows <= NI * RPI || NWB <= P.hb;
  const int parts = alone ? 1 : NWB / P.hb;
  const int64_t gstride = (int64_t)P.gh * PR;  // floats between consecutive splits
  float* sum = &o_lds[0][0][0];                // [part][head][D] (o_lds is free again)
  static_assert(sizeof(o_lds) >= NWB * D * sizeof(float), "parts * hb rows of sums, at most NWB");
  for (int hp = wave; hp < P.hb * parts; hp += NWB) {   // (head, part): several heads in turn where there are fewer wavefronts
    const int head = hp % P.hb, part = hp / P.hb;
    const float* gbase = P.ws + ((int64_t)bh * P.splits * P.gh + hsub * P.hb + head) * PR;
    // buffer descriptor over this head's rows of all splits: out-of-range lanes read 0
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(gbase), 0, (int)(((int64_t)(rows - 1) * gstride + PR) * 4), 0x00020000);
    const int r = lane / C4, c4 = lane % C4;
    const int oob = 0x7FFFFFF0;
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    u32x2 ml[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int sidx = lane + 64 * k;
      ml[k] = __builtin_amdgcn_raw_buffer_load_b64(rs, sidx < rows ? (int)((sidx * gstride + D) * 4) : oob, 0, 16);
    }
    // load i of this wavefront: rows (i * parts + part) * RPI + r; past the last row the descriptor's end makes it zeros
    const int row0 = part * RPI + r, row_step = parts * RPI;
    const uint32_t off0 = r < RPI ? (uint32_t)(row0 * gstride + 4 * c4) * 4 : (uint32_t)oob, off_step = (uint32_t)(row_step * gstride) * 4;
    u32x4 ov[NI];
    auto load_rows = [&](int i0) {               // the i0-th .. (i0 + NI - 1)-th load of this wavefront
      uint32_t off = off0 + i0 * off_step;
#pragma unroll
      for (int i = 0; i < NI; ++i, off += off_step) ov[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 16);
    };
    load_rows(0);
    float w[4], mx = -INFINITY, ls = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w[k] = lane + 64 * k < rows ? __uint_as_float(ml[k][0]) : -INFINITY;
      mx = fmaxf(mx, w[k]);
    }
    mx = rows_max(row_max(mx));
    float* weight = reinterpret_cast<float*>(&p_lds[wave][0][0][0]);   // this wavefront's copy, free again
    static_assert(sizeof(p_lds[0]) >= 256 * sizeof(float), "a weight for each split");
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w[k] = w[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(w[k] - mx);
      ls += w[k] * __uint_as_float(ml[k][1]);    // (0 * 0 past the last row)
      weight[lane + 64 * k] = w[k];
    }
    ls = rows_sum(row_sum(ls));
    wave_lds_sync();
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0;;) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const float wi = weight[(row0 + (i0 + i) * row_step) & 255];   // (past the last row the loads are zeros)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(wi, __uint_as_float(ov[i][e]), acc[e]);
      }
      i0 += NI;
      if (i0 * row_step >= rows) break;
      load_rows(i0);
    }
    // add the RPI row classes (lanes c4, c4 + C4, ...), then the parts, in LDS
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float t = acc[e];
#pragma unroll
      for (int k = 1; k < RPI; ++k) t += from_lane(acc[e], (lane + k * C4) & 63);
      acc[e] = t;
    }
    if (!alone) {
      if (lane < C4) *reinterpret_cast<float4*>(sum + (part * P.hb + head) * D + 4 * c4) = make_float4(acc[0], acc[1], acc[2], acc[3]);
      if (part == 0 && lane == 0) ml_lds[0][head][1] = ls;
    } else if (lane < C4) {
      const float inv = 1.0f / ls;
      *reinterpret_cast<uint2*>(P.out + (head0 + head) * D + 4 * c4) =
          make_uint2((uint32_t)f2t<BF16>(acc[0] * inv) | ((uint32_t)f2t<BF16>(acc[1] * inv) << 16),
                     (uint32_t)f2t<BF16>(acc[2] * inv) | ((uint32_t)f2t<BF16>(acc[3] * inv) << 16));
    }
  }
  if (alone) return;
  __syncthreads();
  for (int idx = threadIdx.x; idx < P.hb * D / 2; idx += 64 * NWB) {
    float2 t = *reinterpret_cast<const float2*>(sum + 2 * idx);
    for (int k = 1; k < parts; ++k) {
      const float2 x = *reinterpret_cast<const float2*>(sum + k * P.hb * D + 2 * idx);
      t.x += x.x; t.y += x.y;
    }
    const float inv = 1.0f / ml_lds[0][2 * idx / D][1];
    *reinterpret_cast<uint32_t*>(P.out + head0 * D + 2 * idx) =
        (uint32_t)f2t<BF16>(t.x * inv) | ((uint32_t)f2t<BF16>(t.y * inv) << 16);
  }
}

template <bool BF16, int D, int NWB, int BITS, int NH, int KIND, int PROG>
static hipError_t launch_mfma_g(const Shape& s, const AttnParams& P, const SeqArg* seq, dim3 grid, hipStream_t st) {
  SeqArgs<KIND> S;
  if constexpr (KIND != EQUAL)
    if (seq && seq->in_args())
      for (int i = 0; i < seq->n; ++i) S.e[i] = seq->host[i];
  switch (s.G) {
    case 32: hipLaunchKernelGGL((attn_mfma_kernel<BF16, D, 32, NWB, BITS, KIND, PROG, NH>), grid, dim3(64 * NWB), 0, st, P, S); break;
    case 64: hipLaunchKernelGGL((attn_mfma_kernel<BF16, D, 64, NWB, BITS, KIND, PROG, NH>), grid, dim3(64 * NWB), 0, st, P, S); break;
    default: hipLaunchKernelGGL((attn_mfma_kernel<BF16, D, 128, NWB, BITS, KIND, PROG, NH>), grid, dim3(64 * NWB), 0, st, P, S); break;
  }
  return launch_status(__func__);
}

template <bool BF16, int D, int NWB, int BITS, int NH, int PROG>
static hipError_t launch_mfma_k(const Shape& s, const AttnParams& P, const SeqArg* seq, dim3 grid, hipStream_t st) {
  if constexpr (PROG != DRAWN || NWB != 4)
    if (s.Wq != s.W) return launch_mfma_g<BF16, D, NWB, BITS, NH, PADDED, PROG>(s, P, seq, grid, st);
  if constexpr (PROG != DRAWN)   // (with counts per row each row decides for itself whether it draws)
    if (seq) return launch_mfma_g<BF16, D, NWB, BITS, NH, PER_ROW, PROG>(s, P, seq, grid, st);
  return launch_mfma_g<BF16, D, NWB, BITS, NH, EQUAL, PROG>(s, P, seq, grid, st);
}

template <bool BF16, int D, int NWB, int BITS, int NH>
static hipError_t launch_mfma_p(const Shape& s, const AttnParams& P, const SeqArg* seq, dim3 grid, hipStream_t st) {
  const int NW = P.splits * NWB, TF = (P.n_fp + 31) / 32, TQ = P.tiles;
  if (P.splits == 1 && P.n_q > 0) return launch_mfma_k<BF16, D, NWB, BITS, NH, ONE_SPLIT>(s, P, seq, grid, st);
  // (With counts per sequence each row decides for itself, in the kernel.  Padded rows of one length are not planned with
  // 4 wavefronts: forced to, they take their tiles in a fixed order.)
  if (P.splits > 1 && !seq && !(NWB == 4 && s.Wq != s.W) && draws_tiles(P.dynamic, NW, P.nwf, TF, TQ))
    return launch_mfma_k<BF16, D, NWB, BITS, NH, DRAWN>(s, P, seq, grid, st);
  if constexpr (NWB == 8)
    if (!keeps_units_together(NW, P.nwf, TQ, (int64_t)grid.x * grid.y * grid.z >= compute_units()))
      return launch_mfma_k<BF16, D, NWB, BITS, NH, APART>(s, P, seq, grid, st);
  return launch_mfma_k<BF16, D, NWB, BITS, NH, BY_SPLIT>(s, P, seq, grid, st);
}

template <bool BF16, int NWB, int BITS, int NH>
static hipError_t launch_mfma_d(const Shape& s, const AttnParams& P, const SeqArg* seq, dim3 grid, hipStream_t st) {
  switch (s.d) {
    case 64: return launch_mfma_p<BF16, 64, NWB, BITS, NH>(s, P, seq, grid, st);
    case 96: return launch_mfma_p<BF16, 96, NWB, BITS, NH>(s, P, seq, grid, st);
    default: return launch_mfma_p<BF16, 128, NWB, BITS, NH>(s, P, seq, grid, st);
  }
}

// One source file for each of these (lq_attn_mfma_w*.hip): 1440 kernels in all, which as one file took many minutes.
template <int NWB, int BITS, int NH>
hipError_t launch_mfma_t(const Shape& s, const AttnParams& P, const SeqArg* seq, dim3 grid, hipStream_t st) {
  return s.bf16 ? launch_mfma_d<true, NWB, BITS, NH>(s, P, seq, grid, st)
                : launch_mfma_d<false, NWB, BITS, NH>(s, P, seq, grid, st);
}

}  // namespace lq
