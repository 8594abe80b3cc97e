// Decode attention: kernel arguments from the call's, and the choice of the kernel shape.
#include <stdlib.h>

#include "lq_attn_mfma.h"

namespace lq {

extern template hipError_t launch_mfma_t<12, 2, 1>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<8, 2, 1>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<8, 4, 1>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<4, 2, 1>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<4, 4, 1>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<8, 2, 2>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<8, 4, 2>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<4, 2, 2>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
extern template hipError_t launch_mfma_t<4, 4, 2>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);

template <int NH>
static hipError_t launch_heads(const Shape& s, const AttnParams& P, int waves_per_block, const SeqArg* seq, dim3 grid, hipStream_t st) {
  if constexpr (NH == 1)
    if (waves_per_block == 12) return launch_mfma_t<12, 2, 1>(s, P, seq, grid, st);
  if (waves_per_block == 4)
    return s.bits == 4 ? launch_mfma_t<4, 4, NH>(s, P, seq, grid, st) : launch_mfma_t<4, 2, NH>(s, P, seq, grid, st);
  return s.bits == 4 ? launch_mfma_t<8, 4, NH>(s, P, seq, grid, st) : launch_mfma_t<8, 2, NH>(s, P, seq, grid, st);
}

// seq == nullptr: every sequence has the counts of `c` and the live buffer c.cur;
// otherwise the kernel reads counts, live buffer and fp-wavefront share per sequence
// from the state array (in its own arguments for small batches, else on the device;
// c.n_fp / c.n_q are then the largest counts, which `plan` was made for).
hipError_t launch_decode_attn_mfma(const Shape& s, const lq_cache& c, const void* q, float scale,
                                   void* out, const Workspace& ws, const lq_plan& plan, hipStream_t st,
                                   const void* k_new, const void* v_new, const SeqArg* seq) {
  AttnParams P;
  P.k_new = (const uint16_t*)k_new; P.v_new = (const uint16_t*)v_new;
  const int first = seq ? 0 : c.cur;
  P.k_fp[0] = (uint16_t*)c.k_fp[first]; P.k_fp[1] = (uint16_t*)c.k_fp[first ^ 1];
  P.v_fp[0] = (uint16_t*)c.v_fp[first]; P.v_fp[1] = (uint16_t*)c.v_fp[first ^ 1];
  P.pos_fp[0] = c.pos_fp[first]; P.pos_fp[1] = c.pos_fp[first ^ 1];
  P.seq = seq ? seq->dev : nullptr; P.seq_mode = seq_mode(seq);
  P.Hkv = s.Hkv;
  P.q = (const uint16_t*)q;
  P.k_codes = c.k_codes; P.v_codes = c.v_codes;
  P.k_scale = (const uint16_t*)c.k_scale; P.k_zero = (const uint16_t*)c.k_zero;
  P.v_scale = (const uint16_t*)c.v_scale; P.v_zero = (const uint16_t*)c.v_zero;
  P.counters = ws.counters;
  P.ws = ws.partials;
  P.out = (uint16_t*)out;
  P.cap = s.cap; P.qcap = s.qcap; P.n_fp = c.n_fp; P.n_q = c.n_q; P.gh = s.gh;
  P.W = s.W; P.Wq = s.Wq; P.live.set(s.W, s.Wq);
  P.dead_bit = (int64_t)s.qcap * s.d * s.bits / 8 <= ((int64_t)1 << 31) ? 0x80000000u : 0u;   // (codes: the largest array)
  P.tiles = tiles_of(s, c.n_q); P.n_tok_q = quantized_tokens(s, c.n_q);
  const int groups = plan.blocks / plan.splits;   // B * Hkv * (gh / hb), as planned
  P.hb = s.gh / (groups / (s.B * s.Hkv));
  P.splits = plan.splits; P.nwf = plan.fp_waves; P.cus = seq && pairs_workgroups(plan) ? 1 << 30 : compute_units();
  P.c = scale * 1.4426950408889634f;
  static const int dynamic = [] { const char* v = getenv("LOGQUANT_ATTN_DYNAMIC"); return v && *v ? atoi(v) : 1; }();
  P.dynamic = dynamic;
  P.across = groups % 8 == 0 ? 8 : 1;
  P.div_subgroups.set(s.gh / P.hb); P.div_kv_heads.set(s.Hkv);
  const dim3 grid(P.across, plan.splits, groups / P.across);
  return P.hb > 4 ? launch_heads<2>(s, P, plan.waves_per_block, seq, grid, st) : launch_heads<1>(s, P, plan.waves_per_block, seq, grid, st);
}

}  // namespace lq
