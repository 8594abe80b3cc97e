// Host-side internals: validated shape bundle and kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/logquant.h"
#include "lq_schedule.h"

namespace lq {

struct Shape {
  int B, Hq, Hkv, d, W, G, cap, qcap, gh;  // gh = Hq/Hkv; cap = fp rows allocated per slice (3W rounded up to 32)
  int full;                                // 3W: list length at which the filtering step runs
  int Wq;                                  // quantized slots per filtering event: ceil(W/G) * G (W when G divides W)
  int nkc, nnt, ngc;                       // d/32, d/16, ceil(d/G)
  int bits;                                // 2 or 4
  bool bf16;
};

// Per-sequence lengths: one entry per batch row in device memory, written by the
// library at the start of every call of the per-sequence entry points and read by
// that call's kernels (a way to hand B sets of counts to a launch, not state).
struct SeqState {
  int n_fp, n_q;      // rows in the fp region, slots in the quantized region
  int cur;            // which fp buffer is live
  int nwf;            // attention: wavefronts of a head group that keep to the fp rows where a share of them does
  int n_tok_q;        // tokens held in the n_q slots
  int item;           // compress: the i-th entry names the i-th sequence that is compressed; attention: tiles_of(n_q)
  int flag;           // append: 1 if the sequence takes a token; prefill: prompt length
  int order;          // attention: the i-th entry names the row with the i-th most tokens
};

constexpr int SEQ_CHUNK = 64;   // entries that fit a launch's own arguments (2 KB)
hipError_t launch_seq_upload(SeqState* dst, const SeqState* host, int n, hipStream_t st);

// How a launch gets the per-sequence state: batches of up to SEQ_CHUNK rows carry it in
// their own kernel arguments (`host`), larger ones read the device array (`dev`), which
// the caller of the launcher has filled with launch_seq_upload on the same stream.
struct SeqArg {
  const SeqState* dev;
  const SeqState* host;
  int n;
  bool in_args() const { return n <= SEQ_CHUNK; }
};
struct SeqInline { SeqState e[SEQ_CHUNK]; };
inline void fill_inline(SeqInline* S, const SeqArg* a) {
  if (a && a->in_args())
    for (int i = 0; i < a->n; ++i) S->e[i] = a->host[i];
}
// Kernel side: the state array inside the launch's own argument block.  It is read through
// the argument segment's address (scalar loads at a run-time index); indexing the by-value
// parameter itself makes the compiler copy all of it into private memory first.
// `offset` = where the array parameter starts in the argument block.
typedef const SeqState __attribute__((address_space(4))) * SeqArgsPtr;
__device__ __forceinline__ SeqArgsPtr seq_in_args(size_t offset) {
  typedef const char __attribute__((address_space(4))) * BytePtr;
  return (SeqArgsPtr)((BytePtr)__builtin_amdgcn_kernarg_segment_ptr() + offset);
}
__device__ __forceinline__ SeqState seq_load(SeqArgsPtr p, int i) {
  SeqState r;
  r.n_fp = p[i].n_fp; r.n_q = p[i].n_q; r.cur = p[i].cur; r.nwf = p[i].nwf;
  r.n_tok_q = p[i].n_tok_q; r.item = p[i].item; r.flag = p[i].flag; r.order = p[i].order;
  return r;
}
constexpr size_t args_offset_after(size_t bytes_before) { return (bytes_before + 3) / 4 * 4; }   // SeqState is 4-byte aligned
// kernel-side selector: 0 = no per-sequence state, 1 = in the kernel arguments, 2 = device array
inline int seq_mode(const SeqArg* a) { return !a ? 0 : a->in_args() ? 1 : 2; }

// Fills `s`; returns LQ_OK or the config error.  Pure host arithmetic.
lq_status make_shape(const lq_config* cfg, Shape* s);

// Query heads of a kv head that one workgroup works on.  Up to eight share the loads and the unpacked codes; beyond four
// they are two sets, each with its own softmax and matrix operands, and a tile or unit takes a wavefront longer.  With
// eight heads per kv head two workgroups of four win in small launches, where latency counts and twice the wavefronts
// share it, and one of eight in large ones, which read every byte once.  Of 110 shapes with eight heads per kv head, the 66
// that read less than 24 MB take 0.91 to 1.54 of the time with one set of eight (1.2 on average), the 44 others 0.68 to 1.10
// (0.88): 30 kv heads x 7872 slots, bf16, 27 MB, 19.8 -> 15.1 us; 184 x 3700, 4 bits, 116 MB, 42.9 -> 29.0; but
// 4 x 46000, 19 MB, 14.5 -> 16.2.  Six heads are the same: two workgroups of three below 24 MB (one set takes 0.98 to 1.43 of
// their time, 1.27 on average, 15 shapes), one set above (0.82, 1.03 and 1.11).  Ten and fourteen are fives or sevens against
// twos: the larger sets from where they save 24 MB of reading, 8 and 4.8 MB of the cache (0.89 to 1.45 of the time below it,
// 1.21 on average, 16 shapes, 0.54 to 1.25, 0.85, above it, 45: 14 heads, 1 kv head x 18750 tokens, 8.2 -> 11.8 us; 24 x 5200,
// d = 96, 41 -> 22).  Twelve and fifteen stay fours and threes: sixes and fives read too little less (above 24 MB 0.96 to
// 1.09, 1.04 on average, 7 shapes).  Five and seven, else one head at a time, always are one set: 0.26 to 1.09 of the time
// from 10 MB, 0.68 on average (16 kv heads of 4096 tokens, 7 heads, 17.2 -> 12.8 us), though 1.05 to 1.50 below 4 MB, 1.27 on
// average (7 heads, 1 kv head x 6250, d = 64, 6.5 -> 8.5).
// Rows of different lengths count as so many of the longest, like the rest of their plan (by what they read 16 rows of 300 to
// 8000 tokens, 8 kv heads, would take 26.5 instead of 30.7 us, but 24 of 600 to 6000, 4 kv heads, 21.0 instead of 17.2).
inline int most_heads(const Shape& s, int limit) {
  int hb = s.gh < limit ? s.gh : limit;
  while (s.gh % hb) --hb;
  return hb;
}
inline int heads_per_group(const Shape& s, int64_t bytes_read) {
  const int many = most_heads(s, 8), few = most_heads(s, 4);
  if (few == 1) return many;
  if (3 * many <= 5 * few) return few;
  const int64_t saved = bytes_read * (s.gh / few - s.gh / many);
  return bytes_read < 24000000 && (many <= 2 * few || saved < 24000000) ? few : many;
}

// Upper bound on context splits per (b, kv head) that decode_attn may use.
int max_splits(const Shape& s);

// The workspace starts with the counters of the attention kernel: per (b, kv head,
// head group) CTR_LINES cache lines of CTR_LINE ints, each holding one counter in
// its first int: line 0 the ticket counter, lines 1..NSUB the tile pool counters.
// The splits' partial results follow.
constexpr int CTR_LINE = 32, CTR_LINES = 1 + NSUB;
inline size_t counter_bytes(const Shape& s) {
  return (size_t)s.B * s.Hkv * s.gh * CTR_LINES * CTR_LINE * sizeof(int);
}
hipError_t launch_workspace_init(const Shape& s, void* ws, hipStream_t st);
// The two parts of a workspace as the attention launchers take them.
struct Workspace {
  int* counters;
  float* partials;
};
inline Workspace split_workspace(const Shape& s, void* ws) {
  return Workspace{(int*)ws, (float*)((char*)ws + counter_bytes(s))};
}
// `n` ints at `p` set to zero by a small kernel (safe to record into a HIP graph).
hipError_t launch_zero_ints(int* p, int n, hipStream_t st);

// Bytes one decode step reads from the cache (live slots only).
int64_t cache_bytes_read(const Shape& s, int n_fp, int n_q);
// Tokens held in n_q quantized slots (n_q is a multiple of Wq; W of every Wq slots are live).
inline int quantized_tokens(const Shape& s, int n_q) { return n_q / s.Wq * s.W; }

// hipGetLastError() also reports failures of earlier, unrelated runtime calls made
// by other code in the process (an expected hipErrorNotReady, say).  Launchers
// clear that state first and report only what their own launch produced.
inline void clear_stale_error() { (void)hipGetLastError(); }
hipError_t launch_status(const char* what);

// --- launchers (enqueue only) -------------------------------------------------
hipError_t launch_append(const Shape& s, const lq_cache& c, const void* k_new, const void* v_new,
                         int n_new, hipStream_t st);
hipError_t launch_append_seq(const Shape& s, const lq_cache& c, const void* k_new, const void* v_new,
                             const SeqArg* seq, hipStream_t st);
// seq == nullptr: every sequence is compressed, from the counts of `c`.  Otherwise the
// n_items sequences named by seq[0..n_items).item, each from its own counts.
hipError_t launch_compress(const Shape& s, const lq_cache& c, hipStream_t st, const SeqArg* seq = nullptr,
                           int n_items = 0);
// seq == nullptr: one prompt length L for all.  Otherwise seq[b].flag is the prompt length of
// sequence b (n_fp / n_q what it leads to), L the row stride of the prompt tensors and
// E / n_fp the largest values over the batch (they size the grid).
hipError_t launch_prefill(const Shape& s, const lq_cache& c, const void* k, const void* v, int L, int E,
                          int n_fp, hipStream_t st, const SeqArg* seq = nullptr);
hipError_t launch_decode_attn(const Shape& s, const lq_cache& c, const void* q, float scale,
                              void* out, const Workspace& ws, const lq_plan& plan, hipStream_t st,
                              const SeqArg* seq = nullptr);
hipError_t launch_decode_step(const Shape& s, const lq_cache& c, const void* k_new, const void* v_new,
                              const void* q, float scale, void* out, const Workspace& ws, const lq_plan& plan,
                              hipStream_t st, const SeqArg* seq = nullptr);
enum Rows { LOCK_STEP, SAME_LENGTH, DIFFERENT_LENGTHS };   // one set of counts, or counts per row
void plan_decode(const Shape& s, int n_fp, int n_q, lq_plan* plan, Rows rows = LOCK_STEP);
int compute_units();   // of the device the launches are planned for
// Rows of different lengths, workgroups of 4 wavefronts that are on the chip all at once, two to a compute unit: the
// longest row shares a compute unit with the shortest, and the workgroups dispatched last, the short ones, get no
// precedence (64 rows of up to 4096 tokens, 16 steps: 702 -> 672 us; 38 of 10277, four layers: 147 -> 143).
inline bool pairs_workgroups(const lq_plan& plan) {
  return plan.waves_per_block == 4 && plan.blocks > compute_units() && plan.blocks <= 2 * compute_units();
}
// Tiles of n_q quantized slots that the attention kernel deals out: those that hold tokens, where padding comes in
// whole tiles (LiveTiles), else all.
inline int tiles_of(const Shape& s, int n_q) { return s.G >= 64 ? n_q / s.Wq * ((s.W + 63) / 64) : (n_q + 63) / 64; }
// How many wavefronts' worth of time (of the NW a head group has) n_fp fp rows take beside
// n_q quantized slots.
int fp_wave_share(const Shape& s, int NW, int n_fp, int n_q);

}  // namespace lq
