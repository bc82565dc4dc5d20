// The whole step loop of a decoder in one launch whose blocks keep the weights on chip from the first step to the
// last ("resident" loop).
//
// What bounds the per-step launches is not their work but their boundaries: three dependent kernels of 4 to 14 us per
// step of which each pays 2 to 3 us of launch head and tail, fetches the weights anew (the caches do not survive a
// kernel boundary) and hands its results over through memory.  Here the utterances are dealt out to groups of blocks
// (one group per 32 compute units where there are as many utterances, each on an XCD of its own; that more, emptier groups beat
// fewer, fuller ones has not been measured) that decode them independently of each other.  A group holds every weight of
// the three contractions once, in registers and LDS: a block owns some 16-row tiles of W_hh (at most 6, with the LSTM
// cells of their four units each), of the output layer and of the prediction projection.  One step of a group:
//   cell    words of the last step -> the owners of W_hh tiles update the cells of their units        -> h
//   P       h    -> the owners of projection tiles: pre = f_proj[frame] + W_pred h + b_pred           -> pre
//   J       pre  -> the owners of output-layer tiles: z = W_out ReLU(pre) + b_out                     -> logits
//   select  z    -> one to four utterances per block (its waves share out the rows of logits, one per utterance selects): the Beam best
//           of all, tree, ..   -> words
//   R       h    -> the owners of W_hh tiles: W_hh h for the next cell update, under the selection
// Hand-over between blocks: an array that one phase writes and another reads is pre-filled with a bit pattern that no
// result has (a NaN with all bits set); the reader loads the data itself, device-coherently, until none of it holds the
// pattern.  No barrier, no flag and no acknowledged store lies between the two (one hop costs 0.5 us; stores, their
// acknowledgement, a counter and then the loads 2.0 us).  Where the blocks of a group find themselves on one XCD they hand over through
// its L2, else their stores are written through.  The words of the selection carry the step's number instead.
// A writer puts the pattern back once a word of a later phase proves that every reader is through (see the clear_
// functions), one or two steps before the place is used again.
//
// Every sum is formed in the order of the per-step kernels (K slices of 1/8 of the contraction, slices added first to last), so the
// results are the same bit for bit.  Float32 models from 320 wide on whose weights can be split multiply on the float16 matrix
// instructions, both operands split in two (see split_f16): in float32, W_hh h took 3.2 us per step and tile of 16 slots, longer than the selection it hides under (2.9), and the other
// two contractions 3 us of the chain.  bf16-joint models keep W_hh h on float32 matrix instructions (a 16x16x4 one rounds like four
// fused multiply-adds in a row): they round activations to 8 bits, and near ties there follow every last bit of the hidden state.
// (ms per decode before / after the splits, the gathers and the ends of waves described below: one utterance 8.65 / 6.95, greedy batch
// 32 9.05 / 7.05, batch 32 beam 4 9.05 / 7.55, TDT batch 64 5.1 / 4.1, LM 16.5 / 13.8.)
//
// Stateless decoders (ST) have no cells and no projection: pre is a sum of table rows, f_proj[frame] + tab_0[last token] +
// tab_1[the one before] + .., and every owner of output-layer tiles forms its own slice of it from the words (see
// res_stateless_pre), so that a step is two hops (words -> z -> words).  The owners keep the slots' last tokens themselves.
// (batch 8, beam 4, bf16 joint, 640 wide, V = 1024: 5.46 ms per decode with the per-step launches, 2.62 here.)
//
// Every wait is bounded: a wave that waits too long raises the abort word and ends, every other wave sees the word (or
// its own limit) and ends too, and the host decodes the batch with the per-step launches instead.
#pragma once
#include <type_traits>

#include "lm_device.h"
#include "select.h"

namespace rb {

constexpr int kResWaves = 8, kResThreads = 64 * kResWaves;
constexpr int kResSlot = 16;         // slots per tile
constexpr int kResMaxNT = 3;         // slot tiles per group
constexpr int kResMaxR = 6;          // W_hh tiles per block
constexpr int kResMaxLdsTiles = 2;   // tiles that wait in LDS: projection tiles and the output-layer tile beyond those in registers
constexpr int kResMaxP = 2;
constexpr int kResMaxSel = 4;        // utterances per selecting block (more where the others find no room, see make_plan)
constexpr int kResMaxRounds = 10;    // rounds of 8 k per wave slice: H, P <= 640
constexpr int kResQuads = 5;         // 16-byte words of a lane of a split tile
constexpr int kResTileFloats = kResWaves * kResQuads * 64 * 4;  // a split tile
constexpr int kResMaxV = 1024;
constexpr int kResStepRing = 4;      // ring of the hand-over arrays
// The words of a step are written in several places, of which a block polls one: the waves of a group, up to 240 of them, that poll one
// line of the L2 hold each other up.
constexpr int kResWordCopies = 4, kResWordPlace = 64;  // and the distance of the places, at least a group's slots
constexpr int kResNotLocal = -2;     // stall_step of a test: the groups take themselves to lie on several XCDs
constexpr uint32_t kResEmpty = 0xffffffffu;
// How a decoder's products are formed: on float32 matrix instructions; W_out and W_pred on bf16 ones (the bf16 joint); on float16 ones
// from split operands (see split_f16).
enum ResForm { kResF32, kResBf16, kResSplit };
constexpr int kResRedBlock = 2048;   // floats of one 16-row tile's partial sums: 8 waves x 64 lanes x 4

// What one block of a group owns (the same table for every group).
struct ResTab {
  int8_t nR, nJ, nP, pad;
  int16_t R[kResMaxR], J[3], P[kResMaxP];
};
// output-layer tiles a block keeps in registers (a tile is 16 rows; 32 with the bf16 matrix instructions)
template <bool BF16>
constexpr int kResRegJ = BF16 ? 1 : 2;
// 16-row tiles whose partial sums one half of the buffer holds, at least (with split operands four where LDS has room: both halves of k
// of two projection tiles)
template <bool BF16>
constexpr int kResRedBlocks = BF16 ? 4 : 3;

// Fragment order of an activation vector set: round (8 k), k-quad kq, slot, 2 floats; element 0 is k = 8 round +
// {0, 4, 1, 5}[kq], element 1 is two further.  A lane (slot, kq) of a wave reads its two matrix operands of a round with one
// 8-byte load.  Unit order within a W_hh tile follows: tile t holds units 8 (t / 2) + t % 2 + {0, 2, 4, 6}, whose 16
// slots are 256 contiguous bytes.
__host__ __device__ inline int res_k_of(int round, int kq, int e) { return 8 * round + (kq & 1) * 4 + (kq >> 1) + 2 * e; }

struct ResArgs {
  const uintx4_t *WR, *WJ, *WP;      // kResSplit: [tile][wave][kResQuads * 64] (see k_pack_split)
  const float *WRf, *WJf, *WPf;      // else, [tile][round][64 lanes][2] (kResBf16: W_hh only)
  const float *hh_unscale, *out_unscale, *pred_unscale;  // of their rows (see k_split_rows)
  const float *WJs;                  // the tile that begins with the blank column, for res_fold_mma: see k_pack_fold
  const uint64_t *WJb, *WPb;         // kResBf16: [32-row tile][round][64 lanes] four bf16 (k of the lane's half)
  const float *b_out, *b_pred, *G, *f_proj;
  const float *emb_tab;              // stateless decoders: [n_ctx][V + 1][H], else null
  int n_ctx;
  const int *lengths;
  float *hb, *pb, *zb;               // rings of the hand-over arrays, all groups
  uint64_t *words;
  const ResTab *tab;                 // of the group's blocks behind the selecting ones
  int *ctl;                          // [0] blocks that have started, [1] abort, [2 + group] the XCDs that its blocks found themselves on
  volatile int *h_abort;             // pinned host word
  SelectArgs sel;
  LmView lm;
  int B, K, T, V, N, Npad, H, P;
  int n_groups, stride;              // groups; block i of the launch is of group i % stride (there may be fewer groups)
  int n_sel, upc;                    // per group: selecting blocks, utterances of each
  int NT, halves, has_lm;            // slot tiles per group
  int red_blocks;                    // see kResRedBlocks
  int rounds_h, rounds_p;            // rounds of 8 k per wave slice over H and over P
  int poll_limit, start_limit;       // polls of a data wait; ticks (10 ns) of the wait for all blocks
  int start_blocks;                  // how many those are
  int fold;                          // the per-step launches would fold the blank and duration columns (see res_fold_mma)
  int stall_step;                    // a test's: from this step on the last tile of slots gets no logits (below 0: never)
};

// whether the blocks of a group, which found themselves on these XCDs, hand over through one XCD's L2 (see res_store)
__host__ __device__ inline bool res_on_one_xcd(int xcds, int stall_step) { return xcds != 0 && (xcds & (xcds - 1)) == 0 && stall_step != kResNotLocal; }

// The kernel's arguments, read from the argument segment anew at the begin of every phase: kept in scalar registers over
// the whole loop they would push the weights out of the vector registers (a thousand spills).  What is left by the compiler's
// report: LSTM forms no vector register spilled but 60 to 70 where the weights are split and less than 640 wide, and 100 to 200 scalar
// ones (into vector lanes), 244 to 256 vector registers in use; stateless forms no vector register, 70 to 105 scalar ones.  The selecting blocks, whose code needs the scalar ones, share the kernel with the owners of the weights.
__device__ __forceinline__ const ResArgs &res_args() {
  typedef const __attribute__((address_space(4))) ResArgs ConstArgs;
  ConstArgs *p = (ConstArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const ResArgs *)p;
}

__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ float lo_f(uint64_t x) { return __uint_as_float((uint32_t)x); }
__device__ __forceinline__ float hi_f(uint64_t x) { return __uint_as_float((uint32_t)(x >> 32)); }
// whether any of a lane's words still holds the pattern in one of its halves: the pattern is the largest 32-bit number
template <int N>
__device__ __forceinline__ bool res_any_empty(const uint64_t (&x)[N]) {
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) m = max(m, max((uint32_t)x[i], (uint32_t)(x[i] >> 32)));
  return m == kResEmpty;
}
// x[i] for an index that is the same in all lanes but not known at compile time
template <int N>
__device__ __forceinline__ uint64_t res_pick(const uint64_t (&x)[N], int i) {
  uint64_t v = x[0];
#pragma unroll
  for (int q = 1; q < N; ++q) v = i == q ? x[q] : v;
  return v;
}
__device__ __forceinline__ uint64_t pack2(float lo, float hi) {
  return (uint64_t)__float_as_uint(hi) << 32 | __float_as_uint(lo);
}

// Giving up is a matter of the whole block: a wave whose wait fails leaves a flag in LDS and ends (the barriers no longer
// count it), and every wave looks at the flag behind each barrier that follows a wait, before it uses or publishes what
// the others should have left in LDS.  (Reading the flag along with that and looking at it last: 1 to 3 % slower.)
// (An LDS address, not a generic pointer: a flat load of the word waited for every store and load that the wave had in flight.)
typedef __attribute__((address_space(3))) int LdsInt;
__device__ __forceinline__ LdsInt *res_gave_up_word() {
  __shared__ int word;
  return (LdsInt *)&word;
}
// (Ending the wave where it gives up, rather than by a result handed up through every caller, leaves the compiler no paths on which
// the awaited words are undefined: those took registers and moves.)
__device__ __forceinline__ void res_end_if_given_up() {
  if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(res_gave_up_word(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0) __builtin_amdgcn_endpgm();
}
// bounded waiting: between two polls; the wave ends here when it has waited too long, or when another one has
struct ResWait {
  int n = 0;
  __device__ __forceinline__ void again() {
    if ((++n & 255) != 0) return;
    const ResArgs &a = res_args();
    if (n < a.poll_limit && !load_agent(a.ctl + 1)) return;
    store_agent(a.ctl + 1, 1);
    *a.h_abort = 1;
    __hip_atomic_store(res_gave_up_word(), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // (ahead of the wave's end)
    __builtin_amdgcn_endpgm();
  }
  // between two polls of all words of a wave: from the 32nd on (10 us, which no hand-over takes) the wave leaves gaps of 1 us, for
  // should the polls be what holds up the data (see res_gather)
  __device__ __forceinline__ void again_wide() {
    if (n >= 32) __builtin_amdgcn_s_sleep(32);
    again();
  }
};

// Hand-over stores.  Blocks on one XCD share its L2: a plain store leaves the data there, and a device-coherent load finds it
// there (such a load passes by the L1 but not by the L2: 107 ns, like any other that the L2 answers).  Across XCDs the store has
// to be written through, which takes longer to be seen and to be acknowledged.  (One word from block to block and back, per
// direction: 272 ns on one XCD with plain stores, 375 with written-through ones, 440 between two XCDs.)
template <typename T>
__device__ __forceinline__ void res_store(bool local, T *p, T v) {
  if (local) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  else store_agent(p, v);
}
__device__ __forceinline__ void res_store_pair(bool local, uint64_t *p, int second, uint64_t v0, uint64_t v1) {
  if (local) {
    __hip_atomic_store(p, v0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    __hip_atomic_store(p + second, v1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  } else {
    store_agent(p, v0);
    store_agent(p + second, v1);
  }
}
__device__ __forceinline__ void res_store16(bool local, float *p, floatx4 v) {
  if (local) asm volatile("global_store_dwordx4 %0, %1, off" ::"v"(p), "v"(v) : "memory");
  else store16_through(p, v);
}

// What a step decided for a slot: step tag (16 bits, step + 1) | utterance finished (1) | parent slot in the group (6) | token + 1 (21) | frame (20)
constexpr int kWordMaxFrames = 1 << 20;
__device__ __forceinline__ uint64_t slot_word(int step, int fin, int src, int tok, int t) {
  return (uint64_t)((step + 1) & 0xffff) | (uint64_t)fin << 16 | (uint64_t)src << 17 | (uint64_t)(tok + 1) << 23 |
         (uint64_t)t << 44;
}
__device__ __forceinline__ int word_tag(uint64_t w) { return (int)(w & 0xffff); }
__device__ __forceinline__ int word_finished(uint64_t w) { return (int)(w >> 16) & 1; }
__device__ __forceinline__ int word_src(uint64_t w) { return (int)(w >> 17) & 63; }
__device__ __forceinline__ int word_tok(uint64_t w) { return ((int)(w >> 23) & 0x1fffff) - 1; }
__device__ __forceinline__ int word_frame(uint64_t w) { return (int)(w >> 44); }
__device__ __forceinline__ uint64_t res_load(const char *p) { return load_agent(reinterpret_cast<const uint64_t *>(p)); }
// N 8-byte words of a lane as soon as all are there (in every lane of the wave).  base: the same in all lanes; at(i, o): address of
// word i, base + one of the lane's offsets + a constant; the first n are used (FULL: all N).  (The offsets are made anew for every
// poll: an address kept per word would take more registers than the words.)  Every poll loads all of the words: with a poll of one
// word per tile first, a trip to the L2 lies between the arrival of the data and their use (batch 32 / beam 4 8.09 instead of 7.52 ms
// per decode).
template <bool FULL, int N, int M, class AT>
__device__ __forceinline__ void res_gather(const uint32_t (&offs)[M], AT at, int n, uint64_t (&x)[N]) {
  ResWait w;
  for (;;) {
    uint32_t o[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      o[m] = offs[m];
      asm volatile("" : "+v"(o[m]));
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      x[i] = 0;
      if (FULL || i < n) x[i] = res_load(at(i, o));
    }
    if (__ballot(res_any_empty(x)) == 0ull) return;
    w.again_wide();
  }
}
// Waits for one word of every tile whose owner writes into the words that the wave gathers next (base + the lane's offset: lanes share
// them out).  For waves that gather 20 words a lane (bf16 joint, two tiles of slots): the polls of eight such waves kept a compute unit's
// memory pipeline so busy that its own stores, which others waited for, did not get out (in one build: 280 us per step; with this poll
// first 11).  With 12 words and less no build has shown it; the gaps of again_wide would bound it at some 10 us per hand-over.
__device__ __forceinline__ void res_probe(const char *base, uint32_t offset) {
  ResWait w;
  for (;;) {
    uint32_t o = offset;
    asm volatile("" : "+v"(o));
    const uint64_t y[1] = {res_load(base + o)};
    if (__ballot(res_any_empty(y)) == 0ull) return;
    w.again();
  }
}

// ---- addresses of the hand-over arrays
struct ResAddr {
  float *hb, *pb, *zb;
  uint64_t *words;
  size_t h_ring, p_ring, z_ring, w_ring, h_tile, p_tile;
  int Npad;
  __device__ __forceinline__ float *h(int step, int nt) const { return hb + (step & (kResStepRing - 1)) * h_ring + nt * h_tile; }
  __device__ __forceinline__ float *p(int step, int nt) const { return pb + (step & (kResStepRing - 1)) * p_ring + nt * p_tile; }
  __device__ __forceinline__ float *z(int step, int slot) const { return zb + (step & (kResStepRing - 1)) * z_ring + (size_t)slot * Npad; }
  __device__ __forceinline__ uint64_t *w(int step) const { return words + (step & (kResStepRing - 1)) * w_ring; }
};
__host__ __device__ inline size_t res_h_floats(const ResArgs &a) { return a.emb_tab ? 0 : (size_t)kResStepRing * a.n_groups * a.NT * a.P * kResSlot; }
__host__ __device__ inline size_t res_p_floats(const ResArgs &a) { return a.emb_tab ? 0 : (size_t)kResStepRing * a.n_groups * a.NT * a.H * kResSlot; }
__host__ __device__ inline size_t res_z_floats(const ResArgs &a) { return (size_t)kResStepRing * a.n_groups * a.NT * kResSlot * a.Npad; }
__host__ __device__ inline size_t res_words(const ResArgs &a) { return (size_t)kResStepRing * a.n_groups * kResWordCopies * kResWordPlace; }
template <bool FULL = false>
__device__ __forceinline__ ResAddr res_addr(const ResArgs &a, int g) {
  ResAddr r;
  r.Npad = a.Npad;
  r.h_tile = (size_t)(FULL ? 8 * 8 * kResMaxRounds : a.P) * kResSlot;
  r.p_tile = (size_t)(FULL ? 8 * 8 * kResMaxRounds : a.H) * kResSlot;
  r.h_ring = (size_t)a.n_groups * a.NT * r.h_tile;
  r.p_ring = (size_t)a.n_groups * a.NT * r.p_tile;
  r.z_ring = (size_t)a.n_groups * a.NT * kResSlot * a.Npad;
  r.w_ring = (size_t)a.n_groups * kResWordCopies * kResWordPlace;
  r.hb = a.hb + (size_t)g * a.NT * r.h_tile;
  r.pb = a.pb + (size_t)g * a.NT * r.p_tile;
  r.zb = a.zb + (size_t)g * a.NT * kResSlot * a.Npad;
  r.words = a.words + (size_t)g * kResWordCopies * kResWordPlace;
  return r;
}

// what a wave knows about itself and its block
struct ResBlock {
  int g, nu, nslots;                 // group, utterances and slots of the group
  int place;                         // of the words that this block polls (see kResWordCopies)
  bool local;                        // the group's blocks share one XCD (see res_store)
  int nt;                            // slot tiles up to the last one with an unfinished utterance: the others are left out
  const int16_t *order;              // LDS: the group's utterances (indices in the batch), longest first
  int nR, nJ, nP;
  int wave;
  int fold;                          // the first output-layer tile holds the blank and duration columns, and they are folded (split
                                     // operands: it is one of them, see res_fold_one)
  int ptile, jtile[2];               // the tile of 16 outputs / columns whose sums this wave finishes (-1: none)
  float *red;                        // LDS: partial sums (two halves that alternate, of so many 16-row tiles)
  int red_blocks;
  const uint64_t *spec;              // LDS: see res_fold_bf16
  const uint64_t *tiles;             // LDS: weights of up to kResMaxLdsTiles tiles
  const floatx4 *par;                // LDS: scales and biases of the rows of the block's tiles (see ResPar)
  const int2 *info;                  // LDS: frames of the slot's utterance, its first row of f_proj
  uint64_t *word;                    // LDS: this wave's copy of the last step's words, [slot tile][16]
  int4 *ctx;                         // LDS, stateless decoders: this wave's copy of the slots' last tokens (-1: none)
  float *pre;                        // LDS, stateless decoders: the waves' slices of pre
  int quads_inv;                     // 2^16 over the quads of k of a slice, rounded up (numbers below 320 are divided by up to 20)
  int phase;                         // which half of the partial sums
};
// A lane's place in the wave.  (Computed anew where it is needed rather than kept: the weights leave no registers to
// spare.)  sl: slot of the tile, kq: k-quad, also the group of four rows of a result tile.
struct ResLane {
  int lane, kq, sl;
};
__device__ __forceinline__ ResLane res_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
  return ResLane{l, l >> 4, l & 15};
}
__device__ __forceinline__ int res_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
// index of utterance u of the group in the batch
__device__ __forceinline__ int res_utt(const ResBlock &k, int u) { return k.order[u]; }

// ---- split operands (see split_f16)
// A lane's part of a wave slice of up to 10 rounds of 8 k, for the 16x16x32 instruction (two quads of rounds) and the 16x16x16 one
// (the last two).  A lane (row or slot, kq) has four k of each of two rounds of a quad, half kq % 2 of rounds 2 (kq / 2) and the
// next, resp. half kq / 2 of round 8 + kq % 2: the eight products that an instruction adds up at once are then those of the
// 32x32x16 instructions of the per-step kernels, in the same order.  Absent rounds are zero.
struct ResW16 {
  uintx4_t h[2], l[2];
  uintx2_t th, tl;
};
// Byte offset, relative to the slice's first, of the word of the hand-over arrays' fragment order that is part i (0 to 3) of a lane's
// operand on a quad of rounds, or part i (0, 1) of its operand on two rounds.
constexpr int kResRoundBytes = 4 * kResSlot * 8, kResWordBytes = 2 * kResSlot * 8;  // of a round; from a word to the one of k + 1
__device__ __forceinline__ uint32_t res_quad_base(const ResLane &l) { return (l.kq >> 1) * 2 * kResRoundBytes + ((l.kq & 1) * kResSlot + l.sl) * 8; }
__device__ __forceinline__ uint32_t res_pair_base(const ResLane &l) { return (l.kq & 1) * kResRoundBytes + ((l.kq >> 1) * kResSlot + l.sl) * 8; }
// Hidden states come split already (a cell's lane does it once, where each reader did it for all of its slice: 100 instructions of each
// wave in the chain h -> pre, and as many under the selection).  A word there holds the hi, or the lo, of the four k of a half of a round,
// {0, 2, 1, 3}: of a round hi of the halves, then lo, so that the words of a quad are the lane's operand as they come.
template <bool SPLIT>
__device__ __forceinline__ constexpr uint32_t res_part(int i) {
  return SPLIT ? (i & 1) * kResRoundBytes + (i >> 1) * kResWordBytes : (i >> 1) * kResRoundBytes + (i & 1) * kResWordBytes;
}
// part i (0 to 9) of ten rounds; pair: that of round 8
template <bool SPLIT>
__device__ __forceinline__ constexpr uint32_t res_split_part(int i) {
  return i < 8 ? (i >> 2) * 4 * kResRoundBytes + res_part<SPLIT>(i & 3) : (i & 1) * kResWordBytes;
}
// a slice of nr rounds, as soon as all of it is there
template <bool FULL, bool SPLIT>
__device__ __forceinline__ void res_split_gather(const ResLane &l, const char *src, int nr, uint64_t (&x)[kResMaxRounds]) {
  // (absent rounds read the slice's first and are cleared)
  const uint32_t offs[2] = {res_quad_base(l), res_pair_base(l) + 8 * kResRoundBytes}, end = nr * kResRoundBytes;
  auto at = [&](int i, const uint32_t (&o)[2]) {
    if constexpr (FULL) return src + o[i < 8 ? 0 : 1] + res_split_part<SPLIT>(i);
    const uint32_t w = o[i < 8 ? 0 : 1] + res_split_part<SPLIT>(i);
    return src + (w < end ? w : l.sl * 8);
  };
  res_gather<true, kResMaxRounds>(offs, at, kResMaxRounds, x);
  if constexpr (!FULL) {
#pragma unroll
    for (int i = 0; i < kResMaxRounds; ++i)
      if (offs[i < 8 ? 0 : 1] + res_split_part<SPLIT>(i) >= end) x[i] = 0;
  }
}
// words of a lane -> operand
__device__ __forceinline__ void res_split_act(const uint64_t (&x)[kResMaxRounds], float scale, ResW16 &o) {
  uint32_t h[kResMaxRounds], l[kResMaxRounds];
#pragma unroll
  for (int i = 0; i < kResMaxRounds; ++i) split_f16(lo_f(x[i]) * scale, hi_f(x[i]) * scale, h[i], l[i]);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    o.h[g] = uintx4_t{h[4 * g], h[4 * g + 1], h[4 * g + 2], h[4 * g + 3]};
    o.l[g] = uintx4_t{l[4 * g], l[4 * g + 1], l[4 * g + 2], l[4 * g + 3]};
  }
  o.th = uintx2_t{h[8], h[9]};
  o.tl = uintx2_t{l[8], l[9]};
}
// words that are split already -> operand
__device__ __forceinline__ uintx4_t res_quad(uint64_t a, uint64_t b) { return uintx4_t{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)}; }
__device__ __forceinline__ uintx2_t res_pair(uint64_t a) { return uintx2_t{(uint32_t)a, (uint32_t)(a >> 32)}; }
__device__ __forceinline__ ResW16 res_split_words(const uint64_t (&x)[kResMaxRounds]) {
  return ResW16{{res_quad(x[0], x[1]), res_quad(x[4], x[5])}, {res_quad(x[2], x[3]), res_quad(x[6], x[7])}, res_pair(x[8]), res_pair(x[9])};
}
// a lane's part of a split tile, p: the wave's
__device__ __forceinline__ ResW16 res_split_load(const uintx4_t *p, const ResLane &l) {
  const uintx4_t v = p[4 * 64 + l.lane];
  return ResW16{{p[l.lane], p[2 * 64 + l.lane]}, {p[64 + l.lane], p[3 * 64 + l.lane]}, uintx2_t{v[0], v[1]}, uintx2_t{v[2], v[3]}};
}
// the 20 words as they lie in a tile that is not split (res_fold_mma's)
__device__ __forceinline__ float res_raw(const ResW16 &w, int i) {
  return __uint_as_float(i < 16 ? ((i >> 2) & 1 ? w.l[i >> 3][i & 3] : w.h[i >> 3][i & 3]) : i < 18 ? w.th[i & 1] : w.tl[i & 1]);
}
// Between 16x16x32 instructions and 16x16x16 ones on the same accumulators.  Instructions of one shape hand their sums on inside the
// matrix unit, back to back; from one shape to the other the second missed addends of the first here (the compiler puts no wait states
// between the two).  In the vector registers, where every instruction finds it, a result of either shape is 8 wait states behind its
// instruction (the compiler's distance to any other reader, s_nop 7); these are 16, behind the last instruction on any of the
// accumulators, since all of them pass through the asm.
__device__ __forceinline__ void res_mma_gap(floatx4 (&a)[1], floatx4 (&b)[1]) { asm volatile("s_nop 15" : "+v"(a[0]), "+v"(b[0])); }
__device__ __forceinline__ void res_mma_gap(floatx4 (&a)[2], floatx4 (&b)[2]) {
  asm volatile("s_nop 15" : "+v"(a[0]), "+v"(b[0]), "+v"(a[1]), "+v"(b[1]));
}
__device__ __forceinline__ void res_mma_gap(floatx4 (&a)[3], floatx4 (&b)[3]) {
  asm volatile("s_nop 15" : "+v"(a[0]), "+v"(b[0]), "+v"(a[1]), "+v"(b[1]), "+v"(a[2]), "+v"(b[2]));
}
// N tiles of 16 rows, from w[T0] on.  n_rounds: of the slice (beyond: zeros).  Not FULL: kSplitLoLo
template <bool FULL, int T0, int N, int M>
__device__ __forceinline__ void res_split_mma(const ResW16 (&w)[M], const ResW16 &x, int n_rounds, floatx4 (&acc)[N], floatx4 (&cor)[N]) {
#pragma unroll
  for (int t = 0; t < N; ++t) acc[t] = cor[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < 2; ++g)
    if (FULL || 4 * g < n_rounds) {
#pragma unroll
      for (int t = 0; t < N; ++t) {
        acc[t] = mfma16_f16(w[T0 + t].h[g], x.h[g], acc[t]);
        cor[t] = mfma16_f16(w[T0 + t].h[g], x.l[g], cor[t]);
      }
#pragma unroll
      for (int t = 0; t < N; ++t) cor[t] = mfma16_f16(w[T0 + t].l[g], x.h[g], cor[t]);
      if constexpr (!FULL) {
        const uintx4_t xl = unscaled_lo(x.l[g]);
#pragma unroll
        for (int t = 0; t < N; ++t) cor[t] = mfma16_f16(w[T0 + t].l[g], xl, cor[t]);
      }
    }
  if (FULL || n_rounds > 8) {
    res_mma_gap(acc, cor);
#pragma unroll
    for (int t = 0; t < N; ++t) {
      acc[t] = mfma16_f16(w[T0 + t].th, x.th, acc[t]);
      cor[t] = mfma16_f16(w[T0 + t].th, x.tl, cor[t]);
    }
#pragma unroll
    for (int t = 0; t < N; ++t) cor[t] = mfma16_f16(w[T0 + t].tl, x.th, cor[t]);
    if constexpr (!FULL) {
      const uintx2_t xl = unscaled_lo(x.tl);
#pragma unroll
      for (int t = 0; t < N; ++t) cor[t] = mfma16_f16(w[T0 + t].tl, xl, cor[t]);
    }
  }
}

// Places in ResBlock::par: of each tile four floats per group of four rows, as the lanes that finish it hold them.
struct ResPar {
  static constexpr int kScale = 0, kBias = 4;                     // of a projection or output-layer tile
  static constexpr int kP = 0, kJ = 8 * kResMaxP, kR = kJ + 8 * 4;  // first of the projection's, the output layer's, W_hh's (no bias)
  static constexpr int kFloats = 4 * (kR + 4 * kResMaxR);
};
// partial sums of a 16-row tile: wave's lane (row group, slot) holds four rows
template <bool BF16>
__device__ __forceinline__ float *res_red(const ResBlock &k, int block) {
  return k.red + ((k.phase & 1) * k.red_blocks + block) * kResRedBlock;
}
template <bool BF16>
__device__ __forceinline__ void res_put(const ResBlock &k, const ResLane &l, int block, floatx4 v) {
  *reinterpret_cast<floatx4 *>(res_red<BF16>(k, block) + (k.wave * 64 + l.lane) * 4) = v;
}
template <bool BF16>
__device__ __forceinline__ floatx4 res_sum(const ResBlock &k, const ResLane &l, int block) {
  const float *r = res_red<BF16>(k, block) + l.lane * 4;
  floatx4 v[kResWaves];
#pragma unroll
  for (int w = 0; w < kResWaves; ++w) v[w] = *reinterpret_cast<const floatx4 *>(r + w * 256);
  floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kResWaves; ++w) s += v[w];
  return s;
}

// Waits for the words of step `step` and leaves them in the wave's LDS copy; slots beyond the group's are idle (finished).
// 1: every utterance of the group has finished, 0: not yet.
__device__ __forceinline__ int res_words(ResBlock &k, int step) {
  const ResArgs &a = res_args();
  const ResLane l = res_lane();
  const uint64_t *p = res_addr(a, k.g).w(step) + k.place + l.sl;
  const int tag = (step + 1) & 0xffff;
  int top = 0;
#pragma unroll 1
  for (int nt = 0; nt < a.NT; ++nt) {
    const int slot = nt * kResSlot + l.sl;
    uint64_t w = slot_word(step, 1, slot, -1, 0);
    ResWait wait;
    for (;;) {
      bool missing = false;
      if (slot < k.nslots) {
        w = load_agent(p + nt * kResSlot);
        missing = word_tag(w) != tag;
      }
      if (__ballot(missing) == 0ull) break;
      wait.again();
    }
    if (__ballot(!word_finished(w))) top = nt + 1;
    if (l.kq == 0) k.word[slot] = w;
  }
  wave_sync();
  k.nt = top;
  return top == 0 ? 1 : 0;
}
// before the first step: hypothesis 0 of every utterance reads the start symbol
__device__ __forceinline__ int res_first_words(const ResArgs &a, ResBlock &k) {
  const ResLane l = res_lane();
  int top = 0;
  for (int nt = 0; nt < a.NT; ++nt) {
    const int slot = nt * kResSlot + l.sl;
    const bool used = slot < k.nslots;
    const bool empty = !used || a.lengths[res_utt(k, used ? slot / a.K : 0)] == 0;
    if (__ballot(!empty)) top = nt + 1;
    if (l.kq == 0) k.word[slot] = slot_word(-1, empty ? 1 : 0, slot, (used && slot % a.K == 0) ? a.V : -1, 0);
  }
  wave_sync();
  k.nt = top;
  return top == 0 ? 1 : 0;
}

// ---- P: pre[step] = f_proj[frame] + W_pred h[step] + b_pred for the block's tiles of 16 outputs
// output row i of tile t: o = 16 t + 8 (i / 8) + (i / 4) % 2 + 2 (i % 4), so that a lane's four rows are two 8-byte words
// of the fragment order.
__host__ __device__ inline int res_p_row(int tile, int i) { return 16 * tile + 8 * (i >> 3) + ((i >> 2) & 1) + 2 * (i & 3); }
__device__ __forceinline__ float *res_p_dst(float *p, int tile, int g, int sl) {  // two words, 32 floats apart
  return p + ((size_t)((2 * tile + (g >> 1)) * 4 + 2 * (g & 1)) * kResSlot + sl) * 2;
}
// every second one of eight floats, from the first or the second on: the four rows of a lane
__device__ __forceinline__ floatx4 res_p_pick(const ResLane &l, const float *p) {
  const floatx4 f0 = *reinterpret_cast<const floatx4 *>(p), f1 = *reinterpret_cast<const floatx4 *>(p + 4);
  return (l.kq & 1) ? floatx4{f0[1], f0[3], f1[1], f1[3]} : floatx4{f0[0], f0[2], f1[0], f1[2]};
}
// The frame's projection of the four outputs that the wave finishes: requested before the activations are waited for.
__device__ __forceinline__ floatx4 res_p_frame(const ResArgs &a, const ResBlock &k, const ResLane &l, int nt) {
  const int2 in = k.info[nt * kResSlot + l.sl];
  int tt = word_frame(k.word[nt * kResSlot + l.sl]);
  tt = tt < in.x ? tt : in.x - 1;
  tt = tt < 0 ? 0 : tt;
  return res_p_pick(l, a.f_proj + ((size_t)in.y + tt) * a.H + 16 * k.ptile + 8 * (l.kq >> 1));
}
// sums of the wave's tile -> pre.  first / second: the blocks of its partial sums of the two halves of k (halves: the
// per-step launches add the bias and the frame's projection to the first half's sum, then the second half's).
template <int FORM>
__device__ __forceinline__ void res_p_finish(const ResArgs &a, const ResBlock &k, const ResLane &l, const ResAddr &ad, int step, int nt, int first,
                                             int second, floatx4 f) {
  const floatx4 *par = k.par + ResPar::kP + 8 * (kResWaves - 1 - k.wave) + l.kq;
  floatx4 v = res_sum<FORM == kResBf16>(k, l, first);
  if constexpr (FORM == kResSplit) v *= par[ResPar::kScale];
  v = (v + par[ResPar::kBias]) + f;
  if (a.halves) {
    floatx4 s = res_sum<FORM == kResBf16>(k, l, second);
    if constexpr (FORM == kResSplit) s *= par[ResPar::kScale];
    v += s;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);  // (once here, not by every reader; not a number: 0)
  float *dst = res_p_dst(ad.p(step, nt), k.ptile, l.kq, l.sl);
  asm volatile("" : "+v"(v));  // (all four before either store: else both sums' operands live on behind the first)
  wait_stores_acknowledged();  // (of the pattern that this wave put back into places of the array meanwhile)
  res_store_pair(k.local, reinterpret_cast<uint64_t *>(dst), kResSlot, pack2(v[0], v[1]), pack2(v[2], v[3]));
}
__device__ __forceinline__ void clear_p(const ResBlock &k, const ResLane &l, const ResAddr &ad, int step, int nt) {
  float *dst = res_p_dst(ad.p(step, nt), k.ptile, l.kq, l.sl);
  res_store_pair(k.local, reinterpret_cast<uint64_t *>(dst), kResSlot, ~0ull, ~0ull);
}
// the wave that finishes a tile of the projection: from the last one down, which own no cells
__device__ __forceinline__ int res_p_wave(int tile_no) { return kResWaves - 1 - tile_no; }

// A round of activations (lane: slot column, half of k) rounded to bf16, the four k in order
__device__ __forceinline__ uint64_t round_bf16(const uint64_t *x) {
  return (uint64_t)pack_bf16_rne(hi_f(x[0]), hi_f(x[1])) << 32 | pack_bf16_rne(lo_f(x[0]), lo_f(x[1]));
}
// bf16 matrix instruction (32 x 32 x 16) on two rounds
__device__ __forceinline__ floatx16 mfma_pair_bf16(uint64_t w0, uint64_t w1, uint64_t x0, uint64_t x1, bool two, floatx16 acc) {
  const uintx4_t w = {(uint32_t)w0, (uint32_t)(w0 >> 32), two ? (uint32_t)w1 : 0u, two ? (uint32_t)(w1 >> 32) : 0u};
  const uintx4_t b = {(uint32_t)x0, (uint32_t)(x0 >> 32), two ? (uint32_t)x1 : 0u, two ? (uint32_t)(x1 >> 32) : 0u};
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, b), acc, 0, 0, 0);
}
// Lane (column c, half): the two words of a round, quads half and half + 2; columns 16..31 are the next slot tile (or a repeat).
// Offset from the slice's first word; rounds follow in even strides of kResWordBytes.
__device__ __forceinline__ uint32_t bf16_src(const ResLane &l, size_t tile_floats, bool second) {
  const int half = l.lane >> 5, c = l.lane & 31;
  return ((c >> 4) && second ? (uint32_t)tile_floats * 4 : 0u) + (half * kResSlot + (c & 15)) * 8;
}
// Ten rounds of a lane's words: five from first on, five from then on (offsets of the slice's rounds from src; the first n of either
// are there, the others repeat the first).  With one tile of slots the lanes of the columns beyond it read the words of k + 1 for
// the others, which halves the loads.
template <bool FULL>
__device__ __forceinline__ void bf16_gather(const ResLane &l, const char *src, uint32_t first, uint32_t then, int n_first, int n_then, bool second, size_t tile_floats,
                                            uint32_t probe, uint64_t (&x)[2 * kResMaxRounds]) {
  constexpr int R = kResMaxRounds / 2;
  const uint32_t lane0 = bf16_src(l, tile_floats, second);
  if (second) {
    const uint32_t offs[2] = {lane0 + first, lane0 + then};
    res_probe(src, probe);
    res_gather<true, 2 * kResMaxRounds>(offs, [&](int i, const uint32_t (&o)[2]) {
      const int r = i / 2 % R;
      return src + o[i / kResMaxRounds] + (FULL || r < (i < kResMaxRounds ? n_first : n_then) ? r * kResRoundBytes : 0) + (i & 1) * kResWordBytes;
    }, 0, x);
  } else {
    const uint32_t odd = (l.lane & 16) ? kResWordBytes : 0;
    const uint32_t offs[2] = {lane0 + first + odd, lane0 + then + odd};
    uint64_t y[kResMaxRounds];
    res_gather<true, kResMaxRounds>(offs, [&](int i, const uint32_t (&o)[2]) {
      const int r = i % R;
      return src + o[i / R] + (FULL || r < (i < R ? n_first : n_then) ? r * kResRoundBytes : 0);
    }, 0, y);
#pragma unroll
    for (int i = 0; i < kResMaxRounds; ++i) {
      const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)y[i], (uint32_t)y[i], false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(y[i] >> 32), (uint32_t)(y[i] >> 32), false, false);
      x[2 * i] = (uint64_t)(uint32_t)hi[0] << 32 | (uint32_t)lo[0];
      x[2 * i + 1] = (uint64_t)(uint32_t)hi[1] << 32 | (uint32_t)lo[1];
    }
  }
}
// Words to probe: a tile of W_hh's four units writes half of a round's words (two per round), a tile of the projection two rounds'
// (one per round).  Of the second slot tile: lanes from 32 on.
__device__ __forceinline__ uint32_t bf16_probe_tile(const ResLane &l, size_t tile_floats, bool second) {
  return (l.lane >> 5) && second ? (uint32_t)tile_floats * 4 : 0u;
}
// 32-row tile's accumulators -> partial sums of its two 16-row tiles (blocks b0, b0 + 1) for columns 16 nt2 .. + 15
__device__ __forceinline__ void bf16_put(const ResBlock &k, const ResLane &l, int b0, int nt2, const floatx16 &acc) {
  const int half = l.lane >> 5, c = l.lane & 31;
  if ((c >> 4) == nt2) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int g = (q & 1) * 2 + half;
      *reinterpret_cast<floatx4 *>(res_red<true>(k, b0 + (q >> 1)) + (k.wave * 64 + g * 16 + (c & 15)) * 4) =
          floatx4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    }
  }
}

template <bool FULL, int FORM>
__device__ __forceinline__ void res_p_phase(ResBlock &k, int step) {
  if (k.nP == 0) return;
  const ResArgs &a = res_args();
  const ResLane l = res_lane();
  const ResAddr ad = res_addr(a, k.g);
  const int nr = FULL ? kResMaxRounds : a.rounds_p;
  const bool halves = a.halves != 0;
  const int nh = halves ? nr / 2 : nr;  // rounds of a slice: the wave has one in either half of k, or one of the whole
  if constexpr (FORM == kResBf16) {  // one tile of 32 outputs: two waves finish 16 each
#pragma unroll 1
    for (int nt = 0; nt < k.nt; nt += 2) {
      const bool second = nt + 1 < k.nt;
      floatx4 f[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
      if (k.ptile >= 0) {
        f[0] = res_p_frame(a, k, l, nt);
        if (second) f[1] = res_p_frame(a, k, l, nt + 1);
      }
      const uint64_t *w = k.tiles + l.lane;
      if (second) __syncthreads();  // (both halves of the buffer are written below; one of them has just been read)
      // words of five rounds of the first half's slice, then of the second's (or of ten of the one slice); absent ones repeat the first
      const int ra = k.wave * nh, rb = halves ? 4 * nr + ra : nr > 5 ? ra + 5 : ra;
      uint64_t x[2 * kResMaxRounds];
      {
        const int pr = (l.lane & 31) < 2 * nr ? (l.lane & 31) >> 1 : 0;
        const uint32_t probe = bf16_probe_tile(l, ad.h_tile, second) + (!halves || pr < nh ? ra + pr : rb + pr - nh) * kResRoundBytes + (l.lane & 1) * kResWordBytes;
        bf16_gather<FULL>(l, reinterpret_cast<const char *>(ad.h(step, nt)), ra * kResRoundBytes, rb * kResRoundBytes, halves ? nh : min(nr, 5),
                          halves ? nh : max(nr - 5, 0), second, ad.h_tile, probe, x);
      }
      auto put = [&](int hf, const floatx16 &acc) {
        bf16_put(k, l, 2 * hf, 0, acc);
        if (second) {  // the other slot tile's sums go to the other half of the buffer
          ++k.phase;
          bf16_put(k, l, 2 * hf, 1, acc);
          --k.phase;
        }
      };
      if (halves) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const uint64_t *wh = w + (hf ? rb : ra) * 64;
          floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
          for (int i = 0; i < 3; ++i)
            if (2 * i < nh) {
              const bool two = i < 2 && 2 * i + 1 < nh;
              const uint64_t *xi = x + kResMaxRounds * hf + 4 * i;
              acc = mfma_pair_bf16(wh[2 * i * 64], wh[(2 * i + (two ? 1 : 0)) * 64], round_bf16(xi), round_bf16(i < 2 ? xi + 2 : xi), two, acc);
            }
          put(hf, acc);
        }
      } else {
        floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < kResMaxRounds / 2; ++i)
          if (2 * i < nr) {
            const bool two = 2 * i + 1 < nr;
            acc = mfma_pair_bf16(w[(ra + 2 * i) * 64], w[(ra + 2 * i + (two ? 1 : 0)) * 64], round_bf16(x + 4 * i),
                                 round_bf16(x + 4 * i + 2), two, acc);
          }
        put(0, acc);
      }
      __syncthreads();
      res_end_if_given_up();
      if (k.ptile >= 0) res_p_finish<kResBf16>(a, k, l, ad, step, nt, k.ptile & 1, 2 + (k.ptile & 1), f[0]);
      ++k.phase;
      if (second) {
        if (k.ptile >= 0) res_p_finish<kResBf16>(a, k, l, ad, step, nt + 1, k.ptile & 1, 2 + (k.ptile & 1), f[1]);
        ++k.phase;
        __syncthreads();  // (both halves of the buffer have just been read)
      }
    }
  } else {
#pragma unroll 1
    for (int nt = 0; nt < k.nt; ++nt) {
      floatx4 f = {0.f, 0.f, 0.f, 0.f};
      if (k.ptile >= 0) f = res_p_frame(a, k, l, nt);
      const char *src = reinterpret_cast<const char *>(ad.h(step, nt)) + k.wave * nh * kResRoundBytes;
      [[maybe_unused]] const uintx4_t *tiles = reinterpret_cast<const uintx4_t *>(k.tiles) + (size_t)k.wave * kResQuads * 64;
      // what the wave finishes of tile tp (a copy per tile: their blocks of partial sums alternate)
      auto finish = [&](int tp) {
        __syncthreads();
        res_end_if_given_up();
        if (k.wave == res_p_wave(tp)) res_p_finish<FORM>(a, k, l, ad, step, nt, 0, 1, f);
        ++k.phase;
      };
      if constexpr (FORM == kResF32) {
        uint64_t x[kResMaxRounds];
        // rounds i < nr / 2 from the wave's slice of the first half of k, the others from its slice of the second half (or
        // all of one slice)
        constexpr int R = kResMaxRounds / 2;
        const int n1 = FULL ? R : nr / 2, jump = halves ? 4 * nr - n1 : 0;
        const uint32_t offs[2] = {(uint32_t)l.lane * 8, (uint32_t)l.lane * 8 + (R + jump) * kResRoundBytes};
        auto at = [&](int i, const uint32_t (&o)[2]) {
          if constexpr (FULL) return src + o[i / R] + i % R * kResRoundBytes;
          return src + o[0] + (i + (i >= n1 ? jump : 0)) * kResRoundBytes;
        };
        res_gather<FULL, kResMaxRounds>(offs, at, nr, x);
#pragma unroll 1
        for (int tp = 0; tp < k.nP; ++tp) {
          const uint64_t *w = k.tiles + (size_t)tp * (a.P * kResSlot / 2) + (size_t)k.wave * nh * 64 + l.lane;
          if (halves) {
            floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll
            for (int i = 0; i < R; ++i)
              if (FULL || i < n1) {
                const uint64_t u = w[i * 64], v = w[(4 * nr + i) * 64], y = FULL ? x[R + i] : res_pick(x, n1 + i);
                acc0 = mfma16(lo_f(u), lo_f(x[i]), acc0);
                acc1 = mfma16(lo_f(v), lo_f(y), acc1);
                acc0 = mfma16(hi_f(u), hi_f(x[i]), acc0);
                acc1 = mfma16(hi_f(v), hi_f(y), acc1);
              }
            res_put<false>(k, l, 0, acc0);
            res_put<false>(k, l, 1, acc1);
          } else {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < kResMaxRounds; ++i)
              if (FULL || i < nr) {
                const uint64_t u = w[i * 64];
                acc = mfma16(lo_f(u), lo_f(x[i]), acc);
                acc = mfma16(hi_f(u), hi_f(x[i]), acc);
              }
            res_put<false>(k, l, 0, acc);
          }
          finish(tp);
        }
      } else {
        // One pass over all tiles, one barrier, where their partial sums find room; else a pass per tile
        const bool together = k.nP == 1 || !halves || k.red_blocks >= 4;
        auto all_tiles = [&](auto tile_mma) {
          if (together) {
#pragma unroll
            for (int tp = 0; tp < kResMaxP; ++tp)
              if (tp < k.nP) tile_mma(tp, halves ? 2 * tp : tp);
            __syncthreads();
            res_end_if_given_up();
            const int mine = kResWaves - 1 - k.wave, first = halves ? 2 * mine : mine;
            if (k.ptile >= 0) {
              __builtin_amdgcn_s_setprio(2);
              res_p_finish<FORM>(a, k, l, ad, step, nt, first, first + 1, f);
              __builtin_amdgcn_s_setprio(0);
            }
            ++k.phase;
          } else {
#pragma unroll 1
            for (int tp = 0; tp < k.nP; ++tp) {
              tile_mma(tp, 0);
              finish(tp);
            }
          }
        };
        if (halves) {
          // a slice of up to five rounds of either half of k: a quad, and a fifth round that the lanes of even kq hold
          uint64_t x[12];
          // (absent rounds: words that are there, cleared below)
          const uint32_t end = nh * kResRoundBytes, second = 4 * nr * kResRoundBytes;
          const uint32_t quad = res_quad_base(l), fifth = (FULL || nh > 4) && (l.kq & 1) == 0 ? 4 * kResRoundBytes + res_pair_base(l) : l.sl * 8;
          const uint32_t offs[4] = {quad, fifth, quad + second, fifth + second};
          auto at = [&](int i, const uint32_t (&o)[4]) {
            const int p = i % 6, hf = i / 6;
            const uint32_t part = p < 4 ? res_part<true>(p) : (p & 1) * kResWordBytes;
            if constexpr (FULL) return src + o[2 * hf + (p >= 4)] + part;
            const uint32_t w = o[2 * hf] + part;
            return src + (p >= 4 ? o[2 * hf + 1] + part : w < end + hf * second ? w : l.sl * 8 + hf * second);
          };
          res_gather<true, 12>(offs, at, 12, x);
#pragma unroll
          for (int i = 0; i < 12; ++i) {
            const int p = i % 6;
            const bool in = p < 4 ? FULL || quad + res_part<true>(p) < end : (FULL || nh > 4) && (l.kq & 1) == 0;
            x[i] = in ? x[i] : 0;
          }
          all_tiles([&](int tp, int block) {
            const uintx4_t *w = tiles + (size_t)tp * (kResTileFloats / 4);
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
              const uintx4_t xh = res_quad(x[6 * hf], x[6 * hf + 1]), xl = res_quad(x[6 * hf + 2], x[6 * hf + 3]);
              const uintx4_t wh = w[160 * hf + l.lane], wl = w[160 * hf + 64 + l.lane];
              floatx4 acc[1] = {floatx4{0.f, 0.f, 0.f, 0.f}}, cor[1] = {acc[0]};
              acc[0] = mfma16_f16(wh, xh, acc[0]);
              cor[0] = mfma16_f16(wh, xl, cor[0]);
              cor[0] = mfma16_f16(wl, xh, cor[0]);
              if constexpr (!FULL) cor[0] = mfma16_f16(wl, unscaled_lo(xl), cor[0]);
              if (FULL || nh > 4) {
                const uintx2_t yh = res_pair(x[6 * hf + 4]), yl = res_pair(x[6 * hf + 5]);
                const uintx4_t v = w[160 * hf + 128 + (l.kq >> 1) * 16 + l.sl];  // (the lanes of odd kq: against zeros)
                const uintx2_t vh = {v[0], v[1]}, vl = {v[2], v[3]};
                res_mma_gap(acc, cor);
                acc[0] = mfma16_f16(vh, yh, acc[0]);
                cor[0] = mfma16_f16(vh, yl, cor[0]);
                cor[0] = mfma16_f16(vl, yh, cor[0]);
                if constexpr (!FULL) cor[0] = mfma16_f16(vl, unscaled_lo(yl), cor[0]);
              }
              res_put<false>(k, l, block + hf, split_join(acc[0], cor[0]));
            }
          });
        } else {
          ResW16 xs;
          {
            uint64_t x[kResMaxRounds];
            res_split_gather<FULL, true>(l, src, nr, x);
            xs = res_split_words(x);
          }
          all_tiles([&](int tp, int block) {
            const ResW16 w[1] = {res_split_load(tiles + (size_t)tp * (kResTileFloats / 4), l)};
            floatx4 acc[1], cor[1];
            res_split_mma<FULL, 0, 1>(w, xs, nr, acc, cor);
            res_put<false>(k, l, block, split_join(acc[0], cor[0]));
          });
        }
      }
    }
  }
}

// ---- J: z[step] = W_out ReLU(pre[step]) + b_out for the block's tiles
// Folded columns of split operands are dealt one by one, as "tiles" from V / 16 on: the column of such a one
__device__ __forceinline__ int res_column(int tile) {
  const int V = res_args().V;
  return V + tile - V / 16;
}
template <int FORM>
__device__ __forceinline__ void res_j_finish(const ResBlock &k, const ResLane &l, const ResAddr &ad, int step, int nt, int tile, int par, int block) {
  const int slot = nt * kResSlot + l.sl, n0 = 16 * tile + 4 * l.kq;
  if (FORM == kResSplit && k.fold && k.wave == 0) {  // (a column alone: see res_fold_one)
    const float *r = res_red<false>(k, block) + l.sl * 4;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kResWaves; ++w) v += r[w * 256];
    v += reinterpret_cast<const float *>(k.par + par + ResPar::kBias)[0];
    wait_stores_acknowledged();
    if (slot < k.nslots && l.kq == 0) res_store(k.local, ad.z(step, slot) + res_column(tile), v);
    return;
  }
  floatx4 v = res_sum<FORM == kResBf16>(k, l, block);
  if constexpr (FORM == kResSplit) v *= k.par[par + ResPar::kScale + l.kq];
  v += k.par[par + ResPar::kBias + l.kq];
  wait_stores_acknowledged();
  if (slot < k.nslots) res_store16(k.local, ad.z(step, slot) + n0, v);
}
template <int FORM>
__device__ __forceinline__ void clear_z(const ResBlock &k, const ResLane &l, const ResAddr &ad, int step, int nt, int tile) {
  const int slot = nt * kResSlot + l.sl;
  const float e = __uint_as_float(kResEmpty);
  if (FORM == kResSplit && k.fold && k.wave == 0) {
    if (slot < k.nslots && l.kq == 0) res_store(k.local, ad.z(step, slot) + res_column(tile), e);
    return;
  }
  if (slot < k.nslots) res_store16(k.local, ad.z(step, slot) + 16 * tile + 4 * l.kq, floatx4{e, e, e, e});
}

// Stateless decoders: the wave's slice of pre of the group's slots, summed up in the order of k_stateless_pre, and from LDS a lane's words of
// it as res_gather / bf16_gather would have read them.  All rows of a pair of tables are requested before the first is needed: the
// time is that of one trip to the L2 (each block of a group reads all of the group's rows, at most 16 x (1 + n_ctx) x 2.5 KB; a
// hand-over of sums formed once would cost a hop more, and the same trip before it).  A lane takes four k of a slot, consecutive lanes
// consecutive ones, and the operands are read from LDS: each lane loading what its operands are made of, 30 times 16 bytes, most of it what
// other lanes, or lanes without a slot, load as well, was bound by the 64 bytes a cycle that a compute unit's L1 hands over (1.6 to 2.3 us;
// batch 8, beam 4, bf16 joint: 2.94 -> 2.62 ms per decode).
// SPLIT (float32 models): a lane's places of split operands (see ResW16), else those of res_k_of.  BF16: ReLU and rounding are done.
constexpr int kResPreSlot = 8 * kResMaxRounds + 4;  // floats of a slot in LDS (bf16: half of them)
template <bool FULL, bool BF16, bool SPLIT>
__device__ __forceinline__ void res_stateless_pre(const ResArgs &a, const ResBlock &k, const ResLane &l, int nr, uint64_t (&x)[kResMaxRounds]) {
  constexpr int N = kResSlot * 2 * kResMaxRounds / 64;  // quads of k of a lane
  const int quads = FULL ? 2 * kResMaxRounds : 2 * nr, total = k.nslots * quads;
  float4 v[N];
  const float *f[N];
  int4 c[N];
  int at[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int q = l.lane + 64 * i < total ? l.lane + 64 * i : 0, slot = FULL ? q / quads : q * k.quads_inv >> 16, quad = q - slot * quads;
    const int2 in = k.info[slot];
    c[i] = k.ctx[slot];
    int tt = word_frame(k.word[slot]);
    tt = tt < in.x ? tt : in.x - 1;
    tt = tt < 0 ? 0 : tt;
    at[i] = slot * kResPreSlot + 4 * quad;
    f[i] = a.f_proj + ((size_t)in.y + tt) * a.H + 8 * k.wave * nr + 4 * quad;
    v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (64 * i < total) v[i] = *reinterpret_cast<const float4 *>(f[i]);
  }
#pragma unroll 1
  for (int j = 0; j < a.n_ctx; j += 2) {
    const int j1 = j + 1 < a.n_ctx ? j + 1 : j;
    float4 d0[N], d1[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int col = 8 * k.wave * nr + (at[i] % kResPreSlot), t0 = j == 0 ? c[i].x : c[i].z, t1 = j1 == j ? t0 : j == 0 ? c[i].y : c[i].w;
      d0[i] = d1[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (64 * i < total) {
        d0[i] = *reinterpret_cast<const float4 *>(a.emb_tab + ((size_t)j * (a.V + 1) + (t0 < 0 ? a.V : t0)) * a.H + col);
        d1[i] = *reinterpret_cast<const float4 *>(a.emb_tab + ((size_t)j1 * (a.V + 1) + (t1 < 0 ? a.V : t1)) * a.H + col);
      }
    }
    auto add = [&](const float4 (&d)[N]) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        v[i].x += d[i].x; v[i].y += d[i].y; v[i].z += d[i].z; v[i].w += d[i].w;
      }
    };
    add(d0);
    if (j1 > j) add(d1);
  }
  float *mine = k.pre + k.wave * kResSlot * kResPreSlot / (BF16 ? 2 : 1);
  wave_sync();
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (l.lane + 64 * i < total) {
      if constexpr (BF16) {
        *reinterpret_cast<uint64_t *>(mine + at[i] / 2) = (uint64_t)pack_bf16_rne(fmaxf(v[i].z, 0.f), fmaxf(v[i].w, 0.f)) << 32 |
                                                          pack_bf16_rne(fmaxf(v[i].x, 0.f), fmaxf(v[i].y, 0.f));
      } else {
        *reinterpret_cast<float4 *>(mine + at[i]) = v[i];
      }
    }
  wave_sync();
  const int slot = l.sl < k.nslots ? l.sl : 0;  // (places without a slot repeat the first one)
  if constexpr (BF16) {
    const uint64_t *r = reinterpret_cast<const uint64_t *>(mine) + slot * (kResPreSlot / 4) + (l.lane >> 5);
#pragma unroll
    for (int i = 0; i < kResMaxRounds; ++i) x[i] = FULL || i < nr ? r[2 * i] : 0;
  } else if constexpr (SPLIT) {
    // (four k of two rounds of either quad, then of the last two rounds)
#pragma unroll
    for (int i = 0; i < kResMaxRounds / 2; ++i) {
      const int round = i < 4 ? 4 * (i >> 1) + 2 * (l.kq >> 1) + (i & 1) : 8 + (l.kq & 1), half = i < 4 ? l.kq & 1 : l.kq >> 1;
      const bool in = FULL || round < nr;
      const float4 d = *reinterpret_cast<const float4 *>(mine + slot * kResPreSlot + 4 * (in ? 2 * round + half : 0));
      x[2 * i] = in ? pack2(d.x, d.z) : 0;
      x[2 * i + 1] = in ? pack2(d.y, d.w) : 0;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kResMaxRounds; ++i) {
      const float4 d = *reinterpret_cast<const float4 *>(mine + slot * kResPreSlot + 4 * (FULL || i < nr ? 2 * i + (l.kq & 1) : 0));
      x[i] = l.kq >> 1 ? pack2(d.y, d.w) : pack2(d.x, d.z);
    }
  }
}
// The blank and duration columns where the per-step launches fold them into the token columns' blocks (see joint_tile): per
// wave slice and half of every eight k a chain of its own, then the halves' sum, then the slices'.
// Float32: one matrix instruction takes the four k of a half.  x: two k of a round, {0, 4, 1, 5}[kq] and two further; the
// swaps (rows 2, 3 of the first with rows 0, 1 of the second, then odd rows with even ones) leave k = kq and 4 + kq.  The
// weights lie that way (k_pack_fold).
// w_at(i): word i of the lane's part of the tile.
template <class W>
__device__ __forceinline__ floatx4 res_fold_mma(W w_at, const uint64_t (&x)[kResMaxRounds]) {
  floatx4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
  for (int i = 0; i < kResMaxRounds; ++i) {
    const auto s32 = __builtin_amdgcn_permlane32_swap((uint32_t)x[i], (uint32_t)(x[i] >> 32), false, false);
    const auto s16 = __builtin_amdgcn_permlane16_swap(s32[0], s32[1], false, false);
    lo = mfma16(w_at(2 * i), __uint_as_float(s16[0]), lo);
    hi = mfma16(w_at(2 * i + 1), __uint_as_float(s16[1]), hi);
  }
  return lo + hi;
}
// Split operands: one of the columns per block.  The operands lie as those of the split products do: a lane has the four k of a half of
// one round after the other, rounds 2 (kq / 2) and the next of either quad (half kq % 2), then round 8 + kq % 2 (half kq / 2), so that a
// chain of fused multiply-adds goes from lane to lane of a slot with them.  (All columns by one block, with matrix instructions and the
// operands read anew in the places that these take: 1.9 us per tile of slots instead of 0.7, which all of the group waited for: batch 32 /
// beam 8 with LM 18.8 / 15.8 us per step, TDT batch 64 16.5 / 14.1.)
__device__ __forceinline__ void res_fold_one(const ResBlock &k, const ResLane &l, const ResW16 &w, const uint64_t (&x)[kResMaxRounds]) {
  auto swap32 = [](float v, int i) { return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false)[i]); };
  auto swap16 = [](float v, int i) { return __uint_as_float(__builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false)[i]); };
  auto round = [&](float acc, int p) {  // parts p, p + 1: k 0 and 2, k 1 and 3
    acc = fmaf(res_raw(w, 2 * p), lo_f(x[p]), acc);
    acc = fmaf(res_raw(w, 2 * p + 2), lo_f(x[p + 1]), acc);
    acc = fmaf(res_raw(w, 2 * p + 1), hi_f(x[p]), acc);
    return fmaf(res_raw(w, 2 * p + 3), hi_f(x[p + 1]), acc);
  };
  float v = round(round(0.f, 0), 2);                     // rounds 0, 1 in the lower half of the wave ..
  v = round(round(swap32(v, 0), 0), 2);                  // .. 2, 3 in the upper one
  v = round(round(swap32(v, 1), 4), 6);
  v = round(round(swap32(v, 0), 4), 6);
  const float lower = swap32(v, 1), upper = swap16(v, 1);
  v = round(l.lane < 32 ? lower : upper, 8);             // round 8 in the first and third 16 lanes,
  v = round(swap16(v, 0), 8);                            // 9 in the second and fourth
  v = swap32(v, 0) + swap32(v, 1);
  if (l.kq == 1) res_red<false>(k, 0)[(k.wave * 64 + l.sl) * 4] = v;
}
// bf16 operands: the lane (column, half) has the half's k in order, and the chain is one of fused multiply-adds.  The weights
// lie in LDS (k.spec), [column][round of all slices][half] four bf16.  (The other columns of the tile are beyond the last one.)
__device__ __forceinline__ void res_fold_bf16(const ResBlock &k, const ResLane &l, int n_cols, bool second,
                                              const uint64_t (&xb)[kResMaxRounds]) {
  const int half = l.lane >> 5, c = l.lane & 31;
  auto up = [](uint32_t lo16) { return __uint_as_float(lo16 << 16); };
#pragma unroll 1
  for (int n = 0; n < n_cols; ++n) {
    const uint64_t *w = k.spec + (n * (8 * kResMaxRounds) + k.wave * kResMaxRounds) * 2 + half;
    float part = 0.f;
#pragma unroll
    for (int i = 0; i < kResMaxRounds; ++i) {
      const uint64_t u = w[2 * i];
      const uint32_t b0 = (uint32_t)xb[i], b1 = (uint32_t)(xb[i] >> 32);
      part = fmaf(up((uint32_t)u & 0xffffu), up(b0 & 0xffffu), part);
      part = fmaf(up((uint32_t)u >> 16), up(b0 >> 16), part);
      part = fmaf(up((uint32_t)(u >> 32) & 0xffffu), up(b1 & 0xffffu), part);
      part = fmaf(up((uint32_t)(u >> 48)), up(b1 >> 16), part);
    }
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(part), __float_as_uint(part), false, false);
    part = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    if (half == 0 && (c < kResSlot || second))
      res_red<true>(k, (c >> 4) * 2)[(k.wave * 64 + (n >> 2) * 16 + (c & 15)) * 4 + (n & 3)] = part;
  }
}
// the slots' last tokens behind the words that the wave holds (a group of a stateless decoder has one tile of slots)
__device__ __forceinline__ void res_update_ctx(const ResBlock &k) {
  const ResLane l = res_lane();
  const uint64_t w = k.word[l.sl];
  const int tok = word_tok(w);
  int4 c = k.ctx[word_src(w)];
  if (tok >= 0) c = make_int4(tok, c.x, c.y, c.z);
  wave_sync();
  if (l.kq == 0) k.ctx[l.sl] = c;
  wave_sync();
}

// split tiles, or two words a round (kResBf16: they are four k); the one that is folded as k_pack_fold leaves it
template <int FORM>
struct ResWJ {
  std::conditional_t<FORM == kResSplit, ResW16[kResRegJ<false>], float[kResRegJ<FORM == kResBf16>][2 * kResMaxRounds]> t;
};
// W_hh: split, or round by round
template <int FORM>
struct ResWR {
  std::conditional_t<FORM == kResSplit, ResW16[kResMaxR], float[kResMaxR][2 * kResMaxRounds]> t;
};
// wj: the tiles that the block keeps in registers; one more may lie in LDS behind the projection's
template <bool FULL, int FORM, bool ST>
__device__ __forceinline__ void res_j_phase(ResBlock &k, int step, const ResWJ<FORM> &wj) {
  if (k.nJ == 0) return;
  constexpr bool BF16 = FORM == kResBf16;
  constexpr int NJ = kResRegJ<BF16>;
  const ResArgs &a = res_args();
  const ResLane l = res_lane();
  const ResAddr ad = res_addr(a, k.g);
  const int nr = FULL ? kResMaxRounds : a.rounds_h;
  if constexpr (BF16) {
    const uint64_t *wx = k.tiles + (size_t)k.nP * (a.P * kResSlot / 2) + (size_t)k.wave * nr * 64 + l.lane;
#pragma unroll 1
    for (int nt = 0; nt < k.nt; nt += 2) {
      const bool second = nt + 1 < k.nt;
      if (step == a.stall_step && nt + 2 >= k.nt) __builtin_amdgcn_endpgm();
      uint64_t x[2 * kResMaxRounds], xb[kResMaxRounds];
      if constexpr (ST) res_stateless_pre<FULL, true, false>(a, k, l, nr, xb);
      else {
        const uint32_t probe = bf16_probe_tile(l, ad.p_tile, second) + ((l.lane & 31) < nr ? l.lane & 31 : 0) * kResRoundBytes;
        bf16_gather<FULL>(l, reinterpret_cast<const char *>(ad.p(step, nt)) + k.wave * nr * kResRoundBytes, 0, nr > 5 ? 5 * kResRoundBytes : 0, min(nr, 5),
                          max(nr - 5, 0), second, ad.p_tile, probe, x);
      }
      if constexpr (!ST) {
#pragma unroll
        for (int i = 0; i < kResMaxRounds; ++i) xb[i] = round_bf16(x + 2 * i);
      }
      auto put_out = [&](int t) {
        __syncthreads();
        res_end_if_given_up();
        if (k.wave < (second ? 4 : 2)) res_j_finish<kResBf16>(k, l, ad, step, nt + (k.wave >> 1), k.jtile[t], ResPar::kJ + 8 * (2 * t + (k.wave & 1)), k.wave);
        ++k.phase;
      };
#pragma unroll
      for (int t = 0; t < NJ + 1; ++t) {
        if (t >= k.nJ) break;
        if constexpr (FULL)
          if (t == 0 && k.fold) {
            res_fold_bf16(k, l, a.N - a.V, second, xb);
            put_out(t);
            continue;
          }
        floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < kResMaxRounds / 2; ++i)
          if (FULL || 2 * i < nr) {
            const bool two = FULL || 2 * i + 1 < nr;
            uint64_t w0, w1;
            if (t < NJ) {
              w0 = pack2(wj.t[t < NJ ? t : 0][4 * i], wj.t[t < NJ ? t : 0][4 * i + 1]);
              w1 = pack2(wj.t[t < NJ ? t : 0][4 * i + 2], wj.t[t < NJ ? t : 0][4 * i + 3]);
            } else {
              w0 = wx[2 * i * 64];
              w1 = wx[(2 * i + (two ? 1 : 0)) * 64];
            }
            acc = mfma_pair_bf16(w0, w1, xb[2 * i], xb[2 * i + 1], two, acc);
          }
        bf16_put(k, l, 0, 0, acc);
        if (second) bf16_put(k, l, 2, 1, acc);
        put_out(t);
      }
    }
  } else {
#pragma unroll 1
    for (int nt = 0; nt < k.nt; ++nt) {
      if (step == a.stall_step && nt + 1 == k.nt) __builtin_amdgcn_endpgm();
      const char *src = reinterpret_cast<const char *>(ad.p(step, nt)) + k.wave * nr * kResRoundBytes;
      [[maybe_unused]] auto relu = [](uint64_t (&x)[kResMaxRounds]) {
#pragma unroll
        for (int i = 0; i < kResMaxRounds; ++i) x[i] = pack2(fmaxf(lo_f(x[i]), 0.f), fmaxf(hi_f(x[i]), 0.f));
      };
      auto done = [&] {
        __syncthreads();
        res_end_if_given_up();
        if (k.jtile[0] >= 0) {
          __builtin_amdgcn_s_setprio(2);
          res_j_finish<FORM>(k, l, ad, step, nt, k.jtile[0], ResPar::kJ + 8 * k.wave, k.wave);
          __builtin_amdgcn_s_setprio(0);
        }
        ++k.phase;
      };
      if constexpr (FORM == kResF32) {
        uint64_t x[kResMaxRounds];
        if constexpr (ST) res_stateless_pre<FULL, false, false>(a, k, l, nr, x);
        else {
          const uint32_t offs[2] = {(uint32_t)l.lane * 8, (uint32_t)l.lane * 8 + 5 * kResRoundBytes};
          res_gather<FULL, kResMaxRounds>(offs, [src](int i, const uint32_t (&o)[2]) { return src + o[i / 5] + i % 5 * kResRoundBytes; }, nr, x);
        }
        if constexpr (ST) relu(x);
        floatx4 acc[NJ];
        // N tiles from the first on
        auto mma = [&](auto first, auto w_at, auto &c) {
          constexpr int t0 = decltype(first)::value;
#pragma unroll
          for (int t = t0; t < NJ; ++t) c[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < kResMaxRounds; ++i)
            if (FULL || i < nr) {
#pragma unroll
              for (int t = t0; t < NJ; ++t) c[t] = mfma16(w_at(t, 2 * i), lo_f(x[i]), c[t]);
#pragma unroll
              for (int t = t0; t < NJ; ++t) c[t] = mfma16(w_at(t, 2 * i + 1), hi_f(x[i]), c[t]);
            }
        };
        auto in_regs = [&](int t, int i) { return wj.t[t][i]; };
        if (FULL && k.fold) {
          mma(std::integral_constant<int, 1>{}, in_regs, acc);
          acc[0] = res_fold_mma([&](int i) { return wj.t[0][i]; }, x);
        } else {
          mma(std::integral_constant<int, 0>{}, in_regs, acc);
        }
#pragma unroll
        for (int t = 0; t < NJ; ++t)
          if (t < k.nJ) res_put<false>(k, l, t, acc[t]);
        if (k.nJ > NJ) {
          const uint64_t *w = k.tiles + (size_t)k.nP * (a.P * kResSlot / 2) + (size_t)k.wave * nr * 64 + l.lane;
          floatx4 c[NJ];
          mma(std::integral_constant<int, NJ - 1>{}, [&](int, int i) { return i & 1 ? hi_f(w[(i >> 1) * 64]) : lo_f(w[(i >> 1) * 64]); }, c);
          res_put<false>(k, l, NJ, c[NJ - 1]);
        }
        done();
        continue;
      } else {
      ResW16 xs;
      float inv;
      uint64_t xr[kResMaxRounds];
      {
        uint64_t (&x)[kResMaxRounds] = xr;
        if constexpr (ST) res_stateless_pre<FULL, false, true>(a, k, l, nr, x);
        else res_split_gather<FULL, false>(l, src, nr, x);
        if constexpr (ST) relu(x);
        uint32_t m = 0;  // (of values from 0 on, whose bits are in order)
#pragma unroll
        for (int i = 0; i < kResMaxRounds; ++i) m = max(m, max((uint32_t)x[i], (uint32_t)(x[i] >> 32)));
        const auto s16 = __builtin_amdgcn_permlane16_swap(m, m, false, false);
        m = max(s16[0], s16[1]);
        const auto s32 = __builtin_amdgcn_permlane32_swap(m, m, false, false);
        const float scale = split_scale(__uint_as_float(max(s32[0], s32[1])), inv);
        res_split_act(x, scale, xs);
      }
      if (FULL && k.fold) {
        floatx4 c1[1], d1[1];
        res_split_mma<FULL, 1, 1>(wj.t, xs, nr, c1, d1);
        res_fold_one(k, l, wj.t[0], xr);
        if (1 < k.nJ) res_put<false>(k, l, 1, split_join(c1[0], d1[0]) * inv);
      } else {
        floatx4 acc[NJ], cor[NJ];
        res_split_mma<FULL, 0, NJ>(wj.t, xs, nr, acc, cor);
#pragma unroll
        for (int t = 0; t < NJ; ++t)
          if (t < k.nJ) res_put<false>(k, l, t, split_join(acc[t], cor[t]) * inv);
      }
      if (k.nJ > NJ) {
        const ResW16 w[1] = {res_split_load(reinterpret_cast<const uintx4_t *>(k.tiles) + (size_t)k.nP * (kResTileFloats / 4) + (size_t)k.wave * kResQuads * 64, l)};
        floatx4 c1[1], d1[1];
        res_split_mma<FULL, 0, 1>(w, xs, nr, c1, d1);
        res_put<false>(k, l, NJ, split_join(c1[0], d1[0]) * inv);
      }
      done();
      }
    }
  }
}

// the block's own pieces of pre[step] and of the logits of `step`: every word of `step` has been seen, i.e. every selecting
// block has read its logits, which needed every piece of pre.
// Who reads a place next (four steps on, see kResStepRing) has seen words that needed what this wave wrote for two steps on,
// which it stores behind the acknowledgement of these.
template <int FORM>
__device__ __forceinline__ void res_clear_pz(const ResArgs &a, const ResBlock &k, const ResAddr &ad, int step) {
  const ResLane l = res_lane();
  for (int nt = 0; nt < k.nt; ++nt) {
    if (k.ptile >= 0) clear_p(k, l, ad, step, nt);
    if constexpr (FORM == kResBf16) {
      if (k.wave >> 1 == (nt & 1)) {
        if (k.jtile[0] >= 0) clear_z<FORM>(k, l, ad, step, nt, k.jtile[0]);
        if (k.jtile[1] >= 0) clear_z<FORM>(k, l, ad, step, nt, k.jtile[1]);
      }
    } else {
      if (k.jtile[0] >= 0) clear_z<FORM>(k, l, ad, step, nt, k.jtile[0]);
    }
  }
}

// ---------------------------------------------------------------------------
// blocks that own tiles
// ---------------------------------------------------------------------------
// place of the lane's unit of W_hh tile t in the fragment order of h (split: of the hi, or the lo, of the two units of a pair of lanes)
template <int FORM>
__device__ __forceinline__ int res_h_ofs(const ResLane &l, int t) {
  if constexpr (FORM == kResSplit) return ((t >> 1) * 4 + (l.kq & 1) * 2 + (l.kq >> 1)) * (2 * kResSlot) + l.sl * 2 + (t & 1);
  return ((t >> 1) * 4 + (t & 1) * 2 + (l.kq >> 1)) * (2 * kResSlot) + l.sl * 2 + (l.kq & 1);
}

// The cells of the wave's tile for N tiles of slots.  (All of them at once, without a branch per slot or tile and with divisions that
// share no condition register: one after the other the five divisions of a cell alone, each a chain of ten instructions, took 0.25 us
// per tile of slots.)
template <bool FULL, int FORM, int N>
__device__ __forceinline__ void res_cells(const ResBlock &k, int step, int mytile, const float *Rl, float *cl, float *hl) {
  const ResArgs &a = res_args();
  const ResLane l = res_lane();
  const ResAddr ad = res_addr<FULL>(a, k.g);
  const int P = FULL ? 8 * 8 * kResMaxRounds : a.P, V = a.V, NT = a.NT;
  const float *G = a.G + 4 * (8 * (mytile >> 1) + (mytile & 1));
  const int hofs = res_h_ofs<FORM>(l, mytile);
  float4 g4[N], r4[N];
  float c[N], h[N];
  int at[N];
  uint64_t w[N];
#pragma unroll
  for (int nt = 0; nt < N; ++nt) w[nt] = k.word[nt * kResSlot + l.sl];
#pragma unroll
  for (int nt = 0; nt < N; ++nt) {
    const int tok = word_tok(w[nt]);
    g4[nt] = *reinterpret_cast<const float4 *>(G + ((uint32_t)(tok < 0 ? V : tok) * (uint32_t)(4 * P) + 8 * l.kq));
    const int src = word_src(w[nt]);
    at[nt] = (k.wave * NT + (src >> 4)) * 64 + l.kq * 16 + (src & 15);
  }
#pragma unroll
  for (int nt = 0; nt < N; ++nt) {
    r4[nt] = *reinterpret_cast<const float4 *>(Rl + at[nt] * 4);
    c[nt] = cl[at[nt]];
    h[nt] = hl[at[nt]];
  }
#pragma unroll
  for (int nt = 0; nt < N; ++nt) {
    float c1 = c[nt];
    const float h1 = lstm_unit(r4[nt], g4[nt], c1);
    const bool on = word_tok(w[nt]) >= 0;
    c[nt] = on ? c1 : c[nt];
    h[nt] = on ? h1 : h[nt];
  }
  uint32_t out[N];
#pragma unroll
  for (int nt = 0; nt < N; ++nt) {
    out[nt] = __float_as_uint(h[nt]);
    if constexpr (FORM == kResSplit) {
      const uint32_t v = split_f16(h[nt] * kHidScale);
      const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);  // of the lanes of even, of odd kq
      out[nt] = __builtin_amdgcn_perm(s[1], s[0], (l.kq & 1) ? 0x07060302u : 0x05040100u);
    }
  }
  wait_stores_acknowledged();
#pragma unroll
  for (int nt = 0; nt < N; ++nt)
    res_store(k.local, reinterpret_cast<uint32_t *>(ad.h(step, nt) + hofs), out[nt]);
  wave_sync();
#pragma unroll
  for (int nt = 0; nt < N; ++nt) {
    const int to = (k.wave * NT + nt) * 64 + l.lane;
    cl[to] = c[nt];
    hl[to] = h[nt];
  }
}

template <bool FULL, int FORM, bool ST>
__device__ __forceinline__ void res_worker(ResBlock k, const ResTab &tab, float *lds) {
  constexpr bool BF16 = FORM == kResBf16, SPLIT = FORM == kResSplit;
  constexpr int NJ = kResRegJ<BF16>, NR = ST ? 0 : kResMaxR;
  const ResArgs &a0 = res_args();
  k.nR = res_uniform(tab.nR);
  k.nJ = res_uniform(tab.nJ);
  k.nP = res_uniform(tab.nP);
  k.fold = res_uniform(FULL && a0.fold && k.nJ > 0 && tab.J[0] >= a0.V / (BF16 ? 32 : 16));
  // which tile's sums this wave finishes, and the tile whose cells it updates
  int pt = -1, jt0 = -1, jt1 = -1;
  if constexpr (BF16) {  // two waves per 32-row tile (output layer: two more for the second slot tile)
    if (k.nP > 0 && k.wave >= kResWaves - 2) pt = 2 * tab.P[0] + (kResWaves - 1 - k.wave);
    if (k.wave < 4) {
      if (k.nJ > 0) jt0 = 2 * tab.J[0] + (k.wave & 1);
      if (k.nJ > 1) jt1 = 2 * tab.J[1] + (k.wave & 1);
    }
  } else {
    if (kResWaves - 1 - k.wave < k.nP) pt = tab.P[kResWaves - 1 - k.wave];
    if (k.wave < k.nJ) jt0 = tab.J[k.wave];
  }
  k.ptile = res_uniform(pt);
  k.jtile[0] = res_uniform(jt0);
  k.jtile[1] = res_uniform(jt1);
  const int mytile = res_uniform(k.wave < k.nR ? tab.R[k.wave] : 0);
  const ResLane l0 = res_lane();
  // weights: projection tiles (and the output-layer tile that finds no registers) to LDS, the others to registers
  {
    const int n4 = SPLIT ? kResTileFloats / 4 : a0.P * kResSlot / 4, h4 = SPLIT ? kResTileFloats / 4 : a0.H * kResSlot / 4;
    auto form = [](const uintx4_t *split, const uint64_t *b, const float *f) {
      return SPLIT ? split : BF16 ? reinterpret_cast<const uintx4_t *>(b) : reinterpret_cast<const uintx4_t *>(f);
    };
    uintx4_t *dst = reinterpret_cast<uintx4_t *>(lds);
    k.tiles = reinterpret_cast<const uint64_t *>(lds);
    for (int tp = 0; tp < k.nP; ++tp) {
      const uintx4_t *src = form(a0.WP, a0.WPb, a0.WPf) + (size_t)tab.P[tp] * n4;
      for (int i = threadIdx.x; i < n4; i += kResThreads) dst[i] = src[i];
      dst += n4;
    }
    if (k.nJ > NJ) {
      const uintx4_t *src = form(a0.WJ, a0.WJb, a0.WJf) + (size_t)tab.J[NJ] * h4;
      for (int i = threadIdx.x; i < h4; i += kResThreads) dst[i] = src[i];
      dst += h4;
    }
    if (BF16 && k.fold) {  // the weights of the blank and duration columns: the words of their lanes, round by round
      uint64_t *spec = reinterpret_cast<uint64_t *>(dst);
      const int n = (a0.N - a0.V) * (a0.H / 8) * 2;
      for (int i = threadIdx.x; i < n; i += kResThreads) {
        const int col = i / (a0.H / 4), at = i % (a0.H / 4);
        spec[i] = a0.WJb[((size_t)tab.J[0] * (a0.H / 8) + (at >> 1)) * 64 + col + 32 * (at & 1)];
      }
      k.spec = spec;
      dst += n / 2;
    }
    k.red = reinterpret_cast<float *>(dst);
  }
  // LDS of the cells: sums W_hh h of the block's tiles, cell state and hidden state of their units, [tile][slot tile][64]
  k.red_blocks = res_uniform(a0.red_blocks);
  float *Rl = k.red + 2 * k.red_blocks * kResRedBlock, *cl = Rl + kResMaxR * a0.NT * 256, *hl = cl + kResMaxR * a0.NT * 64;
  float *par = hl + kResMaxR * a0.NT * 64;
  k.par = reinterpret_cast<const floatx4 *>(par);
  if (threadIdx.x < 16) {
    const int i = threadIdx.x;
    auto tile = [&](int first, int row, const float *unscale, const float *bias) {
      if (unscale) par[4 * (first + ResPar::kScale) + i] = unscale[row];
      if (bias) par[4 * (first + ResPar::kBias) + i] = bias[row];
    };
    constexpr int W = BF16 ? 2 : 1;  // 16-row tiles of a tile
    for (int t = 0; t < W * k.nP; ++t)
      tile(ResPar::kP + 8 * t, res_p_row(W * tab.P[t / W] + t % W, i), a0.pred_unscale, a0.b_pred);
    for (int t = 0; t < W * k.nJ; ++t) {
      const int row = 16 * (W * tab.J[t / W] + t % W) + i;
      if (SPLIT && k.fold && t == 0) {  // (one column, of weights that are not split)
        if (i == 0) par[4 * (ResPar::kJ + ResPar::kBias)] = a0.b_out[a0.V + tab.J[0] - a0.V / 16];
        continue;
      }
      tile(ResPar::kJ + 8 * t, row, a0.out_unscale, a0.b_out);
      if (k.fold && t == 0) par[4 * (ResPar::kJ + ResPar::kScale) + i] = 1.f;  // (folded from weights that are not split)
    }
    for (int t = 0; t < k.nR; ++t) tile(ResPar::kR + 4 * t, 4 * (8 * (tab.R[t] >> 1) + 2 * (i >> 2) + (tab.R[t] & 1)) + (i & 3), a0.hh_unscale, nullptr);
  }
  int2 *info = reinterpret_cast<int2 *>(par + ResPar::kFloats);
  if constexpr (!ST)
    for (int i = threadIdx.x; i < kResMaxR * a0.NT * (256 + 128); i += kResThreads) Rl[i] = 0.f;
  if (threadIdx.x < a0.NT * kResSlot) {
    const int b = res_utt(k, (int)threadIdx.x < k.nslots ? threadIdx.x / a0.K : 0);
    info[threadIdx.x] = make_int2(a0.lengths[b], b * a0.T);
  }
  k.info = info;
  k.word = reinterpret_cast<uint64_t *>(info + a0.NT * kResSlot) + k.wave * a0.NT * kResSlot;
  if constexpr (ST) {  // (in the place of the cells' LDS: 8 waves x NT x 16 x 16 bytes of 6 x NT x 1536)
    k.ctx = reinterpret_cast<int4 *>(Rl) + k.wave * a0.NT * kResSlot;
    for (int i = l0.lane; i < a0.NT * kResSlot; i += 64) k.ctx[i] = make_int4(-1, -1, -1, -1);
    k.quads_inv = res_uniform(65535 / (2 * a0.rounds_h) + 1);
    k.pre = reinterpret_cast<float *>(info + a0.NT * kResSlot) + kResWaves * a0.NT * kResSlot * 2;
  }
  ResWJ<FORM> wj;
  ResWR<FORM> wr;
  {
    if constexpr (!SPLIT) {
      const int nrh = FULL ? kResMaxRounds : a0.rounds_h;
#pragma unroll
      for (int t = 0; t < NJ; ++t)
#pragma unroll
        for (int i = 0; i < kResMaxRounds; ++i) {
          wj.t[t][2 * i] = wj.t[t][2 * i + 1] = 0.f;
          if (t < k.nJ && (FULL || i < nrh)) {
            const bool fold = !BF16 && t == 0 && k.fold;
            const uint64_t *w = BF16 ? a0.WJb : reinterpret_cast<const uint64_t *>(fold ? a0.WJs : a0.WJf);
            const uint64_t v = w[((size_t)(fold ? 0 : tab.J[t]) * (a0.H / 8) + k.wave * nrh + i) * 64 + l0.lane];
            wj.t[t][2 * i] = lo_f(v);
            wj.t[t][2 * i + 1] = hi_f(v);
          }
        }
    } else {
#pragma unroll
      for (int t = 0; t < NJ; ++t) {
        wj.t[t] = ResW16{};
        if (t < k.nJ && !(t == 0 && k.fold)) wj.t[t] = res_split_load(a0.WJ + ((size_t)tab.J[t] * kResWaves + k.wave) * kResQuads * 64, l0);
      }
      if (FULL && k.fold) {  // (words 0 to 19 of the lane, see res_raw: weights of part i of x at 2 i and 2 i + 1)
        uint32_t v[2 * kResMaxRounds];
#pragma unroll
        for (int i = 0; i < kResMaxRounds; ++i) {
          const uint32_t *ws = reinterpret_cast<const uint32_t *>(a0.WJs) + (size_t)k.wave * kResMaxRounds * 128 + 2 * (tab.J[0] - a0.V / 16);
          // the column's weights at the k of the lane's parts (k of a round: see k_pack_fold)
          const int round = i < 8 ? 4 * (i >> 2) + 2 * (l0.kq >> 1) + ((i & 3) >> 1) : 8 + (l0.kq & 1), half = i < 8 ? l0.kq & 1 : l0.kq >> 1;
          v[2 * i] = ws[round * 128 + (i & 1) * 32 + half];
          v[2 * i + 1] = ws[round * 128 + ((i & 1) + 2) * 32 + half];
        }
        wj.t[0] = ResW16{{{v[0], v[1], v[2], v[3]}, {v[8], v[9], v[10], v[11]}}, {{v[4], v[5], v[6], v[7]}, {v[12], v[13], v[14], v[15]}}, {v[16], v[17]}, {v[18], v[19]}};
      }
    }
#pragma unroll
    for (int t = 0; t < NR; ++t) {
      if constexpr (!SPLIT) {
        const int nrp = FULL ? kResMaxRounds : a0.rounds_p;
#pragma unroll
        for (int i = 0; i < kResMaxRounds; ++i) {
          wr.t[t][2 * i] = wr.t[t][2 * i + 1] = 0.f;
          if (t < k.nR && (FULL || i < nrp)) {
            const uint64_t v = reinterpret_cast<const uint64_t *>(a0.WRf)[((size_t)tab.R[t] * (a0.P / 8) + k.wave * nrp + i) * 64 + l0.lane];
            wr.t[t][2 * i] = lo_f(v);
            wr.t[t][2 * i + 1] = hi_f(v);
          }
        }
      } else {
        wr.t[t] = ResW16{};
        if (t < k.nR) wr.t[t] = res_split_load(a0.WR + ((size_t)tab.R[t] * kResWaves + k.wave) * kResQuads * 64, l0);
      }
    }
    // (loaded once; without this the compiler would rather load them again in every step)
    auto keep = [](ResW16 &w) { asm volatile("" : "+v"(w.h[0]), "+v"(w.h[1]), "+v"(w.l[0]), "+v"(w.l[1]), "+v"(w.th), "+v"(w.tl)); };
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
      if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < 2 * kResMaxRounds; ++i) asm volatile("" : "+v"(wj.t[t][i]));
      } else {
        keep(wj.t[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < NR; ++t) {
      if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < 2 * kResMaxRounds; ++i) asm volatile("" : "+v"(wr.t[t][i]));
      } else {
        keep(wr.t[t]);
      }
    }
  }
  __syncthreads();
  int over = res_first_words(a0, k);
  for (int step = 0; over == 0; ++step) {
    // ---- cells
    if (!ST && k.wave < k.nR) {
      // (the later ones of the two waves that have cells on a SIMD would get what the earlier leave)
      if (k.wave >= kResWaves / 2) __builtin_amdgcn_s_setprio(2);
      if (k.nt == 1) res_cells<FULL, FORM, 1>(k, step, mytile, Rl, cl, hl);
      else if (k.nt == 2) res_cells<FULL, FORM, 2>(k, step, mytile, Rl, cl, hl);
      else res_cells<FULL, FORM, 3>(k, step, mytile, Rl, cl, hl);
      __builtin_amdgcn_s_setprio(0);
    }
    if constexpr (!ST)
      res_p_phase<FULL, FORM>(k, step);
    res_j_phase<FULL, FORM, ST>(k, step, wj);
    // (under the selection: ahead of the projection the waits for the activations included these stores)
    if (step > 0) {
      const ResArgs &a = res_args();
      res_clear_pz<FORM>(a, k, res_addr(a, k.g), step - 1);
    }
    // ---- R
    if constexpr (!ST) if (k.nR > 0) {
      const ResArgs &a = res_args();
      const ResLane l = res_lane();
      const ResAddr ad = res_addr(a, k.g);
      const int nrp = FULL ? kResMaxRounds : a.rounds_p;
      // h of two steps ago is cleared under the selection: the words of the last step needed h of the last step from every
      // owner of W_hh tiles, who had multiplied h of two steps ago by then.  Who reads the place next (h of two steps on)
      // has seen words that needed this wave's h of the next step, which it stores behind the acknowledgement of these.
      // (Cleared ahead of the cell update, the acknowledgement was waited for on the critical path: one utterance 9.19 -> 9.03
      // ms.  Behind the products below, the clear delays the next step where they outlast the selection: batch 32 / beam 8
      // 1.3 % slower.)
      if (step > 1 && k.wave < k.nR)
        for (int nt = 0; nt < k.nt; ++nt)
          res_store(k.local, reinterpret_cast<uint32_t *>(ad.h(step - 2, nt) + res_h_ofs<FORM>(l, mytile)), kResEmpty);
#pragma unroll 1
      for (int nt = 0; nt < k.nt; ++nt) {
        ResW16 xs;
        uint64_t x[kResMaxRounds];
        const char *src = reinterpret_cast<const char *>(ad.h(step, nt)) + k.wave * nrp * kResRoundBytes;
        // (nearly always there: the logits needed all of it)
        if constexpr (!SPLIT) {
          const uint32_t offs[2] = {(uint32_t)l.lane * 8, (uint32_t)l.lane * 8 + 5 * kResRoundBytes};
          res_gather<FULL, kResMaxRounds>(offs, [src](int i, const uint32_t (&o)[2]) { return src + o[i / 5] + i % 5 * kResRoundBytes; }, nrp, x);
        } else {
          res_split_gather<FULL, true>(l, src, nrp, x);
          xs = res_split_words(x);
        }
        auto three = [&](auto first) {
          constexpr int t0 = decltype(first)::value;
          if (t0 >= k.nR) return;
          // (tiles that the block does not own have zero weights; fewer branches are worth more than their instructions)
          floatx4 acc[3];
          if constexpr (!SPLIT) {
#pragma unroll
            for (int t = 0; t < 3; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < kResMaxRounds; ++i)
              if (FULL || i < nrp) {
#pragma unroll
                for (int t = 0; t < 3; ++t) acc[t] = mfma16(wr.t[t0 + t][2 * i], lo_f(x[i]), acc[t]);
#pragma unroll
                for (int t = 0; t < 3; ++t) acc[t] = mfma16(wr.t[t0 + t][2 * i + 1], hi_f(x[i]), acc[t]);
              }
          } else {
            floatx4 cor[3];
            res_split_mma<FULL, t0, 3>(wr.t, xs, nrp, acc, cor);
#pragma unroll
            for (int t = 0; t < 3; ++t) acc[t] = split_join(acc[t], cor[t]);
          }
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (t0 + t < k.nR) res_put<BF16>(k, l, t, acc[t]);
          __syncthreads();
          res_end_if_given_up();
          if (k.wave >= t0 && k.wave < t0 + 3 && k.wave < k.nR) {
            floatx4 s = res_sum<BF16>(k, l, k.wave - t0);
            if constexpr (SPLIT) s *= k.par[ResPar::kR + 4 * k.wave + l.kq];
            *reinterpret_cast<floatx4 *>(Rl + ((k.wave * a.NT + nt) * 64 + l.lane) * 4) = s;
          }
          ++k.phase;
        };
        static_assert(kResMaxR == 6);
        three(std::integral_constant<int, 0>{});
        three(std::integral_constant<int, 3>{});
      }
    }
    over = res_words(k, step);
    if constexpr (ST) {
      if (over == 0) res_update_ctx(k);
    }
  }
}

// ---------------------------------------------------------------------------
// selecting blocks
// ---------------------------------------------------------------------------
// One step of an utterance: its rows of logits are read by all waves of the block, which leave statistics of every chunk of 32 columns
// in LDS, and the keys themselves (res_row); one wave then takes the Beam best of all candidates of the utterance at once
// (res_select).  It turns the largest key of every set of chunks into the score that it would have as a candidate: the K-th largest of
// these is a lower bound of the K-th largest of all candidates, a close one, and only the chunks that reach it, few more than K,
// are looked at again.  (With the K best of every row first, ranked among the dozens of keys that reach a bound of the row alone, and
// then the ranking of K (K + 1) candidates, the time from the last logit to the words was, at beam 4 / 8 / 12, 4.4 / 7.0 / 9.0 us, here
// 2.8 / 5.7 / 6.3; ms per decode: one utterance, beam 4, 7.09 -> 6.13, batch 32 beam 4 7.62 -> 6.61, batch 16 beam 12 15.4 -> 12.4, batch
// 32 beam 8 with LM 13.4 -> 12.7, stateless batch 8 3.35 -> 2.89.)
constexpr int kResMaxHyps = 24;  // hypotheses of a selecting block
// floats of a row of keys in LDS (those behind the vocabulary are -inf)
__host__ __device__ inline int res_row_floats(int V) { return V <= 128 ? 128 : V <= 512 ? 512 : kResMaxV; }
// An utterance's hypotheses (up to ctx: kept from step to step) and what a step of its selection needs.
// a hypothesis' tokens as candidates: (score + key) + base + lm (see res_select)
struct __align__(16) ResRow {
  double score, base, lm, pad;
};
struct ResUtt {
  ResRow row[kMaxBeam];            // (of these, score is kept)
  int4 state[kMaxBeam];            // frame, symbols in the frame, length, last token
  uint32_t hash[kMaxBeam];
  int kind[kMaxBeam];              // 0: empty, 1: waits or has finished, 2: expanded, 3: the same, with blank alone
  int ctx[kMaxBeam][kCtxMax];
  // of a step
  double lm_const[kMaxBeam], lse[kMaxBeam], margin[kMaxBeam], delta[kMaxBeam], blank_key[kMaxBeam], blank[kMaxBeam];
  int adv[kMaxBeam];               // frames that a token (low half) and that blank advances
  float set[64];
  int chunk[16 * 32 + 16];         // hypothesis * 32 + chunk of those that reach the bound
  double top_key[kTop + 8], top_val[kTop];
  int top_flat[kTop + 8];
  // new slots (see recombine)
  double n_score[kMaxBeam];
  int n_t[kMaxBeam], n_sym[kMaxBeam], n_len[kMaxBeam], n_last[kMaxBeam], n_live[kMaxBeam];
  uint32_t n_hash[kMaxBeam];
  int n_parent[kMaxBeam], n_code[kMaxBeam];
};
struct ResSelLds {  // LDS of the selection beside its utterances' and the rows of keys
  float zs[kResMaxHyps * 9];
  float2 cst[kResMaxHyps][32];     // (maximum, sum of exponentials) of every chunk of 32 columns
  float kmax[kResMaxHyps][32];     // largest key of every chunk, where keys are not the logits
  LmCtxRec rec[kResWaves][kCtxMax + 1];
};

// floats ahead of the rows of keys
__host__ __device__ inline size_t res_sel_floats(int upc, int NT) {
  return (sizeof(ResSelLds) + 15) / 16 * 4 + (upc * sizeof(ResUtt) + (size_t)NT * kResSlot * kResWaves * 8 + 15) / 16 * 4;
}

// x[i] = max (or sum) of x[i] and the lane that CTRL names, for N values at once: one instruction each plus the wait states of the
// first of four (the compiler's form takes five per value; it does not know of the wait states between these and a DPP instruction of
// its own: none may follow on the results)
#define RB_RES_DPP1(OP, DPP) asm("s_nop 1\n\t" OP " %0, %0, %0 " DPP " row_mask:0xf bank_mask:0xf" : "+v"(x[i]))
#define RB_RES_DPP4(OP, DPP)                                                                             \
  asm("s_nop 1\n\t" OP " %0, %0, %0 " DPP " row_mask:0xf bank_mask:0xf\n\t" OP " %1, %1, %1 " DPP        \
      " row_mask:0xf bank_mask:0xf\n\t" OP " %2, %2, %2 " DPP " row_mask:0xf bank_mask:0xf\n\t" OP       \
      " %3, %3, %3 " DPP " row_mask:0xf bank_mask:0xf"                                                   \
      : "+v"(x[i]), "+v"(x[i + 1]), "+v"(x[i + 2]), "+v"(x[i + 3]))
#define RB_RES_DPP(NAME, OP)                                                                             \
  template <int CTRL, int N>                                                                             \
  __device__ __forceinline__ void NAME(float (&x)[N]) {                                                  \
    _Pragma("unroll") for (int i = 0; i < N / 4 * 4; i += 4) {                                           \
      if constexpr (N >= 4) {                                                                            \
        if constexpr (CTRL == kDppXor1) RB_RES_DPP4(OP, "quad_perm:[1,0,3,2]");                          \
        else if constexpr (CTRL == kDppXor2) RB_RES_DPP4(OP, "quad_perm:[2,3,0,1]");                     \
        else if constexpr (CTRL == kDppHalfMirror) RB_RES_DPP4(OP, "row_half_mirror");                   \
        else RB_RES_DPP4(OP, "row_mirror");                                                              \
      }                                                                                                  \
    }                                                                                                    \
    _Pragma("unroll") for (int i = N / 4 * 4; i < N; ++i) {                                              \
      if constexpr (CTRL == kDppXor1) RB_RES_DPP1(OP, "quad_perm:[1,0,3,2]");                            \
      else if constexpr (CTRL == kDppXor2) RB_RES_DPP1(OP, "quad_perm:[2,3,0,1]");                       \
      else if constexpr (CTRL == kDppHalfMirror) RB_RES_DPP1(OP, "row_half_mirror");                     \
      else RB_RES_DPP1(OP, "row_mirror");                                                                \
    }                                                                                                    \
  }
RB_RES_DPP(dpp_max_n, "v_max_f32_dpp")
RB_RES_DPP(dpp_add_n, "v_add_f32_dpp")
#undef RB_RES_DPP
#undef RB_RES_DPP4
#undef RB_RES_DPP1
template <int LANES, int N>
__device__ __forceinline__ void group_max_n(float (&x)[N]) {
  dpp_max_n<kDppXor1>(x);
  dpp_max_n<kDppXor2>(x);
  if constexpr (LANES >= 8) dpp_max_n<kDppHalfMirror>(x);
  if constexpr (LANES >= 16) dpp_max_n<kDppMirror>(x);
}
template <int LANES, int N>
__device__ __forceinline__ void group_sum_n(float (&x)[N]) {
  dpp_add_n<kDppXor1>(x);
  dpp_add_n<kDppXor2>(x);
  if constexpr (LANES >= 8) dpp_add_n<kDppHalfMirror>(x);
  if constexpr (LANES >= 16) dpp_add_n<kDppMirror>(x);
}

// Columns 128 (part NQ .. part NQ + NQ - 1) of a hypothesis' row of logits, by one wave: statistics of the chunks as the per-step kernels
// form them, the blank and duration logits, and the keys, which go to LDS.  A lane holds columns 128 q + 2 lane + {0, 1}; 16 lanes are a
// chunk of 32.  late_lm: row holds the LM's scores (log10), to which the keys follow.  stash: whether it takes the keys at all.
// (Every load is unconditional, from a clamped address: the wave's time is the latency of this chain.)
template <int NQ, int PLAIN>
__device__ __forceinline__ void res_row(int g, int step, int slot, float *row, bool late_lm, bool stash, int hyp, int part, ResSelLds &L) {
  const ResArgs &a = res_args();
  const int lane = threadIdx.x & 63, V = a.V, nz = a.N - V;
  const int q0 = part * NQ;
  const float *zrow = res_addr(a, g).z(step, slot);
  const int v_last = (V - 1) & ~1;
  uint64_t zz[NQ + 1];  // the last: blank and duration logits, one per lane
  const uint32_t *ps = reinterpret_cast<const uint32_t *>(zrow) + V + (lane < nz ? lane : 0);
  ResWait w;
  for (;;) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) zz[q] = load_agent(reinterpret_cast<const uint64_t *>(zrow + min(128 * (q0 + q) + 2 * lane, v_last)));
    zz[NQ] = load_agent(ps);
    if (__ballot(res_any_empty(zz)) == 0ull) break;
    w.again();
  }
  if (part == 0 && lane < nz) L.zs[hyp * nz + lane] = lo_f(zz[NQ]);
  float z[2 * NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    z[2 * q] = lo_f(zz[q]);
    z[2 * q + 1] = hi_f(zz[q]);
  }
  const bool whole = 128 * (q0 + NQ) <= V;
  auto mask = [&](float (&x)[2 * NQ]) {  // a place without a token: -inf
    if (whole) return;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int n = 128 * (q0 + q) + 2 * lane;
      x[2 * q] = n < V ? x[2 * q] : -INFINITY;
      x[2 * q + 1] = n + 1 < V ? x[2 * q + 1] : -INFINITY;
    }
  };
  mask(z);
  float *keys = row + 128 * q0 + 2 * lane;
  if (PLAIN == 0 && late_lm) {
    float x[2 * NQ], km[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float2 lm = *reinterpret_cast<const float2 *>(keys + 128 * q);
      const float l0 = lm.x * kLn10, l1 = lm.y * kLn10;
      x[2 * q] = z[2 * q] + a.sel.lambda * l0;
      x[2 * q + 1] = z[2 * q + 1] + a.sel.lambda * l1;
    }
    mask(x);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      *reinterpret_cast<float2 *>(keys + 128 * q) = make_float2(x[2 * q], x[2 * q + 1]);
      km[q] = fmaxf(x[2 * q], x[2 * q + 1]);
    }
    group_max_n<16>(km);
    if ((lane & 15) == 0)
#pragma unroll
      for (int q = 0; q < NQ; ++q) L.kmax[hyp][4 * (q0 + q) + (lane >> 4)] = km[q];
  } else if (PLAIN || stash) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) *reinterpret_cast<float2 *>(keys + 128 * q) = make_float2(z[2 * q], z[2 * q + 1]);
  }
  // chunk statistics
  float mx[NQ], sum[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) mx[q] = fmaxf(z[2 * q], z[2 * q + 1]);
  group_max_n<16>(mx);
  bool odd = false;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const float m = fmaxf(mx[q], -3.4028235e38f);  // (a chunk of -inf only: sum 0)
    sum[q] = __expf(z[2 * q] - m);
    sum[q] += __expf(z[2 * q + 1] - m);
    odd |= sum[q] != sum[q];
  }
  if (__ballot(odd) != 0ull) {  // (logits that are no numbers count for nothing)
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      sum[q] = z[2 * q] > -INFINITY ? __expf(z[2 * q] - mx[q]) : 0.f;
      sum[q] += z[2 * q + 1] > -INFINITY ? __expf(z[2 * q + 1] - mx[q]) : 0.f;
    }
  }
  group_sum_n<16>(sum);
  if ((lane & 15) == 0)
#pragma unroll
    for (int q = 0; q < NQ; ++q) L.cst[hyp][4 * (q0 + q) + (lane >> 4)] = make_float2(mx[q], sum[q]);
}

// LM scores (log10) of every token after a hypothesis, by one wave, into an LDS row: see lm_row_block
__device__ __forceinline__ void res_lm_row(const LmView &lm, const int *hist, int len, float *row, LmCtxRec *rec) {
  const int lane = threadIdx.x & 63, nj = lm.order - 1;
  int toks[kCtxMax], have = 0;
#pragma unroll
  for (int i = 0; i < kCtxMax; ++i) {
    toks[i] = hist[i];
    if (toks[i] >= 0 && have == i) have = i + 1;
  }
  int jmax = nj < have ? nj : have;
  jmax = len < jmax ? len : jmax;
  constexpr int NU = kResMaxV / 64;
  float uni[NU];
#pragma unroll
  for (int q = 0; q < NU; ++q) {
    const int v = lane + 64 * q;
    uni[q] = lm.uni[v < lm.V ? v : 0];
  }
  if (lane >= 1 && lane <= kCtxMax) rec[lane] = lm_probe(lm, toks, lane, jmax);
  wave_sync();
  double bo[kCtxMax + 1];
  {
    double acc = 0.0;
#pragma unroll
    for (int j = kCtxMax; j >= 1; --j) {
      bo[j] = acc;
      if (j <= nj) acc += (double)rec[j].backoff;
    }
    bo[0] = acc;
  }
  const float base = (float)bo[0];
#pragma unroll
  for (int q = 0; q < NU; ++q) {
    const int v = lane + 64 * q;
    if (v < lm.V) row[v] = uni[q] + base;
  }
#pragma unroll
  for (int j = 1; j <= kCtxMax; ++j) {
    if (j > nj) break;
    wave_sync();
    const float add = (float)bo[j];
    const int beg = rec[j].begin, cnt = rec[j].count;
    for (int i0 = lane; i0 < cnt; i0 += 4 * 64) {  // four successors of a lane in flight at once
      int st[4];
      float sp[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 + 64 * q;
        st[q] = lm.succ_tok[beg + (i < cnt ? i : 0)];
        sp[q] = lm.succ_p[beg + (i < cnt ? i : 0)];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (i0 + 64 * q < cnt) row[st[q]] = sp[q] + add;
    }
  }
  wave_sync();
}

// a word, in all of its places
__device__ __forceinline__ void res_put_word(bool local, uint64_t *p, uint64_t w) {
#pragma unroll
  for (int i = 0; i < kResWordCopies; ++i) {
    if (local) __hip_atomic_store(p + i * kResWordPlace, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    else store_agent(p + i * kResWordPlace, w);
  }
}
// The Beam best of an utterance's candidates, expansion, words, recombination and tree, by one wave.  rows: the utterance's rows of
// keys in LDS (early pruning: of LM scores; the keys are the logits where they came from).  h0: its first hypothesis in the block, u
// in the group, b in the batch.  Returns whether its last step is done.
template <int KC, int PLAIN>
__device__ __forceinline__ bool res_select(const ResBlock &k, int step, int u, int b, int T_b, int h0, const float *rows, ResUtt &s, const ResSelLds &L) {
  const ResArgs &ra = res_args();
  const SelectArgs &a = ra.sel;
  const int K = ra.K, V = ra.V, nz = ra.N - V, stride = res_row_floats(V), lane = threadIdx.x & 63;
  const int ND = PLAIN ? 0 : nz - 1;
  const bool has_lm = PLAIN == 0 && ra.has_lm, early = PLAIN == 0 && a.lm_early, late_lm = has_lm && !early;
  const bool aes = PLAIN == 0 && a.algo == 1, use_gamma = aes && a.gamma < INFINITY;
  const bool prefix = PLAIN == 0 && a.prefix && aes && !early;
  // LPR lanes per hypothesis, of which each takes NC chunks: e, e + LPR, ..
  constexpr int LPR = 64 / KC, NC = 32 / LPR;
  const int e = lane & (LPR - 1), r = lane / LPR, row = r < K ? r : 0;
  const int n_cst = 4 * ((V + 127) / 128);
  const double sc = s.row[row].score;
  const int kind = r < K ? s.kind[row] : 0;
  float2 c[NC];
  float km[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int i = e + LPR * q;
    const float2 v = L.cst[h0 + row][i];
    c[q] = i < n_cst ? v : make_float2(-INFINITY, 0.f);
    km[q] = c[q].x;
    if constexpr (PLAIN == 0) {
      const float x = L.kmax[h0 + row][i];
      km[q] = !late_lm ? km[q] : i < n_cst ? x : -INFINITY;
    }
  }
  const float *zs = L.zs + (h0 + row) * nz;
  const float zb = zs[0];
  // ---- soft-max statistics of the row, added up in the order of the per-step kernels
  float m[1] = {c[0].x}, st_sum = 0.f;
#pragma unroll
  for (int q = 1; q < NC; ++q) m[0] = fmaxf(m[0], c[q].x);
  group_max_n<LPR>(m);
  const float st_mx = m[0];
  if constexpr (KC < 16) {
    float t[1] = {0.f};
#pragma unroll
    for (int q = 0; q < NC; ++q) t[0] = c[q].x > -INFINITY ? t[0] + c[q].y * __expf(c[q].x - st_mx) : t[0];
    group_sum_n<LPR>(t);
    st_sum = t[0];
  } else {  // (a chunk per lane there, in a tree over 16 lanes, then the two sixteens)
    float t[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) t[q] = c[q].x > -INFINITY ? c[q].y * __expf(c[q].x - st_mx) : 0.f;
    group_sum_n<LPR>(t);
    st_sum = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
  }
  const float lse_nb = st_mx + __logf(st_sum);
  const float hi = fmaxf(lse_nb, zb), lo = fminf(lse_nb, zb);
  const float lse_all = hi + __logf(1.f + __expf(lo - hi));
  const double logp_b = (double)zb - (double)lse_all;
  double x_tok = 0.0, x_blank = 0.0;
  int adv = 1 << 16;
  if (ND > 0) {
    float dl[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) dl[d] = zs[1 + (d < ND ? d : 0)];
    adv = best_durations(dl, ND, a.dur_bytes, x_tok, x_blank);
  }
  // ---- candidates.  A token's: what it is ranked by (key) and its score (val), which differ under early pruning and with the prefix
  // search's credit.  Eq. (4): tokens get lambda (ln(1 - p_blank) + lm), blank (1 + lambda) ln p_blank; Eq. (3): tokens lambda lm, blank
  // unchanged.  Late pruning: lambda lm is in the row's keys; early: added to the score of those that are kept.
  const double lm_const = (has_lm && !a.lm_rule3) ? (double)a.lambda * ((double)lse_nb - (double)lse_all) : 0.0;
  const double tok_base = x_tok - (double)lse_all;
  const double lm_key = early ? 0.0 : lm_const;
  const double thr = use_gamma ? (double)fmaxf(st_mx, zb) - (double)lse_all - (double)a.gamma : -INFINITY;
  auto token_key = [&](float z, double score, double base, double lm) {
    double key = score + (double)z + base;
    if (PLAIN == 0) key = key + lm;
    return z >= kLeastKey ? key : -INFINITY;
  };
  double bkey = -INFINITY, bval = -INFINITY;
  if (kind >= 2) {
    double bl = logp_b;
    if (use_gamma && logp_b < thr && kind == 2) bl = -INFINITY;
    bkey = sc + bl + x_blank;
    bval = (has_lm && !a.lm_rule3 && bl > -INFINITY) ? bkey + (double)a.lambda * bl : bkey;
    if (!early) bkey = bval;
  } else if (kind == 1) {
    bkey = bval = sc;  // a waiting or finished hypothesis stays as it is
  }
  if (e == 0 && r < K) {
    s.row[r].base = tok_base;
    if (PLAIN == 0) {
      s.row[r].lm = lm_key;
      s.adv[r] = adv;
      if (early) s.lm_const[r] = lm_const;
      if (use_gamma) {
        s.lse[r] = (double)lse_all;
        s.margin[r] = thr;
      }
    }
  }
  double delta = 0.0;
  if (prefix) {
    // AES++, maximum-length prefix search (Sec. 2.2, "AES"), as select_utterance has it: hypotheses i and j expanded at this step in the
    // same frame with transcript(i) = transcript(j) + v; (j, v), if among j's Beam best tokens, is credited to i for the ranking.
    wave_sync();
    const int i = lane < K ? lane : 0;
    const int4 st = s.state[i];
    const bool open = lane < K && s.kind[i] >= 2 && st.z >= 1;
    double add = -INFINITY;
    for (int j = 0; j < K; ++j) {
      const int4 sj = s.state[j];
      bool pair = open && j != i && s.kind[j] == 2 && sj.x == st.x && sj.z + 1 == st.z && (s.adv[j] & 0xffff) == 0;
      if (pair) pair = mod_mersenne31((uint64_t)s.hash[j] * kHashBase + (uint64_t)(st.w + 1)) == s.hash[i];
      for (unsigned long long todo = __ballot(pair); todo; todo &= todo - 1ull) {
        const int who = __builtin_ctzll(todo), v = __builtin_amdgcn_readlane(st.w, who);
        const float *rj = rows + j * stride;
        const float z = rj[v];
        int ahead = 0;
        for (int n = lane; n < V; n += 64) ahead += comes_before_count(rj[n], n, z, v);
        ahead = wave_sum_i(ahead);
        const ResRow rw = s.row[j];
        double val = token_key(z, rw.score, rw.base, rw.lm);
        if (use_gamma && (double)z - s.lse[j] < s.margin[j]) val = -INFINITY;
        if (lane == who && ahead < K && val > -INFINITY) add = logaddexp_d(add, val);
      }
    }
    if (lane < K) s.delta[lane] = add > -INFINITY ? logaddexp_d(s.row[lane].score, add) - s.row[lane].score : 0.0;
    wave_sync();
    delta = s.delta[row];
    bkey = bkey + delta;
  }
  // ---- a lower bound of the K-th largest: the K-th largest of the maxima of disjoint sets of candidates, those of one, two or four
  // lanes (in float32, rounded down)
  float kmx = km[0];
#pragma unroll
  for (int q = 1; q < NC; ++q) kmx = fmaxf(kmx, km[q]);
  double best = kind == 2 ? token_key(kmx, sc, tok_base, lm_key) : -INFINITY;
  if (use_gamma && (double)kmx - (double)lse_all < thr) best = -INFINITY;
  if (prefix) best = best + delta;
  if (e == LPR - 1) best = bkey > best || !(best > -INFINITY) ? bkey : best;
  float fl = score_floor(best);
  constexpr int SETS = KC == 4 ? 16 : KC == 8 ? 32 : 64, LANES = 64 / SETS;
  if constexpr (LANES > 1) {
    float q[1] = {fl};
    dpp_max_n<kDppXor1>(q);
    if constexpr (LANES == 4) dpp_max_n<kDppXor2>(q);
    fl = q[0];
  }
  if ((lane & (LANES - 1)) == 0) s.set[lane / LANES] = fl;
  wave_sync();
  double tau = (double)kth_largest<SETS>(s.set, fl, K);
  // Where few hypotheses are expanded (at first, and while the others of AES++ wait) these sets may be fewer than K, or say little of the
  // one row that has candidates: there the K-th largest of a row's chunks as well, the largest of the rows'.
  if constexpr (KC > 4) {
    const int open = __popcll(__ballot(kind == 2 && e == 0));
    if (open * (LPR / LANES) < K + 4) {
      for (unsigned long long todo = __ballot(kind == 2 && e == 0); todo; todo &= todo - 1ull) {
        const int first = __builtin_ctzll(todo), h = first / LPR, i = lane & 31;
        const float z = late_lm ? L.kmax[h0 + h][i] : L.cst[h0 + h][i].x;
        double x = token_key(i < n_cst ? z : -INFINITY, readlane_d(sc, first), readlane_d(tok_base, first), readlane_d(lm_key, first));
        if (use_gamma && (double)z - readlane_d((double)lse_all, first) < readlane_d(thr, first)) x = -INFINITY;
        if (prefix) x = x + readlane_d(delta, first);
        const float f = score_floor(x);
        wave_sync();
        if (lane < 32) s.set[lane] = f;
        wave_sync();
        tau = fmax(tau, (double)kth_largest<32>(s.set, f, K));
      }
    }
  }
  // ---- the chunks that reach it, and of these and the blanks the candidates that do
  const float reach = key_reach(tau, sc, tok_base, PLAIN ? 0.0 : prefix ? delta + lm_key : lm_key);
  int n_chunks = 0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const bool in = kind == 2 && km[q] >= reach;
    const unsigned long long mask = __ballot(in);
    const int pos = n_chunks + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
    if (in) s.chunk[pos] = r << 5 | (e + LPR * q);
    n_chunks += __popcll(mask);
  }
  int total = 0;
  auto append = [&](bool in, double key, double val, int flat) {
    const unsigned long long mask = __ballot(in);
    const int pos = total + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
    if (in && pos < kTop) {
      s.top_key[pos] = key;
      if (PLAIN == 0) s.top_val[pos] = val;
      s.top_flat[pos] = flat;
    }
    total += __popcll(mask);
  };
  append(e == LPR - 1 && bkey > -INFINITY && bkey >= tau, bkey, bval, r << kFlatShift | V);
  wave_sync();
  // a candidate of hypothesis h: its key and score
  const float *zr = early ? res_addr(ra, k.g).z(step, u * K) : rows;  // (early: a row of Npad, in global memory)
  const int zstride = early ? ra.Npad : stride;
  auto token = [&](int h, int n, float z, double &key, double &val) {
    const ResRow &rw = s.row[h];
    val = token_key(z, rw.score, rw.base, PLAIN ? 0.0 : rw.lm);
    if (use_gamma && (double)z - s.lse[h] < s.margin[h]) val = -INFINITY;
    key = val;
    if (PLAIN == 0) {
      if (prefix) key = val + s.delta[h];
      if (early) val = key + s.lm_const[h] + (double)a.lambda * (double)(rows[h * stride + (n < V ? n : 0)] * kLn10);
    }
  };
  constexpr int U = KC / 4;  // fours of chunks in flight
  for (int i0 = 0; i0 < n_chunks; i0 += 4 * U) {
    int id[U];
    float2 z[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int at = i0 + 4 * i + (lane >> 4);
      id[i] = s.chunk[at < n_chunks ? at : i0];
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int n = 32 * (id[i] & 31) + 2 * (lane & 15);
      if (PLAIN == 0 && early) {
        const uint64_t x = load_agent(reinterpret_cast<const uint64_t *>(zr + (size_t)(id[i] >> 5) * zstride + min(n, (V - 1) & ~1)));
        z[i] = make_float2(n < V ? lo_f(x) : -INFINITY, n + 1 < V ? hi_f(x) : -INFINITY);
      } else {
        z[i] = *reinterpret_cast<const float2 *>(rows + (id[i] >> 5) * stride + n);
      }
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (i > 0 && i0 + 4 * i >= n_chunks) break;
      const int h = id[i] >> 5, n = 32 * (id[i] & 31) + 2 * (lane & 15);
      const bool there = i0 + 4 * i + (lane >> 4) < n_chunks;
      double k0, v0, k1, v1;
      token(h, n, z[i].x, k0, v0);
      token(h, n + 1, z[i].y, k1, v1);
      append(there && k0 > -INFINITY && k0 >= tau, k0, v0, h << kFlatShift | n);
      append(there && k1 > -INFINITY && k1 >= tau, k1, v1, h << kFlatShift | (n + 1));
    }
  }
  if (total > kTop) {
    if (e == LPR - 1 && r < K) {
      s.blank_key[r] = bkey;
      s.blank[r] = bval;
    }
    wave_sync();
    auto collect = [&](auto in, int most) {  // until there are that many (more than that of the last 64 may be)
      for (int h = 0; h < K && total < most; ++h) {
        if (__builtin_amdgcn_readfirstlane(s.kind[h]) == 2)
          for (int n0 = 0; n0 < V && total < most; n0 += 64) {
            const int n = n0 + lane;
            const float *p = zr + (size_t)h * zstride + min(n, V - 1);
            const float z = PLAIN == 0 && early ? load_agent(p) : rows[h * stride + min(n, V - 1)];
            double key, val;
            token(h, n, z, key, val);
            append(n < V && in(key), key, val, h << kFlatShift | n);
          }
        if (total >= most) break;
        append(lane == 0 && in(s.blank_key[h]), s.blank_key[h], s.blank[h], h << kFlatShift | V);
      }
    };
    narrow_top(s.top_key, K, tau, total, collect);
  }
  // ---- rank and expansion: a lane whose candidate is kept makes slot `rank` of it
  const NewSlot x = rank_and_expand<PLAIN != 0, PLAIN != 0>(s, total, K, V, T_b);
  // The words leave here, ahead of the recombination, which changes none of their fields: the slots of a class stand in the same frame
  // and one of them stays live, so whether any slot is open is known already.  The group's other blocks go on while this wave merges and
  // writes the tree (batch 32 / beam 4: 10.79 -> 10.50 ms per decode, one utterance 9.53 -> 9.33).
  const bool last_step = __ballot(x.alive && x.state.x < T_b) == 0ull || step + 1 >= T_b * (a.max_sym + 1);
  const int slot0 = u * K, n_kept = __popcll(__ballot(x.kept));
  uint64_t *words = res_addr(ra, k.g).w(step) + slot0;
  if (x.kept) res_put_word(k.local, words + x.rank, slot_word(step, last_step ? 1 : 0, slot0 + (x.alive ? x.parent : x.rank), x.appended, x.state.x));
  if (n_kept < K && lane >= n_kept && lane < K) res_put_word(k.local, words + lane, slot_word(step, last_step ? 1 : 0, slot0 + lane, -1, 0));
  put_new_slots(s, x, n_kept, K);
  int ctx[kCtxMax];
  if (a.use_ctx && x.kept) {
#pragma unroll
    for (int i = 0; i < kCtxMax; ++i) ctx[i] = s.ctx[x.parent][i];
  }
  wave_sync();
  if (a.use_ctx) {  // (every read of the old histories lies before)
    if (x.kept)
#pragma unroll
      for (int i = 0; i < kCtxMax; ++i) s.ctx[x.rank][i] = !x.alive ? -1 : x.appended < 0 ? ctx[i] : i == 0 ? x.appended : ctx[i > 0 ? i - 1 : 0];
    if (n_kept < K && lane >= n_kept && lane < K)
#pragma unroll
      for (int i = 0; i < kCtxMax; ++i) s.ctx[lane][i] = -1;
  }
  // ---- recombination, tree, and what the hypotheses do next
  int next = 0, frame = 0;
  if (lane < K) {
    const int j = lane;
    double score;
    bool live;
    const int merged = recombine<KC>(s, K, j, score, live);
    const int4 now = make_int4(s.n_t[j], s.n_sym[j], s.n_len[j], s.n_last[j]);
    s.row[j].score = score;
    s.state[j] = now;
    s.hash[j] = s.n_hash[j];
    if (last_step) {  // what the back-trace ranks and sizes the transcripts by
      store_through(a.score + b * K + j, score);
      store_through(a.len + b * K + j, now.z);
    }
    write_tree(a, b, step, K, j, s.n_parent[j], s.n_code[j], merged);
    if (j == 0 && last_step) end_utterance(a, b, step);
    next = hyp_kind(live, now, T_b, a.max_sym);
    frame = now.x;
  }
  if (aes) {  // only those in the earliest frame are expanded
    const int first = __builtin_amdgcn_readlane(group_min_i<16>(next >= 2 ? frame : 0x7fffffff), 0);
    if (next >= 2 && frame != first) next = 1;
  }
  if (lane < K) s.kind[lane] = next;
  wave_sync();
  return last_step;
}

template <int KC, int PLAIN>
__device__ __forceinline__ void res_selector(ResBlock k, int sel, float *lds) {
  const ResArgs &a0 = res_args();
  const int K = a0.K, lane = threadIdx.x & 63, upc = a0.upc, stride = res_row_floats(a0.V);
  const bool has_lm = a0.has_lm != 0, late_lm = has_lm && !a0.sel.lm_early, early = has_lm && a0.sel.lm_early;
  ResSelLds &L = *reinterpret_cast<ResSelLds *>(lds);
  float *rows = lds + res_sel_floats(upc, a0.NT);
  ResUtt *utt = reinterpret_cast<ResUtt *>(lds + (sizeof(ResSelLds) + 15) / 16 * 4);
  k.word = reinterpret_cast<uint64_t *>(utt + upc) + k.wave * a0.NT * kResSlot;
  const int u0 = sel * upc, nu = min(upc, k.nu - u0);  // the block's utterances of the group (none: nu <= 0)
  const int n_hyp = nu * K;
  // waves per row: two where that leaves less to the wave that has most (at beams up to 4, and from 9 to 12)
  const int parts = stride == kResMaxV && (2 * n_hyp + kResWaves - 1) / kResWaves < 2 * ((n_hyp + kResWaves - 1) / kResWaves) ? 2 : 1;
  int T_b = 0;
  bool finished = true;
  if (k.wave < nu) {  // the wave that selects for utterance u0 + wave
    const int u = u0 + k.wave;
    ResUtt &s = utt[k.wave];
    T_b = res_uniform(a0.lengths[res_utt(k, u)]);
    finished = T_b == 0;
    if (lane < K) {
      const int4 none = make_int4(0, 0, 0, -1);
      s.row[lane].score = lane == 0 ? 0.0 : -INFINITY;
      s.state[lane] = none;
      s.hash[lane] = 0;
      s.kind[lane] = hyp_kind(lane == 0, none, T_b, a0.sel.max_sym);
      for (int i = 0; i < kCtxMax; ++i) s.ctx[lane][i] = -1;
    }
  }
  __syncthreads();
  int over = res_first_words(a0, k);
  for (int step = 0; over == 0; ++step) {
    // rows in the tiles that are left out (their utterances have finished) do not come
    const int n_rows = min(n_hyp, k.nt * kResSlot - u0 * K);
    if (has_lm)  // rows of the hypotheses as the last step left them (their histories: behind its last barrier)
      for (int q = k.wave; q < n_rows; q += kResWaves)
        res_lm_row(res_args().lm, utt[q / K].ctx[q % K], utt[q / K].state[q % K].z, rows + (size_t)q * stride, L.rec[k.wave]);
    // (with two waves per row of logits a wave reads an LM row that another one has written)
    if (late_lm && parts == 2) __syncthreads();
    // (every other row is waited for, also those of finished utterances: a word of this step tells the group's other blocks that
    // all logits of the step were there)
    auto read_rows = [&](auto nq) {
      constexpr int NQ = decltype(nq)::value;
      for (int i = k.wave; i < n_rows * parts; i += kResWaves) {
        const int q = parts == 2 ? i >> 1 : i;
        res_row<NQ, PLAIN>(k.g, step, u0 * K + q, rows + (size_t)q * stride, late_lm, !early, q, parts == 2 ? i & 1 : 0, L);
      }
    };
    if (stride == 128) read_rows(std::integral_constant<int, 1>{});
    else if (stride == 512 || parts == 2) read_rows(std::integral_constant<int, 4>{});
    else read_rows(std::integral_constant<int, 8>{});
    __syncthreads();
    res_end_if_given_up();
    if (k.wave < nu) {
      const int u = u0 + k.wave, b = res_utt(k, u);
      if (finished) {
        if (lane < K) res_put_word(k.local, res_addr(res_args(), k.g).w(step) + u * K + lane, slot_word(step, 1, u * K + lane, -1, 0));
      } else {
        finished = res_select<KC, PLAIN>(k, step, u, b, T_b, k.wave * K, rows + (size_t)k.wave * K * stride, utt[k.wave], L);
      }
    }
    if (has_lm) __syncthreads();
    over = res_words(k, step);
  }
}

// FULL: H = P = 640 (loops of known length).  ST: stateless decoder (P does not count).  KC: beams up to 4, 8, 16.  PLAIN: 1 = ALSD++ on a plain RNN-T (see
// select_utterance), 0 = any.  One block of 8 waves per compute unit (the LDS it asks for is more than half of a unit's).
// The first n_sel blocks of a group select, the others own the tiles.
template <bool FULL, int FORM, bool ST, int KC, int PLAIN>
__global__ __launch_bounds__(kResThreads, 2) void k_decode_resident(ResArgs) {
  extern __shared__ __align__(16) float smem[];
  __shared__ int s_ok;
  __shared__ int16_t s_order[kResMaxNT * kResSlot];
  const ResArgs &a = res_args();
  if (*reinterpret_cast<const volatile int *>(a.sel.done)) return;
  // every block of the launch must be on the chip before any of them waits for another's data
  const int g = (int)blockIdx.x % a.stride;  // (workgroup i runs on XCD i % 8)
  if (g >= a.n_groups) return;
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_or(a.ctl + 2 + g, 1 << (__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_stores_acknowledged();
    __hip_atomic_fetch_add(a.ctl, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const long long t0 = wall_clock64();
    int ok = 0;
    for (;;) {
      if (load_agent(a.ctl + 1)) break;
      if (load_agent(a.ctl) >= a.start_blocks) {
        ok = 1;
        break;
      }
      if (wall_clock64() - t0 > a.start_limit) {
        store_agent(a.ctl + 1, 1);
        *a.h_abort = 1;
        break;
      }
      __builtin_amdgcn_s_sleep(4);
    }
    s_ok = ok && res_on_one_xcd(load_agent(a.ctl + 2 + g), a.stall_step) ? 2 : ok;
  }
  ResBlock k;
  k.g = g;
  const int rank = (int)blockIdx.x / a.stride;
  k.place = rank % kResWordCopies * kResWordPlace;
  k.nu = (a.B - k.g + a.n_groups - 1) / a.n_groups;
  // utterances of the group, g + n_groups i, the longest first: the ends of the slots run empty first, and tiles behind
  // the last unfinished utterance are left out of every phase (TDT, 64 utterances of 4 to 20 s, beam 4: 5.90 -> 5.22 ms;
  // 16 utterances of 3 to 10 s, beam 12: 19.70 -> 18.53)
  if ((int)threadIdx.x < k.nu) {
    const int mine = a.lengths[k.g + a.n_groups * threadIdx.x];
    int at = 0;
    for (int i = 0; i < k.nu; ++i) {
      const int other = a.lengths[k.g + a.n_groups * i];
      at += other > mine || (other == mine && i < (int)threadIdx.x);
    }
    s_order[at] = (int16_t)(k.g + a.n_groups * threadIdx.x);
  }
  if (threadIdx.x == 0) *res_gave_up_word() = 0;
  k.order = s_order;
  k.nt = a.NT;
  __syncthreads();
  if (!s_ok) return;
  k.local = res_uniform(s_ok) == 2;
  k.nslots = k.nu * a.K;
  k.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  k.phase = 0;
  if (rank < a.n_sel) {
    res_selector<KC, PLAIN>(k, rank, smem);
  } else {
    const ResTab &tab = a.tab[rank - a.n_sel];
    if (tab.nR + tab.nJ + tab.nP > 0) res_worker<FULL, FORM, ST>(k, tab, smem);
  }
}

typedef void (*ResKernel)(ResArgs);
// each in a translation unit of its own (resident_kernels.hip), so that they build at once
template <bool FULL, int FORM, bool ST>
ResKernel resident_kernel(int K, bool plain);

}  // namespace rb
