// Selection of a beam-search step (top Beam of an utterance's candidates, tree write, hypothesis state, recombination,
// end-of-utterance detection) as device functions, for the kernels of the per-step launches and for the resident loop.
#pragma once
#include "device_utils.h"

namespace rb {

// ---------------------------------------------------------------------------
// Selection, tree write, state update and recombination: one block per utterance.
// ---------------------------------------------------------------------------
struct SelectArgs {
  // hypothesis state, [M] each (ctx: [M][kCtxMax])
  double *score;
  int *t, *sym, *len, *last;
  uint32_t *hash;
  int *ctx;
  const int *lengths;
  // candidate lists from the joint (k_step_main, k_row_select) or k_inject
  const float *p_max, *p_sum;
  const uint64_t *p_cand;  // [M, K, n_chunks] packed (key, token): entry j of every chunk's list (best first) side by
                           // side, so that lanes that take neighbouring chunks read neighbouring words
  const float *zs;
  int n_chunks;
  int use_ctx;     // 1: the token history of each hypothesis is kept (stateless prediction network, LM)
  int normalized;  // 1: keys are log-probabilities already (injected mode)
  // configuration
  int B, K, V, ND;
  int dur[8];
  uint64_t dur_bytes;   // the same, one byte each (durations are at most 255): one scalar register pair instead of eight
  int algo, max_sym;
  float gamma;
  int has_lm;
  int lm_rule3;         // 1: Eq. (3) (LM on tokens only, blank as it is); 0: Eq. (4)
  int lm_early;         // 1: early pruning: keys carry no LM term; the kept candidates are charged it here
  int prefix;           // 1: AES++ maximum-length prefix search (ranking credit, see select_utterance)
  const float *lm_rows; // [M, V] natural-log LM scores (read for the kept candidates under early pruning)
  float lambda;
  // what the prediction step has to do for each new slot
  int *src_row, *tok;
  // tree [B][S_max][K]
  int *tree_parent, *tree_token, *tree_merged;
  int S_max;
  // loop control
  const int *step_base;
  int step_off;
  int *finished, *utt_steps, *n_finished, *done;
  volatile int *h_done;  // pinned host word, set when every utterance has finished
};

// Where the selection finds the candidate lists of its utterance: the arrays of SelectArgs (rows indexed by
// hypothesis), or arrays in LDS that hold the rows of this utterance only (row0 = its first hypothesis).
struct CandView {
  const uint64_t *cand;
  const float *pmax, *psum, *zs;
  int row0;
};
__device__ __forceinline__ CandView cand_view(const SelectArgs &a) { return CandView{a.p_cand, a.p_max, a.p_sum, a.zs, 0}; }

__device__ __forceinline__ float logaddexp_f(float a, float b) {
  const float m = fmaxf(a, b), d = fminf(a, b) - m;  // d <= 0
  return d > -INFINITY ? m + log1pf(expf(d)) : m;
}

// LDS scratch of one wave while it handles one utterance
template <int CAND>
struct SelectScratchT {
  double score[kMaxBeam];
  double rc_val[CAND];
  double rc_key[CAND];  // early pruning only: what the candidates are ranked by
  double sel_val[kMaxBeam];
  double n_score[kMaxBeam];
  double delta[kMaxBeam];  // prefix search: what the ranking adds to every candidate of the hypothesis
  int t[kMaxBeam], sym[kMaxBeam], len[kMaxBeam], last[kMaxBeam], kind[kMaxBeam];
  uint32_t hash[kMaxBeam];
  int ctx[kMaxBeam][kCtxMax];
  int advt[kMaxBeam], advb[kMaxBeam];
  int rc_flat[CAND];
  int sel_flat[kMaxBeam];
  // more than 64 candidates: those that can be among the Beam best (and what the ranking reads beyond them)
  double top_key[64 + 8];
  int top_flat[64 + 8], top_src[64];
  int n_t[kMaxBeam], n_sym[kMaxBeam], n_len[kMaxBeam], n_last[kMaxBeam], n_live[kMaxBeam];
  uint32_t n_hash[kMaxBeam];
};
// K (K + 1) candidates per utterance: K tokens and blank / stay of every hypothesis
typedef SelectScratchT<kMaxBeam * (kMaxBeam + 1)> SelectScratch;
// TDT with every (symbol, duration) pair as a candidate: K (K + 1) ND of them, for beams up to 8
constexpr int kPairsMaxBeam = 8;
typedef SelectScratchT<kPairsMaxBeam * (kPairsMaxBeam + 1) * 8> SelectScratchPairs;

// the lanes of one wave see each other's LDS writes after this (they run in lockstep; this
// only stops the compiler and the memory pipeline from re-ordering)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// candidate order inside an utterance: (hypothesis k, token v) -> k * 2^20 + v, the same order as
// k * (V + 1) + v for V < 2^20, without a division on the way back
constexpr int kFlatShift = 20;

// x mod (2^31 - 1) for x < 2^62
__device__ __forceinline__ uint32_t mod_mersenne31(uint64_t x) {
  uint64_t y = (x & kHashMod) + (x >> 31);
  y = (y & kHashMod) + (y >> 31);
  return (uint32_t)(y >= kHashMod ? y - kHashMod : y);
}

// Rank of the calling lane's candidate (value mv, index mf) among the cnt candidates in LDS: the number of those that
// come before it.  Every lane reads all candidates (the same address in all lanes: broadcasts, many in flight), eight
// at a time; the arrays hold eight entries beyond cnt that come before nothing.  First on the values alone (one
// comparison per candidate): when no two finite values are equal, which the sum of the counts tells, that is the
// rank; otherwise once more in the full order (value, then index).
__device__ __forceinline__ int rank_by_counting(const double *keys, const int *flats, int cnt, double mv, int mf) {
  int ge = 0;  // candidates not below mine, myself included
  for (int c0 = 0; c0 < cnt; c0 += 8) {
    double cv[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) cv[q] = keys[c0 + q];
#pragma unroll
    for (int q = 0; q < 8; ++q) ge += (int)(cv[q] >= mv);
  }
  const bool finite = mv > -INFINITY;
  const int F = __popcll(__ballot(finite));
  if (wave_sum_i(finite ? ge : 0) == F * (F + 1) / 2) return ge - 1;
  int rank = 0;
  for (int c0 = 0; c0 < cnt; c0 += 8) {
    double cv[8];
    int cf[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      cv[q] = keys[c0 + q];
      cf[q] = flats[c0 + q];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) rank += comes_before_count(cv[q], cf[q], mv, mf);
  }
  return rank;
}

// The Beam best of more than 64 candidates (beams from 8 on), candidate r * (K + 1) + j of hypothesis r, tokens (best first) and then
// blank.  The K-th largest of a few candidates is a lower bound of the K-th largest of all: with each hypothesis' two best tokens and
// its blank (a lane each) few more than K candidates reach it, and those are ranked against each other.  Where more than 64 do (wide
// beams of hypotheses of much the same score), the K-th largest of the first 64 of them is a better bound.  false: many equal ones.
// (Ranking the K (K + 1) / 2 candidates that the order of the sorted lists leaves took 4.5 us at beam 12 and 2.0 at beam 8.  Without
// the second bound beams of 16 fell back to K rounds over all: stateless, batch
// 24, 64 wide, V = 1000 10.19 ms per decode of 40 frames, with it 6.03, with the ranking by the sorted lists 6.59.)
template <class Scratch>
__device__ __forceinline__ bool rank_best(Scratch &s, const double *rank_of, int K, int n) {
  const int lane = threadIdx.x & 63;
  const int r = (171 * lane) >> 9, j = lane - 3 * r;  // lane / 3
  double v = lane < 3 * K ? rank_of[r * (K + 1) + (j == 2 ? K : j)] : -INFINITY;
  s.top_key[lane] = v;
  int total, few = 3 * K;
#pragma unroll 1
  for (int pass = 0;; ++pass) {
    wave_sync();
    int ge = 0;  // of these, not below mine
    for (int c0 = 0; c0 < few; c0 += 8) {
      double cv[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) cv[q] = s.top_key[c0 + q];
#pragma unroll
      for (int q = 0; q < 8; ++q) ge += (int)(cv[q] >= v);
    }
    ge = v > -INFINITY && ge >= K ? ge : 65;
    int least = group_min_i<16>(ge);
    least = min(min(__builtin_amdgcn_readlane(least, 0), __builtin_amdgcn_readlane(least, 16)),
                min(__builtin_amdgcn_readlane(least, 32), __builtin_amdgcn_readlane(least, 48)));
    const double tau = least < 65 ? readlane_d(v, __builtin_ctzll(__ballot(ge == least))) : -INFINITY;
    wave_sync();
    total = 0;
    for (int c0 = 0; c0 < n; c0 += 64) {
      const int c = c0 + lane;
      const double x = rank_of[c < n ? c : 0];
      const bool in = c < n && x > -INFINITY && x >= tau;
      const unsigned long long mask = __ballot(in);
      const int pos = total + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
      if (in && pos < 64) {
        s.top_key[pos] = x;
        s.top_flat[pos] = s.rc_flat[c];
        s.top_src[pos] = c;
      }
      total += __popcll(mask);
    }
    if (total <= 64) break;
    if (pass == 2) return false;
    wave_sync();
    v = s.top_key[lane];
    few = 64;
  }
  if (lane < 8) {  // (the ranking reads in eights)
    s.top_key[total + lane] = -INFINITY;
    s.top_flat[total + lane] = 0x7fffffff;
  }
  wave_sync();
  const bool mine = lane < total;
  const double mv = mine ? s.top_key[lane] : -INFINITY;
  const int mf = mine ? s.top_flat[lane] : 0x7fffffff;
  const int rank = rank_by_counting(s.top_key, s.top_flat, total, mv, mf);
  if (mine && rank < K) {
    s.sel_val[rank] = s.rc_val[s.top_src[lane]];
    s.sel_flat[rank] = mf;
  }
  return true;
}

constexpr float kLn10 = 2.302585092994046f;

// Recombination: equal (hash, length, last token, frame, symbols in frame).  Slot j of the K new ones: which slot it is merged into
// (-1: it holds nothing), its score behind that and whether it stays.
template <int KMAX, class Scratch>
__device__ __forceinline__ int recombine(const Scratch &s, int K, int j, double &score, bool &live) {
  int merged = -1;
  score = s.n_score[j];
  live = s.n_live[j] != 0;
  if (live) {
    // which slots hold the same (hash, length, last token, frame, symbols in frame): all keys are read without
    // branches in between, so that the LDS reads go out together
    const uint32_t mh = s.n_hash[j];
    const int ml = s.n_len[j], mla = s.n_last[j], mt = s.n_t[j], ms = s.n_sym[j];
    // (the hashes first, read without branches in between; the other fields only of the few slots whose hash is equal)
    uint32_t same_hash = 0;
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
      const bool e = (i < K) & (s.n_live[i] != 0) & (s.n_hash[i] == mh);
      same_hash |= (uint32_t)e << i;
    }
    uint32_t same = 1u << j;
    for (uint32_t r = same_hash & ~(1u << j); r; r &= r - 1u) {
      const int i = __builtin_ctz(r);
      const bool e = (s.n_len[i] == ml) & (s.n_last[i] == mla) & (s.n_t[i] == mt) & (s.n_sym[i] == ms);
      same |= (uint32_t)e << i;
    }
    const uint32_t lower = same & ((1u << j) - 1u);
    if (lower == 0) {  // the lowest slot of its class keeps the log-sum, added up in slot order
      merged = j;
      for (uint32_t higher = same & ~((2u << j) - 1u); higher; higher &= higher - 1u)
        score = logaddexp_d(score, s.n_score[__builtin_ctz(higher)]);
    } else {
      merged = __builtin_ctz(lower);
      live = false;
      score = -INFINITY;
    }
  }
  return merged;
}
__device__ __forceinline__ void write_tree(const SelectArgs &a, int b, int S, int K, int j, int parent, int code, int merged) {
  if (S < a.S_max) {
    const size_t ti = ((size_t)b * a.S_max + S) * K + j;
    store_through(a.tree_parent + ti, parent);
    store_through(a.tree_token + ti, code);
    store_through(a.tree_merged + ti, merged);
  }
}
// (one lane) utterance b's last step was S
__device__ __forceinline__ void end_utterance(const SelectArgs &a, int b, int S) {
  store_through(a.finished + b, 1);
  store_through(a.utt_steps + b, S + 1);
  __threadfence();
  const int old = atomicAdd(a.n_finished, 1);
  if (old + 1 == a.B) {
    *reinterpret_cast<volatile int *>(a.done) = 1;
    __threadfence_system();
    *a.h_done = 1;
  }
}

// ---- the Beam best of the few candidates of an utterance that reach a lower bound of the K-th largest, in LDS (see res_select and
// k_utt_few): top_key[0 .. kTop - 1] what they are ranked by, top_val their scores (where they differ), top_flat (hypothesis << kFlatShift | token);
// state, hash, kind, adv of the hypotheses; n_* of the new slots.
constexpr int kTop = 64;  // candidates that are ranked (and eight more are read)
// what a hypothesis does at a step.  0: empty, 1: waits or has finished, 2: expanded, 3: the same, with blank alone.  state: frame, symbols in
// the frame, length, last token
__device__ __forceinline__ int hyp_kind(bool live, int4 state, int T_b, int max_sym) {
  return !live ? 0 : state.x >= T_b ? 1 : state.y >= max_sym ? 3 : 2;
}
// A score as a float that is not above it (no number: -inf).  The K-th largest of such is below the K-th largest score.
__device__ __forceinline__ float score_floor(double x) {
  const float f = (float)x;
  return f > -INFINITY ? f - (fabsf(f) * 2.4e-7f + 1e-30f) : -INFINITY;
}
// K-th largest of SETS values in LDS, one of which each lane holds as well (with fewer sets, some do).  -inf where there are fewer than K.
template <int SETS>
__device__ __forceinline__ float kth_largest(const float *set, float mine, int K) {
  int n[4] = {0, 0, 0, 0};  // not below mine
#pragma unroll
  for (int i = 0; i < SETS; i += 4) {
    const float4 v = *reinterpret_cast<const float4 *>(set + i);
    n[0] += (int)(v.x >= mine);
    n[1] += (int)(v.y >= mine);
    n[2] += (int)(v.z >= mine);
    n[3] += (int)(v.w >= mine);
  }
  const int ge = (n[0] + n[1]) + (n[2] + n[3]);
  const unsigned long long kth = __ballot(mine > -INFINITY && ge == K);
  if (kth != 0ull) return readlane_f(mine, __builtin_ctzll(kth));
  return wave_max(mine > -INFINITY && ge >= K ? mine : -INFINITY);
}
// A bound of keys that a hypothesis' candidates reach which reach tau, (score + key) + base + extra, in float32 and with room for the rounding
// of all of this (no token at -inf is a candidate)
constexpr float kLeastKey = -3.4028235e38f;
__device__ __forceinline__ float key_reach(double tau, double score, double base, double extra) {
  float reach = (float)(((tau - extra) - base) - score);
  reach -= fabsf(reach) * 2.4e-7f + (fabsf((float)score) + fabsf((float)tau)) * 1e-14f + 1e-6f;
  return tau > -INFINITY ? fmaxf(reach, kLeastKey) : kLeastKey;
}
// Many candidates reach the bound: there were fewer than K sets (a single hypothesis at first), or keys are equal.  collect(in, most)
// appends those for which in(key), in the candidates' own order, until there are `most` (more than that of the last 64 may be), and
// counts them in total.  The K-th largest of the first kTop is the next bound; one that cannot be raised is that of the K best itself, and of those
// equal to it the first ones count.
template <class Collect>
__device__ __forceinline__ void narrow_top(const double *top_key, int K, double tau, int &total, Collect collect) {
  const int lane = threadIdx.x & 63;
  bool above = false;  // whether the bound itself is left out
  for (;;) {
    total = 0;
    collect([&](double x) { return x > -INFINITY && (above ? x > tau : x >= tau); }, kTop + 1);
    if (total <= kTop && (!above || total >= K)) break;
    if (total < K) {
      collect([&](double x) { return x == tau; }, K);
      total = min(total, kTop);
      break;
    }
    wave_sync();
    const int have = min(total, kTop);  // (kTop of them, or, above the bound, K or more)
    const double x = top_key[lane];
    int n = 0;
    for (int i = 0; i < have; ++i) n += (int)(top_key[i] >= x);
    // the K-th largest: the largest that K are not below
    double t = lane < have && n >= K ? x : -INFINITY;
    int dummy = 0;
    wave_best(t, dummy);
    above = !(t > tau);
    if (!above) tau = t;
    wave_sync();
  }
}
// The candidate of a lane (of the first `total`): its place among all, and the slot that it becomes if that is below K.
struct NewSlot {
  bool kept, alive;  // alive: as most kept ones (early pruning: the LM's score may be no number)
  int rank, parent, code, appended;  // code: for the tree
  int4 state;
  uint32_t hash;
  double val;
};
// SAME: keys are the scores.  NO_DUR: no durations (adv is not read)
template <bool SAME, bool NO_DUR, class S>
__device__ __forceinline__ NewSlot rank_and_expand(S &s, int total, int K, int V, int T_b) {
  const int lane = threadIdx.x & 63;
  if (lane < 8) {  // (read in eights)
    s.top_key[total + lane] = -INFINITY;
    s.top_flat[total + lane] = 0x7fffffff;
  }
  wave_sync();
  const bool mine = lane < total;
  const int at = mine ? lane : 0;
  const double key = s.top_key[at];
  const int flat = s.top_flat[at];
  NewSlot x;
  if constexpr (SAME) x.val = key; else x.val = s.top_val[at];
  x.parent = (flat >> kFlatShift) & (kMaxBeam - 1);
  const int v = flat & ((1 << kFlatShift) - 1);
  x.state = s.state[x.parent];
  x.hash = s.hash[x.parent];
  const int kind = s.kind[x.parent];
  const int adv = NO_DUR ? 1 << 16 : s.adv[x.parent];
  int ge = 0, gt = 0;
  for (int c0 = 0; c0 < total; c0 += 8) {
    double y[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) y[q] = s.top_key[c0 + q];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      ge += (int)(y[q] >= key);
      gt += (int)(y[q] > key);
    }
  }
  x.rank = gt;
  if (__ballot(mine && ge != gt + 1) != 0ull) {  // equal ones: the full order
    x.rank = 0;
    for (int c = 0; c < total; ++c) x.rank += comes_before_count(s.top_key[c], s.top_flat[c], key, flat);
  }
  x.kept = mine && x.rank < K;
  x.code = -2;
  x.appended = -1;
  if (kind >= 2) {
    if (v == V) {
      x.code = -1;
      x.state.x += adv >> 16;
      x.state.y = 0;
    } else {
      x.code = x.appended = v;
      x.state.z += 1;
      x.state.w = v;
      x.hash = mod_mersenne31((uint64_t)x.hash * kHashBase + (uint64_t)(v + 1));
      x.state.x += adv & 0xffff;
      x.state.y = (adv & 0xffff) == 0 ? x.state.y + 1 : 0;
    }
  }
  x.state.x = min(x.state.x, T_b);
  x.alive = x.kept && (SAME || x.val > -INFINITY);
  if (!SAME && !x.alive) {
    x.state = make_int4(0, 0, 0, -1);
    x.hash = 0;
    x.code = -3;
    x.appended = -1;
  }
  return x;
}
// the new slots, for recombine; those behind the n_kept candidates are empty
template <class S>
__device__ __forceinline__ void put_new_slots(S &s, const NewSlot &x, int n_kept, int K) {
  const int lane = threadIdx.x & 63;
  if (x.kept) {
    const int j = x.rank;
    s.n_live[j] = x.alive;
    s.n_score[j] = x.alive ? x.val : -INFINITY;
    s.n_t[j] = x.state.x;
    s.n_sym[j] = x.state.y;
    s.n_len[j] = x.state.z;
    s.n_last[j] = x.state.w;
    s.n_hash[j] = x.hash;
    s.n_parent[j] = x.alive ? x.parent : -1;
    s.n_code[j] = x.code;
  }
  if (n_kept < K && lane >= n_kept && lane < K) {
    s.n_live[lane] = 0;
    s.n_score[lane] = -INFINITY;
    s.n_t[lane] = s.n_sym[lane] = s.n_len[lane] = 0;
    s.n_last[lane] = s.n_parent[lane] = -1;
    s.n_hash[lane] = 0;
    s.n_code[lane] = -3;
  }
}
// TDT: scores of the most likely duration (the first of equal ones) and of the most likely one that advances, from the logits of ND
// durations; frames that a token (low half) and that blank advances with them.  (Every index is a compile-time constant: see
// select_utterance.)
__device__ __forceinline__ int best_durations(float (&dl)[8], int ND, uint64_t dur_bytes, double &x_tok, double &x_blank) {
  float dmx = -INFINITY, sm = 0.f;
#pragma unroll
  for (int d = 0; d < 8; ++d)
    if (d < ND) dmx = fmaxf(dmx, dl[d]);
#pragma unroll
  for (int d = 0; d < 8; ++d)
    if (d < ND) sm += __expf(dl[d] - dmx);
  const float l = dmx + __logf(sm);
#pragma unroll
  for (int d = 0; d < 8; ++d)
    if (d < ND) dl[d] -= l;
  bool have = false, have_b = false;
  float best_v = 0.f, best_bv = 0.f;
  int best_adv = 0, best_badv = 1;
#pragma unroll
  for (int d = 0; d < 8; ++d)
    if (d < ND) {
      const int du = (int)((dur_bytes >> (8 * d)) & 0xff);
      if (!have || dl[d] > best_v) {
        have = true;
        best_v = dl[d];
        best_adv = du;
      }
      if (du >= 1 && (!have_b || dl[d] > best_bv)) {
        have_b = true;
        best_bv = dl[d];
        best_badv = du;
      }
    }
  x_tok = (double)best_v;
  x_blank = (double)best_bv;
  return best_adv | best_badv << 16;
}

// One beam-search step of utterance b by one wave: the K best tokens and blank of every
// hypothesis (LPR lanes per hypothesis, all hypotheses at once), the Beam best of those,
// expansion, tree write, recombination, end-of-utterance detection.
// NCH > 0: a lane keeps the lists of NCH chunks in registers (n_chunks <= LPR * NCH, K <= KMAX) and
// the K best of the hypothesis come out of a K-way merge of list heads; NCH == 0: the lists are
// scanned in memory at every round instead (any size).
// MULTI: the beam may be wider than the 64 / LPR hypotheses handled at once; the per-hypothesis part then
// runs in several passes.
// PAIRS (TDT): every (symbol, duration) pair of a hypothesis is a candidate of its own (blank only with
// durations >= 1) instead of one duration per symbol; candidate (k, j, d) sits at ((k (K + 1) + j) ND + d.
// ONE: every hypothesis comes with exactly one list (n_chunks == 1, NCH == 1), known at compile time: the merge
// of list heads and its registers drop out.
template <int LPR, int NCH, int KMAX, bool MULTI = false, bool PAIRS = false, class Scratch = SelectScratch,
          bool ONE = false, int PLAIN = 0, bool DYNDUR = false>
__device__ __forceinline__ void select_utterance(const SelectArgs &a, int b, Scratch &s, const CandView cv) {
  const int K = a.K, V = a.V, lane = threadIdx.x & 63;
  // PLAIN (the caller has checked): 1 = ALSD++, 2 = AES++ without prune margin and prefix search, both without
  // durations and LM: the code of the other cases drops out
  const int a_ND = PLAIN ? 0 : a.ND;
  const int a_has_lm = PLAIN ? 0 : a.has_lm, a_lm_early = PLAIN ? 0 : a.lm_early, a_lm_rule3 = PLAIN ? 0 : a.lm_rule3;
  const int a_prefix = PLAIN ? 0 : a.prefix;
  const float a_gamma = PLAIN ? INFINITY : a.gamma;
  const int a_algo = PLAIN ? PLAIN - 1 : a.algo;
  const int m_base = b * K;
  const int nz = 1 + a_ND;
  // ---- every load of the prologue is requested before anything waits on one of them
  const int fin = load_agent(a.finished + b);  // (a wave-uniform word that changes: never through the scalar cache)
  const int S = *a.step_base + a.step_off;
  const int T_b = a.lengths[b];
  double my_score = -INFINITY;
  int my_t = 0, my_sym = 0, my_len = 0, my_last = -1;
  uint32_t my_hash = 0;
  if (lane < K) {
    const int m = m_base + lane;
    my_score = a.score[m];
    my_t = a.t[m];
    my_sym = a.sym[m];
    my_len = a.len[m];
    my_last = a.last[m];
    my_hash = a.hash[m];
  }
  // LPR lanes per hypothesis, 64 / LPR hypotheses at once; a beam wider than that takes several passes
  // over the per-hypothesis part (lists -> K best tokens -> candidate scores in LDS)
  constexpr int kRowsPerPass = 64 / LPR;
  const int e = lane % LPR;  // position inside the lane group
  const int ncand = a.n_chunks * K;
  int rk = 0;                // hypothesis of this lane in the current pass
  bool row_ok = false;
  const uint64_t *cands = nullptr;
  const float *pmax = nullptr, *psum = nullptr;
  uint64_t list[NCH > 0 ? NCH : 1][KMAX];
  float pm[NCH > 0 ? NCH : 1], ps[NCH > 0 ? NCH : 1];
  float zb = 0.f;
  float dl[8];
  // a single chunk's list IS the K best of the hypothesis: lane e takes entries e, e + LPR, .. as they are
  constexpr int kMine = (KMAX + LPR - 1) / LPR;
  const bool one_list = ONE || (NCH == 1 && a.n_chunks == 1);
  uint64_t direct[kMine];
  auto load_rows = [&](int r0) {
    rk = r0 + lane / LPR;
    row_ok = rk < K;
    const int krow = row_ok ? rk : 0;
    const int crow = m_base - cv.row0 + krow;
    cands = cv.cand + (size_t)crow * ncand;
    pmax = cv.pmax + (size_t)crow * a.n_chunks;
    psum = cv.psum + (size_t)crow * a.n_chunks;
    const float *zsr = cv.zs + (size_t)crow * nz;
    // (every load is unconditional, from a clamped address, and what does not apply is replaced afterwards: a load
    // under a condition of its own costs a branch each)
    if constexpr (NCH > 0) {
#pragma unroll
      for (int q = 0; q < NCH; ++q) {
        const int ch = e + LPR * q;
        const bool ok = row_ok && ch < a.n_chunks;
        const int chs = min(ch, a.n_chunks - 1);  // (lanes without a chunk repeat their group's last address: no extra line)
        if constexpr (!ONE) {
          if (!one_list) {
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {
              const uint64_t x = load_agent(cands + (j < K ? j : 0) * a.n_chunks + chs);
              list[q][j] = (ok && j < K) ? x : no_cand();
            }
          }
        }
        const float xm = load_agent(pmax + chs), xs = load_agent(psum + chs);
        pm[q] = (ok && !a.normalized) ? xm : -INFINITY;
        ps[q] = (ok && !a.normalized) ? xs : 0.f;
      }
      if (one_list) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
          const int j = e + LPR * i;
          const uint64_t x = load_agent(cands + (j < K ? j : 0));
          direct[i] = (row_ok && j < K) ? x : no_cand();
        }
      }
    }
    zb = load_agent(zsr);
    if (a_ND > 0) {
#pragma unroll
      for (int d = 0; d < 8; ++d) dl[d] = load_agent(zsr + 1 + (d < a_ND ? d : 0));
    }
  };
  auto process_rows = [&]() {
    // ---- K rounds of "best remaining candidate" in every lane group at once.
    // Lane e keeps the winners of rounds e, e + LPR, ... (at most KMAX / LPR + 1 of them).
    uint64_t mine[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) mine[i] = no_cand();
    if (one_list) {
#pragma unroll
      for (int i = 0; i < kMine; ++i) mine[i] = direct[i];
    } else if constexpr (ONE) {
    } else if constexpr (NCH > 0) {
#pragma unroll
      for (int j = 0; j < KMAX; ++j) {
        if (j < K) {
          uint64_t best = list[0][0];
#pragma unroll
          for (int q = 1; q < NCH; ++q) best = list[q][0] > best ? list[q][0] : best;
          best = group_max_u64<LPR>(best);
#pragma unroll
          for (int q = 0; q < NCH; ++q)
            if (list[q][0] == best) {  // the winner's list moves up (real candidates are unique)
#pragma unroll
              for (int x = 0; x + 1 < KMAX; ++x) list[q][x] = list[q][x + 1];
              list[q][KMAX - 1] = no_cand();
            }
          if (e == j % LPR) mine[j / LPR] = best;
        }
      }
    } else {
      uint64_t last = ~0ull;
      for (int j = 0; j < K; ++j) {
        uint64_t best = no_cand();
        if (row_ok)
          for (int c = e; c < ncand; c += LPR) {
            const uint64_t v = load_agent(cands + c);
            if (v < last && v > best) best = v;
          }
        best = group_max_u64<LPR>(best);
#pragma unroll
        for (int i = 0; i < kMine; ++i)
          if (e == j % LPR && i == j / LPR) mine[i] = best;
        last = best > no_cand() ? best : no_cand() + 1;  // nothing below "no candidate" is eligible again
      }
    }
    // ---- soft-max statistics of the hypothesis (float transcendental math, scores accumulate in double)
    float lse_all = 0.f, lse_nb = 0.f, max_nb = -INFINITY;
    if (!a.normalized) {
      float st_mx = -INFINITY, st_sum = 0.f;
      if constexpr (NCH > 0) {
#pragma unroll
        for (int q = 0; q < NCH; ++q) st_mx = fmaxf(st_mx, pm[q]);
        st_mx = group_max<LPR>(st_mx);
#pragma unroll
        for (int q = 0; q < NCH; ++q)
          if (pm[q] > -INFINITY) st_sum += ps[q] * __expf(pm[q] - st_mx);
      } else {
        if (row_ok)
          for (int c = e; c < a.n_chunks; c += LPR) st_mx = fmaxf(st_mx, load_agent(pmax + c));
        st_mx = group_max<LPR>(st_mx);
        if (row_ok)
          for (int c = e; c < a.n_chunks; c += LPR) {
            const float p = load_agent(pmax + c);
            if (p > -INFINITY) st_sum += load_agent(psum + c) * __expf(p - st_mx);
          }
      }
      st_sum = group_sum<LPR>(st_sum);
      lse_nb = st_mx + __logf(st_sum);
      const float hi = fmaxf(lse_nb, zb), lo = fminf(lse_nb, zb);
      lse_all = hi + __logf(1.f + __expf(lo - hi));
      max_nb = st_mx;
    } else {
      // keys are log-probabilities already; the best token of the row is round 0's winner, the largest
      // of the winners spread over the group's lanes
      max_nb = cand_key(group_max_u64<LPR>(mine[0]));
    }
    const double logp_b = (double)zb - (double)lse_all;
    const double nb = (double)lse_nb - (double)lse_all;
    const double maxlogp = (double)fmaxf(max_nb, zb) - (double)lse_all;
    // TDT durations
    double x_tok = 0.0, x_blank = 0.0;
    int adv_tok = 0, adv_blank = 1;
    if (a_ND > 0) {
      if constexpr (DYNDUR) {
        // The form with indices computed at run time (every access a dependent load: 2.4 us at five durations).  Kept
        // for the main kernel's instantiation for 256 slots and more, where the selection is not what the launch
        // waits for and the kernel as a whole came out 0.9 us SLOWER with the form below (its joint blocks end 0.8 us
        // later: the compiler's placement of the whole kernel, not this block's own time).
        if (!a.normalized) {
          float dmx = -INFINITY, sm = 0.f;
          for (int d = 0; d < a_ND; ++d) dmx = fmaxf(dmx, dl[d]);
          for (int d = 0; d < a_ND; ++d) sm += __expf(dl[d] - dmx);
          const float l = dmx + __logf(sm);
          for (int d = 0; d < a_ND; ++d) dl[d] -= l;
        }
        int best = -1, best_b = -1;
        for (int d = 0; d < a_ND; ++d) {
          if (best < 0 || dl[d] > dl[best]) best = d;
          if (a.dur[d] >= 1 && (best_b < 0 || dl[d] > dl[best_b])) best_b = d;
        }
        if constexpr (!PAIRS) {
          x_tok = (double)dl[best];
          x_blank = (double)dl[best_b];
          adv_tok = a.dur[best];
          adv_blank = a.dur[best_b];
        }
      } else {
        // (every index into dl and a.dur below is a compile-time constant: an index computed at run time turns each
        // access into a dependent load from memory, 2.4 us for this block at five durations)
        if (!a.normalized) {
          float dmx = -INFINITY, sm = 0.f;
#pragma unroll
          for (int d = 0; d < 8; ++d)
            if (d < a_ND) dmx = fmaxf(dmx, dl[d]);
#pragma unroll
          for (int d = 0; d < 8; ++d)
            if (d < a_ND) sm += __expf(dl[d] - dmx);
          const float l = dmx + __logf(sm);
#pragma unroll
          for (int d = 0; d < 8; ++d)
            if (d < a_ND) dl[d] -= l;
        }
        // the most likely duration (the first of equal ones), and the most likely one that advances
        bool have = false, have_b = false;
        float best_v = 0.f, best_bv = 0.f;
        int best_adv = 0, best_badv = 1;
#pragma unroll
        for (int d = 0; d < 8; ++d)
          if (d < a_ND) {
            const int du = (int)((a.dur_bytes >> (8 * d)) & 0xff);
            if (!have || dl[d] > best_v) {
              have = true;
              best_v = dl[d];
              best_adv = du;
            }
            if (du >= 1 && (!have_b || dl[d] > best_bv)) {
              have_b = true;
              best_bv = dl[d];
              best_badv = du;
            }
          }
        if constexpr (!PAIRS) {  // one duration per candidate: the most likely one (for blank: that advances)
          x_tok = (double)best_v;
          x_blank = (double)best_bv;
          adv_tok = best_adv;
          adv_blank = best_badv;
        }
      }
    }
    wave_sync();  // s.kind / s.score / s.sym are needed per row from here on
    // candidate c of the utterance is rc[k * (K + 1) + j]: j < K tokens, j == K blank / stay
    if (row_ok) {
      const int kind = s.kind[rk];
      const bool forced = s.sym[rk] >= a.max_sym;
      const bool use_gamma = a_algo == 1 && a_gamma < INFINITY;
      const double thr = maxlogp - (double)a_gamma;
      const double sc = s.score[rk];
      const int flat0 = rk << kFlatShift;
      // Eq. (4): tokens get lambda (ln(1 - p_blank) + lm), blank (1 + lambda) ln p_blank; Eq. (3): tokens lambda lm,
      // blank unchanged.  Late pruning: lambda * lm is in the key already; early: added here, after the ranking value.
      const double lm_const = (a_has_lm && !a_lm_rule3) ? (double)a.lambda * nb : 0.0;
      const double tok_base = x_tok - (double)lse_all;
      const bool early = a_lm_early != 0;
      // where candidate (hypothesis rk, j-th symbol[, duration d]) goes and how it is numbered for the tie-break
      const int nd = PAIRS ? a_ND : 1;
      auto put = [&](int j, int token, double key, double val) {
        if constexpr (PAIRS) {
          for (int d = 0; d < nd; ++d) {
            // blank must advance by at least one frame; a waiting hypothesis is the single candidate d = 0
            const bool ok = key > -INFINITY && (kind == 1 ? d == 0 : (token < V || a.dur[d] >= 1));
            const double x = kind == 1 ? 0.0 : (double)dl[d];
            const int c = (rk * (K + 1) + j) * nd + d;
            s.rc_val[c] = ok ? val + x : -INFINITY;
            if (early) s.rc_key[c] = ok ? key + x : -INFINITY;
            s.rc_flat[c] = ((flat0 + token) << 3) | d;
          }
        } else {
          const int c = rk * (K + 1) + j;
          s.rc_val[c] = val;
          if (early) s.rc_key[c] = key;
          s.rc_flat[c] = flat0 + token;
        }
      };
#pragma unroll
      for (int i = 0; i < kMine; ++i) {
        const int j = e + LPR * i;
        if (j < K) {
          const float wk = cand_key(mine[i]);
          const int wi = cand_idx(mine[i]);
          double val = -INFINITY, key = -INFINITY;
          if (kind == 2 && wk > -INFINITY && !forced) {
            const double lp = (double)wk - (double)lse_all;  // pre-LM log-probability when no LM is in the key
            if (!(use_gamma && lp < thr)) {
              key = sc + (double)wk + tok_base;
              val = key + lm_const;
              if (early)
                val += (double)a.lambda * (double)a.lm_rows[(size_t)(m_base + rk) * V + wi];
            }
          }
          put(j, wi < V ? wi : V - 1, key, val);
        }
      }
      if (e == LPR - 1) {  // blank / stay: the group's last lane (least loaded with winners)
        double val = -INFINITY, key = -INFINITY;
        if (kind == 2) {
          double bl = logp_b;
          if (use_gamma && logp_b < thr && !forced) bl = -INFINITY;
          key = sc + bl + x_blank;
          val = (a_has_lm && !a_lm_rule3 && bl > -INFINITY) ? key + (double)a.lambda * bl : key;
          s.advt[rk] = adv_tok;
          s.advb[rk] = adv_blank;
        } else if (kind == 1) {
          val = key = sc;  // a waiting or finished hypothesis stays as it is
        }
        put(K, V, key, val);
      }
    }
    wave_sync();
  };
  auto per_utterance = [&]() -> bool {  // false: the utterance had finished before this step
    if (a.use_ctx)
      for (int i = lane; i < K * kCtxMax; i += 64) s.ctx[i / kCtxMax][i % kCtxMax] = a.ctx[m_base * kCtxMax + i];
    if (fin) {  // a finished utterance is frozen; its slots tell the prediction step to copy
      if (lane < K) {
        store_through(a.src_row + m_base + lane, m_base + lane);
        store_through(a.tok + m_base + lane, -1);
      }
      return false;
    }
    if (lane < K) {
      s.score[lane] = my_score;
      s.t[lane] = my_t;
      s.sym[lane] = my_sym;
      s.len[lane] = my_len;
      s.last[lane] = my_last;
      s.hash[lane] = my_hash;
      s.sel_val[lane] = -INFINITY;
      s.sel_flat[lane] = -1;
    }
    // frame of the earliest unfinished hypothesis (lanes >= K hold neutral values)
    const bool my_live = my_score > -INFINITY;
    int t_cur = group_min_i<16>((my_live && my_t < T_b) ? my_t : T_b);
    t_cur = __builtin_amdgcn_readlane(t_cur, 0);
    if (lane < K) s.kind[lane] = my_live ? ((my_t < T_b && (a_algo == 0 || my_t == t_cur)) ? 2 : 1) : 0;
    return true;
  };
  if constexpr (MULTI) {
    for (int r0 = 0; r0 < K; r0 += kRowsPerPass) {
      load_rows(r0);
      if (r0 == 0 && !per_utterance()) return;
      process_rows();
    }
  } else {
    load_rows(0);
    if (!per_utterance()) return;
    process_rows();
  }

  const int n = K * (K + 1) * (PAIRS ? a_ND : 1);
  // ---- AES++, maximum-length prefix search (Sec. 2.2, "AES").  Hypotheses i and j expanded at this step in the
  // same frame with transcript(i) = transcript(j) + v: the step's own expansion (j, v), if it is among j's Beam best
  // tokens and stays in the frame, is credited to i for the RANKING of i's candidates; the new scores stay as they
  // are (the expansion competes on its own and meets i in the recombination; adding it to i's score too would count
  // that alignment twice).  Pairs are found through Eq. (1), like equal transcripts in the recombination.
  const bool prefix = !PAIRS && a_prefix && a_algo == 1 && !a_lm_early;
  if constexpr (!PAIRS) {
    if (prefix) {
      if (lane < K) {
        const int i = lane;
        double add = -INFINITY;
        if (s.kind[i] == 2 && s.len[i] >= 1) {
          const uint32_t hi = s.hash[i];
          const int li = s.len[i], la = s.last[i], ti = s.t[i];
          for (int j = 0; j < K; ++j) {
            if (j == i || s.kind[j] != 2 || s.t[j] != ti || s.len[j] + 1 != li) continue;
            if (s.advt[j] != 0) continue;
            if (mod_mersenne31((uint64_t)s.hash[j] * kHashBase + (uint64_t)(la + 1)) != hi) continue;
            for (int c = 0; c < K; ++c) {  // j's Beam best tokens: is v among them, with a finite score?
              const int idx = j * (K + 1) + c;
              if (s.rc_flat[idx] == (j << kFlatShift) + la && s.rc_val[idx] > -INFINITY) add = logaddexp_d(add, s.rc_val[idx]);
            }
          }
        }
        s.delta[i] = add > -INFINITY ? logaddexp_d(s.score[i], add) - s.score[i] : 0.0;
      }
      wave_sync();
      for (int c = lane; c < n; c += 64) s.rc_key[c] = s.rc_val[c] + s.delta[c / (K + 1)];
      wave_sync();
    }
  }
  // ---- the Beam best of all K * (K + 1) candidates, by (ranking value desc, (k, v) asc); the ranking
  // value is the new score itself except under early pruning and with a prefix credit
  double *rank_of = (a_lm_early || prefix) ? s.rc_key : s.rc_val;
  // candidates a lane may own in the counting form below
  constexpr int kOwn = 1;  // (measured: from 65 candidates up the rounds below are faster than two owned candidates)
  if (n <= 64 * kOwn) {
    // Each lane counts, for each candidate it owns (lane, lane + 64, ..), how many candidates come before it; that
    // count is the candidate's new slot.  (Every lane reads all n candidates back from LDS, the same address in all
    // lanes: such reads are broadcasts and, unlike lane reads into scalar registers, can be requested many at a time.)
    double mv[kOwn];
    int mf[kOwn], rank[kOwn];
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      const int c = lane + 64 * q;
      mv[q] = c < n ? rank_of[c] : -INFINITY;
      mf[q] = c < n ? s.rc_flat[c] : 0x7fffffff;
      rank[q] = 0;
    }
    // the loop below reads in eights: the (up to seven) places after the last candidate hold one that comes before
    // nothing, so that no comparison needs a bound check (the arrays have room beyond n; nothing else uses it)
    if (lane < 8) {
      rank_of[n + lane] = -INFINITY;
      s.rc_flat[n + lane] = 0x7fffffff;
    }
    wave_sync();
    rank[0] = rank_by_counting(rank_of, s.rc_flat, n, mv[0], mf[0]);
#pragma unroll
    for (int q = 0; q < kOwn; ++q)
      if (mv[q] > -INFINITY && rank[q] < K) {
        s.sel_val[rank[q]] = s.rc_val[lane + 64 * q];
        s.sel_flat[rank[q]] = mf[q];
      }
  } else if (!PAIRS && KMAX > 7 && rank_best(s, rank_of, K, n)) {
    // (beams from 8 on)
  } else {
    double last_v = INFINITY;
    int last_i = -1;
    for (int j = 0; j < K; ++j) {
      double bv = -INFINITY;
      int bi = 0x7fffffff;
      for (int c = lane; c < n; c += 64) {
        const double v = rank_of[c];
        const int i = s.rc_flat[c];
        const bool eligible = v > -INFINITY && (v < last_v || (v == last_v && i > last_i));
        if (eligible && comes_before(v, i, bv, bi)) {
          bv = v;
          bi = i;
        }
      }
      wave_best(bv, bi);
      if (!(bv > -INFINITY)) break;
      for (int c = lane; c < n; c += 64)  // the candidate's own lane hands over its score ((k, v) is unique)
        if (s.rc_flat[c] == bi && rank_of[c] == bv) {
          s.sel_val[j] = s.rc_val[c];
          s.sel_flat[j] = bi;
        }
      last_v = bv;
      last_i = bi;
    }
  }
  wave_sync();

  // ---- expansion into the new slots
  int code = -3, parent = -1, appended = -1;
  int ctx_new[kCtxMax];
  if (lane < K) {
    const int j = lane;
    const double val = s.sel_val[j];
#pragma unroll
    for (int i = 0; i < kCtxMax; ++i) ctx_new[i] = -1;
    if (!(val > -INFINITY)) {
      s.n_live[j] = 0;
      s.n_score[j] = -INFINITY;
      s.n_t[j] = 0;
      s.n_sym[j] = 0;
      s.n_len[j] = 0;
      s.n_last[j] = -1;
      s.n_hash[j] = 0;
    } else {
      const int kv = PAIRS ? s.sel_flat[j] >> 3 : s.sel_flat[j];
      const int k = kv >> kFlatShift, v = kv & ((1 << kFlatShift) - 1);
      const int adv_b = PAIRS ? a.dur[s.sel_flat[j] & 7] : s.advb[k];  // frames the step advances: the pair's own
      const int adv_t = PAIRS ? a.dur[s.sel_flat[j] & 7] : s.advt[k];  // duration, or the hypothesis' chosen one
      parent = k;
      int t = s.t[k], sym = s.sym[k], len = s.len[k], last = s.last[k];
      uint32_t hash = s.hash[k];
      if (a.use_ctx) {
#pragma unroll
        for (int i = 0; i < kCtxMax; ++i) ctx_new[i] = s.ctx[k][i];
      }
      if (s.kind[k] == 1) {
        code = -2;
      } else if (v == V) {
        code = -1;
        t += adv_b;
        sym = 0;
      } else {
        code = v;
        appended = v;
        len += 1;
        last = v;
        hash = mod_mersenne31((uint64_t)hash * kHashBase + (uint64_t)(v + 1));
        t += adv_t;
        sym = adv_t == 0 ? sym + 1 : 0;
#pragma unroll
        for (int i = kCtxMax - 1; i > 0; --i) ctx_new[i] = ctx_new[i - 1];
        ctx_new[0] = v;
      }
      if (t > T_b) t = T_b;
      s.n_live[j] = 1;
      s.n_score[j] = val;
      s.n_t[j] = t;
      s.n_sym[j] = sym;
      s.n_len[j] = len;
      s.n_last[j] = last;
      s.n_hash[j] = hash;
    }
  }
  wave_sync();

  if (lane < K) {
    const int j = lane;
    double score;
    bool live;
    const int merged = recombine<KMAX>(s, K, j, score, live);
    const int m = m_base + j;
    // finished when no surviving slot has frames left
    const bool last_step = __ballot(live && s.n_t[j] < T_b) == 0ull || S + 1 >= T_b * (a.max_sym + 1);
    // written through (see store_through): nothing of a step's results waits in an L2 for the kernel's end
    store_through(a.score + m, score);
    store_through(a.t + m, s.n_t[j]);
    store_through(a.sym + m, s.n_sym[j]);
    store_through(a.len + m, s.n_len[j]);
    store_through(a.last + m, s.n_last[j]);
    store_through(a.hash + m, s.n_hash[j]);
    if (a.use_ctx) {
#pragma unroll
      for (int i = 0; i < kCtxMax; ++i) {
        store_through(a.ctx + m * kCtxMax + i, ctx_new[i]);
        s.ctx[j][i] = ctx_new[i];  // (every read of the parents' histories lies before the last wave_sync)
      }
    }
    store_through(a.src_row + m, parent >= 0 ? m_base + parent : m);
    store_through(a.tok + m, appended);
    write_tree(a, b, S, K, j, parent, code, merged);
    if (j == 0 && last_step) end_utterance(a, b, S);
  }
  wave_sync();
}

// picks the lane-group width and register budget for the beam and list sizes at hand.
// FORMS: 0 = beams up to 8 (what the main kernel of a step runs in its tail); 1 = those plus wider beams
// whose hypotheses come with a single list; 2 = wider beams with many lists (several passes, many
// registers).  The heavy forms are kept out of the kernels that do not need them.
template <int FORMS, class Scratch = SelectScratch>
__device__ __forceinline__ void select_dispatch(const SelectArgs &a, int b, Scratch &s, const CandView cv) {
  if constexpr (FORMS == 3) {  // TDT, every (symbol, duration) pair a candidate, beams up to 8
    if (a.K <= 4) {
      if (a.n_chunks <= 16 * 3) select_utterance<16, 3, 4, false, true, Scratch>(a, b, s, cv);
      else select_utterance<16, 0, 4, false, true, Scratch>(a, b, s, cv);
    } else {
      if (a.n_chunks <= 8 * 5) select_utterance<8, 5, 8, false, true, Scratch>(a, b, s, cv);
      else select_utterance<8, 0, 8, false, true, Scratch>(a, b, s, cv);
    }
  } else if constexpr (FORMS == 17) {  // forms 5 and 6 with the durations' older code (see select_utterance)
    select_utterance<16, 3, 4, false, false, Scratch, false, 0, true>(a, b, s, cv);
  } else if constexpr (FORMS == 18) {
    select_utterance<8, 5, 8, false, false, Scratch, false, 0, true>(a, b, s, cv);
  } else if constexpr (FORMS == 5) {  // one form alone (the caller has checked 2 < K <= 4, n_chunks <= 48) ...
    select_utterance<16, 3, 4>(a, b, s, cv);
  } else if constexpr (FORMS == 11) {  // ... the same for ALSD++ on a plain RNN-T (no durations, no LM): beams 3, 4,
    select_utterance<16, 3, 4, false, false, Scratch, false, 1>(a, b, s, cv);
  } else if constexpr (FORMS == 13) {  // ... 1, 2 (n_chunks <= 48),
    select_utterance<16, 3, 2, false, false, Scratch, false, 1>(a, b, s, cv);
  } else if constexpr (FORMS == 14) {  // ... 5 to 8 (n_chunks <= 40);
    select_utterance<8, 5, 8, false, false, Scratch, false, 1>(a, b, s, cv);
  } else if constexpr (FORMS == 15) {  // AES++ without prune margin and prefix search on a plain RNN-T, beams 3, 4
    select_utterance<16, 3, 4, false, false, Scratch, false, 2>(a, b, s, cv);
  } else if constexpr (FORMS == 6) {  // ... (4 < K <= 8, n_chunks <= 40): a kernel a third the size
    select_utterance<8, 5, 8>(a, b, s, cv);
  } else if constexpr (FORMS == 2) {
    if (a.n_chunks <= 16 * 3) select_utterance<16, 3, 16, true>(a, b, s, cv);  // four hypotheses per pass
    else select_utterance<4, 0, 16>(a, b, s, cv);
  } else {
    if (a.K <= 2 && a.n_chunks <= 16 * 3) {  // (a form of its own: the lists are loaded and merged KMAX entries wide)
      select_utterance<16, 3, 2>(a, b, s, cv);
    } else if (a.K <= 4) {
      if (a.n_chunks <= 16 * 3) select_utterance<16, 3, 4>(a, b, s, cv);
      else select_utterance<16, 0, 4>(a, b, s, cv);
    } else if (a.K <= 8) {
      if (a.n_chunks <= 8 * 5) select_utterance<8, 5, 8>(a, b, s, cv);
      else select_utterance<8, 0, 8>(a, b, s, cv);
    } else if constexpr (FORMS == 1) {
      select_utterance<4, 1, 16>(a, b, s, cv);
    }
  }
}
template <int FORMS, class Scratch = SelectScratch>
__device__ __forceinline__ void select_dispatch(const SelectArgs &a, int b, Scratch &s) {
  select_dispatch<FORMS, Scratch>(a, b, s, cand_view(a));
}
// One list per hypothesis, of beams up to KC (4, 8, 12 or 16: chosen on the host, or narrow beams would pay for the ranking of wide ones:
// k_utt_select with all four took 149 scalar spills, 197 since the ranking of wide beams finds a bound first).  PLAIN: see
// select_utterance.
template <int KC, int PLAIN>
__device__ __forceinline__ void select_one_list(const SelectArgs &a, int b, SelectScratch &s, const CandView cv) {
  select_utterance<(KC == 4 ? 16 : KC == 8 ? 8 : 4), 1, KC, false, false, SelectScratch, true, PLAIN>(a, b, s, cv);
}
// which stand-alone selection kernel takes a beam of K with n_chunks lists per hypothesis
__host__ __device__ inline bool select_needs_wide_forms(int K, int n_chunks) { return K > 8 && n_chunks > 4; }

}  // namespace rb
