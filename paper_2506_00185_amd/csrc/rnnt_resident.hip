// Host side of the resident step loop: see resident.h and kernels_resident.h.
#include "resident.h"

#include <algorithm>
#include <cmath>
#include <cstring>

#include "kernels_resident.h"

namespace rb {

namespace {

__device__ __forceinline__ size_t k4_at(int k, int row, int rows) { return ((size_t)(k >> 2) * rows + row) * 4 + (k & 3); }

// row r of a 16-row tile.  MAP 0: rows as they are; 1: tiles of four LSTM units; 2: tiles of projection outputs
template <int MAP>
__device__ __forceinline__ int res_tile_row(int tile, int r) {
  return MAP == 0 ? 16 * tile + r : MAP == 1 ? 4 * (8 * (tile >> 1) + 2 * (r >> 2) + (tile & 1)) + (r & 3) : res_p_row(tile, r);
}

// W (k4-major, `rows` rows, split by k_split_rows) -> [tile of 16 rows][wave][kResQuads * 64 words of 16 bytes] (see ResW16),
// rounds of 8 k, absent ones zero.
// One slice of k per wave: [quadword of a lane][64 lanes], hi and lo of the first two quads of rounds, then those of the last two
// rounds.  halves: two slices of up to five rounds, one of either half of k; of each hi and lo of a quad, [64 lanes] each, then the
// fifth round's [32 lanes]: the lanes of even kq.
template <int MAP>
__global__ void k_pack_split(const uint32_t *W, int rows, int K, int n_tiles, bool halves, uint32_t *out) {
  const int n_rounds = halves ? K / 128 : K / 64;
  const size_t n = (size_t)n_tiles * kResWaves * kResQuads * 64 * 4;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int e = (int)(i & 3), wave = (int)((i >> 8) / kResQuads) % kResWaves, tile = (int)((i >> 8) / kResQuads / kResWaves);
    int at = (int)((i >> 2) % (kResQuads * 64)), slice = wave * n_rounds;
    if (halves) {
      slice += at / 160 * 8 * n_rounds;
      at %= 160;
    }
    const int q = at >> 6, most = halves ? 4 : 8;
    const bool tail = q == (halves ? 2 : 4), lo = tail ? e >> 1 : q & 1;
    int r = at & 15, kq = (at >> 4) & 3;
    if (halves && tail) kq = 2 * (kq & 1);
    const int round = tail ? most + (kq & 1) : 4 * (q >> 1) + 2 * (kq >> 1) + (e >> 1), half = tail ? kq >> 1 : kq & 1;
    const int row = res_tile_row<MAP>(tile, r);
    // the word of a lane holds k and k + 2 (see res_k_of)
    uint32_t v = 0;
    if (round < n_rounds && row < rows) {
      const uint32_t *g = W + ((size_t)((slice + round) * 2 + half) * rows + row) * 4 + (lo ? 2 : 0);  // k pairs (0, 1), (2, 3)
      v = (e & 1) == 0 ? (g[0] & 0xffffu) | g[1] << 16 : g[0] >> 16 | (g[1] & 0xffff0000u);
    }
    out[i] = v;
  }
}
// W as it is -> [tile of 16 rows][round][64 lanes][2].  MAP: as above
template <int MAP>
__global__ void k_pack_f32(const float *W, int rows, int K, int n_tiles, float *out) {
  const int n_rounds = K / 8;
  const size_t n = (size_t)n_tiles * n_rounds * 128;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int e = (int)(i & 1), lane = (int)(i >> 1) & 63;
    const int round = (int)((i >> 7) % n_rounds), tile = (int)((i >> 7) / n_rounds), row = res_tile_row<MAP>(tile, lane & 15);
    out[i] = row < rows ? W[k4_at(res_k_of(round, lane >> 4, e), row, rows)] : 0.f;
  }
}
// rows row0 .. + 15 as res_fold_mma reads them: [round][64 lanes][2], k = 8 round + lane / 16 and four further
__global__ void k_pack_fold(const float *W, int rows, int row0, int K, float *out) {
  const int n = K / 8 * 128;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int e = i & 1, lane = (i >> 1) & 63, row = row0 + (lane & 15);
    out[i] = row < rows ? W[k4_at(8 * (i >> 7) + 4 * e + (lane >> 4), row, rows)] : 0.f;
  }
}
// For the bf16 matrix instructions: [tile of 32 rows][round][64 lanes] four bf16 (values are bf16 already)
template <int MAP>
__global__ void k_pack_bf16(const float *W, int rows, int K, int n_tiles, uint64_t *out) {
  const int n_rounds = K / 8;
  const size_t n = (size_t)n_tiles * n_rounds * 64;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int lane = (int)(i & 63), r = lane & 31, half = lane >> 5;
    const int round = (int)((i >> 6) % n_rounds), tile = (int)((i >> 6) / n_rounds);
    const int row = MAP == 0 ? 32 * tile + r : res_p_row(2 * tile + (r >> 4), r & 15);
    float v[4];
    for (int q = 0; q < 4; ++q) v[q] = row < rows ? W[k4_at(8 * round + 4 * half + q, row, rows)] : 0.f;
    out[i] = (uint64_t)pack_bf16_rne(v[2], v[3]) << 32 | pack_bf16_rne(v[0], v[1]);
  }
}

constexpr int kResCtlWords = 64, kResMaxGroups = kResCtlWords - 2;

// pre-fill of the hand-over arrays, zero words and counters
__global__ void k_resident_init(ResArgs a) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, n = (size_t)gridDim.x * blockDim.x;
  const uintx4_t e = {kResEmpty, kResEmpty, kResEmpty, kResEmpty};
  for (size_t i = gid; i < res_h_floats(a) / 4; i += n) reinterpret_cast<uintx4_t *>(a.hb)[i] = e;
  for (size_t i = gid; i < res_p_floats(a) / 4; i += n) reinterpret_cast<uintx4_t *>(a.pb)[i] = e;
  for (size_t i = gid; i < res_z_floats(a) / 4; i += n) reinterpret_cast<uintx4_t *>(a.zb)[i] = e;
  for (size_t i = gid; i < res_words(a); i += n) a.words[i] = 0;
  if (gid < kResCtlWords) a.ctl[gid] = 0;
}

constexpr int kResShortSpin = 1000;  // a test's limit: the launch waits, for a microsecond, for one block more than it has

constexpr int kResStallPolls = 4096;  // a test's wait for data that does not come

constexpr size_t kResOwnLds = 256;  // the kernel's own words beside the dynamic ones, at most

// kernels whose loops have known lengths (FULL)
bool whole_width(const rnnt_config_t &c) {
  return c.H == 8 * 8 * kResMaxRounds && (c.pred != RNNT_PRED_LSTM || c.P == 8 * 8 * kResMaxRounds);
}

struct Plan {
  bool ok = false, columns = false;
  int n_groups = 0, stride = 0, n_blocks = 0, nu = 0, n_sel = 0, upc = 0, NT = 0, red_blocks = 0;
  size_t lds = 0;
  std::vector<ResTab> tab;
};

// Who owns what among the n_blocks blocks of a group that do not select.  Every tile goes to the block that has least of
// its kind (the phases of a step follow each other, so what counts is the largest number per block and kind), then least of
// all.  False: they do not fit.
// columns: the blank and duration columns are dealt one by one (see res_fold_one).
bool assign_tiles(const rnnt_config_t &c, int n_blocks, bool columns, std::vector<ResTab> &tab) {
  const bool bf = c.prec == RNNT_BF16_JOINT;
  const int N = c.V + 1 + c.n_durations;
  const bool lstm = c.pred == RNNT_PRED_LSTM;
  const int nR = lstm ? 4 * c.P / 16 : 0, nJ = columns ? c.V / 16 + N - c.V : bf ? (N + 31) / 32 : (N + 15) / 16;
  const int nP = !lstm ? 0 : bf ? c.H / 32 : c.H / 16;
  const int reg_j = bf ? kResRegJ<true> : kResRegJ<false>, max_p = bf ? 1 : kResMaxP;
  tab.assign(n_blocks, ResTab{});
  auto total = [&](const ResTab &t) { return t.nR + t.nJ + t.nP; };
  auto put = [&](int tile, auto count, auto room, auto store) {
    int best = -1;
    for (int i = 0; i < n_blocks; ++i) {
      if (!room(tab[i])) continue;
      if (best < 0 || count(tab[i]) < count(tab[best]) || (count(tab[i]) == count(tab[best]) && total(tab[i]) < total(tab[best])))
        best = i;
    }
    if (best < 0) return false;
    store(tab[best], tile);
    return true;
  };
  for (int t = 0; t < nR; ++t)
    if (!put(t, [](const ResTab &x) { return (int)x.nR; }, [](const ResTab &x) { return x.nR < kResMaxR; },
             [](ResTab &x, int tile) { x.R[x.nR++] = (int16_t)tile; }))
      return false;
  // (the tile with the blank column, or the columns, are dealt first, as a block reads them from its first place where they are
  // folded, and count as two tiles)
  const int blank_tile = c.V / (bf ? 32 : 16), n_first = columns ? N - c.V : 1;
  auto special = [&](const ResTab &x) { return x.nJ > 0 && x.J[0] >= blank_tile && x.J[0] < blank_tile + n_first; };
  for (int i = 0; i < nJ; ++i) {
    const int t = i < n_first ? blank_tile + i : i - n_first < blank_tile ? i - n_first : i;
    if (!put(t, [&](const ResTab &x) { return x.nJ + special(x); }, [&](const ResTab &x) { return i < n_first ? x.nJ == 0 : x.nJ < reg_j + 1; },
             [](ResTab &x, int tile) { x.J[x.nJ++] = (int16_t)tile; }))
      return false;
  }
  for (int t = 0; t < nP; ++t)
    if (!put(t, [](const ResTab &x) { return (int)x.nP; },
             [&](const ResTab &x) { return x.nP < max_p && x.nP + std::max(0, x.nJ - reg_j) < kResMaxLdsTiles; },
             [](ResTab &x, int tile) { x.P[x.nP++] = (int16_t)tile; }))
      return false;
  return true;
}

// Decoders that stay with the per-step launches although they fit the loop: narrow ones, whose per-step launches are short, with
// several tiles of slots or wide beams.  Both sides timed, time of the per-step launches over the loop's.  The lines were drawn while the
// loop's selection took each row's Beam best first; what is given first at each of them is from then.  With the selection of the Beam
// best of all at once the loop is the faster one behind each of them as well, 1.02 to 3.3 times at 273 shapes (V = 29 to 1000, beams 3 to 16),
// as given after "since": they hold back decodes that could take it.
// Not held back, then: split decoders (320 wide and more) 1.01 and more at each of 250 shapes of two and three tiles (to 512 wide, V = 29
// to 1000, beams 5 to 16, LM and TDT among them; means 1.33 in float32, 1.23 with the bf16 joint); 640 wide 1.07 and more.
// Not split, 64 to 256 wide: one tile 1.23 to 1.94, two tiles at beams up to 8 1.24 to 1.52.
bool stays_with_launches(const Resident &r, const rnnt_config_t &c, int B, int K, int n_tiles) {
  const bool bf = c.prec == RNNT_BF16_JOINT;
  // 64 and 128 wide, V = 1000: one utterance 0.95 to 1.08, eight 1.01 to 1.15; 320 wide, bf16, one utterance 1.09 and 1.11.  Since: 1.53 to
  // 3.3
  if (c.pred != RNNT_PRED_LSTM) return K > 8 && (c.H <= 128 || (bf && B == 1 && c.H <= 320));
  if (std::max(c.H, c.P) <= 192) {
    // float32, three tiles: V = 1000 at beams up to 8 1.17 to 1.26; else 0.85 to 1.50, V = 260 at beams above 4 and V = 29 above 1.  Since:
    // 1.08 to 2.25
    if (!bf && n_tiles == 3 && !(c.V > 512 && K <= 8)) return true;
    // two tiles, beams above 8, float32: V = 29 and 260 1.12 to 1.65, V = 500 0.98 to 1.27, V = 1000 1.04 to 1.13;
    // bf16: V = 450 0.97 to 1.84, V > 512 1.00 to 1.34.  Since: float32 1.54 to 2.85, bf16 1.46 to 1.86
    return n_tiles > 1 && K > 8 && c.V > (bf ? 512 : 384);
  }
  // 256 wide, three tiles: V up to 500 at beam 4 0.93 to 0.99, else 0.94 to 1.40.  Since, beams up to 4: 1.02 to 1.18
  return r.form == kResF32 && n_tiles == 3 && K <= 4 && c.V <= 512;
}

Plan make_plan(const Resident &r, const rnnt_config_t &c, int B, int K, bool has_lm, bool fold) {
  Plan p;
  // One group per 32 compute units at most (they hold the weights of a 640-wide decoder), and never more than utterances.
  // Each group is on one XCD (see res_store); the others stay free when there are fewer utterances.  (One utterance of 125 frames
  // on all 256 units, with written-through stores between the XCDs: 9.4 ms, on the 32 of one: 8.6; 7 utterances in 4 groups 7.3,
  // in 7 groups 6.4.)
  p.stride = std::min(std::max(1, r.n_cus / 32), kResMaxGroups);
  const int G = std::min(B, p.stride);
  p.n_groups = G;
  p.n_blocks = r.n_cus / p.stride;
  p.nu = (B + G - 1) / G;
  const int slots = p.nu * K;
  p.NT = (slots + kResSlot - 1) / kResSlot;
  if (p.NT > kResMaxNT) return p;
  // Stateless decoders: one tile of slots, whose last tokens the owners of output-layer tiles keep.  (A form for more, float32, 640 wide, us
  // per step here / there, before hand-overs stayed in the L2: two tiles, batch 16 beam 16 34.8 / 33.3; three, batch 32 beam 12 37.3 / 36.0.
  // It has not been tried since.)
  if (c.pred != RNNT_PRED_LSTM && p.NT > 1) return p;
  if (stays_with_launches(r, c, B, K, p.NT)) return p;
  const bool bf = c.prec == RNNT_BF16_JOINT;
  p.columns = fold && r.form == kResSplit && whole_width(c);
  int most_sel = std::max(1, p.n_blocks / 8);
  p.upc = (p.nu + most_sel - 1) / most_sel;
  if (p.upc > kResMaxSel || p.upc * K > kResMaxHyps) return p;
  p.n_sel = (p.nu + p.upc - 1) / p.upc;
  while (!assign_tiles(c, p.n_blocks - p.n_sel, p.columns, p.tab)) {
    // Columns dealt one by one take more places than the tile that they lie in: with eight durations and V = 1024 one more than 28
    // blocks have (64 + 9 of the output layer, 40 of the projection, 4 in each).  Then fewer blocks select, for more utterances each
    // (ms per decode of 100 frames, here / by the per-step launches: batch 32 beam 8 1.50 / 3.46, beam 12 1.94 / 5.23, batch 113 beam 2 1.54 / 3.56).
    if (!p.columns || --most_sel == 0) return p;
    p.upc = (p.nu + most_sel - 1) / most_sel;
    if (p.upc > kResWaves || p.upc * K > kResMaxHyps) return p;  // (a wave per utterance)
    p.n_sel = (p.nu + p.upc - 1) / p.upc;
  }
  int lds_tiles = 0;
  for (const ResTab &t : p.tab) lds_tiles = std::max(lds_tiles, t.nP + std::max(0, t.nJ - (bf ? kResRegJ<true> : kResRegJ<false>)));
  auto worker_lds = [&](int red_blocks) {
    return (size_t)lds_tiles * (r.form == kResSplit ? kResTileFloats : std::max(c.pred == RNNT_PRED_LSTM ? c.P : 0, c.H) * kResSlot) * 4 +
           (bf && fold ? (size_t)(1 + c.n_durations) * c.H * 2 : 0) + (size_t)2 * red_blocks * kResRedBlock * 4 +
           (size_t)kResMaxR * p.NT * (256 + 128) * 4 + ResPar::kFloats * 4 + (size_t)p.NT * kResSlot * (sizeof(int2) + kResWaves * 8) +
           (c.pred == RNNT_PRED_LSTM ? 0 : (size_t)kResWaves * kResSlot * kResPreSlot * (bf ? 2 : 4));
  };
  // (640 wide: with one tile of slots)
  p.red_blocks = bf ? kResRedBlocks<true> : kResRedBlocks<false>;
  if (r.form == kResSplit && worker_lds(4) + kResOwnLds <= (size_t)r.max_lds) p.red_blocks = 4;
  const size_t worker = worker_lds(p.red_blocks);
  const size_t sel = (res_sel_floats(p.upc, p.NT) + (size_t)p.upc * K * res_row_floats(c.V)) * 4;
  p.lds = std::max(worker, sel);
  p.lds = std::max<size_t>(p.lds, 84 * 1024);  // more than half of a compute unit's: two blocks never share one
  if (p.lds + kResOwnLds > (size_t)r.max_lds) return p;
  p.ok = true;
  return p;
}

template <bool FULL, bool ST>
ResKernel pick_form(int form, int K, bool plain) {
  return form == kResSplit ? resident_kernel<FULL, kResSplit, ST>(K, plain)
         : form == kResBf16 ? resident_kernel<FULL, kResBf16, ST>(K, plain) : resident_kernel<FULL, kResF32, ST>(K, plain);
}
template <bool ST>
ResKernel pick_kernel(const rnnt_config_t &c, int form, int K, bool plain) {
  return whole_width(c) ? pick_form<true, ST>(form, K, plain) : pick_form<false, ST>(form, K, plain);
}

}  // namespace

void resident_destroy(Resident &r) {
  for (void *p : r.allocs) hipFree(p);
  if (r.h_abort) hipHostFree(r.h_abort);
  r = Resident{};
}

int resident_create(Resident &r, const rnnt_config_t &c, const ResidentWeights &w, std::string &err, int fail_alloc) {
  r.usable = false;
  // decoders whose contractions split into eight slices of whole rounds and fit the registers (stateless ones: P is not
  // that of a contraction); vocabularies that one wave holds in registers
  const bool lstm = c.pred == RNNT_PRED_LSTM;
  const int most = 8 * 8 * kResMaxRounds;
  if (c.tdt_all_pairs || c.H % 64 || c.H > most || (lstm && (c.P % 64 || c.P > most)) || c.V > kResMaxV) return RNNT_OK;
  hipError_t e;
  auto fail = [&](const char *what) {
    err = std::string(what) + ": " + hipGetErrorString(e);
    resident_destroy(r);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();  // (handled: no later check is to find it)
      return RNNT_OK;
    }
    return RNNT_E_HIP;
  };
  int dev = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return fail("hipGetDevice");
  if ((e = hipDeviceGetAttribute(&r.n_cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return fail("CU count");
  if ((e = hipDeviceGetAttribute(&r.max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev)) != hipSuccess) return fail("LDS size");
  if (r.n_cus < 32) return RNNT_OK;
  const bool bf = c.prec == RNNT_BF16_JOINT;
  const int N = c.V + 1 + c.n_durations, G = r.n_cus / 32;
  const size_t rows = (size_t)G * kResMaxNT * kResSlot;
  auto alloc = [&](auto **p, size_t n) {
    void *q = nullptr;
    e = fail_alloc == (int)r.allocs.size() ? hipErrorOutOfMemory : hipMalloc(&q, n * sizeof(**p));
    if (e == hipSuccess) {
      r.allocs.push_back(q);
      *p = static_cast<std::remove_reference_t<decltype(*p)>>(q);
    }
    return e == hipSuccess;
  };
  const int nR = 4 * c.P / 16, nJ = bf ? (N + 31) / 32 : (N + 15) / 16, nP = bf ? c.H / 32 : c.H / 16;
  constexpr size_t kTileWords = kResTileFloats;
  const bool split = w.split;
  r.form = bf ? kResBf16 : split ? kResSplit : kResF32;
  bool ok = bf ? alloc(&r.WJb, (size_t)nJ * (c.H / 8) * 64)
               : (split ? alloc(&r.WJ, nJ * kTileWords) : alloc(&r.WJf, (size_t)nJ * 16 * c.H)) && alloc(&r.WJs, (size_t)16 * c.H);
  if (lstm) {
    ok = ok && (split ? alloc(&r.WR, nR * kTileWords) : alloc(&r.WRf, (size_t)nR * 16 * c.P)) && alloc(&r.hb, kResStepRing * rows * c.P) && alloc(&r.pb, kResStepRing * rows * c.H);
    ok = ok && (bf      ? alloc(&r.WPb, (size_t)nP * (c.P / 8) * 64)
                : split ? alloc(&r.WP[0], nP * kTileWords) && (c.P % 128 || alloc(&r.WP[1], nP * kTileWords))
                        : alloc(&r.WPf, (size_t)nP * 16 * c.P));
  }
  ok = ok && alloc(&r.zb, kResStepRing * rows * w.out_rows) &&
       alloc(&r.words, (size_t)kResStepRing * G * kResWordCopies * kResWordPlace) && alloc(&r.ctl, kResCtlWords) && alloc(&r.tab, r.n_cus);
  if (!ok) return fail("resident loop: hipMalloc");
  if ((e = hipHostMalloc(reinterpret_cast<void **>(&r.h_abort), 128, hipHostMallocMapped)) != hipSuccess) return fail("hipHostMalloc");
  if ((e = hipHostGetDevicePointer(reinterpret_cast<void **>(&r.h_abort_dev), r.h_abort, 0)) != hipSuccess) return fail("pinned word");
  const dim3 grid(512), block(256);
  if (bf) hipLaunchKernelGGL(k_pack_bf16<0>, grid, block, 0, nullptr, w.W_out, w.out_rows, c.H, nJ, r.WJb);
  else {
    if (split) hipLaunchKernelGGL(k_pack_split<0>, grid, block, 0, nullptr, reinterpret_cast<const uint32_t *>(w.W_out_s), w.out_rows, c.H, nJ, false, r.WJ);
    else hipLaunchKernelGGL(k_pack_f32<0>, grid, block, 0, nullptr, w.W_out, w.out_rows, c.H, nJ, r.WJf);
    r.out_unscale = w.out_unscale;
    hipLaunchKernelGGL(k_pack_fold, grid, block, 0, nullptr, w.W_out, w.out_rows, c.V / 16 * 16, c.H, r.WJs);
  }
  if (lstm) {
    if (!split) hipLaunchKernelGGL(k_pack_f32<1>, grid, block, 0, nullptr, w.W_hh, 4 * c.P, c.P, nR, r.WRf);
    else hipLaunchKernelGGL(k_pack_split<1>, grid, block, 0, nullptr, reinterpret_cast<const uint32_t *>(w.W_hh), 4 * c.P, c.P, nR, false, r.WR);
    r.hh_unscale = w.hh_unscale;
    if (bf) hipLaunchKernelGGL(k_pack_bf16<2>, grid, block, 0, nullptr, w.W_pred, c.H, c.P, nP, r.WPb);
    else if (!split) hipLaunchKernelGGL(k_pack_f32<2>, grid, block, 0, nullptr, w.W_pred, c.H, c.P, nP, r.WPf);
    else {
      for (int halves = 0; halves < 2; ++halves)
        if (r.WP[halves])
          hipLaunchKernelGGL(k_pack_split<2>, grid, block, 0, nullptr, reinterpret_cast<const uint32_t *>(w.W_pred), c.H, c.P, nP, halves != 0,
                             r.WP[halves]);
      r.pred_unscale = w.pred_unscale;
    }
  }
  if ((e = hipGetLastError()) != hipSuccess || (e = hipDeviceSynchronize()) != hipSuccess) return fail("resident loop: packing");
  r.usable = true;
  return RNNT_OK;
}

bool resident_fits(const Resident &r, const rnnt_config_t &c, int B, int K, int T, int max_steps, bool has_lm, bool fold) {
  if (!r.usable) return false;
  if (T >= kWordMaxFrames || max_steps > 60000) return false;  // fields of the words
  return make_plan(r, c, B, K, has_lm, fold).ok;
}

hipError_t resident_launch(Resident &r, const rnnt_config_t &c, const ResidentBatch &b, hipStream_t s) {
  Plan p = make_plan(r, c, b.B, b.K, b.has_lm, b.fold);
  if (!p.ok) return hipErrorInvalidValue;
  ResArgs a{};
  a.WR = reinterpret_cast<const uintx4_t *>(r.WR); a.WJ = reinterpret_cast<const uintx4_t *>(r.WJ);
  a.WP = reinterpret_cast<const uintx4_t *>(r.WP[b.halves ? 1 : 0]);
  a.hh_unscale = r.hh_unscale; a.out_unscale = r.out_unscale; a.pred_unscale = r.pred_unscale; a.WRf = r.WRf; a.WJf = r.WJf; a.WPf = r.WPf; a.WJs = r.WJs; a.WJb = r.WJb; a.WPb = r.WPb;
  a.emb_tab = b.emb_tab; a.n_ctx = b.n_ctx;
  a.b_out = b.b_out; a.b_pred = b.b_pred; a.G = b.G; a.f_proj = b.f_proj;
  a.lengths = b.lengths;
  a.hb = r.hb; a.pb = r.pb; a.zb = r.zb; a.words = r.words;
  a.tab = r.tab;
  a.ctl = r.ctl;
  a.h_abort = r.h_abort_dev;
  a.sel = b.sel;
  a.lm = b.lm;
  a.B = b.B; a.K = b.K; a.T = b.T; a.V = c.V; a.N = c.V + 1 + c.n_durations; a.Npad = b.Npad; a.H = c.H; a.P = c.P;
  a.n_groups = p.n_groups; a.stride = p.stride; a.n_sel = p.n_sel; a.upc = p.upc;
  a.NT = p.NT; a.red_blocks = p.red_blocks; a.halves = b.halves ? 1 : 0; a.has_lm = b.has_lm ? 1 : 0;
  a.rounds_h = c.H / 64; a.rounds_p = c.P / 64;
  a.fold = b.fold ? 1 : 0;
  a.stall_step = b.stall_step;
  a.poll_limit = std::min(b.stall_step < 0 ? 1 << 19 : kResStallPolls, b.spin_limit);
  const bool short_spin = b.spin_limit < kResShortSpin;
  r.n_groups = p.n_groups;
  r.last_stall_step = b.stall_step;
  a.start_blocks = p.n_groups * p.n_blocks + (short_spin ? 1 : 0);
  a.start_limit = short_spin ? 100 : 5000000;  // 50 ms
  *reinterpret_cast<volatile int *>(r.h_abort) = 0;
  hipError_t e = hipSuccess;
  if (r.tab_blocks != p.n_blocks || r.tab_sel != p.n_sel || r.tab_columns != p.columns) {
    // (pageable memory: the call returns when it has been read; the last launch that read the table is over, as its
    // decode waited for it)
    e = hipMemcpyAsync(r.tab, p.tab.data(), sizeof(ResTab) * p.tab.size(), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    r.tab_blocks = p.n_blocks;
    r.tab_sel = p.n_sel;
    r.tab_columns = p.columns;
  }
  hipLaunchKernelGGL(k_resident_init, dim3(512), dim3(256), 0, s, a);
  const bool plain = c.n_durations == 0 && !b.has_lm && b.algo == RNNT_ALSD;
  ResKernel k = b.emb_tab ? pick_kernel<true>(c, r.form, b.K, plain) : pick_kernel<false>(c, r.form, b.K, plain);
  e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(p.stride * p.n_blocks), dim3(kResThreads), p.lds, s, a);
  return hipGetLastError();
}

hipError_t resident_local_groups(const Resident &r, int *groups, int *local) {
  int words[kResCtlWords];
  *groups = r.n_groups;
  *local = 0;
  if (r.n_groups == 0) return hipSuccess;
  const hipError_t e = hipMemcpy(words, r.ctl, sizeof words, hipMemcpyDeviceToHost);
  for (int g = 0; e == hipSuccess && g < r.n_groups; ++g) *local += res_on_one_xcd(words[2 + g], r.last_stall_step);
  return e;
}

}  // namespace rb
