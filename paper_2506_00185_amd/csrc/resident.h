// Host side of the resident step loop (kernels_resident.h): weights in its layout, plan per batch shape, launch.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <string>
#include <vector>

#include "../../include/rnnt_beam.h"
#include "lm_device.h"
#include "select.h"

namespace rb {

struct ResTab;

// Per-handle state: owned by the handle, everything on the device it was created on.
struct Resident {
  bool usable = false;
  int n_cus = 0, max_lds = 0;
  int misses = 0, skip = 0;       // launches in a row that gave up; decodes left to the per-step launches before the next try
  int form = 0;                   // ResForm
  const float *hh_unscale = nullptr, *out_unscale = nullptr, *pred_unscale = nullptr;  // the handle's
  uint32_t *WR = nullptr, *WJ = nullptr, *WP[2] = {nullptr, nullptr};  // see k_pack_split
  float *WRf = nullptr, *WJf = nullptr, *WPf = nullptr, *WJs = nullptr;
  uint64_t *WJb = nullptr, *WPb = nullptr;
  float *hb = nullptr, *pb = nullptr, *zb = nullptr;
  uint64_t *words = nullptr;
  int *ctl = nullptr;
  ResTab *tab = nullptr;          // who owns what in a group, as uploaded for the last launch:
  int tab_blocks = 0, tab_sel = 0;
  bool tab_columns = false;
  int n_groups = 0, last_stall_step = -1;  // of the last launch
  int *h_abort = nullptr, *h_abort_dev = nullptr;  // pinned
  std::vector<void *> allocs;
};
// A launch that gives up costs the decode up to 50 ms, several decodes' time: after the n-th in a row the next 4, 8, 16, ..
// 256 decodes of the handle use the per-step launches.  One that succeeds starts the count anew.
constexpr int kResidentSkip = 4, kResidentMaxSkip = 256;
inline void resident_missed(Resident &r) {
  r.skip = kResidentSkip << r.misses;
  if (r.skip >= kResidentMaxSkip) r.skip = kResidentMaxSkip;
  else ++r.misses;
}

// What the packing reads: the handle's k4-major weights (see kernels.h, k4_index)
struct ResidentWeights {
  // split: W_hh, W_out_s and W_pred are (k_split_rows), the output layer is there as it is as well
  bool split;
  const float *W_hh, *hh_unscale, *W_out, *W_out_s, *out_unscale, *W_pred, *pred_unscale;
  int out_rows;  // padded rows of W_out
};

// RNNT_OK with r.usable == false: the decoder does not fit the loop, or its second copy of the weights finds no memory (the
// per-step launches do without it).  fail_alloc: a test's, the allocation that is taken to fail (-1: none).
int resident_create(Resident &r, const rnnt_config_t &c, const ResidentWeights &w, std::string &err, int fail_alloc = -1);
void resident_destroy(Resident &r);

struct ResidentBatch {
  int B, T, K, algo, spin_limit;
  int stall_step;   // see ResArgs
  bool halves;      // the per-step launches would split the projection along k at this size
  bool fold;        // they would fold the blank and duration columns into the token columns' blocks
  const float *b_out, *b_pred, *G, *f_proj;
  const float *emb_tab;  // stateless decoders (see ResArgs), else null
  int n_ctx;
  const int *lengths;
  int Npad;
  bool has_lm;
  LmView lm;
  SelectArgs sel;   // n_chunks = 1
};
// whether a batch of this shape can run as one resident launch
bool resident_fits(const Resident &r, const rnnt_config_t &c, int B, int K, int T, int max_steps, bool has_lm, bool fold);
// groups of the last launch, and how many of them handed over through the L2 of one XCD; waits for the device
hipError_t resident_local_groups(const Resident &r, int *groups, int *local);
hipError_t resident_launch(Resident &r, const rnnt_config_t &c, const ResidentBatch &b, hipStream_t s);

}  // namespace rb
