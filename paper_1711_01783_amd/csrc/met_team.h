// Interface of the team decoder (met_team.hip) to the other entry points.
#pragma once

#include <hip/hip_runtime.h>

#include "met_internal.h"

namespace met {

constexpr int kTeamSlots = 8;  // groups in work at once, at most: one per XCD

struct TeamClass {
  int32_t shape, tile0, first_check, n_checks, first_msg, first_leaf;
};

// One decode, passed to the kernel by value.
struct TeamJob {
  const int32_t *edge_msgvn, *vn_ptr, *vn_edges, *msg_vn_user, *leaf_vn, *vn_slot, *chk_msg_ptr, *chk_leaf_ptr,
      *chk_pos;
  int64_t N;
  int32_t M, N2, EL;
  int32_t B, G, max_iter, early;
  const float *llr;
  const uint8_t *syn;
  uint8_t *bits;
  int32_t *iters;
  uint8_t *converged;
  float *posterior;
  char *ws;               // control words, then the slots
  size_t off_slots;
  // offsets of a slot's arrays in bytes (c2v at 0); an array ends where the next begins
  uint32_t off_P, off_L2, off_Lphi, off_Lraw, off_P1, off_syn, off_B1, slot_bytes;
  int32_t n_slots, expected, lanes_per_vn;
  int32_t dies;           // workgroups on an XCD of this number or above take no part
  uint32_t late_ticks;    // delays of workgroups (tests), in ticks of 10 ns
  uint32_t poll_limit;    // polls after which a workgroup gives up waiting for its team
  int32_t n_classes, check_tiles;
  TeamClass cls[kMaxClasses];
};

// Bytes of one group's state; fills the offsets of *job if given.
size_t team_slot(const met_code *c, int W, bool post, size_t c2v_bytes, TeamJob *job);

// Bytes ahead of the slots in the workspace.
size_t team_control_bytes();

// *width: frames per group with which the team decoder takes this decode, or 0
// where the per-phase launches are the better path or the workspace is too small.
int team_width(const met_code *c, int B, bool post, size_t c2v_bytes, bool lut, int max_iter, bool early,
               size_t ws_bytes, int *width);

// Bytes of workspace with which team_width is free in its choice.
size_t team_bytes(const met_code *c, int B, bool post, size_t c2v_bytes);

// Whether the teams' states in groups of W frames fit in a workspace.
bool team_fits(const met_code *c, int B, bool post, size_t c2v_bytes, int W, size_t ws_bytes);

int team_decode(const met_code *c, const DeviceCode *d, int W, const float *llr, const uint8_t *syn, int B,
                int max_iter, uint32_t flags, uint8_t *bits, int32_t *iters, uint8_t *conv, float *post,
                char *ws, hipStream_t st, const met_team_options *opt = nullptr);

}  // namespace met
