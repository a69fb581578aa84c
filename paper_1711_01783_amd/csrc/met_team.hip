// Decoding in teams: one launch decodes a whole batch, each frame group by the
// workgroups of one accelerator die (XCD).
//
// Frames are independent, so a batch of B frames is cut into small groups of W
// frames and each group is decoded from set-up to outputs by one team: the
// workgroups that run on one XCD.  A group's state (messages, posteriors, leaf
// inputs) lives in that die's L2, the phases of an iteration (Methods, Steps
// 3-5: check update, variable update) are separated by a barrier among the
// team's workgroups alone, and a team whose frames have all stopped takes the
// next group.  No launch, host round trip or device-wide barrier remains
// inside a decode, and a frame that needs many iterations holds up only the
// few frames of its group.  Teams take every group, their first one too, from
// one counter, so that however many teams form (a partitioned device shows
// fewer dies) all groups are decoded.
//
// Coherence inside a team.  All workgroups of a team share one L2, so data
// written by one is visible to the others once its stores are acknowledged
// (vmcnt(0)) if the readers bypass their own first-level cache: loads of words
// that other workgroups write carry the sc1 (device scope) bit, which this
// cache does not serve and the L2 does.  No cache is flushed or invalidated (an
// acquire fence costs 1.8 us for each wave that issues it).  The barrier is one
// store and a poll of all members' flags: 0.46 us for 32 workgroups.
//
// Forming teams.  A workgroup reads the number of its XCD and registers with
// that XCD's counter.  The first to register waits until the expected number
// has arrived, or 20 us; the team is who has registered by then.  Where other
// work holds compute units at that moment, it is joined by those that come
// later: the first member admits them at the end of an iteration, and hands
// them the state of the decode.  Nobody ever waits for a workgroup that is not
// running, so concurrent launches on other streams or in other processes cannot
// block each other; they only make teams smaller while they run.  (Teams that
// kept their first size: one frame of N = 65536 beside 64-frame decodes of
// N = 300000 ran up to 11 ms, against 0.66 ms in the median.)
//
// The arithmetic is that of met_gpu.h's kernels, operation by operation, so
// the results equal the per-phase launches' bit for bit.
#include <cmath>

#include "met_gpu.h"
#include "met_team.h"

namespace met {
namespace {

constexpr int kTeamBlock = 1024;
constexpr int kTeamWaves = kTeamBlock / 64;
constexpr int kMaxTeam = 64;            // workgroups of one team
constexpr uint32_t kEnded = 0x80000000u;
constexpr uint64_t kFormTicks = 2000;   // 20 us of the 100 MHz counter
constexpr uint32_t kPollLimit = 1u << 22;  // polls of about 0.4 us (TeamJob::poll_limit)

// Control words at the start of the workspace, cleared before the launch.
struct TeamControl {
  uint64_t taken, pad0[15];             // groups taken, and slots in the high word
  struct {
    uint32_t count, pad0[31];
    uint64_t pub, pad1[15];             // members + 256 (slot + 1) + 65536 group, set once
    uint32_t grown, pad2[31];           // members with those admitted since, or kEnded
    uint32_t state[5], stop[16], pad3[11];  // for those: epoch, group, iteration, frames that run, last
  } reg[kTeamSlots];
  uint64_t flag[kTeamSlots][2][kMaxTeam];  // epoch in the low word, payload in the high one
};

// Outcome (iterations) of frames that no team has taken, and of those whose team
// gave up.
constexpr int32_t kUntaken = -1, kGivenUp = -2;
constexpr int32_t kSatisfied = 1 << 30;  // in TeamShared::stop

__global__ __launch_bounds__(kTeamBlock) void k_team_clear(uint32_t *ctl, int32_t *iters, uint8_t *converged,
                                                           int32_t B) {
  for (size_t i = threadIdx.x; i < sizeof(TeamControl) / 4; i += kTeamBlock) ctl[i] = 0u;
  for (int32_t f = threadIdx.x; f < B; f += kTeamBlock) {
    iters[f] = kUntaken;
    converged[f] = 0;
  }
}

// ---- Memory -----------------------------------------------------------------
// State arrays are addressed as buffers: a descriptor in scalar registers and a
// 32-bit byte offset per lane; reads past the end return 0.

using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr int kSc1 = 16;                 // cache policy bit of the buffer instructions
// Offsets past the end of every array, also after the scaling of element
// numbers to bytes (1, 2 or 4 per element); kMaxSlotBytes keeps arrays below.
constexpr uint32_t kNowhere = 0xFFFFFFF0u;
constexpr size_t kMaxTeamBytes = 192u << 20;  // states of all slots: within the Infinity Cache
constexpr size_t kMaxSlotBytes = kNowhere / 4u - 1024u;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ rsrc_t buffer_of(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

template <int F, int AUX>
__device__ __forceinline__ void ld_f32(rsrc_t r, uint32_t off, float (&v)[F]) {
  if constexpr (F == 4) {
    const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX);
#pragma unroll
    for (int f = 0; f < 4; ++f) v[f] = __uint_as_float(t[f]);
  } else if constexpr (F == 2) {
    const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
    v[0] = __uint_as_float(t[0]);
    v[1] = __uint_as_float(t[1]);
  } else {
    v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, AUX));
  }
}

template <int F>
__device__ __forceinline__ void st_f32(rsrc_t r, uint32_t off, const float (&v)[F]) {
  if constexpr (F == 4) {
    u32x4 t;
#pragma unroll
    for (int f = 0; f < 4; ++f) t[f] = __float_as_uint(v[f]);
    __builtin_amdgcn_raw_buffer_store_b128(t, r, off, 0, 0);
  } else if constexpr (F == 2) {
    u32x2 t;
    t[0] = __float_as_uint(v[0]);
    t[1] = __float_as_uint(v[1]);
    __builtin_amdgcn_raw_buffer_store_b64(t, r, off, 0, 0);
  } else {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[0]), r, off, 0, 0);
  }
}

// Tables of the 8-bit storage in LDS.
struct Tables {
  const float *q8;       // [128] grid values
  const float *phi;      // [kLutSize] (table-driven check update)
  const uint8_t *code;   // [kLutSize]
};

__device__ __forceinline__ float q8_value(uint32_t c, const Tables &tab) {
  const float m = tab.q8[c & 127u];
  return (c & 128u) ? -m : m;
}

// F messages of storage type CT; F > 1 reads one aligned word.
template <int F, typename CT, int AUX>
__device__ __forceinline__ void ld_msgs(rsrc_t r, uint32_t elem, const Tables &tab, float (&v)[F]) {
  if constexpr (std::is_same<CT, float>::value) {
    ld_f32<F, AUX>(r, elem * 4u, v);
  } else if constexpr (std::is_same<CT, half_t>::value) {
    static_assert(F == 4 || F == 1, "half rows are read by one or four frames");
    if constexpr (F == 4) {
      const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(r, elem * 2u, 0, AUX);
#pragma unroll
      for (int f = 0; f < 4; ++f)
        v[f] = (float)__builtin_bit_cast(half_t, (uint16_t)(t[f / 2] >> (16 * (f & 1))));
    } else {
      v[0] = (float)__builtin_bit_cast(half_t, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, elem * 2u, 0, AUX));
    }
  } else {
    static_assert(F == 4 || F == 1, "8-bit rows are read by one or four frames");
    if constexpr (F == 4) {
      const uint32_t t = __builtin_amdgcn_raw_buffer_load_b32(r, elem, 0, AUX);
#pragma unroll
      for (int f = 0; f < 4; ++f) v[f] = q8_value(t >> (8 * f), tab);
    } else {
      v[0] = q8_value((uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, elem, 0, AUX), tab);
    }
  }
}

template <int F, typename CT>
__device__ __forceinline__ void st_msgs(rsrc_t r, uint32_t elem, const float (&v)[F]) {
  if constexpr (std::is_same<CT, float>::value) {
    st_f32<F>(r, elem * 4u, v);
  } else if constexpr (std::is_same<CT, half_t>::value) {
    uint16_t h[F];
#pragma unroll
    for (int f = 0; f < F; ++f) h[f] = __builtin_bit_cast(uint16_t, (half_t)v[f]);
    if constexpr (F == 4) {
      u32x2 t;
      t[0] = h[0] | ((uint32_t)h[1] << 16);
      t[1] = h[2] | ((uint32_t)h[3] << 16);
      __builtin_amdgcn_raw_buffer_store_b64(t, r, elem * 2u, 0, 0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b16(h[0], r, elem * 2u, 0, 0);
    }
  } else {
    uint32_t t = 0;
#pragma unroll
    for (int f = 0; f < F; ++f) t |= q8_encode(v[f]) << (8 * f);
    if constexpr (F == 4)
      __builtin_amdgcn_raw_buffer_store_b32(t, r, elem, 0, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b8((uint8_t)t, r, elem, 0, 0);
  }
}

// ---- One group's work ---------------------------------------------------------

// Lanes of a wave in the check phase: an item (check) takes W / F lanes, each of
// which holds F frames in registers, so that an index is read once for F frames
// and rows are read as whole words.
template <int W>
constexpr int kFramesPerLane = W < 4 ? W : 4;

struct GroupState {
  const TeamJob *job;
  char *base;
  rsrc_t c2v, P, L2, Lphi, syn, B1;
  uint32_t b1_half;  // bytes of one of the two buffers of B1
  // arrays of decodes with posterior output
  __device__ rsrc_t Lraw() const { return buffer_of(base + job->off_Lraw, job->off_P1 - job->off_Lraw); }
  __device__ rsrc_t P1(int it) const {
    const uint32_t half = (job->off_syn - job->off_P1) / 2;
    return buffer_of(base + job->off_P1 + ((it & 1) ? half : 0u), half);
  }
};

// The frames named by `lanes`, a mask over lanes of which each holds frames
// FL (lane % (W / FL)) + f of its check.
template <int W, int FL>
__device__ __forceinline__ uint32_t frames_of(const uint64_t (&lanes)[FL]) {
  constexpr int LPI = W / FL;
  uint32_t word = 0;
#pragma unroll
  for (int f = 0; f < FL; ++f)
#pragma unroll
    for (int wl = 0; wl < LPI; ++wl) {
      uint64_t those = 0;
#pragma unroll
      for (int l = wl; l < 64; l += LPI) those |= 1ull << l;
      word |= (lanes[f] & those) ? 1u << (wl * FL + f) : 0u;
    }
  return word;
}

// What a phase does besides the message update.
struct Phase {
  bool first;   // iteration 1: P = L, c2v = 0
  bool test;    // syndrome test of the previous iteration
  bool decide;  // leaf decisions of this iteration are needed
  bool post;    // leaf posteriors of this iteration are needed
  int it;
  uint32_t act; // frames of the group that run
};

// Wide checks take one lane per frame (a tile of them would otherwise be the
// longest chain of a phase), narrow ones kFramesPerLane frames per lane.
template <int W, int NM, int NL, typename CT>
__device__ __forceinline__ void check_tile(const GroupState &s, const int32_t *edge_msgvn, const TeamClass &c,
                                           uint32_t tile, const Phase &ph, const Tables &tab, uint32_t &unsat) {
  constexpr int F = NM > 4 ? 1 : kFramesPerLane<W>, LPI = W / F, D = NM + NL;
  constexpr int FW = kFramesPerLane<W>, WPI = W / FW;  // decisions and syndrome bits: WPI bytes of FW bits
  static_assert(NL == 0 || F == FW, "a lane owns whole bytes of decisions");
  constexpr bool lut = std::is_same<CT, q8lut_t>::value;
  const uint32_t lane = threadIdx.x & 63, wl = lane % LPI;
  const uint32_t i = tile * (64 / LPI) + lane / LPI;
  const bool valid = i < (uint32_t)c.n_checks;
  const uint32_t item = valid ? i : 0u;
  const uint32_t m0 = (uint32_t)c.first_msg + item * NM, l0 = (uint32_t)c.first_leaf + item * NL;
  const uint32_t chk = (uint32_t)c.first_check + item;
  // the class's messages lie plane by plane (edge m of every check together),
  // so that a wave's rows are contiguous: rows of 16 bytes at a stride of 48
  // were stored at the rate of scattered ones (1.9 ns per row and CU)
  const uint32_t p0 = (uint32_t)c.first_msg + item;
  const bool partial = ph.act != (uint32_t)wmask<W>();
  const uint32_t b1_in = ((ph.it - 1) & 1) ? s.b1_half : 0u, b1_out = (ph.it & 1) ? s.b1_half : 0u;
  float x[NM][F], cv[NM][F], lf[NL > 0 ? NL : 1][F];
  uint32_t b1[NL > 0 ? NL : 1], old[NL > 0 ? NL : 1];
  uint32_t vi[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) vi[m] = (uint32_t)edge_msgvn[m0 + m];
  uint32_t sb = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.syn, chk * WPI + wl * F / FW, 0, kSc1);
#pragma unroll
  for (int m = 0; m < NM; ++m) ld_f32<F, kSc1>(ph.first ? s.L2 : s.P, (vi[m] * W + wl * F) * 4u, x[m]);
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    // this thread's own words of the previous iteration
    if (!ph.first) {
      ld_msgs<F, CT, 0>(s.c2v, (p0 + m * (uint32_t)c.n_checks) * W + wl * F, tab, cv[m]);
    } else {
#pragma unroll
      for (int f = 0; f < F; ++f) cv[m][f] = 0.0f;
    }
  }
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    ld_f32<F, kSc1>(s.Lphi, ((l0 + l) * W + wl * F) * 4u, lf[l]);
    b1[l] = ph.test ? (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.B1, b1_in + (l0 + l) * WPI + wl, 0, kSc1) : 0u;
    old[l] = ph.decide && partial
                 ? (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.B1, b1_out + (l0 + l) * WPI + wl, 0, kSc1)
                 : 0u;
  }
  if constexpr (F != FW) sb >>= wl % FW;
  const uint64_t mvalid = __ballot(valid);
  uint32_t tb = sb;  // parity of the syndrome bit and the leaf decisions
#pragma unroll
  for (int l = 0; l < NL; ++l) tb ^= b1[l];
  // Signs, parities and decisions are lane masks in scalar registers (one
  // vector compare each, the logic on the scalar unit).
  uint64_t bad[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    bad[f] = __ballot(tb & (1u << f));
#pragma unroll
    for (int m = 0; m < NM; ++m) bad[f] ^= __ballot(x[m][f] < 0.0f);
    bad[f] &= mvalid;
  }
  if (ph.test) unsat |= frames_of<W, F>(bad);
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int f = 0; f < F; ++f) x[m][f] = clamp_llr(x[m][f] - cv[m][f]);
  uint32_t dec[NL > 0 ? NL : 1], code[NM];
  float Sl[NL > 0 ? NL : 1][F];  // phi-domain sum of a leaf's message, with that message's sign
#pragma unroll
  for (int l = 0; l < NL; ++l) dec[l] = 0;
#pragma unroll
  for (int m = 0; m < NM; ++m) code[m] = 0;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    float A[D];
    uint32_t sg[D], tot = sb << (31 - f);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if constexpr (lut)
        A[m] = tab.phi[lut_index(fabsf(x[m][f]))];
      else
        A[m] = phi(fabsf(x[m][f]));
      sg[m] = __float_as_uint(x[m][f]);
      tot ^= sg[m];
    }
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      A[NM + l] = fabsf(lf[l][f]);
      sg[NM + l] = __float_as_uint(lf[l][f]);
      tot ^= sg[NM + l];
    }
    // leave-one-out sums by prefix and suffix sums, as check_fixed_body
    float pre[D], suf[D], S[D];
    pre[1] = A[0];
#pragma unroll
    for (int m = 2; m < D; ++m) pre[m] = pre[m - 1] + A[m - 1];
    suf[D - 2] = A[D - 1];
#pragma unroll
    for (int m = D - 3; m >= 0; --m) suf[m] = suf[m + 1] + A[m + 1];
    S[0] = suf[0];
    S[D - 1] = pre[D - 1];
#pragma unroll
    for (int m = 1; m < D - 1; ++m) S[m] = pre[m] + suf[m];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if constexpr (lut) {
        code[m] |= (tab.code[lut_index(S[m])] | (((tot ^ sg[m]) >> 24) & 128u)) << (8 * f);
      } else {
        const uint32_t mag = __float_as_uint(phi(S[m]));
        x[m][f] = __uint_as_float(mag | ((tot ^ sg[m]) & 0x80000000u));
      }
    }
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      // leaf_bit on masks: where the message agrees with the LLR's sign the
      // decision is that sign, unless both are zero; otherwise the larger one
      // decides, a tie 0
      const float S1 = S[NM + l], A1 = A[NM + l];
      const uint64_t mt = __ballot((int32_t)tot < 0), ml = __ballot((int32_t)sg[NM + l] < 0);
      const uint64_t lt = __ballot(S1 < A1), gt = __ballot(S1 > A1), inf = __ballot(A1 == __builtin_huge_valf());
      const uint64_t bits = (~mt & ml & (lt | ~inf)) | (mt & ((lt & ~ml) | (gt & ml)));
      dec[l] |= __builtin_amdgcn_inverse_ballot_w64(bits) ? 1u << f : 0u;
      Sl[l][f] = __uint_as_float(__float_as_uint(S1) | ((tot ^ sg[NM + l]) & 0x80000000u));
    }
  }
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const uint32_t elem = (p0 + m * (uint32_t)c.n_checks) * W + wl * F;
    if (!valid) continue;
    if constexpr (!lut)
      st_msgs<F, CT>(s.c2v, elem, x[m]);
    else if constexpr (F == 4)
      __builtin_amdgcn_raw_buffer_store_b32(code[m], s.c2v, elem, 0, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b8((uint8_t)code[m], s.c2v, elem, 0, 0);
  }
  if (NL > 0 && ph.decide && valid) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const uint32_t own = (ph.act >> (wl * F)) & ((1u << F) - 1u);
      __builtin_amdgcn_raw_buffer_store_b8((uint8_t)((old[l] & ~own) | (dec[l] & own)), s.B1,
                                           b1_out + (l0 + l) * WPI + wl, 0, 0);
      if (ph.post) {
        float lr[F], p1[F];
        const uint32_t off = ((l0 + l) * W + wl * F) * 4u;
        ld_f32<F, kSc1>(s.Lraw(), off, lr);
        ld_f32<F, kSc1>(s.P1(ph.it), off, p1);
#pragma unroll
        for (int f = 0; f < F; ++f)
          if ((own >> f) & 1u) p1[f] = lr[f] + 1.0f * copysignf(phi(fabsf(Sl[l][f])), Sl[l][f]);
        st_f32<F>(s.P1(ph.it), off, p1);
      }
    }
  }
}

// Run-time degrees, one lane per frame.  A check's inputs are formed once, U
// message rows at a time, and kept with their suffix sums in private memory:
// arrays of the largest degree in registers would set the whole kernel's
// register count.
template <int W, typename CT>
__device__ __forceinline__ void check_tile_generic(const GroupState &s, const TeamJob &job, const TeamClass &c,
                                                   uint32_t tile, const Phase &ph, const Tables &tab,
                                                   uint32_t &unsat) {
  constexpr int FW = kFramesPerLane<W>, WPI = W / FW, U = 8;
  const uint32_t lane = threadIdx.x & 63, w = lane % W;
  const uint32_t i = tile * (64 / W) + lane / W;
  const bool valid = i < (uint32_t)c.n_checks;
  const uint32_t chk = (uint32_t)c.first_check + (valid ? i : 0u);
  const uint32_t m0 = (uint32_t)job.chk_msg_ptr[chk], l0 = (uint32_t)job.chk_leaf_ptr[chk];
  const int nm = (int)((uint32_t)job.chk_msg_ptr[chk + 1] - m0);
  const int nl = (int)((uint32_t)job.chk_leaf_ptr[chk + 1] - l0);
  const uint32_t b1_in = ((ph.it - 1) & 1) ? s.b1_half : 0u, b1_out = (ph.it & 1) ? s.b1_half : 0u;
  const bool on = (ph.act >> w) & 1u;
  auto bit_of = [&](rsrc_t r, uint32_t at) {
    return ((uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, at + w / FW, 0, kSc1) >> (w % FW)) & 1u;
  };
  float in[MET_MAX_CHECK_DEGREE], suf[MET_MAX_CHECK_DEGREE];  // inputs in the phi domain with their signs
  float run = 0.0f;
  uint32_t parity = bit_of(s.syn, chk * WPI), tot = parity;
#pragma unroll 1
  for (int l = nl - 1; l >= 0; --l) {
    float lf[1];
    ld_f32<1, kSc1>(s.Lphi, ((l0 + l) * W + w) * 4u, lf);
    if (ph.test) parity ^= bit_of(s.B1, b1_in + (l0 + l) * WPI);
    in[nm + l] = lf[0];
    suf[nm + l] = run;
    run = run + fabsf(lf[0]);
    tot ^= sign_bit(lf[0]);
  }
#pragma unroll 1
  for (int k = nm; k > 0; k -= U) {
    uint32_t vi[U];
    float pv[U][1], cv[U][1];
#pragma unroll
    for (int u = 0; u < U; ++u) vi[u] = (uint32_t)job.edge_msgvn[m0 + max(k - 1 - u, 0)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ld_f32<1, kSc1>(ph.first ? s.L2 : s.P, (vi[u] * W + w) * 4u, pv[u]);
      cv[u][0] = 0.0f;
      if (!ph.first) ld_msgs<1, CT, 0>(s.c2v, (m0 + max(k - 1 - u, 0)) * W + w, tab, cv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k - 1 - u >= 0) {
        parity ^= (uint32_t)(pv[u][0] < 0.0f);
        const float x = clamp_llr(pv[u][0] - cv[u][0]);
        const float a = phi(fabsf(x));
        in[k - 1 - u] = copysignf(a, x);
        suf[k - 1 - u] = run;
        run = run + a;
        tot ^= sign_bit(x);
      }
  }
  if (ph.test) {
    const uint64_t bad[1] = {__ballot((parity & (uint32_t)valid) != 0u)};
    unsat |= frames_of<W, 1>(bad);
  }
  run = 0.0f;
#pragma unroll 1
  for (int k = 0; k < nm; ++k) {
    const float a = in[k], mag = phi(run + suf[k]);
    run = run + fabsf(a);
    const float out[1] = {(tot ^ sign_bit(a)) & 1u ? -mag : mag};
    if (valid) st_msgs<1, CT>(s.c2v, (m0 + k) * W + w, out);
  }
  const int leaves = ph.decide && valid ? nl : 0;
#pragma unroll 1
  for (int l = 0; __any(l < leaves); ++l) {
    const bool has = l < leaves;
    const float a = has ? in[nm + l] : 0.0f, S = run + (has ? suf[nm + l] : 0.0f);
    run = run + fabsf(a);
    const uint32_t neg = sign_bit(a), neg_c = (tot ^ neg) & 1u, le = l0 + l;
    const uint64_t ones = __ballot(has && leaf_bit(neg, neg_c, S, fabsf(a)));
    if (has && w % FW == 0) {  // the byte of FW frames
      const uint32_t at = b1_out + le * WPI + w / FW, own = (ph.act >> w) & ((1u << FW) - 1u);
      const uint32_t was = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.B1, at, 0, kSc1);
      __builtin_amdgcn_raw_buffer_store_b8((uint8_t)((was & ~own) | ((uint32_t)(ones >> lane) & own)), s.B1, at, 0, 0);
    }
    if (has && on && ph.post) {
      const float mag = phi(S);
      float lr[1];
      const uint32_t off = (le * W + w) * 4u;
      ld_f32<1, kSc1>(s.Lraw(), off, lr);
      const float p1[1] = {lr[0] + 1.0f * (neg_c ? -mag : mag)};
      st_f32<1>(s.P1(ph.it), off, p1);
    }
  }
}

// Variable update of 64 / (W K) nodes: K lanes share a node's edges, each with U
// gathers in flight; the sum runs through the K lanes in list order (a chain of
// shuffles), so it is the sequential sum of variable_body.
template <int W, int K, int U, typename CT>
__device__ __forceinline__ void variable_tile(const GroupState &s, const int32_t *vn_ptr, const int32_t *vn_edges,
                                              uint32_t n2, uint32_t tile, uint32_t act, const Tables &tab) {
  const uint32_t lane = threadIdx.x & 63, w = lane % W, sub = (lane / W) % K;
  const uint32_t v = tile * (64 / (W * K)) + lane / (W * K);
  const bool on = v < n2 && ((act >> w) & 1u);
  const uint32_t vv = v < n2 ? v : 0u;
  uint32_t e = (uint32_t)vn_ptr[vv];
  const uint32_t e1 = on ? (uint32_t)vn_ptr[vv + 1] : 0u;
  float acc[1];
  ld_f32<1, kSc1>(s.L2, (vv * W + w) * 4u, acc);
  while (__any(e < e1)) {
    float a[U][1];
    uint32_t at[U];
    const uint32_t first = e + sub * U;
    int cnt = e1 > first ? (int)min(e1 - first, (uint32_t)U) : 0;  // this lane's edges
#pragma unroll
    for (int u = 0; u < U; ++u) at[u] = u < cnt ? (uint32_t)vn_edges[first + u] * W + w : kNowhere / 4u;
#pragma unroll
    for (int u = 0; u < U; ++u) ld_msgs<1, CT, kSc1>(s.c2v, at[u], tab, a[u]);
    asm volatile("" : "+v"(cnt));  // compared again below: keeping U masks spills scalar registers
    float in = acc[0];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float x = in;
#pragma unroll
      for (int u = 0; u < U; ++u) x = u < cnt ? x + a[u][0] : x;
      // the partial sum of lane k goes to all lanes of the node
      in = K > 1 ? __shfl(x, (int)((lane & ~(uint32_t)(W * K - 1)) + k * W + w)) : x;
    }
    acc[0] = in;
    e += K * U;
  }
  if (on && sub == 0) st_f32<1>(s.P, (vv * W + w) * 4u, acc);
}

// ---- The team -----------------------------------------------------------------

struct TeamShared {
  uint32_t rank, n, slot, group, err;
  uint32_t last;    // no group is left for this team after the present one
  uint32_t epoch, it, act;  // where a member that was admitted later begins; it = 0: at the start
  uint32_t word;    // OR of the waves' payloads
  uint32_t result;  // OR of the members' payloads
  int32_t stop[16]; // iteration at which each frame of the group stopped, and kSatisfied
};

// The next group that nobody has taken (low word), and with `slots` = 1 the next
// slot (high word).  One addition for both: there are 8 slots, one per die, or
// one per group if there are fewer groups, so that a team without a slot finds
// no group left either.
__device__ __forceinline__ uint64_t take_group(TeamControl *ctl, uint32_t slots) {
  return __hip_atomic_fetch_add(&ctl->taken, (uint64_t)slots << 32 | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A check's messages are read through the first-level cache, by the workgroup
// that wrote them.  Where the checks change hands that cache may hold older ones.
__device__ __forceinline__ void forget_cached() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }

__device__ __forceinline__ uint32_t ld_agent(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Registers the workgroup with its XCD's team; false if it has no part in it.
__device__ bool join_team(TeamControl *ctl, uint32_t xcc, const TeamJob &job, TeamShared &sh) {
  if (xcc >= (uint32_t)job.dies) return false;
  if (threadIdx.x == 0) {
    auto &r = ctl->reg[xcc];
    const uint32_t expected = (uint32_t)job.expected;
    if (job.late_ticks) {  // every eighth workgroup of a die comes in time
      const uint64_t t0 = wall_clock64();
      const uint64_t late = (uint64_t)job.late_ticks * (blockIdx.x / kTeamSlots % 8);
      while (wall_clock64() - t0 < late) __builtin_amdgcn_s_sleep(8);
    }
    const uint32_t rank = __hip_atomic_fetch_add(&r.count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t pub = 0;
    if (rank == 0) {
      const uint64_t t0 = wall_clock64();
      const uint64_t first = take_group(ctl, 1);  // waited for after the loop
      uint32_t n;
      do {
        n = ld_agent(&r.count);
      } while (n < expected && wall_clock64() - t0 < kFormTicks);
      pub = min(n, (uint32_t)kMaxTeam);
      const uint32_t slot = (uint32_t)(first >> 32), g = (uint32_t)first;
      if (g < (uint32_t)job.G && slot < (uint32_t)job.n_slots) pub |= (slot + 1) << 8 | (uint64_t)g << 16;
      __hip_atomic_store(&r.pub, pub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      for (uint32_t i = 0; i < job.poll_limit; ++i) {
        pub = __hip_atomic_load(&r.pub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (pub) break;
        __builtin_amdgcn_s_sleep(1);
      }
    }
    sh.err = 0;
    sh.word = 0;
    sh.rank = rank;
    sh.n = (uint32_t)pub & 255u;
    sh.slot = (uint32_t)(pub >> 8) & 255u;  // slot + 1, 0: nothing to do
    sh.group = (uint32_t)(pub >> 16);
    sh.epoch = sh.it = sh.act = sh.last = 0;
    if (sh.slot && rank >= sh.n) {
      // too late for the start: until the first member admits it or ends
      sh.slot = 0;
      for (uint64_t i = 0; rank < expected && i < (uint64_t)job.poll_limit * 64; ++i) {
        const uint32_t grown = ld_agent(&r.grown);
        if (grown == kEnded) break;
        if (rank < grown) {
          // (the words below were in the L2 before `grown`)
          asm volatile("" ::: "memory");
          sh.slot = (uint32_t)(pub >> 8) & 255u;
          sh.n = grown;
          sh.epoch = ld_agent(&r.state[0]);
          sh.group = ld_agent(&r.state[1]);
          sh.it = ld_agent(&r.state[2]);
          sh.act = ld_agent(&r.state[3]);
          sh.last = ld_agent(&r.state[4]);
          for (int f = 0; f < 16; ++f) sh.stop[f] = (int32_t)ld_agent(&r.stop[f]);
          break;
        }
        __builtin_amdgcn_s_sleep(16);
      }
    }
  }
  __syncthreads();
  return sh.slot != 0 && sh.rank < sh.n;
}

// Barrier of the team's workgroups; returns the OR of everything the members
// put into sh.word before it.  sh.err is set if a member never came (it cannot:
// every member is running), and the caller marks its group's frames and leaves;
// no member passes the barrier after the next one then, so the team ends.
struct TeamBarrier {
  TeamControl *ctl;
  uint32_t xcc, rank, n, poll_limit, epoch;
  __device__ uint32_t operator()(TeamShared &sh) {
    ++epoch;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x < 64) {
      uint64_t *fl = ctl->flag[xcc][epoch & 1];
      if (threadIdx.x == 0) {
        const uint64_t mine = ((uint64_t)sh.word << 32) | epoch;
        sh.word = 0;
        // stays in the XCD's L2, where the members' polls find it
        __hip_atomic_store(fl + rank, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      uint64_t v = 0;
      uint32_t i = 0;
      for (;; ++i) {
        v = threadIdx.x < n ? __hip_atomic_load(fl + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : epoch;
        if (__all((uint32_t)v == epoch)) break;
        if (i == poll_limit) break;
      }
      uint32_t w = (uint32_t)(v >> 32);
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) w |= __shfl_xor(w, d);
      if (threadIdx.x == 0) {
        sh.result = w;
        if (i == poll_limit) sh.err = 1;
      }
    }
    __syncthreads();
    return sh.result;
  }
};

// The first member hands the state after iteration `it - 1` to new members, which
// begin with check update `it` and the team's barrier after it.
__device__ void admit(TeamControl *ctl, uint32_t xcc, const TeamShared &sh, uint32_t n, uint32_t epoch, uint32_t g,
                      int it, uint32_t act) {
  if (threadIdx.x >= 64) return;
  auto &r = ctl->reg[xcc];
  if (threadIdx.x < 16) r.stop[threadIdx.x] = (uint32_t)sh.stop[threadIdx.x];
  if (threadIdx.x == 0) {
    r.state[0] = epoch;
    r.state[1] = g;
    r.state[2] = (uint32_t)it;
    r.state[3] = act;
    r.state[4] = sh.last;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (threadIdx.x == 0) __hip_atomic_store(&r.grown, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int W, typename CT>
__device__ __forceinline__ void check_phase(const TeamJob &job, const GroupState &s, const Phase &ph,
                                            uint32_t wave, uint32_t waves, const Tables &tab, TeamShared &sh) {
  uint32_t unsat = 0;
  int c = 0;
  for (uint32_t t = wave; t < (uint32_t)job.check_tiles; t += waves) {
    while (c + 1 < job.n_classes && t >= (uint32_t)job.cls[c + 1].tile0) ++c;
    const TeamClass k = job.cls[c];
    const uint32_t tile = t - (uint32_t)k.tile0;
    switch (k.shape) {
      case 0: check_tile<W, 3, 1, CT>(s, job.edge_msgvn, k, tile, ph, tab, unsat); break;
      case 1: check_tile<W, 2, 1, CT>(s, job.edge_msgvn, k, tile, ph, tab, unsat); break;
      case 2: check_tile<W, 12, 0, CT>(s, job.edge_msgvn, k, tile, ph, tab, unsat); break;
      case 3: check_tile<W, 11, 0, CT>(s, job.edge_msgvn, k, tile, ph, tab, unsat); break;
      case 4: check_tile<W, 6, 0, CT>(s, job.edge_msgvn, k, tile, ph, tab, unsat); break;
      case 5: check_tile<W, 5, 0, CT>(s, job.edge_msgvn, k, tile, ph, tab, unsat); break;
      case 6: check_tile<W, 4, 0, CT>(s, job.edge_msgvn, k, tile, ph, tab, unsat); break;
      default: check_tile_generic<W, CT>(s, job, k, tile, ph, tab, unsat);
    }
  }
  if (unsat && (threadIdx.x & 63) == 0) atomicOr(&sh.word, unsat);
}

// Parity of the final decisions (after the last iteration).
template <int W>
__device__ __forceinline__ void test_phase(const TeamJob &job, const GroupState &s, int it, uint32_t wave,
                                           uint32_t waves, TeamShared &sh) {
  constexpr int F = kFramesPerLane<W>, LPI = W / F;
  const uint32_t lane = threadIdx.x & 63, wl = lane % LPI;
  const uint32_t b1 = (it & 1) ? s.b1_half : 0u;
  uint32_t word = 0;
  for (uint32_t t = wave; t * (64 / LPI) < (uint32_t)job.M; t += waves) {
    const uint32_t j = t * (64 / LPI) + lane / LPI;
    if (j >= (uint32_t)job.M) continue;
    uint32_t par = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.syn, j * LPI + wl, 0, kSc1);
    for (int32_t e = job.chk_msg_ptr[j]; e < job.chk_msg_ptr[j + 1]; ++e) {
      float pv[F];
      ld_f32<F, kSc1>(s.P, ((uint32_t)job.edge_msgvn[e] * W + wl * F) * 4u, pv);
#pragma unroll
      for (int f = 0; f < F; ++f) par ^= (uint32_t)(pv[f] < 0.0f) << f;
    }
    for (int32_t e = job.chk_leaf_ptr[j]; e < job.chk_leaf_ptr[j + 1]; ++e)
      par ^= (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.B1, b1 + (uint32_t)e * LPI + wl, 0, kSc1);
    word |= (par & ((1u << F) - 1u)) << (wl * F);
  }
  if (word) atomicOr(&sh.word, word);
}

// A group's inputs into its state: channel LLRs of the message nodes, leaf
// inputs in the phi domain, syndrome bits.
template <int W>
__device__ __forceinline__ void setup_phase(const TeamJob &job, const GroupState &s, uint32_t g, uint32_t wave,
                                            uint32_t waves) {
  constexpr int F = kFramesPerLane<W>, LPI = W / F;
  const uint32_t lane = threadIdx.x & 63, wl = lane % LPI;
  const uint32_t items = (uint32_t)(job.EL + job.N2);
  for (uint32_t t = wave; t * (64 / LPI) < items; t += waves) {
    const uint32_t i = t * (64 / LPI) + lane / LPI;
    if (i >= items) continue;
    const bool leaf = i < (uint32_t)job.EL;
    const uint32_t k = leaf ? i : i - (uint32_t)job.EL;
    const int64_t v = leaf ? job.leaf_vn[k] : job.msg_vn_user[k];
    float l[F];
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const uint32_t frame = g * W + wl * F + f;
      l[f] = frame < (uint32_t)job.B ? job.llr[(int64_t)frame * job.N + v] : 0.0f;
    }
    const uint32_t off = (k * W + wl * F) * 4u;
    if (leaf) {
      float ph[F];
#pragma unroll
      for (int f = 0; f < F; ++f) ph[f] = copysignf(phi(fabsf(clamp_llr(l[f]))), l[f]);
      st_f32<F>(s.Lphi, off, ph);
      if (job.posterior) st_f32<F>(s.Lraw(), off, l);
    } else {
      st_f32<F>(s.L2, off, l);
    }
  }
  for (uint32_t t = wave; t * (64 / LPI) < (uint32_t)job.M; t += waves) {
    const uint32_t j = t * (64 / LPI) + lane / LPI;
    if (j >= (uint32_t)job.M) continue;
    uint32_t b = 0;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const uint32_t frame = g * W + wl * F + f;
      if (frame < (uint32_t)job.B) b |= (uint32_t)(job.syn[(int64_t)frame * job.M + j] & 1u) << f;
    }
    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)b, s.syn, (uint32_t)job.chk_pos[j] * LPI + wl, 0, 0);
  }
}

// Outputs in user order, 64 consecutive nodes per wave and store.
template <int W>
__device__ __forceinline__ void output_phase(const TeamJob &job, const GroupState &s, uint32_t g, uint32_t wave,
                                             uint32_t waves, const TeamShared &sh) {
  constexpr int F = kFramesPerLane<W>, LPI = W / F;
  const uint32_t lane = threadIdx.x & 63;
  for (uint32_t t = wave; t * 64 < (uint32_t)job.N; t += waves) {
    const uint32_t v = t * 64 + lane;
    if (v >= (uint32_t)job.N) continue;
    const int32_t slot = job.vn_slot[v];
    const uint32_t k = slot >= 0 ? (uint32_t)slot : (uint32_t)(-(slot + 1));
#pragma unroll
    for (int wl = 0; wl < LPI; ++wl) {
      float post[F];
      uint32_t b = 0;
      const uint32_t off = (k * W + wl * F) * 4u;
      if (slot >= 0) {
        ld_f32<F, kSc1>(s.P, off, post);
#pragma unroll
        for (int f = 0; f < F; ++f) b |= (uint32_t)(post[f] < 0.0f) << f;
      } else {
        const uint32_t ba = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.B1, k * LPI + wl, 0, kSc1);
        const uint32_t bb = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(s.B1, s.b1_half + k * LPI + wl, 0, kSc1);
#pragma unroll
        for (int f = 0; f < F; ++f) b |= ((sh.stop[wl * F + f] & 1) ? bb : ba) & (1u << f);
        if (job.posterior) {
          float pa[F], pb[F];
          ld_f32<F, kSc1>(s.P1(0), off, pa);
          ld_f32<F, kSc1>(s.P1(1), off, pb);
#pragma unroll
          for (int f = 0; f < F; ++f) post[f] = (sh.stop[wl * F + f] & 1) ? pb[f] : pa[f];
        }
      }
#pragma unroll
      for (int f = 0; f < F; ++f) {
        const uint32_t frame = g * W + wl * F + f;
        if (frame >= (uint32_t)job.B) continue;
        job.bits[(int64_t)frame * job.N + v] = (uint8_t)((b >> f) & 1u);
        if (job.posterior) job.posterior[(int64_t)frame * job.N + v] = post[f];
      }
    }
  }
}

template <int W, typename CT>
__device__ __forceinline__ void variable_phase(const TeamJob &job, const GroupState &s, uint32_t act, uint32_t wave,
                                               uint32_t waves, const Tables &tab) {
  const uint32_t n2 = (uint32_t)job.N2;
  auto sweep = [&](auto kc, auto uc) {
    constexpr int K = decltype(kc)::value, U = decltype(uc)::value;
    if constexpr (W * K <= 64) {
      constexpr uint32_t per = 64 / (W * K);
      for (uint32_t t = wave; t * per < n2; t += waves)
        variable_tile<W, K, U, CT>(s, job.vn_ptr, job.vn_edges, n2, t, act, tab);
    }
  };
  switch (job.lanes_per_vn) {
    case 16: sweep(std::integral_constant<int, 16>{}, std::integral_constant<int, 8>{}); break;
    case 4: sweep(std::integral_constant<int, 4>{}, std::integral_constant<int, 16>{}); break;
    default: sweep(std::integral_constant<int, 1>{}, std::integral_constant<int, 24>{});
  }
}

// A frame's outcome, written by its team's first member, and the mark of a
// member that gave up, before that or after: the mark stays.  The waits keep
// converged at 0 with it: the flag is stored before the outcome is offered, and
// cleared after the mark.
__device__ __forceinline__ void give_up(const TeamJob &job, uint32_t f) {
  (void)__hip_atomic_exchange(job.iters + f, kGivenUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  job.converged[f] = 0;
}
__device__ __forceinline__ bool set_outcome(const TeamJob &job, uint32_t f, int32_t stop) {
  job.converged[f] = (uint8_t)((stop & kSatisfied) != 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  int32_t was = kUntaken;
  return __hip_atomic_compare_exchange_strong(job.iters + f, &was, stop & ~kSatisfied, __ATOMIC_RELAXED,
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int W, typename CT>
__global__ __launch_bounds__(kTeamBlock) void k_team(const TeamJob job) {
  __shared__ TeamShared sh;
  __shared__ float s_q8[std::is_class<CT>::value ? 128 : 1];
  __shared__ float s_phi[std::is_same<CT, q8lut_t>::value ? kLutSize : 1];
  __shared__ uint8_t s_code[std::is_same<CT, q8lut_t>::value ? kLutSize : 1];
  TeamControl *ctl = reinterpret_cast<TeamControl *>(job.ws);
  const uint32_t xcc = xcc_id();
  if (!join_team(ctl, xcc, job, sh)) return;
  if constexpr (std::is_class<CT>::value)
    for (int i = threadIdx.x; i < 128; i += kTeamBlock) s_q8[i] = kQ8Table.v[i];
  if constexpr (std::is_same<CT, q8lut_t>::value)
    for (int i = threadIdx.x; i < kLutSize; i += kTeamBlock) {
      s_phi[i] = kPhiTables.a[i];
      s_code[i] = kPhiTables.out[i];
    }
  __syncthreads();
  const Tables tab{s_q8, s_phi, s_code};
  const uint32_t rank = sh.rank, slot = sh.slot - 1;
  TeamBarrier barrier{ctl, xcc, rank, sh.n, job.poll_limit, sh.epoch};
  uint32_t wave = rank + barrier.n * (uint32_t)wave_id(), waves = barrier.n * kTeamWaves;
  char *base = job.ws + job.off_slots + (size_t)slot * job.slot_bytes;
  auto buf = [&](uint32_t off, uint32_t end) { return buffer_of(base + off, end - off); };
  GroupState s;
  s.job = &job;
  s.base = base;
  s.c2v = buf(0, job.off_P);
  s.P = buf(job.off_P, job.off_L2);
  s.L2 = buf(job.off_L2, job.off_Lphi);
  s.Lphi = buf(job.off_Lphi, job.off_Lraw);
  s.syn = buf(job.off_syn, job.off_B1);
  s.B1 = buf(job.off_B1, job.slot_bytes);
  s.b1_half = (job.slot_bytes - job.off_B1) / 2;

  // the last wave, which has the least to set up and put out, keeps the books
  // (numbers from 0 in it, beyond every frame elsewhere)
  const uint32_t clerk = threadIdx.x - (kTeamBlock - 64);
  uint32_t g = sh.group;
  int it = (int)sh.it;
  if (it) forget_cached();
  uint32_t act = sh.act;
  while (g < (uint32_t)job.G) {
    if (it == 0) {
      act = (1u << min((uint32_t)W, (uint32_t)job.B - g * W)) - 1u;
      if (threadIdx.x < W) sh.stop[threadIdx.x] = job.max_iter;
      setup_phase<W>(job, s, g, wave, waves);
      // where every group has been taken by now, the team need not meet again
      // after its outputs
      if (rank == 0 && clerk == 0 &&
          (uint32_t)__hip_atomic_load(&ctl->taken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= (uint32_t)job.G)
        atomicOr(&sh.word, 1u);
      const uint32_t last = barrier(sh);
      if (threadIdx.x == 0) sh.last = last;
      it = 1;
    }
    for (; it <= job.max_iter && !sh.err; ++it) {
      Phase ph;
      ph.first = it == 1;
      ph.test = job.early && it >= 2;
      ph.decide = job.early || it == job.max_iter;
      ph.post = ph.decide && job.posterior;
      ph.it = it;
      ph.act = act;
      check_phase<W, CT>(job, s, ph, wave, waves, tab, sh);
      const uint32_t unsat = barrier(sh);
      if (ph.test) {
        const uint32_t done = act & ~unsat;
        if (threadIdx.x < W && ((done >> threadIdx.x) & 1u)) sh.stop[threadIdx.x] = (it - 1) | kSatisfied;
        act &= unsat;
        if (!act) break;
      }
      variable_phase<W, CT>(job, s, act, wave, waves, tab);
      // a team that is not complete takes in who has registered since
      if (rank == 0 && threadIdx.x == 0 && barrier.n < (uint32_t)job.expected && it < job.max_iter) {
        const uint32_t n = min(ld_agent(&ctl->reg[xcc].count), (uint32_t)job.expected);
        if (n > barrier.n) sh.word = n;
      }
      const uint32_t grown = barrier(sh);
      if (grown && !sh.err) {
        forget_cached();
        barrier.n = grown;
        wave = rank + grown * (uint32_t)wave_id();
        waves = grown * kTeamWaves;
        if (rank == 0) admit(ctl, xcc, sh, grown, barrier.epoch, g, it + 1, act);
      }
    }
    if (act && !sh.err) {  // frames that ran the whole budget
      test_phase<W>(job, s, job.max_iter, wave, waves, sh);
      const uint32_t done = act & ~barrier(sh);
      if (threadIdx.x < W && ((done >> threadIdx.x) & 1u)) sh.stop[threadIdx.x] |= kSatisfied;
    }
    __syncthreads();  // sh.stop
    const bool mine = clerk < min((uint32_t)W, (uint32_t)job.B - g * W);  // a thread per frame
    if (sh.err) {
      if (mine) give_up(job, g * W + clerk);
      break;
    }
    // (both waited for after the outputs)
    uint32_t next = 0;
    bool set = true;
    if (rank == 0 && threadIdx.x == 0 && !sh.last) next = (uint32_t)take_group(ctl, 0);
    if (rank == 0 && mine) set = set_outcome(job, g * W + clerk, sh.stop[clerk]);
    output_phase<W>(job, s, g, wave, waves, sh);
    if (!set) job.converged[g * W + clerk] = 0;
    if (sh.last) break;
    if (rank == 0 && threadIdx.x == 0) sh.word = next;
    g = barrier(sh);
    if (sh.err) break;
    it = 0;
  }
  if (rank == 0 && threadIdx.x == 0)
    __hip_atomic_store(&ctl->reg[xcc].grown, kEnded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int W, typename CT>
void launch_team(const TeamJob &job, unsigned grid, hipStream_t st) {
  hipLaunchKernelGGL((k_team<W, CT>), dim3(grid), dim3(kTeamBlock), 0, st, job);
}

template <typename CT>
void launch_reduced(int W, const TeamJob &job, unsigned grid, hipStream_t st) {
  W == 4   ? launch_team<4, CT>(job, grid, st)
  : W == 8 ? launch_team<8, CT>(job, grid, st)
           : launch_team<16, CT>(job, grid, st);
}

// Dies that the device shows: eight, or fewer where it is partitioned.
constexpr int kCusPerDie = 32;
int device_dies(int *dies, int *cus) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  HIP_TRY(hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev));
  *dies = std::max(1, std::min(*cus / kCusPerDie, kTeamSlots));
  return MET_OK;
}

// Lanes per variable node: as many as still leave one tile per wave of a full
// team (a second round of tiles costs more than shorter gather chains save),
// as the node degrees can use, and as W allows.
int lanes_per_vn(const met_code *c, int W) {
  const int64_t lanes = 32 * (int64_t)kTeamBlock;
  for (int k : {16, 4})
    if (W * k <= 64 && c->N2 * W * k <= lanes && c->max_vn_deg > 8 * (k / 4)) return k;
  return 1;
}

// Message edges (in millions) of checks without a compiled shape.
double generic_edges(const met_code *c) {
  int64_t compiled = 0;
  for (const CheckClass &k : c->classes)
    if (k.shape != kShapeGeneric) compiled += k.n_checks * kShapeMsg[k.shape];
  return 1e-6 * (double)(c->E12 - compiled);
}

}  // namespace

size_t team_control_bytes() { return align256(sizeof(TeamControl)); }

size_t team_slot(const met_code *c, int W, bool post, size_t c2v_bytes, TeamJob *job) {
  const int F = W < 4 ? W : 4, LPI = W / F;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += align256(bytes);
    return at;
  };
  const size_t e = (size_t)c->E12 * W, v = (size_t)c->N2 * W * 4, l = (size_t)c->EL * W * 4;
  (void)take(e * c2v_bytes);
  const size_t off[] = {take(v), take(v), take(l), take(post ? l : 0), take(post ? 2 * align256(l) : 0),
                        take((size_t)c->M * LPI), take(2 * align256((size_t)c->EL * LPI))};
  if (job) {
    job->off_P = (uint32_t)off[0];
    job->off_L2 = (uint32_t)off[1];
    job->off_Lphi = (uint32_t)off[2];
    job->off_Lraw = (uint32_t)off[3];
    job->off_P1 = (uint32_t)off[4];
    job->off_syn = (uint32_t)off[5];
    job->off_B1 = (uint32_t)off[6];
    job->slot_bytes = (uint32_t)o;
  }
  return o;
}


// Estimated times (us) of an iteration and of a decode's set-up and outputs on both
// paths, fitted to fixed-iteration runs: rates 0.1, 0.05 and 0.02 and regular codes
// of check degrees 6 to 20, N = 1000 to 262144, groups of 1 to 16 frames, batches of
// 1 to 256 (E: message edges, V: nodes of degree >= 2, G: message edges of checks
// with run-time degrees, N: in millions; F: frames in whole groups).  Measured
// iterations:
//                                  teams, W = 1 / 4 / 16     launches, 1 / 16 / 64 / 256
//   rate 0.1, N = 4096             6.1 / 6.4 / 8.3           15 / 6.4 / 9.3 / 14
//   rate 0.1, N = 32000            10 / 13 / 34              15 / 13 / 20 / 60
//   rate 0.1, N = 65536            15 / 24 / 67              22 / 19 / 37 / 119
//   rate 0.1, N = 160000           40 / 55 / 162             20 / 30 / 75 / -
//   rate 0.02, N = 100001          23 / 54 / 117             36 / 24 / 50 / -
//   rate 0.05, N = 65536 (4 checks 19 / 32 / 76              36 / 30 / 47 / -
//     with run-time degrees)
//   (3,6) regular, N = 60000       16 / 34 / 124             9 / 18 / 57 / 190
//   (3,9) regular, N = 60000 (all  27 / 57 / 182             16 / 32 / 78 / 283
//     with run-time degrees)
//   8-bit, rate 0.1, N = 65536     - / - / 73                - / - / 60 / -
//     with the table               - / - / 56                - / - / 52 / -
namespace {

struct Run {
  double iteration, frames, once;  // per iteration; part of it that goes with the frames; per decode
};

// A group of W frames on one die.  A tile's chain of loads has a floor of 5 us an
// iteration; nodes whose edges are more than their lanes have under way add
// their further gathers; one or two frames per check leave the larger codes with
// many short tiles.
Run team_run(const met_code *c, int W, size_t c2v_bytes, bool lut) {
  const double E = 1e-6 * c->E12, V = 1e-6 * c->N2, N = 1e-6 * c->N;
  const int K = lanes_per_vn(c, W);
  const double under_way = K == 16 ? 128 : K == 4 ? 64 : 24;
  const double per_edge = c2v_bytes > 1 ? 32 + 15.5 * W : lut ? 24 + 14 * W : 36 + 19 * W;
  double t = 5 + per_edge * E + 60 * V * W + (K == 1 ? 4.5 : 1.5) * std::max(0.0, c->max_vn_deg / under_way - 1);
  if (W <= 2) t += 40 * std::max(0.0, E - 0.2);
  if (const double G = generic_edges(c); G > 0) t += 0.5 * c->max_check_deg + 25 * G * W;
  return {t, t, 4 + 60 * N + 95 * N * W};
}

Run launch_run(const met_code *c, int B, size_t c2v_bytes, bool lut) {
  const int W = choose_interleave(B);
  const double F = (double)((B + W - 1) / W) * W, E = 1e-6 * c->E12, V = 1e-6 * c->N2, G = generic_edges(c);
  const int generic = G > 0, compiled = (int)c->classes.size() - generic;
  const int launches = 1 + generic + (W >= 16 && c2v_bytes > 1 ? std::min(compiled, 1) : compiled);
  const double each = c2v_bytes > 1 ? 3.2 : lut ? 5.2 : 6.2;
  double t = each * launches, f = ((c2v_bytes == 4 ? 2.2 : c2v_bytes == 2 ? 1.45 : lut ? 1.55 : 1.7) * E + (c2v_bytes == 4 ? 5 : 4) * V) * F;
  // long lists: one frame per item reads them and their rows scattered
  const double longer = std::max(0, c->max_vn_deg - 24);
  t += W >= 16 ? 0.065 * longer : 4.5 + 0.17 * longer * std::min(1.0, 1e-5 * c->N);
  if (generic) {
    t += 3 + 0.5 * c->max_check_deg;
    f += 1.8 * G * F;
  }
  return {t + f, f, 25 + 12e-6 * c->N * F};
}

}  // namespace

// The rule compares the two.  With early exit, taken to last two fifths of the budget,
// the launches have the host's reads to wait for and frames to move (us an
// iteration: 7.2 up to 32 frames, 12 where one group is squeezed, 16 where there
// are several), save by that 80 or 70 % of what goes with the frames, and run until
// the slowest of all frames stops; with posteriors they write them in every
// iteration.  A team runs until the slowest of each of its groups: in units of the
// former a group of W out of B frames takes about m = (W / B)^0.175, and the eight
// teams end after max(1, m groups / 8) + 0.74 m (1 where each has one group).  (How
// many frames never stop is not known beforehand: rate 0.02, N = 40000, 48 frames of a
// good channel 4.4 ms by launches and 3.6 by teams, of a bad one 4.5 and 6.8.)  A team
// that would be slower by more than 15 % if every frame ran its whole budget is not
// taken, nor one whose states leave the Infinity Cache (64 frames of N = 10^6 in
// groups of 8: 87 ms).  Fixed-iteration launches take 10 % more than their estimate
// where teams come into question.  Of 3400 decodes (the codes above, 1 to 400 frames,
// good and bad channels, all storage types, early exit and fixed) 84 are more than
// 5 % slower than the launches would be, and in the mean they are 3.3 % off the best
// of launches and five widths; estimates by edges alone: 255, and 4.7 %.
int team_width(const met_code *c, int B, bool post, size_t c2v_bytes, bool lut, int max_iter, bool early,
               size_t ws_bytes, int *width) {
  *width = 0;
  int dies = 0, cus = 0;
  if (const int rc = device_dies(&dies, &cus)) return rc;
  const Run l = launch_run(c, B, c2v_bytes, lut);
  const bool squeezed = early && !post && choose_interleave(B) == 64;
  const double iterations = early ? 0.4 * max_iter + 0.5 : max_iter;
  const double waits = !early ? 0 : !squeezed ? 7.2 : B <= 64 ? 12 : 16;
  const double whole =
      (l.iteration + (early && post ? 0.4 * l.frames : 0.0) + waits + l.once / iterations) * (early ? 1.0 : 1.1);
  int best = 0;
  double best_t = squeezed ? whole - l.frames * (B > 64 ? 0.7 : 0.8) : whole;
  for (int W : {16, 8, 4, 2, 1}) {
    if (c2v_bytes != sizeof(float) && W < 4) continue;
    const int G = (B + W - 1) / W, rounds = (G + dies - 1) / dies;
    const size_t slot = team_slot(c, W, post, c2v_bytes, nullptr), all = slot * std::min(G, kTeamSlots);
    if (slot >= kMaxSlotBytes || team_control_bytes() + all > ws_bytes || all > kMaxTeamBytes) continue;
    const Run r = team_run(c, W, c2v_bytes, lut);
    const double once = (20 + rounds * r.once) / iterations;
    if (rounds * r.iteration + once > 1.15 * whole) continue;
    const double m = std::min(1.0, std::pow((double)W / B, 0.175));
    const double t = once + r.iteration * (early && rounds > 1 ? std::max(1.0, m * G / dies) + 0.74 * m : rounds);
    if (t < best_t) {
      best = W;
      best_t = t;
    }
  }
  *width = best;
  return MET_OK;
}

int team_decode(const met_code *c, const DeviceCode *d, int W, const float *llr, const uint8_t *syn, int B,
                int max_iter, uint32_t flags, uint8_t *bits, int32_t *iters, uint8_t *conv, float *post,
                char *ws, hipStream_t st, const met_team_options *opt) {
  int dies = 0, cus = 0;
  if (const int rc = device_dies(&dies, &cus)) return rc;
  const size_t cb = (flags & MET_C2V_Q8) ? 1 : (flags & MET_C2V_FP16) ? 2 : 4;
  TeamJob job{};
  job.edge_msgvn = d->edge_msgvn;
  job.vn_ptr = d->vn_ptr;
  job.vn_edges = d->vn_edges_plane;
  job.msg_vn_user = d->msg_vn_user;
  job.leaf_vn = d->leaf_vn;
  job.vn_slot = d->vn_slot;
  job.chk_msg_ptr = d->chk_msg_ptr;
  job.chk_leaf_ptr = d->chk_leaf_ptr;
  job.chk_pos = d->chk_pos;
  job.N = c->N;
  job.M = (int32_t)c->M;
  job.N2 = (int32_t)c->N2;
  job.EL = (int32_t)c->EL;
  job.llr = llr;
  job.syn = syn;
  job.bits = bits;
  job.iters = iters;
  job.converged = conv;
  job.posterior = post;
  job.ws = ws;
  job.B = B;
  job.G = (B + W - 1) / W;
  job.max_iter = max_iter;
  job.early = !(flags & MET_FIXED_ITERS);
  job.n_slots = std::min(job.G, kTeamSlots);
  job.dies = opt && opt->dies ? opt->dies : kTeamSlots;
  job.late_ticks = opt ? 100u * (uint32_t)opt->late_us : 0u;
  job.poll_limit = opt && opt->polls ? (uint32_t)opt->polls : kPollLimit;
  job.off_slots = team_control_bytes();
  job.lanes_per_vn = lanes_per_vn(c, W);
  team_slot(c, W, post != nullptr, cb, &job);
  int32_t tiles = 0;
  for (const CheckClass &k : c->classes) {
    TeamClass &t = job.cls[job.n_classes++];
    t.shape = k.shape;
    t.tile0 = tiles;
    t.first_check = (int32_t)k.first_check;
    t.n_checks = (int32_t)k.n_checks;
    t.first_msg = (int32_t)k.first_msg;
    t.first_leaf = (int32_t)k.first_leaf;
    const bool wide = k.shape == kShapeGeneric || kShapeMsg[k.shape] > 4;
    const int per = 64 / (wide ? W : W / std::min(W, 4));  // checks per wave, as check_tile
    tiles += (int32_t)((k.n_checks + per - 1) / per);
  }
  job.check_tiles = tiles;
  job.expected = std::min(cus, kCusPerDie);
  hipLaunchKernelGGL(k_team_clear, dim3(1), dim3(kTeamBlock), 0, st, reinterpret_cast<uint32_t *>(ws), iters, conv, B);
  {
    ScopedTimer t(st, "k_team");
    const unsigned grid = (unsigned)cus;
    if (flags & MET_C2V_FP16) {
      launch_reduced<half_t>(W, job, grid, st);
    } else if (flags & MET_CHECK_LUT) {
      launch_reduced<q8lut_t>(W, job, grid, st);
    } else if (flags & MET_C2V_Q8) {
      launch_reduced<q8_t>(W, job, grid, st);
    } else {
      switch (W) {
        case 1: launch_team<1, float>(job, grid, st); break;
        case 2: launch_team<2, float>(job, grid, st); break;
        case 4: launch_team<4, float>(job, grid, st); break;
        case 8: launch_team<8, float>(job, grid, st); break;
        default: launch_team<16, float>(job, grid, st);
      }
    }
  }
  HIP_TRY(hipGetLastError());
  return MET_OK;
}

// What the widest groups take that team_width would choose on eight dies: none
// wider than the narrowest that hold the batch in one round.
size_t team_bytes(const met_code *c, int B, bool post, size_t c2v_bytes) {
  size_t most = 0;
  const int narrowest = c2v_bytes == sizeof(float) ? 1 : 4;
  for (int W = narrowest; W <= 16 && (W == narrowest || B > W / 2 * kTeamSlots); W *= 2) {
    const size_t slot = team_slot(c, W, post, c2v_bytes, nullptr), all = slot * std::min((B + W - 1) / W, kTeamSlots);
    if (slot < kMaxSlotBytes && all <= kMaxTeamBytes) most = std::max(most, team_control_bytes() + all);
  }
  return most;
}

// Whether the teams' states in groups of W frames fit in ws_bytes.
bool team_fits(const met_code *c, int B, bool post, size_t c2v_bytes, int W, size_t ws_bytes) {
  const size_t slot = team_slot(c, W, post, c2v_bytes, nullptr);
  return slot < kMaxSlotBytes && team_control_bytes() + slot * std::min((B + W - 1) / W, kTeamSlots) <= ws_bytes;
}

}  // namespace met
