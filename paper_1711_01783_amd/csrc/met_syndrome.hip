// Syndromes S = H x mod 2 of many frames (Methods, Step 1: Bob's syndrome).
//
// A check's bit is the parity of a few bits at random positions of the frame.
// Gathering them byte by byte, frame by frame, reads the adjacency once per
// frame and costs a cache line per bit: 64 frames of N = 10^6 (rate 0.1, 3.76
// million edges) took 995 us.  With room for packed words the frames are
// transposed instead: one word per variable node holds its bit in up to 64
// frames, each edge is gathered once for all of them, and the parities are
// written back as bytes in runs of 256 checks.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "met_internal.h"

#define HIP_TRY(expr)                                                                     \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess) return met::fail(MET_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

namespace met {
namespace {

constexpr int kSynBlock = 256;

__global__ __launch_bounds__(kSynBlock) void k_syndrome(const int32_t *all_vn, const int32_t *all_ptr, int64_t N,
                                                        int64_t M, const uint8_t *bits, uint8_t *syn) {
  const int f = blockIdx.y;
  const int64_t j = (int64_t)blockIdx.x * kSynBlock + threadIdx.x;
  if (j >= M) return;
  uint32_t s = 0;
  for (int32_t e = all_ptr[j]; e < all_ptr[j + 1]; ++e) s ^= bits[(int64_t)f * N + all_vn[e]] & 1u;
  syn[(int64_t)f * M + j] = (uint8_t)s;
}

// Four consecutive bytes of a row; rows of odd length start at any address.
__device__ __forceinline__ uint32_t ld4(const uint8_t *p) {
  uint32_t x;
  __builtin_memcpy(&x, p, 4);
  return x;
}
__device__ __forceinline__ void st4(uint8_t *p, uint32_t x) { __builtin_memcpy(p, &x, 4); }

// Words of the nodes of one group of frames: a thread takes four nodes, reads
// them as one 32-bit word per frame (256 bytes per wave) and is bound by the
// read of the bytes.
template <typename T>
__global__ __launch_bounds__(kSynBlock) void k_pack_frames(const uint8_t *bits, int64_t N, int32_t B, T *words) {
  constexpr int W = 8 * sizeof(T);
  const int64_t v = ((int64_t)blockIdx.x * kSynBlock + threadIdx.x) * 4;
  if (v >= N) return;
  const int f0 = blockIdx.y * W, nf = min(W, B - f0);
  const uint8_t *row = bits + (int64_t)f0 * N + v;
  T *out = words + (int64_t)blockIdx.y * N + v;
  T w[4] = {0, 0, 0, 0};
  if (v + 4 <= N) {
#pragma unroll 8
    for (int f = 0; f < nf; ++f, row += N) {
      const uint32_t x = ld4(row);
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] |= (T)((x >> (8 * i)) & 1u) << f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = w[i];
  } else {
    for (int i = 0; v + i < N; ++i) {
      T x = 0;
      for (int f = 0; f < nf; ++f) x |= (T)(row[(int64_t)f * N + i] & 1u) << f;
      out[i] = x;
    }
  }
}

// Parities of 256 checks, one per thread, then their bytes frame by frame.
// Bound by the gathers: a word per edge, from a table of N words.
template <typename T>
__global__ __launch_bounds__(kSynBlock) void k_syndrome_words(const int32_t *all_vn, const int32_t *all_ptr, int64_t N,
                                                              int64_t M, int32_t B, const T *words, uint8_t *syn) {
  constexpr int W = 8 * sizeof(T);
  __shared__ T par[kSynBlock];
  const int64_t j0 = (int64_t)blockIdx.x * kSynBlock, j = j0 + threadIdx.x;
  const T *table = words + (int64_t)blockIdx.y * N;
  T s = 0;
  if (j < M) {
    int32_t e = all_ptr[j];
    const int32_t e1 = all_ptr[j + 1];
    for (; e + 4 <= e1; e += 4) {
      const T a = table[all_vn[e]], b = table[all_vn[e + 1]], c = table[all_vn[e + 2]], d = table[all_vn[e + 3]];
      s ^= a ^ b ^ c ^ d;
    }
    for (; e < e1; ++e) s ^= table[all_vn[e]];
  }
  par[threadIdx.x] = s;
  __syncthreads();
  const int lane = threadIdx.x & 63, f0 = blockIdx.y * W, nf = min(W, B - f0);
  const int64_t jj = j0 + 4 * lane;
  T w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = par[4 * lane + i];
  for (int f = threadIdx.x >> 6; f < nf; f += kSynBlock / 64) {
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) x |= (uint32_t)((w[i] >> f) & 1u) << (8 * i);
    uint8_t *out = syn + (int64_t)(f0 + f) * M + jj;
    if (jj + 4 <= M) {
      st4(out, x);
    } else {
      for (int i = 0; jj + i < M; ++i) out[i] = (uint8_t)(x >> (8 * i));
    }
  }
}

// Bytes of a word of the packed table: the smallest that holds the frames, so
// that the gathered table stays small (N bytes up to 8 frames).
int word_bytes(int B) { return B <= 8 ? 1 : B <= 16 ? 2 : B <= 32 ? 4 : 8; }

size_t packed_bytes(const met_code *c, int B) {
  const int wb = word_bytes(B);
  return (size_t)((B + 8 * wb - 1) / (8 * wb)) * c->N * wb;
}

template <typename T>
void launch_packed(const met_code *c, const DeviceCode *d, const uint8_t *bits, int B, uint8_t *syn, void *ws,
                   hipStream_t st) {
  const unsigned G = (unsigned)((B + 8 * (int)sizeof(T) - 1) / (8 * (int)sizeof(T)));
  const int64_t per = (int64_t)kSynBlock * 4;
  hipLaunchKernelGGL(k_pack_frames<T>, dim3((unsigned)((c->N + per - 1) / per), G), dim3(kSynBlock), 0, st, bits, c->N,
                     B, static_cast<T *>(ws));
  hipLaunchKernelGGL(k_syndrome_words<T>, dim3((unsigned)((c->M + kSynBlock - 1) / kSynBlock), G), dim3(kSynBlock), 0,
                     st, d->all_vn, d->all_ptr, c->N, c->M, B, static_cast<const T *>(ws), syn);
}

}  // namespace
}  // namespace met

using met::fail;

extern "C" int met_syndrome_workspace_bytes(const met_code *c, int32_t B, size_t *bytes) { return met::guarded("met_syndrome_workspace_bytes", [&]() -> int {
  met::clear_error();
  if (!c || !bytes) return fail(MET_EINVAL, "met_syndrome_workspace_bytes: NULL argument");
  if (B < 1 || B > 65535) return fail(MET_EINVAL, "met_syndrome_workspace_bytes: B = %d outside 1..65535", B);
  *bytes = met::packed_bytes(c, B);
  return MET_OK;
  });
}

extern "C" int met_syndrome_ex(const met_code *c, const uint8_t *bits, int32_t B, uint8_t *syn, void *workspace,
                               size_t ws_bytes, void *stream) { return met::guarded("met_syndrome", [&]() -> int {
  met::clear_error();
  if (!c || !bits || !syn) return fail(MET_EINVAL, "met_syndrome: NULL argument");
  if (B < 1 || B > 65535) return fail(MET_EINVAL, "met_syndrome: B = %d outside 1..65535", B);
  if ((uintptr_t)workspace & 7) return fail(MET_EINVAL, "met_syndrome: workspace must be 8-byte aligned");
  if (workspace && ws_bytes < met::packed_bytes(c, B))
    return fail(MET_EINVAL, "met_syndrome: workspace of %zu bytes, %zu needed", ws_bytes, met::packed_bytes(c, B));
  const met::DeviceCode *d = nullptr;
  int rc = met::device_code(c, &d);
  if (rc) return rc;
  const hipStream_t st = (hipStream_t)stream;
  if (!workspace) {
    hipLaunchKernelGGL(met::k_syndrome, dim3((unsigned)((c->M + met::kSynBlock - 1) / met::kSynBlock), B),
                       dim3(met::kSynBlock), 0, st, d->all_vn, d->all_ptr, c->N, c->M, bits, syn);
  } else {
    switch (met::word_bytes(B)) {
      case 1: met::launch_packed<uint8_t>(c, d, bits, B, syn, workspace, st); break;
      case 2: met::launch_packed<uint16_t>(c, d, bits, B, syn, workspace, st); break;
      case 4: met::launch_packed<uint32_t>(c, d, bits, B, syn, workspace, st); break;
      default: met::launch_packed<uint64_t>(c, d, bits, B, syn, workspace, st);
    }
  }
  HIP_TRY(hipGetLastError());
  return MET_OK;
  });
}

extern "C" int met_syndrome(const met_code *c, const uint8_t *bits, int32_t B, uint8_t *syn, void *stream) {
  return met_syndrome_ex(c, bits, B, syn, nullptr, 0, stream);
}
