// Environment of one gate (Sec. 3, Eq. 10; Fig. env_calc_tensor) straight from the caller's
// row-major state sets: qfs_environment, with its partial sums in a buffer kept between calls,
// and qfs_environment_noalloc, with them in a fixed device array of this library.
#include <algorithm>
#include <mutex>

#include "qfs_internal.h"
#include "wave_sums.h"

namespace qfs {
namespace {

constexpr int kNaThreads = 256;                  // threads per work-group
constexpr int kNaBlocks = 1024;                  // most work-groups, so most partials
constexpr int64_t kNaItemsPerThread = 1 << 10;   // most (sample, other-qubit) items a thread sums
constexpr int64_t kNaMaxItems = (int64_t)kNaBlocks * kNaThreads * kNaItemsPerThread;  // 2^28

// The partials: 16 complex128 per work-group, 256 KiB. Each GPU the library runs on holds
// its own copy until the process ends; every call on a GPU shares it.
static __device__ __align__(256) c128 scratch[kNaBlocks * 16];

// Item it = (sample j, value r of the n - 2 other qubits): the four amplitudes of a_j and
// b_j that differ in qubits qa, qb (qubit q is bit n - 1 - q of the amplitude index; the
// local index of the pair is 2 bit(qa) + bit(qb)); the sample number lies above the amplitude's
// bits in the flat index of the set. Each thread sums its items' 16 products a(q) conj(b(p));
// the work-group's sums go to part[blockIdx.x][q * 4 + p], reduced in a fixed order.
// Bound by its launches and the wave sums at 10 qubits and 64 states (one item a thread), by
// memory on large sets: a call takes 22 us at that size, 33 with both sets first converted to
// the sweep's layout.
__global__ __launch_bounds__(kNaThreads) void k_env_rows(int n, int64_t items, const c128 *a, const c128 *b,
                                                         int qa, int qb, c128 *part) {
  __shared__ double red[kNaThreads / 64][32];
  const int pa = n - 1 - qa, pb = n - 1 - qb;
  const int lo = std::min(pa, pb), hi = std::max(pa, pb);
  c128 acc[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = cmake(0.0, 0.0);
  for (int64_t it = blockIdx.x * (int64_t)kNaThreads + threadIdx.x; it < items;
       it += (int64_t)gridDim.x * kNaThreads) {
    // zero bits at positions lo and hi
    int64_t r = it + (it & ~((int64_t(1) << lo) - 1));
    r += r & ~((int64_t(1) << hi) - 1);
    c128 av[4], bv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t off = r + ((int64_t((q >> 1) & 1) << pa) | (int64_t(q & 1) << pb));
      av[q] = a[off];
      bv[q] = b[off];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 4; ++p) cfma_conj(acc[q * 4 + p], av[q], bv[p]);
  }
  double v[32];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    v[2 * e] = acc[e].re;
    v[2 * e + 1] = acc[e].im;
  }
  const double ws = wave_sums<double, 32>(v);
  const int lane = threadIdx.x & 63;
  if (lane < 32) red[threadIdx.x >> 6][wave_sums_index<32>(lane)] = ws;
  __syncthreads();
  if (threadIdx.x < 32) {
    double t = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kNaThreads / 64; ++w) t += red[w][threadIdx.x];
    reinterpret_cast<double *>(part + (int64_t)blockIdx.x * 16)[threadIdx.x] = t;
  }
}

// gamma[e] = sum over the P partials: thread 16 g + e those g, g + 16, .. in order, then the
// sixteen sums in order.
__global__ __launch_bounds__(kNaThreads) void k_env_rows_sum(const c128 *part, int P, c128 *gamma) {
  __shared__ c128 red[kNaThreads];
  const int e = threadIdx.x & 15;
  c128 s = cmake(0.0, 0.0);
  for (int p = threadIdx.x >> 4; p < P; p += kNaThreads / 16) s = s + part[(int64_t)p * 16 + e];
  red[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x < 16) {
    for (int g = 1; g < kNaThreads / 16; ++g) s = s + red[16 * g + e];
    gamma[e] = s;
  }
}

int blocks_of(int64_t items) { return (int)std::min<int64_t>(kNaBlocks, (items + kNaThreads - 1) / kNaThreads); }

int env_rows(int n, int64_t items, const qfs_c128 *a, const qfs_c128 *b, int qa, int qb, c128 *part, qfs_c128 *gamma,
             hipStream_t s) {
  const int P = blocks_of(items);
  hipLaunchKernelGGL(k_env_rows, dim3(P), dim3(kNaThreads), 0, s, n, items, reinterpret_cast<const c128 *>(a),
                     reinterpret_cast<const c128 *>(b), qa, qb, part);
  QFS_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_env_rows_sum, dim3(1), dim3(kNaThreads), 0, s, part, P, reinterpret_cast<c128 *>(gamma));
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

// Device address of `scratch` on each GPU, looked up once per device (the array's name in
// host code is only a stand-in, not a device address).
int scratch_ptr(c128 **out) {
  constexpr int kDevices = 64;
  static std::mutex mu;
  static c128 *ptr[kDevices] = {};
  int dev = 0;
  QFS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kDevices) {
    set_error_detail("qfs_environment_noalloc: device index out of range");
    return QFS_EUNSUPPORTED;
  }
  std::lock_guard<std::mutex> lk(mu);
  if (!ptr[dev]) {
    void *p = nullptr;
    QFS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) {
      set_error_detail("qfs_environment_noalloc: no device address for the partials array");
      return QFS_EDEVICE;
    }
    ptr[dev] = static_cast<c128 *>(p);
  }
  *out = ptr[dev];
  return QFS_OK;
}

}  // namespace
}  // namespace qfs

using namespace qfs;

extern "C" int qfs_environment_noalloc(int32_t n, int32_t M, const qfs_c128 *a, const qfs_c128 *b, int32_t qa,
                                       int32_t qb, qfs_c128 *gamma, void *hip_stream) {
  if (n < 2 || n > 24 || qa < 0 || qb < 0 || qa >= n || qb >= n || qa == qb) {
    set_error_detail("qfs_environment_noalloc: need 2 <= n <= 24 and two distinct qubits below n");
    return QFS_EINVAL;
  }
  if (M < 1 || !a || !b || !gamma) return QFS_EINVAL;
  const int64_t items = (int64_t)M << (n - 2);
  if (items > kNaMaxItems) {
    set_error_detail("qfs_environment_noalloc: M 2^(n-2) = " + std::to_string(items) + " exceeds " +
                     std::to_string(kNaMaxItems) + " (1024 work-group partials of 256 x 1024 items)");
    return QFS_EINVAL;
  }
  c128 *part = nullptr;
  QFS_TRY(scratch_ptr(&part));
  return env_rows(n, items, a, b, qa, qb, part, gamma, static_cast<hipStream_t>(hip_stream));
}

extern "C" int qfs_environment(int32_t n, int32_t M, const qfs_c128 *a, const qfs_c128 *b, int32_t qa, int32_t qb,
                               qfs_c128 *gamma, void *hip_stream) {
  if (n < 2 || n > 24 || qa < 0 || qb < 0 || qa >= n || qb >= n || qa == qb) {
    set_error_detail("qfs_environment: need 2 <= n <= 24 and two distinct qubits below n");
    return QFS_EINVAL;
  }
  if (M < 1 || !a || !b || !gamma) return QFS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int64_t items = (int64_t)M << (n - 2);
  BufferScope scope;
  DevBuf part;
  QFS_TRY(part.alloc(sizeof(c128) * 16 * blocks_of(items)));
  QFS_TRY(env_rows(n, items, a, b, qa, qb, part.as<c128>(), gamma, s));
  return scope.done(s);
}
