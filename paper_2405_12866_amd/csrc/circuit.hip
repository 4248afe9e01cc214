// Simulation of a whole gate list on a set of FP64 states (Fig. pre-comp without a B list; the
// circuit form of the target, Sec. 2.3): each work-group takes some samples into LDS, applies
// every gate there, and writes them out, so the set is read and written once instead of once
// per gate.
#include <algorithm>

#include "qfs_internal.h"
#include "stream_common.h"

namespace qfs {

namespace {

constexpr int kCircuitGates = 120;   // gates of one launch (their bit positions are arguments)
constexpr int kCircuitMaxBits = 13;  // 2^13 amplitudes of 16 bytes and their padding in LDS

struct CircuitArgs {
  const c128 *src;
  c128 *dst;
  int64_t si, sj;      // element (amplitude i, sample j) of either set at i si + j sj
  const c128 *gates;   // the first gate applied
  int32_t n, M, lspw;  // samples per work-group: 2^lspw
  int32_t L, step;     // gate t of the launch at gates + 16 t step
  uint8_t pa[kCircuitGates], pb[kCircuitGates];  // bit positions of its qubits
};

// 16 bytes of padding per 256: gates on the lowest amplitude bits stay free of bank conflicts
__device__ __forceinline__ uint32_t amp_slot(uint32_t i) { return i + (i >> 4); }

// Bound by FP64 issue and LDS throughput alike (a gate is 16 complex FMAs, four 16-byte reads
// and four writes per group of four amplitudes) and by the barrier after each gate: 12 qubits,
// 256 states, 44 gates in 55 us (1.3 us a gate on every compute unit, 19 us of FP64 issue in
// all), against 44 launches of 9.0 us, and 14 us of layout conversions, with one gate a launch.
// That is a caller's set, rows of amplitudes. A run's sets have the samples contiguous: with one
// sample a work-group each 16-byte read then takes a whole line, and the same launch 82 us.
template <int T, bool DAG>
__global__ __launch_bounds__(T) void k_circuit(CircuitArgs A) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  c128 *st = reinterpret_cast<c128 *>(lds_raw);
  const int n = A.n;
  const uint32_t N = 1u << n, spw = 1u << A.lspw;
  const int64_t j0 = (int64_t)blockIdx.x << A.lspw;
  const uint32_t cnt = (uint32_t)min((int64_t)spw, (int64_t)A.M - j0);
  const uint32_t total = N << A.lspw;
  // along the set's contiguous index, samples or amplitudes
  auto each = [&](auto f) {
    for (uint32_t e = threadIdx.x; e < total; e += T) {
      const uint32_t j = A.si == 1 ? e >> n : e & (spw - 1), i = A.si == 1 ? e & (N - 1) : e >> A.lspw;
      if (j < cnt) f(amp_slot((j << n) + i), (int64_t)i * A.si + (j0 + j) * A.sj);
    }
  };
  each([&](uint32_t s, int64_t o) { st[s] = A.src[o]; });
  lds_barrier();
  const uint32_t groups = cnt << (n - 2);
  for (int t = 0; t < A.L; ++t) {
    const int pa = A.pa[t], pb = A.pb[t];
    const int lo = min(pa, pb), hi = max(pa, pb);
    const cptr<c128> g = as_const(A.gates + (int64_t)16 * t * A.step);
    c128 u[16];
    load_gate<double>(g, u, DAG);
    for (uint32_t gi = threadIdx.x; gi < groups; gi += T) {
      uint32_t i0 = ((gi >> lo) << (lo + 1)) | (gi & ((1u << lo) - 1u));
      i0 = ((i0 >> hi) << (hi + 1)) | (i0 & ((1u << hi) - 1u));
      const uint32_t o[4] = {amp_slot(i0), amp_slot(i0 + (1u << pb)), amp_slot(i0 + (1u << pa)),
                             amp_slot(i0 + (1u << pa) + (1u << pb))};
      c128 x[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) x[p] = st[o[p]];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c128 acc = cmake(0.0, 0.0);
#pragma unroll
        for (int p = 0; p < 4; ++p) cfma(acc, u[q * 4 + p], x[p]);
        st[o[q]] = acc;
      }
    }
    lds_barrier();
  }
  each([&](uint32_t s, int64_t o) { A.dst[o] = st[s]; });
}

template <int T, bool DAG>
int launch_t(const CircuitArgs &A, size_t lds, hipStream_t s) {
  static size_t attr = 0;
  QFS_TRY(ensure_dynamic_lds(reinterpret_cast<const void *>(&k_circuit<T, DAG>), lds, &attr));
  const int64_t spw = int64_t(1) << A.lspw;
  hipLaunchKernelGGL((k_circuit<T, DAG>), dim3((unsigned)((A.M + spw - 1) / spw)), dim3(T), lds, s, A);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

}  // namespace

// LDS of a work-group with 2^bits amplitudes
static size_t circuit_lds(int bits) { return sizeof(c128) * ((size_t(1) << bits) + ((size_t(1) << bits) >> 4)); }

bool circuit_fits(int n) { return n >= 2 && n <= kCircuitMaxBits && circuit_lds(n) <= lds_max_bytes(); }

int launch_circuit(int n, int M, const c128 *src, c128 *dst, int64_t si, int64_t sj, int L, const int32_t *pairs,
                   const c128 *gates, bool dagger, hipStream_t s) {
  if (!circuit_fits(n) || M < 1) return QFS_EINVAL;
  // one group of four amplitudes per thread and gate: 1024 threads where a state alone has as
  // many groups or the set fills the device with such work-groups; else 256, so that small
  // sets spread over more compute units
  const bool wide = n >= 12 || ((int64_t)M << n >= int64_t(256) * 4096 && circuit_lds(12) <= lds_max_bytes());
  const int groups_log = wide ? 12 : 10;  // amplitudes of a work-group
  CircuitArgs A{};
  A.dst = dst;
  A.si = si;
  A.sj = sj;
  A.n = n;
  A.M = M;
  A.lspw = std::max(0, groups_log - n);
  while (A.lspw > 0 && (int64_t(1) << (A.lspw - 1)) >= M) --A.lspw;
  const size_t lds = circuit_lds(n + A.lspw);
  for (int t0 = 0; t0 == 0 || t0 < L; t0 += kCircuitGates) {
    A.src = t0 == 0 ? src : dst;
    A.L = std::min(kCircuitGates, L - t0);
    A.step = dagger ? -1 : 1;
    for (int t = 0; t < A.L; ++t) {
      const int k = dagger ? L - 1 - (t0 + t) : t0 + t;
      if (t == 0) A.gates = gates + (int64_t)16 * k;
      A.pa[t] = (uint8_t)(n - 1 - pairs[2 * k]);
      A.pb[t] = (uint8_t)(n - 1 - pairs[2 * k + 1]);
    }
    if (wide)
      QFS_TRY(dagger ? (launch_t<1024, true>(A, lds, s)) : (launch_t<1024, false>(A, lds, s)));
    else
      QFS_TRY(dagger ? (launch_t<256, true>(A, lds, s)) : (launch_t<256, false>(A, lds, s)));
  }
  return QFS_OK;
}

}  // namespace qfs
