// Batched QFactor-Sample: thousands of small instantiation problems x multistarts in
// persistent launches (one work-group per (problem, start) job, jobs pulled from a
// device work queue, longest first).
//
// Per job the two working state sets live in LDS when they fit (else in a per-work-group
// global scratch slot): the forward pass runs Psi through the gates in place, and the
// backward pass recovers each intermediate state B_k = u_k^dag B_{k+1} with the gate as
// it was before the sweep (gate k is updated only after its environment is reduced),
// so no B list is stored. The paper's per-sweep steps are unchanged (Sec. 3, Fig.
// pre-comp, Fig. env_calc_tensor); the control decisions of App. A run on the device
// after every sweep; doublings and the complex128 refinement switch are applied by the
// host between launches.
#include <algorithm>

#include "batch.h"
#include "philox.h"
#include "polar2.h"
#include "polar4.h"
#include "stream_common.h"
#include "wave_sums.h"

namespace qfs {

namespace {

template <typename R>
__device__ __forceinline__ R bwave_sum(R x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// Zero bits put in at positions lo < hi: each moves the bits from its position on up by one,
// which adds that part once more. Bits beyond a state's index (the sample number of a flat
// [rows][N] group index) move along, so the result indexes the whole set.
__device__ __forceinline__ uint32_t deposit2(uint32_t r, int lo, int hi) {
  r += r & ~((1u << lo) - 1u);
  return r + (r & ~((1u << hi) - 1u));
}

// Sum over the work-group; result valid in every thread. `red` holds NT/64 values.
template <int NT>
__device__ __forceinline__ double block_sum(double x, double *red) {
  x = bwave_sum<double>(x);
  if (NT == 64) return x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = x;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) t += red[i];
  return t;
}

// Pointers of known address space: through generic ones (a problem's pointers come out of
// memory, and the sets lie in LDS or in global scratch) every access is a flat one.
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ gptr<T> as_global(T *p) {
  return (gptr<T>)p;
}

// A working set: packets of V samples of one amplitude (16 bytes: two complex64 or one
// complex128), packet (j / V) 2^n + i for samples j .. and amplitude i, at slot pk + pk / 16
// (16 bytes of padding per 256, so the groups of gates on the lowest bits fall on different
// banks). Samples beyond the set's rows are zero.
__device__ __forceinline__ uint32_t bslot(uint32_t pk) { return pk + (pk >> 4); }

template <typename R>
struct BSet {
  Pk<R> *p;          // (LDS or scratch)
  uint32_t packets;  // packet rows << n
  __device__ __forceinline__ BSet(Pk<R> *p_, int rows, int n)
      : p(p_), packets((uint32_t)((rows + Pk<R>::V - 1) / Pk<R>::V) << n) {}
  __device__ __forceinline__ BSet(Pk<R> *p_, uint32_t packets_) : p(p_), packets(packets_) {}
};

template <typename R>
__device__ __forceinline__ void gate_regs(const cx<R> *u, bool dagger, cx<R> (&m)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int p = 0; p < 4; ++p) m[q * 4 + p] = dagger ? cconj(u[p * 4 + q]) : u[q * 4 + p];
}

// Apply u (or u^dagger) of qubit bit positions (pa, pb) to a set.
template <typename R, int NT>
__device__ __forceinline__ void apply_states(BSet<R> S, int pa, int pb, const cx<R> *u, bool dagger) {
  constexpr int V = Pk<R>::V;
  cx<R> m[16];
  gate_regs<R>(u, dagger, m);
  const int lo = min(pa, pb), hi = max(pa, pb);
  const uint32_t ma = 1u << pa, mb = 1u << pb;
  const uint32_t total = S.packets >> 2;
  for (uint32_t g = threadIdx.x; g < total; g += NT) {
    const uint32_t i0 = deposit2(g, lo, hi);
    const uint32_t o[4] = {bslot(i0), bslot(i0 + mb), bslot(i0 + ma), bslot(i0 + ma + mb)};
    Pk<R> x[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) x[p] = S.p[o[p]];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      Pk<R> y;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        cx<R> acc = cmake<R>(0, 0);
#pragma unroll
        for (int p = 0; p < 4; ++p) cfma(acc, m[q * 4 + p], x[p].v[e]);
        y.v[e] = acc;
      }
      S.p[o[q]] = y;
    }
  }
}

// B_k <- u^dagger B_{k+1} in place (as apply_states), and acc += a conj(B_k) over the same groups
// on the way: the environment of the gate on (pa, pb). Its products and sums are FP64 for either
// state precision: some of the small environments here are so badly conditioned that FP32 sums of a
// thread's groups show in the gates (over 30 sets of 128 problems, four sweeps, the error against
// FP64 states is 5 % less in the geometric mean). The vector units do them at the FP32 rate; the
// conversions and registers cost 5 % of the call.
template <typename R, int NT>
__device__ __forceinline__ void unapply_env(BSet<R> B, const Pk<R> *a, int pa, int pb, const cx<R> *u,
                                            c128 (&acc)[16]) {
  constexpr int V = Pk<R>::V;
  cx<R> m[16];
  gate_regs<R>(u, true, m);
  const int lo = min(pa, pb), hi = max(pa, pb);
  const uint32_t ma = 1u << pa, mb = 1u << pb;
  const uint32_t total = B.packets >> 2;
  for (uint32_t g = threadIdx.x; g < total; g += NT) {
    const uint32_t i0 = deposit2(g, lo, hi);
    const uint32_t o[4] = {bslot(i0), bslot(i0 + mb), bslot(i0 + ma), bslot(i0 + ma + mb)};
    Pk<R> x[4], av[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) x[p] = B.p[o[p]];
#pragma unroll
    for (int p = 0; p < 4; ++p) av[p] = a[o[p]];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      Pk<R> y;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        cx<R> t = cmake<R>(0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) cfma(t, m[p * 4 + q], x[q].v[e]);
        y.v[e] = t;
        const c128 td = cmake((double)t.re, (double)t.im);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          cfma_conj(acc[q * 4 + p], cmake((double)av[q].v[e].re, (double)av[q].v[e].im), td);
      }
      B.p[o[p]] = y;
    }
  }
}

// Packets of a set's load in flight per thread (the sets come from L2 or memory: one at a time, a
// set of 8192 amplitudes took 32 round trips of 256 threads).
constexpr int kSetLoads = 4;

// Packet pk's samples of the FP64 states [rows][N] in global (zero beyond the rows).
template <typename R>
__device__ __forceinline__ void fetch_pk(gptr<const c128> src, int rows, int n, uint32_t pk, c128 (&v)[Pk<R>::V]) {
  const uint32_t i = pk & ((1u << n) - 1u), j = (pk >> n) * Pk<R>::V;
#pragma unroll
  for (int e = 0; e < Pk<R>::V; ++e) {
    const bool in = (int)(j + e) < rows;
    const gptr<const c128> q = src + (((size_t)(in ? j + e : j) << n) + i);
    const double re = q->re, im = q->im;
    v[e] = in ? cmake(re, im) : cmake(0.0, 0.0);
  }
}

// The set from FP64 states [rows][N] in global.
template <typename R, int NT>
__device__ __forceinline__ void load_states(BSet<R> S, const c128 *src_, int rows, int n) {
  constexpr int V = Pk<R>::V;
  const gptr<const c128> src = as_global(src_);
  for (uint32_t e0 = threadIdx.x; e0 < S.packets; e0 += kSetLoads * NT) {
    c128 v[kSetLoads][V];
#pragma unroll
    for (int i = 0; i < kSetLoads; ++i) fetch_pk<R>(src, rows, n, min(e0 + i * NT, S.packets - 1), v[i]);
#pragma unroll
    for (int i = 0; i < kSetLoads; ++i) {
      Pk<R> y;
#pragma unroll
      for (int e = 0; e < V; ++e) y.v[e] = cmake<R>((R)v[i][e].re, (R)v[i][e].im);
      if (e0 + i * NT < S.packets) S.p[bslot(e0 + i * NT)] = y;
    }
  }
}

// (1/rows) sum |x - ref|^2 with ref FP64 in global; every thread gets the result.
template <typename R, int NT>
__device__ __forceinline__ double dist_states(BSet<R> S, const c128 *ref_, int rows, int n, double *red) {
  constexpr int V = Pk<R>::V;
  const gptr<const c128> ref = as_global(ref_);
  double acc = 0.0;
  for (uint32_t e0 = threadIdx.x; e0 < S.packets; e0 += kSetLoads * NT) {
    c128 v[kSetLoads][V];
#pragma unroll
    for (int i = 0; i < kSetLoads; ++i) fetch_pk<R>(ref, rows, n, min(e0 + i * NT, S.packets - 1), v[i]);
#pragma unroll
    for (int i = 0; i < kSetLoads; ++i) {
      if (e0 + i * NT >= S.packets) continue;
      const Pk<R> x = S.p[bslot(e0 + i * NT)];
#pragma unroll
      for (int e = 0; e < V; ++e) {  // (padding samples: zero against zero)
        const double dr = (double)x.v[e].re - v[i][e].re, di = (double)x.v[e].im - v[i][e].im;
        acc += dr * dr + di * di;
      }
    }
  }
  return block_sum<NT>(acc, red) / (double)rows;
}

// ------------------------------------------------------------------ job sweeps
template <int NW>
struct SweepShared {
  c128 wred[NW][16];
  c128 gam[16];
  c128 pg[16], pv[16];
  double ps[4];
  double red[NW];
  int flag;   // control decision after a sweep
  int pause;  // pause at the top of a sweep (a separate word: waves may still be reading
              // flag from the previous sweep's decision when thread 0 writes this one)
};

// Jobs with at most kGatesInLds gates keep all their gates (state precision) in LDS for
// the whole launch; longer templates stage one gate at a time from the FP64 masters.
constexpr int kGatesInLds = 24;

template <typename R, int NT>
__device__ __forceinline__ void run_job(const BatchArgs &A, int jid, Pk<R> *buf, SweepShared<NT / 64> &sh, cx<R> *gl,
                                        cx<R> *gates_l) {
  BJob &J = A.jobs[jid];
  BProb &P = A.probs[J.prob];
  const int n = P.n, L = P.L, M = P.M, Mv = P.Mv;
  // set A (validation states forward, the backward state), and behind it set B (training states,
  // B_k); for n >= 4 whole padding blocks, so that A's and B's packets are one run
  const uint32_t pkA = BSet<R>(buf, max(M, Mv), n).packets;
  Pk<R> *bufB = buf + bslot((pkA + 15u) & ~15u);
  const BSet<R> setA(buf, M, n), setB(bufB, M, n), setV(buf, Mv, n), both(buf, 2 * pkA);
  const bool one_run = Mv == M && n >= 4;
  const gptr<const int32_t> pairs = as_global(P.pairs), kinds = as_global(P.kinds);
  c128 *g64 = P.g64 + (size_t)J.start * L * 16;
  c128 *vst = P.vst + (size_t)J.start * L * 16;
  const BParams &hp = A.hp;
  const double beta = effective_beta(hp.beta, hp.beta_normalized != 0, M);

  // gate k of this job in R precision: resident in LDS (short templates), or staged
  // from the FP64 master into the slot gl
  const bool resident = L <= kGatesInLds;
  if (resident) {
    for (int e = threadIdx.x; e < L * 16; e += NT) {
      const c128 u = g64[e];
      gates_l[e] = cmake<R>((R)u.re, (R)u.im);
    }
    __syncthreads();
  }
  auto gate = [&](int k) -> const cx<R> * {
    if (resident) return gates_l + k * 16;
    if (threadIdx.x < 16) {
      const c128 u = g64[k * 16 + threadIdx.x];
      gl[threadIdx.x] = cmake<R>((R)u.re, (R)u.im);
    }
    __syncthreads();
    return gl;
  };
  // forward: set B <- C Psi (training), set A <- C Psi_val; returns c_val; c0 optional
  auto forward = [&](double *c0) {
    load_states<R, NT>(setB, P.psi, M, n);
    if (Mv > 0) load_states<R, NT>(setV, P.psiv, Mv, n);
    // the loads fill one element per thread while a gate reads groups of four written by
    // other waves (and gate(k) returns without a barrier when the gates are resident)
    __syncthreads();
    for (int k = 0; k < L; ++k) {
      const cx<R> *u = gate(k);
      const int pa = n - 1 - pairs[2 * k], pb = n - 1 - pairs[2 * k + 1];
      if (one_run) {
        apply_states<R, NT>(both, pa, pb, u, false);
      } else {
        apply_states<R, NT>(setB, pa, pb, u, false);
        if (Mv > 0) apply_states<R, NT>(setV, pa, pb, u, false);
      }
      __syncthreads();
    }
    if (c0) *c0 = dist_states<R, NT>(setB, P.phi, M, n, sh.red);
    return Mv > 0 ? dist_states<R, NT>(setV, P.phiv, Mv, n, sh.red) : -1.0;
  };

  const int Kmax = A.sweeps_per_launch;
  double c0 = 0.0;
  // read once: thread 0 clears the flag below, and every wave must take the same branch
  // to the barrier inside it
  const bool need_c0 = J.need_c0 != 0;
  double cval = forward(need_c0 ? &c0 : nullptr);
  if (need_c0) {
    if (threadIdx.x == 0) {
      J.c_prev = c0;
      J.c_train = c0;
      J.c_val = Mv > 0 ? cval : c0;
      J.need_c0 = 0;
    }
    __syncthreads();
  }
  for (int sw = 0; sw < Kmax; ++sw) {
    // stop at a sweep boundary the problem already decided on
    if (threadIdx.x == 0) {
      const int ds = __hip_atomic_load(&P.done_sweep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int os = __hip_atomic_load(&P.over_sweep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sh.pause = (!hp.independent && (J.total >= ds || J.total >= os)) ? 1 : 0;
    }
    __syncthreads();
    if (sh.pause) {
      if (threadIdx.x == 0) J.status = BJ_PAUSED;
      return;
    }
    // ---- backward (right to left), set B holds C Psi on entry
    load_states<R, NT>(setA, P.phi, M, n);
    __syncthreads();
    for (int k = L - 1; k >= 0; --k) {
      const int pa = n - 1 - pairs[2 * k], pb = n - 1 - pairs[2 * k + 1];
      const int kind = P.kinds ? kinds[k] : QFS_GATE_2Q;
      if (k < L - 1) {
        const cx<R> *u1 = gate(k + 1);  // already updated
        const int qa = n - 1 - pairs[2 * (k + 1)], qb = n - 1 - pairs[2 * (k + 1) + 1];
        apply_states<R, NT>(setA, qa, qb, u1, true);
        __syncthreads();
      }
      const cx<R> *u0 = gate(k);  // not yet updated
      if (kind == QFS_GATE_FIXED) {  // applied only, no environment
        apply_states<R, NT>(setB, pa, pb, u0, true);  // B_k
        __syncthreads();
        continue;
      }
      // B_k and the environment of gate k
      c128 acc[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = cmake(0.0, 0.0);
      unapply_env<R, NT>(setB, setA.p, pa, pb, u0, acc);
      const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
      {
        // value 2e of entry e's real part, 2e + 1 of its imaginary part
        double v[32];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          v[2 * e] = acc[e].re;
          v[2 * e + 1] = acc[e].im;
        }
        const double ws = wave_sums<double, 32>(v);
        if (lane < 32) reinterpret_cast<double *>(&sh.wred[w][0])[wave_sums_index<32>(lane)] = ws;
      }
      __syncthreads();
      if (threadIdx.x < 16) {
        c128 t = sh.wred[0][threadIdx.x];
        for (int ww = 1; ww < NT / 64; ++ww) t = t + sh.wred[ww][threadIdx.x];
        sh.gam[threadIdx.x] = t;
      }
      __syncthreads();
      // the new gate k goes to the FP64 master and (state precision) to its LDS slot;
      // the old one has served its last use (B_k above)
      cx<R> *unew = resident ? gates_l + k * 16 : gl;
      if (kind == QFS_GATE_1Q) {
        if (threadIdx.x == 0) polar2_update<R>(sh.gam, beta, g64 + k * 16, unew);
      } else if (threadIdx.x < 64) {
        polar4_wave<R>(sh.gam, beta, g64 + k * 16, g64 + k * 16, unew, sh.pg, sh.pv, sh.ps, vst + k * 16);
      }
      __syncthreads();
    }
    // cost of the updated gates: a_0 = u_0^dag a
    {
      const int pa = n - 1 - pairs[0], pb = n - 1 - pairs[1];
      apply_states<R, NT>(setA, pa, pb, resident ? gates_l : gl, true);  // the new u_0
      __syncthreads();
    }
    const double ct = dist_states<R, NT>(setA, P.psi, M, n, sh.red);
    __syncthreads();
    cval = forward(nullptr);
    // ---- control (App. A), one thread
    if (threadIdx.x == 0) {
      const double cv = Mv > 0 ? cval : ct;
      J.iter += 1;
      J.total += 1;
      J.work += (double)(M + Mv) * (double)(1u << n) * (double)L;
      const bool improved = fabs(J.c_prev) - fabs(ct) > hp.diff_tol_r * fabs(ct);
      J.z = improved ? 0 : J.z + 1;
      J.c_prev = ct;
      J.c_train = ct;
      J.c_val = cv;
      const bool gen_ok = P.full || Mv == 0 || cv <= (1.0 + hp.overtrain_ratio) * ct;
      int st = BJ_RUN;
      if (ct < hp.dist_tol && gen_ok) {
        st = BJ_SUCCESS;
        __hip_atomic_fetch_min(&P.done_sweep, J.total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (J.iter >= hp.min_iter && !gen_ok && M < P.mcap) {
        st = BJ_OVER;
        __hip_atomic_fetch_min(&P.over_sweep, J.total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (J.iter >= hp.min_iter && !gen_ok && ct < hp.dist_tol) {
        st = BJ_NOT_GEN;
      } else if (J.iter >= hp.min_iter && J.z >= hp.plateau_window) {
        st = BJ_PLATEAU;
      } else if (J.total >= hp.max_iter) {
        st = BJ_MAX_ITER;
      } else if (sizeof(R) == 4 && hp.mixed && ct < hp.refine_below) {
        st = BJ_REFINE;
      }
      J.status = st;
      sh.flag = st;
    }
    __syncthreads();
    if (sh.flag != BJ_RUN) return;
  }
}

// SCR: the sets in this work-group's global slot instead of LDS (an instantiation of its own, so
// that either kind is accessed by its own instructions). Two waves a SIMD:
// with three the FP64 environment spills (128 problems of 5-7 qubits: the longest class takes 2.86
// ms instead of 2.74, the next 0.80 instead of 0.95, the call 3 % more).
template <typename R, int NT, bool SCR>
__global__ __launch_bounds__(NT, 2) void k_batch_sweep(BatchArgs A) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ SweepShared<NT / 64> sh;
  __shared__ int qi_s;
  __shared__ __align__(16) cx<R> gl[16];
  __shared__ __align__(16) cx<R> gates_l[kGatesInLds * 16];
  for (;;) {
    if (threadIdx.x == 0) qi_s = atomicAdd(A.queue_head, 1);
    __syncthreads();
    const int qi = qi_s;
    __syncthreads();
    if (qi >= A.njobs) break;
    const int jid = A.queue[qi];
    if constexpr (SCR)
      run_job<R, NT>(A, jid, reinterpret_cast<Pk<R> *>(A.scratch + (size_t)blockIdx.x * A.scratch_slot_bytes), sh, gl,
                     gates_l);
    else
      run_job<R, NT>(A, jid, reinterpret_cast<Pk<R> *>(lds_raw), sh, gl, gates_l);
    __syncthreads();
  }
}

// ------------------------------------------------------------------ per-problem setup
// Two work-groups per problem: training columns [m0, m1) of the Ginibre stream (role 1,
// stream 0, index j N + i) orthonormalised against all previous columns (the unique QR with
// positive diag R), and U psi for them; and a fresh validation set (role 2, stream =
// generation) with its U psi. All FP64, states [M][N] in global memory.

constexpr int kSetupBlock = 512;

// Wave sum in every lane: DPP moves within the 16-lane rows, then across them.
__device__ __forceinline__ double bwave_all(double x) {
  x += xor_lane<1>(x);
  x += xor_lane<2>(x);
  x += xor_lane<4>(x);
  x += xor_lane<8>(x);
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// Columns c0 .. c1 - 1 of Q ([col][N]) orthonormalised in order against every column before
// them (those below c0 are orthonormal already): modified Gram-Schmidt column by column over
// the later ones, run twice, which leaves the orthogonality error at rounding level for any
// full-rank set (the unique QR with positive diag(R)). Step j needs one barrier: every wave
// takes column j (EL elements a lane) and its norm for itself and removes it from the later
// columns dealt to the wave, two at a time; the scaled column is written one step later, when
// no wave reads it any more. Bound by the latency of a step's loads and wave sums: the set-up of
// 128 problems of 5-7 qubits (up to 64 training and 64 validation states of 128 amplitudes)
// takes 0.56 ms, against 5.1 ms with one column at a time, a thread per projection walking
// down both columns, and the validation set after the training set.
template <int EL>
__device__ void orth_columns_el(c128 *Q, int n, int c0, int c1) {
  const int N = 1 << n, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int NW = kSetupBlock / 64;
  auto load = [&](c128 (&x)[EL], int col) {
#pragma unroll
    for (int i = 0; i < EL; ++i) {
      const int e = lane + 64 * i;
      x[i] = e < N ? Q[((size_t)col << n) + e] : cmake(0.0, 0.0);
    }
  };
  auto store = [&](const c128 (&x)[EL], int col) {
#pragma unroll
    for (int i = 0; i < EL; ++i) {
      const int e = lane + 64 * i;
      if (e < N) Q[((size_t)col << n) + e] = x[i];
    }
  };
  for (int pass = 0; pass < 2; ++pass) {
    c128 q[EL];
    for (int j = 0; j < c1; ++j) {
      if (w == 0 && j > c0) store(q, j - 1);  // column j - 1, scaled in the step before
      load(q, j);
      if (j >= c0) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < EL; ++i) s += cabs2(q[i]);
        const double inv = 1.0 / sqrt(bwave_all(s));
#pragma unroll
        for (int i = 0; i < EL; ++i) q[i] = cscale(q[i], inv);
      }
      for (int k = max(j + 1, c0) + w; k < c1; k += 2 * NW) {
        const int k2 = k + NW;
        const bool two = k2 < c1;
        c128 x[EL], y[EL];
        load(x, k);
        if (two) load(y, k2);
        c128 d = cmake(0.0, 0.0), f = cmake(0.0, 0.0);
#pragma unroll
        for (int i = 0; i < EL; ++i) {
          cfma(d, cconj(q[i]), x[i]);
          if (two) cfma(f, cconj(q[i]), y[i]);
        }
        d = cmake(bwave_all(d.re), bwave_all(d.im));
        if (two) f = cmake(bwave_all(f.re), bwave_all(f.im));
#pragma unroll
        for (int i = 0; i < EL; ++i) {
          x[i] = x[i] - d * q[i];
          if (two) y[i] = y[i] - f * q[i];
        }
        store(x, k);
        if (two) store(y, k2);
      }
      __syncthreads();
    }
    if (w == 0 && c1 > c0) store(q, c1 - 1);
    __syncthreads();
  }
}

__device__ void orth_columns(c128 *Q, int n, int c0, int c1) {
  if (n <= 6) orth_columns_el<1>(Q, n, c0, c1);
  else if (n == 7) orth_columns_el<2>(Q, n, c0, c1);
  else if (n == 8) orth_columns_el<4>(Q, n, c0, c1);
  else if (n == 9) orth_columns_el<8>(Q, n, c0, c1);
  else orth_columns_el<16>(Q, n, c0, c1);  // n <= 10
}

__device__ void target_columns(const BProb &P, const c128 *psi, c128 *phi, int c0, int c1) {
  const int n = P.n, N = 1 << n;
  if (P.kind == QFS_TARGET_DENSE) {
    for (uint32_t e = threadIdx.x; e < (uint32_t)(c1 - c0) * N; e += blockDim.x) {
      const int j = c0 + (int)(e >> n), row = (int)(e & (N - 1));
      c128 acc = cmake(0.0, 0.0);
      for (int col = 0; col < N; ++col) cfma(acc, P.U[(size_t)row * N + col], psi[((size_t)j << n) + col]);
      phi[((size_t)j << n) + row] = acc;
    }
    __syncthreads();
    return;
  }
  for (uint32_t e = threadIdx.x; e < (uint32_t)(c1 - c0) * N; e += blockDim.x)
    phi[((size_t)c0 << n) + e] = psi[((size_t)c0 << n) + e];
  __syncthreads();
  for (int k = 0; k < P.Lt; ++k) {
    const int pa = n - 1 - P.tpairs[2 * k], pb = n - 1 - P.tpairs[2 * k + 1];
    const c128 *u = P.tgates + (size_t)k * 16;
    const int lo = min(pa, pb), hi = max(pa, pb);
    const uint32_t ma = 1u << pa, mb = 1u << pb, gper = 1u << (n - 2);
    for (uint32_t g = threadIdx.x; g < gper * (uint32_t)(c1 - c0); g += blockDim.x) {
      const uint32_t j = c0 + (g >> (n - 2)), r = g & (gper - 1u);
      c128 *s = phi + ((size_t)j << n);
      const uint32_t i0 = deposit2(r, lo, hi);
      const uint32_t o[4] = {i0, i0 + mb, i0 + ma, i0 + ma + mb};
      c128 x[4];
      for (int p = 0; p < 4; ++p) x[p] = s[o[p]];
      for (int q = 0; q < 4; ++q) {
        c128 y = cmake(0.0, 0.0);
        for (int p = 0; p < 4; ++p) cfma(y, u[q * 4 + p], x[p]);
        s[o[q]] = y;
      }
    }
    __syncthreads();
  }
}

// Work-group (t, 0): the training set of problem todo[t]; (t, 1): its validation set (a
// SAMPLES target's two sets are copied by the first).
__global__ __launch_bounds__(kSetupBlock) void k_batch_setup(BProb *probs, const int32_t *todo, int ntodo,
                                                             const int32_t *m0s) {
  const int t = blockIdx.x;
  if (t >= ntodo) return;
  BProb &P = probs[todo[t]];
  const int n = P.n, N = 1 << n;
  const int m0 = m0s[t], m1 = P.M;
  const bool val = blockIdx.y == 1;
  if (P.kind == QFS_TARGET_SAMPLES) {
    if (val) return;
    for (uint32_t e = threadIdx.x; e < (uint32_t)(m1 - m0) * N; e += blockDim.x) {
      const size_t o = ((size_t)m0 << n) + e;
      P.psi[o] = P.s_psi[o];
      P.phi[o] = P.s_phi[o];
    }
    if (m0 == 0)
      for (uint32_t e = threadIdx.x; e < (uint32_t)P.Mv * N; e += blockDim.x) {
        P.psiv[e] = P.s_psi[((size_t)P.n_train << n) + e];
        P.phiv[e] = P.s_phi[((size_t)P.n_train << n) + e];
      }
    return;
  }
  const int c0 = val ? 0 : m0, c1 = val ? P.Mv : m1;
  if (c1 <= c0) return;
  c128 *psi = val ? P.psiv : P.psi, *phi = val ? P.phiv : P.phi;
  const uint32_t role = val ? 2u : 1u, gen = val ? (uint32_t)P.generation : 0u;
  for (uint32_t e = threadIdx.x; e < (uint32_t)(c1 - c0) * N; e += blockDim.x) {
    const int j = c0 + (int)(e >> n), i = (int)(e & (N - 1));
    psi[((size_t)j << n) + i] = complex_normal(P.seed, role, gen, (uint64_t)j * N + i);
  }
  __syncthreads();
  orth_columns(psi, n, c0, c1);
  target_columns(P, psi, phi, c0, c1);
}

// Haar 4x4 per (problem, start, gate), role 3, stream = start, index 16 gate + 4 col + row.
__global__ void k_batch_gates(BProb *probs, const int32_t *prob_of, const int32_t *first_gate,
                              int total) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  const int pidx = prob_of[t];
  const BProb &P = probs[pidx];
  const int local = t - first_gate[pidx];
  const int s = local / P.L, k = local % P.L;
  const int kind = P.kinds ? P.kinds[k] : QFS_GATE_2Q;
  c128 *u = P.g64 + ((size_t)s * P.L + k) * 16;
  c128 *v = P.vst + ((size_t)s * P.L + k) * 16;
  for (int e = 0; e < 16; ++e) v[e] = cmake((e % 5 == 0) ? 1.0 : 0.0, 0.0);
  if (kind == QFS_GATE_FIXED) {
    for (int e = 0; e < 16; ++e) u[e] = P.fixed[(size_t)k * 16 + e];
    return;
  }
  if (kind == QFS_GATE_1Q) {
    // v (x) I_2 with v Haar on U(2) from indices 16 k + 2 col + row of the same stream
    c128 h[2][2];
    for (int c = 0; c < 2; ++c)
      for (int r = 0; r < 2; ++r) h[c][r] = complex_normal(P.seed, 3u, (uint32_t)s, (uint64_t)k * 16u + 2u * c + r);
    for (int c = 0; c < 2; ++c) {
      for (int rep = 0; rep < 2; ++rep)
        for (int o = 0; o < c; ++o) {
          const c128 d = cconj(h[o][0]) * h[c][0] + cconj(h[o][1]) * h[c][1];
          for (int r = 0; r < 2; ++r) h[c][r] = h[c][r] - d * h[o][r];
        }
      const double inv = 1.0 / sqrt(cabs2(h[c][0]) + cabs2(h[c][1]));
      for (int r = 0; r < 2; ++r) h[c][r] = cscale(h[c][r], inv);
    }
    for (int r = 0; r < 4; ++r)
      for (int c = 0; c < 4; ++c) u[r * 4 + c] = ((r & 1) == (c & 1)) ? h[c >> 1][r >> 1] : cmake(0.0, 0.0);
    return;
  }
  c128 q[4][4];
  for (int c = 0; c < 4; ++c)
    for (int r = 0; r < 4; ++r) q[c][r] = complex_normal(P.seed, 3u, (uint32_t)s, (uint64_t)k * 16u + 4u * c + r);
  for (int c = 0; c < 4; ++c) {
    for (int rep = 0; rep < 2; ++rep)
      for (int o = 0; o < c; ++o) {
        c128 d = cmake(0.0, 0.0);
        for (int r = 0; r < 4; ++r) cfma(d, cconj(q[o][r]), q[c][r]);
        for (int r = 0; r < 4; ++r) q[c][r] = q[c][r] - d * q[o][r];
      }
    double nrm = 0.0;
    for (int r = 0; r < 4; ++r) nrm += cabs2(q[c][r]);
    const double inv = 1.0 / sqrt(nrm);
    for (int r = 0; r < 4; ++r) q[c][r] = cscale(q[c][r], inv);
  }
  for (int r = 0; r < 4; ++r)
    for (int c = 0; c < 4; ++c) u[r * 4 + c] = q[c][r];
}

__global__ void k_batch_move(const BMove *moves) {
  const BMove m = moves[blockIdx.x];
  for (int e = threadIdx.x; e < m.count; e += blockDim.x) m.dst[e] = m.src[e];
}

}  // namespace

// ------------------------------------------------------------------ launchers
int launch_batch_move(const BMove *moves, int count, hipStream_t s) {
  if (count <= 0) return QFS_OK;
  hipLaunchKernelGGL(k_batch_move, dim3(count), dim3(256), 0, s, moves);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

int launch_batch_setup(BProb *probs_dev, const int32_t *todo, int ntodo, const int32_t *m0s,
                       hipStream_t s) {
  if (ntodo <= 0) return QFS_OK;
  hipLaunchKernelGGL(k_batch_setup, dim3(ntodo, 2), dim3(kSetupBlock), 0, s, probs_dev, todo, ntodo, m0s);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

int launch_batch_gates(BProb *probs_dev, const int32_t *prob_of, const int32_t *first_gate, int total,
                       hipStream_t s) {
  if (total <= 0) return QFS_OK;
  hipLaunchKernelGGL(k_batch_gates, dim3((total + 127) / 128), dim3(128), 0, s, probs_dev, prob_of,
                     first_gate, total);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

template <typename R, int NT>
static int launch_sweep_t(const BatchArgs &a, int grid, size_t lds, hipStream_t s) {
  static size_t attr = 0;
  if (a.scratch) {
    hipLaunchKernelGGL((k_batch_sweep<R, NT, true>), dim3(grid), dim3(NT), 0, s, a);
  } else {
    QFS_TRY(ensure_dynamic_lds(reinterpret_cast<const void *>(&k_batch_sweep<R, NT, false>), lds, &attr));
    hipLaunchKernelGGL((k_batch_sweep<R, NT, false>), dim3(grid), dim3(NT), lds, s, a);
  }
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

int launch_batch_sweep(const BatchArgs &a, bool fp64, int threads, int grid, size_t lds, hipStream_t s) {
  if (a.njobs <= 0) return QFS_OK;
  if (fp64) {
    switch (threads) {
      case 64: return launch_sweep_t<double, 64>(a, grid, lds, s);
      case 128: return launch_sweep_t<double, 128>(a, grid, lds, s);
      case 512: return launch_sweep_t<double, 512>(a, grid, lds, s);
      default: return launch_sweep_t<double, 256>(a, grid, lds, s);
    }
  }
  switch (threads) {
    case 64: return launch_sweep_t<float, 64>(a, grid, lds, s);
    case 128: return launch_sweep_t<float, 128>(a, grid, lds, s);
    case 512: return launch_sweep_t<float, 512>(a, grid, lds, s);
    default: return launch_sweep_t<float, 256>(a, grid, lds, s);
  }
}

}  // namespace qfs
