// FP64 4x4 unitary polar factor on one wave, shared by the per-gate and the grouped
// backward passes (sweep.hip, group.hip).
#pragma once

#include "qfs_internal.h"

namespace qfs {

// ------------------------------------------------------------------ FP64 4x4 polar
// One-sided (Hestenes) Jacobi on one wave: lane l = 4c + r (of each 16-lane group)
// holds column c, row r of the working matrix G and of V. Each round rotates the two
// disjoint column pairs c <-> c ^ (m >> 2), m in {4, 8, 12}; the pair's Gram entries
// are summed over the four rows of a quad, so both columns' lanes compute bitwise
// equal rotations. Then W = normalised columns of G (re-orthonormalised and completed
// when a singular value is negligible) and u = W V^dagger.
//
// Warm start (vstore != nullptr): Jacobi starts from G V_prev and V_prev, the right
// singular vectors this gate had after its previous update (the environment changes
// little between sweeps), so it converges in one or two sweeps instead of ~6. V_prev is
// first made unitary to rounding by one Newton-Schulz step V (3I - V^dag V) / 2, so no
// error accumulates across sweeps; the new V is stored back.
__device__ __forceinline__ c128 shfl_c(c128 x, int src) {
  return cmake(__shfl(x.re, src), __shfl(x.im, src));
}

// Exchange between the lanes of a 16-lane row by DPP moves (no trip through the LDS
// crossbar): lane i receives lane i ^ M's value, M in {1, 2, 4, 8, 12}. xor 1 and 2 are quad
// permutations, xor 8 the rotation of the row by 8, xor 4 the reversal of each half row
// followed by the reversal of each quad.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
template <int M>
__device__ __forceinline__ double xor_lane(double x) {
  if constexpr (M == 1) {
    return dpp_move<0xB1>(x);  // quad_perm [1, 0, 3, 2]
  } else if constexpr (M == 2) {
    return dpp_move<0x4E>(x);  // quad_perm [2, 3, 0, 1]
  } else if constexpr (M == 8) {
    return dpp_move<0x128>(x);  // row_ror:8
  } else if constexpr (M == 4) {
    return dpp_move<0x1B>(dpp_move<0x141>(x));  // row_half_mirror, then quad_perm [3, 2, 1, 0]
  } else {
    static_assert(M == 12, "lane exchange within a row");
    return xor_lane<8>(xor_lane<4>(x));
  }
}

__device__ __forceinline__ c128 quad_sum(c128 x) {
  x.re += xor_lane<1>(x.re);
  x.im += xor_lane<1>(x.im);
  x.re += xor_lane<2>(x.re);
  x.im += xor_lane<2>(x.im);
  return x;
}

// 1/sqrt(x) and 1/x from the hardware estimates, each refined by two Newton steps (about
// one ulp; the rotations below need cs^2 + sn^2 = 1 and |e| = 1 to rounding, not the
// correctly rounded values, and the estimates shorten their dependent chain).
__device__ __forceinline__ double rsq_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  y = y * fma(-hx * y, y, 1.5);
  y = y * fma(-hx * y, y, 1.5);
  return y;
}
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  double e = fma(-x, y, 1.0);
  y = fma(y, e, y);
  e = fma(-x, y, 1.0);
  return fma(y, e, y);
}

// One round of the one-sided Jacobi below: the column pairs c <-> c ^ (M >> 2).
template <int M>
__device__ __forceinline__ void jacobi_round(int l, c128 &g, c128 &v, int &large) {
  const c128 go = cmake(xor_lane<M>(g.re), xor_lane<M>(g.im));
  const c128 vo = cmake(xor_lane<M>(v.re), xor_lane<M>(v.im));
  const bool is_p = (l ^ M) > l;
  const c128 gp = is_p ? g : go, gq = is_p ? go : g;
  const c128 vp = is_p ? v : vo, vq = is_p ? vo : v;
  double al = cabs2(gp), be = cabs2(gq);
  double gr = gp.re * gq.re + gp.im * gq.im;  // conj(gp) * gq
  double gi = gp.re * gq.im - gp.im * gq.re;
  al += xor_lane<1>(al);
  be += xor_lane<1>(be);
  gr += xor_lane<1>(gr);
  gi += xor_lane<1>(gi);
  al += xor_lane<2>(al);
  be += xor_lane<2>(be);
  gr += xor_lane<2>(gr);
  gi += xor_lane<2>(gi);
  // |Gram_pq|^2 against the product of the column norms squared: rotate when |Gram_pq| >
  // 1e-15 sqrt(al be), and count the round as large above 1e-7 sqrt(al be)
  const double x2 = gr * gr + gi * gi, ab = al * be;
  if (x2 > 1e-30 * ab) {
    large |= x2 > 1e-14 * ab;
    const double rag = rsq_nr(x2);  // 1 / |Gram_pq|
    const c128 ec = cmake(gr * rag, -gi * rag);  // conj(e^{i phi})
    const double tau = (be - al) * (0.5 * rag);
    const double t1 = fma(tau, tau, 1.0);
    const double tt = (tau >= 0.0 ? 1.0 : -1.0) * rcp_nr(fabs(tau) + t1 * rsq_nr(t1));
    const double cs = rsq_nr(fma(tt, tt, 1.0)), sn = cs * tt;
    const c128 egq = ec * gq, evq = ec * vq;
    if (is_p) {
      g = cmake(cs * gp.re - sn * egq.re, cs * gp.im - sn * egq.im);
      v = cmake(cs * vp.re - sn * evq.re, cs * vp.im - sn * evq.im);
    } else {
      g = cmake(sn * gp.re + cs * egq.re, sn * gp.im + cs * egq.im);
      v = cmake(sn * vp.re + cs * evq.re, sn * vp.im + cs * evq.im);
    }
  }
}

// Entry (r, c + J) of the matrix for lane 4c + r (columns cyclic): the 16-lane row rotated
// left by 4 J (row_ror moves right). Entry (r + I, c): a rotation of each quad.
template <int J>
__device__ __forceinline__ c128 col_rot(c128 x) {
  return cmake(dpp_move<0x120 + 16 - 4 * J>(x.re), dpp_move<0x120 + 16 - 4 * J>(x.im));
}
template <int I>
__device__ __forceinline__ c128 row_rot(c128 x) {
  constexpr int q = I == 1 ? 0x39 : I == 2 ? 0x4E : 0x93;  // quad_perm [I, I+1, I+2, I+3] mod 4
  return cmake(dpp_move<q>(x.re), dpp_move<q>(x.im));
}
__device__ __forceinline__ double first_lane(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double row4_sum(double x) {  // over the columns c
  x += dpp_move<0x124>(x);
  return x + dpp_move<0x128>(x);
}
__device__ __forceinline__ double row16_sum(double x) {
  x = row4_sum(x);
  x += xor_lane<1>(x);
  return x + xor_lane<2>(x);
}
__device__ __forceinline__ double row16_max(double x) {
  x = fmax(x, xor_lane<1>(x));
  x = fmax(x, xor_lane<2>(x));
  x = fmax(x, xor_lane<4>(x));
  return fmax(x, xor_lane<8>(x));
}

// Unitary polar factor of a well-conditioned 4x4 matrix by the scaled Newton iteration
// (Higham, Functions of Matrices, Sec. 8.6): X <- (g X + X^-H / g) / 2, g = (|X^-1|_F /
// |X|_F)^(1/2), which keeps the polar factor and squares the distance to it. Lane 4c + r of
// every 16-lane row holds entry (r, c). X^-H[r][c] = conj(cof[r][c] / det), and a lane forms
// its cofactor from the nine entries of the three other rows and columns, taken in cyclic
// order (a rotation of three is even, so the sign is that of r + c) by DPP moves: no LDS, no
// barrier, one reciprocal per iteration. Bound by the issue of one wave (about 150
// instructions, 700 cycles an iteration, five or six iterations). Against the Jacobi SVD of
// every matrix: 64 updates in one launch 7.1 -> 4.2 us, the finalize of a group of two gates
// (8 qubits, cold start) 14.0 -> 9.3 us.
// Returns false, x undefined, when |X|_F |X^-1|_F exceeds 64 in the first iteration: cofactors
// lose digits with the square of the condition number (largest error of the factor at 16, 64, 200
// and 640: 1e-15, 1.2e-14, 9e-14, 1.1e-12, where an SVD's is 9e-15, 9e-15, 1.7e-14, 5e-14), and
// the SVD takes those, singular matrices, and extreme scales.
__device__ __forceinline__ bool polar4_newton(int l, c128 &x) {
  const double sgn = ((l ^ (l >> 2)) & 1) ? -1.0 : 1.0;
  for (int it = 0; it < 16; ++it) {
    const c128 z1 = col_rot<1>(x), z2 = col_rot<2>(x), z3 = col_rot<3>(x);
    const c128 m00 = row_rot<1>(z1), m01 = row_rot<1>(z2), m02 = row_rot<1>(z3);
    const c128 m10 = row_rot<2>(z1), m11 = row_rot<2>(z2), m12 = row_rot<2>(z3);
    const c128 m20 = row_rot<3>(z1), m21 = row_rot<3>(z2), m22 = row_rot<3>(z3);
    c128 cof = m00 * (m11 * m22 - m12 * m21);
    cfma(cof, m01, m12 * m20 - m10 * m22);
    cfma(cof, m02, m10 * m21 - m11 * m20);
    cof = cmake(sgn * cof.re, sgn * cof.im);
    c128 det = x * cof;
    det.re = row4_sum(det.re);
    det.im = row4_sum(det.im);
    const double d2 = cabs2(det);
    const double id2 = rcp_nr(d2);
    const c128 w = cmake((cof.re * det.re + cof.im * det.im) * id2, (cof.re * det.im - cof.im * det.re) * id2);
    const double e = cabs2(x - w);
    double g = 0.5, gi = 0.5;
    const bool far = __any(e > 1e-3);
    if (it == 0 || far) {
      const double n1 = row16_sum(cabs2(x)), n2 = row16_sum(cabs2(w));
      if (it == 0) {
        // (of a matrix of rank two or less, cofactors and determinant are rounding errors of
        // one size, and the quotient says nothing: the cofactors are held to the entries' cube)
        const double nc = n2 * d2;
        if (__any(!(d2 > 1e-280 && d2 < 1e280 && n1 * n2 <= 4096.0 && nc > 1e-10 * (n1 * n1 * n1)))) return false;
      }
      // far from unitary: scaled. Any positive factors keep the polar factor, so the hardware estimates do; they must
      // be the same on every lane (the lanes' sums differ in rounding, and an estimate of
      // inputs one ulp apart may differ by 1e-9)
      if (far) {
        const double ratio = first_lane(n2 * __builtin_amdgcn_rcp(n1));
        const double y = __builtin_amdgcn_rsq(ratio), f = __builtin_amdgcn_rsq(y);
        g = 0.5 * f;
        gi = 0.5 * f * y;
      }
    }
    x = cmake(g * x.re + gi * w.re, g * x.im + gi * w.im);
    // entries of X within 5e-9 of unitary before the step: to rounding after it
    if (!__any(e > 1e-16)) return true;
  }
  return false;
}

// The polar factor of (1 - beta) G + beta u_prev: polar4_newton where it may, else the
// Jacobi SVD.
template <typename R>
__device__ __forceinline__ void polar4_wave(const c128 *G, double beta, const c128 *u_prev, c128 *out64,
                            cx<R> *out32, c128 *lds_g, c128 *lds_v, double *lds_s,
                            c128 *vstore = nullptr) {
  const int lane = threadIdx.x & 63;
  const int l = lane & 15, c = l >> 2, r = l & 3, base = lane & ~15;
  double scale = 1.0;
  auto gm = [&](int row, int col) {
    c128 x = G[row * 4 + col];
    if (beta != 0.0) {
      const c128 up = u_prev[row * 4 + col];
      x = cmake((1.0 - beta) * x.re + beta * up.re, (1.0 - beta) * x.im + beta * up.im);
    }
    return cscale(x, scale);
  };
  c128 g, v;
  {
    c128 x = gm(r, c);
    if (polar4_newton(l, x)) {
      if (lane < 16) {
        out64[r * 4 + c] = x;
        if (out32) out32[r * 4 + c] = cmake<R>((R)x.re, (R)x.im);
      }
      return;
    }
    // the Jacobi forms fourth powers of the entries: scaled by a power of two (exact, and the
    // polar factor does not change) where those leave the range of a double (a subnormal entry
    // asks for more than the largest power of two; 2^1000 brings it far enough)
    const c128 x0 = gm(r, c);
    const double big = row16_max(fmax(fabs(x0.re), fabs(x0.im)));
    if (big > 1e60 || big < 1e-60) scale = big > 0.0 ? ldexp(1.0, min(-ilogb(big), 1000)) : 1.0;
  }
  if (vstore) {
    // lane 4c + r holds X[r][c]; Y[a][c] = sum_k conj(X[k][a]) X[k][c] (quad c);
    // Z[r][c] = (3 X[r][c] - sum_a X[r][a] Y[a][c]) / 2
    const c128 x = vstore[r * 4 + c];
    c128 acc = cmake(0.0, 0.0);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const c128 xca = shfl_c(x, base + 4 * a + r);  // X[r][a]
      const c128 yac = quad_sum(cconj(xca) * x);     // Y[a][c]
      cfma(acc, xca, yac);
    }
    v = cmake(0.5 * (3.0 * x.re - acc.re), 0.5 * (3.0 * x.im - acc.im));
    g = cmake(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 4; ++k) cfma(g, gm(r, k), shfl_c(v, base + 4 * c + k));  // (G V)[r][c]
  } else {
    g = gm(r, c);
    v = cmake(r == c ? 1.0 : 0.0, 0.0);
  }
  // Cyclic Jacobi converges quadratically: a sweep whose rotations all started from a
  // relative off-diagonal Gram entry below 1e-7 leaves them at the 1e-14 level, so the
  // iteration stops after it instead of running a further sweep that rotates nothing.
  bool converged = false;
  for (int sweep = 0; sweep < 40; ++sweep) {
    int large = 0;
    jacobi_round<4>(l, g, v, large);
    jacobi_round<8>(l, g, v, large);
    jacobi_round<12>(l, g, v, large);
    if (!__any(large)) {
      converged = true;
      break;
    }
  }
  double s2 = cabs2(g);
  s2 += xor_lane<1>(s2);
  s2 += xor_lane<2>(s2);
  const double sig = sqrt(s2);
  double smin = sig, smax = sig;
  smin = fmin(smin, xor_lane<4>(smin));
  smin = fmin(smin, xor_lane<8>(smin));
  smax = fmax(smax, xor_lane<4>(smax));
  smax = fmax(smax, xor_lane<8>(smax));
  if (converged && smin > 1e-200 && smin > 1e-15 * smax) {
    // W = G diag(1/sigma) is unitary to the Jacobi tolerance; u = W V^dagger with
    // lane 4q + p computing u[q][p] = sum_k W[q][k] conj(V[p][k]); W[q][k] and V[p][k]
    // live on lanes 4k + q and 4k + p.
    const c128 w = cscale(g, 1.0 / sig);
    const int q = l >> 2, p = l & 3, base = lane & ~15;
    c128 acc = cmake(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int lw = base + 4 * k + q, lv = base + 4 * k + p;
      const c128 wk = cmake(__shfl(w.re, lw), __shfl(w.im, lw));
      const c128 vk = cmake(__shfl(v.re, lv), __shfl(v.im, lv));
      cfma_conj(acc, wk, vk);
    }
    if (lane < 16) {
      out64[l] = acc;
      if (out32) out32[l] = cmake<R>((R)acc.re, (R)acc.im);
      if (vstore) vstore[r * 4 + c] = v;
    }
    return;
  }
  // Rank-deficient (or unconverged) case: lane 0 orders the columns by singular value,
  // re-orthonormalises them and completes W with unit vectors where sigma vanishes.
  if (lane < 16) {
    lds_g[c * 4 + r] = g;
    lds_v[c * 4 + r] = v;
    if (r == 0) lds_s[c] = sig;
    if (vstore) vstore[r * 4 + c] = v;
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) {
    // everything stays in LDS and the loops stay rolled: this path is rare, and its registers
    // would count for the whole kernel
    int ord = 0xE4;  // column of the k-th largest singular value at bits 2k, 2k + 1
#pragma unroll 1
    for (int a = 0; a < 4; ++a)
#pragma unroll 1
      for (int b = a + 1; b < 4; ++b) {
        const int ca = (ord >> (2 * a)) & 3, cb = (ord >> (2 * b)) & 3;
        if (lds_s[cb] > lds_s[ca]) ord ^= ((ca ^ cb) << (2 * a)) | ((ca ^ cb) << (2 * b));
      }
    auto col = [&](int k) { return lds_g + 4 * ((ord >> (2 * k)) & 3); };
    // x <- x minus its components along the first k columns, twice; returns |x|^2
    auto orth = [&](c128 (&x)[4], int k) {
#pragma unroll 1
      for (int i = 0; i < 2 * k; ++i) {
        const c128 *w = col(i < k ? i : i - k);
        c128 d = cmake(0.0, 0.0);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) cfma(d, cconj(w[rr]), x[rr]);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) x[rr] = x[rr] - d * w[rr];
      }
      return ((cabs2(x[0]) + cabs2(x[1])) + (cabs2(x[2]) + cabs2(x[3])));
    };
    const double sm = lds_s[ord & 3];
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
      c128 *wk = col(k);
      const double sk = lds_s[(ord >> (2 * k)) & 3];
      c128 x[4];
      double nn = 0.0;
      if (sk > 0.0 && sk > 1e-13 * sm) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) x[rr] = cscale(wk[rr], 1.0 / sk);
        nn = orth(x, k);
      }
      if (!(nn > 0.25)) {  // complete with the unit vector of largest orthogonal remainder
        int pick = 0;
        double best = -1.0;
#pragma unroll 1
        for (int e = 0; e < 5; ++e) {
          const int at = e < 4 ? e : pick;
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) x[rr] = cmake(rr == at ? 1.0 : 0.0, 0.0);
          nn = orth(x, k);
          if (e < 4 && nn > best) {
            best = nn;
            pick = e;
          }
        }
      }
      const double inv = 1.0 / sqrt(nn);
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) wk[rr] = cscale(x[rr], inv);
    }
#pragma unroll 1
    for (int e = 0; e < 16; ++e) {
      c128 acc = cmake(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 4; ++k) cfma_conj(acc, lds_g[k * 4 + (e >> 2)], lds_v[k * 4 + (e & 3)]);
      out64[e] = acc;
      if (out32) out32[e] = cmake<R>((R)acc.re, (R)acc.im);
    }
  }
}

}  // namespace qfs
