// Operands of the triangular-normaliser forward (psi_tri.h) and its dispatch.
//
// k_tri_qr: one workgroup per site builds the folded matrix
// B = [A_0 v_0; ..; A_3 v_3] (4chi rows, chi d + 1 columns, column-major) from
// the packed parameters and takes it to upper triangular form by Householder
// reflections (backward stable: each column of R is exact for a column of B
// moved by a few ulp of its norm, the size of the rounding of the candidates
// themselves).  k_tri_pack writes the operand blocks.
#include "psi_tri.h"

namespace nqs {
namespace {

constexpr int kQrThreads = 512;

__device__ inline double wave_sum(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

__device__ inline double wave_max(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
  return x;
}

__global__ __launch_bounds__(kQrThreads) void k_tri_qr(TriBuild B) {
#pragma clang fp contract(off)
  __shared__ double v[256];
  __shared__ double s_tau;
  const int i = blockIdx.x, chi = B.chi, tid = threadIdx.x;
  const int e0 = B.pptr[i], d = B.pptr[i + 1] - e0;
  const int rows = 4 * chi, cols = chi * d + 1;
  double* G = B.G + int64_t(i) * B.gstride;
  const double* eta = B.prm + B.offEta[i];
  for (int x = tid; x < rows * cols; x += kQrThreads) {
    const int c = x / rows, r = x % rows, s = r / chi, u = r % chi;
    const double su = sqrt(eta[u]);
    double val;
    if (c == cols - 1) {
      val = su * B.prm[B.offV[i] + s * chi + u];
    } else {
      const int e = e0 + c / chi, k = c % chi;
      val = su * B.prm[B.offM[e] + (int64_t(s) * chi + u) * chi + k] / sqrt(B.prm[B.offEta[B.pidx[e]] + k]);
    }
    G[int64_t(c) * rows + r] = val;
  }
  __syncthreads();
  const int wv = tid >> 6, lane = tid & 63, nw = kQrThreads / 64;
  const int steps = rows - 1 < cols ? rows - 1 : cols;
  for (int k = 0; k < steps; ++k) {
    if (wv == 0) {
      double* a = G + int64_t(k) * rows;
      double ss = 0.0;
      for (int r = k + lane; r < rows; r += 64) {
        v[r] = a[r];
        ss = tfma(a[r], a[r], ss);
      }
      ss = wave_sum(ss);
      // the squares of entries beyond 1e+-154, and the products of v with other columns
      // long before, leave the range of a double: a column far from 1 is taken times a
      // power of two that brings its largest entry to [1/2, 1) (the reflection does not
      // depend on v's length)
      int ex = 0;
      if (!(ss > 1e-40 && ss < 1e40)) {
        double big = 0.0;
        for (int r = k + lane; r < rows; r += 64) big = fmax(big, fabs(a[r]));
        (void)frexp(wave_max(big), &ex);
        ss = 0.0;
        for (int r = k + lane; r < rows; r += 64) {
          v[r] = ldexp(a[r], -ex);
          ss = tfma(v[r], v[r], ss);
        }
        ss = wave_sum(ss);
      }
      const double a0 = ldexp(a[k], -ex), nrm = sqrt(ss);
      // v = a -+ |a| e_k, H = 1 - tau v v^T with tau = 2 / v^T v
      const double beta = a0 < 0.0 ? nrm : -nrm;
      const double vv = 2.0 * (ss - a0 * beta);
      if (lane == 0) {
        v[k] = a0 - beta;
        s_tau = vv > 0.0 ? 2.0 / vv : 0.0;
        if (vv > 0.0) a[k] = ldexp(beta, ex);
      }
    }
    __syncthreads();
    const double tau = s_tau;
    if (tau > 0.0)
      for (int c = k + 1 + wv; c < cols; c += nw) {
        double* a = G + int64_t(c) * rows;
        double x[4], dot = 0.0;
        int q = 0;
#pragma unroll
        for (q = 0; q < 4; ++q) {
          const int r = k + lane + 64 * q;
          x[q] = r < rows ? a[r] : 0.0;
          if (r < rows) dot = tfma(v[r], x[q], dot);
        }
        dot = wave_sum(dot) * tau;
#pragma unroll
        for (q = 0; q < 4; ++q) {
          const int r = k + lane + 64 * q;
          if (r < rows) a[r] = tfma(-dot, v[r], x[q]);
        }
      }
    __syncthreads();
  }
}

// one workgroup of 64 threads per (block of the stream, site)
__global__ __launch_bounds__(64) void k_tri_pack(TriBuild B, TriParams P, double* Q, double* rho) {
#pragma clang fp contract(off)
  const int i = blockIdx.y, chi = B.chi, CH = B.chip, TPC = CH / 16;
  const int e0 = B.pptr[i], d = B.pptr[i + 1] - e0, df = d > 0 ? d : 1;
  const int n = df * TPC, RP = tri_rp(CH), rows = 4 * chi, cols = chi * d + 1;
  const int LR = tri_lr(CH, df), LC = tri_lc(CH, df);
  const double* G = B.G + int64_t(i) * B.gstride;
  // column of B (row of R) at padded position p; -1: padding
  auto col = [&](int p) { return p / CH < d && p % CH < chi ? (p / CH) * chi + p % CH : -1; };
  const int b = blockIdx.x, l = threadIdx.x;
  if (b == 0) {
    double* V = Q + P.vofs / 8 + size_t(i) * (P.dmax + 6) * CH;
    const double* eta = B.prm + B.offEta[i];
    for (int p = l; p < P.dmax * CH; p += 64) {
      const int r = col(p);
      V[p] = r >= 0 && r < rows ? G[int64_t(cols - 1) * rows + r] : 0.0;
    }
    V += P.dmax * CH;
    for (int p = l; p < 4 * CH; p += 64)
      V[p] = p % CH < chi ? sqrt(eta[p % CH]) * B.prm[B.offV[i] + (p / CH) * chi + p % CH] : 0.0;
    V += 4 * CH;
    for (int u = l; u < CH; u += 64) {
      V[u] = u < chi ? eta[chi + u] / sqrt(eta[u]) : 0.0;
      V[CH + u] = u < chi && B.offW2 ? B.prm[B.offW2[i] + u] / sqrt(eta[u]) : 0.0;
    }
    if (l == 0) {
      const double x = cols - 1 < rows ? G[int64_t(cols - 1) * rows + cols - 1] : 0.0;
      rho[i] = x * x;
    }
  }
  if (b >= LR + 4 * LC) return;
  // the block's (row tile, column tile) in its part, by the kernel's order
  const int s = b < LR ? -1 : (b - LR) / LC;
  const int want = b < LR ? b : (b - LR) % LC, nr = s < 0 ? n : TPC;
  int rt = -1, ct = -1, at = 0;
  for (int r0 = 0; r0 < nr; r0 += RP)
    for (int kt = s < 0 ? r0 : 0; kt < n; ++kt)
      for (int r = r0; r < r0 + RP && r < nr; ++r)
        if (s >= 0 || kt >= r) {
          if (at == want) { rt = r; ct = kt; }
          ++at;
        }
  const int mrow = l & 15;
  const int row = 16 * rt + 4 * (mrow & 3) + (mrow >> 2);
  double* q = Q + (int64_t(P.qoff[i]) + b) * 256 + 4 * l;
  for (int v = 0; v < 4; ++v) {
    double val = 0.0;
    if (rt >= 0) {
      const int cp = 16 * ct + 4 * (l >> 4) + v, c = col(cp);
      if (c >= 0 && s < 0) {
        const int r = col(row);
        if (r >= 0 && r <= c && r < rows) val = G[int64_t(c) * rows + r];
      } else if (c >= 0 && row < chi) {
        const int e = e0 + cp / CH, k = cp % CH;
        val = sqrt(B.prm[B.offEta[i] + row]) * B.prm[B.offM[e] + (int64_t(s) * chi + row) * chi + k] /
              sqrt(B.prm[B.offEta[B.pidx[e]] + k]);
      }
    }
    q[v] = val;
  }
}

}  // namespace

hipError_t launch_tri_build(const TriBuild& B, const TriParams& P, double* Q, double* rho,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_tri_qr, dim3(P.K), dim3(kQrThreads), 0, st, B);
  hipLaunchKernelGGL(k_tri_pack, dim3(tri_site_blocks(B.chip, P.dmax), P.K), dim3(64), 0, st, B, P, Q, rho);
  return hipGetLastError();
}

namespace {

template <typename T>
hipError_t dispatch_tri(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi, hipStream_t st,
                        const PsiStates<T>& states, int mode, double* phs) {
  if (R <= 0) return hipSuccess;
  PsiStates<T> X = states;
  if (mode == PSI_STORE || mode == PSI_ROWS) X.perm = nullptr;   // the kernel takes a null order as rows from site 0
  const bool resumed = mode == PSI_SEED || mode == PSI_NODE;
  if ((mode == PSI_STORE && !X.pm) || (resumed && !X.perm)) return hipErrorInvalidValue;
  if (mode == PSI_ROWS && sizeof(T) == 8 && (!X.owner || !X.samples)) return hipErrorInvalidValue;
  if (phs && (!P.c2 || ((resumed || mode == PSI_STORE) && !X.pz) ||
              (((resumed && X.unode) || mode == PSI_NODE) && !X.npz)))
    return hipErrorInvalidValue;
  switch (P.chip) {
    case 16: return launch_tri_16(P, m, R, lphi, sphi, st, X, mode, phs);
    case 32: return launch_tri_32(P, m, R, lphi, sphi, st, X, mode, phs);
    case 48: return launch_tri_48(P, m, R, lphi, sphi, st, X, mode, phs);
    case 64: return launch_tri_64(P, m, R, lphi, sphi, st, X, mode, phs);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_psi_tri(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi,
                          hipStream_t st, const PsiStates<double>& X, int mode, double* phs) {
  return dispatch_tri(P, m, R, lphi, sphi, st, X, mode, phs);
}
hipError_t launch_psi_tri(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi,
                          hipStream_t st, const PsiStates<float>& X, int mode, double* phs) {
  return dispatch_tri(P, m, R, lphi, sphi, st, X, mode, phs);
}

}  // namespace nqs
