// Parameter layouts of an ansatz, made on the device from the packed vector
// (nqs_ansatz_bind_params).  A VMC step binds once per update, so this is on its
// path: building the layouts on the host (with a download, a dozen uploads and
// reallocations per precision) took 2.5 of the 7.5 ms of a K = 20, chi = 16 step
// with the Ising-RBM.  Every kernel here writes each entry of its output, from at
// most three parameters, so they are bound by the writes (a few MB).
#include "internal.h"
#include <cmath>

namespace nqs {
namespace {

// forward edge fe -> its site and its edge of the graph (-1: a parentless site's
// zero edge, or the fetch-ahead edge past the last)
__device__ inline void forward_edge(const PackParams& P, int fe, int& site, int& edge) {
  int i = 0;
  while (i + 1 < P.K && P.fptr[i + 1] <= fe) ++i;
  site = i;
  edge = fe < P.fptr[P.K] && P.pptr[i + 1] > P.pptr[i] ? P.pptr[i] + (fe - P.fptr[i]) : -1;
}

// sigma_i[u] M_ij^s[u][k] / sigma_j[k] with sigma = sqrt(eta) (fold) or 1
__device__ inline double edge_value(const PackParams& P, int site, int edge, int s, int u, int k) {
#pragma clang fp contract(off)
  const double M = P.prm[P.offM[edge] + (int64_t(s) * P.chi + u) * P.chi + k];
  if (!P.fold) return M;
  return sqrt(P.prm[P.offEta[site] + u]) * M / sqrt(P.prm[P.offEta[P.pidx[edge]] + k]);
}

// A: forward MFMA operands per forward edge, [k-step q][output tile ot][lane]:
// lane l holds W^T[o][k] = M_ij^s[u][k] with s = o / chip, u = o % chip (zero
// outside chi), tile row m = l%16 and parent unit k = 16 (q/4) + 4 (l/16) + q%4.
// The 16x16x4 f32 MFMA returns row m = 4 g + v of the tile in register v of lane
// group g = l/16, the f64 MFMA row m = g + 4 v: tile row m therefore carries unit
// o = 16 ot + m for f32 and o = 16 ot + 4 (m%4) + m/4 for f64, so that lane group g
// ends up with units 16 ot + 4 g + v, and k-step q of lane group g reads the parent
// unit that the same lane produced in register q%4 of output tile q/4.
// AF, BT (unfolded layout only, per graph edge): the adjoint's operands.  AF is A;
// BT: k-step q = (s*TPC + t)*4 + v over the candidate units (s, 16t + 4k' + v) and
// output tiles ot over the parent unit kk = 16 ot + n: B[k'][n] = M_ij^s[u][kk].
template <typename T>
__global__ __launch_bounds__(256) void k_pack_edges(PackParams P, T* A, T* AF, T* BT) {
  const int CH = P.chip, KS = CH / 4, NT = CH / 4, TPC = CH / 16;
  const int64_t ES = int64_t(KS) * NT * 64;
  const int64_t x = int64_t(blockIdx.x) * 256 + threadIdx.x;
  int site, edge;
  forward_edge(P, blockIdx.y, site, edge);
  if (x >= ES) return;
  const int l = int(x & 63), mrow = l & 15;
  {
    const int q = int(x / (NT * 64)), ot = int(x / 64) % NT;
    const int o = ot * 16 + (sizeof(T) == 8 ? 4 * (mrow & 3) + (mrow >> 2) : mrow);
    const int k = 16 * (q >> 2) + 4 * (l >> 4) + (q & 3);
    const int s = o / CH, u = o % CH;
    const T val = edge >= 0 && u < P.chi && k < P.chi ? T(edge_value(P, site, edge, s, u, k)) : T(0);
    A[int64_t(blockIdx.y) * ES + x] = val;
    if (AF && edge >= 0) AF[int64_t(edge) * ES + x] = val;
  }
  if (BT && edge >= 0) {
    const int q = int(x / (TPC * 64)), ot = int(x / 64) % TPC;
    const int v = q & 3, t = (q >> 2) % TPC, s = (q >> 2) / TPC;
    const int u = 16 * t + 4 * (l >> 4) + v, kk = 16 * ot + mrow;
    BT[int64_t(edge) * ES + x] = u < P.chi && kk < P.chi ? T(edge_value(P, site, edge, s, u, kk)) : T(0);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_pack_sites(PackParams P, T* v, T* eta, T* w, T* c, T* w2, T* c2) {
#pragma clang fp contract(off)
  const int i = blockIdx.x, CH = P.chip, chi = P.chi;
  const double* e = P.prm + P.offEta[i];   // eta, then w, then c
  for (int x = threadIdx.x; x < 4 * CH; x += 256) {
    const int s = x / CH, u = x % CH;
    double val = 0.0;
    if (u < chi) {
      val = P.prm[P.offV[i] + s * chi + u];
      if (P.fold) val = sqrt(e[u]) * val;
    }
    v[int64_t(i) * 4 * CH + x] = T(val);
  }
  for (int u = threadIdx.x; u < CH; u += 256) {
    const double sg = u < chi && P.fold ? sqrt(e[u]) : 1.0;
    eta[int64_t(i) * CH + u] = u < chi ? T(e[u]) : T(0);
    w[int64_t(i) * CH + u] = u < chi ? T(e[chi + u] / sg) : T(0);
    if (w2) w2[int64_t(i) * CH + u] = u < chi ? T(P.prm[P.offW2[i] + u] / sg) : T(0);
  }
  if (threadIdx.x == 0) {
    c[i] = T(e[2 * chi]);
    if (c2) c2[i] = T(P.prm[P.offW2[i] + chi]);
  }
}

__device__ inline uint16_t to_bf16(float f) {
  uint32_t b = __float_as_uint(f);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return uint16_t(b >> 16);
}

// BF16 forward A stream (psi_bf16.hip): per forward edge, TPC/2 pair k-steps of
// [output tile ot][lane][8] then, when TPC = chip/16 is odd, one k-step of
// [ot][lane][4].  Lane l holds tile row m = l%16 (output unit o = 16 ot + m, the
// FP32 output layout) and, for lane group g = l/16, the parent units
// k = 16 (2q + e/4) + 4 g + e%4 (pair step q, element e) or 16 (TPC-1) + 4 g + e
// (odd step): each lane's own quads of the parent state.  Round to nearest
// even; the lo stream holds bf16(x - bf16(x)), the difference taken in FP64.
__global__ __launch_bounds__(256) void k_pack_bf16(PackParams P, uint16_t* A, uint16_t* Alo) {
  const int CH = P.chip, NT = CH / 4, TPC = CH / 16, NP = TPC / 2;
  const int64_t EP = int64_t(NP) * NT * 64 * 8, EQ = EP + int64_t(TPC & 1) * NT * 64 * 4;
  const int64_t x = int64_t(blockIdx.x) * 256 + threadIdx.x;
  int site, edge;
  forward_edge(P, blockIdx.y, site, edge);
  if (x >= EQ) return;
  int ot, l, k;
  if (x < EP) {
    const int el = int(x & 7), q = int(x / (int64_t(NT) * 512));
    l = int(x >> 3) & 63;
    ot = int(x / 512) % NT;
    k = 16 * (2 * q + el / 4) + 4 * (l >> 4) + el % 4;
  } else {
    const int64_t y = x - EP;
    const int el = int(y & 3);
    l = int(y >> 2) & 63;
    ot = int(y / 256);
    k = 16 * (TPC - 1) + 4 * (l >> 4) + el;
  }
  const int o = 16 * ot + (l & 15), s = o / CH, u = o % CH;
  uint16_t hi = 0, lo = 0;
  if (edge >= 0 && u < P.chi && k < P.chi) {
    const double v = edge_value(P, site, edge, s, u, k);
    hi = to_bf16(float(v));
    lo = to_bf16(float(v - double(__uint_as_float(uint32_t(hi) << 16))));
  }
  A[int64_t(blockIdx.y) * EQ + x] = hi;
  Alo[int64_t(blockIdx.y) * EQ + x] = lo;
}

// The FP32 rows' stream (psi_tri.h): per site, candidate s, unit tile tt and parent
// tile kt one block [lane][4]: lane l holds row 16 tt + l % 16 and columns
// 16 kt + 4 (l / 16) + 0..3; block 0 of a site also writes its vectors.  One
// workgroup per (block, site).
__global__ __launch_bounds__(64) void k_pack_tri32(PackParams P, const int* qoff, int dmax, float* Q, int vofs) {
#pragma clang fp contract(off)
  const int i = blockIdx.y, CH = P.chip, TPC = CH / 16, b = blockIdx.x, l = threadIdx.x;
  const int d = P.pptr[i + 1] - P.pptr[i], n = (d > 0 ? d : 1) * TPC, LC = tri_lc32(CH, d > 0 ? d : 1);
  if (b == 0) {
    float* V = Q + vofs / 4 + int64_t(i) * 6 * CH;
    const double* e = P.prm + P.offEta[i];
    for (int x = l; x < 4 * CH; x += 64) {
      const int u = x % CH;
      V[x] = u < P.chi ? float(sqrt(e[u]) * P.prm[P.offV[i] + (x / CH) * P.chi + u]) : 0.0f;
    }
    for (int u = l; u < CH; u += 64) {
      V[4 * CH + u] = u < P.chi ? float(e[P.chi + u] / sqrt(e[u])) : 0.0f;
      V[5 * CH + u] = u < P.chi && P.offW2 ? float(P.prm[P.offW2[i] + u] / sqrt(e[u])) : 0.0f;
    }
  }
  if (b >= 4 * LC) return;
  const int s = b / LC, t = b % LC, tt = t / n, kt = t % n;
  const int u = 16 * tt + (l & 15);
  for (int v = 0; v < 4; ++v) {
    const int p = 16 * kt + 4 * (l >> 4) + v, e = p / CH, k = p % CH;
    const bool in = t < TPC * n && e < d && k < P.chi && u < P.chi;
    Q[(int64_t(qoff[i]) + b) * 256 + 4 * l + v] = in ? float(edge_value(P, i, P.pptr[i] + e, s, u, k)) : 0.0f;
  }
}

// the correlator's W transposed (hidden unit fastest: [P][k])
__global__ __launch_bounds__(256) void k_pack_wt(int nv, int nh, const double* W, double* Wt) {
  const int64_t x = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (x >= int64_t(nv) * nh) return;
  Wt[x] = W[(x % nh) * nv + x / nh];
}

// S [P][Q][k] = (W2[k][P][Q] + W2[k][Q][P]) / 2, in FP64 and FP32
__global__ __launch_bounds__(256) void k_pack_s(int nv, int nh, const double* W2, double* S, float* S32) {
  const int64_t x = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (x >= int64_t(nv) * nv * nh) return;
  const int64_t k = x % nh, P = x / nh / nv, Q = x / nh % nv;
  const double s = 0.5 * (W2[(k * nv + P) * nv + Q] + W2[(k * nv + Q) * nv + P]);
  S[x] = s;
  S32[x] = float(s);
}

// flags: [0] lowest i chi + u with eta < 0 or NaN (2^31 - 1: none), [1] an eta is
// zero, [2] an entry is infinite or NaN
__global__ void k_flags_init(int* flags) {
  if (threadIdx.x < 3) flags[threadIdx.x] = threadIdx.x == 0 ? 0x7FFFFFFF : 0;
}
__global__ __launch_bounds__(256) void k_check(int K, int chi, const int64_t* offEta, const double* prm, int64_t n,
                                               int* flags) {
  const int64_t stride = int64_t(gridDim.x) * 256, t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  bool odd = false;
  for (int64_t x = t; x < n; x += stride) odd |= !isfinite(prm[x]);
  if (odd) flags[2] = 1;
  for (int64_t x = t; x < int64_t(K) * chi; x += stride) {
    const double e = prm[offEta[x / chi] + x % chi];
    if (!(e >= 0.0)) atomicMin(&flags[0], int(x));
    if (e == 0.0) flags[1] = 1;
  }
}

// complex parameters: the realified vector.  Per edge and state
// M_r = [[Re M, -Im M], [Im M, Re M]]; v_r = [Re v; Im v], eta_r = [eta; eta],
// w_r = [Re w; -Im w], c_r = Re c, w2 = [Im w; Re w], c2 = Im c; the correlator
// block as it is
__global__ __launch_bounds__(256) void k_realify_edges(CxMap M, const double* p, double* r) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int n = M.chi, n2 = 2 * n;
  const int64_t per = int64_t(4) * n * n;
  if (t >= per * M.n_edges) return;
  const int64_t e = t / per;
  const int x = int(t % per), s = x / (n * n), u = x / n % n, k = x % n;
  const double re = p[M.cM[e] + 2 * x], im = p[M.cM[e] + 2 * x + 1];
  double* B = r + M.rM[e] + int64_t(s) * n2 * n2;
  B[int64_t(u) * n2 + k] = re;
  B[int64_t(u) * n2 + k + n] = -im;
  B[int64_t(u + n) * n2 + k] = im;
  B[int64_t(u + n) * n2 + k + n] = re;
}
__global__ __launch_bounds__(256) void k_realify_sites(CxMap M, const double* p, double* r) {
  const int i = blockIdx.x, n = M.chi, n2 = 2 * n;
  for (int x = threadIdx.x; x < 4 * n; x += 256) {
    const int s = x / n, u = x % n;
    r[M.rV[i] + s * n2 + u] = p[M.cV[i] + 2 * x];
    r[M.rV[i] + s * n2 + n + u] = p[M.cV[i] + 2 * x + 1];
  }
  for (int u = threadIdx.x; u < n; u += 256) {
    const double et = p[M.cEta[i] + u], wr = p[M.cW[i] + 2 * u], wi = p[M.cW[i] + 2 * u + 1];
    r[M.rEta[i] + u] = et;
    r[M.rEta[i] + n + u] = et;
    r[M.rW[i] + u] = wr;
    r[M.rW[i] + n + u] = -wi;
    r[M.rW2[i] + u] = wi;
    r[M.rW2[i] + n + u] = wr;
  }
  if (threadIdx.x == 0) {
    r[M.rC[i]] = p[M.cC[i]];
    r[M.rC2[i]] = p[M.cC[i] + 1];
  }
}

inline unsigned blocks(int64_t n) { return unsigned((n + 255) / 256); }

template <typename T>
hipError_t pack(const PackParams& P, T* A, T* AF, T* BT, T* v, T* eta, T* w, T* c, T* w2, T* c2, hipStream_t st) {
  const int64_t ES = int64_t(P.chip / 4) * (P.chip / 4) * 64;
  hipLaunchKernelGGL(k_pack_edges<T>, dim3(blocks(ES), P.n_fwd + 1), dim3(256), 0, st, P, A, AF, BT);
  hipLaunchKernelGGL(k_pack_sites<T>, dim3(P.K), dim3(256), 0, st, P, v, eta, w, c, w2, c2);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pack_f64(const PackParams& P, double* A, double* AF, double* BT, double* v, double* eta, double* w,
                           double* c, double* w2, double* c2, hipStream_t st) {
  return pack<double>(P, A, AF, BT, v, eta, w, c, w2, c2, st);
}
hipError_t launch_pack_f32(const PackParams& P, float* A, float* AF, float* BT, float* v, float* eta, float* w,
                           float* c, float* w2, float* c2, hipStream_t st) {
  return pack<float>(P, A, AF, BT, v, eta, w, c, w2, c2, st);
}

hipError_t launch_pack_tri32(const PackParams& P, const int* qoff, int dmax, float* Q, int vofs, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_tri32, dim3(4 * tri_lc32(P.chip, dmax), P.K), dim3(64), 0, st, P, qoff, dmax, Q, vofs);
  return hipGetLastError();
}

int64_t bf16_edge_values(int chip) {
  const int NT = chip / 4, TPC = chip / 16;
  return int64_t(TPC / 2) * NT * 64 * 8 + int64_t(TPC & 1) * NT * 64 * 4;
}

hipError_t launch_pack_bf16(const PackParams& P, uint16_t* A, uint16_t* Alo, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_bf16, dim3(blocks(bf16_edge_values(P.chip)), P.n_fwd + 1), dim3(256), 0, st, P, A, Alo);
  return hipGetLastError();
}

hipError_t launch_pack_corr(int nv, int nh, const double* W, double* Wt, const double* W2, double* S, float* S32,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_pack_wt, dim3(blocks(int64_t(nv) * nh)), dim3(256), 0, st, nv, nh, W, Wt);
  if (W2)
    hipLaunchKernelGGL(k_pack_s, dim3(blocks(int64_t(nv) * nv * nh)), dim3(256), 0, st, nv, nh, W2, S, S32);
  return hipGetLastError();
}

hipError_t launch_check_params(int K, int chi, const int64_t* offEta, const double* prm, int64_t n, int* flags,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_flags_init, dim3(1), dim3(64), 0, st, flags);
  const int64_t b = (n + 1023) / 1024;
  hipLaunchKernelGGL(k_check, dim3(unsigned(b < 256 ? b : 256)), dim3(256), 0, st, K, chi, offEta, prm, n, flags);
  return hipGetLastError();
}

hipError_t launch_realify(const CxMap& M, int K, const double* p, double* r, hipStream_t st) {
  const int64_t ne = int64_t(4) * M.chi * M.chi * M.n_edges;
  if (ne > 0) hipLaunchKernelGGL(k_realify_edges, dim3(blocks(ne)), dim3(256), 0, st, M, p, r);
  hipLaunchKernelGGL(k_realify_sites, dim3(K), dim3(256), 0, st, M, p, r);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || M.n_corr == 0) return e;
  return hipMemcpyAsync(r + M.r_corr, p + M.c_corr, size_t(M.n_corr) * sizeof(double), hipMemcpyDeviceToDevice, st);
}

}  // namespace nqs
