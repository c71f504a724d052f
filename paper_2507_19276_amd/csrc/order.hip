// Row order for the resumed amplitude pass: a stable counting sort of the
// amplitude rows by their first changed site t0, the lowest site at which a
// row's ONV differs from its sample's (K when they are equal; the fill kernel
// writes it with the row).  The autoregressive conditionals of Eqs. (9)-(10)
// at sites below t0 depend only on the occupations below t0, which the row
// shares with its sample, so a row can resume at t0 from its sample's carried
// state; grouping rows by t0 lets a whole wavefront skip the shared prefix.
//
// Three launches, all deterministic:
//   count:   per block of kOrderChunk rows, a histogram of t0 (LDS atomics;
//            counts do not depend on their order);
//   scan:    one block per bucket: exclusive offsets of the bucket over the
//            blocks, and the bucket total;
//   scatter: each block walks its rows in order, 256 at a time; a row's
//            position is the bucket's base (sum of the lower totals) plus its
//            block offset, the rows of the bucket in earlier rounds, the rows
//            of the bucket in lower wavefronts of the round and the rows of the
//            bucket in lower lanes (one ballot per key bit), so equal keys
//            keep row order.
#include "internal.h"

namespace nqs {
namespace {

__global__ __launch_bounds__(256) void k_t0_count(const uint8_t* __restrict__ t0, int64_t R, int K,
                                                  int32_t* __restrict__ cnt) {
  __shared__ int h[65];
  for (int k = threadIdx.x; k <= K; k += 256) h[k] = 0;
  __syncthreads();
  const int64_t r0 = int64_t(blockIdx.x) * kOrderChunk;
  const int64_t r1 = r0 + kOrderChunk < R ? r0 + kOrderChunk : R;
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) atomicAdd(&h[t0[r]], 1);
  __syncthreads();
  for (int k = threadIdx.x; k <= K; k += 256) cnt[int64_t(blockIdx.x) * (K + 1) + k] = h[k];
}

// block k scans column k of cnt[nb][K+1] in place (exclusive) and writes tot[k]
__global__ __launch_bounds__(256) void k_t0_scan(int32_t* __restrict__ cnt, int64_t nb, int K,
                                                 int64_t* __restrict__ tot) {
  __shared__ int64_t part[256];
  const int k = blockIdx.x, tid = threadIdx.x;
  const int64_t per = (nb + 255) / 256;
  const int64_t b0 = tid * per;
  const int64_t b1 = b0 + per < nb ? b0 + per : nb;
  int64_t s = 0;
  for (int64_t b = b0; b < b1; ++b) s += cnt[b * (K + 1) + k];
  part[tid] = s;
  __syncthreads();
  // inclusive scan of the 256 partial sums (Hillis-Steele)
  for (int d = 1; d < 256; d <<= 1) {
    const int64_t v = tid >= d ? part[tid - d] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  int64_t run = tid > 0 ? part[tid - 1] : 0;
  for (int64_t b = b0; b < b1; ++b) {
    const int c = cnt[b * (K + 1) + k];
    cnt[b * (K + 1) + k] = int(run);
    run += c;
  }
  if (tid == 255) tot[k] = part[255];
}

__global__ __launch_bounds__(256) void k_t0_scatter(const uint8_t* __restrict__ t0, int64_t R, int K,
                                                    const int32_t* __restrict__ off,
                                                    const int64_t* __restrict__ tot, int32_t* __restrict__ perm,
                                                    uint8_t* __restrict__ t0s) {
  __shared__ int run[65];
  __shared__ int wc[4][65];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (threadIdx.x == 0) {
    int64_t acc = 0;
    for (int k = 0; k <= K; ++k) {
      run[k] = int(acc);
      acc += tot[k];
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k <= K; k += 256) {
    run[k] += off[int64_t(blockIdx.x) * (K + 1) + k];
    for (int w = 0; w < 4; ++w) wc[w][k] = 0;
  }
  __syncthreads();
  const int64_t r0 = int64_t(blockIdx.x) * kOrderChunk;
  const int64_t r1 = r0 + kOrderChunk < R ? r0 + kOrderChunk : R;
  const uint64_t below = (1ull << lane) - 1ull;
  for (int64_t rb = r0; rb < r1; rb += 256) {
    const int64_t r = rb + threadIdx.x;
    const bool valid = r < r1;
    const int t = valid ? int(t0[r]) : K;
    // the lanes of this wavefront with the same key (keys <= 64: one ballot per
    // key bit), and the rank among the lower ones
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 7; ++b) {
      const bool bit = (t >> b) & 1;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const int rank = __popcll(peers & below);
    if (valid && (peers & below) == 0) wc[wv][t] = __popcll(peers);
    __syncthreads();
    int pos = 0;
    if (valid) {
      pos = run[t] + rank;
      for (int w = 0; w < wv; ++w) pos += wc[w][t];
    }
    __syncthreads();
    for (int k = threadIdx.x; k <= K; k += 256) {
      int sum = 0;
      for (int w = 0; w < 4; ++w) {
        sum += wc[w][k];
        wc[w][k] = 0;
      }
      run[k] += sum;
    }
    __syncthreads();
    if (valid) {
      perm[pos] = int32_t(r);
      t0s[pos] = uint8_t(t);
    }
  }
}

// Order of the FP64 rows (psi_tri.h): by resume site, then sample, then the
// row's state at the resume site and its next changed site after it, so that the
// rows of a wavefront agree on nearly every site they evaluate.  The rows of
// a sample are contiguous, so one workgroup per sample (per kRowPart of its rows
// where it has more: one workgroup alone took 2 ms over the 572 k rows of an exact
// K = 50 sample, a fifth of the call) counts its rows per resume site (launch 1),
// the columns are scanned over the workgroups (k_t0_scan), and the workgroup places
// its rows with LDS counters over (resume site, state, next change).  Rows with
// equal keys take their places in any order (LDS atomics): which rows share a
// wavefront does not change a bit of any.
constexpr int kRowOrderThreads = 512;

// the rows of part blockIdx.y of sample n0 + blockIdx.x, counted from row_base; the
// parts of all samples are numbered sample by sample
__device__ inline int64_t row_part(const int64_t* rowptr, int64_t n0, int64_t row_base, int64_t part_rows,
                                   int64_t& r0, int64_t& r1) {
  const int64_t n = n0 + blockIdx.x, end = rowptr[n + 1] - row_base;
  r0 = rowptr[n] - row_base + int64_t(blockIdx.y) * part_rows;
  r1 = r0 + part_rows < end ? r0 + part_rows : end;
  return int64_t(blockIdx.x) * gridDim.y + blockIdx.y;
}

__global__ __launch_bounds__(kRowOrderThreads) void k_row_count(const uint8_t* __restrict__ site,
                                                                const int64_t* __restrict__ rowptr, int64_t n0,
                                                                int64_t row_base, int64_t part_rows, int K,
                                                                int32_t* __restrict__ cnt) {
  __shared__ int h[65];
  const int tid = threadIdx.x;
  if (tid <= K) h[tid] = 0;
  __syncthreads();
  int64_t r0, r1;
  const int64_t part = row_part(rowptr, n0, row_base, part_rows, r0, r1);
  for (int64_t r = r0 + tid; r < r1; r += kRowOrderThreads) atomicAdd(&h[site[r]], 1);
  __syncthreads();
  if (tid <= K) cnt[part * (K + 1) + tid] = h[tid];
}

// LDS bin of a row: (resume site, state there, next changed site)
__device__ inline int row_bin(int t, uint64_t lo, uint64_t hi, uint64_t nlo, uint64_t nhi, int K) {
  if (t >= K) return K * 4 * (K + 1);
  const uint64_t ev = 0x5555555555555555ull;
  uint64_t xl = lo ^ nlo, xh = hi ^ nhi;
  xl = (xl | (xl >> 1)) & ev;
  xh = (xh | (xh >> 1)) & ev;
  // keep the changes above site t
  if (t < 31) xl &= ~0ull << (2 * t + 2);
  else {
    xl = 0;
    if (t > 31) xh = t < 63 ? xh & (~0ull << (2 * t - 62)) : 0;
  }
  const int next = xl ? __builtin_ctzll(xl) >> 1 : (xh ? 32 + (__builtin_ctzll(xh) >> 1) : K);
  const int s = t < 32 ? int((lo >> (2 * t)) & 3ull) : int((hi >> (2 * t - 64)) & 3ull);
  return (t * 4 + s) * (K + 1) + next;
}

__global__ __launch_bounds__(kRowOrderThreads) void k_row_place(
    const uint8_t* __restrict__ site, const uint64_t* __restrict__ m, const uint64_t* __restrict__ samples,
    const int64_t* __restrict__ rowptr, int64_t n0, int64_t row_base, int64_t part_rows, int K,
    const int32_t* __restrict__ off, const int64_t* __restrict__ tot, int32_t* __restrict__ perm, uint8_t* __restrict__ t0s) {
  extern __shared__ int bins[];   // [K + 1][4][K + 1], the last site's one bin
  __shared__ int start[65];
  const int tid = threadIdx.x, per = 4 * (K + 1), nbin = K * per + 1;
  const int64_t n = n0 + blockIdx.x;
  int64_t r0, r1;
  const int64_t part = row_part(rowptr, n0, row_base, part_rows, r0, r1);
  if (r0 >= r1) return;
  const uint64_t nlo = samples[2 * n], nhi = samples[2 * n + 1];
  for (int k = tid; k < nbin; k += kRowOrderThreads) bins[k] = 0;
  if (tid < 64) {
    // first position of each site: the lower sites' totals and the lower parts' rows
    int64_t a = tid <= K ? tot[tid] : 0;
    const int64_t own = a;
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t x = __shfl_up(a, o);
      if (tid >= o) a += x;
    }
    if (tid <= K) start[tid] = int(a - own) + off[part * (K + 1) + tid];
    if (tid == 63 && K == 64) start[64] = int(a) + off[part * 65 + 64];
  }
  __syncthreads();
  for (int64_t r = r0 + tid; r < r1; r += kRowOrderThreads)
    atomicAdd(&bins[row_bin(site[r], m[2 * r], m[2 * r + 1], nlo, nhi, K)], 1);
  __syncthreads();
  // exclusive scan of each site's bins from its first position, a wavefront per site
  const int wv = tid >> 6, lane = tid & 63;
  for (int t = wv; t <= K; t += kRowOrderThreads / 64) {
    int run = start[t];
    const int len = t < K ? per : 1;
    for (int k0 = 0; k0 < len; k0 += 64) {
      const int k = k0 + lane;
      const int c = k < len ? bins[t * per + k] : 0;
      int a = c;
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(a, o);
        if (lane >= o) a += x;
      }
      if (k < len) bins[t * per + k] = run + a - c;
      run += __shfl(a, 63);
    }
  }
  __syncthreads();
  for (int64_t r = r0 + tid; r < r1; r += kRowOrderThreads) {
    const int t = site[r];
    const int pos = atomicAdd(&bins[row_bin(t, m[2 * r], m[2 * r + 1], nlo, nhi, K)], 1);
    perm[pos] = int32_t(r);
    t0s[pos] = uint8_t(t);
  }
}

// Order of the node units of the triangular-normaliser forward.  A
// wavefront runs from its units' lowest changed site to their last site and pays
// for every local state that occurs among them, so its units should be of one
// sample and end together: the units that run to the last site (about a third,
// with two thirds of the sites at K = 50) come first, then the others, each in
// sample order, a sample's units by changed site upwards in even samples and
// downwards in odd ones, so that a wavefront across two samples joins
// neighbouring sites.  (NN+NNN chain K = 50, 16384 samples: node pass 213 ms
// in the order of the changed site alone, 129 ms here; the four-candidate
// kernel took 114 ms.)
__global__ __launch_bounds__(256) void k_norder_count(const uint8_t* __restrict__ e1, const int64_t* __restrict__ nbase,
                                                      const int32_t* __restrict__ ncnt, int K,
                                                      int32_t* __restrict__ cnt) {
  __shared__ int c;
  if (threadIdx.x == 0) c = 0;
  __syncthreads();
  const int64_t b = nbase[blockIdx.x];
  const int n = b < 0 ? 0 : ncnt[blockIdx.x];
  int own = 0;
  for (int k = threadIdx.x; k < n; k += 256) own += e1[b + k] >= K;
  if (own) atomicAdd(&c, own);
  __syncthreads();
  if (threadIdx.x == 0) cnt[blockIdx.x] = c;
}

__global__ __launch_bounds__(64) void k_norder_place(const uint8_t* __restrict__ c1, const uint8_t* __restrict__ e1,
                                                     const int64_t* __restrict__ nbase,
                                                     const int32_t* __restrict__ ncnt, int K,
                                                     const int32_t* __restrict__ off, const int64_t* __restrict__ tot,
                                                     int64_t ns, int64_t nn, int32_t* __restrict__ perm,
                                                     uint8_t* __restrict__ c1s) {
  const int64_t s = blockIdx.x, b = nbase[s];
  if (b < 0) return;
  const int n = ncnt[s], lane = threadIdx.x;
  const int64_t l0 = off[s], h0 = tot[0] + b - l0;   // the sample's first place among the long and the short units
  const int64_t lend = s + 1 < ns ? int64_t(off[s + 1]) : tot[0];
  const int nl = int(lend - l0), nh = n - nl;
  const uint64_t below = (1ull << lane) - 1ull;
  int rl = 0, rh = 0;
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int k = k0 + lane;
    const bool in = k < n, lg = in && e1[b + (in ? k : 0)] >= K;
    const uint64_t ml = __ballot(lg), mh = __ballot(in && !lg);
    if (in) {
      const int r = lg ? rl + __popcll(ml & below) : rh + __popcll(mh & below);
      const int len = lg ? nl : nh;
      const int64_t pos = (lg ? l0 : h0) + ((s & 1) ? len - 1 - r : r);
      if (pos < nn) {
        perm[pos] = int32_t(b + k);
        c1s[pos] = c1[b + k];
      }
    }
    rl += __popcll(ml);
    rh += __popcll(mh);
  }
}

// dst[p] = src[perm[p]]
__global__ __launch_bounds__(256) void k_gather_u8(const uint8_t* __restrict__ src, const int32_t* __restrict__ perm,
                                                   int64_t n, uint8_t* __restrict__ dst) {
  const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (p < n) dst[p] = src[perm[p]];
}

// out[p] = a[b[p]]
__global__ __launch_bounds__(256) void k_compose(const int32_t* __restrict__ a, const int32_t* __restrict__ b,
                                                 int64_t n, int32_t* __restrict__ out) {
  const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (p < n) out[p] = a[b[p]];
}

}  // namespace

hipError_t launch_order_t0(const uint8_t* t0, int64_t R, int K, int32_t* cnt, int64_t* tot, int32_t* perm,
                           uint8_t* t0s, hipStream_t st) {
  if (R <= 0) return hipSuccess;
  if (K < 1 || K > 64 || R >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  const int64_t nb = order_blocks(R);
  hipLaunchKernelGGL(k_t0_count, dim3(unsigned(nb)), dim3(256), 0, st, t0, R, K, cnt);
  hipLaunchKernelGGL(k_t0_scan, dim3(unsigned(K + 1)), dim3(256), 0, st, cnt, nb, K, tot);
  hipLaunchKernelGGL(k_t0_scatter, dim3(unsigned(nb)), dim3(256), 0, st, t0, R, K, cnt, tot, perm, t0s);
  return hipGetLastError();
}

hipError_t launch_order_rows(const uint8_t* site, const uint64_t* m, const uint64_t* samples, const int64_t* rowptr,
                             int64_t n0, int64_t n1, int64_t row_base, int64_t R, const RowParts& parts, int K,
                             int32_t* cnt, int64_t* tot, int32_t* perm, uint8_t* t0s, hipStream_t st) {
  if (R <= 0) return hipSuccess;
  if (K < 1 || K > 64 || R >= (int64_t(1) << 31) || parts.n < 1 || parts.n > 65535) return hipErrorInvalidValue;
  const int64_t ns = n1 - n0;
  const dim3 grid(unsigned(ns), unsigned(parts.n));
  hipLaunchKernelGGL(k_row_count, grid, dim3(kRowOrderThreads), 0, st, site, rowptr, n0, row_base, parts.rows, K, cnt);
  hipLaunchKernelGGL(k_t0_scan, dim3(unsigned(K + 1)), dim3(256), 0, st, cnt, ns * parts.n, K, tot);
  const size_t lds = size_t(K * 4 * (K + 1) + 1) * sizeof(int);
  hipLaunchKernelGGL(k_row_place, grid, dim3(kRowOrderThreads), lds, st, site, m, samples, rowptr, n0, row_base,
                     parts.rows, K, cnt, tot, perm, t0s);
  return hipGetLastError();
}

hipError_t launch_order_nodes(const uint8_t* c1, const uint8_t* e1, const int64_t* nbase, const int32_t* ncnt,
                              int64_t ns, int64_t nn, int K, int32_t* cnt, int64_t* tot, int32_t* perm, uint8_t* c1s,
                              hipStream_t st) {
  if (nn <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_norder_count, dim3(unsigned(ns)), dim3(256), 0, st, e1, nbase, ncnt, K, cnt);
  hipLaunchKernelGGL(k_t0_scan, dim3(1), dim3(256), 0, st, cnt, ns, 0, tot);
  hipLaunchKernelGGL(k_norder_place, dim3(unsigned(ns)), dim3(64), 0, st, c1, e1, nbase, ncnt, K, cnt, tot, ns, nn,
                     perm, c1s);
  return hipGetLastError();
}

// order by (t0, t1) ascending: a stable sort by t1, then a stable sort of
// the result by t0 (least significant key first); tmp: 2 R int32 and 2 R bytes
hipError_t launch_order_t0_t1(const uint8_t* t0, const uint8_t* t1, int64_t R, int K, int32_t* cnt, int64_t* tot,
                              int32_t* tmp_perm, uint8_t* tmp_key, int32_t* perm, uint8_t* t0s, hipStream_t st) {
  if (R <= 0) return hipSuccess;
  if (K < 1 || K > 64 || R >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  int32_t* p1 = tmp_perm;       // position -> row, sorted by t1
  int32_t* p2 = tmp_perm + R;   // position -> position of the first sort, sorted by t0
  uint8_t* k1 = tmp_key;        // t1 in the first order (not used further)
  uint8_t* g0 = tmp_key + R;    // t0 in the first order
  hipError_t e = launch_order_t0(t1, R, K, cnt, tot, p1, k1, st);
  if (e != hipSuccess) return e;
  const unsigned blocks = unsigned((R + 255) / 256);
  hipLaunchKernelGGL(k_gather_u8, dim3(blocks), dim3(256), 0, st, t0, p1, R, g0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_order_t0(g0, R, K, cnt, tot, p2, t0s, st)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_compose, dim3(blocks), dim3(256), 0, st, p1, p2, R, perm);
  return hipGetLastError();
}

}  // namespace nqs
