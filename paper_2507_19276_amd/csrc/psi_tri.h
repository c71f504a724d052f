// Forward of the BDG-RNN / MPS-RNN rows of a local energy, sorted so that a
// wavefront's rows agree on nearly every site; in FP64 with the conditional's
// normaliser from a triangular factor (arXiv:2507.19276, Sec. 2.1 Eqs.
// (9)-(10), Sec. 2.2 Eq. (12) without the tensor term; realified complex
// parameters as in psi.hip).
//
// A row needs of site i the candidate of its own local state, h = A_s x + v_s
// (x: the parents' states, sqrt(eta) folded in, P^s = |h|^2), and the sum Z of
// P^s over the allowed states.  psi.hip evaluates all four candidates for it.
// Where all four states are allowed, Z = |[A_0 v_0; ..; A_3 v_3] [x; 1]|^2, and
// with the QR factorisation of that 4chi x (chi d + 1) matrix
//   Z = |R x + r|^2 + rho,  R upper triangular chi d x chi d,
// so a site costs (chi d)^2 / 2 multiply-adds for Z and chi^2 d for each local
// state that occurs among a wavefront's rows, against 4 chi^2 d.  The rows come
// sorted so that a wavefront holds rows of one sample that agree on nearly
// every site (order.hip): mostly one state.  At chi = 32, d = 2 that is 18
// blocks of 16x16 instead of 32, at chi = 16, d = 1 2 instead of 4.  Where the
// particle-number mask forbids a state, Z is the sum over the allowed
// candidates as in psi.hip.  Which form a row takes depends on the row alone, so
// its bits do not depend on the rows that share its wavefront.
//
// What bounds it: FP64 MFMA and VALU instructions share the SIMD's FP64 units
// (they never overlap, measured), so its time is its matrix instructions plus its
// epilogue plus what the resident wavefronts do not hide.  Hence two tiles of rows
// per wavefront (each operand block feeds two MFMA chains; one tile in launches too
// small to fill the chip, see kTriOneTileRows) at registers for two
// or three wavefronts per SIMD: at chi = 32 four tiles at one wavefront ran
// 160 against 119 ms.  Row kernels before (psi.hip) and now: NN+NNN K = 50, chi = 32,
// 4096 samples 202 -> 119 ms (MFMA busy 84%); 3x3x2 lattice chi = 64, 1024 samples
// 119 -> 62 ms; dense K = 20 chi = 64, 256 samples 26.0 -> 11.4 ms; chain K = 20
// chi = 16, 4096 samples 12.0 -> 8.9 ms (MFMA busy 44%: eight sites per row, and a
// wavefront's start, four dependent reads, is a third of its life); the same with
// complex parameters, 1024 samples 10.8 -> 5.7 ms.
//
// FP32 rows (QUAD false) keep the four-candidate sum and psi.hip's order of
// operations, so their bits are psi.hip's; what they take from here is the work
// that the row order saves and psi.hip's four-candidates-at-once form cannot:
//  - one candidate at a time, so chip / 16 accumulators per tile of rows instead of
//    chip / 4, and two wavefronts per SIMD at chi = 64 instead of one;
//  - no candidate that is forbidden to every row of the wavefront (near the chain's
//    end and in every site of a row whose mask has closed);
//  - the choice of the carried state is a register copy when the rows agree.
// FP32 MFMA and VALU instructions share their units too (chip 16: MFMA busy 42% +
// VALU 44%).  Two tiles of rows to chip 32, one above (3x3x2 lattice chi = 64, 2048
// samples: row kernel 102 ms in psi.hip, 112 with two tiles, 70 with one; chi = 48:
// 54 with two, 39 with one; dense K = 20 chi = 16: 6.8 in psi.hip, 5.0 with two, 4.8
// with four; lattice chi = 16: 4.7, 3.2, 4.7).  Row kernels, psi.hip and now: dense
// K = 20 chi = 64 100 -> 51 ms, chi = 64 chain 68 -> 40 ms, chi = 32 K = 50 NN+NNN
// (512 samples) 13.5 -> 12.1 ms, complex chain 5.7 -> 4.4 ms.
#pragma once
#include "device.h"

namespace nqs {

namespace {

// wavefronts per SIMD the registers are kept to (FP32 needs at most what two leave
// at every size; one instead ran dense chi = 64 at 59 against 51 ms)
template <typename T> constexpr int tri_occ(int CH, int DM) {
  if (sizeof(T) == 4) return 2;
  return CH == 16 ? (DM == 3 ? 2 : 3) : (CH == 32 ? 2 : 1);
}

template <typename T, int CH, int NTL, int DM, int STORE, bool CPLX>
__global__ __launch_bounds__(64, tri_occ<T>(CH, DM)) void k_psi_tri(TriParams P, const uint64_t* __restrict__ m,
                                                                    int64_t R, double* __restrict__ lphi,
                                                                    int8_t* __restrict__ sphi, PsiStates<T> X,
                                                                    double* __restrict__ phs) {
  // as in psi.hip every operation is written out: a resumed row ends
  // bit-identical to one evaluated from site 0
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char smem[];
  typedef typename V4<T>::type V;
  constexpr bool QUAD = sizeof(T) == 8;   // Z from the triangular factor; else from the four candidates
  constexpr int TPC = CH / 16, RW = 16 * NTL, PW = QUAD ? tri_pw(CH) : kTriWindow32, RP = tri_rp(CH);
  constexpr int SLOT = NTL * TPC * 64;
  // an FP64 MFMA's result takes its 16 passes and more to arrive: with one tile
  // of rows a row group is squared only after the next group's MFMAs
  constexpr bool LATE = NTL == 1;
  const int lane = threadIdx.x;
  const int j = lane & 15, g = lane >> 4;
  const int own = NTL == 2 ? (g >> 1) : 0;
  const int64_t base = int64_t(blockIdx.x) * RW;
  V* ring = reinterpret_cast<V*>(smem) + lane;
  const CInt* fptr = (const CInt*)(P.pptr);
  const CInt* slots = (const CInt*)(P.slot);
  const CInt* wsl = (const CInt*)(P.wsl);
  const CInt* qoff = (const CInt*)(P.qoff);
  const CT<T>* cc = (const CT<T>*)(P.c);
  const CT<T>* cc2 = (const CT<T>*)(P.c2);
  const CT<double>* rho = (const CT<double>*)(P.rho);
  // rows come in the order of their resume sites; node units in the order of
  // launch_order_nodes, whose wavefronts start at their lowest changed site
  int i0 = 0;
  if (STORE == 2) {
    i0 = P.K;
    for (int p = lane; p < RW; p += 64)
      if (base + p < R) {
        const int c = X.t0[base + p];
        i0 = c < i0 ? c : i0;
      }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const int x = __shfl_xor(i0, o);
      i0 = x < i0 ? x : i0;
    }
    i0 = __builtin_amdgcn_readfirstlane(i0);
  } else if (X.perm) {
    i0 = int(((const __attribute__((address_space(4))) uint8_t*)X.t0)[base]);
  }
  uint64_t lo[NTL], hi[NTL];
  int64_t rowt[NTL];
  uint64_t olo = 0, ohi = 0;
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    const int64_t r = base + 16 * t + j;
    const int64_t rr = r < R ? r : R - 1;
    rowt[t] = X.perm ? int64_t(X.perm[rr]) : rr;
    lo[t] = m[2 * rowt[t]];
    hi[t] = m[2 * rowt[t] + 1];
    if (t == own) { olo = lo[t]; ohi = hi[t]; }
  }
  const bool olive = base + 16 * own + j < R;
  int64_t orow = rowt[0];
#pragma unroll
  for (int t = 1; t < NTL; ++t)
    if (t == own) orow = rowt[t];
  // QUAD: the samples' own amplitudes have Z summed over the candidates, as psi.hip;
  // STORE 1: all rows are samples, STORE 3: those that equal their sample
  bool self = STORE == 1;
  if constexpr (STORE == 3) {
    const int64_t o = X.owner[orow];
    self = olo == X.samples[2 * o] && ohi == X.samples[2 * o + 1];
  }
  const bool sums = QUAD && (STORE == 1 || (STORE == 3 && __builtin_amdgcn_ballot_w64(self) != 0));
  T prod = T(1), prod2 = T(1);   // prod2: with that sum, kept where the wavefront has such a row
  T zr = T(1), zi = T(0);
  int pexp = 0, pexp2 = 0, sgn = 1;
  const SpinEnds ends(olo, ohi, P.K, P.na, P.nb);
  if (X.perm && i0 > 0) {
    // the states live at i0 and the log-product state before it, from the
    // row's node at the sites the node covers, else from its sample (psi.hip)
    int nb[NTL];
    int64_t no[NTL], nco[NTL];
    uint64_t nmk[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      const int nd = X.unode ? X.unode[rowt[t]] : -1;
      NodeRec q{0, 0, 0ull, P.K + 1, 0};
      if (nd >= 0) q = X.nrec[nd];
      nb[t] = q.c1;
      no[t] = q.off;
      nco[t] = q.coff;
      nmk[t] = q.need;
    }
    for (uint64_t lv = ((const __attribute__((address_space(4))) uint64_t*)P.live)[i0]; lv; lv &= lv - 1) {
      const int s = __builtin_ctzll(lv);
      V* wr = ring + size_t(wsl[s]) * SLOT;
#pragma unroll
      for (int t = 0; t < NTL; ++t) {
        const T* src = s >= nb[t] ? X.nhs + size_t(nco[t] + __popcll(nmk[t] & low_bits(s))) * CH + 4 * g
                                       : X.hs + (size_t(s) * X.ns + X.owner[rowt[t]]) * CH + 4 * g;
#pragma unroll
        for (int tt = 0; tt < TPC; ++tt) wr[(t * TPC + tt) * 64] = *reinterpret_cast<const V*>(src + 16 * tt);
      }
    }
    int onb = nb[0];
    int64_t ono = no[0];
#pragma unroll
    for (int t = 1; t < NTL; ++t)
      if (t == own) { onb = nb[t]; ono = no[t]; }
    if (i0 >= onb) {
      const size_t so = size_t(ono + (i0 - onb));
      const LogProd<T> lp = X.nlp[so];
      prod = lp.m;
      pexp = lp.e;
      sgn = lp.s;
      if (CPLX) {
        zr = X.npz[2 * so];
        zi = X.npz[2 * so + 1];
      }
    } else {
      const size_t so = size_t(i0) * X.ns + X.owner[orow];
      prod = X.pm[so];
      pexp = X.pe[so];
      sgn = X.pg[so];
      if (CPLX) {
        zr = X.pz[2 * so];
        zi = X.pz[2 * so + 1];
      }
    }
  }
  int sc1 = 0, se1 = -1;
  int64_t soff = 0;
  if (STORE == 2) {
    const NodeRec q = X.nrec[orow];
    sc1 = q.c1;
    se1 = q.e1;
    soff = q.off;
  }
  int te1[NTL];
  int64_t toff[NTL];
  uint64_t tneed[NTL];
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    NodeRec q{0, 0, 0ull, 0, -1};
    if (STORE == 2) q = X.nrec[rowt[t]];
    te1[t] = q.e1;
    toff[t] = q.coff;
    tneed[t] = q.need;
  }
  const bool writer = NTL == 2 ? (g & 1) == 0 : g == 0;
  auto store_pre = [&](int i) {
    if (STORE == 1 && writer && olive && orow < X.ns) {
      const size_t so = size_t(i) * X.ns + orow;
      X.pm[so] = prod;
      X.pe[so] = pexp;
      X.pg[so] = int8_t(sgn);
      if (CPLX) {
        X.pz[2 * so] = zr;
        X.pz[2 * so + 1] = zi;
      }
    }
    if (STORE == 2 && writer && olive && i >= sc1 && i <= se1) {
      const size_t so = size_t(soff + (i - sc1));
      X.nlp[so] = LogProd<T>{prod, pexp, sgn};
      if (CPLX) {
        X.npz[2 * so] = zr;
        X.npz[2 * so + 1] = zi;
      }
    }
  };
  int iend = P.K;
  if constexpr (STORE == 2) {
    int em = 0;
#pragma unroll
    for (int t = 0; t < NTL; ++t) em = te1[t] > em ? te1[t] : em;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const int x = __shfl_xor(em, o);
      em = x > em ? x : em;
    }
    iend = __builtin_amdgcn_readfirstlane(em < P.K ? em : P.K);
  }
  // The rows' masks at one site as lane masks of the own rows: allowed states,
  // all four allowed, own state; and the wavefront's parts there: bit 0 = some
  // row has all four states allowed (Z from R), bit 1 + s = candidate s is some
  // row's state, or an allowed state of a row whose mask forbids another (not
  // QUAD: of any row; all four where `sums`).
  struct Masks {
    uint64_t full, a0, a1, b0, b1;   // state s = a + 2 b is allowed where a's and b's masks have the lane
    uint32_t pt, own;                // own: bit s = s is some row's state
  };
  auto masks = [&](int i, int s) {
    Masks M;
    M.a0 = __builtin_amdgcn_ballot_w64(i <= ends.ah);
    M.a1 = __builtin_amdgcn_ballot_w64(i <= ends.ae);
    M.b0 = __builtin_amdgcn_ballot_w64(i <= ends.bh);
    M.b1 = __builtin_amdgcn_ballot_w64(i <= ends.be);
    const uint64_t sl = __builtin_amdgcn_ballot_w64((s & 1) != 0), sh = __builtin_amdgcn_ballot_w64(s >= 2);
    M.full = M.a0 & M.a1 & M.b0 & M.b1;
    M.pt = M.full ? 1u : 0u;
    M.own = 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t st = ((k & 1) ? sl : ~sl) & ((k & 2) ? sh : ~sh);
      const uint64_t al = ((k & 1) ? M.a1 : M.a0) & ((k & 2) ? M.b1 : M.b0);
      const uint64_t need = sums ? ~0ull : (st | (QUAD ? al & ~M.full : al));
      M.pt |= need ? 2u << k : 0u;
      M.own |= st ? 1u << k : 0u;
    }
    return M;
  };
  // Operands and vectors come through one buffer resource: the lane's part of
  // the offset is fixed and the rest is scalar, so a load takes no vector
  // arithmetic.
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.Q), 0, P.qbytes, 0x00020000);
  const int laneq = int(sizeof(V)) * lane, gq = int(sizeof(V)) * g;
  auto quad = [&](int vofs, int sofs) {
    if constexpr (QUAD) {
      typedef double d2 __attribute__((ext_vector_type(2)));
      const d2 x = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vofs, sofs, 0));
      const d2 y = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vofs + 16, sofs, 0));
      return V{x.x, x.y, y.x, y.y};
    } else {
      return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vofs, sofs, 0));
    }
  };
  auto ld = [&](int blk) { return quad(laneq, blk * int(256 * sizeof(T))); };
  // vectors of site i: (QUAD: r [DM][CH],) v [4][CH], w [CH], w2 [CH]
  constexpr int VR = 0, VV = QUAD ? DM * CH : 0, VW = VV + 4 * CH, VW2 = VW + CH, VS = VW2 + CH;
  auto vec = [&](int i, int at) { return quad(gq, P.vofs + (i * VS + at) * int(sizeof(T))); };
  // first operand block of site i's parts pt
  auto first_part = [&](int i, uint32_t pt) {
    const int d = fptr[i + 1] - fptr[i];
    const int b0 = qoff[i];
    return (pt & 1u) ? b0 : b0 + tri_lr(CH, d) + int(__builtin_ctz(pt >> 1)) * tri_lc(CH, d);
  };
  Masks M{};
  V an[PW];   // window of operand blocks, PW ahead of the MFMAs
  V rb[RP];   // r of the site's first row group, fetched during the site before
  auto fetch_rb = [&](int i) {
#pragma unroll
    for (int r = 0; r < RP; ++r) rb[r] = vec(i, VR + 16 * r);
  };
  if (i0 < iend) {
    if (QUAD) fetch_rb(i0);
    M = masks(i0, site_state(olo, ohi, i0));
    const int p = QUAD ? first_part(i0, M.pt) : qoff[i0];
#pragma unroll
    for (int q = 0; q < PW; ++q) an[q] = ld(p + q);
  }
  auto site = [&](int i, auto DD) {
    constexpr int D = decltype(DD)::value, n = D * TPC;
    constexpr int LR = QUAD ? tri_lr(CH, D) : 0, LC = QUAD ? tri_lc(CH, D) : tri_lc32(CH, D);
    const int b0 = qoff[i];
    const int e0 = fptr[i];
    V b[n][NTL];
#pragma unroll
    for (int e = 0; e < D; ++e) {
      const int sl = slots[e0 + e];
      const bool zero = sl >= P.W;
      const V* rp = ring + size_t(zero ? 0 : sl) * SLOT;
#pragma unroll
      for (int t = 0; t < NTL; ++t)
#pragma unroll
        for (int tt = 0; tt < TPC; ++tt) b[e * TPC + tt][t] = zero ? V{0, 0, 0, 0} : rp[(t * TPC + tt) * 64];
    }
    const uint32_t cand = M.pt >> 1;
    V vb[TPC];   // v_s of the next candidate
    auto fetch_v = [&](int s) {
#pragma unroll
      for (int tt = 0; tt < TPC; ++tt)
        vb[tt] = vec(i, VV + s * CH + 16 * tt);
    };
    fetch_v(QUAD ? __builtin_ctz(cand) : 0);
    // the next site's parts: they follow from the occupations alone, and their
    // scalar work runs beside the MFMAs of the candidate
    const int osi = site_state(olo, ohi, i);
    Masks Mn{};
    int pn = 0;
    auto look_ahead = [&]() {
      if (i + 1 < iend) {
        Mn = masks(i + 1, site_state(olo, ohi, i + 1));
        if (QUAD) pn = first_part(i + 1, Mn.pt);
      }
    };
    // one block: four k-steps into acc, then its window slot takes the block PW
    // further on (past the part's end: of the next part)
    auto block = [&](int blk, int len, int cur, int nxt, const V (&x)[NTL], V (&acc)[NTL]) {
      const V a = an[blk % PW];
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int t = 0; t < NTL; ++t) acc[t] = mfma(a[v], x[t][v], acc[t]);
      an[blk % PW] = ld(blk + PW < len ? cur + (blk + PW) : nxt + (blk + PW - len));
      // keep the window's distance (scalar and vector arithmetic may move): the
      // scheduler would otherwise bring loads next to their uses and every block
      // would wait for its operands
      __builtin_amdgcn_sched_barrier(6);
    };
    // the padding blocks of a part: only the window moves on
    auto skip = [&](int from, int len, int cur, int nxt) {
#pragma unroll
      for (int k = from; k < len; ++k) an[k % PW] = ld(k + PW < len ? cur + (k + PW) : nxt + (k + PW - len));
    };
    auto square = [&](const V (&x)[RP][NTL], T (&q)[NTL]) {
#pragma unroll
      for (int r = 0; r < RP; ++r)
#pragma unroll
        for (int t = 0; t < NTL; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) q[t] = tfma(x[r][t][v], x[r][t][v], q[t]);
    };
    T zz[NTL], Z = T(0);
    V last[RP][NTL];   // the last rows of R x + r, squared after the next part's MFMAs
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      zz[t] = T(0);
#pragma unroll
      for (int r = 0; r < RP; ++r) last[r][t] = V{0, 0, 0, 0};
    }
    const int C0 = b0 + LR;
    if (QUAD && (M.pt & 1u)) {
      const int cur = b0, nxt = C0 + LC * int(__builtin_ctz(cand));
      int blk = 0;
#pragma unroll
      for (int r0 = 0; r0 < n; r0 += RP) {
        V acc[RP][NTL];
#pragma unroll
        for (int r = 0; r < RP; ++r) {
#pragma unroll
          for (int t = 0; t < NTL; ++t) acc[r][t] = r0 + r < n ? rb[r] : V{0, 0, 0, 0};
          if (r0 + RP + r < n) rb[r] = vec(i, VR + 16 * (r0 + RP + r));
        }
#pragma unroll
        for (int kt = r0; kt < n; ++kt)
#pragma unroll
          for (int r = 0; r < RP; ++r)
            if (r0 + r < n && kt >= r0 + r) block(blk++, LR, cur, nxt, b[kt], acc[r]);
        if (!LATE) square(acc, zz);
        if (LATE && r0 > 0) square(last, zz);
#pragma unroll
        for (int r = 0; r < RP; ++r)
#pragma unroll
          for (int t = 0; t < NTL; ++t)
            if (LATE) last[r][t] = acc[r][t];
      }
      skip(n * (n + 1) / 2, LR, cur, nxt);
      if (!LATE) Z = ReduceOwn<T, NTL>::run(zz) + T(rho[i]);
    }
    V ww[TPC], w2[TPC];
#pragma unroll
    for (int tt = 0; tt < TPC; ++tt) {
      ww[tt] = vec(i, VW + 16 * tt);
      if (CPLX) w2[tt] = vec(i, VW2 + 16 * tt);
    }
    if (QUAD) fetch_rb(i + 1 < iend ? i + 1 : i);
    V h[TPC][NTL];
    T Zs = T(0), pc = T(0);
    // candidate s of all rows into x, P^s of the own row returned; Z on the way
    // when its last rows are still to be squared
    auto candidate = [&](int s, const int& nxt, int s_next, auto with_z, auto&& take, auto&& beside) {
      const int cur = C0 + LC * s;
      T pp[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) pp[t] = T(0);
      int blk = 0;
      V acc[TPC][NTL];
#pragma unroll
      for (int tt = 0; tt < TPC; ++tt)
#pragma unroll
        for (int t = 0; t < NTL; ++t) acc[tt][t] = vb[tt];
      if (s_next >= 0) fetch_v(s_next);
      if (LC == PW) beside();   // it sets nxt, which the last PW blocks read
      auto finish = [&](int t0) {
#pragma unroll
        for (int tt = t0; tt < t0 + RP; ++tt)
          if (tt < TPC)
#pragma unroll
            for (int t = 0; t < NTL; ++t) {
#pragma unroll
              for (int v = 0; v < 4; ++v) pp[t] = tfma(acc[tt][t][v], acc[tt][t][v], pp[t]);
              take(tt, t, acc[tt][t]);
            }
      };
#pragma unroll
      for (int t0 = 0; t0 < TPC; t0 += RP) {
#pragma unroll
        for (int kt = 0; kt < n; ++kt)
#pragma unroll
          for (int r = 0; r < RP; ++r)
            if (t0 + r < TPC) {
              block(blk, LC, cur, nxt, b[kt], acc[t0 + r]);
              if (LC > PW && blk == 0) beside();
              ++blk;
            }
        if (t0 > 0) finish(t0 - RP);
      }
      skip(TPC * n, LC, cur, nxt);
      if (LATE && decltype(with_z)::value) {
        square(last, zz);
        Z = ReduceOwn<T, NTL>::run(zz) + T(rho[i]);
      }
      finish((TPC - 1) / RP * RP);
      return ReduceOwn<T, NTL>::run(pp);
    };
    if constexpr (!QUAD) {
      // the four candidates one after the other: their operands are one run of
      // the stream, so the window needs no look-ahead, and a candidate that no row
      // needs (forbidden to all, near the chain's end) only moves it on
      int si[NTL];
      const bool one = (M.own & (M.own - 1)) == 0;   // every row has the same state
#pragma unroll
      for (int t = 0; t < NTL; ++t) si[t] = site_state(lo[t], hi[t], i);
      auto step = [&](int s, auto off) {
        constexpr int O = decltype(off)::value;   // window slot of the part's first block
        const int cur = C0 + LC * s;
        if ((cand >> s) & 1u) {
          V acc[TPC][NTL];
          T pp[NTL];
#pragma unroll
          for (int tt = 0; tt < TPC; ++tt)
#pragma unroll
            for (int t = 0; t < NTL; ++t) acc[tt][t] = vb[tt];
#pragma unroll
          for (int t = 0; t < NTL; ++t) pp[t] = T(0);
          if (s < 3) fetch_v(s + 1);
#pragma unroll
          for (int blk = 0; blk < LC; ++blk) {
            constexpr int NB = TPC * n;
            if (blk < NB) {
              const V a = an[(O + blk) % PW];
#pragma unroll
              for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int t = 0; t < NTL; ++t) acc[blk / n][t] = mfma(a[v], b[blk % n][t][v], acc[blk / n][t]);
            }
            an[(O + blk) % PW] = ld(cur + blk + PW);
            __builtin_amdgcn_sched_barrier(6);   // as in block()
          }
#pragma unroll
          for (int tt = 0; tt < TPC; ++tt)
#pragma unroll
            for (int t = 0; t < NTL; ++t)
#pragma unroll
              for (int v = 0; v < 4; ++v) pp[t] = tfma(acc[tt][t][v], acc[tt][t][v], pp[t]);
          if ((M.own >> s) & 1u) {
            if (one) {
#pragma unroll
              for (int tt = 0; tt < TPC; ++tt)
#pragma unroll
                for (int t = 0; t < NTL; ++t) h[tt][t] = acc[tt][t];
            } else {
#pragma unroll
              for (int tt = 0; tt < TPC; ++tt)
#pragma unroll
                for (int t = 0; t < NTL; ++t)
#pragma unroll
                  for (int v = 0; v < 4; ++v) h[tt][t][v] = si[t] == s ? acc[tt][t][v] : h[tt][t][v];
            }
          }
          const T ps = ReduceOwn<T, NTL>::run(pp);
          const uint64_t al = ((s & 1) ? M.a1 : M.a0) & ((s & 2) ? M.b1 : M.b0);
          if (osi == s) pc = ps;
          if ((al >> lane) & 1u) Zs += ps;
        } else {
          if (s < 3) fetch_v(s + 1);
#pragma unroll
          for (int blk = 0; blk < LC; ++blk) an[(O + blk) % PW] = ld(cur + blk + PW);
        }
      };
      look_ahead();
      if constexpr (LC % PW == 0) {
#pragma unroll 1
        for (int s = 0; s < 4; ++s) step(s, std::integral_constant<int, 0>{});
      } else {
        step(0, std::integral_constant<int, 0>{});
        step(1, std::integral_constant<int, LC % PW>{});
        step(2, std::integral_constant<int, 2 * LC % PW>{});
        step(3, std::integral_constant<int, 3 * LC % PW>{});
      }
    } else if ((cand & (cand - 1)) == 0) {
      // one candidate: every row's own
      pc = candidate(__builtin_ctz(cand), pn, -1, std::true_type{}, [&](int tt, int t, const V& x) { h[tt][t] = x; }, look_ahead);
      Zs = pc;
    } else {
      int si[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) si[t] = site_state(lo[t], hi[t], i);
      if (LATE) {
        square(last, zz);
        Z = ReduceOwn<T, NTL>::run(zz) + T(rho[i]);
      }
      look_ahead();
      bool first = true;   // the first candidate's state for every row, the later ones' for theirs
#pragma unroll 1
      for (uint32_t rem = cand; rem; rem &= rem - 1) {
        const int s = __builtin_ctz(rem);
        const uint32_t later = rem & (rem - 1);
        const int s2 = later ? __builtin_ctz(later) : -1;
        const uint64_t al = ((s & 1) ? M.a1 : M.a0) & ((s & 2) ? M.b1 : M.b0);
        const int nxt = later ? C0 + LC * s2 : pn;
        const T ps = candidate(
            s, nxt, s2, std::false_type{},
            [&](int tt, int t, const V& x) {
              const bool mine = first || si[t] == s;
#pragma unroll
              for (int v = 0; v < 4; ++v) h[tt][t][v] = mine ? x[v] : h[tt][t][v];
            },
            [] {});
        first = false;
        if (osi == s) pc = ps;
        if ((al >> lane) & 1u) Zs += ps;
      }
    }
    // the carried state and the sign (or phase) of w.h + c
    T dp[NTL], dq[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) dp[t] = dq[t] = T(0);
    V* wr = ring + size_t(wsl[i]) * SLOT;
#pragma unroll
    for (int tt = 0; tt < TPC; ++tt) {
#pragma unroll
      for (int t = 0; t < NTL; ++t) {
        const V x = h[tt][t];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          dp[t] = tfma(ww[tt][v], x[v], dp[t]);
          if (CPLX) dq[t] = tfma(w2[tt][v], x[v], dq[t]);
        }
        wr[(t * TPC + tt) * 64] = x;
        if (STORE == 1) {
          const int64_t r = base + 16 * t + j;
          if (r < X.ns) *reinterpret_cast<V*>(X.hs + (size_t(i) * X.ns + r) * CH + 16 * tt + 4 * g) = x;
        }
        if (STORE == 2 && base + 16 * t + j < R && i < te1[t] && ((tneed[t] >> i) & 1ull))
          *reinterpret_cast<V*>(X.nhs + size_t(toff[t] + __popcll(tneed[t] & low_bits(i))) * CH + 16 * tt + 4 * g) = x;
      }
    }
    const T dot = ReduceOwn<T, NTL>::run(dp) + T(cc[i]);
    if (CPLX) {
      const T di = ReduceOwn<T, NTL>::run(dq) + T(cc2[i]);
      if (dot != T(0) || di != T(0)) {
        const T nr = zr * dot - zi * di;
        const T ni = zr * di + zi * dot;
        const T an_ = fabs(nr) > fabs(ni) ? fabs(nr) : fabs(ni);
        int ez;
        (void)tfrexp(an_, &ez);
        zr = ldexp(nr, -ez);
        zi = ldexp(ni, -ez);
      }
    }
    int ex;
    prod = tfrexp(prod * (pc / (QUAD && ((M.full >> lane) & 1u) ? Z : Zs)), &ex);
    pexp += ex;
    if (sums) {
      prod2 = tfrexp(prod2 * (pc / Zs), &ex);
      pexp2 += ex;
    }
    if (!CPLX && dot < T(0)) sgn = -sgn;
    M = Mn;
  };
  for (int i = i0; i < iend; ++i) {
    store_pre(i);
    if constexpr (DM == 1) {
      site(i, std::integral_constant<int, 1>{});
    } else {
      const int d = fptr[i + 1] - fptr[i];
      if (d == 2) site(i, std::integral_constant<int, 2>{});
      else if (DM == 2 || d == 1) site(i, std::integral_constant<int, 1>{});
      else site(i, std::integral_constant<int, DM == 3 ? 3 : 1>{});
    }
  }
  store_pre(iend);
  if (writer && olive) {
    const bool bad = ends.bad;
    const bool two = QUAD && self;
    const T pf = two ? prod2 : prod;
    lphi[orow] = bad ? -INFINITY : 0.5 * (log(double(pf)) + double(two ? pexp2 : pexp) * 0.69314718055994530942);
    sphi[orow] = int8_t(bad ? 0 : sgn);
    if (CPLX) phs[orow] = bad ? 0.0 : atan2(double(zi), double(zr));
  }
}

template <typename T, int CH, int NTL, int DM, int STORE, bool CPLX>
hipError_t run_tri(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi, hipStream_t st,
                   const PsiStates<T>& X, double* phs) {
  static_assert(NTL <= 2, "a lane group owns the rows of one of at most two tiles");
  const size_t per_wave = size_t(P.W) * 16 * NTL * CH * sizeof(T);
  if (per_wave > 160 * 1024) return hipErrorInvalidValue;
  // one wavefront per workgroup: its LDS goes to the next as soon as it ends
  // (four to a workgroup: K = 50 FP64 row kernel 127 against 119 ms at 4096 samples)
  hipLaunchKernelGGL((k_psi_tri<T, CH, NTL, DM, STORE, CPLX>), dim3(unsigned((R + 16 * NTL - 1) / (16 * NTL))),
                     dim3(64), per_wave, st, P, m, R, lphi, sphi, X, phs);
  return hipGetLastError();
}

// FP64: one tile of rows per wavefront in launches of at most kTriOneTileRows rows
// (one wavefront of one tile per SIMD, 256 CUs x 4): such a launch lasts as long as
// one wavefront's chain of matrix instructions, which a second tile doubles.  The
// samples' own pass (STORE 1) evaluates all four candidates besides the triangular
// factor and is that small up to 16384 samples, so it has this form alone.  One
// sample at K = 36, NN+NNN, chi = 64, us in psi.hip / with two tiles / with one: own
// pass 635 / 1340 / 711, its 8 k rows 721 / 654 / 342, its nodes 709 / 801 / 390.
constexpr int64_t kTriOneTileRows = 16 * 256 * 4;
template <typename T, int CH, int DM, int STORE, bool CPLX>
hipError_t run_tri_tiles(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi, hipStream_t st,
                         const PsiStates<T>& X, double* phs) {
  constexpr int NTL = sizeof(T) == 8 ? tri_tiles(CH, DM) : tri_tiles32(CH);
  constexpr bool one = sizeof(T) == 8 && NTL > 1;
  if constexpr (one && STORE == 1) {
    return run_tri<T, CH, 1, DM, STORE, CPLX>(P, m, R, lphi, sphi, st, X, phs);
  } else {
    if constexpr (one)
      if (R <= kTriOneTileRows) return run_tri<T, CH, 1, DM, STORE, CPLX>(P, m, R, lphi, sphi, st, X, phs);
    return run_tri<T, CH, NTL, DM, STORE, CPLX>(P, m, R, lphi, sphi, st, X, phs);
  }
}

template <typename T, int CH, int DM>
hipError_t run_tri_modes(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi, hipStream_t st,
                         const PsiStates<T>& X, int mode, double* phs) {
  // (FP32 rows have one form of Z)
  const int store = mode == PSI_STORE ? 1 : (mode == PSI_NODE ? 2 : (mode == PSI_ROWS && sizeof(T) == 8 ? 3 : 0));
  if (phs) {
    switch (store) {
      case 0: return run_tri_tiles<T, CH, DM, 0, true>(P, m, R, lphi, sphi, st, X, phs);
      case 1: return run_tri_tiles<T, CH, DM, 1, true>(P, m, R, lphi, sphi, st, X, phs);
      case 2: return run_tri_tiles<T, CH, DM, 2, true>(P, m, R, lphi, sphi, st, X, phs);
      default:
        if constexpr (sizeof(T) == 8) return run_tri_tiles<T, CH, DM, 3, true>(P, m, R, lphi, sphi, st, X, phs);
        return hipErrorInvalidValue;
    }
  }
  if constexpr (sizeof(T) == 4 && CH == 16 && DM == 1) {
    return hipErrorInvalidValue;   // psi.hip's (tri32 in runtime.cpp)
  } else {
    switch (store) {
      case 0: return run_tri_tiles<T, CH, DM, 0, false>(P, m, R, lphi, sphi, st, X, phs);
      case 1: return run_tri_tiles<T, CH, DM, 1, false>(P, m, R, lphi, sphi, st, X, phs);
      case 2: return run_tri_tiles<T, CH, DM, 2, false>(P, m, R, lphi, sphi, st, X, phs);
      default:
        if constexpr (sizeof(T) == 8) return run_tri_tiles<T, CH, DM, 3, false>(P, m, R, lphi, sphi, st, X, phs);
        return hipErrorInvalidValue;
    }
  }
}

template <typename T, int CH>
hipError_t run_tri_ch(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi, hipStream_t st,
                      const PsiStates<T>& X, int mode, double* phs) {
  switch (P.dmax) {
    case 1: return run_tri_modes<T, CH, 1>(P, m, R, lphi, sphi, st, X, mode, phs);
    case 2: return run_tri_modes<T, CH, 2>(P, m, R, lphi, sphi, st, X, mode, phs);
    case 3: return run_tri_modes<T, CH, 3>(P, m, R, lphi, sphi, st, X, mode, phs);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace nqs
