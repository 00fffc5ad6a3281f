// Oversampled-grid FFTs of the two NUFFTs (Section 2, eqs. 2.5-2.6 and the
// deconvolution step; the type-2 transform runs the type-1 steps in reverse).
//
// Each 3D FFT is three passes of batched 1D transforms, one per axis.  A pass
// stages LB lines of length L in LDS, runs a Stockham autosort FFT with radices
// 8, 4, 2, 3, 5 (also 16 in Algorithm 2's float32 paired passes; twiddles from
// a float64 table rounded to the working type), and writes the lines back.
// Zero padding is never stored: forward passes place the N nonzero inputs of a
// line at fine indices (m mod L), m in [-N/2, N/2), and zero the rest in LDS;
// inverse passes write only those N outputs (the crop to the physical grid).
//
//   forward (type-2 front, sign -1):
//     Z: rho (N0 N1 N2 reals) x H/(phi^0 phi^1 phi^2)  -> A1 [N0][N1][nf2]
//     Y: A1 -> A2 [N0][nf1][nf2]
//     X: A2 -> F  [nf0][nf1][nf2]
//   inverse (type-1 back, sign +1):
//     X: G  -> B2 [N0][nf1][nf2]
//     Y: B2 -> B1 [N0][N1][nf2]
//     Z: B1 -> u = Re(.) / (phi^0 phi^1 phi^2), and partial sums of rho u
//
// Algorithm 2 (JGB_FLAG_SPLIT) changes four things: the forward Z pass also
// places rho H in the imaginary part (two real transforms in one complex
// one); the potential's forward FFT stops before the last axis (X in 3D, Y in
// 2D) and a paired unmix pass along it writes the type-2 grid into the tiles
// the interpolation reads; the inverse's first pass is a fused paired pass that
// transforms the same inputs forward again, forms the combined spectrum of both
// halves and transforms it back (so the full forward spectrum is never
// stored); and the last pass adds the imaginary part (I1) to u.  The
// energy-only and transform calls run the full forward FFT into F.
#include <algorithm>
#include <cmath>

#include "regpair.h"

namespace jgb {

using namespace fft;

namespace {

template <typename T, int KIND, int MAXV, int NT>
__global__ void __launch_bounds__(NT) k_fft_pass(PassArgs<T> a) {
  fft_pass_body<T, KIND, MAXV, NT>(a, blockIdx.x);
}
// Algorithm 2's paired passes along the last forward / first inverse axis.  A
// block takes P lines (a, b) of one row a and their mirrors
// ((A - a) mod A, (B - b) mod B), loads the lines' N inputs from the output of
// the forward pass before (the other axes already transformed), zero-pads them
// to L in LDS and runs the forward transform there, so that Z(q) and Z(-q)
// (element (L - e) mod L of the mirror line) sit in the block's LDS together.
//   PAIR_UNMIX: writes A = (Z(q) + conj Z(-q)) / 2 into the gather tiles of G
//     that the interpolation reads (only blocks with such a tile run);
//   PAIR_FUSED: forms the inverse transform's spectrum
//       Y(q) = (G(q) + conj G(-q)) / 2 + M'(q) (Z(q) - conj Z(-q)) / 2  (splitsym.h),
//     each thread writing Y at q and at -q, transforms both lines back and
//     stores the cropped outputs.
// Z is never stored: the unmix pass touches a few lines, and the fused pass
// reads the N-point inputs instead of the L-point spectrum.  Every line is
// owned by one block; a line that is its own mirror sits in two rows of its
// block, which end up equal.  Registers are capped at 128 (four waves per SIMD).
template <typename T, int MODE, int MAXV, int NT>
__global__ void __launch_bounds__(NT, 4) k_fft_pair_pass(PassArgs<T> a) {
  extern __shared__ unsigned char smem_raw[];
  C2<T>* lds = reinterpret_cast<C2<T>*>(smem_raw);
  const int L = a.L;
  const int ldl = L + 1;
  const int P = a.P;
  const int LB = 2 * P;
  // The logical block.  Unmix: from the plan's list.  Fused: workgroups are
  // dealt round robin to the eight XCDs, so workgroup w runs on XCD w mod 8;
  // the logical ids are dealt out in runs, one run per XCD, so that
  // neighbouring chunks share an L2 (a chunk's mirror run is misaligned by one
  // element and shares its edge segments with the next chunk's).
  int bid;
  if constexpr (MODE == PAIR_UNMIX) {
    bid = a.blist[blockIdx.x];
  } else {
    const int nb = (int)gridDim.x, w = (int)blockIdx.x;
    const int x = w & 7, q = nb >> 3, r = nb & 7;
    bid = x * q + (x < r ? x : r) + (w >> 3);
  }
  // the block's row and chunk
  int ar, c;
  bool self;
  if (bid < a.nb1) {
    ar = 1 + bid / a.cb;
    c = bid % a.cb;
    self = false;
  } else {
    const int sb = bid - a.nb1;
    ar = (sb / a.cs == 0) ? 0 : a.A / 2;
    c = sb % a.cs;
    self = true;
  }
  // line slot l < P: own line (ar, c P + l); l >= P: the mirror of slot l - P
  // (ar <= A/2 and bq < B, so the mirror indices need no division)
  auto line_of = [&](int l, int& la, int& lb) {
    const int j = (l < P) ? l : l - P;
    int bq = c * P + j;
    const bool valid = self ? (bq <= a.B / 2) : (bq < a.B);
    if (!valid) bq = 0;
    if (l < P) {
      la = ar;
      lb = bq;
    } else {
      la = ar ? a.A - ar : 0;
      lb = bq ? a.B - bq : 0;
    }
    return valid;
  };
  const C2<T>* X = (const C2<T>*)a.in;
  const SplitSym& sy = a.sym;
  // tables after the lines: the element axis's frequencies and window values,
  // per line slot the constant parts of |k|^2, p, n.k and m.k, and the line's
  // row of gather-tile flags along the element axis
  const int ea = a.dim3 ? 0 : 1;                              // the element axis
  const int gse = a.dim3 ? sy.gs0 : sy.gs1;                    // its tile shift
  const int ngte = (L + (1 << gse) - 1) >> gse;                // its tiles
  double* sk = reinterpret_cast<double*>(smem_raw + (size_t)LB * ldl * sizeof(C2<T>));
  double* se = sk + L;
  double* lkk = se + L;
  double* lw = lkk + LB;
  double* lnk = lw + LB;
  double* lmk = lnk + LB;
  unsigned char* ltf = reinterpret_cast<unsigned char*>(lmk + LB);  // LB x ngte
  const int N = a.nin;
  // zero the padding of every line: fine positions [N - N/2, L - N/2)
  for (int idx = threadIdx.x; idx < LB * (L - N); idx += NT) {
    const int e = (int)a.dLB.div(idx), l = idx - e * LB;
    lds[l * ldl + (N - N / 2) + e] = C2<T>{T(0), T(0)};
  }
  // load the N inputs of both line sets, all loads issued before the LDS writes
  {
    const int total_in = LB * N;
    C2<T> buf[MAXV];
    int dst[MAXV];
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      if (i * NT >= total_in) {  // uniform: the inputs are N of L per line
        buf[i] = C2<T>{T(0), T(0)};
        dst[i] = -1;
        continue;
      }
      const int idx0 = threadIdx.x + i * NT;
      const bool ok = idx0 < total_in;
      const int idx = ok ? idx0 : 0;
      const int e = (int)a.dLB.div(idx);
      const int l = idx - e * LB;
      int la, lb;
      const bool valid = line_of(l, la, lb) && ok;
      const C2<T> v = X[(int64_t)e * a.es_in + (int64_t)la * a.B + lb];
      buf[i] = valid ? v : C2<T>{T(0), T(0)};
      dst[i] = ok ? l * ldl + fine_pos(e, N, L) : -1;
    }
    for (int t = threadIdx.x; t < L + LB + LB * ngte; t += NT) {
      if (t < L) {
        sk[t] = sy.kt[sy.koff[ea] + t];
        se[t] = sy.kt[sy.eoff[ea] + t];
      } else if (t < L + LB) {
        const int l = t - L;
        int la, lb;
        line_of(l, la, lb);
        const double k2 = sy.kt[sy.koff[2] + lb];
        double k1 = 0.0, w = 1.0;
        if (a.dim3) {
          k1 = sy.kt[sy.koff[1] + la];
          w = sy.kt[sy.eoff[1] + la] * sy.kt[sy.eoff[2] + lb];
        }
        lkk[l] = k1 * k1 + k2 * k2;
        lw[l] = w;
        // n.k over the physical axes: 3D (x1, x2, x3) = (a0, a1, a2), the
        // element carrying n_1; 2D (x1, x2) = (a1, a2), the element again n_1
        lnk[l] = a.dim3 ? sy.axis[1] * k1 + sy.axis[2] * k2 : sy.axis[1] * k2;
        lmk[l] = a.dim3 ? sy.axis2[1] * k1 + sy.axis2[2] * k2 : sy.axis2[1] * k2;
      } else {
        const int r = t - L - LB;
        const int l = r / ngte, te = r - l * ngte;
        int la, lb;
        line_of(l, la, lb);
        const int tile = a.dim3 ? ((te * sy.gnt1 + (la >> sy.gs1)) * sy.gnt2 + (lb >> sy.gs2))
                                : (te * sy.gnt2 + (lb >> sy.gs2));
        ltf[l * ngte + te] = sy.tflag[tile];
      }
    }
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
      if (dst[i] >= 0) lds[dst[i]] = buf[i];
  }
  __syncthreads();
  // forward transform of the 2P lines (sign -1): Z
  {
    int Ns = 1;
    for (int st = 0; st < a.nrad; ++st) {
      const int R = a.rad[st];
      const FastDiv& dNs = a.dNs[st];
      const int tws = a.tws[st];
      switch (R) {
        case 16:
          // float32 only: the radix-16 stage's registers would cost the float64
          // kernels occupancy (the plan never gives them radix 16)
          if constexpr (sizeof(T) == 4) stage<T, 16, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(-1));
          break;
        case 8: stage<T, 8, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(-1)); break;
        case 5: stage<T, 5, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(-1)); break;
        case 4: stage<T, 4, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(-1)); break;
        case 3: stage<T, 3, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(-1)); break;
        default: stage<T, 2, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(-1)); break;
      }
      Ns *= R;
    }
  }
  C2<T>* G = (C2<T>*)a.G;
  if constexpr (MODE == PAIR_UNMIX) {
    // A at every element pair (own line l, element e) <-> (mirror slot l + P,
    // (L - e) mod L) whose gather tile the interpolation reads; A(-q) = conj A(q)
    for (int idx = threadIdx.x; idx < P * L; idx += NT) {
      const int e = (int)a.dP.div(idx);
      const int l = idx - e * P;
      int la, lb;
      if (!line_of(l, la, lb)) continue;
      const int em = e ? L - e : 0;
      const int lm = l + P;
      const C2<T> zq = lds[l * ldl + e], zm = lds[lm * ldl + em];
      const C2<T> aq{T(0.5) * (zq.x + zm.x), T(0.5) * (zq.y - zm.y)};
      if (ltf[l * ngte + (e >> gse)]) {
        const int q0 = a.dim3 ? e : 0, q1 = a.dim3 ? la : e;
        G[((int64_t)q0 * sy.nf1 + q1) * sy.nf2 + lb] = aq;
      }
      if (ltf[lm * ngte + (em >> gse)]) {
        int ma, mb;
        line_of(lm, ma, mb);
        const int m0 = a.dim3 ? em : 0, m1 = a.dim3 ? ma : em;
        G[((int64_t)m0 * sy.nf1 + m1) * sy.nf2 + mb] = C2<T>{aq.x, -aq.y};
      }
    }
    return;
  }
  // form Y at every element pair (own line l, element e) <-> (mirror slot l + P, (L - e) mod L)
  {
    const bool dip = sy.kernel == JGB_DIPOLE_3D || sy.kernel == JGB_DIPOLE_2D;
    for (int idx = threadIdx.x; idx < P * L; idx += NT) {
      const int e = (int)a.dP.div(idx);
      const int l = idx - e * P;
      int la, lb;
      if (!line_of(l, la, lb)) continue;
      const int em = e ? L - e : 0;
      const int lm = l + P;
      const double ke = sk[e];
      double M = split_symbol_core(sy, ke * ke + lkk[l], se[e] * lw[l], sy.axis[0] * ke + lnk[l],
                                   sy.axis2[0] * ke + lmk[l]);
      if (dip && (2 * e == L || 2 * lb == a.B || (a.dim3 && 2 * la == a.A))) {
        // on a Nyquist plane, the mean with the mirror's symbol; off them the
        // mirror's k is exactly -k (the frequencies are 2 pi q' / (2 R) with
        // q' a signed integer) and its symbol equals M bit for bit
        const double km = sk[em];
        M = 0.5 * (M + split_symbol_core(sy, km * km + lkk[lm], se[em] * lw[lm], sy.axis[0] * km + lnk[lm],
                                         sy.axis2[0] * km + lmk[lm]));
      }
      C2<T>* pq = lds + l * ldl + e;
      C2<T>* pm = lds + lm * ldl + em;
      const C2<T> zq = *pq, zm = *pm;
      const T hm = (T)(0.5 * M);
      // D(q) = Z(q) - conj Z(-q) = 2 i B(q); D(-q) = -conj D(q)
      const T dx = zq.x - zm.x, dy = zq.y + zm.y;
      C2<T> gq{T(0), T(0)}, gm{T(0), T(0)};
      if (ltf[l * ngte + (e >> gse)]) {
        const int q0 = a.dim3 ? e : 0, q1 = a.dim3 ? la : e;
        gq = G[((int64_t)q0 * sy.nf1 + q1) * sy.nf2 + lb];
      }
      if (ltf[lm * ngte + (em >> gse)]) {
        int ma, mb;
        line_of(lm, ma, mb);
        const int m0 = a.dim3 ? em : 0, m1 = a.dim3 ? ma : em;
        gm = G[((int64_t)m0 * sy.nf1 + m1) * sy.nf2 + mb];
      }
      *pq = C2<T>{T(0.5) * (gq.x + gm.x) + hm * dx, T(0.5) * (gq.y - gm.y) + hm * dy};
      *pm = C2<T>{T(0.5) * (gm.x + gq.x) - hm * dx, T(0.5) * (gm.y - gq.y) + hm * dy};
    }
  }
  __syncthreads();
  // inverse transform of the 2P lines (sign +1)
  {
    int Ns = 1;
    for (int st = 0; st < a.nrad; ++st) {
      const int R = a.rad[st];
      const FastDiv& dNs = a.dNs[st];
      const int tws = a.tws[st];
      switch (R) {
        case 16:
          // float32 only: the radix-16 stage's registers would cost the float64
          // kernels occupancy (the plan never gives them radix 16)
          if constexpr (sizeof(T) == 4) stage<T, 16, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(1));
          break;
        case 8: stage<T, 8, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(1)); break;
        case 5: stage<T, 5, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(1)); break;
        case 4: stage<T, 4, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(1)); break;
        case 3: stage<T, 3, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(1)); break;
        default: stage<T, 2, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, a.tw, T(1)); break;
      }
      Ns *= R;
    }
  }
  // store the cropped outputs of both line sets
  {
    const int total_out = LB * a.nout;
    C2<T> buf[MAXV];
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      if (i * NT >= total_out) {
        buf[i] = C2<T>{T(0), T(0)};
        continue;
      }
      const int idx0 = threadIdx.x + i * NT;
      const int idx = idx0 < total_out ? idx0 : 0;
      const int e = (int)a.dLB.div(idx);
      const int l = idx - e * LB;
      buf[i] = lds[l * ldl + fine_pos(e, a.nout, L)];
    }
    C2<T>* out = (C2<T>*)a.out;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      const int idx = threadIdx.x + i * NT;
      if (idx >= total_out) continue;
      const int e = (int)a.dLB.div(idx);
      const int l = idx - e * LB;
      int la, lb;
      if (!line_of(l, la, lb)) continue;
      out[(int64_t)e * a.es_out + (int64_t)la * a.B + lb] = buf[i];
    }
  }
}

void factor(int L, int* rad, int& nrad, bool radix16 = false) {
  nrad = 0;
  int m = L;
  while (radix16 && m % 16 == 0) {
    rad[nrad++] = 16;
    m /= 16;
  }
  while (m % 8 == 0) {
    rad[nrad++] = 8;
    m /= 8;
  }
  while (m % 4 == 0) {
    rad[nrad++] = 4;
    m /= 4;
  }
  while (m % 2 == 0) {
    rad[nrad++] = 2;
    m /= 2;
  }
  while (m % 3 == 0) {
    rad[nrad++] = 3;
    m /= 3;
  }
  while (m % 5 == 0) {
    rad[nrad++] = 5;
    m /= 5;
  }
}

static_assert(pass_cap<double, PASS_COMPLEX>() >= 1024 && pass_cap<float, PASS_COMPLEX>() >= 1024 &&
                  pass_cap<double, PASS_FWD_Z>() >= 1024 && pass_cap<float, PASS_FWD_Z>() >= 1024 &&
                  pass_cap<double, PASS_COMPLEX_Z>() >= 1024 && pass_cap<double, PASS_PAIR>() >= 2048 &&
                  pass_cap<float, PASS_PAIR>() >= 2048,
              "a block must stage at least one line of nf = 1024 points");
// The first forward and last inverse passes run the same lines with the same
// shape: their per-block partial sums (d_mparts, d_eparts) are counted once,
// by fft_inverse_z_blocks.
static_assert(pass_cap<double, PASS_FWD_Z>() == pass_cap<double, PASS_INV_Z>() &&
                  pass_cap<float, PASS_FWD_Z>() == pass_cap<float, PASS_INV_Z>(),
              "the Z passes share their block shape");

template <typename T, int KIND = PASS_PAIR>
int lines_per_block(int L) {
  const int cap = pass_elems<T, KIND>() * pass_threads<T, KIND>();  // complex elements staged per block
  const int maxlb = sizeof(T) == 8 ? 16 : 32;
  int lb = cap / L;
  if (lb > maxlb) lb = maxlb;
  if (lb < 1) lb = 1;
  if (KIND == PASS_HSYM)  // a power of two, dividing the block's threads
    while (lb & (lb - 1)) lb &= lb - 1;
  return lb;
}

// The oversampled grid's passes (half the line zero on input or cropped on
// output) of a length with a kernel of its own go there; the kernels below
// take every other length and the periodic passes.
template <typename T, int KIND>
hipError_t run_reg_pass(const PassArgs<T>& a, hipStream_t s) {
  if constexpr (KIND == PASS_FWD_Z) return launch_reg_pass<T, RP_FWD_Z>(a, s);
  if constexpr (KIND == PASS_INV_Z) return launch_reg_pass<T, RP_INV_Z>(a, s);
  if constexpr (KIND == PASS_HSYM) return launch_reg_pass<T, RP_HSYM>(a, s);
  if constexpr (KIND == PASS_COMPLEX) return a.nin < a.L ? launch_reg_pass<T, RP_FWD>(a, s) : launch_reg_pass<T, RP_INV>(a, s);
  return hipErrorInvalidValue;
}

template <typename T, int KIND>
bool reg_pass_fits(const PassArgs<T>& a) {
  if (!reg_length<T>(a.L) || a.nlines >= (1 << 30)) return false;
  if (KIND == PASS_FWD_Z) return 2 * a.nin == a.L && a.nout == (a.half_out ? a.L / 2 + 1 : a.L);
  if (KIND == PASS_INV_Z) return 2 * a.nout == a.L && a.nin == (a.half_in ? a.L / 2 + 1 : a.L);
  // the float32 kernels of the strided passes move two neighbouring lines at a
  // time: even strides, and rows at least one longer than an odd count of lines
  const bool pairs = sizeof(T) == 8 ||
                     (a.in_is == 1 && a.out_is == 1 && a.in_es % 2 == 0 && a.out_es % 2 == 0 && a.in_os % 2 == 0 &&
                      a.out_os % 2 == 0 && std::min(a.in_es, a.out_es) >= a.ic + a.ic % 2 && std::min(a.in_os, a.out_os) >= a.ic + a.ic % 2);
  if (KIND == PASS_HSYM) return pairs && a.nin == a.L && 2 * a.nout == a.L && a.lext;
  if (KIND == PASS_COMPLEX)
    return pairs && (a.sign < 0 ? 2 * a.nin == a.L && a.nout == a.L : a.nin == a.L && 2 * a.nout == a.L);
  return false;
}

// The batched form of an any-length pass is the register passes' own, so that
// a site of the batch's pipeline is one launch whatever its members' lengths.
template <typename T, int RP>
hipError_t record_as(const PassArgs<T>& a, unsigned blocks, size_t smem) {
  launch_recorded(a, &launch_reg_batch<T, RP>, blocks, reg_batch_threads<T, RP>(), smem);
  return hipSuccess;
}
template <typename T, int KIND>
hipError_t record_any_pass(const PassArgs<T>& a, unsigned blocks, size_t smem) {
  if constexpr (KIND == PASS_FWD_Z) return record_as<T, RP_FWD_Z>(a, blocks, smem);
  if constexpr (KIND == PASS_INV_Z) return record_as<T, RP_INV_Z>(a, blocks, smem);
  if constexpr (KIND == PASS_HSYM) return record_as<T, RP_HSYM>(a, blocks, smem);
  if constexpr (KIND == PASS_COMPLEX)
    return a.sign < 0 ? record_as<T, RP_FWD>(a, blocks, smem) : record_as<T, RP_INV>(a, blocks, smem);
  return hipErrorInvalidValue;  // the periodic passes are never batched
}

template <typename T, int KIND>
hipError_t run_pass(const Plan& pl, int stage, PassArgs<T> a, hipStream_t s) {
  a.dic = FastDiv((uint32_t)a.ic);
  a.dn1 = FastDiv((uint32_t)(a.n1 > 0 ? a.n1 : 1));
  if (reg_pass_fits<T, KIND>(a)) {
    // two neighbouring lines per thread in float32 (RegShape::V)
    const int64_t per = sizeof(T) == 4 ? (a.ic + 1) / 2 : a.ic;
    a.dgrp = FastDiv((uint32_t)per);
    a.ngroups = a.nlines / a.ic * per;
    stage_mark(pl, stage, 0, s);
    const hipError_t e = run_reg_pass<T, KIND>(a, s);
    stage_mark(pl, stage, 1, s);
    return e;
  }
  factor(a.L, a.rad, a.nrad);
  a.LB = lines_per_block<T, KIND>(a.L);
  // with an output reach per line, a thread's elements must lie on one line:
  // the lines per block divide the thread count
  if (KIND == PASS_COMPLEX && a.oext)
    while (pass_threads<T, KIND>() % a.LB != 0) --a.LB;
  {
    int Ns = 1;
    for (int st = 0; st < a.nrad; ++st) {
      a.dNs[st] = FastDiv((uint32_t)Ns);
      a.tws[st] = a.L / (Ns * a.rad[st]);
      Ns *= a.rad[st];
    }
  }
  if (a.nlines >= (1 << 30) || (int64_t)a.LB * a.L >= (1 << 30)) return hipErrorInvalidValue;
  // whole lines, with reaches; a thread's elements on one line
  if (KIND == PASS_HSYM && (a.nin != a.L || !a.lext || pass_threads<T, KIND>() % a.LB != 0)) return hipErrorInvalidValue;
  // an output reach per line, the thread's elements on one whole line
  if (a.oext && (KIND != PASS_COMPLEX || a.nout != a.L || pass_threads<T, KIND>() % a.LB != 0))
    return hipErrorInvalidValue;
  a.dLB = FastDiv((uint32_t)a.LB);
  a.dnin = FastDiv((uint32_t)a.nin);
  a.dnout = FastDiv((uint32_t)a.nout);
  unsigned blocks = (unsigned)((a.nlines + a.LB - 1) / a.LB);
  // lines, deconvolution factors (Z passes), twiddles (strided passes)
  constexpr bool TW_LDS = KIND == PASS_COMPLEX || KIND == PASS_KINETIC || KIND == PASS_HSYM;
  const size_t smem = pass_twiddle_offset<T>(a.LB, a.L, has_factors<KIND>()) + (TW_LDS ? (size_t)a.L * sizeof(C2<T>) : 0);
  constexpr int NT = pass_threads<T, KIND>();
  constexpr int MAXV = pass_elems<T, KIND>();
  stage_mark(pl, stage, 0, s);
  hipError_t e = hipSuccess;
  if (launch_record()) {
    e = record_any_pass<T, KIND>(a, blocks, smem);
  } else {
    hipLaunchKernelGGL((k_fft_pass<T, KIND, MAXV, NT>), dim3(blocks), dim3(NT), smem, s, a);
    e = hipGetLastError();
  }
  stage_mark(pl, stage, 1, s);
  return e;
}

// The paired passes of Algorithm 2 along the internal axis `axis` (0 in 3D:
// lines (q1, q2); 1 in 2D: lines q2): block geometry, shared with the plan's
// list of unmix blocks.
template <typename T>
unsigned pair_geometry(PassArgs<T>& a) {
  // float32: radix 16 (two stages for L = 256 instead of three; the pass runs
  // two transforms per line, and fewer LDS round trips pay there)
  factor(a.L, a.rad, a.nrad, sizeof(T) == 4);
  {
    int Ns = 1;
    for (int st = 0; st < a.nrad; ++st) {
      a.dNs[st] = FastDiv((uint32_t)Ns);
      a.tws[st] = a.L / (Ns * a.rad[st]);
      Ns *= a.rad[st];
    }
  }
  const int lb = lines_per_block<T>(a.L), own = a.dim3 ? reg_pair_lines<T>(a.L) : 0;
  a.P = own > 0 ? own : lb / 2 > 0 ? lb / 2 : 1;
  a.LB = 2 * a.P;
  a.dLB = FastDiv((uint32_t)a.LB);
  a.dP = FastDiv((uint32_t)a.P);
  a.cb = (a.B + a.P - 1) / a.P;
  a.cs = (a.B / 2 + 1 + a.P - 1) / a.P;
  a.nb1 = (a.A > 1) ? (a.A / 2 - 1) * a.cb : 0;
  return (unsigned)(a.nb1 + (a.A > 1 ? 2 : 1) * a.cs);
}

template <typename T, int MODE>
hipError_t run_pair_pass(const Plan& pl, int stage, PassArgs<T> a, hipStream_t s) {
  unsigned blocks = pair_geometry<T>(a);
  if (MODE == PAIR_UNMIX) {
    blocks = (unsigned)pl.nublocks;
    a.blist = pl.d_ublocks;
    if (blocks == 0) return hipSuccess;
  }
  if (a.dim3 && reg_pair_lines<T>(a.L) > 0 && 2 * a.nin == a.L && 2 * a.nout == a.L) {
    hipError_t e = hipErrorInvalidValue;
    stage_mark(pl, stage, 0, s);
    if constexpr (sizeof(T) == 8) e = launch_reg_pair<T, MODE>(a, blocks, s);
    stage_mark(pl, stage, 1, s);
    return e;
  }
  const int gse = a.dim3 ? a.sym.gs0 : a.sym.gs1;
  const int ngte = (a.L + (1 << gse) - 1) >> gse;
  const size_t smem = (size_t)a.LB * (a.L + 1) * sizeof(C2<T>) + sizeof(double) * (2 * a.L + 4 * a.LB) +
                      (size_t)a.LB * ngte;
  constexpr int NT = pass_threads<T>();
  constexpr int MAXV = pass_elems<T>();
  stage_mark(pl, stage, 0, s);
  hipLaunchKernelGGL((k_fft_pair_pass<T, MODE, MAXV, NT>), dim3(blocks), dim3(NT), smem, s, a);
  stage_mark(pl, stage, 1, s);
  return hipGetLastError();
}

template <typename T>
PassArgs<T> base_args(const Plan& pl, int axis, T sign) {
  PassArgs<T> a{};
  a.L = pl.nf[axis];
  a.sign = sign;
  a.tw = (const C2<T>*)pl.d_tw[axis];
  a.n1 = pl.n[1];
  a.n2 = pl.n[2];
  return a;
}

// Algorithm 2's paired passes run along the last forward axis (a0 in 3D, a1 in
// 2D) on the output of the forward pass before it, which sits in W: 3D
// [n0][f1][f2], 2D [1][n1][f2].
template <typename T>
PassArgs<T> split_pair_args(const Plan& pl, int axis) {
  const bool has_x = pl.nf[0] > 1;
  PassArgs<T> a = base_args<T>(pl, axis, T(1));
  a.nin = (int)pl.n[axis];
  a.nout = (int)pl.n[axis];
  a.A = has_x ? (int)pl.nf[1] : 1;
  a.B = (int)pl.nf[2];
  a.es_in = has_x ? (int64_t)pl.nf[1] * pl.nf[2] : pl.nf[2];
  a.es_out = a.es_in;
  a.dim3 = has_x ? 1 : 0;
  a.in = pl.d_W;
  a.G = pl.d_G;
  a.sym = make_split_sym(pl);
  return a;
}

// The forward passes; with last = false the pass along the last axis (a0 in
// 3D, a1 in 2D) is left to Algorithm 2's paired passes.
template <typename T>
hipError_t forward_passes(const Plan& pl, const T* rho, hipStream_t s, bool last) {
  const int64_t n0 = pl.n[0], n1 = pl.n[1], n2 = pl.n[2];
  const int64_t f0 = pl.nf[0], f1 = pl.nf[1], f2 = pl.nf[2];
  const bool has_x = f0 > 1;
  // lines along axis 2 that the later passes keep (the Hermitian half
  // 0 .. f2/2 for a real input; all f2 otherwise) and their row stride
  const int64_t c2 = pl.r2c ? pl.h2 : f2, r2 = pl.r2c ? pl.hs2 : f2;
  // G belongs to the spreading: the intermediates use F and W
  void* A1 = has_x ? pl.d_F : pl.d_W;
  void* A2 = has_x ? pl.d_W : pl.d_F;
  hipError_t e;
  {  // Z: rho -> A1 [n0][n1][r2]
    PassArgs<T> a = base_args<T>(pl, 2, T(-1));
    a.nlines = n0 * n1;
    a.nin = (int)n2;
    a.nout = (int)c2;
    a.half_out = pl.r2c ? 1 : 0;
    a.ic = 1;
    a.in_os = n2;
    a.in_is = 0;
    a.in_es = 1;
    a.out_os = r2;
    a.out_is = 0;
    a.out_es = 1;
    a.in = rho;
    a.out = A1;
    a.dec0 = pl.d_deconv[0];
    a.dec1 = pl.d_deconv[1];
    a.dec2 = pl.d_deconv[2];
    a.scale = pl.H;
    a.split = pl.split ? 1 : 0;
    a.mparts = (pl.c0 != 0.0) ? pl.d_mparts : nullptr;
    if ((e = run_pass<T, PASS_FWD_Z>(pl, ST_FWD_Z, a, s)) != hipSuccess) return e;
  }
  if (has_x || last) {  // Y: A1 -> A2 [n0][f1][r2]
    PassArgs<T> a = base_args<T>(pl, 1, T(-1));
    a.nlines = n0 * c2;
    a.nin = (int)n1;
    a.nout = (int)f1;
    a.ic = c2;
    a.in_os = n1 * r2;
    a.in_is = 1;
    a.in_es = r2;
    a.out_os = f1 * r2;
    a.out_is = 1;
    a.out_es = r2;
    a.in = A1;
    a.out = A2;
    if ((e = run_pass<T, PASS_COMPLEX>(pl, ST_FWD_Y, a, s)) != hipSuccess) return e;
  }
  if (has_x && last) {  // X: A2 -> F [f0][f1][r2]
    PassArgs<T> a = base_args<T>(pl, 0, T(-1));
    a.nlines = f1 * c2;
    a.nin = (int)n0;
    a.nout = (int)f0;
    a.ic = c2;
    a.in_os = r2;
    a.in_is = 1;
    a.in_es = f1 * r2;
    a.out_os = r2;
    a.out_is = 1;
    a.out_es = f1 * r2;
    a.in = A2;
    a.out = pl.d_F;
    // Algorithm 1: the interpolation by tiles reads F only within each
    // line's reach (Algorithm 2's unmixing and Fourier-side energy read all
    // of F)
    a.oext = pl.tile_interp && !pl.split ? pl.d_fext : nullptr;
    if ((e = run_pass<T, PASS_COMPLEX>(pl, ST_FWD_X, a, s)) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

template <typename T>
hipError_t launch_fft_forward(const Plan& pl, const T* rho, hipStream_t s) {
  return forward_passes<T>(pl, rho, s, true);
}

template <typename T>
hipError_t launch_split_forward(const Plan& pl, const T* rho, hipStream_t s) {
  hipError_t e = forward_passes<T>(pl, rho, s, false);
  if (e != hipSuccess) return e;
  return run_pair_pass<T, PAIR_UNMIX>(pl, ST_SPLIT_UNMIX, split_pair_args<T>(pl, pl.nf[0] > 1 ? 0 : 1), s);
}

std::vector<int> split_unmix_blocks(const Plan& pl, const std::vector<unsigned char>& tf) {
  const int axis = pl.nf[0] > 1 ? 0 : 1;
  PassArgs<double> a = base_args<double>(pl, axis, 1.0);
  const SplitSym sy = make_split_sym(pl);
  a.A = pl.nf[0] > 1 ? (int)pl.nf[1] : 1;
  a.B = (int)pl.nf[2];
  a.dim3 = pl.nf[0] > 1 ? 1 : 0;
  unsigned nblocks;
  if (pl.fp64) {
    nblocks = pair_geometry<double>(a);
  } else {
    PassArgs<float> b{};
    b.L = a.L;
    b.A = a.A;
    b.B = a.B;
    b.dim3 = a.dim3;
    nblocks = pair_geometry<float>(b);
    a.P = b.P;
    a.cb = b.cb;
    a.cs = b.cs;
    a.nb1 = b.nb1;
  }
  const int gse = a.dim3 ? sy.gs0 : sy.gs1;
  const int ngte = (a.L + (1 << gse) - 1) >> gse;
  std::vector<int> out;
  for (int bid = 0; bid < (int)nblocks; ++bid) {
    int ar, c;
    bool self;
    if (bid < a.nb1) {
      ar = 1 + bid / a.cb;
      c = bid % a.cb;
      self = false;
    } else {
      const int sb = bid - a.nb1;
      ar = (sb / a.cs == 0) ? 0 : a.A / 2;
      c = sb % a.cs;
      self = true;
    }
    bool any = false;
    for (int l = 0; l < 2 * a.P && !any; ++l) {
      const int j = l < a.P ? l : l - a.P;
      const int bq = c * a.P + j;
      if (!(self ? (bq <= a.B / 2) : (bq < a.B))) continue;
      const int la = l < a.P ? ar : (ar ? a.A - ar : 0);
      const int lb = l < a.P ? bq : (bq ? a.B - bq : 0);
      for (int te = 0; te < ngte && !any; ++te) {
        const int tile = a.dim3 ? ((te * sy.gnt1 + (la >> sy.gs1)) * sy.gnt2 + (lb >> sy.gs2))
                                : (te * sy.gnt2 + (lb >> sy.gs2));
        any = tf[tile] != 0;
      }
    }
    if (any) out.push_back(bid);
  }
  return out;
}

template <typename T>
hipError_t launch_fft_inverse(const Plan& pl, T* u, const T* rho_for_energy, hipStream_t s) {
  const int64_t n0 = pl.n[0], n1 = pl.n[1], n2 = pl.n[2];
  const int64_t f0 = pl.nf[0], f1 = pl.nf[1], f2 = pl.nf[2];
  const bool has_x = f0 > 1;
  // the input spectrum: the spreading grid; Algorithm 2's first pass instead
  // forms its spectrum from the forward passes' output in W and from G, line
  // pairs at a time (k_fft_pair_pass), and in 2D runs in place on W (each
  // block reads all of its lines before it writes them back, and no two blocks
  // share a line)
  void* src = pl.d_G;
  void* B2 = has_x ? pl.d_F : src;  // (2D: the input grid itself)
  void* B1 = pl.d_W;
  // a real output needs only the Hermitian part of the spectrum,
  // (G(q) + conj G(-q)) / 2, at the lines 0 .. f2/2 of axis 2: the first pass
  // forms it from G and G's mirror (rows of r2), the last completes each line
  const int64_t c2 = pl.r2c ? pl.h2 : f2, r2 = pl.r2c ? pl.hs2 : f2;
  hipError_t e;
  if (has_x) {  // X: src -> B2 [n0][f1][r2]
    PassArgs<T> a = base_args<T>(pl, 0, T(1));
    a.nlines = f1 * c2;
    a.nin = (int)f0;
    a.nout = (int)n0;
    a.ic = c2;
    a.in_os = f2;
    a.in_is = 1;
    a.in_es = f1 * f2;
    a.out_os = r2;
    a.out_is = 1;
    a.out_es = f1 * r2;
    a.sym_no = (int)f1;
    a.sym_ni = (int)f2;
    a.lext = pl.d_gext;
    a.in = src;
    a.out = B2;
    if (pl.split) {
      PassArgs<T> b = split_pair_args<T>(pl, 0);
      b.out = B2;
      e = run_pair_pass<T, PAIR_FUSED>(pl, ST_INV_X, b, s);
    } else {
      e = run_pass<T, PASS_HSYM>(pl, ST_INV_X, a, s);  // r2c: Algorithm 1
    }
    if (e != hipSuccess) return e;
  }
  if (pl.split && !has_x) {  // 2D Algorithm 2: Y: W -> B1 = W [1][n1][f2], paired
    PassArgs<T> b = split_pair_args<T>(pl, 1);
    b.out = B1;
    if ((e = run_pair_pass<T, PAIR_FUSED>(pl, ST_INV_Y, b, s)) != hipSuccess) return e;
  } else {  // Y: B2 -> B1 [n0][n1][r2]; in 2D the first pass, reading G [1][f1][f2]
    PassArgs<T> a = base_args<T>(pl, 1, T(1));
    const int64_t rin = has_x ? r2 : f2;
    a.nlines = n0 * c2;
    a.nin = (int)f1;
    a.nout = (int)n1;
    a.ic = c2;
    a.in_os = f1 * rin;
    a.in_is = 1;
    a.in_es = rin;
    a.out_os = n1 * r2;
    a.out_is = 1;
    a.out_es = r2;
    a.sym_no = 1;
    a.sym_ni = (int)f2;
    a.lext = pl.d_gext;
    a.in = B2;
    a.out = B1;
    // in 2D the first pass (Algorithm 1, real output), else a plain strided pass
    e = has_x ? run_pass<T, PASS_COMPLEX>(pl, ST_INV_Y, a, s) : run_pass<T, PASS_HSYM>(pl, ST_INV_Y, a, s);
    if (e != hipSuccess) return e;
  }
  {  // Z: B1 -> u [n0][n1][n2], real part, deconvolution, energy partials
    PassArgs<T> a = base_args<T>(pl, 2, T(1));
    a.nlines = n0 * n1;
    a.nin = (int)c2;
    a.half_in = pl.r2c ? 1 : 0;
    a.nout = (int)n2;
    a.ic = 1;
    a.in_os = r2;
    a.in_is = 0;
    a.in_es = 1;
    a.out_os = n2;
    a.out_is = 0;
    a.out_es = 1;
    a.in = B1;
    a.out = u;
    a.dec0 = pl.d_deconv[0];
    a.dec1 = pl.d_deconv[1];
    a.dec2 = pl.d_deconv[2];
    a.rho = rho_for_energy;
    a.eparts = rho_for_energy ? pl.d_eparts : nullptr;
    a.split = pl.split ? 1 : 0;
    a.shift = (pl.c0 != 0.0) ? pl.d_origin : nullptr;
    if ((e = run_pass<T, PASS_INV_Z>(pl, ST_INV_Z, a, s)) != hipSuccess) return e;
  }
  return hipSuccess;
}

// Periodic complex FFT of a grid of n0 x n1 x n2 points in place (no padding,
// no crop): the GPE driver's kinetic step.  tw[a]: exp(-2 pi i t / n_a), t < n_a.
template <typename T>
hipError_t launch_fft_periodic(const Plan& pl, void* const tw[3], void* data, int sign, hipStream_t s) {
  const int64_t n0 = pl.n[0], n1 = pl.n[1], n2 = pl.n[2];
  const T sg = (T)sign;
  hipError_t e;
  auto common = [&](int axis) {
    PassArgs<T> a{};
    a.L = pl.n[axis];
    a.nin = a.nout = a.L;
    a.sign = sg;
    a.tw = (const C2<T>*)tw[axis];
    a.n1 = (int)n1;
    a.n2 = (int)n2;
    a.in = data;
    a.out = data;
    return a;
  };
  {  // axis 2, contiguous: lines [n0][n1]
    PassArgs<T> a = common(2);
    a.nlines = n0 * n1;
    a.ic = 1;
    a.in_os = a.out_os = n2;
    a.in_is = a.out_is = 0;
    a.in_es = a.out_es = 1;
    if ((e = run_pass<T, PASS_COMPLEX_Z>(pl, -1, a, s)) != hipSuccess) return e;
  }
  {  // axis 1: lines [n0][n2]
    PassArgs<T> a = common(1);
    a.nlines = n0 * n2;
    a.ic = n2;
    a.in_os = a.out_os = n1 * n2;
    a.in_is = a.out_is = 1;
    a.in_es = a.out_es = n2;
    if ((e = run_pass<T, PASS_COMPLEX>(pl, -1, a, s)) != hipSuccess) return e;
  }
  if (n0 > 1) {  // axis 0: lines [n1 n2]
    PassArgs<T> a = common(0);
    a.nlines = n1 * n2;
    a.ic = n1 * n2;
    a.in_os = a.out_os = 0;
    a.in_is = a.out_is = 1;
    a.in_es = a.out_es = n1 * n2;
    if ((e = run_pass<T, PASS_COMPLEX>(pl, -1, a, s)) != hipSuccess) return e;
  }
  return hipSuccess;
}

template hipError_t launch_fft_periodic<double>(const Plan&, void* const[3], void*, int, hipStream_t);
template hipError_t launch_fft_periodic<float>(const Plan&, void* const[3], void*, int, hipStream_t);

// The GPE kinetic step in place: forward passes along a2 (and a1 in 3D), one
// kinetic pass along the last axis (a0, or a1 when a0 is a unit axis) that
// transforms forward, multiplies and transforms back, then the inverse passes
// in reverse order.  kt: k per internal axis at offsets koff.
template <typename T>
hipError_t launch_fft_periodic_kinetic(const Plan& pl, void* const tw[3], void* data, const double* kt,
                                       const int koff[3], double h, int imaginary, double inv_n, hipStream_t s) {
  const int64_t n0 = pl.n[0], n1 = pl.n[1], n2 = pl.n[2];
  const bool has_x = n0 > 1;
  auto common = [&](int axis, T sg) {
    PassArgs<T> a{};
    a.L = pl.n[axis];
    a.nin = a.nout = a.L;
    a.sign = sg;
    a.tw = (const C2<T>*)tw[axis];
    a.n1 = (int)n1;
    a.n2 = (int)n2;
    a.in = data;
    a.out = data;
    a.kt = kt;
    for (int i = 0; i < 3; ++i) a.koff[i] = koff[i];
    a.kin_h = h;
    a.inv_n = inv_n;
    a.kin_imag = imaginary;
    a.dkb = FastDiv((uint32_t)n2);  // a line's other two axes: (line / n2, line mod n2)
    return a;
  };
  auto pass_z = [&](T sg) {  // axis 2, contiguous: lines [n0][n1]
    PassArgs<T> a = common(2, sg);
    a.nlines = n0 * n1;
    a.ic = 1;
    a.in_os = a.out_os = n2;
    a.in_is = a.out_is = 0;
    a.in_es = a.out_es = 1;
    return run_pass<T, PASS_COMPLEX_Z>(pl, -1, a, s);
  };
  auto pass_y = [&](T sg, bool kinetic) {  // axis 1: lines [n0][n2], line = i0 n2 + i2
    PassArgs<T> a = common(1, sg);
    a.nlines = n0 * n2;
    a.ic = n2;
    a.in_os = a.out_os = n1 * n2;
    a.in_is = a.out_is = 1;
    a.in_es = a.out_es = n2;
    a.kax = 1;
    return kinetic ? run_pass<T, PASS_KINETIC>(pl, -1, a, s) : run_pass<T, PASS_COMPLEX>(pl, -1, a, s);
  };
  auto pass_x_kinetic = [&]() {  // axis 0: lines [n1 n2], line = i1 n2 + i2
    PassArgs<T> a = common(0, T(-1));
    a.nlines = n1 * n2;
    a.ic = n1 * n2;
    a.in_os = a.out_os = 0;
    a.in_is = a.out_is = 1;
    a.in_es = a.out_es = n1 * n2;
    a.kax = 0;
    return run_pass<T, PASS_KINETIC>(pl, -1, a, s);
  };
  hipError_t e;
  if ((e = pass_z(T(-1))) != hipSuccess) return e;
  if (has_x) {
    if ((e = pass_y(T(-1), false)) != hipSuccess) return e;
    if ((e = pass_x_kinetic()) != hipSuccess) return e;
    if ((e = pass_y(T(1), false)) != hipSuccess) return e;
  } else {
    if ((e = pass_y(T(-1), true)) != hipSuccess) return e;
  }
  return pass_z(T(1));
}

template hipError_t launch_fft_periodic_kinetic<double>(const Plan&, void* const[3], void*, const double*,
                                                        const int[3], double, int, double, hipStream_t);
template hipError_t launch_fft_periodic_kinetic<float>(const Plan&, void* const[3], void*, const double*,
                                                       const int[3], double, int, double, hipStream_t);

// d_origin = {c0 H sum rho, c0 (H sum rho)^2} from the first forward pass's
// per-block sums (one block, fixed order).
struct OriginArgs {
  const double* parts;
  int n;
  double H, c0;
  double* out;
};

__device__ __forceinline__ void origin_body(const OriginArgs& a) {
  const double* parts = a.parts;
  const int n = a.n;
  const double H = a.H, c0 = a.c0;
  double* out = a.out;
  __shared__ double s[256];
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) acc += parts[i];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double r0 = H * s[0];
    out[0] = c0 * r0;
    out[1] = c0 * r0 * r0;
  }
}

__global__ void __launch_bounds__(256) k_origin(OriginArgs a) { origin_body(a); }
__global__ void __launch_bounds__(256) k_origin_b(const OriginArgs* __restrict__ tab, const int* __restrict__ bstart, int nm) {
  int m;
  if (batch_block(bstart, nm, blockIdx.x, m) < 0) return;
  origin_body(tab[m]);
}

hipError_t launch_origin(const Plan& pl, hipStream_t s) {
  const OriginArgs a{pl.d_mparts, fft_inverse_z_blocks(pl), pl.H, pl.c0, pl.d_origin};
  return launch<OriginArgs, k_origin, k_origin_b>(a, 1, 256, 0, s);
}

int fft_inverse_z_blocks(const Plan& pl) {
  int lb = pl.fp64 ? lines_per_block<double, PASS_INV_Z>(pl.nf[2]) : lines_per_block<float, PASS_INV_Z>(pl.nf[2]);
  if (pl.fp64 ? reg_length<double>(pl.nf[2]) : reg_length<float>(pl.nf[2]))
    lb = pl.fp64 ? reg_z_lines<double>(pl.nf[2]) : reg_z_lines<float>(pl.nf[2]);
  int64_t nl = (int64_t)pl.n[0] * pl.n[1];
  return (int)((nl + lb - 1) / lb);
}

template hipError_t launch_fft_forward<double>(const Plan&, const double*, hipStream_t);
template hipError_t launch_split_forward<double>(const Plan&, const double*, hipStream_t);
template hipError_t launch_split_forward<float>(const Plan&, const float*, hipStream_t);
template hipError_t launch_fft_forward<float>(const Plan&, const float*, hipStream_t);
template hipError_t launch_fft_inverse<double>(const Plan&, double*, const double*, hipStream_t);
template hipError_t launch_fft_inverse<float>(const Plan&, float*, const float*, hipStream_t);

}  // namespace jgb
