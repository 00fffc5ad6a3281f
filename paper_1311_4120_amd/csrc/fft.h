// Types shared by the FFT passes: the complex element, the pass kinds and the
// argument block of a pass (fft.hip launches the passes; regfft.h holds the
// kernels whose line length is fixed at compile time).
#pragma once

#include "splitsym.h"

namespace jgb {
namespace fft {

template <typename T>
struct alignas(2 * sizeof(T)) C2 {  // one 16-byte (fp64) or 8-byte (fp32) access
  T x, y;
};

// The arithmetic of the passes, with every rounding written out: which product
// of a sum goes into a fused multiply-add is the compiler's choice otherwise,
// and may differ from one kernel that holds a butterfly to the next -- a batch
// runs the passes from other kernels than a plan, with the same bits.
#pragma clang fp contract(off)

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

template <typename T>
__device__ __forceinline__ C2<T> cadd(C2<T> a, C2<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ C2<T> csub(C2<T> a, C2<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ C2<T> cmul(C2<T> a, C2<T> b) {
  return {fma_(a.x, b.x, -(a.y * b.y)), fma_(a.y, b.x, a.x * b.y)};
}
// a + r b (r real)
template <typename T>
__device__ __forceinline__ C2<T> cfma(T r, C2<T> b, C2<T> a) { return {fma_(r, b.x, a.x), fma_(r, b.y, a.y)}; }
// a + i r b
template <typename T>
__device__ __forceinline__ C2<T> cfma_i(T r, C2<T> b, C2<T> a) { return {fma_(-r, b.y, a.x), fma_(r, b.x, a.y)}; }

#pragma clang fp contract(fast)

// FWD_Z / INV_Z: the oversampled grid's first and last passes (real in or out,
// deconvolution factors); COMPLEX: a complex pass along a strided axis;
// COMPLEX_Z: a complex pass along the contiguous axis (the periodic FFT).
// KINETIC: the GPE driver's kinetic step along one strided axis: the forward
// transform, the multiplier exp(-i h |k|^2 / 2) / N (imaginary time:
// exp(-h |k|^2 / 2) / N), and the inverse transform, in LDS.
// HSYM: the inverse's first pass on a real output, a strided complex pass
// whose input is the Hermitian part of the spreading grid.
enum PassKind { PASS_FWD_Z = 0, PASS_COMPLEX = 1, PASS_INV_Z = 2, PASS_COMPLEX_Z = 3, PASS_KINETIC = 4, PASS_HSYM = 5 };
template <int KIND>
constexpr bool has_factors() { return KIND == PASS_FWD_Z || KIND == PASS_INV_Z; }

template <typename T>
struct PassArgs {
  int L;            // line length
  int64_t nlines;
  int LB;           // lines per block
  int nin;          // inputs per line (L, or N when the input is zero-padded)
  int nout;         // outputs per line (L, or N when the output is cropped)
  int64_t ic;       // lines per outer group; line l = (outer, inner) = (l / ic, l % ic)
  int64_t ngroups;  // strided register passes: groups of neighbouring lines, dgrp.d per outer group
  FastDiv dgrp;
  int64_t in_os, in_is, in_es;
  int64_t out_os, out_is, out_es;
  T sign;
  int nrad;
  int rad[12];
  int tws[12];      // twiddle stride of each radix stage, L / (Ns R)
  FastDiv dNs[12];  // Ns of each radix stage (product of the earlier radices)
  FastDiv dLB, dnin, dnout, dic, dn1;
  const C2<T>* tw;  // exp(-2 pi i t / L), t < L
  const void* in;
  void* out;
  // forward Z: deconvolution and cell volume; inverse Z: deconvolution and energy
  const double* dec0;
  const double* dec1;
  const double* dec2;
  double scale;
  int n1, n2;         // physical grid sizes of axes 1 and 2 (Z passes)
  const T* rho;       // inverse Z: density for the energy partial (nullable)
  double* eparts;     // inverse Z: per-block partials of sum rho u
  int split;          // Z passes of Algorithm 2: forward imag = rho H; inverse u += imag
  double* mparts;     // forward Z: per-block sums of rho (the node at k = 0), nullable
  const double* shift;  // inverse Z: constant added to u (the node at k = 0), nullable
  // Hermitian half along the last axis (real input, Algorithm 1): the forward
  // Z pass stores only outputs 0 .. nout - 1 = L/2 (half_out); the inverse Z
  // pass loads those nin = L/2 + 1 values and completes the line by
  // v(L - p) = conj v(p) (half_in); the inverse's first pass (PASS_HSYM)
  // averages each element with the conjugate of its mirror,
  // v(q) = (g(q) + conj g(-q)) / 2, the mirror of line (outer, inner) and
  // element e being (-outer mod sym_no, -inner mod sym_ni, -e mod L)
  int half_out, half_in, sym_no, sym_ni;
  // PASS_HSYM: per input line (outer sym_ni + inner), the circular range
  // {first, span} of elements the spreading can have written; the pass takes
  // the other elements as zero without loading them
  const int2* lext;
  // PASS_COMPLEX (optional): per output line, the circular range {first,
  // span} of elements that are read later; the pass stores no others
  const int2* oext;
  // the paired passes of Algorithm 2 (k_fft_pair_pass): lines are
  // (a, b) of an A x B set, element stride es_in / es_out; P lines and their
  // mirrors per block; nb1 blocks for the rows 0 < a < A/2 (cb per row), then cs
  // per row for the rows that are their own mirror (a = 0 and a = A/2)
  int P, A, B, nb1, cb, cs, dim3;
  FastDiv dP;
  const int* blist;   // the unmix pass's logical blocks
  int64_t es_in, es_out;
  const void* G;
  SplitSym sym;
  // the kinetic pass: k per internal axis in kt (offsets koff), the pass's
  // axis kax (0, or 1 when axis 0 is a unit axis), a line's two other axes
  // (a, b) = (line / nb, line mod nb) with the divisor in dkb
  const double* kt;
  int koff[3];
  int kax;
  FastDiv dkb;
  double kin_h, inv_n;
  int kin_imag;
};

// ---------------------------------------------- passes of any length
//
// The kernel for lengths without one of their own (regfft.h) and for the
// periodic passes: the line length, its radices and every extent are run-time
// values, and the line stays in LDS from load to store.

#pragma clang fp contract(off)

// In-register DFTs of small radix, y_k = sum_n x_n exp(s 2 pi i n k / R), s = +-1.
template <typename T>
__device__ inline void dft2(C2<T>* v, T) {
  C2<T> a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

template <typename T>
__device__ inline void dft4(C2<T>* v, T s) {
  C2<T> a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
  C2<T> c = cadd(v[1], v[3]), d = csub(v[1], v[3]);
  v[0] = cadd(a, c);
  v[2] = csub(a, c);
  v[1] = cfma_i(s, d, b);
  v[3] = cfma_i(-s, d, b);
}

template <typename T>
__device__ inline void dft3(C2<T>* v, T s) {
  const T h = s * T(0.86602540378443864676);  // sin(2 pi / 3)
  C2<T> t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
  C2<T> m = cfma(T(-0.5), t, v[0]);
  v[0] = cadd(v[0], t);
  v[1] = cfma_i(h, d, m);
  v[2] = cfma_i(-h, d, m);
}

template <typename T>
__device__ inline void dft5(C2<T>* v, T s) {
  const T c1 = T(0.30901699437494742410), c2 = T(-0.80901699437494742410);
  const T s1 = T(0.95105651629515357212), s2 = T(0.58778525229247312917);
  C2<T> a1 = cadd(v[1], v[4]), b1 = csub(v[1], v[4]);
  C2<T> a2 = cadd(v[2], v[3]), b2 = csub(v[2], v[3]);
  C2<T> x0 = v[0];
  C2<T> r1 = cfma(c2, a2, cfma(c1, a1, x0));
  C2<T> r2 = cfma(c1, a2, cfma(c2, a1, x0));
  C2<T> q1 = {fma_(s2, b2.x, s1 * b1.x), fma_(s2, b2.y, s1 * b1.y)};
  C2<T> q2 = {fma_(s2, b1.x, -(s1 * b2.x)), fma_(s2, b1.y, -(s1 * b2.y))};
  v[0] = cadd(x0, cadd(a1, a2));
  v[1] = cfma_i(s, q1, r1);
  v[4] = cfma_i(-s, q1, r1);
  v[2] = cfma_i(s, q2, r2);
  v[3] = cfma_i(-s, q2, r2);
}

template <typename T>
__device__ inline void dft8(C2<T>* v, T s) {
  const T r = T(0.70710678118654752440);
  C2<T> e[4] = {v[0], v[2], v[4], v[6]};
  C2<T> o[4] = {v[1], v[3], v[5], v[7]};
  dft4(e, s);
  dft4(o, s);
  // twiddles w^k, w = exp(s 2 pi i / 8)
  const C2<T> t1 = cfma_i(s, o[1], o[1]), t3 = cfma_i(s, o[3], C2<T>{-o[3].x, -o[3].y});
  v[0] = cadd(e[0], o[0]);
  v[4] = csub(e[0], o[0]);
  v[1] = cfma(r, t1, e[1]);
  v[5] = cfma(-r, t1, e[1]);
  v[2] = cfma_i(s, o[2], e[2]);
  v[6] = cfma_i(-s, o[2], e[2]);
  v[3] = cfma(r, t3, e[3]);
  v[7] = cfma(-r, t3, e[3]);
}

#pragma clang fp contract(fast)

// Radix 16 as 4 x 4: with n = 4 n1 + n2 and k = k1 + 4 k2,
// y_k = sum_n2 w16^(n2 k1) [sum_n1 x_(4 n1 + n2) w4^(n1 k1)] w4^(n2 k2).
// Only the float32 paired passes use it, which no batch runs: its products'
// roundings are the compiler's.
template <typename T>
__device__ inline void dft16(C2<T>* v, T s) {
  const T c1 = T(0.92387953251128675613), s1 = T(0.38268343236508977173);  // cos, sin of pi/8
  const T r = T(0.70710678118654752440);
  C2<T> a[4][4];  // a[n2][k1]
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    C2<T> t[4] = {v[n2], v[4 + n2], v[8 + n2], v[12 + n2]};
    dft4(t, s);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) a[n2][k1] = t[k1];
  }
  // twiddles w16^m = (cos(2 pi m / 16), s sin(2 pi m / 16)) for m = n2 k1
  auto mul = [](C2<T> a, C2<T> b) { return C2<T>{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; };
  const C2<T> w1{c1, s * s1}, w2{r, s * r}, w3{s1, s * c1}, w6{-r, s * r}, w9{-c1, -s * s1};
  a[1][1] = mul(a[1][1], w1);
  a[1][2] = mul(a[1][2], w2);
  a[1][3] = mul(a[1][3], w3);
  a[2][1] = mul(a[2][1], w2);
  a[2][2] = C2<T>{-s * a[2][2].y, s * a[2][2].x};
  a[2][3] = mul(a[2][3], w6);
  a[3][1] = mul(a[3][1], w3);
  a[3][2] = mul(a[3][2], w6);
  a[3][3] = mul(a[3][3], w9);
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    C2<T> t[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
    dft4(t, s);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = t[k2];
  }
}

template <typename T, int R>
__device__ inline void dft(C2<T>* v, T s) {
  if constexpr (R == 2) dft2(v, s);
  if constexpr (R == 3) dft3(v, s);
  if constexpr (R == 4) dft4(v, s);
  if constexpr (R == 5) dft5(v, s);
  if constexpr (R == 8) dft8(v, s);
  if constexpr (R == 16) dft16(v, s);
}

// Byte offset of a pass block's twiddle table in LDS: after LB padded lines
// and, for the Z passes, LB + L deconvolution factors; 16-byte aligned.
template <typename T>
__host__ __device__ inline size_t pass_twiddle_offset(int LB, int L, bool factors) {
  size_t off = (size_t)LB * (L + 1) * sizeof(C2<T>);
  if (factors) off += sizeof(double) * (LB + L);
  return (off + 15) & ~(size_t)15;
}

// Position on the fine grid of physical index i of a line of N: (i - N/2) mod L.
__device__ inline int fine_pos(int i, int N, int L) {
  int m = i - N / 2;
  return m < 0 ? m + L : m;
}

template <typename T, int R, int MAXV, int NT>
__device__ inline void stage(C2<T>* lds, int ldl, int L, int LB, int Ns, const FastDiv& dLB, const FastDiv& dNs,
                             int stride_tw, const C2<T>* tw, T sign) {
  const int nbf = L / R;           // butterflies per line
  const int nb = LB * nbf;         // butterflies in the block
  constexpr int MAXB = (MAXV + R - 1) / R;   // butterflies per thread at most
  C2<T> v[MAXB][R];
  int dst[MAXB];
#pragma unroll
  for (int i = 0; i < MAXB; ++i) {
    int b = threadIdx.x + i * NT;
    if (b < nb) {
      const int j = (int)dLB.div(b);
      const int l = b - j * LB;
      const int jq = (int)dNs.div(j);
      const int k = j - jq * Ns;
      C2<T>* row = lds + l * ldl;
#pragma unroll
      for (int r = 0; r < R; ++r) v[i][r] = row[j + r * nbf];
      if (Ns > 1) {
        // r k stride_tw < R Ns L / (Ns R) = L: no reduction needed
#pragma unroll
        for (int r = 1; r < R; ++r) {
          C2<T> w = tw[r * k * stride_tw];
          w.y *= -sign;  // table holds exp(-2 pi i t/L); sign +1 needs the conjugate
          v[i][r] = cmul(v[i][r], w);
        }
      }
      dft<T, R>(v[i], sign);
      dst[i] = l * ldl + jq * Ns * R + k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MAXB; ++i) {
    int b = threadIdx.x + i * NT;
    if (b < nb) {
#pragma unroll
      for (int r = 0; r < R; ++r) lds[dst[i] + r * Ns] = v[i][r];
    }
  }
  __syncthreads();
}

// One block transforms LB lines.  Global traffic is issued in bulk: every
// thread computes clamped (always valid) addresses for all of its up to MAXV
// elements and issues the loads back to back, and only then writes LDS, so
// that the loads are in flight together; the store phase reads LDS into
// registers first and then stores.  The pass kind fixes the access order:
// the complex passes run along a strided axis with consecutive threads on
// consecutive lines, the Z passes along the contiguous axis.
template <typename T, int KIND, int MAXV, int NT>
__device__ __forceinline__ void fft_pass_body(const PassArgs<T>& a, const int blk) {
  constexpr bool LINES_FASTEST = (KIND == PASS_COMPLEX || KIND == PASS_KINETIC || KIND == PASS_HSYM);
  extern __shared__ unsigned char smem_raw[];
  C2<T>* lds = reinterpret_cast<C2<T>*>(smem_raw);
  const int L = a.L;
  const int ldl = L + 1;
  const int LB = a.LB;
  const int line0 = blk * LB;
  // Z passes: deconvolution factors of the block's lines and of the elements,
  // staged after the lines
  double* fline = reinterpret_cast<double*>(smem_raw + (size_t)LB * ldl * sizeof(C2<T>));
  double* felem = fline + LB;
  // the strided passes stage the line's twiddles after the lines (16-byte
  // aligned) and their radix stages read them from LDS; the Z passes, whose
  // blocks are smaller and more numerous per CU, read them from global memory
  constexpr bool TW_LDS = LINES_FASTEST;
  C2<T>* const twl = reinterpret_cast<C2<T>*>(smem_raw + pass_twiddle_offset<T>(LB, L, has_factors<KIND>()));
  const C2<T>* const ltw = TW_LDS ? twl : a.tw;

  // staged while the element loads are in flight (below)
  auto stage_factors = [&]() {
    const int ne = (KIND == PASS_FWD_Z) ? a.nin : a.nout;
    for (int t = threadIdx.x; t < LB + ne; t += NT) {
      if (t < LB) {
        int line = line0 + t;
        if (line >= a.nlines) line = 0;
        const int i0 = (int)a.dn1.div(line), i1 = line - i0 * a.n1;
        fline[t] = (KIND == PASS_FWD_Z ? a.scale : 1.0) * a.dec0[i0] * a.dec1[i1];
      } else {
        felem[t - LB] = a.dec2[t - LB];
      }
    }
  };

  // the output reach of the thread's line (its elements all lie on one line
  // here), read now and used by the stores
  int2 ox{0, L - 1};
  if constexpr (KIND == PASS_COMPLEX) {
    if (a.oext) {
      const int line = line0 + (int)(threadIdx.x - a.dLB.div(threadIdx.x) * LB);
      ox = a.oext[line < a.nlines ? line : 0];
    }
  }

  // zero the padding region of every line when the input is padded
  if (a.nin < L && !a.half_in) {
    const int N = a.nin;
    const int nz = L - N;  // fine positions [N - N/2, L - N/2) stay zero
    for (int idx = threadIdx.x; idx < LB * nz; idx += NT) {
      const int e = (int)a.dLB.div(idx), l = idx - e * LB;
      lds[l * ldl + (N - N / 2) + e] = C2<T>{T(0), T(0)};
    }
  }

  double macc = 0.0;  // forward Z: the block's sum of rho
  // load: every load is issued before any loaded value is used, so that they
  // are in flight together; masked elements load from a valid index instead
  // of branching around the load, and their values are dropped afterwards
  {
    const int total_in = LB * a.nin;
    constexpr bool HSYM = KIND == PASS_HSYM;
    C2<T> buf[MAXV];
    T rbuf[KIND == PASS_FWD_Z ? MAXV : 1];
    C2<T> mir[HSYM ? MAXV : 1];
    int dst[MAXV];
    int le[MAXV];  // Z pass: line (high bits) and element (low 16 bits)
    unsigned keep = 0, keepm = 0;  // bit i: element i's value (its mirror's) is used
    // HSYM: LB divides NT, so all of a thread's elements lie on one line, whose
    // mirror line and reaches are read once, before the element loads
    int hl = 0, hlo = 0, hli = 0, hmo = 0, hmi = 0;
    bool hlok = false;
    int2 xp{0, -1}, xm{0, -1};
    if constexpr (HSYM) {
      hl = threadIdx.x - (int)a.dLB.div(threadIdx.x) * LB;
      const int line = line0 + hl;
      hlok = line < a.nlines;
      const int ln = hlok ? line : 0;
      hlo = (int)a.dic.div(ln);
      hli = ln - hlo * (int)a.ic;
      hmo = hlo ? a.sym_no - hlo : 0;
      hmi = hli ? a.sym_ni - hli : 0;
      xp = a.lext[(int64_t)hlo * a.sym_ni + hli];
      xm = a.lext[(int64_t)hmo * a.sym_ni + hmi];
    }
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      // slots past the block's inputs (padded passes load N of L) issue nothing;
      // the test is uniform across the block.  HSYM takes no such branch:
      // past one, the compiler no longer knows that the line's reaches have
      // arrived and waits for every load in flight before using them; its
      // empty slots are masked lanes instead
      if (!HSYM && i * NT >= total_in) {
        dst[i] = -1;
        le[i] = 0;
        continue;
      }
      const int idx0 = threadIdx.x + i * NT;
      const bool ok = idx0 < total_in;
      const int idx = ok ? idx0 : 0;
      int l, e;
      if constexpr (LINES_FASTEST) {
        e = (int)a.dLB.div(idx);
        l = idx - e * LB;
      } else {
        l = (int)a.dnin.div(idx);
        e = idx - l * a.nin;
      }
      if constexpr (HSYM) {
        // elements beyond their line's reach are zero: not fetched
        const bool lok = ok && hlok;
        const int me = e ? L - e : 0;
        int dp = e - xp.x, dm = me - xm.x;
        dp += dp < 0 ? L : 0;
        dm += dm < 0 ? L : 0;
        const bool in_p = lok && dp <= xp.y, in_m = lok && dm <= xm.y;
        const int64_t base = (int64_t)hlo * a.in_os + (int64_t)hli * a.in_is + (int64_t)e * a.in_es;
        const int64_t mbase = (int64_t)hmo * a.in_os + (int64_t)hmi * a.in_is + (int64_t)me * a.in_es;
        buf[i] = ((const C2<T>*)a.in)[in_p ? base : 0];
        mir[i] = ((const C2<T>*)a.in)[in_m ? mbase : 0];
        keep |= (unsigned)in_p << i;
        keepm |= (unsigned)in_m << i;
        dst[i] = ok ? hl * ldl + e : -1;
        le[i] = 0;
        continue;
      }
      const int line = line0 + l;
      const bool lok = ok && line < a.nlines;
      const int ln = lok ? line : 0;
      const int lo = (int)a.dic.div(ln);
      const int li = ln - lo * (int)a.ic;
      const int64_t base = (int64_t)lo * a.in_os + (int64_t)li * a.in_is + (int64_t)e * a.in_es;
      if constexpr (KIND == PASS_FWD_Z) {
        rbuf[i] = ((const T*)a.in)[base];
        keep |= (unsigned)lok << i;
      } else {
        buf[i] = ((const C2<T>*)a.in)[base];
        keep |= (unsigned)lok << i;
      }
      const int pos = (a.nin < L && !a.half_in) ? fine_pos(e, a.nin, L) : e;
      dst[i] = ok ? l * ldl + pos : -1;
      le[i] = (l << 16) | e;
    }
    // the twiddles or the deconvolution factors, copied while the element
    // loads are in flight
    if constexpr (TW_LDS)
      for (int t = threadIdx.x; t < L; t += NT) twl[t] = a.tw[t];
    if constexpr (has_factors<KIND>()) stage_factors();
    if constexpr (KIND == PASS_FWD_Z) __syncthreads();  // factors staged: the LDS writes below apply them
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      if (dst[i] >= 0) {
        const bool use = (keep >> i) & 1u;
        C2<T> v;
        if constexpr (KIND == PASS_FWD_Z) {
          // deconvolution and cell volume, applied in float64
          const T r = use ? rbuf[i] : T(0);
          const double d = fline[le[i] >> 16] * felem[le[i] & 0xffff];
          macc += (double)r;
          v.y = a.split ? (T)((double)r * a.scale) : T(0);
          v.x = (T)((double)r * d);
        } else if constexpr (HSYM) {
          const bool usem = (keepm >> i) & 1u;
          const T px = use ? buf[i].x : T(0), py = use ? buf[i].y : T(0);
          const T mx = usem ? mir[i].x : T(0), my = usem ? mir[i].y : T(0);
          v = C2<T>{T(0.5) * (px + mx), T(0.5) * (py - my)};
        } else {
          v = use ? buf[i] : C2<T>{T(0), T(0)};
        }
        lds[dst[i]] = v;
      }
    }
  }
  __syncthreads();
  if (a.half_in) {
    // the rest of each line from the Hermitian symmetry of its spectrum
    const int nfill = L - a.nin;
    for (int idx = threadIdx.x; idx < LB * nfill; idx += NT) {
      const int e = (int)a.dLB.div(idx), l = idx - e * LB;
      const int p = a.nin + e;
      const C2<T> v = lds[l * ldl + (L - p)];
      lds[l * ldl + p] = C2<T>{v.x, -v.y};
    }
    __syncthreads();
  }

  // FFT stages
  auto transform = [&](T sign) {
    int Ns = 1;
    for (int st = 0; st < a.nrad; ++st) {
      const int R = a.rad[st];
      const FastDiv& dNs = a.dNs[st];
      const int tws = a.tws[st];
      switch (R) {
        case 8: stage<T, 8, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, ltw, sign); break;
        case 5: stage<T, 5, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, ltw, sign); break;
        case 4: stage<T, 4, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, ltw, sign); break;
        case 3: stage<T, 3, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, ltw, sign); break;
        default: stage<T, 2, MAXV, NT>(lds, ldl, L, LB, Ns, a.dLB, dNs, tws, ltw, sign); break;
      }
      Ns *= R;
    }
  };
  if constexpr (KIND == PASS_KINETIC) {
    transform(T(-1));
    // the multiplier at every element, |k|^2 summed in axis order
    for (int idx = threadIdx.x; idx < LB * L; idx += NT) {
      const int e = (int)a.dLB.div(idx), l = idx - e * LB;
      const int line = line0 + l;
      if (line >= a.nlines) continue;
      const int ia = (int)a.dkb.div(line), ib = line - ia * (int)a.dkb.d;
      const double ke = a.kt[a.koff[a.kax] + e];
      const double kb = a.kt[a.koff[2] + ib];
      const double kx = a.kax == 0 ? ke : a.kt[a.koff[0] + ia];
      const double ky = a.kax == 0 ? a.kt[a.koff[1] + ia] : ke;
      const double ex = 0.5 * a.kin_h * (kx * kx + ky * ky + kb * kb);
      double fr, fi;
      if (a.kin_imag) {
        fr = exp(-ex) * a.inv_n;
        fi = 0.0;
      } else {
        sincos(-ex, &fi, &fr);
        fr *= a.inv_n;
        fi *= a.inv_n;
      }
      C2<T>* pv = lds + l * ldl + e;
      const C2<T> p = *pv;
      const double re = fr * p.x - fi * p.y, im = fr * p.y + fi * p.x;
      *pv = C2<T>{(T)re, (T)im};
    }
    __syncthreads();
    transform(T(1));
  } else {
    transform(a.sign);
  }

  // store: LDS reads first, then the global stores
  double eacc = 0.0;
  double ushift = 0.0;
  if constexpr (KIND == PASS_INV_Z) {
    if (a.shift) ushift = *a.shift;
  }
  {
    const int total_out = LB * a.nout;
    C2<T> buf[MAXV];
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      if (i * NT >= total_out) {  // cropped passes store N of L (uniform test)
        buf[i] = C2<T>{T(0), T(0)};
        continue;
      }
      const int idx0 = threadIdx.x + i * NT;
      const int idx = idx0 < total_out ? idx0 : 0;
      int l, e;
      if constexpr (LINES_FASTEST) {
        e = (int)a.dLB.div(idx);
        l = idx - e * LB;
      } else {
        l = (int)a.dnout.div(idx);
        e = idx - l * a.nout;
      }
      const int pos = (a.nout < L && !a.half_out) ? fine_pos(e, a.nout, L) : e;
      buf[i] = lds[l * ldl + pos];
    }
    T rho_v[KIND == PASS_INV_Z ? MAXV : 1];
    if constexpr (KIND == PASS_INV_Z) {
      // density values for the energy partials, loaded together
#pragma unroll
      for (int i = 0; i < MAXV; ++i) {
        if (i * NT >= total_out) {
          rho_v[i] = T(0);
          continue;
        }
        const int idx0 = threadIdx.x + i * NT;
        const int idx = idx0 < total_out ? idx0 : 0;
        const int l = (int)a.dnout.div(idx), e = idx - l * a.nout;
        int line = line0 + l;
        if (line >= a.nlines) line = 0;
        rho_v[i] = a.rho ? a.rho[(int64_t)line * a.out_os + e] : T(0);
      }
    }
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      const int idx = threadIdx.x + i * NT;
      if (idx >= total_out) continue;
      int l, e;
      if constexpr (LINES_FASTEST) {
        e = (int)a.dLB.div(idx);
        l = idx - e * LB;
      } else {
        l = (int)a.dnout.div(idx);
        e = idx - l * a.nout;
      }
      const int line = line0 + l;
      if (line >= a.nlines) continue;
      const int lo = (int)a.dic.div(line);
      const int64_t base = (int64_t)lo * a.out_os + (int64_t)(line - lo * (int)a.ic) * a.out_is + (int64_t)e * a.out_es;
      if constexpr (KIND == PASS_COMPLEX) {
        int dp = e - ox.x;
        dp += dp < 0 ? L : 0;
        if (dp > ox.y) continue;  // never read: not stored
      }
      if constexpr (KIND == PASS_INV_Z) {
        double u = __builtin_fma((double)buf[i].x, fline[l] * felem[e], ushift);
        if (a.split) u += (double)buf[i].y;
        ((T*)a.out)[base] = (T)u;
        eacc = __builtin_fma((double)rho_v[i], u, eacc);
      } else {
        ((C2<T>*)a.out)[base] = buf[i];
      }
    }
  }

  if constexpr (KIND == PASS_FWD_Z) {
    if (a.mparts) {
      // deterministic block sum of rho: wave shuffle, then waves in order
      for (int off = 32; off > 0; off >>= 1) macc += __shfl_xor(macc, off, 64);
      __shared__ double msum[NT / 64];
      __syncthreads();
      if ((threadIdx.x & 63) == 0) msum[threadIdx.x >> 6] = macc;
      __syncthreads();
      if (threadIdx.x == 0) {
        double s = 0.0;
        for (int i = 0; i < NT / 64; ++i) s += msum[i];
        a.mparts[blk] = s;
      }
    }
  }
  if constexpr (KIND == PASS_INV_Z) {
    if (a.eparts) {
      // deterministic block sum: wave shuffle, then waves in order
      for (int off = 32; off > 0; off >>= 1) eacc += __shfl_xor(eacc, off, 64);
      __shared__ double wsum[NT / 64];
      __syncthreads();
      if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = eacc;
      __syncthreads();
      if (threadIdx.x == 0) {
        double s = 0.0;
        for (int i = 0; i < NT / 64; ++i) s += wsum[i];
        a.eparts[blk] = s;
      }
    }
  }
}

// Block shapes (threads x complex elements per thread; the staged elements
// cap / L give the lines per block).  Measured on the 256-point lines of the
// 128^3 grids: the strided passes keep every row of a block at 128 contiguous
// bytes (8 fp64 or 16 fp32 lines) with four or more blocks per CU, the Z
// passes stage 2048 elements per block, and the paired pass of Algorithm 2
// runs 256 threads (4 fp64 or 8 fp32 line pairs).  Every cap holds a whole
// line of the largest grid (nf = 1024), the paired pass's a line and its
// mirror.
constexpr int PASS_PAIR = 9;
template <typename T, int KIND = PASS_PAIR>
constexpr int pass_threads() {
  if (KIND == PASS_COMPLEX || KIND == PASS_KINETIC || KIND == PASS_HSYM) return sizeof(T) == 8 ? 256 : 512;
  if (KIND == PASS_FWD_Z || KIND == PASS_INV_Z) return 256;
  if (KIND == PASS_PAIR) return 256;
  return 512;
}
template <typename T, int KIND = PASS_PAIR>
constexpr int pass_elems() {
  if (KIND == PASS_COMPLEX || KIND == PASS_KINETIC || KIND == PASS_HSYM || KIND == PASS_FWD_Z || KIND == PASS_INV_Z)
    return 8;
  return sizeof(T) == 8 ? 8 : 16;
}
template <typename T, int KIND>
constexpr int pass_cap() { return pass_threads<T, KIND>() * pass_elems<T, KIND>(); }

}  // namespace fft
}  // namespace jgb
