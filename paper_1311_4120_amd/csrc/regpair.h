// Algorithm 2's paired passes (Section 3.3) in 3D for lengths fixed at compile time,
// on the register butterflies of regfft.h.
//
// A block takes P neighbouring lines (a, b) of one row a and their mirrors
// ((A - a) mod A, (B - b) mod B), a thread per butterfly and line.  The last
// forward stage leaves Z in registers; the mirror's value Z(-q) comes through
// LDS, and the combined spectrum Y (splitsym.h) is formed in registers.  The
// last radix is the first one, so that Y is already the first inverse stage's
// input.  A line of 8 x 4 x 8 points goes through LDS five times, against nine
// round trips with the line in LDS throughout: at 128^3 in float64 the pass
// went from 160 to 136 us, of which loading, storing and the symbol take 100
// (skipping the stages).
#pragma once

#include "regfft.h"

namespace jgb {
namespace fft {

enum PairMode { PAIR_UNMIX = 0, PAIR_FUSED = 1 };

// P line pairs: 2 P line slots (own lines, then their mirrors), 128-byte rows
// each, halved while LDS or the block is too large.
template <typename T, typename SEQ>
struct PairShape : SEQ {
  using SEQ::L;
  using SEQ::TPL;
  static constexpr int V = 1, R1 = SEQ::radix(0), JB = L / SEQ::RL;
  static constexpr int pitch = L + L / R1;  // LDS rows of a line (RegShape)
  // the exchange buffer, then the symbol at every position of the own lines
  static constexpr int lds_values(int p) { return 2 * p * pitch + p * L; }
  static constexpr int pairs() {
    int p = 128 / (2 * (int)sizeof(T));
    while (lds_values(p) * (int)sizeof(T) > 65536 || 2 * p * TPL > 512) p /= 2;
    return p;
  }
  static constexpr int P = pairs();
  static constexpr int NT = 2 * P * TPL;
  static constexpr size_t lds = (size_t)lds_values(P) * sizeof(T);
  static constexpr int row = 2 * P;
  static constexpr bool wave_sync = false;
  static __device__ __forceinline__ int line_base(int l) { return l; }
  static_assert(SEQ::RL == R1 && SEQ::nb(SEQ::NS - 1) == 1,
                "the last forward stage's positions are the first inverse stage's inputs");
  static_assert(P >= 1 && NT <= 1024, "pair shape");
};

// Y(q) from Z(q), Z(-q), g = (G(q) + conj G(-q)) / 2 and hm = M / 2: hm times
// the difference Z(q) - conj Z(-q), rounded, then added to g.
#pragma clang fp contract(off)
template <typename T>
__device__ __forceinline__ C2<T> pair_combine(C2<T> zq, C2<T> zm, C2<T> g, T hm) {
  const T dx = hm * (zq.x - zm.x), dy = hm * (zq.y + zm.y);
  return C2<T>{g.x + dx, g.y + dy};
}
#pragma clang fp contract(fast)

// The same value, which the compiler must take for another: offsets derived from
// it are computed again where they are needed instead of being held in
// registers from one transform to the next.
__device__ __forceinline__ int again(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

template <typename T, int MODE, typename SEQ>
__device__ __forceinline__ void reg_pair_body(const PassArgs<T>& a) {
  typedef PairShape<T, SEQ> S;
  constexpr int L = S::L, TPL = S::TPL, P = S::P, R1 = S::R1, Q = R1 / 4, RL = SEQ::RL, JB = S::JB, row = S::row;
  constexpr int NL = SEQ::NS - 1, NBL = SEQ::nb(NL);
  extern __shared__ unsigned char smem_raw[];
  void* const smem = smem_raw;
  // The logical block.  Unmix: from the plan's list.  Fused: workgroup w runs
  // on XCD w mod 8; the logical ids are dealt out in runs, one run per XCD, so
  // that neighbouring chunks share an L2 (a chunk's mirror run is misaligned
  // by one element and shares its edge segments with the next chunk's).
  int bid;
  if constexpr (MODE == PAIR_UNMIX) {
    bid = a.blist[blockIdx.x];
  } else {
    const int nb = (int)gridDim.x, w = (int)blockIdx.x;
    const int x = w & 7, q = nb >> 3, r = nb & 7;
    bid = x * q + (x < r ? x : r) + (w >> 3);
  }
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
  const int l = threadIdx.x % (2 * P), j = threadIdx.x / (2 * P);
  const int lp = l % P;
  int bq = c * P + lp;
  const bool valid = self ? (bq <= a.B / 2) : (bq < a.B);
  if (!valid) bq = 0;
  // the slot's line (u = 0) and its mirror (u = 1)
  const int ma = ar ? a.A - ar : 0, mb = bq ? a.B - bq : 0;
  const int la[2] = {l < P ? ar : ma, l < P ? ma : ar}, lb[2] = {l < P ? bq : mb, l < P ? mb : bq};
  C2<T> v[1][SEQ::NV];
  {
    const C2<T>* p = (const C2<T>*)a.in + (int64_t)la[0] * a.B + lb[0] + (int64_t)j * a.es_in;
    const int64_t st = (int64_t)TPL * a.es_in;
#pragma unroll
    for (int r = 0; r < 2 * Q; ++r) v[0][r < Q ? 3 * Q + r : r - Q] = p[r * st];
  }
  // whether some node's tile lies on one of the block's lines (the same for the
  // whole block), and on position e of line u
  const SplitSym& sy = a.sym;
  bool tiles = false;
  {
    const int b0 = c * P, b1 = min(c * P + P - 1, a.B - 1);  // own lines
    const int m0 = max(a.B - b1, 0), m1 = a.B - max(b0, 1);    // mirrors of b0 .. b1 (0 is its own)
    const int ro = (ar >> sy.gs1) * sy.gnt2, rm = (ma >> sy.gs1) * sy.gnt2;
    for (int t = b0 >> sy.gs2; t <= b1 >> sy.gs2; ++t) tiles |= sy.tcol[ro + t] != 0;
    for (int t = m0 >> sy.gs2; t <= m1 >> sy.gs2; ++t) tiles |= sy.tcol[rm + t] != 0;
    if (b0 == 0) tiles |= sy.tcol[rm] != 0;
  }
  auto flagged = [&](int u, int e) {
    return sy.tflag[((e >> sy.gs0) * sy.gnt1 + (la[u] >> sy.gs1)) * sy.gnt2 + (lb[u] >> sy.gs2)] != 0;
  };
  auto at_g = [&](int u, int e) { return ((int64_t)e * sy.nf1 + la[u]) * sy.nf2 + lb[u]; };
  C2<T>* G = (C2<T>*)a.G;
  // the symbol hm = M / 2 at the own lines' positions, while the loads are in
  // flight (the mirror lines share it, and the work)
  T* const hms = reinterpret_cast<T*>(smem) + 2 * P * S::pitch;
  if constexpr (MODE == PAIR_FUSED) {
    const double* ks = sy.kt + sy.koff[0];
    const double* es = sy.kt + sy.eoff[0];
    // the constant parts of |k|^2, p, n.k and m.k on a line
    struct LineK {
      double kk, w, nk, mk;
    };
    auto line_k = [&](int a1, int a2) {
      const double k1 = sy.kt[sy.koff[1] + a1], k2 = sy.kt[sy.koff[2] + a2];
      return LineK{k1 * k1 + k2 * k2, sy.kt[sy.eoff[1] + a1] * sy.kt[sy.eoff[2] + a2],
                   sy.axis[1] * k1 + sy.axis[2] * k2, sy.axis2[1] * k1 + sy.axis2[2] * k2};
    };
    const LineK k = line_k(ar, bq);
    const bool dip = sy.kernel == JGB_DIPOLE_3D;
    const bool nyq = 2 * bq == a.B || 2 * ar == a.A;
#pragma unroll 1
    for (int e = j + (l < P ? 0 : TPL); e < L; e += 2 * TPL) {
      const double ke = ks[e];
      double M = split_symbol_core3(sy, ke * ke + k.kk, es[e] * k.w, sy.axis[0] * ke + k.nk, sy.axis2[0] * ke + k.mk);
      if (dip && (nyq || 2 * e == L)) {
        // on a Nyquist plane, the mean with the mirror's symbol; off them the
        // mirror's k is exactly -k (the frequencies are 2 pi q' / (2 R) with
        // q' a signed integer) and its symbol equals M bit for bit
        const LineK m = line_k(ma, mb);
        const int em = e ? L - e : 0;
        const double km = ks[em];
        M = 0.5 * (M + split_symbol_core3(sy, km * km + m.kk, es[em] * m.w, sy.axis[0] * km + m.nk,
                                          sy.axis2[0] * km + m.mk));
      }
      hms[e * P + lp] = (T)(0.5 * M);
    }
  }
  reg_butterfly<T, -1, SEQ, 0, true>(v[0]);
  reg_stages<T, S, -1, 1>(smem, v, l, again(j), a.tw);

  // the mirror's values: element i RL + r of a line is position q + r JB, q the
  // thread's butterfly i; its image is position JB - q + (RL - 1 - r) JB of the
  // mirror line, or, from butterfly 0, (RL - r) JB mod L
  const int jm = again(j);
  C2<T> zm[NBL * RL];
  {
    constexpr int st = in_step<SEQ, NL>();
    T* const own = reinterpret_cast<T*>(smem) + l;
    const T* const mir = reinterpret_cast<const T*>(smem) + (l < P ? l + P : l - P);
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NBL; ++i) {
        T* const w = own + row * in_row<SEQ, NL>(SEQ::template bf<NL>(jm, i));
#pragma unroll
        for (int r = 0; r < RL; ++r) w[r * st * row] = part ? v[0][i * RL + r].y : v[0][i * RL + r].x;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NBL; ++i) {
        const int q = SEQ::template bf<NL>(jm, i);
        const int last = q ? in_row<SEQ, NL>(JB - q) + (RL - 1) * st : RL * st;
        const T* const w = mir + row * last;
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          const T x = r == 0 ? mir[row * (q ? last : 0)] : w[-r * st * row];
          if (part) zm[i * RL + r].y = x;
          else zm[i * RL + r].x = x;
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NBL; ++i) {
    const int q = SEQ::template bf<NL>(jm, i);
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const int e = q + r * JB;
      if constexpr (MODE == PAIR_UNMIX) {
        // A = (Z(q) + conj Z(-q)) / 2 where the interpolation reads it
        const C2<T> z = v[0][i * RL + r], m = zm[i * RL + r];
        if (valid && tiles && flagged(0, e)) G[at_g(0, e)] = C2<T>{T(0.5) * (z.x + m.x), T(0.5) * (z.y - m.y)};
      } else {
        // I2's share of the spectrum, where the block's lines have any
        C2<T> g{T(0), T(0)};
        if (tiles) {
          const int em = e ? L - e : 0;
          C2<T> gq{T(0), T(0)}, gm{T(0), T(0)};
          if (flagged(0, e)) gq = G[at_g(0, e)];
          if (flagged(1, em)) gm = G[at_g(1, em)];
          g = C2<T>{T(0.5) * (gq.x + gm.x), T(0.5) * (gq.y - gm.y)};
        }
        // (the symbol is even: a mirror line's position e is the own line's L - e)
        const int eo = l < P ? e : e ? L - e : 0;
        v[0][i * RL + r] = pair_combine(v[0][i * RL + r], zm[i * RL + r], g, hms[eo * P + lp]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (MODE == PAIR_UNMIX) return;
  reg_butterfly<T, 1, SEQ, 0, false>(v[0]);
  __syncthreads();
  reg_stages<T, S, 1, 1>(smem, v, l, again(j), a.tw);
  // the cropped outputs
  if (!valid) return;
  const int js = again(j);
  C2<T>* out = (C2<T>*)a.out + (int64_t)la[0] * a.B + lb[0];
#pragma unroll
  for (int i = 0; i < NBL; ++i) {
    const int q = SEQ::template bf<NL>(js, i);
    if (!SEQ::template own<NL>(js, i)) continue;
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      if (RL % 4 == 0 && r >= RL / 4 && r < 3 * RL / 4) continue;
      const int p = q + r * JB;
      if (RL % 4 == 0 || 4 * p < L || 4 * p >= 3 * L)
        out[(int64_t)(4 * p < L ? p + L / 4 : p - 3 * L / 4) * a.es_out] = v[0][i * RL + r];
    }
  }
}

template <typename T, int MODE, int R1, int R2, int R3, int R4>
__global__ void __launch_bounds__((PairShape<T, RegSeq<R1, R2, R3, R4>>::NT), 4) k_reg_pair(PassArgs<T> a) {
  reg_pair_body<T, MODE, RegSeq<R1, R2, R3, R4>>(a);
}

// The lengths with a kernel of their own (float64): a last radix that is the
// first one, eight line pairs (128-byte rows) within the LDS of a block, and no
// more than eight values a thread.  Of the lengths that meet this, 32 (4 x 2 x 4)
// and 64 (8 x 8) are left to the any-length kernel although theirs would be the
// faster (whole evaluations: 16^3 72 us, 69 with it; 32^3 78 and 76; 32 x 128 x
// 128 145 and 122).  Beyond, the any-length kernel is the faster
// one (320 points, four pairs: 350 against 381 us at 160^3; 288 points as
// 12 x 2 x 12: 305 against 375 at 144^3); in float32 it is by what the
// transforms' own radices leave of the gain (16 x 4 x 5 points: 204 against
// 354 us at 160 x 144 x 160).
#define JGB_PAIR_LENGTHS(X) \
  X(4, 3, 4, 1) X(4, 5, 4, 1) X(4, 6, 4, 1) X(8, 2, 8, 1) X(4, 10, 4, 1) X(8, 3, 8, 1) X(8, 4, 8, 1)

// line pairs per block of the paired passes (0: no kernel of its own)
template <typename T>
constexpr int reg_pair_lines(int L) {
#define JGB_PAIR_P(R1, R2, R3, R4) \
  if (L == R1 * R2 * R3 * R4) return PairShape<T, RegSeq<R1, R2, R3, R4>>::P;
  if constexpr (sizeof(T) == 8) {
    JGB_PAIR_LENGTHS(JGB_PAIR_P)
  }
#undef JGB_PAIR_P
  return 0;
}

// Launch a paired pass of a length with reg_pair_lines<T>(a.L) > 0
// (instantiated per mode and precision in regpair_*.hip).
template <typename T, int MODE>
hipError_t launch_reg_pair(const PassArgs<T>& a, unsigned blocks, hipStream_t s);
#define JGB_PAIR_DECLARE(TYPE, MODE_) \
  template <>                         \
  hipError_t launch_reg_pair<TYPE, MODE_>(const PassArgs<TYPE>&, unsigned, hipStream_t);
JGB_PAIR_DECLARE(double, PAIR_UNMIX)
JGB_PAIR_DECLARE(double, PAIR_FUSED)
#undef JGB_PAIR_DECLARE

template <typename T, int MODE, int R1, int R2, int R3, int R4>
hipError_t launch_pair_shape(const PassArgs<T>& a, unsigned blocks, hipStream_t s) {
  typedef PairShape<T, RegSeq<R1, R2, R3, R4>> S;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL((k_reg_pair<T, MODE, R1, R2, R3, R4>), dim3(blocks), dim3(S::NT), S::lds, s, a);
  return hipGetLastError();
}

#define JGB_PAIR_CASE(R1, R2, R3, R4) \
  case R1 * R2 * R3 * R4: return launch_pair_shape<T, MODE, R1, R2, R3, R4>(a, blocks, s);
#define JGB_PAIR_INSTANTIATE(TYPE, MODE_)                                                          \
  template <typename T, int MODE>                                                                  \
  static hipError_t pair_switch(const PassArgs<T>& a, unsigned blocks, hipStream_t s) {            \
    switch (a.L) {                                                                                 \
      JGB_PAIR_LENGTHS(JGB_PAIR_CASE)                                                              \
      default: return hipErrorInvalidValue;                                                        \
    }                                                                                              \
  }                                                                                                \
  template <>                                                                                      \
  hipError_t launch_reg_pair<TYPE, MODE_>(const PassArgs<TYPE>& a, unsigned blocks, hipStream_t s) { \
    return pair_switch<TYPE, MODE_>(a, blocks, s);                                                 \
  }

}  // namespace fft
}  // namespace jgb
