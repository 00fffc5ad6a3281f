// FFT passes whose line length L = R1 R2 R3 R4 is fixed at compile time.
//
// A thread holds the R1 inputs of one butterfly of the first stage in
// registers, loaded straight from the grid, and the outputs of its butterflies
// of the last stage, stored straight to it; the line goes through LDS only
// between stages.  Against a kernel that stages the line in LDS before the
// first stage and after the last, an L = 256 pass makes one (float64, 16 x 16)
// or two (float32, 8 x 8 x 4) LDS round trips instead of four and waits at as
// many fewer barriers: what bounds these passes is that chain of dependent
// steps per block, not HBM.  With N = L / 2 nonzero inputs the middle half of
// a first butterfly's inputs is zero and not loaded.
//
// Stockham order: a stage of radix R with Ns the product of the earlier radices
// takes butterfly q from elements q + r L / R, r < R, multiplies by
// w_(Ns R)^(r (q mod Ns)), transforms, and puts output r at
// (q / Ns) Ns R + q mod Ns + r Ns.
//
// float64 uses large radices (fewer exchanges), float32 the radix sequence and
// butterflies of the any-length kernel (fft.h): the digits of a mixed plan's
// results are those of that kernel (u has the same bits as where it runs every
// length on 288 3D and 192 planar grids with sides of 8 to 512 points).  Both
// write every rounding out, so that a kernel's batched form gives its bits too.
#pragma once

#include "fft.h"

namespace jgb {
namespace fft {

// cos of k half degrees, k = 0 .. 180
constexpr double kCos720[181] = {
    1.0, 0.9999619230641713, 0.9998476951563913, 0.9996573249755573, 0.9993908270190958, 0.9990482215818578,
    0.9986295347545738, 0.9981347984218669, 0.9975640502598242, 0.996917333733128, 0.9961946980917455, 0.9953961983671789,
    0.9945218953682733, 0.9935718556765875, 0.992546151641322, 0.9914448613738104, 0.9902680687415704, 0.9890158633619168,
    0.9876883405951378, 0.9862856015372314, 0.984807753012208, 0.9832549075639546, 0.981627183447664, 0.9799247046208296,
    0.9781476007338057, 0.9762960071199334, 0.9743700647852352, 0.9723699203976766, 0.9702957262759965, 0.9681476403781077,
    0.9659258262890683, 0.963630453208623, 0.9612616959383189, 0.958819734868193, 0.9563047559630354, 0.9537169507482269,
    0.9510565162951535, 0.9483236552061993, 0.9455185755993168, 0.9426414910921784, 0.9396926207859084, 0.9366721892483976,
    0.9335804264972017, 0.9304175679820246, 0.9271838545667874, 0.9238795325112867, 0.9205048534524404, 0.917060074385124,
    0.9135454576426009, 0.9099612708765432, 0.9063077870366499, 0.9025852843498606, 0.898794046299167, 0.8949343616020251,
    0.8910065241883679, 0.8870108331782217, 0.882947592858927, 0.8788171126619654, 0.8746197071393959, 0.8703556959398997,
    0.8660254037844386, 0.8616291604415257, 0.8571673007021123, 0.8526401643540922, 0.848048096156426, 0.8433914458128857,
    0.838670567945424, 0.8338858220671682, 0.8290375725550417, 0.8241261886220157, 0.8191520442889918, 0.8141155183563192,
    0.8090169943749475, 0.8038568606172173, 0.7986355100472928, 0.7933533402912352, 0.7880107536067219, 0.7826081568524139,
    0.7771459614569709, 0.77162458338772, 0.766044443118978, 0.7604059656000309, 0.754709580222772, 0.7489557207890022,
    0.7431448254773942, 0.7372773368101241, 0.7313537016191705, 0.7253743710122876, 0.7193398003386512, 0.7132504491541816,
    0.7071067811865476, 0.7009092642998509, 0.6946583704589973, 0.688354575693754, 0.6819983600624985, 0.6755902076156602,
    0.6691306063588582, 0.6626200482157375, 0.6560590289905073, 0.6494480483301837, 0.6427876096865394, 0.636078220277764,
    0.6293203910498375, 0.6225146366376195, 0.6156614753256583, 0.6087614290087207, 0.6018150231520483, 0.5948227867513413,
    0.5877852522924731, 0.5807029557109398, 0.573576436351046, 0.5664062369248328, 0.5591929034707468, 0.5519369853120581,
    0.5446390350150271, 0.5372996083468239, 0.5299192642332049, 0.5224985647159489, 0.5150380749100542, 0.5075383629607042,
    0.5, 0.4924235601034671, 0.484809620246337, 0.4771587602596084, 0.46947156278589075, 0.4617486132350339,
    0.4539904997395468, 0.44619781310980877, 0.4383711467890774, 0.43051109680829514, 0.42261826174069944, 0.414693242656239,
    0.4067366430758002, 0.3987490689252462, 0.39073112848927377, 0.3826834323650898, 0.374606593415912, 0.3665012267242973,
    0.35836794954530027, 0.3502073812594675, 0.3420201433256687, 0.3338068592337709, 0.32556815445715664, 0.31730465640509214,
    0.30901699437494745, 0.3007057995042731, 0.2923717047227367, 0.2840153447039226, 0.27563735581699916, 0.2672383760782569,
    0.25881904510252074, 0.25038000405444144, 0.24192189559966773, 0.23344536385590542, 0.224951054343865, 0.21643961393810288,
    0.20791169081775934, 0.1993679344171972, 0.1908089953765448, 0.18223552549214744, 0.17364817766693036, 0.16504760586067765,
    0.15643446504023087, 0.14780941112961063, 0.13917310096006544, 0.1305261922200516, 0.12186934340514748, 0.11320321376790672,
    0.10452846326765347, 0.095845752520224, 0.08715574274765818, 0.07845909572784494, 0.0697564737441253, 0.06104853953485687,
    0.052335956242943835, 0.043619387365336, 0.03489949670250097, 0.026176948307873153, 0.01745240643728351, 0.008726535498373935,
    0.0,
};
constexpr double cos720(int t) {
  t %= 720;
  if (t < 0) t += 720;
  if (t > 360) t = 720 - t;
  return t <= 180 ? kCos720[t] : -kCos720[360 - t];
}
// exp(2 pi i K / N) for N dividing 720
template <int K, int N>
struct Root {
  static_assert(720 % N == 0, "roots of unity come from a table of 720");
  static constexpr int t = ((K * (720 / N)) % 720 + 720) % 720;
  static constexpr double c = cos720(t), s = cos720(t + 540);
};

#pragma clang fp contract(off)  // every rounding written out (fft.h)

// a exp(SG 2 pi i K / N)
template <int SG, int K, int N, typename T>
__device__ __forceinline__ C2<T> rot(C2<T> a) {
  constexpr int t = Root<SG * K, N>::t;
  if constexpr (t == 0) return a;
  else if constexpr (t == 180) return C2<T>{-a.y, a.x};
  else if constexpr (t == 360) return C2<T>{-a.x, -a.y};
  else if constexpr (t == 540) return C2<T>{a.y, -a.x};
  else {
    constexpr T c = (T)Root<SG * K, N>::c, s = (T)Root<SG * K, N>::s;
    return C2<T>{fma_(a.x, c, -(a.y * s)), fma_(a.x, s, a.y * c)};
  }
}

// In-register DFTs in natural order, y_k = sum_n x_n exp(SG 2 pi i n k / N).
template <int SG, int N, typename T>
__device__ __forceinline__ void rdft(C2<T>* v) {
  if constexpr (N == 2) {
    const C2<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (N == 3) {
    constexpr T h = (T)(SG * Root<1, 3>::s);
    const C2<T> t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const C2<T> m = cfma(T(-0.5), t, v[0]);
    v[0] = cadd(v[0], t);
    v[1] = cfma_i(h, d, m);
    v[2] = cfma_i(-h, d, m);
  } else if constexpr (N == 4) {
    const C2<T> a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
    const C2<T> c = cadd(v[1], v[3]), d = rot<SG, 1, 4>(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[2] = csub(a, c);
    v[1] = cadd(b, d);
    v[3] = csub(b, d);
  } else if constexpr (N == 5) {
    constexpr T c1 = (T)Root<1, 5>::c, c2 = (T)Root<2, 5>::c;
    constexpr T s1 = (T)(SG * Root<1, 5>::s), s2 = (T)(SG * Root<2, 5>::s);
    const C2<T> a1 = cadd(v[1], v[4]), b1 = csub(v[1], v[4]);
    const C2<T> a2 = cadd(v[2], v[3]), b2 = csub(v[2], v[3]);
    const C2<T> x0 = v[0];
    const C2<T> r1 = cfma(c2, a2, cfma(c1, a1, x0));
    const C2<T> r2 = cfma(c1, a2, cfma(c2, a1, x0));
    const C2<T> q1 = {-fma_(s1, b1.y, s2 * b2.y), fma_(s1, b1.x, s2 * b2.x)};
    const C2<T> q2 = {-fma_(s2, b1.y, -(s1 * b2.y)), fma_(s2, b1.x, -(s1 * b2.x))};
    v[0] = cadd(x0, cadd(a1, a2));
    v[1] = cadd(r1, q1);
    v[4] = csub(r1, q1);
    v[2] = cadd(r2, q2);
    v[3] = csub(r2, q2);
  } else {
    static_assert(N % 2 == 0, "radix");
    // even and odd elements, N / 2 points each
    constexpr int H = N / 2;
    C2<T> e[H], o[H];
#pragma unroll
    for (int n = 0; n < H; ++n) {
      e[n] = v[2 * n];
      o[n] = v[2 * n + 1];
    }
    rdft<SG, H>(e);
    rdft<SG, H>(o);
    static_assert(H <= 5, "radix");
    if constexpr (H > 0) { const C2<T> q = rot<SG, 0, N>(o[0]); v[0] = cadd(e[0], q); v[H] = csub(e[0], q); }
    if constexpr (H > 1) { const C2<T> q = rot<SG, 1, N>(o[1]); v[1] = cadd(e[1], q); v[H + 1] = csub(e[1], q); }
    if constexpr (H > 2) { const C2<T> q = rot<SG, 2, N>(o[2]); v[2] = cadd(e[2], q); v[H + 2] = csub(e[2], q); }
    if constexpr (H > 3) { const C2<T> q = rot<SG, 3, N>(o[3]); v[3] = cadd(e[3], q); v[H + 3] = csub(e[3], q); }
    if constexpr (H > 4) { const C2<T> q = rot<SG, 4, N>(o[4]); v[4] = cadd(e[4], q); v[H + 4] = csub(e[4], q); }
  }
}

// v[K] *= exp(SG 2 pi i J K / N) over K = 0 .. Q - 1
template <int SG, int J, int Q, int N, int K = 0, typename T>
__device__ __forceinline__ void rot_row(C2<T>* v) {
  if constexpr (K < Q) {
    v[K] = rot<SG, J * K, N>(v[K]);
    rot_row<SG, J, Q, N, K + 1>(v);
  }
}

// First-stage DFT of 4 Q points: the four-point columns of elements n2,
// Q + n2, 2 Q + n2, 3 Q + n2 first, then Q-point rows, y_(k1 + 4 k2).  PAD:
// elements Q .. 3 Q - 1 are zero (never read).
template <int SG, int Q, bool PAD, typename T>
__device__ __forceinline__ void dft_first(C2<T>* v) {
  C2<T> a[4][Q];  // a[k1][n2]
#pragma unroll
  for (int n2 = 0; n2 < Q; ++n2) {
    if constexpr (PAD) {
      const C2<T> x = v[n2], z = v[3 * Q + n2], q = rot<SG, 3, 4>(z);
      a[0][n2] = cadd(x, z);
      a[1][n2] = cadd(x, q);
      a[2][n2] = csub(x, z);
      a[3][n2] = csub(x, q);
    } else {
      C2<T> t[4] = {v[n2], v[Q + n2], v[2 * Q + n2], v[3 * Q + n2]};
      rdft<SG, 4>(t);
#pragma unroll
      for (int k1 = 0; k1 < 4; ++k1) a[k1][n2] = t[k1];
    }
  }
  rot_row<SG, 1, Q, 4 * Q>(a[1]);
  rot_row<SG, 2, Q, 4 * Q>(a[2]);
  rot_row<SG, 3, Q, 4 * Q>(a[3]);
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    if constexpr (Q > 1) rdft<SG, Q>(a[k1]);
#pragma unroll
    for (int k2 = 0; k2 < Q; ++k2) v[k1 + 4 * k2] = a[k1][k2];
  }
}

// Last-stage DFT of 4 Q points: Q-point DFTs over the elements n1 + 4 n2
// first, then the four-point ones, y_(Q k1 + k2): the caller uses all outputs
// or only those with k1 = 0 and k1 = 3 (the compiler drops the others' work).
template <int SG, int Q, typename T>
__device__ __forceinline__ void dft_last(C2<T>* v) {
  C2<T> a[4][Q];  // a[n1][k2]
#pragma unroll
  for (int n1 = 0; n1 < 4; ++n1) {
#pragma unroll
    for (int n2 = 0; n2 < Q; ++n2) a[n1][n2] = v[n1 + 4 * n2];
    if constexpr (Q > 1) rdft<SG, Q>(a[n1]);
  }
  rot_row<SG, 1, Q, 4 * Q>(a[1]);
  rot_row<SG, 2, Q, 4 * Q>(a[2]);
  rot_row<SG, 3, Q, 4 * Q>(a[3]);
#pragma unroll
  for (int k2 = 0; k2 < Q; ++k2) {
    C2<T> t[4] = {a[0][k2], a[1][k2], a[2][k2], a[3][k2]};
    rdft<SG, 4>(t);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) v[Q * k1 + k2] = t[k1];
  }
}

// float32: the any-length kernel's butterflies (fft.h) for a direction known at
// compile time.
// a + SG i d, a - SG i d
template <int SG>
__device__ __forceinline__ C2<float> xadd_i(C2<float> a, C2<float> d) {
  return SG > 0 ? C2<float>{a.x - d.y, a.y + d.x} : C2<float>{a.x + d.y, a.y - d.x};
}
template <int SG>
__device__ __forceinline__ void xdft4(C2<float>* v) {
  const C2<float> a{v[0].x + v[2].x, v[0].y + v[2].y}, b{v[0].x - v[2].x, v[0].y - v[2].y};
  const C2<float> c{v[1].x + v[3].x, v[1].y + v[3].y}, d{v[1].x - v[3].x, v[1].y - v[3].y};
  v[0] = C2<float>{a.x + c.x, a.y + c.y};
  v[2] = C2<float>{a.x - c.x, a.y - c.y};
  v[1] = xadd_i<SG>(b, d);
  v[3] = xadd_i<-SG>(b, d);
}
// xdft4 with v[1] = v[2] = 0
template <int SG>
__device__ __forceinline__ void xdft4_pad(C2<float>* v) {
  const C2<float> a = v[0], c = v[3];
  v[0] = C2<float>{a.x + c.x, a.y + c.y};
  v[2] = C2<float>{a.x - c.x, a.y - c.y};
  v[1] = xadd_i<-SG>(a, c);
  v[3] = xadd_i<SG>(a, c);
}
template <int SG, bool PAD>
__device__ __forceinline__ void xdft8(C2<float>* v) {
  constexpr float r = (float)Root<1, 8>::c, s = (float)SG;
  C2<float> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
  if constexpr (PAD) {
    xdft4_pad<SG>(e);
    xdft4_pad<SG>(o);
  } else {
    xdft4<SG>(e);
    xdft4<SG>(o);
  }
  const C2<float> t1{o[1].x - s * o[1].y, o[1].y + s * o[1].x}, t3{-o[3].x - s * o[3].y, -o[3].y + s * o[3].x};
  v[0] = C2<float>{e[0].x + o[0].x, e[0].y + o[0].y};
  v[4] = C2<float>{e[0].x - o[0].x, e[0].y - o[0].y};
  v[1] = C2<float>{__builtin_fmaf(r, t1.x, e[1].x), __builtin_fmaf(r, t1.y, e[1].y)};
  v[5] = C2<float>{__builtin_fmaf(-r, t1.x, e[1].x), __builtin_fmaf(-r, t1.y, e[1].y)};
  v[2] = xadd_i<SG>(e[2], o[2]);
  v[6] = xadd_i<-SG>(e[2], o[2]);
  v[3] = C2<float>{__builtin_fmaf(r, t3.x, e[3].x), __builtin_fmaf(r, t3.y, e[3].y)};
  v[7] = C2<float>{__builtin_fmaf(-r, t3.x, e[3].x), __builtin_fmaf(-r, t3.y, e[3].y)};
}
template <int SG>
__device__ __forceinline__ void xdft3(C2<float>* v) {
  constexpr float h = (float)(SG * Root<1, 3>::s);
  const C2<float> t{v[1].x + v[2].x, v[1].y + v[2].y}, d{v[1].x - v[2].x, v[1].y - v[2].y};
  const C2<float> m{__builtin_fmaf(-0.5f, t.x, v[0].x), __builtin_fmaf(-0.5f, t.y, v[0].y)};
  v[0] = C2<float>{v[0].x + t.x, v[0].y + t.y};
  v[1] = C2<float>{__builtin_fmaf(-h, d.y, m.x), __builtin_fmaf(h, d.x, m.y)};
  v[2] = C2<float>{__builtin_fmaf(h, d.y, m.x), __builtin_fmaf(-h, d.x, m.y)};
}
template <int SG>
__device__ __forceinline__ void xdft5(C2<float>* v) {
  constexpr float c1 = (float)Root<1, 5>::c, c2 = (float)Root<2, 5>::c;
  constexpr float s1 = (float)Root<1, 5>::s, s2 = (float)Root<2, 5>::s;
  const C2<float> a1{v[1].x + v[4].x, v[1].y + v[4].y}, b1{v[1].x - v[4].x, v[1].y - v[4].y};
  const C2<float> a2{v[2].x + v[3].x, v[2].y + v[3].y}, b2{v[2].x - v[3].x, v[2].y - v[3].y};
  const C2<float> x0 = v[0], a{a1.x + a2.x, a1.y + a2.y};
  const C2<float> r1{__builtin_fmaf(c2, a2.x, __builtin_fmaf(c1, a1.x, x0.x)),
                     __builtin_fmaf(c2, a2.y, __builtin_fmaf(c1, a1.y, x0.y))};
  const C2<float> r2{__builtin_fmaf(c1, a2.x, __builtin_fmaf(c2, a1.x, x0.x)),
                     __builtin_fmaf(c1, a2.y, __builtin_fmaf(c2, a1.y, x0.y))};
  const C2<float> q1{__builtin_fmaf(s2, b2.x, s1 * b1.x), __builtin_fmaf(s2, b2.y, s1 * b1.y)};
  const C2<float> q2{__builtin_fmaf(s2, b1.x, -(s1 * b2.x)), __builtin_fmaf(s2, b1.y, -(s1 * b2.y))};
  v[0] = C2<float>{x0.x + a.x, x0.y + a.y};
  v[1] = xadd_i<SG>(r1, q1);
  v[4] = xadd_i<-SG>(r1, q1);
  v[2] = xadd_i<SG>(r2, q2);
  v[3] = xadd_i<-SG>(r2, q2);
}
template <int SG, bool PAD>
__device__ __forceinline__ void xdft16(C2<float>* v) {
  constexpr float c1 = (float)Root<1, 16>::c, s1 = (float)Root<1, 16>::s, r = (float)Root<1, 8>::c, s = (float)SG;
  C2<float> a[4][4];  // a[n2][k1]
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    C2<float> t[4] = {v[n2], v[4 + n2], v[8 + n2], v[12 + n2]};
    if constexpr (PAD) xdft4_pad<SG>(t);
    else xdft4<SG>(t);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) a[n2][k1] = t[k1];
  }
  const C2<float> w1{c1, s * s1}, w2{r, s * r}, w3{s1, s * c1}, w6{-r, s * r}, w9{-c1, -s * s1};
  a[1][1] = cmul(a[1][1], w1);
  a[1][2] = cmul(a[1][2], w2);
  a[1][3] = cmul(a[1][3], w3);
  a[2][1] = cmul(a[2][1], w2);
  a[2][2] = C2<float>{-s * a[2][2].y, s * a[2][2].x};
  a[2][3] = cmul(a[2][3], w6);
  a[3][1] = cmul(a[3][1], w3);
  a[3][2] = cmul(a[3][2], w6);
  a[3][3] = cmul(a[3][3], w9);
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    C2<float> t[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
    xdft4<SG>(t);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = t[k2];
  }
}
template <int SG, int R, bool PAD>
__device__ __forceinline__ void xdft(C2<float>* v) {
  static_assert(!PAD || R == 4 || R == 8 || R == 16, "padded radix");
  if constexpr (R == 2) {
    const C2<float> a = v[0], b = v[1];
    v[0] = C2<float>{a.x + b.x, a.y + b.y};
    v[1] = C2<float>{a.x - b.x, a.y - b.y};
  }
  if constexpr (R == 3) xdft3<SG>(v);
  if constexpr (R == 4 && PAD) xdft4_pad<SG>(v);
  if constexpr (R == 4 && !PAD) xdft4<SG>(v);
  if constexpr (R == 5) xdft5<SG>(v);
  if constexpr (R == 8) xdft8<SG, PAD>(v);
  if constexpr (R == 16) xdft16<SG, PAD>(v);
}

#pragma clang fp contract(fast)

// ------------------------------------------------------------------ geometry

// What a pass does beside the transform.  RP_FWD_Z, RP_INV_Z: the first and
// last pass along the contiguous axis (real input or output, deconvolution);
// RP_FWD: zero-padded input, whole output, strided; RP_INV: whole input,
// cropped output, strided; RP_HSYM: RP_INV on the Hermitian part of the input.
enum RegPass { RP_FWD_Z = 0, RP_INV_Z = 1, RP_FWD = 2, RP_INV = 3, RP_HSYM = 4 };

template <int KIND>
constexpr bool reg_strided() { return KIND != RP_FWD_Z && KIND != RP_INV_Z; }

// The stages of a line and the threads that run them: a thread for each
// butterfly of the first stage.  A stage of radix R has L / R butterflies,
// nb of them per thread: thread j takes j, j + TPL, ... (a butterfly past the
// last is the last one again: the same values computed and written twice).
template <int R1, int R2, int R3, int R4>
struct RegSeq {
  static constexpr int L = R1 * R2 * R3 * R4;
  static constexpr int NS = R4 > 1 ? 4 : R3 > 1 ? 3 : 2;  // stages
  static constexpr int TPL = L / R1;
  static constexpr int radix(int s) { return s == 0 ? R1 : s == 1 ? R2 : s == 2 ? R3 : R4; }
  static constexpr int ns(int s) { return s == 0 ? 1 : s == 1 ? R1 : s == 2 ? R1 * R2 : R1 * R2 * R3; }
  static constexpr int RL = radix(NS - 1);
  static constexpr int nb(int s) { return (L / radix(s) + TPL - 1) / TPL; }
  static constexpr int held(int s) { return s < NS ? nb(s) * radix(s) : 0; }
  static constexpr int cmax(int a, int b) { return a > b ? a : b; }
  static constexpr int NV = cmax(cmax(held(0), held(1)), cmax(held(2), held(3)));  // values a thread holds at most
  static_assert(R1 % 4 == 0, "the padding is the middle half of a first butterfly's inputs");
  // butterfly i of thread j in stage s
  template <int s>
  static __device__ __forceinline__ int bf(int j, int i) {
    constexpr int n = L / radix(s);
    return n % TPL == 0 ? j + i * TPL : min(j + i * TPL, n - 1);
  }
  // whether it is the thread's own (not a repeated one)
  template <int s>
  static __device__ __forceinline__ bool own(int j, int i) {
    constexpr int n = L / radix(s);
    return n % TPL == 0 || j + i * TPL < n;
  }
};

// Strided passes: V LB lines side by side in memory, a thread holding V
// neighbouring lines (two in float32: 16-byte accesses in both precisions) and
// consecutive threads on consecutive ones: rows of 256 bytes, halved until the
// block fits 64 KB of LDS and 512 threads (128-byte rows were 10-20% slower on
// 256-point float64 lines: 27.0 -> 23.9 us for the second forward pass of a
// 128^3 grid).  Contiguous passes: consecutive threads along the line, as many
// lines as fit 256 threads.
template <typename T, bool STR, typename SEQ>
struct RegShape : SEQ {
  using SEQ::L;
  using SEQ::TPL;
  static constexpr int V = STR && sizeof(T) == 4 ? 2 : 1;
  // the exchange moves the real and then the imaginary parts: half the LDS, so
  // twice the blocks per CU (45.3 against 47.2 us for the first inverse pass of
  // a 128^3 grid in float64)
  static constexpr int es = V * (int)sizeof(T);  // bytes of an LDS element
  static constexpr int R1 = SEQ::radix(0);
  // LDS rows of a line: one pad per R1 elements, so that the elements that
  // consecutive butterflies write together (R1 apart) fall on different banks,
  // at a constant stride per output
  static constexpr int pitch = L + L / R1;
  static constexpr int str_lines() {
    int lb = 256 / (2 * V * (int)sizeof(T));
    while (lb * pitch * es > 65536 || lb * TPL > 512) lb /= 2;
    return lb;
  }
  static constexpr int LB = STR ? str_lines() : (TPL >= 256 ? 1 : 256 / TPL);  // line groups of V
  static constexpr int NT = LB * TPL;
  static constexpr bool wave_sync = !STR && 64 % TPL == 0;  // a line never leaves its wavefront
  static constexpr size_t lds = (size_t)LB * pitch * es < NT * sizeof(double) ? NT * sizeof(double) : (size_t)LB * pitch * es;
  static_assert(NT <= 1024 && lds <= 65536, "pass shape");
  // LDS elements between two rows, and the first of line group l
  static constexpr int row = STR ? LB : 1;
  static __device__ __forceinline__ int line_base(int l) { return STR ? l : l * pitch; }
};

// V neighbouring complex values, one access.
template <typename T, int V>
struct alignas(2 * V * sizeof(T)) CV {
  C2<T> u[V];
};

template <bool WAVE>
__device__ __forceinline__ void reg_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// V values of one part (real or imaginary), one LDS access.
template <typename T, int V>
struct alignas(V * sizeof(T)) PV {
  T u[V];
};

// The first row of butterfly q's outputs of stage s, and the rows between two
// of them; likewise of its inputs.
template <typename SEQ, int s>
__device__ __forceinline__ int out_row(int q) {
  constexpr int R1 = SEQ::radix(0), R = SEQ::radix(s), NS = SEQ::ns(s);
  if constexpr (s == 0) return q * (R1 + 1);
  const int k = q % NS, e = (q - k) * R + k;
  return e + e / R1;
}
template <typename SEQ, int s>
constexpr int out_step() { return s == 0 ? 1 : SEQ::ns(s) + SEQ::ns(s) / SEQ::radix(0); }
template <typename SEQ, int s>
__device__ __forceinline__ int in_row(int q) { return q + q / SEQ::radix(0); }
template <typename SEQ, int s>
constexpr int in_step() {
  constexpr int n = SEQ::L / SEQ::radix(s);
  static_assert(n % SEQ::radix(0) == 0, "a later stage's inputs are a multiple of R1 apart");
  return n + n / SEQ::radix(0);
}

// Exchange through LDS from stage s - 1's outputs in v to stage s's inputs: the
// real parts, then the imaginary ones.
template <typename T, typename S, int s>
__device__ __forceinline__ void reg_exchange(void* smem, C2<T> (&v)[S::V][S::NV], int l, int j) {
  constexpr int V = S::V, P = S::radix(s - 1), NW = S::nb(s - 1), R = S::radix(s), NR = S::nb(s), row = S::row;
  constexpr int os = out_step<S, s - 1>(), is = in_step<S, s>();
  typedef PV<T, V> E;
  E* const m = reinterpret_cast<E*>(smem) + S::line_base(l);
  T re[V][NR * R];
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    if (part || s > 1) reg_sync<S::wave_sync>();  // what was there has been read
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      E* const w = m + row * out_row<S, s - 1>(S::template bf<s - 1>(j, i));
#pragma unroll
      for (int r = 0; r < P; ++r) {
        E x;
#pragma unroll
        for (int u = 0; u < V; ++u) x.u[u] = part ? v[u][i * P + r].y : v[u][i * P + r].x;
        w[r * os * row] = x;
      }
    }
    reg_sync<S::wave_sync>();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const E* const q = m + row * in_row<S, s>(S::template bf<s>(j, i));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const E x = q[r * is * row];
#pragma unroll
        for (int u = 0; u < V; ++u) {
          if (part == 0) re[u][i * R + r] = x.u[u];
          else v[u][i * R + r] = C2<T>{re[u][i * R + r], x.u[u]};
        }
      }
    }
  }
}

// One butterfly of stage s.  PAD: the middle half of its inputs is zero.
template <typename T, int SG, typename SEQ, int s, bool PAD>
__device__ __forceinline__ void reg_butterfly(C2<T>* v) {
  constexpr int R = SEQ::radix(s);
  if constexpr (sizeof(T) == 4) {
    xdft<SG, R, PAD>(v);
  } else if constexpr (s == 0) {
    dft_first<SG, R / 4, PAD>(v);
  } else if constexpr (s == SEQ::NS - 1 && R % 4 == 0) {
    dft_last<SG, R / 4>(v);
  } else {
    rdft<SG, R>(v);
  }
}

// Table entry t by a 32-bit byte offset from the table's base (the base stays in
// scalar registers).
template <typename T>
__device__ __forceinline__ C2<T> table_at(const C2<T>* __restrict__ tw, int t) {
  return *reinterpret_cast<const C2<T>*>(reinterpret_cast<const char*>(tw) + (uint32_t)t * (uint32_t)sizeof(C2<T>));
}

// Stages s .. NS - 1, from stage s - 1's outputs in v to the last stage's
// (butterfly i's output r at v[i RL + r]).
template <typename T, typename S, int SG, int s>
__device__ __forceinline__ void reg_stages(void* smem, C2<T> (&v)[S::V][S::NV], int l, int j,
                                           const C2<T>* __restrict__ tw) {
  if constexpr (s < S::NS) {
    constexpr int L = S::L, R = S::radix(s), NS = S::ns(s);
    constexpr int NB = S::nb(s);
    reg_exchange<T, S, s>(smem, v, l, j);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int k = S::template bf<s>(j, i) % NS;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        // w_(Ns R)^(r k); the table holds exp(-2 pi i t / L)
        C2<T> w = table_at(tw, r * k * (L / (NS * R)));
        if constexpr (SG > 0) w.y = -w.y;
#pragma unroll
        for (int u = 0; u < S::V; ++u) {
          v[u][i * R + r] = cmul(v[u][i * R + r], w);
        }
      }
#pragma unroll
      for (int u = 0; u < S::V; ++u) reg_butterfly<T, SG, S, s, false>(v[u] + i * R);
    }
    reg_stages<T, S, SG, s + 1>(smem, v, l, j, tw);
  }
}

// Deterministic sum of v over the block into *out, through the pass's LDS:
// thread t of the first wavefront adds the values of threads t, t + 64, ... in
// order, then a fixed tree.
template <int NT>
__device__ __forceinline__ void reg_block_sum(void* smem, double v, double* out) {
  static_assert(NT >= 64, "block");
  double* s = reinterpret_cast<double*>(smem);
  __syncthreads();
  s[threadIdx.x] = v;
  __syncthreads();
  if (threadIdx.x < 64) {
    double a = 0.0;
    for (int t = threadIdx.x; t < NT; t += 64) a += s[t];
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
    if (threadIdx.x == 0) *out = a;
  }
}

template <typename T, int KIND, typename SEQ>
__device__ __forceinline__ void reg_pass_body(const PassArgs<T>& a, const int blk) {
  constexpr bool STR = reg_strided<KIND>();
  typedef RegShape<T, STR, SEQ> S;
  constexpr int L = S::L, TPL = S::TPL, LB = S::LB, V = S::V, R1 = SEQ::radix(0), RL = SEQ::RL, NBL = SEQ::nb(SEQ::NS - 1);
  constexpr int SG = (KIND == RP_FWD_Z || KIND == RP_FWD) ? -1 : 1;
  constexpr int Q = R1 / 4;
  extern __shared__ unsigned char smem_raw[];
  void* const smem = smem_raw;
  const int tid = threadIdx.x;
  const int l = STR ? tid % LB : tid / TPL, j = STR ? tid / LB : tid % TPL;
  // contiguous passes: the line; strided ones: group li .. li + V - 1 of the
  // lines of outer index lo (an odd count of lines leaves the last group one
  // past them, into the row's padding or, reading, the next column)
  const int line = blk * LB + l;
  const bool lok = line < (int)(STR ? a.ngroups : a.nlines);
  const int ln = lok ? line : 0;
  const int lo = STR ? (int)a.dgrp.div(ln) : 0, li = STR ? V * (ln - lo * (int)a.dgrp.d) : 0;
  C2<T> v[V][SEQ::NV];

  if constexpr (KIND == RP_FWD_Z) {
    // rho H / (phi^0 phi^1 phi^2), in float64; input element n sits at fine
    // position n - N/2 mod L, so butterfly inputs Q .. 3 Q - 1 are padding
    const T* in = (const T*)a.in + (int64_t)ln * a.in_os + j;
    T x[2 * Q];
    double d2[2 * Q];
#pragma unroll
    for (int r = 0; r < 2 * Q; ++r) x[r] = in[r * TPL];
#pragma unroll
    for (int r = 0; r < 2 * Q; ++r) d2[r] = a.dec2[j + r * TPL];
    const int i0 = (int)a.dn1.div(ln), i1 = ln - i0 * a.n1;
    const double f = a.scale * a.dec0[i0] * a.dec1[i1];
    double macc = 0.0;
#pragma unroll
    for (int r = 0; r < 2 * Q; ++r) {
      const T xv = lok ? x[r] : T(0);
      const double d = f * d2[r];
      macc += (double)xv;
      C2<T> c;
      c.x = (T)((double)xv * d);
      c.y = a.split ? (T)((double)xv * a.scale) : T(0);
      v[0][r < Q ? 3 * Q + r : r - Q] = c;
    }
    if (a.mparts) {
      reg_block_sum<S::NT>(smem, macc, a.mparts + blk);
      __syncthreads();
    }
    reg_butterfly<T, SG, SEQ, 0, true>(v[0]);
  } else if constexpr (KIND == RP_INV_Z) {
    const C2<T>* in = (const C2<T>*)a.in + (int64_t)ln * a.in_os;
    // the Hermitian half holds positions 0 .. L/2: v(p) = conj v(L - p) beyond
#pragma unroll
    for (int r = 0; r < R1; ++r) {
      const int p = j + r * TPL;
      const bool mir = a.half_in && 2 * p > L;
      const C2<T> x = in[mir ? L - p : p];
      v[0][r] = C2<T>{x.x, mir ? -x.y : x.y};
    }
    reg_butterfly<T, SG, SEQ, 0, false>(v[0]);
  } else {
    typedef CV<T, V> E;
    const C2<T>* in = (const C2<T>*)a.in;
    const int64_t bp = (int64_t)lo * a.in_os + (int64_t)li * a.in_is;
    if constexpr (KIND == RP_FWD || KIND == RP_INV) {
      constexpr bool PAD = KIND == RP_FWD;
      const C2<T>* p = in + bp + (int64_t)j * a.in_es;
      const int64_t st = (int64_t)TPL * a.in_es;
#pragma unroll
      for (int r = 0; r < (PAD ? 2 * Q : R1); ++r) {
        const E x = *reinterpret_cast<const E*>(p + r * st);
#pragma unroll
        for (int u = 0; u < V; ++u) v[u][!PAD ? r : r < Q ? 3 * Q + r : r - Q] = x.u[u];
      }
#pragma unroll
      for (int u = 0; u < V; ++u) reg_butterfly<T, SG, SEQ, 0, PAD>(v[u]);
    } else {
      // the Hermitian part (g(q) + conj g(-q)) / 2; elements beyond the
      // lines' reaches are zero and not fetched (they load element 0 instead)
      const int mo = lo ? a.sym_no - lo : 0;
      int2 xp[V], xm[V];
      int64_t bm[V];
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const int mi = li + u ? a.sym_ni - (li + u) : 0;
        xp[u] = a.lext[(int64_t)lo * a.sym_ni + li + u];
        xm[u] = a.lext[(int64_t)mo * a.sym_ni + mi];
        if (!lok) xp[u].y = xm[u].y = -1;
        bm[u] = (int64_t)mo * a.in_os + (int64_t)mi * a.in_is;
      }
      constexpr int BATCH = R1 > 8 ? R1 / 2 : R1;  // elements (and mirrors) in flight
#pragma unroll
      for (int r0 = 0; r0 < R1; r0 += BATCH) {
        E g[BATCH];
        C2<T> m[V][BATCH];
        unsigned keep[V] = {};
#pragma unroll
        for (int r = 0; r < BATCH; ++r) {
          const int e = j + (r0 + r) * TPL, me = e ? L - e : 0;
          bool any = false;
#pragma unroll
          for (int u = 0; u < V; ++u) {
            int dp = e - xp[u].x, dm = me - xm[u].x;
            dp += dp < 0 ? L : 0;
            dm += dm < 0 ? L : 0;
            const bool ip = dp <= xp[u].y, im = dm <= xm[u].y;
            any |= ip;
            m[u][r] = in[im ? bm[u] + (int64_t)me * a.in_es : 0];
            keep[u] |= ((unsigned)ip | ((unsigned)im << 1)) << (2 * r);
          }
          g[r] = *reinterpret_cast<const E*>(in + (any ? bp + (int64_t)e * a.in_es : 0));
        }
#pragma unroll
        for (int r = 0; r < BATCH; ++r)
#pragma unroll
          for (int u = 0; u < V; ++u) {
            const bool ip = (keep[u] >> (2 * r)) & 1u, im = (keep[u] >> (2 * r + 1)) & 1u;
            const T px = ip ? g[r].u[u].x : T(0), py = ip ? g[r].u[u].y : T(0);
            const T mx = im ? m[u][r].x : T(0), my = im ? m[u][r].y : T(0);
            v[u][r0 + r] = C2<T>{T(0.5) * (px + mx), T(0.5) * (py - my)};
          }
      }
#pragma unroll
      for (int u = 0; u < V; ++u) reg_butterfly<T, SG, SEQ, 0, false>(v[u]);
    }
  }

  // the last stage's output i RL + r is position bf(i) + r JB; a cropped
  // output keeps N/2 positions at either end, position p as element
  // p + N/2 mod L.  With RL a multiple of four which r are kept is known here.
  constexpr int JB = L / RL;
  auto pos = [&](int i, int r) { return S::template bf<SEQ::NS - 1>(j, i) + r * JB; };
  auto own = [&](int i) { return S::template own<SEQ::NS - 1>(j, i); };
  auto maybe = [](int r) { return RL % 4 || r < RL / 4 || r >= 3 * RL / 4; };
  auto kept = [](int p) { return 4 * p < L || 4 * p >= 3 * L; };
  auto elem = [](int p) { return 4 * p < L ? p + L / 4 : p - 3 * L / 4; };

  // the density values of the energy partials, in flight with the exchange
  T rho[KIND == RP_INV_Z ? NBL * RL : 1];
  if constexpr (KIND == RP_INV_Z) {
    if (a.rho) {
#pragma unroll
      for (int i = 0; i < NBL; ++i)
#pragma unroll
        for (int r = 0; r < RL; ++r)
          if (maybe(r)) {
            const int p = pos(i, r);
            rho[i * RL + r] = a.rho[(int64_t)ln * a.out_os + (kept(p) ? elem(p) : 0)];
          }
    }
  }

  reg_stages<T, S, SG, 1>(smem, v, l, j, a.tw);

  if constexpr (KIND == RP_FWD_Z) {
    C2<T>* out = (C2<T>*)a.out + (int64_t)ln * a.out_os;
#pragma unroll
    for (int i = 0; i < NBL; ++i)
      if (lok && own(i)) {
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          const int p = pos(i, r);
          if (!a.half_out || 2 * p <= L) out[p] = v[0][i * RL + r];
        }
      }
  } else if constexpr (KIND == RP_INV_Z) {
    const int i0 = (int)a.dn1.div(ln), i1 = ln - i0 * a.n1;
    const double f = a.dec0[i0] * a.dec1[i1];
    const double shift = a.shift ? *a.shift : 0.0;
    double eacc = 0.0;
    T* out = (T*)a.out + (int64_t)ln * a.out_os;
#pragma unroll
    for (int i = 0; i < NBL; ++i)
      if (lok && own(i)) {
#pragma unroll
        for (int r = 0; r < RL; ++r)
          if (maybe(r)) {
            const int p = pos(i, r);
            if (RL % 4 == 0 || kept(p)) {
              const int e = elem(p);
              const C2<T> x = v[0][i * RL + r];
              const double d = f * a.dec2[e];
              double u = __builtin_fma((double)x.x, d, shift);
              if (a.split) u += (double)x.y;
              out[e] = (T)u;
              if (a.rho) eacc = __builtin_fma((double)rho[i * RL + r], u, eacc);
            }
          }
      }
    if (a.eparts) reg_block_sum<S::NT>(smem, eacc, a.eparts + blk);
  } else {
    typedef CV<T, V> E;
    C2<T>* out = (C2<T>*)a.out + (int64_t)lo * a.out_os + (int64_t)li * a.out_is;
    int2 ox[V];
    if constexpr (KIND == RP_FWD) {
      // elements beyond a line's output range are never read: not stored where
      // no line of the group has them
#pragma unroll
      for (int u = 0; u < V; ++u)
        ox[u] = a.oext ? a.oext[(int64_t)lo * a.ic + (li + u < (int)a.ic ? li + u : li)] : int2{0, L - 1};
    }
#pragma unroll
    for (int i = 0; i < NBL; ++i)
      if (lok && own(i)) {
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          const int p = pos(i, r);
          E x;
#pragma unroll
          for (int u = 0; u < V; ++u) x.u[u] = v[u][i * RL + r];
          if constexpr (KIND == RP_FWD) {
            bool any = false;
#pragma unroll
            for (int u = 0; u < V; ++u) {
              int dp = p - ox[u].x;
              dp += dp < 0 ? L : 0;
              any |= dp <= ox[u].y;
            }
            if (any) *reinterpret_cast<E*>(out + (int64_t)p * a.out_es) = x;
          } else {
            if (maybe(r) && (RL % 4 == 0 || kept(p))) *reinterpret_cast<E*>(out + (int64_t)elem(p) * a.out_es) = x;
          }
        }
      }
  }
}

template <typename T, int KIND, int R1, int R2, int R3, int R4>
using RegPassShape = RegShape<T, reg_strided<KIND>(), RegSeq<R1, R2, R3, R4>>;

template <typename T, int KIND, int R1, int R2, int R3, int R4>
__global__ void __launch_bounds__((RegPassShape<T, KIND, R1, R2, R3, R4>::NT)) k_reg_pass(PassArgs<T> a) {
  reg_pass_body<T, KIND, RegSeq<R1, R2, R3, R4>>(a, blockIdx.x);
}

// The lengths with a kernel of their own and their radices: in float64 the
// largest that end in few stages, in float32 those of the any-length kernel.
// They are 40 of the 49 that a grid can have (2 N, N even from 8 to 512, a
// product of 2, 3 and 5): those that take at most four stages in float32, save
// 500 = 4 x 5 x 5 x 5.  Of the others (324, 432, 500, 540, 648, 720, 864, 900,
// 972) float32 needs five stages and more, which the any-length kernel runs in
// both precisions.
#define JGB_REG_LENGTHS_F64(X)                                                                                        \
  X(4, 4, 1, 1) X(4, 5, 1, 1) X(4, 6, 1, 1) X(4, 8, 1, 1) X(12, 3, 1, 1) X(4, 10, 1, 1) X(4, 12, 1, 1)               \
  X(12, 5, 1, 1) X(8, 8, 1, 1) X(12, 6, 1, 1) X(8, 10, 1, 1) X(8, 12, 1, 1) X(4, 5, 5, 1) X(12, 3, 3, 1)            \
  X(12, 10, 1, 1) X(8, 16, 1, 1) X(12, 12, 1, 1) X(8, 4, 5, 1) X(12, 3, 5, 1) X(12, 16, 1, 1) X(20, 10, 1, 1)       \
  X(12, 3, 6, 1) X(8, 5, 6, 1) X(16, 16, 1, 1) X(12, 2, 12, 1) X(20, 3, 5, 1) X(16, 20, 1, 1) X(12, 3, 10, 1)      \
  X(12, 2, 16, 1) X(20, 20, 1, 1) X(12, 2, 20, 1) X(16, 2, 16, 1) X(12, 4, 12, 1) X(20, 3, 10, 1) X(16, 2, 20, 1)    \
  X(16, 3, 16, 1) X(20, 2, 20, 1) X(16, 3, 20, 1) X(20, 5, 10, 1) X(16, 4, 16, 1)
#define JGB_REG_LENGTHS_F32(X)                                                                                        \
  X(8, 2, 1, 1) X(4, 5, 1, 1) X(8, 3, 1, 1) X(8, 4, 1, 1) X(4, 3, 3, 1) X(8, 5, 1, 1) X(8, 2, 3, 1) X(4, 3, 5, 1)     \
  X(8, 8, 1, 1) X(8, 3, 3, 1) X(8, 2, 5, 1) X(8, 4, 3, 1) X(4, 5, 5, 1) X(4, 3, 3, 3) X(8, 3, 5, 1) X(8, 8, 2, 1)     \
  X(8, 2, 3, 3) X(8, 4, 5, 1) X(4, 3, 3, 5) X(8, 8, 3, 1) X(8, 5, 5, 1) X(8, 3, 3, 3) X(8, 2, 3, 5) X(8, 8, 4, 1)     \
  X(8, 4, 3, 3) X(4, 3, 5, 5) X(8, 8, 5, 1) X(8, 3, 3, 5) X(8, 8, 2, 3) X(8, 2, 5, 5) X(8, 4, 3, 5) X(8, 8, 8, 1)     \
  X(8, 8, 3, 3) X(8, 3, 5, 5) X(8, 8, 2, 5) X(8, 8, 4, 3) X(8, 4, 5, 5) X(8, 8, 3, 5) X(8, 5, 5, 5) X(8, 8, 8, 2)

template <typename T>
constexpr bool reg_length(int L) {
#define JGB_REG_IS(R1, R2, R3, R4) \
  if (L == R1 * R2 * R3 * R4) return true;
  if constexpr (sizeof(T) == 8) {
    JGB_REG_LENGTHS_F64(JGB_REG_IS)
  } else {
    JGB_REG_LENGTHS_F32(JGB_REG_IS)
  }
#undef JGB_REG_IS
  return false;
}

// lines per block of a contiguous pass (its per-block partial sums)
template <typename T>
constexpr int reg_z_lines(int L) {
#define JGB_REG_ZL(R1, R2, R3, R4) \
  if (L == R1 * R2 * R3 * R4) return RegShape<T, false, RegSeq<R1, R2, R3, R4>>::LB;
  if constexpr (sizeof(T) == 8) {
    JGB_REG_LENGTHS_F64(JGB_REG_ZL)
  } else {
    JGB_REG_LENGTHS_F32(JGB_REG_ZL)
  }
#undef JGB_REG_ZL
  return 0;
}

// The kind of the any-length kernel that runs pass KIND.
constexpr PassKind any_kind(int kind) {
  return kind == RP_FWD_Z ? PASS_FWD_Z : kind == RP_INV_Z ? PASS_INV_Z : kind == RP_HSYM ? PASS_HSYM : PASS_COMPLEX;
}

// Threads of a batched block: the largest of any member's (those past a
// member's own block leave at once).
template <typename T, int KIND>
constexpr int reg_batch_threads() {
  int n = pass_threads<T, any_kind(KIND)>();
#define JGB_REG_NT(R1, R2, R3, R4) \
  if (RegPassShape<T, KIND, R1, R2, R3, R4>::NT > n) n = RegPassShape<T, KIND, R1, R2, R3, R4>::NT;
  if constexpr (sizeof(T) == 8) {
    JGB_REG_LENGTHS_F64(JGB_REG_NT)
  } else {
    JGB_REG_LENGTHS_F32(JGB_REG_NT)
  }
#undef JGB_REG_NT
  return (n + 63) / 64 * 64;
}

// One launch for the members of a batch, whatever their lengths: a site of the
// batch's pipeline stays one launch when its members' grids differ.
template <typename T, int KIND>
__global__ void __launch_bounds__((reg_batch_threads<T, KIND>()))
    k_reg_pass_b(const PassArgs<T>* __restrict__ tab, const int* __restrict__ bstart, int nm) {
  int m;
  const int blk = batch_block(bstart, nm, blockIdx.x, m);
  if (blk < 0) return;
  const PassArgs<T>& a = tab[m];
#define JGB_REG_BODY(R1, R2, R3, R4)                                           \
  if (a.L == R1 * R2 * R3 * R4) {                                              \
    if (threadIdx.x >= RegPassShape<T, KIND, R1, R2, R3, R4>::NT) return;      \
    reg_pass_body<T, KIND, RegSeq<R1, R2, R3, R4>>(a, blk);                    \
    return;                                                                    \
  }
  if constexpr (sizeof(T) == 8) {
    JGB_REG_LENGTHS_F64(JGB_REG_BODY)
  } else {
    JGB_REG_LENGTHS_F32(JGB_REG_BODY)
  }
#undef JGB_REG_BODY
  if (threadIdx.x >= pass_threads<T, any_kind(KIND)>()) return;
  fft_pass_body<T, any_kind(KIND), pass_elems<T, any_kind(KIND)>(), pass_threads<T, any_kind(KIND)>()>(a, blk);
}

// Launch pass KIND for a length with reg_length<T>(a.L), and the batched form
// of any length (instantiated per kind and precision in regfft_*.hip).
template <typename T, int KIND>
hipError_t launch_reg_pass(const PassArgs<T>& a, hipStream_t s);
template <typename T, int KIND>
hipError_t launch_reg_batch(const void* table, const int* bstart, int nm, unsigned blocks, unsigned threads, size_t smem,
                            hipStream_t s);
#define JGB_REG_DECLARE1(TYPE, KIND_)                                          \
  template <>                                                                  \
  hipError_t launch_reg_pass<TYPE, KIND_>(const PassArgs<TYPE>&, hipStream_t); \
  template <>                                                                  \
  hipError_t launch_reg_batch<TYPE, KIND_>(const void*, const int*, int, unsigned, unsigned, size_t, hipStream_t);
#define JGB_REG_DECLARE(KIND_)    \
  JGB_REG_DECLARE1(double, KIND_) \
  JGB_REG_DECLARE1(float, KIND_)
JGB_REG_DECLARE(RP_FWD_Z)
JGB_REG_DECLARE(RP_INV_Z)
JGB_REG_DECLARE(RP_FWD)
JGB_REG_DECLARE(RP_INV)
JGB_REG_DECLARE(RP_HSYM)
#undef JGB_REG_DECLARE
#undef JGB_REG_DECLARE1

template <typename T, int KIND, int R1, int R2, int R3, int R4>
hipError_t launch_reg_shape(const PassArgs<T>& a, hipStream_t s) {
  typedef RegPassShape<T, KIND, R1, R2, R3, R4> S;
  const unsigned blocks = (unsigned)(((reg_strided<KIND>() ? a.ngroups : a.nlines) + S::LB - 1) / S::LB);
  if (launch_recorded(a, &launch_reg_batch<T, KIND>, blocks, reg_batch_threads<T, KIND>(), S::lds)) return hipSuccess;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL((k_reg_pass<T, KIND, R1, R2, R3, R4>), dim3(blocks), dim3(S::NT), S::lds, s, a);
  return hipGetLastError();
}

#define JGB_REG_CASE(R1, R2, R3, R4) \
  case R1 * R2 * R3 * R4: return launch_reg_shape<T, KIND, R1, R2, R3, R4>(a, s);
#define JGB_REG_INSTANTIATE(TYPE, KIND_, LENGTHS)                                                                  \
  template <typename T, int KIND>                                                                                  \
  static hipError_t reg_switch_##KIND_(const PassArgs<T>& a, hipStream_t s) {                                      \
    switch (a.L) {                                                                                                 \
      LENGTHS(JGB_REG_CASE)                                                                                        \
      default: return hipErrorInvalidValue;                                                                        \
    }                                                                                                              \
  }                                                                                                                \
  template <>                                                                                                      \
  hipError_t launch_reg_pass<TYPE, KIND_>(const PassArgs<TYPE>& a, hipStream_t s) {                                \
    return reg_switch_##KIND_<TYPE, KIND_>(a, s);                                                                  \
  }                                                                                                                \
  template <>                                                                                                      \
  hipError_t launch_reg_batch<TYPE, KIND_>(const void* table, const int* bstart, int nm, unsigned blocks,          \
                                           unsigned threads, size_t smem, hipStream_t s) {                         \
    return batch_launch<PassArgs<TYPE>, k_reg_pass_b<TYPE, KIND_>>(table, bstart, nm, blocks, threads, smem, s);   \
  }

}  // namespace fft
}  // namespace jgb
