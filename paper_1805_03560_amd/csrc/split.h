// Building blocks of the stencil kernels that give each of a site's eight directions a wavefront: a
// workgroup of 512 threads holds 64 output sites, the half spinors of the eight directions meet in LDS,
// and six of the wavefronts sum and store two of the sites' twelve components each.
#pragma once
#include <type_traits>

#include "internal.h"
#include "stencil.h"

namespace whmc {

constexpr int kSplitSites = 64, kSplitWG = 512;

// ------------------------------------------------------------------ addresses
// A site of a field as a byte offset from the field's (uniform) base and the distance of its entries, both
// 32 bits: the half fields these kernels are used on stay below 4 GiB (split_fits, sweep_rhs).
struct At {
  unsigned off, w;
  int i;
};
template <class S> struct entries;   // 16-byte entries of a site
template <> struct entries<SpinorF64> { static constexpr int n = 12; };
template <> struct entries<SpinorF32> { static constexpr int n = 6; };
template <> struct entries<SpinorF16> { static constexpr int n = 3; };

template <class S> WHMC_DEV At at(const S& f, int i) {
  const int blk = i >> 6;
  const unsigned w = blk < (f.stride >> 6) ? 64u : (unsigned)(f.stride & 63);
  return {((unsigned)blk * 64u * entries<S>::n + (unsigned)(i & 63)) * 16u, w * 16u, i};
}
template <class T, class U> WHMC_DEV T* byte_at(U* p, unsigned off) {
  return (T*)((std::conditional_t<std::is_const<T>::value, const char*, char*>)p + off);
}

// as load_raw()
WHMC_DEV double load_site(const SpinorF64& f, const At& a, Spinor<double>& s) {
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const double2 v = *byte_at<const double2>(f.p, a.off + k * a.w);
    s.c[k / 3][k % 3] = {v.x, v.y};
  }
  return 1.0;
}
WHMC_DEV float load_site(const SpinorF32& f, const At& a, Spinor<float>& s) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const float4 v = *byte_at<const float4>(f.p, a.off + k * a.w);
    s.c[(2 * k) / 3][(2 * k) % 3] = {v.x, v.y};
    s.c[(2 * k + 1) / 3][(2 * k + 1) % 3] = {v.z, v.w};
  }
  return 1.f;
}
WHMC_DEV float load_site(const SpinorF16& f, const At& a, Spinor<float>& s) {
  const float sc = *byte_at<const float>(f.scale, 4u * (unsigned)a.i);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint4 v = *byte_at<const uint4>(f.p, a.off + k * a.w);
    const unsigned int w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int comp = 4 * k + j;
      s.c[comp / 3][comp % 3] = {h2f((unsigned short)(w[j] & 0xffffu)), h2f((unsigned short)(w[j] >> 16))};
    }
  }
  return sc;
}

// ------------------------------------------------------------------ two components of a site
// pair q (0..5) is components 2q and 2q + 1 in every storage format
WHMC_DEV unsigned pair_off(const SpinorF64&, const At& a, int q) { return a.off + 2u * (unsigned)q * a.w; }
WHMC_DEV unsigned pair_off(const SpinorF32&, const At& a, int q) { return a.off + (unsigned)q * a.w; }
WHMC_DEV unsigned pair_off(const SpinorF16&, const At& a, int q) {
  return a.off + (unsigned)(q >> 1) * a.w + 8u * (unsigned)(q & 1);
}
WHMC_DEV void load2(const SpinorF64& f, const At& a, int q, cplx<double>* v) {
  const unsigned o = pair_off(f, a, q);
  const double2 x = *byte_at<const double2>(f.p, o), y = *byte_at<const double2>(f.p, o + a.w);
  v[0] = {x.x, x.y};
  v[1] = {y.x, y.y};
}
WHMC_DEV void load2(const SpinorF32& f, const At& a, int q, cplx<float>* v) {
  const float4 w = *byte_at<const float4>(f.p, pair_off(f, a, q));
  v[0] = {w.x, w.y};
  v[1] = {w.z, w.w};
}
WHMC_DEV void load2(const SpinorF16& f, const At& a, int q, cplx<float>* v) {
  const uint2 w = *byte_at<const uint2>(f.p, pair_off(f, a, q));
  const float sc = *byte_at<const float>(f.scale, 4u * (unsigned)a.i);
  v[0] = {sc * h2f((unsigned short)(w.x & 0xffffu)), sc * h2f((unsigned short)(w.x >> 16))};
  v[1] = {sc * h2f((unsigned short)(w.y & 0xffffu)), sc * h2f((unsigned short)(w.y >> 16))};
}
// m: the largest modulus of the site's components (used by FP16 only)
WHMC_DEV void store2(const SpinorF64& f, const At& a, int q, const cplx<double>* v, float) {
  const unsigned o = pair_off(f, a, q);
  *byte_at<double2>(f.p, o) = make_double2(v[0].re, v[0].im);
  *byte_at<double2>(f.p, o + a.w) = make_double2(v[1].re, v[1].im);
}
WHMC_DEV void store2(const SpinorF32& f, const At& a, int q, const cplx<float>* v, float) {
  *byte_at<float4>(f.p, pair_off(f, a, q)) = make_float4(v[0].re, v[0].im, v[1].re, v[1].im);
}
WHMC_DEV void store2(const SpinorF16& f, const At& a, int q, const cplx<float>* v, float m) {
  const float inv = m > 0.f ? 1.0f / m : 0.f;
  if (q == 0) *byte_at<float>(f.scale, 4u * (unsigned)a.i) = m;
  uint2 w;
  w.x = (unsigned int)f2h(inv * v[0].re) | ((unsigned int)f2h(inv * v[0].im) << 16);
  w.y = (unsigned int)f2h(inv * v[1].re) | ((unsigned int)f2h(inv * v[1].im) << 16);
  *byte_at<uint2>(f.p, pair_off(f, a, q)) = w;
}
template <typename R> WHMC_DEV float pair_max(const cplx<R>* v) {
  return fmaxf(fmaxf(fabsf((float)v[0].re), fabsf((float)v[0].im)), fmaxf(fabsf((float)v[1].re), fabsf((float)v[1].im)));
}

// sum over the eight directions of components 2Q, 2Q + 1 of the site in column s, as accumulate() does it
template <int DAG, int Q, typename R>
WHMC_DEV void gather2_q(const cplx<R> (*u)[6][kSplitSites], int s, cplx<R>* acc) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    constexpr bool up = Q < 3;
    const int k = 2 * Q + j, sp = k / 3;
    const int same = up ? k : k - 6;                        // spin s - 2 of the half spinor
    const int swap = up ? k : (3 - sp) * 3 + (k - 3 * sp);  // the other spin
    cplx<R> a = {R(0), R(0)};
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      const int mu = d >> 1;
      const R sg = ((d & 1) == 0) == (DAG != 0) ? R(1) : R(-1);
      const cplx<R> v = u[d][mu == 0 || mu == 3 ? same : swap][s];
      const R f = up ? R(1) : (mu >= 2 && sp == 3 ? -sg : sg);
      const bool rot = (mu & 1) && !up;   // times i
      a.re += f * (rot ? -v.im : v.re);
      a.im += f * (rot ? v.re : v.im);
    }
    acc[j] = a;
  }
}
// q: uniform over the wavefront, 0 .. 5
template <int DAG, typename R>
WHMC_DEV void gather2(const cplx<R> (*u)[6][kSplitSites], int q, int s, cplx<R>* acc) {
  switch (q) {
    case 0: gather2_q<DAG, 0>(u, s, acc); break;
    case 1: gather2_q<DAG, 1>(u, s, acc); break;
    case 2: gather2_q<DAG, 2>(u, s, acc); break;
    case 3: gather2_q<DAG, 3>(u, s, acc); break;
    case 4: gather2_q<DAG, 4>(u, s, acc); break;
    default: gather2_q<DAG, 5>(u, s, acc); break;
  }
}

// sum over the workgroup in a fixed order, valid in every thread after the barrier in between
WHMC_DEV void wave_total(double v, double* lds) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
}
WHMC_DEV double add_waves(const double* lds) {
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kSplitWG / 64; ++w) s += lds[w];
  return s;
}
// this thread's share of one rhs's partial sums
WHMC_DEV double my_partials(const double* p, int n) {
  double t = 0.0;
  for (int k = threadIdx.x; k < n; k += kSplitWG) t += p[k];
  return t;
}

// ------------------------------------------------------------------ the first half of a hop
// wavefront d = 2 mu + (0 forward, 1 backward): neighbour of the site and the half spinor from it
WHMC_DEV int neighbour_d(const Geom& g, const Coords& c, int d, bool& wrap) {
  switch (d) {
    case 0: return neighbour<0, +1>(g, c, wrap);
    case 1: return neighbour<0, -1>(g, c, wrap);
    case 2: return neighbour<1, +1>(g, c, wrap);
    case 3: return neighbour<1, -1>(g, c, wrap);
    case 4: return neighbour<2, +1>(g, c, wrap);
    case 5: return neighbour<2, -1>(g, c, wrap);
    case 6: return neighbour<3, +1>(g, c, wrap);
    default: return neighbour<3, -1>(g, c, wrap);
  }
}
template <int DAG, bool SCALED, typename R>
WHMC_DEV void hop_apply_d(int d, const SU3<R>& U, const Spinor<R>& s, R sc, bool wrap, HalfSpinor<R>& u) {
  switch (d) {
    case 0: hop_apply<0, +1, DAG, SCALED>(U, s, sc, wrap, u); break;
    case 1: hop_apply<0, -1, DAG, SCALED>(U, s, sc, wrap, u); break;
    case 2: hop_apply<1, +1, DAG, SCALED>(U, s, sc, false, u); break;
    case 3: hop_apply<1, -1, DAG, SCALED>(U, s, sc, false, u); break;
    case 4: hop_apply<2, +1, DAG, SCALED>(U, s, sc, false, u); break;
    case 5: hop_apply<2, -1, DAG, SCALED>(U, s, sc, false, u); break;
    case 6: hop_apply<3, +1, DAG, SCALED>(U, s, sc, false, u); break;
    default: hop_apply<3, -1, DAG, SCALED>(U, s, sc, false, u); break;
  }
}

struct SplitK2 {
  double v[kMaxRhs];
};

// ------------------------------------------------------------------ fields from pointers
inline SpinorF64 f64(const void* p, int Vh) { return SpinorF64{(double2*)p, Vh}; }
inline SpinorF32 f32(const void* p, int Vh) { return SpinorF32{(float4*)p, Vh}; }
inline SpinorF16 f16(const void* p, int Vh) {
  return SpinorF16{(uint4*)p, p ? (float*)((uint4*)p + (size_t)3 * Vh) : nullptr, Vh};
}

}  // namespace whmc
