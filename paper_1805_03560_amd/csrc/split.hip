// The even/odd stencil and the CG iteration on lattices too small to fill the chip with one thread
// per output site: the eight hops into a site are eight wavefronts of one workgroup.
//
// A workgroup of 512 threads holds 64 output sites of one right-hand side.  Wavefront d = 2 mu + (0
// forward, 1 backward) loads the neighbour spinor and the link of its direction for all 64 sites,
// projects and multiplies (hop_half, the same arithmetic as the one-thread-per-site kernels) and puts
// the resulting half spinor into LDS; then every thread sums two of a site's twelve components over
// the eight directions, in the order of the one-thread kernels, and does that pair's share of the
// epilogue.  A hop is then one memory round trip and one barrier deep instead of eight dependent
// direction steps, and 12^3 x 24 (20736 output sites) gives 2592 wavefronts to the 1024 SIMDs
// instead of 324.  The results of a hop are bit for bit those of the other stencil kernels.
//
// The sums of a CG iteration need no kernels of their own here: the workgroups of the step that uses a
// sum add up the few partial sums themselves, all in the same order, so an iteration is five launches
// instead of seven, and four where launches are most of it (k_split_ph).  What bounds it: at 8^4 the
// launches (about 6 us each with their wait for the previous one); at 12^3x24 FP64 the links and spinors,
// which every kernel reads anew from the Infinity Cache (an XCD's L2 starts a kernel empty: 31 MB counted
// per hop, 6.7 us, 5.2 TB/s); in FP16 the arithmetic and address instructions of a wavefront (about 400).
#include <type_traits>
#include <utility>

#include "internal.h"
#include "split.h"

namespace whmc {

// keeps the loads of these kernel arguments above the first branch, so that they wait for memory once
// together instead of once per branch
WHMC_DEV void pin(const Geom& g, const void* links, const void* in) {
  asm volatile("" ::"s"(g.L[0]), "s"(g.L[1]), "s"(g.L[2]), "s"(g.L[3]), "s"(g.Vh), "s"(g.Lxh), "s"(g.dx.m), "s"(g.dx.sh),
               "s"(g.dy.m), "s"(g.dy.sh), "s"(g.dz.m), "s"(g.dz.sh), "s"(links), "s"(in));
}

// s as load_raw() would give it back from a field (the scale is returned), and the store if asked for
WHMC_DEV double as_stored(const SpinorF64& f, const At& a, Spinor<double>& s, bool store) {
  if (store)
#pragma unroll
    for (int k = 0; k < 12; ++k)
      *byte_at<double2>(f.p, a.off + k * a.w) = make_double2(s.c[k / 3][k % 3].re, s.c[k / 3][k % 3].im);
  return 1.0;
}
WHMC_DEV float as_stored(const SpinorF32& f, const At& a, Spinor<float>& s, bool store) {
  if (store)
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const cplx<float>&v = s.c[(2 * k) / 3][(2 * k) % 3], &w = s.c[(2 * k + 1) / 3][(2 * k + 1) % 3];
      *byte_at<float4>(f.p, a.off + k * a.w) = make_float4(v.re, v.im, w.re, w.im);
    }
  return 1.f;
}
WHMC_DEV float as_stored(const SpinorF16& f, const At& a, Spinor<float>& s, bool store) {
  float m = 0.f;
#pragma unroll
  for (int k = 0; k < 12; ++k) m = fmaxf(m, fmaxf(fabsf(s.c[k / 3][k % 3].re), fabsf(s.c[k / 3][k % 3].im)));
  const float inv = m > 0.f ? 1.0f / m : 0.f;
  unsigned int w[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    cplx<float>& z = s.c[k / 3][k % 3];
    const unsigned short re = f2h(inv * z.re), im = f2h(inv * z.im);
    w[k] = (unsigned int)re | ((unsigned int)im << 16);
    z = {h2f(re), h2f(im)};
  }
  if (store) {
    *byte_at<float>(f.scale, 4u * (unsigned)a.i) = m;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      *byte_at<uint4>(f.p, a.off + k * a.w) = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
  }
  return m;
}

// ------------------------------------------------------------------ kernels
enum { kPlain, kXpay, kFullM, kCgHop, kCgU, kCgR, kRes };

// MODE kPlain: out = k2 H in;  kXpay: out = a x + k2 H in;  kFullM: out = x - k2 H in on the whole lattice,
// where field 2 r + parity is a half of full field r;  and the steps of a CG iteration, which skip a
// stopped right-hand side:  kCgHop: out = H in;  kCgU: out = x - k2 H in, |out|^2 to part_out;
// kCgR: with (p, A p) from part_in, alpha = |r|^2 / (p, A p), A p = x - k2 H in, r -= alpha A p,
// xs += alpha p, |r|^2 to part_out.  kRes: out = p - (x - k2 H in), |out|^2 to part_out (the last hop of a
// residual).  The steps after kXpay work on the right-hand sides of the set `mask` that are not stopped
// (sc may be null: none is).
template <int DAG, int MODE, class Lnk, class S, class SR>
__global__ __launch_bounds__(kSplitWG) void k_split(FastDiv by_nrhs, int nrhs, unsigned mask, CGScalars* sc, Geom g, int par,
                                                    Lnk L, S in0, S x0, S out0, S p0, SR r0, SR xs0, double a,
                                                    const double* part_in, double* part_out, int nb, SplitK2 k2) {
  using R = typename S::Real;
  using RR = typename SR::Real;
  constexpr bool cg = MODE >= kCgHop;
  const int B = xcd_remap(blockIdx.x, gridDim.x);   // the right-hand sides of a block run back to back
  const int sb = by_nrhs.div(B), r = B - sb * nrhs;
  pin(g, L.p, in0.p);
  // scalars of the epilogue, read now so that their latency overlaps the hop
  const R kk = MODE == kCgHop ? R(0) : R(k2.v[MODE == kFullM ? r >> 1 : r]);
  if (MODE == kFullM) par = r & 1;
  const double rr_cur = MODE == kCgR ? sc[r].rr : 0.0;
  if (cg && (!((mask >> r) & 1u) || (sc && (sc[r].done | sc[r].pause)))) return;
  __shared__ cplx<R> lds[8][6][kSplitSites];
  __shared__ double lred[kSplitWG / 64], lsum[kSplitWG / 64];
  __shared__ float lmax[std::is_same<S, SpinorF16>::value ? 6 : 1][kSplitSites];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double part = MODE == kCgR ? my_partials(part_in + (size_t)r * nb, nb) : 0.0;
  // lanes past the last site work on it and store nothing
  const bool here = sb * kSplitSites + lane < g.Vh;
  const int i = here ? sb * kSplitSites + lane : g.Vh - 1;
  // second half: wavefront q < 6 has the component pair q of the same sites
  const int q = wave;
  const bool act = q < 6 && here;
  const At a2 = at(in0, i), b2 = at(r0, i);
  cplx<R> xv[2], pv[2];
  cplx<RR> rv[2], xsv[2];
  {
    const Coords c = coords_of(g, i, par);
    bool wrap = false;
    Spinor<R> s;
    SU3<R> U;
    HalfSpinor<R> u;
    const int j = neighbour_d(g, c, wave, wrap);
    const R sc_in = load_site(field(in0, MODE == kFullM ? r ^ 1 : r), at(in0, j), s);
    L.load(par ^ (wave & 1), wave >> 1, wave & 1 ? j : i, U);
    hop_apply_d<DAG, S::scaled>(wave, U, s, sc_in, wrap, u);
#pragma unroll
    for (int k = 0; k < 6; ++k) lds[wave][k][lane] = u.c[k / 3][k % 3];
  }
  // the epilogue's vectors, on their way while the workgroup meets (before the hop they would hold its
  // registers: 142 VGPRs in FP64, one
  // workgroup per compute unit: 14.1 against 11.3 us for the last step at 12^3x24)
  if (MODE != kPlain && MODE != kCgHop && act) load2(field(x0, r), a2, q, xv);
  if ((MODE == kCgR || MODE == kRes) && act) load2(field(p0, r), a2, q, pv);
  if (MODE == kCgR && act) {
    load2(field(r0, r), b2, q, rv);
    load2(field(xs0, r), b2, q, xsv);
  }
  if (MODE == kCgR) wave_total(part, lsum);
  __syncthreads();
  double nrm = 0.0;
  cplx<R> acc[2];
  if (act) gather2<DAG>(lds, q, lane, acc);
  if (MODE == kCgR) {
    const double pAp = add_waves(lsum);
    const bool ok = pAp > 0.0 && pAp < INFINITY;   // else a breakdown: p = 0 or not finite
    const double alpha = ok ? rr_cur / pAp : 0.0;
    if (sb == 0 && threadIdx.x == 0) {   // fields that nothing else in this launch reads
      sc[r].pAp = pAp;
      sc[r].alpha = alpha;
      sc[r].brk = !ok;
    }
    if (act && ok) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const cplx<R> ap = xv[j] - kk * acc[j];
        rv[j].re -= RR(alpha) * RR(ap.re);
        rv[j].im -= RR(alpha) * RR(ap.im);
        xsv[j].re += RR(alpha) * RR(pv[j].re);
        xsv[j].im += RR(alpha) * RR(pv[j].im);
      }
      nrm = double(norm2(rv[0]) + norm2(rv[1]));
    }
    if (act && ok) {
      store2(field(r0, r), b2, q, rv, 0.f);
      store2(field(xs0, r), b2, q, xsv, 0.f);
    }
  } else {
    if (act) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (MODE == kPlain) acc[j] = kk * acc[j];
        if (MODE == kXpay) acc[j] = axpby(R(a), xv[j], kk, acc[j]);
        if (MODE == kCgU || MODE == kFullM) acc[j] = xv[j] - kk * acc[j];
        if (MODE == kRes) acc[j] = pv[j] - (xv[j] - kk * acc[j]);
      }
      if (MODE == kCgU || MODE == kRes) nrm = double(norm2(acc[0]) + norm2(acc[1]));
    }
    float m = 0.f;
    if (std::is_same<S, SpinorF16>::value) {
      if (act) lmax[q][lane] = pair_max(acc);
      __syncthreads();
      if (act)
#pragma unroll
        for (int k = 0; k < 6; ++k) m = fmaxf(m, lmax[k][lane]);
    }
    if (act) store2(field(out0, r), a2, q, acc, m);
  }
  if (MODE == kCgU || MODE == kCgR || MODE == kRes) {
    wave_total(nrm, lred);
    __syncthreads();
    if (threadIdx.x == 0) part_out[(size_t)r * nb + sb] = add_waves(lred);
  }
}

// The scalars of the next iteration, written by the first thread of a rhs: as they are for a right-hand side
// that has stopped or breaks down here (then true) ...
WHMC_DEV bool beta_halted(const CGScalars* o, CGScalars* n, bool first) {
  const int halt = o->done | o->pause | o->brk;
  if (halt && first) {
    n->rr = o->rr, n->pAp = o->pAp, n->alpha = o->alpha, n->beta = o->beta, n->rr_old = o->rr_old;
    n->stop_rr = o->stop_rr, n->rmax2 = o->rmax2, n->delta2 = o->delta2;
    n->done = o->done | o->brk, n->pause = o->pause, n->iter = o->iter, n->active = o->active, n->brk = 0;
  }
  return halt;
}
// ... or from the new |r|^2;  false: it stops here
template <bool MIXED>
WHMC_DEV bool beta_step(const CGScalars* o, CGScalars* n, bool first, double old_rr, double stop_rr, double delta2,
                        double old_rmax2, double rr, double& beta) {
  beta = rr / old_rr;
  const double rmax2 = fmax(old_rmax2, rr);
  const bool finite = rr < INFINITY;
  const bool pause = MIXED && finite && (rr <= stop_rr || rr < delta2 * rmax2);
  const bool done = !finite || (!MIXED && rr <= stop_rr);
  if (first) {
    n->rr = rr, n->pAp = o->pAp, n->alpha = o->alpha, n->beta = beta, n->rr_old = old_rr;
    n->stop_rr = stop_rr, n->rmax2 = MIXED && finite ? rmax2 : old_rmax2, n->delta2 = delta2;
    n->done = done, n->pause = pause, n->iter = o->iter + 1, n->active = o->active, n->brk = 0;
  }
  return !(pause | done);
}

// out = r + beta p (p where the rhs stops here), beta = |r|^2 / |r_old|^2 from the partial sums; every
// workgroup adds them up in the same order, the first one of a rhs writes the scalars of the next
// iteration into the other buffer.  out may be p.
template <bool MIXED, class S, class SR>
__global__ __launch_bounds__(kSplitWG) void k_split_p(FastDiv by_nrhs, int nrhs, int Vh, S p0, S out0, SR r0,
                                                      const CGScalars* cur, CGScalars* nxt, const double* part, int nb) {
  using R = typename S::Real;
  const int B = xcd_remap(blockIdx.x, gridDim.x);
  const int sb = by_nrhs.div(B), r = B - sb * nrhs;
  const bool first = sb == 0 && threadIdx.x == 0;
  const CGScalars* o = cur + r;
  const double old_rr = o->rr, stop_rr = o->stop_rr, delta2 = o->delta2, old_rmax2 = o->rmax2;
  if (beta_halted(o, nxt + r, first)) return;
  const int lane = threadIdx.x & 63, i = sb * kSplitSites + lane;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool act = q < 6 && i < Vh;
  const At ap = at(p0, i), ar = at(r0, i);
  cplx<R> pv[2];
  cplx<typename SR::Real> rv[2];
  if (act) {
    load2(field(p0, r), ap, q, pv);
    load2(field(r0, r), ar, q, rv);
  }
  __shared__ double lsum[kSplitWG / 64];
  __shared__ float lmax[std::is_same<S, SpinorF16>::value ? 6 : 1][kSplitSites];
  wave_total(my_partials(part + (size_t)r * nb, nb), lsum);
  __syncthreads();
  double beta;
  if (beta_step<MIXED>(o, nxt + r, first, old_rr, stop_rr, delta2, old_rmax2, add_waves(lsum), beta)) {
    if (act) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        pv[j].re = R(rv[j].re) + R(beta) * pv[j].re;
        pv[j].im = R(rv[j].im) + R(beta) * pv[j].im;
      }
    }
  } else if (p0.p == out0.p) {
    return;
  }
  float m = 0.f;
  if (std::is_same<S, SpinorF16>::value) {
    if (act) lmax[q][lane] = pair_max(pv);
    __syncthreads();
    if (act)
#pragma unroll
      for (int k = 0; k < 6; ++k) m = fmaxf(m, lmax[k][lane]);
  }
  if (act) store2(field(out0, r), ap, q, pv, m);
}

// k_split_p and the hop t = H p of the next iteration in one launch.  Each wavefront makes the new p of its
// neighbours itself, as the fields hold it; wavefront 0, whose neighbours are all the sites of the other
// parity, once each, stores it.  pout is not p: other workgroups still read that.
template <bool MIXED, class Lnk, class S, class SR>
__global__ __launch_bounds__(kSplitWG, 4) void k_split_ph(FastDiv by_nrhs, int nrhs, Geom g, Lnk L, S p0, S pout0, S t0, SR r0,
                                                       const CGScalars* cur, CGScalars* nxt, const double* part, int nb) {
  using R = typename S::Real;
  const int B = xcd_remap(blockIdx.x, gridDim.x);
  const int sb = by_nrhs.div(B), r = B - sb * nrhs;
  pin(g, L.p, p0.p);
  const bool first = sb == 0 && threadIdx.x == 0;
  const CGScalars* o = cur + r;
  const double old_rr = o->rr, stop_rr = o->stop_rr, delta2 = o->delta2, old_rmax2 = o->rmax2;
  if (beta_halted(o, nxt + r, first)) return;
  __shared__ cplx<R> lds[8][6][kSplitSites];
  __shared__ double lsum[kSplitWG / 64];
  __shared__ float lmax[std::is_same<S, SpinorF16>::value ? 6 : 1][kSplitSites];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double mine = my_partials(part + (size_t)r * nb, nb);
  const bool here = sb * kSplitSites + lane < g.Vh;
  const int i = here ? sb * kSplitSites + lane : g.Vh - 1;
  const int q = wave;
  const bool act = q < 6 && here;
  const At a2 = at(t0, i);
  {
    const Coords c = coords_of(g, i, 0);
    bool wrap = false;
    const int j = neighbour_d(g, c, wave, wrap);
    const At aj = at(p0, j);
    Spinor<R> s;
    Spinor<typename SR::Real> rv;
    SU3<R> U;
    HalfSpinor<R> u;
    const R sc_in = load_site(field(p0, r), aj, s);
    load_site(field(r0, r), at(r0, j), rv);
    if (sizeof(R) == 4) L.load(wave & 1, wave >> 1, wave & 1 ? j : i, U);
    wave_total(mine, lsum);
    __syncthreads();
    double beta;
    const bool live = beta_step<MIXED>(o, nxt + r, first, old_rr, stop_rr, delta2, old_rmax2, add_waves(lsum), beta);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      cplx<R>& z = s.c[k / 3][k % 3];
      const cplx<typename SR::Real>& y = rv.c[k / 3][k % 3];
      if (S::scaled) z = sc_in * z;
      if (live) z = {R(y.re) + R(beta) * z.re, R(y.im) + R(beta) * z.im};
    }
    const R sc = as_stored(field(pout0, r), aj, s, wave == 0 && here);
    if (!live) return;
    if (sizeof(R) == 8) L.load(wave & 1, wave >> 1, wave & 1 ? j : i, U);
    hop_apply_d<0, S::scaled>(wave, U, s, sc, wrap, u);
#pragma unroll
    for (int k = 0; k < 6; ++k) lds[wave][k][lane] = u.c[k / 3][k % 3];
  }
  __syncthreads();
  cplx<R> acc[2];
  if (act) gather2<0>(lds, q, lane, acc);
  float m = 0.f;
  if (std::is_same<S, SpinorF16>::value) {
    if (act) lmax[q][lane] = pair_max(acc);
    __syncthreads();
    if (act)
#pragma unroll
      for (int k = 0; k < 6; ++k) m = fmaxf(m, lmax[k][lane]);
  }
  if (act) store2(field(t0, r), a2, q, acc, m);
}

// ------------------------------------------------------------------ host side
// f(link accessor, spinor maker) for a format; the links are cached, never streamed, on these lattices
template <class F>
static whmc_status with_links(whmc_ctx* c, int prec, int links, F&& f) {
  WHMC_TRY(ensure_links(c, prec, links));
  const int Vh = c->Vh;
  if (prec == WHMC_F64) {
    if (links == WHMC_L18) return f(LinkF64_18T<false>{c->U18, Vh}, f64);
    if (links == WHMC_L12) return f(LinkF64_12T<false>{c->U12, Vh}, f64);
    return f(LinkF64_8T<false>{c->U8, Vh}, f64);
  }
  if (prec == WHMC_F32) {
    if (links == WHMC_L18) return f(LinkF32_18T<false>{c->U32_18, Vh}, f32);
    if (links == WHMC_L12) return f(LinkF32_12T<false>{c->U32_12, Vh}, f32);
    return f(LinkF32_8T<false>{c->U32_8, Vh}, f32);
  }
  if (links == WHMC_L12) return f(LinkF16_12T<false>{c->U16_12, Vh}, f16);
  return f(LinkF16_8T<false>{c->U16_8, Vh}, f16);
}

static int split_blocks(const whmc_ctx* c) { return (c->Vh + kSplitSites - 1) / kSplitSites; }

// Which calls gain from these kernels: lattices whose one-thread-per-site grid leaves SIMDs idle or with a
// single wavefront, as long as the workgroups are few enough that reading a link once per right-hand side
// (from L2) and the spinors of a 64-site block without the 128-site slice schedule costs less than the
// idle SIMDs.  us per CG iteration, one thread per site -> split: 8^4 FP64 39.6 -> 30.7, 12^3x24 FP64
// 52.5 -> 42.8, two rhs FP32 58.1 -> 43.6 and FP16 63.1 -> 44.0, 16^3x32 two rhs FP64 157 -> 141,
// 16^3x20x40 two rhs FP32 147 -> 126; beyond the lines: 16^3x32 two rhs FP16 81 -> 84, 12-rhs hops at
// 16^3x32 FP64 129 -> 139 and FP16 39 -> 53, 20^3x40 one rhs FP64 250 -> 271.  FP16 has the least work
// per site, so its line lies at a total of output sites; FP64 and FP32 have one for the lattice and FP64
// one for the total.  WHMC_OPT_HOP_KERNEL = 1, which a schedule or cap that the caller sets brings with it, selects
// the one-thread-per-site kernels, and so do streamed links.
bool split_fits(const whmc_ctx* c, int prec, int links, int nrhs) {
  if (c->split_off || c->stream_links(prec, links)) return false;
  const long long total = (long long)c->Vh * nrhs;
  if (prec == WHMC_F16) return total <= 98304;
  return c->Vh <= 131072 && (prec == WHMC_F32 || total <= 524288);
}

// ... and which of them take them where the sweep kernels can have the call too: FP64 on two right-hand sides
// (16^4: 79 us per CG iteration against 84, 16^3 x 40: 174 against 178; on three 107 against 104 and 255
// against 237).  The line of FP32 is in sweep_rhs.
bool split_hops(const whmc_ctx* c, int prec, int links, int nrhs) {
  if (!split_fits(c, prec, links, nrhs)) return false;
  return !sweep_rhs(c, prec, links, nrhs) || (prec == WHMC_F64 && nrhs == 2);
}

// ... and of single right-hand sides' CG solves.  Where time slices are whole blocks the other kernels have their
// schedule and an XCD its part of every slice; up to this size these are ahead of it all the same.  Where they are not,
// the line is lower for 12- and 18-real links, us per iteration with one thread per site and so: 30x20x18x20
// (108 000) FP64-12 137.0, 134.9, FP32-12 79.4, 77.9;  32x20x20x18 (115 200) FP64-18 165.4, 167.1, FP64-12 141.2,
// 146.3, FP32-12 80.7, 82.1, FP64-8 134.3, 131.1;  whole slices, 36x16x20x20 (115 200) FP64-18 180.3, 162.7, FP64-12
// 156.0, 143.2, FP32-12 91.3, 80.6.
bool split_solves(const whmc_ctx* c, int prec, int links) {
  return split_hops(c, prec, links, 1) && (c->g.nbs > 0 || links == WHMC_L8 || c->Vh <= 110592);
}

template <int DAG, int MODE, class Lnk, class S, class SR>
static void launch_split(whmc_ctx* c, int par, int nrhs, const Lnk& L, S in, S x, S out, S p, SR r, SR xs, double a,
                         const SplitK2& k2, unsigned mask, CGScalars* sc, const double* part_in,
                         double* part_out) {
  const int nb = split_blocks(c);
  hipLaunchKernelGGL((k_split<DAG, MODE, Lnk, S, SR>), dim3(nb * nrhs), dim3(kSplitWG), 0, c->stream, fast_div(nrhs),
                     nrhs, mask, sc, c->g, par, L, in, x, out, p, r, xs, a, part_in, part_out, nb, k2);
}

whmc_status split_hop(whmc_ctx* c, int prec, int links, int par, int dag, int nrhs, void* out, const void* in,
                      const void* x, double a, const double* b) {
  SplitK2 kb{};
  for (int q = 0; q < nrhs; ++q) kb.v[q] = b[q];
  auto run = [&](auto L, auto mk) {
    const auto I = mk(in, c->Vh), X = mk(x, c->Vh), O = mk(out, c->Vh);
    auto go = [&](auto dagc, auto mode) {
      launch_split<decltype(dagc)::value, decltype(mode)::value>(c, par, nrhs, L, I, X, O, X, X, X, a, kb, 0u, nullptr,
                                                                 nullptr, nullptr);
    };
    using D0 = std::integral_constant<int, 0>;
    using D1 = std::integral_constant<int, 1>;
    using Plain = std::integral_constant<int, kPlain>;
    using Xpay = std::integral_constant<int, kXpay>;
    if (x) dag ? go(D1{}, Xpay{}) : go(D0{}, Xpay{});
    else dag ? go(D1{}, Plain{}) : go(D0{}, Plain{});
    return WHMC_OK;
  };
  WHMC_TRY(with_links(c, prec, links, run));
  WHMC_HIP(hipGetLastError());
  return WHMC_OK;
}

whmc_status split_fullM(whmc_ctx* c, int dag, int nrhs, double* out, const double* in, const double* kappas) {
  SplitK2 kk{};
  for (int q = 0; q < nrhs; ++q) kk.v[q] = kappas[q];
  const LinkF64_18T<false> L{c->U18, c->Vh};
  const SpinorF64 I = f64(in, c->Vh), O = f64(out, c->Vh);
  if (dag) launch_split<1, kFullM>(c, 0, 2 * nrhs, L, I, I, O, I, I, I, 0.0, kk, 0u, nullptr, nullptr, nullptr);
  else launch_split<0, kFullM>(c, 0, 2 * nrhs, L, I, I, O, I, I, I, 0.0, kk, 0u, nullptr, nullptr, nullptr);
  WHMC_HIP(hipGetLastError());
  return WHMC_OK;
}

// sum of nb partials of each rhs in mask, one workgroup per rhs
__global__ __launch_bounds__(kFinWG) void k_split_sum(unsigned mask, const double* part, int nb, double* out) {
  const int r = blockIdx.x;
  if (!((mask >> r) & 1u)) return;
  const double t = sum_partials(part + (size_t)r * nb, nb);
  if (threadIdx.x == 0) out[r] = t;
}

whmc_status split_residual(whmc_ctx* c, unsigned mask, int nrhs, const double* x, const double* b, const double* k2,
                           void* t, void* u, void* v, void* r, double* rr_dev) {
  SplitK2 kk{};
  for (int q = 0; q < nrhs; ++q) kk.v[q] = k2[q];
  const int Vh = c->Vh;
  const LinkF64_18T<false> L{c->U18, Vh};
  const SpinorF64 X = f64(x, Vh), B = f64(b, Vh), T = f64(t, Vh), U = f64(u, Vh), V = f64(v, Vh), R = f64(r, Vh);
  double* pa = c->red.partials;
  launch_split<0, kCgHop>(c, 0, nrhs, L, X, X, T, X, R, R, 0.0, kk, mask, nullptr, pa, pa);
  launch_split<0, kCgU>(c, 1, nrhs, L, T, X, U, X, R, R, 0.0, kk, mask, nullptr, pa, pa);
  launch_split<1, kCgHop>(c, 0, nrhs, L, U, U, V, U, R, R, 0.0, kk, mask, nullptr, pa, pa);
  launch_split<1, kRes>(c, 1, nrhs, L, V, U, R, B, R, R, 0.0, kk, mask, nullptr, pa, pa);
  hipLaunchKernelGGL(k_split_sum, dim3(nrhs), dim3(fin_threads(split_blocks(c))), 0, c->stream, mask, pa,
                     split_blocks(c), rr_dev);
  WHMC_HIP(hipGetLastError());
  return WHMC_OK;
}

// One launch instead of two for p and the next hop where the launches are most of an iteration: eight
// wavefronts now make each p, so it is a loss on more work.  us per iteration, two launches -> one:  FP32 8^4
// 35.8 -> 33.0, 12^3x24 38.0 -> 35.1, 16^4 42.4 -> 39.9, 12^3x24 four rhs 63.5 -> 65.1, 16^3x32 56.0 -> 57.0;
// FP16 35.5 -> 32.5, 36.9 -> 35.1, 41.1 -> 39.7, 60.0 -> 62.2, 48.5 -> 49.3;  FP64 8^4 26.7 -> 25.9, four rhs
// 31.1 -> 29.7, 12^3x24 41.0 -> 44.3 (22 of its registers spill).
static bool fuse_p(const whmc_ctx* c, int prec, int nrhs) {
  return (long long)c->Vh * nrhs <= (prec == WHMC_F64 ? 8192 : 49152);
}

whmc_status split_cg(whmc_ctx* c, int prec, int links, int nrhs, void* p, void* t, void* u, void* v, void* r, void* x,
                     const double* k2, int n) {
  SplitK2 kk{};
  for (int q = 0; q < nrhs; ++q) kk.v[q] = k2[q];
  auto run = [&](auto L, auto mk) {
    const int Vh = c->Vh, nb = split_blocks(c);
    const auto P = mk(p, Vh), T = mk(t, Vh), U = mk(u, Vh), V = mk(v, Vh);
    using S = std::remove_cv_t<decltype(P)>;
    constexpr bool mixed = !std::is_same<S, SpinorF64>::value;
    std::conditional_t<mixed, SpinorF32, SpinorF64> R, X;
    if constexpr (mixed) R = f32(r, Vh), X = f32(x, Vh);
    else R = f64(r, Vh), X = f64(x, Vh);
    using SR = decltype(R);
    double* pa = c->red.partials;                 // (p, A p)
    double* pb = pa + (size_t)kMaxRhs * nb;       // |r|^2
    // p moves between two fields where its update and the next iteration's first hop are one launch
    void* other = nullptr;
    if (n > 1 && fuse_p(c, prec, nrhs) && workspace(c, "split_p", (size_t)Vh * (mixed ? (prec == WHMC_F32 ? 96 : 52) : 192) * nrhs, &other) != WHMC_OK) {
      (void)hipGetLastError();   // no memory for it: two launches
      other = nullptr;
    }
    S now = P, next = mk(other, Vh);
    for (int it = 0; it < n; ++it) {
      TraceRange tr(mixed ? "whmc cg iteration (mixed)" : "whmc cg iteration");
      CGScalars* cur = c->scal;
      CGScalars* nxt = cur == c->scal_base ? c->scal_base + kMaxRhs : c->scal_base;
      const dim3 grid(nb * nrhs), block(kSplitWG);
      if (it == 0 || !other) launch_split<0, kCgHop>(c, 0, nrhs, L, now, now, T, now, R, X, 0.0, kk, ~0u, cur, pa, pa);
      launch_split<0, kCgU>(c, 1, nrhs, L, T, now, U, now, R, X, 0.0, kk, ~0u, cur, pa, pa);
      launch_split<1, kCgHop>(c, 0, nrhs, L, U, U, V, U, R, X, 0.0, kk, ~0u, cur, pa, pa);
      launch_split<1, kCgR>(c, 1, nrhs, L, V, U, V, now, R, X, 0.0, kk, ~0u, cur, pa, pb);
      if (other && it + 1 < n) {
        hipLaunchKernelGGL((k_split_ph<mixed, decltype(L), S, SR>), grid, block, 0, c->stream, fast_div(nrhs), nrhs, c->g,
                           L, now, next, T, R, cur, nxt, pb, nb);
        std::swap(now, next);
      } else {
        hipLaunchKernelGGL((k_split_p<mixed, S, SR>), grid, block, 0, c->stream, fast_div(nrhs), nrhs, Vh, now, P, R, cur,
                           nxt, pb, nb);
      }
      c->scal = nxt;
    }
    return WHMC_OK;
  };
  WHMC_TRY(with_links(c, prec, links, run));
  WHMC_HIP(hipGetLastError());
  return WHMC_OK;
}

}  // namespace whmc
