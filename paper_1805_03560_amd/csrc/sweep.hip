// The stencil and CG steps on several right-hand sides: a workgroup takes 64 output sites through all of
// them, eight wavefronts for the eight directions (split.h).
//
// A thread loads the link of its direction once and keeps it (and the neighbour's address) while it steps
// through the right-hand sides.  The workgroups in flight on an XCD (64 in FP64, about 4000 sites) pass
// through the right-hand sides together, so what its L2 has to hold between a spinor's use as an x, y, z
// and t neighbour is one right-hand side of those sites.  With one right-hand side a thread per site reads
// as much and waits less: 24^3 x 48 FP64 98 us a hop.
#include <type_traits>

#include "split.h"

namespace whmc {

enum { kSwHop, kSwU, kSwR, kSwRes };

// On the right-hand sides in mask that are not stopped (sc may be null):  kSwHop: out = H in;
// kSwU: out = x - k2 H in, |out|^2;  kSwR: A p = x - k2 H in, r -= alpha A p, xs += alpha p, |r|^2;
// kSwRes: r = p - (x - k2 H in), |r|^2.  The norms go to part[rhs][nparts], unless it is null.
//
// 128 registers in FP64 hold the link, a neighbour and its half spinor, and no more: what the sums need is
// loaded after the barrier (with the loads before it 84 to 148 bytes of a thread spill, and a CG iteration
// on four right-hand sides at 24^3 x 48 takes 1937 us, 1256 so).  24^3 x 48, against the better blocking
// of a thread per site:  FP64 hop on four 264 -> 205 us, on twelve 679 -> 549, CG iteration 1434 -> 1256
// and 3846 -> 3421;  FP32 122 -> 98, 334 -> 264, 782 -> 699, 2154 -> 1946.
template <int DAG, int MODE, class Lnk, class S>
__global__ __launch_bounds__(kSplitWG, 4) void k_sweep(Geom g, int par, int nrhs, unsigned mask, const CGScalars* sc,
                                                       Lnk L, S in0, S x0, S out0, S p0, S r0, S xs0, double* part,
                                                       int nparts, SplitK2 k2) {
  using R = typename S::Real;
  static_assert(!std::is_same<S, SpinorF16>::value, "the store has no norm over a site's six pairs");
  int half, slot;
  const int sb = site_block_grp(g, blockIdx.x, gridDim.x, 2, half, slot);
  const int base = sb * kBlock + half * kSplitSites;
  // next right-hand side from r on that this launch works on (uniform)
  auto live_from = [&](int r) {
    while (r < nrhs && (!((mask >> r) & 1u) || (sc && (sc[r].done | sc[r].pause)))) ++r;
    return r;
  };
  int r = live_from(0);
  if (r >= nrhs) return;
  if (base >= g.Vh) {   // a padding workgroup of the schedule, or no sites in this half of the last block
    if (MODE != kSwHop && part && threadIdx.x == 0)
      for (; r < nrhs; r = live_from(r + 1)) part[(size_t)r * nparts + 2 * slot + half] = 0.0;
    return;
  }
  __shared__ cplx<R> lds[8][6][kSplitSites];
  __shared__ double lred[kSplitWG / 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // lanes past the last site work on it and store nothing
  const bool here = base + lane < g.Vh;
  const int i = here ? base + lane : g.Vh - 1;
  const int q = wave;   // second half: wavefront q < 6 has the component pair q of the same sites
  const bool act = q < 6 && here;
  const At a2 = at(in0, i);
  bool wrap = false;
  const Coords c = coords_of(g, i, par);
  const int j = neighbour_d(g, c, wave, wrap);
  const At n = at(in0, j);   // the neighbour of this thread's direction
  SU3<R> U;
  L.load(par ^ (wave & 1), wave >> 1, wave & 1 ? j : i, U);
#pragma unroll 1
  while (r < nrhs) {
    {
      Spinor<R> s;
      HalfSpinor<R> u;
      At m = n;   // opaque, or its eleven sums would stay in registers over the loop
      asm volatile("" : "+v"(m.off), "+v"(m.w));
      const R sc_in = load_site(field(in0, r), m, s);
      hop_apply_d<DAG, S::scaled>(wave, U, s, sc_in, wrap, u);
#pragma unroll
      for (int k = 0; k < 6; ++k) lds[wave][k][lane] = u.c[k / 3][k % 3];
    }
    __syncthreads();
    cplx<R> xv[2], acc[2];
    double nrm = 0.0;
    if (act) {
      if (MODE != kSwHop) load2(field(x0, r), a2, q, xv);
      gather2<DAG>(lds, q, lane, acc);
      if (MODE != kSwHop) {
        const R kk = R(k2.v[r]);
#pragma unroll
        for (int m = 0; m < 2; ++m) acc[m] = xv[m] - kk * acc[m];
      }
      if (MODE == kSwR) {
        const R alpha = R(sc[r].alpha);
        cplx<R> pv[2], rv[2];
        load2(field(r0, r), a2, q, rv);
        load2(field(p0, r), a2, q, pv);
        load2(field(xs0, r), a2, q, xv);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          rv[m].re -= alpha * acc[m].re;
          rv[m].im -= alpha * acc[m].im;
          xv[m].re += alpha * pv[m].re;
          xv[m].im += alpha * pv[m].im;
          acc[m] = rv[m];
        }
        store2(field(xs0, r), a2, q, xv, 0.f);
      }
      if (MODE == kSwRes) {
        load2(field(p0, r), a2, q, xv);
#pragma unroll
        for (int m = 0; m < 2; ++m) acc[m] = xv[m] - acc[m];
      }
      if (MODE != kSwHop && part) nrm = double(norm2(acc[0]) + norm2(acc[1]));
      store2(field(MODE == kSwR || MODE == kSwRes ? r0 : out0, r), a2, q, acc, 0.f);
    }
    if (MODE != kSwHop && part) wave_total(nrm, lred);
    __syncthreads();   // the sums are read: the next right-hand side may take their place
    if (MODE != kSwHop && part && threadIdx.x == 0) part[(size_t)r * nparts + 2 * slot + half] = add_waves(lred);
    r = live_from(r + 1);
  }
}

// ------------------------------------------------------------------ host side
template <bool NT, class F>
static void with_links_nt(whmc_ctx* c, int prec, int links, F&& f) {
  const int Vh = c->Vh;
  if (prec == WHMC_F64) {
    if (links == WHMC_L18) f(LinkF64_18T<NT>{c->U18, Vh}, f64);
    else if (links == WHMC_L12) f(LinkF64_12T<NT>{c->U12, Vh}, f64);
    else f(LinkF64_8T<NT>{c->U8, Vh}, f64);
  } else if (links == WHMC_L12) {
    f(LinkF32_12T<NT>{c->U32_12, Vh}, f32);
  } else {
    f(LinkF32_8T<NT>{c->U32_8, Vh}, f32);
  }
}
// a launch reads each link once: streamed where the link array is large
template <class F>
static whmc_status with_links(whmc_ctx* c, int prec, int links, F&& f) {
  WHMC_TRY(ensure_links(c, prec, links));
  if (c->stream_links(prec, links)) with_links_nt<true>(c, prec, links, f);
  else with_links_nt<false>(c, prec, links, f);
  WHMC_HIP(hipGetLastError());
  return WHMC_OK;
}

template <int DAG, int MODE, class Lnk, class S>
static void launch_sweep(whmc_ctx* c, int par, int nrhs, const Lnk& L, S in, S x, S out, S p, S r, S xs, double* part,
                         const SplitK2& k2, unsigned mask, const CGScalars* sc) {
  const int n = 2 * c->stencil_blocks();
  hipLaunchKernelGGL((k_sweep<DAG, MODE, Lnk, S>), dim3(n), dim3(kSplitWG), 0, c->stream, c->g, par, nrhs, mask, sc, L,
                     in, x, out, p, r, xs, part, n, k2);
}

int sweep_parts(const whmc_ctx* c) { return 2 * c->stencil_blocks(); }

// From two workgroups per CU on (32768 sites; below, the chip is idle while the right-hand sides pass: 12^3 x
// 24, twelve right-hand sides, 244 us per CG iteration against 236 with a thread per site, 151 in FP32
// against 171; 16^4 306 against 378, 203 against 217).  FP32, which has half the work per site, also needs
// right-hand sides enough: 16^3 x 32 with two 97 against 91, with eight 269 against 275, 20^3 x 32 with two 157
// each.  FP16 keeps a thread per site: 24^3 x 48, four right-hand sides 63.5 us a hop against 69 here, twelve
// 212 against 221.  An address is 32 bits into a field.
bool sweep_rhs(const whmc_ctx* c, int prec, int links, int nrhs) {
  if (nrhs < 2 || c->Vh < 32768 || (unsigned long long)c->Vh * 192ull > 0xFFFFFFFFull) return false;
  if (prec == WHMC_F32) return links != WHMC_L18 && (long long)c->Vh * nrhs > 262144;
  return prec == WHMC_F64;
}

static SplitK2 k2s(const double* k2, int nrhs) {
  SplitK2 kk{};
  for (int q = 0; q < nrhs; ++q) kk.v[q] = k2[q];
  return kk;
}

whmc_status sweep_hop(whmc_ctx* c, int prec, int links, int par, int dag, int nrhs, void* out, const void* in,
                      unsigned mask, const CGScalars* sc) {
  return with_links(c, prec, links, [&](auto L, auto mk) {
    const auto I = mk(in, c->Vh), O = mk(out, c->Vh);
    if (dag) launch_sweep<1, kSwHop>(c, par, nrhs, L, I, I, O, I, I, I, nullptr, SplitK2{}, mask, sc);
    else launch_sweep<0, kSwHop>(c, par, nrhs, L, I, I, O, I, I, I, nullptr, SplitK2{}, mask, sc);
  });
}

whmc_status sweep_u(whmc_ctx* c, int prec, int links, int nrhs, void* u, const void* t, const void* p, const double* k2) {
  return with_links(c, prec, links, [&](auto L, auto mk) {
    const auto P = mk(p, c->Vh);
    launch_sweep<0, kSwU>(c, 1, nrhs, L, mk(t, c->Vh), P, mk(u, c->Vh), P, P, P, c->red.partials, k2s(k2, nrhs), ~0u,
                          c->scal);
  });
}

whmc_status sweep_r(whmc_ctx* c, int prec, int links, int nrhs, void* r, void* x, const void* v, const void* u,
                    const void* p, const double* k2) {
  return with_links(c, prec, links, [&](auto L, auto mk) {
    const auto P = mk(p, c->Vh);
    launch_sweep<1, kSwR>(c, 1, nrhs, L, mk(v, c->Vh), mk(u, c->Vh), P, P, mk(r, c->Vh), mk(x, c->Vh), c->red.partials,
                          k2s(k2, nrhs), ~0u, c->scal);
  });
}

whmc_status sweep_residual(whmc_ctx* c, unsigned mask, int nrhs, const double* x, const double* b, const double* k2,
                           void* t, void* u, void* v, void* r) {
  const SplitK2 kk = k2s(k2, nrhs);
  double* part = c->red.partials;
  return with_links(c, WHMC_F64, WHMC_L18, [&](auto L, auto mk) {
    const int Vh = c->Vh;
    const auto X = mk(x, Vh), B = mk(b, Vh), T = mk(t, Vh), U = mk(u, Vh), V = mk(v, Vh), R = mk(r, Vh);
    launch_sweep<0, kSwHop>(c, 0, nrhs, L, X, X, T, X, X, X, nullptr, kk, mask, nullptr);
    launch_sweep<0, kSwU>(c, 1, nrhs, L, T, X, U, X, X, X, nullptr, kk, mask, nullptr);
    launch_sweep<1, kSwHop>(c, 0, nrhs, L, U, U, V, U, U, U, nullptr, kk, mask, nullptr);
    launch_sweep<1, kSwRes>(c, 1, nrhs, L, V, U, U, B, R, U, part, kk, mask, nullptr);
  });
}

// 24^3 x 48: two masses 847 -> 546 us, four 1749 -> 907, against one after the other
whmc_status sweep_mdagm(whmc_ctx* c, double* out, const double* in, const double* kappas, int nrhs, double* te, double* to) {
  double k2[kMaxRhs];
  for (int q = 0; q < nrhs; ++q) k2[q] = kappas[q] * kappas[q];
  const SplitK2 kk = k2s(k2, nrhs);
  return with_links(c, WHMC_F64, WHMC_L18, [&](auto L, auto mk) {
    const int Vh = c->Vh;
    const auto I = mk(in, Vh), O = mk(out, Vh), E = mk(te, Vh), T = mk(to, Vh);
    launch_sweep<0, kSwHop>(c, 0, nrhs, L, I, I, E, I, I, I, nullptr, kk, ~0u, nullptr);
    launch_sweep<0, kSwU>(c, 1, nrhs, L, E, I, T, I, I, I, nullptr, kk, ~0u, nullptr);
    launch_sweep<1, kSwHop>(c, 0, nrhs, L, T, T, E, T, T, T, nullptr, kk, ~0u, nullptr);
    launch_sweep<1, kSwU>(c, 1, nrhs, L, E, T, O, T, T, T, nullptr, kk, ~0u, nullptr);
  });
}

}  // namespace whmc
