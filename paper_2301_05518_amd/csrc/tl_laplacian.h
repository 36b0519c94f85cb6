// One application of the Laplacian (eq. tlLapl1, or the one-link nabla^2 = H - 6) straight from
// and to natural complex128 fields:
//   out(x) = S(alpha v(x) + beta sum_hops W v),  v = S(in)
// where S rounds a colour vector to the storage format and back (Exch encode and decode, the
// bits that packing, one step and unpacking give).
//
// What bounds a call is latency: at 32^3 FP64 its 17 MB take 4 us at the rate of a large copy,
// three launches and a waited-for table upload took 51 us.  One launch without tables does it
// all: a thread per site, workgroups of one wave so that small slices still spread over the
// chip, the site's seven vectors and six links loaded before the first is used (unrolled
// directions).  Neighbour vectors are rounded again by every reader, which is cheaper than a
// packed copy written and read back.
#pragma once

#include "tl_run.h"

namespace tl {

namespace {

// S of a natural colour vector: v in the arithmetic's precision, rounded to the storage format.
template <int P, typename real>
__device__ __forceinline__ void load_natural(const v2d* __restrict__ in, int64_t i, real (&v)[6]) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    const v2d w = in[3 * i + c];
    v[2 * c] = (real)w.x;
    v[2 * c + 1] = (real)w.y;
  }
}
template <int P, typename real>
__device__ __forceinline__ void round_storage(real (&v)[6]) {
  if constexpr (P == F16S || P == BF16) {
    uint32_t d[Exch<P>::ND];
    Exch<P>::encode(v, d);
    Exch<P>::decode(d, v);
  }
}

template <int P>
__global__ __launch_bounds__(64) void laplacian_kernel(const char* __restrict__ W, int64_t w_mu_stride, int Vp, int Lx,
                                                       int Ly, int Lz, int hop, bool w12, const v2d* __restrict__ in,
                                                       v2d* __restrict__ out, typename Fmt<P>::real alpha,
                                                       typename Fmt<P>::real beta) {
  using real = typename Fmt<P>::real;
  const int V3 = Lx * Ly * Lz;
  // the workgroups of one XCD take a contiguous part of the slice (see xcd_sweep)
  const TileSweep sw = xcd_sweep((V3 + 63) / 64, 0);
  const int site = sw.n > 0 ? sw.tile(0) * 64 + (int)threadIdx.x : V3;
  if (site >= V3) return;
  const int x = site % Lx, yz = site / Lx, y = yz % Ly, z = yz / Ly;
  const int st[3] = {1, Lx, Lx * Ly}, c[3] = {x, y, z}, L[3] = {Lx, Ly, Lz};
  real acc[6], v[6], own[6];
  load_natural<P>(in, site, own);
#pragma unroll
  for (int k = 0; k < 6; k++) acc[k] = (real)0;
#pragma unroll
  for (int mu = 0; mu < 3; mu++) {
    const int f = site + (wrap_sel(c[mu] + hop, L[mu]) - c[mu]) * st[mu];
    const int b = site + (wrap_sel(c[mu] - hop, L[mu]) - c[mu]) * st[mu];
    real m[18];
    run_load_w<P>(w12, W + mu * w_mu_stride, Vp, site, m);
    load_natural<P>(in, f, v);
    round_storage<P>(v);
    mv_acc(m, v, acc);
    run_load_w<P>(w12, W + mu * w_mu_stride, Vp, b, m);
    load_natural<P>(in, b, v);
    round_storage<P>(v);
    mdv_acc(m, v, acc);
  }
  round_storage<P>(own);
  real o[6];
#pragma unroll
  for (int k = 0; k < 6; k++) o[k] = fma_(beta, acc[k], alpha * own[k]);
  round_storage<P>(o);
#pragma unroll
  for (int k = 0; k < 3; k++) out[3 * (int64_t)site + k] = v2d{(double)o[2 * k], (double)o[2 * k + 1]};
}

template <int P>
hipError_t launch_laplacian_p(const char* W, int64_t w_mu_stride, int Vp, const int32_t L[4], int hop, bool w12,
                              const void* in, void* out, double alpha, double beta, hipStream_t s) {
  using real = typename Fmt<P>::real;
  const int64_t V3 = (int64_t)L[0] * L[1] * L[2];
  laplacian_kernel<P><<<(unsigned)((V3 + 63) / 64), 64, 0, s>>>(W, w_mu_stride, Vp, L[0], L[1], L[2], hop, w12,
                                                                static_cast<const v2d*>(in), static_cast<v2d*>(out),
                                                                (real)alpha, (real)beta);
  return hipGetLastError();
}

}  // namespace

}  // namespace tl
