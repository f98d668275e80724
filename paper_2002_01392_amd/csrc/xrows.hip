// x transforms on their own: physical rows of nx reals <-> nkx complex (row
// stride nkxp).  Two real rows (2a, 2a+1) share one complex transform:
// z[n] = x_2a[n] + i x_2a+1[n].
//
// Bound by memory: each row is read and written once.  Lengths of the wavefront
// transforms (x_wave_rows) keep a row pair in registers, 8 points per lane,
// with no workgroup barrier; other lengths go through LDS tiles: 8 lines over 256
// threads up to 256 points (4 lines over 512 left 5 of 6 threads idle at 160 points in
// the radix stages), 4 lines over 512 above, where 256 threads have too few rows in
// flight (set_state at 500 x 128 x 97 485 us with 512 threads, 549 with 256; no
// difference up to 320 points).
// Projection of 160 x 160 x 161, which has four of them: 730 -> 624 us; filtered
// nonlinear term of 256 x 192 x 129: 1.61 -> 1.36 ms.
#include "kernels.hpp"
#include "xwave.hpp"

#include <algorithm>

namespace fcns {

// ---------------------------------------------------------------- wavefront rows
// One row pair per N / 8 lanes; lane t of a pair holds points t + S m.  Rows
// past the end (the last pair of an odd count, the last wave's spare pairs)
// read an in-bounds row and store nothing.
template <int N>
struct XwRows {
  static constexpr int S = N / 8, RPW = 64 / S;
};

template <int N>
__global__ __launch_bounds__(64 * XW_WAVES) void k_xw_r2c(XArgs a, const double* __restrict__ phys,
                                                          cpx<double>* __restrict__ xy,
                                                          long long pfs, long long xfs,
                                                          long long nrows) {
  constexpr int S = XwRows<N>::S, RPW = XwRows<N>::RPW;
  __shared__ cpx<double> tw[XW_TW];
  __shared__ cpx<double> xbuf[XW_WAVES][XW_BUF];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  phys += blockIdx.y * pfs;
  xy += blockIdx.y * xfs;
  xw_twiddles<double, N>(tw, tid);
  __syncthreads();
  const bool spare = lane >= S * RPW;
  const int ln = spare ? lane - S : lane;
  const int t = ln % S, half = ln / S;
  cpx<double>* buf = xbuf[wv] + half * (XW_BUF / RPW);
  const long long npair = (nrows + 1) / 2;
  for (long long rw = (long long)blockIdx.x * XW_WAVES + wv; rw * RPW < npair;
       rw += (long long)gridDim.x * XW_WAVES) {
    const long long pr0 = rw * RPW + half, pr = pr0 < npair ? pr0 : npair - 1;
    const bool st = pr0 < npair && !spare;
    const long long ra = 2 * pr, rb = ra + 1 < nrows ? ra + 1 : ra;
    const double *pa = phys + ra * N, *pb = phys + rb * N;
    cpx<double> z[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) z[m] = mk(pa[t + S * m], pb[t + S * m]);
    wave_fft<double, N>(z, buf, tw, t);
#pragma unroll
    for (int m = 0; m < 8; ++m) buf[xw_nat(t + S * m)] = z[m];
    wave_sync();
    cpx<double> *oa = xy + ra * a.nkxp, *ob = xy + rb * a.nkxp;
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      const int k = t + S * m;
      if (k <= N / 2) {
        const cpx<double> Z = buf[xw_nat(k)], Zm = conj(buf[xw_nat(k == 0 ? 0 : N - k)]);
        if (st) oa[k] = (Z + Zm) * 0.5;
        if (st && rb != ra) ob[k] = mul_mi(Z - Zm) * 0.5;
      }
    }
    wave_sync();
  }
}

// The imaginary parts of the kx = 0 and kx = nx/2 bins are dropped, as a c2r
// transform does.
template <int N>
__global__ __launch_bounds__(64 * XW_WAVES) void k_xw_c2r(XArgs a,
                                                          const cpx<double>* __restrict__ xy,
                                                          double* __restrict__ phys, long long xfs,
                                                          long long pfs, long long nrows) {
  constexpr int S = XwRows<N>::S, RPW = XwRows<N>::RPW;
  __shared__ cpx<double> tw[XW_TW];
  __shared__ cpx<double> xbuf[XW_WAVES][XW_BUF];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  phys += blockIdx.y * pfs;
  xy += blockIdx.y * xfs;
  xw_twiddles<double, N>(tw, tid);
  __syncthreads();
  const bool spare = lane >= S * RPW;
  const int ln = spare ? lane - S : lane;
  const int t = ln % S, half = ln / S;
  cpx<double>* buf = xbuf[wv] + half * (XW_BUF / RPW);
  const double sc = 1.0 / N;
  const long long npair = (nrows + 1) / 2;
  for (long long rw = (long long)blockIdx.x * XW_WAVES + wv; rw * RPW < npair;
       rw += (long long)gridDim.x * XW_WAVES) {
    const long long pr0 = rw * RPW + half, pr = pr0 < npair ? pr0 : npair - 1;
    const bool st = pr0 < npair && !spare;
    const long long ra = 2 * pr, rb = ra + 1 < nrows ? ra + 1 : ra;
    const cpx<double> *pa = xy + ra * a.nkxp, *pb = xy + rb * a.nkxp;
    cpx<double> r[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int k = t + S * m, kk = k <= N / 2 ? k : N - k;
      cpx<double> A = pa[kk], B = pb[kk];
      if (kk == 0 || kk == N / 2) A.y = B.y = 0.0;
      // Z[k] = A + i B (k <= N/2), conj(A) + i conj(B) (k > N/2); inverse via conj
      r[m] = conj(k <= N / 2 ? mk(A.x - B.y, A.y + B.x) : mk(A.x + B.y, B.x - A.y));
    }
    wave_fft<double, N>(r, buf, tw, t);
    double *oa = phys + ra * N, *ob = phys + rb * N;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      if (st) oa[t + S * m] = r[m].x * sc;
      if (st && rb != ra) ob[t + S * m] = -r[m].y * sc;
    }
  }
}

// ---------------------------------------------------------------- LDS tiles
// LL complex lines (2 LL rows) per workgroup of xt_threads(LL); element n of line
// l at lds_pos<true>(l, n, 1, x_ls(nx)).
constexpr int xt_threads(int lines) { return lines == 8 ? 256 : 512; }

template <int LL, int PM>
__global__ __launch_bounds__(xt_threads(LL), 4) void k_x_r2c(XArgs a, const double* __restrict__ phys,
                                                 cpx<double>* __restrict__ xy, long long pfs,
                                                 long long xfs, long long nrows) {
  constexpr int XT_NT = xt_threads(LL);
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x;
  const int nx = a.nx, nkx = a.nkx, nkxp = a.nkxp, ls = x_ls(nx);
  cpx<double>* tw = reinterpret_cast<cpx<double>*>(smem);
  cpx<double>* X0 = tw + a.pl.tsize;
  cpx<double>* X1 = X0 + LL * ls;
  phys += blockIdx.y * pfs;
  xy += blockIdx.y * xfs;
  const cpx<double>* gtw = reinterpret_cast<const cpx<double>*>(a.tw);
  for (int i = tid; i < a.pl.tsize; i += XT_NT) tw[i] = gtw[i];
  const long long r0 = (long long)blockIdx.x * (2 * LL);
  // the tile's rows are contiguous
  const int have = (int)(nrows - r0 < 2 * LL ? nrows - r0 : 2 * LL);
  double* Xs = reinterpret_cast<double*>(X0);
  const float rnx = 1.0f / (float)nx;
  for (int e = tid; e < 2 * LL * nx; e += XT_NT) {
    const int rl = x_div(e, nx, rnx), n = e - rl * nx;
    Xs[2 * lds_pos<true>(rl >> 1, n, 1, ls) + (rl & 1)] = rl < have ? phys[r0 * nx + e] : 0.0;
  }
  __syncthreads();
  const cpx<double>* R = fft_fwd<double, LL, PM, true>(X0, X1, 1, ls, a.pl, tw, tid, XT_NT);
  const float rnk = 1.0f / (float)nkxp;
  for (int e = tid; e < LL * nkxp; e += XT_NT) {
    const int al = x_div(e, nkxp, rnk), k = e - al * nkxp;
    if (k >= nkx) continue;
    const cpx<double> Z = R[lds_pos<true>(al, k, 1, ls)];
    const cpx<double> Zm = conj(R[lds_pos<true>(al, k == 0 ? 0 : nx - k, 1, ls)]);
    if (2 * al < have) xy[(r0 + 2 * al) * nkxp + k] = (Z + Zm) * 0.5;
    if (2 * al + 1 < have) xy[(r0 + 2 * al + 1) * nkxp + k] = mul_mi(Z - Zm) * 0.5;
  }
}

template <int LL, int PM>
__global__ __launch_bounds__(xt_threads(LL), 4) void k_x_c2r(XArgs a, const cpx<double>* __restrict__ xy,
                                                 double* __restrict__ phys, long long xfs,
                                                 long long pfs, long long nrows) {
  constexpr int XT_NT = xt_threads(LL);
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x;
  const int nx = a.nx, nkx = a.nkx, nkxp = a.nkxp, ls = x_ls(nx);
  cpx<double>* tw = reinterpret_cast<cpx<double>*>(smem);
  cpx<double>* X0 = tw + a.pl.tsize;
  cpx<double>* X1 = X0 + LL * ls;
  phys += blockIdx.y * pfs;
  xy += blockIdx.y * xfs;
  const cpx<double>* gtw = reinterpret_cast<const cpx<double>*>(a.tw);
  for (int i = tid; i < a.pl.tsize; i += XT_NT) tw[i] = gtw[i];
  const long long r0 = (long long)blockIdx.x * (2 * LL);
  const int have = (int)(nrows - r0 < 2 * LL ? nrows - r0 : 2 * LL);
  const float rnk = 1.0f / (float)nkxp;
  for (int e = tid; e < LL * nkxp; e += XT_NT) {
    const int al = x_div(e, nkxp, rnk), k = e - al * nkxp;
    if (k >= nkx) continue;
    cpx<double> A = 2 * al < have ? xy[(r0 + 2 * al) * nkxp + k] : zero<double>();
    cpx<double> B = 2 * al + 1 < have ? xy[(r0 + 2 * al + 1) * nkxp + k] : zero<double>();
    if (k == 0 || 2 * k == nx) A.y = B.y = 0.0;
    // Z[k] = A + i B, Z[nx - k] = conj(A) + i conj(B); stored conjugated
    X0[lds_pos<true>(al, k, 1, ls)] = conj(mk(A.x - B.y, A.y + B.x));
    if (k > 0 && 2 * k < nx)
      X0[lds_pos<true>(al, nx - k, 1, ls)] = conj(mk(A.x + B.y, B.x - A.y));
  }
  __syncthreads();
  const cpx<double>* R = fft_fwd<double, LL, PM, true>(X0, X1, 1, ls, a.pl, tw, tid, XT_NT);
  const double sc = 1.0 / nx;
  const float rnx = 1.0f / (float)nx;
  for (int e = tid; e < 2 * LL * nx; e += XT_NT) {
    const int rl = x_div(e, nx, rnx), n = e - rl * nx;
    if (rl >= have) break;   // (rows ascend with e)
    // z = conj(R) / nx: row 2a = Re z, row 2a+1 = Im z
    const cpx<double> z = R[lds_pos<true>(rl >> 1, n, 1, ls)];
    phys[r0 * nx + e] = ((rl & 1) ? -z.y : z.x) * sc;
  }
}

// ---------------------------------------------------------------- launchers
#define FCNS_XW_SWITCH(NV, CALL)                                \
  switch (NV) {                                                 \
    case 512: { constexpr int N = 512; CALL; } break;           \
    case 256: { constexpr int N = 256; CALL; } break;           \
    case 192: { constexpr int N = 192; CALL; } break;           \
    case 128: { constexpr int N = 128; CALL; } break;           \
    case 96: { constexpr int N = 96; CALL; } break;             \
    case 64: { constexpr int N = 64; CALL; } break;             \
    default: { constexpr int N = 32; CALL; } break;             \
  }

// the wavefront grid: each workgroup builds its twiddles once, so no more than
// are resident (about 4 per CU)
static dim3 xw_grid(int nx, long long nrows, int nfields) {
  const long long rpw = 64 / (nx / 8), pairs = (nrows + 1) / 2;
  const long long need = (pairs + rpw * XW_WAVES - 1) / (rpw * XW_WAVES);
  return dim3((unsigned)std::min<long long>(need, std::max(1, 1024 / nfields)), nfields);
}
static int x_tile_lines(int nx) { return nx <= 256 ? 8 : 4; }

#define FCNS_XT(KERNEL, ...)                                                             \
  do {                                                                                   \
    const int LL = x_tile_lines(a.nx);                                                   \
    dim3 grid((unsigned)((nrows + 2 * LL - 1) / (2 * LL)), nfields);                     \
    const size_t sh = ((size_t)a.pl.tsize + 2 * LL * x_ls(a.nx)) * sizeof(cpx<double>);  \
    const int pm = prime_form(a.pl, big, LL, xt_threads(LL));                            \
    if (LL == 8)                                                                         \
      FCNS_PM_SWITCH(pm, FCNS_LAUNCH((KERNEL<8, PM>), grid, dim3(xt_threads(8)), sh, st, __VA_ARGS__)) \
    else                                                                                 \
      FCNS_PM_SWITCH(pm, FCNS_LAUNCH((KERNEL<4, PM>), grid, dim3(xt_threads(4)), sh, st, __VA_ARGS__)) \
  } while (0)

void launch_x_r2c(const XArgs& a, bool big, const double* phys, cpx<double>* xy, long long pfs,
                  long long xfs, long long nrows, int nfields, hipStream_t st) {
  if (x_wave_rows(a.nx)) {
    FCNS_XW_SWITCH(a.nx, hipLaunchKernelGGL(k_xw_r2c<N>, xw_grid(a.nx, nrows, nfields),
                                            dim3(64 * XW_WAVES), 0, st, a, phys, xy, pfs, xfs,
                                            nrows))
    return;
  }
  FCNS_XT(k_x_r2c, a, phys, xy, pfs, xfs, nrows);
}

void launch_x_c2r(const XArgs& a, bool big, const cpx<double>* xy, double* phys, long long xfs,
                  long long pfs, long long nrows, int nfields, hipStream_t st) {
  if (x_wave_rows(a.nx)) {
    FCNS_XW_SWITCH(a.nx, hipLaunchKernelGGL(k_xw_c2r<N>, xw_grid(a.nx, nrows, nfields),
                                            dim3(64 * XW_WAVES), 0, st, a, xy, phys, xfs, pfs,
                                            nrows))
    return;
  }
  FCNS_XT(k_x_c2r, a, xy, phys, xfs, pfs, nrows);
}

}  // namespace fcns
