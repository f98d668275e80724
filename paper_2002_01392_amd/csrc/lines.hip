// FC-Gram continuation of real lines (fc_extend).
#include "kernels.hpp"

#include <algorithm>

namespace fcns {

// ---------------------------------------------------------------- general strides
// One thread per line: consecutive lanes are consecutive lines, so the
// accesses are contiguous where the line index is the fastest one.
__global__ __launch_bounds__(256) void k_fc_extend(const double* __restrict__ in, long long nlines,
                                                   long long ips, long long ils,
                                                   double* __restrict__ out, long long ops,
                                                   long long ols, int nz, int C, int d,
                                                   const double* __restrict__ M) {
  const long long line = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (line >= nlines) return;
  const double* f = in + line * ils;
  double* o = out + line * ols;
  for (int s = 0; s < nz; ++s) o[s * ops] = f[s * ips];
  for (int i = 0; i < C; ++i) {
    double acc = 0.0;
    for (int j = 0; j < d; ++j) acc += M[i * d + j] * f[(nz - d + j) * ips];
    for (int j = 0; j < d; ++j) acc += M[(C - 1 - i) * d + (d - 1 - j)] * f[j * ips];
    o[(nz + i) * ops] = acc;
  }
}

// ---------------------------------------------------------------- contiguous lines
// Points contiguous (in_ps = out_ps = 1): one wavefront per EXT_U lines at a
// time, lanes along the points, so that loads and stores are whole
// cache lines (a thread per line reads 64 lines at once, 8 bytes of each).
// Bound by memory: a line is read and written once.  The C continuation values
// are one lane each (rows i = lane of [M_r | M_l], held in registers across the
// lines for the d of the stored tables); the 2 d boundary points are loaded
// once, one per lane, and broadcast through scalar registers.
// 50001 lines of 193 + 25 points (164 MB; the cache holds 256), against the thread per
// line: eight pairs of buffers in turn 256 -> 49 us (3.4 TB/s; a large copy runs at
// 4.9), one pair again and again 163 -> 32; one call after 1 GiB of other reads 258 ->
// 41, of other writes, which have to leave the cache first, 290 -> 62.
constexpr int EXT_U = 4;
constexpr int EXT_NT = 256;

__device__ __forceinline__ double ext_lane(double v, int k) {
  typedef int i2 __attribute__((ext_vector_type(2)));
  i2 w = __builtin_bit_cast(i2, v);
  w.x = __builtin_amdgcn_readlane(w.x, k);
  w.y = __builtin_amdgcn_readlane(w.y, k);
  return __builtin_bit_cast(double, w);
}

// D: matching points (M_r, M_l rows in registers; C <= 64), or 0: any d, C
// with 2 d <= 64 (coefficients read from M)
template <int D>
__global__ __launch_bounds__(EXT_NT) void k_fc_extend_rows(
    const double* __restrict__ in, long long nlines, long long ils, double* __restrict__ out,
    long long ols, int nz, int C, int d, const double* __restrict__ M) {
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if constexpr (D > 0) d = D;
  auto coef = [&](int i, int k) {
    return k < d ? M[i * d + k] : M[(C - 1 - i) * d + (d - 1 - (k - d))];
  };
  double m[D > 0 ? 2 * D : 1];
  if constexpr (D > 0) {
    const int i = min(lane, C - 1);
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) m[k] = coef(i, k);
  }
  // lane k < 2 d holds boundary point k: the right end, then the left end
  const int bs = lane < d ? nz - d + lane : min(lane - d, d - 1);
  constexpr int WPB = EXT_NT / 64;
  for (long long g = (long long)blockIdx.x * WPB + wv; g * EXT_U < nlines;
       g += (long long)gridDim.x * WPB) {
    const double* f[EXT_U];
    double* o[EXT_U];
    double b[EXT_U];
    bool ok[EXT_U];
#pragma unroll
    for (int u = 0; u < EXT_U; ++u) {
      const long long l = g * EXT_U + u, lc = l < nlines ? l : nlines - 1;
      ok[u] = l < nlines;   // (a line past the end reads the last one, stores nothing)
      f[u] = in + lc * ils;
      o[u] = out + lc * ols;
      b[u] = f[u][bs];
    }
    for (int s = lane; s < nz; s += 64) {
      double t[EXT_U];
#pragma unroll
      for (int u = 0; u < EXT_U; ++u) t[u] = f[u][s];
#pragma unroll
      for (int u = 0; u < EXT_U; ++u)
        if (ok[u]) o[u][s] = t[u];
    }
    if constexpr (D > 0) {
#pragma unroll
      for (int u = 0; u < EXT_U; ++u) {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < 2 * D; ++k) acc += m[k] * ext_lane(b[u], k);
        if (ok[u] && lane < C) o[u][nz + lane] = acc;
      }
    } else {
      for (int i = lane; i - lane < C; i += 64) {
        const int ic = min(i, C - 1);
        double acc[EXT_U] = {};
        for (int k = 0; k < 2 * d; ++k) {
          const double c = coef(ic, k);
#pragma unroll
          for (int u = 0; u < EXT_U; ++u) acc[u] += c * ext_lane(b[u], k);
        }
#pragma unroll
        for (int u = 0; u < EXT_U; ++u)
          if (ok[u] && i < C) o[u][nz + i] = acc[u];
      }
    }
  }
}

// Contiguous points take the wavefront rows (2 d <= 64: a boundary point per
// lane); any other strides, and longer boundaries, one thread per line.
void launch_fc_extend(const double* in, long long nlines, long long ips, long long ils, double* out,
                      long long ops, long long ols, int nz, int C, int d, const double* M,
                      hipStream_t st) {
  if (ips == 1 && ops == 1 && 2 * d <= 64) {
    const long long per = EXT_U * (EXT_NT / 64);
    dim3 grid((unsigned)std::min<long long>((nlines + per - 1) / per, 4096));
    if (d == 5 && C <= 64)
      FCNS_LAUNCH(k_fc_extend_rows<5>, grid, dim3(EXT_NT), 0, st, in, nlines, ils, out, ols, nz,
                  C, d, M);
    else if (d == 7 && C <= 64)
      FCNS_LAUNCH(k_fc_extend_rows<7>, grid, dim3(EXT_NT), 0, st, in, nlines, ils, out, ols, nz,
                  C, d, M);
    else
      FCNS_LAUNCH(k_fc_extend_rows<0>, grid, dim3(EXT_NT), 0, st, in, nlines, ils, out, ols, nz,
                  C, d, M);
    return;
  }
  const int nt = 256;
  dim3 grid((unsigned)((nlines + nt - 1) / nt));
  FCNS_LAUNCH(k_fc_extend, grid, dim3(nt), 0, st, in, nlines, ips, ils, out, ops, ols, nz,
                     C, d, M);
}

}  // namespace fcns
