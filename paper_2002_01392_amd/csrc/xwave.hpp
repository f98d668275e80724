// Transforms of rows of N points by wavefronts (x direction), shared by the x
// kernels.
#pragma once
#include "kernels.hpp"

namespace fcns {

// ---------------------------------------------------------------- x pass, wave-level rows
// Rows of N = 512, 256, 192, 128, 96, 64 or 32 points with 8 points per
// lane: a row occupies S = N / 8 lanes (one row per wavefront at 512, two at
// 256 and 192, four at 128, five at 96, eight at 64, sixteen at 32), and
// lane t of a row (t < S) holds index t + S m (m = 0..7) of every
// transform, in and out.
//
// N = 512 = 8 x 8 x 8: n = n0 + 8 n1 + 64 n2, k = k0 + 8 k1 + 64 k2 (t = n0 + 8 n1):
//   a radix-8 DFT over n2 in registers, twiddle w64^(n1 k0);
//   exchange so that lane n0 + 8 k0 holds n1 = 0..7, radix-8 over n1,
//   twiddle w512^(n0 (k0 + 8 k1));
//   exchange so that lane k0 + 8 k1 holds n0 = 0..7, radix-8 over n0,
// which leaves X[t + 64 k2] in lane t.
// N = 256 = 8 x 32: n = t + 32 m, k = a + 8 b:
//   a radix-8 DFT over m in registers, twiddle w256^(t a);
//   the eight 32-point DFTs over t = t0 + 4 t1 (b = j1 + 8 j0): exchange so
//   that lane t0 + 4 a holds t1 = 0..7, radix-8 over t1, twiddle w32^(t0 j1);
//   exchange so that lane L holds t0 = 0..3 of c = a + 8 j1 = L and L + 32,
//   two radix-4 DFTs over t0,
// which leaves X[c + 64 j0] = X[L + 32 (h + 2 j0)] (c = L + 32 h) in lane L.
// N = 128 = 8 x 16: n = t + 16 m, k = a + 8 b:
//   a radix-8 DFT over m in registers, twiddle w128^(t a);
//   the eight 16-point DFTs over t = h + 2 t1 (b = j + 8 c): exchange so that
//   lane 2 a + h holds t1 = 0..7, radix-8 over t1, twiddle w16^(h j);
//   exchange so that lane a + 8 j0 holds, for j = j0 + 2 j1 (j1 = 0..3),
//   both halves h of output j, and a radix-2 DFT over h,
// which leaves X[a + 8 j + 64 c] = X[L + 16 (j1 + 4 c)] in lane L.
// N = 64 = 8 x 8: a radix-8 DFT over m, twiddle w64^(t a), one exchange so
// that lane a holds t = 0..7, radix-8 over t: X[a + 8 b] in lane a.
// N = 32 = 8 x 4: a radix-8 DFT over m, twiddle w32^(t a), one exchange so
// that lane L holds t = 0..3 of a = 2L and 2L + 1, two radix-4 DFTs, and a
// last exchange into natural order.
// N = 192 = 8 x 24 and 96 = 8 x 12 (S = 24, 12 lanes; 2 and 5 rows per
// wavefront, the 64 mod S spare lanes repeat a row's last lanes and store
// nothing): a radix-8 DFT over m, twiddle wN^(t a); the S-point DFTs over
// t = h + 3 t1 (b = j + (S/3) c): exchange so that a lane holds, for its
// (a, h), t1 = 0..S/3-1 (at 96 two values of a per lane), radix-8 (192) or
// two radix-4 (96) DFTs over t1, twiddle wS^(h j); exchange, radix-3 DFTs
// over h (X[a + 8 j + (8 S/3) c], c = 0..2) spread over the lanes, and a
// last exchange into natural order.
// The exchanges go through a padded per-row LDS buffer (conflict-free
// 16-byte accesses) and need only wave-level ordering, no workgroup barrier.
// Two real transforms share one complex transform: z = a + i b (inverse from
// the spectra A, B; forward of two nonlinear terms).
constexpr int XW_WAVES = 4;        // waves per workgroup
constexpr int XW_BUF = 512 + 64;   // padded slots of one wave's exchange buffer(s)

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A place in an LDS array, kept as the array and one index: where direct loads are
// in flight into another array, an access through a longer chain of pointers is
// no longer known to be of this one, and would wait for them.
template <typename T>
struct XwBuf {
  cpx<T>* base;
  int o;
  __device__ __forceinline__ XwBuf operator+(int i) const { return {base, o + i}; }
  __device__ __forceinline__ cpx<T>& operator[](int i) const { return base[o + i]; }
  __device__ __forceinline__ operator cpx<T>*() const { return base + o; }
};

// Padded slots, written with the per-lane part separate so that the
// per-register part is an instruction offset.  N = 512: element
// 64 n0 + 8 k0 + n1 of exchange 1 sits at 65 n0 + 8 k0 + n1, element
// 8 j + n0 of exchange 2 at 9 j + n0.  N = 256: element (a, t) of exchange 1
// at 36 a + t, element (c, t0) of exchange 2 at 4 c + c / 4 + t0.  Both: element
// i of the natural-order buffer at i + i / 8.
__device__ __forceinline__ int xw_nat(int i) { return i + (i >> 3); }

// Per-lane twiddles, stored [register][t] in LDS (read at t + offset).
// N = 512: tw[k0 - 1][t] = w64^(n1 k0) (k0 = 1..7) with t = n0 + 8 n1, and
// tw[7 + k1][t] = w512^(n0 (k0' + 8 k1)) with t = n0 + 8 k0'.
// N = 256: tw[a - 1][t] = w256^(t a) (a = 1..7), tw[6 + j1][t] = w32^(t0 j1)
// (j1 = 1..7) with t = t0 + 4 a.  N = 128: tw[a - 1][t] = w128^(t a),
// tw[6 + j][L] = w16^(h j) with h = L & 1.  N = 64: tw[a - 1][t] = w64^(t a).
// N = 192, 96: tw[a - 1][t] = wN^(t a), tw[6 + j][L] = w(N/8)^(h j) with
// h = L mod 3.  N = 32: tw[a - 1][t] = w32^(t a).
constexpr int XW_TW = 15 * 64;

template <typename T, int N, int NT = 64 * XW_WAVES>   // NT threads
__device__ __forceinline__ void xw_twiddles(cpx<T>* tw, int tid) {
  constexpr int S = N / 8, NTW = (N == 512 ? 15 : N <= 64 ? 7 : 14) * S;
  static_assert(NTW <= XW_TW, "twiddle table");
  for (int e = tid; e < NTW; e += NT) {
    const int reg = e / S, t = e % S;
    int j;  // power of wN
    if (N == 512)
      j = reg < 7 ? 8 * (t >> 3) * (reg + 1) : (t & 7) * ((t >> 3) + 8 * (reg - 7));
    else if (N == 256)
      j = reg < 7 ? t * (reg + 1) : 8 * (t & 3) * (reg - 6);
    else if (N == 128)   // tw[6 + j][L] = w16^(h j), h = L & 1
      j = reg < 7 ? t * (reg + 1) : 8 * (t & 1) * (reg - 6);
    else if (N == 192 || N == 96)   // tw[6 + j][L] = w(N/8)^(h j), h = L mod 3
      j = reg < 7 ? t * (reg + 1) : 8 * (t % 3) * (reg - 6);
    else
      j = reg < 7 ? t * (reg + 1) : 0;
    double sn, cs;
    sincospi(2.0 * j / N, &sn, &cs);
    tw[e] = mk((T)cs, (T)(-sn));   // exp(-2 pi i j / N)
  }
}

template <typename T, typename B>
__device__ __forceinline__ void wave_fft512(cpx<T> (&r)[8], B buf,
                                            const cpx<T>* __restrict__ tw, int lane) {
  const int n0 = lane & 7, hi = lane >> 3;  // hi = n1 before, k0 after exchange 1
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int k0 = 1; k0 < 8; ++k0) r[k0] = r[k0] * tw[(k0 - 1) * 64 + lane];
  cpx<T>* w1 = buf + 65 * n0 + hi;
#pragma unroll
  for (int k0 = 0; k0 < 8; ++k0) w1[8 * k0] = r[k0];
  wave_sync();
  const cpx<T>* r1 = buf + 65 * n0 + 8 * hi;
#pragma unroll
  for (int n1 = 0; n1 < 8; ++n1) r[n1] = r1[n1];
  wave_sync();
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int k1 = 0; k1 < 8; ++k1) r[k1] = r[k1] * tw[(7 + k1) * 64 + lane];
  cpx<T>* w2 = buf + 9 * hi + n0;
#pragma unroll
  for (int k1 = 0; k1 < 8; ++k1) w2[72 * k1] = r[k1];
  wave_sync();
  const cpx<T>* r2 = buf + 9 * lane;
#pragma unroll
  for (int q = 0; q < 8; ++q) r[q] = r2[q];
  wave_sync();
  Codelet<T, 8>::run(r, nullptr);
}

template <typename T, typename B>
__device__ __forceinline__ void wave_fft256(cpx<T> (&r)[8], B buf,
                                            const cpx<T>* __restrict__ tw, int t) {
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int a = 1; a < 8; ++a) r[a] = r[a] * tw[(a - 1) * 32 + t];
  cpx<T>* w1 = buf + t;
#pragma unroll
  for (int a = 0; a < 8; ++a) w1[36 * a] = r[a];
  wave_sync();
  const int t0 = t & 3, a = t >> 2;  // the lane's (t0, a) after exchange 1
  const cpx<T>* r1 = buf + 36 * a + t0;
#pragma unroll
  for (int t1 = 0; t1 < 8; ++t1) r[t1] = r1[4 * t1];
  wave_sync();
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int j1 = 1; j1 < 8; ++j1) r[j1] = r[j1] * tw[(6 + j1) * 32 + t];
  // c = a + 8 j1: 4 c + c / 4 + t0 = (4 a + a / 4 + t0) + 34 j1
  cpx<T>* w2 = buf + 4 * a + (a >> 2) + t0;
#pragma unroll
  for (int j1 = 0; j1 < 8; ++j1) w2[34 * j1] = r[j1];
  wave_sync();
  // c = t + 32 h: 4 c + c / 4 = (4 t + t / 4) + 136 h
  const cpx<T>* r2 = buf + 4 * t + (t >> 2);
  cpx<T> q[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) q[i] = r2[136 * (i >> 2) + (i & 3)];
  wave_sync();
  dft4_reg<T>(q[0], q[1], q[2], q[3]);
  dft4_reg<T>(q[4], q[5], q[6], q[7]);
  // q[4 h + j0] = X[t + 32 (h + 2 j0)]
#pragma unroll
  for (int m = 0; m < 8; ++m) r[m] = q[4 * (m & 1) + (m >> 1)];
}

template <typename T, typename B>
__device__ __forceinline__ void wave_fft128(cpx<T> (&r)[8], B buf,
                                            const cpx<T>* __restrict__ tw, int t) {
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int a = 1; a < 8; ++a) r[a] = r[a] * tw[(a - 1) * 16 + t];
  // exchange 1: element (a, t) at 17 a + t
  cpx<T>* w1 = buf + t;
#pragma unroll
  for (int a = 0; a < 8; ++a) w1[17 * a] = r[a];
  wave_sync();
  const int a = t >> 1, h = t & 1;  // the lane's (a, h) after exchange 1
  const cpx<T>* r1 = buf + 17 * a + h;
#pragma unroll
  for (int t1 = 0; t1 < 8; ++t1) r[t1] = r1[2 * t1];
  wave_sync();
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int j = 1; j < 8; ++j) r[j] = r[j] * tw[(6 + j) * 16 + t];
  // exchange 2: output j of lane L = 2 a + h at 9 L + j
  cpx<T>* w2 = buf + 9 * t;
#pragma unroll
  for (int j = 0; j < 8; ++j) w2[j] = r[j];
  wave_sync();
  const int a2 = t & 7, j0 = t >> 3;
  const cpx<T>* r2 = buf + 18 * a2 + j0;
#pragma unroll
  for (int j1 = 0; j1 < 4; ++j1) {
    const cpx<T> p0 = r2[2 * j1], p1 = r2[9 + 2 * j1];
    r[j1] = p0 + p1;
    r[j1 + 4] = p0 - p1;
  }
  wave_sync();
}

template <typename T, typename B>
__device__ __forceinline__ void wave_fft64(cpx<T> (&r)[8], B buf,
                                           const cpx<T>* __restrict__ tw, int t) {
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int a = 1; a < 8; ++a) r[a] = r[a] * tw[(a - 1) * 8 + t];
  // element (a, t) at 9 a + t; lane a then reads t = 0..7
  cpx<T>* w1 = buf + t;
#pragma unroll
  for (int a = 0; a < 8; ++a) w1[9 * a] = r[a];
  wave_sync();
  const cpx<T>* r1 = buf + 9 * t;
#pragma unroll
  for (int t1 = 0; t1 < 8; ++t1) r[t1] = r1[t1];
  wave_sync();
  Codelet<T, 8>::run(r, nullptr);
}

// Outputs of the N = 192 and 96 transforms: P_h[a][j] (twiddled) sits at
// PS h + b, b = a + 8 j < Q = 8 S / 3; lane t takes the radix-3 DFTs over h
// of b = t, t + S, ... (< Q), X[b + Q c] for c = 0, 1, 2, writes them in
// natural order (slots xw_nat), and reads back its own X[t + S m].
template <typename T, int S, int PS, typename B>
__device__ __forceinline__ void xw_radix3_out(cpx<T> (&r)[8], B buf,
                                              int t) {
  constexpr int Q = 8 * S / 3;          // radix-3 DFTs per row (64 at 192, 32 at 96)
  constexpr int NB = (Q + S - 1) / S;   // per lane, the last one partial
  const T s3 = T(0.86602540378443864676);  // sqrt(3) / 2
  cpx<T> o[3 * NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = t + S * i;
    if (b < Q) {
      const cpx<T> p0 = buf[b], p1 = buf[PS + b], p2 = buf[2 * PS + b];
      const cpx<T> sm = p1 + p2, df = p1 - p2;
      const cpx<T> e = mul_i(df) * s3;
      const cpx<T> base = p0 - sm * T(0.5);
      o[3 * i] = p0 + sm;
      o[3 * i + 1] = base - e;   // w3 = -1/2 - i sqrt(3)/2
      o[3 * i + 2] = base + e;
    }
  }
  wave_sync();
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = t + S * i;
    if (b < Q) {
#pragma unroll
      for (int c = 0; c < 3; ++c) buf[xw_nat(b + Q * c)] = o[3 * i + c];
    }
  }
  wave_sync();
#pragma unroll
  for (int m = 0; m < 8; ++m) r[m] = buf[xw_nat(t + S * m)];
}

template <typename T, typename B>
__device__ __forceinline__ void wave_fft192(cpx<T> (&r)[8], B buf,
                                            const cpx<T>* __restrict__ tw, int t) {
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int a = 1; a < 8; ++a) r[a] = r[a] * tw[(a - 1) * 24 + t];
  // exchange 1: element (a, t) at 25 a + t; lane 3 a + h reads t = h + 3 t1
  cpx<T>* w1 = buf + t;
#pragma unroll
  for (int a = 0; a < 8; ++a) w1[25 * a] = r[a];
  wave_sync();
  const int a = t / 3, h = t - 3 * a;
  const cpx<T>* r1 = buf + 25 * a + h;
#pragma unroll
  for (int t1 = 0; t1 < 8; ++t1) r[t1] = r1[3 * t1];
  wave_sync();
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int j = 1; j < 8; ++j) r[j] = r[j] * tw[(6 + j) * 24 + t];
  // exchange 2: P_h[a][j] at 65 h + a + 8 j
  cpx<T>* w2 = buf + 65 * h + a;
#pragma unroll
  for (int j = 0; j < 8; ++j) w2[8 * j] = r[j];
  wave_sync();
  xw_radix3_out<T, 24, 65>(r, buf, t);
  wave_sync();
}

template <typename T, typename B>
__device__ __forceinline__ void wave_fft96(cpx<T> (&r)[8], B buf,
                                           const cpx<T>* __restrict__ tw, int t) {
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int a = 1; a < 8; ++a) r[a] = r[a] * tw[(a - 1) * 12 + t];
  // exchange 1: element (a, t) at 13 a + t; lane 3 ap + h reads t = h + 3 t1
  // of a = 2 ap (registers 0..3) and 2 ap + 1 (registers 4..7)
  cpx<T>* w1 = buf + t;
#pragma unroll
  for (int a = 0; a < 8; ++a) w1[13 * a] = r[a];
  wave_sync();
  const int ap = t / 3, h = t - 3 * ap;
  const cpx<T>* r1 = buf + 26 * ap + h;
#pragma unroll
  for (int t1 = 0; t1 < 4; ++t1) {
    r[t1] = r1[3 * t1];
    r[4 + t1] = r1[13 + 3 * t1];
  }
  wave_sync();
  dft4_reg(r[0], r[1], r[2], r[3]);
  dft4_reg(r[4], r[5], r[6], r[7]);
#pragma unroll
  for (int j = 1; j < 4; ++j) {
    const cpx<T> f = tw[(6 + j) * 12 + t];
    r[j] = r[j] * f;
    r[4 + j] = r[4 + j] * f;
  }
  // exchange 2: P_h[a][j] at 33 h + a + 8 j
  cpx<T>* w2 = buf + 33 * h + 2 * ap;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    w2[8 * j] = r[j];
    w2[8 * j + 1] = r[4 + j];
  }
  wave_sync();
  xw_radix3_out<T, 12, 33>(r, buf, t);
  wave_sync();
}

template <typename T, typename B>
__device__ __forceinline__ void wave_fft32(cpx<T> (&r)[8], B buf,
                                           const cpx<T>* __restrict__ tw, int t) {
  Codelet<T, 8>::run(r, nullptr);
#pragma unroll
  for (int a = 1; a < 8; ++a) r[a] = r[a] * tw[(a - 1) * 4 + t];
  // element (a, t) at 4 a + t; lane L reads a = 2L (registers 0..3) and
  // 2L + 1 (registers 4..7)
  cpx<T>* w1 = buf + t;
#pragma unroll
  for (int a = 0; a < 8; ++a) w1[4 * a] = r[a];
  wave_sync();
  const cpx<T>* r1 = buf + 8 * t;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = r1[i];
  wave_sync();
  dft4_reg(r[0], r[1], r[2], r[3]);
  dft4_reg(r[4], r[5], r[6], r[7]);
  // X[2L + 8 b] and X[2L + 1 + 8 b] into natural order, then X[t + 4 m]
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    buf[xw_nat(2 * t + 8 * b)] = r[b];
    buf[xw_nat(2 * t + 1 + 8 * b)] = r[4 + b];
  }
  wave_sync();
#pragma unroll
  for (int m = 0; m < 8; ++m) r[m] = buf[xw_nat(t + 4 * m)];
  wave_sync();
}

template <typename T, int N, typename B>
__device__ __forceinline__ void wave_fft(cpx<T> (&r)[8], B buf,
                                         const cpx<T>* __restrict__ tw, int t) {
  if constexpr (N == 512)
    wave_fft512<T>(r, buf, tw, t);
  else if constexpr (N == 256)
    wave_fft256<T>(r, buf, tw, t);
  else if constexpr (N == 192)
    wave_fft192<T>(r, buf, tw, t);
  else if constexpr (N == 128)
    wave_fft128<T>(r, buf, tw, t);
  else if constexpr (N == 96)
    wave_fft96<T>(r, buf, tw, t);
  else if constexpr (N == 64)
    wave_fft64<T>(r, buf, tw, t);
  else
    wave_fft32<T>(r, buf, tw, t);
}

}  // namespace fcns
