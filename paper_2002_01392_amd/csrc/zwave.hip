// Wall-normal (z) kernels for continued lengths N' = 32 K (K = 2..9), one
// wavefront per two pencils.
//
// A wavefront holds the whole continued line of its two pencils in registers,
// K rows per lane, and transforms it without workgroup barriers: a K-point DFT
// in the lane's registers and a 32-point DFT across the 32 lanes of the pencil
// by cross-lane moves (DPP and the gfx950 permlane swaps).  The waves of a
// workgroup never wait for each other, so one wave's loads and stores run
// under the others' arithmetic; the workgroup engine of zpass.hip (256
// threads, two LDS ping-pong buffers, a barrier per radix stage) holds two
// workgroups per CU in lock step and waits for latency between its phases.
//
// Rows.  N = 32 K, lane index j (0..31) of a pencil.  Natural order: register m
// holds row n = j + 32 m.  With k = r + K k2,
//   X[r + K k2] = sum_j w_32^{j k2} ( w_N^{j r} sum_m w_K^{m r} x[j + 32 m] ),
// so the forward transform is a K-point DFT over the registers, a twiddle per
// register, and a 32-point decimation-in-frequency transform over the lanes,
// which leaves k2 = bitrev(j) in lane j: register r holds coefficient
// l = r + K bitrev(j).  The inverse runs the same steps backwards (decimation
// in time from bit-reversed lanes) on data with real and imaginary part
// swapped, which turns the conjugated twiddles into the forward ones; the
// pointwise work in between does not care about the order, and a row of a
// field is one contiguous access of a lane pair either way.
//
// Lanes.  The five butterfly steps exchange with lane ^ 32, ^ 16 (permlane
// swaps), ^ 8, ^ 7 and ^ 3 (single DPP moves: row_ror:8, row_half_mirror,
// quad_perm).  These masks and 1 (the pencil) are a basis of the lane bits, so
// lane = p + ... is read as coordinates in it: b4 = bit 5, b3 = bit 4,
// b2 = bit 3, b1 = bit 2, b0 = bit 1 ^ bit 2, p = bit 0 ^ bit 1, j = b4..b0.
// Lanes 2 i and 2 i + 1 hold the same row of the two pencils.
#include "kernels.hpp"

namespace fcns {

constexpr int ZW_WAVES = 4;             // wavefronts per workgroup
constexpr int ZW_PPB = 2 * ZW_WAVES;    // pencils per workgroup
constexpr int ZW_MAXD = 6;              // matching points (the continuation's
                                        // boundary rows per end)

typedef unsigned zwu2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------- exchanges
template <int CTRL>
__device__ __forceinline__ double zw_dpp(double v) {
  zwu2 w = __builtin_bit_cast(zwu2, v);
  w.x = __builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xf, 0xf, true);
  w.y = __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, w);
}
template <int CTRL>
__device__ __forceinline__ float zw_dpp(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
constexpr int ZW_X3 = 0x1B;    // quad_perm [3,2,1,0]: lane ^ 3
constexpr int ZW_X7 = 0x141;   // row_half_mirror: lane ^ 7
constexpr int ZW_X8 = 0x128;   // row_ror:8: lane ^ 8
template <int CTRL, typename T>
__device__ __forceinline__ cpx<T> zw_dpp(cpx<T> a) {
  return mk(zw_dpp<CTRL>(a.x), zw_dpp<CTRL>(a.y));
}

// a's upper half (bit BIT of the lane set) exchanged with b's lower half: a
// becomes (a.lower, b.lower), b becomes (a.upper, b.upper).
template <int BIT>
__device__ __forceinline__ void zw_swap32(unsigned& a, unsigned& b) {
  if constexpr (BIT == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  }
}
template <int BIT>
__device__ __forceinline__ void zw_swap(double& a, double& b) {
  zwu2 x = __builtin_bit_cast(zwu2, a), y = __builtin_bit_cast(zwu2, b);
  unsigned x0 = x.x, x1 = x.y, y0 = y.x, y1 = y.y;
  zw_swap32<BIT>(x0, y0);
  zw_swap32<BIT>(x1, y1);
  x.x = x0;
  x.y = x1;
  y.x = y0;
  y.y = y1;
  a = __builtin_bit_cast(double, x);
  b = __builtin_bit_cast(double, y);
}
template <int BIT>
__device__ __forceinline__ void zw_swap(float& a, float& b) {
  unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
  zw_swap32<BIT>(x, y);
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}
template <int BIT, typename T>
__device__ __forceinline__ void zw_swap(cpx<T>& a, cpx<T>& b) {
  zw_swap<BIT>(a.x, b.x);
  zw_swap<BIT>(a.y, b.y);
}

// ---------------------------------------------------------------- K-point DFTs
// Odd prime P with constant roots, symmetric form (as CodeletOdd).
template <int P>
struct ZwRoots;
template <>
struct ZwRoots<5> {
  static constexpr double c[3] = {1.0, 0.30901699437494742410, -0.80901699437494742410};
  static constexpr double s[3] = {0.0, 0.95105651629515357212, 0.58778525229247312917};
};
template <>
struct ZwRoots<7> {
  static constexpr double c[4] = {1.0, 0.62348980185873353053, -0.22252093395631440429,
                                  -0.90096886790241912624};
  static constexpr double s[4] = {0.0, 0.78183148246802980871, 0.97492791218182360702,
                                  0.43388373911755812048};
};
template <typename T, int P>
__device__ __forceinline__ void zw_dft_odd(cpx<T>* v) {
  constexpr int H = (P - 1) / 2;
  cpx<T> a[H], b[H];
  const cpx<T> x0 = v[0];
  cpx<T> s = x0;
#pragma unroll
  for (int q = 1; q <= H; ++q) {
    a[q - 1] = v[q] + v[P - q];
    b[q - 1] = v[q] - v[P - q];
    s = s + a[q - 1];
  }
  v[0] = s;
#pragma unroll
  for (int k = 1; k <= H; ++k) {
    cpx<T> re = x0, im = zero<T>();
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      const int e = (q * k) % P, h = e <= H ? e : P - e;
      const double sn = e <= H ? ZwRoots<P>::s[h] : -ZwRoots<P>::s[h];
      re = re + a[q - 1] * (T)ZwRoots<P>::c[h];
      im = im + b[q - 1] * (T)sn;
    }
    v[k] = re + mul_mi(im);
    v[P - k] = re + mul_i(im);
  }
}

template <typename T, int K>
__device__ __forceinline__ void zw_dft(cpx<T> (&v)[K]) {
  if constexpr (K == 2 || K == 4 || K == 8) {
    Codelet<T, K>::run(v, nullptr);
  } else if constexpr (K == 3) {
    dft3_reg<T>(v[0], v[1], v[2]);
  } else if constexpr (K == 6) {
    dft6_reg<T>(v);
  } else if constexpr (K == 5 || K == 7) {
    zw_dft_odd<T, K>(v);
  } else {
    // 9 = 3 x 3: n = 3 a + b, k = c + 3 e; DFTs over a, twiddles w9^(b c),
    // DFTs over b
    static_assert(K == 9, "K = 2..9");
    constexpr double c1 = 0.76604444311897803520, s1 = 0.64278760968653932632;
    constexpr double c2 = 0.17364817766693034885, s2 = 0.98480775301220805937;
    constexpr double c4 = -0.93969262078590838405, s4 = 0.34202014332566873304;
#pragma unroll
    for (int b = 0; b < 3; ++b) dft3_reg<T>(v[b], v[3 + b], v[6 + b]);
    v[4] = rot(v[4], c1, s1);
    v[5] = rot(v[5], c2, s2);
    v[7] = rot(v[7], c2, s2);
    v[8] = rot(v[8], c4, s4);
#pragma unroll
    for (int c = 0; c < 3; ++c) dft3_reg<T>(v[3 * c], v[3 * c + 1], v[3 * c + 2]);
    // v[3 c + e] = X[c + 3 e]
    cpx<T> t;
    t = v[1]; v[1] = v[3]; v[3] = t;
    t = v[2]; v[2] = v[6]; v[6] = t;
    t = v[5]; v[5] = v[7]; v[7] = t;
  }
}

// ---------------------------------------------------------------- the wave's view
// Twiddles of the lane steps (per lane): w16, w8 for the swap steps (applied
// to a butterfly's difference, whichever register it belongs to), and for the
// DPP steps the factor of this lane's own result (1 in the lower half).
template <typename T>
struct ZwLane {
  cpx<T> w32, w16, w8, w4;
  T s8, s7, s3;   // +1 in the lower, -1 in the upper half of the step
  bool u32, u16;  // upper half of the swap steps
};

struct ZwIdx {
  int j, k2;          // lane index in the pencil, bitrev(j)
  int p;              // pencil
  bool pv;            // not kx padding
};

__device__ __forceinline__ void zw_lanes(ZwIdx& q) {
  const int lane = threadIdx.x & 63;
  const int b1 = (lane >> 2) & 1, b0 = ((lane >> 1) ^ (lane >> 2)) & 1;
  q.j = ((lane >> 3) << 2) | (b1 << 1) | b0;
  q.k2 = (int)(__builtin_bitreverse32((unsigned)q.j) >> 27);
}
// which of the wave's two pencils
__device__ __forceinline__ int zw_pencil() {
  const int lane = threadIdx.x & 63;
  return (lane ^ (lane >> 1)) & 1;
}

// rt: the N' roots exp(-2 pi i q / N') in FP64
template <typename T, int K>
__device__ __forceinline__ ZwLane<T> zw_lane(const cpx<double>* rt, int j) {
  ZwLane<T> w;
  const cpx<T> one = mk(T(1), T(0));
  w.w32 = cvt<T>(rt[K * (j & 15)]);
  w.w16 = cvt<T>(rt[2 * K * (j & 7)]);
  w.u32 = j & 16;
  w.u16 = j & 8;
  const cpx<T> a = cvt<T>(rt[4 * K * (j & 3)]), b = cvt<T>(rt[8 * K * (j & 1)]);
  w.w8 = (j & 4) ? a : one;
  w.w4 = (j & 2) ? b : one;
  w.s8 = (j & 4) ? T(-1) : T(1);
  w.s7 = (j & 2) ? T(-1) : T(1);
  w.s3 = (j & 1) ? T(-1) : T(1);
  return w;
}

// The wave's tables in LDS, shared by the workgroup (read-only after the
// barrier of zw_tables): register twiddles tw[(r - 1) * 32 + j] = w_N^(j r),
// the continuation's coefficients M[k * 32 + j] of row 32 (K - 1) + j on the 2 d
// boundary rows (right end first; zero rows below nz), the roots of the N'
// transform and the filter factors; bnd is a wave's own exchange buffer.
template <typename T, int K>
struct ZwLds {
  cpx<T>* tw;
  double* M;
  cpx<T>* bnd;
};

template <typename T, int K>
struct ZwShared {
  cpx<T> tw[(K - 1) * 32];
  double M[2 * ZW_MAXD * 32];
  cpx<T> bnd[ZW_WAVES][2 * ZW_MAXD * 2];
};

template <typename T, int K>
__device__ __forceinline__ void zw_tables(ZwShared<T, K>& sh, const ZArgs& a, bool ext) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const Geom& g = a.g;
  for (int e = tid; e < (K - 1) * 32; e += nt)
    sh.tw[e] = cvt<T>(a.tw64[(e / 32 + 1) * (e % 32)]);
  if (ext) {
    const int d = g.d, C = g.C;
    for (int e = tid; e < 2 * d * 32; e += nt) {
      const int k = e / 32, i = 32 * (K - 1) + e % 32 - g.nz;
      double m = 0.0;
      if (i >= 0) m = k < d ? a.fc[i * d + k] : a.fc[(C - 1 - i) * d + (d - 1 - (k - d))];
      sh.M[e] = m;
    }
  }
  __syncthreads();
}

__device__ __forceinline__ void zw_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- lane steps
// One swap step (distance 16 or 8 in j) over pairs of registers: after the
// swap one lane holds both ends of a butterfly of register r (lower lanes)
// or r + 1 (upper lanes).
template <int BIT, bool DIF, typename T, int K>
__device__ __forceinline__ void zw_step_swap(cpx<T> (&x)[K], cpx<T> w, bool up) {
#pragma unroll
  for (int r = 0; r + 1 < K; r += 2) {
    cpx<T> a = x[r], b = x[r + 1];
    zw_swap<BIT>(a, b);
    cpx<T> s, d;
    if constexpr (DIF) {
      s = a + b;
      d = (a - b) * w;
    } else {
      b = b * w;
      s = a + b;
      d = a - b;
    }
    zw_swap<BIT>(s, d);
    x[r] = s;
    x[r + 1] = d;
  }
  if constexpr (K % 2 == 1) {
    cpx<T> a = x[K - 1], b = a;
    zw_swap<BIT>(a, b);
    if constexpr (DIF) {
      const cpx<T> s = a + b, d = (a - b) * w;
      x[K - 1] = mk(up ? d.x : s.x, up ? d.y : s.y);
    } else {
      b = b * w;
      const T sg = up ? T(-1) : T(1);
      x[K - 1] = mk(a.x + sg * b.x, a.y + sg * b.y);
    }
  }
}

// One DPP step (distance 4, 2 or 1 in j); TW: with a twiddle.
template <int CTRL, bool DIF, bool TW, typename T, int K>
__device__ __forceinline__ void zw_step_dpp(cpx<T> (&x)[K], cpx<T> w, T s) {
#pragma unroll
  for (int r = 0; r < K; ++r) {
    cpx<T> v = x[r];
    if constexpr (TW && !DIF) v = v * w;
    const cpx<T> q = zw_dpp<CTRL>(v);
    v = mk(q.x + s * v.x, q.y + s * v.y);
    if constexpr (TW && DIF) v = v * w;
    x[r] = v;
  }
}

// Scheduling boundary between the phases of a transform: twiddle and row loads
// hoisted across it would only add live registers.
__device__ __forceinline__ void zw_phase() { __builtin_amdgcn_sched_barrier(0); }

// Forward transform, natural rows -> coefficients l = r + K bitrev(j).
template <typename T, int K>
__device__ __forceinline__ void zw_fft(cpx<T> (&x)[K], const ZwLane<T>& w, const cpx<T>* tw,
                                       int j) {
  zw_phase();
  zw_dft<T, K>(x);
#pragma unroll
  for (int r = 1; r < K; ++r) x[r] = x[r] * tw[(r - 1) * 32 + j];
  zw_phase();
  zw_step_swap<32, true>(x, w.w32, w.u32);
  zw_step_swap<16, true>(x, w.w16, w.u16);
  zw_phase();
  zw_step_dpp<ZW_X8, true, true>(x, w.w8, w.s8);
  zw_step_dpp<ZW_X7, true, true>(x, w.w4, w.s7);
  zw_step_dpp<ZW_X3, true, false>(x, w.w4, w.s3);
  zw_phase();
}

// Unnormalised inverse transform, coefficients -> natural rows.
template <typename T, int K>
__device__ __forceinline__ void zw_ifft(cpx<T> (&x)[K], const ZwLane<T>& w, const cpx<T>* tw,
                                        int j) {
  zw_phase();
#pragma unroll
  for (int r = 0; r < K; ++r) x[r] = mk(x[r].y, x[r].x);
  zw_step_dpp<ZW_X3, false, false>(x, w.w4, w.s3);
  zw_step_dpp<ZW_X7, false, true>(x, w.w4, w.s7);
  zw_step_dpp<ZW_X8, false, true>(x, w.w8, w.s8);
  zw_phase();
  zw_step_swap<16, false>(x, w.w16, w.u16);
  zw_step_swap<32, false>(x, w.w32, w.u32);
  zw_phase();
#pragma unroll
  for (int r = 1; r < K; ++r) x[r] = x[r] * tw[(r - 1) * 32 + j];
  zw_dft<T, K>(x);
  zw_phase();
#pragma unroll
  for (int r = 0; r < K; ++r) x[r] = mk(x[r].y, x[r].x);
}

// Continuation rows nz..N'-1 of the line (Sec. 3; M_l = J M_r J): all of them
// are in the last register (C <= 32).  The 2 d boundary rows go through the
// wave's LDS buffer and are read back as broadcasts.
template <int K>
__device__ __forceinline__ void zw_extend(cpx<double> (&x)[K], const Geom& g, const double* M,
                                          cpx<double>* bnd, int j, int pen) {
  const int d = g.d, r0 = g.nz - d;
  if (j < d) bnd[2 * (d + j) + pen] = x[0];
#pragma unroll
  for (int m = (K > 2 ? K - 2 : 0); m < K; ++m) {
    const int n = j + 32 * m;
    if (n >= r0 && n < g.nz) bnd[2 * (n - r0) + pen] = x[m];
  }
  zw_sync();
  double ar = 0.0, ai = 0.0;
  for (int k = 0; k < 2 * d; ++k) {
    const double c = M[k * 32 + j];
    const cpx<double> b = bnd[2 * k + pen];
    ar += c * b.x;
    ai += c * b.y;
  }
  zw_sync();
  if (j + 32 * (K - 1) >= g.nz) x[K - 1] = mk(ar, ai);
}

// A fresh copy of the lane's indices: what is derived from them is recomputed
// in each phase instead of being kept in registers across all of them.
__device__ __forceinline__ ZwIdx zw_fresh(ZwIdx q) {
  asm volatile("" : "+v"(q.j), "+v"(q.k2), "+v"(q.p));
  return q;
}

// ---------------------------------------------------------------- derivative of lines
// fc_derivative: two real lines per complex line (the multipliers i k~z and
// -kz^2 map real lines to real lines), four lines per wavefront; both
// transforms and the continuation stay in registers, so a line is read and
// written once and nothing waits at a barrier in between.  65537 lines of 257
// points (N' = 288): 128 -> 76 us per call on changing inputs (3.5 TB/s of the
// 269 MB it moves; a large copy takes 54 us) against the workgroup engine.
template <int K>
__global__ __launch_bounds__(64 * ZW_WAVES) void k_zw_deriv(ZArgs a,
                                                            const double* __restrict__ in,
                                                            double* __restrict__ out,
                                                            long long nlines, long long ls,
                                                            int order) {
  constexpr int N = 32 * K;
  __shared__ ZwShared<double, K> sh;
  zw_tables<double, K>(sh, a, true);
  const Geom& g = a.g;
  ZwIdx q{};
  zw_lanes(q);
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int pen = zw_pencil();
  const ZwLane<double> w = zw_lane<double, K>(a.tw64, q.j);
  const long long ngrp = (nlines + 2 * ZW_PPB - 1) / (2 * ZW_PPB);
  for (long long grp = blockIdx.x; grp < ngrp; grp += gridDim.x) {
    q = zw_fresh(q);
    const long long l0 = 2 * (grp * ZW_PPB + 2 * wv + pen), l1 = l0 + 1;
    // (a line past the end reads the last one and stores nothing)
    const double* fa = in + (l0 < nlines ? l0 : nlines - 1) * ls;
    const double* fb = in + (l1 < nlines ? l1 : nlines - 1) * ls;
    cpx<double> x[K];
#pragma unroll
    for (int m = 0; m < K; ++m) {
      const int n = m < K - 1 ? q.j + 32 * m : min(q.j + 32 * m, g.nz - 1);
      x[m] = mk(fa[n], fb[n]);
    }
    zw_extend<K>(x, g, sh.M, sh.bnd[wv], q.j, pen);
    zw_fft<double, K>(x, w, sh.tw, q.j);
    q = zw_fresh(q);
#pragma unroll
    for (int r = 0; r < K; ++r) {
      const int l = r + K * q.k2;
      if (order == 1) {
        x[r] = mul_i(x[r]) * k_odd(l, N, g.kzs);
      } else {
        const double k = k_true(l, N, g.kzs);
        x[r] = x[r] * (-k * k);
      }
    }
    zw_ifft<double, K>(x, w, sh.tw, q.j);
    const double inv = 1.0 / N;
    double* oa = out + l0 * ls;
    double* ob = out + l1 * ls;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      const int z = q.j + 32 * m;
      if (m < K - 1 || z < g.nz) {
        if (l0 < nlines) oa[z] = x[m].x * inv;
        if (l1 < nlines) ob[z] = x[m].y * inv;
      }
    }
  }
}

// ---------------------------------------------------------------- launchers
// N' = 32 K, K = 2..9; the continuation in one register (C <= 32), at most
// ZW_MAXD matching points.
static bool zw_lines_fit(const ZArgs& a) {
  const Geom& g = a.g;
  return g.npr % 32 == 0 && g.npr >= 64 && g.npr <= 288 && g.C <= 32 && g.d <= ZW_MAXD &&
         a.tw64;
}
#define FCNS_ZW_SWITCH(KV, CALL)                \
  switch (KV) {                                 \
    case 2: { constexpr int K = 2; CALL; } break; \
    case 3: { constexpr int K = 3; CALL; } break; \
    case 4: { constexpr int K = 4; CALL; } break; \
    case 5: { constexpr int K = 5; CALL; } break; \
    case 6: { constexpr int K = 6; CALL; } break; \
    case 7: { constexpr int K = 7; CALL; } break; \
    case 8: { constexpr int K = 8; CALL; } break; \
    default: { constexpr int K = 9; CALL; } break; \
  }

// Contiguous points only: with the line index fastest a wave's accesses would
// be 32 bytes wide, and the workgroup engine's 128 are better.
bool zw_deriv_fits(const ZArgs& a, long long ps) { return zw_lines_fit(a) && ps == 1; }

void launch_zw_deriv(const ZArgs& a, const double* in, double* out, long long nlines,
                     long long ls, int order, hipStream_t st) {
  // 4 workgroups per CU are resident: whole rounds of groups over them
  const long long grp = (nlines + 2 * ZW_PPB - 1) / (2 * ZW_PPB);
  const long long rounds = (grp + 1023) / 1024;
  dim3 grid((unsigned)((grp + rounds - 1) / rounds));
  FCNS_ZW_SWITCH(a.g.npr / 32, hipLaunchKernelGGL(k_zw_deriv<K>, grid, dim3(64 * ZW_WAVES), 0, st,
                                                  a, in, out, nlines, ls, order))
}

}  // namespace fcns
