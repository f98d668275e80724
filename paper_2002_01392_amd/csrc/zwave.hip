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
constexpr int ZW_MAXD = 7;              // matching points (the continuation's
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
// Twiddles of the lane steps (per lane): w32, w16 for the swap steps (applied
// to a butterfly's difference, whichever register it belongs to), and for the
// DPP steps the factor of this lane's own result (1 in the lower half).
template <typename T>
struct ZwLane {
  cpx<T> w32, w16, w8, w4;
  T s8, s7, s3;   // +1 in the lower, -1 in the upper half of the step
  bool u32, u16;  // upper half of the swap steps
};

// 1 / a (a normal, positive): the hardware estimate and two Newton steps, in half
// the instructions of the IEEE division.  With an estimate within 2^-22 the result
// was the division's in each of 5e7 random trials on the CPU.
__device__ __forceinline__ double zw_rcp(double a) {
  double r = __builtin_amdgcn_rcp(a);
  r = fma(fma(-a, r, 1.0), r, r);
  return fma(fma(-a, r, 1.0), r, r);
}

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

__device__ __forceinline__ ZwIdx zw_index(const Geom& g, int p0) {
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  ZwIdx q;
  zw_lanes(q);
  q.p = p0 + 2 * wv + zw_pencil();
  q.pv = q.p % g.nkxp < g.nkx;   // (npen is a multiple of ZW_PPB)
  return q;
}

// The lane's factors from the table of zw_fill (read at the start of each
// transform: they would cost 22 registers between transforms).
template <typename T>
__device__ __forceinline__ ZwLane<T> zw_lane(const cpx<T>* lt, int j) {
  ZwLane<T> w;
  w.w32 = lt[j];
  w.w16 = lt[32 + j];
  w.w8 = lt[64 + j];
  w.w4 = lt[96 + j];
  w.u32 = j & 16;
  w.u16 = j & 8;
  w.s8 = (j & 4) ? T(-1) : T(1);
  w.s7 = (j & 2) ? T(-1) : T(1);
  w.s3 = (j & 1) ? T(-1) : T(1);
  return w;
}

// The workgroup's tables in LDS, read-only after a barrier.  Transforms: register
// twiddles tw[(r - 1) * 32 + j] = w_N^(j r) and the lane steps' factors
// lt[step * 32 + j].
template <typename T, int K>
struct ZwTw {
  cpx<T> tw[(K - 1) * 32];
  cpx<T> lt[4 * 32];
};
// Continuation: coefficients M[i][k * 32 + j] of row 32 (K - 1 - i) + j on the 2 d
// boundary rows (right end first; zero for rows below nz); bnd: each wave's own
// exchange buffer.
struct ZwExt {
  double M[2][2 * ZW_MAXD * 32];
  cpx<double> bnd[ZW_WAVES][2 * ZW_MAXD * 2];
};
// The z pass: filter factors, and the roots top[l] = exp(2 pi i l (nz - 1) / N')
// of the value at row nz - 1.
template <int K>
struct ZwRows {
  double sig[32 * K];
  cpx<double> top[32 * K];
};

template <typename T, int K>
__device__ __forceinline__ void zw_fill(ZwTw<T, K>& sh, const ZArgs& a) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int e = tid; e < (K - 1) * 32; e += nt)
    sh.tw[e] = cvt<T>(a.tw64[(e / 32 + 1) * (e % 32)]);
  for (int e = tid; e < 128; e += nt) {
    // step s (distance D = 16, 8, 4, 2 in j): w_{2 D}^(j mod D), for the DPP
    // steps 1 in the lower half
    const int s = e / 32, j = e % 32, D = 16 >> s;
    sh.lt[e] = (s >= 2 && !(j & D)) ? mk(T(1), T(0)) : cvt<T>(a.tw64[(K << s) * (j & (D - 1))]);
  }
}
template <int K>
__device__ __forceinline__ void zw_fill(ZwExt& sh, const ZArgs& a) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int d = a.g.d, C = a.g.C;
  for (int e = tid; e < (C > 32 ? 2 : 1) * 2 * d * 32; e += nt) {
    const int h = e / (2 * d * 32), k = e / 32 % (2 * d), j = e % 32;
    const int i = 32 * (K - 1 - h) + j - a.g.nz;
    double m = 0.0;
    if (i >= 0) m = k < d ? a.fc[i * d + k] : a.fc[(C - 1 - i) * d + (d - 1 - (k - d))];
    sh.M[h][k * 32 + j] = m;
  }
}
template <int K>
__device__ __forceinline__ void zw_fill(ZwRows<K>& sh, const ZArgs& a) {
  for (int e = threadIdx.x; e < 32 * K; e += blockDim.x) {
    sh.sig[e] = a.sigz[e];
    sh.top[e] = conj(a.tw64[(e * (a.g.nz - 1)) % (32 * K)]);
  }
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
__device__ __forceinline__ void zw_fft(cpx<T> (&x)[K], const ZwTw<T, K>& sh, int j) {
  const cpx<T>* tw = sh.tw;
  zw_phase();
  zw_dft<T, K>(x);
#pragma unroll
  for (int r = 1; r < K; ++r) x[r] = x[r] * tw[(r - 1) * 32 + j];
  zw_phase();
  const ZwLane<T> w = zw_lane<T>(sh.lt, j);
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
__device__ __forceinline__ void zw_ifft(cpx<T> (&x)[K], const ZwTw<T, K>& sh, int j) {
  const cpx<T>* tw = sh.tw;
  zw_phase();
  const ZwLane<T> w = zw_lane<T>(sh.lt, j);
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

// Continuation rows nz..N'-1 of the line (Sec. 3; M_l = J M_r J), in the last
// register (C > 32: the last two).  The 2 d boundary rows, all in the last two
// and the first register, go through the wave's LDS buffer and are read back
// as broadcasts.
template <int K>
__device__ __forceinline__ void zw_extend(cpx<double> (&x)[K], const Geom& g,
                                          ZwExt& sh, int wv, int j, int pen) {
  cpx<double>* bnd = sh.bnd[wv];
  const int d = g.d, r0 = g.nz - d;
  if (j < d) bnd[2 * (d + j) + pen] = x[0];
#pragma unroll
  for (int m = K - 2; m < K; ++m) {
    const int n = j + 32 * m;
    if (n >= r0 && n < g.nz) bnd[2 * (n - r0) + pen] = x[m];
  }
  zw_sync();
  auto rows = [&](int h, cpx<double>& v) {
    const double* M = sh.M[h] + j;
    double ar = 0.0, ai = 0.0;
    for (int k = 0; k < 2 * d; ++k) {
      const double c = M[k * 32];
      const cpx<double> b = bnd[2 * k + pen];
      ar += c * b.x;
      ai += c * b.y;
    }
    if (j + 32 * (K - 1 - h) >= g.nz) v = mk(ar, ai);
  };
  rows(0, x[K - 1]);
  if (g.C > 32) rows(1, x[K - 2]);
  zw_sync();
}

// ---------------------------------------------------------------- pieces of the pass
template <int K>
__device__ __forceinline__ int zw_coef(const ZwIdx& q, int r) { return r + K * q.k2; }

// A fresh copy of the lane's indices: what is derived from them is recomputed
// in each phase instead of being kept in registers across all of them.
__device__ __forceinline__ ZwIdx zw_fresh(ZwIdx q) {
  asm volatile("" : "+v"(q.j), "+v"(q.k2), "+v"(q.p));
  return q;
}

// The lane's coefficients r = 0..K-1 (rows K k2 + r of its pencil's group);
// 32-bit offsets (a field has at most 288 x 266240 elements).
template <int K, typename C>
__device__ __forceinline__ C* zw_spec(C* base, const ZwIdx& q) {
  const unsigned o = (unsigned)(q.p / SPEC_ROW) * (unsigned)(SPEC_ROW * 32 * K) +
                     (unsigned)(q.p % SPEC_ROW) + (unsigned)(SPEC_ROW * K * q.k2);
  return base + o;
}
template <int K>
__device__ __forceinline__ void zw_load_coef(cpx<double> (&x)[K], const cpx<double>* src,
                                             const ZwIdx& q) {
  const cpx<double>* s = zw_spec<K>(src, q);
#pragma unroll
  for (int r = 0; r < K; ++r) x[r] = s[SPEC_ROW * r];
}
template <int K>
__device__ __forceinline__ void zw_store_coef(const cpx<double> (&x)[K], cpx<double>* dst,
                                              const ZwIdx& q) {
  cpx<double>* s = zw_spec<K>(dst, q);
  if (q.pv) {
#pragma unroll
    for (int r = 0; r < K; ++r) s[SPEC_ROW * r] = x[r];
  }
}

// The stage: rows z < nz of the workgroup's 8 pencils in LDS, [z][8], through
// which mixed rows are read and written 128 bytes at a time (a wavefront's own two
// pencils are 32).  Pencil pair w of row z sits in pair slot w ^ ((z / 2) mod 4):
// a wave reads its pair of 8 consecutive rows from all banks.
__device__ __forceinline__ int zw_slot(int pair, int z) { return 2 * (pair ^ ((z >> 1) & 3)); }

// A workgroup-wide field into the stage by direct loads (no registers: they
// land while the waves compute; rows past nz repeat the last).  Wave wv takes
// rows 8 (wv + 4 i) .. + 7, one row per 8 lanes.  zw_stage_wait and a barrier
// before the rows are read.
template <int K>
__device__ __forceinline__ void zw_stage_load(cpx<double>* stage, const cpx<double>* src,
                                              const Geom& g, long long p0, int wv) {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int zr = lane >> 3, s = lane & 7;
  const int pen = zw_slot(s >> 1, zr) + (s & 1);   // (the slot map is its own inverse)
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const int z0 = 8 * (wv + ZW_WAVES * i), z = min(z0 + zr, g.nz - 1);
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(src + (long long)z * g.npen + p0 + pen),
        (__attribute__((address_space(3))) void*)(stage + 8 * z0), 16, 0, 0);
  }
}
__device__ __forceinline__ void zw_stage_wait() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

// The stage's rows to a mixed field.
template <int K, typename T>
__device__ __forceinline__ void zw_stage_store(const cpx<T>* stage, cpx<T>* dst, const Geom& g,
                                               long long p0, int wv) {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int zr = lane >> 3, s = lane & 7;
  const long long p = p0 + zw_slot(s >> 1, zr) + (s & 1);
  const bool pv = (int)(p % g.nkxp) < g.nkx;
  cpx<T> v[K];
#pragma unroll
  for (int i = 0; i < K; ++i) v[i] = stage[64 * (wv + ZW_WAVES * i) + lane];
  if (pv) {
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int z = 8 * (wv + ZW_WAVES * i) + zr;
      if (i < K - 2 || z < g.nz) dst[(long long)z * g.npen + p] = v[i];
    }
  }
}

// x[m] = the wave's natural rows of the stage (rows past nz, in the last two
// registers, are replaced by the continuation) / the rows z < nz into it.
template <int K>
__device__ __forceinline__ void zw_stage_get(cpx<double> (&x)[K], const cpx<double>* stage,
                                             const Geom& g, int j, int wv, int pen) {
  const cpx<double>* s = stage + 8 * j + zw_slot(wv, j) + pen;
#pragma unroll
  for (int m = 0; m < K; ++m)
    x[m] = (m < K - 2 || j + 32 * m < g.nz) ? s[256 * m] : zero<double>();
}
template <int K, typename T>
__device__ __forceinline__ void zw_stage_put(const cpx<T> (&x)[K], cpx<T>* stage, const Geom& g,
                                             int j, int wv, int pen) {
  cpx<T>* s = stage + 8 * j + zw_slot(wv, j) + pen;
#pragma unroll
  for (int m = 0; m < K; ++m)
    if (m < K - 2 || j + 32 * m < g.nz) s[256 * m] = x[m];
}

template <int K>
__device__ __forceinline__ void zw_check(const ZArgs& a, const cpx<double> (&x)[K],
                                         const ZwIdx& q) {
  if (!a.nonfinite) return;
  bool bad = false;
#pragma unroll
  for (int r = 0; r < K; ++r)
    bad = bad || !__builtin_isfinite(x[r].x) || !__builtin_isfinite(x[r].y);
  if (bad && q.pv) *a.nonfinite = 1;
}

// sum over the 32 lanes of a pencil, in every lane
__device__ __forceinline__ double zw_sum(double v) {
  v += zw_dpp<ZW_X3>(v);
  v += zw_dpp<ZW_X7>(v);
  v += zw_dpp<ZW_X8>(v);
  double a = v, b = v;
  zw_swap<16>(a, b);
  v = a + b;
  a = b = v;
  zw_swap<32>(a, b);
  return a + b;
}
__device__ __forceinline__ cpx<double> zw_sum(cpx<double> v) {
  return mk(zw_sum(v.x), zw_sum(v.y));
}

// Wavenumbers of a pencil: k~x, k~y, |k_h|^2 with the true and the
// Nyquist-zeroed ones, and the filter factor.
struct ZwWave {
  double kxo, kyo, kh2t, kh2o, sxy;
};
__device__ __forceinline__ ZwWave zw_wave(const ZArgs& a, int p) {
  const Geom& g = a.g;
  const int iy = p / g.nkxp, ix = p - iy * g.nkxp;
  const double kxt = g.kxs * ix, kyt = k_true(iy, g.ny, g.kys);
  ZwWave w;
  w.kxo = (2 * ix == g.nx) ? 0.0 : kxt;
  w.kyo = k_odd(iy, g.ny, g.kys);
  w.kh2t = kxt * kxt + kyt * kyt;
  w.kh2o = w.kxo * w.kxo + w.kyo * w.kyo;
  w.sxy = a.sigy[iy] * a.sigx[ix < g.nkx ? ix : 0];
  return w;
}

// ---------------------------------------------------------------- stage A
// V* of one field from its nonlinear rows in x: N = sigma F_z(NL);
// S = V^t + c (N - diff |k|^2 W) [+ c gamma W_other]; v* = B_z S with the body
// force, the wall values injected; V* = F_z v* (Sec. 4.4 steps 1-3), left in
// x in coefficient order.  The rows vt, w of V^t and W were loaded before
// (WV: W is V^t).
template <int K, bool WV>
__device__ __forceinline__ void zw_stageA(cpx<double> (&x)[K], cpx<double> (&vt)[K],
                                          const cpx<double> (&w)[WV ? 1 : K], const ZArgs& a,
                                          const StageAArgs& s, int f, ZwIdx q,
                                          const ZwWave* wks, const ZwTw<double, K>& sh,
                                          ZwExt& ex, const ZwRows<K>& rows, int wv, int pen,
                                          cpx<double>* stage, const void* nl_next,
                                          long long p0) {
  constexpr int N = 32 * K;
  const Geom& g = a.g;
  const cpx<double>* wb = reinterpret_cast<const cpx<double>*>(s.buoy[f]);
  const double c = s.c, diff = (f == 3) ? s.kappa : s.nu;
  zw_extend<K>(x, g, ex, wv, q.j, pen);
  // V^t - c diff |k|^2 W, formed before the transform: one array of rows
  // instead of two stays live through it
  const double kh2t = wks[2 * wv + pen].kh2t;
#pragma unroll
  for (int r = 0; r < K; ++r) {
    const double kz = k_true(zw_coef<K>(q, r), N, g.kzs);
    vt[r] = vt[r] - (WV ? vt[r] : w[WV ? 0 : r]) * (c * diff * (kh2t + kz * kz));
  }
  // the next field's rows, in flight through this field's transforms (issued
  // behind the last use of vt's and w's loads, which complete in order)
  zw_phase();
  // (the other field's rows for the buoyancy, during the transform where there
  // are registers for them)
  constexpr bool EARLY = K <= 6;
  cpx<double> ow[EARLY ? K : 1];
  if constexpr (EARLY)
    if (wb) zw_load_coef<K>(ow, wb, q);
  if (nl_next)
    zw_stage_load<K>(stage, reinterpret_cast<const cpx<double>*>(nl_next), g, p0, wv);
  zw_fft<double, K>(x, sh, q.j);
  q = zw_fresh(q);
  const double sc = wks[2 * wv + pen].sxy * c;
#pragma unroll
  for (int r = 0; r < K; ++r) x[r] = vt[r] + x[r] * (rows.sig[zw_coef<K>(q, r)] * sc);
  if (wb) {
    const double cg = c * s.gamma;
    if constexpr (EARLY) {
#pragma unroll
      for (int r = 0; r < K; ++r) x[r] = x[r] + ow[r] * cg;
    } else {
      zw_load_coef<K>(vt, wb, q);
#pragma unroll
      for (int r = 0; r < K; ++r) x[r] = x[r] + vt[r] * cg;
    }
  }
  // wall values: c times the previous stage's gradient for u and v, 0 for theta
  // (row 0 in the first register, row nz - 1 in one of the last two)
  cpx<double> gw0 = zero<double>(), gw1 = zero<double>();
  auto load_gw = [&] {
    if (f < 2) {
      gw0 = s.gwall[f * g.npen + q.p];
      gw1 = s.gwall[(2 + f) * g.npen + q.p];
    }
  };
  if constexpr (EARLY) load_gw();
  zw_ifft<double, K>(x, sh, q.j);
  q = zw_fresh(q);
  if constexpr (!EARLY) load_gw();
  const double inv = 1.0 / N;
  const double force = (f == 0 && q.p == 0) ? c * s.forcing_sum : 0.0;
#pragma unroll
  for (int m = 0; m < K; ++m) x[m] = mk(x[m].x * inv + force, x[m].y * inv);
  if (f != 2) {
    if (q.j == 0) x[0] = gw0 * c;
#pragma unroll
    for (int m = K - 2; m < K; ++m)
      if (q.j + 32 * m == g.nz - 1) x[m] = gw1 * c;
  }
  zw_extend<K>(x, g, ex, wv, q.j, pen);
  zw_fft<double, K>(x, sh, q.j);
}

// ---------------------------------------------------------------- projection
// Sec. 4.2 and 4.4 steps 3-5 on V* of the three velocity fields held in
// coefficient order (see z_stageB_body of zpass.hip for the formulas).  The
// homogeneous solution needs F_z of e+ = e^{gamma (z - Lz)} and
// e- = e^{-gamma z}: the continuation's tables are mirror images, so the
// continued line of e+ is that of e- read backwards from nz - 1 and
// F(e+)_l = conj(e_l F(e-)_l) with e_l = exp(2 pi i l (nz - 1) / N'), the root
// that the wall sum at z = Lz uses: one line is transformed.  e- at rows
// j + 32 m is formed as e^{-gamma dz j} (e^{-32 gamma dz})^m.
// (s of a row, and what hangs on the row index, is formed again in each of the
// passes over the rows: kept, it would not fit in registers.)
template <int K>
__device__ __forceinline__ void zw_project(cpx<double> (&V0)[K], cpx<double> (&V1)[K],
                                           cpx<double> (&V2)[K], const ZArgs& a,
                                           const StageBArgs& s, ZwIdx q, const ZwWave* wks,
                                           const ZwTw<double, K>& sh, ZwExt& ex,
                                           const ZwRows<K>& rows, int wv, int pen) {
  constexpr int N = 32 * K;
  const Geom& g = a.g;
  q = zw_fresh(q);
  const ZwWave wk = wks[2 * wv + pen];
  auto svec = [&](int r, double& kz) {
    const int l = zw_coef<K>(q, r);
    kz = k_odd(l, N, g.kzs);
    const double k2 = wk.kh2o + kz * kz;
    double ik = zw_rcp(k2 > 0.0 ? k2 : 1.0);
    ik = k2 > 0.0 ? ik : 0.0;
    return (V0[r] * wk.kxo + V1[r] * wk.kyo + V2[r] * kz) * ik;
  };
  cpx<double> b = zero<double>(), t = b, s0 = b, s1 = b;
#pragma unroll
  for (int r = 0; r < K; ++r) {
    zw_phase();   // (one row at a time: V* alone takes 12 K registers)
    double kz;
    const cpx<double> sv = svec(r, kz);
    const cpx<double> rz = V2[r] - sv * kz;
    const cpx<double> et = rows.top[zw_coef<K>(q, r)];
    b = b + rz;
    t = t + rz * et;
    s0 = s0 + sv;
    s1 = s1 + sv * et;
  }
  const double inv = 1.0 / N;
  b = zw_sum(b) * inv;
  t = zw_sum(t) * inv;
  s0 = zw_sum(s0) * inv;
  s1 = zw_sum(s1) * inv;
  const double gam = sqrt(wk.kxo * wk.kxo + wk.kyo * wk.kyo);
  // A = B = 0 for gamma = 0, D = 0 otherwise: the sums below take all three
  cpx<double> A = zero<double>(), B = A, D = A;
  double E = 0.0;
  if (gam > 0.0) {
    E = exp(-gam * g.lz);
    const double den = 1.0 / (gam * (1.0 - E * E));
    A = (t - b * E) * den;
    B = (b - t * E) * (-den);
  } else {
    D = (b + t) * 0.5;
  }
  if (s.gwall && q.pv && q.j == 0) {
    const cpx<double> h0 = mul_i(A * E + B), h1 = mul_i(A + B * E);
    const double ic = 1.0 / s.c;
    s.gwall[(0 * 2 + 0) * g.npen + q.p] = (s0 + h0) * (wk.kxo * ic);
    s.gwall[(0 * 2 + 1) * g.npen + q.p] = (s0 + h0) * (wk.kyo * ic);
    s.gwall[(1 * 2 + 0) * g.npen + q.p] = (s1 + h1) * (wk.kxo * ic);
    s.gwall[(1 * 2 + 1) * g.npen + q.p] = (s1 + h1) * (wk.kyo * ic);
  }
  const double e1 = exp(-gam * g.dz * q.j), e32 = exp(-gam * g.dz * 32.0);
  cpx<double> x[K];
  q = zw_fresh(q);
  if (s.pmix) {
    // pressure: (B_z(-i s) + phi^H) / c at the rows z < nz
#pragma unroll
    for (int r = 0; r < K; ++r) {
      zw_phase();
      double kz;
      x[r] = mul_mi(svec(r, kz));
    }
    zw_ifft<double, K>(x, sh, q.j);
    // e+ on its own at the rows of the last two registers (those past the box are
    // not stored), downwards from the last one inside it for every lane
    const double ic = 1.0 / s.c;
    auto eplus = [&](int m) {
      return exp(gam * fmin((q.j + 32 * m) * g.dz - g.lz, 0.0));
    };
    double ep[K], em[K];
    em[0] = e1;
#pragma unroll
    for (int m = 1; m < K; ++m) em[m] = em[m - 1] * e32;
    ep[K - 1] = eplus(K - 1);
    ep[K - 2] = eplus(K - 2);
    if constexpr (K > 2) ep[K - 3] = eplus(K - 3);
#pragma unroll
    for (int m = K - 4; m >= 0; --m) ep[m] = ep[m + 1] * e32;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      const int z = q.j + 32 * m;
      const cpx<double> ph = A * ep[m] + B * em[m] + D * (z * g.dz);
      x[m] = (x[m] * inv + ph) * ic;
    }
    if (q.pv) {
      cpx<double>* o = s.pmix + (long long)q.j * g.npen + q.p;
#pragma unroll
      for (int m = 0; m < K; ++m)
        if (m < K - 2 || q.j + 32 * m < g.nz) o[32LL * m * g.npen] = x[m];
    }
  }
  {
    double em = e1;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      x[m] = mk(em, 0.0);
      em *= e32;
    }
  }
  zw_extend<K>(x, g, ex, wv, q.j, pen);
  zw_fft<double, K>(x, sh, q.j);
  q = zw_fresh(q);
#pragma unroll
  for (int r = 0; r < K; ++r) {
    zw_phase();
    double kz;
    const cpx<double> sv = svec(r, kz);
    const cpx<double> em = x[r], ep = conj(rows.top[zw_coef<K>(q, r)] * em);
    const cpx<double> pa = A * ep, pb = B * em, sym = mul_i(pa + pb) + sv;
    V0[r] = V0[r] - sym * wk.kxo;
    V1[r] = V1[r] - sym * wk.kyo;
    V2[r] = V2[r] - sv * kz - (pa - pb) * gam - D * em;
  }
}

template <int K>
__device__ __forceinline__ void zw_copy(cpx<double> (&d)[K], const cpx<double> (&s)[K]) {
#pragma unroll
  for (int r = 0; r < K; ++r) d[r] = s[r];
}

// B_z of the coefficients v into dst and, where dz is set, of i k~z v into dz,
// through the stage (free on entry and on return, up to a barrier).
template <typename T, int K>
__device__ __forceinline__ void zw_back2(const cpx<double> (&v)[K], cpx<T>* dst, cpx<T>* dz,
                                         const Geom& g, ZwIdx q, const ZwTw<T, K>& sh,
                                         cpx<T>* stage, long long p0, int wv, int pen) {
  constexpr double inv = 1.0 / (32 * K);
#pragma unroll 1
  for (int pass = 0; pass < (dz ? 2 : 1); ++pass) {
    q = zw_fresh(q);
    cpx<T> x[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
      const double kz = pass ? k_odd(zw_coef<K>(q, r), 32 * K, g.kzs) * inv : inv;
      const cpx<double> y = v[r] * kz;
      x[r] = mk((T)(pass ? -y.y : y.x), (T)(pass ? y.x : y.y));
    }
    zw_ifft<T, K>(x, sh, q.j);
    __syncthreads();   // (the stage's previous rows are stored)
    zw_stage_put<K, T>(x, stage, g, q.j, wv, pen);
    __syncthreads();
    zw_stage_store<K, T>(stage, pass ? dz : dst, g, p0, wv);
  }
}

// ---------------------------------------------------------------- one fused z pass
// The whole z pass of one RK stage (FP64) for two pencils per wavefront.
// blockIdx.y = 0: the velocity; V* of its three fields stays in registers from
// stage A through the projection to the back transforms, and nothing is read
// back.  blockIdx.y = 1: theta, its stage A and back transforms.  The two meet
// only in the buoyancy, which reads the other's previous state, so the output
// buffer must not be the input buffer.
// WV: W is V^t itself (the first RK stage); it is read once.
//
// Bound by latency at two waves per SIMD (V* of three fields is 12 K registers):
// at 512 x 512 x 257 with theta the vector units are busy a third of the time and
// memory moves 12.6 GB at 3.4 TB/s.  What it took there, ms per stage: each wave
// reading its own 32-byte pieces of strided rows 6.8; state by pencil groups 5.7;
// mixed rows through the LDS stage, loaded without registers while the waves
// compute, and stored 128 bytes wide 4.15; theta on its own workgroups and the
// projection without branches 3.7 (the workgroup pass it replaces: 4.27).
// 192 x 192 x 193: 0.41 (0.55, separate kernels 0.72), 128: 0.146 (0.187, 0.28),
// 64: 0.038 (separate kernels 0.068).
template <int K, bool WV>
__device__ __forceinline__ void zw_pass_group(const ZArgs& a, const StageAArgs& sa,
                                              const StageBArgs& sb, const ZBackArgs& zb,
                                              long long p0, bool scalar) {
  // (separate variables: reads of the tables need not wait for loads into the stage)
  __shared__ cpx<double> stage[32 * K * ZW_PPB];
  __shared__ ZwTw<double, K> sh;
  __shared__ ZwExt ex;
  __shared__ ZwRows<K> rows;
  __shared__ ZwWave wks[ZW_PPB];
  const Geom& g = a.g;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  zw_stage_load<K>(stage, reinterpret_cast<const cpx<double>*>(sa.nl[scalar ? 3 : 2]), g, p0,
                   wv);
  if (threadIdx.x < ZW_PPB) wks[threadIdx.x] = zw_wave(a, (int)p0 + (int)threadIdx.x);
  zw_fill(sh, a);
  zw_fill<K>(ex, a);
  zw_fill(rows, a);
  const ZwIdx q0 = zw_index(g, (int)p0);
  const int pen = zw_pencil();
  // (v's V* is the last one formed: V1 is not live inside the loop)
  cpx<double> V0[K], V1[K], V2[K];
#pragma unroll 1
  for (int it = scalar ? 3 : 0;; ++it) {
    // w, u, v; or theta
    const int f = it == 0 ? 2 : it == 3 ? 3 : it - 1;
    const ZwIdx q = zw_fresh(q0);
    zw_stage_wait();
    __syncthreads();
    cpx<double> vt[K], w[WV ? 1 : K];
    zw_stage_get<K>(V1, stage, g, q.j, wv, pen);
    zw_load_coef<K>(vt, sa.vt[f], q);
    if constexpr (!WV) zw_load_coef<K>(w, sa.w[f], q);
    __syncthreads();
    zw_stageA<K, WV>(V1, vt, w, a, sa, f, q, wks, sh, ex, rows, wv, pen, stage,
                     it < 2 ? sa.nl[it] : nullptr, p0);
    if (it >= 2) break;
    if (it == 0)
      zw_copy(V2, V1);
    else
      zw_copy(V0, V1);
  }
  const ZwIdx q = zw_fresh(q0);
  if (scalar) {
    zw_copy(V0, V1);
  } else {
    zw_project<K>(V0, V1, V2, a, sb, q, wks, sh, ex, rows, wv, pen);
    zw_check<K>(a, V1, q);
    zw_check<K>(a, V2, q);
    zw_store_coef<K>(V1, sb.vout[1], q);
    zw_store_coef<K>(V2, sb.vout[2], q);
  }
  zw_check<K>(a, V0, q);
  zw_store_coef<K>(V0, scalar ? sa.out[3] : sb.vout[0], q);
  cpx<double>* mv = zb.mv + (scalar ? 6 * zb.ms : 0);
#pragma unroll 1
  for (int f = 0; f < (scalar ? 1 : 3); ++f) {
    cpx<double> x[K];
    if (f == 0) zw_copy(x, V0);
    else if (f == 1) zw_copy(x, V1);
    else zw_copy(x, V2);
    zw_back2<double, K>(x, mv + 2 * f * zb.ms, mv + (2 * f + 1) * zb.ms, g, q, sh, stage, p0, wv,
                        pen);
  }
}

template <int K, bool WV>
__global__ __launch_bounds__(64 * ZW_WAVES, 2) void k_zw_pass(ZArgs a, StageAArgs sa,
                                                              StageBArgs sb, ZBackArgs zb) {
  zw_pass_group<K, WV>(a, sa, sb, zb, (long long)blockIdx.x * ZW_PPB, blockIdx.y == 1);
}

// The same for several problems of one N' in one launch: workgroup b serves
// problem r with d[r].wg0 <= b < d[r + 1].wg0.
template <int K>
__global__ __launch_bounds__(64 * ZW_WAVES, 2) void k_zw_pass_batch(const ZPassDesc* d, int n) {
  int r = 0;
  while (r + 1 < n && (long long)blockIdx.x >= d[r + 1].wg0) ++r;
  const ZPassDesc& D = d[r];
  if (blockIdx.y == 1 && D.nf < 4) return;
  zw_pass_group<K, false>(D.a, D.sa, D.sb, D.zb, ((long long)blockIdx.x - D.wg0) * ZW_PPB,
                          blockIdx.y == 1);
}

// ---------------------------------------------------------------- transforms alone
// mixed -> continued spectral: F_z (times the filter if asked); one field per
// blockIdx.y, as the next.
template <int K>
__global__ __launch_bounds__(64 * ZW_WAVES) void k_zw_fwd(ZArgs a,
                                                          const cpx<double>* __restrict__ src,
                                                          cpx<double>* __restrict__ dst,
                                                          long long sfs, long long dfs,
                                                          int filter) {
  __shared__ cpx<double> stage[32 * K * ZW_PPB];
  __shared__ ZwTw<double, K> sh;
  __shared__ ZwExt ex;
  const Geom& g = a.g;
  const long long p0 = (long long)blockIdx.x * ZW_PPB;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  zw_stage_load<K>(stage, src + blockIdx.y * sfs, g, p0, wv);
  zw_fill(sh, a);
  zw_fill<K>(ex, a);
  zw_stage_wait();
  __syncthreads();
  ZwIdx q = zw_index(g, (int)blockIdx.x * ZW_PPB);
  const int pen = zw_pencil();
  cpx<double> x[K];
  zw_stage_get<K>(x, stage, g, q.j, wv, pen);
  zw_extend<K>(x, g, ex, wv, q.j, pen);
  zw_fft<double, K>(x, sh, q.j);
  q = zw_fresh(q);
  if (filter) {
    const double sxy = zw_wave(a, q.p).sxy;
#pragma unroll
    for (int r = 0; r < K; ++r) x[r] = x[r] * (a.sigz[zw_coef<K>(q, r)] * sxy);
  }
  zw_store_coef<K>(x, dst + blockIdx.y * dfs, q);
}

// continued spectral -> mixed: B_z and, where dz is set, B_z(i k~z .).
template <typename T, int K>
__global__ __launch_bounds__(64 * ZW_WAVES) void k_zw_back(ZArgs a,
                                                           const cpx<double>* __restrict__ src,
                                                           cpx<T>* __restrict__ dst,
                                                           cpx<T>* __restrict__ dz,
                                                           long long sfs, long long mfs) {
  __shared__ cpx<T> stage[32 * K * ZW_PPB];
  __shared__ ZwTw<T, K> sh;
  const Geom& g = a.g;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const ZwIdx q = zw_index(g, (int)blockIdx.x * ZW_PPB);
  cpx<double> v[K];
  zw_load_coef<K>(v, src + blockIdx.y * sfs, q);
  zw_fill(sh, a);
  zw_check<K>(a, v, q);
  __syncthreads();
  const long long o = blockIdx.y * mfs;
  zw_back2<T, K>(v, dst + o, dz ? dz + o : nullptr, g, q, sh, stage,
                 (long long)blockIdx.x * ZW_PPB, wv, zw_pencil());
}

// ---------------------------------------------------------------- derivative of lines
// fc_derivative: two real lines per complex line (the multipliers i k~z and
// -kz^2 map real lines to real lines), four lines per wavefront; both
// transforms and the continuation stay in registers, so a line is read and
// written once and nothing waits at a barrier in between.  65537 lines of 257
// points (N' = 288, 269 MB) against the workgroup engine: eight pairs of buffers
// in turn 129 -> 70 us (3.9 TB/s; a large copy takes 54), one pair 109 -> 64; one
// call after 1 GiB of other reads 130 -> 73, of other writes 147 -> 90.
template <int K>
__global__ __launch_bounds__(64 * ZW_WAVES) void k_zw_deriv(ZArgs a,
                                                            const double* __restrict__ in,
                                                            double* __restrict__ out,
                                                            long long nlines, long long ls,
                                                            int order) {
  constexpr int N = 32 * K;
  __shared__ ZwTw<double, K> sh;
  __shared__ ZwExt ex;
  zw_fill(sh, a);
  zw_fill<K>(ex, a);
  __syncthreads();
  const Geom& g = a.g;
  ZwIdx q{};
  zw_lanes(q);
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int pen = zw_pencil();
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
      const int n = m < K - 2 ? q.j + 32 * m : min(q.j + 32 * m, g.nz - 1);
      x[m] = mk(fa[n], fb[n]);
    }
    zw_extend<K>(x, g, ex, wv, q.j, pen);
    zw_fft<double, K>(x, sh, q.j);
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
    zw_ifft<double, K>(x, sh, q.j);
    const double inv = 1.0 / N;
    double* oa = out + l0 * ls;
    double* ob = out + l1 * ls;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      const int z = q.j + 32 * m;
      if (m < K - 2 || z < g.nz) {
        if (l0 < nlines) oa[z] = x[m].x * inv;
        if (l1 < nlines) ob[z] = x[m].y * inv;
      }
    }
  }
}

// ---------------------------------------------------------------- launchers
// N' = 32 K, K = 2..9; the continuation and the right boundary rows in the last
// two registers (C + d <= 64), at most ZW_MAXD matching points: every stored
// table (C = 15, 25, 31, 33).
static bool zw_lines_fit(const ZArgs& a) {
  const Geom& g = a.g;
  return g.npr % 32 == 0 && g.npr >= 64 && g.npr <= 288 && g.C + g.d <= 64 && g.d <= ZW_MAXD &&
         a.tw64;
}
bool z_wave_fits(const ZArgs& a) { return zw_lines_fit(a) && a.g.npen % ZW_PPB == 0; }

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

void launch_zw_pass(const ZArgs& a, const StageAArgs& sa, const StageBArgs& sb,
                    const ZBackArgs& zb, int nfields, hipStream_t st) {
  dim3 grid((unsigned)(a.g.npen / ZW_PPB), nfields == 4 ? 2 : 1);
  bool wv = true;   // W is V^t for every field (the first RK stage)
  for (int f = 0; f < nfields; ++f) wv = wv && sa.w[f] == sa.vt[f];
  if (wv)
    FCNS_ZW_SWITCH(a.g.npr / 32, hipLaunchKernelGGL((k_zw_pass<K, true>), grid,
                                                    dim3(64 * ZW_WAVES), 0, st, a, sa, sb, zb))
  else
    FCNS_ZW_SWITCH(a.g.npr / 32, hipLaunchKernelGGL((k_zw_pass<K, false>), grid,
                                                    dim3(64 * ZW_WAVES), 0, st, a, sa, sb, zb))
}

void launch_zw_pass_batch(const ZPassDesc* d, int n, long long groups, int npr, hipStream_t st) {
  dim3 grid((unsigned)groups, 2);
  FCNS_ZW_SWITCH(npr / 32, hipLaunchKernelGGL(k_zw_pass_batch<K>, grid, dim3(64 * ZW_WAVES), 0, st,
                                              d, n))
}

void launch_zw_fwd(const ZArgs& a, const cpx<double>* src, cpx<double>* dst, long long sfs,
                   long long dfs, int nfields, int filter, hipStream_t st) {
  dim3 grid((unsigned)(a.g.npen / ZW_PPB), nfields);
  FCNS_ZW_SWITCH(a.g.npr / 32, hipLaunchKernelGGL(k_zw_fwd<K>, grid, dim3(64 * ZW_WAVES), 0, st,
                                                  a, src, dst, sfs, dfs, filter))
}

template <typename T>
void launch_zw_back(const ZArgs& a, const cpx<double>* src, cpx<T>* dst, cpx<T>* dzdst,
                    long long sfs, long long mfs, int nfields, hipStream_t st) {
  dim3 grid((unsigned)(a.g.npen / ZW_PPB), nfields);
  FCNS_ZW_SWITCH(a.g.npr / 32, hipLaunchKernelGGL((k_zw_back<T, K>), grid, dim3(64 * ZW_WAVES), 0,
                                                  st, a, src, dst, dzdst, sfs, mfs))
}
template void launch_zw_back<double>(const ZArgs&, const cpx<double>*, cpx<double>*, cpx<double>*,
                                     long long, long long, int, hipStream_t);
template void launch_zw_back<float>(const ZArgs&, const cpx<double>*, cpx<float>*, cpx<float>*,
                                    long long, long long, int, hipStream_t);

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
