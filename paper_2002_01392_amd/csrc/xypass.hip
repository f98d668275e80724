// Periodic-direction kernels: FFTs along y (c2c) and x (r2c / c2r), and the
// fused x-pass that evaluates the advective products in physical space.
//
// Layouts (x fastest): physical real fields [planes][ny][nx]; (kx, y) and
// (kx, ky) complex fields [planes][ny][nkxp] holding nkx = nx/2 + 1 modes per
// row, the row stride nkxp padded to a multiple of 4 (64 B).  Inverse
// transforms use IFFT(y) = conj(FFT(conj(y))) / n with the conjugations folded
// into loads and stores.
#include "kernels.hpp"
#include "xwave.hpp"

#include <type_traits>

namespace fcns {

// ---------------------------------------------------------------- y pass
// Lines q = plane * nkxp + kx; a tile is YL consecutive lines, staged in LDS
// interleaved (element ky of line l at l + YL ky, y_span slots per buffer).  Each thread keeps one line of the tile (l = tid % YL,
// YNT being a multiple of YL) and the rows ky = tid / YL + r * YNT / YL.
// Workgroups loop over tiles and load the next tile into registers before
// transforming the current one, so the loads overlap the FFT.  mode 1
// (inverse only): a second pass transforms i k~y times the input into dst2.
// Lines are interleaved without padding: two workgroups of 512-point lines
// (2 x 4 lines x 512 points x 2 buffers) then fit the 160 KB of LDS per CU,
// which matters more than the 2-way bank conflicts of the first stage.
__host__ __device__ inline int y_span(int ny, int lines) { return lines * ny; }

size_t y_lds_bytes(int ny, int tsize, size_t elem, int lines) {
  return ((size_t)tsize + 2 * (size_t)y_span(ny, lines)) * elem;
}

constexpr int Y_DYN8 = 192;   // y_tile_lines

bool y_wide_tiles(const YArgs& a) { return a.ny == 512 && plan_is(a.pl, {8, 8, 8}); }

// PF: load the next tile into registers while the current one is transformed
// (more registers, fewer waves per SIMD) or load each tile when it is needed.
// LT lines per tile, NT threads.
// Waves per SIMD asked of the compiler where it would otherwise take more registers
// than they leave (matrix accumulators on top of the tile, or two tiles of 8 or 9
// rows), and where that was faster: y back with d/dy at 96 x 300 x 69 135 -> 82 us, at
// 2 x 127 points 213 -> 138; mixed, at 2 x 257 619 -> 354.  Not more than 9
// rows in FP64 (2 x 307: 880 -> 1050, one workgroup per CU by its LDS anyway), nor
// FP32 without such primes (640: 80 -> 84).
template <typename T, class FP, int OWN>
constexpr int y_waves() {
  if constexpr (!FP::dynamic) {
    return 1;
  } else {
    constexpr int pm = FP::primes;
    if (sizeof(T) == 8) return OWN <= 9 && (OWN >= 8 || pm == PRIMES_MATRIX) ? 2 : 1;
    if (pm == PRIMES_NONE || (pm == PRIMES_PAIRS && OWN < 8)) return 1;
    return OWN <= 4 ? 4 : OWN <= 9 ? 3 : 2;
  }
}
template <typename T, class FP, int OWN, bool PF, int LT, int NT>
__global__ __launch_bounds__(NT, (y_waves<T, FP, OWN>())) void k_y(YArgs a, const cpx<T>* src, cpx<T>* dst,
                                               cpx<T>* dst2, long long sfs, long long dfs,
                                               long long nlines, int inv, int mode) {
  constexpr int YL = LT, YNT = NT;
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x;
  const int ny = FP::dynamic ? a.ny : FP::n;
  const int nkx = a.nkx, nkxp = a.nkxp;
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
  cpx<T>* X0 = tw + a.pl.tsize;
  cpx<T>* X1 = X0 + y_span(ny, YL);
  src += blockIdx.y * sfs;
  dst += blockIdx.y * dfs;
  if (mode == 1) dst2 += blockIdx.y * dfs;
  const cpx<T>* gtw = reinterpret_cast<const cpx<T>*>(a.tw);
  for (int i = tid; i < a.pl.tsize; i += YNT) tw[i] = gtw[i];
  const int l = tid % YL, ky0 = tid / YL;
  constexpr int KYS = YNT / YL;
  // the 512-point compiled plan keeps its first and last stages in registers
  constexpr bool RE = std::is_same<FP, SPlan<8, 8, 8>>::value && OWN == 8 && KYS == 64;
  const long long ntiles = (nlines + YL - 1) / YL;
  const T sc = inv ? T(1) / (T)ny : T(1);
  const int npass = (mode == 1) ? 2 : 1;
  cpx<T> cur[OWN], nxt[PF ? OWN : 1];
  // XCD-aware tile order: workgroups are dispatched to the 8 XCDs in turn
  // (workgroup b on XCD b % 8), and a tile may be less than a 128-byte line
  // wide (4 columns; 8 in FP32), so neighbouring tiles share lines.  Each round of G tiles
  // is cut into chunks of 64; in a chunk, XCD x takes the run of 8 tiles
  // 8x .. 8x + 7, one per workgroup of that XCD, so that neighbours meet
  // their shared lines in one L2 and a partial last round still spreads
  // over all XCDs.
  const long long G = gridDim.x;
  long long t = blockIdx.x;
  if (G % 64 == 0) {
    const int j = blockIdx.x / 8, x = blockIdx.x % 8;
    t = (long long)(j / 8) * 64 + x * 8 + j % 8;
  }
  // element ky of line (plane, kx) at base + ky * stride: row-major
  // (stride nkxp) or blocked (stride 4: the 4 columns of a tile contiguous)
  const bool sblk = a.blk & 1, dblk = a.blk & 2;
  const int sstr = sblk ? 4 : nkxp, dstr = dblk ? 4 : nkxp;
  auto line_at = [&](long long tt, bool& ok, bool blocked) {
    const long long q = tt * YL + l;
    const long long pl = q / nkxp, kx = q - pl * nkxp;
    ok = q < nlines && kx < nkx;
    if (!ok) return 0LL;
    return pl * ny * nkxp + (blocked ? (kx >> 2) * ny * 4 + (kx & 3) : kx);
  };
  auto line_base = [&](long long tt, bool& ok) { return line_at(tt, ok, sblk); };
  if constexpr (PF) {
    bool ok;
    const long long base = line_base(t, ok);
#pragma unroll
    for (int r = 0; r < OWN; ++r) {
      const int ky = ky0 + r * KYS;
      cur[r] = (ok && ky < ny) ? src[base + (long long)ky * sstr] : zero<T>();
    }
  }
  for (; t < ntiles; t += gridDim.x) {
    bool ok;
    const long long base = line_base(t, ok);
    const long long dbase = line_at(t, ok, dblk);
    if constexpr (PF) {
      bool okn;
      const long long basen = line_base(t + gridDim.x, okn);
#pragma unroll
      for (int r = 0; r < OWN; ++r) {
        const int ky = ky0 + r * KYS;
        nxt[r] = (okn && ky < ny) ? src[basen + (long long)ky * sstr] : zero<T>();
      }
    } else {
#pragma unroll
      for (int r = 0; r < OWN; ++r) {
        const int ky = ky0 + r * KYS;
        cur[r] = (ok && ky < ny) ? src[base + (long long)ky * sstr] : zero<T>();
      }
    }
    for (int pass = 0; pass < npass; ++pass) {
      if constexpr (RE) {
        // 512 = 8 x 8 x 8 with one butterfly per thread in every stage: the
        // first stage's inputs are this thread's rows ky0 + 64 m (its DFT
        // over m needs no twiddles), and so are the last stage's outputs.
        // Only the middle stage goes through LDS: two barriers per
        // transform.  Reuse of X0 / X1 by the next transform is ordered by
        // these barriers (a thread writes X0 only after the barrier that
        // ends every read of it, and X1 only after the next one).
        cpx<T> v[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          cpx<T> x = cur[m];
          if (pass == 1) x = mul_i(x) * (T)k_odd(ky0 + 64 * m, 512, a.kys);
          v[m] = inv ? conj(x) : x;
        }
        Codelet<T, 8>::run(v, nullptr);
#pragma unroll
        for (int m = 0; m < 8; ++m) X0[lds_pos<false>(l, 8 * ky0 + m, YL, 1)] = v[m];
        __syncthreads();
        sfft_stage<T, 8, 8, 512, YL, YNT, false>(X0, X1, YL, 1, tw + a.pl.toff[1], nullptr, tid);
        __syncthreads();
        const cpx<T>* tws = tw + a.pl.toff[2];
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = X1[lds_pos<false>(l, ky0 + 64 * m, YL, 1)];
#pragma unroll
        for (int m = 1; m < 8; ++m) v[m] = v[m] * tws[(m - 1) * 64 + ky0];
        Codelet<T, 8>::run(v, nullptr);
        cpx<T>* out = pass ? dst2 : dst;
        if (ok) {
#pragma unroll
          for (int m = 0; m < 8; ++m)
            out[dbase + (long long)(ky0 + 64 * m) * dstr] = (inv ? conj(v[m]) : v[m]) * sc;
        }
        continue;
      }
#pragma unroll
      for (int r = 0; r < OWN; ++r) {
        const int ky = ky0 + r * KYS;
        if (ky < ny) {
          cpx<T> v = cur[r];
          if (pass == 1) v = mul_i(v) * (T)k_odd(ky, ny, a.kys);
          X0[lds_pos<false>(l, ky, YL, 1)] = inv ? conj(v) : v;
        }
      }
      __syncthreads();
      const cpx<T>* R = fft_run<T, YL, YNT, false, FP>(X0, X1, YL, 1, a.pl, tw, tid);
      cpx<T>* out = pass ? dst2 : dst;
      if (ok) {
#pragma unroll
        for (int r = 0; r < OWN; ++r) {
          const int ky = ky0 + r * KYS;
          if (ky < ny) {
            const cpx<T> v = R[lds_pos<false>(l, ky, YL, 1)];
            out[dbase + (long long)ky * dstr] = (inv ? conj(v) : v) * sc;
          }
        }
      }
      __syncthreads();
    }
    if constexpr (PF) {
#pragma unroll
      for (int r = 0; r < OWN; ++r) cur[r] = nxt[r];
    }
  }
}

// ---------------------------------------------------------------- x helpers
// Two real rows share one complex line, staged in LDS line-contiguous with the
// padded layout of the FFT engine, element n of line a at xp(a, n) (x_ls:
// line stride).
__device__ __forceinline__ int xp(int a, int n, int ls) { return lds_pos<true>(a, n, 1, ls); }

// ---------------------------------------------------------------- x pass with products
// NL_f = -(u dq_f/dx + v dq_f/dy + w dq_f/dz) at the physical points of RR
// rows (Sec. 4.2: derivatives in Fourier space, products in real space, no
// padding), then its r2c transform.  Passes: 0-2 physical u, v, w; then per
// field f: dq/dx, dq/dy, dq/dz (inverse), and the forward transform of NL_f.
// A workgroup of NT threads owns spectral columns k = tid + c NT and physical
// columns n = tid + c NT (c < CC, CC NT >= nx) of its RR rows; each thread
// loads the next pass's spectral inputs while the current pass is transformed.
// (two waves per SIMD asked for where the matrix accumulators would leave one)
template <class FP>
constexpr int x_waves() {
  if constexpr (FP::dynamic) return FP::primes == PRIMES_MATRIX ? 2 : 1;
  return 1;
}
template <typename T, class FP, int RR, int NT, int CC>
__global__ __launch_bounds__(NT, x_waves<FP>()) void k_x_nl(XArgs a, const cpx<T>* __restrict__ xyb,
                                             cpx<T>* __restrict__ nl, long long fs,
                                             long long nrows, int nfields) {
  constexpr int LL = RR / 2;
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x;
  // with a compile-time plan every row length below is a constant
  const int nx = FP::dynamic ? a.nx : FP::n;
  const int nkx = nx / 2 + 1, nkxp = (nkx + 3) / 4 * 4, ls = x_ls(nx);
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
  cpx<T>* X0 = tw + a.pl.tsize;
  cpx<T>* X1 = X0 + LL * ls;
  const cpx<T>* gtw = reinterpret_cast<const cpx<T>*>(a.tw);
  for (int i = tid; i < a.pl.tsize; i += NT) tw[i] = gtw[i];
  const long long r0 = (long long)blockIdx.x * RR;
  const T sc = T(1) / (T)nx;
  T U[3][CC][RR];
  T acc[CC][RR];
  cpx<T> in[CC][RR];
  // source slot of c2r pass p (-1: forward pass)
  auto slot = [&](int p) {
    if (p < 3) return 3 * p;
    const int f = (p - 3) >> 2, kk = (p - 3) & 3;
    return kk == 3 ? -1 : 3 * f + (kk == 0 ? 0 : kk);
  };
  auto load = [&](int p) {
    const int sl = slot(p);
    if (sl < 0) return;
    const cpx<T>* src = xyb + sl * fs;
#pragma unroll
    for (int c = 0; c < CC; ++c) {
      const int k = tid + c * NT;
#pragma unroll
      for (int r = 0; r < RR; ++r)
        in[c][r] = (k < nkx && r0 + r < nrows) ? src[(r0 + r) * nkxp + k] : zero<T>();
    }
  };
  const int npass = 3 + 4 * nfields;
  load(0);
  for (int pass = 0; pass < npass; ++pass) {
    const int f = (pass - 3) >> 2, kk = (pass - 3) & 3;
    const bool fwd = pass >= 3 && kk == 3;
    if (!fwd) {
      const bool dx = pass >= 3 && kk == 0;
#pragma unroll
      for (int c = 0; c < CC; ++c) {
        const int k = tid + c * NT;
        if (k < nkx) {
          const T kx = (2 * k == nx) ? T(0) : (T)(a.kxs * k);
#pragma unroll
          for (int al = 0; al < LL; ++al) {
            cpx<T> A = in[c][2 * al], B = in[c][2 * al + 1];
            if (dx) {
              A = mul_i(A) * kx;
              B = mul_i(B) * kx;
            }
            if (k == 0 || 2 * k == nx) {
              A.y = T(0);
              B.y = T(0);
            }
            // Z[k] = A + i B, Z[nx - k] = conj(A) + i conj(B); stored conjugated
            X0[xp(al, k, ls)] = conj(mk(A.x - B.y, A.y + B.x));
            if (k > 0 && 2 * k < nx) X0[xp(al, nx - k, ls)] = conj(mk(A.x + B.y, B.x - A.y));
          }
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < CC; ++c) {
        const int n = tid + c * NT;
        if (n < nx) {
#pragma unroll
          for (int al = 0; al < LL; ++al)
            X0[xp(al, n, ls)] = mk(acc[c][2 * al], acc[c][2 * al + 1]);
        }
      }
    }
    // next pass's spectral inputs, in flight during this pass's transform
    int pn = pass + 1;
    if (pn < npass && slot(pn) < 0) ++pn;
    if (pn < npass) load(pn);
    __syncthreads();
    const cpx<T>* R = fft_run<T, LL, NT, true, FP>(X0, X1, 1, ls, a.pl, tw, tid);
    if (!fwd) {
#pragma unroll
      for (int c = 0; c < CC; ++c) {
        const int n = tid + c * NT;
        if (n >= nx) continue;
        T v[RR];
#pragma unroll
        for (int al = 0; al < LL; ++al) {
          const cpx<T> z = R[xp(al, n, ls)];
          v[2 * al] = z.x * sc;
          v[2 * al + 1] = -z.y * sc;
        }
        if (pass < 3) {
#pragma unroll
          for (int r = 0; r < RR; ++r) {
            if (pass == 0) U[0][c][r] = v[r];
            else if (pass == 1) U[1][c][r] = v[r];
            else U[2][c][r] = v[r];
          }
        } else {
#pragma unroll
          for (int r = 0; r < RR; ++r) {
            const T u = (kk == 0) ? U[0][c][r] : ((kk == 1) ? U[1][c][r] : U[2][c][r]);
            if (kk == 0) acc[c][r] = -u * v[r];
            else acc[c][r] -= u * v[r];
          }
        }
      }
    } else {
      // unpack the r2c spectra of the RR rows
#pragma unroll
      for (int al = 0; al < LL; ++al) {
        const long long ra = r0 + 2 * al, rb = ra + 1;
        cpx<T>* dst = nl + f * fs;
        for (int k = tid; k < nkx; k += NT) {
          const cpx<T> Z = R[xp(al, k, ls)];
          const cpx<T> Zm = conj(R[xp(al, ((k == 0) ? 0 : nx - k), ls)]);
          if (ra < nrows) dst[ra * nkxp + k] = (Z + Zm) * T(0.5);
          if (rb < nrows) dst[rb * nkxp + k] = mul_mi(Z - Zm) * T(0.5);
        }
      }
    }
    __syncthreads();
  }
}

// The same for run-time plans of short rows: 8 rows per workgroup, and three
// quantities (u, v, w; dq/dx, dq/dy, dq/dz of a field) transformed together as 12
// complex lines, so that a radix stage of 12 nx / R butterflies fills the 256
// threads (4 lines of 120 points leave three quarters idle) and the row tile
// makes 2 + F rounds of transforms and barriers instead of 3 + 4 F.  The next
// round's spectra are loaded during a round's transform.  A convection solve of
// 120 x 84 x 81 with this kernel and 8-line y tiles: 18.6 -> 12.9 ms (x pass 0.21 ms
// per stage before).
constexpr int X3_NT = 256, X3_L = 12, X3_CE = 5, X3_CP = 3;
constexpr int X3_MAXNX = 192;   // 12 nkxp <= X3_CE X3_NT, 4 nx <= X3_CP X3_NT
template <typename T>
static size_t x3_lds(const XArgs& a) {
  return ((size_t)a.pl.tsize + 2 * X3_L * x_ls(a.nx)) * sizeof(cpx<T>);
}

// (two waves per SIMD asked for: with primes above 7 the compiler would take more than
// 256 registers, and at 154 points, FP64, four fields, 258 us instead of 177)
template <typename T, int NF, int PM>
__global__ __launch_bounds__(X3_NT, 2) void k_x_nl3(XArgs a, const cpx<T>* __restrict__ xyb,
                                                 cpx<T>* __restrict__ nl, long long fs,
                                                 long long nrows) {
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x;
  const int nx = a.nx, nkx = a.nkx, nkxp = a.nkxp, ls = x_ls(nx);
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
  cpx<T>* X0 = tw + a.pl.tsize;
  cpx<T>* X1 = X0 + X3_L * ls;
  const cpx<T>* gtw = reinterpret_cast<const cpx<T>*>(a.tw);
  for (int i = tid; i < a.pl.tsize; i += X3_NT) tw[i] = gtw[i];
  const long long r0 = (long long)blockIdx.x * 8;
  const T sc = T(1) / (T)nx;
  const float rnk = 1.0f / (float)nkxp, rnx = 1.0f / (float)nx;
  // this thread's spectral elements: column ek of line el (quantity el / 4, row
  // pair el % 4) at e = tid + c X3_NT of the 12 nkxp; -1: none
  int el[X3_CE], ek[X3_CE];
#pragma unroll
  for (int c = 0; c < X3_CE; ++c) {
    const int e = tid + c * X3_NT;
    el[c] = x_div(e, nkxp, rnk);
    ek[c] = e - el[c] * nkxp;
    if (el[c] >= X3_L || ek[c] >= nkx) el[c] = -1;
  }
  // and physical points: column pn of row pair pa; -1: none
  int pa[X3_CP], pn[X3_CP];
#pragma unroll
  for (int c = 0; c < X3_CP; ++c) {
    const int e = tid + c * X3_NT;
    pa[c] = x_div(e, nx, rnx);
    pn[c] = e - pa[c] * nx;
    if (pa[c] >= 4) pa[c] = -1;
  }
  cpx<T> in[X3_CE][2];
  // round 0: u, v, w; round 1 + f: the derivatives of field f
  auto load = [&](int round) {
#pragma unroll
    for (int c = 0; c < X3_CE; ++c) {
      const int q = el[c] >> 2, al = el[c] & 3;
      const int slot = round == 0 ? 3 * q : 3 * (round - 1) + q;
      const long long ra = r0 + 2 * al;
      const cpx<T>* src = xyb + slot * fs + ra * nkxp + ek[c];
      in[c][0] = (el[c] >= 0 && ra < nrows) ? src[0] : zero<T>();
      in[c][1] = (el[c] >= 0 && ra + 1 < nrows) ? src[nkxp] : zero<T>();
    }
  };
  T U[3][X3_CP][2], acc[NF][X3_CP][2];
  load(0);
#pragma unroll
  for (int round = 0; round <= NF; ++round) {
#pragma unroll
    for (int c = 0; c < X3_CE; ++c) {
      if (el[c] < 0) continue;
      const int k = ek[c];
      cpx<T> A = in[c][0], B = in[c][1];
      if (round > 0 && el[c] < 4) {
        const T kx = (2 * k == nx) ? T(0) : (T)(a.kxs * k);
        A = mul_i(A) * kx;
        B = mul_i(B) * kx;
      }
      if (k == 0 || 2 * k == nx) A.y = B.y = T(0);
      // Z[k] = A + i B, Z[nx - k] = conj(A) + i conj(B); stored conjugated
      X0[lds_pos<true>(el[c], k, 1, ls)] = conj(mk(A.x - B.y, A.y + B.x));
      if (k > 0 && 2 * k < nx)
        X0[lds_pos<true>(el[c], nx - k, 1, ls)] = conj(mk(A.x + B.y, B.x - A.y));
    }
    if (round < NF) load(round + 1);
    __syncthreads();
    const cpx<T>* R = fft_fwd<T, X3_L, PM, true>(X0, X1, 1, ls, a.pl, tw, tid, X3_NT);
#pragma unroll
    for (int c = 0; c < X3_CP; ++c) {
      if (pa[c] < 0) continue;
      T v[3][2];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const cpx<T> z = R[lds_pos<true>(4 * d + pa[c], pn[c], 1, ls)];
        v[d][0] = z.x * sc;
        v[d][1] = -z.y * sc;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (round == 0) {
          U[0][c][h] = v[0][h];
          U[1][c][h] = v[1][h];
          U[2][c][h] = v[2][h];
        } else {
          T s = -U[0][c][h] * v[0][h];
          s -= U[1][c][h] * v[1][h];
          s -= U[2][c][h] * v[2][h];
          acc[round > 0 ? round - 1 : 0][c][h] = s;
        }
      }
    }
    __syncthreads();
  }
  // forward transforms: fields 0..2 together, then theta
  auto forward = [&](auto lc, int f0) {
    constexpr int L = decltype(lc)::value;
#pragma unroll
    for (int c = 0; c < X3_CP; ++c) {
      if (pa[c] < 0) continue;
#pragma unroll
      for (int f = 0; f < L / 4; ++f)
        X0[lds_pos<true>(4 * f + pa[c], pn[c], 1, ls)] =
            mk(acc[(L == 4 ? NF - 1 : f)][c][0], acc[(L == 4 ? NF - 1 : f)][c][1]);
    }
    __syncthreads();
    const cpx<T>* R = fft_fwd<T, L, PM, true>(X0, X1, 1, ls, a.pl, tw, tid, X3_NT);
#pragma unroll
    for (int c = 0; c < X3_CE; ++c) {
      if (el[c] < 0 || el[c] >= L) continue;
      const int k = ek[c], al = el[c] & 3;
      const cpx<T> Z = R[lds_pos<true>(el[c], k, 1, ls)];
      const cpx<T> Zm = conj(R[lds_pos<true>(el[c], k == 0 ? 0 : nx - k, 1, ls)]);
      const long long ra = r0 + 2 * al;
      cpx<T>* dst = nl + (f0 + (el[c] >> 2)) * fs + ra * nkxp + k;
      if (ra < nrows) dst[0] = (Z + Zm) * T(0.5);
      if (ra + 1 < nrows) dst[nkxp] = mul_mi(Z - Zm) * T(0.5);
    }
  };
  forward(std::integral_constant<int, 12>{}, 0);
  if constexpr (NF == 4) {
    __syncthreads();
    forward(std::integral_constant<int, 4>{}, 3);
  }
}

// ---------------------------------------------------------------- x pass, wave-level rows
// (rows of N points by wavefronts: xwave.hpp)
// Forward transform of two finished real fields (b: none when !two), unpacked
// into the r2c spectra of rows `row` of fields fa and fa + 1; nothing is
// stored for a row past the end (valid false).
template <typename T, int N, typename B>
__device__ __forceinline__ void xw_forward(cpx<T> (&z)[8], B buf,
                                           const cpx<T>* __restrict__ tw, int t,
                                           cpx<T>* __restrict__ nl, long long fs, long long row,
                                           int nkxp, int fa, bool two, bool valid) {
  constexpr int S = N / 8, SN = S + S / 8;  // SN: natural-order slots per register
  wave_fft<T, N>(z, buf, tw, t);
  // slot of element t + S m (S a multiple of 8: a fixed step per register)
  const int t0 = xw_nat(t);
  auto slot = [&](int m) { return S % 8 == 0 ? t0 + SN * m : xw_nat(t + S * m); };
#pragma unroll
  for (int m = 0; m < 8; ++m) buf[slot(m)] = z[m];
  wave_sync();
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const int k = t + S * m;
    if (k <= N / 2 && valid) {
      const cpx<T> Zk = buf[slot(m)];
      const cpx<T> Zm = conj(buf[xw_nat(k == 0 ? 0 : N - k)]);
      nl[fa * fs + row * nkxp + k] = (Zk + Zm) * T(0.5);
      if (two) nl[(fa + 1) * fs + row * nkxp + k] = mul_mi(Zk - Zm) * T(0.5);
    }
  }
  wave_sync();
}

// Input addressing of the wave-level x pass: element kk of (kx, y) row `row`
// (plane row / ny) at rb + xo, with rb per row and xo per register; row-major
// rows (stride nkxp) or the blocked layout of the y pass (the 4 kx columns of
// a block contiguous over y, blocks ny * 4 apart).
__device__ __forceinline__ long long xw_row_base(long long row, int ny, int nkxp, bool blk) {
  if (!blk) return row * nkxp;
  const long long pl = row / ny;
  return pl * ny * nkxp + (row - pl * ny) * 4;
}
__device__ __forceinline__ int xw_col_off(int kk, int ny, bool blk) {
  return blk ? (kk >> 2) * ny * 4 + (kk & 3) : kk;
}

// NL_f = -(u dq_f/dx + v dq_f/dy + w dq_f/dz) on rows of N points.
// The generic schedule: real quantities in the order u, v, w, then per field
// dq/dx, dq/dy, dq/dz, consecutive pairs sharing one inverse transform (the
// value slots are read twice), and the forward transform of a pair of
// finished fields as soon as both are complete.  Used for three fields at
// 512 points, where the one-read schedule below needs more registers than
// two waves per SIMD allow (three fields elsewhere: the one-read schedule, 7%
// faster at 256 and 9% at 128).
template <typename T, int NF, int N, bool BLK>
__global__ __launch_bounds__(64 * XW_WAVES) void k_x_nlw_q(XArgs a, const cpx<T>* __restrict__ xyb,
                                                           cpx<T>* __restrict__ nl, long long fs,
                                                           long long nrows) {
  constexpr int NQ = 3 + 3 * NF, NP = (NQ + 1) / 2;
  constexpr int S = N / 8, RPW = 64 / S;  // lanes per row, rows per wave
  __shared__ cpx<T> tw[XW_TW];
  __shared__ cpx<T> xbuf[XW_WAVES][XW_BUF];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  xw_twiddles<T, N>(tw, tid);
  __syncthreads();
  // the 64 mod S spare lanes (192, 96) repeat the last lanes of row RPW - 1
  const bool spare = lane >= S * RPW;
  const int ln = spare ? lane - S : lane;
  const int t = ln % S, half = ln / S;
  cpx<T>* buf = xbuf[wv] + half * (XW_BUF / RPW);
  const int nkxp = a.nkxp;
  const T kxs = (T)a.kxs;
  const T sc = T(1) / T(N);
  // input offsets per register: kk itself (row-major, folded into the
  // loads) or its place in the blocked layout
  constexpr bool blk = BLK;
  int xo[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int k = t + S * m;
    xo[m] = xw_col_off(k <= N / 2 ? k : N - k, a.ny, blk);
  }
  for (long long rw = (long long)blockIdx.x * XW_WAVES + wv; rw * RPW < nrows;
       rw += (long long)gridDim.x * XW_WAVES) {
    // a row past the end (in the last wave) computes on a copy of the last
    // row and stores nothing; spare lanes compute what their twin lanes do
    const long long row0 = rw * RPW + half;
    const bool inr = RPW == 1 || row0 < nrows;
    const bool valid = inr && !spare;
    const long long row = inr ? row0 : nrows - 1;
    T U[3][8];
    T acc[NF][8];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      // keep each pair's loads next to its transform (hoisting them all would
      // multiply the live registers)
      __builtin_amdgcn_sched_barrier(0);
      // the two quantities of this pair (qb = NQ: none)
      const int qa = 2 * p, qb = 2 * p + 1;
      cpx<T> r[8];
      const long long rb = xw_row_base(row, a.ny, nkxp, blk);
      auto src = [&](int q, bool& dx) -> const cpx<T>* {
        dx = false;
        if (q < 3) return xyb + (3 * q) * fs + rb;
        const int f = (q - 3) / 3, d = (q - 3) % 3;
        dx = d == 0;
        return xyb + (3 * f + d) * fs + rb;
      };
      bool dxa, dxb = false;
      const cpx<T>* pa = src(qa, dxa);
      const cpx<T>* pb = qb < NQ ? src(qb, dxb) : nullptr;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int k = t + S * m;
        const int kk = k <= N / 2 ? k : N - k;
        cpx<T> A = pa[xo[m]];
        cpx<T> B = pb ? pb[xo[m]] : zero<T>();
        const T kx = (kk == N / 2) ? T(0) : kxs * (T)kk;
        if (dxa) A = mul_i(A) * kx;
        if (dxb) B = mul_i(B) * kx;
        if (kk == 0 || kk == N / 2) {
          A.y = T(0);
          B.y = T(0);
        }
        // Z[k] = A + i B (k <= N/2), conj(A) + i conj(B) (k > N/2); inverse via conj
        const cpx<T> Z = (k <= N / 2) ? mk(A.x - B.y, A.y + B.x) : mk(A.x + B.y, B.x - A.y);
        r[m] = conj(Z);
      }
      wave_fft<T, N>(r, buf, tw, t);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int q = 2 * p + h;
        if (q >= NQ) continue;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const T val = h == 0 ? r[m].x * sc : -r[m].y * sc;
          if (q < 3) {
            U[q][m] = val;
          } else {
            const int f = (q - 3) / 3, d = (q - 3) % 3;
            if (d == 0)
              acc[f][m] = -U[0][m] * val;
            else
              acc[f][m] -= U[d][m] * val;
          }
        }
        // a pair of fields finished: forward transform and unpack
        if (q >= 3 && (q - 3) % 3 == 2) {
          const int f = (q - 3) / 3;
          if (f % 2 == 1 || f == NF - 1) {
            const int fa = f % 2 == 1 ? f - 1 : f;
            const bool two = f % 2 == 1;
            cpx<T> z[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) z[m] = mk(acc[fa][m], two ? acc[fa + 1][m] : T(0));
            xw_forward<T, N>(z, buf, tw, t, nl, fs, row, nkxp, fa, two, valid);
          }
        }
      }
    }
  }
}

// Does the pair's next input land in LDS by direct loads while it is transformed?
// Bound by LDS bandwidth (some 60 16-byte accesses per lane and transform) and, at
// two waves per SIMD, by the wait for each pair's rows; a direct load also fetches
// a coefficient once, not once more for its mirror.  192 x 192 x 193 x pass with four
// fields 0.351 -> 0.321 ms, three 0.294 -> 0.252, mixed 0.241 -> 0.198; 128: 0.087 ->
// 0.081, 0.0645 -> 0.062; 256 x 256 x 257, three fields 0.374 -> 0.360, mixed 0.232 ->
// 0.207.  Not 256 with four FP64 fields (0.482 -> 0.490: no registers left), 96 (0.037
// -> 0.041), and 512, where a second workgroup's buffers would not fit.
template <typename T, int NF, int N>
constexpr bool x_direct() {
  return N == 192 || N == 128 || (N == 256 && (NF == 3 || sizeof(T) == 4));
}
// And do so few workgroups gain by it?  Not FP64 rows of 128 points while two
// workgroups per CU hold them all (2600 rows, three fields 18.6 us plain, 20.1 direct;
// 7720: 28.0, 29.7), nor three FP32 fields at 128 or 256 points where three per CU, which
// the buffers of the direct form rule out, do in one round (or little more) what two do
// in two (256: 6240 rows 26.1, 29.0, 7720 27.5, 30.2; 128: 9312 rows 21.2, 22.9).
template <typename T, int NF, int N>
static bool x_direct_pays(long long groups) {
  if (sizeof(T) == 8) return N != 128 || groups > 512;
  return NF == 4 || N == 192 || groups <= 512 || groups > (N == 256 ? 1024 : 768);
}

// DMA: direct loads.  (Two waves per SIMD asked for explicitly where the compiler would
// otherwise go past 256 registers.)
template <typename T, int NF, int N, bool BLK, bool DMA>
__global__ __launch_bounds__(64 * XW_WAVES, (N == 192 || N == 128 || N == 96 || DMA) ? 2 : 1)
void k_x_nlw(XArgs a, const cpx<T>* __restrict__ xyb, cpx<T>* __restrict__ nl, long long fs,
             long long nrows) {
  // Three or four fields: pairs of real quantities per complex transform,
  // each spectral slot read once: (u, du/dx), (v, dv/dx), (w, dw/dx) from
  // one load each (the x derivative is i k~x times the same coefficients),
  // then (dq_f/dy, dq_f/dz) for f = 0..2, and for theta (dq/dx, dq/dy), (dq/dz).
  // NL_f = -(u dq_f/dx + v dq_f/dy + w dq_f/dz) accumulates in that order
  // as soon as u is known; each pair of finished fields is transformed
  // forward together.
  static_assert(NF == 3 || NF == 4, "three or four fields");
  constexpr int NP = NF == 4 ? 8 : 6;
  constexpr int TH = NF - 1;  // theta's accumulator (four fields)
  constexpr int S = N / 8, RPW = 64 / S;  // lanes per row, rows per wave
  constexpr int EPL = 16 / sizeof(cpx<T>);                   // elements per direct load
  constexpr int NI = (RPW * N / 2 / EPL + 63) / 64;          // direct loads per slot
  constexpr int PB = 64 * EPL * NI;                          // elements of one slot
  // (without direct loads no LDS is short, and at 64 points in FP32 the rows behind a table
  // of just its size took 16.0 us instead of 15.0)
  __shared__ cpx<T> tw[DMA ? 14 * S : XW_TW];
  __shared__ cpx<T> xbuf[XW_WAVES * XW_BUF];
  __shared__ cpx<T> pre[DMA ? XW_WAVES : 1][DMA ? 2 * PB + 64 * EPL : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  xw_twiddles<T, N>(tw, tid);
  __syncthreads();
  // the 64 mod S spare lanes (192, 96) repeat the last lanes of row RPW - 1
  const bool spare = lane >= S * RPW;
  const int ln = spare ? lane - S : lane;
  const int t = ln % S, half = ln / S;
  const auto buf = [&] {
    const int o = wv * XW_BUF + half * (XW_BUF / RPW);
    if constexpr (DMA)
      return XwBuf<T>{xbuf, o};
    else
      return xbuf + o;
  }();
  const int nkxp = a.nkxp;
  const T kxs = (T)a.kxs;
  const T sc = T(1) / T(N);
  // input offsets per register: kk itself (row-major, folded into the
  // loads) or its place in the blocked layout
  constexpr bool blk = BLK;
  int xo[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int k = t + S * m;
    xo[m] = xw_col_off(k <= N / 2 ? k : N - k, a.ny, blk);
  }
  // slots of pair p: A, and B: the x derivative of A (p < 3), another slot, or none
  auto slot_a = [](int p) { return p < 3 ? 3 * p : p < 6 ? 3 * (p - 3) + 1 : (p == 6 ? 9 : 11); };
  auto slot_b = [](int p) { return p < 6 ? 3 * (p - 3) + 2 : 10; };
  // direct loads of pair p of the rows whose offsets are in off, offn: k < N/2 of
  // the wave's rows in order, then the Nyquist columns of A and B
  unsigned off[NI], offn = 0;
  auto offsets = [&](long long rw) {
    auto at = [&](int r, int k) {
      const long long row = rw * RPW + r;
      return (unsigned)(xw_row_base(row < nrows ? row : nrows - 1, a.ny, nkxp, blk) +
                        xw_col_off(k, a.ny, blk));
    };
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = (64 * i + lane) * EPL, v = e < RPW * N / 2 ? e : 0;
      off[i] = at(v / (N / 2), v % (N / 2));
    }
    offn = at(lane % RPW, N / 2);
  };
  auto issue = [&](int p) {
    const bool two = p >= 3 && p < 7;
    const cpx<T>* pa = xyb + slot_a(p) * fs;
    const cpx<T>* pb = two ? xyb + slot_b(p) * fs : pa;
    auto load = [&](const cpx<T>* g, cpx<T>* l) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                       (__attribute__((address_space(3))) void*)l, 16, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      load(pa + off[i], pre[wv] + 64 * EPL * i);
      if (two) load(pb + off[i], pre[wv] + PB + 64 * EPL * i);
    }
    load((lane / RPW == 1 ? pb : pa) + offn, pre[wv] + 2 * PB);
  };
  const long long rw0 = (long long)blockIdx.x * XW_WAVES + wv;
  if constexpr (DMA) {
    if (rw0 * RPW < nrows) {
      offsets(rw0);
      issue(0);
    }
  }
  for (long long rw = rw0; rw * RPW < nrows; rw += (long long)gridDim.x * XW_WAVES) {
    // a row past the end (in the last wave) computes on a copy of the last
    // row and stores nothing; spare lanes compute what their twin lanes do
    const long long row0 = rw * RPW + half;
    const bool inr = RPW == 1 || row0 < nrows;
    const bool valid = inr && !spare;
    const long long row = inr ? row0 : nrows - 1;
    T U[3][8];
    T acc[NF][8];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      // keep each pair's loads next to its transform (hoisting them all would
      // multiply the live registers)
      __builtin_amdgcn_sched_barrier(0);
      const bool dxA = p == 6;
      const bool sameB = p < 3;
      const bool hasB = p < 7;
      const long long rb = DMA ? 0 : xw_row_base(row, a.ny, nkxp, blk);
      const cpx<T>* pa = xyb + slot_a(p) * fs + rb;
      const cpx<T>* pb = xyb + slot_b(p) * fs + rb;
      if constexpr (DMA) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): pair p is there
      cpx<T> r[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int k = t + S * m;
        const int kk = k <= N / 2 ? k : N - k;
        const T kx = (kk == N / 2) ? T(0) : kxs * (T)kk;
        cpx<T> A, B = zero<T>();
        if constexpr (DMA) {
          // (m = 4: the lane of index 0 holds the Nyquist column)
          const cpx<T>* at = pre[wv] + half * (N / 2) + (m < 4 ? k : N - k);
          const cpx<T>* an = pre[wv] + 2 * PB + half * EPL;
          const bool nyq = m == 4 && t == 0;
          A = *(nyq ? an : at);
          if (hasB && !sameB) B = *(nyq ? an + RPW * EPL : at + PB);
        } else {
          A = pa[xo[m]];
          if (hasB && !sameB) B = pb[xo[m]];
        }
        if (sameB) B = mul_i(A) * kx;
        if (dxA) A = mul_i(A) * kx;
        if (kk == 0 || kk == N / 2) {
          A.y = T(0);
          B.y = T(0);
        }
        // Z[k] = A + i B (k <= N/2), conj(A) + i conj(B) (k > N/2); inverse via conj
        const cpx<T> Z = (k <= N / 2) ? mk(A.x - B.y, A.y + B.x) : mk(A.x + B.y, B.x - A.y);
        r[m] = conj(Z);
      }
      if constexpr (DMA) {
        // the next pair lands during this one's transform, behind its last reads
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        if (p + 1 < NP) {
          issue(p + 1);
        } else {
          const long long next = rw + (long long)gridDim.x * XW_WAVES;
          if (next * RPW < nrows) {
            offsets(next);
            issue(0);
          }
        }
      }
      wave_fft<T, N>(r, buf, tw, t);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const T va = r[m].x * sc, vb = -r[m].y * sc;
        if (p < 3) {
          U[p][m] = va;
          acc[p][m] = -U[0][m] * vb;        // -u dq_p/dx (U[0] set by pair 0)
        } else if (p < 6) {
          acc[p - 3][m] -= U[1][m] * va;    // -v dq/dy
          acc[p - 3][m] -= U[2][m] * vb;    // -w dq/dz
        } else if (p == 6) {
          acc[TH][m] = -U[0][m] * va;
          acc[TH][m] -= U[1][m] * vb;
        } else {
          acc[TH][m] -= U[2][m] * va;
        }
      }
      if (p == 4) {
        cpx<T> z[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) z[m] = mk(acc[0][m], acc[1][m]);
        xw_forward<T, N>(z, buf, tw, t, nl, fs, row, nkxp, 0, true, valid);
      }
      if (p == NP - 1) {
        // the last field(s): 2 and theta together, or 2 alone
        cpx<T> z[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) z[m] = mk(acc[2][m], NF == 4 ? acc[TH][m] : T(0));
        xw_forward<T, N>(z, buf, tw, t, nl, fs, row, nkxp, 2, NF == 4, valid);
      }
    }
    // (the next row's loads stay behind this row's last transform)
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ---------------------------------------------------------------- helpers
__global__ void k_fill(cpx<double>* p, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = zero<double>();
}

// Remove the physical mean of a mixed-space field: the (0,0) pencil holds
// sum_xy at every z, so subtract its z-average from every z.
__global__ void k_sub_mean00(cpx<double>* pmix, long long npen, int nz) {
  __shared__ double part[256];
  double s = 0.0;
  for (int z = threadIdx.x; z < nz; z += blockDim.x) s += pmix[(long long)z * npen].x;
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < (int)blockDim.x; ++i) t += part[i];
    part[0] = t / nz;
  }
  __syncthreads();
  const double m = part[0];
  for (int z = threadIdx.x; z < nz; z += blockDim.x) pmix[(long long)z * npen].x -= m;
}

// ---------------------------------------------------------------- launchers
// Compiled plans (launch_y).
static bool y_compiled(const YArgs& a) {
  return y_wide_tiles(a) || (a.ny == 256 && plan_is(a.pl, {8, 8, 4})) ||
         (a.ny == 192 && plan_is(a.pl, {8, 8, 3})) || (a.ny == 128 && plan_is(a.pl, {8, 8, 2})) ||
         (a.ny == 96 && plan_is(a.pl, {8, 4, 3})) || (a.ny == 64 && plan_is(a.pl, {8, 8}));
}

// Lines per tile: 4 or, at 512 points, 8 by choice; 8 over 256 threads for the
// shorter compiled plans and for run-time plans up to Y_DYN8 points, whose stages
// of ny / radix butterflies per line leave most threads idle with 4 lines (at 84
// points 48 to 112 of 256, at 128 64 of 256 in a radix-8 stage), and whose tiles are
// then whole 128-byte lines in FP64.  A channel solve of 32 x 32 x 33 with them: 1.64 -> 1.48 ms;
// back with d/dy, back, forward at 256 x 256 x 257 with theta 0.437, 0.280, 0.219 ->
// 0.382, 0.252, 0.216 ms, mixed (three fields) 0.219, 0.160, 0.125 -> 0.167, 0.132,
// 0.102; 128: 0.054, 0.040, 0.036 -> 0.049, 0.041, 0.033; 96: 0.027, 0.020, 0.021 ->
// 0.024, 0.017, 0.018.  Not 192 points in FP64: three such workgroups per CU, 0.166,
// 0.126, 0.093 -> 0.172, 0.124, 0.100.  Above Y_DYN8 8 lines leave one or two
// workgroups per CU: 96 x 200 x 105 0.083, 0.055, 0.053 -> 0.106, 0.068, 0.068, mixed
// 0.047, 0.034, 0.034 -> 0.058, 0.037, 0.038.
int y_tile_lines(const YArgs& a, size_t real) {
  if (y_wide_tiles(a)) return a.lines == 8 ? 8 : YL;
  if (y_compiled(a)) return a.ny == 192 && real == 8 ? YL : 8;
  return a.ny <= Y_DYN8 ? 8 : YL;
}

template <typename T>
void launch_y(const YArgs& a, bool big, bool inv, int mode, const cpx<T>* src, cpx<T>* dst,
              cpx<T>* dst2, long long sfs, long long dfs, int nplanes, int nfields,
              hipStream_t st) {
  const int L = y_tile_lines(a, sizeof(T));
  const bool compiled = y_compiled(a);
  const long long nlines = (long long)nplanes * a.nkxp;
  const long long ntiles = (nlines + L - 1) / L;
  const size_t sh = y_lds_bytes(a.ny, a.pl.tsize, sizeof(cpx<T>), L);
  const long long yg = a.grid > 0 ? a.grid : Y_GRID;
  // fewer tiles than the persistent grid: one workgroup per tile, rounded up
  // to whole chunks of 64 so that the XCD-aware order still applies
  long long gx = ntiles < yg ? ntiles : yg;
  if (gx < yg && gx % 64) gx = std::min(yg, (gx + 63) / 64 * 64);
  dim3 grid((unsigned)gx, nfields);
  const int iv = inv ? 1 : 0;
#define FCNS_YN(FPV, OWNV, LV, NTV)                                                         \
  do {                                                                                      \
    if (a.noprefetch)                                                                       \
      FCNS_LAUNCH((k_y<T, FPV, OWNV, false, LV, NTV>), grid, dim3(NTV), sh, st, a, src, dst, \
                  dst2, sfs, dfs, nlines, iv, mode);                                        \
    else                                                                                    \
      FCNS_LAUNCH((k_y<T, FPV, OWNV, true, LV, NTV>), grid, dim3(NTV), sh, st, a, src, dst,  \
                  dst2, sfs, dfs, nlines, iv, mode);                                        \
  } while (0)
#define FCNS_Y(FPV, OWNV) FCNS_YN(FPV, OWNV, YL, YNT)
  if (y_wide_tiles(a)) {
    using P512 = SPlan<8, 8, 8>;
    if (L == 8)
      FCNS_YN(P512, 8, 8, 512);
    else
      FCNS_Y(P512, 8);
  } else if (compiled && a.ny == 256) {
    using P256 = SPlan<8, 8, 4>;
    FCNS_YN(P256, 8, 8, 256);
  } else if (compiled && a.ny == 192) {
    using P192 = SPlan<8, 8, 3>;
    if constexpr (sizeof(T) == 4)
      FCNS_YN(P192, 6, 8, 256);
    else
      FCNS_Y(P192, 3);
  } else if (compiled && a.ny == 128) {
    using P128 = SPlan<8, 8, 2>;
    FCNS_YN(P128, 4, 8, 256);
  } else if (compiled && a.ny == 96) {
    using P96 = SPlan<8, 4, 3>;
    FCNS_YN(P96, 3, 8, 256);
  } else if (compiled) {
    using P64 = SPlan<8, 8>;
    FCNS_YN(P64, 2, 8, 256);
  } else if (L == 8) {
    const int pm = prime_form(a.pl, big, L, YNT);
    if (a.ny <= 128)
      FCNS_PM_SWITCH(pm, FCNS_YN(DynPlan<PM>, 4, 8, 256))
    else
      FCNS_PM_SWITCH(pm, FCNS_YN(DynPlan<PM>, 6, 8, 256))
  } else {
    const int pm = prime_form(a.pl, big, L, YNT);
    if (a.ny <= 256)
      FCNS_PM_SWITCH(pm, FCNS_Y(DynPlan<PM>, 4))
    else if (a.ny <= 512)
      FCNS_PM_SWITCH(pm, FCNS_Y(DynPlan<PM>, 8))
    else
      FCNS_PM_SWITCH(pm, FCNS_Y(DynPlan<PM>, 16))
  }
#undef FCNS_Y
#undef FCNS_YN
}
template void launch_y<double>(const YArgs&, bool, bool, int, const cpx<double>*, cpx<double>*,
                               cpx<double>*, long long, long long, int, int, hipStream_t);
template void launch_y<float>(const YArgs&, bool, bool, int, const cpx<float>*, cpx<float>*,
                              cpx<float>*, long long, long long, int, int, hipStream_t);

template <typename T, int NF, int N>
static void launch_x_nlw(const XArgs& a, dim3 grid, const cpx<T>* xyb, cpx<T>* nl, long long fs,
                         long long nrows, hipStream_t st) {
#define FCNS_XD(BLKV, DMAV)                                                                 \
  FCNS_LAUNCH((k_x_nlw<T, NF, N, BLKV, DMAV>), grid, dim3(64 * XW_WAVES), 0, st, a, xyb, nl, \
              fs, nrows)
  if constexpr (x_direct<T, NF, N>()) {
    if (x_direct_pays<T, NF, N>(grid.x)) {
      if (a.blk_in) FCNS_XD(true, true); else FCNS_XD(false, true);
      return;
    }
  }
  if (a.blk_in) FCNS_XD(true, false); else FCNS_XD(false, false);
#undef FCNS_XD
}

template <typename T, class FP, int RR, int NT, int CC>
static void launch_x_nl_v(const XArgs& a, const cpx<T>* xyb, cpx<T>* nl, long long fs,
                          long long nrows, int nfields, hipStream_t st) {
  dim3 grid((unsigned)((nrows + RR - 1) / RR));
  const size_t sh = ((size_t)a.pl.tsize + 2 * (RR / 2) * x_ls(a.nx)) * sizeof(cpx<T>);
  FCNS_LAUNCH((k_x_nl<T, FP, RR, NT, CC>), grid, dim3(NT), sh, st, a, xyb, nl, fs, nrows,
              nfields);
}

bool x_reads_blocked(const XArgs& a) { return x_wave_rows(a.nx) && a.variant == 0; }

// nx = 512, 256, 192, 128, 96, 64 and 32: wave-level rows (variant 0) or the tiled kernels; other
// nx: three quantities at a time over 8 rows (variant 0, short rows), 4 rows x
// 256 threads (variant 0 beyond those, and 1) or 8 rows x 512 threads (variant 2),
// with compile-time plans for 512 and 256; nx <= 256: 8 rows x nx threads
// (variant 3)
template <typename T>
void launch_x_nl(const XArgs& a, bool big, const cpx<T>* xyb, cpx<T>* nl, long long fs,
                 long long nrows, int nfields, hipStream_t st) {
  if (a.variant == 3 && a.nx <= 256) {
    // short rows: 8 rows (4 complex lines) per workgroup and one thread per
    // column (a radix-8 stage keeps half the threads busy; 4 or 16 rows, or
    // 4 rows over 256 threads, measured slower)
    const int nt = (a.nx + 63) / 64 * 64;
    const int pm = prime_form(a.pl, big, 4, nt);
#define FCNS_XS(NTV)                                                                        \
  do {                                                                                      \
    FCNS_PM_SWITCH(pm, (launch_x_nl_v<T, DynPlan<PM>, 8, NTV, 1>(a, xyb, nl, fs, nrows,     \
                                                                 nfields, st)))             \
  } while (0)
    if (nt == 64)
      FCNS_XS(64);
    else if (nt == 128)
      FCNS_XS(128);
    else if (nt == 192)
      FCNS_XS(192);
    else
      FCNS_XS(256);
#undef FCNS_XS
  } else if (a.variant == 2 && a.nx <= 512) {
    if (a.nx == 512 && plan_is(a.pl, {8, 8, 8}))
      launch_x_nl_v<T, SPlan<8, 8, 8>, 8, 512, 1>(a, xyb, nl, fs, nrows, nfields, st);
    else
      FCNS_PM_SWITCH(prime_form(a.pl, big, 4, 512),
                     (launch_x_nl_v<T, DynPlan<PM>, 8, 512, 1>(a, xyb, nl, fs, nrows, nfields, st)))
  } else if (x_wave_rows(a.nx) && a.variant == 0) {
    // wave-level rows; enough workgroups to fill the chip several times
    const long long rpw = 64 / (a.nx / 8);
    const long long need = (nrows + rpw * XW_WAVES - 1) / (rpw * XW_WAVES);
    dim3 grid((unsigned)(need < 4096 ? need : 4096));
#define FCNS_XW(NFV, NV) launch_x_nlw<T, NFV, NV>(a, grid, xyb, nl, fs, nrows, st)
    if (a.nx == 512 && nfields == 4)
      FCNS_XW(4, 512);
    else if (a.nx == 512 && a.blk_in)
      FCNS_LAUNCH((k_x_nlw_q<T, 3, 512, true>), grid, dim3(64 * XW_WAVES), 0, st, a, xyb, nl, fs,
                  nrows);
    else if (a.nx == 512)
      FCNS_LAUNCH((k_x_nlw_q<T, 3, 512, false>), grid, dim3(64 * XW_WAVES), 0, st, a, xyb, nl, fs,
                  nrows);
    else if (a.nx == 256 && nfields == 4)
      FCNS_XW(4, 256);
    else if (a.nx == 256)
      FCNS_XW(3, 256);
    else if (a.nx == 192 && nfields == 4)
      FCNS_XW(4, 192);
    else if (a.nx == 192)
      FCNS_XW(3, 192);
    else if (a.nx == 128 && nfields == 4)
      FCNS_XW(4, 128);
    else if (a.nx == 128)
      FCNS_XW(3, 128);
    else if (a.nx == 96 && nfields == 4)
      FCNS_XW(4, 96);
    else if (a.nx == 96)
      FCNS_XW(3, 96);
    else if (a.nx == 64 && nfields == 4)
      FCNS_XW(4, 64);
    else if (a.nx == 64)
      FCNS_XW(3, 64);
    else if (nfields == 4)
      FCNS_XW(4, 32);
    else
      FCNS_XW(3, 32);
#undef FCNS_XW
  } else if (a.variant == 0 && a.nx <= X3_MAXNX && 2 * x3_lds<T>(a) <= 160 * 1024) {
    // (two workgroups per CU, by LDS and by the registers asked for: FP64 rows up to
    // 160 points)
    dim3 grid((unsigned)((nrows + 7) / 8));
#define FCNS_X3(NFV, BV)                                                                      \
  FCNS_LAUNCH((k_x_nl3<T, NFV, BV>), grid, dim3(X3_NT), x3_lds<T>(a), st, a, xyb, nl, fs, nrows)
    const int pm = prime_form(a.pl, big, X3_L, X3_NT);
    if (nfields == 4)
      FCNS_PM_SWITCH(pm, FCNS_X3(4, PM))
    else
      FCNS_PM_SWITCH(pm, FCNS_X3(3, PM))
#undef FCNS_X3
  } else if (a.nx == 512 && plan_is(a.pl, {8, 8, 8}))
    launch_x_nl_v<T, SPlan<8, 8, 8>, 4, 256, 2>(a, xyb, nl, fs, nrows, nfields, st);
  else if (a.nx == 256 && plan_is(a.pl, {8, 8, 4}))
    launch_x_nl_v<T, SPlan<8, 8, 4>, 4, 256, 1>(a, xyb, nl, fs, nrows, nfields, st);
  else
    FCNS_PM_SWITCH(prime_form(a.pl, big, 2, 256),
                   (launch_x_nl_v<T, DynPlan<PM>, 4, 256, 2>(a, xyb, nl, fs, nrows, nfields, st)))
}
template void launch_x_nl<double>(const XArgs&, bool, const cpx<double>*, cpx<double>*, long long,
                                  long long, int, hipStream_t);
template void launch_x_nl<float>(const XArgs&, bool, const cpx<float>*, cpx<float>*, long long,
                                 long long, int, hipStream_t);

void launch_fill(cpx<double>* p, long long n, hipStream_t st) {
  const int nt = 256;
  FCNS_LAUNCH(k_fill, dim3((unsigned)((n + nt - 1) / nt)), dim3(nt), 0, st, p, n);
}

void launch_sub_mean00(cpx<double>* pmix, long long npen, int nz, double, hipStream_t st) {
  FCNS_LAUNCH(k_sub_mean00, dim3(1), dim3(256), 0, st, pmix, npen, nz);
}

}  // namespace fcns
