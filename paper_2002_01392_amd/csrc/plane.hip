// The nonlinear term of small planes in one launch: y back transforms, x pass
// with products and y forward transform of a z plane without leaving the CU.
#include "xwave.hpp"

namespace fcns {

// ---------------------------------------------------------------- one plane, one field
// NL_f = -(u dq_f/dx + v dq_f/dy + w dq_f/dz) of plane z by one workgroup: for
// p = 0, 1, 2 the pair (velocity p, derivative p of q_f) goes through the inverse
// y transform (a wavefront takes 64 / (NY / 8) lines), transposed through LDS, and
// the inverse x transform of its packed rows (xwave.hpp), where the products are
// summed; the sum goes back through the forward x and y transforms.  u, v and w
// are transformed again for every field: a workgroup per (plane, field) fills the
// chip at 65 planes, and the extra transforms cost less than three passes over
// memory and launches.  Bound by the vector units and by the two workgroups that
// some CUs hold at 260.  As four launches and as this one, us (both with the
// events around them): 32 x 32 x 33, three fields 48 -> 15; 64 x 64 x 65, four fields
// 53 -> 32, mixed 45 -> 21; 64 x 64 x 257 121 -> 72; 64 x 32 x 129 128 -> 28.
// The four fields of a plane run on one XCD, which reads u, v and w once.
//
// LDS: a region per wavefront holds its rows of the pair ([field][row][RS]), and
// serves as the exchange buffer of that wavefront's transforms; the Nyquist
// columns (of which the c2r transform takes the real part) of all six quantities
// are transformed first.  64 x 64 in FP64: 77 KB, two workgroups per CU.
template <int NX, int NY>
struct PlaneShape {
  static constexpr int SX = NX / 8, SY = NY / 8;   // lanes per row, per line
  static constexpr int RX = 64 / SX, LY = 64 / SY; // rows, lines per wavefront
  static constexpr int NT = NX * NY / 8, NW = NT / 64;
  static constexpr int XS = XW_BUF / RX;           // slots of a row's exchange
  // of a line's: neighbouring lanes hold neighbouring lines, on different banks
  static constexpr int YS = NY == 64 ? 73 : 37;
  static constexpr int RS = NX == 64 ? 36 : 20;    // row stride (>= NX / 2 + 1)
  static constexpr int cmax(int a, int b) { return a > b ? a : b; }
  static constexpr int REG = cmax(cmax(RX * XS, LY * YS), 2 * RX * RS);
  static constexpr int TWX = 7 * SX, TWY = NX == NY ? 0 : 7 * SY;
};

template <typename T, int NX, int NY>
__global__ __launch_bounds__(NX * NY / 8, NX * NY == 4096 ? 4 : 2) void k_plane_nl(
    XArgs xa, double kys, const cpx<T>* __restrict__ mv, cpx<T>* __restrict__ nl, long long M,
    int nz, int nf) {
  using P = PlaneShape<NX, NY>;
  constexpr int HX = NX / 2;
  __shared__ cpx<T> twx[P::TWX + P::TWY];
  __shared__ cpx<T> reg[P::NW * P::REG];
  __shared__ T nyq[6][NY];
  const int j = blockIdx.x >> 3;
  const int z = (j / nf) * 8 + (blockIdx.x & 7), f = j % nf;
  if (z >= nz) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const cpx<T>* twy = NX == NY ? twx : twx + P::TWX;
  xw_twiddles<T, NX, P::NT>(twx, tid);
  if constexpr (NX != NY) xw_twiddles<T, NY, P::NT>(twx + P::TWX, tid);
  const int nkxp = xa.nkxp;
  const T kxs = (T)xa.kxs;
  const long long zo = (long long)z * NY * nkxp;
  cpx<T>* own = reg + wv * P::REG;
  // quantity h of pair p: the velocity p, or q_f, q_f (times i k~y), dq_f/dz
  auto slot = [&](int p, int h) {
    return mv + (h == 0 ? 2 * p : 2 * f + (p == 2 ? 1 : 0)) * M + zo;
  };
  // this lane in the y transforms (line ly, index ty + SY m) and in the x ones
  const int ly = lane % P::LY, ty = lane / P::LY;
  const int tx = lane % P::SX, rx = lane / P::SX;
  __syncthreads();
  if (wv == P::NW - 1) {
    const int q = ly < 6 ? ly : 0, p = q >> 1;
    const cpx<T>* s = slot(p, q & 1) + HX;
    cpx<T> r[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int ky = ty + P::SY * m;
      cpx<T> v = s[ky * nkxp];
      if (q == 3) v = mul_i(v) * (T)k_odd(ky, NY, kys);
      r[m] = conj(v);
    }
    wave_fft<T, NY>(r, own + ly * P::YS, twy, ty);
    if (ly < 6) {
#pragma unroll
      for (int m = 0; m < 8; ++m) nyq[ly][ty + P::SY * m] = r[m].x * (T(1) / T(NY));
    }
  }
  const int line = wv * P::LY + ly;
  const int h = line / HX, kxl = line % HX;   // (h wave-uniform)
  T acc[8];
#pragma unroll 1
  for (int p = 0; p < 3; ++p) {
    {
      cpx<T> r[8];
      const cpx<T>* s = slot(p, h) + kxl;
      const bool dy = h == 1 && p == 1;
#pragma unroll
      for (int m = 0; m < 8; ++m) r[m] = s[(ty + P::SY * m) * nkxp];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        if (dy) r[m] = mul_i(r[m]) * (T)k_odd(ty + P::SY * m, NY, kys);
        r[m] = conj(r[m]);
      }
      wave_fft<T, NY>(r, own + ly * P::YS, twy, ty);
      __syncthreads();   // every region's last reads are done
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int y = ty + P::SY * m;
        reg[(y / P::RX) * P::REG + (h * P::RX + y % P::RX) * P::RS + kxl] =
            conj(r[m]) * (T(1) / T(NY));
      }
      __syncthreads();
    }
    cpx<T> r[8];
    const T n0 = nyq[2 * p][wv * P::RX + rx], n1 = p == 0 ? T(0) : nyq[2 * p + 1][wv * P::RX + rx];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int k = tx + P::SX * m;
      const int kk = m < 4 ? k : NX - k;
      const bool ny = m == 4 && tx == 0;
      const int ks = m < 4 ? k : (ny ? 0 : kk);
      cpx<T> A = own[rx * P::RS + ks], B = own[(P::RX + rx) * P::RS + ks];
      if (p == 0) B = mul_i(B) * (kxs * (T)ks);
      if (m == 0 && tx == 0) {
        A.y = T(0);
        B.y = T(0);
      }
      if (ny) {
        A = mk(n0, T(0));
        B = mk(n1, T(0));
      }
      // Z[k] = A + i B (k <= N/2), conj(A) + i conj(B) (k > N/2); inverse via conj
      const cpx<T> Z = m < 4 ? mk(A.x - B.y, A.y + B.x) : mk(A.x + B.y, B.x - A.y);
      r[m] = conj(Z);
    }
    wave_sync();
    wave_fft<T, NX>(r, own + rx * P::XS, twx, tx);
    const T sc = T(1) / T(NX);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const T va = r[m].x * sc, vb = -r[m].y * sc;
      acc[m] = p == 0 ? -va * vb : acc[m] - va * vb;
    }
  }
  {
    cpx<T> r[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) r[m] = mk(acc[m], T(0));
    wave_fft<T, NX>(r, own + rx * P::XS, twx, tx);
    wave_sync();
#pragma unroll
    for (int m = 0; m < 4; ++m) own[rx * P::RS + tx + P::SX * m] = r[m];
    if (tx == 0) own[rx * P::RS + HX] = r[4];
  }
  __syncthreads();
  cpx<T> r[8];
  const bool on = wv * P::LY <= HX;   // wave-uniform
  const bool ok = line <= HX;
  const int kx = ok ? line : HX;
  if (on) {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int y = ty + P::SY * m;
      r[m] = reg[(y / P::RX) * P::REG + (y % P::RX) * P::RS + kx];
    }
  }
  __syncthreads();
  if (on) {
    wave_fft<T, NY>(r, own + ly * P::YS, twy, ty);
    cpx<T>* o = nl + f * M + zo + kx;
    if (ok) {
#pragma unroll
      for (int m = 0; m < 8; ++m) o[(ty + P::SY * m) * nkxp] = r[m];
    }
  }
}

bool plane_fits(const XArgs& a) {
  return (a.nx == 64 || a.nx == 32) && (a.ny == 64 || a.ny == 32);
}

template <typename T>
void launch_plane_nl(const XArgs& a, double kys, const cpx<T>* mv, cpx<T>* nl, long long M, int nz,
                     int nfields, hipStream_t st) {
  const dim3 grid((unsigned)((nz + 7) / 8 * 8 * nfields));
#define FCNS_PL(NXV, NYV)                                                                     \
  FCNS_LAUNCH((k_plane_nl<T, NXV, NYV>), grid, dim3(NXV * NYV / 8), 0, st, a, kys, mv, nl, M, \
              nz, nfields)
  if (a.nx == 64) {
    if (a.ny == 64) FCNS_PL(64, 64); else FCNS_PL(64, 32);
  } else {
    if (a.ny == 64) FCNS_PL(32, 64); else FCNS_PL(32, 32);
  }
#undef FCNS_PL
}
template void launch_plane_nl<double>(const XArgs&, double, const cpx<double>*, cpx<double>*,
                                      long long, int, int, hipStream_t);
template void launch_plane_nl<float>(const XArgs&, double, const cpx<float>*, cpx<float>*,
                                     long long, int, int, hipStream_t);

}  // namespace fcns
