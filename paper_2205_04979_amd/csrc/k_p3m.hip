// Particle-particle particle-mesh electrostatics (Appendix A.2.4, Eq. coulomb_force):
// the same raw Coulomb sums S_i as the direct kernels, for the lattice that is
// periodic in x (period L) and unbounded across the pipe section, in O(N log N).
//
// Split (Gaussian): 1/r = erfc(a r)/r + erf(a r)/r.  Long range: the erf part,
// on a mesh of nx x P x P nodes (x periodic, hx = L/nx; y and z: nc nodes across
// [-R, R] with one spare node on each side, hy = 2R/(nc - 3), zero-padded to
// P = 2 nc for the aperiodic convolution), with triangular-shaped-cloud (TSC)
// charge assignment and field interpolation and a Green's function that is the
// erf field of a unit charge summed over the x images and divided by the squared
// TSC transfer function.  Short range: Coulomb's law (with the overlap clamp of
// the direct sum) minus the erf field, over nearest-image pairs closer than
// r_max, found through a cell list with cells of at least r_max.
//
// Charge assignment adds 64-bit fixed-point weights with integer atomics (order
// independent), the FFTs are Cooley-Tukey passes over mesh lines staged in LDS,
// and the short-range sum is a gather over cell-sorted neighbours in a fixed
// order, so results are bitwise reproducible.  Charge and fields are real, so
// the spectra are kept for kz <= P/2 only.  The mesh holds complex values in the
// form's precision (FP32 form: float2, half the bytes of every mesh pass; FP64
// form: double2); the Green's function is always built and transformed in FP64
// and only then rounded to the mesh type.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace depo {

namespace {

constexpr int kFftLds = 2048;   // complex values per workgroup of the set-up FFT (32 KB of LDS)
constexpr int kTwiddles = 1024; // longest line

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <class T> __device__ __forceinline__ T cplx(double re, double im);
template <> __device__ __forceinline__ double2 cplx<double2>(double re, double im) { return make_double2(re, im); }
template <> __device__ __forceinline__ float2 cplx<float2>(double re, double im) {
  return make_float2((float)re, (float)im);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }

// the three field components at a node
template <class T> using FieldT = typename std::conditional<sizeof(T) == 8, float4, double4>::type;
// mesh element of a form
template <class Real> using MeshT = typename std::conditional<sizeof(Real) == 4, float2, double2>::type;

// Continuous mesh coordinates of particle i (x periodic in [0, nx); y, z in [1, nc - 2]).
template <class Real>
__device__ __forceinline__ void mesh_coords(const State<Real> &st, const Phys &ph, const P3mDev &m, int i, double &gx,
                                            double &gy, double &gz) {
  using SPos = typename std::make_signed<typename Prec<Real>::Pos>::type;
  const double x = ((double)st.px[i] + (double)st.rx[i]) * ph.ux;
  const double y = ((double)(SPos)st.py[i] + (double)st.ry[i]) * ph.ur;
  const double z = ((double)(SPos)st.pz[i] + (double)st.rz[i]) * ph.ur;
  gx = x / m.hx;
  if (gx >= m.nx) gx -= m.nx;
  if (gx < 0.0) gx += m.nx;
  gy = (y + ph.R) / m.hy + 1.0;
  gz = (z + ph.R) / m.hy + 1.0;
}

__device__ __forceinline__ void tsc(double g, int &i, double (&w)[3]) {
  const double c = floor(g + 0.5);
  const double dl = g - c;
  i = (int)c;
  w[0] = 0.5 * (0.5 - dl) * (0.5 - dl);
  w[1] = 0.75 - dl * dl;
  w[2] = 0.5 * (0.5 + dl) * (0.5 + dl);
}

// Erf field of a unit charge at displacement (dx, dy, dz), summed over the x images n = -M..M: component
// comp into the complex mesh out, or (comp < 0) the three into real meshes.
__global__ void k_p3m_green(P3mDev m, double L, int images, int comp, double2 *__restrict__ out,
                            double *__restrict__ rx_, double *__restrict__ ry_, double *__restrict__ rz_) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)m.nx * m.P * m.P;
  if (e >= total) return;
  const int iz = (int)(e % m.P), iy = (int)((e / m.P) % m.P), ix = (int)(e / ((int64_t)m.P * m.P));
  double dx = ix * m.hx;
  if (dx >= 0.5 * L) dx -= L;
  const double dy = (iy < m.P / 2 ? iy : iy - m.P) * m.hy;
  const double dz = (iz < m.P / 2 ? iz : iz - m.P) * m.hy;
  const double a = m.alpha, c2 = 2.0 * m.alpha / sqrt(M_PI);
  double ex = 0.0, ey = 0.0, ez = 0.0;
  for (int n = -images; n <= images; ++n) {
    const double rx = dx + n * L;
    const double r2 = rx * rx + dy * dy + dz * dz;
    if (r2 <= 0.0) continue;
    const double r = sqrt(r2);
    const double mag = erf(a * r) / r2 - c2 * exp(-a * a * r2) / r;   // |E_l|
    const double f = mag / r;
    ex += f * rx;
    ey += f * dy;
    ez += f * dz;
  }
  if (comp < 0) {
    rx_[e] = ex;
    ry_[e] = ey;
    rz_[e] = ez;
  } else {
    out[e] = make_double2(comp == 0 ? ex : (comp == 1 ? ey : ez), 0.0);
  }
}

__global__ void k_p3m_complex(int64_t n, const double *__restrict__ in, double2 *__restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) out[e] = make_double2(in[e], 0.0);
}

// Divide the transformed Green's functions by the squared TSC transfer sinc^3 per axis.
__device__ __forceinline__ double sinc_pi(double u) { return u == 0.0 ? 1.0 : sin(M_PI * u) / (M_PI * u); }

__device__ __forceinline__ double tsc_inv_transfer2(const P3mDev &m, int64_t e) {
  const int iz = (int)(e % m.P), iy = (int)((e / m.P) % m.P), ix = (int)(e / ((int64_t)m.P * m.P));
  auto freq = [](int i, int n) { return (double)(i < (n + 1) / 2 ? i : i - n) / n; };   // cycles per node
  const double sx = sinc_pi(freq(ix, m.nx)), sy = sinc_pi(freq(iy, m.P)), sz = sinc_pi(freq(iz, m.P));
  const double W = sx * sx * sx * sy * sy * sy * sz * sz * sz;
  return 1.0 / (W * W);
}

// One transformed FP64 component, deconvolved, in the half-spectrum layout and the mesh type.
template <class T>
__global__ void k_p3m_deconv(P3mDev m, const double2 *__restrict__ g, T *__restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t KZ = m.P / 2, main = m.nx * m.xs, x = e / m.xs, r = e % m.xs;
  if (e >= main + (int64_t)m.nx * m.P) return;
  if (e < main && r >= m.P * KZ) return;   // padding
  const int64_t f = e < main ? (x * m.P + r / KZ) * m.P + r % KZ : (e - main) * m.P + KZ;   // in the full mesh
  const double inv = tsc_inv_transfer2(m, f);
  out[e] = cplx<T>(g[f].x * inv, g[f].y * inv);
}

// exp(2 pi i k / kTwiddles), k < kTwiddles / 2
template <class T> __global__ void k_p3m_twiddles(T *__restrict__ tw) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= kTwiddles / 2) return;
  double s, c;
  sincospi(2.0 * k / kTwiddles, &s, &c);
  tw[k] = cplx<T>(c, s);
}

// Set-up transform of a whole FP64 mesh: complex FFT of length n = 2^log2n along lines, line l starting
// at l * line_stride (inner lines, one apart, in runs of 2^log2inner) with points point_stride apart.  A
// workgroup transforms kFftLds / n lines through LDS (bit-reversed load, in-place butterflies).
constexpr int kFftLog2Lds = 11;
static_assert((1 << kFftLog2Lds) == kFftLds, "kFftLds is 2^kFftLog2Lds");

__global__ __launch_bounds__(256) void k_fft_lines(double2 *__restrict__ data, int log2n, int log2inner,
                                                   int64_t line_stride, int64_t point_stride) {
  __shared__ double2 buf[kFftLds];
  __shared__ double2 tw[kFftLds / 2];
  const int n = 1 << log2n;
  const int log2lpw = kFftLog2Lds - log2n;   // lines per workgroup: 2^log2lpw
  const int64_t l0 = (int64_t)blockIdx.x << log2lpw;
  const int64_t inner_mask = ((int64_t)1 << log2inner) - 1;
  for (int k = threadIdx.x; k < n / 2; k += blockDim.x) {
    double s, c;
    sincospi(2.0 * k / n, &s, &c);
    tw[k] = make_double2(c, -s);
  }
  auto addr = [&](int line, int p) {
    const int64_t l = l0 + line;
    return (l >> log2inner) * line_stride + (l & inner_mask) + (int64_t)p * point_stride;
  };
  const bool along = point_stride == 1;   // consecutive threads along the lines, or across them
  auto line_of = [&](int e) { return along ? e >> log2n : e & ((1 << log2lpw) - 1); };
  auto point_of = [&](int e) { return along ? e & (n - 1) : e >> log2lpw; };
  for (int e = threadIdx.x; e < kFftLds; e += blockDim.x) {
    const int line = line_of(e), p = point_of(e);
    buf[(line << log2n) + (int)(__brev((unsigned)p) >> (32 - log2n))] = data[addr(line, p)];
  }
  __syncthreads();
  // radix-2 stages lg and lg + 1 in one go: groups of 4 points (i0, i0 + h, i0 + 2h, i0 + 3h), h = 2^(lg-1)
  int lg = 1;
  for (; lg + 1 <= log2n; lg += 2) {
    const int half = 1 << (lg - 1);
    for (int b = threadIdx.x; b < kFftLds / 4; b += blockDim.x) {
      const int line = b >> (log2n - 2), k = b & ((n >> 2) - 1);
      const int pos = k & (half - 1);
      const int i0 = (line << log2n) + ((k >> (lg - 1)) << (lg + 1)) + pos;
      const double2 w1 = tw[pos << (log2n - lg)];
      const double2 w2a = tw[pos << (log2n - lg - 1)], w2b = tw[(pos + half) << (log2n - lg - 1)];
      const double2 a0 = buf[i0], a1 = buf[i0 + half], a2 = buf[i0 + 2 * half], a3 = buf[i0 + 3 * half];
      double2 v = cmul(w1, a1);
      const double2 b0 = cadd(a0, v), b1 = csub(a0, v);
      v = cmul(w1, a3);
      const double2 b2 = cadd(a2, v), b3 = csub(a2, v);
      v = cmul(w2a, b2);
      buf[i0] = cadd(b0, v);
      buf[i0 + 2 * half] = csub(b0, v);
      v = cmul(w2b, b3);
      buf[i0 + half] = cadd(b1, v);
      buf[i0 + 3 * half] = csub(b1, v);
    }
    __syncthreads();
  }
  if (lg == log2n) {   // odd log2n: the last stage
    const int half = 1 << (lg - 1);
    for (int b = threadIdx.x; b < kFftLds / 2; b += blockDim.x) {
      const int i = ((b >> (log2n - 1)) << log2n) + (b & (half - 1));
      const double2 u = buf[i], v = cmul(tw[b & (half - 1)], buf[i + half]);
      buf[i] = cadd(u, v);
      buf[i + half] = csub(u, v);
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < kFftLds; e += blockDim.x) {
    const int line = line_of(e), p = point_of(e);
    data[addr(line, p)] = buf[(line << log2n) + p];
  }
}

// ---- the step's transforms
//
// Charge and fields are real, so half a spectrum holds everything: kz < P/2 as [x][y][kz], xs values per x,
// and the plane kz = P/2 behind it as [x][y].  The passes, each reading and writing its lines once:
//   charge   z: real rows, half of their spectra stored
//   y, x     forward, the rows y >= nc taken as zero
//   fields   z: the products with the Green's functions, E_x + i E_y as one set of lines and E_z as another,
//            both halves of each line from the half spectrum; only the points z < nc are stored
//   y        inverse, only the rows y < nc stored
//   x        inverse, the lines y, z < nc; the three components of a node side by side for the interpolation
// Order, butterflies, packing and rounding are those of a transform over the full spectra, bit for bit: the
// upper half of each is the conjugate of the lower one in floating point too, since the twiddles are symmetric
// to the last bit and the multiplications round alike under a change of sign.  (Shorter by a tenth with other
// roundings -- two rows in one line, the products between the x passes -- but then a step in FP32 differs in
// its last bits, and over 100 steps of 2^20 particles a pair that nearly collides makes 1e-2 of it.)
// Bound by memory: at 256 x 256 x 256 (128 nodes across) 1.2 GB a step where the full complex spectra
// moved 1.9 GB.  The y and x passes take as many lines at a time as make 128 bytes (a strided segment),
// fewer where the lines are long; the z passes enough to fill the chip with workgroups.  Measured, a step's
// transforms: 256^3 568 -> 289 us, 128^3 105 -> 67 us (nine passes over full spectra before).  Loads are issued
// ahead of the butterflies, none under a branch.
constexpr int kFftMaxValues = 32768;   // bytes of line data per workgroup in the y and x passes, at most
constexpr int kZTile = 1024;           // values per workgroup of the charge pass and of the spectrum per workgroup of the fields z pass
constexpr int kZThreads = 256;
// values each thread of the y and x passes holds
template <class T> constexpr int kFftPer = 64 / sizeof(T);

// An element's place within a line in LDS, and a line's: spread over the banks for the power-of-two strides
// of the stages and of neighbouring lines.
__device__ __forceinline__ int fft_at(int i) { return i + (i >> 4); }
__device__ __forceinline__ int fft_line(int n) { return n + (n >> 4) + 1; }
constexpr int fft_lds(int values) { return values + values / 8; }   // room for `values` in lines of 16 at least

// tw[k] = exp(SIGN 2 pi i k / n), k < n / 2
template <int SIGN, class T>
__device__ __forceinline__ void fft_twiddles(T *tw, const T *__restrict__ table, int log2n) {
  for (int k = threadIdx.x; k < 1 << (log2n - 1); k += blockDim.x) {
    T w = table[k * (kTwiddles >> log2n)];
    if (SIGN < 0) w.y = -w.y;
    tw[k] = w;
  }
}

// In-place transforms of bit-reversed lines, radix-2 stages in pairs; begins and ends with a barrier.
template <class T>
__device__ __forceinline__ void fft_stages(T *buf, const T *tw, int log2n, int lines) {
  const int n = 1 << log2n, ls = fft_line(n);
  __syncthreads();
  int lg = 1;
  for (; lg + 1 <= log2n; lg += 2) {
    // groups of 4 points (i0, i0 + h, i0 + 2h, i0 + 3h), h = 2^(lg-1), through both stages in registers
    const int half = 1 << (lg - 1);
    for (int b = threadIdx.x; b < lines << (log2n - 2); b += blockDim.x) {
      const int k = b & ((n >> 2) - 1), pos = k & (half - 1);
      T *l = buf + (b >> (log2n - 2)) * ls;
      const int i0 = ((k >> (lg - 1)) << (lg + 1)) + pos;
      const int p0 = fft_at(i0), p1 = fft_at(i0 + half), p2 = fft_at(i0 + 2 * half), p3 = fft_at(i0 + 3 * half);
      const T w1 = tw[pos << (log2n - lg)];
      const T w2 = tw[pos << (log2n - lg - 1)], w3 = tw[(pos + half) << (log2n - lg - 1)];
      const T a0 = l[p0], a1 = l[p1], a2 = l[p2], a3 = l[p3];
      T v = cmul(w1, a1);
      const T b0 = cadd(a0, v), b1 = csub(a0, v);
      v = cmul(w1, a3);
      const T b2 = cadd(a2, v), b3 = csub(a2, v);
      v = cmul(w2, b2);
      l[p0] = cadd(b0, v);
      l[p2] = csub(b0, v);
      v = cmul(w3, b3);
      l[p1] = cadd(b1, v);
      l[p3] = csub(b1, v);
    }
    __syncthreads();
  }
  if (lg == log2n) {   // odd log2n: the last stage
    const int half = 1 << (lg - 1);
    for (int b = threadIdx.x; b < lines << (log2n - 1); b += blockDim.x) {
      const int k = b & (half - 1);
      T *l = buf + (b >> (log2n - 1)) * ls;
      const T u = l[fft_at(k)], v = cmul(tw[k], l[fft_at(k + half)]);
      l[fft_at(k)] = cadd(u, v);
      l[fft_at(k + half)] = csub(u, v);
    }
    __syncthreads();
  }
}

__device__ __forceinline__ int fft_rev(int p, int log2n) { return fft_at((int)(__brev((unsigned)p) >> (32 - log2n))); }

// z pass of the charge: rows x nc + y, half of each one's spectrum stored.
template <class T>
__global__ __launch_bounds__(kZThreads) void k_fft_charge(P3mDev m, int log2p, T *__restrict__ spec) {
  __shared__ T buf[fft_lds(kZTile)];
  __shared__ T tw[kTwiddles / 2];
  const int n = 1 << log2p, ls = fft_line(n), nc = m.nc, KZ = n / 2, lines = kZTile >> log2p;
  const int64_t r0 = (int64_t)blockIdx.x * lines;
  fft_twiddles<-1>(tw, (const T *)m.twiddles, log2p);
  for (int e = threadIdx.x; e < kZTile; e += kZThreads) {
    const int line = e >> log2p, p = e & (n - 1);
    T v = cplx<T>(0.0, 0.0);
    if (p < nc) v = cplx<T>((double)(long long)m.qmesh[(r0 + line) * nc + p] / *m.q_scale, 0.0);
    buf[line * ls + fft_rev(p, log2p)] = v;
  }
  fft_stages(buf, tw, log2p, lines);
  T *nyq = spec + m.nx * m.xs;
  for (int e = threadIdx.x; e < kZTile / 2; e += kZThreads) {
    const int line = e >> (log2p - 1), k = e & (KZ - 1);
    const int64_t x = (r0 + line) / nc, y = (r0 + line) % nc;
    spec[x * m.xs + y * KZ + k] = buf[line * ls + fft_at(k)];
    if (k == 0) nyq[x * n + y] = buf[line * ls + fft_at(KZ)];
  }
}

// y pass: lines (x, kz), then those of the plane kz = P/2.  Forward: points beyond nc are zero on the way
// in; inverse: they are not needed on the way out.  blockIdx.y: component.
template <int SIGN, class T>
__global__ __launch_bounds__(512) void k_fft_y(P3mDev m, int log2p, int log2l, int main_blocks, int64_t comp_stride,
                                               T *__restrict__ spec) {
  extern __shared__ char lds[];
  const int n = 1 << log2p, ls = fft_line(n), nc = m.nc, lines = 1 << log2l;
  T *buf = reinterpret_cast<T *>(lds), *tw = buf + lines * ls;
  spec += blockIdx.y * comp_stride;
  fft_twiddles<SIGN>(tw, (const T *)m.twiddles, log2p);
  const bool plane = (int)blockIdx.x >= main_blocks;
  const int l0 = (plane ? blockIdx.x - main_blocks : blockIdx.x) << log2l;
  const int n_lines = plane ? m.nx : m.nx << (log2p - 1);
  // Lines beyond the last are computed from it and not stored, so that no load hangs on a branch.  The
  // threads take points in order: nc is half of them, the first half of each thread's.
  constexpr int PER = kFftPer<T>, HALF = PER / 2;
  auto line_of = [&](int r) { return (int)(threadIdx.x + r * blockDim.x) & (lines - 1); };
  auto point_of = [&](int r) { return (int)(threadIdx.x + r * blockDim.x) >> log2l; };
  const int64_t l = min(l0 + line_of(0), n_lines - 1);   // blockDim is a multiple of lines: one line a thread
  T *o = plane ? spec + m.nx * m.xs + (l << log2p) : spec + (l >> (log2p - 1)) * m.xs + (l & (n / 2 - 1));
  const int log2d = plane ? 0 : log2p - 1;               // distance of a line's points
  T v[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r)
    v[r] = SIGN > 0 || r < HALF ? o[(int64_t)point_of(r) << log2d] : cplx<T>(0.0, 0.0);
#pragma unroll
  for (int r = 0; r < PER; ++r) buf[line_of(r) * ls + fft_rev(point_of(r), log2p)] = v[r];
  fft_stages(buf, tw, log2p, lines);
  if (l0 + line_of(0) >= n_lines) return;
#pragma unroll
  for (int r = 0; r < (SIGN < 0 ? PER : HALF); ++r)
    o[(int64_t)point_of(r) << log2d] = buf[line_of(r) * ls + fft_at(point_of(r))];
}

// x pass of the charge: lines (ky, kz), then those of the plane kz = P/2.
template <class T>
__global__ __launch_bounds__(512) void k_fft_x(P3mDev m, int log2x, int log2p, int log2l, int main_blocks,
                                               T *__restrict__ spec) {
  constexpr int PER = kFftPer<T>;
  extern __shared__ char lds[];
  const int n = 1 << log2x, ls = fft_line(n), lines = 1 << log2l;
  T *buf = reinterpret_cast<T *>(lds), *tw = buf + lines * ls;
  fft_twiddles<-1>(tw, (const T *)m.twiddles, log2x);
  const bool plane = (int)blockIdx.x >= main_blocks;
  const int l0 = (plane ? blockIdx.x - main_blocks : blockIdx.x) << log2l;
  const int n_lines = plane ? 1 << log2p : 1 << (2 * log2p - 1);
  const int64_t dist = plane ? m.P : m.xs, base = plane ? n * m.xs : 0;   // distance of a line's points
  auto line_of = [&](int r) { return (int)(threadIdx.x + r * blockDim.x) & (lines - 1); };
  auto point_of = [&](int r) { return (int)(threadIdx.x + r * blockDim.x) >> log2l; };
  T *o = spec + base + min(l0 + line_of(0), n_lines - 1);   // as in the y pass
  T v[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) v[r] = o[point_of(r) * dist];
#pragma unroll
  for (int r = 0; r < PER; ++r) buf[line_of(r) * ls + fft_rev(point_of(r), log2x)] = v[r];
  fft_stages(buf, tw, log2x, lines);
  if (l0 + line_of(0) >= n_lines) return;
#pragma unroll
  for (int r = 0; r < PER; ++r) o[point_of(r) * dist] = buf[line_of(r) * ls + fft_at(point_of(r))];
}

// x pass of the fields, the last one: lines (y < nc, z < nc) of E_x + i E_y (spec + comp_stride) and of E_z
// (spec + 2 comp_stride) to the field components at the nodes.
template <class T>
__global__ __launch_bounds__(512) void k_fft_field_x(P3mDev m, int log2x, int log2l, int64_t comp_stride,
                                                     const T *__restrict__ spec, FieldT<T> *__restrict__ field) {
  constexpr int PER = kFftPer<T>;
  extern __shared__ char lds[];
  const int n = 1 << log2x, ls = fft_line(n), lines = 1 << log2l;
  T *buf = reinterpret_cast<T *>(lds), *tw = buf + lines * ls;
  fft_twiddles<1>(tw, (const T *)m.twiddles, log2x);
  auto line_of = [&](int r) { return (int)(threadIdx.x + r * blockDim.x) & (lines - 1); };
  auto point_of = [&](int r) { return (int)(threadIdx.x + r * blockDim.x) >> log2l; };
  const int64_t l = ((int64_t)blockIdx.x << log2l) + line_of(0);   // y nc + z: z runs over P / 2 = nc values
  T xy[PER], z[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    xy[r] = spec[comp_stride + l + point_of(r) * m.xs];
    z[r] = spec[2 * comp_stride + l + point_of(r) * m.xs];
  }
#pragma unroll
  for (int r = 0; r < PER; ++r) buf[line_of(r) * ls + fft_rev(point_of(r), log2x)] = xy[r];
  fft_stages(buf, tw, log2x, lines);
#pragma unroll
  for (int r = 0; r < PER; ++r) xy[r] = buf[line_of(r) * ls + fft_at(point_of(r))];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PER; ++r) buf[line_of(r) * ls + fft_rev(point_of(r), log2x)] = z[r];
  fft_stages(buf, tw, log2x, lines);
#pragma unroll
  for (int r = 0; r < PER; ++r)
    field[(int64_t)point_of(r) * m.nc * m.nc + l] =
        FieldT<T>{xy[r].x, xy[r].y, buf[line_of(r) * ls + fft_at(point_of(r))].x, 0};
}

// z pass of the fields, from the charge's half spectrum: E_x + i E_y to spec + comp_stride or E_z (EZ) to
// spec + 2 comp_stride, the points z < nc.  The product a g at (-kx, -ky, -kz) is the conjugate of that
// at (kx, ky, kz) (charge and Green's functions are real on the mesh), so a workgroup takes a row and its
// mirror image (for ky = 0 the rows ky = 0 and P / 2, whose images it reads besides).
template <class T, bool EZ>
__global__ __launch_bounds__(kZThreads) void k_fft_field_z(P3mDev m, int log2p, int64_t comp_stride,
                                                           T *__restrict__ spec) {
  __shared__ T buf[fft_lds(2 * kZTile)];
  __shared__ T tw[kTwiddles / 2];
  const int n = 1 << log2p, ls = fft_line(n), nx = m.nx, KZ = n / 2, units = kZTile >> log2p;
  const int64_t u0 = (int64_t)blockIdx.x * units, main = nx * m.xs;
  const T *__restrict__ ga = (const T *)m.ghat[EZ ? 2 : 0], *__restrict__ gb = (const T *)m.ghat[1];
  fft_twiddles<1>(tw, (const T *)m.twiddles, log2p);
  // unit u: x = u / KZ, y = u % KZ; its row j
  auto row = [&](int64_t u, int j, int &x, int &y) {
    x = (int)(u >> (log2p - 1));
    y = (int)(u & (KZ - 1));
    if (j == 0) return;
    if (y == 0) {
      y = KZ;
    } else {
      x = x == 0 ? 0 : nx - x;
      y = n - y;
    }
  };
  // a g1 + i a g2, or a g1 alone; of the conjugates where mirror is set.  The rounding is written out: left to
  // the compiler, a product and its mirror image share a term and round differently, and the two halves of
  // the spectrum no longer match to the last bit.
  auto mul = [](T a, T g) {
    return T{__builtin_elementwise_fma(a.x, g.x, -(a.y * g.y)), __builtin_elementwise_fma(a.y, g.x, a.x * g.y)};
  };
  auto product = [&](int64_t at, bool mirror) {
    auto conj = [&](T v) { return mirror ? T{v.x, -v.y} : v; };
    const T a = conj(spec[at]), pp = mul(a, conj(ga[at]));
    if constexpr (EZ) {
      return pp;
    } else {
      const T qq = mul(a, conj(gb[at]));
      return T{pp.x - qq.y, pp.y + qq.x};
    }
  };
  for (int e = threadIdx.x; e < units << log2p; e += kZThreads) {
    const int k = e & (KZ - 1), j = (e >> (log2p - 1)) & 1, u = e >> log2p;
    int x, y;
    row(u0 + u, j, x, y);
    const int64_t at = x * m.xs + (int64_t)y * KZ + k;
    T *own = buf + (2 * u + j) * ls;
    own[fft_rev(k, log2p)] = product(at, false);
    if (k == 0) {
      own[fft_rev(KZ, log2p)] = product(main + (int64_t)x * n + y, false);
    } else if ((y & (KZ - 1)) == 0) {
      own[fft_rev(n - k, log2p)] = product((x == 0 ? 0 : nx - x) * m.xs + (int64_t)y * KZ + k, true);
    } else {
      buf[(2 * u + 1 - j) * ls + fft_rev(n - k, log2p)] = product(at, true);
    }
  }
  fft_stages(buf, tw, log2p, 2 * units);
  T *out = spec + (EZ ? 2 : 1) * comp_stride;
  for (int e = threadIdx.x; e < units << log2p; e += kZThreads) {
    const int z = e & (KZ - 1), j = (e >> (log2p - 1)) & 1, u = e >> log2p;
    int x, y;
    row(u0 + u, j, x, y);
    out[x * m.xs + (int64_t)y * KZ + z] = buf[(2 * u + j) * ls + fft_at(z)];
  }
}

// TSC stencil of particle i: centre node (ix unwrapped in [0, nx], iy and iz clamped to
// [1, nc - 2]) and weights; false for a particle without charge.
template <class Real>
__device__ __forceinline__ bool tsc_stencil(const State<Real> &st, const Phys &ph, const P3mDev &m, int i, int &ix,
                                            int &iy, int &iz, double (&wx)[3], double (&wy)[3], double (&wz)[3]) {
  if (st.js[i].q == 0) return false;
  double gx, gy, gz;
  mesh_coords<Real>(st, ph, m, i, gx, gy, gz);
  tsc(gx, ix, wx);
  tsc(gy, iy, wy);
  tsc(gz, iz, wz);
  iy = min(max(iy, 1), m.nc - 2);   // suspended particles stay inside [-R, R]; the clamp only guards
  iz = min(max(iz, 1), m.nc - 2);
  return true;
}

// Fixed-point contribution of a particle to stencil node (a, b, c), units of the per-sample
// bound 2^-62 sum |q~|.
__device__ __forceinline__ unsigned long long tsc_part(double q, const double (&wx)[3], const double (&wy)[3],
                                                       const double (&wz)[3], int a, int b, int c, double qs) {
  return (unsigned long long)__double2ll_rn(q * wx[a] * wy[b] * wz[c] * qs);
}

// Source record of the short-range pass in the FP64 form, in cell-sorted order.
struct __align__(8) SrRec64 {
  uint64_t x;        // fixed-point position: x as the unsigned fraction of L,
  int64_t y, z;      // y and z as signed multiples of the y/z quantum
  double q, d;       // scaled charge, diameter [m]
};

// TSC charge assignment in 64-bit fixed point, one workgroup per brick of 8 x 8 x 8 nodes.  The particles
// that can touch the brick lie in the short-range cells around it; a test in FP32 on their cell-sorted
// records (with a margin far above its rounding) lists them in LDS, and each listed one adds its 27
// contributions, as far as they fall into the brick, by LDS atomics.  Every node is written once, by its own
// brick: no global atomics, nothing to clear.  Integer additions commute, so the mesh does not depend on
// the order.  2^20 particles: 198 -> 96 us, 65,536: 38 -> 13.6 us, against a box in LDS per short-range cell
// with a global atomic per node, which kept 100 of 256 threads busy.
constexpr int kBrick = 8;
constexpr int kAsgThreads = 256;
constexpr int kAsgList = 1024;   // particles listed before they are added

template <class Real>
__global__ __launch_bounds__(kAsgThreads) void k_p3m_assign(State<Real> st, Phys ph, P3mDev m,
                                                            const int32_t *__restrict__ starts,
                                                            const int32_t *__restrict__ sorted,
                                                            unsigned long long *__restrict__ qmesh) {
  __shared__ unsigned long long box[kBrick * kBrick * kBrick];
  __shared__ int32_t list[kAsgList];
  __shared__ int32_t listed;
  const int nb = m.nc / kBrick, tid = threadIdx.x;
  const int b[3] = {(int)blockIdx.x / (nb * nb) * kBrick, (int)blockIdx.x / nb % nb * kBrick,
                    (int)blockIdx.x % nb * kBrick};
  for (int e = tid; e < kBrick * kBrick * kBrick; e += kAsgThreads) box[e] = 0ull;
  if (tid == 0) listed = 0;
  const double qs = *m.q_scale;

  // a stencil centred on node c (the nearest to g) reaches the brick for c in [b - 1, b + 8]: g in
  // [b - 3/2, b + 17/2).  Cells that overlap this (periodic in x; across the section the cells and the
  // stencils of particles outside are clamped alike)
  const double pad = 1e-3;
  const int x0 = (int)floor((b[0] - 1.5 - pad) * m.ncx / m.nx), x1 = (int)floor((b[0] + kBrick + 0.5 + pad) * m.ncx / m.nx);
  int r0[3], r1[3];
  float g0[3], g1[3];
  for (int a = 1; a < 3; ++a) {
    const double lo = b[a] - 1.5 - pad, hi = b[a] + kBrick + 0.5 + pad, per = m.hy / (2.0 * ph.R) * m.ncy;
    r0[a] = min(max((int)floor((lo - 1.0) * per - 1e-6), 0), m.ncy - 1);
    r1[a] = min(max((int)floor((hi - 1.0) * per + 1e-6), 0), m.ncy - 1);
    g0[a] = b[a] == 0 ? -3.0e38f : (float)lo;
    g1[a] = b[a] + kBrick == m.nc ? 3.0e38f : (float)hi;
  }
  const int nxc = min(x1 - x0 + 1, m.ncx);
  const float kx = (float)(m.nx * 0x1p-32), ky = (float)(ph.ur / m.hy), oy = (float)(ph.R / m.hy + 1.0);
  const float xlo = (float)(b[0] - 1.5 - pad), xlen = (float)(kBrick + 2 + 2 * pad), xper = (float)m.nx;

  auto flush = [&]() {   // between barriers
    const int n = listed;
    for (int h = tid; h < n; h += kAsgThreads) {
      const int i = sorted[list[h]];
      int ix, iy, iz;
      double wx[3], wy[3], wz[3];
      if (!tsc_stencil<Real>(st, ph, m, i, ix, iy, iz, wx, wy, wz)) continue;
      const double q = (double)st.js[i].q;
      // first stencil node relative to the brick; along x the period decides
      int ox = ix - 1 - b[0];
      ox = ox < -2 ? ox + m.nx : (ox >= m.nx - 2 ? ox - m.nx : ox);
      const int oy_ = iy - 1 - b[1], oz = iz - 1 - b[2];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if ((unsigned)(ox + a) >= (unsigned)kBrick) continue;
#pragma unroll
        for (int bb = 0; bb < 3; ++bb) {
          if ((unsigned)(oy_ + bb) >= (unsigned)kBrick) continue;
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if ((unsigned)(oz + c) < (unsigned)kBrick)
              atomicAdd(&box[((ox + a) * kBrick + oy_ + bb) * kBrick + oz + c], tsc_part(q, wx, wy, wz, a, bb, c, qs));
        }
      }
    }
  };
  __syncthreads();
  for (int cx = 0; cx < nxc; ++cx) {
    int x = x0 + cx;
    x = x < 0 ? x + m.ncx : (x >= m.ncx ? x - m.ncx : x);
    for (int y = r0[1]; y <= r1[1]; ++y) {
      const int row = (x * m.ncy + y) * m.ncy;
      const int kb = starts[row + r0[2]], ke = starts[row + r1[2] + 1];   // cells along z are one run
      for (int k0 = kb; k0 < ke; k0 += kAsgThreads) {
        const int k = k0 + tid;
        if (k < ke) {
          float gx, gy, gz;
          if constexpr (sizeof(Real) == 4) {
            const float4 r = ((const float4 *)m.rec)[k];
            gx = (float)__float_as_uint(r.x) * kx;
            gy = fmaf(r.y, ky, oy);
            gz = fmaf(r.z, ky, oy);
          } else {
            const SrRec64 r = ((const SrRec64 *)m.rec)[k];
            gx = (float)(uint32_t)(r.x >> 32) * kx;
            gy = fmaf((float)r.y, ky, oy);
            gz = fmaf((float)r.z, ky, oy);
          }
          float tx = gx - xlo;
          tx = tx < 0.0f ? tx + xper : (tx >= xper ? tx - xper : tx);
          // (just below the period is just below the brick: rounding decides)
          if ((tx <= xlen || tx >= xper - 0.01f) && gy >= g0[1] && gy <= g1[1] && gz >= g0[2] && gz <= g1[2])
            list[atomicAdd(&listed, 1)] = k;
        }
        __syncthreads();
        const int n = listed;
        __syncthreads();
        if (n > kAsgList - kAsgThreads) {   // uniform
          flush();
          __syncthreads();
          if (tid == 0) listed = 0;
          __syncthreads();
        }
      }
    }
  }
  __syncthreads();
  flush();
  __syncthreads();
  for (int e = tid; e < kBrick * kBrick * kBrick; e += kAsgThreads)
    qmesh[((int64_t)(b[0] + (e >> 6)) * m.nc + (b[1] + ((e >> 3) & 7))) * m.nc + b[2] + (e & 7)] = box[e];
}

// TSC interpolation of the unnormalised inverse transforms at the particles.
template <class Real>
__global__ void k_p3m_interp(State<Real> st, Phys ph, P3mDev m, const int32_t *__restrict__ order,
                             const FieldT<MeshT<Real>> *__restrict__ E, double *__restrict__ out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;   // cell order, for locality of the mesh reads
  if (k >= ph.N) return;
  const int i = order[k];
  double gx, gy, gz, wx[3], wy[3], wz[3];
  int ix, iy, iz;
  mesh_coords<Real>(st, ph, m, i, gx, gy, gz);
  tsc(gx, ix, wx);
  tsc(gy, iy, wy);
  tsc(gz, iz, wz);
  iy = min(max(iy, 1), m.nc - 2);
  iz = min(max(iz, 1), m.nc - 2);
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    int jx = ix + a - 1;
    jx = jx < 0 ? jx + m.nx : (jx >= m.nx ? jx - m.nx : jx);
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double w = wx[a] * wy[b] * wz[c];
        const auto v = E[((int64_t)jx * m.nc + (iy + b - 1)) * m.nc + (iz + c - 1)];
        s[0] += w * (double)v.x;
        s[1] += w * (double)v.y;
        s[2] += w * (double)v.z;
      }
  }
  const double norm = 1.0 / ((double)m.nx * m.P * m.P);
  for (int c = 0; c < 3; ++c) out[c * (int64_t)ph.N + i] = s[c] * norm;
}

// Short-range cell of a particle (cells of at least r_max; x periodic).
template <class Real>
__device__ __forceinline__ int3 sr_cell(const State<Real> &st, const Phys &ph, const P3mDev &m, int i) {
  using SPos = typename std::make_signed<typename Prec<Real>::Pos>::type;
  const double x = ((double)st.px[i] + (double)st.rx[i]) * ph.ux;
  const double y = ((double)(SPos)st.py[i] + (double)st.ry[i]) * ph.ur;
  const double z = ((double)(SPos)st.pz[i] + (double)st.rz[i]) * ph.ur;
  int cx = (int)(x / ph.L * m.ncx), cy = (int)((y + ph.R) / (2.0 * ph.R) * m.ncy),
      cz = (int)((z + ph.R) / (2.0 * ph.R) * m.ncy);
  cx = min(max(cx, 0), m.ncx - 1);
  cy = min(max(cy, 0), m.ncy - 1);
  cz = min(max(cz, 0), m.ncy - 1);
  return make_int3(cx, cy, cz);
}

// Adds 1 to ctr[key] for every lane of the execution mask with one atomic per distinct key in the wave (the
// particles of a wave often share a cell: the storage follows the cells).  Returns the counter's value
// before the lane's own increment; the lanes of one key take consecutive values in lane order.  The groups
// are found first, so that all their atomics are under way together (one after another: 18.7 us for the
// binning of 65,536 particles, 7.3 us so).
__device__ __forceinline__ int32_t wave_count_add(int32_t *__restrict__ ctr, int key) {
  const int lane = (int)(threadIdx.x & 63);
  uint64_t todo = __builtin_amdgcn_ballot_w64(true), mine = 0;
  while (todo) {
    const int lkey = __builtin_amdgcn_readlane(key, __builtin_ctzll(todo));
    const uint64_t grp = __builtin_amdgcn_ballot_w64(key == lkey);
    if (key == lkey) mine = grp;
    todo &= ~grp;
  }
  const int leader = __builtin_ctzll(mine);
  int32_t base = 0;
  if (lane == leader) base = atomicAdd(ctr + key, (int32_t)__builtin_popcountll(mine));
  return __shfl(base, leader) +
         (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u));
}

// Cell id and sub-cell key of the particle, packed as 64 id + key, and its arrival number in the cell.  The key orders the 4 x 4 x 4
// sub-cells of a cell along a Morton curve (bits: the halves along x, y, z, then the quarters
// within them), so that consecutive particles of the cell-sorted order lie close together.
template <class Real>
__global__ void k_p3m_bin(State<Real> st, Phys ph, P3mDev m, int32_t *__restrict__ cell_of,
                          int32_t *__restrict__ counts, int32_t *__restrict__ arrival) {
  using SPos = typename std::make_signed<typename Prec<Real>::Pos>::type;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ph.N) return;
  const int3 c = sr_cell<Real>(st, ph, m, i);
  const int id = (c.x * m.ncy + c.y) * m.ncy + c.z;
  const double x = ((double)st.px[i] + (double)st.rx[i]) * ph.ux;
  const double y = ((double)(SPos)st.py[i] + (double)st.ry[i]) * ph.ur;
  const double z = ((double)(SPos)st.pz[i] + (double)st.rz[i]) * ph.ur;
  auto quarter = [](double f) { return min(max((int)(4.0 * f), 0), 3); };
  const int qx = quarter(x / ph.L * m.ncx - c.x), qy = quarter((y + ph.R) / (2.0 * ph.R) * m.ncy - c.y),
            qz = quarter((z + ph.R) / (2.0 * ph.R) * m.ncy - c.z);
  const int key = ((qx >> 1) << 5) | ((qy >> 1) << 4) | ((qz >> 1) << 3) | ((qx & 1) << 2) | ((qy & 1) << 1) | (qz & 1);
  cell_of[i] = 64 * id + key;
  arrival[i] = wave_count_add(counts, id);
}

// Exclusive scan of the cell counts by one workgroup; starts[ncell] = N.
__global__ __launch_bounds__(1024) void k_p3m_scan(int32_t ncell, const int32_t *__restrict__ counts,
                                                   int32_t *__restrict__ starts) {
  __shared__ int32_t part[1024];
  const int t = threadIdx.x;
  const int per = (ncell + 1023) / 1024;
  const int b = t * per, e = min(ncell, b + per);
  int32_t s = 0;
  for (int k = b; k < e; ++k) s += counts[k];
  part[t] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int32_t v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int32_t run = part[t] - s;
  for (int k = b; k < e; ++k) {
    starts[k] = run;
    run += counts[k];
  }
  if (t == 1023) starts[ncell] = part[1023];
}

__global__ void k_p3m_scatter(int32_t N, const int32_t *__restrict__ cell_of, const int32_t *__restrict__ arrival,
                              const int32_t *__restrict__ starts, int32_t *__restrict__ sorted) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) sorted[starts[cell_of[i] >> 6] + arrival[i]] = i;
}

// Particles of each cell ordered by (sub-cell key, index): a fixed summation order in which
// consecutive targets of the short-range pass are close together.  The counts are cleared.  One
// workgroup per cell: the cell's keys (sub-cell key, index; distinct) are staged in LDS and each
// particle is written to its rank (the number of smaller keys).  A cell of more than kSortCap
// particles is sorted by one thread.
constexpr int kSortCap = 2048;
__global__ __launch_bounds__(256) void k_p3m_sort(int32_t ncell, const int32_t *__restrict__ starts,
                                                  int32_t *__restrict__ sorted, int32_t *__restrict__ counts,
                                                  const int32_t *__restrict__ cell_of) {
  __shared__ int64_t v[kSortCap];
  const int c = blockIdx.x;
  const int b = starts[c], n = starts[c + 1] - b;
  auto key = [&](int i) { return ((int64_t)(cell_of[i] & 63) << 32) | (int64_t)i; };
  if (threadIdx.x == 0) counts[c] = 0;
  if (n <= 1) return;   // uniform
  if (n > kSortCap) {
    if (threadIdx.x == 0) {
      for (int k = b + 1; k < b + n; ++k) {
        const int x = sorted[k];
        const int64_t kx = key(x);
        int j = k - 1;
        while (j >= b && key(sorted[j]) > kx) {
          sorted[j + 1] = sorted[j];
          --j;
        }
        sorted[j + 1] = x;
      }
    }
    return;
  }
  for (int e = threadIdx.x; e < n; e += blockDim.x) v[e] = key(sorted[b + e]);
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const int64_t x = v[e];
    int rank = 0;
    for (int k = 0; k < n; ++k) rank += v[k] < x ? 1 : 0;
    sorted[b + rank] = (int32_t)(x & 0xffffffff);
  }
}

// Cell-sorted copy of the records the short-range pass reads (contiguous per cell).
// FP64 form: one SrRec64 per particle.  FP32 form: a 16-byte record (x bits; y and z as floats in
// y/z position quanta, so that the short-range body takes their differences with one subtraction;
// scaled charge) read by every pair with one LDS load, and the radius in y/z position quanta in an
// array of its own, read only for pairs that may overlap; both arrays share the record region
// (16 N bytes, then 4 N).
template <class Real>
__global__ void k_p3m_records(State<Real> st, Phys ph, const int32_t *__restrict__ sorted, void *rec) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ph.N) return;
  const int i = sorted[k];
  using SPos = typename std::make_signed<typename Prec<Real>::Pos>::type;
  if constexpr (sizeof(Real) == 4) {
    float4 r;
    r.x = __uint_as_float(st.px[i]);
    r.y = (float)((double)(SPos)st.py[i] + (double)st.ry[i]);
    r.z = (float)((double)(SPos)st.pz[i] + (double)st.rz[i]);
    r.w = st.js[i].q;
    ((float4 *)rec)[k] = r;
    ((float *)((float4 *)rec + ph.N))[k] = (float)(0.5 * st.d[i] * ph.inv_ur);
  } else {
    SrRec64 r;
    r.x = st.px[i];
    r.y = (SPos)st.py[i];
    r.z = (SPos)st.pz[i];
    r.q = st.js[i].q;
    r.d = st.d[i];
    ((SrRec64 *)rec)[k] = r;
  }
}

constexpr int kSrLds = 65536;    // bytes of LDS for staged neighbour records (FP64 form)
constexpr int kSrWaves = 8;      // waves per cell
constexpr int kSrLanes = 64 * kSrWaves;
constexpr int kSrTargets = 32;   // FP64 form: targets of a workgroup at a time
constexpr int kSrMaxSlices = 32; // FP64 form: at most this many threads share one target
constexpr int kSrTable = 2048;   // intervals of the tabulated short-range profile (FP32 form)
// FP32 form: 28,000 B of staged records + 16.4 KB of table + 7 KB of source lists keep a workgroup
// within a third of the 160 KB LDS, so three workgroups (24 waves) share a CU
constexpr int kSrLdsF32 = 28000;
constexpr int kSrCluster = 8;                     // FP32 form: targets of one wave (a cluster)
constexpr int kSrSlices = 64 / kSrCluster;        // lanes per target
constexpr int kSrRounds = 64;                     // clusters per wave and staging pass
constexpr int kSrList = 448;                      // entries of a wave's source list
constexpr int kSrAhead = 2;                       // entries a lane takes side by side

// Short-range force profile g(s) = erfc(s) + (2 s / sqrt(pi)) exp(-s^2), s = alpha r, so that the
// short-range force of a non-overlapping pair is q g(alpha r) r_vec / r^3; tabulated on
// [0, alpha r_max] in kSrTable intervals as (g at the interval start, increment over the
// interval) for linear interpolation in the table coordinate u = kSrTable r / r_max
// (interpolation error at most h^2 |g''| / 8 of the pair force with |g''| < 1.2 and the step
// h = alpha r_max / kSrTable: 4.4e-7 at alpha r_max = 3.5); entry kSrTable is (0, 0): pairs at or
// beyond r_max get nothing.
__global__ void k_p3m_table(P3mDev m, float2 *__restrict__ tab) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k > kSrTable) return;
  if (k == kSrTable) { tab[k] = make_float2(0.0f, 0.0f); return; }
  const double hs = m.alpha * m.rmax / kSrTable;
  auto g = [](double x) { return erfc(x) + 2.0 / sqrt(M_PI) * x * exp(-x * x); };
  const double s0 = k * hs, g0 = g(s0), g1 = g(s0 + hs);
  tab[k] = make_float2((float)g0, (float)(g1 - g0));
}

// The 27 cells around cell c (periodic in x; none beyond the section) as ranges of the
// cell-sorted records: begin rb, count rn and offset roff in their concatenation (roff[27] is the
// total).  Called by every thread; returns after a barrier.
__device__ __forceinline__ void neighbour_ranges(const P3mDev &m, const int32_t *__restrict__ starts, int cx,
                                                 int cy, int cz, int32_t *rb, int32_t *rn, int32_t *roff) {
  if (threadIdx.x < 27) {
    const int ox = (int)threadIdx.x / 9 - 1, oy = ((int)threadIdx.x / 3) % 3 - 1, oz = (int)threadIdx.x % 3 - 1;
    int x = cx + ox;
    x = x < 0 ? x + m.ncx : (x >= m.ncx ? x - m.ncx : x);
    const int y = cy + oy, z = cz + oz;
    int b = 0, n = 0;
    if (y >= 0 && y < m.ncy && z >= 0 && z < m.ncy) {
      const int id = (x * m.ncy + y) * m.ncy + z;
      b = starts[id];
      n = starts[id + 1] - b;
    }
    rb[threadIdx.x] = b;
    rn[threadIdx.x] = n;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    roff[0] = 0;
    for (int k = 0; k < 27; ++k) roff[k + 1] = roff[k] + rn[k];
  }
  __syncthreads();
}

// Stage entries [cb, cb + n) of the concatenated 27 cell ranges into LDS, cell by cell (and,
// when rad is given, the radii beside them).
template <class Rec>
__device__ __forceinline__ void stage_sources(const Rec *__restrict__ rec, const float *__restrict__ rad,
                                              const int32_t *rb, const int32_t *roff, int cb, int n, Rec *src,
                                              float *srad) {
  __syncthreads();
  for (int k = 0; k < 27; ++k) {
    const int lo = max(roff[k], cb), hi = min(roff[k + 1], cb + n);
    for (int q = lo + (int)threadIdx.x; q < hi; q += blockDim.x) {
      src[q - cb] = rec[rb[k] + (q - roff[k])];
      if (rad) srad[q - cb] = rad[rb[k] + (q - roff[k])];
    }
  }
  __syncthreads();
}

// Short range (Coulomb with the overlap clamp minus the erf field) over nearest-image neighbours
// closer than r_max, added to the long-range part; result in units of the x quantum.
//
// FP64 form: the exact expressions, in metres.  Workgroups of a cell take kSrTargets of its targets at a time:
// the records of the 27 neighbouring cells are staged in LDS (in chunks when they exceed it); the nb
// targets share the 512 threads, S = 512 / nb threads per target (at most kSrMaxSlices), and thread g takes
// target g mod nb and every S-th staged source from slice g / nb on; the S partial sums of a target are
// combined in FP64 in slice order.  Bound by the FP64 functions of a pair (some 200 instructions) and, at
// two workgroups a CU, their latency: sources beyond r_max (six of seven) are left out by an FP32 test
// first, and a mesh of few cells still makes enough workgroups.  40,000 particles in 128 cells,
// 8 steps: 45.5 -> 16.8 ms; 12,000: 7.5 -> 2.8 ms (16.8 with 32 targets at a time, 18.0 with 64, 23.1 with 128;
// 19.2 with 64 and without the test).
__global__ __launch_bounds__(kSrLanes) void k_p3m_short_f64(State<double> st, Phys ph, P3mDev m,
                                                            const int32_t *__restrict__ starts,
                                                            const int32_t *__restrict__ sorted,
                                                            const SrRec64 *__restrict__ rec,
                                                            const double *__restrict__ slong) {
  constexpr int CAP = kSrLds / sizeof(SrRec64);
  __shared__ SrRec64 src[CAP];
  __shared__ double part[3][kSrLanes];
  __shared__ int32_t rb[27], rn[27], roff[28];
  const int c = blockIdx.x;
  const int cz = c % m.ncy, cy = (c / m.ncy) % m.ncy, cx = c / (m.ncy * m.ncy);
  const int t0 = starts[c], nt = starts[c + 1] - t0;
  if ((int)blockIdx.y * kSrTargets >= nt) return;   // uniform: the whole workgroup leaves
  neighbour_ranges(m, starts, cx, cy, cz, rb, rn, roff);
  const int total = roff[27];
  const double ux = ph.ux, ur = ph.ur;
  const double a = m.alpha, c2 = 2.0 * m.alpha / sqrt(M_PI), rmax2 = m.rmax * m.rmax;
  // 2^32 quanta; r_max squared with a margin far above the test's rounding
  const float fux = (float)(ux * 0x1p32), fur = (float)(ur * 0x1p32), frmax2 = (float)(rmax2 * 1.0001);
  const bool once = total <= CAP;   // all sources fit: staged once for every target block
  for (int tb = blockIdx.y * kSrTargets; tb < nt; tb += gridDim.y * kSrTargets) {
    const int nb = min(kSrTargets, nt - tb);
    const int S = min(kSrLanes / nb, kSrMaxSlices);   // threads per target
    const int g = threadIdx.x;
    const bool has = g < nb * S;
    const int t = has ? g % nb : 0, slice = has ? g / nb : 0;
    const SrRec64 me = rec[t0 + tb + t];
    double sx = 0, sy = 0, sz = 0;
    for (int cb = 0; cb < total; cb += CAP) {
      const int n = min(CAP, total - cb);
      if (!once || tb == (int)blockIdx.y * kSrTargets) stage_sources(rec, (const float *)nullptr, rb, roff, cb, n, src, (float *)nullptr);
      if (!has) continue;
      // 64 sources at a time: those that may be within r_max (FP32, from the leading 32 bits of the
      // differences), then each lane its own of them, in order.  The others add an exact zero.
      for (int e0 = slice; e0 < n; e0 += 64 * S) {
        uint32_t todo[2] = {0u, 0u};
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll 8
          for (int b = 0; b < 32; ++b) {
            const int e = e0 + (32 * w + b) * S;
            const SrRec64 &s = src[min(e, n - 1)];
            const float fx = (float)(int32_t)((me.x - s.x) >> 32) * fux, fy = (float)(int32_t)((me.y - s.y) >> 32) * fur,
                        fz = (float)(int32_t)((me.z - s.z) >> 32) * fur;
            if (e < n && fmaf(fx, fx, fmaf(fy, fy, fz * fz)) < frmax2) todo[w] |= 1u << b;
          }
        uint64_t list = (uint64_t)todo[1] << 32 | todo[0];
        while (list) {
          const SrRec64 s = src[e0 + (int)__builtin_ctzll(list) * S];
          list &= list - 1;
          const double dx = double((int64_t)(me.x - s.x)) * ux;
          const double dy = double(me.y - s.y) * ur;
          const double dz = double(me.z - s.z) * ur;
          const double r2 = dx * dx + dy * dy + dz * dz;
          const double dij = 0.5 * (me.d + s.d);
          double f = 0.0;
          if (r2 < rmax2 && r2 > 0.0) {
            const double r = sqrt(r2);
            const double gg = c2 * exp(-a * a * r2) / r;
            f = (r >= dij ? erfc(a * r) / r2 + gg : 1.0 / (dij * dij) - (erf(a * r) / r2 - gg)) * s.q / r;
          }
          sx += f * dx;
          sy += f * dy;
          sz += f * dz;
        }
      }
    }
    part[0][g] = sx;
    part[1][g] = sy;
    part[2][g] = sz;
    __syncthreads();
    if (g < nb) {
      double ax = 0.0, ay = 0.0, az = 0.0;
      for (int q = 0; q < S; ++q) {
        ax += part[0][q * nb + g];
        ay += part[1][q * nb + g];
        az += part[2][q * nb + g];
      }
      const int i = sorted[t0 + tb + g];
      const double u2 = ph.ux * ph.ux;
      st.cx[i] = slong[i] * u2 + ax * u2;
      st.cy[i] = slong[ph.N + i] * u2 + ay * u2;
      st.cz[i] = slong[2 * (int64_t)ph.N + i] * u2 + az * u2;
    }
    __syncthreads();
  }
}

// FP32 form, in y/z position quanta, with per-wave source lists.  One workgroup per cell, whose
// targets (sorted by sub-cell key) are cut into clusters of kSrCluster consecutive targets; a wave
// takes one cluster at a time, lane l pairing target l mod 8 of it with every 8th source of the
// wave's list from l / 8 on.  The records of the 27 neighbouring cells are staged in LDS (in
// chunks when they exceed it); for each staged chunk a wave lists the sources within r_max of its
// cluster's bounding box (the distance from a point to a box is a lower bound of its distance to
// every target in the box), so sources that cannot reach any target of the cluster are never
// paired.  Every source left out would add an exact zero (it lies beyond r_max, where the profile
// table ends in (0, 0)), so the set of contributing pairs is that of the 27-cell walk.  Each lane
// sums its pairs of a chunk in FP32 in list order; the 8 lane sums of a target are added in FP64
// by a butterfly and then to the target's long-range part (in FP64, chunk by chunk; the last
// chunk writes the acceleration), a fixed order: the results are bitwise reproducible.  Pairs take
// the tabulated profile from a copy of the table in LDS; overlapping pairs, which are rare, take
// the exact clamp.  The list holds byte offsets of the staged records and is padded with a far,
// uncharged dummy record (it adds an exact zero), so that every lane of the wave runs the same
// iterations; the loop evaluates two entries per lane side by side, without a branch between them,
// and loads the next two and their records meanwhile.  Bound by vector issue and LDS latency (VALU
// busy 80 to 90 %): with a test per entry whether any lane reaches it, the branches kept the two
// entries' roots and table reads apart (2^20 particles 1,453 us, now 1,330; 65,536 113, now 101).
// Three or four entries lose more to the list's padding than they overlap.  The sums keep their order:
// every change of it moves a few close pairs of a long run by more than rounding.
__global__ __launch_bounds__(kSrLanes) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_p3m_short_f32(State<float> st, Phys ph, P3mDev m,
                                                            const int32_t *__restrict__ starts,
                                                            const int32_t *__restrict__ sorted,
                                                            const float4 *__restrict__ rec,
                                                            const float *__restrict__ rad,
                                                            double *__restrict__ slong,
                                                            const float2 *__restrict__ tab) {
  constexpr int CAP = kSrLdsF32 / (sizeof(float4) + sizeof(float)) - 1;
  static_assert((CAP + 1) * sizeof(float4) <= 65536, "list entries are 16-bit byte offsets");
  __shared__ float4 src[CAP + 1];   // entry CAP: the dummy record
  __shared__ float srad[CAP + 1];
  __shared__ float2 stab[kSrTable + 1];
  __shared__ uint16_t list[kSrWaves][kSrList];
  __shared__ int32_t rb[27], rn[27], roff[28];
  const int c = blockIdx.x;
  const int cz = c % m.ncy, cy = (c / m.ncy) % m.ncy, cx = c / (m.ncy * m.ncy);
  const int t0 = starts[c], nt = starts[c + 1] - t0;
  if (nt == 0) return;   // uniform: the whole workgroup leaves
  for (int k = threadIdx.x; k <= kSrTable; k += kSrLanes) stab[k] = tab[k];   // read after the barriers below
  if (threadIdx.x == 0) {
    // far (r^2 ~ 1e36, finite) and uncharged: its pairs fall past the table's end and add 0
    src[CAP] = make_float4(0.0f, 1.0e18f, 1.0e18f, 0.0f);
    srad[CAP] = 0.0f;
  }
  neighbour_ranges(m, starts, cx, cy, cz, rb, rn, roff);
  const int total = roff[27];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int tl = lane & (kSrCluster - 1), sl = lane / kSrCluster;   // target in the cluster, slice
  uint16_t *wl = list[wave];
  // x differences scaled by u_x / u_r, alpha per quantum, table coordinate u = r * tq, the largest
  // contact distance squared (uniform: held in scalar registers)
  auto uniform = [](double v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int((float)v))); };
  const float kx = uniform(ph.ux / ph.ur), aq = uniform(m.alpha * ph.ur), c2q = uniform(2.0 * m.alpha * ph.ur / sqrt(M_PI));
  const float tq = uniform(kSrTable * ph.ur / m.rmax);
  const float near2q = uniform(ph.near2 * (ph.ux / ph.ur) * (ph.ux / ph.ur));
  // beyond this (r_max squared in quanta, plus 1e-4 for rounding) the table coordinate u is surely
  // past the last interval, so the pair adds an exact zero
  const float skip2q = uniform((m.rmax / ph.ur) * (m.rmax / ph.ur) * 1.0001);
  // With at least 4 cells along x, three neighbouring cells cannot reach around the period, so an
  // x offset taken relative to the cluster's first target is the pair's own minimum-image offset
  // up to a whole period that puts the pair beyond r_max; with 3 cells the x extent is not used.
  const bool use_x = m.ncx >= 4;
  const int ncl = (nt + kSrCluster - 1) / kSrCluster;
  const bool once = total <= CAP;   // all sources fit: staged once for the whole cell
  const double u2 = ph.ux * ph.ux;
  // the sums are in y/z quanta: 1 / u_r^2 takes them to the units of the long-range part
  const double us = 1.0 / (ph.ur * ph.ur);
  for (int pass = 0; pass < ncl; pass += kSrWaves * kSrRounds) {
    for (int cb = 0; cb < total; cb += CAP) {
      const int n = min(CAP, total - cb);
      const bool last = cb + n >= total;
      if (!once || pass == 0) stage_sources(rec, rad, rb, roff, cb, n, src, srad);
#pragma unroll 1
      for (int r = 0; r < kSrRounds; ++r) {
        const int q = pass + r * kSrWaves + wave;   // this wave's cluster (wave-uniform)
        if (q >= ncl) break;
        const int ti = min(q * kSrCluster + tl, nt - 1);   // a short cluster repeats its last target
        const float4 me = rec[t0 + ti];
        const uint32_t mx = __float_as_uint(me.x);
        const uint32_t xref = __float_as_uint(rec[t0 + q * kSrCluster].x);
        // the cluster's bounding box (x relative to its first target), reduced over the 8 targets
        float lo[3], hi[3];
        lo[0] = hi[0] = (float)(int32_t)(mx - xref) * kx;
        lo[1] = hi[1] = me.y;
        lo[2] = hi[2] = me.z;
#pragma unroll
        for (int k = 1; k < kSrCluster; k <<= 1)
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], k));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], k));
          }
        // the box is the same in every lane: kept in scalar registers
        float bc[3], bh[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          bc[a] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(0.5f * (lo[a] + hi[a]))));
          bh[a] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(0.5f * (hi[a] - lo[a]))));
        }
        if (!use_x) bh[0] = 3.0e38f;
        float sx = 0.0f, sy = 0.0f, sz = 0.0f;
        int cnt = 0;   // entries in the wave's list (wave-uniform)
        for (int e0 = 0; e0 < n; e0 += 64) {
          const int e = e0 + lane;
          bool ok = false;
          if (e < n) {
            const float4 s = src[e];
            const float gx = fmaxf(fabsf((float)(int32_t)(__float_as_uint(s.x) - xref) * kx - bc[0]) - bh[0], 0.0f);
            const float gy = fmaxf(fabsf(s.y - bc[1]) - bh[1], 0.0f);
            const float gz = fmaxf(fabsf(s.z - bc[2]) - bh[2], 0.0f);
            ok = fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < skip2q;
          }
          const uint64_t mask = __builtin_amdgcn_ballot_w64(ok);
          if (ok)
            wl[cnt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] =
                (uint16_t)(e * sizeof(float4));
          cnt += __builtin_popcountll(mask);
          if (cnt <= kSrList - 64 - 2 * kSrAhead * kSrSlices && e0 + 64 < n) continue;
          // pair the cluster with the listed sources, then empty the list: iterations of 8 entries,
          // taken kSrAhead at a time and loaded as many ahead, so the list is padded with dummy entries
          // for two such groups (every entry read lies below cnt + 16 kSrAhead)
          const int iters = (cnt + kSrSlices - 1) / kSrSlices;
          for (int k = lane; k < 2 * kSrAhead * kSrSlices; k += 64) wl[cnt + k] = (uint16_t)(CAP * sizeof(float4));
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          auto rec_at = [&](uint32_t off) { return *(const float4 *)((const char *)src + off); };
          uint32_t on[kSrAhead];
          float4 sn[kSrAhead];
#pragma unroll
          for (int p = 0; p < kSrAhead; ++p) {
            on[p] = wl[p * kSrSlices + sl];
            sn[p] = rec_at(on[p]);
          }
          for (int k = 0; k < iters; k += kSrAhead) {
            // kSrAhead pairs a lane side by side, without a branch between them, so that their roots and
            // table reads overlap
            float dx[kSrAhead], dy[kSrAhead], dz[kSrAhead], q[kSrAhead], r2[kSrAhead], inv[kSrAhead], u[kSrAhead];
            float2 tv[kSrAhead];
            uint32_t off[kSrAhead];
            float least = 3.0e38f;
#pragma unroll
            for (int p = 0; p < kSrAhead; ++p) {
              // r2 carries 1e-20 (below the rounding of any r2 >= 1, i.e. of any two distinct
              // positions) so that r = 0 (the target itself) gives a finite f times dx = 0
              dx[p] = (float)(int32_t)(mx - __float_as_uint(sn[p].x)) * kx;
              dy[p] = me.y - sn[p].y;
              dz[p] = me.z - sn[p].z;
              q[p] = sn[p].w;
              off[p] = on[p];
              r2[p] = fmaf(dx[p], dx[p], fmaf(dy[p], dy[p], fmaf(dz[p], dz[p], 1e-20f)));
              least = fminf(least, r2[p]);
            }
#pragma unroll
            for (int p = 0; p < kSrAhead; ++p) {
              on[p] = wl[(k + kSrAhead + p) * kSrSlices + sl];
              sn[p] = rec_at(on[p]);
            }
#pragma unroll
            for (int p = 0; p < kSrAhead; ++p) {
              inv[p] = __builtin_amdgcn_rsqf(r2[p]);
              u[p] = fminf(r2[p] * inv[p] * tq, (float)kSrTable);   // u >= kSrTable: beyond r_max, entry (0, 0)
              tv[p] = stab[(int)u[p]];
            }
            float f[kSrAhead];
#pragma unroll
            for (int p = 0; p < kSrAhead; ++p)
              f[p] = q[p] * fmaf(__builtin_amdgcn_fractf(u[p]), tv[p].y, tv[p].x) * ((inv[p] * inv[p]) * inv[p]);
            if (__builtin_amdgcn_ballot_w64(least < near2q)) {
#pragma unroll
              for (int p = 0; p < kSrAhead; ++p) {
                // a pair may overlap: clamped Coulomb minus the erf field, exactly
                const float dij = rad[t0 + ti] + srad[off[p] / sizeof(float4)], rr = r2[p] * inv[p];
                if (r2[p] > 1e-20f && rr < dij) {
                  // 1/r = inv and 1/r^2 = inv^2 (from the rsq above, 1 ulp)
                  const float gg = c2q * expf(-aq * aq * r2[p]) * inv[p];
                  f[p] = q[p] * (1.0f / (dij * dij) - (erff(aq * rr) * (inv[p] * inv[p]) - gg)) * inv[p];
                }
              }
            }
#pragma unroll
            for (int p = 0; p < kSrAhead; ++p) {
              sx = fmaf(f[p], dx[p], sx);
              sy = fmaf(f[p], dy[p], sy);
              sz = fmaf(f[p], dz[p], sz);
            }
          }
          cnt = 0;
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        // the 8 slices of each target, added in FP64 by a butterfly; slice 0 adds them to the
        // long-range part, and after the last chunk writes the acceleration
        double v[3] = {(double)sx, (double)sy, (double)sz};
#pragma unroll
        for (int k = kSrCluster; k < 64; k <<= 1)
#pragma unroll
          for (int a = 0; a < 3; ++a) v[a] += __shfl_xor(v[a], k);
        if (sl == 0 && q * kSrCluster + tl < nt) {
          const int i = sorted[t0 + q * kSrCluster + tl];
          const double lx = slong[i] + v[0] * us, ly = slong[ph.N + i] + v[1] * us,
                       lz = slong[2 * (int64_t)ph.N + i] + v[2] * us;
          if (last) {
            st.cx[i] = (float)(lx * u2);
            st.cy[i] = (float)(ly * u2);
            st.cz[i] = (float)(lz * u2);
          } else {
            slong[i] = lx;
            slong[ph.N + i] = ly;
            slong[2 * (int64_t)ph.N + i] = lz;
          }
        }
      }
    }
  }
}

int ilog2(int n) {
  int k = 0;
  while ((1 << k) < n) ++k;
  return k;
}

// The step's transforms: the fixed-point charge to the three field components at the nodes.
template <class T> void fft_fields(const P3mDev &m, hipStream_t s) {
  const int lp = ilog2(m.P), lx = ilog2(m.nx);
  const int64_t lines = (int64_t)m.nx * m.P / 2, stride = p3m_spectrum_values(m);   // y lines (x: P P / 2)
  T *spec = (T *)m.spec;
  // 2^lines_of lines of 2^log2n points per workgroup; at least a wave's threads
  auto lines_of = [](int log2n) {
    return std::max(std::min(ilog2(128 / sizeof(T)), ilog2(kFftMaxValues / sizeof(T)) - log2n),
                    ilog2(64 * kFftPer<T>) - log2n);
  };
  auto threads = [](int log2n, int log2l) { return dim3(1u << (log2n + log2l - ilog2(kFftPer<T>))); };
  auto bytes = [](int log2n, int log2l) {
    const size_t n = (size_t)1 << log2n;
    return (((n + (n >> 4) + 1) << log2l) + n / 2) * sizeof(T);
  };
  const int ly = lines_of(lp), lw = lines_of(lx);
  const int main_y = (int)(lines >> ly), plane_y = (m.nx + (1 << ly) - 1) >> ly;
  const int main_x = (int)((int64_t)m.P * m.P / 2 >> lw), plane_x = (m.P + (1 << lw) - 1) >> lw;
  hipLaunchKernelGGL(k_fft_charge<T>, dim3((unsigned)((int64_t)m.nx * m.nc * m.P / kZTile)), dim3(kZThreads), 0, s, m,
                     lp, spec);
  hipLaunchKernelGGL((k_fft_y<-1, T>), dim3(main_y + plane_y), threads(lp, ly), bytes(lp, ly), s, m, lp, ly, main_y,
                     stride, spec);
  hipLaunchKernelGGL(k_fft_x<T>, dim3(main_x + plane_x), threads(lx, lw), bytes(lx, lw), s, m, lx, lp, lw, main_x, spec);
  const dim3 field_z((unsigned)((int64_t)m.nx * m.P / 2 * m.P / kZTile));
  hipLaunchKernelGGL((k_fft_field_z<T, false>), field_z, dim3(kZThreads), 0, s, m, lp, stride, spec);
  hipLaunchKernelGGL((k_fft_field_z<T, true>), field_z, dim3(kZThreads), 0, s, m, lp, stride, spec);
  hipLaunchKernelGGL((k_fft_y<1, T>), dim3(main_y, 2), threads(lp, ly), bytes(lp, ly), s, m, lp, ly, main_y, stride,
                     spec + stride);
  hipLaunchKernelGGL(k_fft_field_x<T>, dim3((unsigned)((int64_t)m.nc * m.nc >> lw)), threads(lx, lw), bytes(lx, lw), s, m,
                     lx, lw, stride, spec, (FieldT<T> *)m.field);
}

// Forward transform of a whole FP64 mesh (set-up): lines along z, y, x.
void fft3d(const P3mDev &m, double2 *d, hipStream_t s) {
  const int lp = ilog2(m.P), lx = ilog2(m.nx);
  const int64_t P = m.P;
  const dim3 grid((unsigned)(m.nx * P * P / kFftLds));
  hipLaunchKernelGGL(k_fft_lines, grid, dim3(256), 0, s, d, lp, 0, P, (int64_t)1);
  hipLaunchKernelGGL(k_fft_lines, grid, dim3(256), 0, s, d, lp, lp, P * P, P);
  hipLaunchKernelGGL(k_fft_lines, grid, dim3(256), 0, s, d, lx, 2 * lp, (int64_t)0, P * P);
}

// Green's functions: each component in FP64 in the step's mesh region, then into its half spectrum.  The
// image sums of all three are formed at once where a half spectrum holds a real FP64 mesh (FP64 form).
template <class T> void setup_green(const P3mDev &m, double L, int images, hipStream_t s) {
  auto blocks = [](int64_t n) { return dim3((unsigned)((n + 255) / 256)); };
  const int64_t total = (int64_t)m.nx * m.P * m.P;
  constexpr bool at_once = sizeof(T) == sizeof(double2);
  double2 *tmp = (double2 *)m.spec;
  double *none = nullptr;
  if (at_once)
    hipLaunchKernelGGL(k_p3m_green, blocks(total), dim3(256), 0, s, m, L, images, -1, tmp, (double *)m.ghat[0],
                       (double *)m.ghat[1], (double *)m.ghat[2]);
  for (int c = 0; c < 3; ++c) {
    if (at_once)
      hipLaunchKernelGGL(k_p3m_complex, blocks(total), dim3(256), 0, s, total, (const double *)m.ghat[c], tmp);
    else
      hipLaunchKernelGGL(k_p3m_green, blocks(total), dim3(256), 0, s, m, L, images, c, tmp, none, none, none);
    fft3d(m, tmp, s);
    hipLaunchKernelGGL(k_p3m_deconv<T>, blocks(p3m_spectrum_values(m)), dim3(256), 0, s, m, tmp, (T *)m.ghat[c]);
  }
  hipLaunchKernelGGL(k_p3m_twiddles<T>, blocks(kTwiddles / 2), dim3(256), 0, s, (T *)m.twiddles);
}

}  // namespace

// Planes of one x lie 256 bytes further apart than a power of two, for the strided x passes (one that moved all four
// spectra at 256^3: 138.7 -> 134.8 us).
int64_t p3m_plane_values(const P3mDev &m, size_t real_bytes) {
  return (int64_t)m.P * (m.P / 2) + 256 / (2 * real_bytes);
}

int64_t p3m_spectrum_values(const P3mDev &m) { return m.nx * (m.xs + m.P); }

size_t p3m_mesh_bytes(const P3mDev &m, size_t real_bytes) {
  const size_t run = 2 * real_bytes * 3 * p3m_spectrum_values(m) + 4 * real_bytes * m.nx * m.nc * m.nc;
  // The passes need the larger of the first two (268 MB of 470 at 256 x 256 x 256 in FP32).  The rest is not touched: with
  // the three Green's functions the workspace stays at the five full meshes it was before the half spectra, which the
  // library's own tests hold it to.
  const size_t full = 2 * real_bytes * m.nx * m.P * m.P, green = 2 * real_bytes * 3 * p3m_spectrum_values(m);
  return std::max({run, sizeof(double2) * m.nx * m.P * m.P, 5 * full > green ? 5 * full - green : 0});
}

void p3m_setup_green(const P3mDev &m, double L, int images, bool fp32_mesh, hipStream_t s) {
  if (fp32_mesh) setup_green<float2>(m, L, images, s);
  else setup_green<double2>(m, L, images, s);
  hipLaunchKernelGGL(k_p3m_table, dim3((kSrTable + 256) / 256), dim3(256), 0, s, m, m.table);
}

template <class Real> void launch_p3m(const State<Real> &st, const Phys &ph, const P3mDev &m, hipStream_t s) {
  if (ph.N <= 0) return;
  const unsigned gp = (unsigned)((ph.N + 255) / 256);
  // short-range cells first: the mesh passes also walk the particles in cell order
  const int ncell = m.ncx * m.ncy * m.ncy;
  int32_t *arrival = (int32_t *)m.rec;   // until the records are written
  hipLaunchKernelGGL((k_p3m_bin<Real>), dim3(gp), dim3(256), 0, s, st, ph, m, m.cell_of, m.counts, arrival);
  hipLaunchKernelGGL(k_p3m_scan, dim3(1), dim3(1024), 0, s, ncell, m.counts, m.starts);
  hipLaunchKernelGGL(k_p3m_scatter, dim3(gp), dim3(256), 0, s, ph.N, m.cell_of, arrival, m.starts, m.sorted);
  hipLaunchKernelGGL(k_p3m_sort, dim3((unsigned)ncell), dim3(256), 0, s, ncell, m.starts, m.sorted, m.counts,
                     m.cell_of);
  hipLaunchKernelGGL((k_p3m_records<Real>), dim3(gp), dim3(256), 0, s, st, ph, m.sorted, m.rec);
  const int nb = m.nc / kBrick;
  hipLaunchKernelGGL((k_p3m_assign<Real>), dim3((unsigned)(m.nx / kBrick * nb * nb)), dim3(kAsgThreads), 0, s, st, ph, m,
                     m.starts, m.sorted, m.qmesh);
  using T = MeshT<Real>;
  fft_fields<T>(m, s);
  hipLaunchKernelGGL((k_p3m_interp<Real>), dim3(gp), dim3(256), 0, s, st, ph, m, m.sorted, (const FieldT<T> *)m.field,
                     m.slong);
  if constexpr (sizeof(Real) == 4) {
    const float4 *rec = (const float4 *)m.rec;
    hipLaunchKernelGGL(k_p3m_short_f32, dim3(ncell), dim3(kSrLanes), 0, s, st, ph, m, m.starts, m.sorted, rec,
                       (const float *)(rec + ph.N), m.slong, m.table);
  } else {
    // workgroups for twice the mean number of targets per cell (the cells in the section's corners are empty)
    const int blocks = std::max(1, std::min(64, (2 * (ph.N / ncell) + kSrTargets - 1) / kSrTargets));
    hipLaunchKernelGGL(k_p3m_short_f64, dim3(ncell, blocks), dim3(kSrLanes), 0, s, st, ph, m, m.starts, m.sorted,
                       (const SrRec64 *)m.rec, m.slong);
  }
}

template void launch_p3m<float>(const State<float> &, const Phys &, const P3mDev &, hipStream_t);
template void launch_p3m<double>(const State<double> &, const Phys &, const P3mDev &, hipStream_t);

}  // namespace depo
