// Cell-list neighbour search and short-range pair forces: soft-sphere normal
// contact (Appendix A.2.2) and van der Waals cohesion (Eq. vdw, Appendix A.2.3).
//
// Build (after the histogram made by k_prepare): exclusive scan of the cell
// counts -> scatter with per-cell atomic slots -> per-cell ascending sort of
// the particle indices, so the neighbour walk and hence every force sum runs
// in a fixed order (bitwise reproducible).  The sort pass also clears the
// counts for the next build, so no memset is ever enqueued.  Up to 131,072
// particles k_cells_fused, one launch for these five and the histogram, builds the
// same list (below a hundred thousand it is the faster one by itself), but not on a
// branch beside a one-sided pair kernel.
#include "common.hpp"
#include "launch.hpp"

namespace depo {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER_THREAD = 4;
constexpr int SCAN_BLOCK = SCAN_THREADS * SCAN_PER_THREAD;

__device__ __forceinline__ int block_exclusive_scan(int v, int *sh, int &total) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int off = 1; off < SCAN_THREADS; off <<= 1) {
    int add = t >= off ? sh[t - off] : 0;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  total = sh[SCAN_THREADS - 1];
  int excl = sh[t] - v;
  __syncthreads();
  return excl;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_reduce(const int32_t *__restrict__ count, int n,
                                                              int32_t *__restrict__ part) {
  __shared__ int sh[SCAN_THREADS];
  const int base = blockIdx.x * SCAN_BLOCK + threadIdx.x * SCAN_PER_THREAD;
  int v = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER_THREAD; ++k) v += base + k < n ? count[base + k] : 0;
  int total;
  block_exclusive_scan(v, sh, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_top(int32_t *__restrict__ part, int nb,
                                                           int32_t *__restrict__ start, int n) {
  __shared__ int sh[SCAN_THREADS];
  int carry = 0;
  for (int b0 = 0; b0 < nb; b0 += SCAN_THREADS) {
    const int b = b0 + threadIdx.x;
    const int v = b < nb ? part[b] : 0;
    int total;
    const int ex = block_exclusive_scan(v, sh, total);
    if (b < nb) part[b] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) start[n] = carry;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_apply(int32_t *__restrict__ count, int n,
                                                             const int32_t *__restrict__ part,
                                                             int32_t *__restrict__ start) {
  __shared__ int sh[SCAN_THREADS];
  const int base = blockIdx.x * SCAN_BLOCK + threadIdx.x * SCAN_PER_THREAD;
  int c[SCAN_PER_THREAD];
  int v = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER_THREAD; ++k) {
    c[k] = base + k < n ? count[base + k] : 0;
    v += c[k];
  }
  int total;
  int run = block_exclusive_scan(v, sh, total) + part[blockIdx.x];
#pragma unroll
  for (int k = 0; k < SCAN_PER_THREAD; ++k)
    if (base + k < n) {
      start[base + k] = run;
      count[base + k] = 0;
      run += c[k];
    }
}

__global__ __launch_bounds__(256) void k_scatter(const int32_t *__restrict__ cell_of, int N,
                                                 const int32_t *__restrict__ start, int32_t *__restrict__ count,
                                                 int32_t *__restrict__ idx) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int c = cell_of[i];
  if (c < 0) return;
  const int slot = start[c] + atomicAdd(&count[c], 1);
  idx[slot] = i;
}

__global__ __launch_bounds__(256) void k_cell_sort(const int32_t *__restrict__ start, int n_cells,
                                                   int32_t *__restrict__ count, int32_t *__restrict__ idx) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_cells) return;
  const int b = start[c], e = start[c + 1];
  for (int k = b + 1; k < e; ++k) {
    const int v = idx[k];
    int j = k - 1;
    while (j >= b && idx[j] > v) {
      idx[j + 1] = idx[j];
      --j;
    }
    idx[j + 1] = v;
  }
  count[c] = 0;
}

// The whole cell list in one kernel, from the cells that k_prepare wrote: each workgroup owns kOwn
// consecutive cells and reads every particle's cell.  Particles of earlier cells are counted (the first slot of
// the workgroup's own), those of its own cells are collected in LDS, and each one's place in its cell is the
// number of smaller indices there: the order of the general build.  Bound by latency and, beyond a few tens
// of workgroups, by their reading the cells over and over; 1,024 cells per workgroup is one per
// thread.  3,001 particles: 18.7 -> 7.8 us for the build, 49.6 -> 38.1 us for the whole step.
constexpr int kOwn = 1024;      // cells (and threads) per workgroup
constexpr int kHits = 4096;     // particles of its own cells that a workgroup holds in LDS

__global__ __launch_bounds__(kOwn) void k_cells_fused(const int32_t *__restrict__ cell_of, int N, int n_cells,
                                                      int32_t *__restrict__ start, int32_t *__restrict__ idx) {
  __shared__ int count[kOwn], first[kOwn];
  __shared__ int hit_i[kHits], hit_at[kHits], ids[kHits];
  __shared__ int n_hits, wave_sum[16], wave_pre[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int c0 = blockIdx.x * kOwn, own = min(kOwn, n_cells - c0);
  count[t] = 0;
  if (t == 0) n_hits = 0;
  __syncthreads();
  int before = 0;
  auto take = [&](int c, int i) {
    if (c >= c0) {
      const int k = c - c0;
      if (k < own) {
        const int at = atomicAdd(&count[k], 1), h = atomicAdd(&n_hits, 1);
        if (h < kHits) { hit_i[h] = i; hit_at[h] = at << 10 | k; }
      }
    } else if (c >= 0) {
      ++before;
    }
  };
  const int n4 = N >> 2;
  for (int q = t; q < n4; q += kOwn) {
    const int4 c = reinterpret_cast<const int4 *>(cell_of)[q];
    take(c.x, 4 * q); take(c.y, 4 * q + 1); take(c.z, 4 * q + 2); take(c.w, 4 * q + 3);
  }
  if (4 * n4 + t < N) take(cell_of[4 * n4 + t], 4 * n4 + t);
  __syncthreads();
  // exclusive scan of the counts; sum of `before`
  const int mine = count[t];
  int inc = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(inc, off);
    if (lane >= off) inc += v;
    before += __shfl_xor(before, off);
  }
  if (lane == 63) { wave_sum[w] = inc; wave_pre[w] = before; }
  __syncthreads();
  int base = 0, pre = 0, total = 0;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    base += q < w ? wave_sum[q] : 0;
    total += wave_sum[q];
    pre += wave_pre[q];
  }
  first[t] = base + inc - mine;
  if (t < own) start[c0 + t] = pre + base + inc - mine;
  if (t == 0 && c0 + own == n_cells) start[n_cells] = pre + total;
  __syncthreads();
  if (total <= kHits) {
    for (int h = t; h < total; h += kOwn) ids[first[hit_at[h] & (kOwn - 1)] + (hit_at[h] >> 10)] = hit_i[h];
    __syncthreads();
    for (int h = t; h < total; h += kOwn) {
      const int i = hit_i[h], k = hit_at[h] & (kOwn - 1), b = first[k], e = b + count[k];
      int rank = b;
      for (int q = b; q < e; ++q) rank += ids[q] < i ? 1 : 0;
      idx[pre + rank] = i;
    }
  } else {
    // more particles than LDS holds (a crowd in few cells): kOwn particles at a time in index order, each
    // placed after those of its cell so far
    count[t] = 0;
    for (int i0 = 0; i0 < N; i0 += kOwn) {
      const int i = i0 + t, k = i < N ? cell_of[i] - c0 : -1;
      const bool hit = k >= 0 && k < own;
      hit_at[t] = hit ? k : -1;
      if (!__syncthreads_or(hit ? 1 : 0)) continue;
      if (hit) {
        int rank = 0;
        for (int q = 0; q < t; ++q) rank += hit_at[q] == k ? 1 : 0;
        idx[pre + first[k] + count[k] + rank] = i;
      }
      __syncthreads();
      if (hit) atomicAdd(&count[k], 1);
      __syncthreads();
    }
  }
}

__global__ void k_clear_int(int32_t *p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Cohesive force magnitude of two spheres (diameters di, dj) at surface gap
// gs: -dU/dr of Hamaker's two-sphere energy, written as the single product
// (32/3) A R1^3 R2^3 r / (P^2 Q^2), P = r^2 - (R1+R2)^2 = gs (gs + 2 (R1+R2)),
// Q = r^2 - (R1-R2)^2, which equals Eq. vdw for equal spheres.  Lengths are
// handled in micrometres so that every intermediate stays in FP32 range.
template <class Real>
__device__ __forceinline__ Real vdw_force(Real gs_m, Real di_m, Real dj_m, Real A) {
  const Real u = Real(1e6);
  const Real r1 = Real(0.5) * di_m * u, r2 = Real(0.5) * dj_m * u, g = gs_m * u;
  const Real s = r1 + r2, t = r1 - r2;
  const Real r = s + g;
  const Real P = g * (g + Real(2) * s);
  const Real Q = (r - t) * (r + t);
  const Real r13 = r1 * r1 * r1, r23 = r2 * r2 * r2;
  const Real PQ = P * Q;
  return Real(32.0 / 3.0) * A * u * (r13 * r23) * r / (PQ * PQ);
}

// kShortRangeLanes threads per alive particle, taken in cell order (the sorted index
// array), so the threads of a wavefront walk neighbouring cells and share their loads.
// Bound by the latency of its dependent reads (cell bounds, index, position); cells
// adjacent along z are one run of the index, read as one row.
// Removed particles are not visited; their short-range slots are never read.
template <class Real>
__global__ __launch_bounds__(256) void k_short_range(State<Real> st, Phys ph, int n_cells) {
  constexpr int G = kShortRangeLanes;
  const int t = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / G), g = threadIdx.x % G;
  if (t >= st.cell_start[n_cells]) return;
  const int i = st.cell_idx[t];
  const SampleDev sp = st.samples[st.sid[i]];
  const auto px = st.px[i], py = st.py[i], pz = st.pz[i];
  const double rxi = st.rx[i], ryi = st.ry[i], rzi = st.rz[i];
  const Real vix = st.vx[i], viy = st.vy[i], viz = st.vz[i];
  int cx, cy, cz, mx, my, mz;
  short_range_cells(px, py, pz, sp, cx, cy, cz, mx, my, mz);
  const double di_d = st.d[i];
  const Real di = Real(di_d);
  const Real mi = Real(ph.mass_coef) * di * di * di;
  const Real A = Real(sp.hamaker);
  const Real dsat = Real(ph.delta_sat);
  const bool vdw = (ph.flags & F_VDW) != 0, col = (ph.flags & F_COLLIDE) != 0;
  Real a0 = 0, a1 = 0, a2 = 0;
  int nb = 0;
  // only the neighbour cells whose shared face is closer than the reach can hold a partner
  const NearRows rows(cx, cy, cz, mx, my, mz, sp);
  for (int r = g; r < rows.n; r += G) {
    const int c = rows.first(r, sp);
    const int e = st.cell_start[c + 1 + rows.z1 - rows.z0];
    for (int k = st.cell_start[c]; k < e; ++k) {
      const int j = st.cell_idx[k];
      if (j == i) continue;
      // geometry and the range test in FP64 (the gap near contact is a small fraction of |r|)
      const double dj_d = st.d[j];
      double gx, gy, gz, gd;
      const double most = 0.25 * fmin(di_d, dj_d);
      const double gap_d = pair_gap_within(most, px, py, pz, st.px[j], st.py[j], st.pz[j], rxi - (double)st.rx[j],
                                           ryi - (double)st.ry[j], rzi - (double)st.rz[j], ph.ux, ph.ur,
                                           0.5 * (di_d + dj_d), gx, gy, gz, gd);
      if (gap_d > most || gd == 0.0) continue;
      ++nb;
      const double inv_d = 1.0 / gd;
      const Real nx = Real(gx * inv_d), ny = Real(gy * inv_d), nz = Real(gz * inv_d);
      const Real dj = Real(dj_d);
      const Real gap = Real(gap_d);
      Real f = 0;   // along +n (away from j), per unit mass of i
      if (vdw) f -= vdw_force(fmax(gap, dsat), di, dj, A) / mi;
      if (col && gap < Real(0)) {
        const Real mj = Real(ph.mass_coef) * dj * dj * dj;
        const Real vn = (vix - st.vx[j]) * nx + (viy - st.vy[j]) * ny + (viz - st.vz[j]) * nz;
        f += mj / (mi + mj) * (Real(ph.col_K) * (-gap) - Real(ph.col_H) * vn);
      }
      a0 += f * nx; a1 += f * ny; a2 += f * nz;
    }
  }
  // the lanes' sums, pairwise
#pragma unroll
  for (int m = 1; m < G; m <<= 1) {
    a0 += __shfl_xor(a0, m); a1 += __shfl_xor(a1, m); a2 += __shfl_xor(a2, m);
    nb += __shfl_xor(nb, m);
  }
  if (g == 0) {
    st.sx[i] = a0; st.sy[i] = a1; st.sz[i] = a2;
    st.nbr[i] = nb;
  }
}

template <class Real>
void launch_cells(const State<Real> &st, const Phys &ph, int n_cells, int n_scan_blocks, hipStream_t s) {
  if (ph.cells_fused) {
    hipLaunchKernelGGL(k_cells_fused, dim3((n_cells + kOwn - 1) / kOwn), dim3(kOwn), 0, s, st.cell_of, ph.N, n_cells,
                       st.cell_start, st.cell_idx);
    return;
  }
  hipLaunchKernelGGL(k_scan_reduce, dim3(n_scan_blocks), dim3(SCAN_THREADS), 0, s, st.cell_count, n_cells,
                     st.scan_part);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(SCAN_THREADS), 0, s, st.scan_part, n_scan_blocks, st.cell_start,
                     n_cells);
  hipLaunchKernelGGL(k_scan_apply, dim3(n_scan_blocks), dim3(SCAN_THREADS), 0, s, st.cell_count, n_cells,
                     st.scan_part, st.cell_start);
  if (ph.N > 0)
    hipLaunchKernelGGL(k_scatter, dim3((ph.N + 255) / 256), dim3(256), 0, s, st.cell_of, ph.N, st.cell_start,
                       st.cell_count, st.cell_idx);
  hipLaunchKernelGGL(k_cell_sort, dim3((n_cells + 255) / 256), dim3(256), 0, s, st.cell_start, n_cells,
                     st.cell_count, st.cell_idx);
}

template <class Real>
void launch_short_range(const State<Real> &st, const Phys &ph, int n_cells, hipStream_t s) {
  if (ph.N <= 0) return;
  hipLaunchKernelGGL(k_short_range<Real>, dim3((unsigned)(((int64_t)ph.N * kShortRangeLanes + 255) / 256)),
                     dim3(256), 0, s, st, ph, n_cells);
}

void launch_clear_int(int32_t *p, size_t n, hipStream_t s) {
  if (n) hipLaunchKernelGGL(k_clear_int, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
}

template void launch_cells<float>(const State<float> &, const Phys &, int, int, hipStream_t);
template void launch_cells<double>(const State<double> &, const Phys &, int, int, hipStream_t);
template void launch_short_range<float>(const State<float> &, const Phys &, int, hipStream_t);
template void launch_short_range<double>(const State<double> &, const Phys &, int, hipStream_t);

}  // namespace depo
