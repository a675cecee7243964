// Host-side launchers of the device kernels (one translation unit per kernel family).
#pragma once

#include "common.hpp"

namespace depo {

// k_prepare modes
enum : int { P_KICK_DRIFT = 1, P_COULOMB = 2, P_CELLS = 4, P_SEED = 8 };
// k_finish modes
// F_PAIR_SUMS: the pair kernel ran without its own finishing pass.  FP32 (symmetric): k_finish turns
// the fixed-point accumulators into the FP32 Coulomb sums and clears them, every particle's; FP64: it adds
// the pieces' partial sums
enum : int { F_KICK = 1, F_V_FROM_FLUID = 2, F_FLUID_ONLY = 4, F_PAIR_SUMS = 8 };

// A batch of steps brings the device's step counter up to date in its last k_finish (by `steps`); its other
// kernels that need the step's number are told how many steps `ahead` of the counter they are.
template <class Real>
void launch_prepare(const State<Real> &st, const Phys &ph, int mode, hipStream_t s, int ahead = 0);
template <class Real>
void launch_finish(const State<Real> &st, const Phys &ph, int mode, hipStream_t s, int steps = 1);
// k_finish of one step and k_prepare of the next, `ahead` steps after the counter
template <class Real>
void launch_finish_prepare(const State<Real> &st, const Phys &ph, int finish_mode, int prepare_mode, int ahead,
                           hipStream_t s);
template <class Real> void launch_tally(const State<Real> &st, const Phys &ph, int nstep, hipStream_t s);

// Storage order: at the start of a step that follows a multiple of `every` steps (decided on the
// device from the step counter), permute the per-particle state into the order of the last cell list.
template <class Real>
void launch_order(const State<Real> &st, const OrderScratch<Real> &sc, int n, int n_cells, int every, int ahead,
                  hipStream_t s);

// Cell list: scan of the histogram, scatter, in-cell ordering, short-range forces.
template <class Real>
void launch_cells(const State<Real> &st, const Phys &ph, int n_cells, int n_scan_blocks, hipStream_t s);
template <class Real> void launch_short_range(const State<Real> &st, const Phys &ph, int n_cells, hipStream_t s);
void launch_clear_int(int32_t *p, size_t n, hipStream_t s);

// Coulomb pair sums.
struct CoulombConfig {
  int ipl;     // targets per lane
  int waves;   // waves per workgroup (split the source range; symmetric: each owns 64*ipl targets)
  int block;   // sources per compensated block
  bool compensated;  // Kahan accumulation of the block sums (FP32); plain sums otherwise
  bool symmetric = false;  // FP32: each unordered pair once, reaction on the source (Newton's third law)
  bool int_rec = false;    // symmetric FP32: y and z of the source records as 32-bit integers in x quanta
};
// FP64 with ph.pair_parts > 1: every sample's sources in that many pieces, each with its own partial sums;
// with defer_finish k_finish adds them (F_PAIR_SUMS; the return value says whether it has to).
template <class Real>
bool launch_coulomb(const State<Real> &st, const Phys &ph, int n_tiles, const CoulombConfig &cfg, hipStream_t s,
                    bool defer_finish);
int coulomb_tile_targets(const CoulombConfig &cfg);
bool coulomb_config_supported(int real_bytes, const CoulombConfig &cfg);

// Symmetric FP32 pair sums over the layout's item list, combined in fixed point into cx/cy/cz.
int coulomb_sym_tile(const CoulombConfig &cfg);   // targets per item (a tile)
bool coulomb_sym_supported(const CoulombConfig &cfg);
// defer_finish: leave the fixed-point accumulators for k_finish (mode F_PAIR_SUMS) instead of
// converting them with k_pair_finish
void launch_coulomb_sym(const State<float> &st, const Phys &ph, int n_items, const CoulombConfig &cfg,
                        hipStream_t s, bool defer_finish = false);

// P3M electrostatics (single-sample layouts): mesh geometry, splitting and workspace.
struct P3mDev {
  int nx, nc, P;          // mesh nodes along x; across the section (with spares); padded P = 2 nc
  int ncx, ncy;           // short-range cells along x and across the section (cells >= r_max)
  double hx, hy;          // mesh spacings [m]
  double alpha, rmax;     // splitting parameter [1/m] and short-range cutoff [m]
  const double *q_scale;  // device: fixed-point units per unit of scaled charge
  // complex values: float2 in the FP32 form, double2 in the FP64 form; half spectra (kz < P/2 as
  // [nx] planes of xs values, [P][P/2] and padding, then the plane kz = P/2 as [nx][P])
  int64_t xs;
  void *ghat[3];          // transformed, deconvolved Green's function per field component
  void *spec;             // three spectra (the charge's in the first), p3m_spectrum_values each
  void *field;            // field components at the nodes, nx x nc x nc x 4 reals, behind spec
  void *twiddles;         // 512 complex roots of unity
  unsigned long long *qmesh;   // fixed-point TSC charge, nx x nc x nc
  double *slong;          // [3][N] long-range part at the particles [1/m^2]
  int32_t *cell_of, *counts, *starts, *sorted;   // short-range cell list
  void *rec;              // cell-sorted source records of the short-range pass (N records)
  float2 *table;          // tabulated short-range profile (FP32 form), 2048 intervals + (0, 0)
};
int64_t p3m_plane_values(const P3mDev &m, size_t real_bytes);   // xs
int64_t p3m_spectrum_values(const P3mDev &m);                  // complex values of a half spectrum
size_t p3m_mesh_bytes(const P3mDev &m, size_t real_bytes);     // spec and field (a full FP64 mesh fits)
void p3m_setup_green(const P3mDev &m, double L, int images, bool fp32_mesh, hipStream_t s);
template <class Real> void launch_p3m(const State<Real> &st, const Phys &ph, const P3mDev &m, hipStream_t s);

// One-dimensional Eulerian low-fidelity model.
struct LfConst {
  double R, nu, rho_f, rho_p, re_tau, eps0;
  int n_wall, n_core;
};
void launch_lf(const LfConst &c, int64_t n, const double *d, const double *q, const double *A, double *out,
               hipStream_t s);

}  // namespace depo
