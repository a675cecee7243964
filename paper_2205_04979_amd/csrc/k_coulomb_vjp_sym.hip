// Symmetric Coulomb pair adjoint, FP32 form: the reverse of the symmetric
// direct sums (Eq. coulomb, Appendix A.2.4) under the same item list.
//
// With b_i = c_i a_bar_i (c_i the factor that turns the raw pair sum of particle
// i into its acceleration) and r = r_i - r_j, the pair law's contribution to the
// position adjoints is
//     x_bar_i += (1/u_x) J(r) p_ij,   p_ij = q_j b_i - q_i b_j,
// with J(r) = I/|r|^3 - 3 r r^T/|r|^5 (or (I - r^ r^T)/(|r| d_ij^2) inside the
// overlap clamp).  J is even in r and p_ji = -p_ij, so particle j receives
// exactly the negative: each unordered pair is evaluated once and its term is
// added to i and subtracted from j, as in the forward kernel.
//
// Schedule (same as the forward): the sources of an item are staged in LDS,
// two rounds of 64 at a time, each twice in a row; in step t lane l pairs its IPL targets with
// source (l + t) mod 64 and the three reaction sums travel with the source (DPP
// wave rotate), so after 64 steps they are back in the source's own lane.
// Per pair the fast body uses the point-charge form with |r|^2 + 1 (one rsq);
// a round that holds a pair closer than the largest diameter is recomputed
// with the exact clamp.  Diagonal items form all ordered pairs of their tile on
// the target side; their self pairs (step 0 of one round per target chunk) are
// skipped, since they contribute nothing.
//
// Items are combined with FP64 atomic adds into per-particle accumulators
// (the near-overlap branch of J has no useful a priori bound, so the forward's
// fixed-point scheme does not apply); k_vjp_finish scales by 1/u_x, writes the
// FP32 result and clears the accumulators.  The order of the FP64 additions
// varies from run to run; the FP32 results differ only when an FP64 sum lies
// within its own rounding error of an FP32 rounding boundary.
#include "common.hpp"
#include "launch.hpp"
#include "adjoint.hpp"

namespace depo {

namespace {

template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int IPL, int W> constexpr bool kCombine = IPL <= 2 && W > 1;   // as in the forward kernel
constexpr int kStage = 2;          // rounds of sources held in LDS at a time (a power of two; 8 KB, for 16 waves a CU)
constexpr int kWaveRol1 = 0x134;   // lane l receives the value of lane (l + 1) mod 64

__device__ __forceinline__ void dadd(double *acc, int64_t i, double v) { unsafeAtomicAdd(acc + i, v); }

// One round (64 ring steps) of four targets per lane in machine code, as the forward kernel's: bound by
// the vector instructions a SIMD issues (127 a step), whose three registers must not all be odd or all
// even.  Displacements, sums and reactions sit in odd registers, the products p in even ones.  Two targets go
// through the stages together (four would cost the wave its place beside three others); roots and lane
// rotations are issued at a raised wave priority.  Sixteen samples of 16,384: 1,560 -> 1,287 us per
// reverse step.
// addr: LDS byte address of the lane's record of step 0 (32-byte records); nq: minus the targets' charges.
// s: sums of the target side, r: of the reactions with the opposite sign, both set; returns the lanes in which
// some pair was near.
__device__ __forceinline__ uint64_t vjp_round4(uint32_t addr, const uint32_t (&x)[4], const float (&y)[4],
                                               const float (&z)[4], const float (&nq)[4], const float (&bx)[4],
                                               const float (&by)[4], const float (&bz)[4], float near2, float (&sx)[4],
                                               float (&sy)[4], float (&sz)[4], float &rx, float &ry, float &rz) {
  uint64_t mask;
  uint32_t cnt;
  // registers: sums v33..v55, reactions v57, v59, v61, charges v63..v69, displacements v71..v81 (odd); p v32..v42,
  // |r|^2 + 1 and its reciprocal root v44, v46, its square v48, v50, its cube v52, v54, r.p v56, v58 (even);
  // records v84..v99
#define DEPO_VJP_TWO(X, Y, Z, Q, BX, BY, BZ, A, B, NA, NB, SXA, SYA, SZA, SXB, SYB, SZB)                       \
  "v_sub_u32 v71, %[x" A "], " X "\n v_sub_u32 v73, %[x" B "], " X "\n"                                       \
  "v_sub_f32 v79, %[z" A "], " Z "\n v_sub_f32 v81, %[z" B "], " Z "\n"                                       \
  "v_cvt_f32_i32 v71, v71\n v_sub_f32 v75, %[y" A "], " Y "\n"                                               \
  "v_cvt_f32_i32 v73, v73\n v_sub_f32 v77, %[y" B "], " Y "\n"                                               \
  "v_mul_f32 v32, " Q ", %[bx" A "]\n v_mul_f32 v34, " Q ", %[bx" B "]\n"                                     \
  "v_mul_f32 v36, " Q ", %[by" A "]\n v_mul_f32 v38, " Q ", %[by" B "]\n"                                     \
  "v_mul_f32 v40, " Q ", %[bz" A "]\n v_mul_f32 v42, " Q ", %[bz" B "]\n"                                     \
  "v_fma_f32 v44, v79, v79, 1.0\n v_fma_f32 v46, v81, v81, 1.0\n"                                           \
  "v_fmac_f32 v32, " NA ", " BX "\n v_fmac_f32 v34, " NB ", " BX "\n"                                        \
  "v_fmac_f32 v44, v75, v75\n v_fmac_f32 v46, v77, v77\n"                                                   \
  "v_fmac_f32 v36, " NA ", " BY "\n v_fmac_f32 v38, " NB ", " BY "\n"                                        \
  "v_fmac_f32 v44, v71, v71\n v_fmac_f32 v46, v73, v73\n"                                                   \
  "v_fmac_f32 v40, " NA ", " BZ "\n v_fmac_f32 v42, " NB ", " BZ "\n"                                        \
  "v_mul_f32 v56, v71, v32\n v_mul_f32 v58, v73, v34\n"                                                     \
  "v_cmp_gt_f32 vcc, %[near2], v44\n s_or_b64 %[mask], %[mask], vcc\n"                                       \
  "v_cmp_gt_f32 vcc, %[near2], v46\n s_or_b64 %[mask], %[mask], vcc\n"                                       \
  "s_setprio 1\n v_rsq_f32 v44, v44\n v_rsq_f32 v46, v46\n s_setprio 0\n"                                   \
  "v_fmac_f32 v56, v75, v36\n v_fmac_f32 v58, v77, v38\n"                                                   \
  "v_fmac_f32 v56, v79, v40\n v_fmac_f32 v58, v81, v42\n"                                                   \
  "v_mul_f32 v48, v44, v44\n v_mul_f32 v50, v46, v46\n"                                                     \
  "v_mul_f32 v52, v48, v44\n v_mul_f32 v54, v50, v46\n"                                                     \
  "v_mul_f32 v48, 0xc0400000, v48\n v_mul_f32 v50, 0xc0400000, v50\n"                                       \
  "v_mul_f32 v56, v56, v48\n v_mul_f32 v58, v58, v50\n"                                                     \
  "v_fmac_f32 v32, v56, v71\n v_fmac_f32 v34, v58, v73\n"                                                   \
  "v_fmac_f32 v36, v56, v75\n v_fmac_f32 v38, v58, v77\n"                                                   \
  "v_fmac_f32 v40, v56, v79\n v_fmac_f32 v42, v58, v81\n"                                                   \
  "v_fmac_f32 v57, v52, v32\n v_fmac_f32 v59, v52, v36\n v_fmac_f32 v61, v52, v40\n"                        \
  "v_fmac_f32 " SXA ", v52, v32\n v_fmac_f32 " SYA ", v52, v36\n v_fmac_f32 " SZA ", v52, v40\n"            \
  "v_fmac_f32 v57, v54, v34\n v_fmac_f32 v59, v54, v38\n v_fmac_f32 v61, v54, v42\n"                        \
  "v_fmac_f32 " SXB ", v54, v34\n v_fmac_f32 " SYB ", v54, v38\n v_fmac_f32 " SZB ", v54, v42\n"
#define DEPO_VJP_STEP(X, Y, Z, Q, BX, BY, BZ)                                                                 \
  DEPO_VJP_TWO(X, Y, Z, Q, BX, BY, BZ, "0", "1", "v63", "v65", "v33", "v35", "v37", "v39", "v41", "v43")      \
  DEPO_VJP_TWO(X, Y, Z, Q, BX, BY, BZ, "2", "3", "v67", "v69", "v45", "v47", "v49", "v51", "v53", "v55")      \
  "s_setprio 1\n v_mov_b32_dpp v57, v57 wave_rol:1 row_mask:0xf bank_mask:0xf\n"                              \
  "v_mov_b32_dpp v59, v59 wave_rol:1 row_mask:0xf bank_mask:0xf\n"                                           \
  "v_mov_b32_dpp v61, v61 wave_rol:1 row_mask:0xf bank_mask:0xf\n s_setprio 0\n"
#define DEPO_VJP_A DEPO_VJP_STEP("v84", "v85", "v86", "v87", "v88", "v89", "v90")
#define DEPO_VJP_B DEPO_VJP_STEP("v92", "v93", "v94", "v95", "v96", "v97", "v98")
  // Every load is waited for inside the block (the last one reads entry 64 of the round, which is
  // stored, and is not used).
  asm volatile(
      "s_waitcnt lgkmcnt(0)\n"
      "ds_read_b128 v[84:87], %[addr]\n ds_read_b128 v[88:91], %[addr] offset:16\n"
      "s_mov_b64 %[mask], 0\n"
      "s_mov_b32 %[cnt], 32\n"
      "v_mov_b32 v33, 0\n v_mov_b32 v35, 0\n v_mov_b32 v37, 0\n v_mov_b32 v39, 0\n v_mov_b32 v41, 0\n"
      "v_mov_b32 v43, 0\n v_mov_b32 v45, 0\n v_mov_b32 v47, 0\n v_mov_b32 v49, 0\n v_mov_b32 v51, 0\n"
      "v_mov_b32 v53, 0\n v_mov_b32 v55, 0\n v_mov_b32 v57, 0\n v_mov_b32 v59, 0\n v_mov_b32 v61, 0\n"
      "v_mov_b32 v63, %[q0]\n v_mov_b32 v65, %[q1]\n v_mov_b32 v67, %[q2]\n v_mov_b32 v69, %[q3]\n"
      ".Lvjp%=:\n"
      "ds_read_b128 v[92:95], %[addr] offset:32\n ds_read_b128 v[96:99], %[addr] offset:48\n"
      "s_waitcnt lgkmcnt(2)\n" DEPO_VJP_A
      "ds_read_b128 v[84:87], %[addr] offset:64\n ds_read_b128 v[88:91], %[addr] offset:80\n"
      "v_add_u32 %[addr], 64, %[addr]\n s_waitcnt lgkmcnt(2)\n" DEPO_VJP_B
      "s_sub_u32 %[cnt], %[cnt], 1\n"
      "s_cmp_lg_u32 %[cnt], 0\n"
      "s_cbranch_scc1 .Lvjp%=\n"
      "s_waitcnt lgkmcnt(0)\n"
      : [mask] "=&s"(mask), [cnt] "=&s"(cnt), [addr] "+v"(addr), "=&{v33}"(sx[0]), "=&{v35}"(sy[0]), "=&{v37}"(sz[0]),
        "=&{v39}"(sx[1]), "=&{v41}"(sy[1]), "=&{v43}"(sz[1]), "=&{v45}"(sx[2]), "=&{v47}"(sy[2]), "=&{v49}"(sz[2]),
        "=&{v51}"(sx[3]), "=&{v53}"(sy[3]), "=&{v55}"(sz[3]), "=&{v57}"(rx), "=&{v59}"(ry), "=&{v61}"(rz)
      : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [y0] "v"(y[0]), [y1] "v"(y[1]),
        [y2] "v"(y[2]), [y3] "v"(y[3]), [z0] "v"(z[0]), [z1] "v"(z[1]), [z2] "v"(z[2]), [z3] "v"(z[3]),
        [q0] "v"(nq[0]), [q1] "v"(nq[1]), [q2] "v"(nq[2]), [q3] "v"(nq[3]), [bx0] "v"(bx[0]), [bx1] "v"(bx[1]),
        [bx2] "v"(bx[2]), [bx3] "v"(bx[3]), [by0] "v"(by[0]), [by1] "v"(by[1]), [by2] "v"(by[2]), [by3] "v"(by[3]),
        [bz0] "v"(bz[0]), [bz1] "v"(bz[1]), [bz2] "v"(bz[2]), [bz3] "v"(bz[3]), [near2] "s"(near2)
      : "v32", "v34", "v36", "v38", "v40", "v42", "v44", "v46", "v48", "v50", "v52", "v54", "v56", "v58", "v63", "v65",
        "v67", "v69", "v71", "v73", "v75", "v77", "v79", "v81", "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91",
        "v92", "v93", "v94", "v95", "v96", "v97", "v98", "v99", "vcc", "scc", "memory");
  return mask;
}

template <int IPL, int W, bool REACT>
__device__ __forceinline__ void vjp_item(const SymItem &it, const JAdj<float> *__restrict__ rec,
                                         const float *__restrict__ jr, double *__restrict__ ax,
                                         double *__restrict__ ay, double *__restrict__ az, float near2,
                                         JAdj<float> *src, float (*comb)[3][W][64]) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  uint32_t xi[IPL];
  float yi[IPL], zi[IPL], qi[IPL], bx[IPL], by[IPL], bz[IPL];
  bool valid[IPL];
#pragma unroll
  for (int k = 0; k < IPL; ++k) {
    const int ii = w * 64 * IPL + lane + 64 * k;
    valid[k] = ii < it.icount;
    const int i = it.i0 + (valid[k] ? ii : 0);
    const JAdj<float> me = rec[i];
    xi[k] = me.x; yi[k] = me.y; zi[k] = me.z;
    // absent targets: p = q_j * 0 - 0 * b_j = 0, no reaction
    qi[k] = valid[k] ? me.q : 0.0f;
    bx[k] = valid[k] ? me.bx : 0.0f;
    by[k] = valid[k] ? me.by : 0.0f;
    bz[k] = valid[k] ? me.bz : 0.0f;
  }
  double hx[IPL], hy[IPL], hz[IPL];
#pragma unroll
  for (int k = 0; k < IPL; ++k) hx[k] = hy[k] = hz[k] = 0.0;

  for (int jb = 0; jb < it.jcount; jb += 64) {
    if ((jb & (64 * kStage - 1)) == 0) {
      // stage the next kStage rounds (entry 128 r + k holds source 64 r + (k mod 64)); padding of the
      // last round has q = 0 and b = 0, so p = 0 and it contributes nothing to either side
      const int left = it.jcount - jb, n = 128 * min(kStage, (left + 63) >> 6);
      __syncthreads();
      for (int e = threadIdx.x; e < n; e += 64 * W) {
        const int jj = (e >> 7) * 64 + (e & 63);
        const bool has = jj < left;
        JAdj<float> r = rec[it.j0 + jb + (has ? jj : 0)];
        if (!has) r.q = r.bx = r.by = r.bz = 0.0f;
        src[e] = r;
      }
      __syncthreads();
    }
    const JAdj<float> *rs = src + 2 * (jb & (64 * kStage - 1)) + lane;
    float sx[IPL], sy[IPL], sz[IPL];
    float rx = 0.0f, ry = 0.0f, rz = 0.0f;   // reaction of the source now in this lane
#pragma unroll
    for (int k = 0; k < IPL; ++k) sx[k] = sy[k] = sz[k] = 0.0f;
    uint64_t nearmask = 0;
    auto step = [&](int t, int kskip) {
      const JAdj<float> s = rs[t];
#pragma unroll
      for (int k = 0; k < IPL; ++k) {
        if (k == kskip) continue;
        const float dx = sdiff(xi[k], s.x);
        const float dy = yi[k] - s.y;
        const float dz = zi[k] - s.z;
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, 1.0f)));
        nearmask |= __builtin_amdgcn_ballot_w64(r2 < near2);
        const float inv = __builtin_amdgcn_rsqf(r2);
        const float inv2 = inv * inv;
        const float inv3 = inv2 * inv;
        const float px = fmaf(s.q, bx[k], -qi[k] * s.bx);
        const float py = fmaf(s.q, by[k], -qi[k] * s.by);
        const float pz = fmaf(s.q, bz[k], -qi[k] * s.bz);
        const float t3 = -3.0f * (fmaf(dx, px, fmaf(dy, py, dz * pz)) * inv2);
        const float ux = fmaf(t3, dx, px), uy = fmaf(t3, dy, py), uz = fmaf(t3, dz, pz);
        sx[k] = fmaf(inv3, ux, sx[k]);
        sy[k] = fmaf(inv3, uy, sy[k]);
        sz[k] = fmaf(inv3, uz, sz[k]);
        if constexpr (REACT) {
          rx = fmaf(-inv3, ux, rx);
          ry = fmaf(-inv3, uy, ry);
          rz = fmaf(-inv3, uz, rz);
        }
      }
      if constexpr (REACT) {
        rx = dpp<kWaveRol1>(rx);
        ry = dpp<kWaveRol1>(ry);
        rz = dpp<kWaveRol1>(rz);
      }
    };
    if constexpr (REACT && IPL == 4) {
      float nq[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) nq[k] = -qi[k];
      // LDS addresses are the low 32 bits of a generic pointer into it
      nearmask = vjp_round4((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) JAdj<float> *)rs, xi, yi, zi,
                            nq, bx, by, bz, near2, sx, sy, sz, rx, ry, rz);
      rx = -rx;
      ry = -ry;
      rz = -rz;
    } else {
      const int kself = REACT ? -1 : (it.j0 - it.i0 + jb - w * 64 * IPL) >> 6;   // wave-uniform
      step(0, kself);
#pragma unroll 3
      for (int t = 1; t < 64; ++t) step(t, -1);
    }
    if (nearmask) {
      // exact pair law for this round: J p = k0 p - k1 (r.p / r^2) r, zero at r = 0
#pragma unroll
      for (int k = 0; k < IPL; ++k) sx[k] = sy[k] = sz[k] = 0.0f;
      rx = ry = rz = 0.0f;
      float ri[IPL];   // radii come from memory: this path is rare
#pragma unroll
      for (int k = 0; k < IPL; ++k) {
        const int ii = w * 64 * IPL + lane + 64 * k;
        ri[k] = jr[it.i0 + (ii < it.icount ? ii : 0)];
      }
      for (int t = 0; t < 64; ++t) {
        const JAdj<float> s = rs[t];
        const int jj = jb + ((lane + t) & 63);
        const float rj = jr[it.j0 + (jj < it.jcount ? jj : 0)];
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
          const float dx = sdiff(xi[k], s.x);
          const float dy = yi[k] - s.y;
          const float dz = zi[k] - s.z;
          const float r2 = dx * dx + dy * dy + dz * dz;
          float gx = 0.0f, gy = 0.0f, gz = 0.0f;
          if (r2 > 0.0f) {
            const float r = sqrtf(r2);
            const float dd = ri[k] + rj;
            const float px = s.q * bx[k] - qi[k] * s.bx;
            const float py = s.q * by[k] - qi[k] * s.by;
            const float pz = s.q * bz[k] - qi[k] * s.bz;
            const float rp = (dx * px + dy * py + dz * pz) / r2;
            float k0, k1;
            if (r >= dd) { k0 = 1.0f / (r2 * r); k1 = 3.0f * k0; }
            else { k0 = 1.0f / (r * dd * dd); k1 = k0; }
            gx = k0 * px - k1 * rp * dx;
            gy = k0 * py - k1 * rp * dy;
            gz = k0 * pz - k1 * rp * dz;
          }
          sx[k] += gx; sy[k] += gy; sz[k] += gz;
          if constexpr (REACT) { rx -= gx; ry -= gy; rz -= gz; }
        }
        if constexpr (REACT) {
          rx = dpp<kWaveRol1>(rx);
          ry = dpp<kWaveRol1>(ry);
          rz = dpp<kWaveRol1>(rz);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
      hx[k] += (double)sx[k];
      hy[k] += (double)sy[k];
      hz[k] += (double)sz[k];
    }
    if constexpr (REACT && kCombine<IPL, W>) {
      // after 64 rotations lane l holds the reaction of source jb + l on this wave's targets: the waves'
      // are added first (alternating buffers: one barrier a round)
      float(*c)[W][64] = comb[(jb >> 6) & 1];
      c[0][w][lane] = rx;
      c[1][w][lane] = ry;
      c[2][w][lane] = rz;
      __syncthreads();
      for (int e = threadIdx.x; e < 192; e += 64 * W) {
        const int k = e >> 6, jj = jb + (e & 63);
        if (jj >= it.jcount) continue;
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < W; ++q) v += (double)c[k][q][e & 63];
        dadd(k == 0 ? ax : k == 1 ? ay : az, (int64_t)it.j0 + jj, v);
      }
    } else if constexpr (REACT) {
      // after 64 rotations lane l holds the reaction of source jb + l on this wave's targets
      if (jb + lane < it.jcount) {
        const int64_t j = (int64_t)it.j0 + jb + lane;
        dadd(ax, j, (double)rx);
        dadd(ay, j, (double)ry);
        dadd(az, j, (double)rz);
      }
    }
  }

#pragma unroll
  for (int k = 0; k < IPL; ++k) {
    if (!valid[k]) continue;
    const int64_t i = it.i0 + w * 64 * IPL + lane + 64 * k;
    dadd(ax, i, hx[k]);
    dadd(ay, i, hy[k]);
    dadd(az, i, hz[k]);
  }
}

template <int IPL, int W>
__global__ __launch_bounds__(64 * W) void k_coulomb_vjp_sym(const SymItem *__restrict__ items,
                                                            const JAdj<float> *__restrict__ rec,
                                                            const float *__restrict__ jr, double *__restrict__ ax,
                                                            double *__restrict__ ay, double *__restrict__ az,
                                                            float near2) {
  __shared__ JAdj<float> src[128 * kStage];
  __shared__ float comb[kCombine<IPL, W> ? 2 : 1][3][W][64];
  const SymItem it = items[blockIdx.x];
  if (it.diag)
    vjp_item<IPL, W, false>(it, rec, jr, ax, ay, az, near2, src, comb);
  else
    vjp_item<IPL, W, true>(it, rec, jr, ax, ay, az, near2, src, comb);
}

// Totals (in units of the x quantum) to x_bar contributions; the accumulators are cleared.
__global__ __launch_bounds__(256) void k_vjp_finish(int32_t N, float inv_ux, double *__restrict__ ax,
                                                    double *__restrict__ ay, double *__restrict__ az,
                                                    float *__restrict__ ox, float *__restrict__ oy,
                                                    float *__restrict__ oz) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  ox[i] = (float)(ax[i] * (double)inv_ux);
  oy[i] = (float)(ay[i] * (double)inv_ux);
  oz[i] = (float)(az[i] * (double)inv_ux);
  ax[i] = 0.0;
  ay[i] = 0.0;
  az[i] = 0.0;
}

}  // namespace

void launch_coulomb_vjp_sym(const State<float> &st, const Phys &ph, const AdjState<float> &ad, int n_items,
                            const CoulombConfig &cfg, hipStream_t s) {
  // the forward's fixed-point accumulators are zero between evaluations; the same memory
  // holds the FP64 sums here and is zero again after k_vjp_finish
  double *ax = reinterpret_cast<double *>(st.accx);
  double *ay = reinterpret_cast<double *>(st.accy);
  double *az = reinterpret_cast<double *>(st.accz);
  // The forward's items fix the tile, and they are cut for its waves: the adjoint takes its targets per lane, where
  // those fewer than four fill the chip with more waves (eight reverse steps of four samples of 12,000
  // particles at (1, 8): 2,865 us, 4,183 as (4, 2); of one of 30,000 at (2, 4) 3,330, 3,930 as (4, 2)).
  // Eight per lane are more registers than the sums and products leave: (8, 1) runs as (4, 2) (two of 20,000
  // 8,900 -> 5,600 us with the forward steps).
  auto go = [&](auto kernel, int threads) {
    if (n_items > 0)
      hipLaunchKernelGGL(kernel, dim3(n_items), dim3(threads), 0, s, st.items, ad.rec, st.jr, ax, ay, az,
                         (float)ph.near2);
  };
  switch (coulomb_sym_tile(cfg)) {
    case 256:
      if (cfg.ipl == 1) go(k_coulomb_vjp_sym<1, 4>, 256);
      else if (cfg.ipl == 2) go(k_coulomb_vjp_sym<2, 2>, 128);
      else go(k_coulomb_vjp_sym<4, 1>, 64);
      break;
    case 512:
      if (cfg.ipl == 1) go(k_coulomb_vjp_sym<1, 8>, 512);
      else if (cfg.ipl == 2) go(k_coulomb_vjp_sym<2, 4>, 256);
      else go(k_coulomb_vjp_sym<4, 2>, 128);
      break;
    default: go(k_coulomb_vjp_sym<4, 4>, 256); break;   // 1,024
  }
  if (ph.N > 0)
    hipLaunchKernelGGL(k_vjp_finish, dim3((ph.N + 255) / 256), dim3(256), 0, s, ph.N, (float)ph.inv_ux, ax, ay, az,
                       ad.xc[0], ad.xc[1], ad.xc[2]);
}

}  // namespace depo
