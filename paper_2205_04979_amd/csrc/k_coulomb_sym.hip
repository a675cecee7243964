// Symmetric direct Coulomb sums (Eq. coulomb; F_i = sum_j F_ij n_ij, Appendix A.2.4),
// FP32 form: every unordered pair of a sample is evaluated once and its force
// is applied to both particles (F_ji = -F_ij, Newton's third law).
//
// The pair matrix of a sample is cut into items of T targets (a tile, T = 64 IPL W:
// IPL per lane, 64 IPL per wave) by a whole number of rounds of 64 sources: all
// sources after the tile, in equal pieces, and the tile's own (diagonal items,
// which form all ordered pairs on the target side only).  The number of rounds
// per item is the layout's (few for small ones: an item is the unit that spreads
// over the chip; 3,001 particles 132 -> 18 us per evaluation).  Per pair the body
// is the point-charge form r / (|r|^2 + 1)^(3/2) (one rsq); any round of sources
// that holds a pair closer than the largest diameter (wave-uniform ballot) is
// recomputed with the exact overlap clamp r / (|r| max(|r|, d_ij)^2).
//
// Ring schedule: sources are staged in LDS, four rounds at a time; a wave takes
// them 64 at a time (a round), one per lane, and in step t of a round lane l
// pairs its targets with source (l + t) mod 64, read from LDS (each round is
// stored twice in a row, so that entry l + t needs no wrap-around).  The reaction
// accumulated for a source travels with it: after each step the three
// accumulators move one lane down (DPP wave rotate), so after 64 steps every
// source's reaction from all 64 IPL targets of the wave is back in its own
// lane.  No cross-lane reduction tree; 3 VALU moves per step.
// * Target side: round sums are added to the running sum with Kahan
//   compensation.  Source side: each wave adds its reaction on the round's
//   sources as soon as the round ends.
// * Items are combined in 64-bit fixed point: each item adds its target and
//   source partials, rounded to multiples of 2^-62 of a per-sample bound on
//   |sum| (sum_j |q~_j| / d_min^2, so no total or intermediate sum can
//   overflow), to per-particle integer accumulators with atomic adds.
//   Integer addition is associative, so the result does not depend on the
//   order in which items finish: bitwise reproducible.  k_pair_finish converts
//   the totals back and clears the accumulators for the next evaluation.
#include "common.hpp"
#include "launch.hpp"

namespace depo {

namespace {

// every lane receives a value under a wave rotate, so the old-value operand is never used
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// The waves of a workgroup add their reactions on a source before the accumulators get them, in the shapes of
// small layouts, where the atomic additions count (five samples of 5,000 to 6,000 particles at (1, 4): a
// third of the kernel; 62.8 -> 49.4 us; one of 9,000 37.6 -> 30.4 us, of 16,000 at (2, 2) 75.8 -> 72.8 us);
// the barrier this takes each round would hold up four targets per lane.
template <int IPL, int W> constexpr bool kCombine = IPL <= 2 && W > 1;
constexpr int kStage = 4;          // rounds of sources held in LDS at a time (a power of two)
constexpr int kWaveRol1 = 0x134;   // lane l receives the value of lane (l + 1) mod 64

__device__ __forceinline__ void fx_add(unsigned long long *acc, int64_t i, double v, double scale) {
  atomicAdd(acc + i, (unsigned long long)__double2ll_rn(v * scale));
}

// y or z difference of two records: float records subtract; integer records (bit patterns of
// int32 x-quanta counts) subtract exactly and convert.
template <bool INTREC> __device__ __forceinline__ float rdiff(float a, float b) {
  if constexpr (INTREC) return (float)(__float_as_int(a) - __float_as_int(b));
  else return a - b;
}

// One round (64 ring steps) of four targets per lane and float records, in machine code.  What
// bounds the kernel is the rate at which a SIMD issues vector instructions (79 per step and four
// pairs).  A three-operand instruction whose registers are all odd or all even takes two issue slots
// instead of one (measured: 4.5 against 2.25 cycles for v_fmac_f32); left to the compiler a sixth of the
// accumulations did, and the copies it added made 83 instructions.  Here every accumulator sits in an
// odd register and every weight in an even one, each stage runs over the four targets before the
// next, and the next source record is on its way while one is evaluated.
// The reciprocal roots and the lane rotations hold back the wave that issues them, and waves in step with
// each other wait together; they are issued at a raised wave priority, so that the other waves'
// multiply-adds fill in behind them (without it: 11 % slower).
// Measured (pair sums per step, compiled body with an item per two tiles -> this one): 65,536 particles
// 893 -> 762 us; ten samples of 2,048 to 32,768 740 -> 635 us; 2^20 particles 213 -> 192.5 ms, 70 TFLOP/s
// at 25 operations per unordered pair.
// addr: LDS byte address of the lane's record of step 0 (16-byte records); s: sums of the target
// side, r: reactions, both set; returns the lanes in which some pair was near.
__device__ __forceinline__ uint64_t ring_round4(uint32_t addr, const uint32_t (&x)[4], const float (&y)[4],
                                                const float (&z)[4], const float (&q)[4], float near2,
                                                float (&sx)[4], float (&sy)[4], float (&sz)[4], float &rx, float &ry,
                                                float &rz) {
  uint64_t mask;
  uint32_t cnt;
  // registers: sums v33..v55 and reactions v57, v59, v61 (odd); weights v32..v46 (even); dx v48..v54,
  // dy v56..v62 (even), dz v63..v66; |r|^2 + 1, then its reciprocal root v67..v70; records v72..v79
#define DEPO_RING_STEP(X, Y, Z, Q)                                                                     \
  "v_sub_u32 v48, %[x0], " X "\n v_sub_u32 v50, %[x1], " X "\n"                                        \
  "v_sub_u32 v52, %[x2], " X "\n v_sub_u32 v54, %[x3], " X "\n"                                        \
  "v_sub_f32 v63, %[z0], " Z "\n v_sub_f32 v64, %[z1], " Z "\n"                                        \
  "v_sub_f32 v65, %[z2], " Z "\n v_sub_f32 v66, %[z3], " Z "\n"                                        \
  "v_cvt_f32_i32 v48, v48\n v_sub_f32 v56, %[y0], " Y "\n v_cvt_f32_i32 v50, v50\n"                    \
  "v_sub_f32 v58, %[y1], " Y "\n v_cvt_f32_i32 v52, v52\n v_sub_f32 v60, %[y2], " Y "\n"               \
  "v_cvt_f32_i32 v54, v54\n v_sub_f32 v62, %[y3], " Y "\n"                                            \
  "v_fma_f32 v67, v63, v63, 1.0\n v_fma_f32 v68, v64, v64, 1.0\n"                                     \
  "v_fma_f32 v69, v65, v65, 1.0\n v_fma_f32 v70, v66, v66, 1.0\n"                                     \
  "v_fmac_f32 v67, v56, v56\n v_fmac_f32 v68, v58, v58\n"                                             \
  "v_fmac_f32 v69, v60, v60\n v_fmac_f32 v70, v62, v62\n"                                             \
  "v_fmac_f32 v67, v48, v48\n v_fmac_f32 v68, v50, v50\n"                                             \
  "v_fmac_f32 v69, v52, v52\n v_fmac_f32 v70, v54, v54\n"                                             \
  "v_cmp_gt_f32 vcc, %[near2], v67\n s_or_b64 %[mask], %[mask], vcc\n"                                \
  "v_cmp_gt_f32 vcc, %[near2], v68\n s_or_b64 %[mask], %[mask], vcc\n"                                   \
  "v_cmp_gt_f32 vcc, %[near2], v69\n s_or_b64 %[mask], %[mask], vcc\n"                                   \
  "v_cmp_gt_f32 vcc, %[near2], v70\n s_or_b64 %[mask], %[mask], vcc\n"                                   \
  "s_setprio 1\n v_rsq_f32 v67, v67\n v_rsq_f32 v68, v68\n v_rsq_f32 v69, v69\n v_rsq_f32 v70, v70\n s_setprio 0\n" \
  "v_mul_f32 v32, v67, v67\n v_mul_f32 v34, v68, v68\n"                                               \
  "v_mul_f32 v36, v69, v69\n v_mul_f32 v38, v70, v70\n"                                               \
  "v_mul_f32 v67, v67, v32\n v_mul_f32 v68, v68, v34\n"                                               \
  "v_mul_f32 v69, v69, v36\n v_mul_f32 v70, v70, v38\n"                                               \
  "v_mul_f32 v40, %[q0], v67\n v_mul_f32 v42, %[q1], v68\n"                                           \
  "v_mul_f32 v44, %[q2], v69\n v_mul_f32 v46, %[q3], v70\n"                                           \
  "v_mul_f32 v32, " Q ", v67\n v_mul_f32 v34, " Q ", v68\n"                                           \
  "v_mul_f32 v36, " Q ", v69\n v_mul_f32 v38, " Q ", v70\n"                                           \
  "v_fmac_f32 v57, v40, v48\n v_fmac_f32 v59, v40, v56\n v_fmac_f32 v61, v40, v63\n"                  \
  "v_fmac_f32 v33, v32, v48\n v_fmac_f32 v35, v32, v56\n v_fmac_f32 v37, v32, v63\n"                  \
  "v_fmac_f32 v57, v42, v50\n v_fmac_f32 v59, v42, v58\n v_fmac_f32 v61, v42, v64\n"                  \
  "v_fmac_f32 v39, v34, v50\n v_fmac_f32 v41, v34, v58\n v_fmac_f32 v43, v34, v64\n"                  \
  "v_fmac_f32 v57, v44, v52\n v_fmac_f32 v59, v44, v60\n v_fmac_f32 v61, v44, v65\n"                  \
  "v_fmac_f32 v45, v36, v52\n v_fmac_f32 v47, v36, v60\n v_fmac_f32 v49, v36, v65\n"                  \
  "v_fmac_f32 v57, v46, v54\n v_fmac_f32 v59, v46, v62\n v_fmac_f32 v61, v46, v66\n"                  \
  "v_fmac_f32 v51, v38, v54\n v_fmac_f32 v53, v38, v62\n v_fmac_f32 v55, v38, v66\n"                  \
  "s_setprio 1\n v_mov_b32_dpp v57, v57 wave_rol:1 row_mask:0xf bank_mask:0xf\n"                                    \
  "v_mov_b32_dpp v59, v59 wave_rol:1 row_mask:0xf bank_mask:0xf\n"                                    \
  "v_mov_b32_dpp v61, v61 wave_rol:1 row_mask:0xf bank_mask:0xf\n s_setprio 0\n"
#define DEPO_RING_A DEPO_RING_STEP("v72", "v73", "v74", "v75")
#define DEPO_RING_B DEPO_RING_STEP("v76", "v77", "v78", "v79")
  // Every load is waited for inside the block (the last one reads entry 64 of the round, which is
  // stored, and is not used).
  asm volatile(
      "s_waitcnt lgkmcnt(0)\n"
      "ds_read_b128 v[72:75], %[addr]\n"
      "s_mov_b64 %[mask], 0\n"
      "s_mov_b32 %[cnt], 16\n"
      "v_mov_b32 v33, 0\n v_mov_b32 v35, 0\n v_mov_b32 v37, 0\n v_mov_b32 v39, 0\n v_mov_b32 v41, 0\n"
      "v_mov_b32 v43, 0\n v_mov_b32 v45, 0\n v_mov_b32 v47, 0\n v_mov_b32 v49, 0\n v_mov_b32 v51, 0\n"
      "v_mov_b32 v53, 0\n v_mov_b32 v55, 0\n v_mov_b32 v57, 0\n v_mov_b32 v59, 0\n v_mov_b32 v61, 0\n"
      ".Lring%=:\n"
      "ds_read_b128 v[76:79], %[addr] offset:16\n s_waitcnt lgkmcnt(1)\n" DEPO_RING_A
      "ds_read_b128 v[72:75], %[addr] offset:32\n s_waitcnt lgkmcnt(1)\n" DEPO_RING_B
      "ds_read_b128 v[76:79], %[addr] offset:48\n s_waitcnt lgkmcnt(1)\n" DEPO_RING_A
      "ds_read_b128 v[72:75], %[addr] offset:64\n v_add_u32 %[addr], 64, %[addr]\n s_waitcnt lgkmcnt(1)\n" DEPO_RING_B
      "s_sub_u32 %[cnt], %[cnt], 1\n"
      "s_cmp_lg_u32 %[cnt], 0\n"
      "s_cbranch_scc1 .Lring%=\n"
      "s_waitcnt lgkmcnt(0)\n"
      : [mask] "=&s"(mask), [cnt] "=&s"(cnt), [addr] "+v"(addr), "=&{v33}"(sx[0]), "=&{v35}"(sy[0]), "=&{v37}"(sz[0]),
        "=&{v39}"(sx[1]), "=&{v41}"(sy[1]), "=&{v43}"(sz[1]), "=&{v45}"(sx[2]), "=&{v47}"(sy[2]), "=&{v49}"(sz[2]),
        "=&{v51}"(sx[3]), "=&{v53}"(sy[3]), "=&{v55}"(sz[3]), "=&{v57}"(rx), "=&{v59}"(ry), "=&{v61}"(rz)
      : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [y0] "v"(y[0]), [y1] "v"(y[1]),
        [y2] "v"(y[2]), [y3] "v"(y[3]), [z0] "v"(z[0]), [z1] "v"(z[1]), [z2] "v"(z[2]), [z3] "v"(z[3]),
        [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), [near2] "s"(near2)
      : "v32", "v34", "v36", "v38", "v40", "v42", "v44", "v46", "v48", "v50", "v52", "v54", "v56", "v58", "v60", "v62",
        "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v72", "v73", "v74", "v75", "v76", "v77", "v78",
        "v79", "vcc", "scc", "memory");
  return mask;
}

template <int IPL, int W, bool REACT, bool INTREC>
__device__ __forceinline__ void ring_item(const SymItem &it, const JSrc<float> *__restrict__ js,
                                          const float *__restrict__ jr, double scale,
                                          unsigned long long *__restrict__ accx, unsigned long long *__restrict__ accy,
                                          unsigned long long *__restrict__ accz, float near2, JSrc<float> *src,
                                          float (*comb)[3][W][64]) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  uint32_t xi[IPL];
  float yi[IPL], zi[IPL], qi[IPL], ri[IPL];
  bool valid[IPL];
#pragma unroll
  for (int k = 0; k < IPL; ++k) {
    const int ii = w * 64 * IPL + lane + 64 * k;
    valid[k] = ii < it.icount;
    const int i = it.i0 + (valid[k] ? ii : 0);
    const JSrc<float> me = js[i];
    xi[k] = me.x; yi[k] = me.y; zi[k] = me.z;
    qi[k] = valid[k] ? me.q : 0.0f;   // absent targets exert no reaction
    ri[k] = jr[i];
  }
  float hx[IPL], hy[IPL], hz[IPL], cx[IPL], cy[IPL], cz[IPL];
#pragma unroll
  for (int k = 0; k < IPL; ++k) hx[k] = hy[k] = hz[k] = cx[k] = cy[k] = cz[k] = 0.0f;

  for (int jb = 0; jb < it.jcount; jb += 64) {
    if ((jb & (64 * kStage - 1)) == 0) {
      // stage the next kStage rounds, each twice in a row (entry 128 r + k holds source
      // 64 r + (k mod 64)); charge 0 beyond jcount: padding of the last round
      const int left = it.jcount - jb, n = 128 * min(kStage, (left + 63) >> 6);
      __syncthreads();
      for (int e = threadIdx.x; e < n; e += 64 * W) {
        const int jj = (e >> 7) * 64 + (e & 63);
        const bool has = jj < left;
        JSrc<float> r = js[it.j0 + jb + (has ? jj : 0)];
        if (!has) r.q = 0.0f;
        src[e] = r;
      }
      __syncthreads();
    }
    const JSrc<float> *rs = src + 2 * (jb & (64 * kStage - 1)) + lane;
    float sx[IPL], sy[IPL], sz[IPL];
    float rx = 0.0f, ry = 0.0f, rz = 0.0f;   // reaction of the source now in this lane
#pragma unroll
    for (int k = 0; k < IPL; ++k) sx[k] = sy[k] = sz[k] = 0.0f;
    uint64_t nearmask = 0;
    // one ring step; target kskip (if any) is skipped: in a diagonal item, step 0 of the round
    // that holds target chunk k pairs every lane with itself (zero force, but never "near")
    auto step = [&](int t, int kskip) {
      const JSrc<float> s = rs[t];
#pragma unroll
      for (int k = 0; k < IPL; ++k) {
        if (k == kskip) continue;
        const float dx = sdiff(xi[k], s.x);
        const float dy = rdiff<INTREC>(yi[k], s.y);
        const float dz = rdiff<INTREC>(zi[k], s.z);
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, 1.0f)));
        nearmask |= __builtin_amdgcn_ballot_w64(r2 < near2);
        const float inv = __builtin_amdgcn_rsqf(r2);
        const float i3 = (inv * inv) * inv;
        const float wt = s.q * i3;
        sx[k] = fmaf(wt, dx, sx[k]);
        sy[k] = fmaf(wt, dy, sy[k]);
        sz[k] = fmaf(wt, dz, sz[k]);
        if constexpr (REACT) {
          const float ws = qi[k] * i3;
          rx = fmaf(ws, dx, rx);
          ry = fmaf(ws, dy, ry);
          rz = fmaf(ws, dz, rz);
        }
      }
      if constexpr (REACT) {
        // as in ring_round4 (18,000 particles, two targets per lane: 93 -> 87 us; raised for the root
        // too it gains nothing here; with four and more per lane it only loses: see below)
        if constexpr (IPL <= 2) __builtin_amdgcn_s_setprio(1);
        rx = dpp<kWaveRol1>(rx);
        ry = dpp<kWaveRol1>(ry);
        rz = dpp<kWaveRol1>(rz);
        if constexpr (IPL <= 2) __builtin_amdgcn_s_setprio(0);
      }
    };
    if constexpr (REACT && IPL == 4 && !INTREC) {
      // LDS addresses are the low 32 bits of a generic pointer into it
      nearmask = ring_round4((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) JSrc<float> *)rs, xi, yi, zi,
                             qi, near2, sx, sy, sz, rx, ry, rz);
    } else if constexpr (REACT && IPL <= 2) {
#pragma unroll 4
      for (int t = 0; t < 64; ++t) step(t, -1);
    } else if constexpr (REACT) {
      // The integer records' four targets per lane, and eight: two steps at a time and no raised priority.  2^20
      // particles in integer records at (4, 4): 255.6 ms with four steps and the priority raised, 245.1 with four, 237.7
      // so; 65,536 at (4, 1) 1,075, 1,027, 1,001 us, at (8, 1) 1,249 with both, 1,046 with four.
#pragma unroll 2
      for (int t = 0; t < 64; ++t) step(t, -1);
    } else {
      // wave-uniform; outside [0, IPL) when no self pair
      const int kself = (it.j0 - it.i0 + jb - w * 64 * IPL) >> 6;
      step(0, kself);
#pragma unroll 3
      for (int t = 1; t < 64; ++t) step(t, -1);
    }
    if (nearmask) {
      // exact overlap clamp for this round, both sides: r / (|r| max(|r|, d_ij)^2), zero at r = 0
#pragma unroll
      for (int k = 0; k < IPL; ++k) sx[k] = sy[k] = sz[k] = 0.0f;
      rx = ry = rz = 0.0f;
      for (int t = 0; t < 64; ++t) {
        const JSrc<float> s = rs[t];
        const int jj = jb + ((lane + t) & 63);   // radii come from memory: this path is rare
        const float rj = jr[it.j0 + (jj < it.jcount ? jj : 0)];
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
          const float dx = sdiff(xi[k], s.x);
          const float dy = rdiff<INTREC>(yi[k], s.y);
          const float dz = rdiff<INTREC>(zi[k], s.z);
          const float r2 = dx * dx + dy * dy + dz * dz;
          const float dd = ri[k] + rj;
          const float rc2 = fmaxf(r2, dd * dd);
          const float f = r2 > 0.0f ? 1.0f / (sqrtf(r2) * rc2) : 0.0f;
          const float wt = s.q * f;
          sx[k] = fmaf(wt, dx, sx[k]);
          sy[k] = fmaf(wt, dy, sy[k]);
          sz[k] = fmaf(wt, dz, sz[k]);
          if constexpr (REACT) {
            const float ws = qi[k] * f;
            rx = fmaf(ws, dx, rx);
            ry = fmaf(ws, dy, ry);
            rz = fmaf(ws, dz, rz);
          }
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
      float y, t;
      y = sx[k] - cx[k]; t = hx[k] + y; cx[k] = (t - hx[k]) - y; hx[k] = t;
      y = sy[k] - cy[k]; t = hy[k] + y; cy[k] = (t - hy[k]) - y; hy[k] = t;
      y = sz[k] - cz[k]; t = hz[k] + y; cz[k] = (t - hz[k]) - y; hz[k] = t;
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
        fx_add(k == 0 ? accx : k == 1 ? accy : accz, (int64_t)it.j0 + jj, -v, scale);
      }
    } else if constexpr (REACT) {
      // after 64 rotations lane l holds the reaction of source jb + l on this wave's targets
      if (jb + lane < it.jcount) {
        const int64_t j = (int64_t)it.j0 + jb + lane;
        fx_add(accx, j, -(double)rx, scale);
        fx_add(accy, j, -(double)ry, scale);
        fx_add(accz, j, -(double)rz, scale);
      }
    }
  }

  // target side: this item's partial of each valid target
#pragma unroll
  for (int k = 0; k < IPL; ++k) {
    if (!valid[k]) continue;
    const int64_t i = it.i0 + w * 64 * IPL + lane + 64 * k;
    fx_add(accx, i, (double)hx[k] - (double)cx[k], scale);
    fx_add(accy, i, (double)hy[k] - (double)cy[k], scale);
    fx_add(accz, i, (double)hz[k] - (double)cz[k], scale);
  }
}

template <int IPL, int W, bool INTREC>
__global__ __launch_bounds__(64 * W) void k_coulomb_sym(const SymItem *__restrict__ items,
                                                        const JSrc<float> *__restrict__ js,
                                                        const float *__restrict__ jr,
                                                        const double *__restrict__ fx_scale,
                                                        unsigned long long *__restrict__ accx,
                                                        unsigned long long *__restrict__ accy,
                                                        unsigned long long *__restrict__ accz, float near2) {
  __shared__ JSrc<float> src[128 * kStage];
  __shared__ float comb[kCombine<IPL, W> ? 2 : 1][3][W][64];
  const SymItem it = items[blockIdx.x];
  const double scale = fx_scale[it.sample];
  if (it.diag)
    ring_item<IPL, W, false, INTREC>(it, js, jr, scale, accx, accy, accz, near2, src, comb);
  else
    ring_item<IPL, W, true, INTREC>(it, js, jr, scale, accx, accy, accz, near2, src, comb);
}

// Fixed-point totals back to pair sums; the accumulators are cleared for the next evaluation.
__global__ __launch_bounds__(256) void k_pair_finish(int32_t N, const int32_t *__restrict__ sid,
                                                     const double *__restrict__ fx_scale,
                                                     unsigned long long *__restrict__ accx,
                                                     unsigned long long *__restrict__ accy,
                                                     unsigned long long *__restrict__ accz, float *__restrict__ ox,
                                                     float *__restrict__ oy, float *__restrict__ oz) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const double inv = 1.0 / fx_scale[sid[i]];
  ox[i] = (float)((double)(long long)accx[i] * inv);
  oy[i] = (float)((double)(long long)accy[i] * inv);
  oz[i] = (float)((double)(long long)accz[i] * inv);
  accx[i] = 0ull;
  accy[i] = 0ull;
  accz[i] = 0ull;
}

}  // namespace

// (targets per lane, waves); T = 64 IPL W targets per tile, rounds of 64 sources
#define DEPO_COULOMB_SYM_CASES(X) X(1, 4) X(1, 8) X(2, 2) X(2, 4) X(4, 1) X(4, 2) X(4, 4) X(8, 1)

int coulomb_sym_tile(const CoulombConfig &cfg) { return 64 * cfg.ipl * cfg.waves; }

bool coulomb_sym_supported(const CoulombConfig &cfg) {
  if (!cfg.symmetric || !cfg.compensated || cfg.block != 64) return false;
#define X(I, W) \
  if (cfg.ipl == I && cfg.waves == W) return true;
  DEPO_COULOMB_SYM_CASES(X)
#undef X
  return false;
}

void launch_coulomb_sym(const State<float> &st, const Phys &ph, int n_items, const CoulombConfig &cfg,
                        hipStream_t s, bool defer_finish) {
  const float near2 = (float)ph.near2;
#define X(I, W)                                                                                              \
  if (n_items > 0 && cfg.ipl == I && cfg.waves == W) {                                                       \
    if (cfg.int_rec)                                                                                         \
      hipLaunchKernelGGL((k_coulomb_sym<I, W, true>), dim3(n_items), dim3(64 * W), 0, s, st.items, st.js,    \
                         st.jr, st.fx_scale, st.accx, st.accy, st.accz, near2);                              \
    else                                                                                                     \
      hipLaunchKernelGGL((k_coulomb_sym<I, W, false>), dim3(n_items), dim3(64 * W), 0, s, st.items, st.js,   \
                         st.jr, st.fx_scale, st.accx, st.accy, st.accz, near2);                              \
  }
  DEPO_COULOMB_SYM_CASES(X)
#undef X
  if (ph.N > 0 && !defer_finish)
    hipLaunchKernelGGL(k_pair_finish, dim3((ph.N + 255) / 256), dim3(256), 0, s, ph.N, st.sid, st.fx_scale, st.accx,
                       st.accy, st.accz, st.cx, st.cy, st.cz);
}

}  // namespace depo
