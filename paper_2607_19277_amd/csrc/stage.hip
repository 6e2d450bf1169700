// stage.hip -- the fused SSP Runge-Kutta stage update of one 16^3 block per
// workgroup on gfx950 (the paper's macro-kernel, Sec. 2.1.3, re-designed for
// CDNA4), for the Euler equations (HLL, HLLC, LF) and the SRHD module (LF;
// its con2prim per cell and ghost), with minmod or van Leer slopes.
//
// 256 lanes = 4 wave64; lane (i, j) owns the z-column (i, j) of the block.
// The block is marched plane by plane in z (2.5-D):
//   - the conserved values of the column are streamed through a register
//     ring (cells k, k+1 and k+2, the last one arriving while the plane's x
//     and y faces are computed), so each interior value is read from HBM once
//     per stage;
//   - z faces: each lane keeps the primitives of cells k, k+1 and the left
//     PLM state of face k+1/2, and computes one z-face flux per plane;
//   - x/y faces of plane k: the plane's primitives (interior + 2 ghost
//     columns / rows) go to LDS (double-buffered: plane k+1 is written while
//     plane k's faces are computed, one barrier per plane); every lane takes
//     the lower x and the lower y face of its own cell (its own state from
//     registers, the three others from LDS at fixed offsets), and the 16 + 16
//     upper faces of the plane are one wave's extra task; each face flux is
//     computed exactly once (the paper evaluates both faces of every cell)
//     and read back from LDS by the cell below it;
//   - waves 0 and 1 (rotated over blocks) also load and convert the plane's
//     128 ghost cells, waves 2 and 3 take the extra face task in turn;
//   - update: L = -((dFx + dFy) + dFz)/dx, then
//     SSP-RK2 stage 1: U1 = U + dt L;  stage 2: U' = (U^n + (U1 + dt L))/2;
//     SSP-RK3: U1 = U + dt L, U2 = 3/4 U^n + 1/4 (U1 + dt L),
//     U' = 1/3 U^n + 2/3 (U2 + dt L); written with the x-boundary export and
//     the face fluxes kept for coarse-fine flux correction; the last stage
//     also reduces the CFL signal rate of the new state (cells to be
//     flux-corrected excepted).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "agile_internal.hpp"
#include "device_math.hpp"

namespace agile {

namespace {

constexpr int NV = 5;
// A plane's primitives in LDS, per variable: the two lower y ghost rows (16
// each), the 16 rows with their x ghosts (20 each), the two upper y ghost rows.
constexpr int PW = BN + 2 * NG;
constexpr int PMID = NG * BN, PTOP = PMID + BN * PW, PLANE = PTOP + NG * BN;   // 32, 352, 384
// Its face fluxes: the lower y ones in lane order, the upper y ones, the 17 x
// faces of every row.
constexpr int FYTOP = BN * BN, FX = FYTOP + BN, NFX = BN + 1, NFACE = FX + BN * NFX;   // 256, 272, 17, 544

// Workgroups are dealt to the 8 XCDs of the chip round-robin.  With xcd = 1
// each XCD gets one contiguous range of work items (blocks in level + Morton
// order, slabs of a block adjacent) so that most same-level neighbours run on
// the same XCD and their boundary rows can be served from that XCD's L2.
__device__ __forceinline__ int xcd_item(int w, int n, int xcd) {
    if (!xcd) return w;
    const int chunk = (n + 7) >> 3;
    return (w & 7) * chunk + (w >> 3);
}
inline int xcd_grid(int n, int xcd) { return xcd ? 8 * ((n + 7) >> 3) : n; }

// primitives of a conserved state: Euler (rho, v, p), or for the SRHD
// module (RS = 3) (rho, Gamma v, p) from the root finding in xi
template <int RS>
__device__ __forceinline__ bool phys_prim(const double C[NV], double gamma, double gm1, double q[NV]) {
    if (RS == 3) return srhd_con2prim_fast(C, gamma, q);
    return cons2prim(C, gm1, q);
}

template <int RS, typename R>
__device__ __forceinline__ void to_prim_z(const double C[NV], double gamma, double gm1, R w[NV], bool &ok) {
    double q[NV];
    ok &= phys_prim<RS>(C, gamma, gm1, q);
    // rotated to the z normal: (rho, vz, vx, vy, p)
    w[0] = R(q[0]); w[1] = R(q[3]); w[2] = R(q[1]); w[3] = R(q[2]); w[4] = R(q[4]);
}

} // namespace

#ifndef AGILE_STAGE_WAVES_F64
#define AGILE_STAGE_WAVES_F64 2
#endif
#ifndef AGILE_STAGE_WAVES_F32
#define AGILE_STAGE_WAVES_F32 3
#endif

// RS: 0 HLL, 1 HLLC, 2 local Lax-Friedrichs, 3 the SRHD module (local
// Lax-Friedrichs on (rho, Gamma v, p)); LIM: 0 minmod, 1 van Leer;
// KIND: 1 first stage (U1 = U + dt L), 2 last SSP-RK2 stage
// ((U^n + (U1 + dt L))/2), 3 middle SSP-RK3 stage (3/4 U^n + 1/4 (U1 + dt L)),
// 4 last SSP-RK3 stage (1/3 U^n + 2/3 (U2 + dt L)).  The last stage of a step
// also reduces the signal rate of the new state.
//
// Bound by VALU work and by the waits that 2 waves per SIMD (FP64; 3 with FP32
// fluxes) do not cover, next to HBM.  Counters of 1856 blocks, HLLC, FP64: of its
// cycles a wave issues VALU instructions in 35%, waits for memory, LDS or the
// barrier in 30%, for its turn or a dependency in 22%; with 1.85 waves on a SIMD the
// VALU is busy for 64% of a launch (256^3 blocks of a shear layer 68%, SRHD 82%).
// The first / last stage move 0.93 / 1.23 GB, 4.5 / 5.3 TB/s against the 6.5 of a
// copy.  Output and U^n are each touched once per launch and carry streaming
// (nontemporal) hints, so that they do not displace, in L2, the input planes and
// ghost rows that neighbouring work items read again.  Fixed face ownership (no index arithmetic, no rotation
// selects, own state from registers), ghosts converted once and wave-uniform
// addresses took an HLLC first stage from 673 to 510 VALU instructions per wave
// and plane; with the shorter fluxes, 278 / 308 -> 215 / 241 us (FP32 fluxes
// 171 / 207).  Not faster: three waves per SIMD (168 registers; the face work
// then spills or loses its instruction-level parallelism, 2-15% slower), the
// upper faces of 8 planes at once from global memory (balanced over the waves,
// 4% slower), cells or ghosts loaded one plane further ahead (equal, or up to
// 3% slower).  On noisy data (256^3 shear layer) the clock drops from 2.39 to
// 2.04 GHz under this kernel, so there operations cost their energy too.
template <int RS, int LIM, int KIND, typename R>
__global__ __launch_bounds__(256, sizeof(R) == 8 ? AGILE_STAGE_WAVES_F64 : AGILE_STAGE_WAVES_F32) void k_stage(StageArgs a) {
    constexpr bool FIRST = KIND == 1, LAST = KIND == 2 || KIND == 4;
    // plane primitives and face fluxes, double-buffered by plane parity so
    // that one barrier per plane separates producers from consumers
    __shared__ R sP[2][NV][PLANE];
    __shared__ R sF[2][NV][NFACE];
    // the x-boundary columns of a plane's output, as they stand in XE; stored
    // by consecutive lanes after the next plane's barrier
    __shared__ __align__(16) double sXE[2][2 * NV * BN * NG];

    // work item = (block, slab of kslab planes)
    const int nslab = BN / a.kslab;
    const int item = xcd_item(blockIdx.x, a.nblocks * nslab, a.xcd);
    if (item >= a.nblocks * nslab) return;
    const int bi = item / nslab, slab = item - bi * nslab;
    const int b = a.list ? a.list[bi] : bi;
    const int k0 = slab * a.kslab, k1 = k0 + a.kslab;
    const int tid = threadIdx.x;
    const int i = tid & 15, j = tid >> 4;
    const BlockDesc D = a.desc[b];
    MeshParams &mp = a.mp[D.mesh];
    const double gamma = mp.gamma;
    const double gm1 = gamma - 1.0;
    const R gammaR = R(gamma), igm1R = R(1.0 / gm1);
    const double inv_dx = mp.inv_dx1 * double(1 << (D.level - 1));
    double dtdx = FIRST && a.prev ? 0.0 : mp.dt * inv_dx;
    // In a chain of steps (at most 64 blocks to a mesh) no launch stands between
    // the last stage of a step and the first one of the next: each wave takes
    // the maximum of its mesh itself, a load per lane that is on its way during
    // the prologue, and the mesh's first work item does the bookkeeping of
    // k_mesh_reduce.  A step of 8 blocks 21.6 -> 20.4 us, of 64 34.9 -> 33.1; on more
    // blocks the launch is below 3% of a step.
    unsigned long long before = 0;
    if (FIRST && a.prev && (tid & 63) < mp.nblocks) before = a.prev[mp.first_block + (tid & 63)];
    const size_t blk = size_t(b) * NV * CELLS;
    const double *Ub = a.Uin + blk;
    const int colp = j * 16 + i;
    const unsigned col8 = colp * 8;
    bool ok = true;

    // conserved values of this column's cell at z index kk in [-2, 18)
    auto zload = [&](int kk, double C[NV]) {
        const double *p = Ub + kk * 256;
        int st = CELLS;
        if (kk < 0 || kk >= BN) {
            const int nb = kk < 0 ? D.nb[4] : D.nb[5];
            if (nb >= 0) {
                p = a.Uin + size_t(nb) * NV * CELLS + (kk < 0 ? kk + BN : kk - BN) * 256;
            } else {
                p = a.halo + size_t(-nb - 1) * NV * SLAB + (kk < 0 ? kk + NG : kk - BN) * 256;
                st = SLAB;
            }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) C[v] = *uniform_at(p + v * st, col8);
    };
    // roles of the waves, rotated over the work items: 0 and 1 convert the x
    // and the y ghosts of a plane (64 each, one per lane), 2 and 3 take the
    // extra face task of the even and of the odd planes
    const int role = (__builtin_amdgcn_readfirstlane(tid >> 6) + item) & 3;
    const int gf = 2 * (role & 1) + ((tid >> 5) & 1), gr = tid & 31;   // ghost face and cell
    // its position in a plane's LDS copy, its source and the strides there
    const int glp = gf == 0 ? PMID + (gr >> 1) * PW + (gr & 1)
                            : (gf == 1 ? PMID + (gr >> 1) * PW + BN + NG + (gr & 1) : (gf == 2 ? gr : PTOP + gr));
    const double *gsrc;
    int gks, gst;
    {
        const int nb = gf == 0 ? D.nb[0] : (gf == 1 ? D.nb[1] : (gf == 2 ? D.nb[2] : D.nb[3]));
        if (nb < 0) {
            gsrc = a.halo + size_t(-nb - 1) * NV * SLAB + gr;
            gks = 32;
            gst = SLAB;
        } else if (gf < 2) {
            gsrc = a.XEin + xe_index(NV, nb, 0, gf == 0 ? 1 : 0, 0) + gr;
            gks = 2 * NV * BN * NG;
            gst = BN * NG;
        } else {
            gsrc = a.Uin + size_t(nb) * NV * CELLS + (gf == 2 ? 224 : 0) + gr;
            gks = 256;
            gst = CELLS;
        }
    }
    auto gload = [&](int k, double G[NV]) {
        const double *p = gsrc + size_t(k) * gks;
#pragma unroll
        for (int v = 0; v < NV; ++v) G[v] = p[v * gst];
    };
    auto put_ghost = [&](int buf, const double G[NV]) {
        double q[NV];
        ok &= phys_prim<RS>(G, gamma, gm1, q);
#pragma unroll
        for (int v = 0; v < NV; ++v) sP[buf][v][glp] = R(q[v]);
    };
    // LDS positions of this lane's own cell and of its y neighbours
    const int pown = PMID + j * PW + NG + i;
    auto yrow = [&](int r) { return r < 0 ? (r + NG) * BN + i : (r < BN ? PMID + r * PW + NG + i : PTOP + (r - BN) * BN + i); };
    const int pym2 = yrow(j - 2), pym1 = yrow(j - 1), pyp1 = yrow(j + 1);
    auto put_own = [&](int buf, const R w[NV]) {   // z-rotated primitives
        sP[buf][0][pown] = w[0]; sP[buf][1][pown] = w[2]; sP[buf][2][pown] = w[3];
        sP[buf][3][pown] = w[1]; sP[buf][4][pown] = w[4];
    };
    // flux from the four cells across a face
    auto flux4 = [&](const R c0[NV], const R c1[NV], const R c2[NV], const R c3[NV], R F[NV]) __attribute__((always_inline)) {
        R wL[NV], wR[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            R s0, s1;
            half_slopes<LIM>(c1[v] - c0[v], c2[v] - c1[v], c3[v] - c2[v], s0, s1);
            wL[v] = c1[v] + R(HALF<LIM>) * s0;
            wR[v] = c2[v] - R(HALF<LIM>) * s1;
        }
        riemann<RS, R>(wL, wR, gammaR, igm1R, F);
    };
    // store a boundary face's flux (natural variable order) into register slot `slot`
    auto keep = [&](int slot, int pos, R f0, R f1, R f2, R f3, R f4) {
        double *r = a.freg + size_t(slot) * NV * REG + pos;
        r[0] = double(f0); r[REG] = double(f1); r[2 * REG] = double(f2); r[3 * REG] = double(f3); r[4 * REG] = double(f4);
    };

    // output plane k's x-boundary columns from LDS to XE: 16 bytes per lane,
    // one run of 2560 bytes (stored by their own lanes they were five
    // stores of 64-byte pieces per wave; ten steps of 1856 blocks 5437 -> 5360
    // us, with FP32 fluxes 4977 -> 4885 us)
    const int xpos = (i < NG ? i : NV * BN * NG + i - (BN - NG)) + j * NG;
    auto export_x = [&](int k, int buf) {
        if (tid < NV * BN * NG)
            __builtin_nontemporal_store(reinterpret_cast<const double2v *>(sXE[buf])[tid],
                                        reinterpret_cast<double2v *>(a.XEout + xe_index(NV, b, k, 0, 0)) + tid);
    };

    // ---- prologue: cells k0-2 .. k0+1 of the column, face k0-1/2, plane k0 in
    // LDS.  Its expressions are the loop body's; the library is built with
    // per-expression contraction only, so each expression rounds the same way
    // wherever it is compiled and results do not depend on the slab shape.
    double C0[NV], C1[NV];
    R wk[NV], wk1[NV], wLz[NV], Flo[NV];
    {
        double Cm2[NV], Cm1[NV], G0[NV];
        zload(k0 - 2, Cm2);
        zload(k0 - 1, Cm1);
        zload(k0, C0);
        zload(k0 + 1, C1);
        if (role < 2) gload(k0, G0);
        R wm2[NV], wm1[NV], wL[NV], wR[NV];
        to_prim_z<RS>(Cm2, gamma, gm1, wm2, ok);
        to_prim_z<RS>(Cm1, gamma, gm1, wm1, ok);
        to_prim_z<RS>(C0, gamma, gm1, wk, ok);
        to_prim_z<RS>(C1, gamma, gm1, wk1, ok);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const R sm = half_slope<LIM>(wm1[v] - wm2[v], wk[v] - wm1[v]);
            wL[v] = wm1[v] + R(HALF<LIM>) * sm;
            const R s0 = half_slope<LIM>(wk[v] - wm1[v], wk1[v] - wk[v]);
            wR[v] = wk[v] - R(HALF<LIM>) * s0;
            wLz[v] = wk[v] + R(HALF<LIM>) * s0;
        }
        riemann<RS, R>(wL, wR, gammaR, igm1R, Flo);
        put_own(0, wk);
        if (role < 2) put_ghost(0, G0);
    }
    if (FIRST && a.prev) {
        const double dt = uniform(mp.cfl / __longlong_as_double(wave_max_u64(before)));
        dtdx = dt * inv_dx;
        if (b == mp.first_block && slab == 0 && tid == 0) {
            const double old = mp.dt;
            mp.t = mp.t + old;
            mp.last_dt = old;
            mp.dt = dt;
        }
    }
    if (k0 == 0 && D.freg[4] >= 0) keep(D.freg[4], colp, Flo[0], Flo[2], Flo[3], Flo[1], Flo[4]);
    __syncthreads();

    unsigned long long smax = 0;
    const int cf = D.cf_coarse;
    if (FIRST && slab == 0 && tid == 0) a.smax[b] = 0;   // the last stage takes the maximum

    // One plane of the march: plane k's x and y faces, z face k+1/2, plane
    // k+1 into LDS (the last plane writes one that is not used), barrier,
    // update of plane k.  The column's cell k+2 and the ghosts of plane k+1
    // are loaded at the top and first used after the x and y faces.
    auto plane = [&](const int k, const int cur) __attribute__((always_inline)) {
        const int nxt = cur ^ 1;
        double C2[NV], G[NV], Un[NV];
        zload(k + 2, C2);
        if (role < 2) gload(min(k + 1, k1 - 1), G);

        // (A) lower x and y face of the own cell, and the plane's upper faces
        R Fx[NV], Fy[NV];
        {
            R c0[NV], c1[NV], c3[NV];
            const R c2[NV] = {wk[0], wk[2], wk[3], wk[1], wk[4]};
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                c0[v] = sP[cur][v][pown - 2];
                c1[v] = sP[cur][v][pown - 1];
                c3[v] = sP[cur][v][pown + 1];
            }
            flux4(c0, c1, c2, c3, Fx);
#pragma unroll
            for (int v = 0; v < NV; ++v) sF[cur][v][FX + j * NFX + i] = Fx[v];
        }
        {
            constexpr int nv[NV] = {0, 2, 1, 3, 4};   // rotated to the y normal: (rho, vy, vx, vz, p)
            R c0[NV], c1[NV], c3[NV], F[NV];
            const R c2[NV] = {wk[0], wk[3], wk[2], wk[1], wk[4]};
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                c0[v] = sP[cur][nv[v]][pym2];
                c1[v] = sP[cur][nv[v]][pym1];
                c3[v] = sP[cur][nv[v]][pyp1];
            }
            flux4(c0, c1, c2, c3, F);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                Fy[nv[v]] = F[v];
                sF[cur][nv[v]][colp] = F[v];
            }
        }
        if (role == 2 + cur) {
            const int t = tid & 15;
            const bool yd = tid & 16;
            if (!(tid & 32)) {   // lanes 0..15: upper x face of row t; 16..31: upper y face of column t
                const int p0 = yd ? PMID + (BN - 2) * PW + NG + t : PMID + t * PW + BN;
                const int p1 = p0 + (yd ? PW : 1), p2 = yd ? PTOP + t : p0 + 2, p3 = yd ? PTOP + BN + t : p0 + 3;
                const int v1 = yd ? 2 : 1, v2 = yd ? 1 : 2;
                R c0[NV], c1[NV], c2[NV], c3[NV], F[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const R *q = sP[cur][v == 1 ? v1 : (v == 2 ? v2 : v)];
                    c0[v] = q[p0]; c1[v] = q[p1]; c2[v] = q[p2]; c3[v] = q[p3];
                }
                flux4(c0, c1, c2, c3, F);
                const int o = yd ? FYTOP + t : FX + t * NFX + BN;
#pragma unroll
                for (int v = 0; v < NV; ++v) sF[cur][v == 1 ? v1 : (v == 2 ? v2 : v)][o] = F[v];
                const int slot = yd ? D.freg[3] : D.freg[1];
                if (slot >= 0) keep(slot, k * 16 + t, F[0], yd ? F[2] : F[1], yd ? F[1] : F[2], F[3], F[4]);
            }
        }

        // U^n of plane k, for the update after the barrier
        const unsigned cell8 = col8 + k * 2048;
        if (!FIRST) {
#pragma unroll
            for (int v = 0; v < NV; ++v) Un[v] = __builtin_nontemporal_load(uniform_at(a.Un + blk + v * CELLS, cell8));
        }
        // (B) z face k+1/2, and plane k+1 into the other LDS buffer
        R Fhi[NV];
        {
            R wk2[NV], wR[NV], wLn[NV];
            to_prim_z<RS>(C2, gamma, gm1, wk2, ok);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const R s1 = half_slope<LIM>(wk1[v] - wk[v], wk2[v] - wk1[v]);
                wR[v] = wk1[v] - R(HALF<LIM>) * s1;
                wLn[v] = wk1[v] + R(HALF<LIM>) * s1;
            }
            riemann<RS, R>(wLz, wR, gammaR, igm1R, Fhi);
            put_own(nxt, wk1);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                wLz[v] = wLn[v];
                wk[v] = wk1[v];
                wk1[v] = wk2[v];
            }
        }
        if (role < 2) put_ghost(nxt, G);
        __syncthreads();

        // (C) divergence, stage combination, stores of plane k
        {
            const double fz[NV] = {double(Fhi[0]) - double(Flo[0]), double(Fhi[2]) - double(Flo[2]),
                                   double(Fhi[3]) - double(Flo[3]), double(Fhi[1]) - double(Flo[1]),
                                   double(Fhi[4]) - double(Flo[4])};
            double out[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const R xt = sF[cur][v][FX + j * NFX + i + 1];
                const double dfx = double(xt) - double(Fx[v]);
                const double dfy = double(sF[cur][v][colp + BN]) - double(Fy[v]);
                const double u1 = C0[v] - dtdx * ((dfx + dfy) + fz[v]);   // input + dt L
                if (KIND == 1) out[v] = u1;
                else if (KIND == 3) out[v] = 0.75 * Un[v] + 0.25 * u1;
                else if (KIND == 4) out[v] = (1.0 / 3.0) * Un[v] + (2.0 / 3.0) * u1;
                else out[v] = 0.5 * (Un[v] + u1);
                __builtin_nontemporal_store(out[v], uniform_at(a.Uout + blk + v * CELLS, cell8));
            }
            if (k > k0) export_x(k - 1, nxt);
            if (i < 2 || i >= BN - 2) {
#pragma unroll
                for (int v = 0; v < NV; ++v) sXE[cur][xpos + v * (BN * NG)] = out[v];
            }
            if (LAST) {
                const bool skip = ((cf & 1) && i == 0) || ((cf & 2) && i == BN - 1) || ((cf & 4) && j == 0) ||
                                  ((cf & 8) && j == BN - 1) || ((cf & 16) && k == 0) || ((cf & 32) && k == BN - 1);
                bool ok2;
                const double s = RS == 3 ? srhd_signal(out, gamma, inv_dx, ok2) : signal_rate(out, gamma, inv_dx, ok2);
                ok &= ok2;
                const unsigned long long sb = __double_as_longlong(s);
                if (!skip && sb > smax) smax = sb;
            }
        }
        // flux registers of the lower x / y boundary faces of plane k (the
        // upper ones are kept by the extra task)
        if (D.freg[0] >= 0 && i == 0) keep(D.freg[0], k * 16 + j, Fx[0], Fx[1], Fx[2], Fx[3], Fx[4]);
        if (D.freg[2] >= 0 && j == 0) keep(D.freg[2], k * 16 + i, Fy[0], Fy[1], Fy[2], Fy[3], Fy[4]);
#pragma unroll
        for (int v = 0; v < NV; ++v) {   // slide the conserved ring
            C0[v] = C1[v];
            C1[v] = C2[v];
            Flo[v] = Fhi[v];
        }
    };
    if (sizeof(R) == 8) {
        // two planes per trip (slabs have one plane or an even number): the
        // register ring then needs about half the moves
        for (int k = k0; k < k1; k += 2) {
            plane(k, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (k1 - k0 == 1) break;
            plane(k + 1, 1);
        }
    } else {
        // FP32 runs three waves per SIMD; the longer body would not fit
        for (int k = k0; k < k1; ++k) plane(k, (k - k0) & 1);
    }
    // flux register of the +z face (Flo holds the flux of face 15+1/2)
    if (k1 == BN && D.freg[5] >= 0) keep(D.freg[5], colp, Flo[0], Flo[2], Flo[3], Flo[1], Flo[4]);
    __syncthreads();
    export_x(k1 - 1, (k1 - 1 - k0) & 1);
    if (!ok) atomicOr(&mp.flags, 1);
    if (LAST) {
        unsigned long long *sMax = reinterpret_cast<unsigned long long *>(sP);   // no longer read
        smax = wave_max_u64(smax);
        if ((tid & 63) == 0) sMax[tid >> 6] = smax;
        __syncthreads();
        if (tid == 0) {
            unsigned long long m = sMax[0];
            for (int w = 1; w < 4; ++w) m = sMax[w] > m ? sMax[w] : m;
            atomicMax(&a.smax[b], m);
        }
    }
}

hipError_t launch_stage(const StageArgs &a, int riemann, int precision, hipStream_t s) {
    if (a.nblocks <= 0) return hipSuccess;
    if (a.kslab != 16 && a.kslab != 8 && a.kslab != 4 && a.kslab != 2 && a.kslab != 1) return hipErrorInvalidValue;
    if (a.stage < 1 || a.stage > 4 || riemann < 0 || riemann > 3 || a.limiter < 0 || a.limiter > 1)
        return hipErrorInvalidValue;
    const dim3 grid(xcd_grid(a.nblocks * (BN / a.kslab), a.xcd)), block(256);
#define AGILE_STAGE_KIND(RSV, LIMV, R)                                                        \
    do {                                                                                      \
        if (a.stage == 1) hipLaunchKernelGGL((k_stage<RSV, LIMV, 1, R>), grid, block, 0, s, a); \
        else if (a.stage == 2) hipLaunchKernelGGL((k_stage<RSV, LIMV, 2, R>), grid, block, 0, s, a); \
        else if (a.stage == 3) hipLaunchKernelGGL((k_stage<RSV, LIMV, 3, R>), grid, block, 0, s, a); \
        else hipLaunchKernelGGL((k_stage<RSV, LIMV, 4, R>), grid, block, 0, s, a);             \
    } while (0)
#define AGILE_STAGE_LIM(RSV, R)                                   \
    do {                                                          \
        if (a.limiter == 1) AGILE_STAGE_KIND(RSV, 1, R);          \
        else AGILE_STAGE_KIND(RSV, 0, R);                         \
    } while (0)
#define AGILE_STAGE_LAUNCH(R)                                     \
    do {                                                          \
        if (riemann == 0) AGILE_STAGE_LIM(0, R);                  \
        else if (riemann == 1) AGILE_STAGE_LIM(1, R);             \
        else if (riemann == 2) AGILE_STAGE_LIM(2, R);             \
        else AGILE_STAGE_LIM(3, R);                               \
    } while (0)
    if (precision == 0) AGILE_STAGE_LAUNCH(double);
    else AGILE_STAGE_LAUNCH(float);
#undef AGILE_STAGE_KIND
#undef AGILE_STAGE_LIM
#undef AGILE_STAGE_LAUNCH
    return hipGetLastError();
}

} // namespace agile
