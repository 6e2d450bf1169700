// mhd.hip -- gfx950 kernels of the ideal-MHD + GLM stage update (Sec. 2.3.3),
// nvar 9: (rho, m, e, B, psi).
//
// A stage is one launch of k_mhd_stage, 256 lanes per block (or per slab of 8, 4
// or 2 planes on small meshes) marching in z: PLM minmod on primitives, the GLM
// interface step and the HLL flux (mhd_hll) for the z faces from a per-lane
// register window and for the x and y faces from the plane in LDS, L = -((dFx
// + dFy) + dFz)/dx, the SSP-RK2 stage combination, flux registers and, in stage
// 2, the exact signal rate and GLM speed of the new state (cells about to be
// flux-corrected excepted).  The GLM source is split off exactly: psi decays
// by exp(-dt/2 c_h alpha/dx) before the two stages (k_glm_decay) and after
// them (applied to the output by the last stage, and by the flux correction to
// the cells it corrects, after their last correction).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "agile_internal.hpp"
#include "device_math.hpp"

namespace agile {

namespace {

constexpr int NV = 9;
// A plane's primitives in LDS, per variable: the two lower y ghost rows (16
// each), the 16 rows with their x ghosts (20 each), the two upper y ghost rows.
constexpr int PW = BN + 2 * NG;
constexpr int PMID = NG * BN, PTOP = PMID + BN * PW, PLANE = PTOP + NG * BN;   // 32, 352, 384
// Its face fluxes: the lower y ones in lane order, the upper y ones, the 17 x
// faces of every row.
constexpr int FYTOP = BN * BN, FX = FYTOP + BN, NFX = BN + 1, NFACE = FX + BN * NFX;   // 256, 272, 17, 544

} // namespace

// One work item (block, slab of kslab planes) per workgroup of 256 lanes,
// marching in z (lane (i, j) owns the z-column (i, j)); per plane k:
//   (1) the lower x and the lower y face of the lane's own cell from the
//       plane's primitives in LDS, the 16 + 16 upper faces of the plane as an
//       extra task of one wave, the z face k+1/2 from the column's primitives
//       (cells k, k+1 and the next one, converted as it arrives; the left
//       state of the face carried from the previous plane); x and y fluxes go
//       to LDS;
//   (2) after a barrier: L = -((dFx + dFy) + dFz)/dx, the stage combination
//       with the cell's input (kept in registers from its load two planes
//       earlier) and, in stage 2, U^n; stage 2: the signal rate and GLM speed
//       of the new state; plane k+1's primitives into LDS; a barrier.
// Waves 0 and 1 (rotated over the items) convert the plane's 128 ghosts, waves
// 2 and 3 take the extra task in turn.  Each face flux is computed once; the
// state is read once per stage (x ghosts from the neighbour's x-boundary
// copy), and nothing but the output with the x-boundary copy of its boundary
// columns, the flux registers and the signal maxima is written.
// Two waves per SIMD (256 registers; three, with FP32 fluxes, spill 80 of 168
// and are slower: 262 instead of 145 us for a first stage of 576 blocks).  Bound
// by VALU work and by the waits that two waves cannot cover.  A reload from
// scratch waits for every global load issued before it, so the FP64 stages are
// written to hold as little as they can: addresses of ghosts and rare branches
// formed where they are used (opaque), cells converted twice.  18 944 blocks,
// stages 1 / 2: FP64 5593 / 6515 us with runtime-indexed face tasks and the
// longer flux, 5041 / 5878 with fixed faces and the shorter flux but 50
// spilled registers, 4015 / 4910 with 6 and 8 (now 0 and 8; the form of the flux
// that keeps slow flow's digits takes 3% more VALU instructions, 1.3% of a step);
// FP32 flux, 576 blocks: 164 / 226 -> 139 / 168.
template <int STAGE, typename R>
__global__ __launch_bounds__(256, 2) void k_mhd_stage(SweepArgs a) {
    __shared__ R sP[NV][PLANE];
    __shared__ R sF[NV][NFACE];
    __shared__ __align__(16) double sXE[2 * NV * BN * NG];   // x-boundary columns of a plane's output, as in XE
    const int nslab = BN / a.kslab;
    const int item = blockIdx.x;
    if (item >= a.nblocks * nslab) return;
    const int bi = item / nslab, slab = item - bi * nslab;
    const int b = a.list ? a.list[bi] : bi;
    const int k0 = slab * a.kslab, k1 = k0 + a.kslab;
    const int tid = threadIdx.x;
    const int i = tid & 15, j = tid >> 4;
    const BlockDesc D = a.desc[b];
    MeshParams &mp = a.mp[D.mesh];
    const double gamma = mp.gamma, gm1 = gamma - 1.0;
    const double inv_dx = mp.inv_dx1 * double(1 << (D.level - 1));
    const double dtdx = mp.dt * inv_dx;
    const double ch = __longlong_as_double(mp.cmax);
    // the last stage also applies the second half of the GLM decay of psi
    // (the factor of k_glm_decay for h = dt/2, the same expression) to every
    // cell that no flux correction follows; k_reflux applies it to the
    // corrected cells after their last correction
    const double hdec = 0.5 * mp.dt;
    const double fdec = STAGE == 2 ? exp(-hdec * ch * mp.glm_alpha * inv_dx) : 1.0;
    const R gammaR = R(gamma), igm1R = R(1.0 / gm1), chR = R(ch), inv2chR = R(0.5 / ch);
    const size_t blk = size_t(b) * NV * CELLS;
    const double *Ub = a.Uin + blk;
    const int colp = j * 16 + i;
    const unsigned col8 = colp * 8;
    bool ok = true;
    if (STAGE == 1 && slab == 0 && tid == 0) {
        a.smax[b] = 0;
        a.cmax[b] = 0;
    }

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
    // rotated primitives for the z normal: (rho, vz, vx, vy, p, Bz, Bx, By, psi)
    auto prim_z = [&](const double C[NV], R w[NV]) {
        double q[NV];
        ok &= mhd_cons2prim(C, gm1, q);
        w[0] = R(q[0]); w[1] = R(q[3]); w[2] = R(q[1]); w[3] = R(q[2]); w[4] = R(q[4]);
        w[5] = R(q[7]); w[6] = R(q[5]); w[7] = R(q[6]); w[8] = R(q[8]);
    };
    // roles of the waves, rotated over the work items: 0 and 1 convert the x
    // and the y ghosts of a plane (64 each, one per lane), 2 and 3 take the
    // extra face task of the even and of the odd planes
    const int role = (__builtin_amdgcn_readfirstlane(tid >> 6) + item) & 3;
    const int gf = 2 * (role & 1) + ((tid >> 5) & 1), gr = tid & 31;   // ghost face and cell
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
        const int st = opaque(gst);
#pragma unroll
        for (int v = 0; v < NV; ++v) G[v] = p[v * st];
    };
    auto put_ghost = [&](const double G[NV]) {
        double q[NV];
        ok &= mhd_cons2prim(G, gm1, q);
#pragma unroll
        for (int v = 0; v < NV; ++v) sP[v][glp] = R(q[v]);
    };
    // LDS positions of this lane's own cell and of its y neighbours
    const int pown = PMID + j * PW + NG + i;
    auto yrow = [&](int r) { return r < 0 ? (r + NG) * BN + i : (r < BN ? PMID + r * PW + NG + i : PTOP + (r - BN) * BN + i); };
    const int pym2 = yrow(j - 2), pym1 = yrow(j - 1), pyp1 = yrow(j + 1);
    // natural variable of rotated variable v for the z and the y normal
    // (cyclic: n, n+1, n+2)
    constexpr int zv[NV] = {0, 3, 1, 2, 4, 7, 5, 6, 8};
    constexpr int yv[NV] = {0, 2, 3, 1, 4, 6, 7, 5, 8};
    auto put_own = [&](const R w[NV]) {   // z-rotated primitives
#pragma unroll
        for (int v = 0; v < NV; ++v) sP[zv[v]][pown] = w[v];
    };
    // limited states (natural variable order) from the cells at LDS positions
    // p0 .. p3 across a face
    auto states = [&](int p0, int p1, int p2, int p3, R wL[NV], R wR[NV]) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const R c0 = sP[v][p0], c1 = sP[v][p1], c2 = sP[v][p2], c3 = sP[v][p3];
            R s0, s1;
            half_slopes<0>(c1 - c0, c2 - c1, c3 - c2, s0, s1);
            wL[v] = c1 + R(0.5) * s0;
            wR[v] = c2 - R(0.5) * s1;
        }
    };
    // store a boundary face's flux, rotated by perm, into register slot `slot`
    auto keep = [&](int slot, int pos, const R F[NV], const int (&perm)[NV]) {
        double *r = a.freg + size_t(slot) * NV * REG + pos;
#pragma unroll
        for (int v = 0; v < NV; ++v) r[perm[v] * REG] = double(F[v]);
    };
    const int xpos = (i < NG ? i : NV * BN * NG + i - (BN - NG)) + j * NG;
    auto export_x = [&](int k) {   // sXE to XE, 16 bytes per lane
        const double *out = a.XEout + xe_index(NV, b, k, 0, 0);
        const int q = opaque(tid);
        __builtin_nontemporal_store(reinterpret_cast<const double2v *>(sXE)[q], uniform2_at(out, q * 16));
        if (q < NV * BN * NG - 256)
            __builtin_nontemporal_store(reinterpret_cast<const double2v *>(sXE)[q + 256], uniform2_at(out, (q + 256) * 16));
    };

    // prologue: cells k0-2 .. k0+1 of the column, face k0-1/2, plane k0 in LDS
    double C0[NV], C1[NV];
    R wLz[NV], Flo[NV];
    {
        double Cm2[NV], Cm1[NV], G0[NV];
        zload(k0 - 2, Cm2);
        zload(k0 - 1, Cm1);
        zload(k0, C0);
        zload(k0 + 1, C1);
        if (role < 2) gload(k0, G0);
        R wm2[NV], wm1[NV], wk[NV], wk1[NV], wL[NV], wR[NV];
        prim_z(Cm2, wm2);
        prim_z(Cm1, wm1);
        prim_z(C0, wk);
        prim_z(C1, wk1);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const R sm = half_slope<0>(wm1[v] - wm2[v], wk[v] - wm1[v]);
            wL[v] = wm1[v] + R(0.5) * sm;
            const R s0 = half_slope<0>(wk[v] - wm1[v], wk1[v] - wk[v]);
            wR[v] = wk[v] - R(0.5) * s0;
            wLz[v] = wk[v] + R(0.5) * s0;
        }
        mhd_hll(wL, wR, gammaR, igm1R, chR, inv2chR, Flo);
        put_own(wk);
        if (role < 2) put_ghost(G0);
    }
    if (k0 == 0 && D.freg[4] >= 0) keep(D.freg[4], colp, Flo, zv);
    __syncthreads();

    unsigned long long sm = 0, cm = 0;
    const int cf = D.cf_coarse, fxup = D.freg[1], fyup = D.freg[3];
    auto plane = [&](const int k) __attribute__((always_inline)) {
        double C2[NV], G[NV], Un[NV];
        const unsigned cell8 = col8 + k * 2048;
        auto load_ghost = [&]() __attribute__((always_inline)) {
            if (role < 2) gload(min(k + 1, k1 - 1), G);
        };
        auto lower_y = [&]() __attribute__((always_inline)) {
            R wL[NV], wR[NV], L[NV], Q[NV], F[NV];
            states(pym2, pym1, pown, pyp1, wL, wR);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                L[v] = wL[yv[v]];
                Q[v] = wR[yv[v]];
            }
            mhd_hll(L, Q, gammaR, igm1R, chR, inv2chR, F);
#pragma unroll
            for (int v = 0; v < NV; ++v) sF[yv[v]][colp] = F[v];
        };
        auto lower_x = [&]() __attribute__((always_inline)) {
            R wL[NV], wR[NV], F[NV];
            states(pown - 2, pown - 1, pown, pown + 1, wL, wR);
            mhd_hll(wL, wR, gammaR, igm1R, chR, inv2chR, F);
#pragma unroll
            for (int v = 0; v < NV; ++v) sF[v][FX + j * NFX + i] = F[v];
        };
        auto upper = [&]() __attribute__((always_inline)) {
            if (role != 2 + (k & 1)) return;
            const int e = opaque(tid & 63), t = e & 15;
            if (e & 32) return;   // lanes 0..15: upper x face of row t; 16..31: upper y face of column t
            const bool yd = e & 16;
            const int e0 = yd ? PMID + (BN - 2) * PW + NG + t : PMID + t * PW + BN;
            const int e1 = e0 + (yd ? PW : 1), e2 = yd ? PTOP + t : e0 + 2, e3 = yd ? e2 + BN : e0 + 3;
            const int eout = yd ? FYTOP + t : FX + t * NFX + BN;
            R wL[NV], wR[NV], L[NV], Q[NV], F[NV];
            states(e0, e1, e2, e3, wL, wR);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                L[v] = yd ? wL[yv[v]] : wL[v];
                Q[v] = yd ? wR[yv[v]] : wR[v];
            }
            mhd_hll(L, Q, gammaR, igm1R, chR, inv2chR, F);
#pragma unroll
            for (int v = 0; v < NV; ++v) sF[v][eout] = yd ? F[zv[v]] : F[v];   // the z rotation undoes the y rotation
            if (fxup >= 0 || fyup >= 0) {
                const int slot = opaque(yd ? fyup : fxup);
                double *r = a.freg + size_t(slot < 0 ? 0 : slot) * NV * REG + k * 16 + t;
                if (slot >= 0) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) r[v * REG] = double(yd ? F[zv[v]] : F[v]);
                }
            }
        };

        // (1) lower y and x face of the own cell, the upper faces, z face k+1/2
        // (FP64: the loads after the first face and the upper faces last, where
        // the fewest registers are held)
        if constexpr (sizeof(R) == 8) {
            lower_y();
            zload(k + 2, C2);
            load_ghost();
            lower_x();
            upper();
        } else {
            zload(k + 2, C2);
            lower_y();
            upper();
            load_ghost();
            lower_x();
        }
        // U^n of plane k, for the update after the barrier
        if (STAGE == 2) {
#pragma unroll
            for (int v = 0; v < NV; ++v) Un[v] = __builtin_nontemporal_load(uniform_at(a.Un + blk + v * CELLS, cell8));
        }
        R Fhi[NV];
        {
            R wk1[NV], wk2[NV], wR[NV], wLn[NV];
            prim_z(C1, wk1);   // again: kept from the last plane it would take 18 registers
            prim_z(C2, wk2);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const R s1 = half_slope<0>(wk1[v] - sP[zv[v]][pown], wk2[v] - wk1[v]);
                wR[v] = wk1[v] - R(0.5) * s1;
                wLn[v] = wk1[v] + R(0.5) * s1;
            }
            mhd_hll(wLz, wR, gammaR, igm1R, chR, inv2chR, Fhi);
            __syncthreads();   // plane k's primitives read, its fluxes complete
            put_own(wk1);
            if (role < 2) put_ghost(G);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                wLz[v] = wLn[v];
            }
        }

        // (2) update of cell (i, j, k)
        {
            // cells on a face where a flux correction follows (coarse side of
            // a level jump): left out of the signal maxima and the decay here
            const bool skip = STAGE == 2 &&
                              (((cf & 1) && i == 0) || ((cf & 2) && i == BN - 1) || ((cf & 4) && j == 0) ||
                               ((cf & 8) && j == BN - 1) || ((cf & 16) && k == 0) || ((cf & 32) && k == BN - 1));
            double out[NV];
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const int v = zv[u];
                const double fz = double(Fhi[u]) - double(Flo[u]);
                const double dfx = double(sF[v][FX + j * NFX + i + 1]) - double(sF[v][FX + j * NFX + i]);
                const double dfy = double(sF[v][colp + BN]) - double(sF[v][colp]);
                const double u1 = C0[v] - dtdx * ((dfx + dfy) + fz);   // input + dt L
                if (STAGE == 1) out[v] = u1;
                else out[v] = 0.5 * (Un[v] + u1);
                if (STAGE == 2 && v == 8 && !skip) out[v] = out[v] * fdec;
                __builtin_nontemporal_store(out[v], uniform_at(a.Uout + blk + v * CELLS, cell8));
            }
            if (i < NG || i >= BN - NG) {
#pragma unroll
                for (int v = 0; v < NV; ++v) sXE[xpos + v * (BN * NG)] = out[v];
            }
            if (D.freg[0] >= 0 && i == 0) {   // flux registers of the lower x / y boundary faces
                double *r = a.freg + size_t(D.freg[0]) * NV * REG + k * 16 + opaque(j);
#pragma unroll
                for (int v = 0; v < NV; ++v) r[v * REG] = double(sF[v][FX + j * NFX]);
            }
            if (D.freg[2] >= 0 && j == 0) {
                double *r = a.freg + size_t(D.freg[2]) * NV * REG + k * 16 + opaque(i);
#pragma unroll
                for (int v = 0; v < NV; ++v) r[v * REG] = double(sF[v][i]);
            }
            if (STAGE == 2) {
                bool ok2;
                double c;
                const double sg = mhd_signal(out, gamma, inv_dx, c, ok2);
                ok &= ok2;
                if (!skip) {
                    const unsigned long long sb = __double_as_longlong(sg), cb = __double_as_longlong(c);
                    sm = sb > sm ? sb : sm;
                    cm = cb > cm ? cb : cm;
                }
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                C0[v] = C1[v];
                C1[v] = C2[v];
                Flo[v] = Fhi[v];
            }
        }
        __syncthreads();   // plane k+1 complete; plane k's fluxes read
        export_x(k);
    };
    // slabs have an even number of planes, starting at an even plane
    for (int k = k0; k < k1; k += 2) {
        __builtin_assume((k & 1) == 0);
        plane(k);
        __builtin_amdgcn_sched_barrier(0);
        plane(k + 1);
    }
    if (k1 == BN && D.freg[5] >= 0) keep(D.freg[5], colp, Flo, zv);   // z flux register of face 15+1/2
    if (!ok) atomicOr(&mp.flags, 1);
    if (STAGE == 2) {
        unsigned long long *sMax = reinterpret_cast<unsigned long long *>(sP);   // no longer read
        sm = wave_max_u64(sm);
        cm = wave_max_u64(cm);
        if ((tid & 63) == 0) {
            sMax[tid >> 6] = sm;
            sMax[4 + (tid >> 6)] = cm;
        }
        __syncthreads();
        if (tid == 0) {
            unsigned long long r = sMax[0], rc = sMax[4];
            for (int w = 1; w < 4; ++w) {
                r = sMax[w] > r ? sMax[w] : r;
                rc = sMax[4 + w] > rc ? sMax[4 + w] : rc;
            }
            atomicMax(&a.smax[b], r);
            atomicMax(&a.cmax[b], rc);
        }
    }
}

// psi <- psi exp(-h c_h alpha / dx) for the listed blocks (exact solution of
// the GLM damping term over a time h), and in the x-boundary copy XE.  One
// workgroup per block: the factor once, then the block's 4096 psi values as
// 16-byte pairs, 4 KB per round of the 256 lanes, with streaming hints (each
// value is read and written once); the pairs (0,1) and (14,15) of a row also
// go to XE.
typedef double v2d __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(256) void k_glm_decay(const BlockDesc *desc, MeshParams *mp, double *U, double *XE,
                                                   const int *list, int nblocks, double hfrac) {
    const int bi = blockIdx.x;
    if (bi >= nblocks) return;
    const int b = list ? list[bi] : bi;
    const BlockDesc D = desc[b];
    const MeshParams &P = mp[D.mesh];
    const double inv_dx = P.inv_dx1 * double(1 << (D.level - 1));
    const double h = hfrac * P.dt;
    const double f = exp(-h * __longlong_as_double(P.cmax) * P.glm_alpha * inv_dx);
    v2d *psi = reinterpret_cast<v2d *>(U + (size_t(b) * NV + 8) * CELLS);
#pragma unroll
    for (int r = 0; r < CELLS / 512; ++r) {
        const int q = threadIdx.x + 256 * r;   // cells 2q, 2q + 1: pair q & 7 of row q >> 3 (row = k * 16 + j)
        v2d x = __builtin_nontemporal_load(psi + q);
        x.x *= f;
        x.y *= f;
        __builtin_nontemporal_store(x, psi + q);
        const int ip = q & 7;
        if (XE && (ip == 0 || ip == 7)) *reinterpret_cast<v2d *>(XE + xe_index(NV, b, q >> 7, ip == 7, 8) + ((q >> 3) & 15) * 2) = x;
    }
}

hipError_t launch_mhd_stage(const SweepArgs &a, int stage, int precision, hipStream_t s) {
    if (a.nblocks <= 0) return hipSuccess;
    if (a.kslab != 16 && a.kslab != 8 && a.kslab != 4 && a.kslab != 2) return hipErrorInvalidValue;
    const dim3 grid(a.nblocks * (BN / a.kslab)), block(256);
    if (precision == 0) {
        if (stage == 1) hipLaunchKernelGGL((k_mhd_stage<1, double>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_mhd_stage<2, double>), grid, block, 0, s, a);
    } else {
        if (stage == 1) hipLaunchKernelGGL((k_mhd_stage<1, float>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_mhd_stage<2, float>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_glm_decay(const BlockDesc *desc, MeshParams *mp, double *U, double *XE, const int *list,
                            int nblocks, double hfrac, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_glm_decay, dim3(nblocks), dim3(256), 0, s, desc, mp, U, XE, list, nblocks, hfrac);
    return hipGetLastError();
}

} // namespace agile
