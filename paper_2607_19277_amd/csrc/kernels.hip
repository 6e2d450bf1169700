// kernels.hip -- gfx950 kernels around the stage update: ghost fill at level
// jumps (restriction, prolongation; SRHD prolongs primitives), coarse-fine
// flux correction, signal-speed scan and reduction for dt, block
// permutation, ghost readout, and the regrid's Loehner estimate and data
// transfer.  Mostly one workgroup per task or block.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "agile_internal.hpp"
#include "device_math.hpp"

namespace agile {
// ---------------------------------------------------------------------------
// ghost-slab cell index (c in [0, 512)) -> (g, a, b) and back

// d = 0: [k][j][g], d = 1: [k][g][i], d = 2: [g][j][i]; written as selects
// (branches that each assign the three outputs are merged by the compiler
// into a small scratch array)
__device__ __forceinline__ void slab_coords(int d, int c, int &g, int &ta, int &tb) {
    g = d == 0 ? (c & 1) : (d == 1 ? ((c >> 4) & 1) : (c >> 8));
    ta = d == 0 ? ((c >> 1) & 15) : (c & 15);
    tb = d == 2 ? ((c >> 4) & 15) : (c >> 5);
}

// Value of variable v of block C at local cell (x, y, z), where at most one
// coordinate may lie one or two cells outside [0, 16): then it is a face ghost
// of C (same-level neighbour interior or C's ghost slab).
__device__ __forceinline__ double block_value(const BlockDesc *desc, const double *U, const double *halo, int NV,
                                              int C, int v, int x, int y, int z) {
    int o = -1;
    if (x < 0 || x >= BN) o = 0;
    else if (y < 0 || y >= BN) o = 1;
    else if (z < 0 || z >= BN) o = 2;
    if (o < 0) return U[(size_t(C) * NV + v) * CELLS + (z * 16 + y) * 16 + x];
    int c[3] = {x, y, z};
    const int side = c[o] >= BN;
    const int nb = desc[C].nb[2 * o + side];
    if (nb >= 0) {
        c[o] = side ? c[o] - BN : c[o] + BN;
        return U[(size_t(nb) * NV + v) * CELLS + (c[2] * 16 + c[1]) * 16 + c[0]];
    }
    const int g = side ? c[o] - BN : c[o] + NG;
    const int ta = o == 0 ? c[1] : c[0];
    const int tb = o == 2 ? c[1] : c[2];
    return halo[(size_t(-nb - 1) * NV + v) * SLAB + slab_index(o, g, ta, tb)];
}

// Restriction: coarse ghost = mean of its 8 fine children, summed pairwise
// ((c000+c100)+(c010+c110)) + ((c001+c101)+(c011+c111)) with x fastest.
// One lane per coarse ghost cell c of the slab; all 8 NV children of the cell
// are loaded before its NV sums are stored.
template <int NV>
__device__ __forceinline__ void restrict_cell(const RestrictTask *__restrict__ t, int c,
                                              const double *__restrict__ U, double *__restrict__ halo) {
    const int d = t->face >> 1, side = t->face & 1;
    int g, ta, tb;
    slab_coords(d, c, g, ta, tb);
    const int q = (ta >> 3) + 2 * (tb >> 3);
    const int F = t->fine[q];   // read through the pointer: a local copy indexed by q would live in scratch
    // first fine child along the normal (under coarse ghost layer g) and the
    // two tangential axes a (x, or y for d = 0) and b (z, or y for d = 2);
    // selects rather than an indexed array, which would live in scratch
    const int bn = side ? 2 * g : 12 + 2 * g, ba = 2 * (ta & 7), bb = 2 * (tb & 7);
    const int bx = d == 0 ? bn : ba;
    const int by = d == 1 ? bn : (d == 0 ? ba : bb);
    const int bz = d == 2 ? bn : bb;
    const double2v *u = reinterpret_cast<const double2v *>(U + size_t(F) * NV * CELLS + (bz * 16 + by) * 16 + bx);
    double2v ch[NV][4];   // pairs along x (bx is even)
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int k = 0; k < 4; ++k) ch[v][k] = u[v * (CELLS / 2) + (k >> 1) * 128 + (k & 1) * 8];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const double s = ((ch[v][0].x + ch[v][0].y) + (ch[v][1].x + ch[v][1].y)) +
                         ((ch[v][2].x + ch[v][2].y) + (ch[v][3].x + ch[v][3].y));
        halo[(size_t(t->slot) * NV + v) * SLAB + c] = s * 0.125;
    }
}

// four workgroups of 128 lanes per restriction task
template <int NV>
__global__ __launch_bounds__(128) void k_restrict(const RestrictTask *__restrict__ tasks,
                                                  const double *__restrict__ U, double *__restrict__ halo) {
    restrict_cell<NV>(tasks + (blockIdx.x >> 2), threadIdx.x + 128 * (blockIdx.x & 3), U, halo);
}

// Prolongation: fine ghost = parent + sum over x, y, z (in that order) of
// +/- (1/4) minmod(parent - left, right - parent) of the parent's axis
// neighbours.  One workgroup per task: wave v takes variable v, lane p the
// coarse parent p of the face's 8 x 8 parents; the three limited slopes of a
// parent are formed once and give its 8 fine ghost cells (2 layers x 2 x 2).
// Bound by the chain task -> neighbours -> cells: the coarse block's neighbours
// are read once for the wave, and a lane at the block's edge selects the address
// beyond it, so that all seven cells are in flight together (1152 tasks 16.4
// -> 11.2 us).  The cells of an x face come from the x-boundary copy XE (the
// same values, in whole runs), if there is one.
template <int NV>
__global__ __launch_bounds__(64 * NV) void k_prolong(const ProlongTask *__restrict__ tasks,
                                                     const BlockDesc *__restrict__ desc,
                                                     const double *__restrict__ U, const double *__restrict__ XE,
                                                     double *__restrict__ halo) {
    const ProlongTask t = tasks[blockIdx.x];
    const int d = t.face >> 1, side = t.face & 1;
    const int da = d == 0 ? 1 : 0;
    const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), p = threadIdx.x & 63;
    const int pa = p & 7, pb = p >> 3;
    const int lay = side ? 0 : BN - 1;      // coarse layer next to the face
    const int c[3] = {d == 0 ? lay : t.ta + pa, d == 1 ? lay : (da == 1 ? t.ta + pa : t.tb + pb),
                      d == 2 ? lay : t.tb + pb};
    const BlockDesc *K = desc + t.coarse;
    const bool inx = XE && d == 0;          // then every cell read lies in a boundary column
    auto cell = [&](int block, int x, int y, int z) -> const double * {
        const int xs = x >= BN / 2;
        return inx ? XE + xe_index(NV, block, z, xs, v) + y * 2 + (x - (xs ? BN - NG : 0))
                   : U + (size_t(block) * NV + v) * CELLS + (z * 16 + y) * 16 + x;
    };
    // the parent's neighbour one cell up (s = 1) or down (-1) axis e
    auto next = [&](int e, int s) -> const double * {
        const int x = c[0] + (e == 0 ? s : 0), y = c[1] + (e == 1 ? s : 0), z = c[2] + (e == 2 ? s : 0);
        const bool out = s > 0 ? c[e] == BN - 1 : c[e] == 0;
        const int nb = K->nb[2 * e + (s > 0)];
        const double *o = nb >= 0
                              ? cell(nb, x & (BN - 1), y & (BN - 1), z & (BN - 1))
                              : halo + (size_t(-nb - 1) * NV + v) * SLAB +
                                    slab_index(e, s > 0 ? 0 : NG - 1, e == 0 ? c[1] : c[0], e == 2 ? c[1] : c[2]);
        return out ? o : cell(t.coarse, x & (BN - 1), y & (BN - 1), z & (BN - 1));
    };
    const double vc = *cell(t.coarse, c[0], c[1], c[2]);
    double vm[3], vp[3], q[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        vm[e] = *next(e, -1);
        vp[e] = *next(e, 1);
    }
#pragma unroll
    for (int e = 0; e < 3; ++e) q[e] = 0.25 * minmod(vc - vm[e], vp[e] - vc);
    double *out = halo + (size_t(t.slot) * NV + v) * SLAB;
    auto child = [&](int g, int ca, int cb) {   // fine ghost layer g: the low child for g = 0
        const int sx = d == 0 ? g : ca, sy = d == 1 ? g : (da == 1 ? ca : cb), sz = d == 2 ? g : cb;
        double val = sx ? vc + q[0] : vc - q[0];
        val = sy ? val + q[1] : val - q[1];
        return sz ? val + q[2] : val - q[2];
    };
    // pairs along the slab's fastest axis
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int e = k & 1, cb = k >> 1;
        double2v r;
        int o;
        if (d == 0) {   // layers 0 and 1
            r.x = child(0, e, cb);
            r.y = child(1, e, cb);
            o = slab_index(0, 0, 2 * pa + e, 2 * pb + cb);
        } else {
            r.x = child(e, 0, cb);
            r.y = child(e, 1, cb);
            o = slab_index(d, e, 2 * pa, 2 * pb + cb);
        }
        *reinterpret_cast<double2v *>(out + o) = r;
    }
}

// ---------------------------------------------------------------------------
// SRHD prolongation (Sec. 2.3.4): the same stencil on the primitives (rho,
// Gamma v, p) of the parent and its axis neighbours, each from the IEEE
// con2prim, and each child's primitives converted back with IEEE arithmetic
// without contraction -- the host's operations, so the ghosts and the regrid
// transfer keep the same bits.  Limited interpolation of the conserved
// variables could give |m| > tau + D next to a strong relativistic shock;
// minmod-limited primitives stay between neighbouring values.  A stencil cell
// without a physical state makes its children NaN (the next step reports
// it).

// (D, m, tau) from (rho, u, p): D = Gamma rho, m = Gamma rho h u,
// tau = Gamma^2 rho h - p - D, Gamma = sqrt(1 + u^2), rho h = rho + g/(g-1) p
__device__ __forceinline__ void srhd_prim2con_ieee(const double w[5], double g, double U[5]) {
#pragma clang fp contract(off)
    const double uu = (w[1] * w[1] + w[2] * w[2]) + w[3] * w[3];
    const double G = __builtin_sqrt(1.0 + uu);
    const double rhoh = w[0] + (g / (g - 1.0)) * w[4];
    U[0] = G * w[0];
    U[1] = (G * rhoh) * w[1];
    U[2] = (G * rhoh) * w[2];
    U[3] = (G * rhoh) * w[3];
    U[4] = ((G * G) * rhoh - w[4]) - U[0];
}

// primitives of cell (x, y, z) of block C (its ghosts included)
__device__ __forceinline__ bool srhd_cell_prims(const BlockDesc *desc, const double *U, const double *halo, int C,
                                                int x, int y, int z, double g, double w[5]) {
    double u[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) u[v] = block_value(desc, U, halo, 5, C, v, x, y, z);
    return srhd_con2prim(u, g, w);
}

// the parent cell's primitives wc and the quarter slopes q[axis][var]
__device__ __forceinline__ bool srhd_parent(const BlockDesc *desc, const double *U, const double *halo, int C,
                                            int x, int y, int z, double g, double wc[5], double q[3][5]) {
    bool ok = srhd_cell_prims(desc, U, halo, C, x, y, z, g, wc);
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        double wm[5], wp[5];
        ok &= srhd_cell_prims(desc, U, halo, C, x - (e == 0), y - (e == 1), z - (e == 2), g, wm);
        ok &= srhd_cell_prims(desc, U, halo, C, x + (e == 0), y + (e == 1), z + (e == 2), g, wp);
#pragma unroll
        for (int v = 0; v < 5; ++v) q[e][v] = 0.25 * minmod(wc[v] - wm[v], wp[v] - wc[v]);
    }
    return ok;
}

// conserved state of the child on the (sx, sy, sz) side (1 = upper) of its
// parent: parent primitives +/- quarter slope per axis, in x, y, z order
__device__ __forceinline__ void srhd_child(const double wc[5], const double q[3][5], int sx, int sy, int sz, double g,
                                           bool ok, double out[5]) {
    double w[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        double val = wc[v];
        val = sx ? val + q[0][v] : val - q[0][v];
        val = sy ? val + q[1][v] : val - q[1][v];
        val = sz ? val + q[2][v] : val - q[2][v];
        w[v] = val;
    }
    srhd_prim2con_ieee(w, g, out);
    if (!ok) {
#pragma unroll
        for (int v = 0; v < 5; ++v) out[v] = __builtin_nan("");
    }
}

// one 64-lane workgroup per prolongation task, lane p = coarse parent p
__global__ __launch_bounds__(64) void k_prolong_srhd(const ProlongTask *__restrict__ tasks,
                                                     const BlockDesc *__restrict__ desc,
                                                     const MeshParams *__restrict__ mp, const double *__restrict__ U,
                                                     double *__restrict__ halo) {
    const ProlongTask *t = tasks + blockIdx.x;
    const int d = t->face >> 1, side = t->face & 1;
    const int p = threadIdx.x, pa = p & 7, pb = p >> 3;
    const int da = d == 0 ? 1 : 0;
    const int lay = side ? 0 : BN - 1;      // coarse layer next to the face
    const int x = d == 0 ? lay : t->ta + pa;
    const int y = d == 1 ? lay : (da == 1 ? t->ta + pa : t->tb + pb);
    const int z = d == 2 ? lay : t->tb + pb;
    const double g = mp[desc[t->coarse].mesh].gamma;
    double wc[5], q[3][5];
    const bool ok = srhd_parent(desc, U, halo, t->coarse, x, y, z, g, wc, q);
    double *out = halo + size_t(t->slot) * 5 * SLAB;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int gl = k & 1, ca = (k >> 1) & 1, cb = k >> 2;
        // side of the child along each axis: the ghost layer along d, the
        // in-face offsets along the other two
        const int sx = d == 0 ? gl : ca;
        const int sy = d == 1 ? gl : (da == 1 ? ca : cb);
        const int sz = d == 2 ? gl : cb;
        double c[5];
        srhd_child(wc, q, sx, sy, sz, g, ok, c);
        const int o = slab_index(d, gl, 2 * pa + ca, 2 * pb + cb);
#pragma unroll
        for (int v = 0; v < 5; ++v) out[v * SLAB + o] = c[v];
    }
}

// Coarse-fine flux correction of one coarse block: for each coarse-fine face
// the coarse flux F_c is replaced by the mean of the 4 fine fluxes covering it,
// F_f = ((f00+f10)+(f01+f11))/4, i.e. U += w dt/dx (+/-)(F_c - F_f).  Faces
// are taken in order (a cell on two such faces is corrected twice, in order);
// in the last stage of a step the signal rate of every corrected cell is
// taken from its final value (the lane of its last face) and joins the block
// maximum, which the stage left out for these cells.
template <int NV>
__device__ __forceinline__ void reflux_block(const RefluxTask *__restrict__ t, MeshParams *mp, double *__restrict__ U,
                                             double *__restrict__ XE, const double *__restrict__ freg,
                                             unsigned long long *smax, unsigned long long *cmax, double bw,
                                             int last) {
    // the task is read through its pointer (uniform scalar loads); a local
    // copy indexed by the face number would live in scratch
    const int block = t->block, nface = t->nface;
    MeshParams &P = mp[t->mesh];
    const double inv_dx = P.inv_dx1 * double(1 << (t->level - 1));
    const double w = (bw * P.dt) * inv_dx;   // the stage's weight of dt L
    // psi decay factor of the second half step (MHD; the expression of k_glm_decay)
    const double hdec = 0.5 * P.dt;
    const double fdec = NV == 9 ? exp(-hdec * __longlong_as_double(P.cmax) * P.glm_alpha * inv_dx) : 1.0;
    unsigned long long m = 0, mc = 0;
    bool ok = true;
    // 256 lanes, one face cell each: (ta, tb) along the tangential axes,
    // quadrant q of the 4 fine blocks, first of its 2 x 2 fine faces (fa, fb)
    const int c = threadIdx.x;
    const int ta = c & 15, tb = c >> 4;
    const int q = (ta >> 3) + 2 * (tb >> 3);
    const int fa = 2 * (ta & 7), fb = 2 * (tb & 7);
    for (int n = 0; n < nface; ++n) {
        const int f = t->face[n], d = f >> 1, side = f & 1;
        const int xd = side ? BN - 1 : 0;
        const double *fr = freg + size_t(t->fslot[n][q]) * NV * REG;
        const double *cr = freg + size_t(t->cslot[n]) * NV * REG;
        // the face's cell: layer xd along the normal d, (ta, tb) along the
        // tangential axes (x or y, then z or y)
        const int cx = d == 0 ? xd : ta;
        const int cy = d == 1 ? xd : (d == 0 ? ta : tb);
        const int cz = d == 2 ? xd : tb;
        const size_t cell = (size_t(cz) * 16 + cy) * 16 + cx;
        // every load of the face before its stores
        const bool inx = XE && d == 0;   // the cells of an x face: from their copy, in whole runs
        double2v f4[NV][2];              // fa is even
        double fc[NV], uo[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double2v *fp = reinterpret_cast<const double2v *>(fr + v * REG + fb * 16 + fa);
            f4[v][0] = fp[0];
            f4[v][1] = fp[8];
            fc[v] = cr[v * REG + c];
            uo[v] = inx ? XE[xe_index(NV, block, cz, side, v) + cy * 2 + side]
                        : U[(size_t(block) * NV + v) * CELLS + cell];
        }
        // final unless a later face of the list also holds the cell
        bool fin = true;
        for (int n2 = n + 1; n2 < nface; ++n2) {
            const int f2 = t->face[n2], d2 = f2 >> 1;
            const int cd = d2 == 0 ? cx : (d2 == 1 ? cy : cz);
            fin &= cd != ((f2 & 1) ? BN - 1 : 0);
        }
        double nu[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double fm = ((f4[v][0].x + f4[v][0].y) + (f4[v][1].x + f4[v][1].y)) * 0.25;
            const double diff = fc[v] - fm;
            nu[v] = side ? uo[v] + w * diff : uo[v] - w * diff;
            // MHD, last stage: the second half of the GLM decay of psi, which
            // the stage kernel left out for the corrected cells, after the
            // cell's last correction
            if (NV == 9 && v == 8 && last && fin) nu[v] = nu[v] * fdec;
            U[(size_t(block) * NV + v) * CELLS + cell] = nu[v];
            if (XE && (cx < 2 || cx >= BN - 2)) {
                const int xs = cx >= BN - 2;
                XE[xe_index(NV, block, cz, xs, v) + cy * 2 + (cx - (xs ? BN - 2 : 0))] = nu[v];
            }
        }
        if (last) {
            if (fin) {
                bool ok2;
                double sg, cm = 0.0;
                if (NV == 9) sg = mhd_signal(nu, P.gamma, inv_dx, cm, ok2);
                else if (P.physics == PHYS_SRHD) sg = srhd_signal(nu, P.gamma, inv_dx, ok2);
                else sg = signal_rate(nu, P.gamma, inv_dx, ok2);
                ok &= ok2;
                const unsigned long long sb = __double_as_longlong(sg), cb = __double_as_longlong(cm);
                m = sb > m ? sb : m;
                mc = cb > mc ? cb : mc;
            }
        }
        if (n + 1 < nface) __syncthreads();
    }
    if (last) {
        m = wave_max_u64(m);
        if ((threadIdx.x & 63) == 0) atomicMax(&smax[block], m);
        if (cmax) {
            mc = wave_max_u64(mc);
            if ((threadIdx.x & 63) == 0) atomicMax(&cmax[block], mc);
        }
        if (!ok) atomicOr(&P.flags, 1);
    }
}

template <int NV>
__global__ __launch_bounds__(256) void k_reflux(const RefluxTask *__restrict__ tasks, MeshParams *mp,
                                                double *__restrict__ U, double *__restrict__ XE,
                                                const double *__restrict__ freg, unsigned long long *smax,
                                                unsigned long long *cmax, double bw, int last) {
    reflux_block<NV>(tasks + blockIdx.x, mp, U, XE, freg, smax, cmax, bw, last);
}

// Flux correction of stage output U together with the restriction of the
// ghost fill that follows it, in one launch of 256-lane workgroups:
// [0, nref) correct, the others restrict (two per task).  Only used when no block that is
// corrected is also read by a restriction task, so the two sets are
// independent.
template <int NV>
__global__ __launch_bounds__(256) void k_reflux_restrict(const RefluxTask *__restrict__ rtasks, int nref,
                                                         const RestrictTask *__restrict__ stasks, MeshParams *mp,
                                                         double *__restrict__ U, double *__restrict__ XE,
                                                         const double *__restrict__ freg, double *__restrict__ halo,
                                                         unsigned long long *smax, unsigned long long *cmax,
                                                         double bw, int last) {
    const int bid = blockIdx.x;
    if (bid < nref) {
        reflux_block<NV>(rtasks + bid, mp, U, XE, freg, smax, cmax, bw, last);
    } else {
        const int r = bid - nref;
        restrict_cell<NV>(stasks + (r >> 1), threadIdx.x + 256 * (r & 1), U, halo);
    }
}

// An upload's scan of pool blocks [first, first + n): per-block maximum signal
// rate (and, with cmax, the MHD speed max_d |v_d| + c_f,d) and the x-boundary
// columns of every row into XE, from one read of the state.  With src, the state
// is the caller's (local block q goes to pool block first + map[q]) and is
// written to the pool on the way.  A trip is two planes: lane = cell (x, y), and
// the lanes at x = 0, 1, 14, 15 write a plane's runs of XE.  Bound by HBM on
// large meshes: 512 to 2304 blocks took 55 us for the copy, 58 for the scan and
// 45 for the columns, whose rows share their cache lines with the rest of the
// state, each with a read of its own; scan and columns together 47, all 79.
template <int NV>
__global__ __launch_bounds__(512) void k_smax(const BlockDesc *desc, MeshParams *mp, double *__restrict__ U,
                                              double *__restrict__ XE, unsigned long long *smax,
                                              unsigned long long *cmax, int first, const double *__restrict__ src,
                                              const int *map) {
    __shared__ unsigned long long sMax[2][8];
    const int b = first + (src ? map[blockIdx.x] : int(blockIdx.x));
    const BlockDesc D = desc[b];
    MeshParams &P = mp[D.mesh];
    const double inv_dx = P.inv_dx1 * double(1 << (D.level - 1));
    const int x = threadIdx.x & 15, y = (threadIdx.x >> 4) & 15;
    const double *in = src ? src + size_t(blockIdx.x) * NV * CELLS : U + size_t(b) * NV * CELLS;
    unsigned long long m = 0, mc = 0;
    bool ok = true;
    for (int k = threadIdx.x >> 8; k < BN; k += 2) {
        const int cell = (k * 16 + y) * 16 + x;
        double u[9];
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v] = in[v * CELLS + cell];
        if (src) {
#pragma unroll
            for (int v = 0; v < NV; ++v) U[(size_t(b) * NV + v) * CELLS + cell] = u[v];
        }
        if (XE && ((x + 2) & 15) < 4) {
#pragma unroll
            for (int v = 0; v < NV; ++v) XE[xe_index(NV, b, k, x >> 3, v) + y * 2 + (x & 1)] = u[v];
        }
        bool ok2;
        double s, cm = 0.0;
        if (NV == 9) s = mhd_signal(u, P.gamma, inv_dx, cm, ok2);
        else if (P.physics == PHYS_SRHD) s = srhd_signal(u, P.gamma, inv_dx, ok2);
        else s = signal_rate(u, P.gamma, inv_dx, ok2);
        ok &= ok2;
        const unsigned long long sb = __double_as_longlong(s), cb = __double_as_longlong(cm);
        m = sb > m ? sb : m;
        mc = cb > mc ? cb : mc;
    }
    m = wave_max_u64(m);
    mc = wave_max_u64(mc);
    if ((threadIdx.x & 63) == 0) {
        sMax[0][threadIdx.x >> 6] = m;
        sMax[1][threadIdx.x >> 6] = mc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long r = sMax[0][0], rc = sMax[1][0];
        for (int w = 1; w < 8; ++w) {
            r = sMax[0][w] > r ? sMax[0][w] : r;
            rc = sMax[1][w] > rc ? sMax[1][w] : rc;
        }
        smax[b] = r;
        if (cmax) cmax[b] = rc;
    }
    if (!ok) atomicOr(&P.flags, 1);
}

// Per-mesh reductions, one workgroup per mesh of `meshes` (cmax: MHD only), at
// the end of a step (end = 1: t += dt, last_dt = dt) and after an upload: smax
// (and cmax) = max over the mesh's blocks, and the dt of the next step, dt =
// cfl / smax.  A step starts with no launch of its own: every kernel of it
// reads dt, and c_h = cmax (the launch that set dt cost 2.7 us and its gap,
// an 8-block step 30 -> 26 us).  Bound by latency, so the lanes follow the mesh
// sizes: 4096 blocks take 7.2 us with 256 lanes and 5.4 with 1024, 8 blocks 2.7
// and 3.6.
__device__ __forceinline__ unsigned long long mesh_max(const unsigned long long *x, int n) {
    unsigned long long m = 0;
#pragma unroll 4
    for (int q = threadIdx.x; q < n; q += int(blockDim.x)) m = x[q] > m ? x[q] : m;
    return wave_max_u64(m);
}
__global__ __launch_bounds__(1024) void k_mesh_reduce(MeshParams *mp, const int *meshes,
                                                      const unsigned long long *smax,
                                                      const unsigned long long *cmax, int end) {
    __shared__ unsigned long long sMax[2][16];
    MeshParams &P = mp[meshes[blockIdx.x]];
    const int first = P.first_block, n = P.nblocks;
    const unsigned long long m = mesh_max(smax + first, n), mc = cmax ? mesh_max(cmax + first, n) : 0;
    if ((threadIdx.x & 63) == 0) {
        sMax[0][threadIdx.x >> 6] = m;
        sMax[1][threadIdx.x >> 6] = mc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long r = sMax[0][0], rc = sMax[1][0];
        for (int w = 1; w < int(blockDim.x >> 6); ++w) {
            r = sMax[0][w] > r ? sMax[0][w] : r;
            rc = sMax[1][w] > rc ? sMax[1][w] : rc;
        }
        if (end) {
            const double dt = P.dt;
            P.t = P.t + dt;
            P.last_dt = dt;
        }
        P.smax = r;
        P.cmax = rc;
        P.dt = P.cfl / __longlong_as_double(r);
    }
}

__global__ void k_set_dt(MeshParams *mp, int mesh, double dt) {
    if (threadIdx.x == 0) mp[mesh].dt = dt;
}

// Block copies from the pool (block first + map[b]) to the caller's order (local
// index b).  A workgroup copies 1024 words of a block (W: 16 bytes, or 8 when
// the caller's pointer is only 8-byte aligned), each lane four that are in
// flight together, streaming.  Bound by HBM on large meshes (4096 blocks 247 ->
// 230 us, 5.8 TB/s) and by latency on small ones, where a workgroup per block
// left most of the chip idle (64 blocks 33 -> 7.6 us).
template <typename W>
__global__ __launch_bounds__(256) void k_permute(const W *__restrict__ src, W *__restrict__ dst, const int *map,
                                                 int first, int per_block, int parts) {
    const int b = blockIdx.x / parts, part = blockIdx.x - b * parts;
    const size_t o = size_t(first) + map[b];
    const int w = part * 1024 + threadIdx.x;
    const W *s = src + o * per_block + w;
    W *d = dst + size_t(b) * per_block + w;
    W x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (w + 256 * r < per_block) x[r] = __builtin_nontemporal_load(s + 256 * r);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (w + 256 * r < per_block) __builtin_nontemporal_store(x[r], d + 256 * r);
}

// Streaming copy of n 16-byte words, the measure of the bandwidth the chip
// sustains on a plain read + write stream: one word per lane and pass,
// nontemporal loads and stores (the fastest of the shapes measured on gfx950:
// 4, 8 words in flight per lane and smaller grids were slower).
__global__ __launch_bounds__(256) void k_stream_copy(const double2v *__restrict__ src, double2v *__restrict__ dst, size_t n) {
    const size_t stride = size_t(gridDim.x) * 256;
    for (size_t i = size_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += stride)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

hipError_t launch_stream_copy(const void *src, void *dst, size_t bytes, hipStream_t s) {
    const size_t n = bytes / 16;
    if (n == 0) return hipSuccess;
    const size_t want = (n + 255) / 256;
    const unsigned grid = unsigned(want < (size_t(1) << 22) ? want : (size_t(1) << 22));
    hipLaunchKernelGGL(k_stream_copy, dim3(grid), dim3(256), 0, s, static_cast<const double2v *>(src),
                       static_cast<double2v *>(dst), n);
    return hipGetLastError();
}

// Copies between a caller's state in blocks of (16 te)^3 cells and the pool's
// 16^3 tiles: caller tile q is sub-tile (tx, ty, tz) = (q mod te, ...) of
// caller block q / te^3, and lives at pool tile first + map[q].  gather = 1:
// pool -> caller layout, 0: caller layout -> pool.  A workgroup copies 1024
// words of one variable of a tile as k_permute does (16-byte words: 8 to a row
// of 16 cells; 512 tiles 58 -> 30 us).
template <typename W>
__global__ __launch_bounds__(256) void k_permute_tiles(const W *__restrict__ src, W *__restrict__ dst, const int *map,
                                                       int first, int NV, int te, int gather) {
    constexpr int RW = BN * sizeof(double) / sizeof(W);   // words of a tile's row
    constexpr int CW = BN * BN * RW, parts = CW / 1024;
    const int part = blockIdx.x % parts, tv = blockIdx.x / parts;
    const int v = tv % NV, q = tv / NV, t3 = te * te * te;
    const int bq = q / t3, t = q - bq * t3;
    const int tx = t % te, ty = (t / te) % te, tz = t / (te * te);
    const int B = BN * te;
    const size_t pool = ((size_t(first) + map[q]) * NV + v) * CW + part * 1024 + threadIdx.x;
    W x[4];
    size_t outer[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = part * 1024 + threadIdx.x + 256 * r;
        const int i = c % RW, j = (c / RW) & 15, k = c / (RW * BN);
        outer[r] = (((size_t(bq) * NV + v) * B + (tz * BN + k)) * B + (ty * BN + j)) * (te * RW) + tx * RW + i;
        x[r] = __builtin_nontemporal_load(gather ? src + pool + 256 * r : src + outer[r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) __builtin_nontemporal_store(x[r], gather ? dst + outer[r] : dst + pool + 256 * r);
}

// face ghosts of pool blocks [first, first + n) as the update reads them:
// out[local block][face][var][512]
__global__ __launch_bounds__(256) void k_read_ghosts(const BlockDesc *desc, const double *U, const double *halo,
                                                     double *out, int first, int NV) {
    const int lb = blockIdx.x, b = first + lb;
    for (int e = threadIdx.x; e < 6 * SLAB; e += blockDim.x) {
        const int f = e / SLAB, c = e - f * SLAB;
        const int d = f >> 1, side = f & 1;
        int g, ta, tb;
        slab_coords(d, c, g, ta, tb);
        int x[3];
        x[d] = side ? BN + g : g - NG;
        x[d == 0 ? 1 : 0] = ta;
        x[d == 2 ? 1 : 2] = tb;
        for (int v = 0; v < NV; ++v)
            out[((size_t(lb) * 6 + f) * NV + v) * SLAB + c] = block_value(desc, U, halo, NV, b, v, x[0], x[1], x[2]);
    }
}

// ---------------------------------------------------------------------------
// launch wrappers (host)

hipError_t launch_restrict(const RestrictTask *t, int n, const double *U, double *halo, int NV, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (NV == 9) hipLaunchKernelGGL(k_restrict<9>, dim3(4 * n), dim3(128), 0, s, t, U, halo);
    else hipLaunchKernelGGL(k_restrict<5>, dim3(4 * n), dim3(128), 0, s, t, U, halo);
    return hipGetLastError();
}

hipError_t launch_prolong(const ProlongTask *t, int n, const BlockDesc *desc, const MeshParams *mp, const double *U,
                          const double *XE, double *halo, int NV, int srhd, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (srhd && NV != 5) return hipErrorInvalidValue;
    if (srhd) hipLaunchKernelGGL(k_prolong_srhd, dim3(n), dim3(64), 0, s, t, desc, mp, U, halo);
    else if (NV == 9) hipLaunchKernelGGL(k_prolong<9>, dim3(n), dim3(64 * 9), 0, s, t, desc, U, XE, halo);
    else hipLaunchKernelGGL(k_prolong<5>, dim3(n), dim3(64 * 5), 0, s, t, desc, U, XE, halo);
    return hipGetLastError();
}

hipError_t launch_reflux(const RefluxTask *t, int n, MeshParams *mp, double *U, double *XE, const double *freg,
                         unsigned long long *smax, unsigned long long *cmax, int NV, double bw, int last,
                         hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (NV == 9)
        hipLaunchKernelGGL(k_reflux<9>, dim3(n), dim3(256), 0, s, t, mp, U, XE, freg, smax, cmax, bw, last);
    else hipLaunchKernelGGL(k_reflux<5>, dim3(n), dim3(256), 0, s, t, mp, U, XE, freg, smax, cmax, bw, last);
    return hipGetLastError();
}

hipError_t launch_reflux_restrict(const RefluxTask *rt, int nref, const RestrictTask *st, int nres, MeshParams *mp,
                                  double *U, double *XE, const double *freg, double *halo, unsigned long long *smax,
                                  unsigned long long *cmax, int NV, double bw, int last, hipStream_t s) {
    if (nref <= 0 || nres <= 0) return hipErrorInvalidValue;
    const dim3 grid(nref + 2 * nres), block(256);
    if (NV == 9)
        hipLaunchKernelGGL(k_reflux_restrict<9>, grid, block, 0, s, rt, nref, st, mp, U, XE, freg, halo, smax, cmax, bw,
                           last);
    else
        hipLaunchKernelGGL(k_reflux_restrict<5>, grid, block, 0, s, rt, nref, st, mp, U, XE, freg, halo, smax, cmax, bw,
                           last);
    return hipGetLastError();
}

hipError_t launch_smax(const BlockDesc *desc, MeshParams *mp, double *U, double *XE, unsigned long long *smax,
                       unsigned long long *cmax, int first, int n, int NV, const double *src, const int *map,
                       hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (NV == 9) hipLaunchKernelGGL(k_smax<9>, dim3(n), dim3(512), 0, s, desc, mp, U, XE, smax, cmax, first, src, map);
    else hipLaunchKernelGGL(k_smax<5>, dim3(n), dim3(512), 0, s, desc, mp, U, XE, smax, cmax, first, src, map);
    return hipGetLastError();
}

// nmax: blocks of the largest of the meshes
hipError_t launch_mesh_reduce(MeshParams *mp, const int *meshes, int nmesh, const unsigned long long *smax,
                              const unsigned long long *cmax, int nmax, int end, hipStream_t s) {
    if (nmesh <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mesh_reduce, dim3(nmesh), dim3(nmax > 512 ? 1024 : 256), 0, s, mp, meshes, smax, cmax, end);
    return hipGetLastError();
}

hipError_t launch_set_dt(MeshParams *mp, int mesh, double dt, hipStream_t s) {
    hipLaunchKernelGGL(k_set_dt, dim3(1), dim3(64), 0, s, mp, mesh, dt);
    return hipGetLastError();
}

// 16-byte words need both pointers 16-byte aligned (the pool's is)
static bool aligned16(const void *a, const void *b) {
    return ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0;
}

hipError_t launch_permute(const double *src, double *dst, const int *map, int first, int nblocks, int per_block,
                          hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    if (per_block % 2 == 0 && aligned16(src, dst)) {
        const int parts = (per_block / 2 + 1023) / 1024;
        hipLaunchKernelGGL(k_permute<double2v>, dim3(unsigned(nblocks) * parts), dim3(256), 0, s,
                           reinterpret_cast<const double2v *>(src), reinterpret_cast<double2v *>(dst), map, first,
                           per_block / 2, parts);
    } else {
        const int parts = (per_block + 1023) / 1024;
        hipLaunchKernelGGL(k_permute<double>, dim3(unsigned(nblocks) * parts), dim3(256), 0, s, src, dst, map, first,
                           per_block, parts);
    }
    return hipGetLastError();
}

hipError_t launch_permute_tiles(const double *src, double *dst, const int *map, int first, int ntiles, int NV,
                                int te, int gather, hipStream_t s) {
    if (ntiles <= 0) return hipSuccess;
    if (aligned16(src, dst))
        hipLaunchKernelGGL(k_permute_tiles<double2v>, dim3(unsigned(ntiles) * NV * 2), dim3(256), 0, s,
                           reinterpret_cast<const double2v *>(src), reinterpret_cast<double2v *>(dst), map, first, NV, te, gather);
    else
        hipLaunchKernelGGL(k_permute_tiles<double>, dim3(unsigned(ntiles) * NV * 4), dim3(256), 0, s, src, dst, map,
                           first, NV, te, gather);
    return hipGetLastError();
}

hipError_t launch_read_ghosts(const BlockDesc *desc, const double *U, const double *halo, double *out, int first,
                              int n, int NV, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_read_ghosts, dim3(n), dim3(256), 0, s, desc, U, halo, out, first, NV);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// regrid: error estimate and data transfer

// Loehner's normalised second difference of variable v per cell, summed over
// the three axes without cross terms (face ghosts at block sides),
//   E = sqrt(sum_d a_d^2 / sum_d b_d^2),  a_d = (u+ - u) - (u - u-),
//   b_d = (|u+ - u| + |u - u-|) + eps((|u+| + 2|u|) + |u-|),
// sums in x, y, z order, no contraction and IEEE division and square root
// (E = 0 where v is zero on the whole stencil and both sums vanish),
// so the block maximum is the same number on any machine.  One workgroup per
// block, lane = column and every fourth plane (bound by the latency of the
// stencil's loads: 59 us on 512 to 2304 blocks with a lane per column, now
// 34); out[block - first] = max over the block's cells.
template <int NV>
__global__ __launch_bounds__(1024) void k_lohner(const BlockDesc *__restrict__ desc, const double *__restrict__ U,
                                                const double *__restrict__ halo, int first, int v, double eps,
                                                double *__restrict__ out) {
#pragma clang fp contract(off)
    __shared__ unsigned long long sMax[16];
    const int b = first + blockIdx.x;
    const int i = threadIdx.x & 15, j = (threadIdx.x >> 4) & 15;
    unsigned long long m = 0;
    for (int k = threadIdx.x >> 8; k < BN; k += 4) {
        const double u0 = U[(size_t(b) * NV + v) * CELLS + (k * 16 + j) * 16 + i];
        double num = 0.0, den = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double up = block_value(desc, U, halo, NV, b, v, i + (d == 0), j + (d == 1), k + (d == 2));
            const double um = block_value(desc, U, halo, NV, b, v, i - (d == 0), j - (d == 1), k - (d == 2));
            const double a = (up - u0) - (u0 - um);
            const double c = (__builtin_fabs(up - u0) + __builtin_fabs(u0 - um)) +
                             eps * ((__builtin_fabs(up) + 2.0 * __builtin_fabs(u0)) + __builtin_fabs(um));
            num = num + a * a;
            den = den + c * c;
        }
        const double e = den > 0.0 ? __builtin_sqrt(num / den) : 0.0;   // den = 0: v is 0 on the stencil
        const unsigned long long eb = __double_as_longlong(e);   // e >= 0: bit order = numeric order
        m = eb > m ? eb : m;
    }
    m = wave_max_u64(m);
    if ((threadIdx.x & 63) == 0) sMax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long r = sMax[0];
        for (int w = 1; w < 16; ++w) r = sMax[w] > r ? sMax[w] : r;
        out[blockIdx.x] = __longlong_as_double(r);
    }
}

// Data of the new leaves of a regrid, one workgroup per new leaf and variable:
// kind 0 copies block src[0]; kind 1 is child `octant` of parent src[0] --
// parent cell plus, in x, y, z order, +/- 1/4 minmod of the parent's axis
// differences (the parent's face ghosts at its sides), as the ghost
// prolongation; kind 2 is the mean of the 8 children src[octant], summed
// pairwise as the restriction.  All indices are pool indices of the old mesh,
// whose ghosts must be filled.  SRHD (srhd != 0) prolongs the primitives, as
// its ghost prolongation: one lane per child cell, the cells shared out over
// the leaf's workgroups.  Bound by HBM: rows are read and written in 16-byte
// words, and a lane of kind 1 forms a parent's slopes once for its 8 children
// (512 -> 2304 and 2304 -> 512 blocks 244 us on average with a workgroup per
// leaf, a cell per lane; now 100).
template <int NV>
__global__ __launch_bounds__(256) void k_remap(const RemapTask *__restrict__ tasks, const BlockDesc *__restrict__ desc,
                                               const MeshParams *__restrict__ mp, const double *__restrict__ U,
                                               const double *__restrict__ halo, double *__restrict__ out, int srhd) {
    const int leaf = blockIdx.x / NV, v = blockIdx.x - leaf * NV;
    const RemapTask *t = tasks + leaf;   // read through the pointer (no scratch copy)
    const int kind = t->kind, oc = t->octant;
    double *o = out + (size_t(leaf) * NV + v) * CELLS;
    double2v *o2 = reinterpret_cast<double2v *>(o);
    if (kind == 0) {
        const double2v *src = reinterpret_cast<const double2v *>(U + (size_t(t->src[0]) * NV + v) * CELLS);
        double2v x[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) x[r] = src[256 * r + threadIdx.x];
#pragma unroll
        for (int r = 0; r < 8; ++r) o2[256 * r + threadIdx.x] = x[r];
        return;
    }
    if (kind == 2) {
        // two cells along x per lane and trip
#pragma unroll 2
        for (int e = threadIdx.x; e < CELLS / 2; e += 256) {
            const int i = 2 * (e & 7), j = (e >> 3) & 15, k = e >> 7;
            const int F = t->src[(i >> 3) + 2 * (j >> 3) + 4 * (k >> 3)];
            const double2v *u = reinterpret_cast<const double2v *>(U + (size_t(F) * NV + v) * CELLS +
                                                         ((2 * (k & 7)) * 16 + 2 * (j & 7)) * 16 + 2 * (i & 7));
            double2v r;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double2v a = u[c], b = u[8 + c], d = u[128 + c], f = u[136 + c];
                const double s = ((a.x + a.y) + (b.x + b.y)) + ((d.x + d.y) + (f.x + f.y));
                r[c] = s * 0.125;
            }
            o2[e] = r;
        }
        return;
    }
    const int P = t->src[0];
    const int px = (oc & 1) * 8, py = ((oc >> 1) & 1) * 8, pz = (oc >> 2) * 8;
    if (NV == 5 && srhd) {
        const double g = mp[desc[P].mesh].gamma;
#pragma unroll 1
        for (int cell = v * 256 + threadIdx.x; cell < CELLS; cell += NV * 256) {
            const int i = cell & 15, j = (cell >> 4) & 15, k = cell >> 8;
            double wc[5], q[3][5], c[5];
            const bool ok = srhd_parent(desc, U, halo, P, px + (i >> 1), py + (j >> 1), pz + (k >> 1), g, wc, q);
            srhd_child(wc, q, i & 1, j & 1, k & 1, g, ok, c);
#pragma unroll
            for (int w = 0; w < 5; ++w) out[(size_t(leaf) * NV + w) * CELLS + cell] = c[w];
        }
        return;
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int i = threadIdx.x & 7, j = (threadIdx.x >> 3) & 7, k = (threadIdx.x >> 6) + 4 * half;
        const int cx = px + i, cy = py + j, cz = pz + k;
        const double vc = U[(size_t(P) * NV + v) * CELLS + (cz * 16 + cy) * 16 + cx];
        double q[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double vm = block_value(desc, U, halo, NV, P, v, cx - (d == 0), cy - (d == 1), cz - (d == 2));
            const double vp = block_value(desc, U, halo, NV, P, v, cx + (d == 0), cy + (d == 1), cz + (d == 2));
            q[d] = 0.25 * minmod(vc - vm, vp - vc);
        }
        const double x[2] = {vc - q[0], vc + q[0]};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int sy = c & 1, sz = c >> 1;
            double2v r;
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                const double y = sy ? x[sx] + q[1] : x[sx] - q[1];
                r[sx] = sz ? y + q[2] : y - q[2];
            }
            o2[((2 * k + sz) * 16 + 2 * j + sy) * 8 + i] = r;
        }
    }
}

hipError_t launch_lohner(const BlockDesc *desc, const double *U, const double *halo, int first, int n, int NV, int v,
                         double eps, double *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (v < 0 || v >= NV) return hipErrorInvalidValue;
    if (NV == 9) hipLaunchKernelGGL(k_lohner<9>, dim3(n), dim3(1024), 0, s, desc, U, halo, first, v, eps, out);
    else hipLaunchKernelGGL(k_lohner<5>, dim3(n), dim3(1024), 0, s, desc, U, halo, first, v, eps, out);
    return hipGetLastError();
}

hipError_t launch_remap(const RemapTask *t, int n, const BlockDesc *desc, const MeshParams *mp, const double *U,
                        const double *halo, int NV, int srhd, double *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (srhd && NV != 5) return hipErrorInvalidValue;
    if (NV == 9) hipLaunchKernelGGL(k_remap<9>, dim3(unsigned(n) * 9), dim3(256), 0, s, t, desc, mp, U, halo, out, 0);
    else hipLaunchKernelGGL(k_remap<5>, dim3(unsigned(n) * 5), dim3(256), 0, s, t, desc, mp, U, halo, out, srhd);
    return hipGetLastError();
}

} // namespace agile
