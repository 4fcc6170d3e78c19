// PC2: block-Jacobi preconditioner with a zero-fill incomplete LU factor per
// block (the paper, Section 2.2; MAS factors one block per MPI rank, and
// Section 4.1 notes that its triangular solves are sequential and that PC1
// performed about as well on GPUs).
//
// Blocks are boxes of kPc2I x kPc2J x kPc2K cells (r, theta, phi) tiling the
// grid from index 0; couplings between blocks and the periodic phi coupling
// are left out.  On the scaled system A^ = W^-1 A W^-1 (unit diagonal,
// A^(c, nb) = -c^) with cells in natural order, ILU(0) of a box with the
// 7-point graph changes only the diagonal:
//     d_c = 1 - sum_{lower neighbours nb in the block} c^_{c,nb}^2 / d_nb,
// and M^-1 r is
//     forward   y_c = (r_c + sum_{lower nb} c^ y_nb) / d_c
//     backward  z_c = y_c + (sum_{upper nb} c^ z_nb) / d_c.
// (The ILU(0) factor of the scaled matrix is the scaled ILU(0) factor of A,
// so PCG on A^ with it has the iterates of PCG on A with the ILU(0) of A.)
// The direction and SpMV step of a PC2 iteration (p = z + beta p, q = A^ p,
// (p, q)) is the PCG iteration kernel run without r, q and x inputs.
//
// Factor: one wave per block, lane k' owns phi offset k', the wave walks the
// block's (r, theta) rows in order and solves each row's phi recurrence
// d_k = s_k - c^2 / d_{k-1} by a prefix scan of 2 x 2 matrices (the maps
// d -> (s d - c^2) / d compose as matrix products).
// Solve: one wave per r plane of the block, lane k' owns phi offset k'
// (coalesced rows), the rows taken as a wavefront over (r, theta).  The r and
// theta terms come from the rows already done; along phi the
// forward sweep is the first-order recurrence y_k = c_k y_{k-1} + b_k with
// c_k = c^p_{k-1,k} / d_k, solved by a prefix scan of the affine maps
// y -> c y + b across the lanes (the backward sweep scans the other way).
#pragma once

#include "kernels.hpp"

namespace mas {

constexpr int kPc2I = 8, kPc2J = 8, kPc2K = 64;
static_assert(kPc2K == kWave, "one lane per phi offset of a block");

// The factor kernel's arguments.
struct Pc2FacArgs {
    const double *cr, *ct, *cp;  // scaled couplings to the +r, +theta, +phi neighbours
    Dims dm;
    int nbi, nbj, nbk;           // blocks per direction
};

// Inclusive scan of the affine maps y -> C y + B over the 64 lanes in lane
// order: each lane ends with the composition of its own map after those of
// all lower lanes, i.e. B = y_lane for y_-1 = 0.  DPP moves (GFX9 family):
// row_shr by 1, 2, 4, 8 inside each 16-lane row, then row_bcast:15 (the last
// lane of rows 0 and 2 to rows 1 and 3) and row_bcast:31 (lane 31 to rows 2
// and 3).  A lane that receives nothing gets the identity map (1, 0), which
// composes as a no-op.
template <int CTRL, int ROWS>
__device__ inline double dpp_or(double v, double identity) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v), o = __builtin_bit_cast(uint64_t, identity);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)b,
                                                              CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32),
                                                              (int)(uint32_t)(b >> 32), CTRL, ROWS,
                                                              0xf, false);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

template <int CTRL, int ROWS>
__device__ inline float dpp_or(float v, float identity) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, identity),
                                                                 __builtin_bit_cast(int, v), CTRL,
                                                                 ROWS, 0xf, false));
}

template <int CTRL, int ROWS, typename T>
__device__ inline void affine_step(T &C, T &B) {
    const T Cs = dpp_or<CTRL, ROWS>(C, T(1)), Bs = dpp_or<CTRL, ROWS>(B, T(0));
    B = C * Bs + B;
    C = C * Cs;
}

template <typename T>
__device__ inline T affine_scan(T C, T B) {
    affine_step<0x111, 0xf>(C, B);  // row_shr:1
    affine_step<0x112, 0xf>(C, B);  // row_shr:2
    affine_step<0x114, 0xf>(C, B);  // row_shr:4
    affine_step<0x118, 0xf>(C, B);  // row_shr:8
    affine_step<0x142, 0xa>(C, B);  // row_bcast:15 into rows 1 and 3
    affine_step<0x143, 0xc>(C, B);  // row_bcast:31 into rows 2 and 3
    return B;
}

// Linear-fractional maps d -> (m00 d + m01) / (m10 d + m11) as 2 x 2 matrices
// (projective: a common factor does not change the map).
struct Mob {
    double m00, m01, m10, m11;
};

// Inclusive scan of such maps over the 64 lanes in lane order (the same DPP
// moves as affine_scan; a lane that receives nothing composes with the
// identity).  After the first three steps (products of up to eight maps)
// the product is rescaled by a power of two, exactly, so that the longer
// products of the last three steps neither overflow nor underflow: every
// map [s, -c^2; 1, 0] has entries of magnitude at most 1 (unit diagonal,
// diagonal dominance), so the entries of a product of eight stay within
// [min(s)^8, 2^8].  A power-of-two scale commutes with every rounding here,
// so the result is the same, bit for bit, as with a rescale after every
// step; the map is applied as a ratio, which ignores the scale.
template <int CTRL, int ROWS, bool RESCALE>
__device__ inline void mobius_step(Mob &P) {
    const double q00 = dpp_or<CTRL, ROWS>(P.m00, 1.0), q01 = dpp_or<CTRL, ROWS>(P.m01, 0.0);
    const double q10 = dpp_or<CTRL, ROWS>(P.m10, 0.0), q11 = dpp_or<CTRL, ROWS>(P.m11, 1.0);
    // each entry a sum of two products, the first fused: written out, so
    // that the rounding does not depend on which product the compiler would
    // fuse in a given context
    const double r00 = fma(P.m00, q00, P.m01 * q10), r01 = fma(P.m00, q01, P.m01 * q11);
    const double r10 = fma(P.m10, q00, P.m11 * q10), r11 = fma(P.m10, q01, P.m11 * q11);
    if constexpr (RESCALE) {
        const double m = fmax(fmax(fabs(r00), fabs(r01)), fmax(fabs(r10), fabs(r11)));
        const int ex = (m > 0.0) ? ilogb(m) : 0;
        P = Mob{ldexp(r00, -ex), ldexp(r01, -ex), ldexp(r10, -ex), ldexp(r11, -ex)};
    } else {
        P = Mob{r00, r01, r10, r11};
    }
}

__device__ inline Mob mobius_scan(Mob P) {
    mobius_step<0x111, 0xf, false>(P);  // row_shr:1
    mobius_step<0x112, 0xf, false>(P);  // row_shr:2
    mobius_step<0x114, 0xf, true>(P);   // row_shr:4
    mobius_step<0x118, 0xf, false>(P);  // row_shr:8
    mobius_step<0x142, 0xa, false>(P);  // row_bcast:15 into rows 1 and 3
    mobius_step<0x143, 0xc, false>(P);  // row_bcast:31 into rows 2 and 3
    return P;
}

// d_c for every cell of the block, from the double-precision couplings (a
// single-precision factor is the double one rounded: TOUT = float).  Lanes
// run along phi (coalesced rows) and the wave walks the block's (r, theta)
// rows in order, as the solve does; with the r and theta terms of a row
// known from the rows done, the phi recurrence
//     d_k = s_k - cp_{k-1,k}^2 / d_{k-1},   s_k = 1 - (r and theta terms),
// is the composition of the maps d -> (s_k d - cp^2) / d, solved by a prefix
// scan of their matrices [s_k, -cp^2; 1, 0] (the first lane of a block has
// no phi term: [s_0, 0; 1, 0], which gives d_0 = s_0 from any start).
// Each row's couplings are loaded one plane (eight rows) before it is
// scanned, into one of two register sets that alternate by plane.  Every
// access goes through a buffer resource over one r plane, and whatever is
// not there (the -r coupling of the block's first plane, the -theta one of
// its first row, the -phi one of its first lane, lanes and rows past the
// grid, planes past the block) has bit 31 set in its offset or a resource of
// size zero: it reads zero or is not stored.  The loop body has no branch:
// a missing coupling enters as 0 against a previous d of 1, which leaves s_k
// unchanged bit for bit (1 - 0 * 0 / 1 = 1); lanes past the grid are the
// highest ones, and the scan only moves values to higher lanes, so their
// maps never reach a lane in the grid; planes are taken in pairs, the
// second of an odd last pair storing nothing.  So the compiler waits for
// each plane's loads only where they are used.
struct Pc2Fac {
    double cr, ct, cp;
};
struct Pc2FacPlane {
    __amdgpu_buffer_rsrc_t cr, ct, cp;  // cr over the plane below, ct and cp over this one
};

template <typename TOUT>
__global__ __launch_bounds__(kWave) void k_pc2_factor(Pc2FacArgs a, TOUT *dout) {
    const Dims &dm = a.dm;
    const int blk = blockIdx.x;
    const int bk = blk % a.nbk, bj = (blk / a.nbk) % a.nbj, bi = blk / (a.nbk * a.nbj);
    const int lane = threadIdx.x;
    const int I0 = bi * kPc2I, J0 = bj * kPc2J, k0 = bk * kPc2K;
    const int kn = min(kPc2K, dm.np - k0);
    const bool act = lane < kn;
    const int ni = min(kPc2I, dm.nr - I0), nj = min(kPc2J, dm.nt - J0);
    // an r plane of one array holds fewer than 2^31 / 7 bytes (the grid
    // check keeps seven planes below 2 GiB): byte offsets of its cells stay
    // below bit 31
    const uint32_t pbytes = (uint32_t)(dm.plane * 8);
    const uint32_t lbad = act ? 0u : kOOB;
    const uint32_t pbad = (act && lane > 0) ? 0u : kOOB;
    // this lane's cell of block row jj in a plane, and the bad bit of the row
    auto cell = [&](int jj) -> int { return (J0 + jj) * dm.np + k0 + lane; };
    auto rbad = [&](int jj) -> uint32_t { return (jj < nj ? 0u : kOOB) | lbad; };
    auto plane_rsrc = [&](int ii) {
        const bool in = ii < ni;
        const int m = min(I0 + ii, dm.nr - 1), mb = max(I0 + ii - 1, 0);
        return Pc2FacPlane{make_rsrc(a.cr + (int64_t)mb * dm.plane, (in && ii > 0) ? pbytes : 0u),
                           make_rsrc(a.ct + (int64_t)m * dm.plane, in ? pbytes : 0u),
                           make_rsrc(a.cp + (int64_t)m * dm.plane, in ? pbytes : 0u)};
    };
    auto load = [&](const Pc2FacPlane &R, int jj) {
        const int c = cell(jj);
        const uint32_t bad = rbad(jj);
        Pc2Fac v;
        v.cr = bld<double, 1>(R.cr, ((uint32_t)c * 8u) | bad).v[0];
        v.ct = bld<double, 1>(R.ct, ((uint32_t)(c - dm.np) * 8u) | bad | (jj > 0 ? 0u : kOOB)).v[0];
        v.cp = bld<double, 1>(R.cp, ((uint32_t)(c - 1) * 8u) | bad | pbad).v[0];
        return v;
    };
    double dp[kPc2J];  // d of the previous r plane of the block, per theta row
#pragma unroll
    for (int jj = 0; jj < kPc2J; ++jj) dp[jj] = 1.0;
    // plane ii: rows from `cur`, the rows of plane ii + 1 issued into `nxt`
    auto plane_step = [&](int ii, const Pc2Fac (&cur)[kPc2J], Pc2Fac (&nxt)[kPc2J]) {
        const Pc2FacPlane Rn = plane_rsrc(ii + 1);
        const auto Rd = make_rsrc(dout + (int64_t)min(I0 + ii, dm.nr - 1) * dm.plane,
                                  ii < ni ? (uint32_t)(dm.plane * (int64_t)sizeof(TOUT)) : 0u);
        double drow = 1.0;  // d of the previous theta row
#pragma unroll
        for (int jj = 0; jj < kPc2J; ++jj) {
            const Pc2Fac c = cur[jj];
            nxt[jj] = load(Rn, jj);
            // keeps the loads here: the scheduler would otherwise sink them
            // towards their use a plane later, where they would be waited for
            // right after being issued
            __builtin_amdgcn_sched_barrier(0);
            double sk = 1.0;
            sk -= c.cr * c.cr / dp[jj];  // no -r neighbour in the block: 0
            sk -= c.ct * c.ct / drow;    // no -theta neighbour: 0
            Mob P{sk, -(c.cp * c.cp), 1.0, 0.0};
            P = mobius_scan(P);
            const double dv = (P.m00 + P.m01) / (P.m10 + P.m11);  // the map of d = 1
            bst<TOUT, 1>(Rd, ((uint32_t)cell(jj) * (uint32_t)sizeof(TOUT)) | rbad(jj),
                         VecT<TOUT, 1>{{(TOUT)dv}});
            dp[jj] = dv;
            drow = dv;
        }
    };
    Pc2Fac qa[kPc2J], qb[kPc2J];
    {
        const Pc2FacPlane R0 = plane_rsrc(0);
#pragma unroll
        for (int jj = 0; jj < kPc2J; ++jj) qa[jj] = load(R0, jj);
        // the first plane's rows are waited for here, once per block (an
        // empty statement that takes them as register operands: the
        // compiler waits for their loads before it): the loop is then
        // entered with no loads in flight, and the waits the compiler
        // places in it are those of its own loads, a plane after issue
#pragma unroll
        for (int jj = 0; jj < kPc2J; ++jj)
            asm volatile("" ::"v"(qa[jj].cr), "v"(qa[jj].ct), "v"(qa[jj].cp));
    }
    for (int ii = 0; ii < ni; ii += 2) {
        plane_step(ii, qa, qb);
        plane_step(ii + 1, qb, qa);
    }
}

// z = M^-1 r for NR right-hand sides, first applying r -= alpha q when
// a.update; per-block partials (r, z) and ||W r||^2 of each (values 2 h and
// 2 h + 1 of [][nblk]).  A right-hand side whose control block is
// stopped is left alone.
// With L the strictly lower couplings and D = diag(d), M = (D - L) D^-1 (D - L^T),
// the forward sweep gives y = (D - L)^-1 r and z = (D - L^T)^-1 D y, so
// (r, z) = r^T (D - L^T)^-1 D (D - L)^-1 r = y^T D y: the forward sweep
// accumulates it and the backward sweep need not read r again.
//
// What bounds it: memory, 9 words per cell (r, q, w, d, three couplings; r and
// z written) once nothing is read twice, and on small grids the chain of
// dependent rows.  So the whole block sits in registers between the sweeps,
// and the rows run as a wavefront: wave ii of the block's eight owns r plane ii
// with all its rows in registers, loads everything up front (about 50 loads in
// flight per wave), and works on row jj in step ii + jj, when row jj of the
// plane below (ii - 1, through LDS) and row jj - 1 (its own) are done: 15
// steps a sweep instead of 64, one barrier each.  Every wave passes the same
// number of barriers: ii before its first row, one per row, ni - 1 - ii after.
// In the backward sweep lane l takes phi offset 63 - l, so that the recurrence
// runs up the lanes again: y, 1/d and the phi and theta couplings are turned
// round by a lane permute, the r couplings come reversed from the LDS copy
// that the forward sweep of the plane above read too.
// Right-hand sides run one after the other on the same coefficients; in single
// precision the next one's r and q are in flight while one is swept.  In
// double precision those 32 registers more spill (four waves per SIMD, so that
// two blocks share a CU: one loads while the other sweeps): three right-hand
// sides on 256 x 320 x 640 cells 164 ms a solve with them, 122 ms without.  Two,
// three and four right-hand sides in double precision spill 10, 16 and 29
// registers all the same, four in single precision 13.
// 256 x 320 x 640 cells, one right-hand side: 670 us in double precision (5.6
// TB/s at 72 B per cell) and 360 us in single (40 B), against 1340 and 735 us
// for one wave per block that walked the 64 rows alone, re-read the
// coefficients and y, and moved x (144 and 76 B); 61 x 93 x 187 cells 32
// against 76 us.  Streamed inputs are loaded non-temporally: 128 x 192 x 384
// cells 8.77 against 9.46 ms a solve without the hint.
template <typename T, int NR>
struct Pc2Args {
    const T *cr, *ct, *cp;  // scaled couplings to the +r, +theta, +phi neighbours
    const double *w;
    const T *d;             // modified diagonal
    T *r[NR], *z[NR];
    const T *q[NR];
    double *partials;
    Ctl *ctl;               // [NR]
    BlockCount *count;
    Report rep;
    Dims dm;
    int nbi, nbj, nbk;      // blocks per direction
    int update;             // 1: r -= alpha q first; 0: the solve of a run's initial residual
};

constexpr int kPc2Threads = kWave * kPc2I;

// After the block solves (one thread): the stopping test on RW = ||W r||^2 and
// beta from RZ = (r, z).  ctl->iter counts finished iterations; first marks the
// solve of the initial residual (no iteration finished yet).
__device__ inline void pc2_beta(Ctl *ctl, double RZ, double RW, bool first) {
    const int k = first ? ctl->iter : ctl->iter + 1;
    ctl->iter = k;
    ctl->rw = RW;
    if (RW <= ctl->tol2 || RW == 0.0) {
        ctl->flag = FLAG_CONV;
        ctl->conv_iter = k;
        return;
    }
    if (k >= ctl->max_iter) {
        ctl->flag = FLAG_MAXIT;
        ctl->conv_iter = k;
        return;
    }
    if (!(RZ > 0.0) || !isfinite(RZ)) {
        ctl->flag = FLAG_BREAK;
        ctl->conv_iter = k;
        return;
    }
    ctl->beta = first ? 0.0 : RZ / ctl->rr;
    ctl->rr = RZ;
}

// lane l's value from lane 63 - l
__device__ inline float lane_reverse(float v, int addr) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr, __builtin_bit_cast(int, v)));
}
__device__ inline double lane_reverse(double v, int addr) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)b);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(addr, (int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, lo | (hi << 32));
}

template <typename T, int NR>
__global__ __launch_bounds__(kPc2Threads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_pc2_solve(Pc2Args<T, NR> a) {
    __shared__ T sCr[kPc2I][kPc2J][kPc2K];  // couplings to the +r neighbour
    __shared__ T sY[2][kPc2I][kPc2K];       // the row each plane finished last, by step parity
    __shared__ double sRed[kPc2I][2];
    // whether the next right-hand side's r and q are loaded ahead (see above)
    constexpr bool PF = sizeof(T) == 4;
    bool run[NR];
    bool any = false;
#pragma unroll
    for (int h = 0; h < NR; ++h) {
        run[h] = a.ctl[h].flag == FLAG_RUN;
        any = any || run[h];
    }
    if (!any) return;
    const Dims &dm = a.dm;
    const int nblk = gridDim.x;
    const int blk = xcd_remap(blockIdx.x, nblk);
    const int bk = blk % a.nbk, bj = (blk / a.nbk) % a.nbj, bi = blk / (a.nbk * a.nbj);
    const int lane = threadIdx.x & (kWave - 1);
    const int ii = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int I0 = bi * kPc2I, J0 = bj * kPc2J, k0 = bk * kPc2K;
    const int kn = min(kPc2K, dm.np - k0);
    const int ni = min(kPc2I, dm.nr - I0), nj = min(kPc2J, dm.nt - J0);
    const bool act = lane < kn;
    const bool in = ii < ni;
    const int64_t first = (int64_t)min(I0 + ii, dm.nr - 1) * dm.plane;
    // one r plane of an array (fewer than 2^31 / 7 bytes: the grid check), or nothing
    auto plane_rsrc = [&](const auto *p, bool on) {
        return make_rsrc(p ? p + first : p, (p && on && in) ? (uint32_t)(dm.plane * (int64_t)sizeof(*p)) : 0u);
    };
    // this lane's cell of row jj; rows and lanes past the grid: out of range
    auto cell = [&](int jj) { return (uint32_t)((J0 + jj) * dm.np + k0 + lane); };
    auto off = [&](int jj, bool on, uint32_t es) { return (on && jj < nj) ? cell(jj) * es : kOOB; };
    constexpr uint32_t ES = sizeof(T);
    const bool upd = a.update != 0;

    T rc[kPc2J], qv[kPc2J];
    auto load_rq = [&](int h) {
        const auto Rr = plane_rsrc(a.r[h], run[h]), Rq = plane_rsrc(a.q[h], run[h] && upd);
#pragma unroll
        for (int jj = 0; jj < kPc2J; ++jj) {
            rc[jj] = bld<T, 1, kAuxNT>(Rr, off(jj, act, ES)).v[0];
            qv[jj] = bld<T, 1, kAuxNT>(Rq, off(jj, act, ES)).v[0];
        }
    };
    T crv[kPc2J], d[kPc2J], dinv[kPc2J], ctm[kPc2J], cp[kPc2J];
    double w[kPc2J];
    {
        const auto Rcr = plane_rsrc(a.cr, ii < ni - 1), Rct = plane_rsrc(a.ct, true), Rcp = plane_rsrc(a.cp, true),
                   Rd = plane_rsrc(a.d, true), Rw = plane_rsrc(a.w, true);
#pragma unroll
        for (int jj = 0; jj < kPc2J; ++jj) crv[jj] = bld<T, 1, kAuxNT>(Rcr, off(jj, act, ES)).v[0];
        load_rq(0);
#pragma unroll
        for (int jj = 0; jj < kPc2J; ++jj) {
            d[jj] = bld<T, 1, kAuxNT>(Rd, off(jj, act, ES)).v[0];
            cp[jj] = bld<T, 1, kAuxNT>(Rcp, off(jj, lane < kn - 1, ES)).v[0];
            ctm[jj] = (jj > 0) ? bld<T, 1, kAuxNT>(Rct, off(jj, act, ES) - (uint32_t)dm.np * ES).v[0] : T(0);
        }
#pragma unroll
        for (int jj = 0; jj < kPc2J; ++jj) w[jj] = bld<double, 1, kAuxNT>(Rw, off(jj, act, 8u)).v[0];
    }
#pragma unroll
    for (int jj = 0; jj < kPc2J; ++jj) sCr[ii][jj][lane] = crv[jj];
#pragma unroll
    for (int jj = 0; jj < kPc2J; ++jj) {
        if (!(in && act && jj < nj)) d[jj] = T(1);
        dinv[jj] = T(1) / d[jj];
    }
    const int rlane = kWave - 1 - lane, raddr = 4 * rlane;

#pragma unroll
    for (int h = 0; h < NR; ++h) {
        if (!run[h]) {  // uniform across the block
            if (PF && h + 1 < NR) load_rq(h + 1);
            continue;
        }
        if (!PF && h > 0) load_rq(h);
        const T alpha = upd ? (T)a.ctl[h].alpha : T(0);
        double rz = 0.0, rw = 0.0;
        T y[kPc2J];
        {
            const auto Rr = plane_rsrc(a.r[h], upd);
#pragma unroll
            for (int jj = 0; jj < kPc2J; ++jj) {
                const T v = rc[jj] - alpha * qv[jj];
                y[jj] = v;
                bst<T, 1, kAuxNT>(Rr, off(jj, act, ES), VecT<T, 1>{{v}});
                const double t = w[jj] * (double)v;
                rw = __builtin_fma(t, t, rw);
            }
        }
        if (PF && h + 1 < NR) load_rq(h + 1);
        // ---- forward sweep
        for (int t = 0; t < min(ii, ni + nj - 1); ++t) __syncthreads();
        if (in) {
#pragma unroll
            for (int jj = 0; jj < kPc2J; ++jj) {
                if (jj < nj) {
                    T sc = y[jj];
                    if (ii > 0) sc = fma(sCr[ii - 1][jj][lane], sY[(ii + jj - 1) & 1][ii - 1][lane], sc);
                    if (jj > 0) sc = fma(ctm[jj], y[jj > 0 ? jj - 1 : 0], sc);
                    // the first lane has no -phi neighbour: lane_prev gives it 0
                    const T v = affine_scan(lane_prev(cp[jj]) * dinv[jj], sc * dinv[jj]);
                    y[jj] = v;
                    sY[(ii + jj) & 1][ii][lane] = v;
                    __syncthreads();
                    rz = __builtin_fma((double)d[jj] * (double)v, (double)v, rz);
                }
            }
            for (int t = 0; t < ni - 1 - ii; ++t) __syncthreads();
        } else {
            for (int t = 0; t < ni + nj - 1 - min(ii, ni + nj - 1); ++t) __syncthreads();
        }
        // ---- backward sweep, lanes reversed
        const auto Rz = plane_rsrc(a.z[h], true);
        const uint32_t zoff = (rlane < kn) ? (uint32_t)(J0 * dm.np + k0 + rlane) * ES : kOOB;
        if (in) {
            for (int t = 0; t < ni - 1 - ii; ++t) __syncthreads();
            T zrow = T(0);
#pragma unroll
            for (int jj = kPc2J - 1; jj >= 0; --jj) {
                if (jj < nj) {
                    const int step = (ni - 1 - ii) + (nj - 1 - jj);
                    T sc = T(0);
                    if (ii < ni - 1) sc = sCr[ii][jj][rlane] * sY[(step + 1) & 1][ii + 1 < kPc2I ? ii + 1 : ii][lane];
                    if (jj < kPc2J - 1) sc = fma(lane_reverse(ctm[jj < kPc2J - 1 ? jj + 1 : jj], raddr), zrow, sc);
                    const T di = lane_reverse(dinv[jj], raddr);
                    zrow = affine_scan(lane_reverse(cp[jj], raddr) * di, fma(sc, di, lane_reverse(y[jj], raddr)));
                    sY[step & 1][ii][lane] = zrow;
                    __syncthreads();
                    bst<T, 1>(Rz, (zoff == kOOB) ? kOOB : zoff + (uint32_t)(jj * dm.np) * ES, VecT<T, 1>{{zrow}});
                }
            }
            for (int t = 0; t < ii; ++t) __syncthreads();
        } else {
            for (int t = 0; t < ni + nj - 1; ++t) __syncthreads();
        }
        // ---- the block's sums
        rz = wave_sum(rz);
        rw = wave_sum(rw);
        if (lane == 0) {
            sRed[ii][0] = rz;
            sRed[ii][1] = rw;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            double v = 0.0;
            for (int u = 0; u < ni; ++u) v += sRed[u][threadIdx.x];
            st_agent(a.partials + (int64_t)(2 * h + threadIdx.x) * nblk + blk, v);
        }
        if (h + 1 < NR) __syncthreads();
    }
    // the finalize, by the block that finishes last; thread c takes right-hand
    // side c
    if (!last_block(a.count, (uint32_t)nblk, blockIdx.x)) return;
    __shared__ double sSum[kPc2I * 2 * NR];
    double S[2 * NR];
    sum_partials<kPc2Threads, 2 * NR>(a.partials, nblk, S, sSum);
    const int c = threadIdx.x;
    if (c < NR && a.ctl[c].flag == FLAG_RUN) {
        double rz = S[0], rw = S[1];
#pragma unroll
        for (int h = 1; h < NR; ++h) {
            rz = (c == h) ? S[2 * h] : rz;
            rw = (c == h) ? S[2 * h + 1] : rw;
        }
        pc2_beta(a.ctl + c, rz, rw, !upd);
        report_ctl(a.rep, c, a.ctl + c);
    }
}

// After a PC2 run: x moves in every second direction launch only, two updates
// at a time (IterArgs::xstep: launches 2, 4, ... of a run, each bringing x up
// to the direction before its own), so T finished iterations leave one or two
// updates (none after a breakdown found by such a launch), made here in the
// same order with the same fused multiply-adds.  p of iteration t (0-based)
// is in p[(iter0 + t + 1) & 1]; alpha is the last iteration's, alpha_prev the
// one's before.  blockIdx.y is the right-hand side.
template <typename T>
__global__ __launch_bounds__(256) void k_pc2_catchup(CatchupArgs<T> a) {
    const int c = blockIdx.y;
    const Ctl *ctl = a.ctl + c;
    const int ran = ctl->launches;  // direction launches that did work
    const int last = (ctl->flag == FLAG_RUN) ? ctl->iter : ctl->conv_iter;
    const int T_ = last - a.iter0;             // finished iterations
    const int done = ((ran - 1) / 2) * 2;      // updates made by the launches
    T *x = a.x[c];
    if (ran < 1 || T_ <= done || !x) return;
    const bool two = T_ - done == 2;
    const T a1 = (T)ctl->alpha, a0 = (T)ctl->alpha_prev;
    const T *p1 = a.p[c][(a.iter0 + T_) & 1], *p0 = a.p[c][(a.iter0 + T_ + 1) & 1];
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * 256) {
        T v = x[i];
        if (two) v = v + a0 * p0[i];
        x[i] = v + a1 * p1[i];
    }
}

}  // namespace mas
