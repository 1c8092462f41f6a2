// FV-subgrid multigrid kernels (paper Sec. "Multigrid preconditioner for
// finite volume approximations" and "Smoother / Pseudo time iteration").
//
// f_low on level l is the DG scheme with k = 0 on the subgrid: HLLC on the face
// total states (cell value + Ubar at the face), the k = 0 interior-penalty
// diffusion flux with penalty 1/h, and the gravity source.  The kernels carry
// the flux sum without the constant background-flux term, and each face's
// normal-momentum flux without the face's background pressure pb (the HLLC flux
// is affine in the pressure: F = F' + pb e_D, F' computed from p - pb); every
// use is a difference f(u + eps x) - f(u), in which those state-independent
// terms cancel, and the difference then loses digits only at the scale of
// p - pb and of the other fluxes, not at that of pb (about 10^5 Pa).
//
// Layout: SoA [4][nzl][nxl].  A work-group of the operator kernels is a tile of
// cells (six shapes, below) whose states go to LDS with a halo of one cell; each
// face of the tile gets its flux once.  The streaming kernels take 64 x 4 tiles,
// one wave per row of 64 cells.  Every kernel that produces a vector the next FD
// product needs also produces its squared norm through a deterministic two-level
// reduction.
#include "jfmg_internal.h"

namespace jfmg {

constexpr int FV_SUM_MAX = 3072;   // partials that a consumer sums itself
constexpr int FV_TX = 64, FV_TZ = 4, FV_NTH = FV_TX * FV_TZ;

enum { FVM_LIN = 0, FVM_STAGE = 1, FVM_MATVEC = 2, FVM_DEFECT = 3, FVM_STAGE_PC = 4, FVM_STAGE_TINV = 5 };

// Tile shapes of the FV operator kernels (jfmg_tile; chosen per level, by
// jfmg_autotune or by default):
//   64x4 / 256 threads: one wave per row of 64 cells (loads of a component are
//         512-byte rows); own-cell operands loaded after the face loop and at most
//         128 VGPRs, so four waves fit per SIMD
//   64x8 / 512 threads: the same with fewer halo faces per cell (2.14 vs 2.27)
//   16x4 / 256 threads: more threads than cells, so every face of the tile gets
//         its own thread (latency-bound narrow levels)
//   8x4 / 128 threads: the same with a quarter of the work per work-group
//   32x4 / 256 threads: two threads per cell (x-faces on the first threads,
//         z-faces from the last down), two waves per SIMD
//   64x4 / 512 threads: the 64x4 tile with two threads per cell (twice the waves
//         of the 256-thread form on a level too small to fill the chip)
// z-faces are handed out from the last thread down, so that the threads with a
// second x-face are not those with a second z-face.  Default: fv_default_tile.

// HLLC flux (Toro) for the normal +e_D without the face's background pressure (the
// pressures less pb enter wherever the pressure is added; see the file comment), Davis wave
// speeds.  On the side K of the contact: F_0 = rho*_K S*, F_D = F_0 S* + p*_K,
// F_c = (U_c / rho)_K F_0, rho*_K = rho_K (S_K - q_K) / (S_K - S*),
// p*_K = p_K + rho_K (S_K - q_K)(S* - q_K); S* = q_K in the supersonic cases turns the same
// expressions into the physical flux.  18 operations fewer than the S*-factored form
// (S*(S_K U_K - F_K) + S_K p*_K e_D) / (S_K - S*).  In FP32, where the pressure can round to
// zero and S_K - q_K = c with it, the supersonic rho*_K is rho_K itself instead of 0/0 (in
// FP64 the root of a zero pressure is no number, which the wave speeds leave out).
template <typename T, int D>
__device__ __forceinline__ void fv_hllc(const Gas<T>& G, const T (&UL)[4], const T (&UR)[4], T pL, T pR, T dpL, T dpR,
                                        T irL, T irR, T (&F)[4])
{
    constexpr int E = 3 - D;   // tangential momentum
    const T qL = UL[D] * irL, qR = UR[D] * irR;
    const T cL = psqrt<T>(G.gamma * pL * irL), cR = psqrt<T>(G.gamma * pR * irR);
    const T SL = fmin(qL - cL, qR - cR);
    const T SR = fmax(qL + cL, qR + cR);
    const T mL = UL[0] * (SL - qL), mR = UR[0] * (SR - qR);
    const T Ss = (dpR - dpL + qL * mL - qR * mR) * frcp<T>(mL - mR);
    const bool supL = SL >= T(0), supR = SR <= T(0);
    const bool lk = supL | (!supR & (Ss >= T(0)));
    const T SK = lk ? SL : SR, mK = lk ? mL : mR, qK = lk ? qL : qR, dpK = lk ? dpL : dpR;
    const T uE = lk ? UL[E] * irL : UR[E] * irR, u3 = lk ? UL[3] * irL : UR[3] * irR;
    const bool sup = supL | supR;
    const T S = sup ? qK : Ss;
    if constexpr (std::is_same_v<T, float>) {
        const T rK = lk ? UL[0] : UR[0];
        F[0] = (sup ? rK : mK * frcp<T>(SK - Ss)) * S;
    } else {
        F[0] = mK * frcp<T>(SK - S) * S;
    }
    F[D] = F[0] * S + (dpK + mK * (S - qK));
    F[E] = uE * F[0];
    F[3] = u3 * F[0];
}

// Net flux through one face (HLLC minus the k = 0 interior-penalty diffusion flux, along +x,
// D = 1, or +z, D = 2) from the staged states of its low and high cell.  bg: the face's
// background Ubar, p, 1/(rho theta), dbg (z-faces) its derivative.  A slip wall's missing
// state is a copy of the inside cell (wallL, wallR: the low, the high side's), whose normal
// momentum is negated here.
template <typename T, int D>
__device__ __forceinline__ void fv_flux(const FvArgs<T>& A, const T (&wL)[4], const T (&wR)[4], const T* bg, const T* dbg,
                                        bool wallL, bool wallR, T (&Phi)[4])
{
    T UL[4], UR[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        UL[c] = wL[c] + bg[c];
        UR[c] = wR[c] + bg[c];
    }
    UL[D] = wallL ? -UL[D] : UL[D];
    UR[D] = wallR ? -UR[D] : UR[D];
    const T pb = bg[4], irb = bg[5];
    const T rt[2] = {wL[3], wR[3]}, ir2[2] = {irb, irb}, pb2[2] = {pb, pb};
    T dp[2];
    pert_pressures<T, 2, true>(A.gas, rt, ir2, pb2, dp);
    const T irL = frcp<T>(UL[0]), irR = frcp<T>(UR[0]);
    fv_hllc<T, D>(A.gas, UL, UR, pb + dp[0], pb + dp[1], dp[0], dp[1], irL, irR, Phi);
    if (A.physics == 1) {
        // k = 0 diffusion: mean of mu (G_c - (U_c/rho) G_rho) over both sides, where the
        // only gradient is the background's (z-faces), minus the interior penalty
        // (mu/h) (dw_c - (U_c/rho)_avg dw_rho), dw = w_L - w_R, on the averaged state;
        // none through a wall
        const T mu = (wallL | wallR) ? T(0) : A.mu;
        const T muh = mu / (D == 1 ? A.hx : A.hz);
        const T irs = frcp<T>(UL[0] + UR[0]);
        const T dw0 = (wL[0] - wR[0]) * irs;
        const T hg0 = D == 1 ? T(0) : T(0.5) * mu * dbg[0];
#pragma unroll
        for (int c = 1; c < 4; ++c) {
            if constexpr (D == 2) Phi[c] += hg0 * (UL[c] * irL + UR[c] * irR) - mu * dbg[c];
            Phi[c] += muh * ((wL[c] - wR[c]) - (UL[c] + UR[c]) * dw0);
        }
    }
}

// The flux through face idx of a tile's x-faces (XF: the low faces of the cells row by row,
// then the last column's high faces) or z-faces (row by row).  Beyond a wall the halo holds a
// copy of the inside cell (and beyond the domain's last cells the tile copies of them), so
// that faces outside the domain, which no cell reads, compute with finite values instead of
// behind a branch.
template <typename T, int TX, int TZ, int HZ, int HX, bool XF>
__device__ __forceinline__ void fv_face(const FvArgs<T>& A, const T (&sw)[4][HZ][HX], const T (&sBc)[TZ][6],
                                        const T (&sBf)[TZ + 1][10], T (&sFx)[TZ][TX + 1][4], T (&sFz)[TZ + 1][TX][4],
                                        int I0, int J0, int nxl, int nzl, bool per, int idx)
{
    // tile row (the face's background row) and column
    const int r = XF && idx >= TX * TZ ? idx - TX * TZ : idx / TX;
    const int x = XF && idx >= TX * TZ ? TX : idx % TX;
    const bool wallL = XF ? !per && I0 + x == 0 : J0 + r == 0;
    const bool wallR = XF ? !per && I0 + x == nxl : J0 + r == nzl;
    T wL[4], wR[4], Phi[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        wL[c] = sw[c][XF ? r + 1 : r][XF ? x : x + 1];
        wR[c] = sw[c][r + 1][x + 1];
    }
    fv_flux<T, XF ? 1 : 2>(A, wL, wR, XF ? &sBc[XF ? r : 0][0] : &sBf[r][0], &sBf[XF ? 0 : r][6], wallL, wallR, Phi);
    T* F = XF ? &sFx[XF ? r : 0][x][0] : &sFz[r][XF ? 0 : x][0];
#pragma unroll
    for (int c = 0; c < 4; ++c) F[c] = Phi[c];
}

// FV operator on one tile of TX x TZ cells, face-centric: the perturbed states
// w = u + eps x of the tile and a one-cell halo are staged in LDS, every face
// of the tile gets its net flux Phi (HLLC minus the interior-penalty diffusion
// flux, along +x or +z) exactly once, and each cell then sums its four faces:
//   f~ = -(Phi_{I+1/2} - Phi_{I-1/2}) / hx - (Phi_{J+1/2} - Phi_{J-1/2}) / hz - g w_rho.
// The flux through a face seen from the other cell is the same number with
// the opposite sign (HLLC(L,R;n) = -HLLC(R,L;-n)).
// On the small levels a launch is one chain of latencies: of the 11300 cycles that a
// wave of the 8 x 4 tile lived, 3600 went by before its last load was issued (scalar
// loads of the level's scalars and of the arguments, each waited for in turn, and loads
// behind branches) and 2200 until the partial sums were there.  The kernel now fetches
// its arguments at once, reads the scalars by vector loads, and issues every load before
// it waits for the first, without a branch in between (a wait behind branches is one for
// all loads).  FGMRES iteration of 64 x 32 elements, k = 2: 135 -> 123 us; of the density
// current 216 -> 210 us.
// On the large levels the vector instructions bound it (56 to 75 % of the time): 856 per
// wave in FP32 and 934 in FP64 on the 64x8 tile before, 703 and 831 with a wall's ghost
// state in the halo instead of behind selects, each thread's own cell staged from its own
// loads, 32-bit offsets, the shorter HLLC form and no branch around the faces: step of
// 1024x256 nodes 24.2 -> 23.2 ms, of 2048x1024 (FP32 multigrid) 131.5 -> 126.7 ms; another 76
// less with the faces handed out without a loop: 23.3 -> 22.7 and 118.1 -> 116.9 ms.  Modes:
//   LIN     out = F0 = f~(u); ||u + Ubar||^2 and max(|v| + c) block partials (the level
//           slots and dtau from them: fv_lin_finalize_kernel); with out2 also the next coarser
//           level's state R u
//   STAGE   out = x0 + alpha_j dtau (b - g'x), g'x = x - adt/eps (f~(u + eps x) - F0)
//   MATVEC  out = g'x
//   DEFECT  out(coarse) = R(g'x - b), 2x2 agglomeration inside the tile; with out2 also
//           the coarse level's first RK stage from zero, out2 = alpha_j dtau_c out (dtau_c in
//           slots2), and its ||.||^2 block partials into red
//   STAGE_PC the STAGE result v is not stored: it corrects the next finer level's x in
//           out2 by injection, x_f -= P v (x_f = -P v when fzero is set, x_f being zero), with the
//           ||x_f||^2 block partials into red (the last smoother stage of a coarse level)
//   STAGE_TINV (finest level, tiles of whole DG elements) the STAGE result v is not stored:
//           the tile's elements are transferred back to the DG space, tv.z = T^-1 v with the
//           mass fix when tv.mass_fix is set (the arithmetic of transfer_Tinv_kernel), with the
//           ||z||^2 block partials into red (the last smoother stage of the cycle)
template <typename T, int TX, int TZ, int NTH, int WPE, bool LATE, bool ZREV, bool MB, int MODE, bool RG>
__global__ void __launch_bounds__(NTH, WPE)
fv_tile_kernel(FvArgs<T> Aa, const MemberArgs* __restrict__ mt, const T* __restrict__ u, const T* __restrict__ F0,
               const T* __restrict__ xp,
               const T* __restrict__ x0, const T* __restrict__ b, T* __restrict__ out, T* __restrict__ out2,
               const double* __restrict__ xpart, int xcount, double* __restrict__ slots,
               const double* __restrict__ slots2, double alpha_j, double adt, int fzero, Red red, long ms,
               TinvOut tv)
{
    const FvArgs<T>& A = fv_of<T, RG>(Aa, mt);
    // the arguments that the first loads need, in scalar registers at once (the compiler
    // would fetch them one by one where they are used, a trip to the kernel arguments each)
    gptr<T> u_ = (gptr<T>)u, F0_ = (gptr<T>)F0, xp_ = (gptr<T>)xp, x0_ = (gptr<T>)x0, b_ = (gptr<T>)b;
    gptr<T> rc_ = (gptr<T>)A.rc, rf_ = (gptr<T>)A.rf;
    gptr<double> xpart_ = (gptr<double>)xpart, slots_ = (gptr<double>)slots;
    int nxl = A.nxl, nzl = A.nzl;
    long nc = A.nc;
    asm volatile("" : "+s"(u_), "+s"(F0_), "+s"(xp_), "+s"(x0_), "+s"(b_), "+s"(xpart_), "+s"(xcount), "+s"(slots_),
                 "+s"(rc_), "+s"(rf_), "+s"(nxl), "+s"(nzl), "+s"(nc));
    u = (const T*)u_;
    F0 = (const T*)F0_;
    xp = (const T*)xp_;
    x0 = (const T*)x0_;
    b = (const T*)b_;
    xpart = (const double*)xpart_;
    const T *const rc = (const T*)rc_, *const rf = (const T*)rf_;
    const double* lslots = (const double*)slots_;
    if constexpr (MB) {   // member blockIdx.z of a lock-step batch
        u = mbr(u, ms);
        F0 = mbr(F0, ms);
        xp = mbr(xp, ms);
        x0 = mbr(x0, ms);
        b = mbr(b, ms);
        out = mbr(out, ms);
        out2 = mbr(out2, ms);
        slots2 = mbr(slots2, ms);
        xpart = mbr(xpart, ms);
        lslots = mbr(lslots, ms);
        red = mbr(red, ms);
    }
    double* const zout = MB ? mbr(tv.z, ms) : tv.z;   // STAGE_TINV output (tv stays in the arguments)
    constexpr int NCELL = TX * TZ, HX = TX + 2, HZ = TZ + 2;
    // halo cells that a face reads: the rows below and above the tile, the columns beside it
    constexpr int RING = 2 * TX + 2 * TZ;
    constexpr bool ONE = NTH >= NCELL + RING;   // one staged cell per thread
    static_assert(ONE || (NTH == NCELL && NTH >= 64 + RING), "halo staging");
    constexpr int NFX = TZ * (TX + 1), NFZ = (TZ + 1) * TX;
    constexpr bool PERT = (MODE != FVM_LIN);
    constexpr bool STG = (MODE == FVM_STAGE || MODE == FVM_STAGE_PC || MODE == FVM_STAGE_TINV);
    constexpr bool TI = (MODE == FVM_STAGE_TINV);
    static_assert(NTH >= NCELL && NTH % 64 == 0, "tile shape");
    __shared__ T sw[4][HZ][HX];
    __shared__ T sFx[TZ][TX + 1][4];
    __shared__ T sFz[TZ + 1][TX][4];
    // background of the tile's rows: cell centres [Ubar(4), p, 1/(rho theta)], z-faces
    // [Ubar(4), p, 1/(rho theta), dUbar/dz(4)]
    __shared__ T sBc[TZ][6];
    __shared__ T sBf[TZ + 1][10];
    // STAGE_TINV: V^-1, the Newton-Cotes weights and the first contraction of T^-1
    __shared__ double sVi[TI ? MAXN1 : 1][MAXN1], sWn[TI ? MAXN1 : 1];
    __shared__ double sHt[TI ? 4 : 1][TI ? TZ : 1][TI ? TX : 1];
    const int tid = threadIdx.x;
    // tiles of this member (a one-dimensional grid; in a ragged batch the work-groups
    // beyond a smaller member's tiles only store zero partial sums)
    const unsigned ntx = (unsigned)((nxl + TX - 1) / TX), ntiles = ntx * (unsigned)((nzl + TZ - 1) / TZ);
    if (blockIdx.x >= ntiles || (RG && sits_out(mt))) {
        if (tid == 0) {
            if constexpr (MODE == FVM_LIN) {
                red.partials[blockIdx.x] = 0.0;
                red.partials[gridDim.x + blockIdx.x] = 0.0;
            } else if constexpr (STG) {
                red.partials[blockIdx.x] = 0.0;
            } else if constexpr (MODE == FVM_DEFECT) {
                if (out2) red.partials[blockIdx.x] = 0.0;
            }
        }
        return;
    }
    const unsigned tile = xcd_tile(blockIdx.x, ntiles);
    const int I0 = (int)(tile % ntx) * TX, J0 = (int)(tile / ntx) * TZ;
    // own cell (threads tid < NCELL)
    const int ti = tid % TX, tj = tid / TX;
    const int I = I0 + ti, J = J0 + tj;
    const bool cell = NTH == NCELL || tid < NCELL;
    const bool valid = cell && I < nxl && J < nzl;
    // halo cell r (the last one beyond the list), tile coordinates
    const bool per = A.bc == 1;
    auto ring_cell = [&](int r, int& i, int& j) {
        const int s = r - 2 * TX;
        j = r < TX ? -1 : s < 0 ? TZ : s & (TZ - 1);
        i = s < 0 ? r & (TX - 1) : s < TZ ? -1 : TX;
    };
    static_assert((TX & (TX - 1)) == 0 && (TZ & (TZ - 1)) == 0, "halo staging");
    // index of the cell at tile coordinates (i, j): beyond the domain the wrapped-round
    // column (x-periodic) or the nearest cell
    const int below = per ? nxl - 1 : 0, beyond = per ? 0 : nxl - 1;
    auto cell_index = [&](int i, int j) {
        const int Ig = I0 + i, Jg = min(max(J0 + j, 0), nzl - 1);
        return (unsigned)(Jg * nxl + (Ig < 0 ? below : Ig >= nxl ? beyond : Ig));
    };
    // this thread's staged cell, its own where it has one
    int si = ti, sj = tj;
    if constexpr (ONE)
        if (!cell) ring_cell(min(tid - NCELL, RING - 1), si, sj);
    const unsigned qs = cell_index(si, sj);
    const unsigned q = ONE ? (cell ? qs : 0u) : qs;

    // ---- every global load first (the ||x||^2 partials, the level's scalars and
    // background rows, the own-cell operands, then the halo states), or the own-cell
    // operands only after the face loop (LATE: fewer live registers).  Nothing below
    // waits on memory before the partial sums of ||x||^2 have arrived. ----
    PartialSum<NTH> xsum;
    double s_utot = 0.0, s_iutot = 0.0, s_dtau = 0.0;
    if constexpr (PERT) {
        xsum.load(xpart, xcount);
        s_utot = ldv(lslots + LV_UTOT);
        s_iutot = ldv(lslots + LV_IUTOT);
    }
    if constexpr (STG) s_dtau = ldv(lslots + LV_DTAU);
    if constexpr (MODE == FVM_DEFECT) s_dtau = out2 ? ldv(slots2 + LV_DTAU) : 0.0;
    static_assert(NTH >= 6 * TZ + 10 * (TZ + 1), "background staging");
    // this thread's entry of sBc / sBf: the tile's rows are contiguous in the level's records
    const bool bg_c = tid < 6 * TZ;
    const int bg_i = bg_c ? tid : tid - 6 * TZ;
    const bool bg_ok = bg_c || bg_i < 10 * (TZ + 1);
    // (rows beyond the level's last: the tile's first row)
    const int bg_j = bg_c ? (bg_i < 6 * (nzl - J0) ? bg_i : bg_i % 6)
                          : (bg_i < 10 * min(TZ + 1, nzl + 1 - J0) ? bg_i : bg_i % 10);
    const T* const bg_p = bg_c ? rc + 6L * J0 : rf + 10L * J0;
    const T bg_v = bg_p[bg_j];
    T su[4], own_x[4], ru[4], rx[4];
    T own_f0[4], own_b[4], own_x0[4] = {T(0), T(0), T(0), T(0)};
    // STAGE_PC: the finer level's four children of the cell, read with the own-cell
    // operands (before any of them is written)
    T own_xf[4][4] = {};
    // (threads without a cell read a neighbouring one, or cell 0: loads behind a branch
    // would make the wait for the partial sums one for all loads)
    const unsigned nxf = 2u * (unsigned)nxl;
    const long ncf = 4 * nc;
    const unsigned q00 = MODE == FVM_STAGE_PC ? 4u * q - 2u * (q % (unsigned)nxl) : 0u;
    auto load_own = [&]() {
        if constexpr (MODE == FVM_STAGE_PC)
            if (!fzero) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const T* xf = out2 + c * ncf;
                    own_xf[c][0] = ld(xf, q00); own_xf[c][1] = ld(xf, q00 + 1);
                    own_xf[c][2] = ld(xf, q00 + nxf); own_xf[c][3] = ld(xf, q00 + nxf + 1);
                }
            }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if constexpr (PERT) own_f0[c] = ld(F0 + c * nc, q);
            if constexpr (STG || MODE == FVM_DEFECT) own_b[c] = ld(b + c * nc, q);
        }
        // the first stage of a sweep has x^(0) = x^(j-1): no second load (the copy
        // is taken where x^(0) is used, so that no load waits for another)
        if constexpr (STG)
            if (x0 && x0 != xp)
#pragma unroll
                for (int c = 0; c < 4; ++c) own_x0[c] = ld(x0 + c * nc, q);
    };
    if constexpr (!LATE) load_own();
    auto load_cell = [&](unsigned qc, T (&cu)[4], T (&cx)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            cu[c] = ld(u + c * nc, qc);
            if constexpr (PERT) cx[c] = ld(xp + c * nc, qc);
        }
    };
    load_cell(qs, su, own_x);
    // the halo cells of a tile with a cell for each thread: by waves 1 and up (wave 0 has
    // the x-faces beyond one per thread)
    const bool ring = !ONE && tid >= 64 && tid < 64 + RING;
    int ri = 0, rj = 0;
    if constexpr (!ONE)
        if (ring) {
            ring_cell(tid - 64, ri, rj);
            load_cell(cell_index(ri, rj), ru, rx);
        }
    // eps = sqrt(eps_p) ||u + Ubar|| / ||x|| and adt / eps, from ||x|| and the stored 1/||u + Ubar||
    T eps = T(0), sc = T(0);
    bool xzero = false;   // uniform: g'x = 0 for x = 0
    if constexpr (PERT) {
        // ||x||^2, same order in every block.  The FP64 64x4 tile that transfers back exchanges it
        // through the x-fluxes' array (the barrier behind the staged states comes before the first
        // flux): with 2 KB of its own for it, three of its work-groups would fit a CU, not four.
        constexpr bool LEND = TI && sizeof(T) == 8 && NTH == 256 && NCELL == NTH;
        double xn2;
        if constexpr (LEND) xn2 = xsum.sum(xpart, xcount, reinterpret_cast<double*>(&sFx[0][0][0]));
        else xn2 = xsum.sum(xpart, xcount);
        if (!(xn2 > 0.0)) {
            xzero = true;
        } else {
            const double xn = psqrt(xn2);
            eps = (T)(FdEps<T>::sqrt_eps * s_utot * frcp(xn));
            sc = (T)(adt * xn * (FdEps<T>::inv_sqrt_eps * s_iutot));
        }
    }

    if (!xzero) {
        auto stage = [&](int i, int j, const T (&cu)[4], const T (&cx)[4]) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                T v = cu[c];
                if constexpr (PERT) v = v + eps * cx[c];
                sw[c][j + 1][i + 1] = v;
            }
        };
        stage(si, sj, su, own_x);   // (threads beyond the halo's last cell: that cell again)
        if (ring) stage(ri, rj, ru, rx);
        if (bg_ok) (bg_c ? &sBc[0][0] : &sBf[0][0])[bg_i] = bg_v;
        if constexpr (TI) {
            if (tid < MAXN1 * MAXN1) sVi[tid / MAXN1][tid % MAXN1] = tv.Vinv[tid / MAXN1][tid % MAXN1];
            else if (tid < MAXN1 * MAXN1 + MAXN1) sWn[tid - MAXN1 * MAXN1] = tv.wnc[tid - MAXN1 * MAXN1];
        }
        __syncthreads();
        // ---- one net flux per face: x-faces in thread order, z-faces in reverse
        // thread order (the threads with a second x-face are not those with a
        // second z-face) ----
        auto face = [&](auto xf_tag, int idx) {
            fv_face<T, TX, TZ, HZ, HX, decltype(xf_tag)::value>(A, sw, sBc, sBf, sFx, sFz, I0, J0, nxl, nzl, per, idx);
        };
        // (not loops: the constants of the general power, the rare branch of the pressures,
        // would be set up before each of them, 38 moves and as many registers)
#pragma unroll
        for (int k = 0; k < (NFX + NTH - 1) / NTH; ++k)
            if (NFX >= (k + 1) * NTH || tid < NFX - k * NTH) face(std::true_type{}, tid + k * NTH);
        const int tz = ZREV ? NTH - 1 - tid                          // z-faces from the last thread down
                            : (tid + NTH - NFX % NTH) % NTH;         // or numbered on after the x-faces
#pragma unroll
        for (int k = 0; k < (NFZ + NTH - 1) / NTH; ++k)
            if (NFZ >= (k + 1) * NTH || tz < NFZ - k * NTH) face(std::false_type{}, tz + k * NTH);
        if constexpr (LATE) load_own();
        __syncthreads();
    } else {
        if constexpr (TI) {
            if (tid < MAXN1 * MAXN1) sVi[tid / MAXN1][tid % MAXN1] = tv.Vinv[tid / MAXN1][tid % MAXN1];
            else if (tid < MAXN1 * MAXN1 + MAXN1) sWn[tid - MAXN1 * MAXN1] = tv.wnc[tid - MAXN1 * MAXN1];
        }
        if constexpr (LATE) load_own();
    }

    // ---- per cell ----
    T f[4] = {T(0), T(0), T(0), T(0)};
    if (cell && !xzero) {
        const T ihx = A.hz * A.iarea, ihz = A.hx * A.iarea;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f[c] = -(sFx[tj][ti + 1][c] - sFx[tj][ti][c]) * ihx - (sFz[tj + 1][ti][c] - sFz[tj][ti][c]) * ihz;
            if (c == 2) f[c] -= A.g * sw[0][tj + 1][ti + 1];
        }
    }
    if constexpr (MODE == FVM_LIN) {
        // with out2: the next coarser level's state R u from the staged tile (the 2 x 2
        // means of fv_restrict_kernel, in its order)
        if (out2 && valid && !(ti & 1) && !(tj & 1)) {
            const int nxc = nxl / 2;
            const long ncc = (long)nxc * (nzl / 2), qc = (long)(J / 2) * nxc + I / 2;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                out2[c * ncc + qc] =
                    ((sw[c][tj + 1][ti + 1] + sw[c][tj + 1][ti + 2]) + (sw[c][tj + 2][ti + 1] + sw[c][tj + 2][ti + 2])) * T(0.25);
        }
        double ss = 0.0, lam = 0.0;
        if (valid) {
            T Ut[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                st(out + c * nc, q, f[c]);   // F0
                Ut[c] = su[c] + sBc[tj][c];
                ss += (double)Ut[c] * (double)Ut[c];
            }
            const double rho = Ut[0], uu = Ut[1] / rho, ww = Ut[2] / rho;
            const double p = (double)A.gas.p0 * pow((double)A.gas.R * (double)Ut[3] / (double)A.gas.p0,
                                                    (double)A.gas.gamma);
            lam = sqrt(uu * uu + ww * ww) + sqrt((double)A.gas.gamma * p / rho);
        }
        __shared__ double sh[NTH / 64];
        const double bs = block_sum<NTH>(ss, sh);
        const double bm = block_max<NTH>(lam, sh);
        if (tid == 0) {
            red.partials[blockIdx.x] = bs;
            red.partials[gridDim.x + blockIdx.x] = bm;
        }
        return;
    } else {
        T Ax[4] = {T(0), T(0), T(0), T(0)};
        if (cell && !xzero) {
#pragma unroll
            for (int c = 0; c < 4; ++c) Ax[c] = own_x[c] - sc * (f[c] - own_f0[c]);
        }
        if constexpr (MODE == FVM_MATVEC) {
            if (valid)
#pragma unroll
                for (int c = 0; c < 4; ++c) st(out + c * nc, q, Ax[c]);
        } else if constexpr (MODE == FVM_STAGE) {
            double nrm = 0.0;
            if (valid) {
                const T s = (T)(alpha_j * s_dtau);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const T v = (x0 == xp ? own_x[c] : own_x0[c]) + s * (own_b[c] - Ax[c]);
                    st(out + c * nc, q, v);
                    nrm += (double)v * (double)v;
                }
            }
            put_partial<NTH>(red, nrm);
        } else if constexpr (MODE == FVM_STAGE_PC) {
            double nrm = 0.0;
            if (valid) {
                const T s = (T)(alpha_j * s_dtau);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const T v = (x0 == xp ? own_x[c] : own_x0[c]) + s * (own_b[c] - Ax[c]);
                    T* xf = out2 + c * ncf;
                    T f00 = -v, f01 = -v, f10 = -v, f11 = -v;
                    if (!fzero) {
                        f00 = own_xf[c][0] - v; f01 = own_xf[c][1] - v;
                        f10 = own_xf[c][2] - v; f11 = own_xf[c][3] - v;
                    }
                    st(xf, q00, f00); st(xf, q00 + 1, f01);
                    st(xf, q00 + nxf, f10); st(xf, q00 + nxf + 1, f11);
                    nrm += ((double)f00 * (double)f00 + (double)f01 * (double)f01) +
                           ((double)f10 * (double)f10 + (double)f11 * (double)f11);
                }
            }
            put_partial<NTH>(red, nrm);
        } else if constexpr (MODE == FVM_STAGE_TINV) {
            T v[4] = {T(0), T(0), T(0), T(0)};
            if (valid) {
                const T s = (T)(alpha_j * s_dtau);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = (x0 == xp ? own_x[c] : own_x0[c]) + s * (own_b[c] - Ax[c]);
            }
            __syncthreads();   // the staged states are read no more: the tile of v replaces them
            if (valid)
#pragma unroll
                for (int c = 0; c < 4; ++c) sw[c][tj][ti] = v[c];
            __syncthreads();
            // T^-1 with k + 1 = N1 known at compile time (tiles of whole elements: N1 = 2 or 4)
            double nrm = 0.0;
            auto tinv = [&](auto n1c) {
                constexpr int N1 = decltype(n1c)::value, NP = N1 * N1;
                // first contraction, one thread per subcell (a, bb) of its element:
                // h_{bb,a} = sum_i Vinv_ai t_{i,bb}
                // the element sums of the mass fix (mean and Newton-Cotes quadrature of each
                // component, each in the order of transfer_Tinv_kernel) in the flux rows, which
                // the cell sums have finished reading: one (sum, component) pair per thread
                constexpr int NEX = TX / N1, NEL = NEX * (TZ / N1);
                static_assert(8 * NEL * sizeof(double) <= sizeof(sFz), "element sums");
                double* const sSum = reinterpret_cast<double*>(&sFz[0][0][0]);   // [8][NEL]
                if (valid) {
                    const int a = ti % N1, ea = ti - a, b1 = tj % N1, eb = tj - b1;
                    double va[N1];
#pragma unroll
                    for (int ii = 0; ii < N1; ++ii) va[ii] = sVi[a][ii];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        double s = 0.0;
#pragma unroll
                        for (int ii = 0; ii < N1; ++ii) s += va[ii] * (double)sw[c][tj][ea + ii];
                        sHt[c][tj][ti] = s;
                    }
                    if (tv.mass_fix) {
                        const int el = (eb / N1) * NEX + ea / N1;
                        for (int qs = b1 * N1 + a; qs < 8; qs += NP) {
                            const int c = qs & 3;
                            double acc = 0.0;
                            if (qs < 4) {
#pragma unroll
                                for (int jj = 0; jj < N1; ++jj)
#pragma unroll
                                    for (int ii = 0; ii < N1; ++ii) acc += (double)sw[c][eb + jj][ea + ii];
                            } else {
#pragma unroll
                                for (int jj = 0; jj < N1; ++jj)
#pragma unroll
                                    for (int ii = 0; ii < N1; ++ii) {
                                        const double w = sw[c][eb + jj][ea + ii];
                                        acc += sWn[ii] * sWn[jj] * w;
                                    }
                            }
                            sSum[qs * NEL + el] = acc;
                        }
                    }
                }
                __syncthreads();
                // second contraction and mass fix, one thread per DG node in the order of the
                // DG vector (the tile's elements of one element row are consecutive there)
                constexpr int ROW = TX * N1;   // nodes of one element row of the tile
                if (tid < NCELL) {
                    const int er = tid / ROW, rem = tid - er * ROW, el = rem / NP, nd = rem - el * NP;
                    const int a = nd % N1, bb = nd / N1, ea = el * N1, eb = er * N1;
                    if (I0 + ea < nxl && J0 + eb < nzl) {
                        const long e = (long)((J0 + eb) / N1) * (nxl / N1) + (I0 + ea) / N1;
                        double vb[N1];
#pragma unroll
                        for (int jj = 0; jj < N1; ++jj) vb[jj] = sVi[bb][jj];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            double s = 0.0;
#pragma unroll
                            for (int jj = 0; jj < N1; ++jj) s += vb[jj] * sHt[c][eb + jj][ea + a];
                            double shift = 0.0;
                            if (tv.mass_fix) {
                                const int el2 = er * NEX + el;
                                shift = sSum[(4 + c) * NEL + el2] - sSum[c * NEL + el2] / NP;
                            }
                            const double z = s - shift;
                            zout[c * nc + e * NP + nd] = z;   // the DG vector has nc nodes per component
                            nrm += z * z;
                        }
                    }
                }
            };
            if (tv.n1 == 4) tinv(std::integral_constant<int, 4>{});
            else tinv(std::integral_constant<int, 2>{});
            put_partial<NTH>(red, nrm);
        } else {   // DEFECT: reuse the state tile for d = g'x - b, then agglomerate 2x2
            __syncthreads();
            if (valid)
#pragma unroll
                for (int c = 0; c < 4; ++c) sw[c][tj][ti] = Ax[c] - own_b[c];
            __syncthreads();
            double nrm = 0.0;
            if (valid && !(ti & 1) && !(tj & 1)) {
                const int nxc = nxl / 2;
                const long ncc = (long)nxc * (nzl / 2), qc = (long)(J / 2) * nxc + I / 2;
                const T s1 = out2 ? (T)(alpha_j * s_dtau) : T(0);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const T r = ((sw[c][tj][ti] + sw[c][tj][ti + 1]) + (sw[c][tj + 1][ti] + sw[c][tj + 1][ti + 1])) * T(0.25);
                    out[c * ncc + qc] = r;
                    if (out2) {
                        const T v = s1 * r;
                        out2[c * ncc + qc] = v;
                        nrm += (double)v * (double)v;
                    }
                }
            }
            if (out2) put_partial<NTH>(red, nrm);
        }
    }
}

// The coarsest levels of a V-cycle in one launch, one work-group per member: pre-smoothing,
// defect, the coarser levels and post-smoothing of at most TAIL_LEV levels, and the correction
// of the next finer level's x with its ||x_f||^2 partials.  On such a level a launch is one
// chain of latencies, 4.3 us whatever its size and the gap to the next one; here a stage is
// three barriers of one work-group, and states, right-hand sides and fluxes stay in LDS.  One
// thread per face, one per cell in the order of the 8x4 tiles' threads (half a wave per tile);
// the arithmetic and the order of every sum are those of the 8x4 tile kernels, so that it does
// not matter to the bits which of the two a level takes.  On entry the top level's first stage
// from x = 0 has its ||x||^2 partials at xpart (written with b by the producer).
// FP64, 16x16 and 8x8 cells, three stages: 56 us for the 24 launches' 104 (implicit Euler step
// of that problem 12.6 -> 8.9 ms); FP32, 24x12 cells, one stage: 11.5 us for 13 of three
// launches, without their gaps (step 15.8 -> 14.9 ms).  Halo cells written behind branches
// (a face knows its two cells instead) and one load waited for at a time made it 62 and 12.4.
template <typename T, bool RG>
__global__ void __launch_bounds__(TAIL_NTH)
fv_tail_kernel(const TailArgs<T> a, const MemberArgs* __restrict__ mt, long ms)
{
    __shared__ T sw[4 * TAIL_CELLS];            // staged states, or defects, [component][cell]
    __shared__ T sF[4][TAIL_NTH];               // fluxes, by thread
    __shared__ T sV[16 * TAIL_SUM];             // per level [u, F0, b, x][component][cell]
    __shared__ T sBc[2 * TAIL_ROWS][6], sBf[2 * TAIL_ROWS + TAIL_LEV][10];   // the levels' background rows
    __shared__ double sS[TAIL_LEV][4], part[32];
    const int tid = threadIdx.x, lane = tid & 63;
    const Red red = mbr(a.red, ms);
    if (RG && sits_out(mt)) {
        if (tid < a.nparts) red.partials[tid] = 0.0;
        return;
    }
    const double* const xpart = mbr(a.xpart, ms);
    PartialSum<128> xsum;
    xsum.load(xpart, a.xcount);
    // The arguments of the top level; the coarser ones' differ by powers of two only.
    FvArgs<T> A;
    if constexpr (RG) A = fv_entry<T>(mt, a.lev0);
    else A = a.A;
    const T top_hx = A.hx, top_hz = A.hz, top_ia = A.iarea;
    const bool per = A.bc == 1;
    // everything that the levels need from memory, every load before the first store
    {
        static_assert(4 * TAIL_CELLS <= 2 * TAIL_NTH && 10 * (TAIL_ROWS + 1) <= 2 * TAIL_NTH, "staging");
        T ru[TAIL_LEV][2], rF[TAIL_LEV][2], rb[2], rrc[TAIL_LEV], rrf[TAIL_LEV][2];
        double rs = 0.0;
        const T* b = (const T*)(gptr<T>)mbr(a.b, ms);
        auto fetch = [&](const T* p, int i, int n) { return p[i < n ? i : 0]; };
#pragma unroll
        for (int l = 0; l < TAIL_LEV; ++l) {
            const int m = l < a.n ? l : 0;   // (a level that is not there: the first one's, not stored)
            const int nz = A.nzl >> m, n4 = 4 * (A.nxl >> m) * nz;
            const T *rc = a.rc[m], *rf = a.rf[m];
            if constexpr (RG) {
                rc = fv_entry<T>(mt, a.lev0 + m).rc;
                rf = fv_entry<T>(mt, a.lev0 + m).rf;
            }
            rc = (const T*)(gptr<T>)rc;
            rf = (const T*)(gptr<T>)rf;
            const T *u = (const T*)(gptr<T>)mbr(a.u[m], ms), *F0 = (const T*)(gptr<T>)mbr(a.F0[m], ms);
#pragma unroll
            for (int k = 0; k < (l == 0 ? 2 : 1); ++k) {
                const int i = tid + k * TAIL_NTH;
                ru[l][k] = fetch(u, i, n4);
                rF[l][k] = fetch(F0, i, n4);
                if (l == 0) rb[k] = fetch(b, i, n4);
                rrf[l][k] = fetch(rf, i, 10 * (nz + 1));
            }
            rrc[l] = fetch(rc, tid, 6 * nz);
        }
        if (tid < 4 * a.n) rs = mbr(a.slots, ms)[tid];
        int o = 0, oc = 0, of = 0;
#pragma unroll
        for (int l = 0; l < TAIL_LEV; ++l) {
            if (l < a.n) {
                const int nz = A.nzl >> l, n4 = 4 * (A.nxl >> l) * nz;
#pragma unroll
                for (int k = 0; k < (l == 0 ? 2 : 1); ++k) {
                    const int i = tid + k * TAIL_NTH;
                    if (i < n4) {
                        sV[o + i] = ru[l][k];
                        sV[o + n4 + i] = rF[l][k];
                        if (l == 0) sV[o + 2 * n4 + i] = rb[k];
                    }
                    if (i < 10 * (nz + 1)) (&sBf[of][0])[i] = rrf[l][k];
                }
                if (tid < 6 * nz) (&sBc[oc][0])[tid] = rrc[l];
                o += 4 * n4;
                oc += nz;
                of += nz + 1;
            }
        }
        if (tid < 4 * a.n) (&sS[0][0])[tid] = rs;
    }
    // the level, and this thread's cell of it
    int nxl, nzl, nc, nt, I, J, q, off, oc, of, flo, fhi, frow, fx, fz;
    bool valid, xf, face, fwl, fwr;
    double utot, iutot, dtau;
    auto enter = [&](int l) __attribute__((always_inline)) {
        nxl = A.nxl >> l;
        nzl = A.nzl >> l;
        nc = nxl * nzl;
        off = oc = of = 0;
        for (int m = 0; m < l; ++m) {
            off += 16 * (A.nxl >> m) * (A.nzl >> m);
            oc += A.nzl >> m;
            of += (A.nzl >> m) + 1;
        }
        const T two = (T)(1 << l);
        A.hx = top_hx * two;
        A.hz = top_hz * two;
        A.iarea = top_ia * (T(1) / (two * two));
        const int ntx = (nxl + 7) / 8;
        nt = ntx * ((nzl + 3) / 4);
        const int g = tid >> 5, tile = g < nt ? (int)xcd_tile(g, nt) : 0;
        I = (tile % ntx) * 8 + (tid & 7);
        J = (tile / ntx) * 4 + ((tid >> 3) & 3);
        valid = g < nt && I < nxl && J < nzl;
        I = valid ? I : 0;
        J = valid ? J : 0;
        q = J * nxl + I;
        // this thread's face: x-faces from thread 0, z-faces from the next wave on
        const int nxf = (nxl + 1) * nzl, nxp = (nxf + 63) & ~63, nzf = nxl * (nzl + 1);
        xf = __builtin_amdgcn_readfirstlane(tid) < nxp;
        const int k = xf ? tid : tid - nxp, fw = xf ? nxl + 1 : nxl;
        const int r = k / fw, cc = k - r * fw;
        face = k < (xf ? nxf : nzf);
        // its low and high cell; beyond a wall the inside one (see fv_flux)
        const int e = per ? nxl - 1 : 0;   // x-periodic: the other end
        flo = xf ? r * nxl + (cc > 0 ? cc - 1 : e) : (r > 0 ? k - nxl : k);
        fhi = xf ? r * nxl + (cc < nxl ? cc : nxl - 1 - e) : (r < nzl ? k : k - nxl);
        frow = xf ? oc + r : of + r;
        fwl = xf ? !per && cc == 0 : r == 0;
        fwr = xf ? !per && cc == nxl : r == nzl;
        fx = J * (nxl + 1) + I;
        fz = nxp + q;
        utot = sS[l][LV_UTOT];
        iutot = sS[l][LV_IUTOT];
        dtau = sS[l][LV_DTAU];
    };
    auto vec = [&](int k, int c, int i) -> T& { return sV[off + (4 * k + c) * nc + i]; };   // k: 0 u, 1 F0, 2 b, 3 x
    // sum of v over the level's cells from the tiles' sums, every thread; a barrier inside
    auto tile_sums = [&](double v, double* out) {
        v += dpp_move<0x111, 0xf>(v);
        v += dpp_move<0x112, 0xf>(v);
        v += dpp_move<0x114, 0xf>(v);
        v += dpp_move<0x118, 0xf>(v);
        v += dpp_move<0x142, 0xa>(v);
        if ((tid & 31) == 31 && (tid >> 5) < nt) out[tid >> 5] = v;
    };
    auto total = [&](double v) {
        tile_sums(v, part);
        __syncthreads();
        return wave_sum(lane < nt ? part[lane] : 0.0);
    };
    // g'x of this thread's cell (the states staged in sw)
    T x[4], Ax[4], f0[4], b[4];   // (F0 and b read behind the face)
    auto apply = [&](double xn2) __attribute__((always_inline)) {
        if (!(xn2 > 0.0)) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                Ax[c] = T(0);
                b[c] = vec(2, c, q);
            }
            __syncthreads();
            return;
        }
        const double xn = psqrt(xn2);
        const T eps = (T)(FdEps<T>::sqrt_eps * utot * frcp(xn));
        const T sc = (T)(a.adt * xn * (FdEps<T>::inv_sqrt_eps * iutot));
        if (valid)
#pragma unroll
            for (int c = 0; c < 4; ++c) sw[c * nc + q] = vec(0, c, q) + eps * x[c];
        __syncthreads();
        if (face) {
            T wL[4], wR[4], Phi[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                wL[c] = sw[c * nc + flo];
                wR[c] = sw[c * nc + fhi];
            }
            if (xf) fv_flux<T, 1>(A, wL, wR, &sBc[frow][0], &sBf[0][6], fwl, fwr, Phi);
            else fv_flux<T, 2>(A, wL, wR, &sBf[frow][0], &sBf[frow][6], fwl, fwr, Phi);
#pragma unroll
            for (int c = 0; c < 4; ++c) sF[c][tid] = Phi[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f0[c] = vec(1, c, q);
            b[c] = vec(2, c, q);
        }
        __syncthreads();
        const T ihx = A.hz * A.iarea, ihz = A.hx * A.iarea;
        if (valid)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                T f = -(sF[c][fx + 1] - sF[c][fx]) * ihx - (sF[c][fz + nxl] - sF[c][fz]) * ihz;
                if (c == 2) f -= A.g * sw[q];
                Ax[c] = x[c] - sc * (f - f0[c]);
            }
    };
    int l = 0;
    const double xn2_0 = xsum.sum(xpart, a.xcount);
    __syncthreads();
    enter(0);
    double xn2 = xn2_0;
    T x0[4];   // at the sweep's start
    {
        const T s = (T)(a.alpha[0] * dtau);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            x[c] = s * vec(2, c, q);
            x0[c] = T(0);
        }
    }
    bool post = false;
    for (int sweep = 0, j = 1;;) {   // one product g'x per turn: of a stage, or of the defect after the pre-smoothing
        if (j == a.S) {
            ++sweep;
            j = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) x0[c] = x[c];
        }
        const bool done = !post && sweep == a.pre, defect = done && l < a.n - 1;
        if (done && !defect) {
            post = true;
            sweep = 0;
        }
        apply(xn2);
        if (defect) {
            // down: the coarse level's b = R(g'x - b) and its first stage from zero
            T d[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) d[c] = Ax[c] - b[c];
            __syncthreads();   // the staged states are read no more
            if (valid)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    vec(3, c, q) = x[c];
                    sw[c * nc + q] = d[c];
                }
            __syncthreads();
            const int fnx = nxl, fnc = nc;
            auto coarse = [&](int c, int o) {
                const T* p = sw + c * fnc + o;
                return ((p[0] + p[1]) + (p[fnx] + p[fnx + 1])) * T(0.25);
            };
            // the stage's norm as this level's tiles sum it
            const T s1 = (T)(a.alpha[0] * sS[l + 1][LV_DTAU]);
            double nrm = 0.0;
            if (valid && !(I & 1) && !(J & 1))
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const T v = s1 * coarse(c, q);
                    nrm += (double)v * (double)v;
                }
            xn2 = total(nrm);
            ++l;
            enter(l);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const T r = coarse(c, 2 * J * fnx + 2 * I);
                if (valid) vec(2, c, q) = r;
                x[c] = s1 * r;
                x0[c] = T(0);
            }
            sweep = 0;
            j = 1;
            __syncthreads();   // (the defects are read no more)
            continue;
        }
        const T s = (T)(a.alpha[j] * dtau);
        double nrm = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const T v = x0[c] + s * (b[c] - Ax[c]);
            x[c] = v;
            nrm += (double)v * (double)v;
        }
        ++j;
        if (!(post && sweep == a.post - 1 && j == a.S)) {
            xn2 = total(valid ? nrm : 0.0);
            continue;
        }
        // up: the last result corrects the finer level's x
        const int ncf = 4 * nc, nxf = 2 * nxl, q00 = 2 * J * nxf + 2 * I;
        nrm = 0.0;
        auto correct = [&](T* xf) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                T* p = xf + c * ncf + q00;
                const T v = x[c];
                const T f00 = p[0] - v, f01 = p[1] - v, f10 = p[nxf] - v, f11 = p[nxf + 1] - v;
                p[0] = f00; p[1] = f01;
                p[nxf] = f10; p[nxf + 1] = f11;
                nrm += ((double)f00 * (double)f00 + (double)f01 * (double)f01) +
                       ((double)f10 * (double)f10 + (double)f11 * (double)f11);
            }
        };
        if (l == 0) {
            if (valid) correct(mbr(a.xf, ms));
            tile_sums(nrm, red.partials);
            if (tid >= nt && tid < a.nparts) red.partials[tid] = 0.0;
            return;
        }
        if (valid) correct(sV + off - 4 * ncf);
        xn2 = total(nrm);
        --l;
        enter(l);
#pragma unroll
        for (int c = 0; c < 4; ++c) x0[c] = x[c] = vec(3, c, q);
        sweep = 0;
        j = 0;
    }
}

// The sum of n partials, in the order of a consumer of NTH threads, to p[n]: that entry alone
// gives the consumer the same bits.
template <int NTH>
__global__ void __launch_bounds__(NTH) fv_sum_kernel(double* __restrict__ p, int n, long ms)
{
    p = mbr(p, ms);
    PartialSum<NTH> x;
    x.load(p, n);
    const double s = x.sum(p, n);
    if (threadIdx.x == 0) p[n] = s;
}

// first stage of a sweep from x = 0: out = alpha_1 dtau b, with ||out||^2
template <typename T, bool RG>
__global__ void __launch_bounds__(256)
fv_stage_zero_kernel(FvArgs<T> Aa, const MemberArgs* __restrict__ mt, const T* __restrict__ b, T* __restrict__ out,
                     const double* __restrict__ slots, double alpha_j, Red red, long ms)
{
    const FvArgs<T>& A = fv_of<T, RG>(Aa, mt);
    b = mbr(b, ms);
    out = mbr(out, ms);
    slots = mbr(slots, ms);
    red = mbr(red, ms);
    const long n = sits_out(mt) ? 0 : 4 * A.nc;
    const long nb = (n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024;   // this member's work-groups
    const T s = (T)(alpha_j * slots[LV_DTAU]);
    double nrm = 0.0;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += nb * 256) {
        const T v = s * b[i];
        out[i] = v;
        nrm += (double)v * (double)v;
    }
    put_partial<256>(red, nrm);
}

// coarse = R(-b): the defect of x = 0
template <typename T, bool RG>
__global__ void __launch_bounds__(256)
fv_restrict_neg_kernel(FvArgs<T> Aa, const MemberArgs* __restrict__ mt, const T* __restrict__ f, T* __restrict__ c,
                       long ms)
{
    const FvArgs<T>& A = fv_of<T, RG>(Aa, mt);
    if (RG && sits_out(mt)) return;
    f = mbr(f, ms);
    c = mbr(c, ms);
    const int nxc = A.nxl / 2, nzc = A.nzl / 2;
    const int Ic = blockIdx.x * 64 + (threadIdx.x & 63);
    const int Jc = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (Ic >= nxc || Jc >= nzc) return;
    const long ncc = (long)nxc * nzc, qc = (long)Jc * nxc + Ic;
    const long q00 = (long)(2 * Jc) * A.nxl + 2 * Ic, q01 = q00 + A.nxl;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
        const T* g = f + cc * A.nc;
        c[cc * ncc + qc] = ((-g[q00] + -g[q00 + 1]) + (-g[q01] + -g[q01 + 1])) * T(0.25);
    }
}

// x -= P v (injection) on the fine level, with ||x||^2
template <typename T, bool RG>
__global__ void __launch_bounds__(FV_NTH)
fv_prolong_correct_kernel(FvArgs<T> Aa, const MemberArgs* __restrict__ mt, T* __restrict__ x, const T* __restrict__ v,
                          Red red, long ms)
{
    const FvArgs<T>& A = fv_of<T, RG>(Aa, mt);
    x = mbr(x, ms);
    v = mbr(v, ms);
    red = mbr(red, ms);
    // a one-dimensional grid over this member's 64 x 4 tiles (row-major)
    const unsigned gx = (unsigned)((A.nxl + FV_TX - 1) / FV_TX), nt = gx * (unsigned)((A.nzl + FV_TZ - 1) / FV_TZ);
    if (blockIdx.x >= nt || sits_out(mt)) {   // beyond a smaller member, or one that sits out
        if (threadIdx.x == 0) red.partials[blockIdx.x] = 0.0;
        return;
    }
    const int I = (blockIdx.x % gx) * FV_TX + (threadIdx.x & (FV_TX - 1));
    const int J = (blockIdx.x / gx) * FV_TZ + (threadIdx.x / FV_TX);
    double nrm = 0.0;
    if (I < A.nxl && J < A.nzl) {
        const long q = (long)J * A.nxl + I;
        const long ncc = (long)(A.nxl / 2) * (A.nzl / 2), qc = (long)(J / 2) * (A.nxl / 2) + I / 2;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const T val = x[c * A.nc + q] - v[c * ncc + qc];
            x[c * A.nc + q] = val;
            nrm += (double)val * (double)val;
        }
    }
    put_partial<FV_NTH>(red, nrm);
}

template <typename T, bool RG>
__global__ void __launch_bounds__(FV_NTH)
fv_restrict_kernel(FvArgs<T> Aa, const MemberArgs* __restrict__ mt, const T* __restrict__ f, T* __restrict__ c, long ms)
{
    const FvArgs<T>& A = fv_of<T, RG>(Aa, mt);
    if (RG && sits_out(mt)) return;
    f = mbr(f, ms);
    c = mbr(c, ms);
    const int nxc = A.nxl / 2, nzc = A.nzl / 2;
    const int Ic = blockIdx.x * FV_TX + (threadIdx.x & (FV_TX - 1));
    const int Jc = blockIdx.y * FV_TZ + (threadIdx.x / FV_TX);
    if (Ic >= nxc || Jc >= nzc) return;
    const long ncc = (long)nxc * nzc, qc = (long)Jc * nxc + Ic;
    const long q00 = (long)(2 * Jc) * A.nxl + 2 * Ic, q01 = q00 + A.nxl;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
        const T* g = f + cc * A.nc;
        c[cc * ncc + qc] = ((g[q00] + g[q00 + 1]) + (g[q01] + g[q01 + 1])) * T(0.25);
    }
}

template <typename T, bool RG>
__global__ void __launch_bounds__(FV_NTH)
fv_prolong_kernel(FvArgs<T> Aa, const MemberArgs* __restrict__ mt, const T* __restrict__ c, T* __restrict__ f, long ms)
{
    const FvArgs<T>& A = fv_of<T, RG>(Aa, mt);
    if (RG && sits_out(mt)) return;
    c = mbr(c, ms);
    f = mbr(f, ms);
    const int I = blockIdx.x * FV_TX + (threadIdx.x & (FV_TX - 1));
    const int J = blockIdx.y * FV_TZ + (threadIdx.x / FV_TX);
    if (I >= A.nxl || J >= A.nzl) return;
    const long q = (long)J * A.nxl + I;
    const long ncc = (long)(A.nxl / 2) * (A.nzl / 2), qc = (long)(J / 2) * (A.nxl / 2) + I / 2;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) f[cc * A.nc + q] = c[cc * ncc + qc];
}

template <typename T>
__global__ void __launch_bounds__(256) fv_norm2_kernel(const T* __restrict__ x, long n, Red red, long ms)
{
    x = mbr(x, ms);
    red = mbr(red, ms);
    double s = 0.0;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
        const double v = x[i];
        s += v * v;
    }
    put_partial<256>(red, s);
}

// level slots from the LIN partials: ||u + Ubar||, max(|v| + c), pseudo time step
// The slots of every level from the LIN partials (one work-group per level, level l's
// 2 x nb[l] partials at p + l * pstride): ||u + Ubar||, its inverse, max(|v| + c), dtau
template <typename T>
__global__ void __launch_bounds__(256)
fv_lin_finalize_kernel(const double* __restrict__ p, long pstride, LinLevels lv, double* __restrict__ slots,
                       double mu, double adt, double cfl, long ms, const MemberArgs* __restrict__ mt)
{
    const int lev = blockIdx.x;
    p = mbr(p, ms) + lev * pstride;
    slots = mbr(slots, ms) + 4 * lev;
    const int nb = lv.nb[lev];
    double hx = lv.hx[lev], hz = lv.hz[lev];
    if (mt) {   // a ragged member's own cell widths
        const FvArgs<T>& A = fv_entry<T>(mt, lev);
        hx = (double)A.hx;
        hz = (double)A.hz;
    }
    __shared__ double sh[4];
    double a = 0.0, m = 0.0;
    for (int i = threadIdx.x; i < nb; i += 256) { a += p[i]; m = fmax(m, p[nb + i]); }
    a = block_sum<256>(a, sh);
    m = block_max<256>(m, sh);
    if (threadIdx.x == 0) {
        slots[LV_UTOT] = sqrt(a);
        slots[LV_IUTOT] = a > 0.0 ? 1.0 / sqrt(a) : 0.0;
        slots[LV_LAM] = m;
        slots[LV_DTAU] = cfl / (1.0 + adt * (m * (1.0 / hx + 1.0 / hz) + 2.0 * mu * (1.0 / (hx * hx) + 1.0 / (hz * hz))));
    }
}

static inline dim3 tile_grid(int nx, int nz, int members = 1)
{
    return dim3((unsigned)((nx + FV_TX - 1) / FV_TX), (unsigned)((nz + FV_TZ - 1) / FV_TZ), (unsigned)members);
}
// the same 64 x 4 tiles as a one-dimensional grid
static inline dim3 tile_grid_1d(int nx, int nz, int members = 1)
{
    const dim3 g = tile_grid(nx, nz);
    return dim3(g.x * g.y, 1, (unsigned)members);
}

template <typename T, int TX, int TZ, int NTH, int WPE, bool LATE, bool ZREV, int MODE>
static int tile_launch_shape(const FvArgs<T>& A, const T* u, const T* F0, const T* xp, const T* x0, const T* b,
                             T* out, T* out2, const double* xpart, int xcount, double* slots, const double* slots2,
                             double alpha_j, double adt, int fzero, Red red, hipStream_t st, const Mb& mb,
                             const TinvOut& tv)
{
    const unsigned nt = (unsigned)((A.nxl + TX - 1) / TX) * (unsigned)((A.nzl + TZ - 1) / TZ);
    const dim3 g(nt, 1, (unsigned)mb.n);
    // Every work-group sums all partials of ||x||^2 by itself, which saves a launch (3 us)
    // while they are few; 4608 of them, read by as many work-groups, made the second stage of
    // 2.4 M cells take 82 us where the one after 1024 partials took 45: one launch before it.
    // (Eighteen sweeps with and without that launch, us, 64x4 tiles of a level 1024 cells wide:
    // FP64 2048 partials 391 and 385, 3072 501 and 494, 3328 538 and 558, 5120 766 and 832;
    // FP32 250 and 231, 320 and 314, 343 and 356, 460 and 496.)
    // (Not a timed launch: the caller's kernel class is that of the tile kernel.)
    if (MODE != FVM_LIN && xcount > FV_SUM_MAX) {
        fv_sum_kernel<NTH><<<dim3(1, 1, (unsigned)mb.n), dim3(NTH), 0, st>>>(const_cast<double*>(xpart), xcount,
                                                                             mb.n > 1 ? mb.ms : 0L);
        xpart += xcount;
        xcount = 1;
    }
    if (mb.tab)
        timed_launch(fv_tile_kernel<T, TX, TZ, NTH, WPE, LATE, ZREV, true, MODE, true>, g, dim3(NTH), st, A, mb.tab, u,
                     F0, xp, x0, b, out, out2, xpart, xcount, slots, slots2, alpha_j, adt, fzero, red, mb.ms, tv);
    else if (mb.n > 1)
        timed_launch(fv_tile_kernel<T, TX, TZ, NTH, WPE, LATE, ZREV, true, MODE, false>, g, dim3(NTH), st, A, mb.tab,
                     u, F0, xp, x0, b, out, out2, xpart, xcount, slots, slots2, alpha_j, adt, fzero, red, mb.ms, tv);
    else
        timed_launch(fv_tile_kernel<T, TX, TZ, NTH, WPE, LATE, ZREV, false, MODE, false>, g, dim3(NTH), st, A, mb.tab,
                     u, F0, xp, x0, b, out, out2, xpart, xcount, slots, slots2, alpha_j, adt, fzero, red, 0L, tv);
    return (int)nt;
}

template <typename T, int MODE>
static int tile_launch(const FvArgs<T>& A, const T* u, const T* F0, const T* xp, const T* x0, const T* b, T* out,
                       const double* xpart, int xcount, double* slots, double alpha_j, double adt, int fzero,
                       Red red, hipStream_t st, const Mb& mb, T* out2 = nullptr, const double* slots2 = nullptr,
                       const TinvOut& tv = TinvOut{})
{
    switch (A.tile) {
    case JFMG_TILE_64x8:
        return tile_launch_shape<T, 64, 8, 512, 4, true, true, MODE>(A, u, F0, xp, x0, b, out, out2, xpart, xcount,
                                                                       slots, slots2, alpha_j, adt, fzero, red, st, mb, tv);
    case JFMG_TILE_16x4:
        return tile_launch_shape<T, 16, 4, 256, 1, false, true, MODE>(A, u, F0, xp, x0, b, out, out2, xpart, xcount,
                                                                        slots, slots2, alpha_j, adt, fzero, red, st, mb, tv);
    case JFMG_TILE_8x4:
        return tile_launch_shape<T, 8, 4, 128, 1, false, true, MODE>(A, u, F0, xp, x0, b, out, out2, xpart, xcount,
                                                                       slots, slots2, alpha_j, adt, fzero, red, st, mb, tv);
    case JFMG_TILE_32x4:
        return tile_launch_shape<T, 32, 4, 256, 2, false, true, MODE>(A, u, F0, xp, x0, b, out, out2, xpart, xcount,
                                                                        slots, slots2, alpha_j, adt, fzero, red, st, mb, tv);
    case JFMG_TILE_64x4_512:
        return tile_launch_shape<T, 64, 4, 512, 4, true, true, MODE>(A, u, F0, xp, x0, b, out, out2, xpart, xcount,
                                                                       slots, slots2, alpha_j, adt, fzero, red, st, mb, tv);
    default:
        return tile_launch_shape<T, 64, 4, 256, 4, true, true, MODE>(A, u, F0, xp, x0, b, out, out2, xpart, xcount,
                                                                       slots, slots2, alpha_j, adt, fzero, red, st, mb, tv);
    }
}

template <typename T>
int FvLaunch<T>::lin_level(const FvArgs<T>& A, const T* u, T* F0, T* uc, Red red, double adt, hipStream_t st,
                           const Mb& mb)
{
    return tile_launch<T, FVM_LIN>(A, u, nullptr, nullptr, nullptr, nullptr, F0, nullptr, 0, nullptr, 0.0, adt, 0, red,
                                   st, mb, uc);
}
template <typename T>
void FvLaunch<T>::lin_finalize(const double* partials, long pstride, const LinLevels& lv, int nlev, double* slots,
                               double mu, double adt, double cfl, hipStream_t st, const Mb& mb)
{
    fv_lin_finalize_kernel<T><<<dim3(nlev, 1, mb.n), dim3(256), 0, st>>>(partials, pstride, lv, slots, mu, adt, cfl,
                                                                         mb.ms, mb.tab);
}
template <typename T>
int FvLaunch<T>::stage(const FvArgs<T>& A, const T* u, const T* F0, const T* xp, const T* x0, const T* b, T* xo,
                       const double* xpart, int xcount, const double* slots, double alpha_j, double adt, int zero,
                       Red red, hipStream_t st, const Mb& mb)
{
    if (zero) {
        const long n = 4 * A.nc;
        const int nb = norm_blocks(n);
        if (mb.tab)
            timed_launch(fv_stage_zero_kernel<T, true>, dim3(nb, 1, mb.n), dim3(256), st, A, mb.tab, b, xo, slots,
                         alpha_j, red, mb.ms);
        else
            timed_launch(fv_stage_zero_kernel<T, false>, dim3(nb, 1, mb.n), dim3(256), st, A, mb.tab, b, xo, slots,
                         alpha_j, red, mb.ms);
        return nb;
    }
    return tile_launch<T, FVM_STAGE>(A, u, F0, xp, x0, b, xo, xpart, xcount, const_cast<double*>(slots), alpha_j,
                                     adt, 0, red, st, mb);
}
template <typename T>
int FvLaunch<T>::stage_prolong(const FvArgs<T>& A, const T* u, const T* F0, const T* xp, const T* x0, const T* b,
                               T* xf, bool fine_zero, const double* xpart, int xcount, const double* slots,
                               double alpha_j, double adt, Red red, hipStream_t st, const Mb& mb)
{
    return tile_launch<T, FVM_STAGE_PC>(A, u, F0, xp, x0, b, nullptr, xpart, xcount, const_cast<double*>(slots),
                                        alpha_j, adt, fine_zero ? 1 : 0, red, st, mb, xf);
}
template <typename T>
int FvLaunch<T>::stage_tinv(const FvArgs<T>& A, const T* u, const T* F0, const T* xp, const T* x0, const T* b,
                            const TinvOut& tv, const double* xpart, int xcount, const double* slots, double alpha_j,
                            double adt, Red red, hipStream_t st, const Mb& mb)
{
    return tile_launch<T, FVM_STAGE_TINV>(A, u, F0, xp, x0, b, nullptr, xpart, xcount, const_cast<double*>(slots),
                                          alpha_j, adt, 0, red, st, mb, nullptr, nullptr, tv);
}
template <typename T>
void FvLaunch<T>::matvec(const FvArgs<T>& A, const T* u, const T* F0, const T* x, T* out, const double* xpart,
                         int xcount, const double* slots, double adt, hipStream_t st, const Mb& mb)
{
    tile_launch<T, FVM_MATVEC>(A, u, F0, x, nullptr, nullptr, out, xpart, xcount, const_cast<double*>(slots), 0.0,
                               adt, 0, Red{nullptr, nullptr}, st, mb);
}
template <typename T>
int FvLaunch<T>::defect_restrict(const FvArgs<T>& A, const T* u, const T* F0, const T* x, const T* b, T* rc,
                                 const double* xpart, int xcount, const double* slots, double adt, int zero,
                                 hipStream_t st, const Mb& mb, const ZeroStage<T>& z0)
{
    if (zero) {
        const dim3 g((unsigned)((A.nxl / 2 + 63) / 64), (unsigned)((A.nzl / 2 + 3) / 4), (unsigned)mb.n);
        if (mb.tab) timed_launch(fv_restrict_neg_kernel<T, true>, g, dim3(256), st, A, mb.tab, b, rc, mb.ms);
        else timed_launch(fv_restrict_neg_kernel<T, false>, g, dim3(256), st, A, mb.tab, b, rc, mb.ms);
        return 0;
    }
    const int nb = tile_launch<T, FVM_DEFECT>(A, u, F0, x, nullptr, b, rc, xpart, xcount, const_cast<double*>(slots),
                                              z0.alpha, adt, 0, z0.red, st, mb, z0.x1, z0.slots);
    return z0.x1 ? nb : 0;
}
template <typename T>
int FvLaunch<T>::prolong_correct(const FvArgs<T>& Af, T* x, const T* v, Red red, hipStream_t st, const Mb& mb)
{
    const dim3 g = tile_grid_1d(Af.nxl, Af.nzl, mb.n);
    if (mb.tab) timed_launch(fv_prolong_correct_kernel<T, true>, g, dim3(FV_NTH), st, Af, mb.tab, x, v, red, mb.ms);
    else timed_launch(fv_prolong_correct_kernel<T, false>, g, dim3(FV_NTH), st, Af, mb.tab, x, v, red, mb.ms);
    return (int)g.x;
}
template <typename T>
void FvLaunch<T>::restrict_(const FvArgs<T>& Af, const T* f, T* c, hipStream_t st, const Mb& mb)
{
    const dim3 g = tile_grid(Af.nxl / 2, Af.nzl / 2, mb.n);
    if (mb.tab) fv_restrict_kernel<T, true><<<g, dim3(FV_NTH), 0, st>>>(Af, mb.tab, f, c, mb.ms);
    else fv_restrict_kernel<T, false><<<g, dim3(FV_NTH), 0, st>>>(Af, mb.tab, f, c, mb.ms);
}
template <typename T>
void FvLaunch<T>::prolong(const FvArgs<T>& Af, const T* c, T* f, hipStream_t st, const Mb& mb)
{
    const dim3 g = tile_grid(Af.nxl, Af.nzl, mb.n);
    if (mb.tab) fv_prolong_kernel<T, true><<<g, dim3(FV_NTH), 0, st>>>(Af, mb.tab, c, f, mb.ms);
    else fv_prolong_kernel<T, false><<<g, dim3(FV_NTH), 0, st>>>(Af, mb.tab, c, f, mb.ms);
}
template <typename T>
void FvLaunch<T>::norm2(const T* x, long n, Red red, hipStream_t st, const Mb& mb)
{
    fv_norm2_kernel<T><<<dim3(norm_blocks(n), 1, mb.n), dim3(256), 0, st>>>(x, n, red, mb.ms);
    if (red.out) launch_finalize(red.partials, norm_blocks(n), 1, red.out, st, mb);
}
// The default shape by the level's cells (in a ragged batch those of all members, which
// share a launch).  Stage kernel, FP64 / FP32, us (viscous 256 x 64 and 768 x 192 elements
// of degree 3 and their coarser levels, 24 members of 288 x 144 cells and less):
//     cells    8x4         16x4        64x4_512    64x4        64x8
//      4096    4.1 / 3.7   4.5 / 3.8   6.0 / 5.8   6.1 / 5.3   7.4 / 6.6
//     16384    4.6 / 3.9   4.5 / 4.0   5.8 / 5.9   6.0 / 5.2   7.4 / 6.7
//     65536   10.3 / 6.4   8.3 / 5.8   6.3 / 5.1   6.5 / 5.4   8.0 / 6.1
//    147456   16.8 / 10.4 14.2 / 8.9  12.0 / 8.1  10.1 / 7.0  11.6 / 8.2
//    262144   29.5 / 15.5 22.9 / 13.5 14.8 / 9.9  13.3 / 9.5  12.8 / 9.1
//    580608   51.5 / 26.4 47.7 / 23.6 33.0 / 19.9 24.7 / 16.0 26.5 / 16.9
//   2359296    268 / 101   191 / 84.7  129 / 61.1 93.1 / 50.7  102 / 45.6
// (by the level's width, the rule before, 192 x 96 cells took 8x4, the members 16x4 and a
// level of 2400 x 80 cells 64x8, 11.7 / 8.7 against 10.5 / 7.8 with 64x4).  64x8 is the
// fastest in FP64 where its tiles fill the 512 places of one round (us, 64x8 and 64x4: 10.4 and
// 10.7 at 448 tiles, 10.6 and 10.8 at 480; in FP32 7.6 and 7.5; below, 10.3 and 9.1 at 384; with
// a second round 14.0 and 12.4 at 528), and in FP32 on large levels.
// Rows that leave more than 30 % of the 64-cell rows empty take 16x4.
int fv_default_tile(long cells, long padded64, bool f32)
{
    if (cells < 8192) return JFMG_TILE_8x4;
    if (cells < 32768 || 10 * cells < 7 * padded64) return JFMG_TILE_16x4;
    if (cells < 131072) return JFMG_TILE_64x4_512;
    const long t8 = padded64 / 512;   // tiles of 64x8
    return (t8 > 448 && t8 <= 512) || (f32 && cells >= 655360) ? JFMG_TILE_64x8 : JFMG_TILE_64x4;
}
bool fv_wide_tile(int tile) { return tile == JFMG_TILE_64x4 || tile == JFMG_TILE_64x8 || tile == JFMG_TILE_64x4_512; }
bool fv_tile_fits_elements(int tile, int n1)
{
    const int tx = tile == JFMG_TILE_16x4 ? 16 : tile == JFMG_TILE_8x4 ? 8 : tile == JFMG_TILE_32x4 ? 32 : 64;
    const int tz = tile == JFMG_TILE_64x8 ? 8 : 4;
    return (n1 == 2 || n1 == 4) && tx % n1 == 0 && tz % n1 == 0;   // the stage kernel's two N1
}

long fv_partial_blocks(long nxl, long nzl)
{
    // the most work-groups of any tile shape (8x4) or of the 64x4 streaming kernels, at least 1024
    const long smallest = ((nxl + 7) / 8) * ((nzl + 3) / 4);
    const long pro = ((nxl + FV_TX - 1) / FV_TX) * ((nzl + FV_TZ - 1) / FV_TZ);
    return std::max(std::max(smallest, pro), 1024L);
}
// Levels that the tail kernel takes: its LDS holds them, and the work-group has a thread for
// each face.
bool fv_tail_fits(int nxl, int nzl, int tile)
{
    const int nt = ((nxl + 7) / 8) * ((nzl + 3) / 4);
    return tile == JFMG_TILE_8x4 && nxl * nzl <= TAIL_CELLS && nt <= TAIL_NTH / 32 && nzl <= TAIL_ROWS &&
           (((nxl + 1) * nzl + 63) & ~63) + nxl * (nzl + 1) <= TAIL_NTH;
}
template <typename T> int FvLaunch<T>::tail(const TailArgs<T>& a0, hipStream_t st, const Mb& mb)
{
    TailArgs<T> a = a0;
    a.nparts = ((a.A.nxl + 7) / 8) * ((a.A.nzl + 3) / 4);
    const dim3 g(1, 1, (unsigned)mb.n);
    const long ms = mb.n > 1 ? mb.ms : 0L;
    if (mb.tab) timed_launch(fv_tail_kernel<T, true>, g, dim3(TAIL_NTH), st, a, mb.tab, ms);
    else timed_launch(fv_tail_kernel<T, false>, g, dim3(TAIL_NTH), st, a, mb.tab, ms);
    return a.nparts;
}
template <typename T> int FvLaunch<T>::norm_blocks(long n)
{
    long b = (n + 255) / 256;
    return (int)(b < 1024 ? b : 1024);
}

template struct FvLaunch<double>;
template struct FvLaunch<float>;

}  // namespace jfmg
