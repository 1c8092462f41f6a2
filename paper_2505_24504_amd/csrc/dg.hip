// DG space operator of the well-balanced perturbation system (paper eqs.
// convDiscr, elementint, surfaceint and perturbed-euler) on gfx950.
//
// On Cartesian elements the operator splits by direction: the x-fluxes need only
// x-derivatives and the z-fluxes only z-derivatives, and each is contracted along its
// own direction.  A thread therefore takes one line of k + 1 GL nodes of an element
// along x or along z, holds it in registers and does everything along it there with
// wave-uniform weights: 128 threads of a work-group take the x-lines of a tile of
// elements, 128 the z-lines.  Per tile:
//   T  every line's trace and trace derivative at both ends; those at the high end, and
//      the facing ends of the neighbour elements' lines outside the tile, go to LDS;
//      the background of the tile's rows is staged with them;
//   F  every line's face point at its low end (each face point of the grid once, at a
//      tile's high end once more by the tile): HLLC minus the background HLLC, the
//      interior-penalty terms and both sides' symmetric terms;
//   V  the volume fluxes along the line (total state U' + Ubar minus the background
//      flux, minus the viscous flux), contracted with the GL derivative matrix, and the
//      face terms of both ends lifted to the line's nodes;
//   D  the x-lines add the z-lines' result (through LDS) and write the output.
// In JVP mode the kernel evaluates the fluxes of U' + eps y and differences them
// point by point with those of U' before contracting.  The fluxes of U' are the
// same for every product with one linearization state: mode 5 writes them (volume
// fluxes per node, face terms per face point) once per linearization, and each
// product reads them back instead of evaluating a second state.
//
// What bounds it: memory latency and FP64 issue on large grids, on the density current
// (256 x 64 elements, k = 3, one round of work-groups) the chain of its phases.  With a
// thread per node, every face point evaluated from both sides and the background's HLLC
// at each of them, M^-1 L_h took 705 us at 1024 x 1024 elements (viscous, k = 3) and an
// explicit stage 15.3 us at 256 x 64 and 11.1 us at 197 x 45 (k = 2); this form takes
// 438, 11.8 and 7.4 us with half the VALU and a third of the LDS work per node.  A
// node-per-thread form with each tile face evaluated once reached 636, 13.3 and 7.9 us.
// Six waves per work-group (the neighbours' lines and the high faces on two of their
// own) were slower at k = 3, 18.7 against 15.2 us under counters: two such groups do
// not fit the three wave slots per SIMD that 168 registers leave.
#include "jfmg_internal.h"

namespace jfmg {

// Tiles of TEX x TEZ elements with HALF lines per direction: 32 elements (k = 3),
// 42 (k = 2), 64 (k = 1).  The lines of neighbours (NHX + NHZ of them) and the face
// points at the tile's high ends (NXF + NZF) each fit one wave per direction.
template <int N1> struct DgShape {
    static constexpr int TEX = N1 == 3 ? 7 : 8, TEZ = N1 == 4 ? 4 : N1 == 3 ? 6 : 8;
    static constexpr int NP = N1 * N1, HALF = 128, NTH = 2 * HALF, EPB = TEX * TEZ;
    static constexpr int NXF = TEZ * N1, NZF = TEX * N1;     // high-end face points of x- and z-lines
    static constexpr int NSLOT = NTH + 2 * (NXF + NZF);      // own lines, then left, right, bottom, top
    static constexpr int ROWS = TEZ * N1, NROW = ROWS + TEZ + 1;   // background rows: nodes, then z-faces
    static_assert(EPB * N1 <= HALF && 2 * NXF <= 64 && 2 * NZF <= 64 && NXF + NZF <= 64 && 3 * ROWS + TEZ + 1 <= 64,
                  "tile shape");
};

// work-groups of a grid of nx x nz elements
template <int N1> __host__ __device__ inline int dg_tiles(int nx, int nz)
{
    return ((nx + DgShape<N1>::TEX - 1) / DgShape<N1>::TEX) * ((nz + DgShape<N1>::TEZ - 1) / DgShape<N1>::TEZ);
}

// LDS record of a background row (node row or z-face): rho, rho u, rho theta (the
// background has no vertical wind), pressure, 1/(rho theta), d/dz of the three; with the
// background subtracted also the HLLC flux of the background in the frame of the row's
// faces (normal momentum at 1, tangential at 2) through a face inside the grid (or the
// wall of the bottom or top row), for node rows through a wall on the low and on the
// high side, and the x-momentum and rho theta components of the convective x-flux.
enum { BR_RHO = 0, BR_MX = 1, BR_RT = 2, BR_P = 3, BR_IRT = 4, BR_DRHO = 5, BR_DMX = 6, BR_DRT = 7, BR_H = 8,
       BR_HLO = 12, BR_HHI = 16, BR_F1 = 20, BR_F3 = 21 };
static_assert(DG_REC == 22, "record length");

// Record of node row (zr false) or z-face row i in rec; with bgsub the flux entries of
// case v (0: inside the grid, 1 and 2: a wall on the low or high side), else and for
// v = 0 the state entries.
__device__ __forceinline__ void dg_record(const DgArgs& A, bool zr, int i, int v, bool bgsub, double* __restrict__ rec)
{
    const double* bg = (zr ? A.bg_face : A.bg_node) + 4 * i;
    const double* db = (zr ? A.dbg_face : A.dbg_node) + 4 * i;
    const double pb = zr ? A.pb_face[i] : A.pb_node[i], irt = zr ? A.irt_face[i] : A.irt_node[i];
    const double rho = bg[0], mx = bg[1], rt = bg[3];
    if (v == 0) {
        rec[BR_RHO] = rho;
        rec[BR_MX] = mx;
        rec[BR_RT] = rt;
        rec[BR_P] = pb;
        rec[BR_IRT] = irt;
        rec[BR_DRHO] = db[0];
        rec[BR_DMX] = db[1];
        rec[BR_DRT] = db[3];
    }
    if (bgsub) {
        double UL[4] = {rho, zr ? 0.0 : mx, zr ? mx : 0.0, rt}, UR[4], H[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) UR[c] = UL[c];
        if (v == 1 || (zr && i == 0)) UL[1] = -UL[1];
        if (v == 2 || (zr && i == A.nz)) UR[1] = -UR[1];
        const double ir = frcp(rho);
        hllc(A.gas, UL, UR, pb, pb, ir, ir, H);
#pragma unroll
        for (int c = 0; c < 4; ++c) rec[(v == 0 ? BR_H : v == 1 ? BR_HLO : BR_HHI) + c] = H[c];
        if (v == 0) {
            const double q1 = mx * ir;
            rec[BR_F1] = mx * q1 + pb;
            rec[BR_F3] = rt * q1;
        }
    }
}

// The records of every row of a grid, once per problem: node rows, then z-faces.
__global__ void __launch_bounds__(256) dg_records_kernel(DgArgs A, int rows, double* __restrict__ rec)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= rows + A.nz + 1) return;
    const bool zr = i >= rows;
    for (int v = 0; v < 3; ++v) dg_record(A, zr, zr ? i - rows : i, v, true, rec + (long)DG_REC * i);
}

void launch_dg_records(int k, const DgArgs& A, double* rec, hipStream_t st)
{
    const int rows = (k + 1) * A.nz;
    dg_records_kernel<<<dim3((unsigned)((rows + A.nz + 1 + 255) / 256)), dim3(256), 0, st>>>(A, rows, rec);
}

// Terms at one face point along +e_D, in the face frame (component 1 the normal
// momentum, 2 the tangential one), from both sides' traces tl, th and trace derivatives
// nl, nh (d/d xi):
//   Phi = H(U_lo, U_hi) (minus the background's H when BGSUB) minus, for viscous flow,
//         the average of both sides' F_v . n plus the interior penalty on the jump of
//         the velocity-like variables,
//   slo, shi = the symmetric term's jump of either side, mu/2 (+-[U_c] - (U_c/rho)_side (+-[rho])),
//         [U] = U_lo - U_hi (components 1..3).
// At a slip wall (wlo, whi) the missing side is the inside trace mirrored.
template <bool NS, bool BGSUB>
__device__ __forceinline__ void dg_face(const DgArgs& A, double (&tl)[4], const double (&nl)[4], double (&th)[4],
                                        const double (&nh)[4], const double* __restrict__ row, bool xf, bool wlo,
                                        bool whi, double (&Phi)[4], double (&slo)[3], double (&shi)[3])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {   // slip walls: the inside trace on both sides
        const double a = wlo ? th[c] : tl[c];
        th[c] = whi ? tl[c] : th[c];
        tl[c] = a;
    }
    const double pb = row[BR_P], irt = row[BR_IRT], mx = row[BR_MX];
    const double Ub[4] = {row[BR_RHO], xf ? mx : 0.0, xf ? 0.0 : mx, row[BR_RT]};
    double UL[4], UR[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        UL[c] = tl[c] + Ub[c];
        UR[c] = th[c] + Ub[c];
    }
    if (wlo) UL[1] = -UL[1];
    if (whi) UR[1] = -UR[1];
    const double rt[2] = {tl[3], th[3]}, ir2[2] = {irt, irt}, pb2[2] = {pb, pb};
    double pp[2];
    pert_pressures<double, 2, false>(A.gas, rt, ir2, pb2, pp);
    const double pL = pp[0], pR = pp[1];
    const double irL = frcp(UL[0]), irR = frcp(UR[0]);
    hllc(A.gas, UL, UR, pL, pR, irL, irR, Phi);
    if constexpr (BGSUB) {
        const double* hb = row + (wlo && xf ? BR_HLO : whi && xf ? BR_HHI : BR_H);
#pragma unroll
        for (int c = 0; c < 4; ++c) Phi[c] -= hb[c];
    }
    if constexpr (NS) {
        // F_v(U, G) . n of a Cartesian face involves only the normal derivative (the
        // tangential part enters multiplied by 0): both sides' trace derivatives,
        // plus the background's z-derivative on z-faces; none of it at walls
        const bool wall = wlo | whi;
        const double gs = xf ? A.rdx2 : A.rdz2;
        const double eta = xf ? A.eta_x : A.eta_z;
        const double gb[4] = {xf ? 0.0 : row[BR_DRHO], 0.0, xf ? 0.0 : row[BR_DMX], xf ? 0.0 : row[BR_DRT]};
        const double GL0 = gs * nl[0] + gb[0], GR0 = gs * nh[0] + gb[0];
        const double D0 = tl[0] - th[0];
        const double irm = frcp(0.5 * (UL[0] + UR[0]));
#pragma unroll
        for (int c = 1; c < 4; ++c) {
            const double rl = UL[c] * irL, rr = UR[c] * irR;
            const double fo = (gs * nl[c] + gb[c]) - rl * GL0;
            const double fx = (gs * nh[c] + gb[c]) - rr * GR0;
            const double Dc = tl[c] - th[c];
            const double pen = eta * (Dc - (0.5 * (UL[c] + UR[c]) * irm) * D0);
            const double pv = A.mu * (0.5 * (fo + fx) - pen);
            Phi[c] -= wall ? 0.0 : pv;
            slo[c - 1] = wall ? 0.0 : 0.5 * A.mu * (Dc - rl * D0);
            shi[c - 1] = wall ? 0.0 : -0.5 * A.mu * (Dc - rr * D0);
        }
    }
}

// The line of nodes n0, n0 + 1, ... (x) or n0, n0 + N1, ... (z) of the four components,
// in the line's frame (component 1 the momentum along it).  xd is wave-uniform.
template <int N1>
__device__ __forceinline__ void dg_line(const double* __restrict__ U, long N, unsigned n0, bool xd, double (&v)[4][N1])
{
    if (xd) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < N1; ++j) v[c][j] = ld(U + c * N, n0 + j);
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < N1; ++j) v[c][j] = ld(U + (c == 1 ? 2 : c == 2 ? 1 : c) * N, n0 + j * N1);
    }
}

// The JVP (MODE 3) reads its stored terms ahead and holds a line of both vectors and of the
// halo's at once: two waves per SIMD, the shorter chain where all work-groups run at the same
// time (two per CU, 512).  With more of them, LEAN: the halo's lines after the own, the stored
// terms where they are used, three waves per SIMD; the same products and sums.  Inviscid
// k = 2, 24 members: 34.3 -> 30.6 us per launch, the ensemble's step 71.5 -> 70.3 ms.  Not
// for the viscous kernels and k = 3, whose registers spill (k = 3, viscous, 9.4 M unknowns:
// 169 us, 201 so; inviscid, 16 registers: 46.0 and 50.3 us at 4.2 M, 207 and 237 at 16.8 M).
constexpr long DG_LEAN_TILES = 512;
template <int N1, bool NS> constexpr bool DG_LEAN = !NS && N1 <= 3;

// REC: the background records are read from the problem's table (A.rec); without one
// (the allocation-free residual) wave 0 evaluates the tile's.
template <int N1, bool NS, int MODE, bool RG, bool REC, bool LEAN = false>
__global__ void __launch_bounds__(DgShape<N1>::NTH, MODE == 3 && !LEAN ? 2 : 3)
dg_kernel(DgArgs Aa, const MemberArgs* __restrict__ mt, const double* __restrict__ U, const double* __restrict__ Y,
          const double* __restrict__ Ubar, double* __restrict__ out, const double* __restrict__ yn2p,
          const double* __restrict__ ut2p, int eps_mode, double adt, Red red, long ms, ExStage rk, int ycount)
{
    const DgArgs& A = dg_of<RG>(Aa, mt);
    // the arguments that the first loads need, in scalar registers at once
    gptr<double> U_ = (gptr<double>)U, rec_ = (gptr<double>)A.rec;
    int nx = A.nx, nz = A.nz;
    if constexpr (MODE == 3) {
        gptr<double> Y_ = (gptr<double>)Y, yn2p_ = (gptr<double>)yn2p, ut2p_ = (gptr<double>)ut2p;
        asm volatile("" : "+s"(U_), "+s"(Y_), "+s"(rec_), "+s"(yn2p_), "+s"(ut2p_), "+s"(ycount), "+s"(nx), "+s"(nz));
        Y = (const double*)Y_;
        yn2p = (const double*)yn2p_;
        ut2p = (const double*)ut2p_;
    } else {
        asm volatile("" : "+s"(U_), "+s"(rec_), "+s"(nx), "+s"(nz));
    }
    U = (const double*)U_;
    const double* const grec = (const double*)rec_;
    double* lin0 = A.lin0;
    if (gridDim.z > 1) {   // member of a lock-step batch
        U = mbr(U, ms);
        Y = mbr(Y, ms);
        Ubar = mbr(Ubar, ms);
        out = mbr(out, ms);
        yn2p = mbr(yn2p, ms);
        ut2p = mbr(ut2p, ms);
        red = mbr(red, ms);
        if (!RG) lin0 = mbr(lin0, ms);   // a ragged member's pointer is its own
    }
    using S = DgShape<N1>;
    constexpr int NP = S::NP, NTH = S::NTH, HALF = S::HALF, EPB = S::EPB, TEX = S::TEX, TEZ = S::TEZ;
    constexpr int NXF = S::NXF, NZF = S::NZF, NSLOT = S::NSLOT, ROWS = S::ROWS;
    constexpr bool BGSUB = MODE != 3 && MODE != 5;
    constexpr int BRN = BGSUB ? 22 : 8;               // doubles of a background record
    constexpr int TRN = NS ? 8 : 4;                   // trace (and its derivative)
    constexpr int FLN = NS ? 7 : 4;                   // face terms the low side's element needs
    constexpr int FCN = NS ? 10 : 4;                  // stored face terms of the linearization state
    const int ntx = (nx + TEX - 1) / TEX, ntiles = dg_tiles<N1>(nx, nz);   // this member's work-groups
    if ((int)blockIdx.x >= ntiles || (RG && sits_out(mt))) {   // beyond a smaller member, or one that sits out
        if (MODE == 2 && red.partials && threadIdx.x == 0) red.partials[block_linear()] = 0.0;
        return;
    }
    // traces [component][slot] of the low sides, later the z-lines' result [component][node]
    constexpr int NTR = TRN * NSLOT, NLZ = MODE == 5 ? 1 : 4 * EPB * NP;
    __shared__ double sT[NTR > NLZ ? NTR : NLZ];
    __shared__ double sF[FLN * (NTH + NXF + NZF)];   // face terms [term][own low face, then the tile's high faces]
    __shared__ double sH[NS && MODE != 5 ? 3 : 1][NS && MODE != 5 ? NTH : 1];   // the low faces' terms of the high side
    __shared__ double sB[S::NROW][BRN];
    constexpr int NFS = NTH + NXF + NZF;

    const int t = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool xd = wv < HALF / 64;                       // x- or z-line (wave-uniform)
    const int tile = (int)xcd_tile(blockIdx.x, ntiles);   // XCD-contiguous ranges of tiles
    const int ex0 = (tile % ntx) * TEX, ez0 = (tile / ntx) * TEZ;
    const int wx = min(TEX, nx - ex0), wz = min(TEZ, nz - ez0);   // elements of this tile
    const bool per = A.bc == 1;
    const int lt = xd ? t : t - HALF;
    const int le = lt / N1, ln = lt - le * N1;            // element of the tile, line
    const int lz = le / TEX, lx = le - lz * TEX;
    const bool valid = le < EPB && lx < wx && lz < wz;
    const long N = A.ne * NP;
    double* const vol0 = lin0;              // [8][N]
    double* const face0 = lin0 + 8 * N;     // [FCN][NF]
    const unsigned NF = (unsigned)(N1 * ((nx + 1) * (long)nz + nx * (long)(nz + 1)));
    // (lanes without a line read element 0's: the loads stay free of branches)
    const unsigned e0 = valid ? (unsigned)(((ez0 + lz) * (long)nx + ex0 + lx) * NP) : 0u;
    const unsigned n0 = e0 + (xd ? ln * N1 : ln);         // first node of the line
    const RefTab& R = A.R;

    // ---- every global load first ----
    PartialSum<NTH> ysum;
    double ut2 = 0.0, yn1 = 0.0;
    if constexpr (MODE == 3) {
        if (ycount > 0) ysum.load(yn2p, ycount);
        else yn1 = ldv(yn2p);
        if (eps_mode != 0) ut2 = ldv(ut2p);
    }
    double s[4][N1], y[4][N1];
    dg_line<N1>(U, N, n0, xd, s);
    if constexpr (MODE == 3) dg_line<N1>(Y, N, n0, xd, y);
    // the neighbour elements' lines outside the tile: of bottom and top (z) in wave 2, of
    // left and right (x) in wave 3; at a wall none
    double h[4][N1], hy[4][N1];
    int hslot = -1;
    bool hhigh = false;
    auto load_halo = [&]() {
        if (wv < 2) return;
        const int l = t & 63, n = wv == 2 ? NZF : NXF;
        const bool up = l >= n;                           // top or right neighbours: their low end
        const int q = up ? l - n : l, g = q / N1, r = q - g * N1;
        int ex = wv == 2 ? ex0 + g : (up ? ex0 + wx : ex0 - 1);
        const int ez = wv == 2 ? (up ? ez0 + wz : ez0 - 1) : ez0 + g;
        bool ok = l < 2 * n && g < (wv == 2 ? wx : wz);
        if (wv == 2) ok = ok && ez >= 0 && ez < nz;
        else if (ex < 0 || ex >= nx) { ex = up ? 0 : nx - 1; ok = ok && per; }
        if (ok) hslot = NTH + (wv == 2 ? 2 * NXF : 0) + l;
        hhigh = !up;
        const unsigned o = ok ? (unsigned)((ez * (long)nx + ex) * NP) + (wv == 2 ? r : r * N1) : 0u;
        dg_line<N1>(U, N, o, wv != 2, h);
        if constexpr (MODE == 3) dg_line<N1>(Y, N, o, wv != 2, hy);
    };
    if constexpr (!LEAN) load_halo();
    constexpr int NRL = (BRN * ROWS + NTH - 1) / NTH;   // loads per thread for the node rows
    double rr[NRL], rf = 0.0;
    if constexpr (REC) {
        const double* rn = grec + (long)DG_REC * ez0 * N1;                  // node rows
        const double* rz = grec + (long)DG_REC * ((long)nz * N1 + ez0);     // z-faces
#pragma unroll
        for (int k = 0; k < NRL; ++k) {
            const int i = t + k * NTH < BRN * wz * N1 ? t + k * NTH : 0;
            rr[k] = rn[(i / BRN) * DG_REC + i % BRN];
        }
        const int i = t < BRN * (wz + 1) ? t : 0;
        rf = rz[(i / BRN) * DG_REC + i % BRN];
    } else if (t < (BGSUB ? 3 * ROWS : ROWS) + TEZ + 1) {
        // one lane per row; a node row's three flux cases on three lanes
        const bool zr = t < TEZ + 1;   // a z-face row
        const int q = t - (TEZ + 1), v = zr ? 0 : q / ROWS, r = zr ? t : q - v * ROWS;
        if (zr ? r <= wz : r < wz * N1)
            dg_record(A, zr, zr ? ez0 + r : ez0 * N1 + r, v, BGSUB, sB[zr ? ROWS + r : r]);
    }
    // (JVP) the stored terms of the linearization state at the line's low face
    const unsigned fo0 = valid ? (xd ? (unsigned)(((long)(ez0 + lz) * (nx + 1) + ex0 + lx) * N1 + ln)
                                     : (unsigned)(((long)(nx + 1) * nz + (long)(ez0 + lz) * nx + ex0 + lx) * N1 + ln))
                               : 0u;
    double l0[FCN], urho[N1];
    if constexpr (MODE == 3) {
#pragma unroll
        for (int c = 0; c < FCN; ++c) l0[c] = LEAN ? 0.0 : ld(face0 + (long)c * NF, fo0);
    }
    double eps = 0.0;
    if constexpr (MODE == 3) {
        // ||y||^2: yn2p[0], or with ycount > 0 the sum of the ycount block partials at yn2p
        const double yn2 = ycount > 0 ? ysum.sum(yn2p, ycount) : yn1;
        if (!(yn2 > 0.0)) {   // y = 0: the product is 0 (uniform over the grid)
            if (valid && xd)
                for (int c = 0; c < 4; ++c)
                    for (int j = 0; j < N1; ++j) st(out + c * N, n0 + j, 0.0);
            return;
        }
        eps = uniform(eps_mode == 0 ? FdEps<double>::sqrt_eps / sqrt(yn2)
                                    : FdEps<double>::sqrt_eps * sqrt(ut2) / sqrt(yn2));
#pragma unroll
        for (int j = 0; j < N1; ++j) urho[j] = LEAN ? 0.0 : s[0][j];
        // the line of U' + eps y
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < N1; ++j) {
                s[c][j] = s[c][j] + eps * y[c][j];
                if (!LEAN && wv >= 2) h[c][j] = h[c][j] + eps * hy[c][j];
            }
    }

    // ---- T: traces ----
    double tlo[4], dlo[4];   // at the line's low end
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        double a = 0.0, b = 0.0, da = 0.0, db = 0.0;
#pragma unroll
        for (int j = 0; j < N1; ++j) {
            a += R.em[j] * s[c][j];
            b += R.ep[j] * s[c][j];
            if constexpr (NS) {
                da += R.dm[j] * s[c][j];
                db += R.dp[j] * s[c][j];
            }
        }
        tlo[c] = a;
        dlo[c] = da;
        sT[c * NSLOT + t] = b;
        if constexpr (NS) sT[(4 + c) * NSLOT + t] = db;
    }
    if constexpr (LEAN) {
        load_halo();
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < N1; ++j)
                if (wv >= 2) h[c][j] = h[c][j] + eps * hy[c][j];
    }
    if (hslot >= 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double a = 0.0, da = 0.0;
#pragma unroll
            for (int j = 0; j < N1; ++j) {
                a += (hhigh ? R.ep[j] : R.em[j]) * h[c][j];
                if constexpr (NS) da += (hhigh ? R.dp[j] : R.dm[j]) * h[c][j];
            }
            sT[c * NSLOT + hslot] = a;
            if constexpr (NS) sT[(4 + c) * NSLOT + hslot] = da;
        }
    }
    if constexpr (REC) {
#pragma unroll
        for (int k = 0; k < NRL; ++k)
            if (t + k * NTH < BRN * wz * N1) (&sB[0][0])[t + k * NTH] = rr[k];
        if (t < BRN * (wz + 1)) sB[ROWS + t / BRN][t % BRN] = rf;
    }
    __syncthreads();
    // (JVP) the line's stored volume fluxes, read behind the face work
    double v0[4][N1];
    if constexpr (MODE == 3 && !LEAN) {
        const long vo = xd ? 0 : 4 * N;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < N1; ++q) v0[c][q] = ld(vol0 + vo + c * N, n0 + q * (xd ? 1 : N1));
    }

    // ---- F: the face point at the line's low end, and wave 1 the tile's high faces ----
    auto traces = [&](int slot, double (&tr)[4], double (&dn)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            tr[c] = sT[c * NSLOT + slot];
            if constexpr (NS) dn[c] = sT[(4 + c) * NSLOT + slot];
        }
    };
    auto finish = [&](double (&Phi)[4], double (&slo)[3], double (&shi)[3], unsigned fo, const double (&f0)[FCN], int slot) {
        if constexpr (MODE == 5) {
#pragma unroll
            for (int c = 0; c < 4; ++c) st(face0 + (long)c * NF, fo, Phi[c]);
            if constexpr (NS) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    st(face0 + (long)(4 + c) * NF, fo, slo[c]);
                    st(face0 + (long)(7 + c) * NF, fo, shi[c]);
                }
            }
        } else {
            if constexpr (MODE == 3) {
#pragma unroll
                for (int c = 0; c < 4; ++c) Phi[c] -= f0[c];
                if constexpr (NS) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        slo[c] -= f0[4 + c];
                        shi[c] -= f0[7 + c];
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) sF[c * NFS + slot] = Phi[c];
            if constexpr (NS) {
#pragma unroll
                for (int c = 0; c < 3; ++c) sF[(4 + c) * NFS + slot] = slo[c];
            }
        }
    };
    if (valid) {
        const bool first = xd ? lx == 0 : lz == 0;   // the low neighbour is outside the tile
        const int slot = first ? NTH + (xd ? lz * N1 + ln : 2 * NXF + lx * N1 + ln) : t - (xd ? N1 : TEX * N1);
        double tl[4], nl[4], Phi[4], slo[3], shi[3];
        if constexpr (LEAN) {
#pragma unroll
            for (int c = 0; c < FCN; ++c) l0[c] = ld(face0 + (long)c * NF, fo0);
        }
        traces(slot, tl, nl);
        const bool wlo = first && (xd ? ex0 == 0 && !per : ez0 == 0);
        dg_face<NS, BGSUB>(A, tl, nl, tlo, dlo, sB[xd ? lz * N1 + ln : ROWS + lz], xd, wlo, false, Phi, slo, shi);
        finish(Phi, slo, shi, fo0, l0, t);
        if constexpr (NS && MODE != 5) {   // (in LDS rather than held through V)
#pragma unroll
            for (int c = 0; c < 3; ++c) sH[c][t] = shi[c];
        }
    }
    if (wv == 1) {
        const int l = t & 63;
        const bool xf = l < NXF;
        const int q = xf ? l : l - NXF, g = q / N1, r = q - g * N1;
        if (l < NXF + NZF && g < (xf ? wz : wx)) {
            double tl[4], nl[4], th[4], nh[4], Ph[4], sl[3], sh[3], f1[FCN];
            const unsigned fo = xf ? (unsigned)(((long)(ez0 + g) * (nx + 1) + ex0 + wx) * N1 + r)
                                   : (unsigned)(((long)(nx + 1) * nz + (long)(ez0 + wz) * nx + ex0 + g) * N1 + r);
            if constexpr (MODE == 3) {
#pragma unroll
                for (int c = 0; c < FCN; ++c) f1[c] = ld(face0 + (long)c * NF, fo);
            }
            traces(xf ? (g * TEX + wx - 1) * N1 + r : HALF + ((wz - 1) * TEX + g) * N1 + r, tl, nl);
            traces(NTH + (xf ? NXF : 2 * NXF + NZF) + q, th, nh);
            const bool end = xf ? ex0 + wx == nx : ez0 + wz == nz;
            dg_face<NS, BGSUB>(A, tl, nl, th, nh, sB[xf ? g * N1 + r : ROWS + wz], xf, false, end && !(xf && per), Ph, sl,
                               sh);
            // (mode 5: a face between tiles is stored by the tile of its high side)
            if (MODE != 5 || end)
                finish(Ph, sl, sh, fo, f1, NTH + l);
        }
    }

    // ---- V: volume fluxes along the line and their contraction, over the line's scale
    // 2/dx or 2/dz and the node's mass: M^-1 L_h along this direction ----
    double L[4][N1];
    const double r2 = xd ? A.rdx2 : A.rdz2;
    if (valid) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < N1; ++j) L[c][j] = 0.0;
        double pt[N1], ir1[N1], pb1[N1];
#pragma unroll
        for (int q = 0; q < N1; ++q) {
            const double* row = sB[lz * N1 + (xd ? ln : q)];
            ir1[q] = row[BR_IRT];
            pb1[q] = row[BR_P];
        }
        pert_pressures<double, N1, false>(A.gas, s[3], ir1, pb1, pt);
#pragma unroll
        for (int q = 0; q < N1; ++q) {
            const double* row = sB[lz * N1 + (xd ? ln : q)];
            const double mx = row[BR_MX], pb = pb1[q];
            const double Ut[4] = {s[0][q] + row[BR_RHO], s[1][q] + (xd ? mx : 0.0), s[2][q] + (xd ? 0.0 : mx),
                                  s[3][q] + row[BR_RT]};
            const double ir = frcp(Ut[0]);
            const double qn = Ut[1] * ir;
            double F[4] = {Ut[1], Ut[1] * qn + pt[q], Ut[2] * qn, Ut[3] * qn};
            if constexpr (BGSUB) {
                // the background's flux: along z only its pressure
                F[0] -= xd ? mx : 0.0;
                F[1] -= xd ? row[BR_F1] : pb;
                F[3] -= xd ? row[BR_F3] : 0.0;
            }
            if constexpr (NS) {
                // mu (G_c - (U_c/rho) G_rho) with the derivative along the line
                double G[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    double a = 0.0;
#pragma unroll
                    for (int j = 0; j < N1; ++j) a += R.D[q][j] * s[c][j];
                    G[c] = r2 * a;
                }
                if (!xd) {
                    G[0] += row[BR_DRHO];
                    G[2] += row[BR_DMX];
                    G[3] += row[BR_DRT];
                }
#pragma unroll
                for (int c = 1; c < 4; ++c) F[c] -= A.mu * (G[c] - (Ut[c] * ir) * G[0]);
            }
            if constexpr (MODE == 5) {
                const long vo = xd ? 0 : 4 * N;   // this direction's volume fluxes
#pragma unroll
                for (int c = 0; c < 4; ++c) st(vol0 + vo + c * N, n0 + q * (xd ? 1 : N1), F[c]);
            }
            if constexpr (MODE == 3) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    F[c] -= LEAN ? ld(vol0 + (xd ? 0 : 4 * N) + c * N, n0 + q * (xd ? 1 : N1)) : v0[c][q];
            }
            if constexpr (MODE != 5) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int a = 0; a < N1; ++a) L[c][a] += R.lt[a][q] * F[c];
            }
        }
    }
    if constexpr (MODE == 5) return;
    // (JVP) y again, for the output
    if constexpr (MODE == 3) {
        if (xd) {
            dg_line<N1>(opaque(Y), N, n0, true, y);
            if constexpr (LEAN)
#pragma unroll
                for (int j = 0; j < N1; ++j) urho[j] = ld(opaque(U), n0 + j);
        }
    }
    __syncthreads();
    if (valid) {
        // face terms of the line's ends: the high face's from LDS
        const bool last = xd ? lx == wx - 1 : lz == wz - 1;
        const int slot = last ? NTH + (xd ? lz * N1 + ln : NXF + lx * N1 + ln) : t + (xd ? N1 : TEX * N1);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double pl = sF[c * NFS + t], ph = sF[c * NFS + slot];
#pragma unroll
            for (int a = 0; a < N1; ++a) L[c][a] += R.lt[a][4] * pl - R.lt[a][5] * ph;
            if constexpr (NS) {
                if (c > 0) {
                    const double lo = r2 * sH[c - 1][t], hi = r2 * sF[(3 + c) * NFS + slot];
#pragma unroll
                    for (int a = 0; a < N1; ++a) L[c][a] += R.lt[a][7] * hi - R.lt[a][6] * lo;
                }
            }
        }
        if (!xd) {   // (the traces are read no more)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int a = 0; a < N1; ++a)
                    sT[((c == 1 ? 2 : c == 2 ? 1 : c) * EPB + le) * NP + a * N1 + ln] = r2 * L[c][a];
        }
    }
    __syncthreads();

    // ---- D: both directions, gravity and the output, by the x-lines ----
    double nrm = 0.0;
    if (xd && valid) {
        const double sc = MODE == 3 ? adt / eps : 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int a = 0; a < N1; ++a) {
                const unsigned no = n0 + a;
                double v = r2 * L[c][a] + sT[(c * EPB + le) * NP + ln * N1 + a];
                if (c == 2) {
                    // gravity; JVP: of (U' + eps y)_rho - U'_rho
                    if constexpr (MODE == 3) v -= A.g * (s[0][a] - urho[a]);
                    else v -= A.g * s[0][a];
                }
                if constexpr (MODE == 0) st(out + c * N, no, v * (R.w[a] * R.w[ln] * A.J));
                else if constexpr (MODE == 1) st(out + c * N, no, v);
                else if constexpr (MODE == 2) {
                    const double G = s[c][a] - adt * v - ld(Ubar + c * N, no);
                    st(out + c * N, no, G);
                    nrm += G * G;
                } else if constexpr (MODE == 3) {
                    st(out + c * N, no, y[c][a] - sc * v);
                } else {   // explicit Runge-Kutta stage
                    const double base = rk.a0 != 0.0 ? rk.a0 * ld(Ubar + c * N, no) : 0.0;
                    st(out + c * N, no, base + rk.a1 * s[c][a] + rk.c * v);
                }
            }
    }
    if constexpr (MODE == 2)
        if (red.partials) put_partial<NTH>(red, nrm);
}

int dg_grid(int k, int nx, int nz)
{
    return k == 1 ? dg_tiles<2>(nx, nz) : k == 2 ? dg_tiles<3>(nx, nz) : dg_tiles<4>(nx, nz);
}

template <int N1, bool NS, bool RG>
static void launch_dg_n(int mode, const DgArgs& A0, const double* U, const double* Y, const double* Ubar,
                        double* out, const double* yn2, const double* ut2, int eps_mode, double adt, Red red,
                        hipStream_t st, const Mb& mb, const ExStage& ex, int ycount)
{
    DgArgs A = A0;
    A.rdx2 = 2.0 / A.dx;
    A.rdz2 = 2.0 / A.dz;
    A.eta_x = A.c_ip * (double)(N1 * N1) / A.dx;
    A.eta_z = A.c_ip * (double)(N1 * N1) / A.dz;
    const dim3 grid(dg_tiles<N1>(A.nx, A.nz), 1, mb.n), block(DgShape<N1>::NTH);
    auto launch = [&](auto kernel, int yc) {
        timed_launch(kernel, grid, block, st, A, mb.tab, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, mb.ms, ex, yc);
    };
    switch (mode) {
    case 0: launch(dg_kernel<N1, NS, 0, RG, true>, 0); break;
    case 1: launch(dg_kernel<N1, NS, 1, RG, true>, 0); break;
    case 2:
        if constexpr (!RG) {
            if (!A.rec) launch(dg_kernel<N1, NS, 2, false, false>, 0);
            else launch(dg_kernel<N1, NS, 2, false, true>, 0);
        } else {
            launch(dg_kernel<N1, NS, 2, true, true>, 0);
        }
        if (red.out) launch_finalize(red.partials, (int)grid.x, 1, red.out, st, mb);
        break;
    case 4: launch(dg_kernel<N1, NS, 4, RG, true>, 0); break;
    case 5: launch(dg_kernel<N1, NS, 5, RG, true>, 0); break;
    default:
        if constexpr (DG_LEAN<N1, NS>) {
            if ((long)grid.x * mb.n > DG_LEAN_TILES) {
                launch(dg_kernel<N1, NS, 3, RG, true, true>, ycount);
                break;
            }
        }
        launch(dg_kernel<N1, NS, 3, RG, true>, ycount);
        break;
    }
}

template <int N1>
static void launch_dg_k(bool ns, int mode, const DgArgs& A, const double* U, const double* Y, const double* Ubar,
                        double* out, const double* yn2, const double* ut2, int eps_mode, double adt, Red red,
                        hipStream_t st, const Mb& mb, const ExStage& ex, int yc)
{
    if (mb.tab) {
        if (ns) launch_dg_n<N1, true, true>(mode, A, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, st, mb, ex, yc);
        else launch_dg_n<N1, false, true>(mode, A, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, st, mb, ex, yc);
    } else {
        if (ns) launch_dg_n<N1, true, false>(mode, A, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, st, mb, ex, yc);
        else launch_dg_n<N1, false, false>(mode, A, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, st, mb, ex, yc);
    }
}

void launch_dg(int k, bool ns, int mode, const DgArgs& A, const double* U, const double* Y, const double* Ubar,
               double* out, const double* yn2, const double* ut2, int eps_mode, double adt, Red red, hipStream_t st,
               const Mb& mb, const ExStage& ex, int ycount)
{
    if (k == 1) launch_dg_k<2>(ns, mode, A, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, st, mb, ex, ycount);
    else if (k == 2) launch_dg_k<3>(ns, mode, A, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, st, mb, ex, ycount);
    else launch_dg_k<4>(ns, mode, A, U, Y, Ubar, out, yn2, ut2, eps_mode, adt, red, st, mb, ex, ycount);
}

// ---------------------------------------------------------------------------
// Initial data (eq. add-perturbation): theta' inserted at constant pressure.
// ---------------------------------------------------------------------------
template <int N1>
__global__ void __launch_bounds__(256)
init_kernel(DgArgs A, int shape, double amp, double xc, double zc, double xr, double zr, double aa, double Z,
            double x0, double z0, double u_mean, double* __restrict__ U, long ms)
{
    U = mbr(U, ms);
    constexpr int NP = N1 * N1;
    const long n = A.ne * NP;
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const long e = i / NP;
    const int nd = (int)(i - e * NP);
    const int a = nd % N1, b = nd / N1;
    const int ez = (int)(e / A.nx), ex = (int)(e - (long)ez * A.nx);
    const double x = x0 + (ex + 0.5 * (1.0 + A.R.xi[a])) * A.dx;
    const double z = z0 + (ez + 0.5 * (1.0 + A.R.xi[b])) * A.dz;
    double th1 = 0.0;
    if (shape == 0) {
        const double rx = (x - xc) / xr, rz = (z - zc) / zr;
        const double r = sqrt(rx * rx + rz * rz);
        if (r < 1.0) th1 = 0.5 * amp * (1.0 + cos(M_PI * r));
    } else {
        const double s = (x - xc) / aa;
        th1 = amp / (1.0 + s * s) * sin(M_PI * z / Z);
    }
    const int zi = ez * N1 + b;
    const double rt = A.bg_node[zi * 4 + 3], rhob = A.bg_node[zi * 4 + 0], mb = A.bg_node[zi * 4 + 1];
    const double rho = rt / (A.th_node[zi] + th1);
    U[i] = rho - rhob;
    U[n + i] = rho * u_mean - mb;
    U[2 * n + i] = 0.0;
    U[3 * n + i] = 0.0;
}

void launch_initial_state(int k, const DgArgs& A, int shape, double amp, double xc, double zc, double xr, double zr,
                          double a, double Z, double x0, double z0, double u_mean, double* U, hipStream_t st,
                          const Mb& mb)
{
    const long n = A.ne * (k + 1) * (k + 1);
    const dim3 grid((unsigned)((n + 255) / 256), 1, mb.n), block(256);
    if (k == 1) init_kernel<2><<<grid, block, 0, st>>>(A, shape, amp, xc, zc, xr, zr, a, Z, x0, z0, u_mean, U, mb.ms);
    else if (k == 2) init_kernel<3><<<grid, block, 0, st>>>(A, shape, amp, xc, zc, xr, zr, a, Z, x0, z0, u_mean, U, mb.ms);
    else init_kernel<4><<<grid, block, 0, st>>>(A, shape, amp, xc, zc, xr, zr, a, Z, x0, z0, u_mean, U, mb.ms);
}

// sum over all nodes and components of (U' + Ubar)^2
template <int N1, bool RG>
__global__ void __launch_bounds__(256)
norm_total_kernel(DgArgs Aa, const MemberArgs* __restrict__ mt, const double* __restrict__ U, Red red, long ms)
{
    const DgArgs& A = dg_of<RG>(Aa, mt);
    U = mbr(U, ms);
    red = mbr(red, ms);
    constexpr int NP = N1 * N1;
    const long n = sits_out(mt) ? 0 : A.ne * NP;
    const long nb = (n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024;   // this member's work-groups
    double s = 0.0;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += nb * 256) {
        const long e = i / NP;
        const int b = (int)(i - e * NP) / N1;
        const int zi = (int)(e / A.nx) * N1 + b;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double v = U[c * n + i] + A.bg_node[zi * 4 + c];
            s += v * v;
        }
    }
    put_partial<256>(red, s);   // 0 from the work-groups beyond a smaller member
}

int norm_total_grid(long n)
{
    long b = (n + 255) / 256;
    return (int)(b < 1024 ? b : 1024);
}

template <int N1>
static void launch_norm_total_k(const DgArgs& A, const double* U, Red red, hipStream_t st, const Mb& mb, dim3 grid)
{
    if (mb.tab) norm_total_kernel<N1, true><<<grid, dim3(256), 0, st>>>(A, mb.tab, U, red, mb.ms);
    else norm_total_kernel<N1, false><<<grid, dim3(256), 0, st>>>(A, nullptr, U, red, mb.ms);
}

void launch_norm2_total(int k, const DgArgs& A, const double* U, Red red, hipStream_t st, const Mb& mb)
{
    const long n = A.ne * (k + 1) * (k + 1);
    const dim3 grid(norm_total_grid(n), 1, mb.n);
    if (k == 1) launch_norm_total_k<2>(A, U, red, st, mb, grid);
    else if (k == 2) launch_norm_total_k<3>(A, U, red, st, mb, grid);
    else launch_norm_total_k<4>(A, U, red, st, mb, grid);
    launch_finalize(red.partials, (int)grid.x, 1, red.out, st, mb);
}

}  // namespace jfmg
