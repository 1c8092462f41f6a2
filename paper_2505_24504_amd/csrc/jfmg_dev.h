// Device helpers shared by the gfx950 kernels: gas physics, the HLLC flux
// and wave64 / block / multi-block reductions (fixed
// summation order everywhere, no float atomics).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace jfmg {

// sqrt of the unit roundoff used in finite-difference steps: 2^-26 (FP64), 2^-11.5 (FP32)
template <typename T> struct FdEps;
template <> struct FdEps<double> {
    static constexpr double sqrt_eps = 1.4901161193847656e-08;
    static constexpr double inv_sqrt_eps = 1.0 / sqrt_eps;
};
template <> struct FdEps<float> {
    static constexpr double sqrt_eps = 3.4526698300124393e-04;
    static constexpr double inv_sqrt_eps = 1.0 / sqrt_eps;
};

// Gas constants plus the binomial coefficients C(gamma, k) used to evaluate
// the equation of state around the background pressure (see pert_pressure).
constexpr int GAS_NCOEF = 12;
template <typename T> struct Gas {
    T gamma, R, p0;
    T cg[GAS_NCOEF];   // C(gamma, k), k = 0 .. GAS_NCOEF-1
};

template <typename T> __device__ __forceinline__ T dpow(T a, T b)
{
    if constexpr (std::is_same_v<T, float>) return powf(a, b);
    else return pow(a, b);
}
// Square root of a normal number (sound speeds): hardware 1/sqrt estimate; in FP64 one
// coupled Goldschmidt step for g ~ sqrt(a), h ~ 1/(2 sqrt(a)), then two Newton corrections
// g += h (a - g^2), positive arguments only; in FP32, where the estimate is good to one
// ulp, one correction (7 operations instead of the library's 16), and zero and infinity,
// whose estimate is infinite or zero, are their own roots: an FP32 pressure pb + (p - pb)
// rounds to zero where (1 + s)^gamma is below half an ulp of one.  Without the library's
// rescaling of denormal arguments.
template <typename T> __device__ __forceinline__ T psqrt(T a)
{
    if constexpr (std::is_same_v<T, float>) {
        const float y = __builtin_amdgcn_rsqf(a);
        const float g = a * y;
        constexpr int ZERO_INF = 0x260;   // -0, +0, +inf
        return __builtin_amdgcn_classf(a, ZERO_INF) ? a : fmaf(fmaf(-g, g, a), 0.5f * y, g);
    } else {
        const double y = __builtin_amdgcn_rsq(a);
        double g = a * y, h = 0.5 * y;
        const double r = fma(-h, g, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
        double d = fma(-g, g, a);
        g = fma(d, h, g);
        d = fma(-g, g, a);
        return fma(d, h, g);
    }
}
template <typename T> __device__ __forceinline__ T dabs(T a)
{
    if constexpr (std::is_same_v<T, float>) return fabsf(a);
    else return fabs(a);
}

// Element i of an array addressed by a 32-bit byte offset from its base (usually
// wave-uniform, in scalar registers): one vector register per address instead of
// two.  Arrays must be smaller than 4 GiB.
template <typename T> __device__ __forceinline__ T ld(const T* base, unsigned i)
{
    return *(const T*)((const char*)base + i * (unsigned)sizeof(T));
}
template <typename T> __device__ __forceinline__ void st(T* base, unsigned i, T v)
{
    *(T*)((char*)base + i * (unsigned)sizeof(T)) = v;
}

// A device pointer in the global address space: pointers that went through an asm
// statement are not known to be global any more, and loads through them would be flat.
template <typename T> using gptr = const __attribute__((address_space(1))) T*;

// The same (wave-uniform) pointer, opaque to the optimizer: loads through it are
// issued again instead of being merged with earlier loads of the same address,
// whose values would otherwise be held in registers in between.
template <typename T> __device__ __forceinline__ const T* opaque(const T* p)
{
    gptr<T> g = (gptr<T>)p;
    asm volatile("" : "+s"(g));
    return (const T*)g;
}

// A value that is the same in every lane of the wave, moved to scalar registers
// (keeps it out of the vector register budget).
__device__ __forceinline__ double uniform(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Reciprocal from the hardware estimate refined by Newton's iteration for 1/a,
// r <- r + r (1 - a r): the FP64 estimate (relative error ~5e-8) needs two steps
// to reach the accuracy of a correctly rounded division (measured: within one ulp,
// equal to it for >99.9 % of inputs); the FP32 estimate is accurate to one ulp.
// Shorter dependency chain than the IEEE division sequence.  a must be a finite,
// nonzero normal number (densities and HLLC wave-speed differences are).
template <typename T> __device__ __forceinline__ T frcp(T a)
{
    if constexpr (std::is_same_v<T, float>) {
        return __builtin_amdgcn_rcpf(a);
    } else {
        double r = __builtin_amdgcn_rcp(a);
        double e = fma(-a, r, 1.0);
        r = fma(r, e, r);
        e = fma(-a, r, 1.0);
        return fma(r, e, r);
    }
}

// Equation of state of the potential-temperature form, p = p0 (R rho theta / p0)^gamma,
// evaluated at the total states rho theta = rtb (1 + s), s = (rho theta)' / rtb, as
// p = pb (1 + s)^gamma with the background pressure pb = p0 (R rtb / p0)^gamma, for n
// states at once: p (DEV false) or the deviation p - pb (DEV true: accurate to the unit
// roundoff of p - pb rather than of p; FP32 FV operators, whose values enter only
// differences of two evaluations, carry p - pb where the pressure enters additively).
// (1 + s)^gamma is the binomial series, 12 terms in FP64 and 7 in FP32, truncated below
// the unit roundoff for |s| <= 1/20 and 1 < gamma <= 5/3 (<= 3e-19 in FP64), pow
// beyond.  It is summed as 1 + s g(s) with g in pairs (Estrin): the last step alone
// rounds at the scale of the result, as in Horner's form, but four operations deep
// instead of eleven, and without a branch on |s| that would cut the flux evaluations
// around it in pieces (a face point of the DG kernel spent 1100 of its 4000 cycles in
// the branched Horner form).  s = 0 returns pb (0) exactly, so background and perturbed
// evaluations agree bitwise.  The general power is one copy for all n states, as a rare
// branch after them.
template <typename T, int n, bool DEV>
__device__ __forceinline__ void pert_pressures(const Gas<T>& G, const T (&rt1)[n], const T (&irtb)[n], const T (&pb)[n],
                                               T (&out)[n])
{
    bool far = false;
#pragma unroll
    for (int q = 0; q < n; ++q) {
        const T s = rt1[q] * irtb[q];
        const T* c = G.cg;
        const T s2 = s * s;
        const T s4 = s2 * s2;
        T g;
        if constexpr (std::is_same_v<T, float>) {
            g = (c[1] + c[2] * s) + (c[3] + c[4] * s) * s2 + (c[5] + c[6] * s) * s4;
        } else {
            static_assert(GAS_NCOEF == 12, "series length");
            const T lo = (c[1] + c[2] * s) + (c[3] + c[4] * s) * s2;
            const T mi = (c[5] + c[6] * s) + (c[7] + c[8] * s) * s2;
            const T hi = (c[9] + c[10] * s) + c[11] * s2;
            g = lo + (mi + hi * s4) * s4;
        }
        if constexpr (DEV) out[q] = pb[q] * (g * s);
        else out[q] = pb[q] * (T(1) + g * s);
        far = far || !(dabs<T>(s) <= T(0.05));
    }
    if (far) {
#pragma unroll 1
        for (int q = 0; q < n; ++q) {
            T s = rt1[0] * irtb[0], p = pb[0];
#pragma unroll
            for (int r = 1; r < n; ++r) {
                s = q == r ? rt1[r] * irtb[r] : s;
                p = q == r ? pb[r] : p;
            }
            if (!(dabs<T>(s) <= T(0.05))) {
                T f = dpow<T>(T(1) + s, G.gamma);
                if constexpr (DEV) f = f - T(1);
                const T v = p * f;
#pragma unroll
                for (int r = 0; r < n; ++r) out[r] = q == r ? v : out[r];
            }
        }
    }
}

// HLLC flux (Toro) through a Cartesian face in its frame (component 1 the momentum along the
// positive normal, 2 the tangential one), Davis wave speeds S_L = min(q_L - c_L, q_R - c_R),
// S_R = max(q_L + c_L, q_R + c_R); star flux in the S*-factored form
// (S*(S_K U_K - F_K) + S_K p*_K e_1) / (S_K - S*), p*_K = p_K + rho_K (S_K - q_K)(S* - q_K).
// 1/rho of both states is given (the callers reuse it).
// A face with the opposite normal is the mirror case, H(a, b; -e) = -H(b, a; +e), so every
// Cartesian face (slip walls included, via a mirrored ghost state) needs only this form.
// Without branches: the supersonic cases take the physical flux of the side that the
// star flux is built on, so that one basic block holds the face and its long dependency
// chain overlaps the work around it.
__device__ __forceinline__ void hllc(const Gas<double>& G, const double* UL, const double* UR, double pL, double pR,
                                     double irL, double irR, double* F)
{
    const double rL = UL[0], rR = UR[0];
    const double qL = UL[1] * irL, qR = UR[1] * irR;
    const double cL = psqrt<double>(G.gamma * pL * irL), cR = psqrt<double>(G.gamma * pR * irR);
    const double SL = fmin(qL - cL, qR - cR);
    const double SR = fmax(qL + cL, qR + cR);
    const double Ss =
        (pR - pL + rL * qL * (SL - qL) - rR * qR * (SR - qR)) * frcp<double>(rL * (SL - qL) - rR * (SR - qR));
    const bool supL = SL >= 0.0, supR = SR <= 0.0;
    const bool lk = supL | (!supR & (Ss >= 0.0));
    const double SK = lk ? SL : SR, rK = lk ? rL : rR, qK = lk ? qL : qR, pK = lk ? pL : pR;
    const double u1 = lk ? UL[1] : UR[1], u2 = lk ? UL[2] : UR[2], u3 = lk ? UL[3] : UR[3];
    const double F1 = u1 * qK + pK, F2 = u2 * qK, F3 = u3 * qK;   // the physical flux (first component: u1)
    const double pst = pK + rK * (SK - qK) * (Ss - qK);
    const double iden = frcp<double>(SK - Ss);
    const double G0 = (Ss * (SK * rK - u1)) * iden;
    const double G1 = (Ss * (SK * u1 - F1) + SK * pst) * iden;
    const double G2 = (Ss * (SK * u2 - F2)) * iden;
    const double G3 = (Ss * (SK * u3 - F3)) * iden;
    const bool sup = supL | supR;
    F[0] = sup ? u1 : G0;
    F[1] = sup ? F1 : G1;
    F[2] = sup ? F2 : G2;
    F[3] = sup ? F3 : G3;
}

// ---------------------------------------------------------------------------
// Reductions, in a fixed order everywhere: the wave, then the waves in their order.
// ---------------------------------------------------------------------------

// Value of another lane by data-parallel primitives (VALU moves; a shuffle goes through
// LDS, 120 cycles a step): control CTRL over the rows of ROWS, 0 where no lane is read.
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_move(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)b, CTRL, ROWS, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(b >> 32), CTRL, ROWS, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Sum over the wave's 64 lanes, in every lane (scalar registers).  All lanes must take
// part.  Inclusive sums in each row of 16 lanes (shifts by 1, 2, 4, 8), then of the rows
// (lane 15 of rows 0 and 2 to rows 1 and 3, lane 31 to rows 2 and 3): lane 63 has all.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_move<0x111, 0xf>(v);
    v += dpp_move<0x112, 0xf>(v);
    v += dpp_move<0x114, 0xf>(v);
    v += dpp_move<0x118, 0xf>(v);
    v += dpp_move<0x142, 0xa>(v);
    v += dpp_move<0x143, 0xc>(v);
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, 63), hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), 63);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

// Block sum over NTH threads (a multiple of 64); result valid in thread 0.
template <int NTH> __device__ __forceinline__ double block_sum(double v, double* sh)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < NTH / 64; ++i) s += sh[i];
    __syncthreads();
    return s;
}
template <int NTH> __device__ __forceinline__ double block_max(double v, double* sh)
{
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < NTH / 64; ++i) s = fmax(s, sh[i]);
    __syncthreads();
    return s;
}

// Multi-block reductions without tickets or fences: every block writes its
// partial with a plain store; the partials are summed in a fixed order either
// by a one-block finalize kernel launched right after the producer (scalars the
// host or a later kernel reads) or by each block of the consuming kernel
// itself (PartialSum).  Kernel boundaries make the partials visible; no
// agent-scope fence is executed per block.
struct Red {
    double* partials;   // [nq][number of blocks]
    double* out;        // if non-null the launcher finalizes into out[0..nq)
};

__device__ __forceinline__ unsigned block_linear() { return blockIdx.y * gridDim.x + blockIdx.x; }

// The dispatcher hands work-groups to the 8 XCDs of the chip round-robin by
// linear id, and each XCD has its own L2.  Stencil kernels therefore renumber
// their tiles so that XCD x works on one contiguous range of tiles (rows of
// neighbouring tiles share halo cache lines inside one L2).  Bijective on [0, nb).
constexpr unsigned NUM_XCD = 8;
__device__ __forceinline__ unsigned xcd_tile(unsigned w, unsigned nb)
{
    const unsigned x = w % NUM_XCD, i = w / NUM_XCD, q = nb / NUM_XCD, r = nb % NUM_XCD;
    return x * q + (x < r ? x : r) + i;
}

template <int NTH> __device__ __forceinline__ void put_partial(const Red& r, double v)
{
    __shared__ double sh[NTH / 64];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < NTH / 64; ++i) s += sh[i];
        r.partials[block_linear()] = s;
    }
}

// Lock-step batches: member m of a batched problem lives m * ms bytes after
// member 0 (identical layouts); kernels run with gridDim.z = members and shift
// every per-member pointer by blockIdx.z * ms (ms = 0 for a single problem).
template <typename P> __device__ __forceinline__ P* mbr(P* p, long ms)
{
    return p ? (P*)((char*)p + (long)blockIdx.z * ms) : p;
}
__device__ __forceinline__ Red mbr(Red r, long ms) { return Red{mbr(r.partials, ms), mbr(r.out, ms)}; }

// A uniform value that another kernel wrote, read by a vector load.  The compiler would
// make it a scalar load; scalar loads return out of order, so the first wait for any of
// the kernel's arguments would also wait for this one's trip to memory.
template <typename T> __device__ __forceinline__ T ldv(const T* p)
{
    int z = 0;
    asm volatile("" : "+v"(z));
    return p[z];
}

// Deterministic sum of n partials, returned to every thread of the block; once per
// kernel.  load() issues the first loads, so that a kernel can issue its other loads
// behind them; sum() waits for them.  The order: entry i belongs to lane i mod 64 and
// wave (i / 64) mod NW of a block of NW waves; each lane of each wave adds its entries in
// turn, then each lane over the waves, then the lanes.  Up to 256 entries every wave
// holds them all and follows that order by itself, without an exchange through LDS; more
// are split over the block.  (Entries of zero at the end change nothing: a ragged batch
// passes the count of its largest member.)
template <int NTH> struct PartialSum {
    static constexpr int NW = NTH / 64, NV = 4;
    double v[NV];
    __device__ __forceinline__ void load(const double* p, int n)
    {
        const bool whole = n <= 64 * NV;
        const int i0 = whole ? (int)threadIdx.x & 63 : (int)threadIdx.x, st = whole ? 64 : NTH;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int i = i0 + k * st;
            const double x = p[i < n ? i : 0];   // (no branch: the wait for them would also
            v[k] = i < n ? x : 0.0;              // wait for the loads behind them)
        }
    }
    // with sh: through these NTH doubles of the caller's LDS
    __device__ __forceinline__ double sum(const double* p, int n)
    {
        __shared__ double sh[NTH];
        return sum(p, n, sh);
    }
    __device__ __forceinline__ double sum(const double* p, int n, double* sh)
    {
        double s;
        if (n <= 64 * NV) {
            double w[NW < NV ? NW : NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                if (k < NW) w[k] = v[k];
                else w[k % NW] += v[k];
            }
            s = w[0];
#pragma unroll
            for (int k = 1; k < (NW < NV ? NW : NV); ++k) s += w[k];
        } else {
            double a = ((v[0] + v[1]) + v[2]) + v[3];
            for (int i0 = threadIdx.x + NV * NTH; i0 < n; i0 += 8 * NTH) {   // eight loads in flight
                double x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int i = i0 + k * NTH;
                    const double y = p[i < n ? i : 0];
                    x[k] = i < n ? y : 0.0;
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) a += x[k];
            }
            const int lane = threadIdx.x & 63;
            sh[threadIdx.x] = a;
            __syncthreads();
            s = sh[lane];
#pragma unroll
            for (int k = 1; k < NW; ++k) s += sh[64 * k + lane];
        }
        return wave_sum(s);
    }
};

}  // namespace jfmg
