// FP64 vector kernels of the FGMRES Arnoldi process (classical Gram-Schmidt,
// re-orthogonalized where the first pass cancels most of w): multi-dot products <w, v_i> of one vector
// against the whole basis in a single pass, the basis update w -= V h, scaling,
// and the final combination delta = Z y.  Streaming, HBM bound; every
// reduction is two-level with a fixed summation order (run-to-run identical).
#include "jfmg_internal.h"

#include <algorithm>

namespace jfmg {

constexpr int LA_NTH = 256, LA_EL = 4;   // threads per block, elements per thread
constexpr int UPDATE2_GROUPS = 1024;     // work-groups of the second Gram-Schmidt pass
constexpr int LA_FILL = 2048;            // blocks up to which the multi-dot splits its groups

int la_blocks(long n)
{
    return (int)((n + (long)LA_NTH * LA_EL - 1) / ((long)LA_NTH * LA_EL));
}

// out[q] = sum_b p[q * nb + b], one block per q, fixed order; with host (pinned) also host[m * entries + q], which saves the gather launch of a sum that only the
// host waits for (stage residual and its norm at 1024x256 nodes 28.7 -> 27.5 us)
__global__ void __launch_bounds__(256)
finalize_kernel(const double* __restrict__ p, int nb, double* __restrict__ out, long ms, double* __restrict__ host)
{
    p = mbr(p, ms);
    out = mbr(out, ms);
    __shared__ double sh[4];
    const int q = blockIdx.x;
    // eight loads in flight per thread
    const double* pq = p + (long)q * nb;
    double a = 0.0;
    for (int i0 = 0; i0 < nb; i0 += 8 * 256) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int i = i0 + k * 256 + (int)threadIdx.x;
            const double x = pq[i < nb ? i : 0];
            v[k] = i < nb ? x : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) a += v[k];
    }
    a = block_sum<256>(a, sh);
    if (threadIdx.x == 0) {
        out[q] = a;
        if (host) host[blockIdx.z * gridDim.x + q] = a;
    }
}

void launch_finalize(const double* partials, int nb, int nq, double* out, hipStream_t st, const Mb& mb, double* host)
{
    finalize_kernel<<<dim3(nq, 1, mb.n), dim3(256), 0, st>>>(partials, nb, out, mb.ms, host);
}

// Scalars between the device slots of every member and coherent pinned host
// memory, by kernels (no copy engine): gather host[m * count + i] = slot_m[i],
// scatter slot_m[i] = host[m * hstride + i].
__global__ void __launch_bounds__(64) gather_kernel(const double* __restrict__ src, int count, double* __restrict__ host,
                                                    long ms)
{
    src = mbr(src, ms);
    host += (long)blockIdx.z * count;
    for (int i = threadIdx.x; i < count; i += 64) host[i] = src[i];
}

__global__ void __launch_bounds__(64) scatter_kernel(double* __restrict__ dst, int count, const double* __restrict__ host,
                                                     long hstride, long ms)
{
    dst = mbr(dst, ms);
    host += (long)blockIdx.z * hstride;
    for (int i = threadIdx.x; i < count; i += 64) dst[i] = host[i];
}

void launch_gather(const double* src, int count, double* host, hipStream_t st, const Mb& mb)
{
    gather_kernel<<<dim3(1, 1, mb.n), dim3(64), 0, st>>>(src, count, host, mb.ms);
}

void launch_scatter(double* dst, int count, const double* host, long hstride, hipStream_t st, const Mb& mb)
{
    scatter_kernel<<<dim3(1, 1, mb.n), dim3(64), 0, st>>>(dst, count, host, hstride, mb.ms);
}

__global__ void __launch_bounds__(256)
norm2_kernel(const double* __restrict__ x, long n, Red red, long ms, const MemberArgs* __restrict__ mt)
{
    x = mbr(x, ms);
    red = mbr(red, ms);
    n = len_of(n, mt);
    const long nb = (n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024;   // this member's work-groups
    double s = 0.0;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += nb * 256) s += x[i] * x[i];
    put_partial<256>(red, s);
}

void launch_norm2(const double* x, long n, Red red, hipStream_t st, const Mb& mb)
{
    long b = (n + 255) / 256;
    const int nb = (int)(b < 1024 ? b : 1024);
    norm2_kernel<<<dim3(nb, 1, mb.n), dim3(256), 0, st>>>(x, n, red, mb.ms, mb.tab);
    if (red.out) launch_finalize(red.partials, nb, 1, red.out, st, mb);
}

// Element k of the thread at base = block start + t (wave-wide loads of 512 contiguous bytes).
__device__ __forceinline__ long la_el(long base, int k) { return base + (long)k * LA_NTH; }
__device__ __forceinline__ void ld_els(const double* __restrict__ x, long base, double (&v)[LA_EL])
{
#pragma unroll
    for (int k = 0; k < LA_EL; ++k) v[k] = x[la_el(base, k)];
}

// v of lane l (l wave-uniform), in scalar registers
__device__ __forceinline__ double lane_value(double v, int l)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, l), hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// <w, v_i> for i < nv (and <w, w> as entry nv when self is set) over one block of w, which
// stays in registers: the basis vectors come in groups of G, the next group's loads in
// flight while the current one is reduced (the wave's sums; one LDS exchange at the end
// combines the waves); the block partials [v][block] are summed by the finalize kernel.
// Grids too small to fill the chip split the groups over blockIdx.y, into LA_FILL blocks at
// most (mean launch of a step, us, unsplit and so: 6.8 and 5.5 with 128 blocks, 8.0 and 7.4
// with 256, 11.9 and 11.6 with 512, 18.9 and 19.3 with 1024; twice as many: 19.9 with 1024).
__global__ void __launch_bounds__(LA_NTH)
multidot_kernel(const double* __restrict__ w, const double* __restrict__ V, long ld, int nv, int self, long n, Red red,
                long ms, const MemberArgs* __restrict__ mt)
{
    constexpr int NW = LA_NTH / 64, G = 4;
    n = len_of(n, mt);   // a ragged member's length: blocks beyond it store zero partials
    __shared__ double sh[NW][65];
    w = mbr(w, ms);
    V = mbr(V, ms);
    red = mbr(red, ms);
    const int nt = nv + self;
    const long b0 = (long)blockIdx.x * LA_NTH * LA_EL, base = b0 + threadIdx.x;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const bool whole = b0 + LA_NTH * LA_EL <= n;
    double wv[LA_EL];
    if (whole) {
        ld_els(w, base, wv);
    } else {
#pragma unroll
        for (int k = 0; k < LA_EL; ++k) wv[k] = la_el(base, k) < n ? w[la_el(base, k)] : 0.0;
    }
    auto load = [&](int v0, double (&a)[G][LA_EL]) {
        if (whole) {
#pragma unroll
            for (int q = 0; q < G; ++q) ld_els(V + (long)min(v0 + q, nv - 1) * ld, base, a[q]);
        } else {
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int k = 0; k < LA_EL; ++k)
                    a[q][k] = la_el(base, k) < n ? V[(long)min(v0 + q, nv - 1) * ld + la_el(base, k)] : 0.0;
        }
    };
    auto dots = [&](int v0, const double (&a)[G][LA_EL]) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < LA_EL; ++k) s += wv[k] * a[q][k];
            s = wave_sum(s);
            if (lane == 0 && v0 + q < nv) sh[wid][v0 + q] = s;
        }
    };
    const int step = G * (int)gridDim.y;
    int v0 = G * (int)blockIdx.y;
    if (v0 < nv) {
        double a[G][LA_EL], b[G][LA_EL];
        load(v0, a);
        for (; v0 < nv; v0 += 2 * step) {
            if (v0 + step < nv) load(v0 + step, b);
            dots(v0, a);
            if (v0 + step >= nv) break;
            if (v0 + 2 * step < nv) load(v0 + 2 * step, a);
            dots(v0 + step, b);
        }
    }
    if (self && blockIdx.y == 0) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < LA_EL; ++k) s += wv[k] * wv[k];
        s = wave_sum(s);
        if (lane == 0) sh[wid][nv] = s;
    }
    __syncthreads();
    const int e = threadIdx.x;
    // this block's entries: its groups', and <w, w> in the first row
    if (e < nt && (e == nv ? blockIdx.y == 0 : (e / G) % (int)gridDim.y == (int)blockIdx.y)) {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < NW; ++r) s += sh[r][e];
        red.partials[(long)e * gridDim.x + blockIdx.x] = s;
    }
}

void launch_multidot(const double* w, const double* V, long ld, int nv, int self, long n, Red red, hipStream_t st,
                     const Mb& mb)
{
    const int nb = la_blocks(n), ng = (nv + 3) / 4;
    const int gy = std::min(ng, std::max(1, LA_FILL / (nb * mb.n)));
    timed_launch(multidot_kernel, dim3(nb, gy, mb.n), dim3(LA_NTH), st, w, V, ld, nv, self, n, red, mb.ms, mb.tab);
    if (red.out) launch_finalize(red.partials, nb, nv + self, red.out, st, mb);
}

// w -= sum_v h[v] V_v.
// With dots (the first pass) the gate g2 of the second pass decides: where it opens, the
// kernel goes on to that pass's multi-dot <w, v_q> of the w it has just formed, still in
// registers: the block partials at dots[q * gridDim.x + blockIdx.x], with the multi-dot
// kernel's products, order and partial layout (its launch, one kernel per iteration, is
// saved); where it stays closed, work-group 0 stores ||w||^2 after this pass, by Pythagoras,
// to pub.out and publishes (first thing, so that its loads and host stores overlap the update).
// Publishing stores the scalar block pub.src[0..ns) to host-visible pinned memory, entry idx
// replaced by pub.out's value, entry fidx by 1 where the second pass ran (else 0) and, where
// the gate is closed, entries zoff .. zoff+zn (the skipped pass's coefficients) by 0, so the
// host reads the Hessenberg column after the iteration's completion event without a separate
// copy.  (h lies in that block and is not restrict.)
__global__ void __launch_bounds__(LA_NTH)
update_kernel(double* __restrict__ w, const double* __restrict__ V, long ld, int nv, long n,
              double* h, long ms, const MemberArgs* __restrict__ mt, const double* __restrict__ hpart,
              int hnb, Gate g2, double* __restrict__ dots, Publish pub)
{
    constexpr int G = 4;
    n = len_of(n, mt);
    g2.h = mbr(g2.h, ms);
    pub.out = mbr(pub.out, ms);
    pub.src = mbr(pub.src, ms);
    pub.host += (long)blockIdx.z * pub.host_stride;
    w = mbr(w, ms);
    V = mbr(V, ms);
    h = mbr(h, ms);
    const int lane = threadIdx.x & 63;
    const long b0 = (long)blockIdx.x * LA_NTH * LA_EL, base = b0 + threadIdx.x;
    const bool whole = b0 + LA_NTH * LA_EL <= n;
    // coefficient v in lane v of every wave
    double hl = 0.0, before = 0.0, acc[LA_EL], a[G][LA_EL], b[G][LA_EL];
    if (!hpart) {
        hl = h[min(lane, nv - 1)];
        before = ldv(g2.h + nv);
    }
    auto load = [&](int v0, double (&x)[G][LA_EL]) {   // (beyond nv: the last vector, not used)
        if (whole) {
#pragma unroll
            for (int q = 0; q < G; ++q) ld_els(V + (long)min(v0 + q, nv - 1) * ld, base, x[q]);
        } else {
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int k = 0; k < LA_EL; ++k)
                    x[q][k] = la_el(base, k) < n ? V[(long)min(v0 + q, nv - 1) * ld + la_el(base, k)] : 0.0;
        }
    };
    if (whole) {
        ld_els(w, base, acc);
    } else {
#pragma unroll
        for (int k = 0; k < LA_EL; ++k) acc[k] = la_el(base, k) < n ? w[la_el(base, k)] : 0.0;
    }
    load(0, a);
    bool dots2 = false;
    __shared__ double hs[65];
    if (hpart) {
        // the multi-dot's partials (at most 128 per entry), in the finalize kernel's order
        hpart = mbr(hpart, ms);
        for (int q0 = threadIdx.x >> 6; q0 <= nv; q0 += 4 * (LA_NTH / 64)) {
            double p0[4], p1[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double* p = hpart + (long)min(q0 + r * (LA_NTH / 64), nv) * hnb;
                p0[r] = p[min(lane, hnb - 1)];
                p1[r] = p[min(lane + 64, hnb - 1)];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int q = q0 + r * (LA_NTH / 64);
                const double t = wave_sum(lane < hnb ? p0[r] : 0.0) + wave_sum(lane + 64 < hnb ? p1[r] : 0.0);
                if (lane == 0 && q <= nv) hs[q] = t;
            }
        }
        __syncthreads();
        hl = hs[min(lane, nv - 1)];
        before = hs[nv];
        if (blockIdx.x == 0) {
            if ((int)threadIdx.x <= nv) h[threadIdx.x] = hs[threadIdx.x];
            __syncthreads();   // (published below)
        }
    }
    if (dots) {
        // gate_after from the coefficients that every wave holds
        const double after = before - wave_sum(lane < nv ? hl * hl : 0.0);
        dots2 = after < g2.tau2 * before;   // gate_open's decision
        if (!dots2 && blockIdx.x == 0) {
            if (threadIdx.x == 0) pub.out[0] = after;
            for (int i = threadIdx.x; i < pub.ns; i += LA_NTH)
                pub.host[i] = (i == pub.idx)                             ? after
                              : (i == pub.fidx)                          ? 0.0
                              : (i >= pub.zoff && i < pub.zoff + pub.zn) ? 0.0
                                                                         : pub.src[i];
        }
    }
    auto subtract = [&](int v0, const double (&x)[G][LA_EL]) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const double hv = v0 + q < nv ? lane_value(hl, min(v0 + q, nv - 1)) : 0.0;
            if (v0 + q < nv)
#pragma unroll
                for (int k = 0; k < LA_EL; ++k) acc[k] -= hv * x[q][k];
        }
    };
    for (int v0 = 0; v0 < nv; v0 += 2 * G) {   // the next group's loads in flight
        if (v0 + G < nv) load(v0 + G, b);
        subtract(v0, a);
        if (v0 + G >= nv) break;
        if (v0 + 2 * G < nv) load(v0 + 2 * G, a);
        subtract(v0 + G, b);
    }
#pragma unroll
    for (int k = 0; k < LA_EL; ++k)
        if (la_el(base, k) < n) w[la_el(base, k)] = acc[k];
    if (!dots2) return;
    dots = mbr(dots, ms);
    constexpr int NW = LA_NTH / 64;
    __shared__ double sd[NW][G];
    const int wid = threadIdx.x >> 6;
    if (!whole) {   // (entries beyond the vector: zeros)
#pragma unroll
        for (int k = 0; k < LA_EL; ++k) acc[k] = la_el(base, k) < n ? acc[k] : 0.0;
    }
    for (int v0 = 0; v0 < nv; v0 += G) {
        load(v0, a);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < LA_EL; ++k) t += acc[k] * a[q][k];
            t = wave_sum(t);
            if (lane == 0) sd[wid][q] = t;
        }
        __syncthreads();
        if ((int)threadIdx.x < G && v0 + (int)threadIdx.x < nv) {
            double t = 0.0;
#pragma unroll
            for (int r = 0; r < NW; ++r) t += sd[r][threadIdx.x];
            dots[(long)(v0 + threadIdx.x) * gridDim.x + blockIdx.x] = t;
        }
        __syncthreads();
    }
}

void launch_update(double* w, const double* V, long ld, int nv, long n, double* h, hipStream_t st, const Mb& mb, Gate g2,
                   double* dots, const Publish& pub, const double* hpart)
{
    timed_launch(update_kernel, dim3(la_blocks(n), 1, mb.n), dim3(LA_NTH), st, w, V, ld, nv, n, h, mb.ms, mb.tab, hpart,
                 la_blocks(n), g2, dots, pub);
}

// The gated second Gram-Schmidt pass together with the iteration's last reduction and its
// publication (pub), in one launch.  Where the gate is open h is not given but formed by every
// work-group from the multi-dot's hnb block partials per entry at hpart (lane-strided sums and
// the wave sum, a fixed order; work-group 0 stores it to hout), each work-group updates its
// blocks of w and stores their ||w||^2 partials in red; the last work-group to finish (a
// release fence and a counter in device memory, so no work-group waits for another) sums the
// partials in a fixed order into pub.out, publishes, and clears the counter for the next
// launch.  Where it is closed every work-group returns at once: there are at most
// UPDATE2_GROUPS of them over all members, each taking blocks of w in turn (with one per
// block, 9216 of them, the closed gate, the usual case, took 12 us; 1024 of them 5.7).
__global__ void __launch_bounds__(LA_NTH)
update2_kernel(double* __restrict__ w, const double* __restrict__ V, long ld, int nv, long n, Gate gate, Red red,
               long ms, const MemberArgs* __restrict__ mt, const double* __restrict__ hpart, int hnb,
               double* hout, Publish pub)
{
    constexpr int G = 4;
    __shared__ double hs[64], sh[LA_NTH / 64], total;
    __shared__ bool last;
    n = len_of(n, mt);
    gate.h = mbr(gate.h, ms);
    if (!gate_open(gate)) return;   // every lane takes part in the gate's wave sum
    pub.out = mbr(pub.out, ms);
    pub.src = mbr(pub.src, ms);
    pub.cnt = mbr(pub.cnt, ms);
    pub.host += (long)blockIdx.z * pub.host_stride;
    w = mbr(w, ms);
    V = mbr(V, ms);
    red = mbr(red, ms);
    hpart = mbr(hpart, ms);
    const int lane = threadIdx.x & 63;
    for (int q = threadIdx.x >> 6; q < nv; q += LA_NTH / 64) {
        double t = 0.0;
        for (int i = lane; i < hnb; i += 64) t += hpart[(long)q * hnb + i];
        t = wave_sum(t);
        if (lane == 0) hs[q] = t;
    }
    __syncthreads();
    const double hl = hs[min(lane, nv - 1)];   // coefficient v in lane v of every wave
    if (blockIdx.x == 0 && (int)threadIdx.x < nv) mbr(hout, ms)[threadIdx.x] = hl;
    for (int blk = blockIdx.x; blk < hnb; blk += gridDim.x) {
        const long base = (long)blk * LA_NTH * LA_EL + threadIdx.x;
        double acc[LA_EL];
        long el[LA_EL];   // (beyond the vector: its first elements, not stored)
#pragma unroll
        for (int k = 0; k < LA_EL; ++k) el[k] = la_el(base, k) < n ? la_el(base, k) : 0;
#pragma unroll
        for (int k = 0; k < LA_EL; ++k) acc[k] = w[el[k]];
        for (int v0 = 0; v0 < nv; v0 += G) {
            double a[G][LA_EL];
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int k = 0; k < LA_EL; ++k) a[q][k] = V[(long)min(v0 + q, nv - 1) * ld + el[k]];
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const double hv = lane_value(hl, min(v0 + q, nv - 1));
                if (v0 + q < nv)
#pragma unroll
                    for (int k = 0; k < LA_EL; ++k) acc[k] -= hv * a[q][k];
            }
        }
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < LA_EL; ++k)
            if (la_el(base, k) < n) {
                w[el[k]] = acc[k];
                s += acc[k] * acc[k];
            }
        s = block_sum<LA_NTH>(s, sh);   // in thread 0; ends with a barrier
        if (threadIdx.x == 0) red.partials[blk] = s;
    }
    if (threadIdx.x == 0) {
        // release: this work-group's partials (and work-group 0's hout) before its count
        // (no cache invalidation, which the other work-groups' reads of hpart would pay)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        last = atomicAdd(pub.cnt, 1ull) == (unsigned long long)(gridDim.x - 1);
    }
    __syncthreads();
    if (!last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // every work-group's partials after its count
    double t = 0.0;
    for (int i = threadIdx.x; i < hnb; i += LA_NTH) t += red.partials[i];
    t = block_sum<LA_NTH>(t, sh);   // in thread 0
    if (threadIdx.x == 0) {
        pub.out[0] = t;
        total = t;
        atomicExch(pub.cnt, 0ull);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < pub.ns; i += LA_NTH)
        pub.host[i] = (i == pub.idx) ? total : (i == pub.fidx) ? 1.0 : pub.src[i];
}

void launch_update2_publish(double* w, const double* V, long ld, int nv, long n, Gate gate, const double* hpart,
                            double* hout, double* wpart, const Publish& pub, hipStream_t st, const Mb& mb)
{
    const int nb = la_blocks(n), g = std::min(nb, std::max(1, UPDATE2_GROUPS / mb.n));
    timed_launch(update2_kernel, dim3(g, 1, mb.n), dim3(LA_NTH), st, w, V, ld, nv, n, gate, Red{wpart, nullptr}, mb.ms,
                 mb.tab, hpart, nb, hout, pub);
}

__global__ void __launch_bounds__(256)
scale_kernel(double* __restrict__ out, const double* __restrict__ in, long n, const double* __restrict__ nrm2,
             double sgn, long ms, const MemberArgs* __restrict__ mt)
{
    n = len_of(n, mt);
    out = mbr(out, ms);
    in = mbr(in, ms);
    nrm2 = mbr(nrm2, ms);
    const double s = sgn / sqrt(nrm2[0]);
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) out[i] = in[i] * s;
}

// out = sgn * in / sqrt(nrm2[0]) (per member)
void launch_scale(double* out, const double* in, long n, const double* nrm2, hipStream_t st, double sgn,
                  const Mb& mb)
{
    long b = (n + 255) / 256;
    scale_kernel<<<dim3((unsigned)(b < 4096 ? b : 4096), 1, mb.n), dim3(256), 0, st>>>(out, in, n, nrm2, sgn, mb.ms,
                                                                                       mb.tab);
}

__global__ void __launch_bounds__(LA_NTH)
lincomb_kernel(double* out, const double* base_, const double* __restrict__ Z, long ld, int nv, long n,
               const double* __restrict__ y, long ms, const MemberArgs* __restrict__ mt)
{
    n = len_of(n, mt);
    out = mbr(out, ms);
    base_ = mbr(base_, ms);
    Z = mbr(Z, ms);
    y = mbr(y, ms);
    constexpr int G = 4;
    const int lane = threadIdx.x & 63;
    const long b0 = (long)blockIdx.x * LA_NTH * LA_EL, base = b0 + threadIdx.x;
    if (b0 >= n) return;
    // coefficient v in lane v; columns behind the last nonzero one are not read
    const double yl = lane < nv ? y[lane] : 0.0;
    const unsigned long long nz = __ballot(yl != 0.0);
    nv = nz ? 64 - __builtin_clzll(nz) : 0;
    double acc[LA_EL], a[G][LA_EL], b[G][LA_EL];
    // (elements beyond the vector: its first ones, not stored)
    long el[LA_EL];
#pragma unroll
    for (int k = 0; k < LA_EL; ++k) el[k] = la_el(base, k) < n ? la_el(base, k) : 0;
#pragma unroll
    for (int k = 0; k < LA_EL; ++k) acc[k] = base_ ? base_[el[k]] : 0.0;
    auto load = [&](int v0, double (&x)[G][LA_EL]) {
#pragma unroll
        for (int q = 0; q < G; ++q)
#pragma unroll
            for (int k = 0; k < LA_EL; ++k) x[q][k] = Z[(long)min(v0 + q, nv - 1) * ld + el[k]];
    };
    auto add = [&](int v0, const double (&x)[G][LA_EL]) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const double yv = lane_value(yl, min(v0 + q, 63));
            if (v0 + q < nv && yv != 0.0)   // a zero coefficient adds nothing (its column may be unset)
#pragma unroll
                for (int k = 0; k < LA_EL; ++k) acc[k] += yv * x[q][k];
        }
    };
    if (nv > 0) load(0, a);
    for (int v0 = 0; v0 < nv; v0 += 2 * G) {   // the next group's loads in flight
        if (v0 + G < nv) load(v0 + G, b);
        add(v0, a);
        if (v0 + G >= nv) break;
        if (v0 + 2 * G < nv) load(v0 + 2 * G, a);
        add(v0 + G, b);
    }
#pragma unroll
    for (int k = 0; k < LA_EL; ++k)
        if (la_el(base, k) < n) out[el[k]] = acc[k];
}

void launch_lincomb(double* out, const double* base, const double* Z, long ld, int nv, long n, const double* y,
                    hipStream_t st, const Mb& mb)
{
    lincomb_kernel<<<dim3(la_blocks(n), 1, mb.n), dim3(LA_NTH), 0, st>>>(out, base, Z, ld, nv, n, y, mb.ms, mb.tab);
}

__global__ void __launch_bounds__(256)
axpby_kernel(double* out, double a, const double* x, double b, const double* y,
             long n, long ms, const MemberArgs* __restrict__ mt)
{
    n = len_of(n, mt);
    out = mbr(out, ms);
    x = mbr(x, ms);
    y = mbr(y, ms);
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) out[i] = a * x[i] + b * y[i];
}

void launch_axpby(double* out, double a, const double* x, double b, const double* y, long n, hipStream_t st,
                  const Mb& mb)
{
    long blk = (n + 255) / 256;
    axpby_kernel<<<dim3((unsigned)(blk < 4096 ? blk : 4096), 1, mb.n), dim3(256), 0, st>>>(out, a, x, b, y, n, mb.ms,
                                                                                           mb.tab);
}

// Stage of the DG-level pseudo-time smoother; out may alias x0 or t (no restrict):
// every element is read and written by the same thread.
__global__ void __launch_bounds__(256)
dg_smooth_kernel(double* out, const double* x0, const double* __restrict__ r, const double* t, double alpha,
                 const double* __restrict__ dtau, long n, Red red, long ms)
{
    out = mbr(out, ms);
    x0 = mbr(x0, ms);
    r = mbr(r, ms);
    t = mbr(t, ms);
    dtau = mbr(dtau, ms);
    red = mbr(red, ms);
    const double s = dtau ? alpha * dtau[0] : alpha;
    double a = 0.0;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
        const double d = t ? r[i] - t[i] : r[i];
        const double v = x0 ? x0[i] + s * d : s * d;
        out[i] = v;
        a += v * v;
    }
    if (red.partials) put_partial<256>(red, a);
}

void launch_dg_smooth(double* out, const double* x0, const double* r, const double* t, double alpha,
                      const double* dtau, long n, Red red, hipStream_t st, const Mb& mb)
{
    long b = (n + 255) / 256;
    const int nb = (int)(b < 1024 ? b : 1024);
    if (!red.out) red.partials = nullptr;
    timed_launch(dg_smooth_kernel, dim3(nb, 1, mb.n), dim3(256), st, out, x0, r, t, alpha, dtau, n, red, mb.ms);
    if (red.out) launch_finalize(red.partials, nb, 1, red.out, st, mb);
}

__global__ void __launch_bounds__(64) dg_dtau_kernel(const double* __restrict__ lam, double* __restrict__ out,
                                                     double hx, double hz, double mu, double adt, double cfl,
                                                     long ms)
{
    lam = mbr(lam, ms);
    out = mbr(out, ms);
    if (threadIdx.x == 0)
        out[0] = cfl / (1.0 + adt * (lam[0] * (1.0 / hx + 1.0 / hz) + 2.0 * mu * (1.0 / (hx * hx) + 1.0 / (hz * hz))));
}

void launch_dg_dtau(const double* lam, double* out, double hx, double hz, double mu, double adt, double cfl,
                    hipStream_t st, const Mb& mb)
{
    dg_dtau_kernel<<<dim3(1, 1, mb.n), dim3(64), 0, st>>>(lam, out, hx, hz, mu, adt, cfl, mb.ms);
}

__global__ void __launch_bounds__(256) zero_kernel(unsigned* __restrict__ x, long n, long ms)
{
    x = mbr(x, ms);
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) x[i] = 0u;
}

// x[i] = a fixed pattern of values in [-1/2, 1/2) (test vectors of the autotuner)
template <typename T> __global__ void __launch_bounds__(256) fill_pattern_kernel(T* __restrict__ x, long n, long ms)
{
    x = mbr(x, ms);
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256)
        x[i] = (T)((double)(((unsigned long)i * 2654435761UL) & 0xffffUL) * (1.0 / 65536.0) - 0.5);
}

template <typename T> void launch_fill_pattern(T* x, long n, hipStream_t st, const Mb& mb)
{
    const long nb = (n + 255) / 256 < 2048 ? (n + 255) / 256 : 2048;
    fill_pattern_kernel<T><<<dim3((unsigned)nb, 1, mb.n), dim3(256), 0, st>>>(x, n, mb.ms);
}
template void launch_fill_pattern<double>(double*, long, hipStream_t, const Mb&);
template void launch_fill_pattern<float>(float*, long, hipStream_t, const Mb&);

void launch_zero(void* ptr, size_t bytes, hipStream_t st, const Mb& mb)
{
    const long n = (long)(bytes / 4);
    long blk = (n + 255) / 256;
    zero_kernel<<<dim3((unsigned)(blk < 4096 ? blk : 4096), 1, mb.n), dim3(256), 0, st>>>((unsigned*)ptr, n, mb.ms);
}

__global__ void __launch_bounds__(256) set_live_kernel(MemberArgs* __restrict__ tab, int n, LiveBits bits)
{
    for (int m = blockIdx.x * 256 + threadIdx.x; m < n; m += gridDim.x * 256)
        tab[m].live = (int)((bits.w[m >> 6] >> (m & 63)) & 1ull);
}

void launch_set_live(MemberArgs* tab, int n, const LiveBits& bits, hipStream_t st)
{
    set_live_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(tab, n, bits);
}

}  // namespace jfmg
