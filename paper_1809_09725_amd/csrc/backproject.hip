// Pixel-driven back-projection of the folded sinogram g~ (Sec. 4, eq.
// radadjapr): out_k(z,r,q) = sum_a sum_b w(theta0_a, b, q, r) g~(a,z,b,k), the
// exact transpose of the ray-driven forward projection: the weight of bin b
// for pixel p is max(0, 1 - |s_b - s_p| / c) / c with c = max(|cos|, |sin|),
// Joseph's linear interpolation written from the pixel's side.  The fold-sum
// stores g~ / c, so that the weights here, c times the triangle weights, lie
// in [0, 1].
//
// A workgroup takes a tile of 32 x 8 VPT pixels and NQ channel quads of the
// list of all slices' quads (K = 16: one slice, K = 8: two).  Per class it
// stages in LDS the window of detector bins the tile's pixels reach, then
// every pixel takes the two bins around its s_p.  A pixel's position is formed
// in FP64 once per class and stepped over the thread's rows in 32.32 fixed
// point (the integer part gives the window row, the fraction the weights);
// weights and sums in FP32.  Positions are absolute, so a pixel's bits do not
// depend on its tile's shape.
//
// Stages of BP_CA classes, one per wave, are copied to LDS directly and double
// buffered: a stage is on its way while the one before is summed, and one
// barrier ends it.  A window row is NQ quads and, for NQ = 2 and 4, a spare
// one (an odd number of 16-byte units: the 8 x 8 pixels of a read instruction
// reach fewer than 16 consecutive rows per 16 lanes, which then fall in
// distinct units).  The reads of g~ cost 128 bytes of LDS per pixel, class and
// 16 channels; at 256 bytes per cycle and CU that is 5.3 ms at 512^2 x 128, K =
// 16, 180 classes, and bounds the kernel with the FMAs (4.9 ms).  Measured there:
// 8.33 ms with the windows staged through registers between two barriers per
// round of classes, 6.69 as it is; one 512^2 slice, 180 classes: 193 us in 32 x
// 32 tiles, 98 in smaller ones.
#include "common.h"
#include "internal.h"

namespace rt {
namespace {

constexpr int BP_CA = NT / 64;   // classes per stage
constexpr int BP_CH = 64;        // classes per fill of the class table (two fills kept)
// Thread -> pixel: wave w of the tile takes columns 8w..8w+7 and lane l row
// l / 8 of each 8-row step, so the 64 taps of one read instruction come from
// an 8 x 8 pixel block, whose detector positions span few bins.
__device__ inline int bp_col(int tid) { return 8 * (tid >> 6) + (tid & 7); }
__device__ inline int bp_row(int tid) { return (tid >> 3) & 7; }
// rows of the widest window of a tile of 32 x 8 vpt pixels: the positions'
// span is at most the tile's diagonal; two bins around each position, one to
// spare on either side
constexpr int bp_rows(int vpt) { return vpt == 4 ? 44 + 6 : 32 + 6; }
constexpr int bp_units(int nq) { return nq | 1; }   // 16-byte units per window row
constexpr int bp_copies(int nq, int vpt) { return (bp_rows(vpt) * bp_units(nq) + 63) / 64; }

struct __attribute__((aligned(16))) BpClass {
    double cs, sn;
    long long D;     // 8 sin in 32.32 fixed point
    float ic1, s1;   // 1 - 1/c and 2^-32 / c
    int lo, pad[3];  // bin of the window's row 0
};

struct BpArgs {
    int N, Nz, Ns, K, K4, n0, ntq, ntr;
    unsigned nblocks;
};

// LIST: the quads are of several slices (K4 is no multiple of NQ); lanes
// outside the detector or the list get an offset past the buffer.  Otherwise
// the buffer is the slice's rows of one class and its bounds give the zeros.
template <int NQ, int VPT, bool LIST>
__global__ __launch_bounds__(NT, 4) void k_backproject(const float *__restrict__ gt,
                                                       float *__restrict__ out,
                                                       const double *__restrict__ ccos,
                                                       const double *__restrict__ csin, BpArgs A)
{
    constexpr int NU = bp_units(NQ), NI = bp_copies(NQ, VPT);
    constexpr unsigned CLB = NI * 1024u, STB = BP_CA * CLB;   // bytes of a class's window, of a stage
    extern __shared__ __align__(64) char smem[];              // [2][BP_CA][NI * 64 units]
    __shared__ BpClass tab[2 * BP_CH];                        // class a in entry a mod 2 BP_CH
    typedef float v4 __attribute__((ext_vector_type(4)));
    typedef int i4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const v4 lds_v4;
    const int N = A.N, Nz = A.Nz, Ns = A.Ns, K = A.K, K4 = A.K4, n0 = A.n0;
    unsigned lid = xcd_remap(blockIdx.x, A.nblocks);
    const int tq = lid % A.ntq;
    lid /= A.ntq;
    const int tr = lid % A.ntr;
    const int cg = lid / A.ntr;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double hN = 0.5 * (double)(N - 1), hS = 0.5 * (double)(Ns - 1);
    const int z0 = cg * NQ / K4, kq0 = cg * NQ % K4;   // first quad
    const unsigned Kb = 16u * K4;                      // bytes of a bin of g~

    const int q = tq * 32 + bp_col(tid);
    // rows r0 + 8 j of the 32-row band, j0 <= j < j0 + VPT
    const int band = tr * 8 * VPT / 32 * 32, j0 = (tr * 8 * VPT - band) / 8;
    const int r0 = band + bp_row(tid);
    const double x = (double)q - hN, y0 = (double)r0 - hN;
    const double xlo = (double)(tq * 32) - hN, xhi = xlo + 31.0;
    const double ylo = (double)(tr * 8 * VPT) - hN, yhi = ylo + (8 * VPT - 1);

    auto fill = [&](int a0) {   // classes [a0, a0 + BP_CH) into the table
        const int a = a0 + tid;
        if (tid >= BP_CH || a >= n0) return;
        // s_p is affine in (x, y): the extreme positions are at the tile's
        // corners; one spare bin below
        const double cs = ccos[a], sn = csin[a];
        const double u00 = fma(xlo, cs, fma(ylo, sn, hS)), u10 = fma(xhi, cs, fma(ylo, sn, hS));
        const double u01 = fma(xlo, cs, fma(yhi, sn, hS)), u11 = fma(xhi, cs, fma(yhi, sn, hS));
        const double umin = fmin(fmin(u00, u10), fmin(u01, u11));
        const double ic = 1.0 / fmax(fabs(cs), fabs(sn));
        BpClass &T = tab[a % (2 * BP_CH)];
        T.cs = cs;
        T.sn = sn;
        T.D = (long long)llrint(sn * 34359738368.0);
        T.ic1 = (float)(1.0 - ic);
        T.s1 = (float)ic * 2.3283064365386963e-10f;
        T.lo = (int)floor(umin) - 1;
    };

    // copy i of a wave: unit 64 i + lane of its class's window: row e / NU,
    // quad e % NU (the spare unit and rows past the window take zeros)
    unsigned goff[NI];
    int grow[LIST ? NI : 1];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int e = 64 * i + lane, row = e / NU, u = e % NU;
        const int gq = cg * NQ + u, zq = gq / K4 - z0, kq = gq % K4;
        const bool ok = u < NQ && gq < Nz * K4 && row < bp_rows(VPT);
        goff[i] = row * Kb + (LIST ? zq * (unsigned)Ns * Kb + kq * 16u : (kq0 + u) * 16u);
        if constexpr (LIST) grow[i] = ok ? row : -(1 << 28);
        else if (!ok) goff[i] = 0xc0000000u;   // stays past the buffer for every window start
    }
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char *)smem;
    // stage st into buffer st & 1 (inline assembly: the compiler adds no wait
    // before the reads of the other buffer; the wait is the vmcnt(0) before
    // the barrier that ends the stage)
    auto issue = [&](int st) {
        const int a = BP_CA * st + wave;
        if (a >= n0) return;
        const int lo = __builtin_amdgcn_readfirstlane(tab[a % (2 * BP_CH)].lo);
        const char *base = (const char *)gt + ((size_t)a * Nz + z0) * Ns * Kb;
        const unsigned end = (LIST ? min(Nz - z0, NQ) : 1) * (unsigned)Ns * Kb;
        const i4 rs{(int)(unsigned)(size_t)base, (int)(((size_t)base >> 32) & 0xffff), (int)end, 0x00020000};
        const unsigned dst = lds0 + (st & 1) * STB + wave * CLB;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            unsigned off = goff[i] + (unsigned)lo * Kb;
            if constexpr (LIST)
                if ((unsigned)(grow[i] + lo) >= (unsigned)Ns) off = 0xffffff00u;
            asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds"
                         :: "v"(off), "s"(rs), "{m0}"(__builtin_amdgcn_readfirstlane(dst + i * 1024u))
                         : "memory");
        }
    };

    float acc[VPT][NQ][4];
#pragma unroll
    for (int j = 0; j < VPT; ++j)
#pragma unroll
        for (int k = 0; k < NQ; ++k)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[j][k][t] = 0.f;

    const int nst = (n0 + BP_CA - 1) / BP_CA;
    fill(0);
    __syncthreads();
    issue(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        if (st % (BP_CH / BP_CA) == 0) fill(BP_CA * st + BP_CH);
        if (st + 1 < nst) issue(st + 1);
        const int nc = min(BP_CA, n0 - BP_CA * st);
        for (int c = 0; c < nc; ++c) {
            const BpClass &T = tab[(BP_CA * st + c) % (2 * BP_CH)];
            const float ic1 = T.ic1, s1 = T.s1;
            const double s = fma(x, T.cs, fma(y0, T.sn, hS)), fl = floor(s);
            const unsigned long long D = (unsigned long long)T.D;
            // 32.32 fixed point: the integer part counts window rows; rows 8
            // apart add 8 sin, rounded to 2^-32
            unsigned long long U = ((unsigned long long)(unsigned)((int)fl - T.lo) << 32) |
                                   (unsigned)((s - fl) * 4294967296.0);
            if constexpr (VPT < 4) U += (unsigned long long)j0 * D;
            const unsigned wbase = lds0 + (st & 1) * STB + c * CLB;
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                if (j) {
                    U += D;
                    asm volatile("" : "+v"(U));   // one 64-bit add per row, not j*D
                }
                const float fq = (float)(unsigned)U;   // the fraction in units of 2^-32
                // triangle weights of the bins floor(u) and floor(u)+1 times c:
                // one fma with the clamp to [0, 1] each
                const float w0 = fminf(fmaxf(fmaf(-fq, s1, 1.f), 0.f), 1.f);
                const float w1 = fminf(fmaxf(fmaf(fq, s1, ic1), 0.f), 1.f);
                const unsigned t0 = __umul24((unsigned)(U >> 32), NU * 16u) + wbase;
                v4 x0[NQ], x1[NQ];
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    x0[k] = *(lds_v4 *)(size_t)(t0 + 16 * k);
                    x1[k] = *(lds_v4 *)(size_t)(t0 + 16 * (NU + k));
                }
                __builtin_amdgcn_sched_barrier(0);   // all reads are issued before the first FMA waits
#pragma unroll
                for (int k = 0; k < NQ; ++k)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        acc[j][k][t] = fmaf(w1, x1[k][t], fmaf(w0, x0[k][t], acc[j][k][t]));
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }

    if (q >= N) return;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int r = r0 + 8 * (j0 + j);
        if (r >= N) continue;
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int gq = cg * NQ + k, z = gq / K4, c0 = 4 * (gq % K4);
            if (z >= Nz) continue;
            float *dst = out + (((size_t)z * N + r) * N + q) * K + c0;
            if ((K & 3) == 0) {
                *(v4 *)dst = v4{acc[j][k][0], acc[j][k][1], acc[j][k][2], acc[j][k][3]};
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (c0 + t < K) dst[t] = acc[j][k][t];
            }
        }
    }
}

// Few pixels: a workgroup takes 8 x 8 pixels, and its four waves take every
// fourth class each, with windows of their own (no barriers), and add their sums
// at the end in wave order.  A 64^2 slice is then 64 workgroups of n0 / 4
// classes in sequence instead of 16 of n0: 21 -> 13 us at 90 classes, 8
// channels.  The windows' rows per pixel double, so it is for images whose 32 x 8
// tiles leave most CUs idle.
constexpr int BS_CB = 4;      // classes per batch of copies, two batches in flight
constexpr int BS_ROWS = 17;   // 7 sqrt 2 < 10 positions; two bins, one to spare on either side
constexpr int bs_copies(int nq) { return (BS_ROWS * bp_units(nq) + 63) / 64; }

template <int NQ, bool LIST>
__global__ __launch_bounds__(NT) void k_backproject_small(const float *__restrict__ gt,
                                                          float *__restrict__ out,
                                                          const double *__restrict__ ccos,
                                                          const double *__restrict__ csin, BpArgs A)
{
    constexpr int NU = bp_units(NQ), NI = bs_copies(NQ);
    constexpr unsigned CLB = NI * 1024u, WVB = 2 * BS_CB * CLB;   // bytes of a window, of a wave's ring
    extern __shared__ __align__(64) char smem[];                  // [4 waves][2][BS_CB][NI * 64 units]
    typedef float v4 __attribute__((ext_vector_type(4)));
    typedef int i4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const v4 lds_v4;
    const int N = A.N, Nz = A.Nz, Ns = A.Ns, K = A.K, K4 = A.K4, n0 = A.n0;
    unsigned lid = xcd_remap(blockIdx.x, A.nblocks);
    const int tq = lid % A.ntq;
    lid /= A.ntq;
    const int tr = lid % A.ntr;
    const int cg = lid / A.ntr;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double hN = 0.5 * (double)(N - 1), hS = 0.5 * (double)(Ns - 1);
    const int z0 = cg * NQ / K4, kq0 = cg * NQ % K4;
    const unsigned Kb = 16u * K4;
    const int q = tq * 8 + (lane & 7), r = tr * 8 + (lane >> 3);
    const double x = (double)q - hN, y = (double)r - hN;
    const double xm = (double)(tq * 8) + 3.5 - hN, ym = (double)(tr * 8) + 3.5 - hN;   // tile's middle

    unsigned goff[NI];
    int grow[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int e = 64 * i + lane, row = e / NU, u = e % NU;
        const int gq = cg * NQ + u, zq = gq / K4 - z0, kq = gq % K4;
        goff[i] = row * Kb + (LIST ? zq * (unsigned)Ns * Kb + kq * 16u : (kq0 + u) * 16u);
        grow[i] = u < NQ && gq < Nz * K4 && row < BS_ROWS ? row : -(1 << 28);
    }
    const unsigned ring = (unsigned)(size_t)(__attribute__((address_space(3))) char *)smem + wave * WVB;
    // this wave's class i (past the end: the last class again, not summed)
    auto cls = [&](int i) { return min(4 * i + wave, n0 - 1); };
    // bin of the window's row 0: one below the lowest position of the tile
    auto first = [&](double cs, double sn) {
        return (int)floor(fma(xm, cs, fma(ym, sn, hS)) - 3.5 * (fabs(cs) + fabs(sn))) - 1;
    };
    auto issue = [&](int b) {   // batch b into half b & 1 of the ring
#pragma unroll
        for (int c = 0; c < BS_CB; ++c) {
            const int a = cls(BS_CB * b + c);
            const int lo = __builtin_amdgcn_readfirstlane(first(ccos[a], csin[a]));
            const char *base = (const char *)gt + ((size_t)a * Nz + z0) * Ns * Kb;
            const unsigned end = (LIST ? min(Nz - z0, NQ) : 1) * (unsigned)Ns * Kb;
            const i4 rs{(int)(unsigned)(size_t)base, (int)(((size_t)base >> 32) & 0xffff), (int)end, 0x00020000};
            const unsigned dst = ring + ((b & 1) * BS_CB + c) * CLB;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const unsigned off = (unsigned)(grow[i] + lo) < (unsigned)Ns ? goff[i] + (unsigned)lo * Kb : 0xffffff00u;
                asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds"
                             :: "v"(off), "s"(rs), "{m0}"(__builtin_amdgcn_readfirstlane(dst + i * 1024u))
                             : "memory");
            }
        }
    };

    float acc[NQ][4];
#pragma unroll
    for (int k = 0; k < NQ; ++k)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[k][t] = 0.f;
    const int ncl = (n0 - wave + 3) / 4;   // this wave's classes
    const int nb = (ncl + BS_CB - 1) / BS_CB;
    if (nb > 0) issue(0);
    for (int b = 0; b < nb; ++b) {
        // the taps of batch b - 1 have left the half of the ring that batch b + 1
        // is copied to (the copies' order after LDS reads is nowhere else kept)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(b + 1);   // always, so that the count below is this batch's
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(BS_CB * NI) : "memory");
#pragma unroll
        for (int c = 0; c < BS_CB; ++c) {
            if (BS_CB * b + c >= ncl) break;
            const int a = cls(BS_CB * b + c);
            const double cs = ccos[a], sn = csin[a];
            const float ic = (float)(1.0 / fmax(fabs(cs), fabs(sn)));
            const double s = fma(x, cs, fma(y, sn, hS)), fl = floor(s);
            const float fr = (float)(s - fl);
            const float w0 = fminf(fmaxf(fmaf(-fr, ic, 1.f), 0.f), 1.f);
            const float w1 = fminf(fmaxf(fmaf(fr, ic, 1.f - ic), 0.f), 1.f);
            const unsigned t0 = ring + ((b & 1) * BS_CB + c) * CLB + __umul24((unsigned)((int)fl - first(cs, sn)), NU * 16u);
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
                const v4 x0 = *(lds_v4 *)(size_t)(t0 + 16 * k), x1 = *(lds_v4 *)(size_t)(t0 + 16 * (NU + k));
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[k][t] = fmaf(w1, x1[t], fmaf(w0, x0[t], acc[k][t]));
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // the waves' sums, [wave][NQ][lane]; wave w adds and writes quads w, w + 4, ..
    v4 *sums = (v4 *)smem;
#pragma unroll
    for (int k = 0; k < NQ; ++k)
        sums[(wave * NQ + k) * 64 + lane] = v4{acc[k][0], acc[k][1], acc[k][2], acc[k][3]};
    __syncthreads();
    if (wave >= NQ || q >= N || r >= N) return;
    v4 v = sums[wave * 64 + lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) v += sums[(w * NQ + wave) * 64 + lane];
    const int gq = cg * NQ + wave, z = gq / K4, c0 = 4 * (gq % K4);
    if (z >= Nz) return;
    float *dst = out + (((size_t)z * N + r) * N + q) * K + c0;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (c0 + t < K) dst[t] = v[t];
}

template <int NQ>
static void launch_bp_small(const Plan &p, float *out, hipStream_t s, int ncg, bool list)
{
    const rt_geom &G = p.g;
    BpArgs A{G.N, G.Nz, G.Ns, G.K, (G.K + 3) / 4, p.n0, (G.N + 7) / 8, (G.N + 7) / 8, 0};
    A.nblocks = (unsigned)ncg * A.ntq * A.ntr;
    const size_t lds = (size_t)4 * 2 * BS_CB * bs_copies(NQ) * 1024;
    KTimer kt("k_backproject", s);
    if (list)
        hipLaunchKernelGGL((k_backproject_small<NQ, true>), dim3(A.nblocks), dim3(NT), lds, s, p.d_scr,
                           out, p.d_ccos, p.d_csin, A);
    else
        hipLaunchKernelGGL((k_backproject_small<NQ, false>), dim3(A.nblocks), dim3(NT), lds, s, p.d_scr,
                           out, p.d_ccos, p.d_csin, A);
    kt.stop();
}

template <int NQ, int VPT>
static void launch_bp_t(const Plan &p, float *out, hipStream_t s, int ncg, bool list)
{
    const rt_geom &G = p.g;
    BpArgs A{G.N, G.Nz, G.Ns, G.K, (G.K + 3) / 4, p.n0, (G.N + 31) / 32, (G.N + 8 * VPT - 1) / (8 * VPT), 0};
    A.nblocks = (unsigned)ncg * A.ntq * A.ntr;
    const size_t lds = (size_t)2 * BP_CA * bp_copies(NQ, VPT) * 1024;
    KTimer kt("k_backproject", s);
    if (list)
        hipLaunchKernelGGL((k_backproject<NQ, VPT, true>), dim3(A.nblocks), dim3(NT), lds, s, p.d_scr,
                           out, p.d_ccos, p.d_csin, A);
    else
        hipLaunchKernelGGL((k_backproject<NQ, VPT, false>), dim3(A.nblocks), dim3(NT), lds, s, p.d_scr,
                           out, p.d_ccos, p.d_csin, A);
    kt.stop();
}

}  // namespace

int launch_backproject(const Plan &p, float *out, hipStream_t s)
{
    const rt_geom &G = p.g;
    if (G.Nz == 0) return RT_OK;
    const int K4 = (G.K + 3) / 4, tq = G.Nz * K4;
    const int NQ = tq >= 3 ? 4 : tq;
    const int ncg = (tq + NQ - 1) / NQ;
    const bool list = K4 % NQ != 0;
    // 32 x 32 tiles where they give every CU its four workgroups, else 32 x 8 (a
    // pixel's bits are the same); where those hold less than 1024 channel
    // quads, 8 x 8 tiles, whose sums have an order of their own: the choice
    // follows from nz_ref, not from Nz, so that a slab and its volume agree.
    // Measured, 32 x 8 against 8 x 8: 512 quads (256^2, K = 8) 35 and 30 us,
    // 1024 quads (256^2, K = 16) 42 and 46 us
    const long t32 = (G.N + 31) / 32;
    const long ref = std::max((long)p.nz_ref * K4, 1L) * t32 * ((G.N + 7) / 8);
    const bool small = ncg * t32 * t32 < 1024;
    if (ref < 1024) {
        switch (NQ) {
        case 4: launch_bp_small<4>(p, out, s, ncg, list); break;
        case 2: launch_bp_small<2>(p, out, s, ncg, list); break;
        default: launch_bp_small<1>(p, out, s, ncg, list); break;
        }
        RT_HIP(hipGetLastError());
        return RT_OK;
    }
    switch (NQ) {
    case 4: small ? launch_bp_t<4, 1>(p, out, s, ncg, list) : launch_bp_t<4, 4>(p, out, s, ncg, list); break;
    case 2: small ? launch_bp_t<2, 1>(p, out, s, ncg, list) : launch_bp_t<2, 4>(p, out, s, ncg, list); break;
    default: small ? launch_bp_t<1, 1>(p, out, s, ncg, list) : launch_bp_t<1, 4>(p, out, s, ncg, list); break;
    }
    RT_HIP(hipGetLastError());
    return RT_OK;
}

}  // namespace rt
