// Project-first (PF) FP32 form of the decomposed-time Radon operator and its
// transpose (Sec. 4, eqs. radapr and radadjapr, with the pi-periodicity
// identity and the fold-sum).
//
// Forward  g(i,z,b) = sum_k Phi[i][k] P(a(i), z, b'(i,b), k)
//          P(a,z,b,k) = static projection of f_k at theta0_a in [0,pi)
//          b' = b on even half-turns, Ns-1-b on odd ones (s_{Ns-1-b} = -s_b)
// Adjoint  g~(a,z,b,k) = sum_rot Phi[rot*Ntheta0+a][k] g(rot*Ntheta0+a, z, b')
//          out_k = static back-projection of g~(.,.,.,k) over theta0_a
//
// Kernels
//   k_project      ray-driven projection of up to 16 channel columns for the
//                  rays of a tile of bins and neighbouring angle classes of one
//                  walk direction; the window of each line (row or column) of
//                  the slice that they reach is staged once in LDS.
//   k_contract     sum over the line parts and over k with the s-flip;
//                  optionally fused with the h1 prox of Fig. 2 and an FP64
//                  partial of |R f~ - g|^2.
//   k_fold         the fold-sum g -> g~.
// The back-projection of g~ is in backproject.hip.
// Ray positions start in FP64 and are stepped in 32.32 fixed point; weights and
// accumulation in FP32.
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace rt {
namespace {

// clamp to [0, hi] in one v_med3_i32 (the compiler forms it only for
// constant bounds); hi is uniform and stays in an SGPR
__device__ inline int clamp0_i32(int x, int hi)
{
    int r;
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(x), "s"(hi));
    return r;
}

// What the projection does with its sums P(a,z,b,k): store them (g == NULL),
// or, when one workgroup holds all K channels of its slices and all lines,
// contract them with Phi over the Npi half-turns with the s-flip (Sec. 4, eq.
// radapr and the pi-periodicity) and store g.
struct FwdEpi {
    float *g;
    int n0, Npi;
};

// Work split of k_project (host: RayCfg).
struct RayArgs {
    int N, Nz, Ns, K, K4;      // K4 = channel quads per slice
    int ngroups, NLP;          // ray groups, parts of the lines
    unsigned nblocks;
};

typedef float v4 __attribute__((ext_vector_type(4)));

__device__ inline float dot4(float4 w, v4 x)
{
    return fmaf(w.w, x[3], fmaf(w.z, x[2], fmaf(w.y, x[1], w.x * x[0])));
}

// Joseph's ray-driven projection: P(a,z,b,k) = sum over the lines of slice z
// (rows or columns, whichever the ray crosses once each) of the linear
// interpolation between the two positions around the ray, times the line
// spacing along the ray 1/c.
//
// Columns.  The Nz * K4 channel quads of all slices form one list; a
// workgroup takes NQ consecutive ones, so K = 16 is one slice per workgroup
// and K = 8 two, and a position of a staged line is NQ * 16 bytes in LDS.
// Rays.  A workgroup takes one RayGroup: a tile of bins of neighbouring
// classes of one walk direction, as blocks of 64 rays, PPT blocks per wave.
// Where the detector is no multiple of 64 a block may run on into the next
// class (as the plan finds faster).  Lines no
// ray of a block crosses are skipped (a wave-uniform interval per block): 9%
// of the tap work at Ns = N, more where the detector is wider than the slice.
// Lines.  Only the window of W positions that the group's rays reach on a
// line is staged; it moves with the line along the group's middle slope
// (positions outside the slice are read as zeros by the buffer bounds).
// Two bin blocks of 16 classes need about 250 of 512 positions, 270 of
// 1024, 380 of 2048: a line's read and LDS traffic per ray is 8 to 13 bytes
// per channel quad column instead of 16 to 64 for whole lines, and 4 or 2
// lines fit a stage.  Stages are double buffered, with the loads a stage
// further ahead in registers; one barrier per stage.  With NLP > 1 a
// workgroup walks one of NLP parts of the lines and stores partial sums
// that k_contract adds in part order.
//
// What bounds it: no unit alone.  At 512^2 x 128, K = 16, 180 classes (9.9 ms)
// LDS is active 58% of the time, with the tap reads at 8 bytes per channel
// sample and 5.1 cycles each where 4.3 would be free of conflicts, and the
// vector units issue half of it; the 16 waves of a CU, one workgroup, meet at
// each stage's barrier and leave both idle there.  8.0 ms remain without the
// staging and its barriers.  With whole lines staged for all bins of four
// classes, rows padded to 80 bytes and lanes ordered modulo 16 it was 12.9 ms
// there, and 8.4 ms against 5.6 at 1024^2 x 8 over 300 classes, where whole
// lines allowed 8 channels at a time.
//
// LDS.  A ds_read_b128 is served in four groups of 16 lanes ({0-3, 12-15,
// 20-27}, {4-11, 16-19, 28-31}, and the same + 32), each over 16 units of 16
// bytes, at 4.3 cycles per CU when no two lanes of a group hit different rows
// of one unit.  Rows are unpadded; lane l reads the quads of a row in the
// order quad = kappa ^ rho, rho = (l >> 3) & 3 (NQ = 4), so the four lane
// quads of a group read four different column quads, and the lane tables give
// every lane quad four rays whose positions are about 0, 1, 2, 3 modulo 4
// apart.  Sampled over the angles that is 5.1 cycles per read, against 5.9 for
// rows padded to 80 bytes and lanes ordered modulo 16, and a line takes 20%
// less LDS.
//
// Staging (STG).  STG_LINE: the quads are of one slice; each line is a buffer
// whose bounds give the zeros outside it, and the loads go to LDS directly.
// STG_LIST: the quads are of several slices (K4 is no multiple of NQ); one
// buffer over them, lanes outside get an offset past its end.  STG_FEW: fewer
// than 4 channels, a quad per slice; the same buffer, read into registers with
// one load of K dwords per quad (three masked 4-byte loads took 1.39 ms against
// 0.57 at 551^2 x 36, K = 3, 25 classes, and 0.46 against 0.32 at 256^2 x 64, 128
// classes).  STG_REGS: offsets of more than 32 bits; masked loads through
// registers.  Where K is no multiple of 4, a slice's last quad is staged as
// its last four channels, all of them real; the sums are shifted into place
// at the end.
enum { STG_LINE = 0, STG_LIST = 1, STG_REGS = 2, STG_FEW = 3 };
constexpr bool stg_regs(int stg) { return stg >= STG_REGS; }   // through registers
template <int NQ, int PPT, int PF, bool TL, int NTH, int STG>
__global__ __launch_bounds__(NTH) void k_project(
    const float *__restrict__ f, float *P, const RayGroup *__restrict__ groups,
    const int *__restrict__ wcls, const unsigned char *__restrict__ rlane, const double *__restrict__ ccos,
    const double *__restrict__ csin, const float *__restrict__ phi, RayArgs A, FwdEpi E)
{
    constexpr int NW = NTH / 64;
    constexpr int SH = NQ == 4 ? 6 : NQ == 2 ? 5 : 4;   // log2 of a row's bytes
    constexpr int RPJ = NTH / NQ;                       // rows one float4 per thread covers
    extern __shared__ __align__(64) char smem[];        // [2][NLS][W rows][NQ] float4
    const int N = A.N, Ns = A.Ns, K = A.K, K4 = A.K4;
    unsigned lid = xcd_remap(blockIdx.x, A.nblocks);
    const int grp = lid % A.ngroups;
    lid /= A.ngroups;
    const int lp = lid % A.NLP, cg = lid / A.NLP;
    const int lbeg = (int)((long)lp * N / A.NLP), lend = (int)((long)(lp + 1) * N / A.NLP);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RayGroup G = groups[grp];
    const int walk = G.walk, W = G.W;
    const double hN = 0.5 * (double)(N - 1), hS = 0.5 * (double)(Ns - 1);
    // a line takes PPL float4 per thread, a stage NLS = PF / PPL lines (fewer
    // in a short part)
    const int sh_l = W <= RPJ ? 0 : W <= 2 * RPJ ? 1 : W <= 4 * RPJ ? 2 : 3;   // log2 PPL
    const int NLS = min(PF >> sh_l, lend - lbeg);
    const int lineb = W << SH, bufb = NLS * lineb;

    // ---- rays.  Positions along the lines in 32.32 fixed point: u at the
    // block's first line from FP64, stepped by the slope with an exact
    // integer add per line, so u(l) carries the rounding of its start and of
    // l s alone (below 2^-32 (1 + l) positions).  The integer part less the
    // window's first position is the LDS row of the left tap, the fraction
    // the weight.  The row is clamped to the window, which only moves lanes
    // without a ray (1/c = 0), or, where the window is the whole line with
    // its guard positions, rays off the slice.
    long long U[PPT], S[PPT];
    float invc[PPT], sfr[PPT];
    int cl[PPT], bin[PPT], jb[PPT], je[PPT];   // class (-1: none) and bin of a lane, lines [jb, je) of the block
    const int nrays = G.ncls * G.stride;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        // block n: rays 64 n .. of the list of classes times bins, in the lane
        // order of its first ray's class
        const int first = (j * NW + wave) * 64;
        int a = -1, b = Ns;
        if (first < nrays) {
            const int ray = first + (int)rlane[wcls[G.cls0 + first / G.stride] * 64 + lane], c = ray / G.stride;
            const int off = ray - c * G.stride;
            if (ray < nrays && off < G.nb) {
                a = wcls[G.cls0 + c];
                b = G.b0 + off;
            }
        }
        cl[j] = a;
        bin[j] = b;
        double base = -1.0e6, slope = 0.0, lo = 2.0e6, hi = -2.0e6;
        invc[j] = 0.f;
        if (b < Ns) {
            const double cs = ccos[a], sn = csin[a], sb = (double)b - hS;
            if (walk == 0) {   // |cos| >= |sin|: the ray crosses every row once
                base = sb / cs + hN;
                slope = -sn / cs;
                invc[j] = (float)(1.0 / fabs(cs));
            } else {           // |sin| > |cos|: every column once
                base = sb / sn + hN;
                slope = -cs / sn;
                invc[j] = (float)(1.0 / fabs(sn));
            }
            // lines with -1 <= u < N, a line to spare at each end
            const double u0 = fma(-hN, slope, base);
            if (fabs(slope) * (double)N > 1.0e-3) {
                const double x = (-1.0 - u0) / slope, y = ((double)N - u0) / slope;
                lo = fmin(x, y) - 1.0;
                hi = fmax(x, y) + 2.0;
            } else if (u0 > -2.0 && u0 < (double)N + 1.0) {
                lo = -1.0;
                hi = (double)N;
            }
        }
        int l0 = (int)fmin(fmax(lo, (double)lbeg), (double)lend);
        int l1 = (int)fmin(fmax(hi, (double)lbeg), (double)lend);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            l0 = min(l0, __shfl_xor(l0, o, 64));
            l1 = max(l1, __shfl_xor(l1, o, 64));
        }
        jb[j] = __builtin_amdgcn_readfirstlane(l0);
        je[j] = __builtin_amdgcn_readfirstlane(l1);
        const double u = fmin(fmax(fma((double)jb[j] - hN, slope, base), -1.0e6), 1.0e6);
        U[j] = (long long)llrint(u * 4294967296.0);
        S[j] = (long long)llrint(slope * 4294967296.0);
        sfr[j] = invc[j] * 2.3283064365386963e-10f;   // fraction bits -> weight: 2^-32 / c
    }

    float acc[PPT][NQ][4];
#pragma unroll
    for (int j = 0; j < PPT; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[j][q][t] = 0.f;

    // ---- staging: float4 j of a thread is quad tid % NQ of row tid / NQ +
    // RPJ (j mod PPL) of line j / PPL of the stage
    const unsigned lstep = (walk == 0 ? N * K : K) * 4u;   // next line (bytes)
    const unsigned pstep = (walk == 0 ? K : N * K) * 4u;   // next position
    const int z0 = cg * NQ / K4;
    const int cq = tid % NQ, p0 = tid / NQ, gq = cg * NQ + cq;
    const int zq = gq / K4 - z0, kq = gq % K4;
    const bool qok = gq < A.Nz * K4;             // a quad of the list
    const int kr = K & 3;                        // channels of a slice's last quad (0: 4)
    const unsigned coff = min(4 * kq, max(K - 4, 0)) * 4u;   // channel offset of the load
    const unsigned goff = coff + p0 * pstep + (STG == STG_LIST || STG == STG_FEW ? zq * (unsigned)N * N * K * 4u : 0u);
    const char *fz = (const char *)(f + (size_t)z0 * N * N * K);
    typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));
    typedef int i4 __attribute__((ext_vector_type(4)));
    v4 r[stg_regs(STG) ? PF : 1];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char *)smem;
    auto first_line = [&](int st) { return min(lbeg + st * NLS, lend - NLS); };
    auto wfirst = [&](int l) { return (int)((G.wl0 + l * G.sw) >> 32); };   // window's first position
    // stage st into registers (STG_REGS) or into buffer st & 1: global to LDS
    // copies of 16 bytes per lane to consecutive LDS addresses.  They are
    // issued from inline assembly, so that the compiler, which cannot tell the
    // two buffers apart, adds no wait for them before the tap reads; the wait
    // is the vmcnt(0) before the barrier that ends the stage.
    // STG_FEW: KC channels of a position in one load, zeros from past the buffer's end
    auto load_few = [&](int st, auto kc) __attribute__((always_inline)) {
        constexpr int KC = decltype(kc)::value;
        const int l0 = first_line(st);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void *)fz, 0, (unsigned)min(A.Nz - z0, NQ) * (unsigned)N * N * KC * 4u, 0x00020000);
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int ln = j >> sh_l, row = (j & ((1 << sh_l) - 1)) * RPJ;
            if (ln >= NLS) break;
            const int l = l0 + ln, pos = wfirst(l) + row + p0;
            const bool in = qok && (unsigned)pos < (unsigned)N;
            const unsigned off = in ? goff + (unsigned)(pos - p0) * pstep + l * lstep : 0xffffff00u;
            v4 x = {0.f, 0.f, 0.f, 0.f};
            if constexpr (KC == 3) {
                const auto u = __builtin_amdgcn_raw_buffer_load_b96(rs, off, 0, 0);
                x = v4{__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), 0.f};
            } else if constexpr (KC == 2) {
                const auto u = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
                x[0] = __uint_as_float(u[0]);
                x[1] = __uint_as_float(u[1]);
            } else {
                x[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
            }
            r[j] = x;
        }
    };
    auto load = [&](int st) __attribute__((always_inline)) {
        if constexpr (STG == STG_FEW) {
            if (K == 3) load_few(st, std::integral_constant<int, 3>{});
            else if (K == 2) load_few(st, std::integral_constant<int, 2>{});
            else load_few(st, std::integral_constant<int, 1>{});
            return;
        }
        const int l0 = first_line(st);
        const unsigned buf = lds0 + (st & 1) * bufb + wave * 1024;
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int ln = j >> sh_l, row = (j & ((1 << sh_l) - 1)) * RPJ;
            if (ln >= NLS) break;
            const int l = l0 + ln, w0 = wfirst(l) + row;   // uniform
            if constexpr (STG == STG_REGS) {
                const int pos = w0 + p0;
                const char *src = fz + (qok ? (size_t)zq * N * N * K * 4 : 0) + (size_t)l * lstep +
                                  (size_t)(unsigned)max(pos, 0) * pstep + coff;
                r[j] = v4{0.f, 0.f, 0.f, 0.f};
                if (qok && (unsigned)pos < (unsigned)N) r[j] = *(const v4u *)src;
            } else {
                // STG_LINE: the bytes of the line up to its last position's
                // end; a position before the line (the offset wraps) or past
                // it is out of bounds
                const char *base = fz + (STG == STG_LINE ? (size_t)l * lstep : 0);
                const unsigned end = STG == STG_LINE ? (N - 1) * pstep + K * 4u
                                                     : (unsigned)min(A.Nz - z0, NQ) * (unsigned)N * N * K * 4u;
                const i4 rs{(int)(unsigned)(size_t)base, (int)(((size_t)base >> 32) & 0xffff), (int)end, 0x00020000};
                unsigned off = goff + (unsigned)w0 * pstep;
                if constexpr (STG == STG_LIST) {
                    const bool in = qok && (unsigned)(w0 + p0) < (unsigned)N;
                    off = in ? off + l * lstep : 0xffffff00u;
                }
                if (p0 + row < W)
                    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds"
                                 :: "v"(off), "s"(rs), "{m0}"(__builtin_amdgcn_readfirstlane(buf + ln * lineb + (row << SH)))
                                 : "memory");
            }
        }
    };
    auto store = [&](int st) {   // through registers
        char *dst = smem + (st & 1) * bufb + (tid << 4);
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int ln = j >> sh_l, row = (j & ((1 << sh_l) - 1)) * RPJ;
            if (ln >= NLS) break;
            if (p0 + row < W) *(v4 *)(dst + ln * lineb + (row << SH)) = r[stg_regs(STG) ? j : 0];
        }
    };

    typedef __attribute__((address_space(3))) const v4 lds_v4;
    const unsigned rho = (NQ == 4 ? (lane >> 3) & 3 : NQ == 2 ? (lane >> 4) & 1 : 0) * 16;
    // block j's rays on the staged line at byte offset lb (its low bits hold rho)
    auto taps = [&](int j, unsigned lb, int w0l) {
        const int q0 = (int)(U[j] >> 32);
        const float fr = (float)(unsigned)U[j];
        U[j] += S[j];
        asm volatile("" : "+v"(U[j]));   // one 64-bit add per line, not U(0) + l s rebuilt
        const float w1 = fr * sfr[j];
        const float w0 = invc[j] - w1;
        const unsigned t0 = ((unsigned)clamp0_i32(q0 - w0l, W - 2) << SH) + lb;
        v4 x[NQ], y[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) x[q] = *(lds_v4 *)(size_t)(t0 ^ (16u * q));
#pragma unroll
        for (int q = 0; q < NQ; ++q) y[q] = *(lds_v4 *)(size_t)((t0 ^ (16u * q)) + (1u << SH));
        __builtin_amdgcn_sched_barrier(0);   // all reads are issued before the first FMA waits
        if constexpr (TL) {   // one rounding at the size of the sum per line (see flush)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[j][q][t] += fmaf(w1, y[q][t], w0 * x[q][t]);
        } else {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[j][q][t] = fmaf(w0, x[q][t], acc[j][q][t]);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[j][q][t] = fmaf(w1, y[q][t], acc[j][q][t]);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(acc[j][q][t])::"memory");
    };

    // acc[j][q] holds column quad q ^ (rho / 16) of block j
    const int rq = (int)rho / 16, Kp = 4 * K4, nq = A.Nz * K4;
    // a ragged last quad's kr channels moved to its front
    auto front = [&](v4 x) {
        return v4{kr == 1 ? x[3] : kr == 2 ? x[2] : x[1], kr == 1 ? 0.f : kr == 2 ? x[3] : x[2],
                  kr == 3 ? x[3] : 0.f, 0.f};
    };
    auto sums = [&](int j, int q) {
        v4 x{acc[j][q][0], acc[j][q][1], acc[j][q][2], acc[j][q][3]};
        return kr && K > 4 && (cg * NQ + (q ^ rq)) % K4 == K4 - 1 ? front(x) : x;
    };
    auto psum = [&](int j, int g) {   // where P keeps column quad g of block j's ray
        return (v4 *)(P + ((((size_t)lp * E.n0 + cl[j]) * A.Nz + g / K4) * Ns + bin[j]) * Kp + 4 * (g % K4));
    };
    // TL (two-level sums, planned for N > 512): the taps of LB consecutive
    // lines are summed in registers and then added to P, so that the FP32
    // rounding of a long ray grows with sqrt(LB) + sqrt(N / LB) additions
    // instead of sqrt(N).  A second set of sums in registers would not fit
    // 16 waves per CU; adding to P takes the L2 traffic of 2 KB per ray block
    // and quad column.  All reads of P are issued before the first is used.
    // Both taps of a line are summed before they are added to the block's sum,
    // which is then rounded once a line.  Error of signed volumes (rel-L2, a
    // CPU emulation of the sums at N = 640, 1024, 2048), and k_project at 1024^2
    // x 8, K = 16, 300 classes: LB = 64 and two FMAs a line 2.21, 2.23,
    // 2.29e-7, 5.47 ms; LB = 32 and two FMAs 1.74, 1.87, 2.09e-7, 6.05 ms; LB
    // = 64 as it is 1.67, 1.75, 1.85e-7, 5.79 ms.
    constexpr int LB = 64;
    bool first = true;
    auto flush = [&]() {
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            v4 x[NQ];
            const bool ray = cl[j] >= 0 && bin[j] < Ns;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                x[q] = v4{0.f, 0.f, 0.f, 0.f};
                if (ray && !first && cg * NQ + (q ^ rq) < nq) x[q] = *psum(j, cg * NQ + (q ^ rq));
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                x[q] += sums(j, q);
                if (ray && cg * NQ + (q ^ rq) < nq) *psum(j, cg * NQ + (q ^ rq)) = x[q];
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[j][q][t] = 0.f;
            }
        }
        first = false;
    };

    // Stage st + 1 is on its way during stage st, into the buffer that stage
    // st - 1 has left.  (STG_REGS: at the top of stage st the registers hold
    // stage st + 1 and are refilled with stage st + 2.)
    const int nst = (lend - lbeg + NLS - 1) / NLS;
    load(0);
    if constexpr (stg_regs(STG)) {
        store(0);
        load(min(1, nst - 1));
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        if constexpr (stg_regs(STG)) {
            store(st + 1);
            load(min(st + 2, nst - 1));
        } else {
            if (st + 1 < nst) load(st + 1);
        }
        const int l0 = first_line(st);
        for (int ln = lbeg + st * NLS - l0; ln < NLS; ++ln) {
            const int l = l0 + ln;
            if constexpr (TL)
                if (l % LB == 0 && l > lbeg) flush();
            const unsigned lb = lds0 + (unsigned)((st & 1) * bufb + ln * lineb) + rho;
            const int w0l = wfirst(l);
#pragma unroll
            for (int j = 0; j < PPT; ++j)
                if ((unsigned)(l - jb[j]) < (unsigned)(je[j] - jb[j])) taps(j, lb, w0l);
        }
        if constexpr (!stg_regs(STG)) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }

    // ---- epilogue
    if (TL || !E.g) {
        flush();
        return;
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        // all K channels of the workgroup's NQ / K4 slices are here (K4 = 1,
        // 2 or 4 divides NQ).  The quads are put in order first, so that the Phi
        // rows are uniform over the wave.  A slice's quads are summed as a tree.
        v4 x[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) x[q] = v4{acc[j][q][0], acc[j][q][1], acc[j][q][2], acc[j][q][3]};
#pragma unroll
        for (int bit = 1; bit < NQ; bit *= 2)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (!(q & bit)) {
                        float lo = x[q][t], hi = x[q | bit][t];
                        asm volatile("" : "+v"(lo), "+v"(hi));   // two selects, not an index into x
                        x[q][t] = rq & bit ? hi : lo;
                        x[q | bit][t] = rq & bit ? lo : hi;
                    }
        if (kr && K > 4)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if ((cg * NQ + q) % K4 == K4 - 1) x[q] = front(x[q]);
        // uniform addresses, stepped per half-turn: a wave alone issues an
        // instruction in 8 cycles, and the address of each store formed anew
        // took more of them than the rest
        const size_t pstep_r = (size_t)E.n0 * Kp, gstep_r = (size_t)E.n0 * A.Nz * Ns;
        const int b = bin[j], nsl = min(NQ / K4, A.Nz - z0);   // nsl: slices of the workgroup
        auto contract = [&](int a) __attribute__((always_inline)) {
            const float *pr = phi + (size_t)a * Kp;
            float *gr = E.g + ((size_t)a * A.Nz + z0) * Ns;
#pragma unroll 2
            for (int r = 0; r < E.Npi; ++r, pr += pstep_r, gr += gstep_r) {
                float s[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) s[q] = dot4(*(const float4 *)(pr + 4 * (q & (K4 - 1))), x[q]);
                const unsigned bo = (r & 1) ? Ns - 1 - b : b;
                if (K4 == 1) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
                        if (q < nsl) gr[(size_t)q * Ns + bo] = s[q];
                } else if (K4 == 2) {
#pragma unroll
                    for (int q = 0; q + 1 < NQ; q += 2)
                        if (q / 2 < nsl) gr[(size_t)(q / 2) * Ns + bo] = s[q] + s[q + 1];
                } else if constexpr (NQ == 4) {
                    gr[bo] = (s[0] + s[1]) + (s[2] + s[3]);
                }
            }
        };
        if (cl[j] < 0) continue;
        // one class in the block (uniform addresses), or several
        const int a0 = __builtin_amdgcn_readfirstlane(cl[j]);
        if (__all(cl[j] == a0)) contract(a0);
        else contract(cl[j]);
    }
}

// g(i,z,b) = sum_k Phi[i][k] sum_lp P_lp(a(i), z, b', k): a workgroup takes
// one class and EPT * NT of its (slice, bin) pairs; a thread adds its pair's
// NLP partial sums once, keeps the KQ channel quads in registers and takes
// every half-turn from them (the Phi rows are uniform over the workgroup).  The
// order of the FP64 partials is fixed by the grid.  Bound by HBM: P, g and h1
// once each; 1024^2 x 8, 300 classes, 12 half-turns with the prox: 466 us with
// a thread per (half-turn, slice, bin) reading P each time, 116 as it is.
template <int KQ>
__global__ __launch_bounds__(NT) void k_contract(
    const float *__restrict__ P, const float *__restrict__ phi, float *__restrict__ out,
    const float *__restrict__ gdata, int mode, float sigma, double *__restrict__ part, int Nz,
    int Ns, int K4, int n0, int Npi, int NLP, int EPT, int nch, int RP)
{
    __shared__ double sh[NT / 64];
    const int rp = blockIdx.x % RP, a = blockIdx.x / RP / nch, ch = blockIdx.x / RP % nch;
    const int rbeg = rp * Npi / RP, rend = (rp + 1) * Npi / RP;
    const int Kp = 4 * K4, ne = Nz * Ns;
    const size_t pstride = (size_t)n0 * ne * Kp;   // between the parts
    double d2 = 0.0;
    const float inv1s = 1.f / (1.f + sigma);
    for (int t = 0; t < EPT; ++t) {
        const int e = (ch * EPT + t) * NT + (int)threadIdx.x;
        if (e >= ne) break;
        const int z = e / Ns, b = e % Ns;
        const float *src = P + ((size_t)a * ne + e) * Kp;
        v4 x[KQ];
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            x[q] = v4{0.f, 0.f, 0.f, 0.f};
            if (q >= K4) continue;
            x[q] = *(const v4 *)(src + 4 * q);
            for (int lp = 1; lp < NLP; ++lp) x[q] += *(const v4 *)(src + lp * pstride + 4 * q);
        }
        for (int r = rbeg; r < rend; ++r) {
            const int i = r * n0 + a;
            const float *ph = phi + (size_t)i * Kp;
            float v = 0.f;
#pragma unroll
            for (int q = 0; q < KQ; ++q)
                if (q < K4) v += dot4(*(const float4 *)(ph + 4 * q), x[q]);
            const size_t o = ((size_t)i * Nz + z) * Ns + ((r & 1) ? Ns - 1 - b : b);
            if (mode == CONTRACT_STORE) {
                out[o] = v;
            } else {   // Fig. 2 step 3: h1 <- (h1 + sigma (R f~ - g)) / (1 + sigma)
                const float d = v - gdata[o];
                d2 += (double)d * (double)d;
                out[o] = (out[o] + sigma * d) * inv1s;
            }
        }
    }
    if (part) {
        const double s = block_sum(d2, sh);
        if (threadIdx.x == 0) part[blockIdx.x] = s;
    }
}

// g~(a,z,b,k) / c = sum_rot Phi[rot*n0+a][k] g(rot*n0+a, z, b') / c(a)  (fold-sum,
// Sec. 4, with the back-projection's 1/c), K rounded up to 4 in a bin.  Bound by
// HBM: g is read once, g~ written once.  A workgroup takes one class, whose Phi
// rows it stages in LDS, and a run of its (slice, bin) pairs; a thread owns one
// channel quad of a pair, so that consecutive threads write consecutive 16
// bytes (a thread per pair wrote at 64-byte strides), and has the g values of
// FB half-turns in flight at a time: 425 -> 281 us at 512^2 x 128, 10 half-turns,
// K = 16 (1.23 GB, 4.4 TB/s).
constexpr int FB = 10;
__global__ __launch_bounds__(NT) void k_fold(const float *__restrict__ g,
                                             const float *__restrict__ phi,
                                             const float *__restrict__ invc,
                                             float *__restrict__ gt, int Nz, int Ns, int K4,
                                             int n0, int Npi, int run, int nrun)
{
    extern __shared__ v4 sphi[];   // Phi rows of class a: [Npi][K4]
    const int a = blockIdx.x / nrun, e0 = (blockIdx.x % nrun) * run;
    for (int e = threadIdx.x; e < Npi * K4; e += NT)
        sphi[e] = *(const v4 *)(phi + ((size_t)(e / K4) * n0 + a) * 4 * K4 + 4 * (e % K4));
    __syncthreads();
    const float ic = invc[a];
    const int ne = Nz * Ns * K4, e1 = min(ne, e0 + run);
    const size_t rstep = (size_t)n0 * Nz * Ns;   // next half-turn of the class
    for (int e = e0 + (int)threadIdx.x; e < e1; e += NT) {
        const int q = e % K4, zb = e / K4, z = zb / Ns, b = zb % Ns;
        const float *src = g + ((size_t)a * Nz + z) * Ns;
        v4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int r0 = 0; r0 < Npi; r0 += FB) {
            float v[FB];
#pragma unroll
            for (int u = 0; u < FB; ++u)
                if (r0 + u < Npi) v[u] = src[(r0 + u) * rstep + (((r0 + u) & 1) ? Ns - 1 - b : b)];
#pragma unroll
            for (int u = 0; u < FB; ++u)
                if (r0 + u < Npi) {
                    const v4 w = sphi[(r0 + u) * K4 + q];
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[t] = fmaf(w[t], v[u], acc[t]);
                }
        }
        *(v4 *)(gt + ((size_t)a * ne + e) * 4) = acc * ic;
    }
}

template <int NQ, int PPT, int PF, bool TL, int NTH, int STG>
static int launch_project_t(const Plan &p, const RayCfg &R, const float *f, const FwdEpi &E,
                            hipStream_t s)
{
    const rt_geom &G = p.g;
    auto kern = k_project<NQ, PPT, PF, TL, NTH, STG>;
    if (R.lds > 64 * 1024)   // beyond the default dynamic LDS limit: ask for what this plan needs
        RT_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)R.lds));
    const RayArgs A{G.N, G.Nz, G.Ns, G.K, R.K4, R.ngroups, R.NLP, R.nblocks};
    KTimer kt("k_project", s);
    hipLaunchKernelGGL(kern, dim3(R.nblocks), dim3(NTH), R.lds, s, f, p.d_scr, p.d_groups + R.group0,
                       p.d_wcls, p.d_lanes + (size_t)(NQ == 4 ? 2 : NQ == 2 ? 1 : 0) * p.n0 * 64,
                       p.d_ccos, p.d_csin, p.d_phip, A, E);
    kt.stop();
    return RT_OK;
}

// the instances RayCfg plans for
template <int NQ, int STG>
static int launch_project_s(const Plan &p, const RayCfg &R, const float *f, const FwdEpi &E,
                            hipStream_t s)
{
    if (R.nth == 256) return launch_project_t<NQ, 1, RAY_PF_SMALL, false, 256, STG>(p, R, f, E, s);
    if (R.tl) return launch_project_t<NQ, 2, RAY_PF, true, 1024, STG>(p, R, f, E, s);
    return launch_project_t<NQ, 2, RAY_PF, false, 1024, STG>(p, R, f, E, s);
}

template <int NQ>
static int launch_project_q(const Plan &p, const RayCfg &R, const float *f, const FwdEpi &E,
                            hipStream_t s)
{
    // the buffer loads need every position of a window to have its own 32-bit
    // offset: those before the line and past it included (STG_LINE), all
    // slices of a workgroup's quads, at most 1 + (NQ - 1) / K4 more (STG_LIST;
    // STG_FEW, whose four slices of at most 3 channels take below 2^30 bytes)
    const rt_geom &g = p.g;
    const size_t lim = (size_t)1 << 32, pos = (size_t)g.N * g.K * 4;
    if (g.K >= 4 && R.K4 % NQ == 0 && (g.N + 2 * RAY_WMAX) * pos < lim)
        return launch_project_s<NQ, STG_LINE>(p, R, f, E, s);
    if (g.K >= 4 && (size_t)NQ * g.N * pos < lim - 4096)
        return launch_project_s<NQ, STG_LIST>(p, R, f, E, s);
    if (g.K < 4) return launch_project_s<NQ, STG_FEW>(p, R, f, E, s);
    return launch_project_s<NQ, STG_REGS>(p, R, f, E, s);
}

// workgroups of k_contract: per class, NT * EPT (slice, bin) pairs and one of RP
// parts of the half-turns each.  The half-turns are walked one after the other
// (their Phi rows, g and h1 are read as they come up): where the pairs make
// less than 4 workgroups per CU, they are split, into no more parts than reading
// P in each of them costs 4 MB.  Measured, one part against the split: 64^2 x 4,
// 30 classes, 40 half-turns, K = 8 14.5 and 9.0 us; 64^2, 90 classes, 8 half-turns
// with the prox 8.4 and 7.6; 8^2 x 5, 34 half-turns, K = 45 30 and 7.5; 512^2, 180
// classes (29 MB of P), 10 half-turns 15.3 and, split into six, 54.6.
struct ContractGrid {
    int EPT, nch, RP;
    unsigned nb;
};
static ContractGrid contract_grid(const Plan &p, int NLP)
{
    const long ne = (long)p.g.Nz * p.g.Ns;
    ContractGrid c;
    c.EPT = (int)std::max(1L, std::min(4L, ne * p.n0 / (4096L * NT)));
    c.nch = (int)((ne + (long)NT * c.EPT - 1) / ((long)NT * c.EPT));
    const long nw = std::max((long)p.n0 * c.nch, 1L), pb = std::max(NLP * ne * p.n0 * ((p.g.K + 3) / 4 * 16), 1L);
    c.RP = (int)std::max(1L, std::min<long>({p.g.Npi, (1024 + nw - 1) / nw, 1 + (4L << 20) / pb}));
    c.nb = (unsigned)(nw * c.RP);
    return c;
}

}  // namespace

int launch_forward_pf(const Plan &p, const float *f, float *g, int mode, const float *gdata,
                      float *h1, float sigma, double *part, hipStream_t s)
{
    const rt_geom &G = p.g;
    if (G.Nz == 0) return RT_OK;
    const RayCfg &R = p.ray;
    // The h1 prox runs in k_contract: its reads of g and h1 at the end of the
    // projection, one workgroup per CU, are covered by nothing (512^2 x 32: 2.84
    // ms with the prox inside, 2.69 + 0.12 without).  So is the contraction of
    // more than 16 half-turns where the workgroups are few (8^2 x 22, 234 classes,
    // 19 of them, K = 16: 27.9 us inside, 22.0 outside); in large volumes the two
    // are equal (315^2 x 20, 40 of them 320 and 325 us), and fewer half-turns are
    // better inside (512^2 x 128, 10 of them: 9.90 and 10.03 ms).
    const bool fused = R.fusable && mode == CONTRACT_STORE && G.Npi <= 16;
    const FwdEpi E{fused ? g : nullptr, p.n0, G.Npi};
    const int rc = R.NQ == 4   ? launch_project_q<4>(p, R, f, E, s)
                   : R.NQ == 2 ? launch_project_q<2>(p, R, f, E, s)
                               : launch_project_q<1>(p, R, f, E, s);
    if (rc) return rc;
    RT_HIP(hipGetLastError());
    if (fused) return RT_OK;
    const ContractGrid c = contract_grid(p, R.NLP);
    KTimer kt("k_contract", s);
#define RT_CONTRACT(Q) hipLaunchKernelGGL(k_contract<Q>, dim3(c.nb), dim3(NT), 0, s, p.d_scr, p.d_phip, \
                                          mode == CONTRACT_STORE ? g : h1, gdata, mode, sigma, part, G.Nz, G.Ns, R.K4, p.n0,    \
                                          G.Npi, R.NLP, c.EPT, c.nch, c.RP)
    if (R.K4 <= 2) RT_CONTRACT(2);
    else if (R.K4 <= 4) RT_CONTRACT(4);
    else if (R.K4 <= 8) RT_CONTRACT(8);
    else RT_CONTRACT(16);
#undef RT_CONTRACT
    kt.stop();
    RT_HIP(hipGetLastError());
    return RT_OK;
}

int forward_partials(const Plan &p)   // of the h1 prox
{
    if (p.form == RT_FORM_SF) return (int)sf_partials(p);
    return (int)contract_grid(p, p.ray.NLP).nb;
}

int launch_forward(const Plan &p, const float *f, float *g, int mode, const float *gdata,
                   float *h1, float sigma, double *part, hipStream_t s)
{
    if (p.form == RT_FORM_SF) return launch_forward_sf(p, f, g, mode, gdata, h1, sigma, part, s);
    return launch_forward_pf(p, f, g, mode, gdata, h1, sigma, part, s);
}

int launch_adjoint(const Plan &p, const float *g, float *out, hipStream_t s)
{
    if (p.form == RT_FORM_SF) {
        int rc = launch_fold_mfma(p, g, s);
        return rc ? rc : launch_backproject(p, out, s);
    }
    return launch_adjoint_pf(p, g, out, s);
}

int launch_adjoint_pf(const Plan &p, const float *g, float *out, hipStream_t s)
{
    const rt_geom &G = p.g;
    if (G.Nz == 0) return RT_OK;
    // a workgroup per class and run of 4 NT channel quads, fewer where that
    // gives less than 4 workgroups per CU
    const int K4 = (G.K + 3) / 4;
    const long ne = (long)G.Nz * G.Ns * K4;
    const int run = NT * (int)std::max(1L, std::min(4L, ne * p.n0 / (1024L * NT)));
    const int nrun = (int)((ne + run - 1) / run);
    KTimer kt("k_fold", s);
    hipLaunchKernelGGL(k_fold, dim3((unsigned)p.n0 * nrun), dim3(NT), (size_t)G.Npi * K4 * 16, s, g,
                       p.d_phip, p.d_invc, p.d_scr, G.Nz, G.Ns, K4, p.n0, G.Npi, run, nrun);
    kt.stop();
    RT_HIP(hipGetLastError());
    return launch_backproject(p, out, s);
}

}  // namespace rt
