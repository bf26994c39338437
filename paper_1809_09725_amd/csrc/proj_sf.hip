// Precision form of R_T and R_T*: the basis contraction sum_k Phi[i][k] f_k
// (and its transpose) in BF16 on the matrix cores with FP32 accumulation,
// the projection itself in FP32.
//
// Forward, synthesise-first: for each line (row or column) of slice z the
// states of the line at the Npi half-turns of the workgroup's angle classes
// are formed on MFMA,
//   F[c][pos] = sum_k Phi[i(c)][k] f_k(line, pos),   c = (class slot, half-turn),
// from a BF16 shadow of f (kept beside f~ by the primal update, or converted
// on entry) and Phi split into BF16 hi + lo parts, FP32 accumulate; each ray
// (class, bin) then takes Joseph's two interpolation taps on the frames of
// its class (Sec. 2 eq. Rfwd: the state at time t_i is projected at
// theta_i; the pi-periodicity of Sec. 4 lets every half-turn of a class share
// one ray walk, odd half-turns landing on bin Ns-1-b).
//
// Adjoint: the fold-sum g~(a,z,b,k) = sum_r Phi[r*Ntheta0+a][k] g(r*Ntheta0+a,
// z, b') (Sec. 4) as BF16 MFMA products with FP32 accumulation, then the FP32
// pixel-driven back-projection shared with the plain form.
#include "common.h"
#include "internal.h"

namespace rt {
namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));


// FP32 -> BF16 with round-to-nearest-even (finite inputs).
__device__ inline unsigned short bf16_rne(float x)
{
    const unsigned u = __float_as_uint(x);
    return (unsigned short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline float bf16_val(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

struct SfEpi {
    float *out;           // g (EPI_G) or h1 (EPI_PROX); with line parts: partial sums
    const float *gdata;   // measured sinogram (EPI_PROX)
    double *part;         // per-workgroup FP64 sum of (R f~ - g)^2, or NULL
    size_t pstride;       // line parts: floats between the parts' partial sums
    float sigma;
    int prox, n0, Npi;
};

__device__ inline long long uniform64(long long v)
{
    return (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                       (unsigned)__builtin_amdgcn_readfirstlane((int)v));
}

// The bin offset thread tid (of the NB side by side) takes for class a: its own, reordered within its
// wave's block of 64 bins by the class's lane map (the 16-lane tap reads at
// positions 1/|c| apart then spread over the LDS bank groups; the row stride
// CS is an odd number of 16-byte groups).
__device__ inline int sf_bin(int tid, int a, const unsigned char *__restrict__ lperm)
{
    return a >= 0 ? (tid & ~63) | (int)lperm[a * 64 + (tid & 63)] : tid;
}

// Forward, synthesise-first.  Workgroup: slice z, a group of A classes of one
// walk direction, bins [bt*BT, bt*BT + BT), and part lp of the NLP parts of
// the slice's lines (NLP > 1: the ray sums over those lines are stored at
// E.out + lp * E.pstride for k_sf_finish).  Consecutive workgroups take the
// class groups of one part, so the part's BF16 lines are read while they are
// still cached.  A thread owns the rays (slot, bin) of its half of the A slots
// (of all of them with one slot or fewer than 1024 threads) at UT bins each.
// NPP: frame columns per class (Npi rounded up to 4, the padding columns are
// zero); KB: MFMA k-steps of 16 channels.
//
// The frames F[c][pos] = sum_k Phi[i(c)][k] f_k(pos) of a chunk of PCH
// positions are one v_mfma_f32_32x32x16_bf16 product per 32-position tile,
// one tile per wave: A = Phi rows of the 32 frame columns (hi and lo BF16
// parts), B = the BF16 shadow of f.  They land in LDS position-major, row
// 1 + pos - c0 holding the frames of position pos, so that a ray's tap at one
// position is NPP/4 16-byte reads, the access of the plain form's staged lines.
//
// What bounds it: per line of 1024 positions and 4 classes of 8 half-turns the
// LDS takes about 2100 cycles (1024 for the frames' stores, 1100 for the
// taps' reads), the vector units 1300 and the matrix cores 1024, of 5200 in
// all; the operand loads (128-byte lines, of which a column walk uses half)
// are hidden.  Two frame buffers let one barrier per step do, with the
// products of the next step running under the taps of this one; 16 waves of
// half the rays each (ST = 1024; ST = 512 where these would lack rays: two
// workgroups per CU; 640 and 768 where a line then is one chunk) keep more of the
// LDS reads in flight than 8.  Measured, 1024^2 x 8, 256 classes, 8 half-turns,
// K = 32: 7.4 ms with one buffer and two barriers per chunk, 5.6 with two
// buffers and 8 waves, 4.5 as it is; 512^2 x 16, 180 classes, K = 16: 2.24 ->
// 1.47 ms; 2048^2 x 2, 64 classes, 12 half-turns, K = 32: 3.42 -> 2.20 ms.
// Waves per SIMD asked for: with 33..48 channels and two bins or slots of up
// to 20 half-turns a thread, 512 threads are held to 128 registers (a few more
// otherwise), so that two workgroups do fit a CU: 512^2 x 16, 16 half-turns, K =
// 48: 5.40 -> 4.67 ms.  More sums, or more channels, would spill tens of
// registers (256^2 x 16, 16 half-turns, K = 64: 1.13 -> 1.85 ms).
constexpr int sf_waves(int npp, int kb, int as, int ub, int st)
{
    return st == 512 && kb == 3 && as * ub == 2 && npp <= 20 ? 4 : (st + 255) / 256;
}
template <int NPP, int KB, int AS, int UB, int ST>
__global__ __launch_bounds__(ST, sf_waves(NPP, KB, AS, UB, ST)) void k_project_sf(
    const __bf16 *__restrict__ f16, const float *__restrict__ phi, const int *__restrict__ gcls,
    const int *__restrict__ gwalk, const unsigned char *__restrict__ lperm, const double *__restrict__ ccos,
    const double *__restrict__ csin, int N, int Nz, int Ns, int K, int A, int ngroups, int BT,
    int nbt, int PCH, int NLP, unsigned nblocks, SfEpi E)
{
    constexpr int KP = 16 * KB;
    constexpr int CS = 4 * ((AS * NPP / 4) | 1);   // floats per row
    // waves: with 1024 threads and several slots, the two halves of the
    // workgroup take half of the slots each; NB threads side by side take UT bins each per slot
    constexpr int SH = AS > 1 && ST == 1024 ? 2 : 1, AT = AS / SH, NB = ST / SH, UT = (UB * 512 + NB - 1) / NB;
    constexpr int R = AT * UT;      // rays per thread: slot j0 + rho / UT, bin sf_bin(tb) + NB * (rho % UT)
    extern __shared__ float fr[];   // two buffers [PCH + 3][CS]; rows 0, PCH + 1 and PCH + 2 stay zero
    __shared__ double sh[ST / 64];
    unsigned lid = xcd_remap(blockIdx.x, nblocks);
    const int bt = lid % nbt;
    lid /= nbt;
    const int grp = lid % ngroups;
    lid /= ngroups;
    const int lp = lid % NLP;
    const int z = lid / NLP;
    const int lbeg = (int)((long)lp * N / NLP), lend = (int)((long)(lp + 1) * N / NLP);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = SH > 1 ? wave / (NB / 64) : 0, tb = tid - half * NB, j0 = half * AT;
    const int walk = gwalk[grp];
    const int Npi = E.Npi;
    const double hN = 0.5 * (double)(N - 1), hS = 0.5 * (double)(Ns - 1);

    // ---- rays of this thread: position on line lbeg and its step per line
    // (one value per class), in 32.32 fixed point as in the plain projector:
    // FP64 once, then one exact integer add per line (the position carries the
    // rounding of its start and of l s alone, below 2^-32 (1 + l)).  A ray
    // outside the tile starts at -1e6 and stays outside.
    long long U[R], Sl[AT];
    float invc[AT];
#pragma unroll
    for (int j = 0; j < AT; ++j) {
        const int a = j0 + j < A ? gcls[grp * A + j0 + j] : -1;
        const double cs = a >= 0 ? ccos[a] : 1.0, sn = a >= 0 ? csin[a] : 0.0;
        const double d = a < 0 || walk == 0 ? cs : sn, n = a < 0 || walk == 0 ? sn : cs;
        const double slope = -n / d;
        invc[j] = (float)(1.0 / fabs(d));
        Sl[j] = uniform64((long long)llrint(slope * 4294967296.0));
#pragma unroll
        for (int u = 0; u < UT; ++u) {
            const int bi = sf_bin(tb, a, lperm) + NB * u, b = bt * BT + bi;
            double u0 = -1.0e6;
            if (a >= 0 && bi < BT && b < Ns)
                u0 = fma((double)lbeg - hN, slope, ((double)b - hS) / d + hN);
            U[j * UT + u] = (long long)llrint(fmin(fmax(u0, -1.0e6), 1.0e6) * 4294967296.0);
        }
    }
    float acc[R][NPP];
#pragma unroll
    for (int rho = 0; rho < R; ++rho)
#pragma unroll
        for (int r = 0; r < NPP; ++r) acc[rho][r] = 0.f;

    // ---- MFMA A operand: Phi[i(c)][k] of frame column c = lane % 32 (slot
    // c / NPP, half-turn c % NPP), channels kb*16 + 8*(lane/32) + 0..7
    v8bf ahi[KB], alo[KB];
    {
        const int c = lane & 31, slot = c / NPP, r = c % NPP;
        const int a = (slot < A && r < Npi) ? gcls[grp * A + slot] : -1;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int k = kb * 16 + 8 * (lane >> 5) + q;
                const float v = (a >= 0 && k < K) ? phi[(size_t)(r * E.n0 + a) * K + k] : 0.f;
                const __bf16 h = (__bf16)v;
                ahi[kb][q] = h;
                alo[kb][q] = (__bf16)(v - (float)h);
            }
    }

    const int bufsz = (PCH + 3) * CS;
    for (int e = tid; e < 6 * CS; e += ST) {
        const int k = e / CS, r = k % 3;
        fr[k / 3 * bufsz + (r ? PCH + r : 0) * CS + e % CS] = 0.f;
    }

    const __bf16 *fz = f16 + (size_t)z * N * N * KP;
    const size_t lstep = walk == 0 ? (size_t)N * KP : (size_t)KP;
    const size_t pstep = walk == 0 ? (size_t)KP : (size_t)N * KP;
    const int nch = (N + PCH - 1) / PCH;
    const int nsteps = (lend - lbeg) * nch;   // (line, chunk) steps of this part

    // B operand of one step for the wave's position tile: lane holds
    // position c0 + wave*32 + lane%32, channels kb*16 + 8*(lane/32) + 0..7.
    // Steps are loaded in order; past the last one the last line is read again.
    // Positions past the slice read its last one and are zeroed before the
    // product (zeroed as they were loaded, the waves at a line's end waited for
    // their loads in every step, and the workgroup with them: 300^2 x 2, 567 bins,
    // 329 classes, 18 half-turns, K = 54: 1.84 and 1.21 ms).
    v8bf raw[KB];
    const int lpos = 32 * wave + (lane & 31);
    const unsigned pbytes = (unsigned)pstep * 2;   // a slice is at most 2^31 bytes
    const char *line = (const char *)(fz + (size_t)lbeg * lstep);
    // first position of the chunk: to load next, loaded, of the frames, and tapped
    int lc0 = 0, rc0 = 0, dc0 = 0, c0 = 0;
    int left = lend - lbeg;
    auto load_step = [&]() {
        const unsigned off = (unsigned)min(lc0 + lpos, N - 1) * pbytes + 16 * (lane >> 5);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) raw[kb] = *(const v8bf *)(line + off + kb * 32);
        rc0 = lc0;
        lc0 += PCH;
        if (lc0 >= N) {
            lc0 = 0;
            line += --left > 0 ? 2 * lstep : 0;
        }
    };
    // the frames of one step
    v16f d;
    auto frames = [&]() {
        if (rc0 + 32 * wave + 32 > N) {
            asm volatile("");   // a branch: as selects in every step 3 to 5% slower
            const bool in = rc0 + lpos < N;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) raw[kb] = in ? raw[kb] : v8bf{};
        }
        c0 = dc0;
        dc0 = rc0;
        d = v16f{};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi[kb], raw[kb], d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo[kb], raw[kb], d, 0, 0, 0);
        }
    };
    // ... into a buffer.  D[c][pos]: lane holds position lane%32 of its tile,
    // columns 8g + 4(lane/32) + 0..3
    auto store = [&](int buf) {
        if (wave * 32 >= PCH) return;
        float *row = fr + buf * bufsz + (1 + wave * 32 + (lane & 31)) * CS + 4 * (lane >> 5);
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (8 * g + 8 <= AS * NPP || (8 * g < AS * NPP && lane < 32))
                *(float4 *)(row + 8 * g) = make_float4(d[4 * g], d[4 * g + 1], d[4 * g + 2], d[4 * g + 3]);
    };
    // Taps of the rays whose positions fall in step st's chunk: rows q and
    // q + 1 of the line, -1 <= q < PCH relative to the chunk; the zero rows on
    // both sides stand for the neighbouring chunks' positions and for those
    // outside the slice.  The rays of one bin set are taken together wherever
    // one of the wave's is in the chunk (the group's classes are close in
    // angle), the others reading the two zero rows at the end.
    int row[R];
    float frc[R];
    auto taps = [&](int buf) {
        if (c0 == 0) {   // ray positions on this step's line
#pragma unroll
            for (int rho = 0; rho < R; ++rho) {
                const unsigned q = (unsigned)(int)(U[rho] >> 32) + 1u;
                frc[rho] = (float)(unsigned)U[rho] * 2.3283064365386963e-10f;
                U[rho] += Sl[rho / UT];
                row[rho] = q <= (unsigned)N ? (int)q : 1 << 28;
            }
        }
        const float *fb = fr + buf * bufsz + j0 * NPP;
#pragma unroll
        for (int u = 0; u < UT; ++u) {
            unsigned q[AT];
            bool any = false;
#pragma unroll
            for (int j = 0; j < AT; ++j) {
                q[j] = min((unsigned)(row[j * UT + u] - c0), (unsigned)PCH + 1u);
                any |= q[j] <= (unsigned)PCH;
            }
            if (!__any(any)) continue;
#pragma unroll
            for (int j = 0; j < AT; ++j) {
                const int rho = j * UT + u;
                const float a1 = frc[rho], a0 = 1.f - a1;
                const float *F0 = fb + __umul24(q[j], CS) + j * NPP;
#pragma unroll
                for (int m = 0; m < NPP / 4; ++m) {
                    const float4 x0 = *(const float4 *)(F0 + 4 * m);
                    const float4 x1 = *(const float4 *)(F0 + CS + 4 * m);
                    acc[rho][4 * m + 0] = fmaf(a1, x1.x, fmaf(a0, x0.x, acc[rho][4 * m + 0]));
                    acc[rho][4 * m + 1] = fmaf(a1, x1.y, fmaf(a0, x0.y, acc[rho][4 * m + 1]));
                    acc[rho][4 * m + 2] = fmaf(a1, x1.z, fmaf(a0, x0.z, acc[rho][4 * m + 2]));
                    acc[rho][4 * m + 3] = fmaf(a1, x1.w, fmaf(a0, x0.w, acc[rho][4 * m + 3]));
                }
            }
        }
    };

    // Step st taps buffer st % 2; the matrix cores form the frames of step
    // st + 1 meanwhile, from operands loaded one step ahead, and they are
    // stored to the other buffer at the end.
    if (nsteps > 0) {
        load_step();
        frames();
        load_step();
        store(0);
        __syncthreads();
        for (int st = 0; st < nsteps; ++st) {
            const int buf = st & 1;
            frames();
            load_step();
            taps(buf);
            store(buf ^ 1);
            __syncthreads();
        }
    }

    // ---- epilogue: every half-turn r of class a lands on bin b (even r) or Ns-1-b (odd r)
    double d2 = 0.0;
    const float inv1s = 1.f / (1.f + E.sigma);
    // out and gdata do not overlap: the loads of all half-turns may be issued
    // ahead of the stores
    const float *__restrict__ gd = E.gdata;
    float *__restrict__ out = E.out;
#pragma unroll
    for (int rho = 0; rho < R; ++rho) {
        const int j = rho / UT;
        const int a = j0 + j < A ? gcls[grp * A + j0 + j] : -1;
        const int bi = sf_bin(tb, a, lperm) + NB * (rho % UT), b = bt * BT + bi;
        if (a < 0 || bi >= BT || b >= Ns) continue;
#pragma unroll
        for (int r = 0; r < NPP; ++r) {
            if (r >= Npi) continue;
            const int i = r * E.n0 + a;
            const int bo = (r & 1) ? Ns - 1 - b : b;
            const size_t o = ((size_t)i * Nz + z) * Ns + bo;
            const float v = acc[rho][r] * invc[j];
            if (!E.prox) {
                out[o + lp * E.pstride] = v;
            } else {
                const float d = v - gd[o];
                d2 += (double)d * (double)d;
                out[o] = (out[o] + E.sigma * d) * inv1s;
            }
        }
    }
    if (E.part) {
        const double sum = block_sum(d2, sh);
        if (tid == 0) E.part[blockIdx.x] = sum;
    }
}

// The line parts' partial ray sums added in part order, then stored as g or
// taken into the h1 prox of Fig. 2 step 3 with the FP64 partial sums of
// (R f~ - g)^2; rows grid-strided over a fixed number of workgroups.
__global__ __launch_bounds__(NT) void k_sf_finish(const float *__restrict__ psf, int NLP,
                                                  size_t ng, float *__restrict__ out,
                                                  const float *__restrict__ gdata, int prox,
                                                  float sigma, double *__restrict__ part)
{
    __shared__ double sh[NT / 64];
    double d2 = 0.0;
    const float inv1s = 1.f / (1.f + sigma);
    for (size_t o = (size_t)blockIdx.x * NT + threadIdx.x; o < ng; o += (size_t)gridDim.x * NT) {
        float v = psf[o];
        for (int lp = 1; lp < NLP; ++lp) v += psf[(size_t)lp * ng + o];
        if (!prox) {
            out[o] = v;
        } else {
            const float d = v - gdata[o];
            d2 += (double)d * (double)d;
            out[o] = (out[o] + sigma * d) * inv1s;
        }
    }
    if (part) {
        const double s = block_sum(d2, sh);
        if (threadIdx.x == 0) part[blockIdx.x] = s;
    }
}

unsigned sf_finish_blocks(const rt_geom &G)
{
    const size_t ng = ng_of(G);
    return (unsigned)std::max<size_t>(1, std::min<size_t>((ng + NT - 1) / NT, 8192));
}

// BF16 shadow of f: [Nz][N][N][K] FP32 -> [Nz][N][N][KP] BF16 (round to
// nearest even), channels K..KP-1 zero.  One thread per 8 output channels.
__global__ __launch_bounds__(NT) void k_to_bf16(const float *__restrict__ f,
                                                __bf16 *__restrict__ out, size_t nvox, int K,
                                                int KP)
{
    const int n8 = KP / 8;
    const size_t total = nvox * n8;
    for (size_t e = (size_t)blockIdx.x * NT + threadIdx.x; e < total;
         e += (size_t)gridDim.x * NT) {
        const size_t v = e / n8;
        const int k0 = (int)(e % n8) * 8;
        const float *src = f + v * K;
        v8bf o;
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = (__bf16)(k0 + q < K ? src[k0 + q] : 0.f);
        *(v8bf *)(out + v * KP + k0) = o;
    }
}

// Fold-sum on MFMA (v_mfma_f32_16x16x16 bf16): per (class a, slice z) the
// product [Ns bins x Npi half-turns] x [Npi x K], half-turns padded to a
// multiple of 16.  One wave per 16-bin x 16-channel tile.
// A: lane holds bins row = lane%16, half-turns 4*(lane/16) + 0..3 of the
// current 16-chunk; B: Phi rows of those half-turns, channel lane%16;
// C: bins 4*(lane/16) + 0..3, channel lane%16.  Stored as g~ / c(a) (the
// back-projection's weights), K rounded up to 4 in a bin.
// Both operands are split into BF16 hi + lo parts and the three products
// hi*hi + hi*lo + lo*hi are accumulated in FP32 (the lo*lo term is below
// 2^-16 of the product): the sinogram fed to the adjoint is the dual h1 of
// the data term, whose rounding to a single BF16 would put a 2^-9 relative
// error straight into the primal update when few half-turns and classes
// average it.  The fold is bound by its HBM traffic, so the two extra
// products cost nothing measurable.
__global__ __launch_bounds__(NT) void k_fold_mfma(const float *__restrict__ g,
                                                  const float *__restrict__ phi,
                                                  const float *__restrict__ invc,
                                                  float *__restrict__ gt, int Nz, int Ns, int K,
                                                  int n0, int Npi)
{
    // wave-uniform, so that the tile's numbers and 1/c are formed and read on the
    // scalar unit: with a vector read of 1/c just before the stores 140 us at
    // 1024^2 x 8, 256 classes, 8 half-turns, K = 32, without 1/c 120, as it is 116
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nbt = (Ns + 15) / 16, nkt = (K + 15) / 16, Kp = (K + 3) / 4 * 4;
    const long tiles = (long)n0 * Nz * nbt * nkt;
    for (long t = (long)blockIdx.x * (NT / 64) + wave; t < tiles; t += (long)gridDim.x * (NT / 64)) {
        long u = t;
        const int kt = (int)(u % nkt);
        u /= nkt;
        const int btile = (int)(u % nbt);
        u /= nbt;
        const int z = (int)(u % Nz);
        const int a = (int)(u / Nz);
        const int bin = btile * 16 + (lane & 15);
        const int kcol = kt * 16 + (lane & 15);
        v4f cacc = {0.f, 0.f, 0.f, 0.f};
        for (int r0 = 0; r0 < Npi; r0 += 16) {
            v4s ah, al, bh, bl;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + 4 * (lane >> 4) + q;
                float gv = 0.f, pv = 0.f;
                if (r < Npi) {
                    const int i = r * n0 + a;
                    if (bin < Ns) gv = g[((size_t)i * Nz + z) * Ns + ((r & 1) ? Ns - 1 - bin : bin)];
                    if (kcol < K) pv = phi[(size_t)i * K + kcol];
                }
                const unsigned short gh = bf16_rne(gv);
                ah[q] = (short)gh;
                al[q] = (short)bf16_rne(gv - bf16_val(gh));
                const unsigned short h = bf16_rne(pv);
                bh[q] = (short)h;
                bl[q] = (short)bf16_rne(pv - bf16_val(h));
            }
            cacc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(al, bh, cacc, 0, 0, 0);
            cacc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bl, cacc, 0, 0, 0);
            cacc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bh, cacc, 0, 0, 0);
        }
        if (kcol < Kp) {
            const float ic = invc[a];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int bo = btile * 16 + 4 * (lane >> 4) + q;
                if (bo < Ns) gt[(((size_t)a * Nz + z) * Ns + bo) * Kp + kcol] = cacc[q] * ic;
            }
        }
    }
}

template <int NPP, int KB, int AS, int UB, int ST>
static int launch_sf_s(const Plan &p, const SfEpi &E, hipStream_t s, unsigned nb)
{
    const rt_geom &G = p.g;
    const SfCfg &C = p.sf;
    auto kern = k_project_sf<NPP, KB, AS, UB, ST>;
    if (C.lds > 64 * 1024)
        RT_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)C.lds));
    KTimer kt("k_project_sf", s);
    hipLaunchKernelGGL(kern, dim3(nb), dim3(ST), C.lds, s, (const __bf16 *)p.d_f16, p.d_phi,
                       p.d_gcls_sf, p.d_gwalk_sf, p.d_lanes, p.d_ccos, p.d_csin, G.N, G.Nz, G.Ns, G.K, C.A,
                       C.ngroups, C.BT, C.nbt, C.PCH, C.NLP, nb, E);
    kt.stop();
    return RT_OK;
}

template <int NPP, int KB, int AS, int UB>
static int launch_sf_t(const Plan &p, const SfEpi &E, hipStream_t s, unsigned nb)
{
    if constexpr (UB == 1 || KB >= 3) {   // as the plan chooses ST
        if (p.sf.ST == 512) return launch_sf_s<NPP, KB, AS, UB, 512>(p, E, s, nb);
    }
    if constexpr ((UB == 1 && NPP > 8) || KB >= 3) {
        if (p.sf.ST == 640) return launch_sf_s<NPP, KB, AS, UB, 640>(p, E, s, nb);
        if (p.sf.ST == 768) return launch_sf_s<NPP, KB, AS, UB, 768>(p, E, s, nb);
    }
    return launch_sf_s<NPP, KB, AS, UB, 1024>(p, E, s, nb);
}

// AS slots for one bin per thread; UB bins per thread take AS / UB slots
// the slot count sf_slots gives: at most 96 ray sums and 8 rays per thread
// (64 and 4 when K > 32)
constexpr int acc_cap(int kb) { return kb >= 3 ? 64 : 96; }
constexpr int fit_slots(int as, int ub, int npp, int kb)
{
    return (as > 1 && (as * ub * npp > acc_cap(kb) || as * ub > (kb >= 3 ? 4 : 8)))
               ? fit_slots(as - 1, ub, npp, kb) : as;
}

template <int NPP, int KB, int AS>
static int launch_sf_u(const Plan &p, const SfEpi &E, hipStream_t s, unsigned nb)
{
    constexpr int AS2 = fit_slots(AS, 2, NPP, KB), AS4 = fit_slots(AS, 4, NPP, KB);
    switch (p.sf.UB) {
    case 1: return launch_sf_t<NPP, KB, fit_slots(AS, 1, NPP, KB), 1>(p, E, s, nb);
    case 2: return launch_sf_t<NPP, KB, AS2, 2>(p, E, s, nb);
    default:
        // the plan keeps UB * slots * NPP within acc_cap accumulators per thread
        if constexpr (4 * AS4 * NPP <= acc_cap(KB)) {
            return launch_sf_t<NPP, KB, AS4, 4>(p, E, s, nb);
        } else {
            return fail(RT_E_SHAPE, "no synthesise-first kernel for NPP=%d with 4 bins per thread", NPP);
        }
    }
}

template <int NPP, int AS>
static int launch_sf_k(const Plan &p, const SfEpi &E, hipStream_t s, unsigned nb)
{
    switch (p.sf.KP / 16) {
    case 1: return launch_sf_u<NPP, 1, AS>(p, E, s, nb);
    case 2: return launch_sf_u<NPP, 2, AS>(p, E, s, nb);
    case 3: return launch_sf_u<NPP, 3, AS>(p, E, s, nb);
    default: return launch_sf_u<NPP, 4, AS>(p, E, s, nb);
    }
}

}  // namespace

unsigned sf_blocks(const Plan &p)
{
    return (unsigned)p.g.Nz * p.sf.ngroups * p.sf.nbt * p.sf.NLP;
}

// FP64 partials of the forward's h1 prox: one per projection workgroup, or one
// per k_sf_finish workgroup when the lines come in parts
unsigned sf_partials(const Plan &p) { return p.sf.NLP > 1 ? sf_finish_blocks(p.g) : sf_blocks(p); }

int sf_slots(int npp, int ub, int kb)
{
    int as = npp <= 8 ? 4 : npp <= 16 ? 2 : 1;
    while (as > 1 && (as * ub * npp > (kb >= 3 ? 64 : 96) || as * ub > (kb >= 3 ? 4 : 8))) --as;
    return as;
}

int launch_to_bf16(const Plan &p, const float *f, hipStream_t s)
{
    const rt_geom &G = p.g;
    const size_t nvox = (size_t)G.Nz * G.N * G.N;
    if (nvox == 0) return RT_OK;
    const size_t total = nvox * (p.sf.KP / 8);
    const unsigned nb = (unsigned)std::min<size_t>((total + NT - 1) / NT, 16384);
    KTimer kt("k_to_bf16", s);
    hipLaunchKernelGGL(k_to_bf16, dim3(nb), dim3(NT), 0, s, f, (__bf16 *)p.d_f16, nvox, G.K,
                       p.sf.KP);
    kt.stop();
    RT_HIP(hipGetLastError());
    ++p.shadow_gen;
    return RT_OK;
}

int launch_forward_sf16(const Plan &p, float *g, int mode, const float *gdata, float *h1,
                        float sigma, double *part, hipStream_t s)
{
    const rt_geom &G = p.g;
    if (G.Nz == 0) return RT_OK;
    SfEpi E{};
    float *dst = mode == CONTRACT_STORE ? g : h1;
    const bool parts = p.sf.NLP > 1;
    float *sums = p.d_psf ? p.d_psf : p.d_scr;
    E.out = parts ? sums : dst;
    E.gdata = gdata;
    E.part = parts ? nullptr : part;
    E.pstride = parts ? ng_of(G) : 0;
    E.sigma = sigma;
    E.prox = !parts && mode == CONTRACT_PROX;
    E.n0 = p.n0;
    E.Npi = G.Npi;
    const unsigned nb = sf_blocks(p);
    int rc;
    switch (p.sf.NPP) {
    case 4: rc = launch_sf_k<4, 4>(p, E, s, nb); break;
    case 8: rc = launch_sf_k<8, 4>(p, E, s, nb); break;
    case 12: rc = launch_sf_k<12, 2>(p, E, s, nb); break;
    case 16: rc = launch_sf_k<16, 2>(p, E, s, nb); break;
    case 20: rc = launch_sf_k<20, 1>(p, E, s, nb); break;
    case 24: rc = launch_sf_k<24, 1>(p, E, s, nb); break;
    case 28: rc = launch_sf_k<28, 1>(p, E, s, nb); break;
    default: rc = launch_sf_k<32, 1>(p, E, s, nb); break;
    }
    if (rc) return rc;
    RT_HIP(hipGetLastError());
    if (parts) {
        KTimer kt("k_sf_finish", s);
        hipLaunchKernelGGL(k_sf_finish, dim3(sf_finish_blocks(G)), dim3(NT), 0, s, sums,
                           p.sf.NLP, ng_of(G), dst, gdata, mode == CONTRACT_PROX ? 1 : 0, sigma,
                           part);
        kt.stop();
        RT_HIP(hipGetLastError());
    }
    return RT_OK;
}

int launch_forward_sf(const Plan &p, const float *f, float *g, int mode, const float *gdata,
                      float *h1, float sigma, double *part, hipStream_t s)
{
    if (p.g.Nz == 0) return RT_OK;
    int rc = launch_to_bf16(p, f, s);
    if (rc) return rc;
    return launch_forward_sf16(p, g, mode, gdata, h1, sigma, part, s);
}

int launch_fold_mfma(const Plan &p, const float *g, hipStream_t s)
{
    const rt_geom &G = p.g;
    if (G.Nz == 0) return RT_OK;
    const long tiles = (long)p.n0 * G.Nz * ((G.Ns + 15) / 16) * ((G.K + 15) / 16);
    const unsigned nb = (unsigned)std::max<long>(1, std::min<long>((tiles + 3) / 4, 16384));
    KTimer kt("k_fold_mfma", s);
    hipLaunchKernelGGL(k_fold_mfma, dim3(nb), dim3(NT), 0, s, g, p.d_phi, p.d_invc, p.d_scr, G.Nz,
                       G.Ns, G.K, p.n0, G.Npi);
    kt.stop();
    RT_HIP(hipGetLastError());
    return RT_OK;
}

}  // namespace rt
