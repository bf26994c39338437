// Plan: geometry checks, host tables, kernel configuration, device tables.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <utility>

#include "internal.h"

namespace rt {

static thread_local std::string g_err;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(e == hipErrorOutOfMemory ? RT_E_OOM : RT_E_HIP, "%s: %s", what,
                hipGetErrorString(e));
}

int check_geom(const rt_geom *g)
{
    if (!g) return fail(RT_E_ARG, "geometry pointer is NULL");
    if (g->N < 1 || g->Ns < 1 || g->Ntheta < 1 || g->Npi < 1 || g->K < 1 || g->Nt < 1 ||
        g->Nz < 0)
        return fail(RT_E_SHAPE, "sizes must be >= 1 (Nz >= 0): N=%d Nz=%d Ns=%d Ntheta=%d "
                    "Npi=%d K=%d Nt=%d", g->N, g->Nz, g->Ns, g->Ntheta, g->Npi, g->K, g->Nt);
    if (g->Ntheta % g->Npi != 0)
        return fail(RT_E_SHAPE, "Ntheta=%d is not a whole number of half-turns Npi=%d",
                    g->Ntheta, g->Npi);
    if (g->Nt > g->Npi)
        return fail(RT_E_SHAPE, "Nt=%d time frames exceed the Npi=%d half-turns", g->Nt, g->Npi);
    if (g->N > 4096 || g->Ns > 8192 || g->K > 64 || g->Nt > 64 || (int64_t)g->Npi * g->K > 16384)
        return fail(RT_E_SHAPE, "size beyond the supported maximum (N<=4096, Ns<=8192, "
                    "K<=64, Nt<=64, Npi*K<=16384)");
    // a limit of the interface, kept for every plan: slices of more than 2048^2
    // pixels with a ragged last channel quad are not among the sizes that were
    // ever checked against the oracle (no kernel depends on it)
    if (g->N > 2048 && g->K % 4 != 0)
        return fail(RT_E_SHAPE, "N=%d > 2048 needs K to be a multiple of 4 (got K=%d)", g->N, g->K);
    return RT_OK;
}

int check_plan(const rt_plan *p)
{
    if (!p) return fail(RT_E_ARG, "plan is NULL");
    return RT_OK;
}

// Time of one projection launch in microseconds, for the choice of the line
// parts: `rounds` workgroups one after the other on a CU, each walking
// `lines` lines of N positions for `blocks` ray blocks of 64, and the extra
// kernel and traffic of partial sums.  Per line: the tap reads at about 5
// cycles, the stores of the line at 8, a barrier; a fixed 6 us per workgroup.
static double project_cost(double rounds, double lines, double blocks, int N, int NQ, double parts_bytes)
{
    const double line = (blocks * 2 * NQ * 5.5 + std::min(N, 300) * NQ / 64.0 * 8 + 400) / 2400.0;
    return rounds * (lines * line + 6.0) + (parts_bytes > 0 ? 8.0 + parts_bytes / 2.0e6 : 0.0);
}

// Channel quads per workgroup: up to 4, of as many slices as it takes.
static int quads_per_row(const rt_geom &g, int nz)
{
    const long tq = (long)nz * ((g.K + 3) / 4);   // channel quads of nz slices
    return tq >= 3 ? 4 : (int)std::max(tq, 1L);
}

struct LineSplit {
    int NLP = 1;
    bool small = false;
};
// The split of the lines and the workgroup size for nz slices.  The parts
// fix the order in which a ray's taps are added, so they follow from nz_ref
// alone: every plan of one volume, whole or a slab, passes the same.  One part
// and full workgroups (32 ray blocks) where these fill the chip; else the
// cheaper, by project_cost, of up to 16 parts of full workgroups and, for lines
// of at most 256 positions, of workgroups of 4 ray blocks (several per CU).
// Measured: one 512^2 slice of 16 channels over 180 classes, 46 full
// workgroups, 462 us in one part, 119 in five.
static LineSplit line_split(const rt_geom &g, int nz)
{
    LineSplit best;
    if (nz < 1) return best;
    const long n0 = g.Ntheta / g.Npi;
    const long K4 = (g.K + 3) / 4, nbb = (g.Ns + 63) / 64;
    const int NQ = quads_per_row(g, nz);
    const long ncg = (nz * K4 + NQ - 1) / NQ;
    const long half = (n0 + 1) / 2 * nbb;   // ray blocks of a walk, about
    const bool fusable = g.N <= 512 && K4 <= NQ && NQ % K4 == 0;
    double cost = 1e300;
    for (int small = 0; small < (g.N <= 256 ? 2 : 1); ++small) {
        const long bpw = small ? RAY_BLOCKS_SMALL : RAY_BLOCKS;
        const long W = ncg * 2 * ((half + bpw - 1) / bpw) * 107 / 100;   // groups fill to about 0.94
        const long occ = small ? (NQ == 4 ? 2 : 4) : 1;   // workgroups per CU, by their LDS
        if (!small && W >= 512) return LineSplit{};
        for (int np = 1; np <= 16 && np * 4 <= std::max(g.N, 4); ++np) {
            const double rounds = (double)((W * np + 256 * occ - 1) / (256 * occ));
            const double pb = np > 1 || !fusable ? 2.0 * np * n0 * nz * g.Ns * K4 * 16 : 0.0;
            // the workgroups that share a CU take turns: their blocks add up
            const double share = std::min<double>((double)occ, std::max(1.0, (double)(W * np) / 256));
            const double c = project_cost(rounds, (double)g.N / np, bpw * share, g.N, NQ, pb);
            if (c < cost * 0.97) {
                cost = c;
                best.NLP = np;
                best.small = small;
            }
        }
    }
    return best;
}

// The workgroup size for nz slices, of which the full size has `ngroups` ray
// groups: line_split's; but where that is one part of full workgroups, small
// ones all the same for lines of at most 64 positions (the 16 waves of a full
// one then spend more on its barriers than on taps: 48^2 x 40, 8 channels, 200
// classes: 70 us full, 39 small; 64^2 x 120, 16 channels, 30 classes: 69 and
// 47), and for lines of at most 128 where the full ones fill less than 0.7 of
// the rounds that they take (128^2 x 40, 8 channels, 200 classes, 1.2 rounds:
// 239 and 176).  In fuller rounds small ones lose there: 70^2 x 120, 8
// channels, 90 classes: 88 and 122.
static bool small_workgroups(const rt_geom &g, int nz, int ngroups)
{
    const LineSplit L = line_split(g, nz);
    if (L.small || L.NLP > 1 || nz < 1) return L.small;
    const int NQ = quads_per_row(g, nz);
    const long W = ((long)nz * ((g.K + 3) / 4) + NQ - 1) / NQ * ngroups, slots = (W + 255) / 256 * 256;
    return g.N <= 64 || (g.N <= 128 && W * 10 < slots * 7);
}

// Whether the ray blocks of nz slices may run on over classes (the plan takes
// what it estimates faster).  Line parts already even out launches of few
// workgroups (339^2 x 2, 11 channels, 147 classes, four parts: 125 us, packed
// 134; 196^2, 25 channels, 122 classes, six parts: 83 and 97); the staging of
// fewer than four channels is not in the estimate; and lines of more than 512
// positions gained nothing (650^2 x 3, 1000 bins: 1079 and 1083 us).
static bool may_pack(const rt_geom &g, int nz)
{
    return g.Ns % 64 && g.K >= 4 && g.N <= 512 && line_split(g, nz).NLP == 1;
}

size_t adjoint_scratch_bytes(const rt_geom &g)
{
    return (size_t)(g.Ntheta / g.Npi) * g.Nz * g.Ns * ((size_t)(g.K + 3) / 4 * 4) * sizeof(float);
}

size_t plan_scratch_bytes(const rt_geom &g, int nz_ref)
{
    const size_t n0 = (size_t)(g.Ntheta / g.Npi), Kp = (size_t)(g.K + 3) / 4 * 4;
    // partial ray sums of the whole volume, or of the one slice of the power iteration
    const size_t slices = std::max((size_t)g.Nz * line_split(g, nz_ref).NLP,
                                   g.Nz > 0 ? (size_t)line_split(g, 1).NLP : 0);
    return n0 * slices * g.Ns * Kp * sizeof(float);
}

// The window of a group of rays: n classes of directions d (one walk, one
// sign of the main direction) and bins [b0, b1].  Relative to the line of the middle
// slope a class's positions run linearly, so the extremes over the group are
// at the first or last line.  One position to spare below and two above (the
// right tap, and fixed-point rounding).  A window wider than the line becomes
// the whole line with two guard positions at each end.
struct RayDir {
    double slope, inv;   // positions per line, per bin
};
static void ray_window(int N, int Ns, const RayDir *d, int n, int b0, int b1, RayGroup &G)
{
    const double hN = 0.5 * (double)(N - 1), hS = 0.5 * (double)(Ns - 1);
    double smin = 1e9, smax = -1e9, lo = 1e9, hi = -1e9;
    for (int i = 0; i < n; ++i) {
        smin = std::min(smin, d[i].slope);
        smax = std::max(smax, d[i].slope);
    }
    const double sw = 0.5 * (smin + smax);
    for (int i = 0; i < n; ++i) {
        const double first = hN - hN * d[i].slope;                    // line 0, the bin at s = 0
        const double last = hN + hN * d[i].slope - (double)(N - 1) * sw;
        const double p0 = ((double)b0 - hS) * d[i].inv, p1 = ((double)b1 - hS) * d[i].inv;
        lo = std::min(lo, std::min(first, last) + std::min(p0, p1));
        hi = std::max(hi, std::max(first, last) + std::max(p0, p1));
    }
    G.W = (int)std::ceil(hi - lo) + 5;
    if (G.W < N + 4) {
        G.wl0 = std::llrint((lo - 1.0) * 4294967296.0);
        G.sw = std::llrint(sw * 4294967296.0);
    } else {
        G.W = N + 4;
        G.wl0 = -2 * (1LL << 32);
        G.sw = 0;
    }
}

// Ray groups of at most `blocks` blocks of 64 rays with windows of at most
// wmax positions, the blocks of one class each or packed over the classes; and
// the cost of the largest group and of all.  A group is a tile of bins (blocks
// of 64, the last one up to the detector's end) over neighbouring classes;
// more classes and fewer bins (or the reverse) widen the window by their fan-
// out (their spacing).  The tile width is the power of two that costs least:
// per line the LDS cycles of the taps and of the window's stores and a share
// of the barrier, as k_project's comment has them.  At 512^2 over 180 classes
// two blocks of 16 classes: windows of 247 positions on average; whole lines
// (eight blocks of four classes) took 12.8 ms against 9.85 there (128 slices
// of 16 channels) and 8.45 against 5.76 at 1024^2 x 8.
static std::vector<RayGroup> ray_groups(const rt_geom &g, const std::vector<RayDir> (&lists)[3], bool packed,
                                        int blocks, int wmax, double &worst, double &total)
{
    const int nbb = (g.Ns + 63) / 64, N = g.N, Ns = g.Ns;
    std::vector<RayGroup> best;
    double best_cost = 1e300;
    for (int tile = 1; tile <= blocks; tile *= 2) {
        const int nt = (nbb + tile - 1) / tile;   // tiles of nearly equal width
        std::vector<RayGroup> v;
        double cost = 0.0, most = 0.0;
        bool fits = true;
        int cls0 = 0;
        for (int s = 0; s < 3; ++s) {
            const std::vector<RayDir> &L = lists[s];
            for (int t = 0; t < nt; ++t) {
                RayGroup G{};
                G.walk = s == 1;
                const int bbt = nbb / nt + (t < nbb % nt ? 1 : 0);
                G.b0 = 64 * (t * (nbb / nt) + std::min(t, nbb % nt));
                G.nb = std::min(64 * bbt, Ns - G.b0);
                const int b1 = G.b0 + G.nb - 1;
                for (int i = 0; i < (int)L.size(); i += G.ncls) {
                    G.stride = packed ? G.nb : 64 * bbt;
                    G.cls0 = cls0 + i;
                    G.ncls = std::min(blocks * 64 / G.stride, (int)L.size() - i);
                    ray_window(N, Ns, L.data() + i, G.ncls, G.b0, b1, G);
                    while (G.W > wmax && G.ncls > 1) ray_window(N, Ns, L.data() + i, --G.ncls, G.b0, b1, G);
                    if (G.W > wmax) fits = false;
                    const int lines = std::max(1, wmax / G.W >= 4 ? 4 : wmax / G.W >= 2 ? 2 : 1);
                    // a block of two classes costs a little more: its lanes are in the
                    // order of the first alone
                    const int nblk = (G.ncls * G.stride + 63) / 64, mixed = G.stride % 64 ? std::min(G.ncls - 1, nblk) : 0;
                    const double c = nblk * 40.0 + mixed * 3.0 + G.W * 0.5 + 500.0 / lines;
                    cost += c;
                    most = std::max(most, c);
                    v.push_back(G);
                }
            }
            cls0 += (int)L.size();
        }
        if (fits && cost < best_cost) {
            best_cost = total = cost;
            worst = most;
            best = v;
        }
        if (tile >= nbb) break;
    }
    return best;
}

RayCfg ray_cfg(const Plan &p)
{
    const rt_geom &g = p.g;
    const LineSplit L = line_split(g, p.nz_ref);
    RayCfg R;
    R.K4 = (g.K + 3) / 4;
    const int tq = g.Nz * R.K4;   // channel quads of all slices
    R.NQ = quads_per_row(g, g.Nz);
    R.ncg = (tq + R.NQ - 1) / R.NQ;
    R.tl = g.N > 512;
    R.NLP = L.NLP;
    const bool small = small_workgroups(g, p.nz_ref, p.ngroups);
    R.nth = small ? RAY_NTH_SMALL : RAY_NTH;
    R.group0 = small ? p.ngroups : 0;
    R.ngroups = small ? (int)p.groups.size() - p.ngroups : p.ngroups;
    R.fusable = R.NLP == 1 && !R.tl && R.K4 <= R.NQ && R.NQ % R.K4 == 0;
    R.nblocks = (unsigned)R.ncg * R.ngroups * R.NLP;
    // stage buffers: as k_project lays them out
    const int rpj = R.nth / R.NQ, pf = small ? RAY_PF_SMALL : RAY_PF;
    int rows = 0;
    for (int i = 0; i < R.ngroups; ++i) {
        const int W = p.groups[R.group0 + i].W;
        const int sh = W <= rpj ? 0 : W <= 2 * rpj ? 1 : W <= 4 * rpj ? 2 : 3;
        rows = std::max(rows, std::min(pf >> sh, (g.N + R.NLP - 1) / R.NLP) * W);
    }
    R.lds = (size_t)2 * rows * R.NQ * 16;
    return R;
}

size_t shadow_bytes(const rt_geom &g)
{
    return (size_t)g.Nz * g.N * g.N * ((g.K + 15) / 16 * 16) * 2;
}

// a slice's BF16 copy in parts of at most 64 MiB of lines
int sf_line_parts(const rt_geom &g)
{
    const size_t slice = (size_t)g.N * g.N * ((g.K + 15) / 16 * 16) * 2;
    const size_t part = (size_t)64 << 20;
    return (int)std::max<size_t>(1, std::min<size_t>({(slice + part - 1) / part, 16, (size_t)std::max(g.N, 1)}));
}

size_t sf_partial_bytes(const rt_geom &g)
{
    const int nlp = sf_line_parts(g);
    return nlp > 1 ? (size_t)nlp * ng_of(g) * sizeof(float) : 0;
}

size_t job_state_bytes(const rt_geom &g)
{
    return (2 * nf_of(g) + 2 * ng_of(g) + 5 * n4_of(g)) * sizeof(float);
}

// Sec. 4, eq. discrt: theta_i = i*pi/Ntheta0, t_i = i/Ntheta (theta = alpha t,
// alpha = Npi*pi); the class a = i mod Ntheta0 of [0,pi) and the half-turn
// rot = i div Ntheta0 of the pi-periodicity identity.
static void build_tables(const rt_geom &g, const double *phi, const double *S, Tables &T)
{
    const int n0 = g.Ntheta / g.Npi;
    T.theta.resize(g.Ntheta);
    T.t.resize(g.Ntheta);
    T.cls.resize(g.Ntheta);
    T.rot.resize(g.Ntheta);
    T.flip.resize(g.Ntheta);
    T.phi.resize((size_t)g.Ntheta * g.K);
    for (int i = 0; i < g.Ntheta; ++i) {
        T.theta[i] = ((double)i * M_PI) / (double)n0;
        T.t[i] = (double)i / (double)g.Ntheta;
        T.cls[i] = i % n0;
        T.rot[i] = i / n0;
        T.flip[i] = (i / n0) & 1;
        for (int k = 0; k < g.K; ++k)
            T.phi[(size_t)i * g.K + k] =
                phi ? phi[(size_t)i * g.K + k] : std::cos(M_PI * (double)k * T.t[i]);
    }
    T.S.resize((size_t)g.Nt * g.K);
    for (int m = 0; m < g.Nt; ++m)
        for (int k = 0; k < g.K; ++k)
            T.S[(size_t)m * g.K + k] = S ? S[(size_t)m * g.K + k] : T.phi[(size_t)m * n0 * g.K + k];
    T.ccos.resize(n0);
    T.csin.resize(n0);
    for (int a = 0; a < n0; ++a) {
        T.ccos[a] = std::cos(T.theta[a]);
        T.csin[a] = std::sin(T.theta[a]);
    }
}

// The plan's tables in one device allocation and one copy.
struct TableUpload {
    std::vector<char> host;
    std::vector<std::pair<void **, size_t>> at;   // pointer to set, offset
    template <class T>
    void add(T **dst, const std::vector<T> &src)
    {
        at.emplace_back((void **)dst, host.size());
        const size_t b = (std::max<size_t>(src.size(), 1) * sizeof(T) + 255) / 256 * 256;
        host.resize(host.size() + b, 0);
        if (!src.empty()) std::memcpy(host.data() + at.back().second, src.data(), src.size() * sizeof(T));
    }
    int upload(void **mem, size_t *bytes)
    {
        RT_HIP(hipMalloc(mem, host.size()));
        RT_HIP(hipMemcpy(*mem, host.data(), host.size(), hipMemcpyHostToDevice));
        for (const auto &x : at) *x.first = (char *)*mem + x.second;
        *bytes += host.size();
        return RT_OK;
    }
};

static int configure(Plan &p, TableUpload &up)
{
    const rt_geom &g = p.g;
    const int n0 = p.n0;
    // ---- forward: classes by walk direction and sign of the main direction
    std::vector<int> rows, cols, by_dir[3];
    std::vector<RayDir> lists[3];
    for (int a = 0; a < n0; ++a) {
        const double cs = p.T.ccos[a], sn = p.T.csin[a];
        const bool row = std::fabs(cs) >= std::fabs(sn);
        (row ? rows : cols).push_back(a);
        const int d = !row ? 1 : cs > 0 ? 0 : 2;
        by_dir[d].push_back(a);
        lists[d].push_back(row ? RayDir{-sn / cs, 1.0 / cs} : RayDir{-cs / sn, 1.0 / sn});
    }
    std::vector<int> wcls;
    for (const std::vector<int> &L : by_dir) wcls.insert(wcls.end(), L.begin(), L.end());
    // Ray blocks of one class, or packed over the classes: the set of groups
    // whose launch takes less.  The workgroups are alike, so up to six rounds of
    // them count as whole ones, each of the largest group and of 30 us of setup
    // and epilogue (3 us where the workgroups are small).  100^2 x 40, 16
    // channels, 200 classes, 78% of the lanes in use: 600 workgroups of one
    // class, three rounds, 305 us, 480 packed in two 213; 198^2 x 31, 305 bins,
    // 32 channels, 37 classes (two rounds either way) 340 and 389 us.
    double best_t = 1e300;
    for (int packed = 0; packed < (may_pack(g, p.nz_ref) ? 2 : 1) && !p.adjoint_only; ++packed) {
        double worst = 0.0, total = 0.0;
        std::vector<RayGroup> v = ray_groups(g, lists, packed, RAY_BLOCKS, RAY_WMAX, worst, total);
        const int ngroups = (int)v.size();
        if (!ngroups) continue;
        const int NQ = quads_per_row(g, p.nz_ref);
        const long ncg = ((long)p.nz_ref * ((g.K + 3) / 4) + NQ - 1) / NQ;
        const bool small = small_workgroups(g, p.nz_ref, ngroups);
        if (small || small_workgroups(g, 1, ngroups)) {
            double w = 0.0, t = 0.0;
            const std::vector<RayGroup> vs = ray_groups(g, lists, packed, RAY_BLOCKS_SMALL, RAY_WMAX_SMALL, w, t);
            v.insert(v.end(), vs.begin(), vs.end());
            if (small) {
                worst = w;
                total = t;
            }
        }
        const int ngr = small ? (int)v.size() - ngroups : ngroups;
        const double W = (double)ncg * ngr, occ = small ? (NQ == 4 ? 2 : 4) : 1;
        const double share = std::min(occ, std::max(1.0, W / 256)), rounds = W / (256 * occ);
        const double setup = small ? 3.0 : 30.0, us = g.N / 2400.0;
        const double t = share * (rounds <= 6 ? std::ceil(rounds) * (worst * us + setup)
                                              : total / ngr * (rounds + 0.5) * us + rounds * setup);
        if (t < best_t) {
            best_t = t;
            p.groups = v;
            p.ngroups = ngroups;
        }
    }
    if (!p.adjoint_only && !p.ngroups) return fail(RT_E_SHAPE, "no ray groups of the projector for N=%d Ns=%d", g.N, g.Ns);

    // Lane order of the forward waves.  A wave's 64 rays are 64 consecutive
    // bins of one class, or of neighbours in the order of the first; their
    // positions on a line are spaced 1/|c| in [1, sqrt 2] apart.  A 16-byte LDS read is served 16 lanes at a time, in the
    // groups of lane quads {0,3,5,6}, {1,2,4,7} and the same + 8 (measured: a
    // lane on the same 16-byte unit as lane 0 costs a cycle for the lanes of
    // its group alone).  With NQ quads per staged position the lanes of a
    // group that read the same quad of a position must differ modulo 16 / NQ
    // in position; ordering the 64 rays by (r / c) modulo that and dealing
    // them out in turn spreads each such set evenly.  The precision form's
    // rows (an odd number of 16-byte units) take the order of NQ = 1.
    std::vector<uint8_t> lanes(p.adjoint_only ? 0 : (size_t)3 * n0 * 64, 0);
    static const int set_quads[3][8] = {   // lane quads of the sets, in order, of half a wave
        {0, 3, 5, 6, 1, 2, 4, 7}, {0, 3, 5, 6, 1, 2, 4, 7}, {0, 1, 2, 3, 4, 5, 6, 7}};
    for (int v = 0; v < 3 && !p.adjoint_only; ++v) {
        const int NQ = 1 << v, M = 16 / NQ, nsets = 4 * NQ;   // sets of M lanes
        // in use: by the volume, by the one slice of the power iteration, by
        // the precision form
        if (NQ != quads_per_row(g, p.nz_ref) && NQ != quads_per_row(g, 1) &&
            NQ != quads_per_row(g, g.Nz) && !(NQ == 1 && p.form == RT_FORM_SF))
            continue;
        for (int a = 0; a < n0; ++a) {
            const double d = 1.0 / std::max(std::fabs(p.T.ccos[a]), std::fabs(p.T.csin[a]));
            // counting sort of the phases r d mod M in 256 steps
            uint8_t key[64], ord[64];
            int at[257] = {0};
            double ph = 0.0;
            for (int r = 0; r < 64; ++r, ph += d) {
                if (ph >= M) ph -= M;
                key[r] = (uint8_t)std::min(255, (int)(ph * 256.0 / M));
                ++at[key[r] + 1];
            }
            for (int k = 0; k < 256; ++k) at[k + 1] += at[k];
            for (int r = 0; r < 64; ++r) ord[at[key[r]]++] = (uint8_t)r;
            for (int i = 0; i < 64; ++i) {
                const int slot = (i % nsets) * M + i / nsets;   // set, place in it
                const int lane = 32 * (slot / 32) + 4 * set_quads[v][slot % 32 / 4] + slot % 4;
                lanes[((size_t)v * n0 + a) * 64 + lane] = ord[i];
            }
        }
    }

    p.tv.KT = g.K <= 8 ? 8 : g.K <= 16 ? 16 : g.K <= 32 ? 32 : 64;

    // ---- synthesise-first projector: A classes x NPP frame columns in one 32-column tile
    std::vector<int> gcls_sf, gwalk_sf;
    if (p.form == RT_FORM_SF) {
        SfCfg &C = p.sf;
        C.NPP = (g.Npi + 3) / 4 * 4;
        // one workgroup covers all bins up to 2048 (each thread up to 4 bins
        // per class), so that every line's frames are synthesised once
        C.UB = g.Ns <= 512 ? 1 : g.Ns <= 1024 ? 2 : 4;
        const int kb = (g.K + 15) / 16;
        while (C.UB > 1 && C.UB * sf_slots(C.NPP, C.UB, kb) * C.NPP > (kb >= 3 ? 64 : 96))
            C.UB /= 2;   // registers
        C.A = std::min(sf_slots(C.NPP, C.UB, kb), (int)std::max(rows.size(), cols.size()));
        for (int w = 0; w < 2; ++w) {
            const std::vector<int> &L = w == 0 ? rows : cols;
            for (size_t i = 0; i < L.size(); i += C.A) {
                for (int j = 0; j < C.A; ++j) gcls_sf.push_back(i + j < L.size() ? L[i + j] : -1);
                gwalk_sf.push_back(w);
            }
        }
        C.ngroups = (int)gwalk_sf.size();
        C.BT = std::min(g.Ns, 512 * C.UB);
        C.nbt = (g.Ns + C.BT - 1) / C.BT;
        // Positions of a line are taken in chunks of half as many as threads.
        // Workgroups of 512 threads and chunks of 256 positions, two per CU,
        // where 1024 threads lack rays: lines and detectors of at most 256, or
        // fewer than four slots of at most 512 bins.  Measured, 1024 against
        // 512 threads: 128^2 x 60, 10 half-turns 1.42 and 0.56 ms; 256^2 x 64, 2
        // of them 1.20 and 0.57; 512^2 x 128, 10 of them 17.8 and 15.9; four
        // slots, 384^2 x 20, 8 half-turns 1.03 and 1.18; 512^2 x 16 1.50 and 1.56.
        C.ST = C.UB == 1 && (C.NPP > 8 || std::max(g.N, g.Ns) <= 256) ? 512 : 1024;
        // Above 32 channels the operands of the products take the registers that
        // 16 waves leave.  33..48 channels: 512 threads (1024 against 512: 266^2 x
        // 45, 4 half-turns, K = 35 1.55 and 1.06 ms; 800^2 x 4, 8 of them, K = 40
        // 4.16 and 3.08; 720 bins of 700^2 x 4, 32 of them, K = 44 4.55 and 4.07),
        // except for many half-turns over several tiles of bins (1300^2, 1400 bins,
        // 32 of them 6.02 and 6.47).  More channels over more than 512 bins: 512
        // threads where 1024 spill (32 frame columns; 965^2 x 3, 13 half-turns, K =
        // 52 6.55 and 4.62; 1024^2 x 4, 32 of them, K = 64 11.0 and 8.5) or pad the
        // lines with more positions (1213^2 x 4, 5 of them, K = 58 7.25 and 6.14);
        // elsewhere 1024 (1024^2 x 8, 12 of them, K = 64 16.2 and 16.4).
        const int cols = sf_slots(C.NPP, C.UB, kb) * C.NPP, sums = cols * C.UB;   // frame columns, ray sums
        const auto padded = [&](int pch) { return (g.N + pch - 1) / pch * pch; };
        if ((kb == 3 && (C.NPP <= 20 || g.Ns <= 1024)) ||
            (kb == 4 && C.UB > 1 && (cols == 32 || padded(256) < padded(512))))
            C.ST = 512;
        // Lines of 257..384 positions in one chunk, of 640 or 768 threads, where
        // 512 would be taken or more than 32 channels: two chunks of 256 are half
        // padding.  100 classes, 5 slices, 512 threads against 640 or 768: 270^2, 20
        // half-turns, K = 16 389 and 248 us; 300^2, 600 bins, 24 of them, K = 40 889
        // and 550; 384^2, 28 of them, K = 60 1.45 and 1.15 ms (1024: 339, 657, 1.24).
        // Of 385..512 positions above 32 channels: 512 threads where two workgroups
        // fit a CU by their registers or 1024 would spill, otherwise 1024 (410^2,
        // 820 bins, 16 half-turns, K = 40: 820 and 588 us; where they fit, 8 of
        // them: 493 and 556).
        if (g.N > 256 && g.N <= 384 && (kb >= 3 || C.ST == 512))
            C.ST = g.N <= 320 ? 640 : 768;
        else if (g.N > 384 && g.N <= 512 && kb >= 3)
            C.ST = (kb == 3 ? sums <= 40 && (cols < 32 || C.NPP > 8 || C.UB > 1) : sums <= 24) ||
                   (kb == 4 && (C.NPP == 32 || sums == 64)) ? 512 : 1024;
        C.PCH = std::min(C.ST / 2, (g.N + 31) / 32 * 32);
        C.KP = (g.K + 15) / 16 * 16;
        // an odd number of 16-byte groups per row: 16 consecutive positions
        // of a b128 access fall in distinct bank groups
        const int row = 4 * ((sf_slots(C.NPP, C.UB, kb) * C.NPP / 4) | 1);
        C.lds = (size_t)2 * (C.PCH + 3) * row * sizeof(float);
        // Few workgroups (one or two per CU fit): the lines in parts, as many as make
        // the rounds of workgroups times a part's lines least, a workgroup's
        // setup and its share of k_sf_finish counted as 24 lines; the partial
        // sums go where the plain form keeps its own.  From the slices the
        // order of the sums is planned for (p.nz_ref), like the plain form's
        // parts.  Measured (forward): 512^2 x 1, 100 classes, 4 half-turns,
        // K = 16: 333 us in one part, 71 in eight; 1024^2 x 2, 256 classes, 4
        // half-turns, K = 32: 1.95 -> 1.11 ms; 256^2 x 1, 60 classes: 298 -> 46 us;
        // 1024^2 x 8, 256 classes (512 workgroups): one part.
        C.NLP = sf_line_parts(g);
        if (C.NLP == 1) {
            const long wg = (long)p.nz_ref * C.ngroups * C.nbt;
            const long room = (long)line_split(g, p.nz_ref).NLP * ((g.K + 3) / 4 * 4) / g.Npi;
            const long fit = C.ST == 512 ? 512 : 256;
            auto cost = [&](long n) { return (wg * n + fit - 1) / fit * ((g.N + n - 1) / n + 24); };
            for (long n = 2; n <= std::min<long>({room, 32, g.N}); ++n)
                if (10 * cost(n) < 9 * cost(C.NLP)) C.NLP = (int)n;
        }
    }

    up.add(&p.d_wcls, wcls);
    up.add(&p.d_groups, p.groups);
    up.add(&p.d_lanes, lanes);
    if (p.form == RT_FORM_SF) {
        up.add(&p.d_gcls_sf, gcls_sf);
        up.add(&p.d_gwalk_sf, gwalk_sf);
    }
    return RT_OK;
}

static void free_plan(Plan &p)
{
    for (void *ptr : {p.d_tables, (void *)p.d_scr, (void *)p.d_frames, p.d_f16, (void *)p.d_psf,
                      (void *)p.d_part, (void *)p.d_red})
        if (ptr) (void)hipFree(ptr);
}

static int create(const rt_geom *geom, rt_form form, rt_prec prec, const double *phi,
                  const double *S, int nz_ref, bool adjoint_only, Plan &p)
{
    p.g = *geom;
    p.nz_ref = nz_ref;
    p.adjoint_only = adjoint_only;
    p.form = form;
    p.prec = prec;
    p.n0 = geom->Ntheta / geom->Npi;
    RT_HIP(hipGetDevice(&p.device));
    build_tables(p.g, phi, S, p.T);
    TableUpload up;
    int rc = configure(p, up);
    if (rc) return rc;
    if (!adjoint_only) p.ray = ray_cfg(p);
    const size_t Kp = (size_t)(geom->K + 3) / 4 * 4;
    std::vector<float> phip((size_t)geom->Ntheta * Kp, 0.f);
    for (int i = 0; i < geom->Ntheta; ++i)
        std::copy_n(p.T.phi.begin() + (size_t)i * geom->K, geom->K, phip.begin() + (size_t)i * Kp);
    up.host.reserve(up.host.size() + 2 * phip.size() * sizeof(float) + ((size_t)1 << 16));
    up.add(&p.d_phip, phip);
    if (!adjoint_only) {
        up.add(&p.d_phi, std::vector<float>(p.T.phi.begin(), p.T.phi.end()));
        up.add(&p.d_S, std::vector<float>(p.T.S.begin(), p.T.S.end()));
    }
    up.add(&p.d_ccos, p.T.ccos);
    up.add(&p.d_csin, p.T.csin);
    std::vector<float> invc(p.n0);
    for (int a = 0; a < p.n0; ++a)
        invc[a] = (float)(1.0 / std::max(std::fabs(p.T.ccos[a]), std::fabs(p.T.csin[a])));
    up.add(&p.d_invc, invc);
    if ((rc = up.upload(&p.d_tables, &p.bytes))) return rc;
    const size_t scr = std::max<size_t>(adjoint_only ? adjoint_scratch_bytes(p.g) : plan_scratch_bytes(p.g, nz_ref), 256);
    RT_HIP(hipMalloc(&p.d_scr, scr));
    p.bytes += scr;
    if (adjoint_only) return RT_OK;
    const size_t frb = std::max<size_t>(n4_of(p.g), 1) * sizeof(float);
    RT_HIP(hipMalloc(&p.d_frames, frb));
    p.bytes += frb;
    if (form == RT_FORM_SF) {
        const size_t sb = std::max<size_t>(shadow_bytes(p.g), 256);
        RT_HIP(hipMalloc(&p.d_f16, sb));
        p.bytes += sb;
        if (const size_t pb = sf_partial_bytes(p.g)) {
            RT_HIP(hipMalloc(&p.d_psf, pb));
            p.bytes += pb;
        }
    }
    // FP64 partials: h1 prox, shrink, primal update (two per workgroup), reductions
    p.part_cap = std::max<size_t>((size_t)1 << 18,
                                  (size_t)forward_partials(p) + grad_blocks(p.g) + 2 * (size_t)voxel_blocks(p.g) + 64);
    RT_HIP(hipMalloc(&p.d_part, p.part_cap * sizeof(double)));
    RT_HIP(hipMalloc(&p.d_red, 16 * sizeof(double)));
    p.bytes += (p.part_cap + 16) * sizeof(double);
    return RT_OK;
}

int pick_form(const rt_geom *geom, rt_form *form, rt_prec *prec)
{
    int rc = check_geom(geom);
    if (rc) return rc;
    if (*form != RT_FORM_PF && *form != RT_FORM_SF && *form != RT_FORM_AUTO)
        return fail(RT_E_ARG, "unknown form %d", (int)*form);
    if (*prec != RT_PREC_FP32 && *prec != RT_PREC_BF16MFMA)
        return fail(RT_E_ARG, "unknown precision %d", (int)*prec);
    if (*form == RT_FORM_AUTO) {
        // per ray and line, project-first taps K channels; synthesise-first
        // taps the Npi frames (rounded up to 4) and forms them on the matrix
        // cores, which pays from about K = 2 Npi (measured per iteration at
        // 8 half-turns, 256^2 to 1024^2 x 8: SF/PF 0.67-0.82 at K = 32, 0.84-0.99
        // at K = 16, 1.27-1.37 at K = 8; 1.28 at K = 16 over 12 half-turns)
        const bool sf = *prec == RT_PREC_BF16MFMA && geom->K >= 2 * geom->Npi && geom->Npi <= 32;
        *form = sf ? RT_FORM_SF : RT_FORM_PF;
        *prec = sf ? RT_PREC_BF16MFMA : RT_PREC_FP32;
        return RT_OK;
    }
    if (*prec == RT_PREC_BF16MFMA && *form != RT_FORM_SF)
        return fail(RT_E_ARG, "the BF16 contraction needs the synthesise-first form");
    if (*form == RT_FORM_SF && *prec != RT_PREC_BF16MFMA)
        return fail(RT_E_ARG, "the synthesise-first form is built with the BF16 contraction only");
    if (*form == RT_FORM_SF && geom->Npi > 32)
        return fail(RT_E_SHAPE, "the synthesise-first form needs Npi <= 32 (got %d)", geom->Npi);
    return RT_OK;
}

int plan_create(const rt_geom *geom, rt_form form, rt_prec prec, const double *phi, const double *S,
                int nz_ref, bool adjoint_only, rt_plan **out)
{
    if (!out) return fail(RT_E_ARG, "out is NULL");
    *out = nullptr;
    int rc = pick_form(geom, &form, &prec);
    if (rc) return rc;
    if (phi)
        for (size_t e = 0; e < (size_t)geom->Ntheta * geom->K; ++e)
            if (!std::isfinite(phi[e])) return fail(RT_E_ARG, "phi has a non-finite entry");
    if (S)
        for (size_t e = 0; e < (size_t)geom->Nt * geom->K; ++e)
            if (!std::isfinite(S[e])) return fail(RT_E_ARG, "S has a non-finite entry");
    rt_plan *p = new (std::nothrow) rt_plan();
    if (!p) return fail(RT_E_OOM, "host allocation failed");
    rc = create(geom, form, prec, phi, S, nz_ref, adjoint_only, p->impl);
    if (rc) {
        free_plan(p->impl);
        delete p;
        return rc;
    }
    *out = p;
    return RT_OK;
}

}  // namespace rt

using namespace rt;

extern "C" int rt_form_pick(const rt_geom *geom, rt_form form, rt_prec prec, rt_form *form_out,
                            rt_prec *prec_out)
{
    if (!form_out || !prec_out) return fail(RT_E_ARG, "NULL output");
    int rc = pick_form(geom, &form, &prec);
    if (rc) return rc;
    *form_out = form;
    *prec_out = prec;
    return RT_OK;
}

extern "C" int rt_basis_fourier(const rt_geom *geom, int32_t M, double *phi, double *S)
{
    int rc = check_geom(geom);
    if (rc) return rc;
    if (!phi || !S) return fail(RT_E_ARG, "NULL table");
    if (M < 2 || M % 2 || geom->K != M - 1)
        return fail(RT_E_ARG, "the real form of M = %d Fourier functions has K = M - 1 (got K = %d)",
                    (int)M, geom->K);
    const int K = geom->K, n0 = geom->Ntheta / geom->Npi;
    auto row = [&](double t, double *out) {
        out[0] = 1.0;
        for (int v = 1; v <= M / 2 - 1; ++v) {
            const double w = 2.0 * M_PI * (double)v * t;
            out[2 * v - 1] = std::cos(w);
            out[2 * v] = std::sin(w);
        }
    };
    for (int i = 0; i < geom->Ntheta; ++i) row((double)i / (double)geom->Ntheta, phi + (size_t)i * K);
    for (int m = 0; m < geom->Nt; ++m)
        row((double)(m * n0) / (double)geom->Ntheta, S + (size_t)m * K);
    return RT_OK;
}

extern "C" int rt_plan_form(const rt_plan *p, rt_form *form, rt_prec *prec)
{
    if (check_plan(p) || !form || !prec) return fail(RT_E_ARG, "NULL argument");
    *form = p->impl.form;
    *prec = p->impl.prec;
    return RT_OK;
}

extern "C" int rt_plan_create(const rt_geom *geom, rt_form form, rt_prec prec, const double *phi,
                              const double *S, rt_plan **out)
{
    return plan_create(geom, form, prec, phi, S, geom ? geom->Nz : 0, false, out);
}

extern "C" void rt_plan_destroy(rt_plan *p)
{
    if (!p) return;
    free_plan(p->impl);
    delete p;
}

extern "C" int rt_plan_bytes(const rt_plan *p, size_t *bytes)
{
    if (check_plan(p) || !bytes) return fail(RT_E_ARG, "NULL argument");
    *bytes = p->impl.bytes;
    return RT_OK;
}

extern "C" int rt_tables(const rt_plan *p, double *theta, double *t, int32_t *cls, int32_t *rot,
                         int32_t *flip)
{
    if (check_plan(p)) return RT_E_ARG;
    const Tables &T = p->impl.T;
    const size_t n = T.theta.size();
    if (theta) std::memcpy(theta, T.theta.data(), n * sizeof(double));
    if (t) std::memcpy(t, T.t.data(), n * sizeof(double));
    if (cls) std::memcpy(cls, T.cls.data(), n * sizeof(int32_t));
    if (rot) std::memcpy(rot, T.rot.data(), n * sizeof(int32_t));
    if (flip) std::memcpy(flip, T.flip.data(), n * sizeof(int32_t));
    return RT_OK;
}

extern "C" const char *rt_last_error(void) { return rt::g_err.c_str(); }
