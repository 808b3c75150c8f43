// Metaball-Imaging fit (sec. 2.2): the genetic algorithm's evaluation,
// mutation, crossover and selection, and the gradient search with the
// piecewise objective of Eq. GSloss and the anomaly cleaning.  C ABI in
// include/mifit.h.  Everything is FP64: the fitness decides the selection
// (an integer decision), and the gradient search runs 10^5 dependent
// steps.  Nothing here is a dense contraction (one reciprocal per hull
// point and control point), so it runs on the vector ALUs.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cstdint>
#include <mutex>

#include "../../include/mifit.h"

namespace {

constexpr int BLK = 256;         // threads of the fitness blocks (4 waves)
constexpr int GS_BLK = 1024;     // threads of a gradient-search block (16 waves)
constexpr int GS_SMALL = 192;    // hull points up to which many models take blocks of 256 (mi_gs)
constexpr int CHUNK = 2048;      // hull points per fitness block
constexpr int SEL_MAX = 4096;    // pool size the selection holds in LDS
constexpr int SEL_CHUNKS = 4;    // hull chunks whose sums the selection adds itself (each block for the whole pool)
constexpr double EPS_F = 1e-12;  // floor of f in the 1/f term of the objective

// Fixed-order sum over a block of NW waves: butterfly within each wave, then
// the wave sums in wave order.  Every thread returns the total.
template <int NW = BLK / 64>
__device__ double block_sum(double v, double *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();  // red may still be read from the previous call
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w];
    return s;
}

// f(h) = sum_j k_j / |h - p_j|^2 with the model in LDS ([n][4]: k, x, y, z).
__device__ __forceinline__ double mb_value(const double *sM, int n, double hx, double hy, double hz) {
    double f = 0.0;
    for (int j = 0; j < n; ++j) {
        const double dx = hx - sM[4 * j + 1], dy = hy - sM[4 * j + 2], dz = hz - sM[4 * j + 3];
        f += sM[4 * j] / (dx * dx + dy * dy + dz * dz);
    }
    return f;
}

// 1 / x: the hardware estimate refined by two Newton steps.
__device__ __forceinline__ double rcp_refined(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(e, r, r);
    e = fma(-x, r, 1.0);
    return fma(e, r, r);
}
__device__ __forceinline__ double dist2(const double *sM, int j, double hx, double hy, double hz) {
    const double dx = hx - sM[4 * j + 1], dy = hy - sM[4 * j + 2], dz = hz - sM[4 * j + 3];
    return fma(dx, dx, fma(dy, dy, dz * dz));
}

// The same sum with each quotient k / r^2 as k times the refined reciprocal of
// r^2 (within a few ulp of the quotient; the fitness, a sum of squares of
// f - 1, is compared and ranked, not tested for equality).
__device__ __forceinline__ double mb_value_rcp(const double *sM, int n, double hx, double hy, double hz) {
    double f = 0.0;
    for (int j = 0; j < n; ++j) f = fma(sM[4 * j], rcp_refined(dist2(sM, j, hx, hy, hz)), f);
    return f;
}

// The same sum at NP points at once, four control points over one common
// denominator: a reciprocal (four issue slots, and four of refinement) for
// four quotients, and a control point read from LDS once for NP points.  The
// products stay far inside the range of FP64 while coordinates are below
// TAME_X and weights below TAME_K (r^2 <= 1.2e33, four of them <= 2.1e132); tame
// says whether the model is (wave-uniform).  A point that is not, or that lies so
// near a control point that the denominator falls below 1e-200, is summed
// term by term.
constexpr double TAME_X = 1e16, TAME_K = 1e60;
template <int NP>
__device__ __forceinline__ void mb_values(const double *sM, int n, bool tame, const double hx[NP], const double hy[NP],
                                          const double hz[NP], double f[NP]) {
    bool bad[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        f[q] = 0.0;
        bad[q] = !(tame && fabs(hx[q]) < TAME_X && fabs(hy[q]) < TAME_X && fabs(hz[q]) < TAME_X);
    }
    int j = 0;
    for (; j + 4 <= n; j += 4) {
        const double k0 = sM[4 * j], k1 = sM[4 * j + 4], k2 = sM[4 * j + 8], k3 = sM[4 * j + 12];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const double a = dist2(sM, j, hx[q], hy[q], hz[q]), b = dist2(sM, j + 1, hx[q], hy[q], hz[q]);
            const double c = dist2(sM, j + 2, hx[q], hy[q], hz[q]), d = dist2(sM, j + 3, hx[q], hy[q], hz[q]);
            const double ab = a * b, cd = c * d, den = ab * cd;
            const double nab = fma(k0, b, k1 * a), ncd = fma(k2, d, k3 * c);
            bad[q] |= !(den > 1e-200);
            f[q] = fma(fma(nab, cd, ncd * ab), rcp_refined(den), f[q]);
        }
    }
    for (; j < n; ++j)
#pragma unroll
        for (int q = 0; q < NP; ++q) f[q] = fma(sM[4 * j], rcp_refined(dist2(sM, j, hx[q], hy[q], hz[q])), f[q]);
#pragma unroll
    for (int q = 0; q < NP; ++q)
        if (bad[q]) f[q] = mb_value_rcp(sM, n, hx[q], hy[q], hz[q]);
}
// Whether value t of the model's 4 n stays in that range.
__device__ __forceinline__ bool tame_value(int t, double v) { return fabs(v) < ((t & 3) == 0 ? TAME_K : TAME_X); }

// The per-point term of Eq. GSloss and its slope.
__device__ __forceinline__ double gs_term(double f) {
    if (f >= 2.0) return (f - 1.0) * (f - 1.0);
    if (f >= 1.0) return f - 1.0;
    const double fc = f > EPS_F ? f : EPS_F;
    return (f - 1.0) * (f - 1.0) + 1.0 / fc - 1.0;
}
__device__ __forceinline__ double gs_slope(double f) {
    if (f >= 2.0) return 2.0 * (f - 1.0);
    if (f >= 1.0) return 1.0;
    return 2.0 * (f - 1.0) - (f > EPS_F ? 1.0 / (f * f) : 0.0);
}

// ------------------------------------------------------------- evaluation
// Adds (f - 1)^2 at the NP hull points i, i + BLK, ... of a lane to s.
template <int NP>
__device__ __forceinline__ void fitness_points(const double *__restrict__ hull, long long i, long long i1,
                                               const double *sM, int n, bool tame, double &s) {
    double hx[NP], hy[NP], hz[NP], f[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {  // past the end: the chunk's last point, unused
        const long long k = i + q * BLK < i1 ? i + q * BLK : i1 - 1;
        hx[q] = hull[3 * k];
        hy[q] = hull[3 * k + 1];
        hz[q] = hull[3 * k + 2];
    }
    mb_values<NP>(sM, n, tame, hx, hy, hz, f);
#pragma unroll
    for (int q = 0; q < NP; ++q)
        if (i + q * BLK < i1) {
            const double e = f[q] - 1.0;
            s += e * e;
        }
}

// Sum over the hull points of chunk c of (f - 1)^2 for the model in LDS: up to
// FP points per lane at a time, FP = 0: one, with a reciprocal per quotient.
// Whole block; every thread returns the sum.
// Bound by vector issue: 11.4 instructions per (hull point, control point) with
// the shared reciprocals, 15 with one each (2400 models of 25 points on 4096:
// 117 -> 90 us a call; two points a lane take the same time).  A wave goes
// through the rounds of 256 points that reach it and no others, four, two or
// one at a time: padded to four, hulls that are no multiple of 1024 points took
// longer than with a reciprocal each (2400 models of 25 points on 600: 23.9 us, padded 27.6, now 20.1).
template <int FP>
__device__ __forceinline__ double fitness_chunk(const double *__restrict__ hull, long long m, const double *sM, int n,
                                                int c, double *red) {
    const long long i0 = (long long)c * CHUNK;
    const long long i1 = i0 + CHUNK < m ? i0 + CHUNK : m;
    double s = 0.0;
    long long i = i0 + threadIdx.x;
    if (FP == 0) {
        for (; i < i1; i += BLK) {
            const double e = mb_value_rcp(sM, n, hull[3 * i], hull[3 * i + 1], hull[3 * i + 2]) - 1.0;
            s += e * e;
        }
        return block_sum(s, red);
    }
    // whether the model is tame: each wave looks at all of it
    bool ok = true;
    for (int t = threadIdx.x & 63; t < 4 * n; t += 64) ok = ok && tame_value(t, sM[t]);
    const bool tame = __all(ok);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63);
    int rounds = (int)((i1 - i0 - wave + BLK - 1) / BLK);  // wave-uniform; i1 - i0 >= 1: not below 0
    if (FP >= 4)
        for (; rounds >= 4; rounds -= 4, i += 4 * BLK) fitness_points<4>(hull, i, i1, sM, n, tame, s);
    if (FP >= 2)
        for (; rounds >= 2; rounds -= 2, i += 2 * BLK) fitness_points<2>(hull, i, i1, sM, n, tame, s);
    for (; rounds >= 1; --rounds, i += BLK) fitness_points<1>(hull, i, i1, sM, n, tame, s);
    return block_sum(s, red);
}

// Block (individual p, chunk c): its chunk sum to out[p * nch + c].
template <int FP>
__global__ __launch_bounds__(BLK) void k_fitness(const double *__restrict__ hull, long long m,
                                                 const double *__restrict__ pop, int n, int nch,
                                                 double *__restrict__ out) {
    __shared__ double sM[MI_MAXCP * 4];
    __shared__ double red[4];
    const int p = blockIdx.x / nch, c = blockIdx.x - p * nch;
    const double *M = pop + (size_t)p * n * 4;
    for (int t = threadIdx.x; t < 4 * n; t += BLK) sM[t] = M[t];
    __syncthreads();
    const double s = fitness_chunk<FP>(hull, m, sM, n, c, red);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// F[p] = the chunk sums of individual p added in chunk order.
__global__ void k_fitness_sum(const double *__restrict__ part, int P, int nch, double *__restrict__ F) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    double s = 0.0;
    for (int c = 0; c < nch; ++c) s += part[(size_t)p * nch + c];
    F[p] = s;
}

// ------------------------------------------------------ genetic operators
// One generation's offspring and their evaluation in one launch.  Block
// (offspring a of 2 N, chunk c of the hull): mutant a (a < N) of individual a,
// gene-wise, each gene exactly v + z * sigma (no contraction); or child a - N:
// the pairs (perm[2j], perm[2j+1]) exchange their control points from cut on,
// an odd last individual is copied.  The genes go to LDS and, from the first
// chunk's block, to the pool behind the N parents; then the chunk's fitness.
// (Mutation, crossover and the chunk sums were launches of 5 us each beside the
// evaluation; a generation of 1200 went from 220 to 118 us.)
template <int FP>
__global__ __launch_bounds__(BLK) void k_breed(const double *__restrict__ hull, long long m, double *__restrict__ pool,
                                               const double *__restrict__ U, const double *__restrict__ Z,
                                               const int *__restrict__ perm, int N, int n, int cut, double C_m,
                                               double sx, double sk, int nch, double *__restrict__ out) {
#pragma clang fp contract(off)
    __shared__ double sM[MI_MAXCP * 4];
    __shared__ double red[4];
    const int a = blockIdx.x / nch, c = blockIdx.x - a * nch, g4 = 4 * n, t = threadIdx.x;
    if (t < g4) {  // g4 <= BLK
        double v;
        if (a < N) {
            const size_t i = (size_t)a * g4 + t;
            const int g = t & 3;
            v = pool[i];
            if (U[i] < C_m) v = v + Z[i] * (g == 0 ? sk : sx);
            if (g == 0 && v < 0.0) v = 0.0;
        } else {
            const int b = a - N;
            int src;
            if ((N & 1) && b == N - 1) {
                src = perm[b];
            } else {
                const int first = perm[b & ~1], second = perm[b | 1];
                const bool head = (t >> 2) < cut;
                src = (b & 1) ? (head ? second : first) : (head ? first : second);
            }
            if ((unsigned)src >= (unsigned)N) src = b;  // not a permutation entry: keep the index in range
            v = pool[(size_t)src * g4 + t];
        }
        sM[t] = v;
        if (c == 0) pool[(size_t)(N + a) * g4 + t] = v;
    }
    __syncthreads();
    const double s = fitness_chunk<FP>(hull, m, sM, n, c, red);
    if (t == 0) out[blockIdx.x] = s;
}

// Survivors: the N fittest of the pool's K individuals, ties to the lower
// index (NaN counts as +inf), in order.  Every block holds the whole pool's
// fitness in LDS -- F [F_known] of the parents, then the offspring's chunk
// sums added in chunk order -- and ranks SEL_PER of them: SEL_LANES lanes count
// the individuals before one, the count is its place, and the lanes copy it
// there if it survives.  The comparisons of all pairs over many blocks take
// less time than the dependent passes of a sort in one block (3600 of them:
// 13.9 us with the copy, against 77 for a bitonic sort and 5 for a gather).
constexpr int SEL_LANES = 32, SEL_PER = BLK / SEL_LANES;
__global__ __launch_bounds__(BLK) void k_select(const double *__restrict__ pool, const double *__restrict__ F,
                                                int F_known, const double *__restrict__ part, int nch, int K, int N,
                                                int n, double *__restrict__ pop, double *__restrict__ Fout) {
    __shared__ double key[SEL_MAX];
    auto fitness = [&](int i) {
        if (i < F_known) return F[i];
        double v = 0.0;
        for (int c = 0; c < nch; ++c) v += part[(size_t)(i - F_known) * nch + c];
        return v;
    };
#pragma unroll 4
    for (int i = threadIdx.x; i < K; i += BLK) {
        const double v = fitness(i);
        key[i] = v != v ? HUGE_VAL : v;
    }
    __syncthreads();
    const int l = threadIdx.x % SEL_LANES, i = blockIdx.x * SEL_PER + threadIdx.x / SEL_LANES;
    const double mine = i < K ? key[i] : 0.0;
    int before = 0;
#pragma unroll 8
    for (int j = l; j < K; j += SEL_LANES) {
        const double v = key[j];
        before += (v < mine) | ((v == mine) & (j < i));
    }
#pragma unroll
    for (int d = SEL_LANES / 2; d > 0; d >>= 1) before += __shfl_xor(before, d, SEL_LANES);
    if (i >= K || before >= N) return;
    const int g4 = 4 * n;
    for (int r = l; r < g4; r += SEL_LANES) pop[(size_t)before * g4 + r] = pool[(size_t)i * g4 + r];
    if (l == 0) Fout[before] = fitness(i);
}

// --------------------------------------------------------- gradient search
// n . p + d of a half-space (no contraction: the same sum as a plain dot product).
__device__ __forceinline__ double plane_side(const double *pl, double px, double py, double pz) {
#pragma clang fp contract(off)
    return ((px * pl[0] + py * pl[1]) + pz * pl[2]) + pl[3];
}

// f at one point for the descent, four control points over one common
// denominator (mb_values; here every denominator and the sum are held to a
// range far inside FP64, since the model moves); outside it the plain sum.
__device__ __forceinline__ double gs_value(const double *sM, int n, double hx, double hy, double hz) {
    double f = 0.0;
    bool ok = true;
    int j = 0;
    for (; j + 4 <= n; j += 4) {
        const double a = dist2(sM, j, hx, hy, hz), b = dist2(sM, j + 1, hx, hy, hz);
        const double c = dist2(sM, j + 2, hx, hy, hz), d = dist2(sM, j + 3, hx, hy, hz);
        const double ab = a * b, cd = c * d, den = ab * cd;
        const double nab = fma(sM[4 * j], b, sM[4 * j + 4] * a), ncd = fma(sM[4 * j + 8], d, sM[4 * j + 12] * c);
        ok = ok && den > 1e-200 && den < 1e200;
        f = fma(fma(nab, cd, ncd * ab), rcp_refined(den), f);
    }
    for (; j < n; ++j) f += sM[4 * j] / dist2(sM, j, hx, hy, hz);
    return ok && fabs(f) < 1e200 ? f : mb_value(sM, n, hx, hy, hz);
}

// Chunks of points in pass 2: as many as 1024 threads take, of four points or
// more (two pairs over a reciprocal each).
__host__ __device__ __forceinline__ int gs_chunks(int m, int n) {
    const int most = GS_BLK / n, fours = (m + 3) / 4;
    return most < fours ? most : fours;
}

// Sum over the hull points of the Eq. GSloss terms for the model in LDS.
template <int NT>
__device__ double gs_loss_block(const double *__restrict__ hull, long long m, const double *sM, int n, double *red) {
    double s = 0.0;
    for (long long i = threadIdx.x; i < m; i += NT)
        s += gs_term(mb_value(sM, n, hull[3 * i], hull[3 * i + 1], hull[3 * i + 2]));
    return block_sum<NT / 64>(s, red);
}

// One workgroup per model: E descent steps, cleaning, E steps.  Per step:
// pass 1, one hull point per lane: f and the objective's slope g_i (in
// LDS); pass 2, lanes over (control point j, chunk of points):
// dL/dk_j = sum g_i / r^2, dL/dp_j = sum g_i 2 k_j (h_i - p_j) / r^4 over the
// chunk, two points over one reciprocal; the chunks are added in a fixed
// order (eight lanes a gene, four beyond 32 control points) and the model
// updated in LDS.  A step is one compute unit's vector issue on the 2 m n
// terms, so the block has 16 waves, four per SIMD (four waves in all left
// each SIMD waiting on one), and with STAGED the hull is kept in LDS beside its
// slopes (32 bytes a point) instead of being read again from the caches every
// step.  64 models of 900 to 1500 points, 25 control points: 13.5 us a step, 40
// with four waves, exact quotients and the hull in memory.
// Two more forms for more models than compute units, with the same chunks and
// sums, bit for bit (mi_gs chooses): WPE = 8 holds the block to 64 registers a
// lane, so that two share a compute unit; NT = 256 (hulls of up to 192 points,
// which leave most of 1024 threads idle) lets several, a thread standing for
// four of the 1024 in pass 2.
template <bool STAGED, int NT, int WPE>
__global__ __launch_bounds__(NT, WPE) void k_gs(const double *__restrict__ hulls, const int64_t *__restrict__ hoff,
                                                const double *__restrict__ planes, const int64_t *__restrict__ poff,
                                                int n, int E, double eta, double *__restrict__ Mall,
                                                double *__restrict__ loss) {
    __shared__ double sM[MI_MAXCP * 4];
    __shared__ double red[NT / 64];
    extern __shared__ double pts[];  // STAGED: x, y, z and the slope of each point; else the slopes alone
    const int b = blockIdx.x, t = threadIdx.x;
    const long long h0 = hoff[b];
    const int m = (int)(hoff[b + 1] - h0);  // at most MI_GS_MAXPTS; with NT = 256, at most 256
    const double *hull = hulls + 3 * h0;
    double *M = Mall + (size_t)b * n * 4;
    if (t < 4 * n) sM[t] = M[t];  // 4 n <= 256
    if (STAGED)
        for (int i = t; i < m; i += NT)
            for (int a = 0; a < 3; ++a) pts[4 * i + a] = hull[3 * i + a];
    __syncthreads();
    double L = gs_loss_block<NT>(hull, m, sM, n, red);
    if (t == 0) loss[3 * b] = L;
    const int nch = gs_chunks(m, n);
    const int lp = n <= 32 ? 3 : 2;  // 2^lp lanes per gene in the last sum
    const int j0 = t % n, c0 = t / n, dj = NT % n, dc = NT / n;  // control point and chunk, and their steps
    constexpr int W = STAGED ? 4 : 1;
    constexpr bool FIXED = NT == GS_BLK;  // a place of its own for the sums; else behind the points
    __shared__ double fixed[FIXED ? GS_BLK * 4 : 1];
    double *part = FIXED ? fixed : pts + W * m;
    auto point = [&](int i, double &x, double &y, double &z) {
        const double *h = STAGED ? pts + 4 * i : hull + 3 * (size_t)i;
        x = h[0];
        y = h[1];
        z = h[2];
    };
    for (int phase = 0; phase < 2; ++phase) {
        for (int it = 0; it < E; ++it) {
            for (int i = t; i < m; i += NT) {
                double x, y, z;
                point(i, x, y, z);
                pts[W * i + W - 1] = gs_slope(gs_value(sM, n, x, y, z));
            }
            __syncthreads();
            for (int v = t, j = j0, c = c0; v < nch * n; v += NT) {  // control point j, chunk c; v = c n + j
                const double k2 = 2.0 * sM[4 * j], px = sM[4 * j + 1], py = sM[4 * j + 2], pz = sM[4 * j + 3];
                double gk = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
                auto add = [&](double dx, double dy, double dz, double y, double gi) {
                    const double gy_ = gi * y, w = k2 * gy_ * y;
                    gk += gy_;
                    gx = fma(w, dx, gx);
                    gy = fma(w, dy, gy);
                    gz = fma(w, dz, gz);
                };
                int i = c;
                for (; i + nch < m; i += 2 * nch) {
                    double ax, ay, az, bx, by, bz;
                    point(i, ax, ay, az);
                    point(i + nch, bx, by, bz);
                    ax -= px; ay -= py; az -= pz;
                    bx -= px; by -= py; bz -= pz;
                    const double ra = fma(ax, ax, fma(ay, ay, az * az)), rb = fma(bx, bx, fma(by, by, bz * bz));
                    const double den = ra * rb, inv = rcp_refined(den);
                    double ya = rb * inv, yb = ra * inv;
                    if (!(den > 1e-200 && den < 1e200)) {
                        ya = 1.0 / ra;
                        yb = 1.0 / rb;
                    }
                    add(ax, ay, az, ya, pts[W * i + W - 1]);
                    add(bx, by, bz, yb, pts[W * (i + nch) + W - 1]);
                }
                if (i < m) {
                    double ax, ay, az;
                    point(i, ax, ay, az);
                    ax -= px; ay -= py; az -= pz;
                    add(ax, ay, az, 1.0 / fma(ax, ax, fma(ay, ay, az * az)), pts[W * i + W - 1]);
                }
                part[4 * v] = gk; part[4 * v + 1] = gx;
                part[4 * v + 2] = gy; part[4 * v + 3] = gz;
                if (FIXED) break;  // one round
                j += dj;
                c += dc;
                if (j >= n) {
                    j -= n;
                    ++c;
                }
            }
            __syncthreads();
            for (int v = t; v < 4 * n << lp; v += NT) {  // gene o: 2^lp partial sums, then a butterfly
                const int o = v >> lp, l = v - (o << lp);
                double G = 0.0;
                for (int cc = l; cc < nch; cc += 1 << lp) G += part[4 * cc * n + o];
                for (int d = 1 << (lp - 1); d > 0; d >>= 1) G += __shfl_xor(G, d);
                if (l == 0) sM[o] -= eta * G;
                if (FIXED) break;
            }
            __syncthreads();
        }
        if (phase == 0) {
            L = gs_loss_block<NT>(hull, m, sM, n, red);
            if (t == 0) loss[3 * b + 1] = L;
            // anomaly cleaning: negative weights and control points outside the hull
            if (t < n) {
                const int jj = t;
                bool out = sM[4 * jj] < 0.0;
                const double px = sM[4 * jj + 1], py = sM[4 * jj + 2], pz = sM[4 * jj + 3];
                for (long long q = poff[b]; q < poff[b + 1] && !out; ++q) out = plane_side(planes + 4 * q, px, py, pz) > 0.0;
                if (out) sM[4 * jj] = 0.0;
            }
            __syncthreads();
        }
    }
    L = gs_loss_block<NT>(hull, m, sM, n, red);
    if (t == 0) loss[3 * b + 2] = L;
    if (t < 4 * n) M[t] = sM[t];
}

// Hulls of up to GS_STAGED points are kept in LDS (96 KB beside the 34 KB of
// the model and the sums, of the 160 KB of a compute unit); a larger one leaves its points in
// memory.
constexpr int GS_STAGED = 3072;
constexpr int GS_PAIR = 1400;  // two blocks share the 160 KB

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
inline int chunks(long long m) { return cdiv(m, CHUNK); }

lbm_status launched() { return hipGetLastError() == hipSuccess ? LBM_OK : LBM_E_HIP; }

// The fitness's form.  A reciprocal per quotient while the model has too few
// control points, or the hull too few points beside them, for shared ones to
// make up for their checks (the start of a block, and what is added per
// point).  Time with a reciprocal each over time with shared ones, by control
// points and hull points:
//             40    250    500   1024   2048   4096
//    2      0.85   0.88   0.88   0.90   0.91   0.92
//    4      0.89   0.95   0.97   0.97   1.02   1.02
//    6      0.87   0.95   0.97   1.01   1.05   1.06
//    8      0.89   0.99   1.05   1.08   1.11   1.13
//   12      0.92   1.03   1.13   1.13   1.18   1.18
//   25      0.91   1.12   1.17   1.21   1.25   1.25
// Shared, the points per lane at a time are as many as the hull gives a lane of
// one block, up to four (more registers, fewer waves).
template <class L0, class L1, class L2, class L4>
void by_form(long long m, int n, L0 each, L1 one, L2 two, L4 four) {
    if (n < 8 ? n < 4 || m < 2048 : n * m < 3500) each();
    else if (m <= BLK) one();
    else if (m <= 2 * BLK) two();
    else four();
}

// Fitness of P individuals into F (partials in part when m spans chunks).
lbm_status fitness_launch(const double *hull, long long m, const double *pop, int P, int n, double *F, double *part,
                          hipStream_t s) {
    const int nch = chunks(m);
    double *out = nch == 1 ? F : part;
    by_form(
        m, n, [&] { k_fitness<0><<<P * nch, BLK, 0, s>>>(hull, m, pop, n, nch, out); },
        [&] { k_fitness<1><<<P * nch, BLK, 0, s>>>(hull, m, pop, n, nch, out); },
        [&] { k_fitness<2><<<P * nch, BLK, 0, s>>>(hull, m, pop, n, nch, out); },
        [&] { k_fitness<4><<<P * nch, BLK, 0, s>>>(hull, m, pop, n, nch, out); });
    if (nch > 1) k_fitness_sum<<<cdiv(P, 256), 256, 0, s>>>(part, P, nch, F);
    return launched();
}

struct GaLayout {
    size_t poolA, poolB, FA, FB, part, total;
};
GaLayout ga_layout(long long m, int N, int n) {
    GaLayout L;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t r = o; o = align256(o + bytes); return r; };
    const size_t pool = (size_t)3 * N * n * 4 * sizeof(double);
    L.poolA = take(pool);
    L.poolB = take(pool);
    L.FA = take((size_t)3 * N * sizeof(double));
    L.FB = take((size_t)3 * N * sizeof(double));
    take((size_t)N * sizeof(int));  // unused: the workspace keeps its size
    L.part = take(chunks(m) > 1 ? (size_t)2 * N * chunks(m) * sizeof(double) : 0);
    L.total = o;
    return L;
}

}  // namespace

extern "C" {

size_t mi_fitness_work_bytes(int64_t m, int32_t P) {
    if (m < 1 || P < 1) return 0;
    return chunks(m) > 1 ? (size_t)P * chunks(m) * sizeof(double) : 0;
}

lbm_status mi_fitness(const double *hull, int64_t m, const double *pop, int32_t P, int32_t n, double *F, void *work,
                      size_t work_bytes, void *hip_stream) {
    if (!hull || !pop || !F || m < 1 || P < 1 || n < 1 || n > MI_MAXCP) return LBM_E_INVALID;
    if ((long long)P * chunks(m) > 0x7fffffffll) return LBM_E_INVALID;
    const size_t need = mi_fitness_work_bytes(m, P);
    if (need && (!work || work_bytes < need)) return LBM_E_NOMEM;
    return fitness_launch(hull, m, pop, P, n, F, (double *)work, (hipStream_t)hip_stream);
}

size_t mi_ga_work_bytes(int64_t m, int32_t N_I, int32_t n) {
    if (m < 1 || N_I < 2 || n < 1 || n > MI_MAXCP) return 0;
    return ga_layout(m, N_I, n).total;
}

lbm_status mi_ga(const double *hull, int64_t m, int32_t N_I, int32_t n, int32_t E, double C_m, double C_c,
                 double sigma_x, double sigma_k, const double *U, const double *Z, const int32_t *PERM, double *pop,
                 double *F, void *work, size_t work_bytes, void *hip_stream) {
    if (!hull || !pop || !F || !work || m < 1 || n < 1 || n > MI_MAXCP || N_I < 2 || 3 * N_I > SEL_MAX || E < 0)
        return LBM_E_INVALID;
    if (E > 0 && (!U || !Z || !PERM)) return LBM_E_INVALID;
    if (!(C_c >= 0.0 && C_c <= 1.0) || !(sigma_x >= 0.0) || !(sigma_k >= 0.0)) return LBM_E_INVALID;
    const GaLayout Lw = ga_layout(m, N_I, n);
    if (work_bytes < Lw.total) return LBM_E_NOMEM;
    hipStream_t s = (hipStream_t)hip_stream;
    char *w = (char *)work;
    double *A = (double *)(w + Lw.poolA), *B = (double *)(w + Lw.poolB);
    double *FA = (double *)(w + Lw.FA), *FB = (double *)(w + Lw.FB);
    double *part = (double *)(w + Lw.part);
    const long long genes = (long long)N_I * n * 4;
    const int c = (int)(C_c * n + 0.5);
    if (hipMemcpyAsync(A, pop, genes * sizeof(double), hipMemcpyDeviceToDevice, s) != hipSuccess) return LBM_E_HIP;
    lbm_status st = fitness_launch(hull, m, A, N_I, n, FA, part, s);
    if (st) return st;
    const int nch = chunks(m);
    double *sums = nch == 1 ? FA + N_I : part;  // the offspring's fitness, whole or in chunk sums
    for (int e = 0; e < E; ++e) {
        const double *Ue = U + (size_t)e * genes, *Ze = Z + (size_t)e * genes;
        const int *pe = PERM + (size_t)e * N_I;
        auto breed = [&](auto kernel) {
            kernel<<<2 * N_I * nch, BLK, 0, s>>>(hull, m, A, Ue, Ze, pe, N_I, n, c, C_m, sigma_x, sigma_k, nch, sums);
        };
        by_form(m, n, [&] { breed(k_breed<0>); }, [&] { breed(k_breed<1>); }, [&] { breed(k_breed<2>); }, [&] { breed(k_breed<4>); });
        const bool fold = nch <= SEL_CHUNKS;
        if (!fold) k_fitness_sum<<<cdiv(2 * N_I, 256), 256, 0, s>>>(part, 2 * N_I, nch, FA + N_I);
        k_select<<<cdiv(3 * N_I, SEL_PER), BLK, 0, s>>>(A, FA, fold ? N_I : 3 * N_I, sums, nch, 3 * N_I, N_I, n, B, FB);
        if ((st = launched())) return st;
        double *t = A; A = B; B = t;
        t = FA; FA = FB; FB = t;
        if (nch == 1) sums = FA + N_I;
    }
    if (hipMemcpyAsync(pop, A, genes * sizeof(double), hipMemcpyDeviceToDevice, s) != hipSuccess ||
        hipMemcpyAsync(F, FA, N_I * sizeof(double), hipMemcpyDeviceToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return LBM_E_HIP;
    return launched();
}

lbm_status mi_gs(const double *hulls, const int64_t *hull_off, const double *planes, const int64_t *plane_off,
                 int32_t B, int32_t n, int32_t E, double eta, double *M, double *loss, void *hip_stream) {
    if (!hulls || !hull_off || !planes || !plane_off || !M || !loss || B < 1 || n < 1 || n > MI_MAXCP || E < 0 ||
        !(eta >= 0.0))
        return LBM_E_INVALID;
    // the offsets live on the device: read them to check every hull's size
    hipStream_t s = (hipStream_t)hip_stream;
    int64_t *ho = new int64_t[2 * (size_t)(B + 1)];
    if (hipMemcpyAsync(ho, hull_off, 8 * (size_t)(B + 1), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(ho + B + 1, plane_off, 8 * (size_t)(B + 1), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
        delete[] ho;
        return LBM_E_HIP;
    }
    bool ok = ho[0] >= 0 && ho[B + 1] >= 0;
    int64_t most = 0;
    for (int b = 0; b < B && ok; ++b) {
        most = ho[b + 1] - ho[b] > most ? ho[b + 1] - ho[b] : most;
        ok = ho[b + 1] - ho[b] >= 1 && ho[b + 1] - ho[b] <= MI_GS_MAXPTS && ho[B + 2 + b] >= ho[B + 1 + b];
    }
    delete[] ho;
    if (!ok) return LBM_E_INVALID;
    const bool staged = most <= GS_STAGED;
    // Beyond 64 KB of LDS a kernel asks for it, and the request belongs to the
    // kernel, not to the launch: it is each form's largest (130 and 82 KB with
    // the static 34) in every call, so that calls on several threads agree.
    const size_t points = (staged ? 32 : 8) * (size_t)most;
    auto run = [&](auto kernel, int threads, int max_lds, size_t lds) {
        if (hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds) != hipSuccess)
            return LBM_E_HIP;
        kernel<<<B, threads, lds, s>>>(hulls, hull_off, planes, plane_off, n, E, eta, M, loss);
        return launched();
    };
    constexpr int MAX_STAGED = 32 * GS_STAGED, MAX_SMALL = 32 * GS_SMALL + 32 * GS_BLK, MAX_SLOPES = 8 * MI_GS_MAXPTS;
    // Up to one model a compute unit: the form without a register limit.  More:
    // two blocks a unit where their LDS allows it; beyond two a unit and with
    // small hulls, blocks of 256.  Us a call of 20 steps with the form taken and
    // with the first one:
    //   models   25 control points on 100   300   500       10 on 100
    //     300        143 / 176        199 / 235   250 / 282   103 / 135
    //     512        148 / 180        210 / 242   263 / 288   105 / 136
    //    1024        214 / 306                                130 / 223
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return LBM_E_HIP;
    if (!staged) return run(k_gs<false, GS_BLK, 1>, GS_BLK, MAX_SLOPES, points);
    if (B > 2 * cu && most <= GS_SMALL)
        return run(k_gs<true, 256, 1>, 256, MAX_SMALL, points + 32 * (size_t)n * gs_chunks((int)most, n));
    if (B > cu && most <= GS_PAIR) return run(k_gs<true, GS_BLK, 8>, GS_BLK, MAX_STAGED, points);
    return run(k_gs<true, GS_BLK, 1>, GS_BLK, MAX_STAGED, points);
}

// ---------------------------------------------- fitness without allocation
// For callers that cannot allocate (graph capture, tight loops): the chunk
// sums live in this file-scope array, one copy per GPU, held until the
// process ends.  Host code reaches it only through the address
// hipGetSymbolAddress returns for the current device.
constexpr size_t MI_SCRATCH_DOUBLES = size_t(1) << 17;  // 1 MiB: individuals x chunks <= 131072
__device__ __align__(256) double scratch[MI_SCRATCH_DOUBLES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double *g_scratch[MAX_DEVICES];
}  // namespace

lbm_status mi_fitness_noalloc(const double *hull, int64_t m, const double *pop, int32_t P, int32_t n, double *F,
                              void *hip_stream) {
    if (!hull || !pop || !F || m < 1 || P < 1 || n < 1 || n > MI_MAXCP) return LBM_E_INVALID;
    if ((long long)P * chunks(m) > (long long)MI_SCRATCH_DOUBLES) return LBM_E_INVALID;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return LBM_E_HIP;
    double *ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch[dev]) {
            void *a = nullptr;
            if (hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)) != hipSuccess || !a) return LBM_E_HIP;
            g_scratch[dev] = (double *)a;
        }
        ptr = g_scratch[dev];
    }
    return fitness_launch(hull, m, pop, P, n, F, ptr, (hipStream_t)hip_stream);
}

}  // extern "C"
