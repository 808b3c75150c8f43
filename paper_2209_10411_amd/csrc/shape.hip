// Shape descriptors of a metaball body (sec. 4): volume, surface area,
// principal dimensions and projected area on a grid, then sphericity,
// nominal and surface-equivalent diameters and the Corey shape factor.  C ABI
// in include/shape.h.  Grid points are formed without contraction (the same
// sums as written), the metaball in control-point order with exact
// quotients, so that the inside decisions are those of a plain evaluation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "../../include/shape.h"

namespace {

constexpr int BLK = 256;
constexpr int MAXN = 64;

struct Body {
    double p[MAXN][3];
    double k[MAXN];
    int n;
};

// C(x) - 1 with exact quotients in control-point order (+inf on a control point).
__device__ double cm1(const Body &b, double x, double y, double z) {
#pragma clang fp contract(off)
    double c = 0.0;
    for (int j = 0; j < b.n; ++j) {
        const double dx = x - b.p[j][0], dy = y - b.p[j][1], dz = z - b.p[j][2];
        c += b.k[j] / ((dx * dx + dy * dy) + dz * dz);
    }
    return c - 1.0;
}

__device__ double block_sum(double v, double *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((red[0] + red[1]) + red[2]) + red[3];
}
__device__ double block_min(double v, double *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
}

// Area of the zero surface of the linear interpolant in one tetrahedron.
__device__ double tet_area(const double P[4][3], const double g[4]) {
#pragma clang fp contract(off)
    int pos[4], neg[4], np = 0, nn = 0;
    for (int a = 0; a < 4; ++a) {
        if (g[a] >= 0.0) pos[np++] = a;
        else neg[nn++] = a;
    }
    if (np == 0 || nn == 0) return 0.0;
    auto cut = [&](int a, int b, double q[3]) {
        const double t = g[a] / (g[a] - g[b]);
        for (int c = 0; c < 3; ++c) q[c] = P[a][c] + t * (P[b][c] - P[a][c]);
    };
    auto tri = [](const double a[3], const double b[3], const double c[3]) {
        const double u[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
        const double v[3] = {c[0] - a[0], c[1] - a[1], c[2] - a[2]};
        const double x = u[1] * v[2] - u[2] * v[1], y = u[2] * v[0] - u[0] * v[2], z = u[0] * v[1] - u[1] * v[0];
        return 0.5 * sqrt((x * x + y * y) + z * z);
    };
    double q[4][3];
    if (np == 1 || np == 3) {
        const int lone = np == 1 ? pos[0] : neg[0];
        int o = 0;
        for (int a = 0; a < 4; ++a)
            if (a != lone) cut(lone, a, q[o++]);
        return tri(q[0], q[1], q[2]);
    }
    cut(pos[0], neg[0], q[0]);
    cut(pos[0], neg[1], q[1]);
    cut(pos[1], neg[1], q[2]);
    cut(pos[1], neg[0], q[3]);
    return tri(q[0], q[1], q[2]) + tri(q[0], q[2], q[3]);
}

struct Grid {
    double lo[3], h;
    int n[3];
};
struct Axes {
    double a[9];  // three rows
};

__device__ __forceinline__ void centre(const Grid &G, long long t, double c[3], int idx[3]) {
#pragma clang fp contract(off)
    idx[0] = (int)(t % G.n[0]);
    const long long r = t / G.n[0];
    idx[1] = (int)(r % G.n[1]);
    idx[2] = (int)(r / G.n[1]);
    for (int a = 0; a < 3; ++a) c[a] = G.lo[a] + G.h * ((double)idx[a] + 0.5);
}

// Inside decision at a point: coordinates about the anchor (the mean control
// point) scaled so that sqrt(sum k) is 16, in FP32; terms k * rcp(|d|^2) on the
// hardware reciprocal (1 ulp).  With every |d|^2 >= 1 each component of d is off
// by at most u (|r_a| + |p_a| + |d_a|) (u = 2^-24), so |d|^2 by at most
// u (2.03 (|r|_1 + |p|_1) + 6.5) relative, a term by that plus 3 u, and the
// n-term sum by n u more; with a factor 1.5 (the scaling's own roundings are
// below it) and 1e-12 for the exact sum's.  Within the bound of 1, within
// 1 of a control point, or where the bound exceeds 1/4 (a body 1e5 times as long
// as its radius: the errors' squares, left out of it, then count), the exact
// quotients decide (cm1).
struct Body32 {
    float4 f[MAXN];  // scaled position about the anchor, scaled weight
    double anc[3], scale;
    float bp;  // max |p - anchor|_1
};

__device__ __forceinline__ bool inside(const Body &b, const Body32 &q, double x, double y, double z) {
    const float rx = (float)((x - q.anc[0]) * q.scale), ry = (float)((y - q.anc[1]) * q.scale),
                rz = (float)((z - q.anc[2]) * q.scale);
    float C = 0.f, rmin = 1.f;
    for (int j = 0; j < b.n; ++j) {
        const float4 c = q.f[j];
        const float dx = rx - c.x, dy = ry - c.y, dz = rz - c.z;
        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        rmin = fminf(rmin, d2);
        C = fmaf(c.w, __builtin_amdgcn_rcpf(d2), C);
    }
    if (rmin >= 1.f) {
        const float ax = fabsf(rx) + fabsf(ry) + fabsf(rz);
        const double rel = 1.5 * 5.9604644775390625e-8 * (2.03 * ((double)ax + (double)q.bp) + 9.5 + b.n);
        if (rel < 0.25 && (double)C * (1.0 - rel) > 1.0 + 1e-12) return true;
        if (rel < 0.25 && (double)C * (1.0 + rel) < 1.0 - 1e-12) return false;
    }
    return cm1(b, x, y, z) >= 0.0;
}

// ---------------------------------------------------------- general form
// Every cell by itself (passes 1 to 3); mb_shape_descriptors says when.  All
// but the area needs the inside decisions alone (inside).
// Pass 1: inside count, first moments of the inside centres, surface area.
__global__ __launch_bounds__(BLK) void k_shape_grid(Body b, Grid G, long long cells, double *__restrict__ part) {
#pragma clang fp contract(off)
    __shared__ double red[4];
    const long long t = blockIdx.x * (long long)BLK + threadIdx.x;
    double cnt = 0.0, sx = 0.0, sy = 0.0, sz = 0.0, area = 0.0;
    if (t < cells) {
        double c[3];
        int idx[3];
        centre(G, t, c, idx);
        if (cm1(b, c[0], c[1], c[2]) >= 0.0) {
            cnt = 1.0;
            sx = c[0]; sy = c[1]; sz = c[2];
        }
        if (idx[0] < G.n[0] - 1 && idx[1] < G.n[1] - 1 && idx[2] < G.n[2] - 1) {
            double P[8][3], g[8];
            for (int q = 0; q < 8; ++q) {
                for (int a = 0; a < 3; ++a) P[q][a] = G.lo[a] + G.h * (double)(idx[a] + ((q >> a) & 1));
                g[q] = cm1(b, P[q][0], P[q][1], P[q][2]);
            }
            double gmin = g[0], gmax = g[0];
            for (int q = 1; q < 8; ++q) { gmin = fmin(gmin, g[q]); gmax = fmax(gmax, g[q]); }
            if (gmin < 0.0 && gmax >= 0.0) {
                const int tets[6][4] = {{0, 1, 3, 7}, {0, 3, 2, 7}, {0, 2, 6, 7}, {0, 6, 4, 7}, {0, 4, 5, 7}, {0, 5, 1, 7}};
                for (int e = 0; e < 6; ++e) {
                    double Pt[4][3], gt[4];
                    for (int v = 0; v < 4; ++v) {
                        gt[v] = g[tets[e][v]];
                        for (int a = 0; a < 3; ++a) Pt[v][a] = P[tets[e][v]][a];
                    }
                    area += tet_area(Pt, gt);
                }
            }
        }
    }
    const double v[5] = {cnt, sx, sy, sz, area};
    for (int q = 0; q < 5; ++q) {
        const double s = block_sum(v[q], red);
        if (threadIdx.x == 0) part[5 * blockIdx.x + q] = s;
    }
}

// First moments alone: the sums of pass 1, in its order.
__global__ __launch_bounds__(BLK) void k_shape_centre(Body b, Body32 q, Grid G, long long cells,
                                                      double *__restrict__ part) {
    __shared__ double red[4];
    const long long t = blockIdx.x * (long long)BLK + threadIdx.x;
    double v[3] = {0.0, 0.0, 0.0};
    if (t < cells) {
        double c[3];
        int idx[3];
        centre(G, t, c, idx);
        if (inside(b, q, c[0], c[1], c[2]))
            for (int a = 0; a < 3; ++a) v[a] = c[a];
    }
    for (int a = 0; a < 3; ++a) {
        const double s = block_sum(v[a], red);
        if (threadIdx.x == 0) part[3 * blockIdx.x + a] = s;
    }
}

// Pass 2: second moments about the centroid c of the inside centres.
__global__ __launch_bounds__(BLK) void k_shape_moments(Body b, Body32 q, Grid G, long long cells, double cx, double cy,
                                                       double cz, double *__restrict__ part) {
#pragma clang fp contract(off)
    __shared__ double red[4];
    const long long t = blockIdx.x * (long long)BLK + threadIdx.x;
    double m[6] = {0, 0, 0, 0, 0, 0};
    if (t < cells) {
        double c[3];
        int idx[3];
        centre(G, t, c, idx);
        if (inside(b, q, c[0], c[1], c[2])) {
            const double r[3] = {c[0] - cx, c[1] - cy, c[2] - cz};
            m[0] = r[0] * r[0]; m[1] = r[1] * r[1]; m[2] = r[2] * r[2];
            m[3] = r[0] * r[1]; m[4] = r[0] * r[2]; m[5] = r[1] * r[2];
        }
    }
    for (int e = 0; e < 6; ++e) {
        const double s = block_sum(m[e], red);
        if (threadIdx.x == 0) part[6 * blockIdx.x + e] = s;
    }
}

// Pass 3: min and max of the inside centres projected on the three axes
// (rows of ax), relative to the centroid.
__global__ __launch_bounds__(BLK) void k_shape_extent(Body b, Body32 q, Grid G, long long cells, double cx,
                                                      double cy, double cz, Axes A, double *__restrict__ part) {
#pragma clang fp contract(off)
    __shared__ double red[4];
    const double *ax = A.a;
    const long long t = blockIdx.x * (long long)BLK + threadIdx.x;
    double lo[3] = {HUGE_VAL, HUGE_VAL, HUGE_VAL}, mhi[3] = {HUGE_VAL, HUGE_VAL, HUGE_VAL};
    if (t < cells) {
        double c[3];
        int idx[3];
        centre(G, t, c, idx);
        if (inside(b, q, c[0], c[1], c[2])) {
            const double r[3] = {c[0] - cx, c[1] - cy, c[2] - cz};
            for (int a = 0; a < 3; ++a) {
                const double pr = (r[0] * ax[3 * a] + r[1] * ax[3 * a + 1]) + r[2] * ax[3 * a + 2];
                lo[a] = pr;
                mhi[a] = -pr;
            }
        }
    }
    for (int a = 0; a < 3; ++a) {
        const double mn = block_min(lo[a], red), mx = block_min(mhi[a], red);
        if (threadIdx.x == 0) {
            part[6 * blockIdx.x + a] = mn;
            part[6 * blockIdx.x + 3 + a] = mx;
        }
    }
}

// ------------------------------------------------------------- slab form
// The same decisions, with each grid sample evaluated once, first in FP32
// (inside).
//
// Node and centre coordinates along axis a, as written in pass 1.
__device__ __forceinline__ double node_at(const Grid &G, int a, int i) {
#pragma clang fp contract(off)
    return G.lo[a] + G.h * (double)i;
}
__device__ __forceinline__ double centre_at(const Grid &G, int a, int i) {
#pragma clang fp contract(off)
    return G.lo[a] + G.h * ((double)i + 0.5);
}

// Side of all nodes and centres in the box of nodes [i0, i1] x [j0, j1] x
// [k0, k1]: -1 when even the sum of each point's largest term in the box is below
// 1, 1 when the sum of the smallest terms is above it (a margin of 1e-9 for the
// roundings of this sum and of the exact one), else 0.
__device__ int box_side(const Body &b, const Grid &G, int i0, int i1, int j0, int j1, int k0, int k1) {
    const double lo[3] = {node_at(G, 0, i0), node_at(G, 1, j0), node_at(G, 2, k0)};
    const double hi[3] = {node_at(G, 0, i1), node_at(G, 1, j1), node_at(G, 2, k1)};
    double most = 0.0, least = 0.0;
    for (int j = 0; j < b.n; ++j) {
        double near = 0.0, far = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double d0 = lo[a] - b.p[j][a], d1 = b.p[j][a] - hi[a];
            const double dn = fmax(0.0, fmax(d0, d1)), df = fmax(fabs(d0), fabs(d1));
            near += dn * dn;
            far += df * df;
        }
        most += b.k[j] / near;  // +inf with a control point in the box
        least += b.k[j] / far;
    }
    return most < 1.0 - 1e-9 ? -1 : least > 1.0 + 1e-9 ? 1 : 0;
}

// Area of the interpolated surface in one tetrahedron (corners a, b, c, d of the
// cell at the node o, bit 0 of a corner along x, 1 along y, 2 along z; g: the
// cell's corner values): tet_area with the corners' numbers in place of their
// values, so that nothing is indexed in registers.
__device__ double cell_tet_area(const Grid &G, const int o[3], const double *g, unsigned corners) {
#pragma clang fp contract(off)
    unsigned pos = 0u, neg = 0u, np = 0u, nn = 0u;  // corner numbers, four bits each, in order
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const unsigned id = (corners >> (4 * v)) & 7u;
        if (g[id] >= 0.0) pos |= id << (4 * np++);
        else neg |= id << (4 * nn++);
    }
    if (np == 0 || nn == 0) return 0.0;
    // two and two: p0, p1 against n0, n1; one against three: it takes both p
    const bool two = np == 2;
    const unsigned few = np <= 2 ? pos : neg, many = np <= 2 ? neg : pos;
    const unsigned p0 = few & 7u, p1 = two ? (few >> 4) & 7u : p0;
    const unsigned n0 = many & 7u, n1 = (many >> 4) & 7u, n2 = two ? n1 : (many >> 8) & 7u;
    auto cut = [&](unsigned u, unsigned v, double r[3]) {
        const double t = g[u] / (g[u] - g[v]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double pu = node_at(G, c, o[c] + (int)((u >> c) & 1u)), pv = node_at(G, c, o[c] + (int)((v >> c) & 1u));
            r[c] = pu + t * (pv - pu);
        }
    };
    auto tri = [](const double a[3], const double b[3], const double c[3]) {
        const double u[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
        const double v[3] = {c[0] - a[0], c[1] - a[1], c[2] - a[2]};
        const double x = u[1] * v[2] - u[2] * v[1], y = u[2] * v[0] - u[0] * v[2], z = u[0] * v[1] - u[1] * v[0];
        return 0.5 * sqrt((x * x + y * y) + z * z);
    };
    double q0[3], q1[3], q2[3];
    cut(p0, n0, q0);
    cut(p0, n1, q1);
    cut(p1, n2, q2);
    double area = tri(q0, q1, q2);
    if (two) {
        cut(p1, n0, q1);
        area += tri(q0, q2, q1);
    }
    return area;
}

// Pass 1, slab form.  Block (y, z patch of 15 x 15 cells, segment of SEG cells
// along x): each thread marches its node column through the segment, one node
// and one centre a plane, so a node is evaluated once (and on the patch's rim
// twice) instead of for each of its eight cells; boxes of eight planes that a
// bound on C puts on one side (nineteen in twenty) are not evaluated at all.  Cells with nodes on both
// sides are listed (LDS, in a fixed order) and their area formed afterwards
// from exact values, 32 cells at a time: a lane a corner, then a lane a
// tetrahedron.  Per block: ten integer sums of the
// inside centres' indices relative to the patch (count, first and second
// moments: exact, so the centroid and moments need no second pass), the area,
// and per row of the segment its first and last inside centre (255: none).
// Bound by the longest block, a patch that the surface runs along for its whole
// segment, hence the short segments (16 cells: 84 us, 32: 131, for a body of 8
// points, R 10, cell 0.2, where the general form's first pass takes 481 and its
// second 69).
constexpr int SLAB = 15, SEG = 16, BOX = 8, NSUM = 10, CELLS = BLK / 8;
struct SlabOut {
    int sum[NSUM];  // 1, x, y, z, xx, yy, zz, xy, xz, yz
    int pad[2];
    double area;
};
__global__ __launch_bounds__(BLK) void k_shape_slab(Body b, Body32 q, Grid G, int py, int pz, SlabOut *__restrict__ out,
                                                    uchar2 *__restrict__ rows) {
    __shared__ double red[4];
    __shared__ uint8_t sgn[2][16][16];
    __shared__ uint16_t list[SLAB * SLAB * SEG];
    __shared__ int cnt[4], tot[4][NSUM];
    __shared__ double corner[CELLS][8];
    __shared__ unsigned tets[6];  // corner numbers of the six tetrahedra, four bits each
    if (threadIdx.x < 6) {
        const unsigned all[6] = {0x7310u, 0x7230u, 0x7620u, 0x7460u, 0x7540u, 0x7150u};
        unsigned v = all[0];
#pragma unroll
        for (int e = 1; e < 6; ++e)
            if (threadIdx.x == e) v = all[e];
        tets[threadIdx.x] = v;
    }
    const int t = threadIdx.x, ty = t & 15, tz = t >> 4, lane = t & 63, w = t >> 6;
    const int seg = blockIdx.x / (py * pz), pr = blockIdx.x - seg * (py * pz);
    const int x0 = seg * SEG, y0 = (pr % py) * SLAB, z0 = (pr / py) * SLAB;
    const int iy = y0 + ty, iz = z0 + tz;
    const int nx = min(SEG, G.n[0] - x0);  // centres of the segment
    const bool row = ty < SLAB && tz < SLAB && iy < G.n[1] && iz < G.n[2];
    const bool cell_row = row && iy < G.n[1] - 1 && iz < G.n[2] - 1;
    const double yn = node_at(G, 1, iy), zn = node_at(G, 2, iz), yc = centre_at(G, 1, iy), zc = centre_at(G, 2, iz);
    int n = 0, sx = 0, sxx = 0, first = 255, last = 255, listed = 0;
    auto centre_in = [&](int i) {
        ++n;
        sx += i;
        sxx += i * i;
        if (first == 255) first = i;
        last = i;
    };
    bool in0 = false, out0 = false;  // among the four nodes of the cell's face at the plane before
    bool plane = false;              // those are known
    for (int i0 = 0; i0 < nx; i0 += BOX) {  // block-uniform
        const int i1 = min(i0 + BOX, nx);
        const int side = box_side(b, G, x0 + i0, x0 + i1, y0, y0 + SLAB, z0, z0 + SLAB);
        if (side != 0) {  // planes i0 .. i1 on one side
            in0 = side > 0;
            out0 = side < 0;
            plane = true;
            if (side > 0 && row)
                for (int i = i0; i < i1; ++i) centre_in(i);
            continue;
        }
        for (int i = plane ? i0 + 1 : i0; i <= i1; ++i) {
            sgn[i & 1][tz][ty] = inside(b, q, node_at(G, 0, x0 + i), yn, zn);
            __syncthreads();
            bool in1 = false, out1 = false, mixed = false;
            if (cell_row) {
                const int c4 = sgn[i & 1][tz][ty] + sgn[i & 1][tz][ty + 1] + sgn[i & 1][tz + 1][ty] +
                               sgn[i & 1][tz + 1][ty + 1];
                in1 = c4 > 0;
                out1 = c4 < 4;
                mixed = i > i0 && x0 + i - 1 < G.n[0] - 1 && (in0 || in1) && (out0 || out1);
            }
            const unsigned long long m = __ballot(mixed);
            if (lane == 0) cnt[w] = __popcll(m);
            __syncthreads();
            if (mixed) {
                int at = listed + __popcll(m & ((1ull << lane) - 1ull));
                for (int v = 0; v < w; ++v) at += cnt[v];
                list[at] = (uint16_t)((i - 1) | (ty << 5) | (tz << 9));  // i - 1 < 32
            }
            listed += cnt[0] + cnt[1] + cnt[2] + cnt[3];
            in0 = in1;
            out0 = out1;
            if (i > i0 && row && inside(b, q, centre_at(G, 0, x0 + i - 1), yc, zc)) centre_in(i - 1);
        }
        plane = true;
    }
    if (row) rows[((size_t)seg * G.n[2] + iz) * G.n[1] + iy] = make_uchar2((uint8_t)first, (uint8_t)last);
    int v[NSUM] = {n, sx, n * ty, n * tz, sxx, n * ty * ty, n * tz * tz, sx * ty, sx * tz, n * ty * tz};
#pragma unroll
    for (int k = 0; k < NSUM; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
        if (lane == 0) tot[w][k] = v[k];
    }
    __syncthreads();  // the list and the sums
    double area = 0.0;
    for (int e0 = 0; e0 < listed; e0 += CELLS) {  // block-uniform
        const int e = t / 8, c = list[min(e0 + e, listed - 1)], v = t & 7;
        corner[e][v] = cm1(b, node_at(G, 0, x0 + (c & 31) + (v & 1)), node_at(G, 1, y0 + ((c >> 5) & 15) + ((v >> 1) & 1)),
                           node_at(G, 2, z0 + (c >> 9) + (v >> 2)));
        __syncthreads();
        const int et = t / 6;
        if (et < CELLS && e0 + et < listed) {
            const int ct = list[e0 + et], o[3] = {x0 + (ct & 31), y0 + ((ct >> 5) & 15), z0 + (ct >> 9)};
            area += cell_tet_area(G, o, corner[et], tets[t - 6 * et]);
        }
        __syncthreads();
    }
    area = block_sum(area, red);
    if (t < NSUM) out[blockIdx.x].sum[t] = tot[0][t] + tot[1][t] + tot[2][t] + tot[3][t];
    if (t == 0) out[blockIdx.x].area = area;
}

// Pass 3, slab form: the extents from each row's first and last inside centre
// (along a row the projection is monotone, roundings included).
__global__ __launch_bounds__(BLK) void k_shape_rows(Grid G, int segs, double cx, double cy, double cz,
                                                    Axes A, const uchar2 *__restrict__ rows,
                                                    double *__restrict__ part) {
#pragma clang fp contract(off)
    __shared__ double red[4];
    const double *ax = A.a;
    double lo[3] = {HUGE_VAL, HUGE_VAL, HUGE_VAL}, mhi[3] = {HUGE_VAL, HUGE_VAL, HUGE_VAL};
    const long long N = (long long)segs * G.n[1] * G.n[2];
    for (long long r = blockIdx.x * (long long)BLK + threadIdx.x; r < N; r += (long long)gridDim.x * BLK) {
        const uchar2 f = rows[r];
        if (f.x == 255) continue;
        const int iy = (int)(r % G.n[1]), iz = (int)(r / G.n[1] % G.n[2]), x0 = (int)(r / ((long long)G.n[1] * G.n[2])) * SEG;
        const double ry = centre_at(G, 1, iy) - cy, rz = centre_at(G, 2, iz) - cz;
        for (int e = 0; e < 2; ++e) {
            const double rx = centre_at(G, 0, x0 + (e ? f.y : f.x)) - cx;
            for (int a = 0; a < 3; ++a) {
                const double p = (rx * ax[3 * a] + ry * ax[3 * a + 1]) + rz * ax[3 * a + 2];
                lo[a] = fmin(lo[a], p);
                mhi[a] = fmin(mhi[a], -p);
            }
        }
    }
    for (int a = 0; a < 3; ++a) {
        const double mn = block_min(lo[a], red), mx = block_min(mhi[a], red);
        if (threadIdx.x == 0) {
            part[6 * blockIdx.x + a] = mn;
            part[6 * blockIdx.x + 3 + a] = mx;
        }
    }
}

// Pass 4 (105 -> 14 us with eight lanes a column and the FP32 first decision):
// columns along the shortest axis (aS) over the grid of the plane of
// the two longer ones (aL along u, aI along v) that hold an inside sample: eight
// lanes a column, each every eighth sample, from the middle on (where most
// columns have one), until a lane of the group has found one.
constexpr int COL_LANES = 8;
__global__ __launch_bounds__(BLK) void k_shape_project(Body b, Body32 q, double cx, double cy, double cz,
                                                       Axes A, double hL, double hI, double hS, double h, int nu,
                                                       int nv, int nw, double *__restrict__ part) {
#pragma clang fp contract(off)
    __shared__ double red[4];
    const double *ax = A.a, *aS = ax, *aI = ax + 3, *aL = ax + 6;
    const int l = threadIdx.x % COL_LANES, base = threadIdx.x & 63 & ~(COL_LANES - 1);
    const long long cols = (long long)nu * nv, per = BLK / COL_LANES;
    double hits = 0.0;
    for (long long c0 = blockIdx.x * per; c0 < cols; c0 += gridDim.x * per) {
        const long long t = c0 + threadIdx.x / COL_LANES;
        const bool ok = t < cols;
        const int iu = ok ? (int)(t / nv) : 0, iv = ok ? (int)(t - (long long)iu * nv) : 0;
        const double u = -hL + h * (double)iu, v = -hI + h * (double)iv;
        bool open = ok, hit = false;
        for (int s = 0; s < nw; s += COL_LANES) {  // block-uniform
            if (open && s + l < nw) {
                int iw = nw / 2 + s + l;
                if (iw >= nw) iw -= nw;
                const double w = -hS + h * (double)iw;
                const double x = ((cx + u * aL[0]) + v * aI[0]) + w * aS[0];
                const double y = ((cy + u * aL[1]) + v * aI[1]) + w * aS[1];
                const double z = ((cz + u * aL[2]) + v * aI[2]) + w * aS[2];
                hit = inside(b, q, x, y, z);
            }
            if ((__ballot(hit) >> base) & ((1u << COL_LANES) - 1u)) open = false;
            if (!__any(open)) break;
        }
        if (l == 0 && ok && !open) hits += 1.0;
    }
    const double s = block_sum(hits, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Eigenvectors of a symmetric 3x3 matrix by cyclic Jacobi rotations
// (columns of V).
void jacobi3(double A[3][3], double V[3][3]) {
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) V[i][j] = i == j ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 50; ++sweep) {
        const double off = A[0][1] * A[0][1] + A[0][2] * A[0][2] + A[1][2] * A[1][2];
        const double diag = A[0][0] * A[0][0] + A[1][1] * A[1][1] + A[2][2] * A[2][2];
        if (off <= 1e-32 * diag || off == 0.0) break;
        for (int p = 0; p < 2; ++p)
            for (int q = p + 1; q < 3; ++q) {
                if (A[p][q] == 0.0) continue;
                const double th = (A[q][q] - A[p][p]) / (2.0 * A[p][q]);
                const double t = (th >= 0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(th * th + 1.0));
                const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < 3; ++k) {  // A <- J^T A J
                    const double akp = A[k][p], akq = A[k][q];
                    A[k][p] = c * akp - s * akq;
                    A[k][q] = s * akp + c * akq;
                }
                for (int k = 0; k < 3; ++k) {
                    const double apk = A[p][k], aqk = A[q][k];
                    A[p][k] = c * apk - s * aqk;
                    A[q][k] = s * apk + c * aqk;
                }
                for (int k = 0; k < 3; ++k) {
                    const double vkp = V[k][p], vkq = V[k][q];
                    V[k][p] = c * vkp - s * vkq;
                    V[k][q] = s * vkp + c * vkq;
                }
            }
    }
}

bool make_grid(const double *cp, const double *k, int n, double h, Grid &G, long long &cells) {
    double sk = 0.0;
    for (int j = 0; j < n; ++j) sk += k[j];
    const double r = std::sqrt(sk);
    for (int a = 0; a < 3; ++a) {
        double mn = cp[a], mx = cp[a];
        for (int j = 1; j < n; ++j) {
            mn = std::fmin(mn, cp[3 * j + a]);
            mx = std::fmax(mx, cp[3 * j + a]);
        }
        G.lo[a] = mn - r - h;
        const double hi = mx + r + h;
        const double na = std::ceil((hi - G.lo[a]) / h) + 1.0;
        if (!(na >= 2.0 && na < 2e6)) return false;
        G.n[a] = (int)na;
    }
    G.h = h;
    cells = (long long)G.n[0] * G.n[1] * G.n[2];
    return cells < (1ll << 31);
}

inline long long cdiv(long long a, long long b) { return (a + b - 1) / b; }

}  // namespace

extern "C" {

size_t mb_shape_work_bytes(const double *cp, const double *k, int32_t n, double h) {
    if (!cp || !k || n < 1 || n > MAXN || !(h > 0.0)) return 0;
    Grid G;
    long long cells;
    if (!make_grid(cp, k, n, h, G, cells)) return 0;
    // per-block slots of the widest pass (6 doubles), and the three axes
    const long long blocks = cdiv(cells, BLK);
    return (size_t)(6 * blocks + 16) * sizeof(double);
}

lbm_status mb_shape_descriptors(const double *cp, const double *k, int32_t n, double h, void *work,
                                size_t work_bytes, void *hip_stream, mb_shape *out) {
    if (!cp || !k || !work || !out || n < 1 || n > MAXN || !(h > 0.0)) return LBM_E_INVALID;
    Body b;
    memset(&b, 0, sizeof b);
    b.n = n;
    for (int j = 0; j < n; ++j) {
        if (!(k[j] > 0.0) || !std::isfinite(k[j])) return LBM_E_INVALID;
        for (int a = 0; a < 3; ++a) {
            if (!std::isfinite(cp[3 * j + a])) return LBM_E_INVALID;
            b.p[j][a] = cp[3 * j + a];
        }
        b.k[j] = k[j];
    }
    Grid G;
    long long cells;
    if (!make_grid(cp, k, n, h, G, cells)) return LBM_E_INVALID;
    const long long blocks = cdiv(cells, BLK);
    if (work_bytes < (size_t)(6 * blocks + 16) * sizeof(double)) return LBM_E_NOMEM;
    hipStream_t s = (hipStream_t)hip_stream;
    double *part = (double *)work;
    std::vector<double> hp;
    auto fetch = [&](size_t count, size_t from = 0) {
        hp.resize(count);
        return hipMemcpyAsync(hp.data(), part + from, count * sizeof(double), hipMemcpyDeviceToHost, s) == hipSuccess &&
               hipStreamSynchronize(s) == hipSuccess;
    };
    Body32 q;
    memset(&q, 0, sizeof q);
    double ksum = 0.0;
    for (int j = 0; j < n; ++j) {
        ksum += k[j];
        for (int a = 0; a < 3; ++a) q.anc[a] += cp[3 * j + a] / n;
    }
    q.scale = 16.0 / std::sqrt(ksum);
    for (int j = 0; j < n; ++j) {
        float *f = &q.f[j].x, l1 = 0.f;
        for (int a = 0; a < 3; ++a) {
            f[a] = (float)((cp[3 * j + a] - q.anc[a]) * q.scale);
            l1 += std::fabs(f[a]);
        }
        f[3] = (float)(k[j] * q.scale * q.scale);
        q.bp = std::fmax(q.bp, l1 * (1.f + 1e-6f));
    }
    // The slab form needs its rows and block results in the workspace (they do
    // not fit a short grid of long rows).
    //
    // Where two principal moments are equal but for roundings (a sphere, a
    // dumbbell or a cube that lies with the grid), the roundings of their sums
    // alone choose the axes, and with them dims and A_p: such a body takes its
    // centroid and moments from the general form's sums, the ones it always
    // had, and so do the extents, whose rows share the workspace with them.
    // (Equal: within 1e-4 of the largest; a gap of that leaves the axes, of
    // moments exact to 1e-14, good to 1e-10.)  With the three more passes and
    // read-backs two coincident points, radius 8, take 193 us at cell 0.25 and
    // 488 at 0.1; every pass in the general form, 240 and 920.  One control
    // point, a sphere, does without the slab form.
    const int segs = (int)cdiv(G.n[0], SEG), py = (int)cdiv(G.n[1], SLAB), pz = (int)cdiv(G.n[2], SLAB);
    const long long slabs = (long long)segs * py * pz, n_rows = (long long)segs * G.n[1] * G.n[2];
    const size_t slab_bytes = sizeof(SlabOut) * (size_t)slabs;
    SlabOut *slab = (SlabOut *)part;
    uchar2 *rows = (uchar2 *)((char *)part + slab_bytes);
    const size_t row_end = (slab_bytes + 2 * (size_t)n_rows + 7) / 8;  // in doubles; the extents' slots follow
    const long long room = 6 * blocks - (long long)row_end, ext_blocks = std::min<long long>(256, room / 6);
    const bool slab_form = n > 1 && ext_blocks >= 1 && slabs < (1ll << 31);
    bool rows_kept = slab_form;
    double cnt = 0, area = 0, c[3], m[6] = {0, 0, 0, 0, 0, 0};
    auto sum_moments = [&]() {  // pass 2
        k_shape_moments<<<(unsigned)blocks, BLK, 0, s>>>(b, q, G, cells, c[0], c[1], c[2], part);
        if (hipGetLastError() != hipSuccess || !fetch(6 * blocks)) return false;
        for (int a = 0; a < 6; ++a) m[a] = 0.0;
        for (long long e = 0; e < blocks; ++e)
            for (int a = 0; a < 6; ++a) m[a] += hp[6 * e + a];
        return true;
    };
    if (slab_form) {
        k_shape_slab<<<(unsigned)slabs, BLK, 0, s>>>(b, q, G, py, pz, slab, rows);
        std::vector<SlabOut> so((size_t)slabs);
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(so.data(), slab, slab_bytes, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return LBM_E_HIP;
        __int128 N = 0, S[3] = {0, 0, 0}, T[6] = {0, 0, 0, 0, 0, 0};  // of the cells' indices
        for (long long e = 0; e < slabs; ++e) {
            const int *v = so[e].sum;
            area += so[e].area;
            if (v[0] == 0) continue;
            const long long pr = e % ((long long)py * pz);
            const __int128 o[3] = {(e / ((long long)py * pz)) * SEG, (pr % py) * SLAB, (pr / py) * SLAB};
            const __int128 n1 = v[0], s1[3] = {v[1], v[2], v[3]};
            N += n1;
            for (int a = 0; a < 3; ++a) S[a] += s1[a] + n1 * o[a];
            const int pa[6] = {0, 1, 2, 0, 0, 1}, pb[6] = {0, 1, 2, 1, 2, 2};
            for (int e2 = 0; e2 < 6; ++e2) {
                const int a = pa[e2], d = pb[e2];
                T[e2] += v[4 + e2] + o[a] * s1[d] + o[d] * s1[a] + n1 * o[a] * o[d];
            }
        }
        if (N == 0) return LBM_E_INVALID;
        cnt = (double)N;
        for (int a = 0; a < 3; ++a) c[a] = G.lo[a] + h * ((double)S[a] / cnt + 0.5);
        // second moments about the centroid: h^2 (sum i j - sum i sum j / N)
        const int pa[6] = {0, 1, 2, 0, 0, 1}, pb[6] = {0, 1, 2, 1, 2, 2};
        for (int e2 = 0; e2 < 6; ++e2)
            m[e2] = h * h * (double)(((long double)(N * T[e2] - S[pa[e2]] * S[pb[e2]])) / (long double)N);
        double D[3][3] = {{m[0], m[3], m[4]}, {m[3], m[1], m[5]}, {m[4], m[5], m[2]}}, W[3][3];
        jacobi3(D, W);
        double w[3] = {D[0][0], D[1][1], D[2][2]};
        std::sort(w, w + 3);
        if (std::min(w[1] - w[0], w[2] - w[1]) <= 1e-4 * w[2]) {
            rows_kept = false;
            k_shape_centre<<<(unsigned)blocks, BLK, 0, s>>>(b, q, G, cells, part);
            if (hipGetLastError() != hipSuccess || !fetch(3 * blocks)) return LBM_E_HIP;
            double sum[3] = {0, 0, 0};
            for (long long e = 0; e < blocks; ++e)
                for (int a = 0; a < 3; ++a) sum[a] += hp[3 * e + a];
            for (int a = 0; a < 3; ++a) c[a] = sum[a] / cnt;
            if (!sum_moments()) return LBM_E_HIP;
        }
    } else {
        // pass 1
        k_shape_grid<<<(unsigned)blocks, BLK, 0, s>>>(b, G, cells, part);
        if (hipGetLastError() != hipSuccess || !fetch(5 * blocks)) return LBM_E_HIP;
        double sx = 0, sy = 0, sz = 0;
        for (long long e = 0; e < blocks; ++e) {
            cnt += hp[5 * e]; sx += hp[5 * e + 1]; sy += hp[5 * e + 2]; sz += hp[5 * e + 3]; area += hp[5 * e + 4];
        }
        if (!(cnt > 0.0)) return LBM_E_INVALID;
        c[0] = sx / cnt; c[1] = sy / cnt; c[2] = sz / cnt;
        if (!sum_moments()) return LBM_E_HIP;
    }
    double A[3][3] = {{m[0], m[3], m[4]}, {m[3], m[1], m[5]}, {m[4], m[5], m[2]}}, V[3][3];
    jacobi3(A, V);
    double ax[9];
    for (int j = 0; j < 3; ++j) {  // axis j = column j, signed by its largest component
        int big = 0;
        for (int a = 1; a < 3; ++a)
            if (std::fabs(V[a][j]) > std::fabs(V[big][j])) big = a;
        const double sg = V[big][j] < 0 ? -1.0 : 1.0;
        for (int a = 0; a < 3; ++a) ax[3 * j + a] = sg * V[a][j];
    }
    // pass 3
    Axes A3, A4;
    memcpy(A3.a, ax, sizeof ax);
    const long long eb = rows_kept ? std::min(ext_blocks, cdiv(n_rows, BLK)) : blocks;
    if (rows_kept)
        k_shape_rows<<<(unsigned)eb, BLK, 0, s>>>(G, segs, c[0], c[1], c[2], A3, rows, part + row_end);
    else
        k_shape_extent<<<(unsigned)blocks, BLK, 0, s>>>(b, q, G, cells, c[0], c[1], c[2], A3, part);
    if (hipGetLastError() != hipSuccess || !fetch(6 * eb, rows_kept ? row_end : 0)) return LBM_E_HIP;
    double mn[3] = {HUGE_VAL, HUGE_VAL, HUGE_VAL}, mx[3] = {HUGE_VAL, HUGE_VAL, HUGE_VAL};
    for (long long e = 0; e < eb; ++e)
        for (int a = 0; a < 3; ++a) {
            mn[a] = std::fmin(mn[a], hp[6 * e + a]);
            mx[a] = std::fmin(mx[a], hp[6 * e + 3 + a]);
        }
    double ext[3];
    for (int a = 0; a < 3; ++a) ext[a] = -mx[a] - mn[a];
    int order[3] = {0, 1, 2};  // by increasing extent, stable
    for (int i = 1; i < 3; ++i)
        for (int j = i; j > 0 && ext[order[j]] < ext[order[j - 1]]; --j) std::swap(order[j], order[j - 1]);
    double axs[9], dims[3];
    for (int a = 0; a < 3; ++a) {
        dims[a] = ext[order[a]] + h;
        for (int q = 0; q < 3; ++q) axs[3 * a + q] = ax[3 * order[a] + q];
    }
    // pass 4: the plane of the two longer axes
    double half[3];
    int cntax[3];
    for (int a = 0; a < 3; ++a) {
        half[a] = 0.5 * dims[a] + 2.0 * h;
        cntax[a] = (int)std::ceil(2.0 * half[a] / h) + 1;
    }
    const long long cols = (long long)cntax[2] * cntax[1];
    if (cdiv(cols, BLK) > 6 * blocks) return LBM_E_NOMEM;
    const long long pblocks = std::min<long long>(std::min<long long>(2048, 6 * blocks), cdiv(cols * COL_LANES, BLK));
    memcpy(A4.a, axs, sizeof axs);
    k_shape_project<<<(unsigned)pblocks, BLK, 0, s>>>(b, q, c[0], c[1], c[2], A4, half[2], half[1], half[0], h,
                                                     cntax[2], cntax[1], cntax[0], part);
    if (hipGetLastError() != hipSuccess || !fetch(pblocks)) return LBM_E_HIP;
    double hits = 0;
    for (long long e = 0; e < pblocks; ++e) hits += hp[e];
    mb_shape &o = *out;
    o.V = cnt * h * h * h;
    o.S = area;
    o.A_p = hits * h * h;
    for (int a = 0; a < 3; ++a) {
        o.dims[a] = dims[a];
        o.centroid[a] = c[a];
    }
    memcpy(o.axes, axs, sizeof axs);
    o.d_n = std::cbrt(6.0 * o.V / M_PI);
    o.d_s = std::sqrt(4.0 * o.A_p / M_PI);
    o.Phi = M_PI * o.d_n * o.d_n / o.S;
    o.CSF = dims[0] / std::sqrt(dims[1] * dims[2]);
    o.cells_inside = (int64_t)cnt;
    o.columns_hit = (int64_t)hits;
    return LBM_OK;
}

}  // extern "C"
