// Modified method of characteristics for the temperature (Sec. 6:
// eq:characteristic, eq:departure, eq:mmoc): departure points by the explicit
// midpoint rule backwards along the velocity, and the old temperature
// interpolated there (W1).  One thread per node slot, FP64.
//
// Point location.  A wedge is the set {lam s : s in the flat triangle of its
// three lateral unit vectors, lam in [r_k, r_k+1]} (the isoparametric map
// x = r(zeta) s(xi, eta)), so a point x = a s0 + b s1 + c s2 (Cramer's rule)
// lies over the triangle when a, b, c >= 0, with lam = a + b + c and
// (xi, eta) = (b, c) / lam.  The lateral grid is the recursive midpoint
// refinement of the 20 icosahedron faces (two per diamond), and the child
// triangles of a triangle cover exactly its cone (their outer edges lie on
// the parent's great circles), so the triangle is found by testing the 20
// faces (the one whose centroid is nearest in direction: the faces of the regular
// icosahedron are the Voronoi cells of their centroids) and then descending one refinement
// level at a time into the child (of four): a corner child when the point lies beyond the
// plane of that corner's two edge midpoints, else the centre one.  In a diamond's index
// space a triangle of level size S at origin (i0, j0) is
//   type 0: (i0, j0), (i0+S, j0), (i0, j0+S);  type 1: (i0+S, j0+S), (i0, j0+S), (i0+S, j0)
// and the coarse nodes are the fine nodes at multiples of S, so the finest
// level's unit vectors serve every level.  Bound by FP64 arithmetic and the loads of the
// descent: three plane signs a level and one division per location, instead of Cramer's
// rule with its three divisions for all twenty faces and four children a level ((64,64):
// 790 -> 155 us).
#include <cmath>

#include "batch_dev.hpp"
#include "mg.hpp"
#include "tng_internal.hpp"

namespace tng {
namespace {

struct LocGeo {
    const double* unit;   // [10][m+1][m+1][3]
    int m, n;
    double r_in, r_out, dr;
};

__device__ __forceinline__ const double* unit_at(const LocGeo& G, int d, int i, int j) {
    return G.unit + (((long long)d * (G.m + 1) + i) * (G.m + 1) + j) * 3;
}

__device__ __forceinline__ void cross3(const double* a, const double* b, double* c) {
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ double dot3(const double* a, const double* b) {
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

struct Loc {
    int d, ci, cj, w, k;
    double xi, eta, zeta;
};

// face[2 d + w]: centroid direction of the icosahedron face of diamond d, triangle w
__device__ Loc locate(const LocGeo& G, const double (&face)[20][3], const double x[3]) {
    int best = 0;
    double bs = -1e300;
#pragma unroll 4
    for (int f = 0; f < 20; ++f) {
        const double sc = dot3(x, face[f]);
        if (sc > bs) {
            bs = sc;
            best = f;
        }
    }
    const int d = best >> 1;
    int i0 = 0, j0 = 0, w = best & 1;
    for (int S = G.m; S > 1; S >>= 1) {
        const int h = S >> 1;
        // edge midpoints opposite to corners 2, 0, 1: m01 on the i edge through the first
        // corner, m12 on the split diagonal, m20 on the j edge
        const int o = w == 0 ? 0 : S;
        const double* p01 = unit_at(G, d, i0 + h, j0 + o);
        const double* p12 = unit_at(G, d, i0 + h, j0 + h);
        const double* p20 = unit_at(G, d, i0 + o, j0 + h);
        const double m01[3] = {p01[0], p01[1], p01[2]}, m12[3] = {p12[0], p12[1], p12[2]},
                     m20[3] = {p20[0], p20[1], p20[2]};
        double n0[3], n1[3], n2[3];
        cross3(m01, m20, n0);
        cross3(m12, m01, n1);
        cross3(m20, m12, n2);
        const double c0 = dot3(x, n0), c1 = dot3(x, n1), c2 = dot3(x, n2);
        // corners in the triangle's own order: type 0 (i0, j0), (i0+S, j0), (i0, j0+S), type 1
        // (i0+S, j0+S), (i0, j0+S), (i0+S, j0)
        const int a = w == 0 ? 0 : h, q = h - a;    // offset of corner 0's child, and of the others'
        if (c0 > 0.0) {
            i0 += a;
            j0 += a;
        } else if (c1 > 0.0) {
            i0 += q;
            j0 += a;
        } else if (c2 > 0.0) {
            i0 += a;
            j0 += q;
        } else {
            i0 += a;
            j0 += a;
            w ^= 1;
        }
    }
    const double* s0 = w == 0 ? unit_at(G, d, i0, j0) : unit_at(G, d, i0 + 1, j0 + 1);
    const double* s1 = w == 0 ? unit_at(G, d, i0 + 1, j0) : unit_at(G, d, i0, j0 + 1);
    const double* s2 = w == 0 ? unit_at(G, d, i0, j0 + 1) : unit_at(G, d, i0 + 1, j0);
    double c12[3], c20[3], c01[3];
    cross3(s1, s2, c12);
    cross3(s2, s0, c20);
    cross3(s0, s1, c01);
    const double ca = dot3(x, c12), cb = dot3(x, c20), cc = dot3(x, c01);
    const double sum = ca + cb + cc;
    double lam = sum / dot3(s0, c12);
    Loc L;
    L.d = d;
    L.ci = i0;
    L.cj = j0;
    L.w = w;
    const double inv = 1.0 / sum;
    L.xi = cb * inv;
    L.eta = cc * inv;
    // a point outside the shell is brought back radially onto it
    lam = fmin(fmax(lam, G.r_in), G.r_out);
    int k = (int)floor((lam - G.r_in) / G.dr);
    k = k < 0 ? 0 : (k > G.n - 1 ? G.n - 1 : k);
    L.k = k;
    L.zeta = 2.0 * (lam - (G.r_in + k * G.dr)) / G.dr - 1.0;
    return L;
}

// lateral offsets of the three nodes of a type-0 / type-1 cell triangle
__constant__ int c_mi[2][3] = {{0, 1, 0}, {1, 0, 1}};
__constant__ int c_mj[2][3] = {{0, 0, 1}, {1, 1, 0}};

// W1 interpolant of node field f at a located point
__device__ double interp(const LocGeo& G, const Loc& L, const double* __restrict__ f) {
    const double lat[3] = {1.0 - L.xi - L.eta, L.xi, L.eta};
    const double rad[2] = {0.5 * (1.0 - L.zeta), 0.5 * (1.0 + L.zeta)};
    double v = 0.0;
    for (int a = 0; a < 3; ++a) {
        const long long s = (((long long)L.d * (G.m + 1) + L.ci + c_mi[L.w][a]) * (G.m + 1) + L.cj + c_mj[L.w][a]) *
                            (G.n + 1) + L.k;
        v += lat[a] * (rad[0] * f[s] + rad[1] * f[s + 1]);
    }
    return v;
}

__global__ void __launch_bounds__(128) mmoc_departure_kernel(LocGeo G, MagicDiv dn1, const double* __restrict__ u0,
                                                             const double* __restrict__ u1,
                                                             const double* __restrict__ u2,
                                                             const double* __restrict__ Tn, double dt,
                                                             double* __restrict__ That, unsigned nslots) {
    __shared__ double face[20][3];
    if (threadIdx.x < 20) {
        const int d = threadIdx.x >> 1, w = threadIdx.x & 1, m = G.m;
        const double* a = w == 0 ? unit_at(G, d, 0, 0) : unit_at(G, d, m, m);
        const double* b = unit_at(G, d, m, 0);
        const double* c = unit_at(G, d, 0, m);
        for (int x = 0; x < 3; ++x) face[threadIdx.x][x] = a[x] + b[x] + c[x];
    }
    __syncthreads();
    const unsigned t = xcd_block() * 128u + threadIdx.x;
    if (t >= nslots) return;
    const unsigned lat = mdiv(t, dn1);
    const int k = (int)(t - lat * (unsigned)(G.n + 1));
    const double rk = G.r_in + k * G.dr;
    const double* s = G.unit + (size_t)lat * 3;
    const double x[3] = {rk * s[0], rk * s[1], rk * s[2]};
    // explicit midpoint rule backwards over dt (eq:departure)
    const double xm[3] = {x[0] - 0.5 * dt * u0[t], x[1] - 0.5 * dt * u1[t], x[2] - 0.5 * dt * u2[t]};
    const Loc Lm = locate(G, face, xm);
    const double um[3] = {interp(G, Lm, u0), interp(G, Lm, u1), interp(G, Lm, u2)};
    const double xh[3] = {x[0] - dt * um[0], x[1] - dt * um[1], x[2] - dt * um[2]};
    That[t] = interp(G, locate(G, face, xh), Tn);
}

}  // namespace

void mmoc_departure(const tng_ctx* ctx, const Level& L, const double* const u[3], double dt, const double* Tn,
                    double* That) {
    LocGeo G{L.unit64.p, L.m, L.n, L.r_in, L.r_out, L.dr()};
    const long long ns = L.node_slots();
    ScopedKernelTimer timer(ctx, "mmoc_departure");
    mmoc_departure_kernel<<<(unsigned)((ns + 127) / 128), 128, 0, ctx->stream>>>(
        G, magic_div((unsigned)(L.n + 1)), u[0], u[1], u[2], Tn, dt, That, (unsigned)ns);
    TNG_HIP(hipGetLastError());
    // copies of a duplicate node computed the same value up to rounding of their own
    // coordinates: make them equal
    void* f[1] = {That};
    launch_interface(ctx, L, TNG_F64, 1, 1, f);
}

}  // namespace tng
