// The viscous operator on small multigrid levels, gathered per node and fused with what
// the smoother does with it (Sec. 7): one launch per Chebyshev step, residual or power
// iteration step instead of seam zeroing, operator apply and update.
//
// The streaming apply (stokes_apply.hip) walks the cell rows of a band one after another,
// about ten microseconds on any small level however few cells it has.  Here a workgroup
// takes 62 consecutive node slots and gives each of their six triangles a wave: a lane
// forms the stress of the wedge above its node in its triangle, and the parts of the two
// nodes of that wedge in its column: its own (bottom) and the next lane's (top, handed on
// by a DPP shift; so are the velocities of the layer above, the next lane's, and lanes 0
// and 63 only serve their neighbours).  The six triangles' parts are added in LDS
// in ring order, over all diamonds, so that every copy of a node gets the same bits and no
// interface pass is needed.  A wedge is evaluated for each of its three columns, against
// once in the streaming apply, so this form is for levels whose launches are bound by
// latency (ring_apply_fits).
//
// With E1 = sum over the wedge's two layers of u_1 - u_0, E2 of u_2 - u_0 (node 0 the
// lane's own), C the difference between its layers of u_0 + u_1 + u_2, a_l the lateral
// basis gradients and g3 the radial row (wedge.hpp, rows without their 1/(2 r_m)),
//   2 r_m grad u = L = E1 a_1 + E2 a_2 + 2 r_m C g3,  2 r_m grad phi_0 = a_0 +- 2 r_m g3,
// and V / (2 r_m)^2 = g9 / 4: the wedge's part of row 0 is
//   eta g9/4 (L + L^T - 2/3 tr L) (a_0 +- 2 r_m g3), with no division (+ at its top node).
#include <cstdio>
#include <type_traits>

#include "batch_dev.hpp"
#include "mg.hpp"
#include "tng_internal.hpp"
#include "wedge.hpp"

namespace tng {
namespace {

// Element idx of a field addressed by a 32-bit byte offset from its base (the levels taken
// here are small): one register per address instead of two.
template <typename T>
__device__ __forceinline__ const T& elem(const T* base, unsigned idx) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + idx * (unsigned)sizeof(T));
}

enum { RING_CHEB, RING_RESID, RING_POWER, RING_A, RING_K };

template <typename T>
struct RingArgs {
    const int* __restrict__ ring_tri;
    const int* __restrict__ ring_nb;
    const T* __restrict__ geo;
    const T* __restrict__ eta;
    const T* __restrict__ x;      // velocity the operator is applied to
    const T* __restrict__ b;      // right-hand side (step, residual)
    const T* __restrict__ invd;   // inverse diagonal (step, power iteration)
    T* out;                       // step: x_k-1 in, x_k+1 out; residual; power: D^-1 A_D x
    const double* __restrict__ ab;
    int k;                        // step of the recurrence
    int prev_zero;
    unsigned ns;
    int n;
    MagicDiv dn1;
    T r_in, dr;
    int ns_in, ns_out;
    // operator apply on separate fields (RING_A, RING_K): u and y per component, pressure
    const T* __restrict__ xs[3];
    T* ys[3];
    const T* __restrict__ p;
    T* yp;
    int m;
    unsigned nbu;                 // workgroups of the velocity rows; the pressure rows follow
    MagicDiv dm, dn1p;            // division by m, nc + 1
    const int* __restrict__ ring_tri_p;
    unsigned nsp;
};

// Iso-W1 weights without the radial ones: corner lc of the coarse quad at q_c of wedge w in
// the fine cell (a, b) of it.
template <typename T>
__device__ __forceinline__ T iso_lat(int a, int b, int w, int lc) {
    constexpr IsoWeights<T> iso = make_iso_weights<T>();
    T v = T(0);
#pragma unroll
    for (int q = 0; q < 32; ++q)
        if (q == ((a * 2 + b) * 2 + w) * 4 + lc) v = iso.lw[q >> 4][(q >> 3) & 1][(q >> 2) & 1][q & 3];
    return v;
}

// Pressure rows y_p = B u of four coarse nodes: the 96 threads of a node take the six coarse
// triangles around it, times the four fine triangles in each, times the four fine layers
// around its layer, one wedge each; summed in a fixed order.
template <typename T>
__device__ __forceinline__ void ring_pressure_rows(const RingArgs<T>& a, unsigned blk, T* part) {
    const int node = threadIdx.x & 3, f = (threadIdx.x >> 2) & 3, q = (threadIdx.x >> 4) & 3, r = threadIdx.x >> 6;
    const unsigned t = blk * 4u + node, tc = min(t, a.nsp - 1);
    const int m = a.m, mc = m / 2, nc = a.n / 2;
    const unsigned lat = mdiv(tc, a.dn1p);
    const int K = (int)(tc - lat * (unsigned)(nc + 1));
    const int k = 2 * K - 2 + q;                     // fine layer of cells
    const int code = a.ring_tri_p[lat * 6 + r];
    T acc = T(0);
    if (code >= 0 && k >= 0 && k < a.n) {
        const int cc = code >> 3, wc = (code >> 2) & 1, l = code & 3;
        const int J = cc % mc, I = (cc / mc) % mc, d = cc / (mc * mc);
        // the node's corner of the coarse quad, and its radial weight at the layer
        const int lc = wc == 0 ? l : 3 - l;
        const T wr = q == 0 || q == 3 ? T(0.25) : T(0.75);
        const T rm = a.r_in + (T(k) + T(0.5)) * a.dr, r2 = T(2) * rm;
        const bool z0 = a.ns_in && k == 0, z1 = a.ns_out && k + 1 == a.n;
        // fine triangles of the coarse one: at its three corners, and the centre
        const int ca = wc == 0 ? (f == 1) : (f != 1), cb = wc == 0 ? (f == 2) : (f != 2);
        const int w = f < 3 ? wc : 1 - wc;
        const int i = 2 * I + ca, j = 2 * J + cb;
        const T* g = a.geo + (((size_t)d * m + i) * m + j) * GEO_PER_COL + w * GEO_PER_TRI;
        const unsigned base = ((unsigned)d * (m + 1) + i) * (m + 1) + j;
        const unsigned v[3] = {w == 0 ? base : base + m + 2, w == 0 ? base + m + 1 : base + 1,
                               w == 0 ? base + 1 : base + m + 1};
        T tr = T(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            T b[3], e[3];
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const T* u = a.xs[c] + ((size_t)v[s] * (a.n + 1) + k);
                const T ub = u[0], ue = u[1];
                b[s] = z0 ? T(0) : ub;
                e[s] = z1 ? T(0) : ue;
            }
            tr += ((b[1] - b[0]) + (e[1] - e[0])) * g[c] + ((b[2] - b[0]) + (e[2] - e[0])) * g[3 + c] +
                  r2 * ((e[0] + e[1] + e[2]) - (b[0] + b[1] + b[2])) * g[6 + c];
        }
        acc = -iso_lat<T>(ca, cb, w, lc) * wr * (T(0.5) * rm * g[9]) * tr;
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    T v = T(0);
#pragma unroll
    for (int x = 0; x < 6; ++x) v += part[64 * x + threadIdx.x];
#pragma unroll
    for (int x = 4; x < 64; x <<= 1) v += __shfl_xor(v, x, 64);
    if (threadIdx.x < 4 && t < a.nsp) a.yp[t] = v;
}

template <typename T, int MODE>
__global__ void __launch_bounds__(384) ring_apply_kernel(RingArgs<T> a, SlotBatch sb) {
    constexpr bool FIELDS = MODE == RING_A || MODE == RING_K;
    __shared__ T part[6][3][64];
    const long long so = slot_off(sb);
    if constexpr (FIELDS) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            a.xs[c] = at_slot(a.xs[c], so);
            a.ys[c] = at_slot(a.ys[c], so);
        }
        a.p = at_slot(a.p, so);
        a.yp = at_slot(a.yp, so);
    }
    const unsigned blk = xcd_block();
    if constexpr (MODE == RING_K) {
        if (blk >= a.nbu) {
            ring_pressure_rows<T>(a, blk - a.nbu, &part[0][0][0]);
            return;
        }
    }
    const T* eta = at_slot(a.eta, so);
    const T* x = at_slot(a.x, so);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int ti = (int)(blk * 62u) + lane - 1;      // node slot; lanes 0 and 63: the ones around
    const bool mine = lane > 0 && lane < 63 && ti < (int)a.ns;
    const unsigned t = (unsigned)min(max(ti, 0), (int)a.ns - 1);
    const int n = a.n, n1 = n + 1;
    const unsigned lat = mdiv(t, a.dn1);
    const int k = (int)(t - lat * (unsigned)n1);
    const bool off0 = a.ns_in && k == 0, offn = a.ns_out && k == n;
    T bot[3] = {T(0), T(0), T(0)}, top[3] = {T(0), T(0), T(0)};
    // velocities at the triangle's vertices on the node's layer; the next layer's are the next
    // lane's (every lane of a column has the same vertices)
    const int code = elem(a.ring_tri, lat * 6 + w);
    const unsigned v[3] = {lat, (unsigned)elem(a.ring_nb, lat * 6 + w),
                           (unsigned)elem(a.ring_nb, lat * 6 + (w < 5 ? w + 1 : 0))};
    T u[2][3][3];   // [layer k, k + 1][vertex][component]
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            u[0][s][c] = FIELDS ? elem(a.xs[c], v[s] * (unsigned)n1 + k) : elem(x, c * a.ns + v[s] * (unsigned)n1 + k);
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) u[1][s][c] = lane_above(u[0][s][c]);
    if (code >= 0 && k < n && ti >= 0 && lane < 63) {
        const int cell = code >> 3, wd = (code >> 2) & 1, l = code & 3;
        const T* g = &elem(a.geo, (unsigned)(cell * GEO_PER_COL + wd * GEO_PER_TRI));
        const T ev = T(0.25) * g[9] * elem(eta, ((unsigned)cell * (unsigned)n + k) * 2 + wd);
        const T rm = a.r_in + (T(k) + T(0.5)) * a.dr;
        T vp = T(0);                    // V pbar / (2 r_m) of the wedge
        if constexpr (MODE == RING_K) {
            const unsigned row = mdiv((unsigned)cell, a.dm), d = mdiv(row, a.dm);
            const int j = cell - (int)row * a.m, i = (int)row - (int)d * a.m;
            const unsigned mc1 = a.m / 2 + 1, nc1 = n / 2 + 1;
            const T* pc = a.p + ((size_t)((d * mc1 + i / 2) * mc1 + j / 2) * nc1 + k / 2);
            const T wlo = k & 1 ? T(0.25) : T(0.75), whi = T(1) - wlo;
#pragma unroll
            for (int lc = 0; lc < 4; ++lc) {
                const T* q = pc + (size_t)((lc & 1) * mc1 + (lc >> 1)) * nc1;
                vp += iso_lat<T>(i & 1, j & 1, wd, lc) * (wlo * q[0] + whi * q[1]);
            }
            vp *= T(0.5) * rm * g[9];
        }
        // velocities on no-slip layers count as zero
        const bool z0 = off0, z1 = a.ns_out && k + 1 == n;
        T a1[3], a2[3], g3[3], L[3][3];
        const T r2 = T(2) * rm;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T g0 = g[c], g1 = g[3 + c], gm = -(g0 + g1);
            a1[c] = l == 0 ? g0 : (l == 1 ? g1 : gm);
            a2[c] = l == 0 ? g1 : (l == 1 ? gm : g0);
            g3[c] = r2 * g[6 + c];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T b0 = z0 ? T(0) : u[0][0][c], b1 = z0 ? T(0) : u[0][1][c], b2 = z0 ? T(0) : u[0][2][c];
            const T t0 = z1 ? T(0) : u[1][0][c], t1 = z1 ? T(0) : u[1][1][c], t2 = z1 ? T(0) : u[1][2][c];
            const T E1 = (b1 - b0) + (t1 - t0), E2 = (b2 - b0) + (t2 - t0);
            const T C = (t0 + t1 + t2) - (b0 + b1 + b2);
#pragma unroll
            for (int d = 0; d < 3; ++d) L[c][d] = E1 * a1[d] + E2 * a2[d] + C * g3[d];
        }
        const T tr = T(2.0 / 3.0) * (L[0][0] + L[1][1] + L[2][2]);
        T S[3][3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            S[c][c] = ev * (L[c][c] + L[c][c] - tr) - vp;
            const int d = (c + 1) % 3;
            S[c][d] = S[d][c] = ev * (L[c][d] + L[d][c]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T P = -(S[c][0] * (a1[0] + a2[0]) + S[c][1] * (a1[1] + a2[1]) + S[c][2] * (a1[2] + a2[2]));
            const T Q = S[c][0] * g3[0] + S[c][1] * g3[1] + S[c][2] * g3[2];
            bot[c] = P - Q;
            top[c] = P + Q;
        }
    }
    // what the closing threads (wave w < 3: component w) need (loaded here: held over
    // the stress they cost ten registers and a sixth wave per SIMD, (32,32) FP64 420 -> 388 us)
    T bv = T(0), iv = T(0), xv = T(0), pv = T(0), alpha = T(0), beta = T(0);
    const unsigned e = w * a.ns + t;
    if (w < 3) {
        if constexpr (MODE == RING_CHEB || MODE == RING_RESID) bv = at_slot(a.b, so)[e];
        if constexpr (MODE == RING_CHEB || MODE == RING_POWER) iv = at_slot(a.invd, so)[e];
        xv = FIELDS ? (w == 0 ? a.xs[0] : (w == 1 ? a.xs[1] : a.xs[2]))[t] : x[e];
        if constexpr (MODE == RING_CHEB) {
            const double* ab = at_slot(a.ab, so);
            alpha = T(ab[2 * a.k]);
            beta = T(ab[2 * a.k + 1]);
            if (alpha != T(0) && !a.prev_zero) pv = at_slot(a.out, so)[e];
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) part[w][c][lane] = bot[c] + lane_below(top[c]);
    __syncthreads();
    if (w >= 3 || !mine) return;
    T yv = part[0][w][lane];
#pragma unroll
    for (int r = 1; r < 6; ++r) yv += part[r][w][lane];
    const bool bnd = off0 || offn;
    if (bnd) yv = xv;
    T* out = at_slot(a.out, so);
    if constexpr (FIELDS) {
        (w == 0 ? a.ys[0] : (w == 1 ? a.ys[1] : a.ys[2]))[t] = yv;
    } else if constexpr (MODE == RING_RESID) {
        out[e] = bv - yv;
    } else if constexpr (MODE == RING_POWER) {
        out[e] = iv * yv;
    } else {
        // as cheb_post_update_kernel
        const T r = beta * iv * (bv - yv);
        const bool use_prev = alpha != T(0) && !a.prev_zero;
        out[e] = use_prev ? xv + (alpha * (xv - pv) + r) : (alpha == T(0) ? xv + r : xv + (alpha * xv + r));
    }
}

template <typename T>
RingArgs<T> ring_args(const Level& L, bool ns_in, bool ns_out, const T* eta, const T* x) {
    RingArgs<T> a{};
    constexpr bool is64 = sizeof(T) == 8;
    a.ring_tri = L.ring_tri.p;
    a.ring_nb = L.ring_nb.p;
    a.geo = is64 ? reinterpret_cast<const T*>(L.geo64.p) : reinterpret_cast<const T*>(L.geo32.p);
    a.eta = eta;
    a.x = x;
    a.ns = (unsigned)L.node_slots();
    a.n = L.n;
    a.dn1 = magic_div((unsigned)(L.n + 1));
    a.r_in = T(L.r_in);
    a.dr = T(L.dr());
    a.ns_in = ns_in ? 1 : 0;
    a.ns_out = ns_out ? 1 : 0;
    return a;
}

// workgroups of the velocity rows
unsigned ring_blocks(const Level& L) { return (unsigned)((L.node_slots() + 61) / 62); }

// nb workgroups, timed like the streaming apply (what is fused with the operator included)
template <typename T, int MODE>
void ring_launch(const tng_ctx* ctx, const Level& L, const RingArgs<T>& a, unsigned nb) {
    const SlotBatch sb = launch_batch();
    char detail[48] = {0};
    if (ctx->profile)
        std::snprintf(detail, sizeof(detail), "%s/%s/%dx%d/ring%s", std::is_same<T, double>::value ? "f64" : "f32",
                      MODE == RING_K ? "K" : "A", L.m, L.n, sb.nb > 1 ? "/batch" : "");
    ScopedKernelTimer timer(ctx, "stokes_apply", detail);
    ring_apply_kernel<T, MODE><<<dim3(nb, 1, sb.nb), 384, 0, ctx->stream>>>(a, sb);
    TNG_HIP(hipGetLastError());
}

}  // namespace

// Where one gathered launch beats seam zeroing, streaming apply and update.  A smoother step
// gathered and streamed, FP64: (16,16), 49,130 slots, 6.7 and 19 us; (32,32), 359,370 slots, 28
// and 35; (32,44), 490,050 slots, 36.2 and 37.1; (64,10), 464,750 slots, 36 and 69; (16,170),
// 494,190 slots, 36 and 44.  FP32: (16,16) 4.7 and 20 us; (32,32) 14 and 30; (32,72), 794,970
// slots, 29 and 43.  The gathered form grows with the slots (74 ps each in FP64, 37 in FP32),
// the streaming one with the rows, so the forms meet near the FP64 line on the shells with the
// fewest rows per slot; nothing is measured above either line.
// A forced band count asks for the streaming form on every level.
template <typename T>
bool ring_apply_fits(const tng_ctx* ctx, const Level& L) {
    return ctx->apply_bands == 0 && L.node_slots() <= (sizeof(T) == 8 ? 500000 : 800000);
}

// y = A_D u or K_D [u; p] in one launch (flags: TNG_OP_A, or with TNG_OP_BT and TNG_OP_B,
// and TNG_OP_DIRICHLET), instead of the streaming apply's three launches.
template <typename T>
void ring_apply(const tng_ctx* ctx, const Level& L, const Level* Lp, unsigned flags, const void* eta,
                const void* const u[3], const void* p, void* const yu[3], void* yp) {
    const bool ns = (flags & TNG_OP_DIRICHLET) != 0, full = (flags & TNG_OP_B) != 0;
    RingArgs<T> a = ring_args<T>(L, ns, ns, (const T*)eta, nullptr);
    for (int c = 0; c < 3; ++c) {
        a.xs[c] = (const T*)u[c];
        a.ys[c] = (T*)yu[c];
    }
    a.nbu = ring_blocks(L);
    if (full) {
        a.p = (const T*)p;
        a.yp = (T*)yp;
        a.m = L.m;
        a.dm = magic_div((unsigned)L.m);
        a.dn1p = magic_div((unsigned)(Lp->n + 1));
        a.ring_tri_p = Lp->ring_tri.p;
        a.nsp = (unsigned)Lp->node_slots();
        ring_launch<T, RING_K>(ctx, L, a, a.nbu + (a.nsp + 3) / 4);
    } else {
        ring_launch<T, RING_A>(ctx, L, a, a.nbu);
    }
}

template <typename T>
void ring_cheb_step(const tng_ctx* ctx, const Level& L, bool ns_in, bool ns_out, const T* eta, const double* ab_dev,
                    int k, bool prev_zero, const T* b, const T* invd, const T* xk, T* xo) {
    RingArgs<T> a = ring_args<T>(L, ns_in, ns_out, eta, xk);
    a.b = b;
    a.invd = invd;
    a.out = xo;
    a.ab = ab_dev;
    a.k = k;
    a.prev_zero = prev_zero ? 1 : 0;
    ring_launch<T, RING_CHEB>(ctx, L, a, ring_blocks(L));
}

template <typename T>
void ring_resid(const tng_ctx* ctx, const Level& L, bool ns_in, bool ns_out, const T* eta, const T* b, const T* x,
                T* r) {
    RingArgs<T> a = ring_args<T>(L, ns_in, ns_out, eta, x);
    a.b = b;
    a.out = r;
    ring_launch<T, RING_RESID>(ctx, L, a, ring_blocks(L));
}

template <typename T>
void ring_power(const tng_ctx* ctx, const Level& L, bool ns_in, bool ns_out, const T* eta, const T* invd, const T* x,
                T* z) {
    RingArgs<T> a = ring_args<T>(L, ns_in, ns_out, eta, x);
    a.invd = invd;
    a.out = z;
    ring_launch<T, RING_POWER>(ctx, L, a, ring_blocks(L));
}

#define TNG_RINST(T)                                                                                             \
    template bool ring_apply_fits<T>(const tng_ctx*, const Level&);                                              \
    template void ring_apply<T>(const tng_ctx*, const Level&, const Level*, unsigned, const void*,                  \
                                const void* const[3], const void*, void* const[3], void*);                         \
    template void ring_cheb_step<T>(const tng_ctx*, const Level&, bool, bool, const T*, const double*, int, bool,    \
                                    const T*, const T*, const T*, T*);                                            \
    template void ring_resid<T>(const tng_ctx*, const Level&, bool, bool, const T*, const T*, const T*, T*);          \
    template void ring_power<T>(const tng_ctx*, const Level&, bool, bool, const T*, const T*, const T*, T*);
TNG_RINST(double)
TNG_RINST(float)
#undef TNG_RINST

}  // namespace tng
