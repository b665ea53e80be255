// Energy equation kernels (Sec. 1 eq:energy in Boussinesq form, Sec. 6 scheme
// list: SUPG-stabilised Galerkin) and the buoyancy right-hand side of
// eq:stokes, all with the one-point rule of Sec. 4.
//
// Per wedge e at q_c: V_e, basis gradients grad phi_j, the mean velocity
// ubar = (1/6) sum_j u_j, and the SUPG parameter
//   tau_e = h_e / (2 |ubar|) (coth Pe - 1/Pe),  Pe = |ubar| h_e / 2,  h_e = V_e^(1/3)
// (unit diffusivity).  The backward-Euler operator on a temperature T is
//   (E T)_i = sum_e V_e [ N_i T_i / dt + grad phi_i . grad T
//                          + N_i ubar . grad T + tau (ubar . grad phi_i)(ubar . grad T) ]
// with N_i(q_c) = 1/6, i.e. lumped mass, diffusion, advection and streamline
// diffusion.  Every kernel gathers over the wedges around a node (no atomics)
// and produces per-diamond partial sums that the interface pass completes.
#include <cstdio>
#include <type_traits>

#include "batch_dev.hpp"
#include "mg.hpp"
#include "tng_internal.hpp"

namespace tng {
namespace {

inline unsigned nblk(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

struct NodeIdx4 {
    int d, i, j, k;
};
__device__ __forceinline__ NodeIdx4 decode4(long long t, int m, int n) {
    NodeIdx4 r;
    r.k = (int)(t % (n + 1));
    t /= (n + 1);
    r.j = (int)(t % (m + 1));
    t /= (m + 1);
    r.i = (int)(t % (m + 1));
    r.d = (int)(t / (m + 1));
    return r;
}

// lateral offsets of the three nodes of wedge 0 / wedge 1 in a cell
__constant__ int c_cdi[2][3] = {{0, 1, 0}, {1, 0, 1}};
__constant__ int c_cdj[2][3] = {{0, 0, 1}, {1, 1, 0}};

__device__ __forceinline__ void grad_of(const double* g, double s1, int lat, int top, double out[3]) {
    const double a = lat == 0 ? -1.0 : (lat == 1 ? 1.0 : 0.0);
    const double b = lat == 0 ? -1.0 : (lat == 2 ? 1.0 : 0.0);
    const double c = top ? 1.0 : -1.0;
    for (int x = 0; x < 3; ++x) out[x] = a * s1 * g[x] + b * s1 * g[3 + x] + c * g[6 + x];
}

__device__ __forceinline__ double supg_tau(double unorm, double h) {
    const double pe = 0.5 * unorm * h;
    // coth(Pe) - 1/Pe = Pe/3 - Pe^3/45 + ... ; tau = h/(2|u|) (coth Pe - 1/Pe)
    if (pe < 1e-3) return h * h / 12.0 * (1.0 - pe * pe / 15.0);
    return h / (2.0 * unorm) * (1.0 / tanh(pe) - 1.0 / pe);
}

// Wedges around node (q.d, q.i, q.j, q.k): calls f(ci, cj, ck, wd, lat, top)
// for every wedge having the node as local vertex (lat, top).
template <typename F>
__device__ __forceinline__ void for_node_wedges(const NodeIdx4& q, int m, int n, F&& f) {
    for (int ci = q.i - 1; ci <= q.i; ++ci) {
        if (ci < 0 || ci >= m) continue;
        for (int cj = q.j - 1; cj <= q.j; ++cj) {
            if (cj < 0 || cj >= m) continue;
            const int di = q.i - ci, dj = q.j - cj;
            for (int ck = q.k - 1; ck <= q.k; ++ck) {
                if (ck < 0 || ck >= n) continue;
                const int top = q.k - ck;
                for (int wd = 0; wd < 2; ++wd) {
                    int lat = -1;
                    for (int l = 0; l < 3; ++l)
                        if (c_cdi[wd][l] == di && c_cdj[wd][l] == dj) lat = l;
                    if (lat >= 0) f(ci, cj, ck, wd, lat, top);
                }
            }
        }
    }
}

struct EnergyGeo {
    const double* geo;
    int m, n;
    double r_in, dr;
};

template <typename T>
struct WedgeField {
    // gathers the six nodal values of a field for wedge (d, ci, cj, ck, wd)
    __device__ __forceinline__ static void gather(const T* f, int d, int ci, int cj, int ck, int wd, int m, int n,
                                                  double v[6]) {
        for (int l = 0; l < 6; ++l) {
            const int lat = l % 3, top = l / 3;
            const long long s = (((long long)d * (m + 1) + ci + c_cdi[wd][lat]) * (m + 1) + cj + c_cdj[wd][lat]) *
                                    (n + 1) + ck + top;
            v[l] = (double)f[s];
        }
    }
};

// Flow data of every wedge for the SUPG operator, which depends on the velocity
// only: ubar (3 values) and tau at q_c, FP64, [10][m][m][n][2][4].  Computed once
// per velocity field instead of once per node of the wedge in every apply.
constexpr int WF = 4;
template <typename T>
__global__ void wedge_flow_kernel(EnergyGeo G, const T* __restrict__ u0, const T* __restrict__ u1,
                                  const T* __restrict__ u2, double* __restrict__ wf, long long ncells) {
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncells) return;
    const int m = G.m, n = G.n;
    const int ck = (int)(c % n);
    long long r = c / n;
    const int cj = (int)(r % m);
    r /= m;
    const int ci = (int)(r % m);
    const int d = (int)(r / m);
    const double rm = G.r_in + (ck + 0.5) * G.dr;
    for (int wd = 0; wd < 2; ++wd) {
        const double* g = G.geo + (((long long)d * m + ci) * m + cj) * GEO_PER_COL + wd * GEO_PER_TRI;
        const double V = rm * rm * g[9];
        double uu[3][6];
        WedgeField<T>::gather(u0, d, ci, cj, ck, wd, m, n, uu[0]);
        WedgeField<T>::gather(u1, d, ci, cj, ck, wd, m, n, uu[1]);
        WedgeField<T>::gather(u2, d, ci, cj, ck, wd, m, n, uu[2]);
        double ub[3];
        for (int x = 0; x < 3; ++x)
            ub[x] = (uu[x][0] + uu[x][1] + uu[x][2] + uu[x][3] + uu[x][4] + uu[x][5]) * (1.0 / 6.0);
        const double un = sqrt(ub[0] * ub[0] + ub[1] * ub[1] + ub[2] * ub[2]);
        double* w = wf + (c * 2 + wd) * WF;
        w[0] = ub[0];
        w[1] = ub[1];
        w[2] = ub[2];
        w[3] = supg_tau(un, cbrt(V));
    }
}

// y = E T (mode 0), or the diagonal of E (mode 1).  Dirichlet rows handled later.
template <typename T, int MODE>
__global__ void energy_node_kernel(EnergyGeo G, const T* __restrict__ Tin, const double* __restrict__ wf,
                                   double inv_dt, T* __restrict__ y, long long nslots) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nslots) return;
    const NodeIdx4 q = decode4(t, G.m, G.n);
    const int m = G.m, n = G.n;
    double acc = 0.0;
    for_node_wedges(q, m, n, [&](int ci, int cj, int ck, int wd, int lat, int top) {
        const double* g = G.geo + (((long long)q.d * m + ci) * m + cj) * GEO_PER_COL + wd * GEO_PER_TRI;
        const double rm = G.r_in + (ck + 0.5) * G.dr;
        const double s1 = 0.5 / rm;
        const double V = rm * rm * g[9];
        const double* w = wf + (((((long long)q.d * m + ci) * m + cj) * n + ck) * 2 + wd) * WF;
        const double ub[3] = {w[0], w[1], w[2]};
        const double tau = w[3];
        double gi[3];
        grad_of(g, s1, lat, top, gi);
        const double ugi = ub[0] * gi[0] + ub[1] * gi[1] + ub[2] * gi[2];
        if (MODE == 0) {
            double Tv[6];
            WedgeField<T>::gather(Tin, q.d, ci, cj, ck, wd, m, n, Tv);
            // grad T = A rho1~ + B rho2~ + C rho3' with nodal differences
            const double A = Tv[1] + Tv[4] - Tv[0] - Tv[3];
            const double B = Tv[2] + Tv[5] - Tv[0] - Tv[3];
            const double C = Tv[3] + Tv[4] + Tv[5] - Tv[0] - Tv[1] - Tv[2];
            double gT[3];
            for (int x = 0; x < 3; ++x) gT[x] = A * s1 * g[x] + B * s1 * g[3 + x] + C * g[6 + x];
            const double a = ub[0] * gT[0] + ub[1] * gT[1] + ub[2] * gT[2];
            const double Ti = Tv[lat + 3 * top];
            acc += V * ((1.0 / 6.0) * Ti * inv_dt + gi[0] * gT[0] + gi[1] * gT[1] + gi[2] * gT[2] +
                        (1.0 / 6.0) * a + tau * ugi * a);
        } else {
            // diagonal: T = e_i, grad T = grad phi_i
            acc += V * ((1.0 / 6.0) * inv_dt + gi[0] * gi[0] + gi[1] * gi[1] + gi[2] * gi[2] +
                        (1.0 / 6.0) * ugi + tau * ugi * ugi);
        }
    });
    y[t] = T(acc);
}

constexpr int RING_MAXL = 32;   // lateral slots of a workgroup, at most

// b_i = m_i (T_i / dt + H_i), m_i = sum_e V_e / 6 (lumped mass): with V_e = r_m^2 g9 a
// node's mass is (sum of g9 over its triangles, of all diamonds) times the radial factor
// (r_below^2 + r_above^2) / 6.  Dirichlet rows: T_in, T_out.
template <typename T>
__global__ void __launch_bounds__(256) energy_rhs_kernel(EnergyGeo G, const int* __restrict__ ring_tri, int nlat,
                                                         int nlb, MagicDiv dn1, const T* __restrict__ Tn,
                                                         const T* __restrict__ H, double inv_dt, double T_in,
                                                         double T_out, T* __restrict__ b) {
    __shared__ double ms[RING_MAXL];
    const int lat0 = (int)xcd_block() * nlb;
    if (lat0 >= nlat) return;
    const int nl = min(nlb, nlat - lat0);
    if ((int)threadIdx.x < nl) {
        double v = 0.0;
        for (int r = 0; r < 6; ++r) {
            const int cd = ring_tri[(size_t)(lat0 + threadIdx.x) * 6 + r];
            if (cd >= 0) v += G.geo[(size_t)(cd >> 3) * GEO_PER_COL + ((cd >> 2) & 1) * GEO_PER_TRI + 9];
        }
        ms[threadIdx.x] = v * (1.0 / 6.0);
    }
    __syncthreads();
    const int n1 = G.n + 1;
    const size_t out0 = (size_t)lat0 * n1;
    for (unsigned t = threadIdx.x; t < (unsigned)(nl * n1); t += 256) {
        const int li = (int)mdiv(t, dn1), k = (int)t - li * n1;
        if (k == 0 || k == G.n) {
            b[out0 + t] = T(k == 0 ? T_in : T_out);
            continue;
        }
        const double ra = G.r_in + (k + 0.5) * G.dr, rb = G.r_in + (k - 0.5) * G.dr;
        b[out0 + t] = T(ms[li] * (ra * ra + rb * rb) *
                        ((double)Tn[out0 + t] * inv_dt + (H ? (double)H[out0 + t] : 0.0)));
    }
}

// Buoyancy f_(i,c) = sum_e V_e N_i(q_c) Ra T(q_c) rhat_c(q_c), rhat the direction of
// x(q_c) = r_m s_c (s_c the mean of the triangle's unit vectors); zero on no-slip spheres,
// the tangential part on free-slip ones (fs bit 0 inner, bit 1 outer).  A triangle's
// vector (Ra / 36) g9 rhat does not depend on the layer: a workgroup forms those of its
// lateral slots once in LDS and then streams their layers, 63 nodes per wave and trip: a lane
// forms the force of the six wedges above its node from T at the node and its ring of
// neighbours on two layers, equal at their bottom and top nodes, and hands it to the lane
// above as well.  The sum over the triangles of all diamonds is complete (no interface sum,
// no Dirichlet pass).  FP64 (128,128): 0.30 ms, against 1.42 ms for one thread per node
// gathering its twelve wedges with their square roots; 0.13 ms is what reading T and
// writing f once takes at the copy rate, the rest the seven reads of T through the caches.
template <typename T>
__global__ void __launch_bounds__(256) buoyancy_kernel(EnergyGeo G, const double* __restrict__ unit,
                                                       const int* __restrict__ ring_tri,
                                                       const int* __restrict__ ring_nb, int nlat, int nlb,
                                                       MagicDiv dn1, const T* __restrict__ Tn, double Ra, int fs, T* f0,
                                                       T* f1, T* f2, const double* __restrict__ tbar,
                                                       const double* __restrict__ rhoalpha) {
    __shared__ double vec[RING_MAXL * 6][3];
    __shared__ int nb[RING_MAXL * 6];
    const int lat0 = (int)xcd_block() * nlb;
    if (lat0 >= nlat) return;
    const int nl = min(nlb, nlat - lat0);
    for (int x = threadIdx.x; x < nl * 6; x += 256) {
        const int cd = ring_tri[(size_t)lat0 * 6 + x];
        const int* rn = ring_nb + (size_t)lat0 * 6 + (x / 6) * 6;
        nb[x] = cd >= 0 ? rn[x % 6] : -1 - rn[x % 6];   // past the triangles of a five-ring: negative
        const int sl[3] = {lat0 + x / 6, rn[x % 6], rn[(x + 1) % 6]};
        double sc[3] = {0.0, 0.0, 0.0};
        for (int l = 0; l < 3; ++l)
            for (int c = 0; c < 3; ++c) sc[c] += unit[(size_t)sl[l] * 3 + c];
        double w = 0.0;
        // the shape function's 1/6 and the mean's 1/6, not Ra / 36: its rounding is the same for
        // every triangle and shifts the whole field (FP64 (8,16) 1.05e-15 -> 1.07e-15 of the
        // field's norm off its value)
        if (cd >= 0)
            w = G.geo[(size_t)(cd >> 3) * GEO_PER_COL + ((cd >> 2) & 1) * GEO_PER_TRI + 9] *
                (Ra * (1.0 / 6.0) * (1.0 / 6.0)) /
                sqrt(sc[0] * sc[0] + sc[1] * sc[1] + sc[2] * sc[2]);
        for (int c = 0; c < 3; ++c) vec[x][c] = cd >= 0 ? w * sc[c] : 0.0;
    }
    __syncthreads();
    const int n = G.n, n1 = n + 1;
    const size_t out0 = (size_t)lat0 * n1;
    const int total = nl * n1, lane = threadIdx.x & 63;
    // trip: nodes [t0 + 1, t0 + 64) of the workgroup's columns; lane 0 forms the node below
    for (int t0 = 63 * (int)(threadIdx.x >> 6) - 1; t0 + 1 < total; t0 += 63 * 4) {
        const int t = t0 + lane;
        const unsigned tc = (unsigned)min(max(t, 0), total - 1);
        const int li = (int)mdiv(tc, dn1), k = (int)tc - li * n1;
        const int ka = min(k + 1, n);
        T v[7][2];
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            const int q = r < 6 ? nb[li * 6 + r] : lat0 + li;
            const T* c = Tn + (size_t)(r == 5 && q < 0 ? -1 - q : q) * n1;
            v[r][0] = c[k];
            v[r][1] = c[ka];
        }
        const double ra = G.r_in + (k + 0.5) * G.dr;
        double wa = k < n ? ra * ra : 0.0, ta = 0.0;
        if (tbar) {
            // compressible form: T' = T - Tbar(r) and rhobar alphabar, W1 in the radius
            // (six times Tbar at the wedge, as the sums of six nodes below)
            ta = 3.0 * (tbar[k] + tbar[ka]);
            wa *= 0.5 * (rhoalpha[k] + rhoalpha[ka]);
        }
        const bool five = nb[li * 6 + 5] < 0;
        double acc[3] = {0.0, 0.0, 0.0};
        double sc[7];
#pragma unroll
        for (int r = 0; r < 7; ++r) sc[r] = (double)v[r][0] + (double)v[r][1];
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            double s = sc[6] + (sc[r] + sc[r < 5 ? r + 1 : 0]) - ta;
            if (r == 5 && five) s = 0.0;   // not zero times a temperature that is not finite
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[c] += s * vec[li * 6 + r][c];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double f = k < n && t >= 0 ? wa * acc[c] : 0.0;
            acc[c] = f + lane_below(f);
        }
        if (lane == 0 || t >= total) continue;
        if ((k == 0 && !(fs & 1)) || (k == n && !(fs & 2))) {
            acc[0] = acc[1] = acc[2] = 0.0;
        } else if (k == 0 || k == n) {
            // an impermeable free-slip sphere: the normal rows prescribe zero normal velocity
            const double* rh = unit + 3 * (size_t)(lat0 + li);
            const double dn = rh[0] * acc[0] + rh[1] * acc[1] + rh[2] * acc[2];
            for (int c = 0; c < 3; ++c) acc[c] -= dn * rh[c];
        }
        f0[out0 + t] = T(acc[0]);
        f1[out0 + t] = T(acc[1]);
        f2[out0 + t] = T(acc[2]);
    }
}

// CFL data: per block max of |ubar_e| / h_e over wedges (deterministic max)
template <typename T>
__global__ void cfl_kernel(EnergyGeo G, const T* __restrict__ u0, const T* __restrict__ u1,
                           const T* __restrict__ u2, double* __restrict__ part, long long ncells) {
    __shared__ double sh[256];
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int m = G.m, n = G.n;
    double best = 0.0;
    if (t < ncells) {
        const int ck = (int)(t % n);
        long long r = t / n;
        const int cj = (int)(r % m);
        r /= m;
        const int ci = (int)(r % m);
        const int d = (int)(r / m);
        const double rm = G.r_in + (ck + 0.5) * G.dr;
        for (int wd = 0; wd < 2; ++wd) {
            const double* g = G.geo + (((long long)d * m + ci) * m + cj) * GEO_PER_COL + wd * GEO_PER_TRI;
            const double V = rm * rm * g[9];
            double uu[3][6];
            WedgeField<T>::gather(u0, d, ci, cj, ck, wd, m, n, uu[0]);
            WedgeField<T>::gather(u1, d, ci, cj, ck, wd, m, n, uu[1]);
            WedgeField<T>::gather(u2, d, ci, cj, ck, wd, m, n, uu[2]);
            double ub[3];
            for (int c = 0; c < 3; ++c)
                ub[c] = (uu[c][0] + uu[c][1] + uu[c][2] + uu[c][3] + uu[c][4] + uu[c][5]) * (1.0 / 6.0);
            const double v = sqrt(ub[0] * ub[0] + ub[1] * ub[1] + ub[2] * ub[2]) / cbrt(V);
            best = fmax(best, v);
        }
    }
    sh[threadIdx.x] = best;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Dirichlet temperature rows: value v0 on k = 0 (inner sphere), v1 on k = n
template <typename T>
__global__ void set_layers_kernel(long long ncol, int n, T* y, const T* src, double v0, double v1) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * ncol) return;
    const long long idx = (t >> 1) * (n + 1) + ((t & 1) ? n : 0);
    y[idx] = src ? src[idx] : T((t & 1) ? v1 : v0);
}

EnergyGeo make_geo(const Level& L) { return EnergyGeo{L.geo64.p, L.m, L.n, L.r_in, L.dr()}; }

}  // namespace

template <typename T>
void energy_wedge_flow(const tng_ctx* ctx, const Level& L, const T* const u[3], double* wf) {
    require_unbatched("energy_wedge_flow");
    const long long nc = L.cells();
    wedge_flow_kernel<T><<<nblk(nc, 256), 256, 0, ctx->stream>>>(make_geo(L), u[0], u[1], u[2], wf, nc);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void energy_apply_wf(const tng_ctx* ctx, const Level& L, const double* wf, double dt, const T* Tin, T* y) {
    require_unbatched("energy_apply");
    const long long ns = L.node_slots();
    {
        char detail[48] = {0};
        if (ctx->profile)
            std::snprintf(detail, sizeof(detail), "%s/SUPG/%dx%d", std::is_same<T, double>::value ? "f64" : "f32",
                          L.m, L.n);
        ScopedKernelTimer timer(ctx, "energy_apply", detail);
        energy_node_kernel<T, 0><<<nblk(ns, 256), 256, 0, ctx->stream>>>(make_geo(L), Tin, wf, 1.0 / dt, y, ns);
        TNG_HIP(hipGetLastError());
    }
    void* f[1] = {y};
    launch_interface(ctx, L, prec_of<T>(), 0, 1, f);
    set_layers_kernel<T><<<nblk(2 * L.lat_slots(), 256), 256, 0, ctx->stream>>>(L.lat_slots(), L.n, y, Tin, 0, 0);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void energy_apply(const tng_ctx* ctx, const Level& L, const T* const u[3], double dt, const T* Tin, T* y) {
    if (energy_stream_fits(L)) {
        energy_apply_stream<T>(ctx, L, u, dt, Tin, y);
        return;
    }
    DevBuf<double> wf((size_t)L.cells() * 2 * WF);
    energy_wedge_flow<T>(ctx, L, u, wf.p);
    energy_apply_wf<T>(ctx, L, wf.p, dt, Tin, y);
    TNG_HIP(hipStreamSynchronize(ctx->stream));   // wf is freed on return
}

template <typename T>
void energy_diag(const tng_ctx* ctx, const Level& L, const double* wf, double dt, T* diag) {
    require_unbatched("energy_diag");
    const long long ns = L.node_slots();
    energy_node_kernel<T, 1><<<nblk(ns, 256), 256, 0, ctx->stream>>>(make_geo(L), nullptr, wf, 1.0 / dt, diag, ns);
    TNG_HIP(hipGetLastError());
    void* f[1] = {diag};
    launch_interface(ctx, L, prec_of<T>(), 0, 1, f);
    set_layers_kernel<T><<<nblk(2 * L.lat_slots(), 256), 256, 0, ctx->stream>>>(L.lat_slots(), L.n, diag, nullptr,
                                                                               1.0, 1.0);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void energy_rhs(const tng_ctx* ctx, const Level& L, const T* Tn, const T* H, double dt, double T_in,
                double T_out, T* b) {
    const int nlb = ring_slots_per_block(L, RING_MAXL);
    energy_rhs_kernel<T><<<nblk(L.lat_slots(), nlb), 256, 0, ctx->stream>>>(
        make_geo(L), L.ring_tri.p, (int)L.lat_slots(), nlb, magic_div((unsigned)(L.n + 1)), Tn, H, 1.0 / dt, T_in,
        T_out, b);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void buoyancy_rhs(const tng_ctx* ctx, const Level& L, const T* Tn, double Ra, T* const f[3], const double* tbar,
                  const double* rhoalpha, unsigned fs) {
    require_unbatched("buoyancy_rhs");
    const int nlb = ring_slots_per_block(L, RING_MAXL);
    buoyancy_kernel<T><<<nblk(L.lat_slots(), nlb), 256, 0, ctx->stream>>>(
        make_geo(L), L.unit64.p, L.ring_tri.p, L.ring_nb.p, (int)L.lat_slots(), nlb,
        magic_div((unsigned)(L.n + 1)), Tn, Ra, (int)fs, f[0], f[1], f[2], tbar, rhoalpha);
    TNG_HIP(hipGetLastError());
}

// max over wedges of |ubar| / h into host memory (synchronises)
template <typename T>
double cfl_rate(const tng_ctx* ctx, const Level& L, const T* const u[3], DevBuf<double>& part) {
    const long long nc = L.cells();
    const unsigned nb = nblk(nc, 256);
    if (part.n < nb) part.alloc(nb);
    cfl_kernel<T><<<nb, 256, 0, ctx->stream>>>(make_geo(L), u[0], u[1], u[2], part.p, nc);
    TNG_HIP(hipGetLastError());
    std::vector<double> h(nb);
    TNG_HIP(hipMemcpyAsync(h.data(), part.p, nb * sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
    TNG_HIP(hipStreamSynchronize(ctx->stream));
    double best = 0.0;
    for (double v : h) best = std::max(best, v);
    return best;
}

#define TNG_EINST(T)                                                                                   \
    template void energy_apply<T>(const tng_ctx*, const Level&, const T* const[3], double, const T*, T*); \
    template void energy_wedge_flow<T>(const tng_ctx*, const Level&, const T* const[3], double*);          \
    template void energy_apply_wf<T>(const tng_ctx*, const Level&, const double*, double, const T*, T*);   \
    template void energy_diag<T>(const tng_ctx*, const Level&, const double*, double, T*);                 \
    template void energy_rhs<T>(const tng_ctx*, const Level&, const T*, const T*, double, double, double, T*); \
    template void buoyancy_rhs<T>(const tng_ctx*, const Level&, const T*, double, T* const[3], const double*,  \
                                  const double*, unsigned);                                                       \
    template double cfl_rate<T>(const tng_ctx*, const Level&, const T* const[3], DevBuf<double>&);
TNG_EINST(double)
TNG_EINST(float)
#undef TNG_EINST

}  // namespace tng
