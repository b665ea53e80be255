// Multigrid and Krylov building blocks (Sec. 7): operator diagonal, lumped
// inverse-viscosity pressure mass, W1 transfer operators, Chebyshev update,
// BLAS-1 with deterministic reductions, precision casts, and the dense
// coarsest-level solve.
//
// All velocity vectors are in the duplicated-diamond layout with equal values
// in every copy of a shared node.  Gathers that run per diamond produce
// partial sums on diamond-edge nodes; the interface kernel then adds the
// copies.  Reductions count every unique node once (owner mask).
#include "batch_dev.hpp"
#include "tng_internal.hpp"
#include "mg.hpp"
#include "wedge.hpp"

namespace tng {
namespace {

inline unsigned nblk(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// per-slot vector counts of a batched multi-dot / multi-axpy stay in range
inline void check_counts(const SlotBatch& sb) {
    if (!sb.has_cnt) return;
    for (int z = 0; z < sb.nb; ++z)
        TNG_REQUIRE(sb.cnt[z] >= 1 && sb.cnt[z] <= MAX_MDOT, "per-slot vector count out of range");
}

// Gradient of the wedge basis function of local node (lat, top) at q_c, with
// the constants folded as in wedge.hpp: sign pattern of the reference gradient
// times the folded rows of G^{-1}.
__device__ __forceinline__ void basis_grad(const double* g, double s1, int lat, int top, double out[3]) {
    const double a = lat == 0 ? -1.0 : (lat == 1 ? 1.0 : 0.0);
    const double b = lat == 0 ? -1.0 : (lat == 2 ? 1.0 : 0.0);
    const double c = top ? 1.0 : -1.0;
    for (int x = 0; x < 3; ++x) out[x] = a * s1 * g[x] + b * s1 * g[3 + x] + c * g[6 + x];
}

// Two-radial-point rule (Sec. 4): points zeta = -+1/sqrt 3 on the lateral centroid,
// weight 1/2 each.  There the Jacobian is G diag(r_q, r_q, dr/2) with r_q = r_m +
// zeta dr/2, so the lateral part of a basis gradient carries 1/r_q and the radial
// shape factor (1 + zeta) on the top face, (1 - zeta) on the bottom face; the
// radial part is the one of q_c.  s1q = 1/(2 r_q).
constexpr double TWOPT_ZETA = 0.57735026918962576451;
__device__ __forceinline__ void basis_grad_at(const double* g, double s1q, double zq, int lat, int top,
                                              double out[3]) {
    const double a = lat == 0 ? -1.0 : (lat == 1 ? 1.0 : 0.0);
    const double b = lat == 0 ? -1.0 : (lat == 2 ? 1.0 : 0.0);
    const double c = top ? 1.0 : -1.0;
    const double f = top ? 1.0 + zq : 1.0 - zq;
    for (int x = 0; x < 3; ++x) out[x] = f * (a * s1q * g[x] + b * s1q * g[3 + x]) + c * g[6 + x];
}

// Hourglass-control scale of a wedge (eq:hgstab over the three barycentric
// modes): eps_e = alpha mean(diag A_e) = alpha 5/27 eta V sum_j |grad phi_j|^2,
// sum_j |grad phi_j|^2 = 4 (|rho1~|^2 + |rho2~|^2 + rho1~.rho2~) + 6 |rho3'|^2.
__device__ __forceinline__ double hg_eps(const double* g, double s1, double V, double e, double alpha) {
    const double a = g[0] * g[0] + g[1] * g[1] + g[2] * g[2] + g[3] * g[3] + g[4] * g[4] + g[5] * g[5] +
                     g[0] * g[3] + g[1] * g[4] + g[2] * g[5];
    const double b = g[6] * g[6] + g[7] * g[7] + g[8] * g[8];
    return alpha * (5.0 / 27.0) * e * V * (4.0 * s1 * s1 * a + 6.0 * b);
}

// diag(A)_(node,c) = sum over the node's wedges of V eta (|grad phi|^2 + 1/3 (d_c phi)^2),
// the diagonal of eq:elemmat with the one-point rule, plus 2/3 eps_e with hourglass
// control (sum_a h_a[j]^2 = 2/3 for every node); twopt: the same sum over the two
// radial points, each with V_q = r_q^2 |det G| / 2.  On a free-slip sphere (fs bit 0
// inner, bit 1 outer) the row block is P A_jj P + N with P = I - rhat rhat^T: its two
// tangential diagonal entries are replaced by their mean, the same value in all three
// components, so that D^{-1} maps tangential vectors to tangential vectors:
// trace(P A_jj P) / 2 = sum_e V eta (|grad phi|^2 + (|grad phi|^2 - (rhat.grad phi)^2) / 6).
// Rows of no-slip spheres are 1.  invert: the reciprocal of every entry.
//
// With a the lateral part of the basis gradient (grad phi = s1 a +- g3, s1 = 1/(2 r_m),
// V = r_m^2 g9) an entry of a wedge is eta (A_c +- r_m B_c + r_m^2 C_c), + for the wedge
// below the node and - for the one above, with nine values per triangle that do not
// depend on the layer:
//   A_c = g9/4 (|a|^2 + a_c^2/3), B_c = g9 (a.g3 + a_c g3_c/3), C_c = g9 (|g3|^2 + g3_c^2/3);
// the two-point rule changes the radial factors only (sums over its points: 4/3,
// r_m +- dr/6, r_m^2 + dr^2/12).  A workgroup takes nlb consecutive lateral slots, forms
// their triangles' values once in LDS and then streams the slots' layers, 63 nodes per wave
// and trip: a lane forms the six wedges above its node, for their bottom node (its own) and
// their top node (handed to the lane above), so every viscosity is read once per lateral
// node.  Every node gets its complete sum over the triangles of all diamonds (no interface
// sum, no Dirichlet pass).  FP64 (128,128) with its two coarser levels: 0.33 ms, against
// 1.51 ms (+ 0.08 ms of closing passes) for one thread per node gathering twelve wedges;
// 0.19 ms is what reading eta and writing the diagonal once takes at the copy rate.
constexpr int DIAG_MAXL = 16;   // lateral slots of a workgroup, at most

template <typename T>
__global__ void __launch_bounds__(256) diag_A_kernel(const T* __restrict__ eta, const double* __restrict__ geo,
                                                     const int* __restrict__ ring_tri, int nlat, int nlb, int n,
                                                     MagicDiv dn1, double r_in, double dr, double hg_alpha, int twopt,
                                                     int fs, const double* __restrict__ unit, int invert, T* d0, T* d1,
                                                     T* d2) {
    __shared__ double coef[DIAG_MAXL * 6][9];
    __shared__ int code[DIAG_MAXL * 6];
    const int lat0 = (int)xcd_block() * nlb;
    if (lat0 >= nlat) return;
    const int nl = min(nlb, nlat - lat0);
    for (int x = threadIdx.x; x < nl * 6; x += 256) {
        const int own = ring_tri[(size_t)lat0 * 6 + x];
        // a vertex of five triangles: the sixth is the first one with zero values
        const int cd = own >= 0 ? own : ring_tri[(size_t)lat0 * 6 + x - 5];
        code[x] = cd;
        const double* g = geo + (size_t)(cd >> 3) * GEO_PER_COL + ((cd >> 2) & 1) * GEO_PER_TRI;
        const int lat = cd & 3;
        const double g9 = own >= 0 ? g[9] : 0.0;
        double a[3], aa = 0.0, ag = 0.0, gg = 0.0, as = 0.0;
        for (int c = 0; c < 3; ++c) {
            a[c] = lat == 0 ? -(g[c] + g[3 + c]) : (lat == 1 ? g[c] : g[3 + c]);
            aa += a[c] * a[c];
            ag += a[c] * g[6 + c];
            gg += g[6 + c] * g[6 + c];
            as += g[c] * g[c] + g[3 + c] * g[3 + c] + g[c] * g[3 + c];
        }
        // hourglass control: 2/3 eps_e, eps_e = alpha 5/27 eta V (4 s1^2 as + 6 gg)
        const double h = hg_alpha * (10.0 / 81.0) * g9;
        for (int c = 0; c < 3; ++c) {
            coef[x][c] = 0.25 * g9 * (aa + a[c] * a[c] / 3.0) + h * as;
            coef[x][3 + c] = g9 * (ag + a[c] * g[6 + c] / 3.0);
            coef[x][6 + c] = g9 * (gg + g[6 + c] * g[6 + c] / 3.0) + h * 6.0 * gg;
        }
    }
    __syncthreads();
    const int n1 = n + 1;
    const size_t out0 = (size_t)lat0 * n1;
    const int total = nl * n1, lane = threadIdx.x & 63;
    const double q0 = twopt ? 4.0 / 3.0 : 1.0, q1 = twopt ? dr / 6.0 : 0.0, q2 = twopt ? dr * dr / 12.0 : 0.0;
    bool nan = false;
    // trip: nodes [t0 + 1, t0 + 64) of the workgroup's columns; lane 0 forms the node below
    for (int t0 = 63 * (int)(threadIdx.x >> 6) - 1; t0 + 1 < total; t0 += 63 * 4) {
        const int t = t0 + lane;
        const unsigned tc = (unsigned)min(max(t, 0), total - 1);
        const int li = (int)mdiv(tc, dn1), k = (int)tc - li * n1;
        // the wedges above the node: p = sum eta (A + r^2 C), q = sum eta r B
        const double rm = r_in + (k + 0.5) * dr, w1 = rm + q1, w1b = rm - q1, w2 = rm * rm + q2;
        const int ka = min(k, n - 1);
        T e[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            const int cd = code[li * 6 + r];
            e[r] = eta[((size_t)(cd >> 3) * n + ka) * 2 + ((cd >> 2) & 1)];
        }
        double p[3] = {0.0, 0.0, 0.0}, q[3] = {0.0, 0.0, 0.0}, s[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            const double x = (double)e[r];
            const double* cf = coef[li * 6 + r];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                p[c] += cf[c] * x;
                q[c] += cf[3 + c] * x;
                s[c] += cf[6 + c] * x;
            }
        }
        double acc[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double m = q0 * p[c] + w2 * s[c];
            const double top = lane_below(k < n && t >= 0 ? m + w1 * q[c] : 0.0);
            acc[c] = (k < n ? m - w1b * q[c] : 0.0) + top;
        }
        if (lane == 0 || t >= total) continue;
        if ((k == 0 && !(fs & 1)) || (k == n && !(fs & 2))) {
            acc[0] = acc[1] = acc[2] = 1.0;
        } else if (k == 0 || k == n) {
            // free slip: the wedge below the outer sphere, or above the inner one
            const bool top = k > 0;
            const double rb = r_in + ((top ? k - 1 : k) + 0.5) * dr;
            const double* rh = unit + 3 * (size_t)(lat0 + li);
            acc[0] = 0.0;
            for (int r = 0; r < 6; ++r) {
                const int cd = ring_tri[(size_t)(lat0 + li) * 6 + r];
                if (cd < 0) break;
                const int cell = cd >> 3, wd = (cd >> 2) & 1;
                const double* g = geo + (size_t)cell * GEO_PER_COL + wd * GEO_PER_TRI;
                double gr[3];
                basis_grad(g, 0.5 / rb, cd & 3, top ? 1 : 0, gr);
                const double ev = (double)eta[((size_t)cell * n + (top ? k - 1 : k)) * 2 + wd];
                const double nn = gr[0] * gr[0] + gr[1] * gr[1] + gr[2] * gr[2];
                const double gn = rh[0] * gr[0] + rh[1] * gr[1] + rh[2] * gr[2];
                acc[0] += rb * rb * g[9] * ev * (nn + (nn - gn * gn) / 6.0);
            }
            acc[1] = acc[2] = acc[0];
        }
        if (invert)
            for (int c = 0; c < 3; ++c) acc[c] = (double)(T(1) / T(acc[c]));
        const double any = acc[0] + acc[1] + acc[2];
        nan |= any != any;
        d0[out0 + t] = T(acc[0]);
        d1[out0 + t] = T(acc[1]);
        d2[out0 + t] = T(acc[2]);
    }
    if (!nan) return;
    // An infinite viscosity: infinity minus infinity, or times zero, above.  Every entry is a sum
    // of its wedges' viscosities with positive weights, so it is infinite like their plain sum
    // (after the loop: in it, or with positive weights formed in it, (128,128) takes 285 -> 308
    // us in FP64 and 179 -> 212 us in FP32).
    for (int t0 = 63 * (int)(threadIdx.x >> 6) - 1; t0 + 1 < total; t0 += 63 * 4) {
        const int t = t0 + lane;
        if (lane == 0 || t >= total) continue;
        const T any = d0[out0 + t] + d1[out0 + t] + d2[out0 + t];
        if (any == any) continue;
        const int li = (int)mdiv((unsigned)t, dn1), k = t - li * n1;
        double x = 0.0;
        for (int w = 0; w < 12; ++w) {
            const int cd = code[li * 6 + w / 2], kw = k - (w & 1);
            if (kw >= 0 && kw < n) x += (double)eta[((size_t)(cd >> 3) * n + kw) * 2 + ((cd >> 2) & 1)];
        }
        if (fabs(x) <= 1.7976931348623157e308) continue;
        d0[out0 + t] = d1[out0 + t] = d2[out0 + t] = invert ? T(1) / T(x) : T(x);
    }
}

// Lumped M_{1/eta} on the pressure level: m_I = sum_e (V_e / eta_e) psi_I(q_c^e)
// (eq:pmass, row-sum lumping, one-point rule), per-diamond partial sums.  A workgroup
// owns PM_T x PM_T lateral coarse nodes and PM_K of their layers: first every coarse cell
// around them reduces its sixteen wedges to eight corner values in LDS (one reciprocal
// per wedge, at most 1.7 times per wedge over all workgroups), then every node adds its
// eight cells in a fixed order.  FP64 (128,128): 0.114 ms (0.49 ms for one thread per
// coarse node with its 128 wedges); reading eta once takes 0.065 ms at the copy rate.
constexpr int PM_T = 4, PM_K = 16;

template <typename T>
__global__ void __launch_bounds__(256) pmass_kernel(const T* __restrict__ eta, const double* __restrict__ geo, int m,
                                                    int n, double r_in, double dr, T* __restrict__ out) {
    constexpr int PC = PM_T + 1, PK = PM_K + 1;
    constexpr IsoWeights<double> iso = make_iso_weights<double>();
    __shared__ double part[8][PC * PC][PK];
    const int mc = m / 2, nc = n / 2;
    const int nt = (mc + PM_T) / PM_T, nkt = (nc + PM_K) / PM_K;   // tiles over mc + 1 nodes, nc + 1 layers
    int b = (int)xcd_block();
    const int K0 = (b % nkt) * PM_K;
    b /= nkt;
    const int J0 = (b % nt) * PM_T;
    b /= nt;
    const int I0 = (b % nt) * PM_T, d = b / nt;
    for (int x = threadIdx.x; x < PC * PC * PK; x += 256) {
        const int lk = x % PK, lj = (x / PK) % PC, li = x / (PK * PC);
        const int I = I0 - 1 + li, J = J0 - 1 + lj, K = K0 - 1 + lk;
        double p[4][2] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
        if (I >= 0 && I < mc && J >= 0 && J < mc && K >= 0 && K < nc) {
            const double r0 = r_in + (2 * K + 0.5) * dr, r1 = r_in + (2 * K + 1.5) * dr;
            T e[2][2][4];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int bb = 0; bb < 2; ++bb) {
                    const size_t col = ((size_t)d * m + 2 * I + a) * m + 2 * J + bb;
                    const T* ep = eta + (col * n + 2 * K) * 2;
#pragma unroll
                    for (int q = 0; q < 4; ++q) e[a][bb][q] = ep[q];
                }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int bb = 0; bb < 2; ++bb) {
                    const double* g = geo + (((size_t)d * m + 2 * I + a) * m + 2 * J + bb) * GEO_PER_COL;
#pragma unroll
                    for (int wd = 0; wd < 2; ++wd) {
                        const double g9 = g[wd * GEO_PER_TRI + 9];
                        const double v0 = r0 * r0 * g9 / (double)e[a][bb][wd];
                        const double v1 = r1 * r1 * g9 / (double)e[a][bb][2 + wd];
                        const double bot = iso.rw[0][0] * v0 + iso.rw[1][0] * v1;
                        const double top = iso.rw[0][1] * v0 + iso.rw[1][1] * v1;
#pragma unroll
                        for (int lc = 0; lc < 4; ++lc) {
                            const double w = iso.lw[a][bb][wd][lc];
                            if (w != 0.0) {
                                p[lc][0] += w * bot;
                                p[lc][1] += w * top;
                            }
                        }
                    }
                }
        }
#pragma unroll
        for (int lc = 0; lc < 4; ++lc) {
            part[lc][li * PC + lj][lk] = p[lc][0];
            part[4 + lc][li * PC + lj][lk] = p[lc][1];
        }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < PM_T * PM_T * PM_K; x += 256) {
        const int lk = x % PM_K, lj = (x / PM_K) % PM_T, li = x / (PM_K * PM_T);
        const int I = I0 + li, J = J0 + lj, K = K0 + lk;
        if (I > mc || J > mc || K > nc) continue;
        double acc = 0.0;
        // the cells on either side of the node; its corner in them, and the face (1: the
        // cell below has it on its top)
#pragma unroll
        for (int ci = 0; ci < 2; ++ci)
#pragma unroll
            for (int cj = 0; cj < 2; ++cj)
#pragma unroll
                for (int ck = 0; ck < 2; ++ck)
                    acc += part[(1 - ci) + 2 * (1 - cj) + 4 * (1 - ck)][(li + ci) * PC + lj + cj][lk + ck];
        out[(((size_t)d * (mc + 1) + I) * (mc + 1) + J) * (nc + 1) + K] = T(acc);
    }
}

// Prolongation (W1 interpolation in index space): a fine node that is a
// coarse node copies it, one on a coarse edge takes the mean of the edge's
// end nodes (edges along i, along j, or the split diagonal), radially odd
// layers take the mean of the two coarse layers.  y += P x (add) or y = P x.
struct ProlongNode {
    size_t a, b;      // the ends of the coarse edge that a fine node lies on (the same at a coarse node)
    unsigned edge;    // they differ
    unsigned up;      // 1: on an odd layer, between coarse layers
};
__device__ __forceinline__ ProlongNode prolong_node(unsigned t, int mf, int nf, MagicDiv dn1, MagicDiv dm1) {
    const unsigned mf1 = mf + 1, nc1 = nf / 2 + 1, mc1 = mf / 2 + 1;
    const unsigned lat = mdiv(t, dn1), k = t - lat * (nf + 1);
    const unsigned row = mdiv(lat, dm1), j = lat - row * mf1;
    const unsigned d = mdiv(row, dm1), i = row - d * mf1;
    const unsigned oi = i & 1, oj = j & 1;
    const unsigned a = (d * mc1 + i / 2) * mc1 + j / 2 + (oi & oj);
    const unsigned b = a + (oi ? mc1 : 0u) + (oi & oj ? 0u - 1u : oj);
    return {(size_t)a * nc1 + k / 2, (size_t)b * nc1 + k / 2, oi | oj, k & 1};
}

// y += P x, a component per thread
template <typename T>
__global__ void __launch_bounds__(256) prolong_add_kernel(int mf, int nf, const T* __restrict__ c0,
                                                          const T* __restrict__ c1, const T* __restrict__ c2, T* f0,
                                                          T* f1, T* f2, unsigned nslots, MagicDiv dn1, MagicDiv dm1,
                                                          SlotBatch sb) {
    const long long so = slot_off(sb);
    const unsigned t = blockIdx.x * 256u + threadIdx.x;
    if (t >= nslots) return;
    const T* c = at_slot(blockIdx.y == 0 ? c0 : (blockIdx.y == 1 ? c1 : c2), so);
    T* f = at_slot(blockIdx.y == 0 ? f0 : (blockIdx.y == 1 ? f1 : f2), so);
    const T old = f[t];
    const ProlongNode q = prolong_node(t, mf, nf, dn1, dm1);
    f[t] = old + T(0.25) * ((c[q.a] + c[q.b]) + (c[q.a + q.up] + c[q.b + q.up]));
}

// y = P x: a coarse node is copied, whatever its value.  All components per thread and
// stores past the caches, which the written field would only fill: (128,128) FP64 264 -> 140
// us, FP32 84 -> 70 us (a component per thread with plain stores: 275 and 117 us); in turn with
// a kernel that reads the field, 249 -> 217 and 150 -> 62 us.
template <typename T>
__global__ void __launch_bounds__(256) prolong_kernel(int mf, int nf, const T* __restrict__ c0,
                                                      const T* __restrict__ c1, const T* __restrict__ c2, T* f0, T* f1,
                                                      T* f2, unsigned nslots, MagicDiv dn1, MagicDiv dm1,
                                                      SlotBatch sb) {
    const long long so = slot_off(sb);
    const unsigned t = blockIdx.x * 256u + threadIdx.x;
    if (t >= nslots) return;
    const T* const c[3] = {at_slot(c0, so), at_slot(c1, so), at_slot(c2, so)};
    T* const f[3] = {at_slot(f0, so), at_slot(f1, so), at_slot(f2, so)};
    const ProlongNode q = prolong_node(t, mf, nf, dn1, dm1);
    const T w = (q.edge ? T(0.5) : T(1)) * (q.up ? T(0.5) : T(1));
    T v[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        const T a0 = c[x][q.a], a1 = c[x][q.a + q.up], b0 = c[x][q.b], b1 = c[x][q.b + q.up];
        const T s0 = q.edge ? a0 + b0 : a0, s1 = q.edge ? a1 + b1 : a1;
        v[x] = (q.up ? s0 + s1 : s0) * w;
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) __builtin_nontemporal_store(v[x], &f[x][t]);
}

// Restriction R = P^T: a coarse node gathers the fine nodes that interpolate from it, the
// fine node at its place (weight 1) and that node's ring of neighbours (1/2 each: the
// midpoints of the coarse edges at the node, over all diamonds, so that no interface sum
// follows), on three fine layers (1/2, 1, 1/2).  No-slip layers of the result are zero; the
// layer of a free-slip sphere (fs bit 0 inner, bit 1 outer) is restricted like the interior.
template <typename T>
__global__ void __launch_bounds__(256) restrict_kernel(int mf, int nf, const T* __restrict__ f0,
                                                       const T* __restrict__ f1, const T* __restrict__ f2,
                                                       const int* __restrict__ ring_tri,
                                                       const int* __restrict__ ring_nb, T* c0, T* c1, T* c2,
                                                       unsigned ncslots, MagicDiv dn1, MagicDiv dm1, int fs,
                                                       SlotBatch sb) {
    const long long so = slot_off(sb);
    const unsigned t = blockIdx.x * 256u + threadIdx.x;
    if (t >= ncslots) return;
    const T* f = at_slot(blockIdx.y == 0 ? f0 : (blockIdx.y == 1 ? f1 : f2), so);
    T* c = at_slot(blockIdx.y == 0 ? c0 : (blockIdx.y == 1 ? c1 : c2), so);
    const unsigned mc1 = mf / 2 + 1, nc = nf / 2;
    const unsigned lat = mdiv(t, dn1), k = t - lat * (nc + 1);
    T v = T(0);
    if ((k > 0 || (fs & 1)) && (k < nc || (fs & 2))) {
        const unsigned row = mdiv(lat, dm1), j = lat - row * mc1;      // row = d (mc + 1) + i
        const unsigned d = mdiv(row, dm1), i = row - d * mc1;
        const unsigned fl = (d * (mf + 1) + 2 * i) * (mf + 1) + 2 * j;
        const bool five = ring_tri[fl * 6 + 5] < 0;
        const unsigned kb = k > 0 ? 2 * k - 1 : 0, kt = k < nc ? 2 * k + 1 : 2 * nc;
        const T wb = k > 0 ? T(0.5) : T(0), wt = k < nc ? T(0.5) : T(0);
        T p[7][3];
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            const T* q = f + (size_t)(r < 6 ? (unsigned)ring_nb[fl * 6 + r] : fl) * (nf + 1);
            p[r][0] = q[kb];
            p[r][1] = q[2 * k];
            p[r][2] = q[kt];
        }
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            const T s = p[r][1] + (wb * p[r][0] + wt * p[r][2]);
            v += r == 5 && five ? T(0) : s;
        }
        v = T(0.5) * v + (p[6][1] + (wb * p[6][0] + wt * p[6][2]));
    }
    c[t] = v;
}

// One Chebyshev step of the smoother on D^{-1} A, fused after y = A x:
//   d <- alpha d + beta D^{-1} (b - y),   x <- x + d,
// with (alpha, beta) = ab[2k], ab[2k + 1] (per slot: they scale with the
// slot's eigenvalue estimate).
constexpr int EW_PER = 4;   // elements per thread of the streaming elementwise kernels

template <typename T>
__global__ void __launch_bounds__(256) cheb_update_kernel(long long n, const double* __restrict__ ab, int k,
                                                          const T* __restrict__ b, const T* __restrict__ y,
                                                          const T* __restrict__ invd, T* d, T* x, SlotBatch sb) {
    const long long so = slot_off(sb);
    ab = at_slot(ab, so);
    b = at_slot(b, so);
    y = at_slot(y, so);
    invd = at_slot(invd, so);
    d = at_slot(d, so);
    x = at_slot(x, so);
    const T alpha = T(ab[2 * k]), beta = T(ab[2 * k + 1]);
    const long long t0 = (long long)blockIdx.x * (256 * EW_PER) + threadIdx.x;
    T bv[EW_PER], yv[EW_PER], iv[EW_PER], dv[EW_PER], xv[EW_PER];
#pragma unroll
    for (int e = 0; e < EW_PER; ++e) {
        const long long t = t0 + e * 256;
        const bool in = t < n;
        bv[e] = in ? b[t] : T(0);
        yv[e] = in ? y[t] : T(0);
        iv[e] = in ? invd[t] : T(0);
        dv[e] = in && alpha != T(0) ? d[t] : T(0);   // d may hold garbage on the first step
        xv[e] = in ? x[t] : T(0);
    }
#pragma unroll
    for (int e = 0; e < EW_PER; ++e) {
        const long long t = t0 + e * 256;
        if (t >= n) break;
        const T r = beta * iv[e] * (bv[e] - yv[e]);
        const T nd = alpha == T(0) ? r : alpha * dv[e] + r;
        d[t] = nd;
        x[t] = xv[e] + nd;
    }
}

// The same update with 16-byte vector accesses (every pointer 16-byte aligned):
// vector i of L = 16 / sizeof(T) values per thread, block 0 also the n % L tail;
// the arithmetic of every value is that of cheb_update_kernel.
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
    using type = float4;
};
template <>
struct Vec16<double> {
    using type = double2;
};

template <typename T>
__global__ void __launch_bounds__(256) cheb_update_vec_kernel(long long n, const double* __restrict__ ab, int k,
                                                              const T* __restrict__ b, const T* __restrict__ y,
                                                              const T* __restrict__ invd, T* d, T* x, SlotBatch sb) {
    using V = typename Vec16<T>::type;
    constexpr int L = 16 / sizeof(T);
    const long long so = slot_off(sb);
    ab = at_slot(ab, so);
    b = at_slot(b, so);
    y = at_slot(y, so);
    invd = at_slot(invd, so);
    d = at_slot(d, so);
    x = at_slot(x, so);
    const T alpha = T(ab[2 * k]), beta = T(ab[2 * k + 1]);
    const long long nv = n / L;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < nv) {
        V bv = reinterpret_cast<const V*>(b)[i], yv = reinterpret_cast<const V*>(y)[i];
        V iv = reinterpret_cast<const V*>(invd)[i], xv = reinterpret_cast<const V*>(x)[i];
        V dv{};
        if (alpha != T(0)) dv = reinterpret_cast<const V*>(d)[i];   // d may hold garbage on the first step
        const T* pb = reinterpret_cast<const T*>(&bv);
        const T* py = reinterpret_cast<const T*>(&yv);
        const T* pi = reinterpret_cast<const T*>(&iv);
        T* pd = reinterpret_cast<T*>(&dv);
        T* px = reinterpret_cast<T*>(&xv);
#pragma unroll
        for (int c = 0; c < L; ++c) {
            const T r = beta * pi[c] * (pb[c] - py[c]);
            pd[c] = alpha == T(0) ? r : alpha * pd[c] + r;
            px[c] += pd[c];
        }
        reinterpret_cast<V*>(d)[i] = dv;
        reinterpret_cast<V*>(x)[i] = xv;
    }
    if (blockIdx.x == 0 && threadIdx.x < n - nv * L) {
        const long long t = nv * L + threadIdx.x;
        const T r = beta * invd[t] * (b[t] - y[t]);
        const T dn = alpha == T(0) ? r : alpha * d[t] + r;
        d[t] = dn;
        x[t] += dn;
    }
}

// y <- a x + b y with 16-byte vector accesses (as axpby_kernel)
template <typename T>
__global__ void __launch_bounds__(256) axpby_vec_kernel(long long n, T a, const T* __restrict__ x, T b, T* y,
                                                        SlotBatch sb) {
    using V = typename Vec16<T>::type;
    constexpr int L = 16 / sizeof(T);
    const long long so = slot_off(sb);
    x = at_slot(x, so);
    y = at_slot(y, so);
    const long long nv = n / L;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < nv) {
        V xv = reinterpret_cast<const V*>(x)[i];
        V yv{};
        if (b != T(0)) yv = reinterpret_cast<const V*>(y)[i];
        const T* px = reinterpret_cast<const T*>(&xv);
        T* py = reinterpret_cast<T*>(&yv);
#pragma unroll
        for (int c = 0; c < L; ++c) py[c] = b == T(0) ? a * px[c] : a * px[c] + b * py[c];
        reinterpret_cast<V*>(y)[i] = yv;
    }
    if (blockIdx.x == 0 && threadIdx.x < n - nv * L) {
        const long long t = nv * L + threadIdx.x;
        y[t] = b == T(0) ? a * x[t] : a * x[t] + b * y[t];
    }
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <typename T>
__global__ void invert_kernel(long long n, T* a) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) a[t] = T(1) / a[t];
}

// Free-slip boundary rows of an iterate: x <- P x + N b = x + (rhat.b - rhat.x) rhat at
// the layers of the free-slip spheres (fs bit 0 inner, bit 1 outer), b == nullptr: b = 0.
// The normal rows of P A P + N are identity rows, so this solves them exactly and leaves
// the tangential part to the smoother.
template <typename T>
__global__ void fs_project_kernel(long long ncol, int n, int fs, const T* __restrict__ unit, T* x0, T* x1, T* x2,
                                  const T* __restrict__ b0, const T* __restrict__ b1, const T* __restrict__ b2) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * ncol) return;
    if (!((t & 1) ? (fs & 2) : (fs & 1))) return;
    const long long col = t >> 1;
    const long long idx = col * (n + 1) + ((t & 1) ? n : 0);
    const T r0 = unit[3 * col], r1 = unit[3 * col + 1], r2 = unit[3 * col + 2];
    const T dx = r0 * x0[idx] + r1 * x1[idx] + r2 * x2[idx];
    const T db = b0 ? r0 * b0[idx] + r1 * b1[idx] + r2 * b2[idx] : T(0);
    x0[idx] += (db - dx) * r0;
    x1[idx] += (db - dx) * r1;
    x2[idx] += (db - dx) * r2;
}

// Rigid rotation e_a x x of the shell's nodes (x = r_k rhat), component c at every
// node slot: a null vector of the viscous block with free slip on both spheres.
template <typename T>
__global__ void rotation_fill_kernel(int m, int n, double r_in, double dr, const double* __restrict__ unit, int a,
                                     T* o0, T* o1, T* o2, long long nslots) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nslots) return;
    const long long lat = t / (n + 1);
    const double r = r_in + (double)(t % (n + 1)) * dr;
    const double x = r * unit[3 * lat], y = r * unit[3 * lat + 1], z = r * unit[3 * lat + 2];
    const double v0 = a == 0 ? 0.0 : (a == 1 ? z : -y);
    const double v1 = a == 0 ? -z : (a == 1 ? 0.0 : x);
    const double v2 = a == 0 ? y : (a == 1 ? -x : 0.0);
    o0[t] = T(v0);
    o1[t] = T(v1);
    o2[t] = T(v2);
}

// The coarsest matrix with free slip on both spheres is singular (the three rigid
// rotations).  q: the rotations over the coarse DoFs, orthonormalised (Gram-Schmidt in
// DoF order), and sigma the mean diagonal entry; one thread.
__global__ void coarse_rotation_basis_kernel(int nd, const int* __restrict__ dof_slot, int m, int n, double r_in,
                                             double dr, const double* __restrict__ unit,
                                             const double* __restrict__ Ad, double* q) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    for (int a = 0; a < 3; ++a) {
        double* qa = q + (long long)a * nd;
        for (int d = 0; d < nd; ++d) {
            const long long slot = dof_slot[d] >> 2;
            const int c = dof_slot[d] & 3;
            const long long lat = slot / (n + 1);
            const double r = r_in + (double)(slot % (n + 1)) * dr;
            const double x[3] = {r * unit[3 * lat], r * unit[3 * lat + 1], r * unit[3 * lat + 2]};
            // (e_a x x)_c = eps_{c a b} x_b
            const int b = 3 - a - c;
            qa[d] = a == c ? 0.0 : (((a - c + 3) % 3 == 1) ? x[b] : -x[b]);
        }
        for (int b2 = 0; b2 < a; ++b2) {
            const double* qb = q + (long long)b2 * nd;
            double dt = 0.0;
            for (int d = 0; d < nd; ++d) dt += qa[d] * qb[d];
            for (int d = 0; d < nd; ++d) qa[d] -= dt * qb[d];
        }
        double nn = 0.0;
        for (int d = 0; d < nd; ++d) nn += qa[d] * qa[d];
        const double inv = 1.0 / sqrt(nn);
        for (int d = 0; d < nd; ++d) qa[d] *= inv;
    }
    double tr = 0.0;
    for (int d = 0; d < nd; ++d) tr += Ad[(long long)d * nd + d];
    q[3LL * nd] = tr / nd;
}

// A <- A + sigma sum_a q_a q_a^T: the rotations get eigenvalue sigma, the rest of the
// spectrum is unchanged (the q_a span the null space), so for a right-hand side
// orthogonal to them the inverse gives the solution orthogonal to them.
__global__ void coarse_rotation_shift_kernel(int nd, const double* __restrict__ q, double* Ad) {
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= nd) return;
    const double sigma = q[3LL * nd];
    const double c0 = q[col], c1 = q[nd + col], c2 = q[2LL * nd + col];
    for (int r = 0; r < nd; ++r)
        Ad[(long long)col * nd + r] += sigma * (c0 * q[r] + c1 * q[nd + r] + c2 * q[2LL * nd + r]);
}

template <typename TO, typename TI>
__global__ void cast_kernel(long long n, const TI* __restrict__ a, TO* __restrict__ b, SlotBatch sb) {
    const long long so = slot_off(sb);
    a = at_slot(a, so);
    b = at_slot(b, so);
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) b[t] = TO(a[t]);
}

// y <- a x + b y  (x may alias nothing; pass b = 0 to overwrite)
template <typename T>
__global__ void __launch_bounds__(256) axpby_kernel(long long n, T a, const T* __restrict__ x, T b, T* y,
                                                    SlotBatch sb) {
    const long long so = slot_off(sb);
    x = at_slot(x, so);
    y = at_slot(y, so);
    const long long t0 = (long long)blockIdx.x * (256 * EW_PER) + threadIdx.x;
    T xv[EW_PER], yv[EW_PER];
#pragma unroll
    for (int e = 0; e < EW_PER; ++e) {
        const long long t = t0 + e * 256;
        xv[e] = t < n ? x[t] : T(0);
        yv[e] = t < n && b != T(0) ? y[t] : T(0);
    }
#pragma unroll
    for (int e = 0; e < EW_PER; ++e) {
        const long long t = t0 + e * 256;
        if (t >= n) break;
        y[t] = b == T(0) ? a * xv[e] : a * xv[e] + b * yv[e];
    }
}

// Multi-dot partials: for every vector v_q (q < nq <= NQ) the block sum of
// mask(slot) x v_q over one grid-stride share; a second kernel adds the block
// sums in a fixed order, so the result does not depend on timing.  Node slot
// t lies in radial column t / n1 (division by a magic multiplier, exact for
// all 32-bit t); the owner mask counts every unique node once.  The vector
// pointers are read once per block into scalar registers, and every load of
// an element is issued before the first use.
constexpr int DOT_BS = 256;

// Residual r = b - A_D x from a raw viscous apply y (the closing pass fused as in
// cheb_post_update_kernel: copies summed in group order, identity rows r = b - x); MUL: the
// step r = b A_D x of the power iteration, b the inverse diagonal.
template <typename T, bool MUL>
__global__ void __launch_bounds__(256) resid_post_kernel(int ns, int n1, MagicDiv dn1, const int* __restrict__ lat_grp,
                                                        const int* __restrict__ gp, const int* __restrict__ gs,
                                                        int ns_in, int ns_out, const T* __restrict__ b,
                                                        const T* __restrict__ x, const T* y, T* r, SlotBatch sb) {
    const long long so = slot_off(sb);
    const unsigned t = blockIdx.x * 256u + threadIdx.x;
    if (t >= (unsigned)ns) return;
    const long long e = (long long)blockIdx.y * ns + t;
    const unsigned lat = mdiv(t, dn1);
    const int kk = (int)(t - lat * (unsigned)n1);
    T yv;
    if ((ns_in && kk == 0) || (ns_out && kk == n1 - 1)) {
        yv = at_slot(x, so)[e];
    } else {
        const int g = lat_grp[lat];
        const T* yy = at_slot(y, so) + (long long)blockIdx.y * ns;
        if (g < 0) {
            yv = yy[t];
        } else {
            const int s0 = gp[g], s1 = gp[g + 1];
            yv = yy[(long long)gs[s0] * n1 + kk];
            for (int q = s0 + 1; q < s1; ++q) yv += yy[(long long)gs[q] * n1 + kk];
        }
    }
    const T bv = at_slot(b, so)[e];
    at_slot(r, so)[e] = MUL ? bv * yv : bv - yv;
}

// One Chebyshev step of the smoother in its two-term form
//   x_k+1 = x_k + alpha (x_k - x_k-1) + beta D^-1 (b - A_D x_k)
// (the form with the direction d_k = x_k+1 - x_k needs one more vector per step),
// fused with the closing pass of the raw viscous apply before it (y = A_D x_k with
// each diamond's partial sums on duplicated nodes and nothing on the no-slip rows):
// per node, the completed A_D x_k is the sum of the node's copies in group order
// (the interface pass's order), or x_k itself on an identity row.  xo holds x_k-1
// on entry (read when alpha != 0 and not prev_zero; x_k-1 = 0 otherwise) and x_k+1
// on return, element by element in place.  first: the step from x_k = 0
// (y and x_k are not read).  Each thread takes one 16-byte vector of the flat
// [3][node slots] arrays (16-byte aligned; the tail of fewer than one vector is the
// first block's) and locates its elements' node (component, lateral slot, layer)
// incrementally.
template <typename T>
__global__ void __launch_bounds__(256) cheb_post_update_kernel(unsigned ns, int n1, MagicDiv dns, MagicDiv dn1,
                                                              const int* __restrict__ lat_grp,
                                                              const int* __restrict__ gp, const int* __restrict__ gs,
                                                              int ns_in, int ns_out, const double* __restrict__ ab,
                                                              int k, int first, int prev_zero,
                                                              const T* __restrict__ b, const T* __restrict__ y,
                                                              const T* __restrict__ invd, const T* __restrict__ xk,
                                                              T* xo, SlotBatch sb) {
    using V = typename Vec16<T>::type;
    constexpr int L = 16 / sizeof(T);
    const long long so = slot_off(sb);
    ab = at_slot(ab, so);
    b = at_slot(b, so);
    y = at_slot(y, so);
    invd = at_slot(invd, so);
    xk = at_slot(xk, so);
    xo = at_slot(xo, so);
    const T alpha = T(ab[2 * k]), beta = T(ab[2 * k + 1]);
    const bool use_prev = alpha != T(0) && !prev_zero;
    const unsigned n = 3u * ns, nv = n / L;
    const unsigned v = blockIdx.x * 256u + threadIdx.x;
    // completed A_D x_k at element e (component c, lateral slot lat, layer kk)
    auto yat = [&](unsigned c, unsigned lat, int kk, T yraw, T xv) -> T {
        if ((ns_in && kk == 0) || (ns_out && kk == n1 - 1)) return xv;
        const int g = lat_grp[lat];
        if (g < 0) return yraw;
        const T* yy = y + (size_t)c * ns;
        const int s0 = gp[g], s1 = gp[g + 1];
        T acc = yy[(size_t)gs[s0] * n1 + kk];
        for (int q = s0 + 1; q < s1; ++q) acc += yy[(size_t)gs[q] * n1 + kk];
        return acc;
    };
    auto step = [&](T bq, T iq, T yq, T xq, T pq) -> T {
        const T r = beta * iq * (bq - yq);
        return use_prev ? xq + (alpha * (xq - pq) + r) : (alpha == T(0) ? xq + r : xq + (alpha * xq + r));
    };
    if (v < nv) {
        const V bv = reinterpret_cast<const V*>(b)[v], iv = reinterpret_cast<const V*>(invd)[v];
        const T* pb = reinterpret_cast<const T*>(&bv);
        const T* pi = reinterpret_cast<const T*>(&iv);
        V ov{};
        T* po = reinterpret_cast<T*>(&ov);
        if (first) {
#pragma unroll
            for (int q = 0; q < L; ++q) po[q] = beta * pi[q] * (pb[q] - T(0));
        } else {
            const V yv = reinterpret_cast<const V*>(y)[v], xv = reinterpret_cast<const V*>(xk)[v];
            V pv{};
            if (use_prev) pv = reinterpret_cast<const V*>(xo)[v];
            const T* py = reinterpret_cast<const T*>(&yv);
            const T* px = reinterpret_cast<const T*>(&xv);
            const T* pp = reinterpret_cast<const T*>(&pv);
            const unsigned e0 = v * L;
            unsigned c = mdiv(e0, dns);
            unsigned t = e0 - c * ns;
            unsigned lat = mdiv(t, dn1);
            int kk = (int)(t - lat * (unsigned)n1);
#pragma unroll
            for (int q = 0; q < L; ++q) {
                po[q] = step(pb[q], pi[q], yat(c, lat, kk, py[q], px[q]), px[q], pp[q]);
                // next element: the next layer, column or component
                if (++kk == n1) {
                    kk = 0;
                    if (++t == ns) {
                        t = 0;
                        ++c;
                        lat = 0;
                    } else {
                        ++lat;
                    }
                } else {
                    ++t;
                }
            }
        }
        reinterpret_cast<V*>(xo)[v] = ov;
    }
    if (blockIdx.x == 0 && threadIdx.x < n - nv * L) {
        const unsigned e = nv * L + threadIdx.x;
        if (first) {
            xo[e] = beta * invd[e] * (b[e] - T(0));
        } else {
            const unsigned c = mdiv(e, dns), t = e - c * ns, lat = mdiv(t, dn1);
            const int kk = (int)(t - lat * (unsigned)n1);
            const T xe = xk[e];
            xo[e] = step(b[e], invd[e], yat(c, lat, kk, y[e], xe), xe, use_prev ? xo[e] : T(0));
        }
    }
}

// A pointer read from a table lost its address space; loads through this
// global-memory pointer type are global, not flat, instructions.
template <class T>
using gptr = const __attribute__((address_space(1))) T*;
template <class T>
__device__ __forceinline__ gptr<T> as_global(const T* p) {
    return (gptr<T>)p;
}

// Block sums of acc[q], q < nq, to part[q][blockIdx.x] (fixed order).
template <int NQ>
__device__ __forceinline__ void block_partials(const double (&acc)[NQ], int nq, double* __restrict__ part) {
    __shared__ double sh[DOT_BS / 64][NQ];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q >= nq) break;
        double v = acc[q];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) sh[wv][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < nq) {
        double v = 0.0;
        for (int w = 0; w < DOT_BS / 64; ++w) v += sh[w][threadIdx.x];
        part[(long long)threadIdx.x * DOT_BLOCKS + blockIdx.x] = v;
    }
}

// n slots of up to three node-field components of one level (n1 layers per
// column, nlat lateral slots per component).
template <typename T, int NQ>
__global__ void __launch_bounds__(DOT_BS) mdot_partial_kernel(unsigned n, MagicDiv dn1, unsigned nlat,
                                                              const uint8_t* __restrict__ owner,
                                                              const T* __restrict__ x, const T* const* __restrict__ vs,
                                                              int nq, double* __restrict__ part, SlotBatch sb) {
    const long long so = slot_off(sb);
    x = at_slot(x, so);
    vs = at_slot(vs, so);
    part = at_slot(part, so);
    nq = slot_count(sb, nq);
    gptr<T> vp[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) vp[q] = as_global(vs[q < nq ? q : 0]);
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    // two elements per step, every load (mask and data) issued before the first use
    const unsigned stride = gridDim.x * DOT_BS;
    for (unsigned t0 = blockIdx.x * DOT_BS + threadIdx.x; t0 < n; t0 += 2 * stride) {
        T xv[2], v[2][NQ];
        bool own[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned t = t0 + e * stride;
            const bool in = t < n;
            const unsigned tt = in ? t : 0;
            unsigned lat = mdiv(tt, dn1);
            lat = lat >= nlat ? lat - nlat : lat;
            lat = lat >= nlat ? lat - nlat : lat;
            own[e] = in && owner[lat];
            xv[e] = x[tt];
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[e][q] = q < nq ? vp[q][tt] : T(0);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (!own[e]) continue;
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q] += (double)xv[e] * (double)v[e][q];
        }
    }
    block_partials<NQ>(acc, nq, part);
}

// y <- y + sign * sum_q coef[q] v_q (q < nq <= NQ), coefficients read from
// device memory; pointers and coefficients in scalar registers, all loads of
// an element in flight together.
template <typename T, int NQ>
__global__ void __launch_bounds__(256) maxpy_kernel(unsigned n, const double* __restrict__ coef, double sign,
                                                    const T* const* __restrict__ vs, int nq, T* y, SlotBatch sb) {
    const long long so = slot_off(sb);
    coef = at_slot(coef, so);
    vs = at_slot(vs, so);
    y = at_slot(y, so);
    nq = slot_count(sb, nq);
    gptr<T> vp[NQ];
    double cf[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        vp[q] = as_global(vs[q < nq ? q : 0]);
        cf[q] = q < nq ? sign * coef[q] : 0.0;
    }
    const unsigned stride = gridDim.x * blockDim.x;
    for (unsigned t0 = blockIdx.x * blockDim.x + threadIdx.x; t0 < n; t0 += 2 * stride) {
        T v[2][NQ], yv[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned t = t0 + e * stride;
            const unsigned tt = t < n ? t : 0;
            yv[e] = y[tt];
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[e][q] = q < nq ? vp[q][tt] : T(0);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned t = t0 + e * stride;
            if (t >= n) break;
            double acc = (double)yv[e];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (q < nq) acc += cf[q] * (double)v[e][q];
            y[t] = T(acc);
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(256) copy3_kernel(unsigned n, const T* a0, const T* a1, const T* a2, T* o0, T* o1,
                                                    T* o2) {
    const T* a = blockIdx.y == 0 ? a0 : (blockIdx.y == 1 ? a1 : a2);
    T* o = blockIdx.y == 0 ? o0 : (blockIdx.y == 1 ? o1 : o2);
    for (unsigned t = blockIdx.x * 256u + threadIdx.x; t < n; t += gridDim.x * 256u) o[t] = a[t];
}

template <typename T>
__global__ void mul_kernel(unsigned n, const T* __restrict__ a, const T* __restrict__ b, T* c) {
    for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) c[t] = a[t] * b[t];
}

template <typename T>
__global__ void fillv_kernel(unsigned n, T v, T* a, SlotBatch sb) {
    a = at_slot(a, slot_off(sb));
    for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) a[t] = v;
}

// out[q] = sum of the block partials of vector q = blockIdx.x: every thread a fixed strided
// share of the contiguous partials, then a fixed shuffle tree and the waves in order; the
// order depends only on nblocks.  One workgroup per vector and coalesced reads (a single
// workgroup gathering strided partials took 12.8 us for 4096 blocks).
__global__ void __launch_bounds__(256) mdot_final_kernel(int nblocks, int nq, const double* __restrict__ part,
                                                         double* out, int accumulate, SlotBatch sb) {
    const long long so = slot_off(sb);
    part = at_slot(part, so);
    out = at_slot(out, so);
    const int q = blockIdx.x;
    if (q >= slot_count(sb, nq)) return;
    part += (size_t)q * DOT_BLOCKS;
    double v = 0.0;
#pragma unroll
    for (int u = 0; u < DOT_BLOCKS / 256; ++u) {
        const int b = threadIdx.x + 256 * u;
        v += b < nblocks ? part[b] : 0.0;
    }
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    __shared__ double sh[4];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        v = (sh[0] + sh[1]) + (sh[2] + sh[3]);
        out[q] = accumulate ? out[q] + v : v;
    }
}

// Dense coarsest level ------------------------------------------------------

// One step of the blocked Gauss-Jordan inversion of an SPD matrix (no pivoting is needed):
// with P the pivot block of INV_NB rows and columns and D = A_PP^{-1},
//   A_PP <- D, A_Pj <- D A_Pj, A_iP <- -A_iP D, A_ij <- A_ij - A_iP D A_Pj.
// Workgroup (bi, bj) writes block (i, j) of `out` from `in` (two buffers, so that no
// workgroup waits for another) and inverts A_PP itself, in LDS.  Bound by the latency of
// the INV_NB pivots of that inversion (the products are 32^3): one launch per pivot block
// instead of one workgroup walking the whole matrix once per pivot (126 unknowns: four
// launches of 24 us, 0.68 ms before).
__global__ void __launch_bounds__(256) invert_step_kernel(int nd, int pb, const double* __restrict__ in,
                                                          double* __restrict__ out) {
    static_assert(INV_NB == 32, "256 threads hold a 32 x 32 block, four rows each");
    __shared__ double D[INV_NB][INV_NB + 1], L[INV_NB][INV_NB + 1], R[INV_NB][INV_NB + 1];
    __shared__ double prow[2][INV_NB], pcol[2][INV_NB];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int p0 = pb * INV_NB, i0 = blockIdx.y * INV_NB, j0 = blockIdx.x * INV_NB;
    // rows and columns past the matrix: identity in the pivot block, zero elsewhere
    auto at = [&](int r, int c, double pad) {
        return r < nd && c < nd ? in[(size_t)r * nd + c] : pad;
    };
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = ty + 8 * q;
        v[q] = at(p0 + r, p0 + tx, r == tx ? 1.0 : 0.0);
        L[r][tx] = at(i0 + r, p0 + tx, 0.0);
        R[r][tx] = at(p0 + r, j0 + tx, 0.0);
        if (r == 0) prow[0][tx] = v[q];
        if (tx == 0) pcol[0][r] = v[q];
    }
    // scalar Gauss-Jordan on the pivot block held in registers (row ty + 8 q, column tx);
    // the next pivot's row and column are handed on through LDS, one barrier per pivot
    for (int p = 0; p < INV_NB; ++p) {
        __syncthreads();
        const double* pr = prow[p & 1];
        const double* pc = pcol[p & 1];
        const double ip = 1.0 / pr[p], prx = pr[tx];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = ty + 8 * q;
            const double f = pc[r] * ip;
            if (r == p)
                v[q] = tx == p ? ip : prx * ip;
            else
                v[q] = tx == p ? -f : v[q] - f * prx;
            if (r == p + 1) prow[(p + 1) & 1][tx] = v[q];
            if (tx == p + 1) pcol[(p + 1) & 1][r] = v[q];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) D[ty + 8 * q][tx] = v[q];
    __syncthreads();
    const bool pi = i0 == p0, pj = j0 == p0;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    if (pi && pj) {
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] = v[q];
    } else if (pj) {
        for (int k = 0; k < INV_NB; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] -= L[ty + 8 * q][k] * D[k][tx];
    } else {
        for (int k = 0; k < INV_NB; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] += D[ty + 8 * q][k] * R[k][tx];
        if (!pi) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 4; ++q) R[ty + 8 * q][tx] = t[q];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] = at(i0 + ty + 8 * q, j0 + tx, 0.0);
            for (int k = 0; k < INV_NB; ++k)
#pragma unroll
                for (int q = 0; q < 4; ++q) t[q] -= L[ty + 8 * q][k] * R[k][tx];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = i0 + ty + 8 * q, c = j0 + tx;
        if (r < nd && c < nd) out[(size_t)r * nd + c] = t[q];
    }
}

// x = A^{-1} b on the coarsest level: gather b at owner slots of interior
// DoFs, dense symmetric matvec, scatter to every copy; other rows set to zero
// (their right-hand side is zero in a V-cycle: Dirichlet rows).
template <typename T>
__global__ void __launch_bounds__(1024) coarse_solve_kernel(int nd, const int* __restrict__ dof_slot,
                                                            const int* __restrict__ slot_dof, long long nslots,
                                                            const double* __restrict__ Ainv,
                                                            const T* __restrict__ b0, const T* __restrict__ b1,
                                                            const T* __restrict__ b2, T* x0, T* x1, T* x2,
                                                            SlotBatch sb) {
    const long long so = slot_off(sb);
    dof_slot = at_slot(dof_slot, so);
    slot_dof = at_slot(slot_dof, so);
    Ainv = at_slot(Ainv, so);
    b0 = at_slot(b0, so);
    b1 = at_slot(b1, so);
    b2 = at_slot(b2, so);
    x0 = at_slot(x0, so);
    x1 = at_slot(x1, so);
    x2 = at_slot(x2, so);
    // the columns are split among the G groups of nd threads that the workgroup holds, their
    // sums added in group order (126 unknowns, eight groups: 13 -> 6.7 us a solve)
    __shared__ double rhs[MAX_COARSE_DOF];
    __shared__ double sol[MAX_COARSE_DOF];      // [G][nd], G nd <= 1024
    for (int r = threadIdx.x; r < nd; r += blockDim.x) {
        const int s = dof_slot[r];
        const int c = s & 3;
        const long long slot = s >> 2;
        rhs[r] = (double)(c == 0 ? b0[slot] : (c == 1 ? b1[slot] : b2[slot]));
    }
    __syncthreads();
    const int G = (int)blockDim.x / nd, grp = (int)threadIdx.x / nd, row = (int)threadIdx.x % nd;
    if (grp < G) {
        const int c0 = nd * grp / G, c1 = nd * (grp + 1) / G;
        double v = 0.0;
#pragma unroll 8
        for (int c = c0; c < c1; ++c) v += Ainv[(long long)c * nd + row] * rhs[c];
        sol[grp * nd + row] = v;
    }
    __syncthreads();
    double sum = 0.0;
    if ((int)threadIdx.x < nd)
        for (int g = 0; g < G; ++g) sum += sol[g * nd + threadIdx.x];
    __syncthreads();
    if ((int)threadIdx.x < nd) sol[threadIdx.x] = sum;
    __syncthreads();
    for (long long t = threadIdx.x; t < 3 * nslots; t += blockDim.x) {
        const int c = (int)(t / nslots);
        const long long slot = t % nslots;
        const int dof = slot_dof[c * nslots + slot];
        const T v = dof >= 0 ? T(sol[dof]) : T(0);
        if (c == 0) x0[slot] = v;
        else if (c == 1) x1[slot] = v;
        else x2[slot] = v;
    }
}

// Pressure: zero nodal mean projection helper  p <- p - mean
template <typename T>
__global__ void shift_kernel(long long n, const double* __restrict__ sum_cnt, T* p, SlotBatch sb) {
    const long long so = slot_off(sb);
    sum_cnt = at_slot(sum_cnt, so);
    p = at_slot(p, so);
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] -= T(sum_cnt[0] / sum_cnt[1]);
}

// Schur preconditioner on the pressure: z = -r / m (Sec. 7, eq:pmass)
template <typename T>
__global__ void schur_diag_kernel(long long n, const T* __restrict__ r, const T* __restrict__ mdiag, T* z,
                                  SlotBatch sb) {
    const long long so = slot_off(sb);
    r = at_slot(r, so);
    mdiag = at_slot(mdiag, so);
    z = at_slot(z, so);
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) z[t] = -r[t] / mdiag[t];
}

// Multi-dot over a Stokes vector [u0 u1 u2 p] (velocity slots of one level
// followed by its pressure slots): owner masks of both grids.
template <typename T, int NQ>
__global__ void __launch_bounds__(DOT_BS) smdot_partial_kernel(unsigned ns, MagicDiv dn1u, unsigned nlat_u,
                                                               const uint8_t* __restrict__ ou, unsigned np,
                                                               MagicDiv dn1p, const uint8_t* __restrict__ op,
                                                               const T* __restrict__ x,
                                                               const T* const* __restrict__ vs, int nq,
                                                               double* __restrict__ part, SlotBatch sb) {
    const long long so = slot_off(sb);
    x = at_slot(x, so);
    vs = at_slot(vs, so);
    part = at_slot(part, so);
    nq = slot_count(sb, nq);
    gptr<T> vp[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) vp[q] = as_global(vs[q < nq ? q : 0]);
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    const unsigned nu = 3u * ns, n = nu + np;
    // two elements per step, every load (mask and data) issued before the first use
    const unsigned stride = gridDim.x * DOT_BS;
    for (unsigned t0 = blockIdx.x * DOT_BS + threadIdx.x; t0 < n; t0 += 2 * stride) {
        T xv[2], v[2][NQ];
        bool own[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned t = t0 + e * stride;
            const bool in = t < n;
            const unsigned tt = in ? t : 0;
            if (tt < nu) {
                unsigned lat = mdiv(tt, dn1u);
                lat = lat >= nlat_u ? lat - nlat_u : lat;
                lat = lat >= nlat_u ? lat - nlat_u : lat;
                own[e] = in && ou[lat];
            } else {
                own[e] = in && op[mdiv(tt - nu, dn1p)];
            }
            xv[e] = x[tt];
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[e][q] = q < nq ? vp[q][tt] : T(0);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (!own[e]) continue;
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q] += (double)xv[e] * (double)v[e][q];
        }
    }
    block_partials<NQ>(acc, nq, part);
}

// Gram-Schmidt step fused with the dots that follow it, over a Stokes vector:
//   y <- y - sum_q c_q v_q   (every slot, as maxpy_kernel),
// then, over owned slots, the dots of the new y with the same v_q (NORM false:
// the re-orthogonalisation coefficients) or with itself (NORM true: the
// squared norm), from the stored (rounded) value of y; block partials as in
// smdot_partial_kernel.  One pass instead of a multi-axpy and a multi-dot.
template <typename T, int NQ, bool NORM>
__global__ void __launch_bounds__(DOT_BS) maxpy_dot_kernel(unsigned ns, MagicDiv dn1u, unsigned nlat_u,
                                                           const uint8_t* __restrict__ ou, unsigned np,
                                                           MagicDiv dn1p, const uint8_t* __restrict__ op,
                                                           const double* __restrict__ coef, double sign,
                                                           const T* const* __restrict__ vs, int nq, T* y,
                                                           double* __restrict__ part, SlotBatch sb) {
    const long long so = slot_off(sb);
    coef = at_slot(coef, so);
    vs = at_slot(vs, so);
    y = at_slot(y, so);
    part = at_slot(part, so);
    nq = slot_count(sb, nq);
    gptr<T> vp[NQ];
    double cf[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        vp[q] = as_global(vs[q < nq ? q : 0]);
        cf[q] = q < nq ? sign * coef[q] : 0.0;
    }
    constexpr int NA = NORM ? 1 : NQ;
    double acc[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[q] = 0.0;
    const unsigned nu = 3u * ns, n = nu + np;
    const unsigned stride = gridDim.x * DOT_BS;
    for (unsigned t0 = blockIdx.x * DOT_BS + threadIdx.x; t0 < n; t0 += 2 * stride) {
        T yv[2], v[2][NQ];
        bool own[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned t = t0 + e * stride;
            const bool in = t < n;
            const unsigned tt = in ? t : 0;
            if (tt < nu) {
                unsigned lat = mdiv(tt, dn1u);
                lat = lat >= nlat_u ? lat - nlat_u : lat;
                lat = lat >= nlat_u ? lat - nlat_u : lat;
                own[e] = in && ou[lat];
            } else {
                own[e] = in && op[mdiv(tt - nu, dn1p)];
            }
            yv[e] = y[tt];
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[e][q] = q < nq ? vp[q][tt] : T(0);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned t = t0 + e * stride;
            if (t >= n) break;
            double a = (double)yv[e];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (q < nq) a += cf[q] * (double)v[e][q];
            const T yn = T(a);
            y[t] = yn;
            if (!own[e]) continue;
            if (NORM) {
                acc[0] += (double)yn * (double)yn;
            } else {
#pragma unroll
                for (int q = 0; q < NA; ++q) acc[q] += (double)v[e][q] * (double)yn;
            }
        }
    }
    block_partials<NA>(acc, NORM ? 1 : nq, part);
}

// 16 bytes of T values as a native vector (it loads out of the global address space
// as one 16-byte access)
template <typename T>
struct Pack16 {
    typedef T type __attribute__((ext_vector_type(16 / sizeof(T))));
};

template <typename T>
__device__ __forceinline__ bool stokes_owned(unsigned t, unsigned nu, MagicDiv dn1u, unsigned nlat_u,
                                             const uint8_t* __restrict__ ou, MagicDiv dn1p,
                                             const uint8_t* __restrict__ op) {
    if (t < nu) {
        unsigned lat = mdiv(t, dn1u);
        lat = lat >= nlat_u ? lat - nlat_u : lat;
        lat = lat >= nlat_u ? lat - nlat_u : lat;
        return ou[lat] != 0;
    }
    return op[mdiv(t - nu, dn1p)] != 0;
}

// smdot_partial_kernel and maxpy_dot_kernel with 16-byte accesses, for vectors that are all
// 16-byte aligned (the Krylov basis, also in the slots of a batch): a thread takes
// L = 16 / sizeof(T) consecutive values of every vector per load, block 0 also the n % L
// tail.  Same arithmetic per value (FP64 products and sums); the owner mask of every value.
template <typename T, int NQ>
__global__ void __launch_bounds__(DOT_BS) smdot_vec_kernel(unsigned ns, MagicDiv dn1u, unsigned nlat_u,
                                                           const uint8_t* __restrict__ ou, unsigned np,
                                                           MagicDiv dn1p, const uint8_t* __restrict__ op,
                                                           const T* __restrict__ x,
                                                           const T* const* __restrict__ vs, int nq,
                                                           double* __restrict__ part, SlotBatch sb) {
    using V = typename Pack16<T>::type;
    constexpr int L = 16 / sizeof(T);
    using gvptr = const __attribute__((address_space(1))) V*;
    const long long so = slot_off(sb);
    x = at_slot(x, so);
    vs = at_slot(vs, so);
    part = at_slot(part, so);
    nq = slot_count(sb, nq);
    gvptr vp[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) vp[q] = (gvptr)vs[q < nq ? q : 0];
    const gvptr xp = (gvptr)x;
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    const unsigned nu = 3u * ns, n = nu + np, nv = n / L;
    const unsigned stride = gridDim.x * DOT_BS;
    for (unsigned c = blockIdx.x * DOT_BS + threadIdx.x; c < nv; c += stride) {
        const V xv = xp[c];
        V v[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = vp[q < nq ? q : 0][c];
        const V px = xv;
#pragma unroll
        for (int e = 0; e < L; ++e) {
            if (!stokes_owned<T>(c * L + e, nu, dn1u, nlat_u, ou, dn1p, op)) continue;
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q] += (double)px[e] * (double)v[q][e];
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < n - nv * L) {
        const unsigned t = nv * L + threadIdx.x;
        if (stokes_owned<T>(t, nu, dn1u, nlat_u, ou, dn1p, op)) {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (q < nq) acc[q] += (double)x[t] * (double)vs[q][t];
        }
    }
    block_partials<NQ>(acc, nq, part);
}

template <typename T, int NQ, bool NORM>
__global__ void __launch_bounds__(DOT_BS) maxpy_dot_vec_kernel(unsigned ns, MagicDiv dn1u, unsigned nlat_u,
                                                               const uint8_t* __restrict__ ou, unsigned np,
                                                               MagicDiv dn1p, const uint8_t* __restrict__ op,
                                                               const double* __restrict__ coef, double sign,
                                                               const T* const* __restrict__ vs, int nq, T* y,
                                                               double* __restrict__ part, SlotBatch sb) {
    using V = typename Pack16<T>::type;
    constexpr int L = 16 / sizeof(T);
    using gvptr = const __attribute__((address_space(1))) V*;
    const long long so = slot_off(sb);
    coef = at_slot(coef, so);
    vs = at_slot(vs, so);
    y = at_slot(y, so);
    part = at_slot(part, so);
    nq = slot_count(sb, nq);
    gvptr vp[NQ];
    double cf[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        vp[q] = (gvptr)vs[q < nq ? q : 0];
        cf[q] = q < nq ? sign * coef[q] : 0.0;
    }
    constexpr int NA = NORM ? 1 : NQ;
    double acc[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[q] = 0.0;
    const unsigned nu = 3u * ns, n = nu + np, nv = n / L;
    const unsigned stride = gridDim.x * DOT_BS;
    V* yv = reinterpret_cast<V*>(y);
    for (unsigned c = blockIdx.x * DOT_BS + threadIdx.x; c < nv; c += stride) {
        V w = yv[c];
        V v[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = vp[q < nq ? q : 0][c];
        #pragma unroll
        for (int e = 0; e < L; ++e) {
            double a2 = (double)w[e];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (q < nq) a2 += cf[q] * (double)v[q][e];
            w[e] = T(a2);
        }
        yv[c] = w;
#pragma unroll
        for (int e = 0; e < L; ++e) {
            if (!stokes_owned<T>(c * L + e, nu, dn1u, nlat_u, ou, dn1p, op)) continue;
            const double yn = (double)w[e];
            if (NORM) {
                acc[0] += yn * yn;
            } else {
#pragma unroll
                for (int q = 0; q < NA; ++q) acc[q] += (double)v[q][e] * yn;
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < n - nv * L) {
        const unsigned t = nv * L + threadIdx.x;
        double a2 = (double)y[t];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (q < nq) a2 += cf[q] * (double)vs[q][t];
        const T yn = T(a2);
        y[t] = yn;
        if (stokes_owned<T>(t, nu, dn1u, nlat_u, ou, dn1p, op)) {
            if (NORM) {
                acc[0] += (double)yn * (double)yn;
            } else {
#pragma unroll
                for (int q = 0; q < NA; ++q)
                    if (q < nq) acc[q] += (double)vs[q][t] * (double)yn;
            }
        }
    }
    block_partials<NA>(acc, NORM ? 1 : nq, part);
}

// Counter-based uniform numbers in [-1, 1) (splitmix64 of seed and index).
template <typename T>
__global__ void rand_kernel(unsigned n, unsigned long long seed, T* a) {
    for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        unsigned long long z = seed + 0x9E3779B97F4A7C15ULL * (unsigned long long)(t + 1);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
        z = z ^ (z >> 31);
        a[t] = T((double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0);
    }
}

// y <- x / sqrt(s[0])  (normalise by a device-side squared norm; y may be x)
template <typename T>
__global__ void scale_rsqrt_kernel(unsigned n, const double* __restrict__ s, const T* x, T* y,
                                   SlotBatch sb) {
    const long long so = slot_off(sb);
    s = at_slot(s, so);
    x = at_slot(x, so);
    y = at_slot(y, so);
    const double f = 1.0 / sqrt(s[0]);
    for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x)
        y[t] = T(f * (double)x[t]);
}

// y <- f x with x = src or the table entry src_tab[i], y = dst or dst_tab[i]
// (i: the slot's table index), f = 1 / sqrt(sq[0]) when sq is given, else 1.
// Moves vectors in and out of a Krylov basis whose index differs per slot.
template <typename T>
__global__ void tab_copy_kernel(unsigned n, const T* __restrict__ src, const T* const* __restrict__ src_tab,
                                T* dst, T* const* __restrict__ dst_tab, int idx, const double* __restrict__ sq,
                                SlotBatch sb) {
    using gw = __attribute__((address_space(1))) T*;
    const long long so = slot_off(sb);
    const int i = slot_count(sb, idx);
    const gptr<T> x = src_tab ? as_global(at_slot(src_tab, so)[i]) : as_global(at_slot(src, so));
    const gw y = dst_tab ? (gw)at_slot(dst_tab, so)[i] : (gw)at_slot(dst, so);
    if (sq) {
        const double f = 1.0 / sqrt(at_slot(sq, so)[0]);
        for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x)
            y[t] = T(f * (double)x[t]);
    } else {
        for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) y[t] = x[t];
    }
}

// Short per-slot arrays to and from one shared staging array (row z: slot z).
__global__ void scal_gather_kernel(const double* __restrict__ src, int k, double* __restrict__ dst, SlotBatch sb) {
    src = at_slot(src, slot_off(sb));
    for (int i = threadIdx.x; i < k; i += blockDim.x) dst[(long long)blockIdx.z * k + i] = src[i];
}
__global__ void scal_scatter_kernel(const double* __restrict__ src, int k, double* __restrict__ dst, SlotBatch sb) {
    dst = at_slot(dst, slot_off(sb));
    for (int i = threadIdx.x; i < k; i += blockDim.x) dst[i] = src[(long long)blockIdx.z * k + i];
}

// Entry (row, col) of D A D on the coarsest level, one thread each: the one-point (or
// two-point) element matrices (eq:elemmat) of the wedges around the column's node that
// hold the row's node, in ring order.  With free slip the entry is that of P A P + N,
// P = I - rhat rhat^T at either node on a free-slip sphere: the 3 x 3 block of the two
// nodes is summed first.  126 unknowns: 14 us (0.23 ms with one thread per column).
template <typename T>
__global__ void __launch_bounds__(64) coarse_assemble_kernel(int nd, const int* __restrict__ dof_slot,
                                                             const int* __restrict__ slot_dof, long long nslots,
                                                             const int* __restrict__ ring_tri,
                                                             const int* __restrict__ ring_nb,
                                                             const T* __restrict__ eta, const double* __restrict__ geo,
                                                             int m, int n, double r_in, double dr, double hg_alpha,
                                                             int twopt, int fs, const double* __restrict__ unit,
                                                             double* __restrict__ Ad) {
    const int row = blockIdx.x * 64 + threadIdx.x, col = blockIdx.y;
    if (row >= nd) return;
    auto on_fs = [&](int k) { return ((fs & 1) && k == 0) || ((fs & 2) && k == n); };
    const int cs = dof_slot[col], rs = dof_slot[row];
    const int cc = cs & 3, rc = rs & 3;
    const int clat = (cs >> 2) / (n + 1), ck0 = (cs >> 2) % (n + 1);
    const int rlat = (rs >> 2) / (n + 1), rk0 = (rs >> 2) % (n + 1);
    const bool pc = on_fs(ck0), pr = on_fs(rk0), proj = pc || pr;
    double M[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};   // [row component][column component]
    if (rk0 - ck0 <= 1 && ck0 - rk0 <= 1) {
        for (int r = 0; r < 6; ++r) {
            const int cd = ring_tri[(size_t)clat * 6 + r];
            if (cd < 0) break;
            // which lateral vertex of the triangle the row's node is
            const int v[3] = {clat, ring_nb[(size_t)clat * 6 + r], ring_nb[(size_t)clat * 6 + (r + 1) % 6]};
            int s2 = -1;
            for (int q = 0; q < 3; ++q)
                if (slot_dof[rc * nslots + (long long)v[q] * (n + 1) + rk0] == row) s2 = q;
            if (s2 < 0) continue;
            const int cell = cd >> 3, wd = (cd >> 2) & 1, lat = cd & 3, lat2 = (lat + s2) % 3;
            const double* g = geo + (size_t)cell * GEO_PER_COL + wd * GEO_PER_TRI;
            for (int ck = ck0 - 1; ck <= ck0; ++ck) {
                const int top = ck0 - ck, top2 = rk0 - ck;
                if (ck < 0 || ck >= n || top2 < 0 || top2 > 1) continue;
                const double rm = r_in + (ck + 0.5) * dr;
                const double e = (double)eta[((size_t)cell * n + ck) * 2 + wd];
                // quadrature points: q_c (weight 1), or the two radial points
                for (int qq = 0; qq < (twopt ? 2 : 1); ++qq) {
                    const double zq = twopt ? (qq == 0 ? -TWOPT_ZETA : TWOPT_ZETA) : 0.0;
                    const double rq = twopt ? rm + zq * (0.5 * dr) : rm;
                    const double V = (twopt ? 0.5 : 1.0) * rq * rq * g[9];
                    double gj[3], gl[3];
                    if (twopt) {
                        basis_grad_at(g, 0.5 / rq, zq, lat, top, gj);
                        basis_grad_at(g, 0.5 / rq, zq, lat2, top2, gl);
                    } else {
                        basis_grad(g, 0.5 / rm, lat, top, gj);
                        basis_grad(g, 0.5 / rm, lat2, top2, gl);
                    }
                    const double gg = gj[0] * gl[0] + gj[1] * gl[1] + gj[2] * gl[2];
                    const double eps = hg_alpha != 0.0 ? hg_eps(g, 0.5 / rm, V, e, hg_alpha) : 0.0;
                    // (A_e)_{(l,a),(j,b)} = V eta [delta_ab g_j.g_l + (g_j)_a (g_l)_b - 2/3 (g_j)_b (g_l)_a]
                    // hourglass term: eps delta_ab zeta_j zeta_l (delta_{lat_j, lat_l} - 1/3)
                    for (int a = 0; a < 3; ++a)
                        for (int b = 0; b < 3; ++b) {
                            if (!proj && (a != rc || b != cc)) continue;
                            double w = V * e * ((a == b ? gg : 0.0) + gj[a] * gl[b] - (2.0 / 3.0) * gj[b] * gl[a]);
                            if (a == b)
                                w += eps * (top ? 1.0 : -1.0) * (top2 ? 1.0 : -1.0) *
                                     ((lat == lat2 ? 1.0 : 0.0) - 1.0 / 3.0);
                            M[a][b] += w;
                        }
                }
            }
        }
    }
    double v = 0.0;
    if (!proj) {
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b)
                if (a == rc && b == cc) v = M[a][b];
    } else {
        const double* nc = unit + 3 * (size_t)clat;
        const double* nr = unit + 3 * (size_t)rlat;
        for (int a = 0; a < 3; ++a) {
            double w = 0.0;
            for (int b = 0; b < 3; ++b) w += M[a][b] * ((b == cc ? 1.0 : 0.0) - (pc ? nc[b] * nc[cc] : 0.0));
            v += ((a == rc ? 1.0 : 0.0) - (pr ? nr[a] * nr[rc] : 0.0)) * w;
        }
        // the normal rows of a free-slip node: + N
        if (pc && clat == rlat && ck0 == rk0) v += nc[rc] * nc[cc];
    }
    Ad[(size_t)col * nd + row] = v;
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// Lateral slots per workgroup of a kernel that streams whole columns with per-column data
// in LDS: about 2048 nodes a workgroup, fewer on small levels (at least 512 workgroups, as
// long as 256 nodes a workgroup are left), at most maxl.
int ring_slots_per_block(const Level& L, int maxl) {
    const int n1 = L.n + 1;
    int nlb = std::max(1, std::min(maxl, 2048 / n1));
    while (nlb > 1 && L.lat_slots() < 512LL * nlb && nlb * n1 > 256) nlb = (nlb + 1) / 2;
    return nlb;
}

template <typename T>
void mg_diag_A(const tng_ctx* ctx, const Level& L, const T* eta, double hg_alpha, T* const d[3], bool twopt,
               unsigned fs, bool invert) {
    require_unbatched("mg_diag_A");
    const int nlb = ring_slots_per_block(L, DIAG_MAXL);
    diag_A_kernel<T><<<nblk(L.lat_slots(), nlb), 256, 0, ctx->stream>>>(
        eta, L.geo64.p, L.ring_tri.p, (int)L.lat_slots(), nlb, L.n, magic_div((unsigned)(L.n + 1)), L.r_in, L.dr(),
        hg_alpha, twopt ? 1 : 0, (int)fs, L.unit64.p, invert ? 1 : 0, d[0], d[1], d[2]);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void mg_pmass(const tng_ctx* ctx, const Level& L, const Level& Lp, const T* eta, T* mdiag) {
    require_unbatched("mg_pmass");
    const long long nt = (Lp.m + PM_T) / PM_T, nkt = (Lp.n + PM_K) / PM_K;
    pmass_kernel<T><<<(unsigned)(10 * nt * nt * nkt), 256, 0, ctx->stream>>>(eta, L.geo64.p, L.m, L.n, L.r_in, L.dr(),
                                                                             mdiag);
    TNG_HIP(hipGetLastError());
    void* f[1] = {mdiag};
    launch_interface(ctx, Lp, prec_of<T>(), 0, 1, f);
}

template <typename T>
void mg_prolong(const tng_ctx* ctx, const Level& Lf, const T* const c[3], T* const f[3], bool add) {
    const long long ns = Lf.node_slots();
    const SlotBatch sb = launch_batch();
    auto* kernel = add ? prolong_add_kernel<T> : prolong_kernel<T>;
    kernel<<<dim3(nblk(ns, 256), add ? 3 : 1, sb.nb), 256, 0, ctx->stream>>>(
        Lf.m, Lf.n, c[0], c[1], c[2], f[0], f[1], f[2], (unsigned)ns, magic_div((unsigned)(Lf.n + 1)),
        magic_div((unsigned)(Lf.m + 1)), sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void mg_restrict(const tng_ctx* ctx, const Level& Lf, const Level& Lc, const T* const f[3], T* const c[3],
                 unsigned fs) {
    const long long ns = Lc.node_slots();
    const SlotBatch sb = launch_batch();
    restrict_kernel<T><<<dim3(nblk(ns, 256), 3, sb.nb), 256, 0, ctx->stream>>>(
        Lf.m, Lf.n, f[0], f[1], f[2], Lf.ring_tri.p, Lf.ring_nb.p, c[0], c[1], c[2], (unsigned)ns,
        magic_div((unsigned)(Lc.n + 1)), magic_div((unsigned)(Lc.m + 1)), (int)fs, sb);
    TNG_HIP(hipGetLastError());
    if (fs) vec_fs_project<T>(ctx, Lc, fs, c, nullptr);
}

template <typename T>
void vec_fs_project(const tng_ctx* ctx, const Level& L, unsigned fs, T* const x[3], const T* const b[3]) {
    if (!fs) return;
    require_unbatched("vec_fs_project");
    const T* un = std::is_same<T, double>::value ? (const T*)L.unit64.p : (const T*)L.unit32.p;
    fs_project_kernel<T><<<nblk(2 * L.lat_slots(), 256), 256, 0, ctx->stream>>>(
        L.lat_slots(), L.n, (int)fs, un, x[0], x[1], x[2], b ? b[0] : nullptr, b ? b[1] : nullptr,
        b ? b[2] : nullptr);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_cheb_update(const tng_ctx* ctx, long long n, const double* ab_dev, int k, const T* b, const T* y,
                     const T* invd, T* d, T* x) {
    const SlotBatch sb = launch_batch();
    if (aligned16(b) && aligned16(y) && aligned16(invd) && aligned16(d) && aligned16(x)) {
        const long long nv = n / (16 / (long long)sizeof(T));
        cheb_update_vec_kernel<T><<<dim3(std::max(1u, nblk(nv, 256)), 1, sb.nb), 256, 0, ctx->stream>>>(
            n, ab_dev, k, b, y, invd, d, x, sb);
        TNG_HIP(hipGetLastError());
        return;
    }
    cheb_update_kernel<T><<<dim3(nblk(n, 256 * EW_PER), 1, sb.nb), 256, 0, ctx->stream>>>(n, ab_dev, k, b, y, invd, d, x,
                                                                                  sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_cheb_post_update(const tng_ctx* ctx, const Level& L, bool ns_in, bool ns_out, const double* ab_dev, int k,
                          bool first, bool prev_zero, const T* b, const T* y, const T* invd, const T* xk, T* xo) {
    const SlotBatch sb = launch_batch();
    const long long ns = L.node_slots();
    TNG_REQUIRE(3 * ns < (1LL << 32), "smoother update: more than 2^32 values");
    TNG_REQUIRE(aligned16(b) && aligned16(y) && aligned16(invd) && aligned16(xk) && aligned16(xo),
                "smoother update: vectors must be 16-byte aligned");
    const long long nv = 3 * ns / (16 / (long long)sizeof(T));
    cheb_post_update_kernel<T><<<dim3(std::max(1u, nblk(nv, 256)), 1, sb.nb), 256, 0, ctx->stream>>>(
        (unsigned)ns, L.n + 1, magic_div((unsigned)ns), magic_div((unsigned)(L.n + 1)), L.lat_grp.p, L.grp_ptr.p,
        L.grp_slot.p, ns_in ? 1 : 0, ns_out ? 1 : 0, ab_dev, k, first ? 1 : 0, prev_zero ? 1 : 0, b, y, invd, xk, xo,
        sb);
    TNG_HIP(hipGetLastError());
}

template <typename T, bool MUL>
void launch_resid_post(const tng_ctx* ctx, const Level& L, bool ns_in, bool ns_out, const T* b, const T* x, const T* y,
                       T* r) {
    const SlotBatch sb = launch_batch();
    const long long ns = L.node_slots();
    resid_post_kernel<T, MUL><<<dim3(std::max(1u, nblk(ns, 256)), 3, sb.nb), 256, 0, ctx->stream>>>(
        (int)ns, L.n + 1, magic_div((unsigned)(L.n + 1)), L.lat_grp.p, L.grp_ptr.p, L.grp_slot.p, ns_in ? 1 : 0,
        ns_out ? 1 : 0, b, x, y, r, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_resid_post(const tng_ctx* ctx, const Level& L, bool ns_in, bool ns_out, const T* b, const T* x, const T* y,
                    T* r) {
    launch_resid_post<T, false>(ctx, L, ns_in, ns_out, b, x, y, r);
}

template <typename T>
void vec_mul_post(const tng_ctx* ctx, const Level& L, bool ns_in, bool ns_out, const T* invd, const T* x, const T* y,
                  T* z) {
    launch_resid_post<T, true>(ctx, L, ns_in, ns_out, invd, x, y, z);
}

// Chebyshev coefficients on the device (the arithmetic of chebyshev_coefficients)
__global__ void power_chebyshev_kernel(const double* __restrict__ pw, int deg, double lo, double hi, double* ab) {
    if (threadIdx.x != 0) return;
    const double lam = sqrt(pw[1]) / sqrt(pw[0]);
    const double l = lo * lam, h = hi * lam;
    const double theta = 0.5 * (h + l), delta = 0.5 * (h - l), sigma = theta / delta;
    ab[0] = 0.0;
    ab[1] = 1.0 / theta;
    double rho_old = 1.0 / sigma;
    for (int k = 1; k < deg; ++k) {
        const double rho = 1.0 / (2.0 * sigma - rho_old);
        ab[2 * k] = rho * rho_old;
        ab[2 * k + 1] = 2.0 * rho / delta;
        rho_old = rho;
    }
}

void power_chebyshev(const tng_ctx* ctx, const double* pw, int deg, double lo, double hi, double* ab) {
    require_unbatched("power_chebyshev");
    power_chebyshev_kernel<<<1, 64, 0, ctx->stream>>>(pw, deg, lo, hi, ab);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_invert(const tng_ctx* ctx, long long n, T* a) {
    require_unbatched("vec_invert");
    invert_kernel<T><<<nblk(n, 256), 256, 0, ctx->stream>>>(n, a);
    TNG_HIP(hipGetLastError());
}

template <typename TO, typename TI>
void vec_cast(const tng_ctx* ctx, long long n, const TI* a, TO* b) {
    const SlotBatch sb = launch_batch();
    cast_kernel<TO, TI><<<dim3(nblk(n, 256), 1, sb.nb), 256, 0, ctx->stream>>>(n, a, b, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_axpby(const tng_ctx* ctx, long long n, double a, const T* x, double b, T* y) {
    const SlotBatch sb = launch_batch();
    if (aligned16(x) && aligned16(y)) {
        const long long nv = n / (16 / (long long)sizeof(T));
        axpby_vec_kernel<T><<<dim3(std::max(1u, nblk(nv, 256)), 1, sb.nb), 256, 0, ctx->stream>>>(n, T(a), x, T(b),
                                                                                                 y, sb);
        TNG_HIP(hipGetLastError());
        return;
    }
    axpby_kernel<T><<<dim3(nblk(n, 256 * EW_PER), 1, sb.nb), 256, 0, ctx->stream>>>(n, T(a), x, T(b), y, sb);
    TNG_HIP(hipGetLastError());
}

// smallest compiled vector count >= every slot's count
inline int count_class(const SlotBatch& sb, int nq) {
    int mx = nq;
    if (sb.has_cnt)
        for (int z = 0; z < sb.nb; ++z) mx = std::max(mx, sb.cnt[z]);
    return mx <= 1 ? 1 : mx <= 2 ? 2 : mx <= 4 ? 4 : mx <= 8 ? 8 : mx <= 12 ? 12 : mx <= 16 ? 16 : MAX_MDOT;
}

#define TNG_NQ_DISPATCH(NQV, CALL)                     \
    switch (NQV) {                                     \
        case 1: { constexpr int NQ = 1; CALL; } break;  \
        case 2: { constexpr int NQ = 2; CALL; } break;  \
        case 4: { constexpr int NQ = 4; CALL; } break;  \
        case 8: { constexpr int NQ = 8; CALL; } break;  \
        case 12: { constexpr int NQ = 12; CALL; } break; \
        case 16: { constexpr int NQ = 16; CALL; } break; \
        default: { constexpr int NQ = MAX_MDOT; CALL; } break; \
    }

template <typename T>
void vec_mdot(const tng_ctx* ctx, DotScratch& ds, long long n, int n1, long long nlat, const uint8_t* owner,
              const T* x, const T* const* vs_dev, int nq, double* out_dev, bool accumulate) {
    TNG_REQUIRE(nq >= 1 && nq <= MAX_MDOT, "too many vectors in a multi-dot");
    TNG_REQUIRE(n <= 3LL * nlat * n1 && n < (1LL << 32), "multi-dot length out of range");
    const int nb = (int)std::min<long long>(DOT_BLOCKS, (n + DOT_BS - 1) / DOT_BS);
    const SlotBatch sb = launch_batch();
    check_counts(sb);
    const MagicDiv dn1 = magic_div((unsigned)n1);
    TNG_NQ_DISPATCH(count_class(sb, nq),
                    (mdot_partial_kernel<T, NQ><<<dim3(nb, 1, sb.nb), DOT_BS, 0, ctx->stream>>>(
                        (unsigned)n, dn1, (unsigned)nlat, owner, x, vs_dev, nq, ds.part.p, sb)));
    TNG_HIP(hipGetLastError());
    mdot_final_kernel<<<dim3(count_class(sb, nq), 1, sb.nb), 256, 0, ctx->stream>>>(nb, nq, ds.part.p, out_dev, accumulate ? 1 : 0, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_maxpy(const tng_ctx* ctx, long long n, const double* coef_dev, double sign, const T* const* vs_dev,
               int nq, T* y) {
    TNG_REQUIRE(nq >= 1 && nq <= MAX_MDOT, "too many vectors in a multi-axpy");
    const unsigned nb = (unsigned)std::min<long long>(nblk(n, 256), 8192);
    const SlotBatch sb = launch_batch();
    check_counts(sb);
    TNG_NQ_DISPATCH(count_class(sb, nq),
                    (maxpy_kernel<T, NQ><<<dim3(nb, 1, sb.nb), 256, 0, ctx->stream>>>((unsigned)n, coef_dev, sign,
                                                                                      vs_dev, nq, y, sb)));
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_smdot(const tng_ctx* ctx, DotScratch& ds, const Level& Lu, const Level& Lp, const T* x,
               const T* const* vs_dev, int nq, double* out_dev, bool accumulate, bool vs_aligned) {
    TNG_REQUIRE(nq >= 1 && nq <= MAX_MDOT, "too many vectors in a multi-dot");
    const long long n = 3 * Lu.node_slots() + Lp.node_slots();
    TNG_REQUIRE(n < (1LL << 32), "multi-dot length out of range");
    const SlotBatch sb = launch_batch();
    check_counts(sb);
    const MagicDiv du = magic_div((unsigned)(Lu.n + 1)), dp = magic_div((unsigned)(Lp.n + 1));
    // 16-byte accesses pay in FP32 (four values per load); the FP64 kernel already streams at
    // about 5.6 TB/s with its two 8-byte loads per vector and step
    if (sizeof(T) == 4 && vs_aligned && aligned16(x)) {
        const long long nv = n / (16 / (long long)sizeof(T));
        const int nb = (int)std::max<long long>(1, std::min<long long>(DOT_BLOCKS, (nv + DOT_BS - 1) / DOT_BS));
        TNG_NQ_DISPATCH(count_class(sb, nq), (smdot_vec_kernel<T, NQ><<<dim3(nb, 1, sb.nb), DOT_BS, 0, ctx->stream>>>(
                                (unsigned)Lu.node_slots(), du, (unsigned)Lu.lat_slots(), Lu.owner.p,
                                (unsigned)Lp.node_slots(), dp, Lp.owner.p, x, vs_dev, nq, ds.part.p, sb)));
        TNG_HIP(hipGetLastError());
        mdot_final_kernel<<<dim3(count_class(sb, nq), 1, sb.nb), 256, 0, ctx->stream>>>(nb, nq, ds.part.p, out_dev,
                                                                      accumulate ? 1 : 0, sb);
        TNG_HIP(hipGetLastError());
        return;
    }
    const int nb = (int)std::min<long long>(DOT_BLOCKS, (n + DOT_BS - 1) / DOT_BS);
    TNG_NQ_DISPATCH(count_class(sb, nq),
                    (smdot_partial_kernel<T, NQ><<<dim3(nb, 1, sb.nb), DOT_BS, 0, ctx->stream>>>(
                        (unsigned)Lu.node_slots(), du, (unsigned)Lu.lat_slots(), Lu.owner.p,
                        (unsigned)Lp.node_slots(), dp, Lp.owner.p, x, vs_dev, nq, ds.part.p, sb)));
    TNG_HIP(hipGetLastError());
    mdot_final_kernel<<<dim3(count_class(sb, nq), 1, sb.nb), 256, 0, ctx->stream>>>(nb, nq, ds.part.p, out_dev, accumulate ? 1 : 0, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_maxpy_smdot(const tng_ctx* ctx, DotScratch& ds, const Level& Lu, const Level& Lp, const double* coef_dev,
                     double sign, const T* const* vs_dev, int nq, T* y, double* out_dev, bool norm, bool vs_aligned) {
    TNG_REQUIRE(nq >= 1 && nq <= MAX_MDOT, "too many vectors in a multi-axpy");
    const long long n = 3 * Lu.node_slots() + Lp.node_slots();
    TNG_REQUIRE(n < (1LL << 32), "vector length out of range");
    const SlotBatch sb = launch_batch();
    check_counts(sb);
    const MagicDiv du = magic_div((unsigned)(Lu.n + 1)), dp = magic_div((unsigned)(Lp.n + 1));
    if (sizeof(T) == 4 && vs_aligned && aligned16(y)) {
        const long long nv = n / (16 / (long long)sizeof(T));
        const int nb = (int)std::max<long long>(1, std::min<long long>(DOT_BLOCKS, (nv + DOT_BS - 1) / DOT_BS));
        const dim3 grid(nb, 1, sb.nb);
        if (norm) {
            TNG_NQ_DISPATCH(count_class(sb, nq), (maxpy_dot_vec_kernel<T, NQ, true><<<grid, DOT_BS, 0, ctx->stream>>>(
                                    (unsigned)Lu.node_slots(), du, (unsigned)Lu.lat_slots(), Lu.owner.p,
                                    (unsigned)Lp.node_slots(), dp, Lp.owner.p, coef_dev, sign, vs_dev, nq, y,
                                    ds.part.p, sb)));
        } else {
            TNG_NQ_DISPATCH(count_class(sb, nq), (maxpy_dot_vec_kernel<T, NQ, false><<<grid, DOT_BS, 0, ctx->stream>>>(
                                    (unsigned)Lu.node_slots(), du, (unsigned)Lu.lat_slots(), Lu.owner.p,
                                    (unsigned)Lp.node_slots(), dp, Lp.owner.p, coef_dev, sign, vs_dev, nq, y,
                                    ds.part.p, sb)));
        }
        TNG_HIP(hipGetLastError());
        // the norm has one value for every slot: the per-slot counts do not apply to it
        SlotBatch sf = sb;
        if (norm) sf.has_cnt = 0;
        mdot_final_kernel<<<dim3(norm ? 1 : count_class(sf, nq), 1, sf.nb), 256, 0, ctx->stream>>>(nb, norm ? 1 : nq, ds.part.p, out_dev, 0, sf);
        TNG_HIP(hipGetLastError());
        return;
    }
    const int nb = (int)std::min<long long>(DOT_BLOCKS, (n + DOT_BS - 1) / DOT_BS);
    if (norm) {
        TNG_NQ_DISPATCH(count_class(sb, nq),
                        (maxpy_dot_kernel<T, NQ, true><<<dim3(nb, 1, sb.nb), DOT_BS, 0, ctx->stream>>>(
                            (unsigned)Lu.node_slots(), du, (unsigned)Lu.lat_slots(), Lu.owner.p,
                            (unsigned)Lp.node_slots(), dp, Lp.owner.p, coef_dev, sign, vs_dev, nq, y, ds.part.p, sb)));
    } else {
        TNG_NQ_DISPATCH(count_class(sb, nq),
                        (maxpy_dot_kernel<T, NQ, false><<<dim3(nb, 1, sb.nb), DOT_BS, 0, ctx->stream>>>(
                            (unsigned)Lu.node_slots(), du, (unsigned)Lu.lat_slots(), Lu.owner.p,
                            (unsigned)Lp.node_slots(), dp, Lp.owner.p, coef_dev, sign, vs_dev, nq, y, ds.part.p, sb)));
    }
    TNG_HIP(hipGetLastError());
    // the norm has one value for every slot: the per-slot counts do not apply to it
    SlotBatch sf = sb;
    if (norm) sf.has_cnt = 0;
    mdot_final_kernel<<<dim3(norm ? 1 : count_class(sf, nq), 1, sf.nb), 256, 0, ctx->stream>>>(nb, norm ? 1 : nq, ds.part.p, out_dev, 0, sf);
    TNG_HIP(hipGetLastError());
}

// a node field is a Stokes vector without velocity slots
template <typename T>
void vec_maxpy_mdot(const tng_ctx* ctx, DotScratch& ds, long long n, int n1, const uint8_t* owner,
                    const double* coef_dev, double sign, const T* const* vs_dev, int nq, T* y, double* out_dev,
                    bool norm) {
    TNG_REQUIRE(nq >= 1 && nq <= MAX_MDOT, "too many vectors in a multi-axpy");
    TNG_REQUIRE(n < (1LL << 32), "vector length out of range");
    require_unbatched("vec_maxpy_mdot");
    const SlotBatch sb;
    const MagicDiv dn1 = magic_div((unsigned)n1);
    const int nb = (int)std::min<long long>(DOT_BLOCKS, (n + DOT_BS - 1) / DOT_BS);
    if (norm) {
        TNG_NQ_DISPATCH(count_class(sb, nq), (maxpy_dot_kernel<T, NQ, true><<<nb, DOT_BS, 0, ctx->stream>>>(
                                0u, dn1, 0u, owner, (unsigned)n, dn1, owner, coef_dev, sign, vs_dev, nq, y,
                                ds.part.p, sb)));
    } else {
        TNG_NQ_DISPATCH(count_class(sb, nq), (maxpy_dot_kernel<T, NQ, false><<<nb, DOT_BS, 0, ctx->stream>>>(
                                0u, dn1, 0u, owner, (unsigned)n, dn1, owner, coef_dev, sign, vs_dev, nq, y,
                                ds.part.p, sb)));
    }
    TNG_HIP(hipGetLastError());
    mdot_final_kernel<<<norm ? 1 : nq, 256, 0, ctx->stream>>>(nb, norm ? 1 : nq, ds.part.p, out_dev, 0, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_rand(const tng_ctx* ctx, long long n, unsigned long long seed, T* a) {
    require_unbatched("vec_rand");
    const unsigned nb = (unsigned)std::min<long long>(nblk(n, 256), 8192);
    rand_kernel<T><<<nb, 256, 0, ctx->stream>>>((unsigned)n, seed, a);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_scale_rsqrt(const tng_ctx* ctx, long long n, const double* s, const T* x, T* y) {
    const unsigned nb = (unsigned)std::min<long long>(nblk(n, 256), 8192);
    const SlotBatch sb = launch_batch();
    scale_rsqrt_kernel<T><<<dim3(nb, 1, sb.nb), 256, 0, ctx->stream>>>((unsigned)n, s, x, y, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_tab_copy(const tng_ctx* ctx, long long n, const T* src, const T* const* src_tab, T* dst, T* const* dst_tab,
                  int idx, const double* sq) {
    const SlotBatch sb = launch_batch();
    const unsigned nb = (unsigned)std::min<long long>(nblk(n, 256), 8192);
    tab_copy_kernel<T><<<dim3(nb, 1, sb.nb), 256, 0, ctx->stream>>>((unsigned)n, src, src_tab, dst, dst_tab, idx,
                                                                     sq, sb);
    TNG_HIP(hipGetLastError());
}

void scal_gather(const tng_ctx* ctx, const double* src, int k, double* staging) {
    const SlotBatch sb = launch_batch();
    scal_gather_kernel<<<dim3(1, 1, sb.nb), 64, 0, ctx->stream>>>(src, k, staging, sb);
    TNG_HIP(hipGetLastError());
}

void scal_scatter(const tng_ctx* ctx, const double* staging, int k, double* dst) {
    const SlotBatch sb = launch_batch();
    scal_scatter_kernel<<<dim3(1, 1, sb.nb), 64, 0, ctx->stream>>>(staging, k, dst, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void coarse_assemble(const tng_ctx* ctx, CoarseDense& cd, const Level& L, const T* eta, double hg_alpha,
                     bool twopt, unsigned fs) {
    require_unbatched("coarse_assemble");
    coarse_assemble_kernel<T><<<dim3(nblk(cd.ndof, 64), cd.ndof), 64, 0, ctx->stream>>>(
        cd.ndof, cd.dof_slot.p, cd.slot_dof.p, cd.nslots, L.ring_tri.p, L.ring_nb.p, eta, L.geo64.p, L.m, L.n, L.r_in,
        L.dr(), hg_alpha, twopt ? 1 : 0, (int)fs, L.unit64.p, cd.matrix());
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_copy3(const tng_ctx* ctx, long long n, const T* a0, const T* a1, const T* a2, T* o0, T* o1, T* o2) {
    require_unbatched("vec_copy3");
    const unsigned nb = (unsigned)std::min<long long>(nblk(n, 256), 8192);
    copy3_kernel<T><<<dim3(nb, 3), 256, 0, ctx->stream>>>((unsigned)n, a0, a1, a2, o0, o1, o2);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_mul(const tng_ctx* ctx, long long n, const T* a, const T* b, T* c) {
    require_unbatched("vec_mul");
    const unsigned nb = (unsigned)std::min<long long>(nblk(n, 256), 8192);
    mul_kernel<T><<<nb, 256, 0, ctx->stream>>>((unsigned)n, a, b, c);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_fill(const tng_ctx* ctx, long long n, T v, T* a) {
    if (n <= 0) return;
    const unsigned nb = (unsigned)std::min<long long>(nblk(n, 256), 8192);
    const SlotBatch sb = launch_batch();
    fillv_kernel<T><<<dim3(nb, 1, sb.nb), 256, 0, ctx->stream>>>((unsigned)n, v, a, sb);
    TNG_HIP(hipGetLastError());
}

void coarse_rotation_shift(const tng_ctx* ctx, CoarseDense& cd, const Level& L) {
    require_unbatched("coarse_rotation_shift");
    if (cd.rotq.n != (size_t)(3 * cd.ndof + 1)) cd.rotq.alloc(3 * cd.ndof + 1);
    coarse_rotation_basis_kernel<<<1, 1, 0, ctx->stream>>>(cd.ndof, cd.dof_slot.p, L.m, L.n, L.r_in, L.dr(),
                                                         L.unit64.p, cd.matrix(), cd.rotq.p);
    TNG_HIP(hipGetLastError());
    coarse_rotation_shift_kernel<<<nblk(cd.ndof, 64), 64, 0, ctx->stream>>>(cd.ndof, cd.rotq.p, cd.matrix());
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_rotation(const tng_ctx* ctx, const Level& L, int a, T* const out[3]) {
    require_unbatched("vec_rotation");
    const long long ns = L.node_slots();
    rotation_fill_kernel<T><<<nblk(ns, 256), 256, 0, ctx->stream>>>(L.m, L.n, L.r_in, L.dr(), L.unit64.p, a, out[0],
                                                                   out[1], out[2], ns);
    TNG_HIP(hipGetLastError());
}

void coarse_invert(const tng_ctx* ctx, CoarseDense& cd) {
    require_unbatched("coarse_invert");
    const int nb = cd.inv_steps();
    double* a = cd.matrix();
    for (int pb = 0; pb < nb; ++pb) {
        double* o = a == cd.Ainv.p ? cd.Awork.p : cd.Ainv.p;
        invert_step_kernel<<<dim3(nb, nb), 256, 0, ctx->stream>>>(cd.ndof, pb, a, o);
        TNG_HIP(hipGetLastError());
        a = o;
    }
}

template <typename T>
void coarse_solve(const tng_ctx* ctx, const CoarseDense& cd, const T* const b[3], T* const x[3]) {
    const SlotBatch sb = launch_batch();
    coarse_solve_kernel<T><<<dim3(1, 1, sb.nb), 1024, 0, ctx->stream>>>(
        cd.ndof, cd.dof_slot.p, cd.slot_dof.p, cd.nslots, cd.Ainv.p, b[0], b[1], b[2], x[0], x[1], x[2], sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_shift(const tng_ctx* ctx, long long n, const double* sum_cnt, T* p) {
    const SlotBatch sb = launch_batch();
    shift_kernel<T><<<dim3(nblk(n, 256), 1, sb.nb), 256, 0, ctx->stream>>>(n, sum_cnt, p, sb);
    TNG_HIP(hipGetLastError());
}

template <typename T>
void vec_schur(const tng_ctx* ctx, long long n, const T* r, const T* mdiag, T* z) {
    const SlotBatch sb = launch_batch();
    schur_diag_kernel<T><<<dim3(nblk(n, 256), 1, sb.nb), 256, 0, ctx->stream>>>(n, r, mdiag, z, sb);
    TNG_HIP(hipGetLastError());
}

#define TNG_INST(T)                                                                                        \
    template void mg_diag_A<T>(const tng_ctx*, const Level&, const T*, double, T* const[3], bool, unsigned, bool); \
    template void vec_fs_project<T>(const tng_ctx*, const Level&, unsigned, T* const[3], const T* const[3]);      \
    template void vec_rotation<T>(const tng_ctx*, const Level&, int, T* const[3]);                                \
    template void mg_pmass<T>(const tng_ctx*, const Level&, const Level&, const T*, T*);                  \
    template void mg_prolong<T>(const tng_ctx*, const Level&, const T* const[3], T* const[3], bool);      \
    template void mg_restrict<T>(const tng_ctx*, const Level&, const Level&, const T* const[3],           \
                                 T* const[3], unsigned);                                                   \
    template void vec_resid_post<T>(const tng_ctx*, const Level&, bool, bool, const T*, const T*, const T*, T*); \
    template void vec_mul_post<T>(const tng_ctx*, const Level&, bool, bool, const T*, const T*, const T*, T*);   \
    template void vec_cheb_post_update<T>(const tng_ctx*, const Level&, bool, bool, const double*, int, bool,   \
                                          bool, const T*, const T*, const T*, const T*, T*);                 \
    template void vec_cheb_update<T>(const tng_ctx*, long long, const double*, int, const T*, const T*,   \
                                     const T*, T*, T*);                                                    \
    template void vec_invert<T>(const tng_ctx*, long long, T*);                                           \
    template void vec_axpby<T>(const tng_ctx*, long long, double, const T*, double, T*);                  \
    template void vec_mdot<T>(const tng_ctx*, DotScratch&, long long, int, long long, const uint8_t*,     \
                              const T*, const T* const*, int, double*, bool);                              \
    template void coarse_solve<T>(const tng_ctx*, const CoarseDense&, const T* const[3], T* const[3]);    \
    template void vec_shift<T>(const tng_ctx*, long long, const double*, T*);                             \
    template void vec_schur<T>(const tng_ctx*, long long, const T*, const T*, T*);                       \
    template void vec_maxpy<T>(const tng_ctx*, long long, const double*, double, const T* const*, int, T*); \
    template void vec_fill<T>(const tng_ctx*, long long, T, T*);                                          \
    template void vec_copy3<T>(const tng_ctx*, long long, const T*, const T*, const T*, T*, T*, T*);         \
    template void vec_mul<T>(const tng_ctx*, long long, const T*, const T*, T*);                          \
    template void vec_smdot<T>(const tng_ctx*, DotScratch&, const Level&, const Level&, const T*,         \
                               const T* const*, int, double*, bool, bool);                                 \
    template void vec_maxpy_smdot<T>(const tng_ctx*, DotScratch&, const Level&, const Level&, const double*,  \
                                     double, const T* const*, int, T*, double*, bool, bool);                 \
    template void vec_maxpy_mdot<T>(const tng_ctx*, DotScratch&, long long, int, const uint8_t*, const double*, double, \
                                    const T* const*, int, T*, double*, bool);                                 \
    template void vec_rand<T>(const tng_ctx*, long long, unsigned long long, T*);                         \
    template void vec_scale_rsqrt<T>(const tng_ctx*, long long, const double*, const T*, T*);             \
    template void vec_tab_copy<T>(const tng_ctx*, long long, const T*, const T* const*, T*, T* const*, int, \
                                  const double*);                                                          \
    template void coarse_assemble<T>(const tng_ctx*, CoarseDense&, const Level&, const T*, double, bool,  \
                                     unsigned);
TNG_INST(double)
TNG_INST(float)
#undef TNG_INST
template void vec_cast<float, double>(const tng_ctx*, long long, const double*, float*);
template void vec_cast<double, float>(const tng_ctx*, long long, const float*, double*);
template void vec_cast<float, float>(const tng_ctx*, long long, const float*, float*);
template void vec_cast<double, double>(const tng_ctx*, long long, const double*, double*);

}  // namespace tng
