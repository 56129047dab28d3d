// Expansion kernels: P2M, M2M, L2L, P2L, L2P and M2P (Sec. 2), the M2L
// operator tables built from Eq. 4, and conversion to the paper's
// normalisation for inspection.  See common.hpp for the basis.
#include "common.hpp"
#include "expansions.hpp"
#include "m2l_table.hpp"

#include <algorithm>

namespace hfmm {

// ---------------------------------------------------------------------
// streaming solid harmonics: f(n, m, re, im) for every n < ND, 0 <= m <= n,
// column by column, so only a few values are live at a time
// ---------------------------------------------------------------------
template <typename T, int ND, typename F>
__device__ __forceinline__ void stream_regular(T x, T y, T z, F&& f) {
    const T r2 = x * x + y * y + z * z;
    T dre = T(1), dim = T(0);
#pragma unroll
    for (int m = 0; m < ND; ++m) {
        if (m > 0) {
            const T c = T(-1) / T(2 * m);
            T nr = c * (x * dre - y * dim);
            T ni = c * (x * dim + y * dre);
            dre = nr;
            dim = ni;
        }
        f(m, m, dre, dim);
        T pr = T(0), pi = T(0), cr = dre, ci = dim;
#pragma unroll
        for (int n = m; n + 1 < ND; ++n) {
            const T c = T(1) / T((n + 1) * (n + 1) - m * m);
            const T a = T(2 * n + 1) * z;
            T nr = (a * cr - r2 * pr) * c;
            T ni = (a * ci - r2 * pi) * c;
            pr = cr;
            pi = ci;
            cr = nr;
            ci = ni;
            f(n + 1, m, cr, ci);
        }
    }
}

template <typename T, int ND, typename F>
__device__ __forceinline__ void stream_irregular(T x, T y, T z, F&& f) {
    const T r2 = x * x + y * y + z * z;
    const T ir = rsqrt_fast(r2);
    const T ir2 = ir * ir;
    T dre = ir, dim = T(0);
#pragma unroll
    for (int m = 0; m < ND; ++m) {
        if (m > 0) {
            const T c = T(-(2 * m - 1)) * ir2;
            T nr = c * (x * dre - y * dim);
            T ni = c * (x * dim + y * dre);
            dre = nr;
            dim = ni;
        }
        f(m, m, dre, dim);
        T pr = T(0), pi = T(0), cr = dre, ci = dim;
#pragma unroll
        for (int n = m; n + 1 < ND; ++n) {
            const T a = T(2 * n + 1) * z;
            const T b = T(n * n - m * m);
            T nr = (a * cr - b * pr) * ir2;
            T ni = (a * ci - b * pi) * ir2;
            pr = cr;
            pi = ci;
            cr = nr;
            ci = ni;
            f(n + 1, m, cr, ci);
        }
    }
}

template <typename T>
__device__ __forceinline__ T cre(const double* X, int n, int m) {
    return (T)X[ridx(n, m, 0)];
}
template <typename T>
__device__ __forceinline__ T cim(const double* X, int n, int m) {
    return m == 0 ? T(0) : (T)X[ridx(n, m, 1)];
}
template <typename T>
__device__ __forceinline__ T cre(const float* X, int n, int m) {
    return (T)X[ridx(n, m, 0)];
}
template <typename T>
__device__ __forceinline__ T cim(const float* X, int n, int m) {
    return m == 0 ? T(0) : (T)X[ridx(n, m, 1)];
}

// ---------------------------------------------------------------------
// masses and centres
// ---------------------------------------------------------------------
// masses in sorted order into the FP32 and FP64 records; non-finite masses
// are flagged in the status word
__global__ void k_fill_masses(int64_t n, const int32_t* __restrict__ perm,
                              const double* __restrict__ m, const double* __restrict__ xs,
                              const double* __restrict__ ys, const double* __restrict__ zs,
                              float4* __restrict__ p32, double4* __restrict__ p64,
                              int32_t* __restrict__ status) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    if (s < n) {
        const double q = m[perm[s]];
        bad = !isfinite(q);
        p32[s].w = (float)q;
        p64[s] = make_double4(xs[s], ys[s], zs[s], q);
    }
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(status, (int32_t)ST_MASS_NONFINITE);
}

__global__ void k_centres_geometric(const Cell* __restrict__ cells, int nc,
                                    const Root* __restrict__ root, double4* __restrict__ cen) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    double o[3];
    Cell cell = cells[c];
    cell_centre(*root, cell, o);
    cen[c] = make_double4(o[0], o[1], o[2], 1.0 / cell_side(*root, cell.level));
}

// centres of mass (weights |m|), leaves from particles and parents from
// children, one level at a time (deepest first); w4 = (sum |m| x, y, z, |m|)
__global__ void k_com_level(const Cell* __restrict__ cells, int c0, int c1,
                            const double4* __restrict__ p64, const Root* __restrict__ root,
                            double4* __restrict__ w4, double4* __restrict__ cen) {
#pragma clang fp contract(off)
    int c = c0 + blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= c1) return;
    Cell cell = cells[c];
    double sx = 0, sy = 0, sz = 0, sw = 0;
    if (cell.nchild == 0) {
        for (int s = cell.first; s < cell.first + cell.count; ++s) {
            double4 q = p64[s];
            double a = fabs(q.w);
            sw += a;
            sx += a * q.x;
            sy += a * q.y;
            sz += a * q.z;
        }
    } else {
        for (int k = 0; k < cell.nchild; ++k) {
            double4 q = w4[cell.child + k];
            sx += q.x;
            sy += q.y;
            sz += q.z;
            sw += q.w;
        }
    }
    w4[c] = make_double4(sx, sy, sz, sw);
    double h = cell_side(*root, cell.level);
    if (sw > 0.0) {
        cen[c] = make_double4(sx / sw, sy / sw, sz / sw, 1.0 / h);
    } else {
        double o[3];
        cell_centre(*root, cell, o);
        cen[c] = make_double4(o[0], o[1], o[2], 1.0 / h);
    }
}

// ---------------------------------------------------------------------
// shift tables: R_n^m(u) for the M2M / L2L vectors in units of the child
// side, u = (c_child - c_parent) / h_child.  Octant table (geometric
// centres): u = (ox - 1/2, oy - 1/2, oz - 1/2); per-child table (centres of
// mass).  Stored as (re, im) pairs, triangular, FP64.
// ---------------------------------------------------------------------
template <int NP>
__global__ void k_shift_octants(double2* __restrict__ tab) {
    int o = threadIdx.x;
    if (o >= 8) return;
    double u[3] = {((o >> 2) & 1) - 0.5, ((o >> 1) & 1) - 0.5, (o & 1) - 0.5};
    double2* out = tab + o * ntri(NP);
    stream_regular<double, NP>(u[0], u[1], u[2], [&](int n, int m, double re, double im) {
        out[tri(n, m)] = make_double2(re, im);
    });
}

template <int NP>
__global__ void k_shift_children(const Cell* __restrict__ cells, int nc,
                                 const double4* __restrict__ cen, double2* __restrict__ tab) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    Cell cell = cells[c];
    if (cell.parent < 0) return;
    double4 a = cen[c], b = cen[cell.parent];
    double ih = a.w;
    double u[3] = {(a.x - b.x) * ih, (a.y - b.y) * ih, (a.z - b.z) * ih};
    double2* out = tab + (int64_t)c * ntri(NP);
    stream_regular<double, NP>(u[0], u[1], u[2], [&](int n, int m, double re, double im) {
        out[tri(n, m)] = make_double2(re, im);
    });
}

__device__ inline int octant_idx(const Cell& c) {
    return ((c.ix & 1) << 2) | ((c.iy & 1) << 1) | (c.iz & 1);
}

// X_n^m of a stored m >= 0 triangle with X_n^{-m} = (-1)^m conj(X_n^m)
__device__ inline double2 tri_get(const double2* X, int n, int m) {
    if (m >= 0) return X[tri(n, m)];
    double2 v = X[tri(n, -m)];
    double s = (m & 1) ? -1.0 : 1.0;
    return make_double2(s * v.x, -s * v.y);
}
__device__ inline double2 real_get(const double* X, int n, int m) {
    int a = m < 0 ? -m : m;
    double re = X[ridx(n, a, 0)], im = a == 0 ? 0.0 : X[ridx(n, a, 1)];
    if (m >= 0) return make_double2(re, im);
    double s = (a & 1) ? -1.0 : 1.0;
    return make_double2(s * re, -s * im);
}

// ---------------------------------------------------------------------
// P2M: Mt_n^m = sum_j q_j conj(R_n^m((x_j - c) / h)) (Eq. 2 in the device
// basis).  G lanes per leaf, lanes stride over the leaf's particles, then a
// butterfly reduction across the G lanes.
// ---------------------------------------------------------------------
template <typename T, int NP>
__global__ void __launch_bounds__(256)
k_p2m(const Cell* __restrict__ cells, const int32_t* __restrict__ leaves, int nleaves,
      const double4* __restrict__ cen, const double4* __restrict__ p64,
      double* __restrict__ M, int ld) {
    constexpr int G = 8, P = NP * NP;
    const int gid = (blockIdx.x * blockDim.x + threadIdx.x) / G;
    const int sub = threadIdx.x % G;
    const bool active = gid < nleaves;
    const int c = active ? leaves[gid] : 0;
    T acc[P];
#pragma unroll
    for (int k = 0; k < P; ++k) acc[k] = T(0);
    if (active) {
        const Cell cell = cells[c];
        const double4 q = cen[c];
        const double ih = q.w;
        for (int j = cell.first + sub; j < cell.first + cell.count; j += G) {
            const double4 pj = p64[j];
            const T ux = (T)((pj.x - q.x) * ih), uy = (T)((pj.y - q.y) * ih),
                    uz = (T)((pj.z - q.z) * ih), mj = (T)pj.w;
            stream_regular<T, NP>(ux, uy, uz, [&](int n, int m, T re, T im) {
                acc[ridx(n, m, 0)] += mj * re;
                if (m > 0) acc[ridx(n, m, 1)] -= mj * im;
            });
        }
    }
#pragma unroll
    for (int d = 1; d < G; d <<= 1)
#pragma unroll
        for (int k = 0; k < P; ++k) acc[k] += __shfl_xor(acc[k], d, 64);
    if (active && sub == 0) {
        double* out = M + (int64_t)c * ld;
#pragma unroll
        for (int k = 0; k < P; ++k) out[k] = (double)acc[k];
        for (int k = P; k < ld; ++k) out[k] = 0.0;
    }
}

// ---------------------------------------------------------------------
// M2M (FP64): Mt_p[n,m] = 2^-n sum_children sum_{k,l} conj(R_k^l(u))
//                         Mt_c[n-k, m-l]
// one thread per (parent, output (n, m >= 0))
// ---------------------------------------------------------------------
template <int NP>
__global__ void k_m2m(const Cell* __restrict__ cells, int c0, int c1,
                      const double2* __restrict__ shift, int per_child,
                      double* __restrict__ M, int ld) {
    constexpr int P = NP * NP, NT = ntri(NP);
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int c = c0 + (int)(gid / NT);
    if (c >= c1) return;
    const int t = (int)(gid % NT);
    int n = 0;
    while (tri(n + 1, 0) <= t) ++n;
    const int m = t - tri(n, 0);
    const Cell cell = cells[c];
    if (cell.nchild == 0) return;
    double sr = 0.0, si = 0.0;
    for (int q = 0; q < cell.nchild; ++q) {
        const int ch = cell.child + q;
        const double2* R = per_child ? shift + (int64_t)ch * NT
                                     : shift + octant_idx(cells[ch]) * NT;
        const double* Mc = M + (int64_t)ch * ld;
        for (int k = 0; k <= n; ++k)
            for (int l = -k; l <= k; ++l) {
                const int mm = m - l;
                if (mm > n - k || mm < -(n - k)) continue;
                double2 r = tri_get(R, k, l);  // conj below
                double2 x = real_get(Mc, n - k, mm);
                sr += r.x * x.x + r.y * x.y;
                si += r.x * x.y - r.y * x.x;
            }
    }
    const double sc = ldexp(1.0, -n);
    double* out = M + (int64_t)c * ld;
    out[ridx(n, m, 0)] = sr * sc;
    if (m > 0) out[ridx(n, m, 1)] = si * sc;
}

// ---------------------------------------------------------------------
// P2L for the X list (Eq. 3 in the device basis, FP64):
//   Lt_n^m(B) += sum_j q_j conj(S_n^m((x_j - c_B) / h_B))
// One 64-lane wave per target cell with an X list (from the compact array of
// such cells; the others keep LX = 0).  The particles of the cell's X-list
// leaves are packed into chunks of 64 (a lane per list leaf, a scan of the
// counts, the owner of each slot from wave_run_owner), lane j evaluating
// particle j.  The harmonics come order by order (m): the wave stores the
// weighted terms of one order in LDS, term by term, and its lanes then add
// them up over the particles, lane g T + t taking the g-th part of the
// particles of term t (T terms, up to 8 parts), into an FP64 sum per order;
// the parts are added at the end.  One order's terms are 2 (p - m) reals, so
// LDS holds 64 particles of them (5 KB at p = 10 in FP32) where it held 20
// particles of all p^2 terms, and every lane evaluates.
// T: the type of the terms (FP32 for the FP32 path; the sums are FP64).
// ---------------------------------------------------------------------
constexpr int kP2lStride = 65;  // LDS row stride (bank spread)
constexpr int p2l_terms(int np, int m) { return m == 0 ? np : 2 * (np - m); }
constexpr int p2l_parts(int np, int m) {
    int g = 1;
    while (g < 8 && 2 * g * p2l_terms(np, m) <= 64) g *= 2;
    return g;
}

template <typename T, int NP>
__global__ void __launch_bounds__(64)
k_p2l(const Cell* __restrict__ cells, const int32_t* __restrict__ x_cells,
      const int32_t* __restrict__ x_off, const int32_t* __restrict__ x_items,
      const double4* __restrict__ cen, const double4* __restrict__ p64,
      double* __restrict__ LX, int ld) {
    __shared__ T sh[2 * NP * kP2lStride];
    __shared__ int own[64];
    const int lane = threadIdx.x;
    const int b = x_cells[blockIdx.x];
    const int e0 = x_off[b], e1 = x_off[b + 1];
    double acc[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) acc[m] = 0.0;
    const double4 q = cen[b];
    const double ih = q.w;
    for (int eb = e0; eb < e1; eb += 64) {
        int first = 0, cnt = 0;
        if (eb + lane < e1) {
            const Cell src = cells[x_items[eb + lane]];
            first = src.first;
            cnt = src.count;
        }
        int tot;
        const int off = wave_excl_scan(cnt, lane, tot);
        for (int pb = 0; pb < tot; pb += 64) {
            int o = wave_run_owner(own, off, cnt, pb, 64, lane);
            const bool ok = pb + lane < tot;
            o = ok ? o : 0;
            const int f = __shfl(first, o, 64), fo = __shfl(off, o, 64);
            // (lanes past the last particle: a zero weight at unit distance)
            T ux = T(1), uy = T(0), uz = T(0), w = T(0);
            if (ok) {
                const double4 pj = p64[f + (pb + lane - fo)];
                ux = (T)((pj.x - q.x) * ih);
                uy = (T)((pj.y - q.y) * ih);
                uz = (T)((pj.z - q.z) * ih);
                w = (T)pj.w;
            }
            stream_irregular<T, NP>(ux, uy, uz, [&](int n, int m, T re, T im) {
                if (m == 0) {
                    sh[n * kP2lStride + lane] = w * re;
                } else {
                    sh[2 * (n - m) * kP2lStride + lane] = w * re;
                    sh[(2 * (n - m) + 1) * kP2lStride + lane] = -w * im;
                }
                if (n + 1 < NP) return;
                // the order's terms are complete
                const int terms = p2l_terms(NP, m), parts = p2l_parts(NP, m), len = 64 / parts;
                const int t = lane % terms, g = lane / terms;
                wave_lds_fence();
                if (g < parts) {
                    const T* r = sh + t * kP2lStride + g * len;
                    double a = 0.0;
#pragma unroll 8
                    for (int j = 0; j < len; ++j) a += (double)r[j];
                    acc[m] += a;
                }
                wave_lds_fence();
            });
        }
    }
    double* out = LX + (int64_t)b * ld;
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        const int terms = p2l_terms(NP, m), parts = p2l_parts(NP, m);
        double v = acc[m];
        for (int g = 1; g < parts; ++g)
            v += __shfl(acc[m], min(lane + g * terms, 63), 64);
        if (lane < terms)
            out[m == 0 ? ridx(lane, 0, 0) : ridx(m + lane / 2, m, lane & 1)] = v;
    }
}


// ---------------------------------------------------------------------
// M2P of one expansion (Eq. 2 with its gradient) at u = (x - c) / h:
//   phi = sum Mt S(u) / h,  grad phi from dS_n^m/dz = -S_{n+1}^m and
//   (d/dx + i d/dy) S_n^m = S_{n+1}^{m+1}
// ---------------------------------------------------------------------
template <typename T, int NP, typename MT>
__device__ __forceinline__ void m2p_accumulate(const MT* Mc, T ux, T uy, T uz, T ih,
                                               T& phi, T& ax, T& ay, T& az) {
    T f = T(0), dz = T(0), hr = T(0), hi = T(0);
    stream_irregular<T, NP + 1>(ux, uy, uz, [&](int k, int l, T sr, T si) {
        const T w = l == 0 ? T(1) : T(2);
        if (k < NP) {
            T mr = cre<T>(Mc, k, l), mi = cim<T>(Mc, k, l);
            f += w * (mr * sr - mi * si);
        }
        if (k >= 1) {
            if (l <= k - 1) {
                T mr = cre<T>(Mc, k - 1, l), mi = cim<T>(Mc, k - 1, l);
                dz -= w * (mr * sr - mi * si);
            }
            if (l >= 1) {
                T mr = cre<T>(Mc, k - 1, l - 1), mi = cim<T>(Mc, k - 1, l - 1);
                hr += mr * sr - mi * si;
                hi += mr * si + mi * sr;
            }
            if (l + 1 <= k - 1) {
                T mr = cre<T>(Mc, k - 1, l + 1), mi = cim<T>(Mc, k - 1, l + 1);
                hr -= mr * sr - mi * si;
                hi += mr * si + mi * sr;
            }
        }
    });
    const T ih2 = ih * ih;
    phi += f * ih;
    ax += hr * ih2;
    ay += hi * ih2;
    az += dz * ih2;
}

// ---------------------------------------------------------------------
// Far field of one target leaf per wave, any p.  A batch of up to 64 list
// cells is packed with a ballot: the cell ids and, per cell, the offset from
// its centre to the leaf's reference point cb in units of its side (formed
// in FP64) with 1/h.  Their coefficient rows are then staged FB at a time in
// the wave's LDS slice (the wave copies the rows with 16-byte loads), and
// lane g * TW + t evaluates cells g, g + G, ... of the slice at target t.
// ---------------------------------------------------------------------
template <int NP, typename MT, int BYTES = 8192>
struct FarShape {
    static constexpr int LD = (NP * NP + 15) / 16 * 16;  // row length of M
    // rows staged at once: at most 8 KB of coefficients per wave
    static constexpr int FIT = BYTES / (LD * (int)sizeof(MT));
    static constexpr int FB = FIT < 2 ? 2 : FIT < 16 ? FIT : 16;
};

template <typename T, int NP, typename MT, int G, int BYTES>
__device__ __forceinline__ void farp_batch(bool valid, int k, const double4& cb,
                                           const double4* __restrict__ cen,
                                           const MT* __restrict__ M, int32_t* ids,
                                           typename Vec4<T>::type* offs, MT* rows, T rx, T ry,
                                           T rz, T& phi, T& ax, T& ay, T& az) {
    using V = typename Vec4<T>::type;
    using S = FarShape<NP, MT, BYTES>;
    constexpr int TW = 64 / G, Q = S::LD * (int)sizeof(MT) / 16;  // 16-byte chunks per row
    const int lane = threadIdx.x & 63, g = lane / TW;
    const uint64_t bal = __ballot(valid);
    const int nb = __popcll(bal);
    if (nb == 0) return;  // uniform per wave
    V o{};
    if (valid) {
        const double4 qc = cen[k];
        o = V{(T)((cb.x - qc.x) * qc.w), (T)((cb.y - qc.y) * qc.w), (T)((cb.z - qc.z) * qc.w),
              (T)qc.w};
    }
    const int pos = __popcll(bal & lanes_below(lane));
    wave_lds_fence();
    if (valid) {
        ids[pos] = k;
        offs[pos] = o;
    }
    wave_lds_fence();
    for (int sb = 0; sb < nb; sb += S::FB) {
        const int ns = min(S::FB, nb - sb);
        // rows of cells sb .. sb + ns, 16 bytes per lane and load
        for (int c = lane; c < ns * Q; c += 64) {
            const int i = c / Q, q = c - i * Q;
            const uint4 v = *((const uint4*)(M + (int64_t)ids[sb + i] * S::LD) + q);
            *((uint4*)(rows + i * S::LD) + q) = v;
        }
        wave_lds_fence();
        for (int j0 = 0; j0 < ns; j0 += G) {
            const int j = j0 + g;
            if (j < ns) {
                const V d = offs[sb + j];
                m2p_accumulate<T, NP>(rows + j * S::LD, rx * d.w + d.x, ry * d.w + d.y,
                                      rz * d.w + d.z, d.w, phi, ax, ay, az);
            }
        }
        wave_lds_fence();
    }
}

// The M2P terms of the box's list items[e0, e1) (the FMM's W list, and V
// for a box without sources) at its targets.  red (kFarLongWaves * 256 of T in
// LDS): the waves of the block hold parts of one list, and the block's sums
// are written; otherwise the wave's.
template <typename T, int NP, typename MT, int G, int BYTES = 8192>
__device__ __forceinline__ void farp_box(const TBox& leaf, const double4& cb,
                                          const double4* __restrict__ cen,
                                          const double4* __restrict__ p64,
                                          const int32_t* __restrict__ items, int e0, int e1,
                                          const MT* __restrict__ M, int32_t* ids,
                                          typename Vec4<T>::type* offs, MT* rows,
                                          T* __restrict__ far, int64_t n, T* red) {
    constexpr int TW = 64 / G;
    const int lane = threadIdx.x & 63, t = lane % TW;
    for (int c0 = 0; c0 < leaf.count; c0 += TW) {
        const bool ok = c0 + t < leaf.count;
        const int64_t s = (int64_t)leaf.first + c0 + t;
        T rx = T(0), ry = T(0), rz = T(0);
        if (ok) {
            const double4 pj = p64[s];
            rx = (T)(pj.x - cb.x);
            ry = (T)(pj.y - cb.y);
            rz = (T)(pj.z - cb.z);
        }
        T phi = T(0), ax = T(0), ay = T(0), az = T(0);
        for (int eb = e0; eb < e1; eb += 64) {
            const bool v = eb + lane < e1;
            farp_batch<T, NP, MT, G, BYTES>(v, v ? items[eb + lane] : 0, cb, cen, M, ids, offs,
                                            rows, rx, ry, rz, phi, ax, ay, az);
        }
#pragma unroll
        for (int d = TW; d < 64; d <<= 1) {
            phi += __shfl_xor(phi, d, 64);
            ax += __shfl_xor(ax, d, 64);
            ay += __shfl_xor(ay, d, 64);
            az += __shfl_xor(az, d, 64);
        }
        if (!red) {
            if (ok && lane < TW) {
                far[s] = phi;
                far[n + s] = ax;
                far[2 * n + s] = ay;
                far[3 * n + s] = az;
            }
            continue;
        }
        T* mine = red + (threadIdx.x >> 6) * 256 + lane;
        mine[0] = phi;
        mine[64] = ax;
        mine[128] = ay;
        mine[192] = az;
        __syncthreads();
        // wave c sums component c
        const int c = threadIdx.x >> 6;
        if (c < 4 && ok && lane < TW) {
            T a = red[64 * c + lane];
            for (int w = 1; w < (int)(blockDim.x >> 6); ++w) a += red[256 * w + 64 * c + lane];
            far[c * n + s] = a;
        }
        __syncthreads();
    }
}

// L2P at every target (Eq. 3 with its gradient, dR_n^m/dz = R_{n-1}^m,
// (d/dx + i d/dy) R_n^m = R_{n-1}^{m+1}) from the local expansion of its
// box's host cell (none outside the root), one thread per sorted target;
// ADD: add to far (the M2P terms written there first) instead of storing.
template <typename T, int NP, bool ADD>
__global__ void __launch_bounds__(256)
k_l2p(Targets tg, const double4* __restrict__ cen, const double* __restrict__ L, int ld,
      T* __restrict__ far) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = tg.n;
    if (s >= n) return;
    const int b = tg.box[tg.box_of[s]].host;
    T phi = T(0), ax = T(0), ay = T(0), az = T(0);
    if (b >= 0) {
        const double4 pj = tg.p64[s];
        const double4 q = cen[b];
        const double ihd = q.w;
        const T ux = (T)((pj.x - q.x) * ihd), uy = (T)((pj.y - q.y) * ihd),
                uz = (T)((pj.z - q.z) * ihd);
        const double* Lb = L + (int64_t)b * ld;
        T f = T(0), gz = T(0), gr = T(0), gi = T(0);
        stream_regular<T, NP>(ux, uy, uz, [&](int k, int l, T rr, T ri) {
            const T w = l == 0 ? T(1) : T(2);
            {
                T lr = cre<T>(Lb, k, l), li = cim<T>(Lb, k, l);
                f += w * (lr * rr - li * ri);
            }
            if (k + 1 < NP) {
                T ar = cre<T>(Lb, k + 1, l), ai = cim<T>(Lb, k + 1, l);
                gz += w * (ar * rr - ai * ri);
                if (l >= 1) {
                    T br = cre<T>(Lb, k + 1, l - 1), bi = cim<T>(Lb, k + 1, l - 1);
                    gr += br * rr - bi * ri;
                    gi += br * ri + bi * rr;
                }
                T cr = cre<T>(Lb, k + 1, l + 1), ci = cim<T>(Lb, k + 1, l + 1);
                gr -= cr * rr - ci * ri;
                gi += cr * ri + ci * rr;
            }
        });
        const T ih = (T)ihd, ih2 = ih * ih;
        phi = f * ih;
        ax = gr * ih2;
        ay = gi * ih2;
        az = gz * ih2;
    }
    if (ADD) {
        phi += far[s];
        ax += far[n + s];
        ay += far[2 * n + s];
        az += far[3 * n + s];
    }
    far[s] = phi;
    far[n + s] = ax;
    far[2 * n + s] = ay;
    far[3 * n + s] = az;
}

// geometric centre of a box as the reference point of its targets' offsets
__device__ inline double4 box_ref(const Root& r, const TBox& bx) {
    double c[3];
    cell_centre(r, box_cell(bx), c);
    return make_double4(c[0], c[1], c[2], 0.0);
}

// Lane groups of a box of `count` targets, and whether its list of n cells is
// a long one: more than `most` evaluations one after the other per lane.
__host__ __device__ constexpr int farp_groups(int count) {
    return count <= 4 ? 16 : count <= 8 ? 8 : count <= 16 ? 4 : count <= 32 ? 2 : 1;
}
__device__ __forceinline__ bool farp_long(int count, int n, int most) {
    return n / farp_groups(count) >= most;
}

#define FARP_GROUPS(C_, F) \
    if ((C_) <= 4)         \
        F(16);             \
    else if ((C_) <= 8)    \
        F(8);              \
    else if ((C_) <= 16)   \
        F(4);              \
    else if ((C_) <= 32)   \
        F(2);              \
    else                   \
        F(1);

// W-list M2P of the FMM, one wave per target leaf; MT: the multipoles'
// type (an FP32 copy for the FP32 path).  Short, uneven lists: a wave per
// leaf replaces the divergent per-particle loops.  (The treecode's long,
// even lists keep one thread per particle, k_treecode_far: there every lane
// has a target, while a wave per leaf of ~10 particles leaves lanes idle.)
// The boxes with long lists are left to k_farp_long.
template <typename T, int NP, typename MT>
__global__ void __launch_bounds__(256, sizeof(T) == 4 ? 6 : 1)
k_farp(const Root* __restrict__ root, Targets tg, const double4* __restrict__ cen,
       const int32_t* __restrict__ off, const int32_t* __restrict__ items,
       const MT* __restrict__ M, int most, T* __restrict__ far) {
    using V = typename Vec4<T>::type;
    using S = FarShape<NP, MT>;
    __shared__ int32_t sid[4][64];
    __shared__ V soff[4][64];
    __shared__ __align__(16) MT srow[4][S::FB * S::LD];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = blockIdx.x * 4 + w;
    if (li >= tg.nbox) return;  // uniform per wave
    const TBox bx = tg.box[li];
    const int row = list_row(tg, li, bx);
    const int e0 = off[row], e1 = off[row + 1];
    if (farp_long(bx.count, e1 - e0, most)) return;
    const double4 cb = box_ref(*root, bx);
#define FARP_BOX(G)                                                                           \
    farp_box<T, NP, MT, G>(bx, cb, cen, tg.p64, items, e0, e1, M, sid[w], soff[w], srow[w], \
                           far, tg.n, (T*)nullptr)
    FARP_GROUPS(bx.count, FARP_BOX)
#undef FARP_BOX
}

// the boxes with long lists, in no particular order (each is summed by itself)
__global__ void k_farp_find(Targets tg, const int32_t* __restrict__ off, int most,
                            int32_t* __restrict__ ids, int32_t* __restrict__ count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, lane = threadIdx.x & 63;
    bool lng = false;
    if (i < tg.nbox) {
        const TBox bx = tg.box[i];
        const int row = list_row(tg, i, bx);
        lng = farp_long(bx.count, off[row + 1] - off[row], most);
    }
    const uint64_t bal = __ballot(lng);
    if (!bal) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(count, __popcll(bal));
    at = __shfl(at, 0, 64) + __popcll(bal & lanes_below(lane));
    if (lng) ids[at] = i;
}

// Long lists: a block of 8 waves per box, each wave an eighth of the list,
// summed through LDS in wave order.  These are the large leaves beside finer
// ones, a few hundred to a few thousand boxes whose lists of 30 to 60 cells a
// wave would evaluate one after the other.  The grid loops over the boxes
// found.  W-list M2P, one wave per box -> with this split (4 and more
// evaluations in a row): 31623 uniform particles, p = 8: 160 -> 64 us; 200003
// Plummer, p = 10: 335 -> 179 us; 262147 uniform, p = 8, FP64: 514 -> 390 us.
// From 2^16 boxes on every list is a wave's own, the boxes being enough by
// themselves.  Around that line the split still gains on Plummer spheres and
// loses where many boxes have middling lists (far field at p = 8 in FP32 without
// -> with it, us): Plummer 30367 boxes 335 -> 251, 41066 461 -> 330, 64760 577
// -> 467, 108973 750 -> 699; uniform 112313 (9 cells a list) 664 -> 838; Plummer
// of 4.4e5 1020 -> 1290.
constexpr int kFarLongWaves = 8;
template <typename T, int NP, typename MT>
__global__ void __launch_bounds__(64 * kFarLongWaves)
k_farp_long(const Root* __restrict__ root, Targets tg, const double4* __restrict__ cen,
            const int32_t* __restrict__ off, const int32_t* __restrict__ items,
            const MT* __restrict__ M, const int32_t* __restrict__ ids,
            const int32_t* __restrict__ count, T* __restrict__ far) {
    using V = typename Vec4<T>::type;
    constexpr int NW = kFarLongWaves;
    // rows staged at once: half as many as a wave of k_farp
    using S = FarShape<NP, MT, 4096>;
    __shared__ int32_t sid[NW][64];
    __shared__ V soff[NW][64];
    __shared__ __align__(16) MT srow[NW][S::FB * S::LD];
    __shared__ T red[NW * 256];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = *count;
    for (int k = blockIdx.x; k < n; k += gridDim.x) {
        const int li = ids[k];
        const TBox bx = tg.box[li];
        const int row = list_row(tg, li, bx);
        const int e0 = off[row], len = off[row + 1] - e0;
        const int s0 = e0 + len * w / NW, s1 = e0 + len * (w + 1) / NW;
        const double4 cb = box_ref(*root, bx);
#define FARP_BOX(G)                                                                         \
    farp_box<T, NP, MT, G, 4096>(bx, cb, cen, tg.p64, items, s0, s1, M, sid[w], soff[w],    \
                                 srow[w], far, tg.n, red)
        FARP_GROUPS(bx.count, FARP_BOX)
#undef FARP_BOX
    }
}

// Treecode far field: M2P over the accepted list of the target's box, one
// thread per sorted target (neighbouring threads share a box and read the
// same cells); MT: FP32 copy of the multipoles for the FP32 path.
template <typename T, int NP, typename MT>
__global__ void __launch_bounds__(256)
k_treecode_far(Targets tg, const double4* __restrict__ cen, const int32_t* __restrict__ a_off,
               const int32_t* __restrict__ a_items, const MT* __restrict__ M, int ld,
               T* __restrict__ far) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = tg.n;
    if (s >= n) return;
    const int b = tg.box_of[s];
    const int row = list_row(tg, b, tg.box[b]);
    const double4 pj = tg.p64[s];
    T phi = T(0), ax = T(0), ay = T(0), az = T(0);
    for (int e = a_off[row]; e < a_off[row + 1]; ++e) {
        const int C = a_items[e];
        const double4 qc = cen[C];
        const double ic = qc.w;
        m2p_accumulate<T, NP>(M + (int64_t)C * ld, (T)((pj.x - qc.x) * ic),
                              (T)((pj.y - qc.y) * ic), (T)((pj.z - qc.z) * ic), (T)ic, phi, ax,
                              ay, az);
    }
    far[s] = phi;
    far[n + s] = ax;
    far[2 * n + s] = ay;
    far[3 * n + s] = az;
}

// ---------------------------------------------------------------------
// M2P at p = 3 (monopole, dipole, quadrupole: the treecode's quadrupole
// moments) in Cartesian form.  With the irregular harmonics of degree <= 2
// written out, S_0^0 = 1/r, S_1^0 = z/r^3, S_1^1 = -(x + iy)/r^3,
// S_2^0 = (3z^2 - r^2)/r^5, S_2^1 = -3z(x + iy)/r^5, S_2^2 = 3(x + iy)^2/r^5,
// the truncated expansion of a cell is
//   f(u) = q/r + (D.u)/r^3 + (u.Q.u)/r^5,
// q = M00, D = (-2 Re M11, 2 Im M11, M10) and the traceless symmetric
//   Q = [[6 Re M22 - M20, -6 Im M22, -3 Re M21],
//        [-6 Im M22, -6 Re M22 - M20, 3 Im M21],
//        [-3 Re M21, 3 Im M21, 2 M20]],
// the same function the degree-by-degree sum evaluates, and its gradient is
//   D/r^3 + 2 Q.u/r^5 - u (q/r^3 + 3 (D.u)/r^5 + 5 (u.Q.u)/r^7).
// Per cell, in units of the root's side S (u = (x - c)/h = (x - c)/S 2^level):
// D' = D h/S, Q' = 2 Q (h/S)^2, both exact, as (Dx, Dy, Dz, q), (Qxx, Qyy, Qxy,
// Qxz), Qyz and the FP64 centre (Qzz = -(Qxx + Qyy)): in FP32 one record of 64
// bytes, so that a wave that gathers 64 cells touches one line per cell.
// The sums hold q/r^2 with r down to 2^-21, and Q' carries 4^-level: with the
// masses as they come, both leave the FP32 range for sets whose fields do not
// (10^6 stars of 2e30 kg within 3e16 m sum to 1e39; masses of 1e-34 make
// subnormal Q').  So the moments are divided by the power of two next below the
// largest of them (k_moment_exp: over all cells, since with both signs the
// root's own may vanish), and the sums get it back, with 1/S and 1/S^2, in FP64
// where they are stored.  With moments of at most 2 a term is at most 2^43, and
// the thousands of a list stay 2^70 below the largest FP32 number.
// ---------------------------------------------------------------------
template <typename T>
struct alignas(sizeof(T) == 4 ? 64 : 32) Cart3 {
    typename Vec4<T>::type m0, m1;
    T qyz;
    double c[3];
};
static_assert(sizeof(Cart3<float>) == 64 && sizeof(Cart3<double>) == 96, "Cart3 records");

// maximum over a block of NW waves, in every thread
template <int NW>
__device__ __forceinline__ int block_max(int v) {
    __shared__ int wmax[NW];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = max(v, __shfl_xor(v, d, 64));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = v;
    __syncthreads();
    v = wmax[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) v = max(v, wmax[w]);
    return v;
}

// Exponent of the largest finite moment of degree <= 2, per block (INT_MIN:
// none but zeros).  16 lanes per row, so that a wave reads whole lines, and the
// largest magnitude kept, its exponent taken once.  At most 256 blocks, the
// exponents a block of k_cart3 reads; they are bound by the latency of the rows:
// 16 waves and four rows in flight, 71 -> 27 us at 5e5 cells.
constexpr int kMomentBlocks = 256, kMomentRows = 64;
__global__ void __launch_bounds__(16 * kMomentRows)
k_moment_exp(const double* __restrict__ M, int ld, int ncells, int32_t* __restrict__ part) {
    const int k = threadIdx.x & 15;
    double big = 0.0;
    if (k < 9) {
#pragma unroll 4
        for (int c = blockIdx.x * kMomentRows + (int)(threadIdx.x >> 4); c < ncells;
             c += gridDim.x * kMomentRows) {
            const double v = fabs(M[(int64_t)c * ld + k]);
            if (v < HUGE_VAL) big = fmax(big, v);
        }
    }
    const int e = block_max<kMomentRows / 4>(big > 0.0 ? ilogb(big) : INT_MIN);
    if (threadIdx.x == 0) part[blockIdx.x] = e;
}

// The records; part: the nparts exponents above; their maximum (0 without a
// non-zero moment) is written to *mexp.
template <typename TC>
__global__ void __launch_bounds__(256)
k_cart3(const Cell* __restrict__ cells, const double4* __restrict__ cen,
        const double* __restrict__ M, int ld, int ncells, const int32_t* __restrict__ part,
        int nparts, int32_t* __restrict__ mexp, Cart3<TC>* __restrict__ C) {
    int e = block_max<4>((int)threadIdx.x < nparts ? part[threadIdx.x] : INT_MIN);
    if (e == INT_MIN) e = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) *mexp = e;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncells) return;
    const double* X = M + (int64_t)c * ld;
    auto mom = [&](int k) { return ldexp(X[k], -e); };
    const double m00 = mom(ridx(0, 0, 0)), m10 = mom(ridx(1, 0, 0));
    const double m11r = mom(ridx(1, 1, 0)), m11i = mom(ridx(1, 1, 1));
    const double m20 = mom(ridx(2, 0, 0)), m21r = mom(ridx(2, 1, 0)), m21i = mom(ridx(2, 1, 1));
    const double m22r = mom(ridx(2, 2, 0)), m22i = mom(ridx(2, 2, 1));
    const double f = ldexp(1.0, -(int)cells[c].level), f2 = 2.0 * f * f;
    const double4 x = cen[c];
    Cart3<TC> o;
    o.m0 = {(TC)(-2.0 * m11r * f), (TC)(2.0 * m11i * f), (TC)(m10 * f), (TC)m00};
    o.m1 = {(TC)((6.0 * m22r - m20) * f2), (TC)((-6.0 * m22r - m20) * f2), (TC)(-6.0 * m22i * f2),
            (TC)(-3.0 * m21r * f2)};
    o.qyz = (TC)(3.0 * m21i * f2);
    o.c[0] = x.x;
    o.c[1] = x.y;
    o.c[2] = x.z;
    C[c] = o;
}

// One evaluation at v = (x - c)/S from the staged record of the cell (m2: Qyz
// and the offset).  With e = v.Q'.v / r^2,
//   f = (q + (D'.v + e/2) / r^2) / r,
//   grad f = (D' + Q'.v / r^2 - v t) / r^3,  t = q + (3 D'.v + 5/2 e) / r^2.
// In this order no power of 1/r beyond the third is formed: at the last level
// (r about 2^-21) the FP32 range still holds them, with moments of at most 2.
template <typename T, typename V>
__device__ __forceinline__ void m2p_cart3(const V& m0, const V& m1, T qyz, T qzz, T vx, T vy,
                                          T vz, T& phi, T& ax, T& ay, T& az) {
    const T dx = m0.x, dy = m0.y, dz = m0.z, q = m0.w;
    const T qxx = m1.x, qyy = m1.y, qxy = m1.z, qxz = m1.w;
    const T r2 = fma(vx, vx, fma(vy, vy, vz * vz));
    const T ir = rsqrt_fast(r2), ir2 = ir * ir, ir3 = ir * ir2;
    const T du = fma(dx, vx, fma(dy, vy, dz * vz));
    const T qx = fma(qxx, vx, fma(qxy, vy, qxz * vz));
    const T qy = fma(qxy, vx, fma(qyy, vy, qyz * vz));
    const T qz = fma(qxz, vx, fma(qyz, vy, qzz * vz));
    const T e = fma(vx, qx, fma(vy, qy, vz * qz)) * ir2;
    phi = fma(ir, fma(ir2, fma(T(0.5), e, du), q), phi);
    const T t = fma(ir2, fma(T(2.5), e, T(3) * du), q);
    ax = fma(ir3, fma(-t, vx, fma(ir2, qx, dx)), ax);
    ay = fma(ir3, fma(-t, vy, fma(ir2, qy, dy)), ay);
    az = fma(ir3, fma(-t, vz, fma(ir2, qz, dz)), az);
}

// The targets of a lane: offsets from the box's reference point in units of
// the root's side, and sums.
template <typename T, int TPL>
struct FarTargets {
    T x[TPL], y[TPL], z[TPL];
    T phi[TPL], ax[TPL], ay[TPL], az[TPL];
};

// One batch of list cells of a target leaf: lane j (j < B) offers cell k
// when `valid`; the valid cells are packed at the front of the wave's LDS
// slice, each as its moments and the offset from the cell's centre to the
// box's reference point cb in units of the root's side (is = 1/S), formed in
// FP64.  Lane g * TW + t (g < G) takes targets t, t + TW, .. and the packed
// cells g, g + G, ...; the slots past the batch up to the next multiple of G
// (at most B <= 64, a multiple of G) hold zero moments far away, whose terms
// are exactly zero.  Lanes past G * TW compute on clamped slots and are never
// summed.
template <typename T, int TPL>
__device__ __forceinline__ void far3_batch(bool valid, int k, const double4& cb, double is,
                                           const Cart3<T>* __restrict__ C,
                                           typename Vec4<T>::type* sh, int G, int g,
                                           FarTargets<T, TPL>& me) {
    using V = typename Vec4<T>::type;
    const int lane = threadIdx.x & 63;
    const uint64_t bal = __ballot(valid);
    const int nb = __popcll(bal);
    if (nb == 0) return;  // uniform per wave
    V r0{}, r1{}, r2{};
    if (valid) {
        const Cart3<T> c = C[k];
        r0 = c.m0;
        r1 = c.m1;
        r2 = V{c.qyz, (T)((cb.x - c.c[0]) * is), (T)((cb.y - c.c[1]) * is),
               (T)((cb.z - c.c[2]) * is)};
    }
    const int pos = __popcll(bal & lanes_below(lane));
    const int nr = (nb + G - 1) / G * G;
    wave_lds_fence();
    if (valid) {
        sh[pos] = r0;
        sh[64 + pos] = r1;
        sh[128 + pos] = r2;
    }
    if (lane >= nb && lane < nr) {
        const V z{};
        sh[lane] = z;
        sh[64 + lane] = z;
        sh[128 + lane] = V{T(0), T(1.2345e15), T(0), T(0)};
    }
    wave_lds_fence();
#pragma unroll 2
    for (int j0 = 0; j0 < nr; j0 += G) {
        const int j = min(j0 + g, 63);
        const V a = sh[j], b = sh[64 + j], d = sh[128 + j];
        const T qzz = -(b.x + b.y);
#pragma unroll
        for (int i = 0; i < TPL; ++i)
            m2p_cart3<T>(a, b, d.x, qzz, me.x[i] + d.y, me.y[i] + d.z, me.z[i] + d.w, me.phi[i],
                         me.ax[i], me.ay[i], me.az[i]);
    }
}

// The far field of one target box.  Lane groups are sized to the box:
// TW = ceil(min(count, 64 TPL) / TPL) lanes of TPL targets per group, G = 64 /
// TW groups (a leaf of 10 particles keeps 60 lanes busy where power-of-two
// groups of 16 kept 40), batches of B = G * (64 / G) cells.  WALK: the M2P
// cells are read from the FMM lists (the box's CSR items: W, and V for a box
// without sources; then the V slots of cell b, the box's leaf or its host, and
// of each ancestor, the non-empty ones queued in the wave's id ring `q` so
// that every batch but the last is full); otherwise from the box's CSR list
// items[e0, e1).
template <typename T, bool WALK, int TPL>
__device__ __forceinline__ void far3_box(const Cell* __restrict__ cells, int b, const TBox& leaf,
                                          const double4& cb, double is,
                                          const double4* __restrict__ p64,
                                          const int32_t* __restrict__ items, int e0, int e1,
                                          const int32_t* __restrict__ vsrc,
                                          const Cart3<T>* __restrict__ C, int mexp,
                                          typename Vec4<T>::type* sh, int* q,
                                          T* __restrict__ far, int64_t n) {
    const int lane = threadIdx.x & 63;
    const int TW = (min(leaf.count, 64 * TPL) + TPL - 1) / TPL;
    const int G = 64 / TW, B = G * (64 / G);
    const int g = lane / TW, t = lane - g * TW;  // g == G: an idle lane
    for (int c0 = 0; c0 < leaf.count; c0 += TW * TPL) {
        FarTargets<T, TPL> me;
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            me.x[i] = me.y[i] = me.z[i] = T(0);
            const int k = c0 + i * TW + t;
            if (g < G && k < leaf.count) {
                const double4 pj = p64[leaf.first + k];
                me.x[i] = (T)((pj.x - cb.x) * is);
                me.y[i] = (T)((pj.y - cb.y) * is);
                me.z[i] = (T)((pj.z - cb.z) * is);
            }
            me.phi[i] = me.ax[i] = me.ay[i] = me.az[i] = T(0);
        }
        auto batch = [&](bool valid, int k) {
            far3_batch<T, TPL>(valid, k, cb, is, C, sh, G, g, me);
        };
        for (int eb = e0; eb < e1; eb += B) {
            const bool v = lane < B && eb + lane < e1;
            batch(v, v ? items[eb + lane] : 0);
        }
        if (WALK) {
            // ring of 256 ids: at most B - 1 + 64 <= 127 are queued at once
            const uint64_t below = lanes_below(lane);
            int head = 0, tail = 0;
            for (int a = b; a >= 0; a = cells[a].parent) {
                const int32_t* row = vsrc + (int64_t)a * 216;
                for (int q0 = 0; q0 < 216; q0 += 64) {
                    const int k = q0 + lane < 216 ? row[q0 + lane] : -1;
                    const uint64_t bal = __ballot(k >= 0);
                    wave_lds_fence();
                    if (k >= 0) q[(tail + __popcll(bal & below)) & 255] = k;
                    tail += __popcll(bal);
                    wave_lds_fence();
                    while (tail - head >= B) {
                        batch(lane < B, q[(head + lane) & 255]);
                        head += B;
                    }
                }
            }
            if (tail > head) batch(lane < tail - head, q[(head + lane) & 255]);
        }
        // group 0 adds the other groups' partial sums of its targets
        const double i1 = ldexp(is, mexp), i2 = i1 * is;
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            T sphi = me.phi[i], sax = me.ax[i], say = me.ay[i], saz = me.az[i];
            for (int h = 1; h < G; ++h) {
                const int src = h * TW + (t < TW ? t : 0);
                sphi += __shfl(me.phi[i], src, 64);
                sax += __shfl(me.ax[i], src, 64);
                say += __shfl(me.ay[i], src, 64);
                saz += __shfl(me.az[i], src, 64);
            }
            const int k = c0 + i * TW + t;
            if (g == 0 && k < leaf.count) {
                const int64_t s = (int64_t)leaf.first + k;
                far[s] = (T)((double)sphi * i1);
                far[n + s] = (T)((double)sax * i2);
                far[2 * n + s] = (T)((double)say * i2);
                far[3 * n + s] = (T)((double)saz * i2);
            }
        }
    }
}

// Treecode far field at p = 3 from the Cartesian moments (k_cart3), one
// wave per target box, lane groups sized to its target count.  off/items:
// the box's M2P list (Barnes-Hut), or with WALK its FMM-list part (W, and V
// for a box without sources), the V lists of the cells above being read
// from vsrc.  Bound by the VALU issue of the evaluations: 43 slots each in
// units of the root's side (moments scaled once per cell), where powers of 1/r
// up to the seventh in units of every cell's own side took 56.  In whole
// evaluations, 2^22 Plummer, Barnes-Hut lists 14.2 -> 11.7 to 13.1 ms between
// runs (52 VALU instructions per evaluation with the staging, issued every 3.4
// cycles), FMM lists of 2^20 2.21 -> 1.81 ms.
template <typename T, bool WALK>
__global__ void __launch_bounds__(256, sizeof(T) == 4 ? 6 : 3)
k_treecode_far3(const Cell* __restrict__ cells, const Root* __restrict__ root, Targets tg,
                const int32_t* __restrict__ off, const int32_t* __restrict__ items,
                const int32_t* __restrict__ vsrc, const Cart3<T>* __restrict__ C,
                const int32_t* __restrict__ mexp, T* __restrict__ far) {
    using V = typename Vec4<T>::type;
    __shared__ V shm[4][192];
    __shared__ int idq[4][WALK ? 256 : 1];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = blockIdx.x * 4 + w;
    if (li >= tg.nbox) return;  // uniform per wave
    const TBox bx = tg.box[li];
    if (bx.count <= 0) return;
    const int row = list_row(tg, li, bx);
    const double4 cb = box_ref(*root, bx);
    const double is = 1.0 / cell_side(*root, 0);
    const int walk_from = bx.leaf >= 0 ? bx.leaf : bx.host;
    if (bx.count <= 2)
        far3_box<T, WALK, 1>(cells, walk_from, bx, cb, is, tg.p64, items, off[row],
                             off[row + 1], vsrc, C, *mexp, shm[w], idq[w], far, tg.n);
    else
        far3_box<T, WALK, 2>(cells, walk_from, bx, cb, is, tg.p64, items, off[row],
                             off[row + 1], vsrc, C, *mexp, shm[w], idq[w], far, tg.n);
}

__global__ void k_zero_i32(int32_t* __restrict__ p) {
    if (threadIdx.x == 0) *p = 0;
}

__global__ void k_to_float(const double* __restrict__ a, int64_t n, float* __restrict__ b) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}

// ---------------------------------------------------------------------
// M2L operator tables
// ---------------------------------------------------------------------
// gridDim.y blocks per offset class (343 classes, 27 of them adjacent
// offsets that stay zero).  Each block tabulates, for its class, the Sec. 5.2
// quantity (N-|M|)! P_N^|M|(cos a) / rho^{N+1} for N <= 2p-2 (Eqs. 7-9) and
// cos(M b), sin(M b) in LDS, then its threads fill a share of the real
// entries in the order they are stored (consecutive threads, consecutive
// addresses; the padding is written as zeros).  Layouts: FP64
// T64[cls][ri][ro], or the matrix-core chunks [cls][rb][q][lane][E] holding
// T[16 rb + (lane & 15)][KS q + 4 r + (lane >> 4)] at element r.
__global__ void __launch_bounds__(256)
k_m2l_ops(int p, int layout, void* __restrict__ T, int RB, int KQ) {
    // layout 0: FP64 [class][ri][ro] (vector units); 1: FP32 matrix-core
    // chunks (E = 4, KS = 16); 2: FP64 matrix-core chunks (E = 2, KS = 8).
    // The r-major order puts the padding of the last block into whole
    // products, which the kernel skips.
    __shared__ M2lClassTable tab;
    const int P = p * p;
    const int cls = blockIdx.x;
    const bool far = tab.fill(p, cls);
    const int64_t per = (int64_t)P * P;
    const int64_t step = (int64_t)gridDim.y * blockDim.x;
    const int64_t first = (int64_t)blockIdx.y * blockDim.x + threadIdx.x;
    if (layout == 0) {
        for (int64_t e = first; e < per; e += step) {
            const int ri = (int)(e / P), ro = (int)(e % P);
            ((double*)T)[(int64_t)cls * per + e] = far ? tab.entry(ro, ri) : 0.0;
        }
        return;
    }
    const int E = layout == 1 ? 4 : 2, KS = layout == 1 ? 16 : 8;
    const int64_t tot = (int64_t)RB * KQ * 64 * E;
    for (int64_t o = first; o < tot; o += step) {
        const int r = (int)(o % E);
        const int64_t u = o / E;
        const int lane = (int)(u % 64), q = (int)((u / 64) % KQ), rb = (int)(u / (64 * KQ));
        const int ro = 16 * rb + (lane & 15), ri = KS * q + 4 * r + (lane >> 4);
        const double val = (far && ro < P && ri < P) ? tab.entry(ro, ri) : 0.0;
        if (layout == 1)
            ((float*)T)[(int64_t)cls * tot + o] = (float)val;
        else
            ((double*)T)[(int64_t)cls * tot + o] = val;
    }
}

// Low-precision operators.  pass 0: bexp[j] = max exponent of T_{jn} 2^{mu_n}
// over classes and columns; pass 1: T' = T 2^{mu_n - b_j}, b_j = bexp[j] + 1,
// split into hi and lo (lo may be null) in the layout
// [cls][rb][q][lane][8], element (16 rb + (lane & 15), 32 q + 8 (lane >> 4) + j).
template <typename T16>
__global__ void __launch_bounds__(256)
k_m2l_ops_lp(int p, int pass, int RB, int KQ, int32_t* __restrict__ bexp,
             T16* __restrict__ hi, T16* __restrict__ lo) {
    __shared__ M2lClassTable tab;
    __shared__ int bmax[HFMM_MAX_P];  // pass 0: block maximum per output degree
    const int P = p * p;
    const int cls = blockIdx.x;
    if (threadIdx.x < HFMM_MAX_P) bmax[threadIdx.x] = INT_MIN;
    const bool far = tab.fill(p, cls);
    const int R = 16 * RB, K = 32 * KQ;
    const int per = R * K;
    for (int e = blockIdx.y * blockDim.x + threadIdx.x; e < per; e += gridDim.y * blockDim.x) {
        const int ro = e / K, ri = e % K;
        double val = 0.0;
        int j = 0, n = 0;
        if (far && ro < P && ri < P) {
            val = tab.entry(ro, ri);
            j = tab.dec[ro] & 255;
            n = tab.dec[ri] & 255;
        }
        if (pass == 0) {
            if (val != 0.0) atomicMax(&bmax[j], ilogb(fabs(val)) + m2l_mu(n));
            continue;
        }
        double t = val == 0.0 ? 0.0 : ldexp(val, m2l_mu(n) - (bexp[j] + 1));
        const int rb = ro / 16, il = ro % 16;
        const int q = ri / 32, g = (ri % 32) / 8, jj = ri % 8;
        const int64_t idx = ((((int64_t)cls * RB + rb) * KQ + q) * 64 + g * 16 + il) * 8 + jj;
        const T16 h = (T16)(float)t;
        hi[idx] = h;
        if (lo) lo[idx] = (T16)(float)(t - (double)(float)h);
    }
    if (pass == 0) {
        __syncthreads();
        if ((int)threadIdx.x < p && bmax[threadIdx.x] != INT_MIN)
            atomicMax(&bexp[threadIdx.x], bmax[threadIdx.x]);
    }
}

void run_m2l_ops_lp(int p, int precision, int RB, int KQ, int32_t* bexp, void* hi, void* lo,
                    hipStream_t s) {
    const bool bf = precision == HFMM_M2L_BF16 || precision == HFMM_M2L_BF16X3;
    // four blocks per class for the larger tables: at p = 12 one left 343 blocks
    // with 96 entries a thread, 2 x 141 us instead of 2 x 88
    const int split = p >= 6 ? 4 : 1;
    for (int pass = 0; pass < 2; ++pass) {
        if (bf)
            hipLaunchKernelGGL((k_m2l_ops_lp<__bf16>), dim3(343, split), dim3(256), 0, s, p, pass,
                               RB, KQ, bexp, (__bf16*)hi, (__bf16*)lo);
        else
            hipLaunchKernelGGL((k_m2l_ops_lp<_Float16>), dim3(343, split), dim3(256), 0, s, p, pass,
                               RB, KQ, bexp, (_Float16*)hi, (_Float16*)lo);
        LAUNCH_CHECK();
    }
}

// pack Mt (FP64, p*p per cell) into the M2L operand: ld = Kp (zero padded),
// one extra zero row at index ncells for absent sources
template <typename TO>
// Rows of the matrix-core M2L operand.  Within each block of 4 NR (NR = 4
// floats or 2 doubles per 16-byte chunk), position NR g + r holds element
// 4 NR q + 4 r + g (the operator's r-major contraction order); the zero row
// ncells stands for an absent source.
__global__ void k_pack(const double* __restrict__ M, int ldm, int ncells, int P, int ld,
                       TO* __restrict__ out) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t tot = (int64_t)(ncells + 1) * ld;
    if (gid >= tot) return;
    const int c = (int)(gid / ld), pos = (int)(gid % ld);
    // blocks of 16 floats (4 lane groups x 4 products) or 8 doubles (x 2)
    constexpr int NR = 16 / sizeof(TO);
    const int blk = pos / (4 * NR), w = pos % (4 * NR);
    const int k = blk * 4 * NR + 4 * (w % NR) + w / NR;
    double v = (c < ncells && k < P) ? M[(int64_t)c * ldm + k] : 0.0;
    out[gid] = (TO)v;
}

__device__ inline double factorial_d(int n) {
    double f = 1.0;
    for (int i = 2; i <= n; ++i) f *= (double)i;
    return f;
}

// device basis -> the paper's normalisation:
//   M_n^m = h^n Mt_n^m / A_n^m,  L_n^m = A_n^m Lt_n^m / h^{n+1}
__global__ void k_export(const double* __restrict__ X, int ld, int ncells, int p,
                         const double4* __restrict__ cen, int which,
                         double* __restrict__ out) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int NT = p * (p + 1) / 2;
    if (gid >= (int64_t)ncells * NT) return;
    const int c = (int)(gid / NT), t = (int)(gid % NT);
    int n = 0;
    while ((n + 1) * (n + 2) / 2 <= t) ++n;
    const int m = t - n * (n + 1) / 2;
    const double h = 1.0 / cen[c].w;
    const double A = 1.0 / sqrt(factorial_d(n - m) * factorial_d(n + m));
    double hn = 1.0;
    for (int i = 0; i < n; ++i) hn *= h;
    const double f = which == 0 ? hn / A : A / (hn * h);
    const double* Xc = X + (int64_t)c * ld;
    out[gid * 2] = f * Xc[ridx(n, m, 0)];
    out[gid * 2 + 1] = m == 0 ? 0.0 : f * Xc[ridx(n, m, 1)];
}

// ---------------------------------------------------------------------
// dispatch over p
// ---------------------------------------------------------------------
#define HFMM_DISPATCH_P(p, F)  \
    switch (p) {               \
        case 1: F(1); break;   \
        case 2: F(2); break;   \
        case 3: F(3); break;   \
        case 4: F(4); break;   \
        case 5: F(5); break;   \
        case 6: F(6); break;   \
        case 7: F(7); break;   \
        case 8: F(8); break;   \
        case 9: F(9); break;   \
        case 10: F(10); break; \
        case 11: F(11); break; \
        case 12: F(12); break; \
        case 13: F(13); break; \
        case 14: F(14); break; \
        case 15: F(15); break; \
        case 16: F(16); break; \
        default: throw Status{HFMM_E_UNSUPPORTED}; \
    }

void fill_masses(Tree& t, const double* m, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_masses, dim3(grid_for(t.n, 256)), dim3(256), 0, s, t.n, t.perm,
                       m, t.xs, t.ys, t.zs, t.p32, t.p64, t.status);
    LAUNCH_CHECK();
}

void compute_centres(Tree& t, int method, hipStream_t s) {
    double4* cen = (double4*)t.cen;
    if (method == HFMM_TREECODE) {
        double4* w4 = t.arena.down<double4>(t.ncells);
        for (int l = t.depth; l >= 0; --l) {
            int c0 = t.level_start[l], c1 = t.level_start[l + 1];
            hipLaunchKernelGGL(k_com_level, dim3(grid_for(c1 - c0, 128)), dim3(128), 0, s,
                               t.cells, c0, c1, t.p64, t.root, w4, cen);
            LAUNCH_CHECK();
        }
    } else {
        hipLaunchKernelGGL(k_centres_geometric, dim3(grid_for(t.ncells, 256)), dim3(256), 0, s,
                           t.cells, t.ncells, t.root, cen);
        LAUNCH_CHECK();
    }
}

void run_p2m(Tree& t, int p, bool fp64, hipStream_t s) {
    const int threads = t.nleaves * 8;
#define P2M_CASE(NP)                                                                       \
    if (fp64)                                                                              \
        hipLaunchKernelGGL((k_p2m<double, NP>), dim3(grid_for(threads, 256)), dim3(256), 0, \
                           s, t.cells, t.leaves, t.nleaves, (const double4*)t.cen, t.p64,   \
                           t.M, t.ldm);                                                     \
    else                                                                                    \
        hipLaunchKernelGGL((k_p2m<float, NP>), dim3(grid_for(threads, 256)), dim3(256), 0,  \
                           s, t.cells, t.leaves, t.nleaves, (const double4*)t.cen, t.p64,   \
                           t.M, t.ldm);
    HFMM_DISPATCH_P(p, P2M_CASE);
#undef P2M_CASE
    LAUNCH_CHECK();
}

void run_shift_octants(int p, double2* tab, hipStream_t s) {
#define SH_CASE(NP) hipLaunchKernelGGL((k_shift_octants<NP>), dim3(1), dim3(64), 0, s, tab);
    HFMM_DISPATCH_P(p, SH_CASE);
#undef SH_CASE
    LAUNCH_CHECK();
}

// M2M with a shift vector per child (centres of mass, treecode)
void run_m2m(Tree& t, int p, hipStream_t s) {
    const int NT = p * (p + 1) / 2;
    double2* tab = t.arena.down<double2>((size_t)t.ncells * NT);
#define SH_CASE(NP)                                                                           \
    hipLaunchKernelGGL((k_shift_children<NP>), dim3(grid_for(t.ncells, 128)), dim3(128), 0, s, \
                       t.cells, t.ncells, (const double4*)t.cen, tab);
    HFMM_DISPATCH_P(p, SH_CASE);
#undef SH_CASE
    LAUNCH_CHECK();
    for (int l = t.depth - 1; l >= 0; --l) {
        int c0 = t.level_start[l], c1 = t.level_start[l + 1];
        int64_t threads = (int64_t)(c1 - c0) * NT;
#define M2M_CASE(NP)                                                                     \
    hipLaunchKernelGGL((k_m2m<NP>), dim3(grid_for(threads, 128)), dim3(128), 0, s, t.cells, \
                       c0, c1, tab, 1, t.M, t.ldm);
        HFMM_DISPATCH_P(p, M2M_CASE);
#undef M2M_CASE
        LAUNCH_CHECK();
    }
}

void run_m2l_ops(Tree& t, int p, int layout, void* T, int RB, int KQ, hipStream_t s) {
    // several blocks per class for the larger tables (each recomputes the
    // class's small Legendre table)
    const int split = p >= 6 ? 4 : 1;
    hipLaunchKernelGGL(k_m2l_ops, dim3(343, split), dim3(256), 0, s, p, layout, T, RB, KQ);
    LAUNCH_CHECK();
}

void run_pack(const double* M, int ldm, int ncells, int P, int ld, void* out, bool fp64,
              hipStream_t s) {
    const int64_t tot = (int64_t)(ncells + 1) * ld;
    if (fp64)
        hipLaunchKernelGGL((k_pack<double>), dim3(grid_for(tot, 256)), dim3(256), 0, s, M, ldm,
                           ncells, P, ld, (double*)out);
    else
        hipLaunchKernelGGL((k_pack<float>), dim3(grid_for(tot, 256)), dim3(256), 0, s, M, ldm,
                           ncells, P, ld, (float*)out);
    LAUNCH_CHECK();
}

void run_p2l(Tree& t, int p, bool fp64, double* LX, hipStream_t s) {
    if (t.n_x == 0 || t.n_xcells == 0) return;
#define P2L_CASE(NP)                                                                         \
    if (fp64)                                                                                \
        hipLaunchKernelGGL((k_p2l<double, NP>), dim3(t.n_xcells), dim3(64), 0, s, t.cells,   \
                           t.x_cells, t.x_off, t.x_items, (const double4*)t.cen, t.p64, LX,  \
                           t.ldm);                                                           \
    else                                                                                     \
        hipLaunchKernelGGL((k_p2l<float, NP>), dim3(t.n_xcells), dim3(64), 0, s, t.cells,    \
                           t.x_cells, t.x_off, t.x_items, (const double4*)t.cen, t.p64, LX,  \
                           t.ldm);
    HFMM_DISPATCH_P(p, P2L_CASE);
#undef P2L_CASE
    LAUNCH_CHECK();
}

// FP32 copy of the multipoles (same layout) for the FP32 M2P
static const float* m_as_float(Tree& t, hipStream_t s) {
    const int64_t nel = (int64_t)t.ncells * t.ldm;
    float* m = t.arena.down<float>(nel);
    hipLaunchKernelGGL(k_to_float, dim3(grid_for(nel, 256)), dim3(256), 0, s, t.M, nel, m);
    LAUNCH_CHECK();
    return m;
}

// FMM far field: M2P over the boxes' far lists (the W lists; V too for
// boxes without sources), one wave per target box, then L2P added at every
// target
void run_far(Tree& t, const Targets& tg, int p, bool fp64, const int32_t* off,
             const int32_t* items, int64_t nitems, void* far, hipStream_t s) {
    if (tg.n == 0) return;
    const bool w = nitems > 0;
    const float* M32 = (!fp64 && w) ? m_as_float(t, s) : nullptr;
    const dim3 grid(grid_for(tg.nbox, 4)), block(256), pgrid(grid_for(tg.n, 256));
    const dim3 lgrid(std::min(tg.nbox, 1024)), lblock(64 * kFarLongWaves);
    const double4* cen = (const double4*)t.cen;
    // the boxes with long lists, found on the device
    const bool split = w && tg.nbox < (1 << 16);
    const int most = split ? 4 : INT32_MAX;
    int32_t *lids = nullptr, *lcount = nullptr;
    if (split) {
        lcount = t.arena.down<int32_t>(1 + (size_t)tg.nbox);
        lids = lcount + 1;
        hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, s, lcount);
        LAUNCH_CHECK();
        hipLaunchKernelGGL(k_farp_find, dim3(grid_for(tg.nbox, 256)), block, 0, s, tg, off, most,
                           lids, lcount);
        LAUNCH_CHECK();
    }
#define FAR_CASE(NP)                                                                          \
    if (fp64) {                                                                               \
        if (w) {                                                                              \
            if (split)                                                                        \
                hipLaunchKernelGGL((k_farp_long<double, NP, double>), lgrid, lblock, 0, s, t.root,  \
                               tg, cen, off, items, t.M, lids, lcount, (double*)far);          \
            hipLaunchKernelGGL((k_farp<double, NP, double>), grid, block, 0, s, t.root, tg,     \
                               cen, off, items, t.M, most, (double*)far);                      \
        }                                                                                     \
        if (w)                                                                                \
            hipLaunchKernelGGL((k_l2p<double, NP, true>), pgrid, block, 0, s, tg, cen, t.L,     \
                               t.ldm, (double*)far);                                           \
        else                                                                                  \
            hipLaunchKernelGGL((k_l2p<double, NP, false>), pgrid, block, 0, s, tg, cen, t.L,    \
                               t.ldm, (double*)far);                                           \
    } else {                                                                                  \
        if (w) {                                                                              \
            if (split)                                                                        \
                hipLaunchKernelGGL((k_farp_long<float, NP, float>), lgrid, lblock, 0, s, t.root,    \
                               tg, cen, off, items, M32, lids, lcount, (float*)far);           \
            hipLaunchKernelGGL((k_farp<float, NP, float>), grid, block, 0, s, t.root, tg, cen,  \
                               off, items, M32, most, (float*)far);                            \
        }                                                                                     \
        if (w)                                                                                \
            hipLaunchKernelGGL((k_l2p<float, NP, true>), pgrid, block, 0, s, tg, cen, t.L,      \
                               t.ldm, (float*)far);                                            \
        else                                                                                  \
            hipLaunchKernelGGL((k_l2p<float, NP, false>), pgrid, block, 0, s, tg, cen, t.L,     \
                               t.ldm, (float*)far);                                            \
    }
    HFMM_DISPATCH_P(p, FAR_CASE);
#undef FAR_CASE
    LAUNCH_CHECK();
}

// Treecode far field over the boxes' M2P lists off/items; walk: over the FMM
// lists at p = 3 the lists hold only the boxes' own part and the V lists of
// the cells above are read directly
void run_treecode_far(Tree& t, const Targets& tg, int p, bool fp64, bool walk,
                      const int32_t* off, const int32_t* items, void* far, hipStream_t s) {
    if (tg.n == 0) return;
    const double4* cen = (const double4*)t.cen;
    if (p == 3) {  // quadrupole moments: the Cartesian form
        const dim3 grid(grid_for(tg.nbox, 4)), block(256);
        const int nparts = std::min(kMomentBlocks, grid_for(t.ncells, kMomentRows));
        int32_t* mexp = t.arena.down<int32_t>(1 + kMomentBlocks);
        hipLaunchKernelGGL(k_moment_exp, dim3(nparts), dim3(16 * kMomentRows), 0, s, t.M, t.ldm,
                           t.ncells, mexp + 1);
        LAUNCH_CHECK();
#define FAR3(TT, W)                                                                            \
    hipLaunchKernelGGL((k_treecode_far3<TT, W>), grid, block, 0, s, t.cells, t.root, tg, off,  \
                       items, t.vsrc, c, mexp, (TT*)far)
#define FAR3_T(TT)                                                                             \
    {                                                                                          \
        Cart3<TT>* c = t.arena.down<Cart3<TT>>(t.ncells);                                      \
        hipLaunchKernelGGL(k_cart3<TT>, dim3(grid_for(t.ncells, 256)), dim3(256), 0, s,        \
                           t.cells, cen, t.M, t.ldm, t.ncells, mexp + 1, nparts, mexp, c);     \
        LAUNCH_CHECK();                                                                        \
        if (walk)                                                                              \
            FAR3(TT, true);                                                                    \
        else                                                                                   \
            FAR3(TT, false);                                                                   \
    }
        if (fp64)
            FAR3_T(double)
        else
            FAR3_T(float)
#undef FAR3_T
#undef FAR3
        LAUNCH_CHECK();
        return;
    }
    if (walk) throw Status{HFMM_E_STATE};  // other orders take full lists
    // other orders: the spherical form, one thread per target
    const float* M32 = fp64 ? nullptr : m_as_float(t, s);
#define TF_CASE(NP)                                                                            \
    if (fp64)                                                                                  \
        hipLaunchKernelGGL((k_treecode_far<double, NP, double>), dim3(grid_for(tg.n, 256)),     \
                           dim3(256), 0, s, tg, cen, off, items, t.M, t.ldm, (double*)far);    \
    else                                                                                       \
        hipLaunchKernelGGL((k_treecode_far<float, NP, float>), dim3(grid_for(tg.n, 256)),       \
                           dim3(256), 0, s, tg, cen, off, items, M32, t.ldm, (float*)far);
    HFMM_DISPATCH_P(p, TF_CASE);
#undef TF_CASE
    LAUNCH_CHECK();
}

void run_export(const double* X, int ld, int ncells, int p, const double* cen, int which,
                double* out, hipStream_t s) {
    const int64_t tot = (int64_t)ncells * p * (p + 1) / 2;
    hipLaunchKernelGGL(k_export, dim3(grid_for(tot, 256)), dim3(256), 0, s, X, ld, ncells, p,
                       (const double4*)cen, which, out);
    LAUNCH_CHECK();
}

}  // namespace hfmm
