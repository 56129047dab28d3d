// Near field (P2P, Sec. 5.1) and the direct sum.
//
// Per pair: a_i += m_j (x_j - x_i) / r^3 and phi_i += m_j / r with one
// reciprocal square root (Listing 1 of Sec. 5.1 plus the potential), pairs
// at r^2 == 0 skipped.  The paper gives each target cell a thread block and
// pads the targets to the block size (Secs. 3 and 5.1); leaves here hold up
// to 64 particles (about 32 on average, clustered data about 10), so one
// 64-lane wave takes one target leaf: TW lanes hold TPL targets each, and the
// 64 / TW lane groups share the sources and are summed with cross-lane
// shuffles at the end.  The sources of consecutive list cells are packed into
// chunks of 64 (x, y, z, m) records in LDS, so a chunk is full however few
// particles each cell holds; the target leaf itself, whose coincident points
// need the r^2 == 0 test, is taken on its own.  Each wave owns its LDS slice,
// so there is no block-wide barrier.
#include "common.hpp"
#include "expansions.hpp"

namespace hfmm {


// ZERO: the pair may coincide (r^2 == 0, skipped).  Coincident points share
// a key, hence a leaf, so only a leaf with itself needs the test.  Across
// leaves FP64 separations are never 0; FP32 ones can round to 0 for points
// closer than FP32 resolves at the leaf size, and r^2 starts from 1e-24
// there so that the (then meaningless) pair stays finite: r^2 (+ eps^2) is
// one chain of fused multiply-adds from that start, which leaves r^2 above
// 2e-17 unchanged and needs no separate clamp instruction in the loop.
template <typename T, bool SOFT, bool ZERO>
__device__ __forceinline__ void pair(T xi, T yi, T zi, const typename Vec4<T>::type& s,
                                     T eps2, T& phi, T& ax, T& ay, T& az) {
    const T dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;
    T rinv;
    if (ZERO) {  // the test is on the unsoftened r^2
        const T r2 = fma(dx, dx, fma(dy, dy, dz * dz));
        rinv = rsqrt_fast(SOFT ? r2 + eps2 : r2);
        rinv = r2 > T(0) ? rinv : T(0);
    } else {
        const T r0 = SOFT ? eps2 : (sizeof(T) == 4 ? T(1e-24) : T(0));
        rinv = rsqrt_fast(fma(dx, dx, fma(dy, dy, fma(dz, dz, r0))));
    }
    const T mr = s.w * rinv;
    phi += mr;
    const T sc = mr * rinv * rinv;
    ax += dx * sc;
    ay += dy * sc;
    az += dz * sc;
}

// The targets of a lane: positions and sums.
template <typename T, int TPL>
struct LaneTargets {
    T x[TPL], y[TPL], z[TPL];
    T phi[TPL], ax[TPL], ay[TPL], az[TPL];
};

// Sum over the sources staged in sh[0, nl): lane = g * TW + t, group g of the
// G = 64 / TW takes sources g, g + G, ..., each read once for the lane's TPL
// targets.  Entries past nl up to the next multiple of G are padding (mass 0,
// far away).
template <typename T, int G, int TPL, bool SOFT, bool ZERO>
__device__ __forceinline__ void p2p_staged(const typename Vec4<T>::type* sh, int nl, int g, T eps2,
                                           LaneTargets<T, TPL>& me) {
    const int steps = (nl + G - 1) / G;
#pragma unroll(TPL > 2 ? 4 : 8)
    for (int q = 0; q < steps; ++q) {
        const typename Vec4<T>::type s = sh[q * G + g];
#pragma unroll
        for (int k = 0; k < TPL; ++k)
            pair<T, SOFT, ZERO>(me.x[k], me.y[k], me.z[k], s, eps2, me.phi[k], me.ax[k], me.ay[k],
                                me.az[k]);
    }
}

// Padding record: zero mass far from every target (its terms are exactly 0).
template <typename T>
__device__ __forceinline__ typename Vec4<T>::type p2p_pad() {
    return typename Vec4<T>::type{T(1e18), T(1e18), T(1e18), T(0)};
}

// The target box's own leaf as a source (coincident points possible): the
// sources of cell c against targets me.  In FP32 both are relative to the
// same centre (the box is the leaf), so no offset is added.
template <typename T, int G, int TPL, bool SOFT>
__device__ __forceinline__ void p2p_self(const Cell& c, const typename Vec4<T>::type* __restrict__ P,
                                         typename Vec4<T>::type* sh, T eps2,
                                         LaneTargets<T, TPL>& me) {
    const int lane = threadIdx.x & 63, g = lane / (64 / G);
    const int end = c.first + c.count;
    for (int base = c.first; base < end; base += 64) {
        const int k = base + lane;
        const typename Vec4<T>::type v = k < end ? P[k] : p2p_pad<T>();
        wave_lds_fence();
        sh[lane] = v;
        wave_lds_fence();
        p2p_staged<T, G, TPL, SOFT, true>(sh, min(64, end - base), g, eps2, me);
    }
}

// Sum over the list cells items[e0, e1) other than the target leaf `self`.
// Per batch of 64 cells, lane j holds cell j's range and (FP32) the offset
// between its centre and the target leaf's centre, formed in FP64; a scan
// over the counts places the batch's particles in one sequence, which is
// staged 64 at a time.
template <typename T, int G, int TPL, bool SOFT>
__device__ __forceinline__ void p2p_packed(const Cell* __restrict__ cells, int self,
                                           const int32_t* __restrict__ items, int e0, int e1,
                                           const typename Vec4<T>::type* __restrict__ P,
                                           typename Vec4<T>::type* sh, int* own,
                                           const Root& root, const double cb[3], T eps2,
                                           LaneTargets<T, TPL>& me) {
    using V = typename Vec4<T>::type;
    constexpr bool REL = sizeof(T) == 4;
    const int lane = threadIdx.x & 63, g = lane / (64 / G);
    for (int eb = e0; eb < e1; eb += 64) {
        int first = 0, cnt = 0;
        T ox = T(0), oy = T(0), oz = T(0);
        if (eb + lane < e1) {
            const int ci = items[eb + lane];
            if (ci != self) {
                const Cell c = cells[ci];
                first = c.first;
                cnt = c.count;
                if (REL) {
                    double cc[3];
                    cell_centre(root, c, cc);
                    ox = (T)(cc[0] - cb[0]);
                    oy = (T)(cc[1] - cb[1]);
                    oz = (T)(cc[2] - cb[2]);
                }
            }
        }
        int tot;
        const int off = wave_excl_scan(cnt, lane, tot);
        tot = __builtin_amdgcn_readfirstlane(tot);
        // lane's source of the run [pb, pb + 64) of the batch's particles;
        // the next run's load is issued before the current run's pairs
        auto fetch = [&](int pb, V& v, T& sx, T& sy, T& sz) {
            int o = wave_run_owner(own, off, cnt, pb, 64, lane);
            const bool ok = pb + lane < tot;
            o = ok ? o : 0;
            const int f = __shfl(first, o, 64), fo = __shfl(off, o, 64);
            v = p2p_pad<T>();
            if (REL) {
                sx = __shfl(ox, o, 64);
                sy = __shfl(oy, o, 64);
                sz = __shfl(oz, o, 64);
            }
            if (ok) v = P[f + (pb + lane - fo)];
            if (!ok) sx = sy = sz = T(0);
        };
        V v;
        T sx = T(0), sy = T(0), sz = T(0);
        if (tot > 0) fetch(0, v, sx, sy, sz);
        for (int pb = 0; pb < tot; pb += 64) {
            V cur = v;
            if (REL) {
                cur.x += sx;
                cur.y += sy;
                cur.z += sz;
            }
            if (pb + 64 < tot) fetch(pb + 64, v, sx, sy, sz);
            wave_lds_fence();
            sh[lane] = cur;
            wave_lds_fence();
            p2p_staged<T, G, TPL, SOFT, false>(sh, min(64, tot - pb), g, eps2, me);
        }
    }
}

// The targets of one box against the list cells items[e0, e1) (the box's
// own leaf, when it is in the list, summed on its own with the r^2 == 0
// test).  TP: the sorted targets, P: the sorted sources.
template <typename T, int TW, int TPL, bool SOFT>
__device__ __forceinline__ void p2p_box(const TBox& bx, bool in_list, const Root& root,
                                        const Cell* __restrict__ cells,
                                        const int32_t* __restrict__ items, int e0, int e1,
                                        const typename Vec4<T>::type* __restrict__ P,
                                        const typename Vec4<T>::type* __restrict__ TP,
                                        typename Vec4<T>::type* sh, int* own,
                                        const T* __restrict__ far, int64_t n,
                                        const int32_t* __restrict__ perm, T eps2,
                                        T* __restrict__ phi_o, T* __restrict__ ax_o,
                                        T* __restrict__ ay_o, T* __restrict__ az_o) {
    using V = typename Vec4<T>::type;
    constexpr int G = 64 / TW;
    static_assert(TW <= 16, "the sums of the lane groups end in the lanes' 16-lane rows");
    const int lane = threadIdx.x & 63;
    const int t = lane % TW;
    double cb[3];
    cell_centre(root, box_cell(bx), cb);
    Cell own_leaf;
    if (in_list) own_leaf = cells[bx.leaf];
    for (int c0 = 0; c0 < bx.count; c0 += TW * TPL) {
        LaneTargets<T, TPL> me;
#pragma unroll
        for (int k = 0; k < TPL; ++k) {
            const int i = c0 + k * TW + t;
            const V q = i < bx.count ? TP[bx.first + i] : V{T(0), T(0), T(0), T(0)};
            me.x[k] = q.x;
            me.y[k] = q.y;
            me.z[k] = q.z;
            me.phi[k] = me.ax[k] = me.ay[k] = me.az[k] = T(0);
        }
        if (in_list) p2p_self<T, G, TPL, SOFT>(own_leaf, P, sh, eps2, me);
        p2p_packed<T, G, TPL, SOFT>(cells, bx.leaf, items, e0, e1, P, sh, own, root, cb, eps2, me);
        // sum of the G lane groups: the two halves of the wave take two of the
        // four sums each, their 16-lane rows one each (row 0 phi, 1 ax, 2 ay,
        // 3 az), and the groups left inside a row add theirs
        const bool up = lane & 32, odd = lane & 16;
        const int row = lane >> 4;
        T* __restrict__ o = row == 0 ? phi_o : row == 1 ? ax_o : row == 2 ? ay_o : az_o;
#pragma unroll
        for (int k = 0; k < TPL; ++k) {
            const T a = (up ? me.ay[k] : me.phi[k]) + __shfl_xor(up ? me.phi[k] : me.ay[k], 32, 64);
            const T b = (up ? me.az[k] : me.ax[k]) + __shfl_xor(up ? me.ax[k] : me.az[k], 32, 64);
            T v = (odd ? b : a) + __shfl_xor(odd ? a : b, 16, 64);
#pragma unroll
            for (int d = TW; d < 16; d <<= 1) v += __shfl_xor(v, d, 64);
            const int i = c0 + k * TW + t;
            if (i < bx.count && (lane & 15) < TW) {
                const int s = bx.first + i;
                if (far) v += far[row * n + s];
                o[perm[s]] = v;
            }
        }
    }
}

// One wave per target box; sources from the box's CSR list row.  Bound by the
// VALU issue of the pairs (14.4 instructions each).  The split of the lanes
// (TW of 4, 8 or 16, the TPL that covers the box) leaves at most TW - 1 of
// TW * TPL target slots empty: with one target per lane and TW = 64 beyond 32
// targets, half of the leaves of a uniform set (34 to 45 targets) left 40 % of
// the lanes idle.  In whole evaluations: 2^20 uniform 0.495 -> 0.39 ms (2.2e12
// pairs/s); 2^22 Plummer, leaves of at most 32, 1.31 -> 1.10 ms; FP64, 262147
// uniform, 0.252 -> 0.211 ms.  Waves per SIMD: as many as leave no register spilled (a
// spilled word costs a small box as much as its pairs).  SMALL: for sets whose
// boxes hold few targets, at most two targets per lane, one wave per SIMD
// more (2^22 Plummer: 1.09 against 1.15 ms).
template <typename T, bool SOFT, bool SMALL>
__global__ void __launch_bounds__(256, sizeof(T) == 8 ? 3 : SMALL ? 6 : 5)
k_p2p(const Cell* __restrict__ cells, const Root* __restrict__ rootp, Targets tg,
      const int32_t* __restrict__ off, const int32_t* __restrict__ items,
      const typename Vec4<T>::type* __restrict__ P, const T* __restrict__ far, T eps2,
      T* __restrict__ phi_o, T* __restrict__ ax_o, T* __restrict__ ay_o, T* __restrict__ az_o) {
    using V = typename Vec4<T>::type;
    __shared__ V shm[4][64];
    __shared__ int owm[4][64];
    // (the wave number as a scalar: the box, its list range and the loops over
    // it then live in scalar registers)
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int li = blockIdx.x * 4 + w;
    if (li >= tg.nbox) return;
    const TBox bx = tg.box[li];
    const int row = list_row(tg, li, bx);
    const Root root = *rootp;
    const int e0 = off[row], e1 = off[row + 1];
    const V* TP = sizeof(T) == 4 ? (const V*)tg.p32 : (const V*)tg.p64;
    V* sh = shm[w];
    int* own = owm[w];
    // is the box's own leaf in its list (then it is summed on its own)
    bool mine = false;
    if (bx.leaf >= 0)
        for (int e = e0 + lane; e < e1; e += 64) mine |= items[e] == bx.leaf;
    const bool in_list = __ballot(mine) != 0ull;
#define P2P_BOX(TW, TPL)                                                                       \
    p2p_box<T, TW, TPL, SOFT>(bx, in_list, root, cells, items, e0, e1, P, TP, sh, own, far,    \
                              tg.n, tg.perm, eps2, phi_o, ax_o, ay_o, az_o)
    const int c = bx.count;
    if constexpr (SMALL) {
        if (c <= 4)
            P2P_BOX(4, 1);
        else if (c <= 8)
            P2P_BOX(4, 2);
        else if (c <= 16)
            P2P_BOX(8, 2);
        else
            P2P_BOX(16, 2);
    } else {
        if (c <= 8)
            P2P_BOX(4, 2);
        else if (c <= 12)
            P2P_BOX(4, 3);
        else if (c <= 16)
            P2P_BOX(4, 4);
        else if (c <= 24)
            P2P_BOX(8, 3);
        else if (c <= 32)
            P2P_BOX(8, 4);
        else if (c <= 40)
            P2P_BOX(8, 5);
        else if (c <= 48)
            P2P_BOX(16, 3);
        else
            P2P_BOX(16, 4);
    }
#undef P2P_BOX
}

void launch_p2p(const Tree& t, const Targets& tg, int precision, double eps2,
                const int32_t* src_off, const int32_t* src_items, const void* far, void* phi,
                void* ax, void* ay, void* az, hipStream_t s) {
    if (tg.nbox == 0) return;
    dim3 grid((tg.nbox + 3) / 4), block(256);
    const bool soft = eps2 != 0.0;
    // small boxes: fewer than 16 targets on average
    const bool small = tg.n < 16 * (int64_t)tg.nbox;
#define P2P_LAUNCH(T, SOFT, SMALL, P)                                                        \
    hipLaunchKernelGGL((k_p2p<T, SOFT, SMALL>), grid, block, 0, s, t.cells, t.root, tg,      \
                       src_off, src_items, P, (const T*)far, (T)eps2, (T*)phi, (T*)ax,       \
                       (T*)ay, (T*)az)
    if (precision == HFMM_FP64) {
        if (soft)
            P2P_LAUNCH(double, true, false, t.p64);
        else
            P2P_LAUNCH(double, false, false, t.p64);
    } else if (small) {
        if (soft)
            P2P_LAUNCH(float, true, true, t.p32);
        else
            P2P_LAUNCH(float, false, true, t.p32);
    } else {
        if (soft)
            P2P_LAUNCH(float, true, false, t.p32);
        else
            P2P_LAUNCH(float, false, false, t.p32);
    }
#undef P2P_LAUNCH
    LAUNCH_CHECK();
}

// ---------------------------------------------------------------------
// direct sum: a block of 4 waves takes 64 / G targets, and its 4 G lane
// groups share the sources (wave w the chunks w, w + 4, ... of 64, group g
// every G-th source of a chunk); the groups are summed by shuffles and
// through LDS, so no partial result leaves the block.
// ---------------------------------------------------------------------
template <typename T>
__global__ void k_pack_points(const double* __restrict__ x, const double* __restrict__ y,
                              const double* __restrict__ z, const double* __restrict__ m,
                              int64_t n, typename Vec4<T>::type* __restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = typename Vec4<T>::type{(T)x[i], (T)y[i], (T)z[i], m ? (T)m[i] : T(0)};
}

// Bound by the VALU issue of the pairs.  With one wave per 64 targets over
// all the sources, N = 30011 ran 469 waves on 1024 SIMDs (1.27 ms, 7.1e11
// pairs/s); the split keeps every SIMD's wave slots filled down to a few
// thousand targets (N = 30011: 0.38 ms, 2.4e12 pairs/s).
template <typename T, int G, bool SOFT>
__global__ void __launch_bounds__(256)
k_direct(const typename Vec4<T>::type* __restrict__ src, int64_t ns,
         const typename Vec4<T>::type* __restrict__ tgt, int64_t nt, T eps2,
         T* __restrict__ phi_o, T* __restrict__ ax_o, T* __restrict__ ay_o,
         T* __restrict__ az_o) {
    using V = typename Vec4<T>::type;
    constexpr int TW = 64 / G;
    __shared__ V shm[4][64];
    __shared__ V red[4][TW];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = lane / TW, t = lane % TW;
    const int64_t i = (int64_t)blockIdx.x * TW + t;
    const V q = i < nt ? tgt[i] : V{T(0), T(0), T(0), T(0)};
    LaneTargets<T, 1> me{{q.x}, {q.y}, {q.z}, {T(0)}, {T(0)}, {T(0)}, {T(0)}};
    V* sh = shm[w];
    // the next chunk's load is issued before the current chunk's pairs
    int64_t base = (int64_t)w * 64;
    V v = base + lane < ns ? src[base + lane] : p2p_pad<T>();
    for (; base < ns; base += 256) {
        wave_lds_fence();
        sh[lane] = v;
        wave_lds_fence();
        const int64_t k = base + 256 + lane;
        v = k < ns ? src[k] : p2p_pad<T>();
        p2p_staged<T, G, 1, SOFT, true>(sh, (int)min((int64_t)64, ns - base), g, eps2, me);
    }
    T phi = me.phi[0], ax = me.ax[0], ay = me.ay[0], az = me.az[0];
#pragma unroll
    for (int d = TW; d < 64; d <<= 1) {
        phi += __shfl_xor(phi, d, 64);
        ax += __shfl_xor(ax, d, 64);
        ay += __shfl_xor(ay, d, 64);
        az += __shfl_xor(az, d, 64);
    }
    if (lane < TW) red[w][t] = V{phi, ax, ay, az};
    __syncthreads();
    if (w == 0 && lane < TW && i < nt) {
        V a = red[0][t];
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            const V b = red[k][t];
            a.x += b.x;
            a.y += b.y;
            a.z += b.z;
            a.w += b.w;
        }
        phi_o[i] = a.x;
        ax_o[i] = a.y;
        ay_o[i] = a.z;
        az_o[i] = a.w;
    }
}

template <typename T>
static void direct_t(const double* x, const double* y, const double* z, const double* m,
                     int64_t ns, const double* tx, const double* ty, const double* tz,
                     int64_t nt, double eps2, Arena& A, void* phi, void* ax, void* ay,
                     void* az, hipStream_t s) {
    using V = typename Vec4<T>::type;
    V* src = A.down<V>(ns);
    V* tgt = tx ? A.down<V>(nt) : src;
    hipLaunchKernelGGL((k_pack_points<T>), dim3(grid_for(ns, 256)), dim3(256), 0, s, x, y, z,
                       m, ns, src);
    LAUNCH_CHECK();
    if (tx) {
        hipLaunchKernelGGL((k_pack_points<T>), dim3(grid_for(nt, 256)), dim3(256), 0, s, tx, ty,
                           tz, (const double*)nullptr, nt, tgt);
        LAUNCH_CHECK();
    }
    // the widest target tile that still gives each of the 256 CUs 16 blocks
    // (8 resident at once; 8 more even out the tail); a launch holds less than
    // 2^32 threads, at 64 targets a block 2^30 targets
    const int64_t tiles = 16 * 256, most = (int64_t)1 << 29;
#define DIRECT_LAUNCH(G)                                                                       \
    for (int64_t t0 = 0; t0 < nt; t0 += most) {                                                \
        const int64_t n = std::min(most, nt - t0);                                             \
        const dim3 grid((unsigned)((n + 64 / G - 1) / (64 / G)));                              \
        T *o0 = (T*)phi + t0, *o1 = (T*)ax + t0, *o2 = (T*)ay + t0, *o3 = (T*)az + t0;         \
        if (eps2 != 0.0)                                                                       \
            hipLaunchKernelGGL((k_direct<T, G, true>), grid, dim3(256), 0, s, src, ns,         \
                               tgt + t0, n, (T)eps2, o0, o1, o2, o3);                          \
        else                                                                                   \
            hipLaunchKernelGGL((k_direct<T, G, false>), grid, dim3(256), 0, s, src, ns,        \
                               tgt + t0, n, (T)eps2, o0, o1, o2, o3);                          \
    }
    if (nt >= 64 * tiles)
        DIRECT_LAUNCH(1)
    else if (nt >= 32 * tiles)
        DIRECT_LAUNCH(2)
    else if (nt >= 16 * tiles)
        DIRECT_LAUNCH(4)
    else
        DIRECT_LAUNCH(8)
#undef DIRECT_LAUNCH
    LAUNCH_CHECK();
}

void direct_sum(const double* x, const double* y, const double* z, const double* m, int64_t ns,
                const double* tx, const double* ty, const double* tz, int64_t nt,
                int precision, double eps2, Arena& A, void* phi, void* ax, void* ay, void* az,
                hipStream_t s) {
    if (nt == 0) return;
    if (precision == HFMM_FP64)
        direct_t<double>(x, y, z, m, ns, tx, ty, tz, nt, eps2, A, phi, ax, ay, az, s);
    else
        direct_t<float>(x, y, z, m, ns, tx, ty, tz, nt, eps2, A, phi, ax, ay, az, s);
}

}  // namespace hfmm
