// FP32 M2L (Eq. 4) on the BF16 matrix cores, p = 8 to 11: both operands split
// into three BF16 parts.
//
// A value is written as a sum of parts h + m + l, each the BF16 rounding of
// what the parts before it leave: 8 significant bits and a sign in each part,
// i.e. all of an FP32 value and one bit more of the FP64 operator.  The six
// products h h, h m, m h, h l, l h, m m are added in FP32.  |m| <= 2^-8 |h| and
// |l| <= 2^-17 |h|, so the dropped m l and l m reach 2^-24 of h h, half a
// rounding of FP32, at worst, and are about 2^-28 of it as a rule.  BF16 has
// FP32's exponent range, so nothing is rescaled by level; only the decay of the
// multipoles with the degree n is moved to the operator (2^mu_n, exact, taken
// out of one operand and put into the other), so that the low parts stay normal
// numbers (masses of 2^-112 and more: the same range as the FP32 products).
// Error of the potential against the same FMM in FP64, FP32 matrix products ->
// this form with all else equal, in 1e-7 (means over six seeds; over 24, good to
// 1.5 %, for 100003 equal masses at p = 8 and 9):
//   p                                8            9            10           11
//   100003 uniform, equal masses  1.40 -> 1.41 1.44 -> 1.44 1.49 -> 1.47 1.52 -> 1.51
//   100003 uniform, both signs    3.83 -> 2.77 4.07 -> 3.06 5.23 -> 3.87 5.38 -> 3.96
//   262147 uniform, equal         1.50 -> 1.41 1.53 -> 1.46 1.90 -> 1.55 1.89 -> 1.57
//   100003 Plummer, equal         1.46 -> 1.47 1.48 -> 1.48 1.65 -> 1.55 1.69 -> 1.56
//   300007 Plummer, unequal       2.14 -> 1.87 2.06 -> 1.85 3.05 -> 2.13 3.07 -> 2.14
// (where they agree the error is that of the other phases: the local expansions
// themselves are as good or better).  Of the acceleration: equal or smaller.
//
// At 16 times the rate of the FP32 matrix products six of them cost 3/8.
// Tiles, teams and segments are those of k_m2l_mma (8 waves of 32 targets of
// one octant, all output rows); the sources are gathered as FP32 rows and
// split in registers, which moves the bytes of the FP32 form, two thirds of
// what three stored parts would be.
// Measured in whole evaluations, FP32 products -> this form: 2^20 uniform, p =
// 10: 1.15 -> 0.73 to 0.77 ms between runs (0.70 in a loop of its own: 1.3
// PFLOP/s as executed; a register-only chain of these products on random data
// runs 1.9); 2^22 Plummer, p = 8: 6.7 -> 4.85 to 5.0 ms.  What bounds it now: at
// 2^20, p = 10 the 4.1 GB a launch fetches from beyond L2 (source rows and
// operators, L2 hit rate 0.44), 5.2 TB/s, the rate of a large copy, with the
// matrix cores busy 54 % of the time; at 2^22 Plummer 10.9 GB (hit rate 0.74, 2
// TB/s) and 43 %: the latency of the gathered rows and the barrier of every slot
// (without the gather, one row for all: 0.58 and 3.5 ms).  64 targets per wave
// with half the operator reads (4 waves, 512 registers) were slower, 0.83 and
// 5.1 ms.
//
// v_mfma_f32_16x16x32_bf16: lane group g = lane / 16 feeds the contraction
// elements 32 q + 8 g .. + 7 of its column (target) and row (operator).  The
// elements past the last whole 32 (p^2 mod 32, when at most 16) are not padded
// to 32: a tail product holds the part products of 4 elements side by side,
//   g = 0: h h, h m   1: m h, h l   2: l h, m m   3: zero operator
// so p = 10 takes 19 products per output block instead of 24.
#include "common.hpp"
#include "expansions.hpp"
#include "m2l_items.hpp"
#include "m2l_table.hpp"

#include <algorithm>

namespace hfmm {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Rows (rb) of 16 outputs, whole contraction steps (kf), tail steps (ts),
// operator chunks of 1 KB (64 lanes x 16 B) per class, floats per source row.
struct SplitShape {
    int rb, kf, ts, nch, ld;
};
__host__ __device__ constexpr SplitShape split_shape(int p) {
    const int P = p * p, rest = P % 32;
    SplitShape s{};
    s.rb = (P + 15) / 16;
    s.kf = P / 32 + (rest > 16 ? 1 : 0);
    s.ts = rest > 16 ? 0 : (rest + 3) / 4;
    s.nch = s.rb * (3 * s.kf + s.ts);
    s.ld = 32 * s.kf + 4 * s.ts;
    return s;
}
// two operator buffers in LDS when both fit in 144 KiB
__host__ __device__ constexpr bool split_double(int p) { return 2 * split_shape(p).nch <= 144; }
// Where the five small part products of a step are added.  Added one by one to
// the sum of the h h products (kOneSum) they round it six times a step; at p = 8
// and 9, where the FP32 form has fewest products of its own, the potential's
// error then came out up to 2.6 % larger than the FP32 form's on some sets.  With
// a sum of their own it is at most the FP32 form's (the figures above).  Kept to
// the end of the segment (kLowSum) that sum takes 32 registers at p = 8 (M2L
// 0.362 -> 0.367 ms at 2^20 uniform, 4.83 -> 4.86 at 2^22 Plummer); at p = 9 its 48
// spill (0.55 -> 0.74 ms), so each step's sum is added on its own, one output
// block later, when its products are done (kStepSum: 0.565 -> 0.573 ms, 2^22
// Plummer 8.1 -> 8.35; at p = 8 0.362 -> 0.378 and 4.83 -> 4.98).
enum SplitSum { kOneSum, kLowSum, kStepSum };
__host__ __device__ constexpr SplitSum split_sum(int p) {
    return p == 8 ? kLowSum : p == 9 ? kStepSum : kOneSum;
}

// The orders at which this form is the faster one.  M2L at 2^20 uniform, FP32
// products -> this form, in ms: p = 5 0.18 -> 0.19, p = 6 0.24 -> 0.26, p = 7
// 0.35 -> 0.34, p = 8 0.47 -> 0.37, p = 9 0.80 -> 0.57, p = 10 1.04 -> 0.71,
// p = 11 1.54 -> 0.94, p = 12 2.08 -> 2.50.  Below, two blocks of the FP32
// kernel share a CU, and the slots are too short to hide the splitting; at 12
// the operator (144 KB) leaves one LDS buffer, and the registers that stage
// the next one spill.
bool m2l_uses_split(int p, int precision) {
    return precision == HFMM_FP32 && p >= 8 && p <= 11;
}
int split_row_floats(int p) { return split_shape(p).ld; }
size_t split_ops_bytes(int p) { return (size_t)343 * split_shape(p).nch * 1024; }

// ---------------------------------------------------------------------
// operators and source rows
// ---------------------------------------------------------------------
// T' = T 2^mu_n split into parts, in the chunk order [cls][rb][q][part] then
// [cls][rb][ts]; one thread per 16-byte lane of a (rb, q) or tail chunk.
__global__ void __launch_bounds__(256) k_split_ops(int p, bf16x8* __restrict__ T) {
    __shared__ M2lClassTable tab;
    const int P = p * p;
    const SplitShape sh = split_shape(p);
    const int cls = blockIdx.x;
    const bool far = tab.fill(p, cls);
    const int main = sh.rb * sh.kf * 64, all = main + sh.rb * sh.ts * 64;
    bf16x8* out = T + (int64_t)cls * sh.nch * 64;
    for (int e = blockIdx.y * blockDim.x + threadIdx.x; e < all; e += gridDim.y * blockDim.x) {
        const int lane = e & 63, g = lane >> 4, c = e >> 6;
        const bool tail = e >= main;
        const int rb = tail ? (c - sh.rb * sh.kf) / sh.ts : c / sh.kf;
        const int q = tail ? (c - sh.rb * sh.kf) % sh.ts : c % sh.kf;
        const int ro = 16 * rb + (lane & 15);
        bf16x8 v[3];
        for (int j = 0; j < 8; ++j) {
            // contraction element of slot j of this lane
            const int k = tail ? 32 * sh.kf + 4 * q + (j & 3) : 32 * q + 8 * g + j;
            const double t = far && ro < P && k < P ? tab.entry(ro, k) * tab.up[k] : 0.0;
            const __bf16 h = (__bf16)(float)t;
            const double r1 = t - (double)(float)h;
            const __bf16 m = (__bf16)(float)r1;
            v[0][j] = h;
            v[1][j] = m;
            v[2][j] = (__bf16)(float)(r1 - (double)(float)m);
        }
        if (!tail) {
            for (int a = 0; a < 3; ++a) out[((rb * sh.kf + q) * 3 + a) * 64 + lane] = v[a];
            continue;
        }
        bf16x8 w;
        for (int j = 0; j < 8; ++j)
            w[j] = g == 0   ? v[0][j]
                   : g == 1 ? (j < 4 ? v[1][j] : v[0][j])
                   : g == 2 ? (j < 4 ? v[2][j] : v[1][j])
                            : (__bf16)0.0f;
        out[(sh.rb * sh.kf * 3 + rb * sh.ts + q) * 64 + lane] = w;
    }
}

// Source rows M' = M 2^-mu_n in FP32, ld floats each; the zero row ncells
// stands for an absent source.
__global__ void __launch_bounds__(256)
k_split_pack(const double* __restrict__ M, int ldm, int ncells, int p, int ld,
             float* __restrict__ out) {
    __shared__ double down[HFMM_MAX_P * HFMM_MAX_P];
    const int P = p * p;
    for (int k = threadIdx.x; k < P; k += blockDim.x) down[k] = ldexp(1.0, -m2l_mu(degree_of(k)));
    __syncthreads();
    const int64_t tot = (int64_t)(ncells + 1) * ld;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < tot;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(e / ld), k = (int)(e % ld);
        out[e] = c < ncells && k < P ? (float)(M[(int64_t)c * ldm + k] * down[k]) : 0.0f;
    }
}

// ---------------------------------------------------------------------
// the products
// ---------------------------------------------------------------------
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
}
// two values -> their BF16 parts, packed
__device__ __forceinline__ void split2(float a, float b, uint32_t (&w)[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        w[i] = pk_bf16(a, b);
        if (i < 2) {
            a -= __builtin_bit_cast(float, w[i] << 16);
            b -= __builtin_bit_cast(float, w[i] & 0xffff0000u);
        }
    }
}
__device__ __forceinline__ floatx4 mma_bf16(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int kSplitCB = 2;  // column blocks of 16 targets per wave
constexpr int kSplitNW = 8;  // waves per block

template <int P>
__global__ void __launch_bounds__(64 * kSplitNW)
k_m2l_split(const int32_t* __restrict__ tiles, const uint32_t* __restrict__ tmask,
            const uint32_t* __restrict__ gmask, const int32_t* __restrict__ gpre, int ngroups,
            int gw, int nb, int nparts, const int32_t* __restrict__ order,
            const int32_t* __restrict__ vsrc, const float* __restrict__ M, int ncells,
            const u32x4* __restrict__ T, float* __restrict__ out, int64_t part_stride,
            int zero_fill) {
    constexpr SplitShape SH = split_shape(P);
    constexpr int RB = SH.rb, KF = SH.kf, TS = SH.ts, NCH = SH.nch, LD4 = SH.ld / 4;
    constexpr bool DB = split_double(P);
    constexpr SplitSum SUM = split_sum(P);
    constexpr int CB = kSplitCB, NW = kSplitNW, LDO = 16 * RB;
    // the contraction in S steps of 32 elements, the last with the tail
    constexpr int S = KF;
    constexpr int MU = 4 * CB;  // split units of a step (2 values) ..
    constexpr int TU = CB * TS;  // .. and of the tail (4 values)
    constexpr int NPW = (NCH + NW - 1) / NW;
    // the step at whose start the next operator is requested (large ones late:
    // their registers)
    constexpr int OPAT = NPW > 9 ? S - 1 : S - 2;
    static_assert(S >= 2, "the pipeline looks two steps ahead, at most one slot");
    __shared__ u32x4 sT[NCH * 64];
    __shared__ u32x4 sT2[DB ? NCH * 64 : 1];
    M2lItems it = m2l_items(gpre, ngroups, gw, nb);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = lane >> 4, col = lane & 15;
    const float4* Mv = (const float4*)M;
    for (; it.item < it.iend; ++it.group) {
        const int tile = it.group * gw + it.o;
        int part;
        bool last_seg;
        uint32_t mw[7];
        m2l_segment(tmask, gmask, gpre, tile, nb, it, part, last_seg, mw);
        const int start = tiles[4 * tile], count = tiles[4 * tile + 1], oct = tiles[4 * tile + 2];
        const int ox = (oct >> 2) & 1, oy = (oct >> 1) & 1, oz = oct & 1;
        // the previous segment's products are done before its buffers are
        // written again
        __syncthreads();
        int tgt[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int i = (wave * CB + cb) * 16 + col;
            tgt[cb] = i < count ? order[start + i] : -1;
        }
        floatx4 acc[CB][RB], low[CB][SUM == kLowSum ? RB : 1];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                acc[cb][rb] = floatx4{0.f, 0.f, 0.f, 0.f};
                if constexpr (SUM == kLowSum) low[cb][rb] = floatx4{0.f, 0.f, 0.f, 0.f};
            }

        // V entry of position j (every call issues CB loads, past the last slot
        // and for absent targets of an entry that exists), and the row it
        // names (the zero row for none); apart, so that the loads stay in
        // flight until the row is needed
        auto load_src = [&](int j, int (&sv)[CB]) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                sv[cb] = vsrc[(int64_t)(tgt[cb] >= 0 ? tgt[cb] : 0) * 216 + (j < 216 ? j : 0)];
        };
        auto src_row = [&](int j, const int (&sv)[CB], int64_t (&row)[CB]) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                row[cb] = (int64_t)(j < 216 && tgt[cb] >= 0 && sv[cb] >= 0 ? sv[cb] : ncells) * LD4;
        };
        auto load_op = [&](int j, u32x4 (&r)[NPW]) {
            const int slot = v_slot_at(j);
            const int dx = slot / 36 - 2 - ox, dy = (slot / 6) % 6 - 2 - oy, dz = slot % 6 - 2 - oz;
            const int cls = (dx + 3) * 49 + (dy + 3) * 7 + (dz + 3);
            const u32x4* t = T + (int64_t)cls * (NCH * 64);
#pragma unroll
            for (int i = 0; i < NPW; ++i) r[i] = t[min(wave + NW * i, NCH - 1) * 64 + lane];
        };
        // (the waves past the last chunk write that chunk's bytes again)
        auto store_op = [&](u32x4* buf, const u32x4 (&r)[NPW]) {
#pragma unroll
            for (int i = 0; i < NPW; ++i) buf[min(wave + NW * i, NCH - 1) * 64 + lane] = r[i];
        };
        // Pipeline over the steps of all slots (linear step L: slot L / S, step
        // L mod S).  While step L runs on the matrix cores, the sources of
        // step L + 2 are requested and those of step L + 1 are split, a few
        // values per output block, between its products; the operator chunks
        // of output block rb + 1 are read from LDS during block rb.
        struct Raw {
            float4 m[CB][2], t[CB][TS > 0 ? TS : 1];
        };
        struct Parts {
            u32x4 m[CB][3], t[CB][TS > 0 ? TS : 1];
        };
        struct Chunks {
            u32x4 m[3], t[TS > 0 ? TS : 1];
        };
        auto load_step = [&](const int64_t (&row)[CB], int q, Raw& r) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                r.m[cb][0] = Mv[row[cb] + 8 * q + 2 * g];
                r.m[cb][1] = Mv[row[cb] + 8 * q + 2 * g + 1];
                if (q == S - 1) {
#pragma unroll
                    for (int i = 0; i < TS; ++i) r.t[cb][i] = Mv[row[cb] + 8 * KF + i];
                }
            }
        };
        // split unit u of a step: two values of a column, or four of the tail
        auto split_unit = [&](const Raw& r, Parts& o, int u) {
            uint32_t w[3];
            if (u < MU) {
                const int cb = u / 4, i = u % 4;
                const float4 x = r.m[cb][i / 2];
                split2(i % 2 ? x.z : x.x, i % 2 ? x.w : x.y, w);
#pragma unroll
                for (int a = 0; a < 3; ++a) o.m[cb][a][i] = w[a];
                return;
            }
            const int cb = (u - MU) / (TS > 0 ? TS : 1), ts = (u - MU) % (TS > 0 ? TS : 1);
            const float4 x = r.t[cb][ts];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                split2(i ? x.z : x.x, i ? x.w : x.y, w);
                o.t[cb][ts][i] = w[0];
                o.t[cb][ts][2 + i] = g == 1 ? w[2] : w[1];
            }
        };
        auto load_chunks = [&](const u32x4* buf, int q, int rb, Chunks& c) {
#pragma unroll
            for (int i = 0; i < 3; ++i) c.m[i] = buf[((rb * KF + q) * 3 + i) * 64 + lane];
            if (q == S - 1) {
#pragma unroll
                for (int i = 0; i < TS; ++i)
                    c.t[i] = buf[(RB * KF * 3 + rb * TS + i) * 64 + lane];
            }
        };

        // state at the top of a slot j: its operator in LDS, its first step
        // split (p0) and the sources of the step after in flight (r1), its
        // rows and those of the next slot jn, the V entries of the slot jq
        // after that in srcn
        int j = m2l_next_slot(mw, 0);
        int jn = j < 216 ? m2l_next_slot(mw, j + 1) : 216;
        int jq = jn < 216 ? m2l_next_slot(mw, jn + 1) : 216;  // last slot looked up
        int src[CB], srcn[CB];
        int64_t rw[2][CB];
        load_src(j, src);
        load_src(jn, srcn);
        src_row(j, src, rw[0]);
        src_row(jn, srcn, rw[1]);
        load_src(jq, srcn);
        Raw r0, r1;
        load_step(rw[0], 0, r0);
        load_step(rw[0], 1, r1);
        u32x4 opr[NPW];
        if (j < 216) {
            load_op(j, opr);
            store_op(sT, opr);
        }
        Parts p0;
#pragma unroll
        for (int u = 0; u < MU; ++u) split_unit(r0, p0, u);
        __syncthreads();
        // one body per iteration, the buffers swapped by parity
        for (int par = 0; j < 216; par ^= 1) {
            const u32x4* cur = DB && par ? sT2 : sT;
            u32x4* nxt = DB && !par ? sT2 : sT;
            const int jnext = jq;
            int64_t rwn[CB];
            src_row(jnext, srcn, rwn);
            jq = jq < 216 ? m2l_next_slot(mw, jq + 1) : 216;
            load_src(jq, srcn);
            Parts pt[S + 1];
            Raw rt[S + 2];
            Chunks ch[2];
            floatx4 step[2][CB];  // kStepSum: of this output block and the one before
            pt[0] = p0;
            rt[1] = r1;
            load_chunks(cur, 0, 0, ch[0]);
#pragma unroll
            for (int q = 0; q < S; ++q) {
                // unconditional loads (past the last slot, its operator again),
                // so that the number in flight is the same on every path
                if (q == OPAT) load_op(jn < 216 ? jn : j, opr);
                load_step(rw[(q + 2) / S], (q + 2) % S, rt[q + 2]);
                // keeps the optimiser from sinking the next slot's loads to
                // their use after the barrier (an empty statement, no wait)
                asm volatile("" ::: "memory");
                const bool tail = q == S - 1;
                const int units = MU + ((q + 1) % S == S - 1 ? TU : 0);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const Chunks& c = ch[(q * RB + rb) & 1];
                    Chunks& cn = ch[(q * RB + rb + 1) & 1];
                    if (rb + 1 < RB)
                        load_chunks(cur, q, rb + 1, cn);
                    else if (!tail)
                        load_chunks(cur, q + 1, 0, cn);
                    // part products, the smallest first
#pragma unroll
                    for (int sum = 2; sum >= 0; --sum)
#pragma unroll
                        for (int i = 0; i <= sum; ++i)
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) {
                                floatx4& a = sum == 0 || SUM == kOneSum ? acc[cb][rb]
                                             : SUM == kLowSum ? low[cb][SUM == kLowSum ? rb : 0]
                                                              : step[rb & 1][cb];
                                const bool first = SUM == kStepSum && sum == 2 && i == 0;
                                a = mma_bf16(c.m[i], pt[q].m[cb][sum - i], first ? floatx4{} : a);
                            }
                    if (tail) {
#pragma unroll
                        for (int i = 0; i < TS; ++i)
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb)
                                acc[cb][rb] = mma_bf16(c.t[i], pt[q].t[cb][i], acc[cb][rb]);
                    }
                    if constexpr (SUM == kStepSum) {
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            if (rb > 0) acc[cb][rb > 0 ? rb - 1 : 0] += step[~rb & 1][cb];
                            if (rb == RB - 1) acc[cb][rb] += step[rb & 1][cb];
                        }
                    }
#pragma unroll
                    for (int u = rb * units / RB; u < (rb + 1) * units / RB; ++u)
                        split_unit(rt[q + 1], pt[q + 1], u);
                    // one product, then a vector instruction or two in its
                    // shadow; the loads first
                    __builtin_amdgcn_sched_group_barrier(0x100, 3 + TS, 0);
#pragma unroll
                    for (int i = 0; i < CB * (6); ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (!DB) __syncthreads();  // the one buffer is no longer read
            store_op(nxt, opr);
            __syncthreads();  // nxt holds slot jn; cur is no longer read
            j = jn;
            jn = jnext;
            p0 = pt[S];
            r1 = rt[S + 1];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                rw[0][cb] = rw[1][cb];
                rw[1][cb] = rwn[cb];
            }
        }
        // with zero_fill, the last segment of the group clears the partial
        // results after its own
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            if (tgt[cb] < 0) continue;
            float* o = out + part * part_stride + (int64_t)tgt[cb] * LDO + 4 * g;
            if constexpr (SUM == kLowSum) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) acc[cb][rb] += low[cb][rb];
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                *(float4*)(o + 16 * rb) = make_float4(acc[cb][rb][0], acc[cb][rb][1],
                                                      acc[cb][rb][2], acc[cb][rb][3]);
            if (last_seg && zero_fill)
                for (int q = part + 1; q < nparts; ++q) {
                    o += part_stride;
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        *(float4*)(o + 16 * rb) = make_float4(0.f, 0.f, 0.f, 0.f);
                }
        }
    }
}

// ---------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------
void run_split_ops(int p, void* T, hipStream_t s) {
    hipLaunchKernelGGL(k_split_ops, dim3(343, 4), dim3(256), 0, s, p, (bf16x8*)T);
    LAUNCH_CHECK();
}

void run_split_pack(const Tree& t, int p, float* Mk, hipStream_t s) {
    const int ld = split_row_floats(p);
    const int64_t tot = (int64_t)(t.ncells + 1) * ld;
    hipLaunchKernelGGL(k_split_pack, dim3((unsigned)std::min<int64_t>(8192, (tot + 255) / 256)),
                       dim3(256), 0, s, t.M, t.ldm, t.ncells, p, ld, Mk);
    LAUNCH_CHECK();
}

void run_m2l_split(const Tree& t, int p, const float* Mk, dim3 grid, int nb, int parts,
                   float* out, int64_t part_stride, int fill, hipStream_t s) {
#define SPLIT_CASE(PP)                                                                        \
    case PP:                                                                                  \
        hipLaunchKernelGGL((k_m2l_split<PP>), grid, dim3(64 * kSplitNW), 0, s, t.m2l_tiles,   \
                           t.m2l_tmask, t.m2l_gmask, t.m2l_gpre, t.n_m2l_tiles / t.m2l_gw,    \
                           t.m2l_gw, nb, parts, t.m2l_torder, t.vsrc, Mk, t.ncells,           \
                           (const u32x4*)t.T, out, part_stride, fill);                        \
        break;
    switch (p) {
        SPLIT_CASE(8)
        SPLIT_CASE(9)
        SPLIT_CASE(10)
        SPLIT_CASE(11)
        default: throw Status{HFMM_E_UNSUPPORTED};
    }
#undef SPLIT_CASE
    LAUNCH_CHECK();
}

}  // namespace hfmm
