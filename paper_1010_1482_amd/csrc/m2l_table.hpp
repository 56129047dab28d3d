// The M2L operator of one offset class (Eq. 4), tabulated by a block in LDS.
#pragma once
#include "common.hpp"

namespace hfmm {

// degree n of real-layout index r, and the exponent of the multipoles' decay
// with it: floor(log2((sqrt3/2)^n / n!))
__device__ inline int degree_of(int r) {
    int n = 0;
    while ((n + 1) * (n + 1) <= r) ++n;
    return n;
}
__device__ inline int m2l_mu(int n) {
    double v = 1.0;
    for (int i = 1; i <= n; ++i) v *= 0.8660254037844386 / (double)i;
    return ilogb(v);
}

// M2L operator of one offset class from Eq. 4.  With the identity of Sec. 5.2,
// Y_N^M / (A_N^M rho^{N+1}) = (N-|M|)! P_N^|M|(cos a) e^{iM b} / rho^{N+1},
// and the change to the device basis (Lb = L / A_j^k, Mb = A_n^m M), the
// factors A_n^m A_j^k of Eq. 4 cancel and the complex coefficient of
// M_n^m in L_j^k becomes
//   c(j,k,n,m) = i^{|k-m|-|k|-|m|} (-1)^j (N-|M|)! P_N^|M| e^{iM b} / rho^{N+1}
// with N = j + n, M = m - k, (rho, a, b) the spherical coordinates of
// c_target - c_source in cell units (offsets are source minus target, so the
// vector is -d).  Conjugate symmetry of M folds m and -m into real entries.
// The 343 classes count the 27 adjacent offsets, whose operator is zero.
struct M2lClassTable {
    static constexpr int kNmax = 2 * HFMM_MAX_P - 1;
    static constexpr int kRows = HFMM_MAX_P * HFMM_MAX_P;
    double pt[kNmax][kNmax];  // (N-|M|)! P_N^|M|(cos a) / rho^{N+1}, N <= 2p-2 (Eqs. 7-9)
    double cs[kNmax][2];      // cos(M b), sin(M b)
    int dec[kRows];           // real-layout index -> n | m << 8 | part << 16
    double up[kRows];         // 2^mu_n

    // every thread of the block calls; false for the adjacent offsets
    __device__ bool fill(int p, int cls) {
        const int ND = 2 * p - 1;
        const int dx = cls / 49 - 3, dy = (cls / 7) % 7 - 3, dz = cls % 7 - 3;
        const bool far = max(abs(dx), max(abs(dy), abs(dz))) >= 2;
        for (int r = threadIdx.x; r < p * p; r += blockDim.x) {
            const int n = degree_of(r), o = r - n * n;
            dec[r] = n | (o + 1) / 2 << 8 | (o == 0 ? 0 : (o + 1) % 2) << 16;
            up[r] = ldexp(1.0, m2l_mu(n));
        }
        if (far && (int)threadIdx.x < ND) {
            const int a = threadIdx.x;  // order |M|
            const double vx = -dx, vy = -dy, vz = -dz;
            const double rxy = sqrt(vx * vx + vy * vy);
            const double rho = sqrt(vx * vx + vy * vy + vz * vz);
            const double x = vz / rho, sn = rxy / rho;
            const double beta = (vx == 0.0 && vy == 0.0) ? 0.0 : atan2(vy, vx);
            cs[a][0] = cos(a * beta);
            cs[a][1] = sin(a * beta);
            double pmm = 1.0;  // Eq. 8
            for (int i = 1; i <= a; ++i) pmm *= -(double)(2 * i - 1) * sn;
            double rinv = 1.0 / rho, rpow = rinv;  // 1 / rho^{N+1}
            for (int i = 0; i < a; ++i) rpow *= rinv;
            double pm1 = 0.0, pc = pmm, fct = 1.0;  // P_{N-1}, P_N, (N - a)!
            for (int N = a; N < ND; ++N) {
                pt[N][a] = fct * pc * rpow;
                const double pn =
                    N == a ? x * (2 * a + 1) * pmm                                 // Eq. 9
                           : (x * (2 * N + 1) * pc - (N + a) * pm1) / (N - a + 1);  // Eq. 7
                pm1 = pc;
                pc = pn;
                fct *= (double)(N - a + 1);
                rpow *= rinv;
            }
        }
        __syncthreads();
        return far;
    }

    // real entry (row ro, column ri):
    // c(j,k,n,+-m) = i^{|k-m|-|k|-|m|} (-1)^j pt[j+n][|m-k|] e^{i (m-k) b}
    __device__ double entry(int ro, int ri) const {
        const int j = dec[ro] & 255, k = dec[ro] >> 8 & 255, po = dec[ro] >> 16;
        const int n = dec[ri] & 255, m = dec[ri] >> 8 & 255, pi = dec[ri] >> 16;
        auto coef = [&](int mm) {
            const int M = mm - k, aM = M < 0 ? -M : M;
            const int ev = abs(k - mm) - abs(k) - abs(mm);
            const double sg = (((ev / 2) & 1) ? -1.0 : 1.0) * ((j & 1) ? -1.0 : 1.0);
            const double v = sg * pt[j + n][aM];
            return make_double2(v * cs[aM][0], v * (M < 0 ? -cs[aM][1] : cs[aM][1]));
        };
        if (m == 0) {
            double2 c0 = coef(0);
            return pi == 0 ? (po == 0 ? c0.x : c0.y) : 0.0;
        }
        double2 cp = coef(m), cm = coef(-m);
        if (po == 0) return pi == 0 ? cp.x + cm.x : -(cp.y - cm.y);
        return pi == 0 ? cp.y + cm.y : cp.x - cm.x;
    }
};

}  // namespace hfmm
