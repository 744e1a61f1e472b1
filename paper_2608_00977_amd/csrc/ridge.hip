// Exact one-sided solve of an extension chunk (Section 5.2; Eq. 6 in factored
// form): with the fixed side's factors held constant, each free row x_f is
// the ridge regression
//   x_f = argmin sum_(u in cells of f) (r_u - p_u . x)^2 + lambda ||x||^2
//       = (sum_u p_u p_u^T + lambda I)^{-1} sum_u r_u p_u,
// the fixed point that the gradient steps of k_extend_steps approach (the
// alternating-least-squares step of the paper's Stage II).  Everything is
// fp64: the Gram matrix of a row with fewer cells than k is singular up to
// lambda, and fp32 would lose the directions lambda alone fixes.
//
// One wave per free row:
//  1. Gram and right-hand side.  Four cells at a time, each lane loads one
//     coordinate of each 16-coordinate block of one cell's fixed row (lane l:
//     cell l/16, coordinate 16 I + l%16), which is at once the A operand
//     A[l%16][l/16] and the B operand B[l/16][l%16] of v_mfma_f64_16x16x4f64,
//     so block (I, J) of the Gram matrix accumulates with one MFMA per block
//     pair I <= J (10 at k = 64).  Lane l, slot j of a result holds
//     C[4 j + l/16][l%16].  The right-hand side accumulates per lane, over the
//     cells of its quarter of the wave.
//  2. Cholesky G = U^T U on the matrix cores, four rows at a time, the blocks
//     never leaving the accumulators.  Slot s of block row I holds rows
//     16 I + 4 s + l/16, and that is both the A operand of its transpose and
//     a B operand.  Per group of four rows: the 4 x 4 diagonal block (broadcast
//     with readlane) is factored and inverted by every lane, M = L^-1; one
//     product M x slot per block column gives the rows of U; and the trailing
//     blocks (J, L) take -U_J^T U_L, one product each.
//  3. U^T z = b goes along (z = M b of the group, the rest of b less its rows
//     of U times z, per quarter), then U x = z, group by group from the last:
//     a row's product with x by a sum over its 16 lanes, then M^T.
// A pivot that is not positive (lambda = 0 and fewer independent cells than
// k) raises the non-finite error; a row without cells gets x = 0.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "internal.h"

namespace tsid {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double readlane_f64(double v, int l) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int K>
struct RidgeShape {
    static constexpr int NB = (K + 15) / 16;          // 16-coordinate blocks
    static constexpr int NP = NB * (NB + 1) / 2;      // block pairs I <= J
    static constexpr int PITCH = K + 1;               // LDS row pitch (doubles)
};

// Gram blocks (block pairs I <= J) and right-hand side of one free row's
// cells b0 .. b1 (b1 > b0), by one wave with the operand layout above.  A ring
// of U groups of four cells: a group's fixed rows load while the U - 1 groups
// before it take their products (640 cycles a group at k = 64, 192 at k = 32),
// and its records load a round earlier, so a row alone on its SIMD (long
// rows are few) does not wait for the two memory round trips, and a group's
// conversions issue under the products of the one before.  Loads past the
// row's end re-read its last cell.  The last round stands apart: the full ones
// need no masks (which keeps k = 32 at four waves a SIMD), and it takes only the
// groups that have a cell, so a row of two cells loads and multiplies one group,
// not U.  Chunks of 12 M cells in Gram form (k = 32, 20 steps), rows of 100 /
// 1,000 cells: 1,337 / 752 -> 1,096 / 605 us with the last round apart.
template <int K>
__device__ __forceinline__ void gram_line(const RidgeArgs &A, int64_t b0, int64_t b1, int lane,
                                          d4 (&acc)[RidgeShape<K>::NP], double (&rhs)[RidgeShape<K>::NB]) {
    using S = RidgeShape<K>;
    constexpr int U = K >= 64 ? 4 : 8;
    const int lr = lane & 15, lq = lane >> 4;
#pragma unroll
    for (int q = 0; q < S::NP; ++q) acc[q] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int I = 0; I < S::NB; ++I) rhs[I] = 0.0;
    // the round's first cell and how many are left from it (as far as a round
    // and the loads ahead of it reach)
    const int2 *first = A.stream + b0;
    auto left_from = [&](int64_t c0) { return (int)(b1 - c0 < (1 << 16) ? b1 - c0 : (1 << 16)); };
    int left = left_from(b0);
    int2 rec[U];
    float raw[U][S::NB], val[U];
    auto load_record = [&](int u, int ahead) {
        const int c = ahead + 4 * u + lq;
        rec[u] = first[c < left ? c : left - 1];
    };
    auto load_row = [&](int u) {
        val[u] = __int_as_float(rec[u].y);
        const float *p = A.F + (int64_t)rec[u].x * K;
#pragma unroll
        for (int I = 0; I < S::NB; ++I) raw[u][I] = p[(K % 16 == 0 || 16 * I + lr < K) ? 16 * I + lr : K - 1];
    };
    auto products = [&](const double rv, const double (&pv)[S::NB]) {
        int q = 0;
#pragma unroll
        for (int I = 0; I < S::NB; ++I) {
            rhs[I] = fma(rv, pv[I], rhs[I]);
#pragma unroll
            for (int J = I; J < S::NB; ++J, ++q)
                acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(pv[I], pv[J], acc[q], 0, 0, 0);
        }
    };
    auto inside = [&](int I) { return K % 16 == 0 || 16 * I + lr < K; };
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (4 * u < left) load_record(u, 0);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (4 * u < left) load_row(u);
    if (left > 4 * U) {
#pragma unroll
        for (int u = 0; u < U; ++u) load_record(u, 4 * U);
    }
    for (int64_t c0 = b0; left > 4 * U; c0 += 4 * U, first += 4 * U, left = left_from(c0)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double rv = (double)val[u];
            double pv[S::NB];
#pragma unroll
            for (int I = 0; I < S::NB; ++I) pv[I] = inside(I) ? (double)raw[u][I] : 0.0;
            load_row(u);
            load_record(u, 8 * U);
            products(rv, pv);
        }
    }
    // the last round: the groups that have a cell
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (4 * u >= left) break;
        const bool in = 4 * u + lq < left;
        double pv[S::NB];
#pragma unroll
        for (int I = 0; I < S::NB; ++I) pv[I] = in && inside(I) ? (double)raw[u][I] : 0.0;
        products(in ? (double)val[u] : 0.0, pv);
    }
}

// The Gram blocks and their mirror images to LDS (pitch K + 1); the
// right-hand side summed over the four cell slots, lane i returning b_i.
template <int K>
__device__ __forceinline__ double gram_to_lds(const d4 (&acc)[RidgeShape<K>::NP], double (&rhs)[RidgeShape<K>::NB],
                                              double *G, int lane) {
    using S = RidgeShape<K>;
    const int lr = lane & 15, lq = lane >> 4;
    int q = 0;
#pragma unroll
    for (int I = 0; I < S::NB; ++I) {
#pragma unroll
        for (int J = I; J < S::NB; ++J, ++q) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = 16 * I + 4 * j + lq, col = 16 * J + lr;
                if (row < K && col < K) {
                    G[row * S::PITCH + col] = acc[q][j];
                    G[col * S::PITCH + row] = acc[q][j];
                }
            }
        }
    }
    // coordinate i = 16 (i / 16) + i % 16 sits in lane i after the sums
#pragma unroll
    for (int I = 0; I < S::NB; ++I) {
        rhs[I] += __shfl_xor(rhs[I], 16, 64);
        rhs[I] += __shfl_xor(rhs[I], 32, 64);
    }
    double b = 0.0;
#pragma unroll
    for (int I = 0; I < S::NB; ++I) b = (lq == I) ? rhs[I] : b;
    return b;
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over the four lanes l % 16 + {0, 16, 32, 48}, in every one of them.
__device__ __forceinline__ double sum_quarters(double v) {
    uint64_t u = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    v = __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
        __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
    u = __builtin_bit_cast(uint64_t, v);
    const auto lo2 = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi2 = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)hi2[0] << 32) | lo2[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi2[1] << 32) | lo2[1]);
}

// 1 / sqrt(d) for a pivot d (a pivot that is not positive marks the row bad
// and counts as 1): the hardware's estimate and two third-order Newton steps
// r <- r (1 + e/2 + 3 e^2 / 8), e = 1 - d r^2.
__device__ __forceinline__ double pivot_rsqrt(double d, bool &bad) {
    bad |= !(d > 0.0);
    d = d > 0.0 ? d : 1.0;
    double r = __builtin_amdgcn_rsq(d);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double e = fma(-d * r, r, 1.0);
        r = fma(r * e, fma(0.375, e, 0.5), r);
    }
    return r;
}

// One free row per wave, four to a workgroup; no LDS.  What bounds it: at
// k = 64 the fp64 matrix cores (64 cycles a product, 10 per four cells and 120
// for the factorisation) and the chain through the 16 groups of four rows.
// k = 64, rows of about 97 cells: 446 -> 199 us a chunk of 10,000 rows (the
// earlier form kept a row of the trailing matrix per lane and broadcast each
// column element by element with readlane: 64 dependent steps, half of the
// lanes idle).  Rows of a few cells at k = 8 are bound by the instructions around
// the one block: 1 M rows of 2 cells 1,137 us (1,568 in the earlier form, 2,474
// while all four groups of the padded block were factored and every row took a
// whole round of the Gram matrix).
template <int K>
__global__ __launch_bounds__(256, 2) void k_ridge_rows(const RidgeArgs A) {
    using S = RidgeShape<K>;
    constexpr int NB = S::NB;
    const int lane = threadIdx.x & 63;
    const int64_t f = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // free row
    if (f >= A.rows) return;  // whole waves leave together
    const int64_t b0 = A.ptr[f], b1 = A.ptr[f + 1];
    if (b0 == b1) {  // no cells: the minimiser is 0
        if (lane < K) A.X[f * K + lane] = 0.f;
        return;
    }
    const int lr = lane & 15, lq = lane >> 4;
    d4 acc[S::NP];
    double rhs[NB];  // this quarter's share of b[16 I + lr]
    gram_line<K>(A, b0, b1, lane, acc, rhs);
    auto at = [](int I, int J) { return I * NB - I * (I - 1) / 2 + J - I; };  // block (I, J), I <= J
    // lambda on the diagonal (coordinates past k: 1, they stay apart)
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (lr == 4 * j + lq) acc[at(I, I)][j] += 16 * I + lr < K ? (double)A.lambda : 1.0;
    // groups of four rows of block row I; at k = 8 the block's other half stays apart
    constexpr auto groups = [](int I) constexpr { return K - 16 * I < 16 ? (K - 16 * I) / 4 : 4; };
    const int ma = lr & 3;  // the row of M in this lane's A operand; its column is lq
    double mv[NB][4], zv[NB][4];  // per group: M[ma][lq], and z of row 4 s + lq
    bool bad = false;
#pragma unroll
    for (int I = 0; I < NB; ++I) {
#pragma unroll
        for (int s = 0; s < groups(I); ++s) {
            const double g = acc[at(I, I)][s];
            auto el = [&](int a, int c) { return readlane_f64(g, 16 * a + 4 * s + c); };
            const double d00 = el(0, 0), d01 = el(0, 1), d02 = el(0, 2), d03 = el(0, 3);
            const double d11 = el(1, 1), d12 = el(1, 2), d13 = el(1, 3), d22 = el(2, 2), d23 = el(2, 3), d33 = el(3, 3);
            const double i0 = pivot_rsqrt(d00, bad);
            const double l10 = d01 * i0, l20 = d02 * i0, l30 = d03 * i0;
            const double i1 = pivot_rsqrt(fma(-l10, l10, d11), bad);
            const double l21 = fma(-l10, l20, d12) * i1, l31 = fma(-l10, l30, d13) * i1;
            const double i2 = pivot_rsqrt(fma(-l21, l21, fma(-l20, l20, d22)), bad);
            const double l32 = fma(-l21, l31, fma(-l20, l30, d23)) * i2;
            const double i3 = pivot_rsqrt(fma(-l32, l32, fma(-l31, l31, fma(-l30, l30, d33))), bad);
            const double m10 = -(l10 * i0) * i1, m21 = -(l21 * i1) * i2, m32 = -(l32 * i2) * i3;
            const double m20 = -fma(l21, m10, l20 * i0) * i2, m31 = -fma(l32, m21, l31 * i1) * i3;
            const double m30 = -fma(l32, m20, fma(l31, m10, l30 * i0)) * i3;
            // M[ma][lq], zero above the diagonal
            const double c0 = ma == 0 ? i0 : ma == 1 ? m10 : ma == 2 ? m20 : m30;
            const double c1 = ma == 1 ? i1 : ma == 2 ? m21 : ma == 3 ? m31 : 0.0;
            const double c2 = ma == 2 ? i2 : ma == 3 ? m32 : 0.0;
            const double c3 = ma == 3 ? i3 : 0.0;
            const double m = lq == 0 ? c0 : lq == 1 ? c1 : lq == 2 ? c2 : c3;
            mv[I][s] = m;
            // the group's rows of U: every slot of the product holds them
            double u[NB];
#pragma unroll
            for (int J = I; J < NB; ++J) {
                const d4 p = __builtin_amdgcn_mfma_f64_16x16x4f64(m, acc[at(I, J)][s], d4{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
                u[J] = p[s];
                acc[at(I, J)][s] = u[J];
            }
#pragma unroll
            for (int J = I; J < NB; ++J) {
                if (J == I && s == groups(I) - 1) continue;  // block row I is done
                // A rows of this block row that are already U are zero: they stay as they are
                const double n = J > I || lr >= 4 * (s + 1) ? -u[J] : 0.0;
#pragma unroll
                for (int L = J; L < NB; ++L)
                    acc[at(J, L)] = __builtin_amdgcn_mfma_f64_16x16x4f64(n, u[L], acc[at(J, L)], 0, 0, 0);
            }
            // z = M b for the group, and its part taken out of the rest of b
            const double bs = sum_quarters(rhs[I]);
            const double y0 = readlane_f64(bs, 4 * s), y1 = readlane_f64(bs, 4 * s + 1),
                         y2 = readlane_f64(bs, 4 * s + 2), y3 = readlane_f64(bs, 4 * s + 3);
            const double z0 = i0 * y0, z1 = fma(m10, y0, i1 * y1), z2 = fma(m20, y0, fma(m21, y1, i2 * y2)),
                         z3 = fma(m30, y0, fma(m31, y1, fma(m32, y2, i3 * y3)));
            const double z = lq == 0 ? z0 : lq == 1 ? z1 : lq == 2 ? z2 : z3;
            zv[I][s] = z;
#pragma unroll
            for (int J = I; J < NB; ++J) rhs[J] = fma(-u[J], z, rhs[J]);
        }
    }
    // U x = z: x[16 I + lr] in every quarter, zero until its group is solved
    double x[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) x[I] = 0.0;
#pragma unroll
    for (int I = NB - 1; I >= 0; --I) {
#pragma unroll
        for (int s = groups(I) - 1; s >= 0; --s) {
            double t = 0.0;
#pragma unroll
            for (int J = I; J < NB; ++J) t = fma(acc[at(I, J)][s], x[J], t);
            t += dpp_f64<0xB1>(t);
            t += dpp_f64<0x4E>(t);
            t += dpp_f64<0x141>(t);
            t += dpp_f64<0x140>(t);
            const double w = zv[I][s] - t;  // row 4 s + lq
            const double w0 = readlane_f64(w, 0), w1 = readlane_f64(w, 16), w2 = readlane_f64(w, 32),
                         w3 = readlane_f64(w, 48);
            // x of row lq: sum over a of M[a][lq] w_a, the four lanes of a quad
            double v = mv[I][s] * (ma == 0 ? w0 : ma == 1 ? w1 : ma == 2 ? w2 : w3);
            v += dpp_f64<0xB1>(v);
            v += dpp_f64<0x4E>(v);
            const double x0 = readlane_f64(v, 0), x1 = readlane_f64(v, 16), x2 = readlane_f64(v, 32),
                         x3 = readlane_f64(v, 48);
            const double xs = ma == 0 ? x0 : ma == 1 ? x1 : ma == 2 ? x2 : x3;
            x[I] = (lr >> 2) == s ? xs : x[I];
        }
    }
    double xl = x[0];  // coordinate `lane`
#pragma unroll
    for (int I = 1; I < NB; ++I) xl = lq == I ? x[I] : xl;
    if (lane < K) {
        const float xf = (float)xl;
        A.X[f * K + lane] = xf;
        if (bad || !__builtin_isfinite(xf)) A.err[ERR_NONFINITE] = 1;  // a bad pivot spoils the whole row
    }
}

// One-sided gradient steps in Gram form (Section 5.2's per-row subproblem
// with Eq. 5's update).  With the fixed side held, the gradient of a free
// row's loss is 2 lambda x - 2 (b - G x), G = sum_u p_u p_u^T and
// b = sum_u r_u p_u over the row's cells, so one pass over the cells (fp64,
// as for the exact solve) gives every step: lane i holds row i of G and b_i,
// and a step is the product G x (x broadcast lane by lane), the gradient, the
// step option's scale, the clip and the update, all in fp64 from x = 0.  The
// per-cell kernel (k_extend_steps) gathers every fixed row once per step; for
// rows of at least gram_min cells this one gathers them once.  Rows shorter
// than gram_min are the per-cell kernel's and are left untouched here.
template <int K>
__global__ __launch_bounds__(64) void k_extend_gram(const RidgeArgs A) {
    using S = RidgeShape<K>;
    __shared__ double G[K * S::PITCH];
    const int lane = threadIdx.x;
    const int64_t f = blockIdx.x;
    if (f >= A.rows) return;
    const int64_t b0 = A.ptr[f], b1 = A.ptr[f + 1], deg = b1 - b0;
    if (deg < A.gram_min || deg == 0) return;
    d4 acc[S::NP];
    double rhs[S::NB];
    gram_line<K>(A, b0, b1, lane, acc, rhs);
    const double b = gram_to_lds<K>(acc, rhs, G, lane);
    __syncthreads();
    const int ri = lane < K ? lane : K - 1;  // lanes past k mirror the last row (never stored)
    double g[K];
#pragma unroll
    for (int c = 0; c < K; ++c) g[c] = G[ri * S::PITCH + c];
    const double lam = A.lambda, lr = A.lr, xi = A.xi;
    const double sc = A.degree ? 1.0 / (double)(deg > 1 ? deg : 1) : 1.0;
    double x = 0.0;
    bool bad = false;
    for (int t = 0; t < A.steps; ++t) {
        // G x in four independent sums (a shorter chain of dependent FMAs)
        double gq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < K; ++c) gq[c & 3] = fma(g[c], readlane_f64(x, c), gq[c & 3]);
        const double gx = (gq[0] + gq[1]) + (gq[2] + gq[3]);
        const double grad = 2.0 * lam * x - 2.0 * (b - gx);
        double d;
        if (A.clip == 3) {  // the printed asymmetric form: the scale outside the clip
            d = -grad;
            if (d > xi) d = xi;
            d *= sc;
        } else {
            d = -sc * grad;
            if (A.clip && d > xi) d = xi;
        }
        x = fma(lr, d, x);
        bad |= !__builtin_isfinite(x);
    }
    if (lane < K) {
        const float xf = (float)x;
        A.X[f * K + lane] = xf;
        if (bad || !__builtin_isfinite(xf)) A.err[ERR_NONFINITE] = 1;
    }
}

template <int K>
void ridge_k(const RidgeArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_ridge_rows<K>, dim3((unsigned)ceil_div(a.rows, 4)), dim3(256), 0, s, a);
    TSID_HIP(hipGetLastError());
}

// k = 128: a row of the Gram matrix does not fit one lane's registers, so
// the matrix lives in LDS (128 x 129 doubles, 129 KiB) and a workgroup of
// four waves solves one free row:
//  1. Gram: the 36 block pairs I <= J of the 8 x 8 blocks are dealt to the
//     waves (pair q to wave q % 4); each wave walks all the row's cells, four
//     at a time, with the operand layout of k_ridge_rows, and wave 0 also
//     sums the right-hand side.
//  2. The blocks and their mirror images go to LDS; lambda joins the
//     diagonal.
//  3. Cholesky, right-looking: at column j every thread reads the pivot
//     d = G[j][j], and the trailing lower triangle takes
//     G[r][c] -= G[r][j] G[c][j] / d (two threads per row r > j, alternate
//     columns); column j - 1 is scaled by 1 / sqrt of its pivot in the same
//     phase (no thread reads it any more), so one barrier per column.
//  4. Wave 0 solves L z = b and L^T x = z, lane l holding rows l and l + 64,
//     the pivots of each step broadcast with readlane.
constexpr int kR128 = 128, kR128Pitch = kR128 + 1, kR128Threads = 256;
constexpr int kR128Lds = (kR128 * kR128Pitch + kR128) * 8;

__global__ __launch_bounds__(kR128Threads) void k_ridge_rows_128(const RidgeArgs A) {
    constexpr int K = kR128, NB = K / 16, PITCH = kR128Pitch;
    extern __shared__ double lds[];
    double *G = lds;                  // K x PITCH
    double *rhs = lds + K * PITCH;    // K
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t f = blockIdx.x;
    if (f >= A.rows) return;
    const int lr = lane & 15, lq = lane >> 4;
    const int64_t b0 = A.ptr[f], b1 = A.ptr[f + 1];
    if (b0 == b1) {
        if (tid < K) A.X[f * K + tid] = 0.f;
        return;
    }
    // 1. this wave's block pairs (slot q / 4 of pair q = 4 s + wv)
    d4 acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) acc[q] = d4{0.0, 0.0, 0.0, 0.0};
    double rb[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) rb[I] = 0.0;
    for (int64_t c0 = b0; c0 < b1; c0 += 4) {
        const int64_t c = c0 + lq;
        double pv[NB];
        double rv = 0.0;
#pragma unroll
        for (int I = 0; I < NB; ++I) pv[I] = 0.0;
        if (c < b1) {
            const int2 rec = A.stream[c];
            rv = (double)__int_as_float(rec.y);
            const float *p = A.F + (int64_t)rec.x * K;
#pragma unroll
            for (int I = 0; I < NB; ++I) pv[I] = (double)p[16 * I + lr];
        }
        if (wv == 0) {
#pragma unroll
            for (int I = 0; I < NB; ++I) rb[I] = fma(rv, pv[I], rb[I]);
        }
        int q = 0;
#pragma unroll
        for (int I = 0; I < NB; ++I) {
#pragma unroll
            for (int J = I; J < NB; ++J, ++q)
                if ((q & 3) == wv) acc[q >> 2] = __builtin_amdgcn_mfma_f64_16x16x4f64(pv[I], pv[J], acc[q >> 2], 0, 0, 0);
        }
    }
    // 2. blocks (and mirrors) to LDS; the right-hand side summed over the four cell slots
    {
        int q = 0;
#pragma unroll
        for (int I = 0; I < NB; ++I) {
#pragma unroll
            for (int J = I; J < NB; ++J, ++q) {
                if ((q & 3) != wv) continue;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int row = 16 * I + 4 * j + lq, col = 16 * J + lr;
                    G[row * PITCH + col] = acc[q >> 2][j];
                    G[col * PITCH + row] = acc[q >> 2][j];
                }
            }
        }
    }
    if (wv == 0) {
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            double v = rb[I];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (lq == 0) rhs[16 * I + lr] = v;
        }
    }
    __syncthreads();
    if (tid < K) G[tid * PITCH + tid] += (double)A.lambda;
    __syncthreads();
    // 3. Cholesky
    bool bad = false;
    const int half = tid & 1;
    double dprev = 1.0;  // the previous column's pivot (read before it was overwritten)
    for (int j = 0; j < K; ++j) {
        const double d = G[j * PITCH + j];
        bad |= !(d > 0.0);
        if (j > 0 && tid < K - j + 1) {  // scale column j - 1 (rows j - 1 .. K - 1)
            const int r = j - 1 + tid;
            const double lp = sqrt(dprev > 0.0 ? dprev : 1.0);
            G[r * PITCH + (j - 1)] = r == j - 1 ? lp : G[r * PITCH + (j - 1)] / lp;
        }
        dprev = d;
        const double inv = 1.0 / (d > 0.0 ? d : 1.0);
        const int r = j + 1 + (tid >> 1);
        if (r < K) {
            const double a = G[r * PITCH + j] * inv;
            for (int c = j + 1 + half; c <= r; c += 2) G[r * PITCH + c] = fma(-a, G[c * PITCH + j], G[r * PITCH + c]);
        }
        __syncthreads();
    }
    if (tid == 0)  // the last column's pivot
        G[(K - 1) * PITCH + (K - 1)] = sqrt(dprev > 0.0 ? dprev : 1.0);
    __syncthreads();
    // 4. triangular solves by wave 0: lane l holds rows l and l + 64
    bad = __syncthreads_or(bad);
    if (wv == 0) {
        double bl = rhs[lane], bh = rhs[lane + 64];
        for (int c = 0; c < K; ++c) {  // L z = b, column by column
            const double lcc = G[c * PITCH + c];
            const double zc = (c < 64 ? readlane_f64(bl, c) : readlane_f64(bh, c - 64)) / lcc;
            if (lane == c) bl = zc;
            else if (lane > c) bl = fma(-G[lane * PITCH + c], zc, bl);
            if (lane + 64 == c) bh = zc;
            else if (lane + 64 > c) bh = fma(-G[(lane + 64) * PITCH + c], zc, bh);
        }
        for (int r = K - 1; r >= 0; --r) {  // L^T x = z, row by row
            const double lrr = G[r * PITCH + r];
            const double xr = (r < 64 ? readlane_f64(bl, r) : readlane_f64(bh, r - 64)) / lrr;
            if (lane == r) bl = xr;
            else if (lane < r) bl = fma(-G[r * PITCH + lane], xr, bl);
            if (lane + 64 == r) bh = xr;
            else if (lane + 64 < r) bh = fma(-G[r * PITCH + lane + 64], xr, bh);
        }
        const float xl = (float)bl, xh = (float)bh;
        A.X[f * K + lane] = xl;
        A.X[f * K + lane + 64] = xh;
        if (bad || !__builtin_isfinite(xl) || !__builtin_isfinite(xh)) A.err[ERR_NONFINITE] = 1;
    }
}

void ridge_128(const RidgeArgs &a, hipStream_t s) {
    static const bool lds_ok = [] {
        TSID_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_ridge_rows_128),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kR128Lds));
        return true;
    }();
    (void)lds_ok;
    hipLaunchKernelGGL(k_ridge_rows_128, dim3((unsigned)a.rows), dim3(kR128Threads), kR128Lds, s, a);
    TSID_HIP(hipGetLastError());
}

}  // namespace

bool ridge_supported(int K) { return K == 8 || K == 16 || K == 32 || K == 64 || K == 128; }

// Where the Gram form pays, per free row of d cells.  Gram form: K^2 r fp64
// multiply-adds per cell on the matrix cores (r: the share of the 16 x 16
// blocks it forms, the pairs I <= J) and, per step, the product G x with x
// broadcast lane by lane (about 3 K wave instructions).  Per-cell form: 2 K
// fp32 multiply-adds per cell and step, and the gathers of the row's fixed
// rows.  The line was measured when the per-cell form gathered them again every
// step, as it does now beyond a workgroup's registers only; shorter rows
// are often faster per cell by now (k = 64, 96 cells, a 128 MB table: 388 us a
// chunk against 738), and keep the Gram form for its fp64 sums (error against 64
// bits 4.7e-8 against 9.1e-8).
//  - A fixed table within one XCD's L2 (4 MiB) serves those gathers from L2,
//    and the forms compare by arithmetic: d = T K / (2 T - K r), when
//    2 T > K r.  Rating-shaped rows (k = 64, 20 steps, a 2 MiB table): all in
//    the per-cell form 16.8 ms, Gram form from 96 / 192 / 384 cells 18.5 /
//    17.3 / 17.2 ms; Scientific rows (k = 32, 2 MiB, about 1,500 cells each)
//    0.112 -> 0.094 s in Gram form.
//  - A larger table is gathered from the memory-side cache or HBM, about
//    4 K / 64 wave instructions' worth per cell and step, and the Gram form
//    pays from d = 192 T / (4 T - K r), when 4 T > K r.  Rating-shaped
//    columns (k = 64, a 123 MB table, about 1,160 cells each): 13.2 -> 7.5 ms
//    (7.49-7.56 ms for thresholds 96 to 384); Scientific columns (k = 32,
//    25.6 MB, about 18,000 cells) 1.38 -> 0.73 s.
// At least 16 cells either way.  Tuning knob TSID_EXT_GRAM_MIN: -1 never,
// n > 0 from n cells on.
int64_t extend_gram_min(int K, int32_t steps, int32_t clip, int64_t n_fixed) {
    if (const char *e = std::getenv("TSID_EXT_GRAM_MIN")) {
        const long long v = std::atoll(e);
        if (v != 0) return v < 0 || K > 64 || clip == 2 || steps < 1 ? 0 : (int64_t)v;
    }
    if (K > 64 || clip == 2 || steps < 1) return 0;
    const int nb = (K + 15) / 16, np = nb * (nb + 1) / 2;
    const double r = (double)np / (double)(nb * nb);
    const bool in_l2 = n_fixed * K * 4 <= (int64_t(4) << 20);
    const double den = (in_l2 ? 2.0 : 4.0) * steps - K * r;
    if (den <= 0.0) return 0;
    const double d = in_l2 ? (double)steps * K / den : 192.0 * steps / den;
    return std::max<int64_t>(16, (int64_t)std::ceil(d));
}

void launch_extend_gram(int K, const RidgeArgs &a, hipStream_t s) {
    if (a.rows <= 0 || a.gram_min <= 0) return;
    if (a.rows > INT32_MAX) fail(TSID_E_INVAL, "too many free rows");
    switch (K) {
        case 8: hipLaunchKernelGGL(k_extend_gram<8>, dim3((unsigned)a.rows), dim3(64), 0, s, a); break;
        case 16: hipLaunchKernelGGL(k_extend_gram<16>, dim3((unsigned)a.rows), dim3(64), 0, s, a); break;
        case 32: hipLaunchKernelGGL(k_extend_gram<32>, dim3((unsigned)a.rows), dim3(64), 0, s, a); break;
        case 64: hipLaunchKernelGGL(k_extend_gram<64>, dim3((unsigned)a.rows), dim3(64), 0, s, a); break;
        default: fail(TSID_E_INVAL, "the Gram-form steps support k in {8, 16, 32, 64}");
    }
    TSID_HIP(hipGetLastError());
}

void launch_ridge_rows(int K, const RidgeArgs &a, hipStream_t s) {
    if (a.rows <= 0) return;
    switch (K) {
        case 8: ridge_k<8>(a, s); break;
        case 16: ridge_k<16>(a, s); break;
        case 32: ridge_k<32>(a, s); break;
        case 64: ridge_k<64>(a, s); break;
        case 128: ridge_128(a, s); break;
        default: fail(TSID_E_INVAL, "the exact extension solve supports k in {8, 16, 32, 64, 128}");
    }
}

}  // namespace tsid
