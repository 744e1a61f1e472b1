// Stage II as Eq. 6 states it (Section 5.2): each free line f (a column of
// R outside the template, or a row) is represented in the fixed template
// basis by a coefficient vector c_f with one entry per basis line, and its
// entries are predicted as R*_i c_f.  In factored form R* = P B^T, so the
// prediction of entry (i, f) is p_i . x_f with x_f = B^T c_f (k numbers), and
//   L(C) = sum (r - p . x_f)^2 + lambda ||C||_F^2,
//   dL/dc_f = B g_f + 2 lambda c_f,   g_f = -2 sum (r - p . x_f) p.
// The coefficients move by the Adam method (bias-corrected first and second
// moment estimates, elementwise step lr m^ / (sqrt(w^) + eps)), from C = 0.
//
// A step is two launches (three with long lines), free lines being independent:
//  the item pass  the residual of every entry of f and sum_e e p, with x_f as
//                 the owner row (the sum of the previous step's partial
//                 products, in slice order) and F the gathered table: the
//                 template fit's per-cell kernel, its sums stored per free
//                 line instead of an update.
//  k_adam_update  16 free lines and a slice of 256 basis lines: the gradient
//                 of those coefficients, the Adam step, and the slice's
//                 partial product B^T c_f for the next step.
// No atomics: every sum has a fixed order, so results repeat bit for bit.
#include <hip/hip_ext.h>

#include "internal.h"

namespace tsid {

namespace {

constexpr int kAdamUpdWaves = 4;
constexpr int kAdamLines = 16;  // free lines of a workgroup

typedef float f4v __attribute__((ext_vector_type(4)));

// x_f = B^T c_f: the slices' partial products of free line f, in slice order
// (zero without slices).
template <int K>
__global__ __launch_bounds__(256) void k_adam_x(const AdamArgs A, int32_t n_slices) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= A.n_free * K) return;
    const int64_t f = t / K;
    const int c = (int)(t % K);
    float x = 0.f;
    for (int32_t s = 0; s < n_slices; ++s) x += A.qpart[(f * n_slices + s) * K + c];
    A.X[t] = x;
}

// K / 4 floats from a 16-byte (k = 8: 8-byte) boundary.
template <int KQ>
__device__ __forceinline__ void load_quarter(const float *p, float (&x)[KQ]) {
    if constexpr (KQ % 4 == 0) {
#pragma unroll
        for (int i = 0; i < KQ; i += 4) {
            const float4 t = *reinterpret_cast<const float4 *>(p + i);
            x[i] = t.x, x[i + 1] = t.y, x[i + 2] = t.z, x[i + 3] = t.w;
        }
    } else {
        static_assert(KQ == 2, "ranks are multiples of 8");
        const float2 t = *reinterpret_cast<const float2 *>(p);
        x[0] = t.x, x[1] = t.y;
    }
}

// One workgroup per 16 free lines and slice of 256 basis lines, wave w taking
// the slice's lines 64 w .. + 63 in tiles of 16.  Both products of a step are
// contractions and run on the matrix cores in fp32
// (v_mfma_f32_16x16x4_f32: lane l holds A[l%16][l/16], B[l/16][l%16] and
// C[4(l/16)+j][l%16], j = 0..3); with q = l/16, c = l%16:
//  1. S = B_tile G^T (16 basis lines x 16 free lines): lane l loads
//     coordinates q K/4 .. + K/4 - 1 of basis line c and of free line c's
//     gradient, which orders the contraction the same way on both sides.  It
//     ends with dL/dx . b for basis lines 4 q .. + 3 of free line c: four
//     neighbours of that line's coefficients.
//  2. The Adam step on those four (16-byte loads and stores of C, M and V).
//  3. X += C_tile B_tile: the four coefficients are the A operands as they
//     stand, operand j covering basis lines 4 q + j.
// The waves' partial products are added in wave order through LDS.  fp32 sums
// in long chains lose digits, so S takes four chains of K / 4 coordinates and
// each tile's part of X a chain of its own: errors against 64 bits at k = 64,
// 1,024 basis lines, 8.4e-8 (S) and 4.9e-8 (X), where two chains of K / 2 and one
// chain of 64 basis lines left 1.07e-7 and 6.4e-8.  At k = 64 three waves a SIMD
// need the register cap (47.2 us a step of 1,000 lines x 4,096 basis lines; 49.1
// with two).  What bounds
// it: the coefficients' and moments' 24 bytes each way per coefficient and step
// (they stay in the memory-side cache), and the latency of a tile's chain of
// loads, product, step, product.  500 free lines x 4,096 basis lines at k = 64:
// 44.6 -> 20 us a step (one wave per free line and slice, dot products by lane
// shuffles, before); 8 waves of two tiles each instead of 4 of four, more waves
// in flight without the two tiles in turn, took 25 us.
template <int K, bool FIRST>
__global__ __launch_bounds__(64 * kAdamUpdWaves, K == 64 ? 3 : 1) void k_adam_update(const AdamArgs A, float c1, float c2) {
    constexpr int KQ = K / 4;             // coordinates per lane in step 1
    constexpr int NX = (K + 15) / 16;     // 16-coordinate blocks of step 3
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int q = lane >> 4, c = lane & 15;
    __shared__ float red[kAdamUpdWaves][kAdamLines * K];
    const int64_t f0 = (int64_t)blockIdx.x * kAdamLines;
    const int64_t f = f0 + c;
    const bool own = f < A.n_free;
    const int64_t fl = own ? f : A.n_free - 1;
    const bool live = !(A.skip_after_nonfinite && A.err[ERR_NONFINITE]);
    const int32_t s = blockIdx.y;
    f4v xa[NX];
#pragma unroll
    for (int nb = 0; nb < NX; ++nb) xa[nb] = f4v{0.f, 0.f, 0.f, 0.f};
    const bool vec = (A.n_b & 3) == 0;  // the four coefficients are one 16-byte word
    bool bad = false;
    struct Tile {
        float b[KQ], bx[NX][4], cj[4], m[4], v[4];
    };
    auto load = [&](int64_t l0, Tile &T) {
        const int64_t lb = l0 + c < A.n_b ? l0 + c : A.n_b - 1;
        load_quarter<KQ>(A.B + lb * K + q * KQ, T.b);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t l = l0 + 4 * q + j, lx = l < A.n_b ? l : A.n_b - 1;
#pragma unroll
            for (int nb = 0; nb < NX; ++nb) T.bx[nb][j] = A.B[lx * K + (K >= 16 ? 16 * nb + c : c & (K - 1))];
        }
        if constexpr (!FIRST) {
            const int64_t at = fl * A.n_b + l0 + 4 * q;
            if (vec) {
                const int64_t a4 = l0 + 4 * q < A.n_b ? at : fl * A.n_b;
                const float4 x = *reinterpret_cast<const float4 *>(A.C + a4);
                const float4 y = *reinterpret_cast<const float4 *>(A.M + a4);
                const float4 z = *reinterpret_cast<const float4 *>(A.V + a4);
                T.cj[0] = x.x, T.cj[1] = x.y, T.cj[2] = x.z, T.cj[3] = x.w;
                T.m[0] = y.x, T.m[1] = y.y, T.m[2] = y.z, T.m[3] = y.w;
                T.v[0] = z.x, T.v[1] = z.y, T.v[2] = z.z, T.v[3] = z.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t a1 = l0 + 4 * q + j < A.n_b ? at + j : fl * A.n_b;
                    T.cj[j] = A.C[a1];
                    T.m[j] = A.M[a1];
                    T.v[j] = A.V[a1];
                }
            }
        } else {  // all zero before the first step
#pragma unroll
            for (int j = 0; j < 4; ++j) T.cj[j] = T.m[j] = T.v[j] = 0.f;
        }
    };
    // two tiles in turn, the next one's loads before this one's stores; the
    // first one's go ahead of the chain item_off -> sums
    const int64_t first = (int64_t)s * 256 + wv * 64;
    Tile ta, tb;
    if (first < A.n_b) load(first, ta);
    // dL/dx of line c: the item pass's sum, or the sums that its waves left
    // when the line's items lie in several
    float gv[KQ];
    const uint32_t i0 = A.item_off[fl], i1 = A.item_off[fl + 1], ng = (uint32_t)A.items_per_wave;
    if (i1 - i0 <= 1 || i0 / ng == (i1 - 1) / ng) {
        load_quarter<KQ>(A.gt + fl * K + q * KQ, gv);
    } else {
#pragma unroll
        for (int i = 0; i < KQ; ++i) gv[i] = 0.f;
        // a partial sum keeps the pass's lane order
        constexpr int W = KQ < 4 ? KQ : 4;  // neighbours in both orders
        for (uint32_t it = i0; it < i1; it = (it / ng + 1) * ng) {
            const float *p = A.carry + (int64_t)it * K;
#pragma unroll
            for (int i = 0; i < KQ; i += W) {
                float part[W];
                load_quarter<W>(p + ItemLanes<K>::place(q * KQ + i), part);
#pragma unroll
                for (int j = 0; j < W; ++j) gv[i + j] += part[j];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < KQ; ++i) gv[i] *= -2.f;  // dL/dx_f = -2 sum_e e p
    auto step = [&](int64_t l0, Tile &T) {
        constexpr int NS = KQ < 4 ? KQ : 4;  // chains of the dot product, of K / 4 terms at most (k = 8: 4)
        f4v sc[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) sc[i] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KQ; ++i) sc[i % NS] = __builtin_amdgcn_mfma_f32_16x16x4f32(T.b[i], gv[i], sc[i % NS], 0, 0, 0);
        f4v st = sc[0] + sc[1];
        if constexpr (NS == 4) st += sc[2] + sc[3];
        float cn[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float gr = 2.f * A.lambda * T.cj[j] + st[j];
            T.m[j] = A.beta1 * T.m[j] + (1.f - A.beta1) * gr;
            T.v[j] = A.beta2 * T.v[j] + (1.f - A.beta2) * gr * gr;
            cn[j] = T.cj[j] - A.lr * (T.m[j] * c1) / (sqrtf(T.v[j] * c2) + A.eps);
            if (!live) cn[j] = T.cj[j];
        }
        const int64_t at = fl * A.n_b + l0 + 4 * q;
        if (own && (live || FIRST)) {
            if (vec) {
                if (l0 + 4 * q < A.n_b) {
                    *reinterpret_cast<float4 *>(A.C + at) = make_float4(cn[0], cn[1], cn[2], cn[3]);
                    *reinterpret_cast<float4 *>(A.M + at) = make_float4(T.m[0], T.m[1], T.m[2], T.m[3]);
                    *reinterpret_cast<float4 *>(A.V + at) = make_float4(T.v[0], T.v[1], T.v[2], T.v[3]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (l0 + 4 * q + j < A.n_b) {
                        A.C[at + j] = cn[j];
                        A.M[at + j] = T.m[j];
                        A.V[at + j] = T.v[j];
                    }
            }
        }
        f4v xt[NX];  // this tile's product, a chain of 16 terms
#pragma unroll
        for (int nb = 0; nb < NX; ++nb) xt[nb] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = l0 + 4 * q + j < A.n_b;
            bad |= own && in && !__builtin_isfinite(cn[j]);
            if (!in) cn[j] = 0.f;  // lines past the basis add nothing
#pragma unroll
            for (int nb = 0; nb < NX; ++nb)
                xt[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(cn[j], T.bx[nb][j], xt[nb], 0, 0, 0);
        }
#pragma unroll
        for (int nb = 0; nb < NX; ++nb) xa[nb] += xt[nb];
    };
    for (int i = 0; i < 4; i += 2) {
        const int64_t l0 = first + 16 * i;
        if (l0 >= A.n_b) break;  // the same for the whole wave
        const bool more = l0 + 16 < A.n_b;
        if (more) load(l0 + 16, tb);
        step(l0, ta);
        if (!more) break;
        if (i + 2 < 4 && l0 + 32 < A.n_b) load(l0 + 32, ta);
        step(l0 + 16, tb);
    }
    // lane l holds X[free line 4 q + i][coordinate 16 nb + c]
#pragma unroll
    for (int nb = 0; nb < NX; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (K >= 16 || c < K) red[wv][(4 * q + i) * K + 16 * nb + c] = xa[nb][i];
    __syncthreads();
    for (int o = threadIdx.x; o < kAdamLines * K; o += 64 * kAdamUpdWaves) {
        const int64_t fo = f0 + o / K;
        if (fo < A.n_free) {
            float t = red[0][o];
#pragma unroll
            for (int w = 1; w < kAdamUpdWaves; ++w) t += red[w][o];
            A.qpart[(fo * A.n_slices + s) * K + o % K] = t;
        }
    }
    if (bad) A.err[ERR_NONFINITE] = 1;
}

template <int K>
void adam_k(const AdamArgs &a, int32_t steps, hipStream_t st) {
    const double b1 = a.beta1, b2 = a.beta2;
    double b1t = 1.0, b2t = 1.0;
    const dim3 gu((unsigned)((a.n_free + kAdamLines - 1) / kAdamLines), (unsigned)a.n_slices);
    const unsigned gx = (unsigned)((a.n_free * K + 255) / 256);
    // the gradient's item pass: owner rows x_f (the slices' sums), gathered
    // rows of F, each free line's sum stored in gt instead of an update
    PassArgs g{};
    g.stream = a.stream;
    g.ptr = a.ptr;
    g.items = a.items;
    g.item_off = a.item_off;
    g.item_end = a.item_off + 1;
    g.n_items_dev = a.item_off + a.n_free;
    g.n_items = (int32_t)a.n_items_ub;
    g.rows = (int32_t)a.n_free;
    g.E = a.E;
    g.X = a.qpart;
    g.Y = a.F;
    g.y_rows = a.n_fixed;
    g.carry = a.carry;
    g.err = a.err;
    g.epoch = INT32_MAX;  // skipped once any step has stored a non-finite flag
    g.skip_after_nonfinite = a.skip_after_nonfinite;
    g.partial_out = a.gt;
    // The update's workgroups add the partial sums of lines that span waves
    // themselves, every slice and wave anew, which saves a launch; past 16 MB of such
    // reads, or 32 sums a line (each is a dependent round of the line's chain), one
    // fixup launch is the cheaper one.  us a step, without -> with it: k = 64, 100
    // lines of 5,000 cells, 16 / 64 / 512 slices 39.7 -> 42.2 / 60.5 -> 53.1 / 269
    // -> 187; of 20,000 cells, 4 / 512 slices 97 -> 91 / 718 -> 310; k = 128, 1,000
    // lines of 640 cells, 4 / 16 slices 49.4 -> 52.8 / 101.2 -> 98.6, 100 of 20,000
    // cells, 4 slices 196 -> 156.
    const int64_t sums = (a.n_items_ub - a.n_free) / a.items_per_wave;
    const bool fix = sums * a.n_slices * K > (int64_t(4) << 20) || sums > 32 * a.n_free;
    AdamArgs u = a;
    if (fix) u.items_per_wave = INT32_MAX;  // every line's sum is in gt
    for (int32_t t = 1; t <= steps; ++t) {
        b1t *= b1;
        b2t *= b2;
        const float c1 = (float)(1.0 / (1.0 - b1t)), c2 = (float)(1.0 / (1.0 - b2t));
        launch_item_pass_parts(K, g, t == 1 ? 0 : a.n_slices, st);
        if (fix) launch_fixup(K, TSID_FP32, g, st);
        if (t == 1)
            hipLaunchKernelGGL((k_adam_update<K, true>), gu, dim3(64 * kAdamUpdWaves), 0, st, u, c1, c2);
        else
            hipLaunchKernelGGL((k_adam_update<K, false>), gu, dim3(64 * kAdamUpdWaves), 0, st, u, c1, c2);
        TSID_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_adam_x<K>, dim3(gx), dim3(256), 0, st, a, steps > 0 ? a.n_slices : 0);
    TSID_HIP(hipGetLastError());
}

}  // namespace

bool adam_supported(int K) { return K == 8 || K == 16 || K == 32 || K == 64 || K == 128; }

int32_t adam_slices(int64_t n_b) { return (int32_t)((n_b + 255) / 256); }

void launch_adam(int K, const AdamArgs &a, int32_t steps, hipStream_t s) {
    if (a.n_free <= 0) return;
    switch (K) {
        case 8: adam_k<8>(a, steps, s); break;
        case 16: adam_k<16>(a, steps, s); break;
        case 32: adam_k<32>(a, steps, s); break;
        case 64: adam_k<64>(a, steps, s); break;
        case 128: adam_k<128>(a, steps, s); break;
        default: fail(TSID_E_INVAL, "the Adam extension supports k in {8, 16, 32, 64, 128}");
    }
}

}  // namespace tsid
