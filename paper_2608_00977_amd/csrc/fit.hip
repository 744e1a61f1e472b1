// Template-fit kernels (Stage I, Section 5.1): per observed cell the residual
// e = r - p_a . q_b, the per-cell gradients of Eqs. 3-4 aggregated into the
// owning factor row, and the row update of Eq. 5 with the asymmetric clip of
// Section 5.3.  The same kernels run the one-sided extension steps of Section
// 5.2 (owner = free rows, gathered side = fixed factors).
//
// Layout and mapping (gfx950, wave64):
//  * A bucketed stream holds one 8-byte {other id, value} record per cell,
//    grouped by the owning row (CSR for the P pass, CSC for the Q pass) and
//    read once per pass with non-temporal loads.
//  * A bucket is cut into work items of at most E cells.  Each item belongs
//    to a group of G = K / V lanes; lane g of the group holds V coordinates of
//    the owner row in registers: [g*V, g*V + V) when V coordinates fill one
//    16-byte chunk of the gathered table, else chunks g, g + G, g + 2G, ...
//    (so that each gather instruction reads consecutive bytes; see Lanes).
//  * Per cell the group gathers the other factor row (16 bytes per lane and
//    chunk), forms the dot product with a DPP butterfly inside the group (all
//    lanes end with the same bits), and accumulates e * q into its registers.
//  * The aggregated gradient goes straight to the owner row when the bucket is
//    one item; split buckets leave one partial sum per item and a fixup kernel
//    adds the parts in item order.  No atomics touch factor or gradient memory,
//    so results are bitwise reproducible.
//  * bf16 mode: the gathered side is a bf16 copy (2 bytes per coordinate, dots
//    by v_dot2_f32_bf16 with fp32 accumulation); the owner row's fp32 master
//    takes the update and a round-to-nearest-even bf16 copy is written beside it.
#include <hip/hip_ext.h>

#include <algorithm>

#include "internal.h"

namespace tsid {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

// Sum over an aligned group of G lanes (G <= 16: the group lies inside one DPP
// row).  Butterfly pairs: quad_perm [1,0,3,2], quad_perm [2,3,0,1],
// row_half_mirror, row_mirror.  IEEE addition commutes, so every lane of the
// group ends with the same bits.
template <int G>
__device__ __forceinline__ float group_sum(float x) {
    if constexpr (G >= 2) x += dpp<0xB1>(x);
    if constexpr (G >= 4) x += dpp<0x4E>(x);
    if constexpr (G >= 8) x += dpp<0x141>(x);
    if constexpr (G >= 16) x += dpp<0x140>(x);
    return x;
}

// Value of lane `t` of this lane's aligned group of G lanes, for every lane
// of the group: ds_swizzle in bit mode, new lane = (lane & ~(G-1)) | t within
// each 32-lane half (and_mask in bits 0-4, or_mask in bits 5-9).
template <int CTRL>
__device__ __forceinline__ int dpp_i(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
}

template <int G>
__device__ __forceinline__ int group_bcast(int v, int t) {
    if constexpr (G == 1) {
        return v;
    } else if constexpr (G == 2) {
        // DPP quad_perm [t, t, 2+t, 2+t]: a VALU move, no LDS traffic
        return t == 0 ? dpp_i<0xA0>(v) : dpp_i<0xF5>(v);
    } else if constexpr (G == 4) {
        // DPP quad_perm [t, t, t, t]
        switch (t) {
            case 0: return dpp_i<0x00>(v);
            case 1: return dpp_i<0x55>(v);
            case 2: return dpp_i<0xAA>(v);
            default: return dpp_i<0xFF>(v);
        }
    } else {
        static_assert(G <= 32, "groups live inside one 32-lane half");
        int out = v;
        // t is a compile-time constant after unrolling; the switch keeps the
        // swizzle pattern an immediate.
        switch (t) {
#define TSID_BCAST_CASE(T_) \
    case T_: out = __builtin_amdgcn_ds_swizzle(v, (0x1F & ~(G - 1)) | ((T_) << 5)); break;
            TSID_BCAST_CASE(0) TSID_BCAST_CASE(1) TSID_BCAST_CASE(2) TSID_BCAST_CASE(3)
            TSID_BCAST_CASE(4) TSID_BCAST_CASE(5) TSID_BCAST_CASE(6) TSID_BCAST_CASE(7)
            TSID_BCAST_CASE(8) TSID_BCAST_CASE(9) TSID_BCAST_CASE(10) TSID_BCAST_CASE(11)
            TSID_BCAST_CASE(12) TSID_BCAST_CASE(13) TSID_BCAST_CASE(14) TSID_BCAST_CASE(15)
#undef TSID_BCAST_CASE
            default: break;
        }
        return out;
    }
}

// IEEE round-to-nearest-even of fp32 to bf16 (NaN stays NaN).
__device__ __forceinline__ uint32_t bf16_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

template <int V>
__device__ __forceinline__ void load_f32(const float *p, float (&x)[V]) {
    const float4 *q = reinterpret_cast<const float4 *>(p);
#pragma unroll
    for (int c = 0; c < V / 4; ++c) {
        const float4 t = q[c];
        x[4 * c + 0] = t.x;
        x[4 * c + 1] = t.y;
        x[4 * c + 2] = t.z;
        x[4 * c + 3] = t.w;
    }
}

template <int V>
__device__ __forceinline__ void store_f32(float *p, const float (&x)[V]) {
    float4 *q = reinterpret_cast<float4 *>(p);
#pragma unroll
    for (int c = 0; c < V / 4; ++c) q[c] = make_float4(x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]);
}

// This lane's coordinates of an fp32 row (row points at coordinate 0).
template <int G, int V, bool BF16>
__device__ __forceinline__ void load_coords(const float *row, int lg, float (&x)[V]) {
    using L = Lanes<G, V, BF16>;
#pragma unroll
    for (int n = 0; n < L::N; ++n) {
#pragma unroll
        for (int w = 0; w < L::Q / 4; ++w) {
            const float4 t = *reinterpret_cast<const float4 *>(row + L::coord(lg, n) + 4 * w);
            x[n * L::Q + 4 * w + 0] = t.x;
            x[n * L::Q + 4 * w + 1] = t.y;
            x[n * L::Q + 4 * w + 2] = t.z;
            x[n * L::Q + 4 * w + 3] = t.w;
        }
    }
}

template <int G, int V, bool BF16>
__device__ __forceinline__ void store_coords(float *row, int lg, const float (&x)[V]) {
    using L = Lanes<G, V, BF16>;
#pragma unroll
    for (int n = 0; n < L::N; ++n) {
#pragma unroll
        for (int w = 0; w < L::Q / 4; ++w) {
            const int e = n * L::Q + 4 * w;
            *reinterpret_cast<float4 *>(row + L::coord(lg, n) + 4 * w) = make_float4(x[e], x[e + 1], x[e + 2], x[e + 3]);
        }
    }
}

// Cells a lane group takes per chunk (rounded to a multiple of the group).
#ifndef TSID_CELLS_PER_GROUP
#define TSID_CELLS_PER_GROUP 8
#endif
// 1: stream loads carry the non-temporal hint.
#ifndef TSID_STREAM_NT
#define TSID_STREAM_NT 0
#endif

__device__ __forceinline__ int2 load_cell(const int2 *p) {
#if TSID_STREAM_NT
    const long long v = __builtin_nontemporal_load(reinterpret_cast<const long long *>(p));
#else
    const long long v = *reinterpret_cast<const long long *>(p);
#endif
    return make_int2((int)(uint32_t)(unsigned long long)v, (int)(uint32_t)((unsigned long long)v >> 32));
}

__device__ __forceinline__ bool skip_epoch(const PassArgs &A) {
    if (!A.skip_after_nonfinite) return false;
    const int32_t f = A.err[ERR_NONFINITE];
    return f != 0 && f - 1 < A.epoch;
}

// Row update of Eq. 5 (descent on Eqs. 3-4 summed), optional 1/max(1, deg)
// normalisation and the Section 5.3 clip, for this lane's V coordinates.
template <int G, int V, bool BF16>
__device__ __forceinline__ void finalize_row(const PassArgs &A, int row, int lg, const float (&x)[V],
                                             const float (&acc_in)[V], int64_t deg) {
    if (A.partial_out) {  // a row block's pass: the sum only, the update comes later
        store_coords<G, V, BF16>(A.partial_out + (int64_t)row * (G * V), lg, acc_in);
        return;
    }
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = acc_in[v];
    if (A.dptr) {
        // dense head tiles: the stream holds the other cells only; the degree
        // counts every cell and the tiles' gradient sums are added here
        deg = A.dptr[row + 1] - A.dptr[row];
        if (A.gd_tile_ptr[(row >> 4) + 1] > A.gd_tile_ptr[row >> 4]) {
            float g[V];
            load_coords<G, V, BF16>(A.gd + (int64_t)row * (G * V), lg, g);
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] += g[v];
        }
    }
    const float s = A.degree ? 1.0f / (float)(deg > 1 ? deg : 1) : 1.0f;
    const bool keep = A.keep_empty && deg == 0;
    float gxv[V];
#pragma unroll
    for (int v = 0; v < V; ++v) gxv[v] = 0.f;
    if (A.gx) load_coords<G, V, BF16>(A.gx + (int64_t)row * (G * V), lg, gxv);
    float xn[V];
    bool bad = false;
    float nrm = 0.f;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        float d;
        if (A.clip == 2) {
            d = s * acc[v];  // the cells' clipped directions (per-entry order)
        } else {
            float g = 2.0f * A.lam * x[v] - 2.0f * acc[v];
            if (A.gx) g += A.gx_scale * gxv[v];
            d = clipped_step(g, s, A.clip, A.xi);
        }
        xn[v] = keep ? x[v] : x[v] + A.lr * d;
        bad |= !__builtin_isfinite(xn[v]);
        nrm += x[v] * x[v];
    }
    const int64_t off = (int64_t)row * (G * V);
    store_coords<G, V, BF16>(A.Xn + off, lg, xn);
    if constexpr (BF16) {
        static_assert(V % 8 == 0, "bf16 rows hold a multiple of 8 coordinates per lane");
        if (A.Xn_b) {
#pragma unroll
            for (int c = 0; c < V / 8; ++c) {
                uint32_t w[4];
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    w[p] = bf16_bits(xn[8 * c + 2 * p]) | (bf16_bits(xn[8 * c + 2 * p + 1]) << 16);
                *reinterpret_cast<uint4 *>(A.Xn_b + off + Lanes<G, V, true>::coord(lg, c)) =
                    make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
    nrm = group_sum<G>(nrm);
    if (lg == 0 && A.norm) A.norm[row] = nrm;
    if (bad) A.err[ERR_NONFINITE] = A.epoch + 1;
}

// Gathers of the other factor.  Within the template (tables below 4 GiB) they
// are raw buffer loads: one 32-bit offset register per gather instead of a
// 64-bit address, and the hardware clamps any offset past the table to zero.
// The extension's fixed table may exceed 4 GiB and uses 64-bit global loads.
struct YTable {
    __amdgpu_buffer_rsrc_t rsrc;
    const char *base;
};

template <bool BUF>
__device__ __forceinline__ YTable make_ytable(const PassArgs &A, int row_bytes) {
    YTable t;
    t.base = static_cast<const char *>(A.Y);
    if constexpr (BUF) {
        // raw buffer, 32-bit data format (descriptor word 3 of the gfx9 family)
        t.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(A.Y), (short)0,
                                                   (int)(A.y_rows * row_bytes), 0x00020000);
    }
    return t;
}

// 16 bytes of row b of the table at byte offset `col_byte` within the row.
template <bool BUF>
__device__ __forceinline__ uint4 ygather16(const YTable &t, int b, int row_bytes, int col_byte) {
    if constexpr (BUF) {
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                             t.rsrc, (unsigned)(b * row_bytes + col_byte), 0, 0));
    } else {
        return *reinterpret_cast<const uint4 *>(t.base + (int64_t)b * row_bytes + col_byte);
    }
}

// Stream layout of a group's walk over its item: cells arrive in blocks of
// SB = G * SPL cells (SPL per lane: lane s holds cells s + c*G, c < SPL),
// and are consumed in chunks of CH cells, CH gathers in flight per lane.
#ifndef TSID_PINGPONG
#define TSID_PINGPONG 0
#endif
#ifndef TSID_CHUNK_BARRIER
#define TSID_CHUNK_BARRIER 0
#endif
#ifndef TSID_STREAM_SPL
#define TSID_STREAM_SPL 16
#endif
template <int G>
constexpr int chunk_cells() {
    return TSID_CELLS_PER_GROUP < G ? G : TSID_CELLS_PER_GROUP;
}
template <int G>
constexpr int block_spl() {  // stream cells per lane per block
    return (G * TSID_STREAM_SPL) < chunk_cells<G>() ? (chunk_cells<G>() / G) : TSID_STREAM_SPL;
}

// One stream block of a work item (SB = G * SPL cells starting at j0).  Per
// chunk of CH cells the group broadcasts each cell's column id and issues
// all CH gathers, then does the arithmetic.  After the gathers of the last
// chunk -- and before its arithmetic -- the group issues the loads of the
// next block's cells into `nxt`: loads retire in issue order, so the slow
// stream loads must come after every gather the arithmetic waits for, and
// issuing them once per block exposes their latency once per SB cells.
// NEXT = false skips those loads (the caller's cells all fit one block).
// PE: the per-entry order of the clipped update -- each cell adds its own
// descent direction 2 e y - 2 lambda x, clipped at xi, instead of e y.
template <int K, int V, bool BF16, bool LOSS_ONLY, bool BUF, bool NEXT = true, int SPL = block_spl<K / V>(),
          bool PE = false>
__device__ __forceinline__ void process_block(const PassArgs &A, const YTable &Yt, int64_t j0,
                                              int64_t end, int64_t last, int lg, const int2 (&cur)[SPL],
                                              int2 (&nxt)[SPL], const float (&x)[V],
                                              const uint32_t (&xp)[V / 2], float (&acc)[V], float &e2) {
    constexpr int G = K / V;
    constexpr int SB = G * SPL;
    constexpr int CH = chunk_cells<G>();
    static_assert(SB % CH == 0, "a stream block holds whole chunks");
    const int64_t left = end - j0;
#pragma unroll
    for (int c0 = 0; c0 < SB; c0 += CH) {
        const bool last_chunk = (c0 + CH == SB);
        if (c0 > 0 && c0 >= left) break;  // the item ends inside this block
#if TSID_CHUNK_BARRIER
        __builtin_amdgcn_sched_barrier(0);  // no hoisting across chunks: fewer live registers
#endif
        if constexpr (BF16) {
            uint32_t yw[CH][V / 2];
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const int b = group_bcast<G>(cur[(c0 + t) / G].x, (c0 + t) % G);
#pragma unroll
                for (int c = 0; c < V / 8; ++c) {
                    const uint4 q = ygather16<BUF>(Yt, b, K * 2, Lanes<G, V, true>::coord(lg, c) * 2);
                    yw[t][4 * c + 0] = q.x;
                    yw[t][4 * c + 1] = q.y;
                    yw[t][4 * c + 2] = q.z;
                    yw[t][4 * c + 3] = q.w;
                }
            }
            if (NEXT && last_chunk) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < SPL; ++c) {
                    const int64_t jn = j0 + SB + c * G + lg;
                    nxt[c] = load_cell(A.stream + (jn < last ? jn : last));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const float r = __int_as_float(group_bcast<G>(cur[(c0 + t) / G].y, (c0 + t) % G));
                float d = 0.f;
#pragma unroll
                for (int p = 0; p < V / 2; ++p)
                    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, xp[p]),
                                                         __builtin_bit_cast(bf16x2, yw[t][p]), d, false);
                d = group_sum<G>(d);
                const bool in = c0 + t < left;
                const float e = in ? r - d : 0.f;
                if constexpr (!LOSS_ONLY && PE) {
#pragma unroll
                    for (int p = 0; p < V / 2; ++p) {
                        float d0 = 2.0f * e * __uint_as_float(yw[t][p] << 16) - 2.0f * A.lam * x[2 * p];
                        float d1 = 2.0f * e * __uint_as_float(yw[t][p] & 0xffff0000u) - 2.0f * A.lam * x[2 * p + 1];
                        if (d0 > A.xi) d0 = A.xi;
                        if (d1 > A.xi) d1 = A.xi;
                        acc[2 * p] += in ? d0 : 0.f;
                        acc[2 * p + 1] += in ? d1 : 0.f;
                    }
                } else if constexpr (!LOSS_ONLY) {
#pragma unroll
                    for (int p = 0; p < V / 2; ++p) {
                        acc[2 * p] += e * __uint_as_float(yw[t][p] << 16);
                        acc[2 * p + 1] += e * __uint_as_float(yw[t][p] & 0xffff0000u);
                    }
                }
                e2 += e * e;
            }
        } else {
            float y[CH][V];
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const int b = group_bcast<G>(cur[(c0 + t) / G].x, (c0 + t) % G);
#pragma unroll
                for (int c = 0; c < V / 4; ++c) {
                    const uint4 q = ygather16<BUF>(Yt, b, K * 4, Lanes<G, V, false>::coord(lg, c) * 4);
                    y[t][4 * c + 0] = __uint_as_float(q.x);
                    y[t][4 * c + 1] = __uint_as_float(q.y);
                    y[t][4 * c + 2] = __uint_as_float(q.z);
                    y[t][4 * c + 3] = __uint_as_float(q.w);
                }
            }
            if (NEXT && last_chunk) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < SPL; ++c) {
                    const int64_t jn = j0 + SB + c * G + lg;
                    nxt[c] = load_cell(A.stream + (jn < last ? jn : last));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const float r = __int_as_float(group_bcast<G>(cur[(c0 + t) / G].y, (c0 + t) % G));
                float d = 0.f;
#pragma unroll
                for (int v = 0; v < V; ++v) d += x[v] * y[t][v];
                d = group_sum<G>(d);
                const bool in = c0 + t < left;
                const float e = in ? r - d : 0.f;
                if constexpr (!LOSS_ONLY && PE) {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        float dv = 2.0f * e * y[t][v] - 2.0f * A.lam * x[v];
                        if (dv > A.xi) dv = A.xi;
                        acc[v] += in ? dv : 0.f;
                    }
                } else if constexpr (!LOSS_ONLY) {
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] += e * y[t][v];
                }
                e2 += e * e;
            }
        }
    }
}

// Waves per SIMD the register allocation must allow (0: compiler's choice).
#ifndef TSID_WAVES_PER_EU
#define TSID_WAVES_PER_EU 0
#endif
#if TSID_WAVES_PER_EU > 0
#define TSID_OCCUPANCY __attribute__((amdgpu_waves_per_eu(TSID_WAVES_PER_EU, TSID_WAVES_PER_EU)))
#else
#define TSID_OCCUPANCY
#endif

// Workgroup `bid` of one side's item pass.  PARTS: the owner rows are sums of
// x_parts parts (see launch_item_pass_parts).
template <int K, int V, bool BF16, bool LOSS_ONLY, bool BUF, bool PE, bool PARTS = false>
__device__ __forceinline__ void item_pass_group(const PassArgs &A, const int64_t bid, const int32_t x_parts = 0) {
    constexpr int G = K / V;
    constexpr int NG = 64 / G;
    static_assert(G >= 1 && G <= 16 && (G & (G - 1)) == 0, "group must fit a DPP row");
    if (skip_epoch(A)) return;
    const int lane = threadIdx.x & 63;
    const int grp = lane / G, lg = lane % G;
    const int64_t item = (bid * kWaves + (threadIdx.x >> 6)) * NG + grp;
    const int64_t n_items = A.n_items_dev ? (int64_t)*A.n_items_dev : (int64_t)A.n_items;
    if (item >= n_items) return;  // whole groups leave together
    const int row = A.items[item];  // -1: a pad item that keeps buckets wave-aligned
    uint32_t i0 = 0, i1 = 0;
    int64_t re = 0, beg = 0, end = 0;
    float x[V];
    if (row >= 0) {
        // the bucket's cells split evenly over its items (at most E each)
        i0 = A.item_off[row];
        i1 = A.item_end[row];
        const int64_t rb = A.ptr[row];
        re = A.ptr_end ? A.ptr_end[row] : A.ptr[row + 1];
        const int64_t deg = re - rb, parts = (int64_t)(i1 - i0), q = item - (int64_t)i0;
        beg = rb + q * deg / parts;
        end = rb + (q + 1) * deg / parts;
        const int64_t orow = A.owner_mod ? row % A.owner_mod : row;
        if constexpr (PARTS) {
#pragma unroll
            for (int v = 0; v < V; ++v) x[v] = 0.f;
#pragma unroll 4
            for (int32_t j = 0; j < x_parts; ++j) {
                float part[V];
                load_coords<G, V, BF16>(A.X + (orow * x_parts + j) * K, lg, part);
#pragma unroll
                for (int v = 0; v < V; ++v) x[v] += part[v];
            }
        } else {
            load_coords<G, V, BF16>(A.X + orow * K, lg, x);
        }
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) x[v] = 0.f;
    }
    uint32_t xp[V / 2] = {};  // bf16 pairs of the owner row (bf16 mode)
    if constexpr (BF16) {
#pragma unroll
        for (int p = 0; p < V / 2; ++p) xp[p] = bf16_bits(x[2 * p]) | (bf16_bits(x[2 * p + 1]) << 16);
    }
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.f;
    float e2 = 0.f;

    // The group walks its cells one stream block at a time (see
    // process_block); two cell buffers alternate so the next block's cells
    // load into the buffer not in use.  Loads past the item's end re-read its
    // last cell (always in bounds and unconditional, so outstanding loads are
    // counted exactly); the slots they fill are masked inside process_block.
    constexpr int SPL = block_spl<G>();
    constexpr int SB = G * SPL;
    const int64_t last = end - 1;
    int2 bufA[SPL], bufB[SPL];
    if (end > beg) {
#pragma unroll
        for (int c = 0; c < SPL; ++c) {
            const int64_t jj = beg + c * G + lg;
            bufA[c] = load_cell(A.stream + (jj < last ? jj : last));
        }
    }
    const YTable Yt = make_ytable<BUF>(A, K * (BF16 ? 2 : 4));
#if TSID_PINGPONG
    for (int64_t j0 = beg; j0 < end; j0 += 2 * SB) {
        process_block<K, V, BF16, LOSS_ONLY, BUF, true, block_spl<K / V>(), PE>(A, Yt, j0, end, last, lg, bufA, bufB, x, xp, acc, e2);
        if (j0 + SB >= end) break;
        process_block<K, V, BF16, LOSS_ONLY, BUF, true, block_spl<K / V>(), PE>(A, Yt, j0 + SB, end, last, lg, bufB, bufA, x, xp, acc,
                                                  e2);
    }
#else
    // One block body per iteration; the block's last stream loads land in
    // bufB and are copied over only after the block's arithmetic, where the
    // next block needs them anyway.
    for (int64_t j0 = beg; j0 < end; j0 += SB) {
        process_block<K, V, BF16, LOSS_ONLY, BUF, true, block_spl<K / V>(), PE>(A, Yt, j0, end, last, lg, bufA, bufB, x, xp, acc, e2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < SPL; ++c) bufA[c] = bufB[c];
    }
#endif

    if (A.e2 && lg == 0) A.e2[item] = e2;
    if constexpr (LOSS_ONLY) {
        if (A.norm && row >= 0 && item == (int64_t)i0) {
            float nrm = 0.f;
#pragma unroll
            for (int v = 0; v < V; ++v) nrm += x[v] * x[v];
            nrm = group_sum<G>(nrm);
            if (lg == 0) A.norm[row] = nrm;
        }
    } else {
        // Groups of this wave that hold consecutive items of the same bucket add
        // their partial sums through LDS, in group order, into the segment's
        // first group.  A bucket whose items all sit in this wave is updated
        // here; otherwise the segment leaves one partial sum, at the index of its
        // first item, for the fixup kernel.
        __shared__ float red[kWaves][NG][K];
        __shared__ int seg_row[kWaves][NG];
        const int wv = threadIdx.x >> 6;
        store_f32<V>(&red[wv][grp][lg * V], acc);
        if (lg == 0) seg_row[wv][grp] = row;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // items are in bucket order (pads hold -1), so the group before this one
        // has published its bucket
        const bool head = row >= 0 && ((grp == 0) || (seg_row[wv][grp - 1] != row));
        if (head) {
            int g_end = grp + 1;
            while (g_end < NG && item + (g_end - grp) < n_items && seg_row[wv][g_end] == row) ++g_end;
            for (int g = grp + 1; g < g_end; ++g) {
                float part[V];
                load_f32<V>(&red[wv][g][lg * V], part);
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] += part[v];
            }
            const int64_t seg_last = item + (g_end - grp) - 1;
            if (item == (int64_t)i0 && seg_last == (int64_t)i1 - 1) {
                finalize_row<G, V, BF16>(A, row, lg, x, acc, re - A.ptr[row]);
            } else {
                store_f32<V>(A.carry + (A.carry_per_wave ? item / NG : item) * K + lg * V, acc);
            }
        }
    }
}

template <int K, int V, bool BF16, bool LOSS_ONLY, bool BUF, bool PE = false>
__global__ __launch_bounds__(kThreads) TSID_OCCUPANCY void k_item_pass(const PassArgs A) {
    item_pass_group<K, V, BF16, LOSS_ONLY, BUF, PE>(A, blockIdx.x);
}

template <int K, int V, bool BUF>
__global__ __launch_bounds__(kThreads) TSID_OCCUPANCY void k_item_pass_parts(const PassArgs A, const int32_t x_parts) {
    item_pass_group<K, V, false, false, BUF, false, true>(A, blockIdx.x, x_parts);
}

// Both passes of a simultaneous step in one launch: the Q pass reads only the
// old factors, so the b0 workgroups of the P pass (A0) and then those of the
// Q pass (A1) share one grid, and the Q pass's workgroups start as the P
// pass's leave the compute units.
template <int K, int V, bool BF16, bool BUF, bool PE>
__global__ __launch_bounds__(kThreads) TSID_OCCUPANCY void k_item_pass_pair(const PassArgs A0, const PassArgs A1,
                                                                           const int32_t b0) {
    const int b = blockIdx.x;
    if (b < b0)
        item_pass_group<K, V, BF16, false, BUF, PE>(A0, b);
    else
        item_pass_group<K, V, BF16, false, BUF, PE>(A1, b - b0);
}

// The item pass over a plan laid out in workgroup-sized chunks, in the order
// the host chose (sched[w]: the chunk of workgroup w, < 0 for none).  The
// row-blocked Q pass uses it to give each XCD its own block of the gathered
// table: the dispatcher hands workgroups to the XCDs in turn, so workgroup w
// runs on XCD w % 8.
template <int K, int V, bool BF16, bool BUF, bool PE>
__global__ __launch_bounds__(kThreads) TSID_OCCUPANCY void k_item_pass_sched(const PassArgs A, const int32_t *sched) {
    const int32_t chunk = sched[blockIdx.x];
    if (chunk < 0) return;
    item_pass_group<K, V, BF16, false, BUF, PE>(A, chunk);
}

// Split buckets: add the item partial sums in item order, then update the row.
template <int K, int V, bool BF16>
__device__ __forceinline__ void fixup_group(const PassArgs &A, const int64_t bid) {
    constexpr int G = K / V;
    constexpr int NG = 64 / G;
    if (skip_epoch(A)) return;
    const int lane = threadIdx.x & 63;
    const int grp = lane / G, lg = lane % G;
    const int64_t row = (bid * kWaves + (threadIdx.x >> 6)) * NG + grp;
    if (row >= A.rows) return;
    const uint32_t i0 = A.item_off[row], i1 = A.item_end[row];
    // the pass already updated buckets whose items all sat in one wave
    if (i1 - i0 <= 1 || i0 / NG == (i1 - 1) / NG) return;
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.f;
    // one partial sum per wave segment, stored at the segment's first item:
    // the bucket's first item and every later item that starts a wave
    for (uint32_t it = i0; it < i1; it = (it / NG + 1) * NG) {
        float part[V];
        load_f32<V>(A.carry + (int64_t)(A.carry_per_wave ? it / NG : it) * K + lg * V, part);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] += part[v];
    }
    float x[V];
    load_coords<G, V, BF16>(A.X + (A.owner_mod ? row % A.owner_mod : row) * K, lg, x);
    finalize_row<G, V, BF16>(A, (int)row, lg, x, acc, A.ptr[row + 1] - A.ptr[row]);
}

template <int K, int V, bool BF16>
__global__ __launch_bounds__(kThreads) void k_fixup(const PassArgs A) {
    fixup_group<K, V, BF16>(A, blockIdx.x);
}

// Both sides' fixups in one launch (the P side's b0 workgroups first): each is
// a launch's latency long, 4.8 us on a 4,096 x 2,048 template of 0.76 M cells
// (k = 32, fp32, 100 epochs: 3,051 -> 2,676 us a fit).
template <int K, int V, bool BF16>
__global__ __launch_bounds__(kThreads) void k_fixup_pair(const PassArgs A0, const PassArgs A1, const int32_t b0) {
    const int b = blockIdx.x;
    if (b < b0)
        fixup_group<K, V, BF16>(A0, b);
    else
        fixup_group<K, V, BF16>(A1, b - b0);
}

// Row-blocked passes.  Bounds of every bucket's runs of other indices per
// block (binary search inside the bucket; one thread per bucket and block).
__global__ void k_block_bounds(const int2 *stream, const int64_t *ptr, int32_t rows, int32_t n_blocks,
                               const int64_t *row_bounds, int64_t *bounds) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)(n_blocks + 1) * rows) return;
    const int64_t j = t / rows, x = t % rows;
    const int64_t target = row_bounds[j];
    int64_t lo = ptr[x], hi = ptr[x + 1];  // first position whose other index >= target
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if ((int64_t)stream[mid].x < target) lo = mid + 1;
        else hi = mid;
    }
    bounds[t] = lo;
}

// The blocks' partial sums of a row added in block order, then its update
// (one lane group per row, as in k_fixup).
template <int K, int V, bool BF16>
__global__ __launch_bounds__(kThreads) void k_block_combine(const PassArgs A, const float *part, int32_t n_blocks) {
    constexpr int G = K / V;
    constexpr int NG = 64 / G;
    if (skip_epoch(A)) return;
    const int lane = threadIdx.x & 63;
    const int grp = lane / G, lg = lane % G;
    const int64_t row = ((int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6)) * NG + grp;
    if (row >= A.rows) return;
    float acc[V];
    load_coords<G, V, BF16>(part + row * K, lg, acc);
    for (int32_t j = 1; j < n_blocks; ++j) {
        float p[V];
        load_coords<G, V, BF16>(part + ((int64_t)j * A.rows + row) * K, lg, p);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] += p[v];
    }
    float x[V];
    load_coords<G, V, BF16>(A.X + row * K, lg, x);
    finalize_row<G, V, BF16>(A, (int)row, lg, x, acc, A.ptr[row + 1] - A.ptr[row]);
}

// One-sided extension steps (Section 5.2, Eq. 6 in factored form), all T of
// them in one launch.  A free row's steps need nothing from other rows, so
// the row stays with one wave, or one workgroup of WAVES waves, for the whole
// run, and its fixed rows are gathered once, into registers, whatever the step
// count: the row's cells are split evenly over the lane groups (G = K / V
// lanes, NG per wave), each group holding up to CH cells.  A step is, per
// cell, the residual (dot product and DPP butterfly) and the gradient sum;
// then the groups' sums are added and the row moves (Eq. 5 with the step
// option and the clip).  The row starts at zero and is stored once.
//
// What bounds it: VALU issue, 2 K multiply-adds and log2 G butterfly adds per
// cell and step; so a group only visits its share of the row's cells (the
// share's ceiling is the same for the whole wave), cells past it are zero rows
// with value zero (they add exactly nothing and need no masks), and the sum
// over the groups is a reduce-scatter (WaveSum) after which each lane updates
// only the coordinates it owns.  Measured (2 million cells, 20 steps, the
// chunk's whole compute, before -> now; before, one wave took every row, added
// its groups' sums through LDS and updated all coordinates in every group, and
// a row of more than 64 cells gathered again every step):
//   k = 128, rows of 24 cells  1,595 -> 714 us   (of 6 cells 5,568 -> 1,424)
//   k = 128, 290 cells, 256 MB table 2,815 -> 757 us  (4 MB table 989 -> 730)
//   k = 64, 96 cells, 2 MB table 612 -> 352 us; 384 cells 566 -> 395 us
// Rows that take the Gram form (launch_extend_gram, fp64) keep it, also where
// this form is now the faster one (k = 64, 96 cells, 128 MB table: 388 us here,
// 738 us there): its sums are in fp64.

// Sums over the 64 / G lane groups of a wave, and back.  sum() leaves N of
// the V coordinates of each lane, summed over the groups, in own: halves of
// the wave, then of each half, exchange half of their values
// (v_permlane32_swap, v_permlane16_swap: after the swap of a and b the lower
// part holds both copies of a and the upper part both of b, so one add sums
// two values); inside a row of 16 lanes the exchange is by DPP, and once a
// single value is left, the rest is an all-reduce by row rotations (each add
// commutes, so all lanes end with the same bits).  spread() is the inverse:
// every lane ends with all V coordinates.
template <int G, int V>
struct WaveSum {
    static constexpr int N32 = V / 2;
    static constexpr int N16 = V / 4;
    static constexpr bool SPLIT8 = G <= 8 && N16 >= 2;
    static constexpr int N = SPLIT8 ? N16 / 2 : N16;
    static_assert(V % 4 == 0 && G <= 16, "four quarters of the wave, groups inside a row");

    static __device__ __forceinline__ void swap32(float &a, float &b) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    }
    static __device__ __forceinline__ void swap16(float &a, float &b) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    }
    static __device__ __forceinline__ void sum(const float (&v)[V], float (&own)[N], bool up8) {
        float h[N32], q[N16];
#pragma unroll
        for (int i = 0; i < N32; ++i) {
            float a = v[i], b = v[i + N32];
            swap32(a, b);
            h[i] = a + b;
        }
#pragma unroll
        for (int i = 0; i < N16; ++i) {
            float a = h[i], b = h[i + N16];
            swap16(a, b);
            q[i] = a + b;
        }
        if constexpr (SPLIT8) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float send = up8 ? q[i] : q[i + N], keep = up8 ? q[i + N] : q[i];
                own[i] = keep + dpp<0x128>(send);  // row_ror:8, lane ^ 8
            }
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                own[i] = q[i];
                if constexpr (G <= 8) own[i] += dpp<0x128>(own[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (G <= 4) own[i] += dpp<0x124>(own[i]);  // row_ror:4
            if constexpr (G <= 2) own[i] += dpp<0x122>(own[i]);  // row_ror:2
        }
    }
    static __device__ __forceinline__ void spread(const float (&own)[N], float (&v)[V], bool up8) {
        float h[N32], q[N16];
        if constexpr (SPLIT8) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float o = dpp<0x128>(own[i]);
                q[i] = up8 ? o : own[i];
                q[i + N] = up8 ? own[i] : o;
            }
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) q[i] = own[i];
        }
#pragma unroll
        for (int i = 0; i < N16; ++i) {
            h[i] = q[i];
            h[i + N16] = q[i];
            swap16(h[i], h[i + N16]);
        }
#pragma unroll
        for (int i = 0; i < N32; ++i) {
            v[i] = h[i];
            v[i + N32] = h[i];
            swap32(v[i], v[i + N32]);
        }
    }
};

// Cells a lane group holds (CH) in the one-wave form and in the workgroup
// forms, and how many cells a form of WAVES waves holds.  At k = 64 and 128 a
// cell takes 8 VGPRs: 16 cells leave three waves per SIMD, 24 leave two (one
// workgroup of 8 waves, or two of 4, per compute unit).
#ifndef TSID_EXT_CELLS
#define TSID_EXT_CELLS 16
#endif
#ifndef TSID_EXT_GROUP_CELLS
#define TSID_EXT_GROUP_CELLS 24
#endif
constexpr int kExtCells = TSID_EXT_CELLS;
constexpr int kExtGroupCells = TSID_EXT_GROUP_CELLS;
// waves of the workgroup forms; the last one holds no cells: it takes rows of
// any length, and the others' rows when there are few steps
constexpr int kExtForms[kExtLists] = {2, 4, 8, 4};
template <int K, int V>
constexpr int64_t ext_capacity(int waves) { return (int64_t)waves * (64 / (K / V)) * (waves > 1 ? kExtGroupCells : kExtCells); }
// Cells visited per branch on a group's share: two keep the dot products of
// two cells in flight and waste at most one cell per group and step.
#ifndef TSID_EXT_UNROLL
#define TSID_EXT_UNROLL 2
#endif

// All steps of one free row by WAVES waves (WAVES = 1: this wave alone).
// red: LDS of 2 x WAVES x 64 x N floats (WAVES > 1).  ALONE (with STREAM): this
// wave takes the shares of all WAVES waves in turn and adds their sums in the
// same order, so the bits are those of the workgroup.
template <int K, int V, bool BUF, int WAVES, bool STREAM, bool ALONE = false>
__device__ __forceinline__ void extend_row(const PassArgs &A, const int64_t row, const int64_t rb, const int64_t deg,
                                           const int32_t steps, float *red) {
    constexpr int G = K / V;
    constexpr int NG = 64 / G;
    constexpr int CH = WAVES > 1 ? kExtGroupCells : kExtCells;
    constexpr int UN = TSID_EXT_UNROLL;
    static_assert(CH % UN == 0, "whole branches");
    constexpr int SPLR = (CH + G - 1) / G;
    using W = WaveSum<G, V>;
    const int lane = threadIdx.x & 63;
    const int wv = WAVES > 1 && !ALONE ? (int)(threadIdx.x >> 6) : 0;
    const int grp = wv * NG + lane / G, lg = lane % G;
    const bool up8 = (lane & 8) != 0;
    constexpr int64_t groups = (int64_t)WAVES * NG;
    const int64_t beg = rb + grp * deg / groups, end = rb + (grp + 1) * deg / groups;
    const int64_t last = end - 1;
    static_assert(STREAM || !ALONE, "a wave alone holds no other wave's cells");
    const float s = A.degree ? 1.0f / (float)(deg > 1 ? deg : 1) : 1.0f;
    const YTable Yt = make_ytable<BUF>(A, K * 4);
    float x[V], xo[W::N];
#pragma unroll
    for (int v = 0; v < V; ++v) x[v] = 0.f;
#pragma unroll
    for (int i = 0; i < W::N; ++i) xo[i] = 0.f;
    // The update of the coordinates this lane owns, and the row back to all lanes.
    auto move = [&](const float (&own)[W::N]) {
#pragma unroll
        for (int i = 0; i < W::N; ++i) {
            const float g = 2.0f * A.lam * xo[i] - 2.0f * own[i];
            xo[i] += A.lr * clipped_step(g, s, A.clip, A.xi);
        }
        W::spread(xo, x, up8);
    };
    // The gradient sum over the groups (and the waves, in wave order), then move.
    auto update = [&](const float (&acc)[V], const int st) {
        float own[W::N];
        W::sum(acc, own, up8);
        if constexpr (WAVES > 1) {
            // one barrier per step: the two halves of red alternate
            float *buf = red + (st & 1) * (WAVES * 64 * W::N);
#pragma unroll
            for (int i = 0; i < W::N; ++i) buf[(wv * W::N + i) * 64 + lane] = own[i];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < W::N; ++i) {
                own[i] = buf[i * 64 + lane];
#pragma unroll
                for (int w = 1; w < WAVES; ++w) own[i] += buf[(w * W::N + i) * 64 + lane];
            }
        }
        move(own);
    };
    if constexpr (!STREAM) {
        // the largest share of a group, the same for every lane
        const int most = __builtin_amdgcn_readfirstlane((int)((deg + groups - 1) / groups));
        const int left = (int)(end - beg);
        int2 rec[SPLR];
#pragma unroll
        for (int c = 0; c < SPLR; ++c) rec[c] = make_int2(0, 0);
        if (left > 0) {
#pragma unroll
            for (int c = 0; c < SPLR; ++c) {
                const int64_t jj = beg + c * G + lg;
                rec[c] = load_cell(A.stream + (jj < last ? jj : last));
            }
        }
        float yc[CH][V], rc[CH];
#pragma unroll
        for (int t0 = 0; t0 < CH; t0 += UN) {
            if (t0 < most) {
#pragma unroll
            for (int t = t0; t < t0 + UN; ++t) {
                const int b = group_bcast<G>(rec[t / G].x, t % G);
                rc[t] = __int_as_float(group_bcast<G>(rec[t / G].y, t % G));
#pragma unroll
                for (int c = 0; c < V / 4; ++c) {
                    uint4 q = make_uint4(0u, 0u, 0u, 0u);
                    if (left > 0) q = ygather16<BUF>(Yt, b, K * 4, Lanes<G, V, false>::coord(lg, c) * 4);
                    yc[t][4 * c + 0] = __uint_as_float(q.x);
                    yc[t][4 * c + 1] = __uint_as_float(q.y);
                    yc[t][4 * c + 2] = __uint_as_float(q.z);
                    yc[t][4 * c + 3] = __uint_as_float(q.w);
                }
            }
            }
        }
#pragma unroll
        for (int t0 = 0; t0 < CH; t0 += UN) {
            if (t0 < most) {
#pragma unroll
            for (int t = t0; t < t0 + UN; ++t) {
                const bool in = t < left;
                if (!in) rc[t] = 0.f;
#pragma unroll
                for (int v = 0; v < V; ++v) yc[t][v] = in ? yc[t][v] : 0.f;
            }
            }
        }
        for (int st = 0; st < steps; ++st) {
            float acc[V];
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = 0.f;
#pragma unroll
            for (int t0 = 0; t0 < CH; t0 += UN) {
                if (t0 < most) {
#pragma unroll
                for (int t = t0; t < t0 + UN; ++t) {
                    float d0 = 0.f, d1 = 0.f;
#pragma unroll
                    for (int v = 0; v < V; v += 2) {
                        d0 += x[v] * yc[t][v];
                        d1 += x[v + 1] * yc[t][v + 1];
                    }
                    const float e = rc[t] - group_sum<G>(d0 + d1);
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] += e * yc[t][v];
                }
                }
            }
            update(acc, st);
        }
    } else {
        // longer than a compute unit's registers hold, or few steps: the groups walk
        // their shares through the item pass's blocks again every step
        constexpr int SPL = 4 * G % chunk_cells<G>() == 0 ? 4 : chunk_cells<G>() / G;
        constexpr int SB = G * SPL;
        const uint32_t xp[V / 2] = {};  // bf16 pairs: unused in fp32
        int2 bufA[SPL], bufB[SPL];
        // Wave w's cells are whole rounds of the wave (a chunk for each of its
        // groups) as far as the row goes, so that only the row's last round is
        // padded; a group's cells are neighbours.
        constexpr int64_t C = chunk_cells<G>(), ROUND = NG * C;
        const int64_t rounds = (deg + ROUND - 1) / ROUND;
        auto walk = [&](const int w, float (&acc)[V]) {
            const int64_t r0 = w * rounds / WAVES, r1 = (w + 1) * rounds / WAVES, per = (r1 - r0) * C;
            const int64_t e = rb + (r1 * ROUND < deg ? r1 * ROUND : deg);
            const int64_t b = rb + r0 * ROUND + lane / G * per;
            const int64_t sb = b < e ? b : e, se = sb + per < e ? sb + per : e, sl = se - 1;
            float e2 = 0.f;
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = 0.f;
            if (se > sb) {
#pragma unroll
                for (int c = 0; c < SPL; ++c) {
                    const int64_t jj = sb + c * G + lg;
                    bufA[c] = load_cell(A.stream + (jj < sl ? jj : sl));
                }
            }
            for (int64_t j0 = sb; j0 < se; j0 += SB) {
                process_block<K, V, false, false, BUF, true, SPL>(A, Yt, j0, se, sl, lg, bufA, bufB, x, xp, acc, e2);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < SPL; ++c) bufA[c] = bufB[c];
            }
        };
        for (int st = 0; st < steps; ++st) {
            float acc[V];
            if constexpr (ALONE) {
                float tot[W::N];
#pragma unroll
                for (int i = 0; i < W::N; ++i) tot[i] = 0.f;
#pragma unroll 1
                for (int w = 0; w < WAVES; ++w) {
                    walk(w, acc);
                    float own[W::N];
                    W::sum(acc, own, up8);
#pragma unroll
                    for (int i = 0; i < W::N; ++i) tot[i] = w == 0 ? own[i] : tot[i] + own[i];
                }
                move(tot);
            } else {
                walk(wv, acc);
                update(acc, st);
            }
        }
    }
    if (grp == 0) store_coords<G, V, false>(A.Xn + row * K, lg, x);
    // a value that left the finite range never comes back (the update adds to
    // it), so the last one tells
    bool bad = false;
#pragma unroll
    for (int i = 0; i < W::N; ++i) bad |= !__builtin_isfinite(xo[i]);
    if (bad) A.err[ERR_NONFINITE] = 1;
}

// The rows longer than one wave's capacity, listed by the workgroup form that
// takes them (the lists' order is of no account: rows are independent).  One
// thread per row and one atomic add per list and workgroup: adds to one
// address from every row's wave took 15 ns each.  stream: the forms (bits) whose
// rows go to the last one.
template <int K, int V>
__global__ __launch_bounds__(kThreads) void k_extend_lists(const PassArgs A, const ExtLists L, const uint32_t stream) {
    __shared__ uint32_t n[kExtLists], base[kExtLists];
    if (threadIdx.x < kExtLists) n[threadIdx.x] = 0;
    __syncthreads();
    const int64_t row = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    int w = -1;
    uint32_t at = 0;
    if (row < A.rows) {
        const int64_t deg = A.ptr[row + 1] - A.ptr[row];
        if (deg > ext_capacity<K, V>(1) && !(A.skip_from > 0 && deg >= A.skip_from)) {
            w = 0;
            while (w < kExtLists - 1 && deg > ext_capacity<K, V>(kExtForms[w])) ++w;
            if (stream >> w & 1) w = kExtLists - 1;
            at = atomicAdd(&n[w], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < kExtLists && n[threadIdx.x]) base[threadIdx.x] = atomicAdd(L.count + threadIdx.x, n[threadIdx.x]);
    __syncthreads();
    if (w >= 0) L.rows[w][base[w] + at] = (int32_t)row;
}

// One wave per free row of at most one wave's capacity; longer ones are the
// workgroup forms'.
template <int K, int V, bool BUF>
__global__ __launch_bounds__(kThreads, K >= 64 ? 3 : 4) void k_extend_steps(const PassArgs A, int32_t steps) {
    const int64_t row =
        (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (row >= A.rows) return;  // whole waves leave together
    const int64_t rb = A.ptr[row], deg = A.ptr[row + 1] - rb;
    if (deg > ext_capacity<K, V>(1)) return;
    if (A.skip_from > 0 && deg >= A.skip_from) return;  // the Gram-form kernel's row
    extend_row<K, V, BUF, 1, false>(A, row, rb, deg, steps, nullptr);
}

// The listed rows, one workgroup of WAVES waves each, dealt in turn (the lists
// come in about row order, so neighbours in length); the next row's place is
// read while this one's steps run.  STREAM, with at least `alone` rows listed:
// those of at most alone_cells cells go to one wave each, after the longer ones.
template <int K, int V, bool BUF, int WAVES, bool STREAM>
__global__ __launch_bounds__(64 * WAVES) void k_extend_group(const PassArgs A, int32_t steps, const int32_t *list,
                                                             const uint32_t *count, uint32_t alone,
                                                             int64_t alone_cells) {
    __shared__ float red[2 * WAVES * 64 * WaveSum<K / V, V>::N];
    const uint32_t n = *count;
    const int64_t by_wave = STREAM && n >= alone ? alone_cells : -1;
    uint32_t q = blockIdx.x;
    if (q < n) {
        int64_t row = list[q], rb = A.ptr[row], re = A.ptr[row + 1];
        for (;;) {  // the same turns for the whole workgroup
            q += gridDim.x;
            const int64_t nrow = q < n ? list[q] : row;
            const int64_t nrb = A.ptr[nrow], nre = A.ptr[nrow + 1];
            if (!STREAM || re - rb > by_wave) {
                __syncthreads();  // the previous row's last reads of red are done
                extend_row<K, V, BUF, WAVES, STREAM>(A, row, rb, re - rb, steps, red);
            }
            if (q >= n) break;
            row = nrow;
            rb = nrb;
            re = nre;
        }
    }
    if constexpr (STREAM) {
        if (by_wave < 0) return;
        const uint32_t wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        for (uint32_t p = blockIdx.x * WAVES + wv; p < n; p += gridDim.x * WAVES) {
            const int64_t row = list[p], rb = A.ptr[row], deg = A.ptr[row + 1] - rb;
            if (deg <= by_wave) extend_row<K, V, BUF, WAVES, true, true>(A, row, rb, deg, steps, nullptr);
        }
    }
}

// Lane group sums in fp64 (as group_sum).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)dpp_i<CTRL>((int)(uint32_t)u), hi = (uint32_t)dpp_i<CTRL>((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int G>
__device__ __forceinline__ double group_sum_f64(double x) {
    if constexpr (G >= 2) x += dpp_f64<0xB1>(x);
    if constexpr (G >= 4) x += dpp_f64<0x4E>(x);
    if constexpr (G >= 8) x += dpp_f64<0x141>(x);
    if constexpr (G >= 16) x += dpp_f64<0x140>(x);
    return x;
}

// A whole fp32 fit in one launch, for templates that fit one compute unit's LDS
// (factors twice, both streams, the bucket pointers): one workgroup runs every
// epoch, a lane group of K / V lanes per owner row, with one barrier per epoch
// where separate launches would be.  Such a fit is bound by launches otherwise:
// 200 x 160 rows, 1,440 cells, k = 8, 50 epochs: 405 us a call with two launches
// an epoch and the history's reductions, 210 us in one launch, which writes
// the history straight to pinned host memory.  An epoch is bound by the latency
// of its longest bucket's walk through LDS, so the sums are fp64 at little cost:
// epochs of the plain step amplify a rounding up to a few tens of times, and
// sums in fp32 in this order left the history of a case 1.2e-6 off where the two
// launches leave it 1.7e-7 off.  With fp64 sums the mean error over 36 templates
// and 50 epochs against 64 bits is 1.9e-7 (factors) and 7.3e-8 (history), the
// launches' 1.9e-7 and 8.4e-8.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
template <int K, int V>
__global__ __launch_bounds__(kSmallThreads) void k_fit_small(const SmallFitArgs A) {
    constexpr int G = K / V;
    constexpr int NGRP = kSmallThreads / G;
    extern __shared__ float4 lds4[];
    const int m = A.m, owners = A.m + A.n;
    float *const buf = reinterpret_cast<float *>(lds4);          // 2 x owners x K: rows of P, then of Q
    int2 *const rec = reinterpret_cast<int2 *>(buf + 2 * owners * K);  // 2 x nnz: {place of the other row, value}
    int32_t *const ptr = reinterpret_cast<int32_t *>(rec + 2 * A.nnz);  // owners + 1
    __shared__ double part[2][kSmallWaves];
    __shared__ int stop[2];  // by epoch parity: one epoch reads its flag while the next may set its own
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int grp = t / G, lg = t % G;
    if (t < 2) stop[t] = 0;
    for (int j = t; j < m * K; j += kSmallThreads) buf[j] = A.P[j];
    for (int j = t; j < A.n * K; j += kSmallThreads) buf[m * K + j] = A.Q[j];
    for (int j = t; j <= m; j += kSmallThreads) ptr[j] = (int32_t)A.row_ptr[j];
    for (int j = t; j < A.n; j += kSmallThreads) ptr[m + 1 + j] = A.nnz + (int32_t)A.col_ptr[j + 1];
    for (int j = t; j < A.nnz; j += kSmallThreads) {
        const int2 r = A.stream_r[j], c = A.stream_c[j];
        rec[j] = make_int2((m + r.x) * K, r.y);
        rec[A.nnz + j] = make_int2(c.x * K, c.y);
    }
    __syncthreads();
    int ep = 0;
    for (;; ++ep) {
        const bool last = ep == A.epochs;  // the loss of the last iterate only
        if (last && !A.loss) break;
        const float *cur = buf + (ep & 1) * owners * K;
        float *nxt = buf + ((ep & 1) ^ 1) * owners * K;
        double sum = 0.0;
        for (int o = grp; o < owners; o += NGRP) {
            float x[V];
            load_coords<G, V, false>(cur + o * K, lg, x);
            double acc[V], e2 = 0.0, nrm = 0.0;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                acc[v] = 0.0;
                nrm = fma((double)x[v], (double)x[v], nrm);
            }
            const int b0 = ptr[o], b1 = ptr[o + 1];
            if (!last || o < m) {
                // four cells' records, then their rows, in flight
                for (int j = b0; j < b1; j += 4) {
                    int2 r[4];
                    float y[4][V];
#pragma unroll
                    for (int i = 0; i < 4; ++i) r[i] = rec[j + i < b1 ? j + i : b1 - 1];
#pragma unroll
                    for (int i = 0; i < 4; ++i) load_coords<G, V, false>(cur + r[i].x, lg, y[i]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        double d = 0.0;
#pragma unroll
                        for (int v = 0; v < V; ++v) d = fma((double)x[v], (double)y[i][v], d);
                        const double e =
                            j + i < b1 ? (double)__int_as_float(r[i].y) - group_sum_f64<G>(d) : 0.0;
#pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] = fma(e, (double)y[i][v], acc[v]);
                        e2 = fma(e, e, e2);
                    }
                }
            }
            nrm = group_sum_f64<G>(nrm);
            if (lg == 0) sum += (o < m ? e2 : 0.0) + (double)A.lam * nrm;
            if (!last) {
                const bool scaled = o < m ? A.degree_r : A.degree_c;
                const double s = scaled ? 1.0 / (double)(b1 - b0 > 1 ? b1 - b0 : 1) : 1.0;
                bool bad = false;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    // clipped_step in fp64
                    const double down = 2.0 * acc[v] - 2.0 * (double)A.lam * (double)x[v];
                    double d = A.clip == 3 ? down : s * down;
                    if (A.clip && d > (double)A.xi) d = (double)A.xi;
                    if (A.clip == 3) d *= s;
                    x[v] = (float)fma((double)A.lr, d, (double)x[v]);
                    bad |= !__builtin_isfinite(x[v]);
                }
                store_coords<G, V, false>(nxt + o * K, lg, x);
                if (bad) stop[ep & 1] = 1;
            }
        }
        if (A.loss) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
            if (lane == 0) part[ep & 1][wv] = sum;
        }
        __syncthreads();
        if (A.loss && t == 0) {
            double l = 0.0;
            for (int w = 0; w < kSmallWaves; ++w) l += part[ep & 1][w];
            A.loss[ep] = l;
        }
        if (last || stop[ep & 1]) break;  // a non-finite update: this epoch's factors stay
    }
    const float *fin = buf + (ep & 1) * owners * K;
    for (int j = t; j < m * K; j += kSmallThreads) A.P[j] = fin[j];
    for (int j = t; j < A.n * K; j += kSmallThreads) A.Q[j] = fin[m * K + j];
    if (t == 0) *A.done = ep;
}

template <int K>
__global__ void k_row_norms(const float *X, int32_t rows, float *norm) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    float x[K];
    load_f32<K>(X + r * K, x);
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < K; ++c) s += x[c] * x[c];
    norm[r] = s;
}

__global__ void k_to_bf16(const float *X, int64_t n, uint16_t *Xb) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x)
        Xb[j] = (uint16_t)bf16_bits(X[j]);
}

constexpr int kRedBlocks = 64;

// Four sums per slot: a (stride sa), b, c and d (strides nb, nc, nd); a null
// array sums to zero.
constexpr int kRedTerms = 4;
__global__ __launch_bounds__(256) void k_reduce_partial(const float *a, int64_t sa, int64_t na,
                                                        const float *b, int64_t nb, const float *c,
                                                        int64_t nc, const float *dd, int64_t nd,
                                                        double *partial) {
    __shared__ double lds[256];
    const int slot = blockIdx.y;
    const int which = blockIdx.x / kRedBlocks, blk = blockIdx.x % kRedBlocks;
    const float *src = which == 0   ? (a ? a + slot * sa : nullptr)
                       : which == 1 ? (b ? b + slot * nb : nullptr)
                       : which == 2 ? (c ? c + slot * nc : nullptr)
                                    : (dd ? dd + slot * nd : nullptr);
    const int64_t n = which == 0 ? na : (which == 1 ? nb : (which == 2 ? nc : nd));
    const int64_t chunk = (n + kRedBlocks - 1) / kRedBlocks;
    const int64_t lo = blk * chunk, hi = lo + chunk < n ? lo + chunk : n;
    double s = 0.0;
    if (src)
        for (int64_t j = lo + threadIdx.x; j < hi; j += 256) s += (double)src[j];
    lds[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) lds[threadIdx.x] += lds[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[(int64_t)slot * kRedTerms * kRedBlocks + blockIdx.x] = lds[0];
}

__global__ void k_reduce_final(const double *partial, int n_slots, double lam, double w4, double *out,
                               const int32_t *err, int32_t epoch0) {
    for (int slot = threadIdx.x; slot < n_slots; slot += blockDim.x) {
        if (err && epoch0 >= 0) {
            const int32_t f = err[ERR_NONFINITE];
            if (f != 0 && f - 1 < epoch0 + slot) continue;
        }
        const double *p = partial + (int64_t)slot * kRedTerms * kRedBlocks;
        double s[kRedTerms] = {0.0, 0.0, 0.0, 0.0};
        const int terms = w4 != 0.0 ? kRedTerms : kRedTerms - 1;  // the fourth only when weighted
        for (int w = 0; w < terms; ++w)
            for (int b = 0; b < kRedBlocks; ++b) s[w] += p[w * kRedBlocks + b];
        out[slot] = s[0] + lam * (s[1] + s[2]);
        if (w4 != 0.0) out[slot] += w4 * s[3];
    }
}

template <int K, int V, bool BF16>
void item_pass_kv(bool loss_only, const PassArgs &a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int NG = 64 / (K / V);
    const int grid = ceil_div(a.n_items, (int64_t)kWaves * NG);
    if (grid <= 0) return;
    // buffer-resource gathers need the table (and every offset) below 2^31 bytes
    const bool buf = a.y_rows * (int64_t)K * (BF16 ? 2 : 4) < (int64_t(1) << 31);
    auto go = [&](auto kernel) {
        hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), 0, s, ev0, ev1, 0, a);
    };
    if (loss_only) {
        if (buf) go(k_item_pass<K, V, BF16, true, true>);
        else go(k_item_pass<K, V, BF16, true, false>);
    } else if (a.clip == 2) {
        if (buf) go(k_item_pass<K, V, BF16, false, true, true>);
        else go(k_item_pass<K, V, BF16, false, false, true>);
    } else {
        if (buf) go(k_item_pass<K, V, BF16, false, true>);
        else go(k_item_pass<K, V, BF16, false, false>);
    }
    TSID_HIP(hipGetLastError());
}

template <int K, int V, bool BF16>
void item_pass_parts_kv(const PassArgs &a, int32_t x_parts, hipStream_t s) {
    if constexpr (BF16) {
        fail(TSID_E_INVAL, "rows in parts are fp32");
    } else {
        constexpr int NG = 64 / (K / V);
        const int grid = ceil_div(a.n_items, (int64_t)kWaves * NG);
        if (grid <= 0) return;
        if (a.y_rows * (int64_t)K * 4 < (int64_t(1) << 31))
            hipLaunchKernelGGL((k_item_pass_parts<K, V, true>), dim3(grid), dim3(kThreads), 0, s, a, x_parts);
        else
            hipLaunchKernelGGL((k_item_pass_parts<K, V, false>), dim3(grid), dim3(kThreads), 0, s, a, x_parts);
        TSID_HIP(hipGetLastError());
    }
}

template <int K, int V, bool BF16>
void item_pass_sched_kv(const PassArgs &a, const int32_t *sched, int64_t n_wg, hipStream_t s, hipEvent_t ev0,
                        hipEvent_t ev1) {
    if (n_wg <= 0) return;
    if (n_wg > INT32_MAX) fail(TSID_E_INVAL, "too many workgroups");
    const bool buf = a.y_rows * (int64_t)K * (BF16 ? 2 : 4) < (int64_t(1) << 31);
    auto go = [&](auto kernel) {
        hipExtLaunchKernelGGL(kernel, dim3((unsigned)n_wg), dim3(kThreads), 0, s, ev0, ev1, 0, a, sched);
    };
    if (a.clip == 2) {
        if (buf) go(k_item_pass_sched<K, V, BF16, true, true>);
        else go(k_item_pass_sched<K, V, BF16, false, true>);
    } else {
        if (buf) go(k_item_pass_sched<K, V, BF16, true, false>);
        else go(k_item_pass_sched<K, V, BF16, false, false>);
    }
    TSID_HIP(hipGetLastError());
}

// Both sides' passes in one launch when their gathers use the same addressing;
// else two launches (ev0 on the first, ev1 on the second).
template <int K, int V, bool BF16>
void item_pass_pair_kv(const PassArgs &a0, const PassArgs &a1, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int NG = 64 / (K / V);
    const int64_t g0 = ceil_div(a0.n_items, (int64_t)kWaves * NG), g1 = ceil_div(a1.n_items, (int64_t)kWaves * NG);
    const int64_t elt = BF16 ? 2 : 4;
    const bool buf0 = a0.y_rows * (int64_t)K * elt < (int64_t(1) << 31);
    const bool buf1 = a1.y_rows * (int64_t)K * elt < (int64_t(1) << 31);
    if (g0 <= 0 || g1 <= 0 || buf0 != buf1 || a0.clip != a1.clip || g0 + g1 > INT32_MAX) {
        item_pass_kv<K, V, BF16>(false, a0, s, ev0, nullptr);
        item_pass_kv<K, V, BF16>(false, a1, s, nullptr, ev1);
        return;
    }
    auto go = [&](auto kernel) {
        hipExtLaunchKernelGGL(kernel, dim3((unsigned)(g0 + g1)), dim3(kThreads), 0, s, ev0, ev1, 0, a0, a1,
                              (int32_t)g0);
    };
    if (a0.clip == 2) {
        if (buf0) go(k_item_pass_pair<K, V, BF16, true, true>);
        else go(k_item_pass_pair<K, V, BF16, false, true>);
    } else {
        if (buf0) go(k_item_pass_pair<K, V, BF16, true, false>);
        else go(k_item_pass_pair<K, V, BF16, false, false>);
    }
    TSID_HIP(hipGetLastError());
}

template <int K, int V, bool BUF>
void extend_steps_buf(const PassArgs &a, int32_t steps, int64_t nnz, const ExtLists &l, hipStream_t s) {
    hipLaunchKernelGGL((k_extend_steps<K, V, BUF>), dim3(ceil_div(a.rows, (int64_t)kWaves)), dim3(kThreads), 0, s, a,
                       steps);
    TSID_HIP(hipGetLastError());
    // the longest row that can be listed: the whole chunk, or one cell below the
    // Gram form's threshold.  Forms it does not reach have no row: empty launches of
    // 2 to 3 us each, five a chunk where that threshold is one wave's capacity or less
    // (k = 32, 20 steps, a table in L2: rows from 40 cells, and one wave holds 128)
    const int64_t longest = a.skip_from > 0 ? std::min(nnz, a.skip_from - 1) : nnz;
    if (longest <= ext_capacity<K, V>(1)) return;
    // With few steps a row's one gather into registers is not spread over enough of
    // them: the forms hold two waves a SIMD, and a form that is half empty (rows just
    // beyond the one before it) fewer cells still, where the streaming form keeps
    // more waves and loads in flight.  From the first step on when the table lies
    // beyond L2 (each further step gathers from there again), for a few steps when it
    // lies in L2.  12 M cells, registers -> streaming, us: k = 128, 100 cells, table in L2,
    // 1 / 2 steps 1,021 -> 602 / 1,185 -> 936, beyond L2 1,414 -> 1,075 / 1,546 ->
    // 1,856; k = 32, 780 cells, in L2, 5 / 10 steps 691 -> 542 / 1,032 -> 895; k = 64,
    // 780 cells, in L2, 3 / 4 steps 731 -> 583 / 819 -> 709.
    const bool in_l2 = a.y_rows * (int64_t)K * 4 <= (int64_t(4) << 20);
    constexpr int32_t kFew[3] = {K == 128 ? 2 : K == 32 ? 3 : 1, K == 128 ? 3 : K == 64 ? 2 : K == 32 ? 5 : 1,
                                 K == 128 ? 7 : K == 64 ? 4 : K == 32 ? 10 : 1};
    uint32_t stream = 0;
    for (int w = 0; w < kExtLists - 1; ++w)
        if (steps <= (in_l2 ? kFew[w] : 1)) stream |= 1u << w;
    hipLaunchKernelGGL((k_extend_lists<K, V>), dim3(ceil_div(a.rows, (int64_t)kThreads)), dim3(kThreads), 0, s, a, l,
                       stream);
    TSID_HIP(hipGetLastError());
    // Streaming rows go to one wave each, with the same bits, where they are many:
    // four waves a row pay a barrier a step and drain four times as often, and are
    // worth it while the chip is not full.  Beyond L2, where a wave mostly waits,
    // that is soon so; in L2 a last wave that is nearly empty costs more until the rows
    // are three times the 2,048 waves that fit at k = 128.  A row of more than a
    // 1,024th of the chunk keeps its workgroup, or it would run on alone.  k = 128, 20
    // steps, four waves -> one: 12,000 rows of 1,000 cells, in L2, 5,243 -> 5,116 us; 2,222
    // of 900, in L2, 910 -> 1,095; beyond L2 1,200 of 10,000, 15,400 -> 9,612, and
    // 1,250 of 1,600, 2,705 -> 2,436.
    const uint32_t alone = in_l2 ? 6144 : 1024;
    // at most nnz / (capacity + 1) rows are longer than a form's capacity
    auto group = [&](auto kernel, int w, int waves) {
        if (stream >> w & 1) return;
        int lowest = w;
        if (w == kExtLists - 1 && stream) lowest = __builtin_ctz(stream);
        const int64_t below = ext_capacity<K, V>(lowest ? kExtForms[lowest - 1] : 1);
        const int64_t most = std::min<int64_t>(a.rows, nnz / (below + 1));
        if (longest <= below || most <= 0) return;
        // twice as many workgroups as fit at two waves per SIMD
        const int64_t grid = std::min<int64_t>(most, 2 * 256 * 8 / waves);
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * waves), 0, s, a, steps, (const int32_t *)l.rows[w],
                           (const uint32_t *)(l.count + w), alone, nnz / 1024);
        TSID_HIP(hipGetLastError());
    };
    group(k_extend_group<K, V, BUF, kExtForms[0], false>, 0, kExtForms[0]);
    group(k_extend_group<K, V, BUF, kExtForms[1], false>, 1, kExtForms[1]);
    group(k_extend_group<K, V, BUF, kExtForms[2], false>, 2, kExtForms[2]);
    // streamed rows of k = 64 from beyond L2: 16 lanes a cell read its whole row with one
    // load (1,200 rows of 10,000 cells, 5 steps 1,810 -> 1,446 us), in L2 8 lanes and fewer
    // instructions are faster (4,000 rows of 2,000 cells, 20 steps 2,040 -> 1,814 us)
    constexpr int SV = K == 64 ? 4 : V;
    if (in_l2) group(k_extend_group<K, V, BUF, kExtForms[3], true>, 3, kExtForms[3]);
    else group(k_extend_group<K, SV, BUF, kExtForms[3], true>, 3, kExtForms[3]);
}

template <int K, int V>
void extend_steps_k(const PassArgs &a, int32_t steps, int64_t nnz, const ExtLists &l, hipStream_t s) {
    if (a.rows <= 0) return;  // steps == 0 still runs: it stores the zero start
    if (a.y_rows * (int64_t)K * 4 < (int64_t(1) << 31)) extend_steps_buf<K, V, true>(a, steps, nnz, l, s);
    else extend_steps_buf<K, V, false>(a, steps, nnz, l, s);
}

template <int K, int V, bool BF16>
void block_combine_kv(const PassArgs &a, const float *part, int32_t n_blocks, hipStream_t s, hipEvent_t ev0,
                      hipEvent_t ev1) {
    constexpr int NG = 64 / (K / V);
    const int grid = ceil_div(a.rows, (int64_t)kWaves * NG);
    if (grid <= 0) return;
    hipExtLaunchKernelGGL(k_block_combine<K, V, BF16>, dim3(grid), dim3(kThreads), 0, s, ev0, ev1, 0, a, part,
                          n_blocks);
    TSID_HIP(hipGetLastError());
}

template <int K, int V, bool BF16>
void fixup_kv(const PassArgs &a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int NG = 64 / (K / V);
    const int grid = ceil_div(a.rows, (int64_t)kWaves * NG);
    if (grid <= 0) return;
    hipExtLaunchKernelGGL(k_fixup<K, V, BF16>, dim3(grid), dim3(kThreads), 0, s, ev0, ev1, 0, a);
    TSID_HIP(hipGetLastError());
}

template <int K, int V, bool BF16>
void fixup_pair_kv(const PassArgs &a0, const PassArgs &a1, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int NG = 64 / (K / V);
    const int64_t g0 = ceil_div(a0.rows, (int64_t)kWaves * NG), g1 = ceil_div(a1.rows, (int64_t)kWaves * NG);
    if (g0 <= 0 || g1 <= 0 || g0 + g1 > INT32_MAX) {
        fixup_kv<K, V, BF16>(a0, s, ev0, nullptr);
        fixup_kv<K, V, BF16>(a1, s, nullptr, ev1);
        return;
    }
    hipExtLaunchKernelGGL((k_fixup_pair<K, V, BF16>), dim3((unsigned)(g0 + g1)), dim3(kThreads), 0, s, ev0, ev1, 0, a0,
                          a1, (int32_t)g0);
    TSID_HIP(hipGetLastError());
}

}  // namespace

#define TSID_DISPATCH_K(K_, FN, ...)                                                              \
    switch (K_) {                                                                                 \
        case 8: prec ? FN<8, 8, true>(__VA_ARGS__) : FN<8, TSID_V_F32_8, false>(__VA_ARGS__); break; \
        case 16: prec ? FN<16, 8, true>(__VA_ARGS__) : FN<16, TSID_V_F32_16, false>(__VA_ARGS__); break; \
        case 32: prec ? FN<32, 8, true>(__VA_ARGS__) : FN<32, TSID_V_F32_32, false>(__VA_ARGS__); break; \
        case 64: prec ? FN<64, TSID_V_BF16_64, true>(__VA_ARGS__)                                   \
                      : FN<64, TSID_V_F32_64, false>(__VA_ARGS__); break;                        \
        case 128: prec ? FN<128, TSID_V_BF16_128, true>(__VA_ARGS__)                                \
                       : FN<128, TSID_V_F32_128, false>(__VA_ARGS__); break;                     \
        default: fail(TSID_E_INVAL, "unsupported rank");                                         \
    }

void launch_item_pass(int K, int prec, bool loss_only, const PassArgs &a, hipStream_t s,
                      hipEvent_t ev0, hipEvent_t ev1) {
    TSID_DISPATCH_K(K, item_pass_kv, loss_only, a, s, ev0, ev1)
}

void launch_item_pass_parts(int K, const PassArgs &a, int32_t x_parts, hipStream_t s) {
    const int prec = TSID_FP32;
    TSID_DISPATCH_K(K, item_pass_parts_kv, a, x_parts, s)
}

void launch_item_pass_pair(int K, int prec, const PassArgs &a0, const PassArgs &a1, hipStream_t s, hipEvent_t ev0,
                           hipEvent_t ev1) {
    TSID_DISPATCH_K(K, item_pass_pair_kv, a0, a1, s, ev0, ev1)
}

void launch_fixup(int K, int prec, const PassArgs &a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    TSID_DISPATCH_K(K, fixup_kv, a, s, ev0, ev1)
}

void launch_fixup_pair(int K, int prec, const PassArgs &a0, const PassArgs &a1, hipStream_t s, hipEvent_t ev0,
                       hipEvent_t ev1) {
    TSID_DISPATCH_K(K, fixup_pair_kv, a0, a1, s, ev0, ev1)
}

void launch_block_combine(int K, int prec, const PassArgs &a, const float *part, int32_t n_blocks, hipStream_t s,
                          hipEvent_t ev0, hipEvent_t ev1) {
    TSID_DISPATCH_K(K, block_combine_kv, a, part, n_blocks, s, ev0, ev1)
}

void launch_block_bounds(const int2 *stream, const int64_t *ptr, int32_t rows, int32_t n_blocks,
                         const int64_t *row_bounds, int64_t *bounds, hipStream_t s) {
    const int64_t n = (int64_t)(n_blocks + 1) * rows;
    if (n <= 0) return;
    k_block_bounds<<<ceil_div(n, 256), 256, 0, s>>>(stream, ptr, rows, n_blocks, row_bounds, bounds);
    TSID_HIP(hipGetLastError());
}

void launch_item_pass_sched(int K, int prec, const PassArgs &a, const int32_t *sched, int64_t n_wg, hipStream_t s,
                            hipEvent_t ev0, hipEvent_t ev1) {
    TSID_DISPATCH_K(K, item_pass_sched_kv, a, sched, n_wg, s, ev0, ev1)
}

// V = 4 and 8 coordinates per lane: at k = 64, groups of 8 lanes add a dot
// product in three butterfly steps for 8 cells at once (16 lanes and 4 steps
// for 4 cells cost a third more instructions per cell).
template <int K>
constexpr int kExtV = K >= 64 ? 8 : 4;
#define TSID_EXT_DISPATCH(K_, FN, ...)                       \
    switch (K_) {                                            \
        case 8: FN<8, kExtV<8>>(__VA_ARGS__); break;         \
        case 16: FN<16, kExtV<16>>(__VA_ARGS__); break;      \
        case 32: FN<32, kExtV<32>>(__VA_ARGS__); break;      \
        case 64: FN<64, kExtV<64>>(__VA_ARGS__); break;      \
        case 128: FN<128, kExtV<128>>(__VA_ARGS__); break;   \
        default: fail(TSID_E_INVAL, "unsupported rank");     \
    }

void launch_extend_steps(int K, const PassArgs &a, int32_t steps, int64_t nnz, const ExtLists &l, hipStream_t s) {
    TSID_EXT_DISPATCH(K, extend_steps_k, a, steps, nnz, l, s)
}

namespace {
template <int K, int V, bool BF16>
void groups_per_wave_kv(int &out) { out = 64 / (K / V); }
}  // namespace

int items_per_wave(int K, int prec) {
    int out = 0;
    TSID_DISPATCH_K(K, groups_per_wave_kv, out)
    return out;
}

int items_per_workgroup(int K, int prec) { return kWaves * items_per_wave(K, prec); }

void launch_row_norms(int K, const float *X, int32_t rows, float *norm, hipStream_t s) {
    if (rows <= 0) return;
    const int grid = ceil_div(rows, 256);
    switch (K) {
        case 8: k_row_norms<8><<<grid, 256, 0, s>>>(X, rows, norm); break;
        case 16: k_row_norms<16><<<grid, 256, 0, s>>>(X, rows, norm); break;
        case 32: k_row_norms<32><<<grid, 256, 0, s>>>(X, rows, norm); break;
        case 64: k_row_norms<64><<<grid, 256, 0, s>>>(X, rows, norm); break;
        case 128: k_row_norms<128><<<grid, 256, 0, s>>>(X, rows, norm); break;
        default: fail(TSID_E_INVAL, "unsupported rank");
    }
    TSID_HIP(hipGetLastError());
}

void launch_to_bf16(const float *X, int64_t n, uint16_t *Xb, hipStream_t s) {
    if (n <= 0) return;
    int64_t g = (n + 255) / 256;
    k_to_bf16<<<(int)(g > 65536 ? 65536 : g), 256, 0, s>>>(X, n, Xb);
    TSID_HIP(hipGetLastError());
}

namespace {
template <int K, int V>
void fit_small_k(const SmallFitArgs &a, size_t lds, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    TSID_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_fit_small<K, V>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmallFitLds));
    hipExtLaunchKernelGGL((k_fit_small<K, V>), dim3(1), dim3(kSmallThreads), lds, s, ev0, ev1, 0, a);
    TSID_HIP(hipGetLastError());
}
}  // namespace

size_t fit_small_lds(int K, int64_t m, int64_t n, int64_t nnz) {
    return (size_t)(2 * (m + n) * K * 4 + 2 * nnz * 8 + (m + n + 1) * 4);
}

int fit_small_groups(int K) { return kSmallThreads / (K / 4); }

void launch_fit_small(int K, const SmallFitArgs &a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const size_t lds = fit_small_lds(K, a.m, a.n, a.nnz);
    if (lds > kSmallFitLds) fail(TSID_E_INVAL, "the template does not fit one workgroup");
    switch (K) {
        case 8: fit_small_k<8, 4>(a, lds, s, ev0, ev1); break;
        case 16: fit_small_k<16, 4>(a, lds, s, ev0, ev1); break;
        case 32: fit_small_k<32, 4>(a, lds, s, ev0, ev1); break;
        case 64: fit_small_k<64, 4>(a, lds, s, ev0, ev1); break;
        default: fail(TSID_E_INVAL, "unsupported rank");
    }
}

size_t reduce_scratch_elems(int n_slots) { return (size_t)kRedTerms * kRedBlocks * (n_slots > 0 ? n_slots : 1); }

void launch_loss_reduce(const float *e2, int64_t e2_stride, int64_t ne, const float *np, int64_t nnp,
                        const float *nq, int64_t nnq, double lam, int n_slots, double *partial,
                        double *out, const int32_t *err, int32_t epoch0, hipStream_t s,
                        hipEvent_t ev0, hipEvent_t ev1, const float *ns, int64_t nns, double w4) {
    if (n_slots <= 0) return;
    if (!ns) w4 = 0.0;
    const int terms = w4 != 0.0 ? kRedTerms : kRedTerms - 1;
    hipExtLaunchKernelGGL(k_reduce_partial, dim3(terms * kRedBlocks, n_slots), dim3(256), 0, s, ev0,
                          nullptr, 0, e2, e2_stride, ne, np, nnp, nq, nnq, ns, nns, partial);
    TSID_HIP(hipGetLastError());
    hipExtLaunchKernelGGL(k_reduce_final, dim3(1), dim3(64), 0, s, nullptr, ev1, 0,
                          (const double *)partial, n_slots, lam, w4, out, err, epoch0);
    TSID_HIP(hipGetLastError());
}

}  // namespace tsid
