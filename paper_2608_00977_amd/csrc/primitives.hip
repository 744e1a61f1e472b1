// Index-building primitives for the resident template (Section 3.2; Section
// 5.1 "Sampling the TSID Template Submatrix"): exclusive scans, a stable LSD
// radix sort for the row and column buckets, the order-preserving filter of
// Omega to Omega*, bucket pointers and the per-bucket work plan.
//
// Everything here is deterministic: counts may use LDS atomics, but every
// output position comes from prefix sums over a fixed element order, so the
// buckets are bit-identical from run to run.
#include <algorithm>

#include "internal.h"

namespace tsid {

namespace {

constexpr int kThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kThreads * kScanItems;  // 2048
constexpr int kSortItems = 16;
constexpr int kSortTile = kThreads * kSortItems;  // 4096
constexpr int kFiltItems = 16;
constexpr int kFiltTile = kThreads * kFiltItems;  // 4096

// Exclusive scan of one value per thread over the 256-thread block; returns
// the exclusive prefix and sets `total`.  Uses `lds` (256 entries).
__device__ uint32_t block_scan_excl(uint32_t v, uint32_t *lds, uint32_t &total) {
    const int t = threadIdx.x;
    lds[t] = v;
    __syncthreads();
    for (int off = 1; off < kThreads; off <<= 1) {
        uint32_t add = t >= off ? lds[t - off] : 0u;
        __syncthreads();
        lds[t] += add;
        __syncthreads();
    }
    uint32_t incl = lds[t];
    total = lds[kThreads - 1];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(kThreads) void k_scan_reduce(const uint32_t *in, int64_t n,
                                                          uint32_t *sums) {
    __shared__ uint32_t lds[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    for (int it = 0; it < kScanItems; ++it) {
        int64_t j = base + (int64_t)it * kThreads + threadIdx.x;
        if (j < n) s += in[j];
    }
    uint32_t total;
    block_scan_excl(s, lds, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kThreads) void k_scan_apply(const uint32_t *in, uint32_t *out,
                                                         int64_t n, const uint32_t *block_offs,
                                                         uint32_t *total_out) {
    __shared__ uint32_t tile[kScanTile];
    __shared__ uint32_t lds[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    for (int it = 0; it < kScanItems; ++it) {
        int64_t j = base + (int64_t)it * kThreads + threadIdx.x;
        tile[it * kThreads + threadIdx.x] = j < n ? in[j] : 0u;
    }
    __syncthreads();
    uint32_t loc[kScanItems];
    uint32_t s = 0;
    for (int it = 0; it < kScanItems; ++it) {
        loc[it] = s;
        s += tile[threadIdx.x * kScanItems + it];
    }
    uint32_t total;
    uint32_t pre = block_scan_excl(s, lds, total);
    uint32_t off = block_offs ? block_offs[blockIdx.x] : 0u;
    for (int it = 0; it < kScanItems; ++it) tile[threadIdx.x * kScanItems + it] = off + pre + loc[it];
    __syncthreads();
    for (int it = 0; it < kScanItems; ++it) {
        int64_t j = base + (int64_t)it * kThreads + threadIdx.x;
        if (j < n) out[j] = tile[it * kThreads + threadIdx.x];
    }
    if (total_out && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total_out = off + total;
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x)
        p[j] = v;
}

__global__ void k_scatter_map(const int32_t *ids, int32_t count, int32_t *map) {
    int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a < count) map[ids[a]] = (int32_t)a;
}

// ---------------------------------------------------------------- radix sort
//
// Stable LSD sort, 8 bits a pass, one launch for the digit counts of all
// passes and one per pass: a tile's place among the tiles before it comes from
// their published counts (chained scan with look-back), so no pass reads its
// keys twice or waits for separate scan launches, and a sort whose input turns
// out to be in order costs passes + 1 empty launches.  What bounds a pass: 24 B
// of memory traffic per element, and the writes, which go through LDS so that
// a tile's elements of one digit leave together.  Per pass of 7.2 M elements: 65
// us with counts, three scan launches and direct writes, now 41 (a share of
// the counts among them); a chunk in line order pays 27 us of empty launches
// instead of 84.

constexpr uint32_t kMaxPasses = 8;
// words at the start of the scratch: the tile tickets and the digit counts of each pass
constexpr int kSortCtl = kMaxPasses * 257;

// The digit counts of every pass, and zeros in the first pass's tile states.
template <typename State>
__global__ __launch_bounds__(kThreads) void k_radix_hist(const uint64_t *keys, int64_t n, int bit0, int passes,
                                                         uint32_t *ctl, State *state, int64_t state_n,
                                                         SortFlag unsorted) {
    if (unsorted.word && *unsorted.word != unsorted.mark) return;
    __shared__ uint32_t h[kMaxPasses][256];
    const int t = threadIdx.x, lane = t & 63;
    for (int p = 0; p < passes; ++p) h[p][t] = 0;
    const int64_t step = (int64_t)gridDim.x * kThreads;
    const int64_t id = (int64_t)blockIdx.x * kThreads + t;
    for (int64_t j = id; j < state_n; j += step) state[j] = 0;
    __syncthreads();
    // whole waves go round together, so that a digit which the wave shares
    // (the high digits of nearly sorted keys) counts with one add
    for (int64_t j0 = id - lane; j0 < n; j0 += step) {
        const bool in = j0 + lane < n;
        const uint64_t key = (in ? keys[j0 + lane] : keys[n - 1]) >> bit0;
        const uint64_t live = __ballot(in);
        for (int p = 0; p < passes; ++p) {
            const uint32_t d = (uint32_t)(key >> (8 * p)) & 255u;
            const uint32_t d0 = __builtin_amdgcn_readfirstlane((int)d);
            if (__ballot(in && d != d0) == 0) {
                if (lane == 0) atomicAdd(&h[p][d0], (uint32_t)__popcll(live));
            } else if (in) {
                atomicAdd(&h[p][d], 1u);
            }
        }
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p)
        if (h[p][t]) atomicAdd(&ctl[kMaxPasses + p * 256 + t], h[p][t]);
}

// Inclusive sum over the 256 threads of a block (lds: 4 words).
__device__ __forceinline__ uint32_t block_sum_incl(uint32_t v, uint32_t *lds) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(v, off, 64);
        if (lane >= off) v += o;
    }
    if (lane == 63) lds[w] = v;
    __syncthreads();
    for (int x = 0; x < w; ++x) v += lds[x];
    __syncthreads();
    return v;
}

// One pass.  A tile of 4,096 elements, taken in ticket order, so that every
// tile before this one has started: it ranks its elements by digit (wave w
// holds elements w * 1024 .. + 1023 in order; lanes with equal digits rank by
// lane), publishes its count of each digit, then thread d walks back over the
// tiles before it, adding their counts of digit d, until it meets one whose
// total up to there is known, and publishes its own total.  A tile publishes
// its counts before it waits, and waits only for tiles with smaller tickets,
// so every wait ends.  State word: 2 high bits (0 nothing, 1 the tile's count,
// 2 the total of all tiles up to it), the rest the number; words carry flag
// and number together, so no fence is needed.  `next` is the other pass's
// states, zeroed here for it.
// With the flag saying that the input was in order, the pass only copies its
// tile when copy_if_sorted is set (the last of an odd number of passes, whose
// result the caller expects in the other buffer).
template <typename State>
__global__ __launch_bounds__(kThreads) void k_radix_scatter(const uint64_t *kin, const uint32_t *vin, uint64_t *kout,
                                                            uint32_t *vout, int64_t n, int shift, int pass,
                                                            uint32_t *ctl, State *state, State *next,
                                                            SortFlag unsorted, int copy_if_sorted) {
    constexpr int kBits = sizeof(State) * 8;
    constexpr State kNum = (State(1) << (kBits - 2)) - 1, kCount = State(1) << (kBits - 2),
                    kTotal = State(2) << (kBits - 2);
    __shared__ uint64_t s_key[kSortTile];
    __shared__ uint32_t s_val[kSortTile];
    __shared__ uint32_t s_cnt[4][256], s_off[256], s_pos[256], s_sum[4], s_tile;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (unsorted.word && *unsorted.word != unsorted.mark) {
        if (copy_if_sorted) {
            for (int it = 0; it < kSortItems; ++it) {
                const int64_t j = (int64_t)blockIdx.x * kSortTile + (int64_t)it * kThreads + t;
                if (j < n) {
                    kout[j] = kin[j];
                    vout[j] = vin[j];
                }
            }
        }
        return;
    }
    if (t == 0) s_tile = atomicAdd(&ctl[pass], 1u);
#pragma unroll
    for (int x = 0; x < 4; ++x) s_cnt[x][t] = 0;
    __syncthreads();
    const int64_t tile = s_tile, base = tile * kSortTile;
    const int m = (int)(n - base < kSortTile ? n - base : kSortTile);  // elements of the tile
    const uint32_t before_digit = block_sum_incl(ctl[kMaxPasses + pass * 256 + t], s_sum) -
                                  ctl[kMaxPasses + pass * 256 + t];  // elements of smaller digits
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint64_t key[kSortItems];
    uint32_t val[kSortItems], rank[kSortItems];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int e = w * (kSortTile / 4) + i * 64 + lane;
        key[i] = e < m ? kin[base + e] : ~0ull;
        val[i] = e < m ? vin[base + e] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const bool in = w * (kSortTile / 4) + i * 64 + lane < m;
        const uint32_t d = (uint32_t)(key[i] >> shift) & 255u;
        uint64_t peers = __ballot(in);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const uint32_t first = (uint32_t)__popcll(peers & lt);
        const uint32_t had = s_cnt[w][d];
        rank[i] = had + first;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (in && first == 0) s_cnt[w][d] = had + (uint32_t)__popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread t: digit t
    uint32_t total = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const uint32_t c = s_cnt[x][t];
        s_cnt[x][t] = total;
        total += c;
    }
    State *row = state + tile * 256;
    __hip_atomic_store(row + t, (tile == 0 ? kTotal : kCount) | (State)total, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    next[tile * 256 + t] = 0;
    const uint32_t local = block_sum_incl(total, s_sum) - total;
    s_off[t] = local;
    // eight tiles' words in flight: one at a time, the tiles of a first round
    // of workgroups would wait for half as many load latencies as there are tiles
    State excl = 0;
    auto word = [&](int64_t q) {
        return q >= 0 ? __hip_atomic_load(state + q * 256 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kTotal;
    };
    bool found = tile == 0;
    for (int64_t q = tile - 1; !found; q -= 8) {
        State v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = word(q - x);
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            if (found) continue;
            while ((v[x] >> (kBits - 2)) == 0) {
                __builtin_amdgcn_s_sleep(1);
                v[x] = word(q - x);
            }
            excl += v[x] & kNum;
            found = (v[x] >> (kBits - 2)) == 2;
        }
    }
    if (tile > 0)
        __hip_atomic_store(row + t, kTotal | (State)(excl + total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_pos[t] = before_digit + (uint32_t)excl - local;  // where the tile's element at place 0 would go
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        if (w * (kSortTile / 4) + i * 64 + lane < m) {
            const uint32_t d = (uint32_t)(key[i] >> shift) & 255u;
            const uint32_t at = s_off[d] + s_cnt[w][d] + rank[i];
            s_key[at] = key[i];
            s_val[at] = val[i];
        }
    }
    __syncthreads();
    for (int j = t; j < m; j += kThreads) {
        const uint64_t k = s_key[j];
        const uint32_t to = s_pos[(uint32_t)(k >> shift) & 255u] + (uint32_t)j;
        kout[to] = k;
        vout[to] = s_val[j];
    }
}

// ------------------------------------------------------------------ filter

__global__ __launch_bounds__(kThreads) void k_filter_count(const int32_t *u, const int32_t *i,
                                                           const float *r, int64_t S,
                                                           const int32_t *row_map,
                                                           const int32_t *col_map, int64_t m,
                                                           int64_t n, uint32_t *bcnt, int32_t *err) {
    __shared__ uint32_t lds[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kFiltTile;
    uint32_t c = 0;
    for (int it = 0; it < kFiltItems; ++it) {
        const int64_t j = base + (int64_t)it * kThreads + threadIdx.x;
        if (j >= S) break;
        const int32_t uu = u[j], ii = i[j];
        if (uu < 0 || uu >= m || ii < 0 || ii >= n) {
            err[ERR_RANGE] = 1;
            continue;
        }
        if (row_map[uu] >= 0 && col_map[ii] >= 0) {
            ++c;
            if (!__builtin_isfinite(r[j])) err[ERR_INVAL] = 1;
        }
    }
    uint32_t total;
    block_scan_excl(c, lds, total);
    if (threadIdx.x == 0) bcnt[blockIdx.x] = total;
}

__global__ __launch_bounds__(kThreads) void k_filter_write(
    const int32_t *u, const int32_t *i, const float *r, int64_t S, const int32_t *row_map,
    const int32_t *col_map, int64_t m, int64_t n, const uint32_t *boffs, int64_t base_out,
    int bits_b, uint64_t *out_key, uint32_t *out_val) {
    __shared__ uint32_t s_w[4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t base = (int64_t)blockIdx.x * kFiltTile;
    int64_t run = base_out + boffs[blockIdx.x];
    for (int it = 0; it < kFiltItems; ++it) {
        const int64_t j = base + (int64_t)it * kThreads + t;
        int32_t a = -1, b = -1;
        if (j < S) {
            const int32_t uu = u[j], ii = i[j];
            if (uu >= 0 && uu < m && ii >= 0 && ii < n) {
                a = row_map[uu];
                b = col_map[ii];
            }
        }
        const bool keep = a >= 0 && b >= 0;
        const uint64_t bal = __ballot(keep);
        if (lane == 0) s_w[w] = (uint32_t)__popcll(bal);
        __syncthreads();
        if (keep) {
            int64_t pos = run + __popcll(bal & lt);
            for (int ww = 0; ww < w; ++ww) pos += s_w[ww];
            out_key[pos] = ((uint64_t)(uint32_t)a << bits_b) | (uint32_t)b;
            out_val[pos] = __float_as_uint(r[j]);
        }
        run += s_w[0] + s_w[1] + s_w[2] + s_w[3];
        __syncthreads();
    }
}

// ------------------------------------------------------------- bucket views

__global__ void k_keys_to_stream(const uint64_t *keys, const uint32_t *vals, int64_t n, int low_bits,
                                 int2 *stream, int32_t *err) {
    const uint64_t mask = (low_bits >= 64) ? ~0ull : ((1ull << low_bits) - 1ull);
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t k = keys[j];
        stream[j] = make_int2((int)(uint32_t)(k & mask), (int)vals[j]);
        if (j > 0 && keys[j - 1] == k) err[ERR_DUP] = 1;
    }
}

// Global cell keys u * n + i of a piece of Omega, from offset on.
__global__ void k_cell_keys(const int32_t *u, const int32_t *i, int64_t len, int64_t n, uint64_t *keys,
                            uint32_t *vals) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < len;
         j += (int64_t)gridDim.x * blockDim.x) {
        keys[j] = (uint64_t)(uint32_t)u[j] * (uint64_t)n + (uint64_t)(uint32_t)i[j];
        vals[j] = 0u;
    }
}

// Equal neighbours in sorted keys: a repeated cell.
__global__ void k_adjacent_equal(const uint64_t *keys, int64_t n, int32_t *err) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x + 1; j < n;
         j += (int64_t)gridDim.x * blockDim.x)
        if (keys[j - 1] == keys[j]) err[ERR_DUP] = 1;
}

__global__ void k_ptr_from_keys(const uint64_t *keys, int64_t n, int32_t rows, int low_bits,
                                int64_t *ptr) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x > rows) return;
    const uint64_t target = (uint64_t)x << low_bits;
    int64_t lo = 0, hi = n;  // first position with key >= target
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (keys[mid] < target) lo = mid + 1;
        else hi = mid;
    }
    ptr[x] = lo;
}

__global__ void k_swap_key_halves(const uint64_t *keys, int64_t n, int lo_bits, int hi_bits,
                                  uint64_t *out) {
    const uint64_t mask = (1ull << lo_bits) - 1ull;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t k = keys[j];
        out[j] = ((k & mask) << hi_bits) | (k >> lo_bits);
    }
}

// Keys and values of an extension chunk; *unsorted.word = unsorted.mark if some
// key is smaller than the one before it; `zero` (n_zero words) is cleared for
// the kernels that follow.
__global__ void k_chunk_keys(const int32_t *fixed_id, const int32_t *free_id, const float *r, int64_t nnz,
                             int64_t n_fixed, int32_t n_free, int bits_fixed, uint64_t *keys, uint32_t *vals,
                             int32_t *err, SortFlag unsorted, uint32_t *zero, int n_zero) {
    if (blockIdx.x == 0)
        for (int x = threadIdx.x; x < n_zero; x += blockDim.x) zero[x] = 0u;
    bool range = false, order = false;
    auto key_of = [&](int64_t j) {
        const int32_t fx = fixed_id[j], fr = free_id[j];
        const bool ok = fx >= 0 && fx < n_fixed && fr >= 0 && fr < n_free;
        range |= !ok;
        return ok ? ((uint64_t)(uint32_t)fr << bits_fixed) | (uint32_t)fx : 0ull;
    };
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t k = key_of(j);
        keys[j] = k;
        vals[j] = __float_as_uint(r[j]);
        order |= j > 0 && key_of(j - 1) > k;
    }
    if (range) err[ERR_RANGE] = 1;
    if (order) *unsorted.word = unsorted.mark;
}

__global__ void k_plan_count(const int64_t *ptr, int32_t rows, int32_t E, uint32_t *nparts) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= rows) return;
    const int64_t deg = ptr[x + 1] - ptr[x];
    nparts[x] = deg <= E ? 1u : (uint32_t)((deg + E - 1) / E);
}

__global__ void k_plan_fill(const uint32_t *item_off, int32_t rows, int32_t *items) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= rows) return;
    for (uint32_t it = item_off[x]; it < item_off[x + 1]; ++it) items[it] = (int32_t)x;
}

int grid_for(int64_t n, int threads, int cap = 65536) {
    int64_t g = (n + threads - 1) / threads;
    if (g < 1) g = 1;
    return (int)(g > cap ? cap : g);
}

}  // namespace

// --------------------------------------------------------------- host side

size_t scan_scratch_elems(int64_t n) {
    size_t total = 0;
    while (n > kScanTile) {
        const int64_t nb = (n + kScanTile - 1) / kScanTile;
        total += 2 * (size_t)nb;
        n = nb;
    }
    return total + 1;
}

void scan_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total, uint32_t *scratch,
              hipStream_t s) {
    if (n <= 0) {
        if (total) TSID_HIP(hipMemsetAsync(total, 0, sizeof(uint32_t), s));
        return;
    }
    const int nb = ceil_div(n, kScanTile);
    if (nb == 1) {
        k_scan_apply<<<1, kThreads, 0, s>>>(in, out, n, nullptr, total);
        TSID_HIP(hipGetLastError());
        return;
    }
    uint32_t *sums = scratch, *offs = scratch + nb;
    k_scan_reduce<<<nb, kThreads, 0, s>>>(in, n, sums);
    TSID_HIP(hipGetLastError());
    scan_u32(sums, offs, nb, nullptr, scratch + 2 * (size_t)nb, s);
    k_scan_apply<<<nb, kThreads, 0, s>>>(in, out, n, offs, total);
    TSID_HIP(hipGetLastError());
}

// The counts of a tile's state words fit 30 bits below 2^30 elements.
static int state_words(int64_t n) { return n < (int64_t(1) << 30) ? 1 : 2; }

size_t radix_scratch_elems(int64_t n) {
    const int64_t nb = n > 0 ? (n + kSortTile - 1) / kSortTile : 1;
    return (size_t)(kSortCtl + 2 * nb * 256 * state_words(n));
}

int radix_ctl_elems() { return kSortCtl; }

template <typename State>
static bool radix_passes(uint64_t *keys, uint32_t *vals, uint64_t *keys_alt, uint32_t *vals_alt, int64_t n, int bit0,
                         int passes, uint32_t *scratch, hipStream_t s, SortFlag unsorted) {
    const int nb = ceil_div(n, kSortTile);
    const int64_t ns = (int64_t)nb * 256;
    State *state = reinterpret_cast<State *>(scratch + kSortCtl);
    k_radix_hist<State><<<std::min(nb, 512), kThreads, 0, s>>>(keys, n, bit0, passes, scratch, state, ns, unsorted);
    TSID_HIP(hipGetLastError());
    bool alt = false;
    for (int p = 0; p < passes; ++p) {
        const uint64_t *kin = alt ? keys_alt : keys;
        const uint32_t *vin = alt ? vals_alt : vals;
        uint64_t *kout = alt ? keys : keys_alt;
        uint32_t *vout = alt ? vals : vals_alt;
        k_radix_scatter<State><<<nb, kThreads, 0, s>>>(kin, vin, kout, vout, n, bit0 + 8 * p, p, scratch,
                                                       state + (p & 1) * ns, state + ((p + 1) & 1) * ns, unsorted,
                                                       (p == passes - 1) && (passes & 1));
        TSID_HIP(hipGetLastError());
        alt = !alt;
    }
    return alt;
}

bool radix_sort(uint64_t *keys, uint32_t *vals, uint64_t *keys_alt, uint32_t *vals_alt, int64_t n, int bit0,
                int nbits, uint32_t *scratch, hipStream_t s, SortFlag unsorted, bool ctl_zeroed) {
    if (n <= 1) return false;
    if (!ctl_zeroed) fill_u32(scratch, kSortCtl, 0u, s);
    const int passes = (nbits + 7) / 8;
    return state_words(n) == 1
               ? radix_passes<uint32_t>(keys, vals, keys_alt, vals_alt, n, bit0, passes, scratch, s, unsorted)
               : radix_passes<uint64_t>(keys, vals, keys_alt, vals_alt, n, bit0, passes, scratch, s, unsorted);
}

void fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return;
    k_fill_i32<<<grid_for(n, 256), 256, 0, s>>>(p, n, v);
    TSID_HIP(hipGetLastError());
}

void fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s) {
    fill_i32(reinterpret_cast<int32_t *>(p), n, (int32_t)v, s);
}

void fill_f32(float *p, int64_t n, float v, hipStream_t s) {
    fill_i32(reinterpret_cast<int32_t *>(p), n, (int32_t)__builtin_bit_cast(uint32_t, v), s);
}

void scatter_map(const int32_t *ids, int32_t count, int32_t *map, hipStream_t s) {
    if (count <= 0) return;
    k_scatter_map<<<ceil_div(count, 256), 256, 0, s>>>(ids, count, map);
    TSID_HIP(hipGetLastError());
}

int filter_blocks(int64_t S) { return ceil_div(S > 0 ? S : 1, kFiltTile); }

void filter_count(const int32_t *u, const int32_t *i, const float *r, int64_t S,
                  const int32_t *row_map, const int32_t *col_map, int64_t m, int64_t n,
                  uint32_t *bcnt, int32_t *err, hipStream_t s) {
    if (S <= 0) return;
    k_filter_count<<<filter_blocks(S), kThreads, 0, s>>>(u, i, r, S, row_map, col_map, m, n, bcnt,
                                                         err);
    TSID_HIP(hipGetLastError());
}

void filter_write(const int32_t *u, const int32_t *i, const float *r, int64_t S,
                  const int32_t *row_map, const int32_t *col_map, int64_t m, int64_t n,
                  const uint32_t *boffs, int64_t base, int bits_b, uint64_t *out_key,
                  uint32_t *out_val, hipStream_t s) {
    if (S <= 0) return;
    k_filter_write<<<filter_blocks(S), kThreads, 0, s>>>(u, i, r, S, row_map, col_map, m, n, boffs,
                                                         base, bits_b, out_key, out_val);
    TSID_HIP(hipGetLastError());
}

void keys_to_stream(const uint64_t *keys, const uint32_t *vals, int64_t n, int low_bits,
                    int2 *stream, int32_t *err, hipStream_t s) {
    if (n <= 0) return;
    k_keys_to_stream<<<grid_for(n, 256), 256, 0, s>>>(keys, vals, n, low_bits, stream, err);
    TSID_HIP(hipGetLastError());
}

void cell_keys(const int32_t *u, const int32_t *i, int64_t len, int64_t n, uint64_t *keys, uint32_t *vals,
               hipStream_t s) {
    if (len <= 0) return;
    k_cell_keys<<<grid_for(len, 256), 256, 0, s>>>(u, i, len, n, keys, vals);
    TSID_HIP(hipGetLastError());
}

void adjacent_equal(const uint64_t *keys, int64_t n, int32_t *err, hipStream_t s) {
    if (n <= 1) return;
    k_adjacent_equal<<<grid_for(n, 256), 256, 0, s>>>(keys, n, err);
    TSID_HIP(hipGetLastError());
}

void ptr_from_keys(const uint64_t *keys, int64_t n, int32_t rows, int low_bits, int64_t *ptr,
                   hipStream_t s) {
    k_ptr_from_keys<<<ceil_div((int64_t)rows + 1, 256), 256, 0, s>>>(keys, n, rows, low_bits, ptr);
    TSID_HIP(hipGetLastError());
}

void swap_key_halves(const uint64_t *keys, int64_t n, int lo_bits, int hi_bits, uint64_t *out,
                     hipStream_t s) {
    if (n <= 0) return;
    k_swap_key_halves<<<grid_for(n, 256), 256, 0, s>>>(keys, n, lo_bits, hi_bits, out);
    TSID_HIP(hipGetLastError());
}

void chunk_keys(const int32_t *fixed_id, const int32_t *free_id, const float *r, int64_t nnz, int64_t n_fixed,
                int32_t n_free, int bits_fixed, uint64_t *keys, uint32_t *vals, int32_t *err, SortFlag unsorted,
                uint32_t *zero, int n_zero, hipStream_t s) {
    if (nnz <= 0) return;
    k_chunk_keys<<<grid_for(nnz, 256), 256, 0, s>>>(fixed_id, free_id, r, nnz, n_fixed, n_free, bits_fixed, keys,
                                                    vals, err, unsorted, zero, n_zero);
    TSID_HIP(hipGetLastError());
}

void plan_items(const int64_t *ptr, int32_t rows, int32_t E, uint32_t *item_off, int32_t *items,
                uint32_t *nparts_scratch, uint32_t *scan_scratch, hipStream_t s) {
    if (rows <= 0) {
        TSID_HIP(hipMemsetAsync(item_off, 0, sizeof(uint32_t), s));
        return;
    }
    k_plan_count<<<ceil_div(rows, 256), 256, 0, s>>>(ptr, rows, E, nparts_scratch);
    TSID_HIP(hipGetLastError());
    scan_u32(nparts_scratch, item_off, rows, item_off + rows, scan_scratch, s);
    k_plan_fill<<<ceil_div(rows, 256), 256, 0, s>>>(item_off, rows, items);
    TSID_HIP(hipGetLastError());
}

}  // namespace tsid
