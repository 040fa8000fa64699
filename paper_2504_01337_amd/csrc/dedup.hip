// Zero-redundancy dispatch (Sec. 3.4): a token is sent ONCE to every device that hosts at
// least one of its selected experts and replicated there.  On one GPU this builds the
// index of that exchange and runs the two-level combine that goes with it:
//
//   dedup_count_kernel / dedup_rank_kernel : the list of (device, token) copies, ordered by
//       device then token (a stable counting sort of per-token device SETS: a wave ranks
//       its 64 tokens for device g with one ballot of "token has an expert on g"), and for
//       every assignment the row of the copy it uses;
//   combine_partial_kernel : what each expert device returns - one row per copy, the
//       gate-weighted fp32 sum of the outputs of ITS experts for that token, rounded once;
//   combine_copies_kernel  : what the token's home device does - add the partial rows of the
//       token's copies (+ the shared expert) in fp32, round once.
#include "row_sum.h"

namespace c2r {

constexpr int DB_THREADS = 256;
constexpr int DB_SPAN = DB_THREADS * 4;  // tokens per block (with few tokens a quarter or a half of that)
constexpr int DB_FEW_TOKENS = 32768;

__device__ __forceinline__ int device_of(int e, int E, const int32_t *__restrict__ expert_device, int n_dev) {
    if (e < 0 || e >= E) return -1;
    const int g = expert_device[e];
    return (g >= 0 && g < n_dev) ? g : -1;
}

// The expert -> device map of the call, checked once per workgroup into LDS (-1: no device).
__device__ __forceinline__ void load_device_table(int32_t *tab, int E, const int32_t *__restrict__ expert_device,
                                                  int n_dev) {
    if (threadIdx.x < C2R_MAX_E) {
        const int e = threadIdx.x;
        tab[e] = e < E ? device_of(e, E, expert_device, n_dev) : -1;
    }
    __syncthreads();
}

// Devices of a token's K experts.  The K indices are loaded together (independent loads); for
// K <= 8 the devices are also returned packed, one byte per slot (device + 1, 0: none), so that
// the caller need not load the indices again.
__device__ __forceinline__ uint64_t device_set(const int32_t *__restrict__ topk_idx, int64_t t, int64_t T, int K,
                                               int E, const int32_t *tab, uint64_t *packed = nullptr) {
    uint64_t m = 0, pk = 0;
    if (t < T) {
        if (K <= 8) {
            int32_t e[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) e[s] = topk_idx[t * K + (s < K ? s : K - 1)];  // (no load behind a branch)
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int g = (s < K && e[s] >= 0 && e[s] < E) ? tab[e[s]] : -1;
                if (g >= 0) {
                    m |= 1ull << g;
                    pk |= (uint64_t)(g + 1) << (8 * s);
                }
            }
        } else {
            for (int s = 0; s < K; ++s) {
                const int32_t e = topk_idx[t * K + s];
                const int g = (e >= 0 && e < E) ? tab[e] : -1;
                if (g >= 0) m |= 1ull << g;
            }
        }
    }
    if (packed) *packed = pk;
    return m;
}

// DB_ITEMS: tokens per thread.  fill: not null, T * K entries that become -1 (those that the next launch lists copies in are overwritten).
template <int DB_ITEMS>
__global__ __launch_bounds__(DB_THREADS) void dedup_count_kernel(
    const int32_t *__restrict__ topk_idx, int64_t T, int K, int E, const int32_t *__restrict__ expert_device,
    int n_dev, uint16_t *__restrict__ block_counts, int32_t *__restrict__ fill) {
    __shared__ int32_t hist[C2R_MAX_E], dev_tab[C2R_MAX_E];
    if (threadIdx.x < C2R_MAX_E) hist[threadIdx.x] = 0;
    load_device_table(dev_tab, E, expert_device, n_dev);
    const int lane = threadIdx.x & 63;
    const int64_t base = (int64_t)blockIdx.x * (DB_THREADS * DB_ITEMS);
    uint64_t sets[DB_ITEMS];
#pragma unroll
    for (int i = 0; i < DB_ITEMS; ++i)
        sets[i] = device_set(topk_idx, base + i * DB_THREADS + threadIdx.x, T, K, E, dev_tab);
    if (fill) {
        const int64_t end = base + DB_THREADS * DB_ITEMS < T ? (base + DB_THREADS * DB_ITEMS) * K : T * K;
        for (int64_t i = base * K + threadIdx.x; i < end; i += DB_THREADS) fill[i] = -1;
    }
#pragma unroll
    for (int i = 0; i < DB_ITEMS; ++i) {
        const uint64_t m = sets[i];
        for (int g = 0; g < n_dev; ++g) {
            const int c = __popcll(__ballot((m >> g) & 1ull));
            if (lane == 0 && c) atomicAdd(&hist[g], c);
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < n_dev) block_counts[(size_t)blockIdx.x * n_dev + threadIdx.x] = (uint16_t)hist[threadIdx.x];
}

// Every block derives the start of its (block, device) runs itself from the block
// histograms; block 0 also writes the counts and offsets.
template <int DB_ITEMS>
__global__ __launch_bounds__(DB_THREADS) void dedup_rank_kernel(
    const int32_t *__restrict__ topk_idx, int64_t T, int K, int E, const int32_t *__restrict__ expert_device,
    int n_dev, const uint16_t *__restrict__ block_counts, int nblocks, int32_t *__restrict__ send_counts,
    int32_t *__restrict__ send_offsets, int32_t *__restrict__ send_token, int32_t *__restrict__ send_row) {
    constexpr int DB_STEPS = DB_THREADS * DB_ITEMS / C2R_WAVE;  // wave steps per block
    __shared__ int32_t step_cnt[DB_STEPS][C2R_MAX_E];
    __shared__ int32_t part_tot[DB_THREADS / 64][C2R_MAX_E], part_pre[DB_THREADS / 64][C2R_MAX_E];
    __shared__ int32_t run_base[C2R_MAX_E], dev_tab[C2R_MAX_E];
    load_device_table(dev_tab, E, expert_device, n_dev);
    {
        const int g = threadIdx.x & 63, part = threadIdx.x >> 6;
        int32_t tot = 0, pre = 0;
        if (g < n_dev)
#pragma unroll 8
            for (int b = part; b < nblocks; b += DB_THREADS / 64) {
                const int32_t v = block_counts[(size_t)b * n_dev + g];
                tot += v;
                if (b < (int)blockIdx.x) pre += v;
            }
        part_tot[part][g] = tot;
        part_pre[part][g] = pre;
        __syncthreads();
        if (threadIdx.x < 64) {
            int32_t total = 0, before = 0;
#pragma unroll
            for (int q = 0; q < DB_THREADS / 64; ++q) {
                total += part_tot[q][g];
                before += part_pre[q][g];
            }
            int32_t incl = total;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int32_t v = __shfl_up(incl, off);
                if (g >= off) incl += v;
            }
            run_base[g] = incl - total + before;
            if (blockIdx.x == 0 && g < n_dev) {
                send_counts[g] = total;
                send_offsets[g] = incl - total;
                if (g == n_dev - 1) send_offsets[n_dev] = incl;
            }
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * (DB_THREADS * DB_ITEMS);
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint64_t sets[DB_ITEMS], packed[DB_ITEMS];
#pragma unroll
    for (int i = 0; i < DB_ITEMS; ++i)
        sets[i] = device_set(topk_idx, base + i * DB_THREADS + threadIdx.x, T, K, E, dev_tab, &packed[i]);
#pragma unroll
    for (int i = 0; i < DB_ITEMS; ++i) {
        const int q = i * (DB_THREADS / 64) + wave;  // wave step q covers 64 consecutive tokens
        for (int g = 0; g < n_dev; ++g) {
            const int c = __popcll(__ballot((sets[i] >> g) & 1ull));
            if (lane == 0) step_cnt[q][g] = c;
        }
    }
    __syncthreads();
    // exclusive prefix over the block's wave steps, per device, seeded with the block's start
    if ((int)threadIdx.x < n_dev) {
        int32_t run = run_base[threadIdx.x];
#pragma unroll
        for (int q = 0; q < DB_STEPS; ++q) {
            const int32_t c = step_cnt[q][threadIdx.x];
            step_cnt[q][threadIdx.x] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < DB_ITEMS; ++i) {
        const int64_t t = base + i * DB_THREADS + threadIdx.x;
        const int q = i * (DB_THREADS / 64) + wave;
        for (int g = 0; g < n_dev; ++g) {
            const bool mine = (sets[i] >> g) & 1ull;
            const uint64_t bal = __ballot(mine);
            if (mine) {
                const int32_t pos = step_cnt[q][g] + __popcll(bal & lt);
                send_token[pos] = (int32_t)t;
                if (K <= 8) {
#pragma unroll
                    for (int s = 0; s < 8; ++s)
                        if (s < K && (int)((packed[i] >> (8 * s)) & 0xff) == g + 1) send_row[t * K + s] = pos;
                } else {
                    for (int s = 0; s < K; ++s) {
                        const int32_t e = topk_idx[t * K + s];
                        if (e >= 0 && e < E && dev_tab[e] == g) send_row[t * K + s] = pos;
                    }
                }
            }
        }
        if (t < T) {
            if (K <= 8) {
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    if (s < K && ((packed[i] >> (8 * s)) & 0xff) == 0) send_row[t * K + s] = -1;
            } else {
                for (int s = 0; s < K; ++s) {
                    const int32_t e = topk_idx[t * K + s];
                    if (!(e >= 0 && e < E && dev_tab[e] >= 0)) send_row[t * K + s] = -1;
                }
            }
        }
    }
}

// The same index in one launch, for few tokens of up to four slots: one workgroup per device, its 16 waves each with a contiguous
// sixteenth of the tokens in registers.  They count, per wave, the tokens of this device and the copies for all lower ones, then hand
// out the rows in order (see permute_by_slot_kernel).  The device 0 workgroup also marks the slots without a device.  A few hundred tokens
// cost a launch and two trips to memory; beyond, the scattered stores of the rows are what a CU spends its time on, so a device's
// workgroups share them, every `parts`-th 64-token step each (all of them count all tokens).  Microseconds, 60 experts, top-4, random
// routing, two launches / this: 4 devices, 64 tokens 6.5 / 3.4, 1000 tokens 7.4 / 3.7, 3000 tokens 7.9 / 5.5, 4096 tokens 8.0 / 5.8, 8192
// tokens 8.0 / 8.4 (one workgroup per device 10.9); 8 devices, 8192 tokens 15.3 / 8.5, 60 devices 59.6 / 10.6; top-2, 2 devices, 4096
// tokens 6.8 / 6.5, 8192 tokens 6.7 / 9.9.
constexpr int DD_WAVES = 16, DD_PARTS = 8, DD_STEPS = 8;
constexpr int64_t DD_MAX_TOKENS = DD_WAVES * C2R_WAVE * DD_STEPS;
static inline bool dedup_in_one_launch(int64_t T, int K, int n_dev) {
    return T > 0 && K <= 4 && T <= (n_dev > 4 ? DD_MAX_TOKENS : DD_MAX_TOKENS / 2);
}

template <int STEPS>
__global__ __launch_bounds__(DD_WAVES * 64) void dedup_by_device_kernel(
    const int32_t *__restrict__ topk_idx, int T, int K, int E, const int32_t *__restrict__ expert_device, int n_dev,
    int32_t *__restrict__ send_counts, int32_t *__restrict__ send_offsets, int32_t *__restrict__ send_token,
    int32_t *__restrict__ send_row, const bool fill) {
    __shared__ int32_t dev_tab[C2R_MAX_E], w_mine[DD_WAVES], w_less[DD_WAVES];
    const int g = blockIdx.x % n_dev, part = blockIdx.x / n_dev, parts = gridDim.x / n_dev;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int seg = ((T + DD_WAVES - 1) / DD_WAVES + 63) / 64 * 64, t_begin = wave * seg;  // (seg <= 64 * STEPS)
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    i32x4 e[STEPS];
    if (K == 4 && (reinterpret_cast<uintptr_t>(topk_idx) & 15) == 0) {
#pragma unroll
        for (int u = 0; u < STEPS; ++u) e[u] = reinterpret_cast<const i32x4 *>(topk_idx)[min(t_begin + u * 64 + lane, T - 1)];
    } else {
#pragma unroll
        for (int u = 0; u < STEPS; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s) e[u][s] = topk_idx[(size_t)min(t_begin + u * 64 + lane, T - 1) * K + min(s, K - 1)];
    }
    load_device_table(dev_tab, E, expert_device, n_dev);
    const uint64_t below = (1ull << g) - 1ull;
    int slots[STEPS];  // bits 0..3: the token's slots on this device, 4..7: those without a device
    int mine = 0, less = 0;
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        const bool have = u * 64 < seg && t_begin + u * 64 + lane < T;
        uint64_t set = 0;
        slots[u] = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int dev = (uint32_t)e[u][s] < (uint32_t)E ? dev_tab[e[u][s]] : -1;
            if (have && s < K) {
                set |= dev >= 0 ? 1ull << dev : 0ull;
                slots[u] |= dev == g ? 1 << s : dev < 0 ? 16 << s : 0;
            }
        }
        mine += (slots[u] & 15) != 0;
        less += __popcll(set & below);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        mine += __shfl_xor(mine, off);
        less += __shfl_xor(less, off);
    }
    if (lane == 0) {
        w_mine[wave] = mine;
        w_less[wave] = less;
    }
    __syncthreads();
    int start = 0, total = 0, run = 0;  // this device's first row and its rows; those of the waves before this one
#pragma unroll
    for (int w = 0; w < DD_WAVES; ++w) {
        start += w_less[w];
        total += w_mine[w];
        run += w < wave ? w_mine[w] : 0;
    }
    run += start;
    if (threadIdx.x == 0 && part == 0) {
        send_counts[g] = total;
        send_offsets[g] = start;
        if (g == n_dev - 1) send_offsets[n_dev] = start + total;
    }
    if (fill && g == n_dev - 1)  // (no copies past the last device's)
        for (int i = start + total + part * (int)blockDim.x + threadIdx.x; i < T * K; i += parts * (int)blockDim.x) send_token[i] = -1;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        const int t = t_begin + u * 64 + lane;
        const bool on = (slots[u] & 15) != 0;
        const uint64_t m = __ballot(on);
        if (u % parts != part) {
            run += __popcll(m);
            continue;
        }
        const int pos = run + __popcll(m & lt);
        if (on) send_token[pos] = t;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if ((slots[u] >> s) & 1) send_row[(size_t)t * K + s] = pos;
            if (g == 0 && ((slots[u] >> s) & 16)) send_row[(size_t)t * K + s] = -1;
        }
        run += __popcll(m);
    }
}

template <bool BF16>
struct VecAcc {
    static constexpr int N = BF16 ? 8 : 4;
    float acc[N];
    __device__ __forceinline__ VecAcc() {
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j] = 0.0f;
    }
    __device__ __forceinline__ void add(const uint4 q, float g) {
        if constexpr (BF16) {
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[2 * j] = __builtin_fmaf(g, __uint_as_float(w[j] << 16), acc[2 * j]);
                acc[2 * j + 1] = __builtin_fmaf(g, __uint_as_float(w[j] & 0xffff0000u), acc[2 * j + 1]);
            }
        } else {
            acc[0] = __builtin_fmaf(g, __uint_as_float(q.x), acc[0]);
            acc[1] = __builtin_fmaf(g, __uint_as_float(q.y), acc[1]);
            acc[2] = __builtin_fmaf(g, __uint_as_float(q.z), acc[2]);
            acc[3] = __builtin_fmaf(g, __uint_as_float(q.w), acc[3]);
        }
    }
    __device__ __forceinline__ uint4 rounded() const {
        uint4 out;
        if constexpr (BF16) {
            out.x = pack_bf16x2(acc[0], acc[1]);
            out.y = pack_bf16x2(acc[2], acc[3]);
            out.z = pack_bf16x2(acc[4], acc[5]);
            out.w = pack_bf16x2(acc[6], acc[7]);
        } else {
            out.x = __float_as_uint(acc[0]);
            out.y = __float_as_uint(acc[1]);
            out.z = __float_as_uint(acc[2]);
            out.w = __float_as_uint(acc[3]);
        }
        return out;
    }
};

// One thread per 16-byte vector of a copy's partial row.
template <bool BF16>
__global__ __launch_bounds__(256) void combine_partial_kernel(
    const uint4 *__restrict__ y_perm, const float *__restrict__ gates, const int32_t *__restrict__ inv_perm,
    const int32_t *__restrict__ send_token, const int32_t *__restrict__ send_row,
    const int32_t *__restrict__ n_send_ptr, int64_t T, int64_t cap_rows, int row_vecs, int K,
    uint4 *__restrict__ y_part) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int64_t n_send = *n_send_ptr;
    n_send = n_send < 0 ? 0 : (n_send > cap_rows ? cap_rows : n_send);
    if (i >= n_send * row_vecs) return;
    const int64_t r = i / row_vecs;
    const int v = (int)(i - r * row_vecs);
    const int64_t t = send_token[r];
    VecAcc<BF16> a;
    if (t >= 0 && t < T)
        for (int s = 0; s < K; ++s) {
            const int32_t p = inv_perm[t * K + s];
            if (send_row[t * K + s] != (int32_t)r || p < 0) continue;
            a.add(y_perm[(int64_t)p * row_vecs + v], gates[t * K + s]);
        }
    y_part[i] = a.rounded();
}

// The same sums for rows of whole 2 KB pieces (see combine_rows_kernel): a wave owns one piece of one copy, and the token's rows, positions
// and gates come in one load each, a lane per slot.  Bound by memory; microseconds, top-4 of 60, d 2048, per vector / per piece: 8192
// tokens on 4 devices 39.2 / 36.2 (1.2 copies per token), 30 devices (2.1 copies) 59.4 / 42.8, 500 tokens 4.8 / 4.2.  combine_copies_rows_kernel
// below: 28.2 / 20.6, 40.8 / 33.7, 3.7 / 3.0.
template <bool BF16>
__global__ __launch_bounds__(256) void combine_partial_rows_kernel(
    const uint4 *__restrict__ y_perm, const float *__restrict__ gates, const int32_t *__restrict__ inv_perm,
    const int32_t *__restrict__ send_token, const int32_t *__restrict__ send_row,
    const int32_t *__restrict__ n_send_ptr, int64_t T, int64_t cap_rows, int row_vecs, int K,
    uint4 *__restrict__ y_part) {
    const int lane = threadIdx.x & 63, pieces = row_vecs / (64 * ROW_NV);
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = w / pieces, n_send = *n_send_ptr;
    if (r >= n_send || r >= cap_rows) return;
    const int v = (int)(w - r * pieces) * (64 * ROW_NV) + lane;
    const int64_t t = send_token[r];
    RowSum<BF16> sum;
    if (t >= 0 && t < T) {
        const int64_t a = t * K + (lane < K ? lane : 0);
        const int row = send_row[a], pl = inv_perm[a];
        const float gl = gates[a];
        uint64_t have = __ballot(lane < K && row == (int32_t)r && pl >= 0);
        while (have) {
            const int s = __ffsll((unsigned long long)have) - 1;
            have &= have - 1;
            sum.add(y_perm + (int64_t)__builtin_amdgcn_readlane(pl, s) * row_vecs + v,
                    __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gl), s)));
        }
    }
    sum.store(y_part + r * row_vecs + v);
}

// One thread per 16-byte vector of an output row: the token's copies in order of first use.
template <bool BF16>
__global__ __launch_bounds__(256) void combine_copies_kernel(
    const uint4 *__restrict__ y_part, const int32_t *__restrict__ send_row, int64_t T, int64_t cap_rows,
    int row_vecs, int K, const uint4 *__restrict__ y_shared, uint4 *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= T * row_vecs) return;
    const int64_t t = i / row_vecs;
    const int v = (int)(i - t * row_vecs);
    VecAcc<BF16> a;
    for (int s = 0; s < K; ++s) {
        const int32_t r = send_row[t * K + s];
        bool seen = r < 0 || r >= cap_rows;
        for (int b = 0; b < s && !seen; ++b) seen = send_row[t * K + b] == r;
        if (!seen) a.add(y_part[(int64_t)r * row_vecs + v], 1.0f);
    }
    if (y_shared) a.add(y_shared[i], 1.0f);
    y[i] = a.rounded();
}

// The same for rows of whole 2 KB pieces, a wave per piece.
template <bool BF16>
__global__ __launch_bounds__(256) void combine_copies_rows_kernel(
    const uint4 *__restrict__ y_part, const int32_t *__restrict__ send_row, int64_t T, int64_t cap_rows,
    int row_vecs, int K, const uint4 *__restrict__ y_shared, uint4 *__restrict__ y) {
    const int lane = threadIdx.x & 63, pieces = row_vecs / (64 * ROW_NV);
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = w / pieces;
    if (t >= T) return;
    const int v = (int)(w - t * pieces) * (64 * ROW_NV) + lane;
    const int rl = lane < K ? send_row[t * K + lane] : -1;
    RowSum<BF16> sum;
    uint64_t have = __ballot(rl >= 0 && rl < cap_rows);
    while (have) {
        const int r = __builtin_amdgcn_readlane(rl, __ffsll((unsigned long long)have) - 1);
        have &= ~__ballot(rl == r);  // (the first slot that uses the copy stands for all that do)
        sum.add(y_part + (int64_t)r * row_vecs + v, 1.0f);
    }
    if (y_shared) sum.add(y_shared + t * row_vecs + v, 1.0f);
    sum.store(y + t * row_vecs + v);
}

size_t dedup_workspace_bytes(int64_t T, int n_dev) {
    if (T <= 0 || n_dev <= 0) return 0;
    const int64_t nblocks = (T + DB_SPAN - 1) / DB_SPAN;
    return round_up((size_t)nblocks * n_dev * sizeof(int32_t), 256);
}

}  // namespace c2r

using namespace c2r;

// fill: entries of send_token past the copies become -1.  (Dispatch index and two-level combine, a fill launch ahead / so: 8192 tokens of 60
// experts on 4 devices 62.8 / 60.7 us, 2000 tokens 46.3 / 42.6.)
static int dedup_dispatch(const int32_t *topk_idx, int64_t T, int K, int E, const int32_t *expert_device, int n_dev, int32_t *send_counts,
                          int32_t *send_offsets, int32_t *send_token, int32_t *send_row, bool fill, void *ws, size_t ws_bytes, void *stream) {
    drop_stale_error();
    if (T < 0 || K < 1 || E < 1 || n_dev < 1) return C2R_ERR_INVALID_ARG;
    if (E > C2R_MAX_E || n_dev > C2R_MAX_E) return C2R_ERR_UNSUPPORTED;
    if (T * (int64_t)K >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    if (!expert_device || !send_counts || !send_offsets) return C2R_ERR_INVALID_ARG;
    if (T > 0 && (!topk_idx || !send_token || !send_row)) return C2R_ERR_INVALID_ARG;
    const size_t need = dedup_workspace_bytes(T > 0 ? T : 1, n_dev);
    if (!ws || ws_bytes < need || !aligned(ws, 256)) return C2R_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // (every workgroup of the one launch reads all of topk_idx and the device map while others write: send_row may stand in topk_idx's place, say)
    const size_t a4 = (size_t)(T * K) * 4, g4 = (size_t)n_dev * 4;
    if (dedup_in_one_launch(T, K, n_dev) && all_apart({{send_counts, g4}, {send_offsets, g4 + 4}, {send_token, a4}, {send_row, a4}},
                                                      {{topk_idx, a4}, {expert_device, (size_t)E * 4}})) {
        int parts = 1;
        while (parts < DD_PARTS && parts * (DD_MAX_TOKENS / DD_STEPS) < T && 2 * parts * n_dev <= 64) parts *= 2;
        const dim3 g((unsigned)(n_dev * parts)), b(DD_WAVES * 64);
#define C2R_BY_DEVICE(STEPS)                                                                                             \
    dedup_by_device_kernel<STEPS><<<g, b, 0, st>>>(topk_idx, (int)T, K, E, expert_device, n_dev, send_counts, send_offsets, \
                                                   send_token, send_row, fill)
        if (T <= DD_MAX_TOKENS / DD_STEPS)
            C2R_BY_DEVICE(1);
        else if (T <= DD_MAX_TOKENS / 2)
            C2R_BY_DEVICE(4);
        else
            C2R_BY_DEVICE(DD_STEPS);
#undef C2R_BY_DEVICE
        return launch_status();
    }
    // Few tokens: one per thread, or two, so that more than a handful of CUs work (8192 tokens, 4 devices: 7.4 + 11.9 us with
    // four per thread, 3.8 + 5.4 with one).  The block counts are 16 bits wide: those of half-size blocks take what the scratch has
    // always had to hold at least, those of quarter-size blocks go where there is room.
    const int64_t quarter = (T + DB_SPAN / 4 - 1) / (DB_SPAN / 4);
    const int items = T > DB_FEW_TOKENS ? 4 : ((size_t)quarter * n_dev * sizeof(uint16_t) <= ws_bytes ? 1 : 2);
    const int64_t span = DB_THREADS * items, nblocks = T > 0 ? (T + span - 1) / span : 1;
    if (nblocks >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    uint16_t *block_counts = static_cast<uint16_t *>(ws);
    const dim3 grid((unsigned)nblocks), block(DB_THREADS);
#define C2R_DEDUP_LAUNCH(ITEMS)                                                                                      \
    dedup_count_kernel<ITEMS><<<grid, block, 0, st>>>(topk_idx, T, K, E, expert_device, n_dev, block_counts, fill ? send_token : nullptr); \
    dedup_rank_kernel<ITEMS><<<grid, block, 0, st>>>(topk_idx, T, K, E, expert_device, n_dev, block_counts, (int)nblocks, \
                                                     send_counts, send_offsets, send_token, send_row)
    switch (items) {
        case 1: C2R_DEDUP_LAUNCH(1); break;
        case 2: C2R_DEDUP_LAUNCH(2); break;
        default: C2R_DEDUP_LAUNCH(4);
    }
#undef C2R_DEDUP_LAUNCH
    return launch_status();
}

extern "C" int c2r_dedup_dispatch(const int32_t *topk_idx, int64_t T, int K, int E, const int32_t *expert_device,
                                  int n_dev, int32_t *send_counts, int32_t *send_offsets, int32_t *send_token,
                                  int32_t *send_row, void *ws, size_t ws_bytes, void *stream) {
    return dedup_dispatch(topk_idx, T, K, E, expert_device, n_dev, send_counts, send_offsets, send_token, send_row, false, ws, ws_bytes, stream);
}

extern "C" int c2r_dedup_dispatch_filled(const int32_t *topk_idx, int64_t T, int K, int E, const int32_t *expert_device,
                                         int n_dev, int32_t *send_counts, int32_t *send_offsets, int32_t *send_token,
                                         int32_t *send_row, void *ws, size_t ws_bytes, void *stream) {
    return dedup_dispatch(topk_idx, T, K, E, expert_device, n_dev, send_counts, send_offsets, send_token, send_row, true, ws, ws_bytes, stream);
}

extern "C" int c2r_combine_partial(const void *y_perm, c2r_dtype dt, const float *gates, const int32_t *inv_perm,
                                   const int32_t *send_token, const int32_t *send_row, const int32_t *n_send,
                                   int64_t T, int64_t cap_rows, int d, int K, void *y_part, void *stream) {
    drop_stale_error();
    if (T < 0 || cap_rows < 0 || d < 1 || K < 1) return C2R_ERR_INVALID_ARG;
    if (dt != C2R_F32 && dt != C2R_BF16) return C2R_ERR_INVALID_ARG;
    if (T == 0 || cap_rows == 0) return C2R_OK;
    if (!y_perm || !gates || !inv_perm || !send_token || !send_row || !n_send || !y_part) return C2R_ERR_INVALID_ARG;
    if (d % 8 != 0) return C2R_ERR_UNSUPPORTED;
    if (!aligned(y_perm, 16) || !aligned(y_part, 16)) return C2R_ERR_INVALID_ARG;
    const int row_vecs = d * (dt == C2R_BF16 ? 2 : 4) / 16;
    const int64_t nblk = (cap_rows * row_vecs + 255) / 256;
    if (nblk >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (row_pieces(row_vecs, K)) {
        const int64_t waves = cap_rows * (row_vecs / (64 * ROW_NV));
        const dim3 g((unsigned)((waves + 3) / 4)), b(256);
        const uint4 *yp = static_cast<const uint4 *>(y_perm);
        if (dt == C2R_BF16)
            combine_partial_rows_kernel<true><<<g, b, 0, st>>>(yp, gates, inv_perm, send_token, send_row, n_send, T, cap_rows, row_vecs,
                                                               K, static_cast<uint4 *>(y_part));
        else
            combine_partial_rows_kernel<false><<<g, b, 0, st>>>(yp, gates, inv_perm, send_token, send_row, n_send, T, cap_rows, row_vecs,
                                                                K, static_cast<uint4 *>(y_part));
        return launch_status();
    }
    if (dt == C2R_BF16)
        combine_partial_kernel<true><<<dim3((unsigned)nblk), dim3(256), 0, st>>>(
            static_cast<const uint4 *>(y_perm), gates, inv_perm, send_token, send_row, n_send, T, cap_rows, row_vecs, K,
            static_cast<uint4 *>(y_part));
    else
        combine_partial_kernel<false><<<dim3((unsigned)nblk), dim3(256), 0, st>>>(
            static_cast<const uint4 *>(y_perm), gates, inv_perm, send_token, send_row, n_send, T, cap_rows, row_vecs, K,
            static_cast<uint4 *>(y_part));
    return launch_status();
}

extern "C" int c2r_combine_copies(const void *y_part, c2r_dtype dt, const int32_t *send_row, int64_t T,
                                  int64_t cap_rows, int d, int K, const void *y_shared, void *y, void *stream) {
    drop_stale_error();
    if (T < 0 || cap_rows < 0 || d < 1 || K < 1) return C2R_ERR_INVALID_ARG;
    if (dt != C2R_F32 && dt != C2R_BF16) return C2R_ERR_INVALID_ARG;
    if (T == 0) return C2R_OK;
    if (!y_part || !send_row || !y) return C2R_ERR_INVALID_ARG;
    if (d % 8 != 0) return C2R_ERR_UNSUPPORTED;
    if (!aligned(y_part, 16) || !aligned(y, 16) || (y_shared && !aligned(y_shared, 16))) return C2R_ERR_INVALID_ARG;
    const int row_vecs = d * (dt == C2R_BF16 ? 2 : 4) / 16;
    const int64_t nblk = (T * row_vecs + 255) / 256;
    if (nblk >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (row_pieces(row_vecs, K)) {
        const int64_t waves = T * (row_vecs / (64 * ROW_NV));
        const dim3 g((unsigned)((waves + 3) / 4)), b(256);
        const uint4 *yp = static_cast<const uint4 *>(y_part), *ys = static_cast<const uint4 *>(y_shared);
        if (dt == C2R_BF16)
            combine_copies_rows_kernel<true><<<g, b, 0, st>>>(yp, send_row, T, cap_rows, row_vecs, K, ys, static_cast<uint4 *>(y));
        else
            combine_copies_rows_kernel<false><<<g, b, 0, st>>>(yp, send_row, T, cap_rows, row_vecs, K, ys, static_cast<uint4 *>(y));
        return launch_status();
    }
    if (dt == C2R_BF16)
        combine_copies_kernel<true><<<dim3((unsigned)nblk), dim3(256), 0, st>>>(
            static_cast<const uint4 *>(y_part), send_row, T, cap_rows, row_vecs, K, static_cast<const uint4 *>(y_shared),
            static_cast<uint4 *>(y));
    else
        combine_copies_kernel<false><<<dim3((unsigned)nblk), dim3(256), 0, st>>>(
            static_cast<const uint4 *>(y_part), send_row, T, cap_rows, row_vecs, K, static_cast<const uint4 *>(y_shared),
            static_cast<uint4 *>(y));
    return launch_status();
}
