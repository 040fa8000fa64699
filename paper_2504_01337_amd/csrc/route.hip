// Router logits (Eq. 1) and collaboration-constrained selection (Sec. 3.3, step 2).
//
// Partial sums, then a selection:
//  route_partial_kernel: an fp32 GEMM over one 256-long k-chunk in which every (token,
//    expert) sum is built with one fused multiply-add per k in ascending k - exactly the
//    ABI's declared order - either by one thread on the vector pipe (up to 8 experts) or by
//    a chain of v_mfma_f32_32x32x2_f32 on the matrix pipe, whose two products per
//    instruction are added in that same order.  Chunk results go to scratch as
//    part[tile][chunk][expert][64] (token fastest, one tile's partials contiguous).
//    Small batches: route_partial_small_kernel, the same sums on 16 x 16 x 4 matrix instructions.
//  route_select_kernel: adds the chunk results left to right (four tokens per lane), adds the
//    bias, then does arg max / masked top-(K-1) in registers with one 64-bit collaborator
//    mask per expert held in LDS: four lanes per token over a quarter of the experts each
//    (chunk partials), or one lane per token over all of them (stored logits).
//    Others for its work: route_select_small_kernel (sixteen lanes per token, up to 8192 tokens), route_finish_small_kernel
//    (up to 64 tokens, with the dispatch index), route_select_keys_kernel (top-K of K <= 4 from one chunk result, more than 8192
//    tokens) and route_select_rows_kernel (stored logits, K <= 4).
#include "route_few.h"
#include "ffn_copy.h"

#include <type_traits>

namespace c2r {

// Wp[k][j] = W_g[k][j] zero-padded to a row length that is a multiple of 4 (only needed when
// E is not one), so that W rows can be fetched with 16-byte loads.
__global__ __launch_bounds__(256) void pack_router_kernel(const float *__restrict__ Wg, int d, int E,
                                                          int ep, float *__restrict__ Wp) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)d * ep) return;
    const int j = (int)(i % ep), k = (int)(i / ep);
    Wp[i] = j < E ? Wg[(int64_t)k * E + j] : 0.0f;
}

// What the selection of a batch needs and writes.
struct SelectArgs {
    const float *bias;
    int E, K;
    const int32_t *collab_idx;
    int Tc;
    int32_t *topk_idx;
    float *gates;
};

// One token's selection by the literal rule, for K <= 4: first one standing unless a later one is strictly larger.  pick(m, e, v) finds
// the expert e of the columns m, and its logit; mask_tab: the collaborators of every expert, or null.
template <typename Pick>
__device__ __forceinline__ void literal_scan(Pick pick, int K, uint64_t all, const uint64_t *mask_tab, int (&es)[4], float (&gs)[4],
                                             float &den) {
    float v0;
    pick(all, es[0], v0);
    uint64_t mm = mask_tab ? mask_tab[es[0]] : all & ~(1ull << es[0]);
    gs[0] = expf(v0 - v0);
    den = gs[0];
#pragma unroll
    for (int s = 1; s < 4; ++s) {
        es[s] = -1;
        gs[s] = 0.0f;
        if (s < K) {
            float v;
            pick(mm, es[s], v);
            if (es[s] >= 0) {
                mm &= ~(1ull << es[s]);
                gs[s] = expf(v - v0);
            }
            den += gs[s];
        }
    }
}

// The same by the whole wave: lane = column, v its logit.  The rule picks the first allowed column if that holds a NaN, else the largest
// number, the lowest column among equals.  Every lane must be active; results in every lane.
__device__ __forceinline__ void literal_scan_by_wave(float v, int K, uint64_t all, const uint64_t *mask_tab, int (&es)[4], float (&gs)[4],
                                                     float &den) {
    const int lane = lane_id(), bits = __float_as_int(v), key = bits ^ ((bits >> 31) & 0x7fffffff);
    auto pick_row = [&](uint64_t mm, int &bi, float &bv) __attribute__((always_inline)) {
        bi = -1;
        bv = 0.0f;
        if (mm == 0) return;
        bi = __ffsll((unsigned long long)mm) - 1;
        bv = __int_as_float(__builtin_amdgcn_readlane(bits, bi));
        if (bv != bv) return;
        const bool in = ((mm >> lane) & 1ull) != 0 && v == v;
        const int best = wave_max(in ? key : (int)0x80000000);
        bi = __ffsll((unsigned long long)__ballot(in && key == best)) - 1;
        bv = __int_as_float(__builtin_amdgcn_readlane(bits, bi));
    };
    literal_scan(pick_row, K, all, mask_tab, es, gs, den);
}

// The keys of the selections below: a logit (-0 made +0) whose low 6 bits are replaced by 63 - column, compared as floats (as
// instructions: the compiler would first quiet what it takes for possible NaNs).
constexpr int KEY_EMPTY = (int)0xff800000;  // minus infinity: below the key of every finite logit
__device__ __forceinline__ int key_of(float v, int c) { return (__float_as_int(v) & ~63) | (63 - c); }
__device__ __forceinline__ int key_max(int a, int b) {
    int d;
    asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
__device__ __forceinline__ int key_med3(int a, int b, int c) {
    int d;
    asm("v_med3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ bool keys_apart(int a, int b) { return ((a ^ b) & ~63) != 0; }
// The N largest keys so far, k[0] >= k[1] >= ... throughout, and one more.
template <int N>
__device__ __forceinline__ void keep_key(int (&k)[N], int kk) {
    int nk[N];
    nk[0] = key_max(k[0], kk);
#pragma unroll
    for (int u = 1; u < N; ++u) nk[u] = key_med3(k[u - 1], k[u], kk);
#pragma unroll
    for (int u = 0; u < N; ++u) k[u] = nk[u];
}
// Whether the replaced bits may have decided the order of the keys kept, or what the last one is.
template <int N>
__device__ __forceinline__ bool keys_undecided(const int (&k)[N]) {
    bool any = false;
#pragma unroll
    for (int u = 0; u + 1 < N; ++u) any = any | !(keys_apart(k[u], k[u + 1]) | (k[u] == KEY_EMPTY));
    return any;
}

// Gates before the division, and the divisor, of the experts es (-1: none) with logits vs.
__device__ __forceinline__ void gates_of(const float (&vs)[4], const int (&es)[4], int K, float (&gs)[4], float &den) {
    gs[0] = expf(vs[0] - vs[0]);
    den = gs[0];
#pragma unroll
    for (int s = 1; s < 4; ++s)
        if (s < K) {
            if (es[s] >= 0) gs[s] = expf(vs[s] - vs[0]);
            den += gs[s];
        }
}

// A token's selection out, for K <= 4.
__device__ __forceinline__ void store_selection(int64_t t, int K, const int (&es)[4], float (&gs)[4], float den, int32_t *topk_idx, float *gates) {
#pragma unroll
    for (int s = 0; s < 4; ++s) gs[s] = gs[s] / den;
    if (K == 4 && ((reinterpret_cast<uintptr_t>(topk_idx) | reinterpret_cast<uintptr_t>(gates)) & 15) == 0) {
        typedef int i32x4 __attribute__((ext_vector_type(4)));
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<i32x4 *>(topk_idx + (size_t)t * 4) = i32x4{es[0], es[1], es[2], es[3]};
        *reinterpret_cast<f32x4 *>(gates + (size_t)t * 4) = f32x4{gs[0], gs[1], gs[2], gs[3]};
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (s < K) {
                topk_idx[(size_t)t * K + s] = es[s];
                gates[(size_t)t * K + s] = gs[s];
            }
    }
}

// The collaborators of every expert as a 64-bit mask (without itself; without lists all others).  Every thread of the workgroup calls it.
__device__ __forceinline__ void build_masks(uint64_t *mask_tab, const int32_t *__restrict__ collab_idx, int E, int Tc, uint64_t all) {
    if (threadIdx.x < C2R_MAX_E) mask_tab[threadIdx.x] = collab_idx ? 0ull : all & ~(1ull << threadIdx.x);
    __syncthreads();
    if (!collab_idx) return;
    for (int i = threadIdx.x; i < E * Tc; i += blockDim.x) {
        const int e = i / Tc, v = collab_idx[i];
        if (v >= 0 && v < E && v != e) atomicOr(reinterpret_cast<unsigned long long *>(&mask_tab[e]), 1ull << v);
    }
    __syncthreads();
}

// Undecided tokens of the 32 of a wave below: scanned by the wave one after the other, at 0.95 us each, or by their own lanes all at once, at
// 2 us and 0.1 a column.  Microseconds of the router with n of every 32 tokens undecided (together / alone), 32768 tokens of d 512: 60 experts, n = 6 33.0 /
// 36.1, n = 8 34.6 / 36.3, n = 10 36.5 / 34.2; 32 experts, n = 5 23.0 / 23.3, n = 6 24.0 / 23.2; 20 experts, n = 4 22.1 / 24.0, n = 5 22.8 / 22.0.
__device__ __forceinline__ bool scan_alone(int n, int E) { return 9 * n > E + 20; }

// The selection of 32 tokens by the wave that has their logits in registers, K <= 4: lane (mh, mc) holds experts 32 a + 8 (i / 4) + 4 mh + i % 4
// of token mc.  Both lanes of a token run the keyed chain of route_select_rows_kernel over their experts and then over the other's
// largest; with lists a chain of two keys finds the first expert, one over its collaborators the others.  Experts masked by -infinity stay
// out of the chains and are chosen, by the literal rule, where nothing else is left.  What the keys cannot decide is scanned by that
// rule (see route_select_keys_kernel).  tile (LDS, this wave's): the logits, [expert][32 tokens].
template <int NEB, class Acc>
__device__ __forceinline__ void select_of_sums(const Acc &sums, float *tile, const uint64_t *mask_tab, const SelectArgs &S, int64_t t0, int64_t T) {
    const int lane = lane_id(), mh = lane >> 5, mc = lane & 31, E = S.E, K = S.K;
    const int64_t t = t0 + mc;
    const uint64_t all = E >= 64 ? ~0ull : ((1ull << E) - 1ull);
    const uint64_t *const lists = S.collab_idx ? mask_tab : nullptr;
    float l[NEB * 16];
    float chk = 0.0f;
    int low = 0;
#pragma unroll
    for (int n = 0; n < NEB * 16; ++n) {
        const int e0 = n / 16 * 32 + n % 16 / 4 * 8 + n % 4, e = e0 + mh * 4;
        float v = sums[n / 16][0][n % 16];
        if (S.bias) v = v + S.bias[e < E ? e : 0];
        v = v + 0.0f;
        l[n] = v;
        if (e < E) {
            tile[e * 32 + mc] = v;
            chk = __builtin_fmaf(v, 0.0f, chk);  // NaN once a NaN or an infinity went in
            low |= __float_as_int(v) & 63;
        }
    }
    chk += __shfl_xor(chk, 32);
    low |= __shfl_xor(low, 32);
    uint64_t masked = 0;  // the token's experts at -infinity
    if (__ballot(chk != chk)) {  // (one of them makes a NaN of every token's sum)
        uint32_t mine[2] = {0u, 0u};
        chk = 0.0f;
#pragma unroll
        for (int n = 0; n < NEB * 16; ++n) {
            const int e0 = n / 16 * 32 + n % 16 / 4 * 8 + n % 4;
            const bool out = __float_as_int(l[n]) == KEY_EMPTY;
            if (e0 + mh * 4 < E) {
                mine[n / 16] |= out ? 1u << (e0 % 32) : 0u;
                chk = __builtin_fmaf(out ? 0.0f : l[n], 0.0f, chk);
            }
        }
        chk += __shfl_xor(chk, 32);
        masked = ((uint64_t)mine[1] << 32 | mine[0]) << (mh * 4);
        masked |= (uint64_t)(uint32_t)__shfl_xor((int)(masked >> 32), 32) << 32 | (uint32_t)__shfl_xor((int)masked, 32);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the tile is this wave's alone)
    // the NKEEP largest keys of the token's experts in m, the same in both its lanes
    auto largest = [&](auto &k, uint64_t m) __attribute__((always_inline)) {
        constexpr int NKEEP = sizeof(k) / sizeof(k[0]);
#pragma unroll
        for (int u = 0; u < NKEEP; ++u) k[u] = KEY_EMPTY;
        const uint32_t mine[2] = {(uint32_t)(m >> (mh * 4)), (uint32_t)(m >> 32 >> (mh * 4))};
#pragma unroll
        for (int n = 0; n < NEB * 16; ++n) {
            const int e0 = n / 16 * 32 + n % 16 / 4 * 8 + n % 4;
            keep_key(k, (mine[n / 16] >> (e0 % 32)) & 1u ? (int)((__float_as_uint(l[n]) & ~63u) | (uint32_t)(63 - e0 - mh * 4)) : KEY_EMPTY);
        }
        int other[NKEEP];
#pragma unroll
        for (int u = 0; u < NKEEP; ++u) other[u] = __shfl_xor(k[u], 32);
#pragma unroll
        for (int u = 0; u < NKEEP; ++u) keep_key(k, other[u]);
    };
    bool literal = chk != chk, nonneg;
    int es[4];
    bool bare;  // a slot is left empty
    if (lists) {
        int k[2], r[4];
        largest(k, all & ~masked);
        literal = literal || keys_undecided(k);
        es[0] = 63 - (k[0] & 63);
        const uint64_t allowed = lists[es[0]];
        largest(r, allowed & ~masked);
        literal = literal || keys_undecided(r);
        masked &= k[0] == KEY_EMPTY ? ~0ull : allowed;
        nonneg = k[1] >= 0 && r[3] >= 0;
#pragma unroll
        for (int s = 1; s < 4; ++s) es[s] = r[s - 1] == KEY_EMPTY ? -1 : 63 - (r[s - 1] & 63);
        bare = k[0] == KEY_EMPTY;
    } else {
        int k[5];
        largest(k, all & ~masked);
        literal = literal || keys_undecided(k);
        nonneg = k[4] >= 0;
        es[0] = 63 - (k[0] & 63);
#pragma unroll
        for (int s = 1; s < 4; ++s) es[s] = k[s] == KEY_EMPTY ? -1 : 63 - (k[s] & 63);
        bare = k[0] == KEY_EMPTY;
    }
#pragma unroll
    for (int s = 1; s < 4; ++s) bare = bare || (s < K && es[s] < 0);
    literal = literal || (bare && masked != 0);
    uint64_t todo = __ballot(literal && t < T && mh == 0);
    if (todo & (todo - 1)) {
        // (rows of zeros that pad a batch: where the replaced bits were all zero and the keys kept are not negative, equal logits lie in
        // ascending columns and the chain is right as it stands)
        literal = literal && !(chk == chk && low == 0 && nonneg);
        todo = __ballot(literal && t < T && mh == 0);
    }
    const bool alone = scan_alone(__popcll(todo), E);
    float gs[4] = {0.0f, 0.0f, 0.0f, 0.0f}, den = 1.0f;
    if (!literal) {
        float vs[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= K) es[s] = -1;
            vs[s] = tile[(es[s] < 0 ? 0 : es[s]) * 32 + mc];
        }
        gates_of(vs, es, K, gs, den);
    } else if (alone && t < T) {
        literal_scan(
            [&](uint64_t mm, int &bi, float &bv) __attribute__((always_inline)) {
                bi = __ffsll((unsigned long long)mm) - 1;
                bv = tile[(bi < 0 ? 0 : bi) * 32 + mc];
                for (int e0 = 0; e0 < E; e0 += 8) {  // (eight reads at once; columns past E are not in mm)
                    const uint32_t in = (uint32_t)(mm >> e0);
                    float v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = tile[(e0 + u) * 32 + mc];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const bool take = (in & (1u << u)) != 0 && v[u] > bv;
                        bv = take ? v[u] : bv;
                        bi = take ? e0 + u : bi;
                    }
                }
            },
            K, all, lists, es, gs, den);
    }
    for (todo = alone ? 0 : todo; todo; todo &= todo - 1) {
        const int tk = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)todo) - 1), col = lane < E ? lane : 0;
        int et[4];
        float gt[4], dt;
        literal_scan_by_wave(tile[col * 32 + tk], K, all, lists, et, gt, dt);
        if (mc == tk) {
            den = dt;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                es[s] = et[s];
                gs[s] = gt[s];
            }
        }
    }
    if (t < T && mh == 0) store_selection(t, K, es, gs, den, S.topk_idx, S.gates);
}

// Partial logits of one 256-long k-chunk for NWV token tiles of 8*TQ tokens (one per wave), all
// experts.  A register-tiled fp32 GEMM: lane = (token lane tl, expert lane el) on an 8 x 8 grid; the
// thread owns tokens tl + 8q (q < TQ) and experts el*TE + j (j < TE), i.e. TQ*TE accumulators,
// and walks k upward one fused multiply-add at a time, which is the declared order.  Both
// operands come from LDS (x as stored, 16 bytes = 8 bf16 or 4 fp32 per token per read; W
// rows as fp32), staged in 32-wide k sub-tiles that are double buffered against global
// loads held in registers; the W sub-tile is shared by the workgroup's waves.
// TQ = 4 halves a wave's tile: twice the waves for batches that would otherwise leave one wave
// per SIMD with nothing to hide its LDS latency behind.
//
// MFMA = true does the same sums on the matrix pipe: one v_mfma_f32_32x32x2_f32 adds, to each of
// 32 experts x 32 tokens, the products of k and k+1 - as two fused multiply-adds, k first,
// then k+1, each rounded to nearest even (checked on the chip against chains of fmaf: bit
// identical, denormal and overflow ranges included), so a chain of them over ascending k IS
// the declared order, at twice the rate the vector pipe reaches without packed instructions.
// Lanes 0-31 feed k, lanes 32-63 k+1: one W value and one x value per lane and instruction.
// With 32-token wave tiles the sub-tiles of a workgroup's chunks are software-pipelined (see PIPE below), in one stream across the
// chunks (STREAM).  What bounds it is the matrix pipe, at the clock the power limit leaves (about 2.0 GHz: 131 TFLOP/s of the nominal
// 157), and with one wave per SIMD (32768 tokens) the trips to memory that nothing else hides.  Microseconds of the stage, 60 experts, d
// 2048, a pipeline per chunk (filled and drained at every 256 k) / one stream: 32768 tokens 102 / 86.6, fp32 117 / 90; 65536 tokens
// 162 / 153.5 (116 TFLOP/s on 64 columns); 16384 tokens 56.2 / 53.0.  Where a chunk is a workgroup of its own and the tile 32 experts
// wide, a pipeline per chunk is the faster one: its three smaller buffers leave room for three workgroups on a CU instead of two.  (16
// experts, d 4096: 9000 tokens 35.3 / 38.4, 26000 tokens 75.0 / 83.5; 32 experts, d 2048: 12000 tokens 27.7 / 30.0; 12 experts, d 8192: 16384
// tokens 93.5 / 107.8.  With sub-tiles of half the length the stream takes 36.3, 77.0, 28.2 and 104.4.)
// ALLCHUNKS (matrix pipe only): the workgroup walks ALL the chunks of its tokens and adds the
// chunk results up in registers, left to right - the declared order - so that scratch holds one
// 64-expert vector per token (256 bytes) instead of one per chunk (2 KB at d = 2048, written
// here and read back by the selection).  For batches with about a wave tile per SIMD of the chip (the rule: route_impl);
// smaller batches need the chunks as separate workgroups to fill it.
// HALVES: a token tile's two blocks of 32 experts by a wave each, half the tokens per workgroup.
// SELECT: the wave that has a token's logits selects as well, and nothing goes to scratch.
template <bool BF16, int TE, int NWV, int TQ, bool MFMA, bool ALLCHUNKS = false, bool HALVES = false, bool SELECT = false>
__global__ __launch_bounds__(NWV * 64, HALVES ? 4 : (MFMA && TQ == 4) ? 2 : 1) void route_partial_kernel(const void *__restrict__ x,
                                                                const float *__restrict__ W, int ldw,
                                                                int ep, int64_t T, int d, int nchunk, int cpw,
                                                                int64_t ntiles,
                                                                float *__restrict__ part, const SelectArgs S) {
    static_assert(!SELECT || (ALLCHUNKS && !HALVES), "a wave has all logits of its tokens");
    constexpr int EPAD = 8 * TE;         // experts covered by a wave (HALVES: by two)
    constexpr int NT = HALVES ? NWV / 2 : NWV;  // wave tiles of tokens in a workgroup
    static_assert(!HALVES || (MFMA && EPAD == 64), "halves of 32 experts");
    constexpr int TOK = 8 * TQ;          // tokens covered by a wave
    constexpr bool PIPE = MFMA && TOK == 32, STREAM = PIPE && (EPAD == 64 || ALLCHUNKS);
    constexpr int KS = STREAM && !BF16 ? 16 : 32;  // k per staged sub-tile
    constexpr int VEC = BF16 ? 8 : 4;    // elements per 16-byte vector of x
    constexpr int ESZ = BF16 ? 2 : 4;
    constexpr int XV = KS / VEC;         // 16-byte vectors per token per sub-tile
    constexpr int XPITCH = KS * ESZ + 16;  // bytes; token rows 8 apart land on distinct bank groups
    constexpr int XLOADS = TOK * XV / 64 / (NWV / NT);  // vectors per lane per sub-tile
    static_assert(XLOADS >= 1 && 64 % TOK == 0, "a wave loads whole vectors; wave tiles divide the 64-token tile");
    constexpr int WF4 = KS * EPAD / 4;     // float4 per W sub-tile
    constexpr int WLOADS = (WF4 + NWV * 64 - 1) / (NWV * 64);
    // One wave's matrix instructions of a sub-tile overlap its own operand reads of the next one
    // (PIPE): that takes a third LDS buffer - the stream a fourth - and two operand register sets,
    // which fit 32-token wave tiles only.
    constexpr int NBUF = STREAM ? 4 : PIPE ? 3 : 2;
    // (Counted on the matrix-pipe form at E = 60: SQ_LDS_BANK_CONFLICT = 128 cycles per wave task of
    // 8 sub-tiles, i.e. 16 per sub-tile - one per x operand read: 32 token rows 80 bytes apart fall
    // on 16 banks, a 2-way conflict that any row pitch that keeps the 16-byte staging stores
    // aligned has.  Against the 2048 matrix-pipe cycles of a sub-tile that is under 1 %; padding
    // the W rows instead, 32 floats per 64-wide row, changed neither the counter nor the time.)
    constexpr int WPITCH = EPAD;
    __shared__ __attribute__((aligned(16))) float Wl[NBUF][KS][WPITCH];
    __shared__ __attribute__((aligned(16))) unsigned char Xl[NBUF][NT][TOK * XPITCH];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tl = lane & 7, el = lane >> 3;
    const int64_t nwt = ntiles * (64 / TOK);       // wave tiles
    const int64_t ngroups = (nwt + NT - 1) / NT;
    const int64_t tgroup = blockIdx.x % ngroups;  // token tiles fastest: neighbours share W rows in L2
    const int chunk_first = ALLCHUNKS ? 0 : (int)(blockIdx.x / ngroups) * cpw;
    const int chunk_last = ALLCHUNKS ? nchunk - 1 : min(chunk_first + cpw, nchunk) - 1;
    // this wave's token tile and, with HALVES, its experts; the tile whose x it brings, and the first of its vectors
    const int tt = HALVES ? wave % NT : wave, eo = HALVES ? wave / NT * 32 : 0, xt = HALVES ? wave / 2 : wave;
    const int x0 = HALVES ? (wave & 1) * 64 : 0;
    const int64_t wt = tgroup * NT + tt;           // may be >= nwt: such a wave only helps load W
    const bool live = wt < nwt;
    int chunk = chunk_first, k_begin = chunk * C2R_CANON_CHUNK;
    int k_end = min(d, k_begin + C2R_CANON_CHUNK);
    const int64_t t0 = (tgroup * NT + xt) * TOK;   // of the tile whose x this wave brings
    const unsigned char *xb = static_cast<const unsigned char *>(x);

    // global loads of a sub-tile are held in registers until its LDS buffer is free; several sets (two in the plain loop, three
    // in the pipeline of a chunk, two of W and four of x in the stream), so that a sub-tile is fetched several sub-tiles
    // ahead (on the matrix pipe one sub-tile of compute is shorter than the memory latency)
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    struct Staged {
        f32x4 w[WLOADS];
        u32x4 x[XLOADS];
    };
    // Every load is issued, out-of-range ones on a clamped address: with no branch around a
    // load the compiler counts the loads in flight and waits only for the older set.  What a
    // clamped load brings is never used: k past the end of the chunk is left out by the
    // compute loops, experts >= ep and tokens >= T are accumulated and never stored or read.
    auto gload = [&](Staged &r, int k0) __attribute__((always_inline)) {
        f32x4 (&wreg)[WLOADS] = r.w;
        u32x4 (&xreg)[XLOADS] = r.x;
#pragma unroll
        for (int i = 0; i < WLOADS; ++i) {
            const int idx = tid + i * NWV * 64;
            const int k = idx / (EPAD / 4), c = idx % (EPAD / 4);
            const int kk = min(k0 + k, k_end - 1), cc = c * 4 < ep ? c : 0;
            wreg[i] = *reinterpret_cast<const f32x4 *>(W + (size_t)kk * ldw + cc * 4);
        }
#pragma unroll
        for (int i = 0; i < XLOADS; ++i) {
            const int idx = x0 + lane + i * 64;
            const int tok = idx / XV, c = idx % XV;
            int64_t t = t0 + tok;
            t = t < T ? t : T - 1;  // rows past the end (and dead waves) re-read a valid token
            t = t < 0 ? 0 : t;
            const int kc = min(k0 + c * VEC, k_end - VEC);
            xreg[i] = *reinterpret_cast<const u32x4 *>(xb + ((size_t)t * d + kc) * ESZ);
        }
    };
    // The same loads of a whole sub-tile (nothing to clamp in k): a uniform base per sub-tile
    // plus a 32-bit lane offset that is the same for every sub-tile.
    uint32_t woff[WLOADS], xoff[XLOADS];
#pragma unroll
    for (int i = 0; i < WLOADS; ++i) {
        const int idx = tid + i * NWV * 64;
        const int k = min(idx / (EPAD / 4), KS - 1), c = idx % (EPAD / 4);
        woff[i] = (uint32_t)((k * ldw + (c * 4 < ep ? c * 4 : 0)) * 4);
    }
    const int64_t tb = t0 < T ? t0 : T - 1;  // wave-uniform; dead waves re-read valid tokens
#pragma unroll
    for (int i = 0; i < XLOADS; ++i) {
        const int idx = x0 + lane + i * 64;
        const int64_t room = T - 1 - tb, tok = idx / XV < room ? idx / XV : room;
        xoff[i] = (uint32_t)((tok * d + (idx % XV) * VEC) * ESZ);
    }
    auto lstore = [&](const Staged &r, int buf) __attribute__((always_inline)) {
        const f32x4 (&wreg)[WLOADS] = r.w;
        const u32x4 (&xreg)[XLOADS] = r.x;
#pragma unroll
        for (int i = 0; i < WLOADS; ++i) {
            const int idx = tid + i * NWV * 64;
            if (WF4 % (NWV * 64) == 0 || idx < WF4) *reinterpret_cast<f32x4 *>(&Wl[buf][idx / (EPAD / 4)][(idx % (EPAD / 4)) * 4]) = wreg[i];
        }
#pragma unroll
        for (int i = 0; i < XLOADS; ++i) {
            const int idx = x0 + lane + i * 64;
            *reinterpret_cast<u32x4 *>(&Xl[buf][xt][(idx / XV) * XPITCH + (idx % XV) * 16]) = xreg[i];
        }
    };

    typedef float f32x16 __attribute__((ext_vector_type(16)));
    constexpr int NEB = MFMA ? EPAD / 32 / (NWV / NT) : 1, NTB = MFMA ? TOK / 32 : 1;  // 32-expert / 32-token blocks
    static_assert(!MFMA || (EPAD % 32 == 0 && TOK % 32 == 0), "whole 32 x 32 blocks");
    f32x16 macc[NEB][NTB];
#pragma unroll
    for (int a = 0; a < NEB; ++a)
#pragma unroll
        for (int b = 0; b < NTB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) macc[a][b][i] = 0.0f;
    f32x16 mtot[ALLCHUNKS ? NEB : 1][ALLCHUNKS ? NTB : 1];  // sum of the chunks done so far
    const int mh = lane >> 5, mc = lane & 31;  // k parity and block column fed by this lane
    float acc[TQ][TE];
#pragma unroll
    for (int q = 0; q < TQ; ++q)
#pragma unroll
        for (int j = 0; j < TE; ++j) acc[q][j] = 0.0f;

    auto compute = [&](int buf, int k0) __attribute__((always_inline)) {
        const int nvec = min(KS, k_end - k0) / VEC;  // workgroup-uniform
        if constexpr (MFMA) {
            auto pair = [&](int kp) __attribute__((always_inline)) {
                float wv[NEB], xv[NTB];
#pragma unroll
                for (int a = 0; a < NEB; ++a) wv[a] = Wl[buf][2 * kp + mh][eo + a * 32 + mc];
#pragma unroll
                for (int b = 0; b < NTB; ++b) {
                    const unsigned char *row = &Xl[buf][tt][(b * 32 + mc) * XPITCH];
                    if (BF16) {  // one word holds x[k] (low half) and x[k+1] (high half)
                        const uint32_t word = *reinterpret_cast<const uint32_t *>(row + kp * 4);
                        xv[b] = __uint_as_float(mh ? (word & 0xffff0000u) : (word << 16));
                    } else {
                        xv[b] = *reinterpret_cast<const float *>(row + (2 * kp + mh) * 4);
                    }
                }
#pragma unroll
                for (int a = 0; a < NEB; ++a)
#pragma unroll
                    for (int b = 0; b < NTB; ++b)
                        macc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[a], xv[b], macc[a][b], 0, 0, 0);
            };
            const int npair = nvec * VEC / 2;
            if (npair == KS / 2) {
                // a whole sub-tile: every operand is read first, into registers of its own, so that
                // the matrix instructions never wait for a read issued just before them
                float wv[KS / 2][NEB], xv[KS / 2][NTB];
#pragma unroll
                for (int kp = 0; kp < KS / 2; ++kp)
#pragma unroll
                    for (int a = 0; a < NEB; ++a) wv[kp][a] = Wl[buf][2 * kp + mh][eo + a * 32 + mc];
#pragma unroll
                for (int b = 0; b < NTB; ++b) {
                    const unsigned char *row = &Xl[buf][tt][(b * 32 + mc) * XPITCH];
#pragma unroll
                    for (int kp = 0; kp < KS / 2; ++kp) {
                        if (BF16) {
                            const uint32_t word = *reinterpret_cast<const uint32_t *>(row + kp * 4);
                            xv[kp][b] = __uint_as_float(mh ? (word & 0xffff0000u) : (word << 16));
                        } else {
                            xv[kp][b] = *reinterpret_cast<const float *>(row + (2 * kp + mh) * 4);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);  // (the scheduler would sink each read to its use)
#pragma unroll
                for (int kp = 0; kp < KS / 2; ++kp)
#pragma unroll
                    for (int a = 0; a < NEB; ++a)
#pragma unroll
                        for (int b = 0; b < NTB; ++b)
                            macc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[kp][a], xv[kp][b], macc[a][b], 0, 0, 0);
            } else {
                for (int kp = 0; kp < npair; ++kp) pair(kp);
            }
        } else
        for (int v = 0; v < nvec; ++v) {
            uint4 xp[TQ];
#pragma unroll
            for (int q = 0; q < TQ; ++q)
                xp[q] = *reinterpret_cast<const uint4 *>(&Xl[buf][tt][(tl + 8 * q) * XPITCH + v * 16]);
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                float wv[TE];
#pragma unroll
                for (int j = 0; j < TE; ++j) wv[j] = Wl[buf][v * VEC + u][el * TE + j];
#pragma unroll
                for (int q = 0; q < TQ; ++q) {
                    const uint32_t word = BF16 ? (u < 2 ? xp[q].x : u < 4 ? xp[q].y : u < 6 ? xp[q].z : xp[q].w)
                                               : (u == 0 ? xp[q].x : u == 1 ? xp[q].y : u == 2 ? xp[q].z : xp[q].w);
                    const float xv = BF16 ? __uint_as_float((u & 1) ? (word & 0xffff0000u) : (word << 16))
                                          : __uint_as_float(word);
#pragma unroll
                    for (int j = 0; j < TE; ++j) acc[q][j] = __builtin_fmaf(xv, wv[j], acc[q][j]);
                }
            }
        }
    };
    const int64_t tile = wt / (64 / TOK);           // the 64-token tile and this wave's part of it
    float *const dst_tile = part + ((size_t)tile * (ALLCHUNKS ? 1 : nchunk) * ep) * 64 + (wt % (64 / TOK)) * TOK;
    auto store_sums = [&](const f32x16 (&v)[NEB][NTB], int c) __attribute__((always_inline)) {
        float *dst = dst_tile + (size_t)c * ep * 64;
        uint32_t at = (uint32_t)(eo * 64 + mh * 256 + mc);  // (opaque: the 32 addresses are not held in registers across the chunks)
        asm volatile("" : "+v"(at));
        // register i of a 32 x 32 block: expert (i/4)*8 + 4*(lane/32) + i%4, token lane%32
#pragma unroll
        for (int a = 0; a < NEB; ++a)
#pragma unroll
            for (int b = 0; b < NTB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int e = a * 32 + (i / 4) * 8 + i % 4;
                    if (eo + e + mh * 4 < ep) dst[at + (uint32_t)(e * 64 + b * 32)] = v[a][b][i];
                }
    };
    // A chunk's sums are complete: out to scratch, or onto the sum of the chunks before it - left to right, plain fp32 adds,
    // as the selection kernel does when it reads them from scratch (the first onto -0, which leaves every value what it
    // is) - and the next chunk starts again from +0.
    auto finish_chunk = [&](int c) __attribute__((always_inline)) {
        if constexpr (MFMA) {
            if constexpr (!ALLCHUNKS) {
                if (live) store_sums(macc, c);
            }
#pragma unroll
            for (int a = 0; a < NEB; ++a)
#pragma unroll
                for (int b = 0; b < NTB; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        if constexpr (ALLCHUNKS) mtot[a][b][i] = mtot[a][b][i] + macc[a][b][i];
                        macc[a][b][i] = 0.0f;
                    }
        }
    };
    if constexpr (ALLCHUNKS) {
#pragma unroll
        for (int a = 0; a < NEB; ++a)
#pragma unroll
            for (int b = 0; b < NTB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) mtot[a][b][i] = -0.0f;
    }
    if constexpr (PIPE) {
        // The whole chunks.  The chain of every accumulator still takes k in ascending order, two per instruction.
        struct Ops {
            float w[KS / 2][NEB];
            uint32_t x[KS / 2][NTB];
        };
        auto read_ops = [&](Ops &o, int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int kp = 0; kp < KS / 2; ++kp)
#pragma unroll
                for (int a = 0; a < NEB; ++a) o.w[kp][a] = Wl[buf][2 * kp + mh][eo + a * 32 + mc];
#pragma unroll
            for (int b = 0; b < NTB; ++b) {
                const unsigned char *row = &Xl[buf][tt][(b * 32 + mc) * XPITCH];
#pragma unroll
                for (int kp = 0; kp < KS / 2; ++kp)  // bf16: the word holds x[k] (low) and x[k+1] (high)
                    o.x[kp][b] = *reinterpret_cast<const uint32_t *>(row + (BF16 ? kp : 2 * kp + mh) * 4);
            }
        };
        const int sh = mh ? 0 : 16;
        auto mma = [&](const Ops &o) __attribute__((always_inline)) {
#pragma unroll
            for (int kp = 0; kp < KS / 2; ++kp)
#pragma unroll
                for (int b = 0; b < NTB; ++b) {
                    const float xv = __uint_as_float(BF16 ? (o.x[kp][b] << sh) & 0xffff0000u : o.x[kp][b]);
#pragma unroll
                    for (int a = 0; a < NEB; ++a)
                        macc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.w[kp][a], xv, macc[a][b], 0, 0, 0);
                }
        };
        constexpr int NSUB = C2R_CANON_CHUNK / KS;
        if constexpr (STREAM) {
            // ONE stream of sub-tiles that runs on across chunk ends.  At step j: operands of sub-tile j in
            // registers (set j % 2), sub-tiles j+1 and j+2 in LDS (buffer j % 4), sub-tile j+3 on its way there from its staging
            // registers, W of j+4 and x of j+4 to j+6 (which comes from memory, W from L2) in flight.  (Past the last sub-tile that one
            // again, never used.)
            static_assert(NSUB % 4 == 0, "buffers and register sets take their turns inside a chunk");
            const int nwhole = min(chunk_last + 1, d / C2R_CANON_CHUNK) - chunk_first;
            if (nwhole > 0) {
                const int klast = (chunk_first + nwhole) * C2R_CANON_CHUNK - KS;
                f32x4 SW[2][WLOADS];
                u32x4 SX[4][XLOADS];
                auto load_w = [&](f32x4 (&r)[WLOADS], int k0) __attribute__((always_inline)) {
                    const unsigned char *wb = reinterpret_cast<const unsigned char *>(W + (size_t)min(k0, klast) * ldw);
#pragma unroll
                    for (int i = 0; i < WLOADS; ++i) r[i] = *reinterpret_cast<const f32x4 *>(wb + woff[i]);
                };
                auto load_x = [&](u32x4 (&r)[XLOADS], int k0) __attribute__((always_inline)) {
                    const unsigned char *xs = xb + ((size_t)tb * d + min(k0, klast)) * ESZ;
#pragma unroll
                    for (int i = 0; i < XLOADS; ++i) r[i] = *reinterpret_cast<const u32x4 *>(xs + xoff[i]);
                };
                auto to_lds = [&](const f32x4 (&w)[WLOADS], const u32x4 (&xv)[XLOADS], int buf) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < WLOADS; ++i) {
                        const int idx = tid + i * NWV * 64;
                        if (WF4 % (NWV * 64) == 0 || idx < WF4)
                            *reinterpret_cast<f32x4 *>(&Wl[buf][idx / (EPAD / 4)][(idx % (EPAD / 4)) * 4]) = w[i];
                    }
#pragma unroll
                    for (int i = 0; i < XLOADS; ++i) {
                        const int idx = x0 + lane + i * 64;
                        *reinterpret_cast<u32x4 *>(&Xl[buf][xt][(idx / XV) * XPITCH + (idx % XV) * 16]) = xv[i];
                    }
                };
                Ops O[2];
                int k0 = chunk_first * C2R_CANON_CHUNK;
                load_w(SW[0], k0);
                load_x(SX[0], k0);
                load_w(SW[1], k0 + KS);
                load_x(SX[1], k0 + KS);
                load_x(SX[2], k0 + 2 * KS);
                load_x(SX[3], k0 + 3 * KS);
                to_lds(SW[0], SX[0], 0);
                load_w(SW[0], k0 + 2 * KS);
                load_x(SX[0], k0 + 4 * KS);
                to_lds(SW[1], SX[1], 1);
                load_w(SW[1], k0 + 3 * KS);
                load_x(SX[1], k0 + 5 * KS);
                to_lds(SW[0], SX[2], 2);
                load_w(SW[0], k0 + 4 * KS);
                load_x(SX[2], k0 + 6 * KS);
                lds_hand_over();
                read_ops(O[0], 0);
                lds_hand_over();
                for (int c = 0; c < nwhole; ++c, k0 += C2R_CANON_CHUNK) {
#pragma unroll
                    for (int i = 0; i < NSUB; ++i) {
                        __builtin_amdgcn_sched_barrier(0);
                        read_ops(O[(i + 1) & 1], (i + 1) & 3);
                        to_lds(SW[(i + 3) & 1], SX[(i + 3) & 3], (i + 3) & 3);
                        load_w(SW[(i + 3) & 1], k0 + (i + 5) * KS);
                        load_x(SX[(i + 3) & 3], k0 + (i + 7) * KS);
                        mma(O[i & 1]);
                        // the step's memory instructions go between its matrix instructions, as a rule one each:
                        // the wave issues them while the matrix pipe works
                        constexpr int NMMA = NEB * NTB * KS / 2;
                        constexpr int NRD = KS / 4 * NEB + (BF16 ? KS / 8 : KS / 4) * NTB, NST = WLOADS + XLOADS;
                        constexpr int PER = (NRD + 2 * NST + NMMA - 1) / NMMA;
#pragma unroll
                        for (int m = 0; m < NMMA; ++m) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // a matrix instruction
#pragma unroll
                            for (int n = m * PER; n < (m + 1) * PER; ++n) {
                                if (n < NRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);             // an LDS read
                                else if (n < NRD + NST) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // an LDS write
                                else if (n < NRD + 2 * NST) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // a global load
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        // A buffer is written two steps before it is read and two steps after it was: one barrier per two steps.
                        if (i & 1) lds_hand_over();
                    }
                    finish_chunk(chunk_first + c);
                }
                chunk += nwhole;
                lds_hand_over();  // (a ragged last chunk starts on the same buffers)
            }
        } else if (k_end - k_begin == C2R_CANON_CHUNK) {
            // A workgroup's one chunk.  At step j: operands of sub-tile j in registers (set j % 2), sub-tile j+1 in LDS (buffer
            // j % 3), sub-tile j+2 on its way there from its staging registers (set j % 3), j+3 and j+4 in flight.  Straight-line
            // code, the loads of a whole sub-tile unclamped: only there are the waits for the oldest set alone.
            static_assert(STREAM || NSUB >= 5, "the prologue fetches sub-tiles 0 to 4");
            auto load = [&](Staged &r, int k0) __attribute__((always_inline)) {
                const unsigned char *wb = reinterpret_cast<const unsigned char *>(W + (size_t)k0 * ldw);
                const unsigned char *xs = xb + ((size_t)tb * d + k0) * ESZ;
#pragma unroll
                for (int i = 0; i < WLOADS; ++i) r.w[i] = *reinterpret_cast<const f32x4 *>(wb + woff[i]);
#pragma unroll
                for (int i = 0; i < XLOADS; ++i) r.x[i] = *reinterpret_cast<const u32x4 *>(xs + xoff[i]);
            };
            Staged R[3];
            Ops O[2];
#pragma unroll
            for (int i = 0; i < 3; ++i) load(R[i], k_begin + i * KS);
            lstore(R[0], 0);
            load(R[0], k_begin + 3 * KS);
            __syncthreads();
            read_ops(O[0], 0);
            lstore(R[1], 1);
            load(R[1], k_begin + 4 * KS);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NSUB; ++i) {
                if (i + 1 < NSUB) read_ops(O[(i + 1) & 1], (i + 1) % 3);
                if (i + 2 < NSUB) lstore(R[(i + 2) % 3], (i + 2) % 3);
                if (i + 5 < NSUB) load(R[(i + 2) % 3], k_begin + (i + 5) * KS);
                mma(O[i & 1]);
                // an LDS read after each matrix instruction: the wave issues them while the matrix pipe works
#pragma unroll
                for (int m = 0; m < NEB * NTB * KS / 2; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (i + 1 < NSUB) __syncthreads();
            }
            finish_chunk(chunk);
            ++chunk;
        }
    }
    static_assert(STREAM || !ALLCHUNKS, "otherwise a workgroup has one chunk");
    if (chunk <= chunk_last) {  // the one chunk that is left: a ragged last one, or the only one
    if constexpr (STREAM) {
        k_begin = chunk * C2R_CANON_CHUNK;
        k_end = min(d, k_begin + C2R_CANON_CHUNK);
    }
    Staged r0, r1;
    gload(r0, k_begin);
    lstore(r0, 0);
    gload(r1, k_begin + KS);  // (past the end of the chunk: clamped loads, never stored)
    gload(r0, k_begin + 2 * KS);
    __syncthreads();
    for (int k0 = k_begin; k0 < k_end; k0 += 2 * KS) {
        compute(0, k0);
        if (k0 + KS < k_end) lstore(r1, 1);
        gload(r1, k0 + 3 * KS);
        __syncthreads();
        if (k0 + KS >= k_end) break;
        compute(1, k0 + KS);
        if (k0 + 2 * KS < k_end) lstore(r0, 0);
        gload(r0, k0 + 4 * KS);
        __syncthreads();
    }
    finish_chunk(chunk);
    }
    if constexpr (SELECT) {
        // (the operand buffers, which every wave has read for the last time, hold the logits now)
        __shared__ uint64_t mask_tab[C2R_MAX_E];
        static_assert(sizeof(Xl) >= (size_t)NWV * EPAD * 32 * sizeof(float), "a tile of logits for every wave");
        build_masks(mask_tab, S.collab_idx, S.E, S.Tc, S.E >= 64 ? ~0ull : ((1ull << S.E) - 1ull));
        if (live) select_of_sums<NEB>(mtot, reinterpret_cast<float *>(&Xl[0][0][0]) + wave * (EPAD * 32), mask_tab, S, wt * TOK, T);
        return;
    }
    if (!live) return;
    if constexpr (MFMA) {
        if constexpr (ALLCHUNKS) store_sums(mtot, 0);
        return;
    }
    float *const dst = dst_tile + (size_t)chunk_first * ep * 64;
#pragma unroll
    for (int j = 0; j < TE; ++j) {
        const int e = el * TE + j;
        if (e < ep) {
#pragma unroll
            for (int q = 0; q < TQ; ++q) dst[(size_t)e * 64 + tl + 8 * q] = acc[q][j];
        }
    }
}

// The same partial sums for small batches, on v_mfma_f32_16x16x4_f32: 16 experts x 16 tokens, four k per instruction,
// added as four fused multiply-adds in ascending k (checked on the chip against chains of fmaf like the 32 x 32 x 2 form:
// bit identical), so that this too is the declared order.  What bounds a small batch is the length of ONE chain: 256 k are
// 64 instructions of 32 cycles here, 0.9 us, against two interleaved chains of 128 instructions of 64 cycles in the kernel
// above, 7 us.  A workgroup of four waves takes one k-chunk: NEB expert blocks x 4 / NEB token tiles of 16.  W_g goes
// straight from memory into operand registers (a lane's 64 values of its expert, all in flight together; rows need no
// padding to 16 bytes, so an E that is no multiple of 4 needs no repacked copy), x through LDS.
// Measured (both kernels of the stage, E 60, d 2048): 1 token 21.0 -> 12.8 us; E 8, d 4096: 16.0 -> 8.7 us.
template <bool BF16, int NEB>
__global__ __launch_bounds__(256) void route_partial_small_kernel(const void *__restrict__ x, const float *__restrict__ Wg,
                                                                  int E, int ep, int64_t T, int d, int nchunk,
                                                                  float *__restrict__ part) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef typename std::conditional<BF16, uint16_t, float>::type elem;
    constexpr int NT = 4 / NEB, TOK = 16 * NT, VEC = 16 / sizeof(elem), CH = C2R_CANON_CHUNK;
    constexpr int PITCH = CH + VEC, STEPS = CH / 4;
    __shared__ __attribute__((aligned(16))) elem xs[TOK * PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x % nchunk, k0 = chunk * CH, len = min(d - k0, CH);  // len: a multiple of 8
    const int64_t t0 = (int64_t)(blockIdx.x / nchunk) * TOK;
    const int eb = wave % NEB, tt = wave / NEB, col = lane & 15, kk = lane >> 4;
    const int e = eb * 16 + col;
    const float *wp = Wg + (size_t)(k0 + kk) * E + (e < E ? e : 0);  // (sums of experts past E are never read)
    float w[STEPS];
    const bool whole = len == CH;
    if (whole) {
#pragma unroll
        for (int i = 0; i < STEPS; ++i) w[i] = wp[(size_t)(4 * i) * E];
    }
    // (every load is issued before the first store: in a loop of load and store each would wait for its own trip to memory)
    constexpr int NV = TOK * (CH / VEC) / 256;
    uint4 xv[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int i = tid + u * 256, tok = i / (CH / VEC), c = i % (CH / VEC) * VEC;
        const int64_t t = t0 + tok < T ? t0 + tok : T - 1;
        xv[u] = *reinterpret_cast<const uint4 *>(static_cast<const elem *>(x) + t * d + k0 + min(c, len - VEC));
    }
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int i = tid + u * 256;
        *reinterpret_cast<uint4 *>(&xs[i / (CH / VEC) * PITCH + i % (CH / VEC) * VEC]) = xv[u];
    }
    __syncthreads();
    const elem *xr = &xs[(tt * 16 + col) * PITCH + kk];
    auto xval = [&](int i) __attribute__((always_inline)) {
        if constexpr (BF16) return __uint_as_float((uint32_t)xr[4 * i] << 16);
        else return xr[4 * i];
    };
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    if (whole) {
#pragma unroll
        for (int i = 0; i < STEPS; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], xval(i), acc, 0, 0, 0);
    } else {
        for (int i = 0; i < len / 4; ++i)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wp[(size_t)(4 * i) * E], xval(i), acc, 0, 0, 0);
    }
    // register i: expert 4 * (lane / 16) + i of the block, token lane % 16
    const int64_t t = t0 + tt * 16 + col;
    float *dst = part + ((size_t)(t >> 6) * nchunk + chunk) * ep * 64 + (t & 63);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int ei = eb * 16 + kk * 4 + i;
        if (ei < ep && t < (T + 63) / 64 * 64) dst[(size_t)ei * 64] = acc[i];
    }
}

// Among experts whose bit is set in m: the largest logit, first one standing
// unless a later one is strictly larger (so ties and NaNs go to the lower index).
template <int EP>
__device__ __forceinline__ void pick(const float (&l)[EP], uint64_t m, int &bi, float &bv) {
    bi = -1;
    bv = 0.0f;
    const uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
#pragma unroll
    for (int e = 0; e < EP; ++e) {
        const bool ok = (((e < 32) ? (lo >> (e & 31)) : (hi >> (e & 31))) & 1u) != 0;
        const bool take = ok && (bi < 0 || l[e] > bv);
        bv = take ? l[e] : bv;
        bi = take ? e : bi;
    }
}

// ROWMAJOR (stored logits [T, E]): one wave per 64 tokens.  Otherwise (chunk partials):
// SEL_WAVES waves per 64 tokens; each sums the chunks of a quarter of the experts (the
// loads of one wave alone cover the memory latency four times worse) and leaves its
// logits in LDS, then the first wave selects.
constexpr int SEL_WAVES = 4;

template <int EP, bool ROWMAJOR>
__global__ __launch_bounds__(ROWMAJOR ? 64 : SEL_WAVES * 64) void route_select_kernel(
    const float *__restrict__ src, int nchunk, const float *__restrict__ bias,
    int64_t T, int E, int K, const int32_t *__restrict__ collab_idx, int Tc,
    int32_t *__restrict__ topk_idx, float *__restrict__ gates, float *__restrict__ logits_out) {
    __shared__ uint64_t mask_tab[C2R_MAX_E];
    constexpr int LP = EP + 1;  // odd pitch: per-lane row reads hit distinct banks
    __shared__ float tile[64 * LP];

    const uint64_t all = E >= 64 ? ~0ull : ((1ull << E) - 1ull);
    // one 64-bit collaborator mask per expert; the list entries are spread over all the threads
    // (one thread walking a whole list would wait for Tc loads one after another).  With chunk
    // partials a thread's first four entries are requested ahead of the partial sums and go into
    // the masks after them, so that the two trips to memory are one.
    constexpr int AHEAD = ROWMAJOR ? 0 : 4;
    if (threadIdx.x < C2R_MAX_E)
        mask_tab[threadIdx.x] = (!collab_idx && (int)threadIdx.x < E) ? all & ~(1ull << threadIdx.x) : 0ull;
    const int nlist = collab_idx ? E * Tc : 0;
    auto allow = [&](int i, int v) __attribute__((always_inline)) {
        const int e = i / Tc;
        if (v >= 0 && v < E && v != e)
            atomicOr(reinterpret_cast<unsigned long long *>(&mask_tab[e]), 1ull << v);
    };
    int32_t ahead[AHEAD > 0 ? AHEAD : 1];
    if (collab_idx) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) ahead[u] = collab_idx[min((int)(threadIdx.x + u * blockDim.x), nlist - 1)];
        if (AHEAD == 0) {
#pragma unroll 4
            for (int i = threadIdx.x; i < nlist; i += blockDim.x) allow(i, collab_idx[i]);
        }
    }

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t t = (int64_t)blockIdx.x * 64 + lane;
    float l[EP];
    if constexpr (ROWMAJOR) {
        // wave-private transpose: 64 consecutive rows of E floats are one contiguous run
        float *tl = tile;
        const int64_t tw = (int64_t)blockIdx.x * 64;
        const int64_t rows = T - tw < 64 ? T - tw : 64;  // may be <= 0
        const int64_t nflt = rows > 0 ? rows * E : 0;
        const float *base = src + tw * E;
        const uint32_t rcp = (uint32_t)((0x100000000ull + E - 1) / E);
        auto scatter = [&](uint32_t f, float v) __attribute__((always_inline)) {
            // f / E, exact for f < 4096 (the 32-bit reciprocal of 1 does not exist)
            const uint32_t r = E == 1 ? f : __umulhi(f, rcp);
            tl[r * LP + (f - r * E)] = v;
        };
        if (rows == 64) {
            // a whole tile: 64 E floats (a multiple of 4), fetched with every load in flight at once -
            // unconditional, out-of-range ones on a clamped address - and only then spread over LDS:
            // what this kernel does is stream the logits, and a wave that waits for one 1 KB load
            // at a time (the loop below) leaves the memory pipe a fifth full
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            constexpr int NV = EP / 4;
            f32x4 q[NV];
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const uint32_t i = (uint32_t)lane * 4 + u * 256;
                q[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(base + (i < nflt ? i : 0)));
            }
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const uint32_t i = (uint32_t)lane * 4 + u * 256;
                if (i < nflt) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) scatter(i + j, q[u][j]);
                }
            }
        } else
        for (int64_t i = (int64_t)lane * 4; i < nflt; i += 256) {
            float v[4];
            if (i + 4 <= nflt) {
                const float4 q = *reinterpret_cast<const float4 *>(base + i);
                v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = i + j < nflt ? base[i + j] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t f = (uint32_t)i + j;
                if (f < nflt) scatter(f, v[j]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < EP; ++e) l[e] = (e < E && lane < rows) ? tl[lane * LP + e] : 0.0f;
    } else {
        static_assert(EP % SEL_WAVES == 0, "experts divide over the waves");
        constexpr int EW = EP / SEL_WAVES;   // experts of this wave
        constexpr int ES = (EW + 3) / 4;     // in steps of four
        // A lane adds up four tokens (16-byte loads) of one expert per step: lane = (token quad,
        // expert within the step).  Chunk results are added left to right; eight chunks x ES
        // loads are in flight together (the partial sums were written by other XCDs a moment
        // ago, so every batch costs a trip to memory), all of them unconditional on clamped
        // indices.
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        constexpr int CU = 8;
        const int tq4 = lane & 15, es = lane >> 4;
        const float *p = src + ((size_t)blockIdx.x * nchunk * EP + (size_t)wave * EW) * 64 + 4 * tq4;
        f32x4 sum[ES];
        for (int c0 = 0; c0 < nchunk; c0 += CU) {
            f32x4 v[CU][ES];
#pragma unroll
            for (int u = 0; u < CU; ++u) {
                const int cc = min(c0 + u, nchunk - 1);
#pragma unroll
                for (int j = 0; j < ES; ++j) {
                    const int el = min(4 * j + es, EW - 1);
                    v[u][j] = *reinterpret_cast<const f32x4 *>(p + ((size_t)cc * EP + el) * 64);
                }
            }
#pragma unroll
            for (int u = 0; u < CU; ++u) {
                const bool have = c0 + u < nchunk;  // wave-uniform
#pragma unroll
                for (int j = 0; j < ES; ++j) sum[j] = !have ? sum[j] : (c0 + u == 0) ? v[u][j] : sum[j] + v[u][j];
            }
        }
#pragma unroll
        for (int j = 0; j < ES; ++j) {
            const int el = 4 * j + es, e = wave * EW + el;
            if (el < EW) {
                if (bias && e < E) sum[j] = sum[j] + bias[e];
#pragma unroll
                for (int i = 0; i < 4; ++i) tile[(4 * tq4 + i) * LP + e] = sum[j][i];
            }
        }
        if (collab_idx) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const int i = threadIdx.x + u * blockDim.x;
                if (i < nlist) allow(i, ahead[u]);
            }
            for (int i = threadIdx.x + AHEAD * blockDim.x; i < nlist; i += blockDim.x) allow(i, collab_idx[i]);
        }
        __syncthreads();
        // Selection by all the waves: four lanes per token, each over a quarter of the experts.
        constexpr int EQ = EP / 4;
        const int tl = wave * (64 / SEL_WAVES) + (lane >> 2), sub = lane & 3;
        const int64_t tq = (int64_t)blockIdx.x * 64 + tl;
        if (tq >= T) return;  // (the four lanes of a token leave together)
        float lq[EQ];
#pragma unroll
        for (int j = 0; j < EQ; ++j) lq[j] = tile[tl * LP + sub * EQ + j];
        if (logits_out) {
#pragma unroll
            for (int j = 0; j < EQ; ++j)
                if (sub * EQ + j < E) logits_out[(size_t)tq * E + sub * EQ + j] = lq[j];
        }
        // The scan "first one standing unless a later one is strictly larger" over all experts,
        // taken apart: the largest value that is not a NaN (ties to the lower index) of each
        // quarter, the quarters merged in index order, and at the end the one case in which the
        // scan differs from that: its first allowed expert holds a NaN, which then stands.
        auto pick4 = [&](uint64_t m, int &bi, float &bv) __attribute__((always_inline)) {
            const uint32_t mloc = (uint32_t)(m >> (sub * EQ));
            bi = -1;
            bv = 0.0f;
#pragma unroll
            for (int j = 0; j < EQ; ++j) {
                const bool ok = ((mloc >> j) & 1u) != 0;
                const bool take = ok && (lq[j] > bv || (bi < 0 && lq[j] == lq[j]));
                bv = take ? lq[j] : bv;
                bi = take ? sub * EQ + j : bi;
            }
            merge_lower<0xB1>(sub & 1, bi, bv);  // quad_perm 1,0,3,2
            merge_lower<0x4E>(sub & 2, bi, bv);  // quad_perm 2,3,0,1
            if (m != 0) {
                const int f = __ffsll((unsigned long long)m) - 1;
                const float lf = tile[tl * LP + f];
                if (lf != lf) {
                    bi = f;
                    bv = lf;
                }
            }
        };
        int e0;
        float v0;
        pick4(all, e0, v0);
        uint64_t m = mask_tab[e0];
        const float g0 = expf(v0 - v0);  // 1, or NaN when the largest logit is infinite or a NaN
        float den = g0;
        if (K <= 8) {  // the usual case: the token's slots stay in registers until the gates are known
            int es[8];
            float gs[8];
            es[0] = e0;
            gs[0] = g0;
#pragma unroll
            for (int s = 1; s < 8; ++s) {
                es[s] = -1;
                gs[s] = 0.0f;
                if (s < K) {
                    float v;
                    pick4(m, es[s], v);
                    if (es[s] >= 0) {
                        m &= ~(1ull << es[s]);
                        gs[s] = expf(v - v0);
                    }
                    den += gs[s];
                }
            }
            if (sub == 0) {
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    if (s < K) {
                        topk_idx[(size_t)tq * K + s] = es[s];
                        gates[(size_t)tq * K + s] = gs[s] / den;
                    }
            }
            return;
        }
        if (sub == 0) {
            topk_idx[(size_t)tq * K] = e0;
            gates[(size_t)tq * K] = g0;
        }
        for (int s = 1; s < K; ++s) {
            int e;
            float v;
            pick4(m, e, v);
            float g = 0.0f;
            if (e >= 0) {
                m &= ~(1ull << e);
                g = expf(v - v0);
            }
            den += g;
            if (sub == 0) {
                topk_idx[(size_t)tq * K + s] = e;
                gates[(size_t)tq * K + s] = g;
            }
        }
        if (sub == 0)
            for (int s = 0; s < K; ++s) gates[(size_t)tq * K + s] = gates[(size_t)tq * K + s] / den;
        return;
    }
    if (t >= T) return;

    if (logits_out) {
#pragma unroll
        for (int e = 0; e < EP; ++e)
            if (e < E) logits_out[(size_t)t * E + e] = l[e];
    }

    int e0;
    float v0;
    pick<EP>(l, all, e0, v0);
    uint64_t m = mask_tab[e0];
    const float g0 = expf(v0 - v0);  // 1, or NaN when the largest logit is infinite or a NaN
    float den = g0;
    if (K <= 8) {
        // the usual case: the token's slots stay in registers and leave as 16-byte stores
        int es[8];
        float gs[8];
        es[0] = e0;
        gs[0] = g0;
#pragma unroll
        for (int s = 1; s < 8; ++s) {
            es[s] = -1;
            gs[s] = 0.0f;
            if (s < K) {
                int e;
                float v;
                pick<EP>(l, m, e, v);
                if (e >= 0) {
                    m &= ~(1ull << e);
                    gs[s] = expf(v - v0);
                }
                es[s] = e;
                den += gs[s];
            }
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) gs[s] = gs[s] / den;
        if (K == 4 && ((reinterpret_cast<uintptr_t>(topk_idx) | reinterpret_cast<uintptr_t>(gates)) & 15) == 0) {
            typedef int i32x4 __attribute__((ext_vector_type(4)));
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            const i32x4 ev = {es[0], es[1], es[2], es[3]};
            const f32x4 gv = {gs[0], gs[1], gs[2], gs[3]};
            __builtin_nontemporal_store(ev, reinterpret_cast<i32x4 *>(topk_idx + (size_t)t * 4));
            __builtin_nontemporal_store(gv, reinterpret_cast<f32x4 *>(gates + (size_t)t * 4));
        } else {
#pragma unroll
            for (int s = 0; s < 8; ++s)
                if (s < K) {
                    topk_idx[(size_t)t * K + s] = es[s];
                    gates[(size_t)t * K + s] = gs[s];
                }
        }
        return;
    }
    topk_idx[(size_t)t * K] = e0;
    gates[(size_t)t * K] = g0;
    for (int s = 1; s < K; ++s) {
        int e;
        float v;
        pick<EP>(l, m, e, v);
        float g = 0.0f;
        if (e >= 0) {
            m &= ~(1ull << e);
            g = expf(v - v0);
        }
        den += g;
        topk_idx[(size_t)t * K + s] = e;
        gates[(size_t)t * K + s] = g;
    }
    for (int s = 0; s < K; ++s) gates[(size_t)t * K + s] = gates[(size_t)t * K + s] / den;
}

// Undecided tokens of a 64-token group that the wave scans together, one after the other: up to E / SCAN_TOGETHER; more are scanned by
// their own lanes, all at once.  The one takes 0.9 us a token (four slots), the other 0.2 us a column whatever the number of tokens.
// Microseconds of the selection with n of every 64 tokens undecided (together / alone): 2^20 tokens, 60 experts, n = 8 104 / 140, n = 12
// 135 / 134, n = 16 166 / 134, n = 64 549 / 129; 36 experts, n = 6 74 / 87, n = 8 90 / 87; 16 experts, n = 3 32 / 37, n = 4 38 / 37; 8 experts,
// n = 1 18 / 24, n = 3 29 / 24; 65536 tokens, 60 experts, n = 8 15.1 / 24.8, n = 12 18.9 / 19.6, n = 16 22.6 / 19.6.
constexpr int SCAN_TOGETHER = 5;

// Top-K, K <= 4, from ONE chunk result per token ([tile][expert][64 tokens]), without lists: a wave per 64 tokens, lane = token, its
// logits in registers, chosen by the keyed chain of route_select_rows_kernel below, the literal scan where that cannot decide.
// Such batches are those of one chunk (d up to 256), those whose sums select_of_sums cannot take: 64-token workgroups, logits asked for,
// results that meet the inputs.  Bound by the launch and two trips to memory; the stage with route_select_kernel / with this, in batches that
// now take the other: 60 experts, d 2048: 32768 tokens 87.0 / 84.0, 65536 tokens 155 / 150; 16 experts, 32768 tokens 103.8 / 102.4.  (With lists, the largest two keys and a second chain over the
// first one's list, it was no faster: 15.6 against 12.7 us for the kernel at 32768 tokens.)
constexpr int KEYS_SCAN_TOGETHER = 8;  // as SCAN_TOGETHER; here a token scanned by the wave also waits for its logits out of L2

template <int EP>
__global__ __launch_bounds__(64) void route_select_keys_kernel(const float *__restrict__ part, const float *__restrict__ bias, int64_t T,
                                                               int E, int K, int32_t *__restrict__ topk_idx,
                                                               float *__restrict__ gates, float *__restrict__ logits_out) {
    const int lane = threadIdx.x;
    const int64_t t = (int64_t)blockIdx.x * 64 + lane;
    const uint64_t all = E >= 64 ? ~0ull : ((1ull << E) - 1ull);
    const float *p = part + (size_t)blockIdx.x * EP * 64;
    float l[EP];
#pragma unroll
    for (int e = 0; e < EP; ++e) l[e] = p[e * 64 + lane];
    if (bias) {
#pragma unroll
        for (int e = 0; e < EP; ++e)
            if (e < E) l[e] = l[e] + bias[e];
    }
    if (logits_out && t < T) {
#pragma unroll
        for (int e = 0; e < EP; ++e)
            if (e < E) logits_out[(size_t)t * E + e] = l[e];
    }
    auto logit_of = [&](int e) __attribute__((always_inline)) { return bias ? p[e * 64 + lane] + bias[e] : p[e * 64 + lane]; };
    constexpr int NKEEP = 5;
    int k[NKEEP];
#pragma unroll
    for (int u = 0; u < NKEEP; ++u) k[u] = KEY_EMPTY;
    float chk = 0.0f;
#pragma unroll
    for (int e = 0; e < EP; ++e)
        if (e < E) {  // (uniform)
            l[e] = l[e] + 0.0f;
            chk = __builtin_fmaf(l[e], 0.0f, chk);  // NaN once a NaN or an infinity went in
            keep_key(k, key_of(l[e], e));
        }
    bool literal = chk != chk;
    literal = literal || keys_undecided(k);
    // Undecided tokens come in numbers where rows of zeros pad a batch (their logits are all +0) or an expert is masked by -infinity.
    // Where the replaced bits were all zero and the keys kept are not negative, equal logits lie in ascending columns and the chain
    // is right as it stands; what is left is scanned as in route_select_rows_kernel.
    uint64_t todo = __ballot(literal && t < T);
    if (todo & (todo - 1)) {
        int low = 0;
#pragma unroll
        for (int e = 0; e < EP; ++e)
            if (e < E) low |= __float_as_int(l[e]) & 63;
        literal = literal && !(chk == chk && low == 0 && k[NKEEP - 1] >= 0);
        todo = __ballot(literal && t < T);
    }
    const bool alone = __popcll(todo) * KEYS_SCAN_TOGETHER > E;
    int es[4] = {63 - (k[0] & 63), -1, -1, -1};
#pragma unroll
    for (int u = 1; u < 4; ++u) es[u] = k[u] == KEY_EMPTY ? -1 : 63 - (k[u] & 63);
    float gs[4] = {0.0f, 0.0f, 0.0f, 0.0f}, den = 1.0f;
    if (!literal) {
        float vs[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= K) es[s] = -1;
            vs[s] = logit_of(es[s] < 0 ? 0 : es[s]);
        }
        gates_of(vs, es, K, gs, den);
    }
    if (alone && literal && t < T)
        literal_scan([&](uint64_t mm, int &bi, float &bv) __attribute__((always_inline)) { pick<EP>(l, mm, bi, bv); }, K, all, nullptr, es,
                     gs, den);
    for (todo = alone ? 0 : todo; todo; todo &= todo - 1) {
        const int tk = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)todo) - 1), col = lane < E ? lane : 0;
        float v = p[col * 64 + tk];
        if (bias) v = v + bias[col];
        int et[4];
        float gt[4], dt;
        literal_scan_by_wave(v + 0.0f, K, all, nullptr, et, gt, dt);
        if (lane == tk) {
            den = dt;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                es[s] = et[s];
                gs[s] = gt[s];
            }
        }
    }
    if (t < T) store_selection(t, K, es, gs, den, topk_idx, gates);
}

// Selection from stored logits [T, E] (the profiling pass of Sec. 3.2 routes 2^20 tokens of stored
// router outputs), for E a multiple of 4 and K <= 4.  What the kernel has to do is stream the
// logits, so the arithmetic per token is kept small:
//  * phase 1: a quad of lanes fetches a token's row, lane `sub` the 16-byte pieces at columns
//    16 i + 4 sub (64 contiguous bytes per quad and load, every load of a 64-token group in flight
//    at once), and the values go to LDS transposed, [column][token], the token position XOR-ed with
//    16 sub so that neither these writes nor the reads of phase 2 meet on a bank.
//  * phase 2, one lane per token.  The low 6 bits of a logit (-0 stored as +0) are replaced by 63 - column: the largest few of these
//    keys, compared as floats - a chain of one max and a few med3 per value, no index bookkeeping - are the largest logits WITH
//    their columns, provided the keys' upper 26 bits differ among the ones kept and the next one below them (then the replaced
//    bits decided nothing).  Without lists the
//    chain keeps five keys of the E columns: the token's K experts and the guard.  With lists it
//    keeps two (top-1 and guard), then walks the top-1's collaborator list ONLY (built once per
//    workgroup from the 64-bit masks, ascending: duplicates, the expert itself and out-of-range
//    entries are gone) keeping four: Tc visits instead of (K - 1) E.
//  * A token that fails the proviso, or has a NaN or an infinity among its logits, takes the
//    literal scan (first one standing unless a later one is strictly larger) for every slot.  Of 2^20 tokens of 60 normal logits some
//    300 do, one lane's scan is 15 us of LDS reads one after the other, and a launch ends with its last wave: the whole wave
//    scans such a token, a lane per column (2^20 tokens 60 -> 51.6 us, 65536 tokens 20 -> 14.6; with the keys compared as floats instead
//    of made order-preserving integers first, three instructions of ten per logit, 48.8 and 13.7; the stream alone 40).  A wave that
//    holds many of them (ties of rounded logits, an expert masked by -infinity) lets every lane scan its own: see SCAN_TOGETHER.
// COUNT: the token's expert pairs are added to the co-activation matrix (Eq. 2) on the spot - an LDS
// histogram per workgroup as in coact.hip, one integer atomic per entry at the end - and either
// output may be left out (null): the profiling pass wants the counts, not the selections.
template <int NV, bool LISTS, bool COUNT>
__global__ __launch_bounds__(256) void route_select_rows_kernel(const float *__restrict__ logits, int64_t T, int E, int K,
                                                                const int32_t *__restrict__ collab_idx, int Tc,
                                                                int32_t *__restrict__ topk_idx,
                                                                float *__restrict__ gates, int32_t *__restrict__ Cmat,
                                                                int64_t ngroups) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    // per wave: [column][token ^ 4 * (column >> 2)] floats for 16 NV columns; a power of two, so that
    // offsets inside a tile may be combined with XOR
    constexpr int TILE_BYTES = NV == 1 ? 4096 : NV == 2 ? 8192 : 16384;
    __shared__ __attribute__((aligned(1024))) unsigned char tile_mem[4 * TILE_BYTES];
    __shared__ uint64_t mask_tab[LISTS ? C2R_MAX_E : 1];
    // clist[e][k]: the k-th collaborator c of e (ascending) as the byte offset of its column in a
    // wave's tile, swizzle term included: c * 256 + 64 * ((c >> 2) & 3)
    __shared__ __attribute__((aligned(16))) uint16_t clist[LISTS ? C2R_MAX_E * 64 : 4];
    __shared__ int cnt[LISTS ? C2R_MAX_E : 1];
    __shared__ int maxcnt;
    __shared__ int32_t red[COUNT ? C2R_MAX_E * C2R_MAX_E : 1];  // co-activation counts of this workgroup, red[a][b], a <= b

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t all = E >= 64 ? ~0ull : ((1ull << E) - 1ull);
    auto code_of = [](int c) __attribute__((always_inline)) { return (uint32_t)(c * 256 + ((c >> 2) << 4)); };
    int nmax = 0;
    if constexpr (COUNT) {
        for (int i = tid; i < C2R_MAX_E * C2R_MAX_E; i += 256) red[i] = 0;
        if constexpr (!LISTS) __syncthreads();
    }
    if constexpr (LISTS) {
        if (tid < C2R_MAX_E) mask_tab[tid] = 0ull;
        if (tid == 0) maxcnt = 0;
        for (int i = tid; i < C2R_MAX_E * 64 / 2; i += 256) reinterpret_cast<uint32_t *>(clist)[i] = 0u;
        __syncthreads();
        const int n = E * Tc;
#pragma unroll 4
        for (int i = tid; i < n; i += 256) {
            const int v = collab_idx[i], e = i / Tc;
            if (v >= 0 && v < E && v != e) atomicOr(reinterpret_cast<unsigned long long *>(&mask_tab[e]), 1ull << v);
        }
        __syncthreads();
        if (tid < C2R_MAX_E) {
            uint64_t m = mask_tab[tid];
            int n2 = 0;
            while (m) {
                clist[tid * 64 + n2++] = (uint16_t)code_of(__ffsll((unsigned long long)m) - 1);
                m &= m - 1;
            }
            cnt[tid] = n2;
            atomicMax(&maxcnt, n2);
        }
        __syncthreads();
        nmax = __builtin_amdgcn_readfirstlane(maxcnt);
    }

    constexpr int EMPTY = KEY_EMPTY;
    // A 64-token group is one contiguous run of 64 E floats = E / 4 wave-wide 16-byte loads; lane l's
    // piece of load u holds columns col .. col + 3 of token tok, the same in every group.  Byte offsets
    // into tile_mem: of that piece's first float (the others follow 256 bytes apart), and of this
    // lane's token for the reads of phase 2.
    const int NU = E / 4;  // <= 4 NV
    uint32_t wr_off[4 * NV];
#pragma unroll
    for (int u = 0; u < 4 * NV; ++u) {
        const int f = u * 256 + lane * 4, tok = (f / E) & 63, col = f - (f / E) * E;
        wr_off[u] = (uint32_t)(wave * TILE_BYTES) + (((uint32_t)(tok * 4)) ^ code_of(col));
    }
    const uint32_t lanebase = (uint32_t)(wave * TILE_BYTES + lane * 4);
    auto lds_f = [&](uint32_t off) __attribute__((always_inline)) -> float & {
        return *reinterpret_cast<float *>(tile_mem + off);
    };
    // this token's logit of column c (any c, per lane)
    auto logit_of = [&](int c) __attribute__((always_inline)) { return lds_f(lanebase ^ code_of(c)); };
    // all loads of a 64-token group go out together (a piece past the end of the logits re-reads the start)
    f32x4 q[4 * NV];
    auto request = [&](int64_t g) __attribute__((always_inline)) {
        const int64_t left = T - g * 64;
        const int nflt = (int)(left < 64 ? left : 64) * E;
        const float *base = logits + g * 64 * E;
#pragma unroll
        for (int u = 0; u < 4 * NV; ++u) {
            const int f = u * 256 + lane * 4;
            if (u < 4 * NV - 3 || u < NU)  // (uniform)
                q[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(base + (f < nflt ? f : 0)));
        }
    };
    const int64_t gstep = (int64_t)gridDim.x * 4;
    int64_t g = (int64_t)blockIdx.x * 4 + wave;
    if (g < ngroups) request(g);
    for (; g < ngroups; g += gstep) {
        // ---- phase 1: the group's logits into LDS, transposed (-0 stored as +0)
#pragma unroll
        for (int u = 0; u < 4 * NV; ++u)
            if (u < 4 * NV - 3 || u < NU) {
#pragma unroll
                for (int j = 0; j < 4; ++j) lds_f(wr_off[u] + j * 256) = q[u][j] + 0.0f;
            }
        // ... and the next group's go out and fly while phase 2 runs (two groups of a wave in flight,
        // with a second register set and the loop body twice, measured slower: 72 against 65 us)
        if (g + gstep < ngroups) request(g + gstep);
        // (the wave's own LDS writes, read back by other lanes of the same wave: LDS operations of a
        // wave complete in order; the fences keep the compiler from moving them)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // ---- phase 2: one lane per token
        const int64_t t = g * 64 + lane;
        constexpr int NKEEP = LISTS ? 2 : 5;
        int k[NKEEP];
#pragma unroll
        for (int u = 0; u < NKEEP; ++u) k[u] = EMPTY;
        float chk = 0.0f;
#pragma unroll
        for (int c = 0; c < NV * 16; ++c) {
            if (c < (NV - 1) * 16 || c < E) {  // (uniform)
                const float v = lds_f((lanebase ^ (uint32_t)((c >> 2) << 4)) + c * 256);
                chk = __builtin_fmaf(v, 0.0f, chk);  // NaN once a NaN or an infinity went in
                const int kk = key_of(v, c);
                int nk[NKEEP];
                nk[0] = key_max(k[0], kk);
#pragma unroll
                for (int u = 1; u < NKEEP; ++u) nk[u] = key_med3(k[u - 1], k[u], kk);  // (k[0] >= k[1] >= ... throughout)
#pragma unroll
                for (int u = 0; u < NKEEP; ++u) k[u] = nk[u];
            }
        }
        bool literal = chk != chk;
#pragma unroll
        for (int u = 0; u + 1 < NKEEP; ++u) literal = literal || !(keys_apart(k[u], k[u + 1]) || k[u] == EMPTY);
        int es[4] = {-1, -1, -1, -1};
        float vs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        es[0] = 63 - (k[0] & 63);
        if constexpr (LISTS) {
            // the top-1's list: four keys kept, the three slots and the guard
            const int n = cnt[es[0]];
            const uint16_t *lst = clist + es[0] * 64;
            int m[4] = {EMPTY, EMPTY, EMPTY, EMPTY};
            for (int kq = 0; kq < nmax; kq += 4) {
                const uint2 w = *reinterpret_cast<const uint2 *>(lst + kq);
                uint32_t code[4] = {w.x & 0xffffu, w.x >> 16, w.y & 0xffffu, w.y >> 16};
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = lds_f(lanebase ^ code[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int kk = kq + j < n ? key_of(v[j], (int)(code[j] >> 8)) : EMPTY;
                    const int n0 = key_max(m[0], kk), n1 = key_med3(m[0], m[1], kk), n2 = key_med3(m[1], m[2], kk),
                              n3 = key_med3(m[2], m[3], kk);
                    m[0] = n0;
                    m[1] = n1;
                    m[2] = n2;
                    m[3] = n3;
                }
            }
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                literal = literal || !(keys_apart(m[u], m[u + 1]) || m[u] == EMPTY);
                es[u + 1] = m[u] == EMPTY ? -1 : 63 - (m[u] & 63);
            }
        } else {
#pragma unroll
            for (int u = 1; u < 4; ++u) es[u] = k[u] == EMPTY ? -1 : 63 - (k[u] & 63);
        }
        float gs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float den = 1.0f;
        if (!literal) {
#pragma unroll
            for (int s2 = 1; s2 < 4; ++s2)
                if (s2 >= K) es[s2] = -1;
            if (gates) {  // (uniform)
#pragma unroll
                for (int s2 = 0; s2 < 4; ++s2) vs[s2] = logit_of(es[s2] < 0 ? 0 : es[s2]);
                gs[0] = expf(vs[0] - vs[0]);
                den = gs[0];
#pragma unroll
                for (int s2 = 1; s2 < 4; ++s2)
                    if (s2 < K) {
                        if (es[s2] >= 0) gs[s2] = expf(vs[s2] - vs[0]);
                        den += gs[s2];
                    }
            }
        }
        // The tokens that need the literal scan: a few one after the other, each by the whole wave (lane = column); more, every one
        // by its own lane.
        const bool scan = literal && t < T;
        uint64_t todo = __ballot(scan);
        if (__popcll(todo) * SCAN_TOGETHER > E) {
            todo = 0;
            if (scan)
                literal_scan(
                    [&](uint64_t mm, int &bi, float &bv) __attribute__((always_inline)) {
                        bi = -1;
                        bv = 0.0f;
                        for (int e = 0; e < E; ++e) {
                            const float v = logit_of(e);
                            const bool take = ((mm >> e) & 1ull) != 0 && (bi < 0 || v > bv);
                            bv = take ? v : bv;
                            bi = take ? e : bi;
                        }
                    },
                    K, all, LISTS ? mask_tab : nullptr, es, gs, den);
        }
        for (; todo; todo &= todo - 1) {
            const int tk = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)todo) - 1);
            const float v = lds_f((uint32_t)(wave * TILE_BYTES + tk * 4) ^ code_of(lane < E ? lane : 0));
            int et[4];
            float gt[4], dt;
            literal_scan_by_wave(v, K, all, LISTS ? mask_tab : nullptr, et, gt, dt);
            if (lane == tk) {
                den = dt;
#pragma unroll
                for (int s2 = 0; s2 < 4; ++s2) {
                    es[s2] = et[s2];
                    gs[s2] = gt[s2];
                }
            }
        }
        if (t < T) {
            const bool vec = K == 4 && ((reinterpret_cast<uintptr_t>(topk_idx) | reinterpret_cast<uintptr_t>(gates)) & 15) == 0;
            if (topk_idx) {
                if (vec) {
                    const i32x4 ev = {es[0], es[1], es[2], es[3]};
                    __builtin_nontemporal_store(ev, reinterpret_cast<i32x4 *>(topk_idx + (size_t)t * 4));
                } else {
#pragma unroll
                    for (int s2 = 0; s2 < 4; ++s2)
                        if (s2 < K) topk_idx[(size_t)t * K + s2] = es[s2];
                }
            }
            if (gates) {
#pragma unroll
                for (int s2 = 0; s2 < 4; ++s2) gs[s2] = gs[s2] / den;
                if (vec) {
                    const f32x4 gv = {gs[0], gs[1], gs[2], gs[3]};
                    __builtin_nontemporal_store(gv, reinterpret_cast<f32x4 *>(gates + (size_t)t * 4));
                } else {
#pragma unroll
                    for (int s2 = 0; s2 < 4; ++s2)
                        if (s2 < K) gates[(size_t)t * K + s2] = gs[s2];
                }
            }
            if constexpr (COUNT) {
                // Eq. 2: one count for every pair a <= b of the token's experts, the diagonal included,
                // into the workgroup's histogram (upper triangle)
                uint64_t ma = 0;
#pragma unroll
                for (int s2 = 0; s2 < 4; ++s2)
                    if (es[s2] >= 0) ma |= 1ull << es[s2];
                while (ma) {
                    const int ea = __ffsll((unsigned long long)ma) - 1;
                    uint64_t mb = ma;
                    ma &= ma - 1;
                    while (mb) {
                        const int eb = __ffsll((unsigned long long)mb) - 1;
                        mb &= mb - 1;
                        atomicAdd(&red[ea * C2R_MAX_E + eb], 1);
                    }
                }
            }
        }
        // the next group's logits overwrite the tile: every lane's reads of it come first
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (COUNT) {
        __syncthreads();
        for (int i = tid; i < E * E; i += 256) {
            const int r = i / E, c = i - r * E;
            const int32_t v = red[(r < c ? r : c) * C2R_MAX_E + (r < c ? c : r)];
            if (v) atomicAdd(&Cmat[i], v);
        }
    }
}

// route_select_kernel for batches that its 64-token workgroups would leave most of the chip idle with: sixteen tokens per
// workgroup.  What bounds such a selection is the trip of a workgroup's chunk results - 128 KB for 64 tokens of 60 experts and 8 chunks, at
// the rate one CU pulls from memory - and the length of its scans: a quarter of the one, sixteen lanes per token on the other.
constexpr int SEL16_TOKENS = 16;

__global__ __launch_bounds__(256) void route_select_small_kernel(
    const float *__restrict__ part, int ep, int nchunk, const float *__restrict__ bias, int64_t T, int E, int K,
    const int32_t *__restrict__ collab_idx, int Tc, int32_t *__restrict__ topk_idx, float *__restrict__ gates,
    float *__restrict__ logits_out) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int LP = C2R_MAX_E + 1;
    __shared__ float tile[SEL16_TOKENS * LP];
    __shared__ uint64_t mask_tab[C2R_MAX_E];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * SEL16_TOKENS;
    const uint64_t all = E >= 64 ? ~0ull : ((1ull << E) - 1ull);
    {
        // a thread's share: one expert (its chunk results of four tokens, and a quarter of its list); all loads of the usual sizes in
        // flight together
        const int e = tid >> 2, quad = tid & 3;
        constexpr int AHEAD = 4;
        int32_t listed[AHEAD];
        const int last = E * Tc - 1;
        if (collab_idx) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) listed[u] = collab_idx[min(e * Tc + quad + 4 * u, last)];
        }
        const float *p = part + ((size_t)(t0 >> 6) * nchunk * ep + (e < ep ? e : 0)) * 64 + (t0 & 63) + quad * 4;
        f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int c0 = 0; c0 < nchunk; c0 += 8) {
            f32x4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = *reinterpret_cast<const f32x4 *>(p + (size_t)min(c0 + u, nchunk - 1) * ep * 64);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (c0 + u < nchunk) sum = c0 + u == 0 ? v[u] : sum + v[u];
        }
        if (bias && e < E) sum = sum + bias[e];
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[(quad * 4 + i) * LP + e] = sum[i];
        uint64_t m = collab_idx ? 0ull : all;
        if (collab_idx) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
                if (quad + 4 * u < Tc && listed[u] >= 0 && listed[u] < E) m |= 1ull << listed[u];
            for (int i = quad + 4 * AHEAD; i < Tc; i += 4) {
                const int v = e < E ? collab_idx[e * Tc + i] : -1;
                if (v >= 0 && v < E) m |= 1ull << v;
            }
            m = or_of_lanes<4>(m);
        }
        if (quad == 0) mask_tab[e] = m & ~(1ull << e);
    }
    __syncthreads();
    const int sub = tid & 15;
    const int64_t t = t0 + (tid >> 4);
    if (t >= T) return;  // (the sixteen lanes of a token leave together)
    const float *row = &tile[(tid >> 4) * LP];
    float l[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) l[j] = sub * 4 + j < E ? row[sub * 4 + j] : 0.0f;
    if (logits_out) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (sub * 4 + j < E) logits_out[(size_t)t * E + sub * 4 + j] = l[j];
    }
    int e, mine = -1;  // lane s of a token keeps its slot s (slots past the sixteenth go out at once, unscaled)
    float v, v0 = 0.0f, den = 0.0f, mine_g = 0.0f;
    uint64_t m = all;
    for (int s = 0; s < K; ++s) {
        pick_by_sixteen(l, row, m, sub, e, v);
        float g = 0.0f;
        if (s == 0) {
            v0 = v;
            m = mask_tab[e];
            g = expf(v0 - v0);  // 1, or NaN when the largest logit is infinite or a NaN
        } else if (e >= 0) {
            m &= ~(1ull << e);
            g = expf(v - v0);
        }
        den = s == 0 ? g : den + g;
        if (s == sub) {
            mine = e;
            mine_g = g;
        }
        if (s >= 16 && sub == 0) {
            topk_idx[(size_t)t * K + s] = e;
            gates[(size_t)t * K + s] = g;
        }
    }
    if (sub < K) {
        topk_idx[(size_t)t * K + sub] = mine;
        gates[(size_t)t * K + sub] = mine_g / den;
    }
    if (sub == 0)
        for (int s = 16; s < K; ++s) gates[(size_t)t * K + s] = gates[(size_t)t * K + s] / den;
}

// Selection AND dispatch index of a batch of at most 64 tokens and 1024 assignments, one workgroup: what
// route_select_kernel and permute_by_slot_kernel (permute.hip) do, in one launch instead of two.
// (The smallest batches' gate/up pass does the same at its start, ffn_skinny_few_kernel.)  A launch costs such a batch as much as its
// work: 60 experts, 1 token, 9.3 + 6.4 us in two launches, 6.3 in one.  Sixteen waves, so that the chunk
// results of a whole batch are one load each in flight per thread, and a token has sixteen lanes to scan its experts.
constexpr int FIN_WAVES = 16, FIN_TOKENS = 64, FIN_ASSIGNMENTS = 1024;

__global__ __launch_bounds__(FIN_WAVES * 64) void route_finish_small_kernel(const FewRoute R) {
    __shared__ FewScratch<FIN_WAVES * 64, FIN_ASSIGNMENTS> S;
    int lo, hi;
    route_few<FIN_WAVES * 64>(R, S, true, lo, hi, nullptr);
}

// Selection, dispatch index and row scatter of up to 1024 tokens with few experts, one launch instead of three (route_select_kernel,
// permute_by_slot_kernel, permute_rows_kernel).  Such a batch is launches: its chunk results are a few ten KB.  Every workgroup adds them up
// and selects for all tokens, a thread per token; `parts` workgroups per slot then hand out the slot's rows (the first of them writes
// them) and copy every parts-th of them each.  Microseconds of a layer call, apart / so: 8 experts, d 256, fp32, 512 tokens 34.0 / 30.9, 1000
// tokens 42.1 / 40.6; d 4096, without rows, 8 experts, 70 tokens 73.3 / 71.3, 250 tokens (128 KB) 90.8 / 89.2, 16 experts, 128 tokens (128
// KB) 84.6 / 83.9.
constexpr int SI_THREADS = 1024, SI_PARTS = 8, SI_BYTES = 131072;
static inline bool select_index_takes(int64_t T, int E, int K, int64_t nchunk) {
    return T >= 1 && T <= SI_THREADS && E >= 1 && E <= 16 && K >= 1 && K <= 4 && T * nchunk * ((E + 3) / 4 * 4) * 4 <= SI_BYTES;
}

template <int EP>
__global__ __launch_bounds__(SI_THREADS) void route_select_index_kernel(const FewRoute R, const uint4 *__restrict__ x, int row_vecs,
                                                                        uint4 *__restrict__ x_perm) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int LP = EP + 1, WAVES = SI_THREADS / 64, DEEP = 8;
    __shared__ float tile[SI_THREADS * LP];
    __shared__ uint64_t mask_tab[16];
    __shared__ int32_t slot_tab[16], w_mine[WAVES], w_less[WAVES];
    __shared__ uint16_t token_of[SI_THREADS * 4];  // of the rows of this slot
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = R.T, E = R.E, K = R.K, Tc = R.Tc, E_local = R.E_local, ep = R.ep, nchunk = R.nchunk;
    const int slot_here = blockIdx.x % E_local, part = blockIdx.x / E_local, parts = gridDim.x / E_local;
    const uint64_t all = (1ull << E) - 1ull;

    // ---- logits, four tokens of one expert per thread (chunk results left to right); a wave walks an expert's list ----
    const int32_t listed = R.collab_idx ? R.collab_idx[min(wave * Tc + lane, E * Tc - 1)] : -1;
    int own_slot = tid;
    if (R.local_slot) own_slot = R.local_slot[min(tid, E - 1)];
    const int quads = (T + 3) >> 2;
    for (int i = tid; i < quads * ep; i += SI_THREADS) {
        const int e = i / quads, t4 = (i - e * quads) * 4;
        const float *p = R.part + ((size_t)(t4 >> 6) * nchunk * ep + e) * 64 + (t4 & 63);
        const float bias = R.bias ? R.bias[min(e, E - 1)] : 0.0f;
        f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int c0 = 0; c0 < nchunk; c0 += DEEP) {
            f32x4 v[DEEP];
#pragma unroll
            for (int u = 0; u < DEEP; ++u) v[u] = *reinterpret_cast<const f32x4 *>(p + (size_t)min(c0 + u, nchunk - 1) * ep * 64);
#pragma unroll
            for (int u = 0; u < DEEP; ++u)
                if (c0 + u < nchunk) sum = c0 + u == 0 ? v[u] : sum + v[u];
        }
        if (R.bias && e < E) sum = sum + bias;
#pragma unroll
        for (int j = 0; j < 4; ++j) tile[(t4 + j) * LP + e] = sum[j];
    }
    if (wave < E) {
        uint64_t m = R.collab_idx ? 0ull : all;
        if (R.collab_idx) {
            if (lane < Tc && listed >= 0 && listed < E) m = 1ull << listed;
            for (int i = lane + 64; i < Tc; i += 64) {
                const int v = R.collab_idx[wave * Tc + i];
                if (v >= 0 && v < E) m |= 1ull << v;
            }
            const int row = (int)or_of_lanes<16>(m);  // (E <= 16)
            m = (uint32_t)(__builtin_amdgcn_readlane(row, 0) | __builtin_amdgcn_readlane(row, 16) | __builtin_amdgcn_readlane(row, 32) |
                           __builtin_amdgcn_readlane(row, 48));
        }
        if (lane == 0) mask_tab[wave] = m & ~(1ull << wave);
    }
    if (tid < 16) slot_tab[tid] = tid < E && own_slot >= 0 && own_slot < E_local ? own_slot : -1;
    __syncthreads();

    // ---- selection: see route_select_kernel for the rule ----
    const int t = tid;
    int slots[4];
    int mine = 0, less = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) slots[s] = -1;
    if (t < T) {
        float l[EP];
#pragma unroll
        for (int e = 0; e < EP; ++e) l[e] = e < E ? tile[t * LP + e] : 0.0f;
        int es[4];
        float gs[4], v0 = 0.0f, den = 0.0f;
        uint64_t m = all;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            es[s] = -1;
            gs[s] = 0.0f;
            if (s >= K) continue;
            float v;
            pick<EP>(l, m, es[s], v);
            if (s == 0) {
                v0 = v;
                m = mask_tab[es[0]];
                gs[0] = expf(v0 - v0);  // 1, or NaN when the largest logit is infinite or a NaN
            } else if (es[s] >= 0) {
                m &= ~(1ull << es[s]);
                gs[s] = expf(v - v0);
            }
            den = s == 0 ? gs[0] : den + gs[s];
            slots[s] = es[s] >= 0 ? slot_tab[es[s]] : -1;
            mine += slots[s] == slot_here;
            less += slots[s] >= 0 && slots[s] < slot_here;
        }
        if (blockIdx.x == 0) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (s < K) {
                    R.topk_idx[t * K + s] = es[s];
                    R.gates[t * K + s] = gs[s] / den;
                    if (slots[s] < 0) R.inv_perm[t * K + s] = -1;
                }
        }
    }
    // ---- this slot's rows, in the order of the assignments t * K + s ----
    const int incl = wave_inclusive_scan(mine), incl_less = wave_inclusive_scan(less);
    if (lane == 63) {
        w_mine[wave] = incl;
        w_less[wave] = incl_less;
    }
    __syncthreads();
    int first = 0, total = 0, before = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        first += w_less[w];
        total += w_mine[w];
        before += w < wave ? w_mine[w] : 0;
    }
    int at = before + incl - mine;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (slots[s] == slot_here) {
            token_of[at] = (uint16_t)t;
            if (part == 0) {
                R.perm[first + at] = t * K + s;
                R.inv_perm[t * K + s] = first + at;
            }
            ++at;
        }
    if (tid == 0 && part == 0) {
        R.counts[slot_here] = total;
        R.offsets[slot_here] = first;
        if (slot_here == E_local - 1) R.offsets[E_local] = first + total;
    }
    if (!x_perm) return;
    __syncthreads();
    for (int r = part * WAVES + wave; r < total; r += parts * WAVES) {
        const uint4 *src = x + (size_t)token_of[r] * row_vecs;
        uint4 *dst = x_perm + (size_t)(first + r) * row_vecs;
        for (int v = lane; v < row_vecs; v += 64) dst[v] = src[v];
    }
}

static int check_route_args(int64_t T, int E, int K, const int32_t *collab_idx, int Tc) {
    if (T < 0 || E < 1 || K < 1 || K > E) return C2R_ERR_INVALID_ARG;
    if (collab_idx && Tc < K - 1) return C2R_ERR_INVALID_ARG;
    if (E > C2R_MAX_E) return C2R_ERR_UNSUPPORTED;
    if (T * (int64_t)K >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    return C2R_OK;
}

static inline int ep_of(int E) { return (E + 3) / 4 * 4; }

struct RouteLayout {
    int EP, nchunk;
    int64_t Tpad;
    size_t part_bytes, wpad_bytes;
};

static RouteLayout route_layout(int64_t T, int d, int E) {
    RouteLayout L;
    L.EP = ep_of(E);
    L.nchunk = (d + C2R_CANON_CHUNK - 1) / C2R_CANON_CHUNK;
    if (L.nchunk < 1) L.nchunk = 1;
    L.Tpad = (T + 63) / 64 * 64;
    L.part_bytes = round_up((size_t)L.nchunk * L.EP * (size_t)L.Tpad * sizeof(float), 256);
    L.wpad_bytes = (E % 4) ? round_up((size_t)d * L.EP * sizeof(float), 256) : 0;
    return L;
}

// Whether a batch takes route_partial_small_kernel: up to 6144 waves (16 experts x 16 tokens x one chunk each).  Beyond, every
// workgroup's own copy of its W_g rows is what it spends its time on.  Microseconds of the stage, without / with it:
//   E 60, d 2048: 1 token 21.0 / 12.8, 512 tokens 22.0 / 14.2, 3000 tokens 25.2 / 24.1, 4096 tokens 26.8 / 28.0;
//   E 16, d 4096: 1 token 13.1 / 9.9, 4096 tokens 20.8 / 18.8, 6000 tokens 26.7 / 25.8; E 8, d 4096: 1 token 16.0 / 8.7,
//     4096 tokens 19.4 / 16.6, 6000 tokens 23.3 / 23.9; E 8, d 256: 12.6 / 10.0 at every size up to 12000 tokens.
static inline int route_expert_blocks(int EP) { return EP > 32 ? 4 : EP > 16 ? 2 : 1; }
static inline bool route_small(int64_t T, int nchunk, int EP) {
    return T <= 12288 && (T + 15) / 16 * nchunk * route_expert_blocks(EP) <= 6144;
}

size_t route_workspace_bytes(int64_t T, int d, int E) {
    if (T <= 0 || d <= 0 || E <= 0) return 0;
    RouteLayout L = route_layout(T, d, E);
    return L.part_bytes + L.wpad_bytes;
}

#define C2R_EP_SWITCH(EPV, ...) \
    switch (EPV) {               \
        case 4: { constexpr int EP = 4; __VA_ARGS__; } break;   \
        case 8: { constexpr int EP = 8; __VA_ARGS__; } break;   \
        case 12: { constexpr int EP = 12; __VA_ARGS__; } break; \
        case 16: { constexpr int EP = 16; __VA_ARGS__; } break; \
        case 20: { constexpr int EP = 20; __VA_ARGS__; } break; \
        case 24: { constexpr int EP = 24; __VA_ARGS__; } break; \
        case 28: { constexpr int EP = 28; __VA_ARGS__; } break; \
        case 32: { constexpr int EP = 32; __VA_ARGS__; } break; \
        case 36: { constexpr int EP = 36; __VA_ARGS__; } break; \
        case 40: { constexpr int EP = 40; __VA_ARGS__; } break; \
        case 44: { constexpr int EP = 44; __VA_ARGS__; } break; \
        case 48: { constexpr int EP = 48; __VA_ARGS__; } break; \
        case 52: { constexpr int EP = 52; __VA_ARGS__; } break; \
        case 56: { constexpr int EP = 56; __VA_ARGS__; } break; \
        case 60: { constexpr int EP = 60; __VA_ARGS__; } break; \
        case 64: { constexpr int EP = 64; __VA_ARGS__; } break; \
        default: return C2R_ERR_UNSUPPORTED;             \
    }

}  // namespace c2r

using namespace c2r;

extern "C" int c2r_route_chunk(void) { return C2R_CANON_CHUNK; }

// Selection from chunk results.
static int launch_select(const float *part, int EP_, int nchunk, const float *bias, int64_t T, int E, int K,
                         const int32_t *collab_idx, int Tc, int32_t *topk_idx, float *gates, float *logits_out, hipStream_t st) {
    // Up to 8192 tokens the 64-token workgroups are at most half as many as the CUs; sixteen lanes per token pay with many experts or
    // slots.  Microseconds of the kernel (64 / 16 tokens per workgroup), 60 experts, d 2048: 131 tokens 10.5 / 5.4, 1000 tokens 11.9 / 6.2,
    // 8192 tokens 11.9 / 9.3; of the stage, 32 experts 300 tokens 12 % less, 4096 tokens 1 % more; 16 experts, d 4096, 4096 tokens 17.5 / 18.3, but
    // 16 slots 29 / 27; 8 experts, d 1024, 300 tokens 8.8 / 9.4; 60 experts, 1 slot, 6000 tokens 29.6 / 31.1.  Beyond, with every CU at work, the shorter scans count (the stage, 60
    // experts: 16384 tokens 52.7 / 54.2, 65536 tokens 155 / 157).
    if (T <= (K > 8 ? 8192 : EP_ > 32 ? (K > 2 ? 8192 : 4096) : EP_ > 16 ? 2048 : 0)) {
        route_select_small_kernel<<<dim3((unsigned)((T + SEL16_TOKENS - 1) / SEL16_TOKENS)), dim3(256), 0, st>>>(
            part, EP_, nchunk, bias, T, E, K, collab_idx, Tc, topk_idx, gates, logits_out);
        return launch_status();
    }
    if (nchunk == 1 && K <= 4 && !collab_idx) {
        C2R_EP_SWITCH(EP_, route_select_keys_kernel<EP><<<dim3((unsigned)((T + 63) / 64)), dim3(64), 0, st>>>(part, bias, T, E, K, topk_idx,
                                                                                                            gates, logits_out));
        return launch_status();
    }
    C2R_EP_SWITCH(EP_, route_select_kernel<EP, false><<<dim3((unsigned)((T + 63) / 64)), dim3(SEL_WAVES * 64), 0, st>>>(
                           part, nchunk, bias, T, E, K, collab_idx, Tc, topk_idx, gates, logits_out));
    return launch_status();
}

// What route_finish_small_kernel writes besides the selection.
struct DispatchOut {
    const int32_t *local_slot;
    int E_local;
    int32_t *counts, *offsets, *perm, *inv_perm;
    FewRoute *later;  // not null: the caller's next launch does the work of route_finish_small_kernel, from these arguments
    void *x_perm;     // where route_select_index_kernel scatters the rows, or null
};

// Tokens up to which the waves that have the sums select as well (see the rule): without lists, with nearly as many experts as a wave selects from,
// and with lists where a token's row is short.
constexpr int64_t SELECT_UP_TO = 65536, SELECT_MOST_UP_TO = 131072, SELECT_NARROW_UP_TO = 262144;

static int route_impl(const void *x, c2r_dtype x_dt, const float *Wg, const float *bias, int64_t T, int d, int E, int K,
                      const int32_t *collab_idx, int Tc, int32_t *topk_idx, float *gates, float *logits_out, void *ws,
                      size_t ws_bytes, const DispatchOut *dispatch, void *stream) {
    drop_stale_error();
    int rc = check_route_args(T, E, K, collab_idx, Tc);
    if (rc != C2R_OK) return rc;
    if (d < 1 || (x_dt != C2R_F32 && x_dt != C2R_BF16)) return C2R_ERR_INVALID_ARG;
    if (T == 0) return C2R_OK;
    if (!x || !Wg || !topk_idx || !gates) return C2R_ERR_INVALID_ARG;
    if (d % 8 != 0) return C2R_ERR_UNSUPPORTED;
    if (!aligned(x, 16) || !aligned(Wg, 4)) return C2R_ERR_INVALID_ARG;
    const RouteLayout L = route_layout(T, d, E);
    if (!ws || ws_bytes < L.part_bytes + L.wpad_bytes || !aligned(ws, 256)) return C2R_ERR_WORKSPACE;
    if (Tc == 0) collab_idx = nullptr;  // (K is 1: no list is asked.  The kernels request entries ahead and need one to be there.)
    hipStream_t st = static_cast<hipStream_t>(stream);
    float *part = static_cast<float *>(ws);
    const float *W = Wg;
    int ldw = E;
    if (!L.wpad_bytes && !aligned(Wg, 16)) return C2R_ERR_INVALID_ARG;
    const int64_t ntiles = L.Tpad / 64;
    if (route_small(T, L.nchunk, L.EP)) {
        const int neb = route_expert_blocks(L.EP), tok = 64 / neb;
        const dim3 g((unsigned)((T + tok - 1) / tok * L.nchunk)), b(256);
#define C2R_SMALL_LAUNCH(BF)                                                                               \
    switch (neb) {                                                                                         \
        case 4: route_partial_small_kernel<BF, 4><<<g, b, 0, st>>>(x, Wg, E, L.EP, T, d, L.nchunk, part); break; \
        case 2: route_partial_small_kernel<BF, 2><<<g, b, 0, st>>>(x, Wg, E, L.EP, T, d, L.nchunk, part); break; \
        default: route_partial_small_kernel<BF, 1><<<g, b, 0, st>>>(x, Wg, E, L.EP, T, d, L.nchunk, part);       \
    }
        if (x_dt == C2R_BF16) { C2R_SMALL_LAUNCH(true) } else { C2R_SMALL_LAUNCH(false) }
#undef C2R_SMALL_LAUNCH
        if (dispatch) {
            const FewRoute R = {part, L.EP, L.nchunk, bias, (int)T, E, K, collab_idx, Tc, dispatch->local_slot, dispatch->E_local,
                                topk_idx, gates, dispatch->counts, dispatch->offsets, dispatch->perm, dispatch->inv_perm};
            if (dispatch->later) {
                *dispatch->later = R;
            } else if (T > FIN_TOKENS || dispatch->x_perm) {
                const int row_vecs = d * (x_dt == C2R_BF16 ? 2 : 4) / 16;
                const dim3 gi((unsigned)(dispatch->E_local * (dispatch->x_perm ? SI_PARTS : 1))), bi(SI_THREADS);
                const uint4 *xv = static_cast<const uint4 *>(x);
                uint4 *xp = static_cast<uint4 *>(dispatch->x_perm);
                if (L.EP <= 8)
                    route_select_index_kernel<8><<<gi, bi, 0, st>>>(R, xv, row_vecs, xp);
                else
                    route_select_index_kernel<16><<<gi, bi, 0, st>>>(R, xv, row_vecs, xp);
            } else {
                route_finish_small_kernel<<<dim3(1), dim3(FIN_WAVES * 64), 0, st>>>(R);
            }
            return launch_status();
        }
        return launch_select(part, L.EP, L.nchunk, bias, T, E, K, collab_idx, Tc, topk_idx, gates, logits_out, st);
    }
    if (L.wpad_bytes) {
        float *Wp = reinterpret_cast<float *>(static_cast<char *>(ws) + L.part_bytes);
        const int64_t n = (int64_t)d * L.EP;
        pack_router_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(Wg, d, E, L.EP, Wp);
        W = Wp;
        ldw = L.EP;
    }
    // Four waves per workgroup share the W sub-tiles.  On the matrix pipe a wave tile is always
    // 32 tokens (the pipelined form of the kernel; at E = 60, d = 2048 it beats 64-token tiles
    // at every batch size: 191 vs 238 us for the stage at T = 65536).  On the vector pipe a batch
    // with fewer than two 64-token wave tiles per SIMD of the chip uses half-size wave tiles:
    // with one wave per SIMD nothing hides its latencies.
    const int te = L.EP > 32 ? 8 : L.EP > 16 ? 4 : L.EP > 8 ? 2 : 1;
    const bool wide = ntiles * L.nchunk >= 2048 && te == 1;
    constexpr int NWV = 4;
    const int64_t nwt = wide ? ntiles : ntiles * 2;
    // With about one 32-token wave tile per SIMD of the chip (1024), a workgroup on the matrix pipe walks all the chunks of its tokens
    // and keeps the running sum in registers: scratch then holds ONE vector per token instead of one per chunk.  Smaller
    // batches need the chunks as separate workgroups to fill the chip.  Microseconds of the stage, chunks apart / together: 60 experts,
    // d 2048: 24000 tokens 75 / 85, 26000 tokens 92 / 85.5, 30000 tokens 96 / 86.5; d 4096, 26000 tokens 158 / 156; 16 experts, d 4096: 26000
    // tokens 92 / 103, 30000 tokens 104 / 103.5.
    const bool all_chunks = !wide && te > 1 && nwt >= (te == 8 ? 784 : 1024) && L.nchunk > 1;
    const int nchunk_out = all_chunks ? 1 : L.nchunk;
    // Chunks a workgroup walks otherwise: two with more than 32 experts where that makes a workgroup per CU and the busiest CU has no
    // more chunks for it (E 60, d 2048: 8192 tokens, fp32, 35.2 us with one, 32.9 with two; 16384 tokens 55.2 / 53.0; but 8193 tokens,
    // 260 workgroups of two, 41.8 / 49.0, 20000 tokens 65.1 / 71.2; three or four are never ahead of both by more than 5 %).
    const int64_t ngroups = (nwt + NWV - 1) / NWV, ntwo = ngroups * ((L.nchunk + 1) / 2);
    const bool two = te == 8 && ntwo >= 256 && (ntwo + 255) / 256 * 2 <= (ngroups * L.nchunk + 255) / 256;
    const int cpw = all_chunks ? L.nchunk : two ? 2 : 1;
    // Workgroups of 128 tokens come in rounds of the chip's CUs, and the first batches past a round (or two) leave most of the last one
    // empty: workgroups of 64 tokens, their waves 32 experts each, make it one of half the length.  (33000 tokens 147 / 124 us,
    // 48000 tokens 149 / 126, 72000 tokens 221 / 201, fp32 33000 tokens 152 / 119; full rounds cost 4 to 9 % more that way, x
    // being read by two waves: 32768 tokens 86.5 / 90, 65536 tokens 154 / 167.  Past the third round it is all but even: 106000 tokens
    // 281 / 272, fp32 299 / 298, 140000 tokens 350 / 345, fp32 386 / 387.)
    const int64_t half_rounds = (ngroups + 127) / 128;
    const bool halves = all_chunks && te == 8 && (half_rounds == 3 || half_rounds == 5);
    const SelectArgs sel = {bias, E, K, collab_idx, Tc, topk_idx, gates};
    // The waves that have the sums select as well: the logits go neither out (16 MB at 65536 tokens) nor back, and the selection's launch (10 to
    // 14 us by itself) costs 3 to 5 at the end of this one, whose workgroups all end at once.  Microseconds, in two launches / so: top-K of the
    // profiling call, 60 experts, d 2048: 26000 tokens 98.1 / 94.2, 32768 tokens 99.4 / 94.7, 65536 tokens 166.8 / 161.8, 16 experts of d 4096, 32768
    // tokens 112.6 / 110.6; with lists, the layer call of 15 of 60 experts, 26000 tokens 369 / 362, 32768 tokens 425.5 / 418.  Not with 64-token
    // workgroups, whose waves have half of a token's logits, nor where logits are asked for.
    // Every round of the chip's workgroups (32768 tokens) pays for its selection, at the price of 32 or 64 experts, where one launch for all selects at
    // the memory's pace by what experts there are; from some round on that is ahead.  Microseconds of top-4, in two launches / so, without lists: d 512,
    // 65536 tokens, 9 experts 32.1 / 31.2, 33 experts 49.8 / 47.0, 100000 tokens, 9 experts 51.5 / 54.2, 20 51.1 / 52.2, 33 83.2 / 85.7, 48 82.8 / 83.5, but 32
    // 53.1 / 52.5, 60 84.8 / 83.9; 131072 tokens, 32 experts 56.1 / 54.0, 60 88.6 / 85.2; 400000 tokens, 32 experts 163 / 167, 60 260 / 264; d 2048, 400000
    // tokens, 9 experts 526 / 536.  With lists the other launch costs more: d 512, 400000 tokens, 9 experts 169.7 / 168.6, 60 297 / 281, 10^6 tokens 388 / 386
    // and 699 / 662; but where little is read, d 264, 400000 tokens, 9 experts 110 / 112, 33 178 / 177, 10^6 tokens 262 / 283 and 421 / 437.
    const bool most = E * 8 > (te == 8 ? 64 : 32) * 7;  // of the experts that a wave selects from
    const int64_t select_up_to = collab_idx ? (most || d >= 512 ? T : SELECT_NARROW_UP_TO) : most ? SELECT_MOST_UP_TO : SELECT_UP_TO;
    // (In one launch workgroups write selections while others still read.)
    const size_t a4 = (size_t)(T * K) * 4;
    const bool select = all_chunks && !halves && K <= 4 && !logits_out && T <= select_up_to &&
                        all_apart({{topk_idx, a4}, {gates, a4}}, {{x, (size_t)T * d * (x_dt == C2R_BF16 ? 2 : 4)}, {W, (size_t)d * ldw * 4},
                                                                 {bias, (size_t)E * 4}, {collab_idx, (size_t)E * Tc * 4}});
    const int64_t nblk = ngroups * ((L.nchunk + cpw - 1) / cpw);
    if (nblk >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    // more than 8 experts: the matrix pipe, a wave covering 32 or 64 experts (columns past the packed
    // expert count re-read column 0; their sums are never stored)
#define C2R_ROUTE_LAUNCH(BF, TE, NWV, TQ, MF)                                                     \
    route_partial_kernel<BF, TE, NWV, TQ, MF><<<dim3((unsigned)nblk), dim3(NWV * 64), 0, st>>>(    \
        x, W, ldw, L.EP, T, d, L.nchunk, cpw, ntiles, part, sel)
#define C2R_ROUTE_LAUNCH_ALL(BF, TE, NWV, TQ)                                                          \
    if (select) {                                                                                      \
        route_partial_kernel<BF, TE, NWV, TQ, true, true, false, true><<<dim3((unsigned)nblk), dim3(NWV * 64), 0, st>>>(  \
            x, W, ldw, L.EP, T, d, L.nchunk, cpw, ntiles, part, sel);                                  \
    } else                                                                                             \
    route_partial_kernel<BF, TE, NWV, TQ, true, true><<<dim3((unsigned)nblk), dim3(NWV * 64), 0, st>>>(  \
        x, W, ldw, L.EP, T, d, L.nchunk, cpw, ntiles, part, sel)
#define C2R_ROUTE_LAUNCH_HALVES(BF)                                                                              \
    route_partial_kernel<BF, 8, NWV, 4, true, true, true>                                                          \
        <<<dim3((unsigned)((nwt + NWV / 2 - 1) / (NWV / 2))), dim3(NWV * 64), 0, st>>>(x, W, ldw, L.EP, T, d, L.nchunk, cpw, \
                                                                                       ntiles, part, sel)
#define C2R_ROUTE_TE(BF, NWV, TQ)                                     \
    if (all_chunks) {                                                 \
        if (halves) { C2R_ROUTE_LAUNCH_HALVES(BF); }                  \
        else if (te == 8) { C2R_ROUTE_LAUNCH_ALL(BF, 8, NWV, TQ); }        \
        else { C2R_ROUTE_LAUNCH_ALL(BF, 4, NWV, TQ); }                \
    } else                                                            \
    switch (te) {                                                     \
        case 8: C2R_ROUTE_LAUNCH(BF, 8, NWV, TQ, true); break;        \
        case 4: C2R_ROUTE_LAUNCH(BF, 4, NWV, TQ, true); break;        \
        case 2: C2R_ROUTE_LAUNCH(BF, 4, NWV, TQ, true); break;        \
        default: C2R_ROUTE_LAUNCH(BF, 1, NWV, TQ, false); break;      \
    }
    if (x_dt == C2R_BF16) {
        if (wide) { C2R_ROUTE_LAUNCH(true, 1, NWV, 8, false); } else { C2R_ROUTE_TE(true, NWV, 4) }
    } else {
        if (wide) { C2R_ROUTE_LAUNCH(false, 1, NWV, 8, false); } else { C2R_ROUTE_TE(false, NWV, 4) }
    }
#undef C2R_ROUTE_TE
#undef C2R_ROUTE_LAUNCH_ALL
#undef C2R_ROUTE_LAUNCH_HALVES
#undef C2R_ROUTE_LAUNCH
    if (select) return launch_status();
    return launch_select(part, L.EP, nchunk_out, bias, T, E, K, collab_idx, Tc, topk_idx, gates, logits_out, st);
}

extern "C" int c2r_route(const void *x, c2r_dtype x_dt, const float *Wg, const float *bias,
                         int64_t T, int d, int E, int K, const int32_t *collab_idx, int Tc,
                         int32_t *topk_idx, float *gates, float *logits_out, void *ws,
                         size_t ws_bytes, void *stream) {
    return route_impl(x, x_dt, Wg, bias, T, d, E, K, collab_idx, Tc, topk_idx, gates, logits_out, ws, ws_bytes, nullptr,
                      stream);
}

// Whether a batch's selection and index are route_few's, and whether the gate/up pass may do them (see ffn_few_takes).
static bool route_few_takes(int64_t T, int d, int E, int K) {
    return T >= 1 && T <= FIN_TOKENS && K >= 1 && T * K <= FIN_ASSIGNMENTS && E >= 1 && d >= 1 &&
           route_small(T, (d + C2R_CANON_CHUNK - 1) / C2R_CANON_CHUNK, ep_of(E));
}
bool c2r::route_may_finish_later(int64_t T, int d, int E, int K) { return route_few_takes(T, d, E, K) && T <= FEW_TOKENS && T * K <= FEW_ASSIGNMENTS; }

// c2r_route followed by c2r_permute, for the layer call.
int c2r::route_and_permute(const void *x, c2r_dtype dt, const float *Wg, const float *bias, int64_t T, int d, int E, int K,
                           const int32_t *collab_idx, int Tc, int32_t *topk_idx, float *gates, void *ws_route,
                           size_t ws_route_bytes, const int32_t *local_slot, int E_local, int32_t *counts, int32_t *offsets,
                           int32_t *perm, int32_t *inv_perm, void *x_perm, void *ws_permute, size_t ws_permute_bytes,
                           FewRoute *later, void *stream) {
    int rc;
    const int64_t nchunk = d >= 1 ? ((int64_t)d + C2R_CANON_CHUNK - 1) / C2R_CANON_CHUNK : 1;
    bool with_rows = E >= 1 && route_small(T, (int)nchunk, ep_of(E)) && select_index_takes(T, E, K, nchunk) && (T > FIN_TOKENS || x_perm);
    if (with_rows) {
        // (every workgroup of that launch selects for all tokens, while others write the index and the rows)
        const size_t a4 = (size_t)(T * K) * 4, size = dt == C2R_BF16 ? 2 : 4;
        with_rows = all_apart({{topk_idx, a4}, {gates, a4}, {counts, (size_t)E_local * 4}, {offsets, (size_t)(E_local + 1) * 4}, {perm, a4},
                               {inv_perm, a4}, {x_perm, (size_t)(T * K) * d * size}},
                              {{ws_route, route_workspace_bytes(T, d, E)}, {bias, (size_t)E * 4}, {collab_idx, (size_t)E * Tc * 4},
                               {local_slot, (size_t)E * 4}, {x, (size_t)T * d * size}});
    }
    if (with_rows || route_few_takes(T, d, E, K)) {
        rc = permute_check(x, dt, topk_idx, T, d, E, K, local_slot, E_local, counts, offsets, perm, inv_perm, x_perm,
                           ws_permute, ws_permute_bytes);
        if (rc != C2R_OK) {  // (as ahead of a c2r_permute that fails)
            const int rr = c2r_route(x, dt, Wg, bias, T, d, E, K, collab_idx, Tc, topk_idx, gates, nullptr, ws_route, ws_route_bytes, stream);
            return rr != C2R_OK ? rr : rc;
        }
        const DispatchOut out = {local_slot, E_local, counts, offsets, perm, inv_perm, later, with_rows ? x_perm : nullptr};
        rc = route_impl(x, dt, Wg, bias, T, d, E, K, collab_idx, Tc, topk_idx, gates, nullptr, ws_route, ws_route_bytes, &out,
                        stream);
        if (rc != C2R_OK || !x_perm || with_rows) return rc;
        return permute_rows(x, dt, T, d, K, inv_perm, x_perm, static_cast<hipStream_t>(stream));
    }
    rc = c2r_route(x, dt, Wg, bias, T, d, E, K, collab_idx, Tc, topk_idx, gates, nullptr, ws_route, ws_route_bytes, stream);
    if (rc != C2R_OK) return rc;
    return c2r_permute(x, dt, topk_idx, T, d, E, K, local_slot, E_local, counts, offsets, perm, inv_perm, x_perm, ws_permute,
                       ws_permute_bytes, stream);
}

// Selection from stored logits; with Cmat the tokens' expert pairs are counted as well (then topk_idx
// and gates may be null where the fused kernel runs: E a multiple of 4, K <= 4).
static int route_from_logits_impl(const float *logits, int64_t T, int E, int K, const int32_t *collab_idx, int Tc,
                                  int32_t *topk_idx, float *gates, int32_t *Cmat, hipStream_t st) {
    const int64_t nsel = (T + 63) / 64;
    if (nsel >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    if (E % 4 == 0 && K <= 4) {
        // few, long-lived workgroups: each builds the collaborator lists once and then walks its groups
        // (as many as fit a CU's LDS at once: two with 64-column tiles, four with 32 columns or fewer)
        const int64_t cap = E <= 32 ? 1024 : 512;
        const int64_t nblk = (nsel + 3) / 4 < cap ? (nsel + 3) / 4 : cap;
        const dim3 grid((unsigned)nblk), block(256);
#define C2R_ROWS_ARGS logits, T, E, K, collab_idx, Tc, topk_idx, gates, Cmat, nsel
#define C2R_ROWS_LAUNCH(NVV)                                                               \
    if (Cmat) {                                                                            \
        if (collab_idx)                                                                    \
            route_select_rows_kernel<NVV, true, true><<<grid, block, 0, st>>>(C2R_ROWS_ARGS);   \
        else                                                                               \
            route_select_rows_kernel<NVV, false, true><<<grid, block, 0, st>>>(C2R_ROWS_ARGS);  \
    } else if (collab_idx)                                                                 \
        route_select_rows_kernel<NVV, true, false><<<grid, block, 0, st>>>(C2R_ROWS_ARGS);      \
    else                                                                                   \
        route_select_rows_kernel<NVV, false, false><<<grid, block, 0, st>>>(C2R_ROWS_ARGS)
        switch ((E + 15) / 16) {
            case 1: C2R_ROWS_LAUNCH(1); break;
            case 2: C2R_ROWS_LAUNCH(2); break;
            case 3: C2R_ROWS_LAUNCH(3); break;
            default: C2R_ROWS_LAUNCH(4); break;
        }
#undef C2R_ROWS_LAUNCH
#undef C2R_ROWS_ARGS
        return launch_status();
    }
    if (!topk_idx || !gates) return C2R_ERR_UNSUPPORTED;
    const int EPV = ep_of(E);
    C2R_EP_SWITCH(EPV, route_select_kernel<EP, true><<<dim3((unsigned)nsel), dim3(64), 0, st>>>(
                           logits, 1, (const float *)nullptr, T, E, K, collab_idx, Tc, topk_idx, gates,
                           (float *)nullptr));
    const int rc = launch_status();
    if (rc != C2R_OK || !Cmat) return rc;
    return c2r_build_coactivation(topk_idx, T, K, E, Cmat, st);
}

extern "C" int c2r_route_from_logits(const float *logits, int64_t T, int E, int K,
                                     const int32_t *collab_idx, int Tc, int32_t *topk_idx,
                                     float *gates, void *stream) {
    drop_stale_error();
    int rc = check_route_args(T, E, K, collab_idx, Tc);
    if (rc != C2R_OK) return rc;
    if (T == 0) return C2R_OK;
    if (!logits || !topk_idx || !gates) return C2R_ERR_INVALID_ARG;
    if (!aligned(logits, 16)) return C2R_ERR_INVALID_ARG;
    return route_from_logits_impl(logits, T, E, K, collab_idx, Tc, topk_idx, gates, nullptr,
                                  static_cast<hipStream_t>(stream));
}

extern "C" int c2r_profile_from_logits(const float *logits, int64_t T, int E, int K,
                                       const int32_t *collab_idx, int Tc, int32_t *topk_idx,
                                       float *gates, int32_t *C, void *stream) {
    drop_stale_error();
    int rc = check_route_args(T, E, K, collab_idx, Tc);
    if (rc != C2R_OK) return rc;
    if (T == 0) return C2R_OK;
    if (!logits || !C) return C2R_ERR_INVALID_ARG;
    if (!aligned(logits, 16) || !aligned(C, 4)) return C2R_ERR_INVALID_ARG;
    if (topk_idx && !aligned(topk_idx, 4)) return C2R_ERR_INVALID_ARG;
    return route_from_logits_impl(logits, T, E, K, collab_idx, Tc, topk_idx, gates, C,
                                  static_cast<hipStream_t>(stream));
}
