// Grouped SwiGLU expert FFN in bf16 for batches of few rows (decoding, small serving batches).
//
// Such a pass is bound by streaming the weights: an expert's 17 MB meet a handful of rows.  The tile kernel of
// ffn_bf16_dma.hip hands out 256 weight rows at a time to one CU, so only as many CUs work as there are tiles (8 of 256
// in the down pass of a shared expert with d = 2048, each walking 88 k-slices alone), and one CU pulls at most 44 GB/s of
// cold data.  Here the unit of work is narrow: a workgroup of four waves owns 16 or 32 output columns (with the matching
// gate and up rows in pass 0) for up to 64 rows of one group, and its four waves split the CONTRACTION range, so that a
// launch has thousands of waves whatever the number of groups.  Every weight is used by exactly one wave, so weights go
// from memory straight into the matrix-operand registers (16 weight rows x 64 bytes per load, the two halves of a
// 128-byte line back to back); the few activation rows come the same way out of L2.  No LDS and no barrier until the
// end, where the waves' fp32 partial sums meet in LDS and are added in a fixed order.
//
// Measured in a replayed graph, weights cold, microseconds of the two passes (tile kernel -> this one); in brackets what
// the weights in use take at the 6.2 TB/s that a plain read of them reaches:
//   60 experts + shared (d 2048, F 1408 / 5632, top-4): 1 token 29.5 + 48.6 -> 18.6 + 12.2 (15 + 7), down pass of 16 tokens
//     75.4 -> 29.2 (18); 16 experts (d 4096, F 688, top-4), both passes: 1 token 54.0 -> 19.3.
// Also measured: eight waves per workgroup (a longer reduction, 10-30 % slower but for a single token), weights loaded
// past the caches (8-12 % slower: the second half of each line is fetched again), a software-pipelined ring instead of
// bursts (its remainders cost registers and spills; the CU's other waves fill the gaps between bursts anyway).
//
// The order of summation depends on the contraction length alone (not on the group sizes or the launch), so every entry
// point that computes a row with this kernel computes the same bits.
#include <type_traits>

#include "ffn_common.h"

namespace c2r {

// Three waves per SIMD: the registers left for fragments and, from them, the 64-wide k-units of a burst.
constexpr int SKINNY_WAVES_PER_SIMD = 3, SKINNY_FRAG_VGPRS = 136;
constexpr int skinny_depth(int mf, int nb) {
    const int d = (SKINNY_FRAG_VGPRS - 4 * mf * nb) / (8 * (mf + nb));
    return d > 8 ? 8 : d;
}

// f(integral_constant<n>) for the one n in 1..MAX that equals the (wave-uniform) count.  The markers keep the compiler
// from merging what the bodies have in common ahead of the branches, which costs it all its registers.
template <int MAX, class F>
__device__ __forceinline__ void static_for_count(int count, F &&f) {
    if constexpr (MAX > 0) {
        if (count == MAX) {
            asm volatile("; burst of %0" ::"n"(MAX));
            f(std::integral_constant<int, MAX>{});
            asm volatile("; end of burst of %0" ::"n"(MAX));
        } else {
            static_for_count<MAX - 1>(count, f);
        }
    }
}

// One item.  MF: 16-row fragments of activations, NF: 16-column blocks of the output.
// Contract as in ffn_bf16_dma.hip: A is zero-padded along k to a multiple of 64 (lda >= 64 * ceil(K / 64)); a weight
// chunk past K is re-read from the row's last chunk and multiplied by those zeros.
template <int MODE, int MF, int NF>
__device__ __forceinline__ void skinny_tile(const FfnProblem &P, unsigned char *smem, int expert, int row_begin, int rows,
                                            int n0) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int NB = MODE == 0 ? 2 * NF : NF;  // weight fragments: gate and up rows of the same columns, or down rows
    constexpr int D = skinny_depth(MF, NB);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & 15, fq = lane >> 4;
    const int N = P.N, Kdim = P.Kdim, lda = P.lda;

    // this lane's activation rows and weight rows, as byte offsets from wave-uniform bases
    const unsigned char *baseA = reinterpret_cast<const unsigned char *>(P.gather ? P.A : P.A + (size_t)row_begin * lda);
    const unsigned char *base0 = reinterpret_cast<const unsigned char *>(P.B0 + (size_t)expert * N * Kdim);
    const unsigned char *base1 = MODE == 0 ? reinterpret_cast<const unsigned char *>(P.B1 + (size_t)expert * N * Kdim) : base0;
    uint32_t offA[MF], offB[NF];
    int ra[MF];
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int r = i * 16 + fr;
        ra[i] = r < rows ? r : rows - 1;
    }
    if (P.gather) {
#pragma unroll
        for (int i = 0; i < MF; ++i) ra[i] = P.gather[row_begin + ra[i]];
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const int r = ra[i] > 0 ? (int)((uint32_t)ra[i] / (uint32_t)P.gather_div) : 0;
            ra[i] = r < P.gather_rows ? r : P.gather_rows - 1;  // an out-of-range entry cannot leave A
        }
    }
#pragma unroll
    for (int i = 0; i < MF; ++i) offA[i] = (uint32_t)ra[i] * (uint32_t)lda * 2u + (uint32_t)fq * 16u;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int c = n0 + j * 16 + fr;
        offB[j] = (uint32_t)(c < N ? c : N - 1) * (uint32_t)Kdim * 2u;
    }

    const int nu = (Kdim + 63) / 64;  // 64-wide k-units; this wave takes [u0, u1)
    const int u0 = wave * nu / 4, u1 = (wave + 1) * nu / 4;
    // Byte position of this lane's chunk of half h inside a unit; in the last unit of a contraction length that is no
    // multiple of 64 the chunks past its end become the row's last one.
    const bool ktail = MODE == 1 && (Kdim & 63) != 0;
    uint32_t pos[2], pos_last[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t end = (uint32_t)Kdim * 2u - 16u - (uint32_t)(nu - 1) * 128u;  // of the row's last chunk, >= 0
        pos[h] = (uint32_t)(h * 64 + fq * 16);
        pos_last[h] = pos[h] < end ? pos[h] : end;
    }
    bf16x8 a[D][2][MF], b[D][2][NB];
    auto load_b = [&](int s, int u) __attribute__((always_inline)) {
        const unsigned char *g0 = base0 + (size_t)(uint32_t)u * 128u, *g1 = base1 + (size_t)(uint32_t)u * 128u;
        const bool last = ktail && u == nu - 1;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const uint32_t o = offB[j] + (last ? pos_last[h] : pos[h]);
                b[s][h][j] = *reinterpret_cast<const bf16x8 *>(g0 + o);
                if (MODE == 0) b[s][h][NF + j] = *reinterpret_cast<const bf16x8 *>(g1 + o);
            }
    };
    auto load_a = [&](int s, int u) __attribute__((always_inline)) {
        const unsigned char *ga = baseA + (size_t)(uint32_t)u * 128u;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < MF; ++i) a[s][h][i] = *reinterpret_cast<const bf16x8 *>(ga + offA[i] + h * 64);
    };
    f32x4 acc[MF][NB];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // (operands swapped: a lane's four results are consecutive columns of one row)
    auto mma = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[s][h][j], a[s][h][i], acc[i][j], 0, 0, 0);
    };
    // Bursts of up to D units: all of a burst's loads are in flight together, and the other waves of the CU fill the
    // gap between two bursts.  (No load is redundant: every burst length has code of its own.)
    for (int u = u0; u < u1; u += D) {
        static_for_count<D>(u1 - u < D ? u1 - u : D, [&](auto count) __attribute__((always_inline)) {
            // (weights first: they do not wait for the gather's row numbers)
#pragma unroll
            for (int s = 0; s < count.value; ++s) load_b(s, u + s);
#pragma unroll
            for (int s = 0; s < count.value; ++s) load_a(s, u + s);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < count.value; ++s) mma(s);
        });
    }

    // ---- the waves' partial sums: the upper half of the waves hands its sums to the lower half, and what is left
    // is added up pairwise by all of them, wave w finishing the fragment pairs w, w + 4, ...
    constexpr bool FLAT = MF * NB <= 8;
    constexpr int NH = 2;
    f32x4 *red = reinterpret_cast<f32x4 *>(smem);
    if (FLAT) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) red[((wave * MF + i) * NB + j) * 64 + lane] = acc[i][j];
        __syncthreads();
    } else {
        const int mine = (wave & (NH - 1)) * (MF * NB) * 64 + lane;
        if (wave >= NH) {
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) red[mine + (i * NB + j) * 64] = acc[i][j];
        }
        __syncthreads();
        if (wave < NH) {
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) red[mine + (i * NB + j) * 64] = acc[i][j] + red[mine + (i * NB + j) * 64];
        }
        __syncthreads();
    }
    uint16_t *out = P.out + (size_t)row_begin * P.ldo;
    auto total = [&](int i, int j) __attribute__((always_inline)) {
        const f32x4 *q = red + (i * NB + j) * 64 + lane;
        constexpr int S = MF * NB * 64;
        if constexpr (!FLAT) return q[0] + q[S];
        else return (q[0] + q[2 * S]) + (q[S] + q[3 * S]);
    };
    for (int p = wave; p < MF * NF; p += 4) {
        const int i = p / NF, j = p % NF;
        const int r = i * 16 + fr, col = n0 + j * 16 + fq * 4;
        f32x4 v = total(i, j);
        if (MODE == 0) {
            const f32x4 up = total(i, NF + j);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = silu_mul(v[e], up[e]);
        }
        if (r >= rows) continue;
        uint2 pk = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        if (col >= N) {  // pass 0 keeps the padding columns of h at zero for pass 1's k tail
            if (col >= P.zero_to) continue;
            pk = make_uint2(0, 0);
        }
        *reinterpret_cast<uint2 *>(out + (size_t)r * P.ldo + col) = pk;
    }
}

// M-chunks of 64 rows; an item = (chunk, block of 16 * NF columns), NF = NFR for the ragged problem and NFS for the single
// group.  Every XCD gets an equal share of the single group's items and of the ragged problem's, chunks of one column
// block next to each other (they share its weights in that XCD's L2), the single group's (the longest contraction) first.
constexpr int SKINNY_BM = 64, SKINNY_GATE_UP_ROWS = 32;

template <int MODE, int NF>
__device__ __forceinline__ void skinny_rows(const FfnProblem &P, unsigned char *smem, int expert, int row_begin, int rows,
                                            int n0) {
    if (rows <= 16)
        skinny_tile<MODE, 1, NF>(P, smem, expert, row_begin, rows, n0);
    else if (MODE == 0 || rows <= 32)  // (the gate/up pass takes no more than 32 rows)
        skinny_tile<MODE, 2, NF>(P, smem, expert, row_begin, rows, n0);
    else
        skinny_tile<MODE, 4, NF>(P, smem, expert, row_begin, rows, n0);
}

constexpr int skinny_red_bytes(int mode, int nf) {  // what the reduction of the largest tile takes
    const int frags = mode == 0 ? 2 * 2 * nf : 4 * nf;
    return (frags <= 8 ? 4 * frags : 2 * frags) * 1024;
}

template <int MODE, int NFR, int NFS>
__global__ __launch_bounds__(256, SKINNY_WAVES_PER_SIMD) void ffn_skinny_kernel(const FfnLaunch L) {
    constexpr int BM = SKINNY_BM, BYTES_R = skinny_red_bytes(MODE, NFR), BYTES_S = skinny_red_bytes(MODE, NFS);
    __shared__ __attribute__((aligned(16))) unsigned char smem[BYTES_R > BYTES_S ? BYTES_R : BYTES_S];
    const int xcd = blockIdx.x & 7;
    int slot = blockIdx.x >> 3;
    if (L.has_single) {
        const FfnProblem &P = L.p[1];
        int lo = P.offsets ? P.offsets[0] : P.row_lo, hi = P.offsets ? P.offsets[1] : P.row_hi;
        lo = lo < 0 ? 0 : (lo > P.A_cap ? P.A_cap : lo);
        hi = hi < lo ? lo : (hi > P.A_cap ? P.A_cap : hi);
        const int chunks = (hi - lo + BM - 1) / BM;
        const XcdRange r = equal_range(chunks * P.ntn, xcd);
        if (slot < r.cnt) {
            const int item = r.first + slot, row_begin = lo + item % chunks * BM;
            const int rows = hi - row_begin < BM ? hi - row_begin : BM;
            skinny_rows<MODE, NFS>(P, smem, 0, row_begin, rows, item / chunks * (16 * NFS));
            return;
        }
        slot -= r.cnt;
    }
    if (!L.has_ragged) return;
    const FfnProblem &P = L.p[0];
    const GroupMap gm = build_group_map<BM>(P.offsets, P.E_local, P.A_cap);
    const XcdRange r = equal_range(__builtin_amdgcn_readfirstlane(gm.total_mtiles) * P.ntn, xcd);
    if (slot >= r.cnt) return;
    const int item = r.first + slot;
    // the group whose items hold this number; inside a group its chunks are numbered fastest
    const uint64_t hit = __ballot(item >= gm.first * P.ntn && item < (gm.first + gm.tiles) * P.ntn);
    if (hit == 0) return;
    const int expert = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)hit) - 1);
    const int chunks = __builtin_amdgcn_readlane(gm.tiles, expert);
    const int local = item - __builtin_amdgcn_readlane(gm.first, expert) * P.ntn;
    const int row_begin = __builtin_amdgcn_readlane(gm.lo, expert) + local % chunks * BM;
    const int left = __builtin_amdgcn_readlane(gm.hi, expert) - row_begin;
    skinny_rows<MODE, NFR>(P, smem, expert, row_begin, left < BM ? left : BM, local / chunks * (16 * NFR));
}

template <int MODE, int NFR, int NFS>
static void skinny_launch(FfnLaunch L, hipStream_t st) {
    int64_t per_xcd = 0;
    for (int q = 0; q < 2; ++q) {
        FfnProblem &P = L.p[q];
        const int cols = P.zero_to > P.N ? P.zero_to : P.N, bn = 16 * (q == 0 ? NFR : NFS);
        P.ntn = (cols + bn - 1) / bn;
        if (!(q == 0 ? L.has_ragged : L.has_single)) continue;
        // chunks: one per 64 rows, and one more for every group that can hold a row
        const int64_t groups = P.E_local < P.A_cap ? P.E_local : P.A_cap;
        per_xcd += ((P.A_cap / SKINNY_BM + groups) * P.ntn + 7) / 8;
    }
    ffn_skinny_kernel<MODE, NFR, NFS><<<dim3((unsigned)(per_xcd * 8)), dim3(256), 0, st>>>(L);
}

// Up to this many rows a problem takes this kernel; beyond, ffn_mid.hip.  Microseconds of a layer call with this kernel /
// with that one in the pass:
//   gate/up: 60 experts + shared: 1 token 44.7 / 45.5, 4 tokens 59.9 / 65.0, 8 tokens 76.8 / 78.6, 16 tokens 91 / 86.6, 24 tokens
//     105.5 / 96.4; 16 experts of d 4096: 8 tokens 63.2 / 63.5, 16 tokens 66 / 63.7, 40 tokens 71.9 / 66.1; 8 experts: 8
//     tokens 72.8 / 69.3.
//   down (narrower workgroups, so the longest contraction is cut finer here): 60 experts + shared: 16 tokens 121.7 / 138.1,
//     32 tokens 142.8 / 158.1, 48 tokens 162.2 / 155.1; 16 experts: 40 tokens 80.7 / 81.0, 100 tokens 96.8 / 94.0.
// (At four experts per token both rules cut the routed groups and a shared expert at the same batch.)
bool ffn_skinny_takes(int pass, const FfnProblem &P) {
    if (pass == 1) return P.A_cap <= (P.E_local == 1 ? 40 : 160);
    return P.A_cap <= (P.E_local == 1 ? 8 : (2 * P.E_local < SKINNY_GATE_UP_ROWS ? 2 * P.E_local : SKINNY_GATE_UP_ROWS));
}

int launch_ffn_skinny(int pass, const FfnLaunch &L, hipStream_t st) {
    drop_stale_error();
    // Column blocks.  Wider ones read the activations less often, narrower ones are more numerous: 16 in the gate/up pass (a
    // layer call of 4 / 8 / 16 tokens: 62.2 / 80.0 / 93.0 us, with 32 columns 71.4 / 83.3 / 96.2).  The down pass takes 32
    // for the routed groups (16 tokens: 91.2 us, with 16 columns 93.8) and 16 for the single group, whose contraction is
    // the longest: its workgroups are the last to finish (1 token, the pass: 12.3 against 17.0 us).
    if (pass == 1)
        skinny_launch<1, 2, 1>(L, st);
    else
        skinny_launch<0, 1, 1>(L, st);
    return launch_status();
}

}  // namespace c2r
