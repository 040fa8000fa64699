// Grouped SwiGLU expert FFN in bf16 for batches of few rows (decoding, small serving batches).
//
// Such a pass is bound by streaming the weights: an expert's 17 MB meet a handful of rows.  The tile kernel of
// ffn_bf16_dma.hip hands out 256 weight rows at a time to one CU, so only as many CUs work as there are tiles (8 of 256
// in the down pass of a shared expert with d = 2048, each walking 88 k-slices alone), and one CU pulls at most 44 GB/s of
// cold data.  Here the unit of work is narrow: a workgroup of four waves owns 16 or 32 output columns (with the matching
// gate and up rows in pass 0) for up to 64 rows of one group, and its four waves take the CONTRACTION range in turns, so
// that a launch has thousands of waves with loads in flight whatever the number of groups.  Every weight is used by exactly
// one wave, so weights go from memory straight into the matrix-operand registers (16 weight rows x 64 bytes per load, the two
// halves of a 128-byte line back to back); the few activation rows come the same way out of L2.
//
// Every output is one chain of v_mfma_f32_16x16x32_bf16 over ascending k, as in ffn_bf16_dma.hip and ffn_mid.hip: a row's
// bits are the same at every batch size and through every entry point.  Only the loads are parallel; the waves pass the sums
// on through LDS, each adding the k range that it has loaded.
//
// Measured, microseconds of gate/up + down in a kernel trace, three layers of weights in turn (tile kernel -> this one): 60
// experts + shared (d 2048, F 1408 / 5632, top-4): 1 token 33.3 + 64.8 -> 22.9 + 12.8, down pass of 16 tokens 76.0 -> 27.3; 16 experts
// (d 4096, F 688, top-4): 1 token 41.3 + 17.7 -> 18.0 + 7.4.  A partial sum per wave, added at the end (another order of
// summation), took 21.3 + 14.5, 30.4 and 14.6 + 6.0.
#include <type_traits>

#include "ffn_common.h"
#include "ffn_copy.h"
#include "route_few.h"

namespace c2r {

// WPS: waves per SIMD.  It fixes the registers left for fragments and, from them, the 64-wide k-units of a burst.
constexpr int skinny_depth(int wps, int mf, int nb) {
    const int d = ((wps == 4 ? 100 : 136) - 4 * mf * nb) / (8 * (mf + nb));
    return d > 8 ? 8 : d;
}

// f(integral_constant<n>) for the one n in 1..MAX that equals the (wave-uniform) count.  The markers keep the compiler
// from merging what the bodies have in common ahead of the branches, which costs it all its registers.
template <int MAX, class F>
__device__ __forceinline__ void static_for_count(int count, F &&f) {
    if constexpr (MAX > 0) {
        if (count == MAX) {
            asm volatile("; bursts of %0" ::"n"(MAX));
            f(std::integral_constant<int, MAX>{});
            asm volatile("; end of bursts of %0" ::"n"(MAX));
        } else {
            static_for_count<MAX - 1>(count, f);
        }
    }
}

// One item.  MF: 16-row fragments of activations, NF: 16-column blocks of the output.
// Contract as in ffn_bf16_dma.hip: A is zero-padded along k to a multiple of 64 (lda >= 64 * ceil(K / 64)); a weight
// chunk past K is taken from the start of its row and multiplied by those zeros.
template <int MODE, int WPS, int MF, int NF>
__device__ __forceinline__ void skinny_tile(const FfnProblem &P, unsigned char *smem, int expert, int row_begin, int rows,
                                            int n0, const uint16_t *row_of) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int NB = MODE == 0 ? 2 * NF : NF;  // weight fragments: gate and up rows of the same columns, or down rows
    constexpr int D = skinny_depth(WPS, MF, NB);
    static_assert(D >= 1, "a burst holds at least one unit");
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
    if (row_of) {  // (LDS: the source row of every sorted row)
#pragma unroll
        for (int i = 0; i < MF; ++i) ra[i] = row_of[row_begin + ra[i]];
    } else if (P.gather) {
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

    const int nu = (Kdim + 63) / 64;  // 64-wide k-units
    // In the last unit of a contraction length that is no multiple of 64 a lane's chunk past the end becomes the row's first.
    const bool ktail = MODE == 1 && (Kdim & 63) != 0;
    const uint32_t chunk = (uint32_t)(fq * 16);
    f32x4 acc[MF][NB];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // Bursts of equally many units, at most D, burst j by wave j % 4: its loads are all in flight together while the bursts
    // before it are added, and the sums go from wave to wave through LDS, so that every output is one chain over ascending
    // k.  (The depth is a constant of the code, and every load unconditional - past the last unit that one again: behind
    // a branch the compiler waits for one unit's loads before it requests the next.)
    const int bursts = max(min(4, nu), (nu + D - 1) / D), depth = (nu + bursts - 1) / bursts, nburst = (nu + depth - 1) / depth;
    f32x4 *red = reinterpret_cast<f32x4 *>(smem) + lane;
    static_for_count<D>(depth, [&](auto depth_c) __attribute__((always_inline)) {
        constexpr int DEPTH = decltype(depth_c)::value;
        bf16x8 a[DEPTH][2][MF], b[DEPTH][2][NB];
        auto load_b = [&](int s, int u) __attribute__((always_inline)) {
            const bool last = ktail && u == nu - 1;
            const uint32_t ub = (uint32_t)u * 128u;
            const unsigned char *g0 = base0 + (size_t)(last ? 0u : ub), *g1 = base1 + (size_t)(last ? 0u : ub);
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                uint32_t row = offB[j];
                asm volatile("" : "+v"(row));  // (keeps the widening of the offset next to the load: scalar base + 32 bits)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t at = ub + h * 64 + chunk;  // (from the start of the row)
                    const uint32_t o = row + (last ? (at < (uint32_t)Kdim * 2u ? at : 0u) : h * 64 + chunk);
                    b[s][h][j] = *reinterpret_cast<const bf16x8 *>(g0 + o);
                    if (MODE == 0) b[s][h][NF + j] = *reinterpret_cast<const bf16x8 *>(g1 + o);
                }
            }
        };
        auto load_a = [&](int s, int u) __attribute__((always_inline)) {
            const unsigned char *ga = baseA + (size_t)(uint32_t)u * 128u;
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                uint32_t o = offA[i];
                asm volatile("" : "+v"(o));
#pragma unroll
                for (int h = 0; h < 2; ++h) a[s][h][i] = *reinterpret_cast<const bf16x8 *>(ga + o + h * 64);
            }
        };
        auto load = [&](int j) __attribute__((always_inline)) {
            // (weights first: they do not wait for the gather's row numbers)
#pragma unroll
            for (int s = 0; s < DEPTH; ++s) load_b(s, min(j * DEPTH + s, nu - 1));
#pragma unroll
            for (int s = 0; s < DEPTH; ++s) load_a(s, min(j * DEPTH + s, nu - 1));
        };
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
        if (wave < nburst) load(wave);
        int step = 0;  // bursts that are in the sums
        for (int j = wave; j < nburst; j += 4) {
            for (; step < j; ++step) lds_hand_over();
            if (j > 0) {
#pragma unroll
                for (int i = 0; i < MF; ++i)
#pragma unroll
                    for (int k = 0; k < NB; ++k) acc[i][k] = red[(i * NB + k) * 64];
            }
#pragma unroll
            for (int s = 0; s < DEPTH; ++s)
                if (s == 0 || j * DEPTH + s < nu) mma(s);
            if (j + 1 == nburst) break;
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int k = 0; k < NB; ++k) red[(i * NB + k) * 64] = acc[i][k];
            lds_hand_over();
            ++step;
            if (j + 4 < nburst) load(j + 4);
        }
        for (; step < nburst - 1; ++step) lds_hand_over();
    });
    if (wave != ((nburst - 1) & 3)) return;

    uint16_t *out = P.out + (size_t)row_begin * P.ldo;
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int r = i * 16 + fr;
        if (r >= rows) continue;
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int col = n0 + j * 16 + fq * 4;
            f32x4 v = acc[i][j];
            if (MODE == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = silu_mul(v[e], acc[i][MODE == 0 ? NF + j : j][e]);
            }
            uint2 pk = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
            if (col >= N) {  // pass 0 keeps the padding columns of h at zero for pass 1's k tail
                if (col >= P.zero_to) continue;
                pk = make_uint2(0, 0);
            }
            *reinterpret_cast<uint2 *>(out + (size_t)r * P.ldo + col) = pk;
        }
    }
}

// M-chunks of 64 rows; an item = (chunk, block of 16 * NF columns), NF = NFR for the ragged problem and NFS for the single
// group.  Every XCD gets an equal share of the single group's items and of the ragged problem's, chunks of one column
// block next to each other (they share its weights in that XCD's L2), the single group's (the longest contraction) first.
constexpr int SKINNY_BM = 64;

template <int MODE, int WPS, int NF>
__device__ __forceinline__ void skinny_rows(const FfnProblem &P, unsigned char *smem, int expert, int row_begin, int rows,
                                            int n0, const uint16_t *row_of) {
    if (rows <= 16)
        skinny_tile<MODE, WPS, 1, NF>(P, smem, expert, row_begin, rows, n0, row_of);
    else if (MODE == 0 || rows <= 32)  // (the gate/up pass takes no more than 32 rows)
        skinny_tile<MODE, WPS, 2, NF>(P, smem, expert, row_begin, rows, n0, row_of);
    else
        skinny_tile<MODE, WPS, 4, NF>(P, smem, expert, row_begin, rows, n0, row_of);
}

constexpr int skinny_lds_bytes(int mode, int nf) { return (mode == 0 ? 2 * 2 * nf : 4 * nf) * 1024; }  // the sums of the largest tile

// FEW: the routed groups are not there yet; their workgroups find them out, each for itself, and one more writes them to memory.
template <int MODE, int WPS, int NFR, int NFS, bool FEW>
__device__ __forceinline__ void skinny_item(const FfnLaunch &L, const FewRoute *R, unsigned char *smem) {
    constexpr int BM = SKINNY_BM;
    const int xcd = blockIdx.x & 7;
    int slot = blockIdx.x >> 3;
    const bool writer = FEW && blockIdx.x == gridDim.x - 1;
    if (L.has_single && !writer) {
        const FfnProblem &P = L.p[1];
        int lo = P.offsets ? P.offsets[0] : P.row_lo, hi = P.offsets ? P.offsets[1] : P.row_hi;
        lo = lo < 0 ? 0 : (lo > P.A_cap ? P.A_cap : lo);
        hi = hi < lo ? lo : (hi > P.A_cap ? P.A_cap : hi);
        const int chunks = (hi - lo + BM - 1) / BM;
        const XcdRange r = equal_range(chunks * P.ntn, xcd);
        if (slot < r.cnt) {
            const int item = r.first + slot, row_begin = lo + item % chunks * BM;
            const int rows = hi - row_begin < BM ? hi - row_begin : BM;
            skinny_rows<MODE, WPS, NFS>(P, smem, 0, row_begin, rows, item / chunks * (16 * NFS), nullptr);
            return;
        }
        slot -= r.cnt;
    }
    if (!L.has_ragged) return;
    const FfnProblem &P = L.p[0];
    GroupMap gm;
    const uint16_t *row_of = nullptr;
    if constexpr (FEW) {
        __shared__ FewScratch<256, FEW_ASSIGNMENTS> S;
        __shared__ uint16_t rows[FEW_ASSIGNMENTS];
        int lo, hi;
        route_few<256>(*R, S, writer, lo, hi, rows);
        if (writer) return;
        __syncthreads();
        gm = group_map_of<BM>(lo, hi);
        row_of = rows;
    } else {
        gm = build_group_map<BM>(P.offsets, P.E_local, P.A_cap);
    }
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
    skinny_rows<MODE, WPS, NFR>(P, smem, expert, row_begin, left < BM ? left : BM, local / chunks * (16 * NFR), row_of);
}

constexpr int skinny_smem_bytes(int mode, int nfr, int nfs) {
    return skinny_lds_bytes(mode, nfr) > skinny_lds_bytes(mode, nfs) ? skinny_lds_bytes(mode, nfr) : skinny_lds_bytes(mode, nfs);
}

template <int MODE, int WPS, int NFR, int NFS>
__global__ __launch_bounds__(256, WPS) void ffn_skinny_kernel(const FfnLaunch L) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[skinny_smem_bytes(MODE, NFR, NFS)];
    skinny_item<MODE, WPS, NFR, NFS, false>(L, nullptr, smem);
}

template <int WPS, int NFR, int NFS>
__global__ __launch_bounds__(256, WPS) void ffn_skinny_few_kernel(const FfnLaunch L, const FewRoute R) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[skinny_smem_bytes(0, NFR, NFS)];
    skinny_item<0, WPS, NFR, NFS, true>(L, &R, smem);
}

// Sets the column blocks of the launch's problems; its workgroups per XCD.
template <int NFR, int NFS>
static int64_t skinny_blocks(FfnLaunch &L) {
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
    return per_xcd;
}

template <int MODE, int WPS, int NFR, int NFS>
static void skinny_launch(FfnLaunch L, const FewRoute *few, hipStream_t st) {
    const int64_t per_xcd = skinny_blocks<NFR, NFS>(L);
    if constexpr (MODE == 0) {
        if (few) {
            ffn_skinny_few_kernel<WPS, NFR, NFS><<<dim3((unsigned)(per_xcd * 8 + 1)), dim3(256), 0, st>>>(L, *few);
            return;
        }
    }
    ffn_skinny_kernel<MODE, WPS, NFR, NFS><<<dim3((unsigned)(per_xcd * 8)), dim3(256), 0, st>>>(L);
}

// Whether a launch takes this kernel; beyond, ffn_mid.hip.  Microseconds of the pass, this kernel / that one:
//   gate/up: 60 experts + shared, 1 token 23.2 / 23.0, 3 tokens 36.1 / 41.3, 8 tokens 44.5 / 44.2; 16 experts of d 4096, top-4,
//     1 token 18.9 / 20.9, 4 tokens 36.4 / 37.2, 8 tokens 38.0 / 38.4; 8 experts, top-2, 4 tokens 36.9 / 38.2;
//   down: 60 experts + shared, 1 token 12.9 / 35.0, 8 tokens 23.9 / 33.7, 16 tokens 27.3 / 37.2, 24 tokens 33.8 / 40.3 (a layer call
//     of 32 tokens 117 / 125, 40 tokens 125.7 / 124.7); 8 experts, 4 tokens 15.8 / 18.2; 15 of 60 experts, 16 tokens 9.7 / 12.2.
//     Routed groups alone whose tiles there make two rounds of its 512 workgroups go over at a row per group: 16 experts
//     (N 4096), 4 tokens 19.0 / 20.4, 8 tokens 22.5 / 21.1, 24 tokens 24.5 / 22.0; groups of more than 16 rows, which need the form
//     of three waves per SIMD, go over unless its tiles are few: 8 groups, N 4096, 160 rows 15.1 / 11.2, 4 groups, 100 rows
//     9.5 / 9.0, but 2 groups, N 2048, 100 rows 10.6 / 16.7, N 4096 8.1 / 11.0 (weights warm).
// (The rows per group are those allotted; a device that holds a quarter of the experts has a quarter of them in use.)
constexpr int SKINNY_UP_ROWS = 32, SKINNY_UP_PER_GROUP = 2, SKINNY_UP_SINGLE = 8;
constexpr int SKINNY_DOWN_ROWS = 160, SKINNY_DOWN_BESIDE = 128, SKINNY_DOWN_SINGLE = 32;

bool ffn_skinny_takes(int pass, const FfnLaunch &L) {
    const FfnProblem &R = L.p[0], &S = L.p[1];
    if (L.has_single && S.A_cap > (pass == 0 ? SKINNY_UP_SINGLE : SKINNY_DOWN_SINGLE)) return false;
    if (!L.has_ragged) return true;
    if (pass == 0) return R.A_cap <= SKINNY_UP_ROWS && R.A_cap <= SKINNY_UP_PER_GROUP * R.E_local;
    if (L.has_single) return R.A_cap <= SKINNY_DOWN_BESIDE;
    const int64_t mid_tiles = (int64_t)(R.E_local < R.A_cap ? R.E_local : R.A_cap) * ((R.N + 63) / 64);
    return R.A_cap <= SKINNY_DOWN_ROWS && (R.A_cap <= R.E_local || mid_tiles < 1024) &&
           (R.A_cap <= 16 * R.E_local || mid_tiles <= 128);
}

// Whether the gate/up pass of a few tokens does their selection and index at its start, instead of route_finish_small_kernel before it.  Up
// to three rounds of workgroups (three share a CU): every round pays for it again.  Microseconds of a layer call, apart / so: 60
// experts + shared, 1 token (704 workgroups) 50.8 / 46.5, 3 tokens (1408) 68.0 / 63.5, 5 tokens (2112) 73.1 / 71.4, 8 tokens (3168) 78.3 /
// 83.2; 16 experts of d 4096, 1 token 36.3 / 34.0, 8 tokens (688) 69.0 / 65.7; 15 of 60 experts, 7 tokens 32.0 / 31.0.
bool ffn_skinny_takes_few(FfnLaunch L) {
    return L.has_ragged && L.p[0].gather_rows <= FEW_TOKENS && ffn_skinny_takes(0, L) && skinny_blocks<1, 1>(L) * 8 <= 9 * 8 * CUS_PER_XCD;
}

int launch_ffn_skinny(int pass, const FfnLaunch &L, const FewRoute *few, hipStream_t st) {
    drop_stale_error();
    const FfnProblem &R = L.p[0], &S = L.p[1];
    // Column blocks.  (Figures of a form with a partial sum per wave.)  Wider ones read the activations less often, narrower ones are more numerous: 16 in the gate/up pass (a
    // layer call of 4 / 8 / 16 tokens: 62.2 / 80.0 / 93.0 us, with 32 columns 71.4 / 83.3 / 96.2).  The down pass takes 32
    // for the routed groups (16 tokens: 91.2 us, with 16 columns 93.8) and 16 for the single group, whose contraction is
    // the longest: its workgroups are the last to finish (1 token, the pass: 12.3 against 17.0 us).
    // Four waves per SIMD with short bursts where the down pass has at most one 16-row fragment per group, as a rule, three
    // with longer ones where it has more (four / three, the pass: 60 experts + shared, 8 tokens 23.9 / 26.7, 16 tokens 27.3 / 30.6,
    // 24 tokens 43.8 / 33.8; 16 experts, 4 tokens 19.0 / 20.5) and in the gate/up pass, which has fewer workgroups (60 experts +
    // shared, 3 tokens 33.5 / 36.1, 8 tokens 43.8 / 44.5; 16 experts, 1 token 22.2 / 18.9, 8 tokens 41.1 / 38.0).
    if (pass == 0)
        skinny_launch<0, 3, 1, 1>(L, few, st);
    else if ((L.has_single && S.A_cap > 16) || (L.has_ragged && R.A_cap > 16 * R.E_local))
        skinny_launch<1, 3, 2, 1>(L, nullptr, st);
    else
        skinny_launch<1, 4, 2, 1>(L, nullptr, st);
    return launch_status();
}

}  // namespace c2r
