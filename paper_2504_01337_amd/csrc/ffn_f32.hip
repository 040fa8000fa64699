// Grouped SwiGLU expert FFN in fp32: the full-precision path, on the fp32 matrix instructions.
//   mode 0: h[r, f]  = silu(x[r,:] . w_gate[e,f,:]) * (x[r,:] . w_up[e,f,:])
//   mode 1: y[r, j]  = h[r,:] . w_down[e,j,:]
//
// Bound by the matrix pipe for large batches (157 TFLOP/s, one fp32 fused multiply-add per product and sum), by streaming the weights
// and by the latency of a wave's chain for small ones.  A workgroup of four waves takes 32 MF rows x 32 NP columns, 16 MF x 16 NP
// (with the matching gate and up columns) per wave; 128-byte k-slices pass through a ring of LDS stages that asynchronous copies
// fill ahead.  Small tiles in shallow rings, so that several workgroups share a CU: their copies, barriers and fragment reads are
// covered by each other's matrix instructions.  A lane loads its operands 16 bytes at a time, lane (i, q) taking k = 4q .. 4q + 3 of
// row i of a 16-wide step, so that the four v_mfma_f32_16x16x4_f32 of a step add k = c, 4 + c, 8 + c, 12 + c for c = 0 .. 3: every
// tile shape gives the same bits.
//
// Microseconds gate/up + down of each pass, three sets of weights in turn (register-direct waves for few rows and tiles of 128 x 128
// for many before -> now): 8 experts, d 256, F 512: 1024 rows 21.3 + 18.0 -> 10.2 + 8.8, 4096 rows 42.9 + 35.3 -> 25.5 + 14.5, 16384
// rows 101 + 80 -> 81 + 41; d 1024, F 1376: 64 rows 24.3 + 20.3 -> 21.1 + 11.7, 4096 rows 293 + 201 -> 193 + 108, 16384 rows 869 + 493
// -> 714 + 358 (129 TFLOP/s); 16 experts, d 2048, F 1408: 64 rows 134 + 61 -> 69 + 32, 2048 rows 297 + 207 -> 226 + 115.  A row per group
// is what lost, with a tile or two per CU: 8 experts, d 1024, 8 rows 21.3 -> 22.7 in gate/up; 16 experts, d 2048, 37.1 + 17.4 -> 39.0 + 18.4.
#include <type_traits>

#include "ffn_common.h"
#include "ffn_copy.h"

namespace c2r {

// 32 MF rows x 32 NP columns per workgroup of four waves (2 x 2; pass 0: the gate rows and the up rows of those columns), 128-byte
// k-slices through a ring of NSTAGE LDS stages that asynchronous copies fill NSTAGE - 1 slices ahead.
template <int MODE, int MF, int NP, int NSTAGE>
__global__ __launch_bounds__(256) void ffn_f32_ring_kernel(const float *__restrict__ A, int lda,
                                                           const int32_t *__restrict__ offsets, int E_local, int A_cap, int N,
                                                           int Kdim, const float *__restrict__ B0, const float *__restrict__ B1,
                                                           float *__restrict__ out, int ldo, int ntn) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int NB = MODE == 0 ? 2 * NP : NP, BM = 32 * MF, BN = 32 * NP;  // NB: blocks of 32 weight rows, 16 of each per wave
    constexpr int ROWB = 128, A_BYTES = BM * ROWB, STAGE = A_BYTES + NB * 32 * ROWB;
    constexpr int NC = MF + NB;  // copies per wave and slice, of eight rows each
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NSTAGE * STAGE];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const GroupMap gm = build_group_map<BM>(offsets, E_local, A_cap);
    const XcdRange share = equal_range(__builtin_amdgcn_readfirstlane(gm.total_mtiles) * ntn, blockIdx.x & 7);
    const int slot = blockIdx.x >> 3;
    if (slot >= share.cnt) return;
    const GroupTile g = locate_group_tile(gm, (share.first + slot) / ntn, BM);
    if (g.expert < 0) return;
    const int n0 = (share.first + slot) % ntn * BN;
    const int expert = __builtin_amdgcn_readfirstlane(g.expert), row0 = __builtin_amdgcn_readfirstlane(g.row_begin);
    const int left = __builtin_amdgcn_readfirstlane(g.row_end) - row0, rows = left < BM ? left : BM;

    // ---- copies: lane l of a copy lands on row l/8, chunk l%8 (of 16 bytes) of an 8-row group and therefore fetches chunk
    //      (l%8) ^ key(row); chunks past the end of a row are replaced by its first one and left out of the sums below.  Wave w
    //      brings rows 8w .. 8w + 7 of every block of 32 rows ----
    const int lrow = lane >> 3, chunkc = (lane & 7) ^ swz_key((wave & 1) * 8 + lrow);
    const unsigned char *baseA = uniform_ptr(reinterpret_cast<const unsigned char *>(A + (size_t)row0 * lda));
    const unsigned char *base0 = uniform_ptr(reinterpret_cast<const unsigned char *>(B0 + (size_t)expert * N * Kdim));
    const unsigned char *base1 = MODE == 0 ? uniform_ptr(reinterpret_cast<const unsigned char *>(B1 + (size_t)expert * N * Kdim)) : base0;
    uint32_t rowA[MF], rowB[NP];
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int r = i * 32 + wave * 8 + lrow;
        rowA[i] = (uint32_t)(r < rows ? r : rows - 1) * (uint32_t)lda * 4u;
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int c = n0 + j * 32 + wave * 8 + lrow;
        rowB[j] = (uint32_t)(c < N ? c : N - 1) * (uint32_t)Kdim * 4u;
    }
    const int nk = (Kdim + 31) / 32;
    auto request = [&](int kt, int stage) __attribute__((always_inline)) {
        unsigned char *s = smem + stage * STAGE + wave * 1024;
        const uint32_t k = chunkc * 4 < Kdim - kt * 32 ? (uint32_t)kt * ROWB + (uint32_t)chunkc * 16u : 0u;
#pragma unroll
        for (int i = 0; i < MF; ++i) copy16_to_lds(baseA, rowA[i] + k, s + i * 4096);
#pragma unroll
        for (int j = 0; j < NB; ++j) copy16_to_lds(j < NP ? base0 : base1, rowB[j % NP] + k, s + A_BYTES + j * 4096);
    };

    // ---- fragments: waves 2 (rows, alternating 16 by 16) x 2 (columns) ----
    const int wm = wave >> 1, wn = wave & 1, fr = lane & 15, fq = lane >> 4, sw = swz_key(fr);
    uint32_t rdA[MF], rdB[NB];
#pragma unroll
    for (int i = 0; i < MF; ++i) rdA[i] = (uint32_t)(i * 32 + wm * 16 + fr) * ROWB;
#pragma unroll
    for (int j = 0; j < NB; ++j) rdB[j] = (uint32_t)A_BYTES + (uint32_t)(j / NP * BN + (wn * NP + j % NP) * 16 + fr) * ROWB;
    const int nf = (rows - wm * 16 + 31) / 32;  // this wave's fragments that hold rows (<= 0: none)
    f32x4 acc[MF][NB];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s)
        if (s < nk) request(s, s);
    // FR: this wave's row fragments that hold rows (a wave with none only copies)
    auto walk = [&](auto fr_c) __attribute__((always_inline)) {
        constexpr int FR = decltype(fr_c)::value;
        int cur = 0, kt = 0;
        // AFTER: slices after this one that have been requested; this one has landed once only their copies are outstanding
        auto step = [&](auto after_c, bool more) __attribute__((always_inline)) {
            constexpr int AFTER = decltype(after_c)::value;
            wait_copies_but_and_lds<AFTER * NC>();
            lds_barrier();  // everyone's copies of this slice have landed, everyone's reads of the one before have returned
            const unsigned char *s = smem + cur * STAGE;
            f32x4 a[2][FR ? FR : 1], b[2][NB];  // (all of the slice's fragments are requested before its first matrix instruction)
            if (FR > 0) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t ch = (uint32_t)(((q * 4 + fq) ^ sw) * 16);
#pragma unroll
                    for (int j = 0; j < NB; ++j) b[q][j] = *reinterpret_cast<const f32x4 *>(s + rdB[j] + ch);
#pragma unroll
                    for (int i = 0; i < FR; ++i) a[q][i] = *reinterpret_cast<const f32x4 *>(s + rdA[i] + ch);
                }
            }
            if (more) request(kt + NSTAGE - 1, cur == 0 ? NSTAGE - 1 : cur - 1);  // (into the stage of the slice before)
            if (FR > 0) {
                if (AFTER == 0 && kt * 32 + 32 > Kdim) {
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        if (kt * 32 + q * 16 + fq * 4 >= Kdim) {
#pragma unroll
                            for (int i = 0; i < FR; ++i) a[q][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                            for (int j = 0; j < NB; ++j) b[q][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                        }
                }
                // (operands swapped: a lane's four results are consecutive columns of one row)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int i = 0; i < FR; ++i)
#pragma unroll
                            for (int j = 0; j < NB; ++j)
                                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[q][j][c], a[q][i][c], acc[i][j], 0, 0, 0);
            }
            cur = cur + 1 == NSTAGE ? 0 : cur + 1;
            ++kt;
        };
#pragma unroll 1
        while (kt + NSTAGE - 1 < nk) step(std::integral_constant<int, NSTAGE - 2>{}, true);
        static_assert(NSTAGE >= 2 && NSTAGE <= 4, "the last slices, below");
        if (NSTAGE > 3 && nk > 2) step(std::integral_constant<int, 2>{}, false);
        if (NSTAGE > 2 && nk > 1) step(std::integral_constant<int, 1>{}, false);
        step(std::integral_constant<int, 0>{}, false);
    };
    if (nf >= MF)
        walk(std::integral_constant<int, MF>{});
    else if (MF > 1 && nf > 0)
        walk(std::integral_constant<int, MF == 1 ? 1 : MF - 1>{});
    else
        walk(std::integral_constant<int, 0>{});
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int r = i * 32 + wm * 16 + fr;
        if (r >= rows) continue;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int c = n0 + (wn * NP + j) * 16 + fq * 4;
            if (c >= N) continue;  // (N is a multiple of 4)
            f32x4 v = acc[i][j];
            if (MODE == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = v[e] / (1.0f + expf(-v[e])) * acc[i][MODE == 0 ? NP + j : j][e];
            }
            *reinterpret_cast<f32x4 *>(out + (size_t)(row0 + r) * ldo + c) = v;
        }
    }
}

template <int MODE, int MF, int NP, int NSTAGE>
static int f32_ring(const float *a, const int32_t *offsets, int E_local, int64_t A_cap, int N, int Kdim, const float *b0,
                    const float *b1, float *out, hipStream_t st) {
    const int64_t mtiles = A_cap / (32 * MF) + (E_local < A_cap ? E_local : A_cap);
    const int ntn = (N + 32 * NP - 1) / (32 * NP);
    const int64_t grid = (mtiles * ntn + 7) / 8 * 8;
    if (grid >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    ffn_f32_ring_kernel<MODE, MF, NP, NSTAGE><<<dim3((unsigned)grid), dim3(256), 0, st>>>(a, Kdim, offsets, E_local, (int)A_cap, N,
                                                                                         Kdim, b0, b1, out, N, ntn);
    return launch_status();
}

int launch_ffn_f32_pass(int pass, const float *a, const int32_t *offsets, int E_local, int64_t A_cap, int d,
                        int F, const float *b0, const float *b1, float *out, hipStream_t st) {
    drop_stale_error();
    const int N = pass == 0 ? F : d, Kdim = pass == 0 ? d : F;
    // Tiles of 32 x 32 until 64-row tiles (64 x 32 in gate/up, 64 x 64 in down) make five for every CU; stages by how many
    // workgroups share a CU.  Microseconds of a pass (32 x 32 / 64-row tiles):
    //   gate/up, 8 experts, d 256, F 512: 1024 rows (384 64-row tiles) 10.2 / 12.3, 4096 rows (1152) 25.5 / 26.5, 16384 rows (4224)
    //     80.6 / 78.3; d 1024, F 1376: 256 rows (516) 30 / 36, 4096 rows (3096) 211 / 193; 16 experts, d 2048, F 1408, 2048 rows
    //     (2112) 244 / 226;
    //   down, the same: 1024 rows (96) 8.8 / 12.2, 4096 rows (288) 14.5 / 19.9, 16384 rows (1056) 41 / 44; 256 rows (192) 16.6 / 27.5, 4096
    //     rows (1152) 105 / 108, 16384 rows (4224) 430 / 358; 2048 rows (1536) 129 / 115.  With three / four stages: 4096 rows 14.5 /
    //     15.6; 64 rows 13.3 / 11.7; one group, d 2048, F 2048, 64 rows 18.7 / 16.3.
    const int64_t groups = E_local < A_cap ? E_local : A_cap;
    auto tiles = [&](int rows, int cols) { return (A_cap / rows + groups) * ((N + cols - 1) / cols); };
#define C2R_F32_RING(MODE, MF, NP, NS) f32_ring<MODE, MF, NP, NS>(a, offsets, E_local, A_cap, N, Kdim, b0, b1, out, st)
    if (pass == 0) return tiles(64, 32) < 1280 ? C2R_F32_RING(0, 1, 1, 3) : C2R_F32_RING(0, 2, 1, 3);
    if (tiles(64, 64) >= 1280) return C2R_F32_RING(1, 2, 2, 3);
    return tiles(32, 32) <= 1024 ? C2R_F32_RING(1, 1, 1, 4) : C2R_F32_RING(1, 1, 1, 3);
#undef C2R_F32_RING
}

}  // namespace c2r
