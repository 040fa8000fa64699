// Grouped SwiGLU expert FFN in fp32: the full-precision path, on the fp32 matrix instructions.
//   mode 0: h[r, f]  = silu(x[r,:] . w_gate[e,f,:]) * (x[r,:] . w_up[e,f,:])
//   mode 1: y[r, j]  = h[r,:] . w_down[e,j,:]
//
// Bound by the matrix pipe for large batches (157 TFLOP/s, one fp32 fused multiply-add per product and sum) and by the
// latency of one wave's chain for small ones.  Both kernels load their operands 16 bytes per lane, lane (i, q) taking
// k = 4q .. 4q + 3 of row i of a 16-wide step, so that the four v_mfma_f32_16x16x4_f32 of a step add k = c, 4 + c, 8 + c,
// 12 + c for c = 0 .. 3: they give the same bits.
//   ffn_f32_direct_kernel: every wave works alone, without LDS, on 16 * MF rows x 16 * NC columns; loads go straight into
//     registers, four steps at a time with the next four in flight, and the waves of a workgroup take neighbouring columns of the same rows, which
//     meet in the CU's cache.  Short chains and many waves: for few rows.
//   ffn_f32_tile_kernel: 128 rows x 128 weight rows per workgroup of four waves, 128-byte k-slices through two LDS stages
//     that asynchronous copies fill, two workgroups per CU: a quarter of the other one's traffic out of L2.
// Microseconds gate/up + down of each pass replayed by itself, operands in L2 (vector-pipe kernel before -> now), 8 experts: d 256,
// F 512: 2 rows 24 + 28 -> 7.0 + 6.8, 1024 rows 28 + 34 -> 12.3 + 9.9, 4096 rows 34 + 34 -> 26 + 19.5, 16384 rows 115 + 65 -> 83 + 48
// (103 + 90 TFLOP/s); d 1024, F 1376: 256 rows 109 + 84 -> 36 + 22, 16384 rows 1113 + 604 -> 807 + 402 (115 TFLOP/s).  Inside a layer
// call the operands come from farther away: 1024 rows 30 + 33 -> 22 + 18, 4096 rows 48 + 37 -> 44 + 36 (profiled).  Against
// 64-bit sums the layer's error is what it was (1 to 8192 tokens: 5.6e-7 to 6.1e-7, 5.6e-7 to 6.3e-7 before).
#include "ffn_common.h"
#include "ffn_copy.h"

namespace c2r {

template <int MODE, int MF, int NC>
__global__ __launch_bounds__(256, 2) void ffn_f32_direct_kernel(const float *__restrict__ A, int lda,
                                                                const int32_t *__restrict__ offsets, int E_local,
                                                                int A_cap, int N, int Kdim, const float *__restrict__ B0,
                                                                const float *__restrict__ B1, float *__restrict__ out,
                                                                int ldo, int nwg) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int NB = MODE == 0 ? 2 * NC : NC, BM = 16 * MF, BN = 16 * NC;
    constexpr int U = 4;  // 16-wide steps requested together
    static_assert(MF * NB <= 4, "two sets of U steps fit the registers");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroup -> (row tile, four column blocks), column blocks fastest, a contiguous eighth of them per XCD: the row tile
    // is then read into one L2
    const GroupMap gm = build_group_map<BM>(offsets, E_local, A_cap);
    const XcdRange share = equal_range(__builtin_amdgcn_readfirstlane(gm.total_mtiles) * nwg, blockIdx.x & 7);
    const int slot = blockIdx.x >> 3;
    if (slot >= share.cnt) return;
    const int tile = (share.first + slot) / nwg, n0 = ((share.first + slot) % nwg * 4 + wave) * BN;
    const GroupTile g = locate_group_tile(gm, tile, BM);
    if (g.expert < 0 || n0 >= N) return;
    const int expert = __builtin_amdgcn_readfirstlane(g.expert), row0 = __builtin_amdgcn_readfirstlane(g.row_begin);
    const int row_end = __builtin_amdgcn_readfirstlane(g.row_end);

    const int fr = lane & 15, fq = lane >> 4;
    const float *pa[MF], *pb[NB];
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int r = row0 + i * 16 + fr;
        pa[i] = A + (size_t)(r < row_end ? r : row_end - 1) * lda + fq * 4;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int c = n0 + (j % NC) * 16 + fr;
        pb[j] = (j < NC ? B0 : B1) + ((size_t)expert * N + (c < N ? c : N - 1)) * Kdim + fq * 4;
    }
    f32x4 acc[MF][NB];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    struct Steps {
        f32x4 a[U][MF], b[U][NB];
    };
    auto load = [&](Steps &s, int g) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int j = 0; j < NB; ++j) s.b[u][j] = *reinterpret_cast<const f32x4 *>(pb[j] + (g * U + u) * 16);
#pragma unroll
            for (int i = 0; i < MF; ++i) s.a[u][i] = *reinterpret_cast<const f32x4 *>(pa[i] + (g * U + u) * 16);
        }
    };
    // (operands swapped: a lane's four results are consecutive columns of one row)
    auto mma = [&](const Steps &s) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);  // (the next steps' loads are issued before these instructions)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < MF; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.b[u][j][c], s.a[u][i][c], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    Steps s0, s1;
    const int ng = Kdim / (16 * U);  // whole groups of steps
    if (ng > 0) {
        load(s0, 0);
        int q = 0;
        for (; q + 1 < ng; q += 2) {
            load(s1, q + 1);
            mma(s0);
            load(s0, q + 2 < ng ? q + 2 : q);  // (unconditional: a load behind a branch would make every wait a full one)
            mma(s1);
        }
        if (q < ng) mma(s0);
    }
    if (ng * 16 * U < Kdim) {  // the rest: 4-wide pieces past the end count as zeros (Kdim is a multiple of 4)
        const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (ng * U + u) * 16;
            const bool in = k + fq * 4 < Kdim;
#pragma unroll
            for (int j = 0; j < NB; ++j) s0.b[u][j] = in ? *reinterpret_cast<const f32x4 *>(pb[j] + k) : zero;
#pragma unroll
            for (int i = 0; i < MF; ++i) s0.a[u][i] = in ? *reinterpret_cast<const f32x4 *>(pa[i] + k) : zero;
        }
        mma(s0);
    }

#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int r = row0 + i * 16 + fr;
        if (r >= row_end) continue;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = n0 + j * 16 + fq * 4;
            if (c >= N) continue;  // (N is a multiple of 4)
            f32x4 v = acc[i][j];
            if (MODE == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = v[e] / (1.0f + expf(-v[e])) * acc[i][MODE == 0 ? NC + j : j][e];
            }
            *reinterpret_cast<f32x4 *>(out + (size_t)r * ldo + c) = v;
        }
    }
}

constexpr int F32_BM = 128, F32_BR = 128;

template <int MODE>
__global__ __launch_bounds__(256, 2) void ffn_f32_tile_kernel(const float *__restrict__ A, int lda,
                                                              const int32_t *__restrict__ offsets, int E_local, int A_cap,
                                                              int N, int Kdim, const float *__restrict__ B0,
                                                              const float *__restrict__ B1, float *__restrict__ out, int ldo,
                                                              int ntn) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int BN = MODE == 0 ? F32_BR / 2 : F32_BR, ROWB = 128, A_BYTES = F32_BM * ROWB, STAGE = (F32_BM + F32_BR) * ROWB;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const GroupMap gm = build_group_map<F32_BM>(offsets, E_local, A_cap);
    const XcdRange share = equal_range(__builtin_amdgcn_readfirstlane(gm.total_mtiles) * ntn, blockIdx.x & 7);
    const int slot = blockIdx.x >> 3;
    if (slot >= share.cnt) return;
    const GroupTile g = locate_group_tile(gm, (share.first + slot) / ntn, F32_BM);
    if (g.expert < 0) return;
    const int n0 = (share.first + slot) % ntn * BN;
    const int expert = __builtin_amdgcn_readfirstlane(g.expert), row0 = __builtin_amdgcn_readfirstlane(g.row_begin);
    const int left = __builtin_amdgcn_readfirstlane(g.row_end) - row0, rows = left < F32_BM ? left : F32_BM;

    // ---- copies: lane l of a copy lands on row l/8, chunk l%8 (of 16 bytes) of an 8-row group and therefore fetches chunk
    //      (l%8) ^ key(row); chunks past the end of a row are replaced by its first one and left out of the sums below ----
    const int lrow = lane >> 3, lpos = lane & 7;
    const int chunkc[2] = {lpos ^ swz_key(lrow), lpos ^ swz_key(8 + lrow)};  // in even / odd 8-row groups
    const unsigned char *baseA = uniform_ptr(reinterpret_cast<const unsigned char *>(A + (size_t)row0 * lda));
    const float *B = MODE == 0 && wave >= 2 ? B1 : B0;  // (pass 0: 64 gate rows, then the 64 up rows of their columns)
    const unsigned char *baseB = uniform_ptr(reinterpret_cast<const unsigned char *>(B + (size_t)expert * N * Kdim));
    uint32_t rowA[4], rowB[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = (wave * 4 + i) * 8 + lrow, c = n0 + (MODE == 0 ? r & 63 : r);
        rowA[i] = (uint32_t)(r < rows ? r : rows - 1) * (uint32_t)lda * 4u;
        rowB[i] = (uint32_t)(c < N ? c : N - 1) * (uint32_t)Kdim * 4u;
    }
    const int nk = (Kdim + 31) / 32;
    auto request = [&](int kt, int stage) __attribute__((always_inline)) {
        unsigned char *s = smem + stage * STAGE + wave * 4096;
        const int room = Kdim - kt * 32;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t k = chunkc[i & 1] * 4 < room ? (uint32_t)kt * ROWB + (uint32_t)chunkc[i & 1] * 16u : 0u;
            copy16_to_lds(baseA, rowA[i] + k, s + i * 1024);
            copy16_to_lds(baseB, rowB[i] + k, s + A_BYTES + i * 1024);
        }
    };

    // ---- fragments: waves 2 (rows, alternating 16 by 16) x 2 (columns) ----
    const int wm = wave >> 1, wn = wave & 1, fr = lane & 15, fq = lane >> 4, sw = swz_key(fr);
    uint32_t rdA[4], rdB[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        rdA[i] = (uint32_t)(i * 32 + wm * 16 + fr) * ROWB;
        rdB[i] = (uint32_t)A_BYTES + (uint32_t)((MODE == 0 ? (i >> 1) * 64 + wn * 32 + (i & 1) * 16 : wn * 64 + i * 16) + fr) * ROWB;
    }
    const int nf = (rows - wm * 16 + 31) / 32;  // this wave's fragments that hold rows (<= 0: none)
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    request(0, 0);
    for (int kt = 0; kt < nk; ++kt) {
        wait_copies_but_and_lds<0>();
        lds_barrier();  // every wave's copies of this slice have landed and its reads of the one before have returned
        if (kt + 1 < nk) request(kt + 1, (kt + 1) & 1);
        const unsigned char *s = smem + (kt & 1) * STAGE;
        if (nf <= 0) continue;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t ch = (uint32_t)(((q * 4 + fq) ^ sw) * 16);
            f32x4 a[4], b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const f32x4 *>(s + rdB[j] + ch);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < nf) a[i] = *reinterpret_cast<const f32x4 *>(s + rdA[i] + ch);
            if (kt * 32 + 32 > Kdim && kt * 32 + q * 16 + fq * 4 >= Kdim) {
#pragma unroll
                for (int j = 0; j < 4; ++j) a[j] = b[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
            // (operands swapped: a lane's four results are consecutive columns of one row)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < nf)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][c], a[i][c], acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = i * 32 + wm * 16 + fr;
        if (r >= rows) continue;
#pragma unroll
        for (int j = 0; j < (MODE == 0 ? 2 : 4); ++j) {
            const int c = n0 + (MODE == 0 ? wn * 32 : wn * 64) + j * 16 + fq * 4;
            if (c >= N) continue;  // (N is a multiple of 4)
            f32x4 v = acc[i][j];
            if (MODE == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = v[e] / (1.0f + expf(-v[e])) * acc[i][MODE == 0 ? 2 + j : j][e];
            }
            *reinterpret_cast<f32x4 *>(out + (size_t)(row0 + r) * ldo + c) = v;
        }
    }
}

template <int MODE, int MF, int NC>
static int f32_direct(const float *a, const int32_t *offsets, int E_local, int64_t A_cap, int N, int Kdim, const float *b0,
                      const float *b1, float *out, hipStream_t st) {
    const int64_t mtiles = A_cap / (16 * MF) + (E_local < A_cap ? E_local : A_cap);
    const int nwg = (N + 64 * NC - 1) / (64 * NC);
    const int64_t grid = (mtiles * nwg + 7) / 8 * 8;
    if (grid >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    ffn_f32_direct_kernel<MODE, MF, NC><<<dim3((unsigned)grid), dim3(256), 0, st>>>(a, Kdim, offsets, E_local, (int)A_cap, N,
                                                                                   Kdim, b0, b1, out, N, nwg);
    return launch_status();
}

int launch_ffn_f32_pass(int pass, const float *a, const int32_t *offsets, int E_local, int64_t A_cap, int d,
                        int F, const float *b0, const float *b1, float *out, hipStream_t st) {
    drop_stale_error();
    const int N = pass == 0 ? F : d, Kdim = pass == 0 ? d : F;
    // From 256 tiles on (one per CU) the tile kernel; below, the taller wave tile (fewer reads of the weights) once it makes a
    // wave for every SIMD of the chip, in the down pass both taller and wider where the contraction is long enough to pay
    // for its start.  Microseconds of a pass (direct 16 x 16 / direct 32 rows / tile):
    //   gate/up, 8 experts, d 256, F 512: 512 rows 9.3 / 11.7 / 17.6, 1024 rows 16.5 / 12.2 / 25, 2048 rows 30 / 21.9 / 26.2,
    //     4096 rows 56 / 41 / 28.3; d 1024, F 1376: 256 rows 48 / 34 / 47, 512 rows 69 / 66 / 60;
    //   down, d 256, F 512: 1024 rows 10.4 / 14.0 / 45, 2048 rows 18.3 / 14.3 / 45, 4096 rows 34 / 26 (32 x 32: 18.9) / 45,
    //     16384 rows 128 / 98 (71) / 48; d 520, F 200, 4096 rows 21.1 / 21.9 (26.0) / 22.6.
    const int bn = pass == 0 ? F32_BR / 2 : F32_BR, ntn = (N + bn - 1) / bn;
    const int64_t groups = E_local < A_cap ? E_local : A_cap, tiles = (A_cap / F32_BM + groups) * ntn;
    auto waves = [&](int cols) { return (A_cap / 32 + groups) * ((N + cols - 1) / cols); };
    if (tiles >= 256) {
        const int64_t grid = (tiles + 7) / 8 * 8;
        if (grid >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
        const dim3 gr((unsigned)grid), bl(256);
        if (pass == 0)
            ffn_f32_tile_kernel<0><<<gr, bl, 0, st>>>(a, Kdim, offsets, E_local, (int)A_cap, N, Kdim, b0, b1, out, N, ntn);
        else
            ffn_f32_tile_kernel<1><<<gr, bl, 0, st>>>(a, Kdim, offsets, E_local, (int)A_cap, N, Kdim, b0, nullptr, out, N, ntn);
        return launch_status();
    }
#define C2R_F32_DIRECT(MODE, MF, NC) f32_direct<MODE, MF, NC>(a, offsets, E_local, A_cap, N, Kdim, b0, b1, out, st)
    if (pass == 0) return waves(16) >= 1280 ? C2R_F32_DIRECT(0, 2, 1) : C2R_F32_DIRECT(0, 1, 1);
    if (Kdim >= 512 && waves(32) >= 1024) return C2R_F32_DIRECT(1, 2, 2);
    return waves(16) >= 1152 ? C2R_F32_DIRECT(1, 2, 1) : C2R_F32_DIRECT(1, 1, 1);
#undef C2R_F32_DIRECT
}

}  // namespace c2r
