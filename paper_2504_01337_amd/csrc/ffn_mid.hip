// Grouped SwiGLU expert FFN in bf16 for batches between decoding and prefill (groups of a few to a hundred-odd rows).
//
// Such a pass is still bound by streaming its weights, but it has too many rows for ffn_skinny.hip, whose every wave
// fetches the activations for 16 or 32 columns of its own, and too few tiles for ffn_bf16_dma.hip: that one's weight tiles
// of 1 MB are handed out in one and a quarter rounds, and a narrow single group (a shared expert's down pass: 8 tiles of
// 88 k-slices) keeps 8 CUs busy for 120 us while the rest of the chip waits.  Here a tile is 64 weight rows (64 output
// columns, or 32 with their gate and up rows) x up to 32, 64 or 128 rows of one group, and a workgroup of four waves, two
// of them on a CU, walks a contiguous run of tiles that is its equal share of all the k-slices.  Both operands go through
// a ring of six, four or three LDS stages filled by asynchronous copies, and the ring runs on ACROSS tiles: the next
// tile's first slices are requested while this one's last are computed, so that a workgroup has its copies in flight from
// its first slice to its last.  (One workgroup per tile instead, the same tile: 99 against 72 us for the gate/up pass of
// 16 tokens; each start waits for the launch, the offsets, the row numbers and the first weights one after the other.)
//
// Every output is one chain of v_mfma_f32_16x16x32_bf16 over ascending k, as in ffn_bf16_dma.hip and ffn_skinny.hip: the
// kernels give the same bits, so which of them runs may depend on what else the launch carries.
//
// Microseconds of a layer call, tile kernel -> this one (60 experts + shared, d 2048, F 1408 / 5632, top-4; 16 experts,
// d 4096, F 688, top-4):
//   60 experts: 64 tokens 212 -> 165, 131 tokens 256 -> 169, 256 tokens (down pass only) 210 -> 185;
//   16 experts: 64 tokens 107 -> 78, 180 tokens 115 -> 88, 256 tokens 126 -> 106, 500 tokens 143 -> 128;
//   15 of the 60 experts, 131 tokens 79 -> 65.
#include "ffn_common.h"
#include "ffn_copy.h"

namespace c2r {

constexpr int MID_BR = 64;               // weight rows of a tile: 64 output columns, or 32 with their gate and up rows
constexpr int MID_ROW_TABLE = 4096;      // sorted rows whose source row (16 bits) a workgroup keeps in LDS
constexpr int MID_WG_PER_XCD = 2 * CUS_PER_XCD;

// What a launch walks: items = (chunk of at most AR rows of one group, column block), the single group's first, then the
// ragged problem's; inside a group the chunks of a column block follow one another.
struct MidList {
    GroupMap gm;                 // of the ragged problem (per lane)
    int slo, shi, schunks;       // the single group's row range and chunks
    int n_single, n_ragged;      // items
};

struct MidItem {
    int expert, row_begin, rows, n0, nk;
    bool single;
};

// A group of n rows is cut into ceil(n / AR) chunks of equal height (a multiple of 16, so none is empty).
template <int MODE, int AR>
__device__ __forceinline__ MidItem mid_item_at(const FfnLaunch &L, const MidList &m, int item) {
    constexpr int BN = MODE == 0 ? MID_BR / 2 : MID_BR;
    MidItem t;
    t.single = item < m.n_single;
    int lo, hi, chunks, local;
    if (t.single) {
        t.expert = 0;
        lo = m.slo;
        hi = m.shi;
        chunks = m.schunks;
        local = item;
        t.nk = (L.p[1].Kdim + 63) / 64;
    } else {
        const int ntn = L.p[0].ntn;
        item -= m.n_single;
        const uint64_t hit = __ballot(item >= m.gm.first * ntn && item < (m.gm.first + m.gm.tiles) * ntn);
        const int e = hit ? __ffsll((unsigned long long)hit) - 1 : 0;
        t.expert = __builtin_amdgcn_readfirstlane(e);
        lo = __builtin_amdgcn_readlane(m.gm.lo, t.expert);
        hi = __builtin_amdgcn_readlane(m.gm.hi, t.expert);
        chunks = __builtin_amdgcn_readlane(m.gm.tiles, t.expert);
        local = item - __builtin_amdgcn_readlane(m.gm.first, t.expert) * ntn;
        t.nk = (L.p[0].Kdim + 63) / 64;
    }
    const int height = ((hi - lo + chunks - 1) / chunks + 15) / 16 * 16;  // <= AR
    t.row_begin = lo + local % chunks * height;
    t.rows = hi - t.row_begin < height ? hi - t.row_begin : height;
    t.n0 = local / chunks * BN;
    return t;
}

// First item whose start, in slices, is not below `s` (kS, kR: slices of a single / ragged item).
__device__ __forceinline__ int mid_first_item(int64_t s, const MidList &m, int kS, int kR) {
    const int64_t single = (int64_t)m.n_single * kS;
    return s < single ? (int)((s + kS - 1) / kS) : m.n_single + (int)((s - single + kR - 1) / kR);
}

template <int MODE, int AR, int NSTAGE>
__global__ __launch_bounds__(256, 2) void ffn_mid_kernel(const FfnLaunch L) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int ROWB = 128, A_BYTES = AR * ROWB, STAGE_BYTES = (AR + MID_BR) * ROWB;
    constexpr int GA = AR / 32, GB = 2, NCOPY = GA + GB;  // 8-row copies per wave and slice
    constexpr int MF = AR / 32;                           // 16-row fragments per wave
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NSTAGE * STAGE_BYTES];
    __shared__ uint16_t row_of[MODE == 0 ? MID_ROW_TABLE : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // ---- the list, and this workgroup's share of it: a contiguous run of items with an equal share of the k-slices
    //      (consecutive workgroups of an XCD walk neighbouring items and share their operands in its L2) ----
    MidList m;
    m.slo = m.shi = m.schunks = m.n_single = m.n_ragged = 0;
    if (L.has_single) {
        const FfnProblem &S = L.p[1];
        int lo = S.offsets ? S.offsets[0] : S.row_lo, hi = S.offsets ? S.offsets[1] : S.row_hi;
        lo = lo < 0 ? 0 : (lo > S.A_cap ? S.A_cap : lo);
        hi = hi < lo ? lo : (hi > S.A_cap ? S.A_cap : hi);
        m.slo = __builtin_amdgcn_readfirstlane(lo);
        m.shi = __builtin_amdgcn_readfirstlane(hi);
        m.schunks = (m.shi - m.slo + AR - 1) / AR;
        m.n_single = m.schunks * S.ntn;
    }
    m.gm = build_group_map<AR>(L.p[0].offsets, L.has_ragged ? L.p[0].E_local : 0, L.p[0].A_cap);
    if (L.has_ragged) m.n_ragged = __builtin_amdgcn_readfirstlane(m.gm.total_mtiles) * L.p[0].ntn;
    const int kS = (L.p[1].Kdim + 63) / 64, kR = (L.p[0].Kdim + 63) / 64;
    const int64_t all = (int64_t)m.n_single * kS + (int64_t)m.n_ragged * kR;
    const int nwg = (int)gridDim.x, w = (int)(blockIdx.x & 7) * (nwg >> 3) + (int)(blockIdx.x >> 3);
    const int first = mid_first_item(all * w / nwg, m, kS, kR), last = mid_first_item(all * (w + 1) / nwg, m, kS, kR);
    if (first >= last) return;
    const int s_items = last < m.n_single ? last - first : (first < m.n_single ? m.n_single - first : 0);
    const int total = s_items * kS + (last - first - s_items) * kR;  // slices

    if (MODE == 0 && L.p[L.has_ragged ? 0 : 1].gather) {  // the source row of every sorted row
        const FfnProblem &P = L.p[L.has_ragged ? 0 : 1];
        for (int p = threadIdx.x; p < P.A_cap; p += 256) {
            const int g = P.gather[p], r = g > 0 ? (int)((uint32_t)g / (uint32_t)P.gather_div) : 0;
            row_of[p] = (uint16_t)(r < P.gather_rows ? r : P.gather_rows - 1);  // an out-of-range entry cannot leave A
        }
        __syncthreads();
    }

    // ---- copies: lane l of a copy lands on row l/8, chunk position l%8 of an 8-row group and therefore fetches chunk
    //      (l%8) ^ key(row), which leaves the tile swizzled for the fragment reads ----
    const int lrow = lane >> 3, lpos = lane & 7;
    const int chunkc[2] = {lpos ^ swz_key(lrow), lpos ^ swz_key(8 + lrow)};  // in even / odd 8-row groups
    int i_item = first, i_kt = 0, i_nk = 0, i_K = 0;  // the next slice to request
    const unsigned char *i_A = nullptr, *i_B = nullptr;
    uint32_t offA[GA], rowB[GB];
    auto open_item = [&]() __attribute__((always_inline)) {
        const MidItem t = mid_item_at<MODE, AR>(L, m, i_item);
        const FfnProblem &P = L.p[t.single ? 1 : 0];
        const bool gather = MODE == 0 && P.gather != nullptr;
        i_kt = 0;
        i_nk = t.nk;
        i_K = P.Kdim;
        i_A = uniform_ptr(reinterpret_cast<const unsigned char *>(gather ? P.A : P.A + (size_t)t.row_begin * P.lda));
        const uint16_t *B = MODE == 0 && wave >= 2 ? P.B1 : P.B0;  // (pass 0: 32 gate rows, then their 32 up rows)
        i_B = uniform_ptr(reinterpret_cast<const unsigned char *>(B + (size_t)t.expert * P.N * P.Kdim));
#pragma unroll
        for (int i = 0; i < GA; ++i) {
            int r = (wave * GA + i) * 8 + lrow;
            r = r < t.rows ? r : t.rows - 1;
            if (gather) r = row_of[t.row_begin + r];
            offA[i] = (uint32_t)r * (uint32_t)P.lda * 2u + (uint32_t)chunkc[(wave * GA + i) & 1] * 16u;
        }
#pragma unroll
        for (int i = 0; i < GB; ++i) {
            const int r = (wave * GB + i) * 8 + lrow, c = t.n0 + (MODE == 0 ? r & 31 : r);
            rowB[i] = (uint32_t)(c < P.N ? c : P.N - 1) * (uint32_t)P.Kdim * 2u;
        }
    };
    auto request = [&](int stage) __attribute__((always_inline)) {
        if (i_kt == i_nk) {
            ++i_item;
            open_item();
        }
        unsigned char *s = smem + stage * STAGE_BYTES;
        const uint32_t kb = (uint32_t)i_kt * ROWB;
        const int left = i_K - i_kt * 64;  // a weight chunk past K is taken from the start of its row: it meets A's zeros
#pragma unroll
        for (int i = 0; i < GB; ++i)
            copy16_to_lds(i_B, rowB[i] + (MODE == 1 && chunkc[i] * 8 >= left ? 0u : kb + (uint32_t)chunkc[i] * 16u),
                          s + A_BYTES + (wave * GB + i) * 1024);
#pragma unroll
        for (int i = 0; i < GA; ++i) copy16_to_lds(i_A + kb, offA[i], s + (wave * GA + i) * 1024);
        ++i_kt;
    };
    open_item();

    // ---- fragments: waves 2 (rows) x 2 (columns); a wave's row fragments alternate with its neighbour's ----
    const int wm = wave >> 1, wn = wave & 1, fr = lane & 15, fq = lane >> 4, sw = swz_key(fr);
    uint32_t rdA[MF], rdB[2];
#pragma unroll
    for (int i = 0; i < MF; ++i) rdA[i] = (uint32_t)(i * 32 + wm * 16 + fr) * ROWB;
#pragma unroll
    for (int j = 0; j < 2; ++j)
        rdB[j] = (uint32_t)A_BYTES + (uint32_t)((MODE == 0 ? j * 32 + wn * 16 : wn * 32 + j * 16) + fr) * ROWB;
    f32x4 acc[MF][2];
    int item = first, kt = 0, stage = 0;
    MidItem t = mid_item_at<MODE, AR>(L, m, item);
    int nf = (t.rows - wm * 16 + 31) / 32;  // this wave's fragments that hold rows (<= 0: none)
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s)
        if (s < total) request(s);
    for (int n = 0; n < total; ++n) {
        // my copies of this slice have landed once at most those of the NSTAGE - 2 slices after it are outstanding (copies
        // complete in order; stores of an epilogue in flight only lengthen the wait); near the end fewer follow
        if (n + NSTAGE - 1 <= total)
            wait_copies_but_and_lds<(NSTAGE - 2) * NCOPY>();
        else
            wait_copies_but_and_lds<0>();
        lds_barrier();  // every wave's copies have landed and its reads of the slice before have returned: that stage is free
        if (n + NSTAGE - 1 < total) request(stage == 0 ? NSTAGE - 1 : stage - 1);
        const unsigned char *s = smem + stage * STAGE_BYTES;
        if (nf > 0) {
            bf16x8 a[2][MF], b[2][2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t ch = (uint32_t)(((q * 4 + fq) ^ sw) * 16);
#pragma unroll
                for (int j = 0; j < 2; ++j) b[q][j] = *reinterpret_cast<const bf16x8 *>(s + rdB[j] + ch);
#pragma unroll
                for (int i = 0; i < MF; ++i)
                    if (i < nf) a[q][i] = *reinterpret_cast<const bf16x8 *>(s + rdA[i] + ch);
            }
            // (operands swapped: a lane's four results are consecutive columns of one row)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < MF; ++i)
                    if (i < nf)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[q][j], a[q][i], acc[i][j], 0, 0, 0);
        }
        stage = stage == NSTAGE - 1 ? 0 : stage + 1;
        if (++kt < t.nk) continue;

        // ---- the item's last slice: results out, accumulators cleared, next item ----
        const FfnProblem &P = L.p[t.single ? 1 : 0];
        uint16_t *out = P.out + (size_t)t.row_begin * P.ldo;
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const int r = i * 32 + wm * 16 + fr;
            if (r < t.rows) {
#pragma unroll
                for (int j = 0; j < (MODE == 0 ? 1 : 2); ++j) {
                    const int col = t.n0 + (MODE == 0 ? wn * 16 : wn * 32 + j * 16) + fq * 4;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = MODE == 0 ? silu_mul(acc[i][0][e], acc[i][1][e]) : acc[i][j][e];
                    uint2 pk = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                    if (col >= P.N) {  // pass 0 keeps the padding columns of h at zero for pass 1's k tail
                        if (col >= P.zero_to) continue;
                        pk = make_uint2(0, 0);
                    }
                    *reinterpret_cast<uint2 *>(out + (size_t)r * P.ldo + col) = pk;
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        kt = 0;
        if (++item < last) {
            t = mid_item_at<MODE, AR>(L, m, item);
            nf = (t.rows - wm * 16 + 31) / 32;
        }
    }
}

template <int MODE>
static void mid_launch(int tile_rows, const FfnLaunch &L, hipStream_t st) {
    const dim3 g(8 * MID_WG_PER_XCD), b(256);
    if (tile_rows == 32)
        ffn_mid_kernel<MODE, 32, 6><<<g, b, 0, st>>>(L);
    else if (tile_rows == 64)
        ffn_mid_kernel<MODE, 64, 4><<<g, b, 0, st>>>(L);
    else
        ffn_mid_kernel<MODE, 128, 3><<<g, b, 0, st>>>(L);
}

// Rows of the tiles this kernel should cut the launch into; 0: the tile kernel is the better one (or the only one).
// Lower tiles leave more copies in flight, higher ones read the weights (from L2) less often.  Microseconds of a layer call
// with 32 / 64 / 128 rows / the tile kernel in the pass, r rows per expert on average (16 experts, d 4096, F 688) or n rows
// of a shared expert (60 experts, d 2048, F 1408 / 5632):
//   gate/up: r = 25: 74.5 / 72.7 / 79.6 / 87, r = 55: 114 / 91 / 97 / 110, r = 75: 116 / 105 / 99 / 113, r = 125: - / 146 / 128 /
//     143, r = 175: - / 178 / 172 / 155; n = 64: 137 / 147 / 150 / 156, n = 110: 176 / 162 / 175 / 166, n = 160: 191 / 165 / 172 /
//     169, n = 200: 232 / 200 / 204 / 185;
//   down: r = 25: 80 / 74 / 75.5 / 90, r = 40: 90 / 78 / 80 / 94, r = 55: 106 / 96 / 91 / 101, r = 75: 118 / 108 / 98 / 106, r = 100:
//     - / 118 / 116 / 113; n = 90: 152 / 162 / 162 / 192, n = 131: 173 / 165 / 174 / 204, n = 300: 221 / 194 / 200 / 216,
//     n = 511: - / - / 210 / 212.
// (r counts the rows allotted.  A device that holds a quarter of the experts has a quarter of them in use: its tiles are higher
// than its rows would ask for, 15 of 60 experts at 131 tokens 65.)
int ffn_mid_rows(int pass, const FfnLaunch &L) {
    int rows = 0;
    for (int q = 0; q < 2; ++q) {
        const FfnProblem &P = L.p[q];
        if (!(q == 0 ? L.has_ragged : L.has_single)) continue;
        if (P.gather && (P.A_cap > MID_ROW_TABLE || P.gather_rows > 65536)) return 0;
        static constexpr int up_to[2][2][3] = {{{20, 64, 150}, {64, 179, 179}}, {{20, 45, 90}, {100, 340, 511}}};
        const int mean = q == 0 ? P.A_cap / P.E_local : P.A_cap, *most = up_to[pass][q];
        if (mean > most[2]) return 0;
        const int fit = mean <= most[0] ? 32 : (mean <= most[1] ? 64 : 128);
        rows = fit > rows ? fit : rows;
    }
    return rows;
}

int launch_ffn_mid(int pass, int tile_rows, FfnLaunch L, hipStream_t st) {
    drop_stale_error();
    for (FfnProblem &P : L.p) {
        const int cols = P.zero_to > P.N ? P.zero_to : P.N, bn = pass == 0 ? MID_BR / 2 : MID_BR;
        P.ntn = (cols + bn - 1) / bn;
    }
    if (pass == 0)
        mid_launch<0>(tile_rows, L, st);
    else
        mid_launch<1>(tile_rows, L, st);
    return launch_status();
}

}  // namespace c2r
