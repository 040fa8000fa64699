// Grouped SwiGLU expert FFN in bf16 for batches between decoding and prefill (groups of a few to a hundred-odd rows).
//
// Such a pass is still bound by streaming its weights, but it has too many rows for ffn_skinny.hip, whose every wave
// fetches the activations for 16 or 32 columns of its own, and too few tiles for ffn_bf16_dma.hip: that one's weight tiles
// of 1 MB are handed out in one and a quarter rounds, and a narrow single group (a shared expert's down pass: 8 tiles of
// 88 k-slices) keeps 8 CUs busy for 120 us while the rest of the chip waits.  Here a tile is 64 weight rows (64 output
// columns, or 32 with their gate and up rows) x up to 32, 64 or 128 rows of one group, and a workgroup of four waves, two
// of them on a CU, walks a contiguous run of tiles, an equal share of its problem's (see mid_walk).  Both operands go through
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

constexpr int mid_stages(int ar) { return ar == 32 ? 6 : ar == 64 ? 4 : 3; }
constexpr int mid_lds_bytes(int ar) { return mid_stages(ar) * (ar + MID_BR) * 128; }

// Where gate/up gathers, the source row of every sorted row.
__device__ __forceinline__ void mid_row_table(const FfnProblem &P, uint16_t *row_of) {
    for (int p = threadIdx.x; p < P.A_cap; p += 256) {
        const int g = P.gather[p], r = g > 0 ? (int)((uint32_t)g / (uint32_t)P.gather_div) : 0;
        row_of[p] = (uint16_t)(r < P.gather_rows ? r : P.gather_rows - 1);  // an out-of-range entry cannot leave A
    }
    __syncthreads();
}

// The workgroups that walk one problem: in all, those of the XCDs before this one, this XCD's, and this one's rank among them.
struct MidShare {
    int all, before, here, rank;
    int room;  // ranks from 0 on that have a CU without each other
};

// Walks one problem, its groups in gm (chunks of AR rows).  Items = (chunk of at most AR rows of one
// group, column block); a workgroup takes a contiguous run of them, an equal share (they all have the same k-slices).  Where the shares
// cannot be equal, the first ranks take an item more: workgroups `slot` and `slot` + 32 of an XCD share a CU, and two longer walks on
// one are what a launch then waits for.  More of them than there is room for are spread evenly instead (beyond it the pairs are there
// anyway, and a mixture of pairs and others finishes later than pairs throughout).  Microseconds of the gate/up pass, always spread / the
// first ranks: 60 groups (2640 items for the 512 workgroups) 151 / 134, 15 groups (660) 33.6 / 29.7, 2 groups (128) 14.0 / 12.4; 8 groups of d
// 4096 (352, room for 256) 30.4 / 33.9.
// A group's items are numbered in blocks of `run` columns - the length of a workgroup's run - chunk after chunk inside a block, so that the
// chunks of a column block, which read the same weights, are walked by neighbouring workgroups at the same time and the weights come
// into that XCD's L2 once.  (Chunks of a column block one after the other in one workgroup: by the second the weights were gone; the
// gate/up pass of 131 tokens fetched 1.37 times its weights.)
template <int MODE, int AR>
__device__ __forceinline__ void mid_walk(const FfnProblem &P, const GroupMap &gm, unsigned char *smem, const uint16_t *row_of,
                                         const MidShare &share) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int NSTAGE = mid_stages(AR), ROWB = 128, A_BYTES = AR * ROWB, STAGE_BYTES = (AR + MID_BR) * ROWB;
    constexpr int GA = AR / 32, GB = 2, NCOPY = GA + GB;  // 8-row copies per wave and slice
    constexpr int MF = AR / 32;                           // 16-row fragments per wave
    constexpr int BN = MODE == 0 ? MID_BR / 2 : MID_BR;
    // Tiles of 32 rows have four matrix instructions a slice, and a slice's time is its chain of wait, barrier, fragment reads and those: the reads go
    // ahead of the slice's copies, which the texture-address unit takes one by one.  Microseconds, copies first / reads first, one after the other in
    // one process: the kernel, 60 experts + shared, gate/up, 16 tokens 43.5 / 42.7, 24 tokens 47.0 / 45.8, 40 tokens 61.9 / 60.8, down, 40 tokens 38.9 /
    // 37.1, 64 tokens 39.3 / 38.4; 16 experts of d 4096, 24 tokens 30.5 / 30.1 and 17.5 / 17.2; 15 of 60 experts, 64 tokens 13.5 / 13.0 and 9.3 / 8.3; the
    // layer call, 16 tokens 79.5 / 78.6, 40 tokens 116.8 / 113.6, 64 tokens 135.0 / 134.0; d 4096, 24 tokens 63.3 / 62.1; 15 of 60 experts, 64 tokens
    // 41.5 / 40.1.  Higher tiles are even or lose: 64-row tiles of gate/up, 8 experts of d 4096, 200 tokens 86.6 / 88.8.
    constexpr bool READS_FIRST = AR == 32;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntn = P.ntn, N = P.N, Kdim = P.Kdim, nk = (Kdim + 63) / 64;
    const int n_items = __builtin_amdgcn_readfirstlane(gm.total_mtiles) * ntn;
    const int each = n_items / share.all, run = max(1, min(ntn, each));
    const uint32_t over = n_items - each * share.all;  // (items past an equal share of whole ones, fewer than the workgroups)
    const int over_before = over * (uint32_t)share.before / (uint32_t)share.all;
    const int more = (int)(over * (uint32_t)(share.before + share.here) / (uint32_t)share.all) - over_before;  // this XCD's of them
    const auto start_of = [&](int rank) __attribute__((always_inline)) {
        return (share.before + rank) * each + over_before +
               (more <= share.room ? min(rank, more) : (int)((uint32_t)more * (uint32_t)rank / (uint32_t)share.here));
    };
    const int first = start_of(share.rank), last = start_of(share.rank + 1);
    if (first >= last) return;
    const int total = (last - first) * nk;  // slices

    // A group of n rows is cut into ceil(n / AR) chunks of equal height (a multiple of 16, so none is empty).
    struct Item {
        int expert, row_begin, rows, n0;
    };
    auto item_at = [&](int item) __attribute__((always_inline)) {
        const uint64_t hit = __ballot(item >= gm.first * ntn && item < (gm.first + gm.tiles) * ntn);
        Item t;
        t.expert = __builtin_amdgcn_readfirstlane(hit ? __ffsll((unsigned long long)hit) - 1 : 0);
        const int lo = __builtin_amdgcn_readlane(gm.lo, t.expert), hi = __builtin_amdgcn_readlane(gm.hi, t.expert);
        const int chunks = __builtin_amdgcn_readlane(gm.tiles, t.expert);
        const int local = item - __builtin_amdgcn_readlane(gm.first, t.expert) * ntn;
        const int block = local / (chunks * run), rem = local - block * chunks * run, cols = min(run, ntn - block * run);
        const int height = ((hi - lo + chunks - 1) / chunks + 15) / 16 * 16;  // <= AR
        t.row_begin = lo + rem / cols * height;
        t.rows = hi - t.row_begin < height ? hi - t.row_begin : height;
        t.n0 = (block * run + rem % cols) * BN;
        return t;
    };

    // ---- copies: lane l of a copy lands on row l/8, chunk position l%8 of an 8-row group and therefore fetches chunk
    //      (l%8) ^ key(row), which leaves the tile swizzled for the fragment reads ----
    const int lrow = lane >> 3, lpos = lane & 7;
    const int chunkc[2] = {lpos ^ swz_key(lrow), lpos ^ swz_key(8 + lrow)};  // in even / odd 8-row groups
    const bool gather = MODE == 0 && P.gather != nullptr;
    const uint16_t *const B = MODE == 0 && wave >= 2 ? P.B1 : P.B0;  // (pass 0: 32 gate rows, then their 32 up rows)
    int i_item = first, i_kt = 0;  // the next slice to request
    const unsigned char *i_A = nullptr, *i_B = nullptr;
    uint32_t offA[GA], rowB[GB];
    auto open_item = [&]() __attribute__((always_inline)) {
        const Item t = item_at(i_item);
        i_kt = 0;
        i_A = uniform_ptr(reinterpret_cast<const unsigned char *>(gather ? P.A : P.A + (size_t)t.row_begin * P.lda));
        i_B = uniform_ptr(reinterpret_cast<const unsigned char *>(B + (size_t)t.expert * N * Kdim));
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
            rowB[i] = (uint32_t)(c < N ? c : N - 1) * (uint32_t)Kdim * 2u;
        }
    };
    auto request = [&](int stage) __attribute__((always_inline)) {
        if (i_kt == nk) {
            ++i_item;
            open_item();
        }
        unsigned char *s = smem + stage * STAGE_BYTES;
        const uint32_t kb = (uint32_t)i_kt * ROWB;
        const int left = Kdim - i_kt * 64;  // a weight chunk past K is taken from the start of its row: it meets A's zeros
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
    Item t = item_at(item);
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
        const bool more = n + NSTAGE - 1 < total;
        const int into = stage == 0 ? NSTAGE - 1 : stage - 1;
        if (!READS_FIRST && more) request(into);
        const unsigned char *s = smem + stage * STAGE_BYTES;
        bf16x8 a[2][MF], b[2][2];
        if (nf > 0) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t ch = (uint32_t)(((q * 4 + fq) ^ sw) * 16);
#pragma unroll
                for (int j = 0; j < 2; ++j) b[q][j] = *reinterpret_cast<const bf16x8 *>(s + rdB[j] + ch);
#pragma unroll
                for (int i = 0; i < MF; ++i)
                    if (i < nf) a[q][i] = *reinterpret_cast<const bf16x8 *>(s + rdA[i] + ch);
            }
        }
        if (READS_FIRST && more) request(into);
        if (nf > 0) {
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
        if (++kt < nk) continue;

        // ---- the item's last slice: results out, accumulators cleared, next item ----
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
                    if (col >= N) {  // pass 0 keeps the padding columns of h at zero for pass 1's k tail
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
            t = item_at(item);
            nf = (t.rows - wm * 16 + 31) / 32;
        }
    }
}

// The single group as a map of one group.
template <int AR>
__device__ __forceinline__ GroupMap mid_single_map(const FfnProblem &S) {
    int lo = S.offsets ? S.offsets[0] : S.row_lo, hi = S.offsets ? S.offsets[1] : S.row_hi;
    lo = lo < 0 ? 0 : (lo > S.A_cap ? S.A_cap : lo);
    hi = hi < lo ? lo : (hi > S.A_cap ? S.A_cap : hi);
    GroupMap m;
    m.total_mtiles = (hi - lo + AR - 1) / AR;
    const bool own = lane_id() == 0;
    m.lo = own ? lo : 0;
    m.hi = own ? hi : 0;
    m.tiles = own ? m.total_mtiles : 0;
    m.first = 0;
    return m;
}

// How many column blocks of the single group a workgroup walks when there are ragged items as well: what leaves the longest walk, in
// slices, as short as possible.  ceil(ntn / that) teams of a workgroup per chunk then walk the group, the other workgroups the ragged
// items.  Lane l tries l + 1; 0: none fits.  (Whole teams per XCD only, as many in each, left 448 or 456 workgroups where 453 make the
// longest walk an item shorter.)
__device__ __forceinline__ int mid_single_run(int chunks, int ntn, int kS, int r_items, int kR) {
    const int c = lane_id() + 1, teams = (ntn + c - 1) / c, rest = 8 * MID_WG_PER_XCD - teams * chunks;
    int cost = 0x7fffffff;
    if ((teams + 7) / 8 * chunks < MID_WG_PER_XCD)
        cost = min(max(c * kS, (r_items + rest - 1) / rest * kR), 0xffffff) << 6 | (63 - lane_id());  // (the longer run among equals)
    cost = -wave_max(-cost);
    return cost == 0x7fffffff ? 0 : 64 - (cost & 63);
}

// ARR, ARS: rows of the ragged problem's and of the single group's tiles.  The two walk on workgroups of their own, the single group's
// teams spread evenly over the XCDs (all of them in one XCD made that one finish last: the down pass of 64 tokens 52 against 42 us) and on
// the first workgroups of each, which have a CU each.  Microseconds, 60 experts and a shared one, eight batches each (one list of items
// for both / workgroups apart, longer walks wherever they fell / these): gate/up, 16 tokens 52.8 / 54.6 / 53.8, 32 tokens 62.0 / 63.6 / 60.1, 131
// tokens 93.8 / 90.2 / 87.9; down, 64 tokens 51.0 / 42.3 / 40.6, 131 tokens 53.1 / 52.0 / 49.1.
template <int MODE, int ARR, int ARS>
__global__ __launch_bounds__(256, 2) void ffn_mid_kernel(const FfnLaunch L) {
    constexpr int LDS = mid_lds_bytes(ARR) > mid_lds_bytes(ARS) ? mid_lds_bytes(ARR) : mid_lds_bytes(ARS);
    __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS];
    __shared__ uint16_t row_of[MODE == 0 ? MID_ROW_TABLE : 1];
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    GroupMap gm = {};
    if (L.has_ragged) gm = build_group_map<ARR>(L.p[0].offsets, L.p[0].E_local, L.p[0].A_cap);
    int ns = 0, ns_before = 0, ns_all = 0;  // workgroups that walk the single group: in this XCD, in those before it, in all
    bool long_single = false;               // their walks are longer than the others
    if (L.has_single) {
        const FfnProblem &S = L.p[1];
        const GroupMap sm = mid_single_map<ARS>(S);
        const int chunks = __builtin_amdgcn_readfirstlane(sm.total_mtiles);
        const int r_items = __builtin_amdgcn_readfirstlane(gm.total_mtiles) * L.p[0].ntn;
        if (chunks > 0) {
            const int kS = (S.Kdim + 63) / 64, kR = (L.p[0].Kdim + 63) / 64;
            const int run = r_items > 0 ? mid_single_run(chunks, S.ntn, kS, r_items, kR) : 0;
            const int teams = run ? (S.ntn + run - 1) / run : 8;
            const int size = run ? chunks : r_items > 0 ? 1 : MID_WG_PER_XCD;  // (nothing beside it: all of them)
            ns_before = xcd * teams / 8 * size;
            ns = (xcd + 1) * teams / 8 * size - ns_before;
            ns_all = teams * size;
            long_single = ns <= CUS_PER_XCD && r_items > 0 && run * kS > (r_items / (8 * MID_WG_PER_XCD - ns_all) + 1) * kR;
        }
        if (slot < ns) {
            if (MODE == 0 && S.gather) mid_row_table(S, row_of);  // (one routed group)
            mid_walk<MODE, ARS>(S, sm, smem, row_of, MidShare{ns_all, ns_before, ns, slot, CUS_PER_XCD});
            return;
        }
    }
    if (!L.has_ragged) return;
    if (MODE == 0 && L.p[0].gather) mid_row_table(L.p[0], row_of);
    // (the workgroups beside a longer walk of the single group's come last)
    const int beside = slot - CUS_PER_XCD;
    const int rank = !long_single || beside < 0 ? slot - ns : beside < ns ? MID_WG_PER_XCD - 2 * ns + beside : slot - 2 * ns;
    mid_walk<MODE, ARR>(L.p[0], gm, smem, row_of,
                        MidShare{8 * MID_WG_PER_XCD - ns_all, xcd * MID_WG_PER_XCD - ns_before, MID_WG_PER_XCD - ns, rank,
                                 long_single ? MID_WG_PER_XCD : CUS_PER_XCD - ns});
}

template <int MODE>
static void mid_launch(int ragged_rows, int single_rows, const FfnLaunch &L, hipStream_t st) {
    const dim3 g(8 * MID_WG_PER_XCD), b(256);
#define C2R_MID(ARR, ARS) ffn_mid_kernel<MODE, ARR, ARS><<<g, b, 0, st>>>(L)
#define C2R_MID_S(ARR)                    \
    if (single_rows == 64) {              \
        C2R_MID(ARR, 64);                 \
    } else {                              \
        C2R_MID(ARR, 32);                 \
    }
    switch (ragged_rows) {
        case 128: C2R_MID_S(128) break;
        case 64: C2R_MID_S(64) break;
        default: C2R_MID_S(32)
    }
#undef C2R_MID_S
#undef C2R_MID
}

// Whether a launch takes this kernel, and the rows of its ragged and its single tiles; else the tile kernel is the better one (or the only one).
// Lower tiles leave more copies in flight, higher ones read the weights (from L2) less often.  Microseconds of a layer call with
// 32 / 64 / 128 rows, r rows per expert on average (16 experts, d 4096, F 688) or n rows of a shared expert (60 experts, d 2048, F 1408 /
// 5632):
//   ragged groups alone: r = 6: 72.9 / 74.3 / 86.7, r = 15: 76.7 / 77.5 / 87, r = 25: 90.8 / 82.0 / 90.4, r = 45: 115 / 89 / 95, r = 64: 132 /
//     108 / 104, r = 88: 150 / 132 / 115, r = 125: 167 / 146 / 131 (tile kernel 143; down pass r = 100: 118 / 116 / 113 with it);
//   beside a shared expert, ragged and shared tiles of 32+32 / 64+32 / 32+64 / 64+64 rows: n = 24: 107 / 106 / 108 / 108, n = 64: 133 / 134 / 145 /
//     147, n = 90: 145 / 142 / 147 / 141, n = 131: 163 / 159 / 160 / 161, n = 178: 187 / 190 / 181 / 174; down pass alone n = 300: 197 / 197 /
//     195 / 187, n = 500: 236 / 228 / 234 / 210 (64+128 216, the tile kernel 212 at 511): no shared tiles of 128.  (The skewed groups beside it
//     hold up to eight times the mean: 64 rows from a mean of 5; measured on this one model.)
// (r counts the rows allotted.  A device that holds a quarter of the experts has a quarter of them in use if the load is even; of a skewed
// model, whose quarters have 0.5 to 2.1 times that, the heaviest is the one that a group waits for.  Its tiles are higher than its rows
// would ask for, 15 of 60 experts at 300 tokens 67.0 / 65.0 / 71.9.  The limit of the down pass goes by twice the even share.  Microseconds, 15
// of 60 experts, by the rows allotted / so: the heaviest quarter 400 tokens 88.0 / 82.8, 600 tokens 95.3 / 88.0, 675 tokens 97.7 / 97.9, a
// light one 400 tokens 79.4 / 73.2, 675 tokens 94.1 / 86.6; 20 of 60, 500 tokens 97.1 / 90.4.  With the limits of both passes by the even share
// the light one went on gaining, 700 tokens 91.9 / 82.2, but the heaviest lost: 700 tokens 98.3 / 104.4, 850 tokens 101 / 112, 1000 tokens 105 / 116.)
constexpr int MID_LOW_BESIDE = 4;

// most rows (per group, in the down pass at most twice the likely ones / in the single group), for 32-, 64- and 128-row tiles of gate/up and of down
constexpr int MID_RAGGED_UP_TO[2][3] = {{20, 64, 150}, {20, 45, 90}}, MID_SINGLE_UP_TO[2][2] = {{64, 179}, {100, 511}};

bool ffn_mid_rows(int pass, const FfnLaunch &L, int likely, int (&rows)[2]) {
    for (int q = 0; q < 2; ++q)
        if ((q == 0 ? L.has_ragged : L.has_single) && L.p[q].gather && (L.p[q].A_cap > MID_ROW_TABLE || L.p[q].gather_rows > 65536))
            return false;
    rows[0] = rows[1] = 0;
    if (L.has_ragged) {
        const int mean = L.p[0].A_cap / L.p[0].E_local, *most = MID_RAGGED_UP_TO[pass];
        const int heavy = pass == 0 || 2ll * likely > L.p[0].A_cap ? L.p[0].A_cap : 2 * likely;
        if (heavy / L.p[0].E_local > most[2]) return false;
        rows[0] = mean <= (L.has_single ? MID_LOW_BESIDE : most[0]) ? 32 : (mean <= most[1] ? 64 : 128);
    }
    if (L.has_single) {
        const int n = L.p[1].A_cap, *most = MID_SINGLE_UP_TO[pass];
        if (n > most[1]) return false;
        rows[1] = n <= most[0] ? 32 : 64;
    }
    if (!rows[0]) rows[0] = rows[1];  // (a side that is not there walks nothing)
    if (!rows[1]) rows[1] = rows[0] < 64 ? rows[0] : 64;
    return true;
}

// Whether a down pass over one group alone leaves no workgroup more than one item.
bool ffn_mid_in_one_round(const FfnProblem &down, int rows) {
    return (int64_t)((down.A_cap + rows - 1) / rows) * ((down.N + MID_BR - 1) / MID_BR) <= 8 * MID_WG_PER_XCD;
}

int launch_ffn_mid(int pass, const int (&tile_rows)[2], FfnLaunch L, hipStream_t st) {
    drop_stale_error();
    for (FfnProblem &P : L.p) {
        const int cols = P.zero_to > P.N ? P.zero_to : P.N, bn = pass == 0 ? MID_BR / 2 : MID_BR;
        P.ntn = (cols + bn - 1) / bn;
    }
    if (pass == 0)
        mid_launch<0>(tile_rows[0], tile_rows[1], L, st);
    else
        mid_launch<1>(tile_rows[0], tile_rows[1], L, st);
    return launch_status();
}

}  // namespace c2r
