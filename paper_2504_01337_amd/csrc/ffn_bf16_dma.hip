// Grouped SwiGLU expert FFN in bf16, fast path: global -> LDS copies that bypass the
// register file (global_load_lds_dwordx4), 8 waves per workgroup, 256 x 256 output tiles,
// 64-wide k-slices in LDS (two stages of the activation tile, a ring of three of the weight
// tile: 160 KB), v_mfma_f32_16x16x32_bf16 (measured 4-8 % faster
// here than the 32x32x16 form at equal LDS traffic: a quarter of the accumulator registers
// move per instruction, and under this chip's power limit that buys clock).
//
// Same two passes, tile numbering and epilogue as the generic kernel in ffn_bf16.hip;
// what differs is how a k-slice reaches LDS.  One wave-level copy instruction moves
// 64 x 16 bytes = 8 tile rows of 128 bytes, i.e. whole cache lines (measured: 128-byte
// rows copy at ~25 TB/s chip-wide, 64-byte rows at ~16 TB/s).  Lane l lands at byte 16*l of the 1 KB run, i.e. row l/8, chunk
// position l%8, so the lane fetches the global chunk (l%8) ^ swz_key(row) and the
// swizzled layout falls out without any LDS write instruction.  The copies are
// asynchronous and overlap the MFMAs: the A tile of slice k+2 goes out when the stage of
// slice k is handed over, the B tile of slice k+2 a little earlier into the ring slot of
// slice k-1 (weights stream from HBM and take longest); one "my copies of the next slice
// landed, my reads returned" wait + bare barrier per slice, placed before the slice's last
// k-step, hands the stages over (see slice_step).
//
// Contract (checked by the launcher): the contraction length seen by A is padded to a
// multiple of 64 with zeros (lda >= 64 * ceil(K/64)); a B chunk past K is re-read from
// chunk 0 of the same row and multiplied by those zeros.
#include <atomic>
#include <type_traits>

#include "ffn_common.h"
#include "ffn_copy.h"

namespace c2r {

// The launch arguments as the tile function reads them: through the constant address space
// (scalar loads from the kernel-argument segment).
typedef const __attribute__((address_space(4))) FfnLaunch FfnLaunchConst;
typedef const __attribute__((address_space(4))) FfnProblem FfnProblemConst;
typedef FfnLaunchConst *FfnLaunchArgs;

// Both passes of an FFN in one launch (see ffn_bf16_dma_both_kernel).
struct FfnBothLaunch {
    FfnLaunch pass[2];
};
constexpr int FFN_LINE = 32, FFN_MTILE_INTS = 8;  // ints from one ticket counter to the next / from one M-tile's counter to the next

// What a tile is to the other pass.  Gate/up: the M-tile that it is a part of and its rows.  Down: the launch's counters of finished
// gate/up rows per M-tile, whether all are known to be finished, and the columns of the gate/up pass in tiles, {routed, single}.
struct FfnTileLink {
    int mt, rows, n_mtiles;
    bool ready;
    int up_ntn[2];
    const int *rows_done;
};

// Shapes shared by the per-tile function and the kernel around it.
template <int WM, int WN>
struct FfnShape {
    static constexpr int BM = 256, BN = 256, BK = 64, NW = WM * WN, ROWB = BK * 2;
    static constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB;
    static constexpr int LONG_BYTES = 2 * A_BYTES + 3 * B_BYTES;         // 2 A stages + a ring of 3 B stages
    static constexpr int SHORT_BYTES = 3 * (128 + BN) * ROWB;            // ring of 3 x (128 A rows + B tile)
    static constexpr int SMEM_BYTES = LONG_BYTES > SHORT_BYTES ? LONG_BYTES : SHORT_BYTES;
};

// A store that is complete only once the memory that all XCDs share has it (the policy of an atomic store at device scope).
__device__ __forceinline__ void store16_through(void *p, uint4 v) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 q = {v.x, v.y, v.z, v.w};
    asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(q) : "memory");
#endif
}

// Length of XCD x's list (tiles, with the last round cut into parts): what its queue hands out.
template <bool BESIDE>
__device__ __forceinline__ int xcd_list_slots(int n_tiles) {
    if (n_tiles <= 0) return 0;
    const int full = n_tiles / CUS_PER_XCD * CUS_PER_XCD;
    return full + (n_tiles - full) * last_round_parts<BESIDE>(n_tiles);
}

// One output tile: position `slot` of XCD `xcd`'s list.  Every wave of the workgroup calls it
// with the same arguments; it returns early (all waves alike) when the position holds nothing.
// grp_lo, grp_hi: the row range of this lane's expert of the ragged problem (load_group_range);
// sg_lo, sg_hi: the row range of the single group (clamped), the same in every lane.
// before_epilogue(): called once by every wave after the tile's last k-step (the kernel draws
// the next ticket there, so that the trip to the counter overlaps the epilogue); not called on
// the early returns.
// BOTH: the launch carries both passes; `link` ties the tile to the other one and under_way() is called once by every wave after a
// barrier behind which this wave's and every other wave's memory operations from before the call are complete.  Every wave has waited there
// until no more than its copies of the later slices are outstanding.  That covers the older stores because a wave's loads, stores and copies
// count down ONE counter in the order of their issue on gfx9 targets, and gfx950 is the only one this is built for (LLVM, "User Guide for AMDGPU
// Backend", memory model: vector memory operations' completion is reported to a wavefront in execution order).  A store with sc1 is
// the guide's atomic store at agent scope, whose completion a release at that scope waits for with the same counter.
// EARLY: the single group's tiles come before all others of their pass (see ffn_bf16_dma_both_kernel).
template <int MODE, int WM, int WN, bool BOTH, bool EARLY, class UnderWay, class BeforeEpilogue>
__device__ __forceinline__ void ffn_tile(const FfnLaunchArgs Lp, unsigned char *smem, const int xcd, const int slot,
                                         const int grp_lo, const int grp_hi, const int sg_lo, const int sg_hi,
                                         FfnTileLink &link, UnderWay &&under_way, BeforeEpilogue &&before_epilogue) {
    const FfnLaunchConst &L = *Lp;
    constexpr int BM = 256, BN = 256, BK = 64;
    constexpr int NW = WM * WN;                // waves
    constexpr int TM = BM / WM, TN = BN / WN;  // wave tile
    constexpr int ROWB = BK * 2;               // 128 bytes per tile row: whole cache lines per copy
    constexpr int GA = BM / 8 / NW, GB = BN / 8 / NW;  // 8-row copy groups per wave
    constexpr int A_BYTES = BM * ROWB, STAGE_BYTES = (BM + BN) * ROWB;
    constexpr int BNF = MODE == 0 ? BN / 2 : BN;
    static_assert((BM / 8) % NW == 0 && (BN / 8) % NW == 0, "copy groups divide evenly");
    // Short tiles (<= LM rows, i.e. small experts) are bound by streaming their expert's
    // weights from HBM, not by the MFMAs: they use the same LDS as a three-stage ring of
    // (LM A rows + BN B rows), two slices in flight instead of one.
    constexpr int LM = 128, L_A_BYTES = LM * ROWB, L_STAGE_BYTES = (LM + BN) * ROWB, L_NSTAGE = 3;
    constexpr int L_GA = LM / 8 / NW;  // A copy groups per wave on the short path
    // Long path: two stages of A (rows of the activations: shared through L2 by the workgroups of
    // a tile row, short latency) and a ring of THREE stages of B (rows of the weights: streamed
    // from HBM, long latency), so that a B slice is copied two slices ahead of its use.
    constexpr int B_BYTES = BN * ROWB, B_NSTAGE = 3;
    constexpr int LONG_BYTES = 2 * A_BYTES + B_NSTAGE * B_BYTES;
    // Tiles of at most TM_T rows (experts with a handful of tokens: most of the short tiles) need
    // even less room for A and get a ring of four stages, three slices in flight: what such a
    // tile takes is the latency of its weight slices divided by the slices in flight.
    constexpr int TM_T = 64, T_A_BYTES = TM_T * ROWB, T_STAGE_BYTES = (TM_T + BN) * ROWB, T_NSTAGE = 4;
    static_assert(TM_T / 8 == NW, "one A copy group per wave on the tiny path");
    constexpr int SMEM_BYTES = LONG_BYTES > L_NSTAGE * L_STAGE_BYTES ? LONG_BYTES : L_NSTAGE * L_STAGE_BYTES;
    static_assert(T_NSTAGE * T_STAGE_BYTES <= SMEM_BYTES, "the tiny ring fits");
    static_assert(SMEM_BYTES == FfnShape<WM, WN>::SMEM_BYTES, "the kernel allocates what the tile function lays out");
    static_assert(LM == TM && (LM / 8) % NW == 0, "the short path is the first wave row's M range");
    unsigned char *const st0 = smem, *const st1 = smem + A_BYTES;  // the two A stages
    // B ring slot q lives at smem + 2*A_BYTES + q*B_BYTES.  Copies and fragment reads address B
    // as "stage + A_BYTES + ...", so a B slot is handed to them as the pointer A_BYTES below it.
    unsigned char *bcur = smem + A_BYTES, *bnxt = bcur + B_BYTES, *bwr = bnxt + B_BYTES;

    // (the thread index is made opaque per tile: what is derived from it - copy offsets, fragment
    // addresses - is then recomputed per tile instead of being hoisted out of the kernel's tile
    // loop and held in registers across it)
    int tid_opaque = threadIdx.x;
    asm volatile("" : "+v"(tid_opaque));
    const int tid = tid_opaque, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    // Tile of this workgroup.  The launch carries one problem, or two (the routed groups and an
    // always-on shared expert).  An XCD's list: its share of the single group's tiles, then of
    // the ragged problem's full tiles, then of its short tiles (ffn_common.h).  One group (a
    // shared expert, a plain GEMM) needs no map: its bounds are two scalars.
    // (the launcher puts the ragged problem, if any, in p[0] and the single group in p[1])
    const bool ragged0 = L.has_ragged != 0, have_sg = L.has_single != 0;
    const int slo = sg_lo, shi = sg_hi;
    int smt = 0;
    XcdRange rs, ra, rb;
    rs.first = rs.cnt = ra.first = ra.cnt = rb.first = rb.cnt = 0;
    const int sbm = L.single_rows;
    if (have_sg) {
        smt = (shi - slo + sbm - 1) / sbm;
        rs = equal_range(smt * L.p[1].ntn, xcd);
    }
    RaggedMap rmap;
    if (ragged0) {
        rmap = ragged_map_of<BM>(grp_lo, grp_hi);
        ra = equal_range(rmap.totalA * L.p[0].ntn, xcd);
        rb = equal_range(rmap.totalB * L.p[0].ntn, xcd);
    }
    constexpr bool BESIDE = BOTH && MODE == 0;
    TailSplit ts = split_last_round<BESIDE>(rs.cnt + ra.cnt + rb.cnt, slot);
    if (!ts.valid) return;
    // (the same in every lane, but derived from cross-lane moves: say so, so that everything
    // picked by them - the problem's arguments above all - stays in scalar registers)
    ts.idx = __builtin_amdgcn_readfirstlane(ts.idx);
    ts.sub = __builtin_amdgcn_readfirstlane(ts.sub);
    ts.nsub = __builtin_amdgcn_readfirstlane(ts.nsub);
    const int n_s = __builtin_amdgcn_readfirstlane(rs.cnt), n_a = __builtin_amdgcn_readfirstlane(ra.cnt);
    // Position in the XCD's list -> item.  The short tiles are SPREAD evenly through the list
    // (a short tile streams its expert's weights from HBM at what one CU can pull, ~44 GB/s,
    // with the matrix pipe nearly idle: side by side with compute-bound tiles on the other CUs
    // that costs nothing but the CU; all of them together at the end or at the start of the
    // launch is a phase in which the whole chip waits for HBM - measured 36 us per short tile
    // instead of 28).  The other items keep their order: single group first, then full tiles.
    // ... except that the LAST few short tiles of the range close the list: the CUs that run out
    // of full tiles first take them while the others finish their last full tile, which fills
    // part of the idle tail of the launch with work that would otherwise sit in the middle of
    // it (few enough of them that they do not have to share HBM: FILL_TAIL per XCD).
    constexpr int FILL_TAIL = BESIDE ? 0 : 12;
    const int n_b = __builtin_amdgcn_readfirstlane(rb.cnt);
    const int n_first = EARLY ? n_s : 0;
    const int n_tail = n_b < FILL_TAIL ? n_b : FILL_TAIL, n_bi = n_b - n_tail, n_main = n_s + n_a + n_bi - n_first, idx = ts.idx - n_first;
    const bool in_tail = idx >= n_main, first_of_all = EARLY && idx < 0;
    const int b_before = first_of_all ? 0
                         : in_tail    ? n_bi + (idx - n_main)
                                      : (int)((uint32_t)idx * (uint32_t)n_bi / (uint32_t)(n_main > 0 ? n_main : 1));
    const bool is_b = !first_of_all &&
                      (in_tail || (int)(((uint32_t)idx + 1u) * (uint32_t)n_bi / (uint32_t)(n_main > 0 ? n_main : 1)) > b_before);
    const int o_rank = ts.idx - b_before;  // rank among the other items
    const bool second = !is_b && o_rank < n_s;  // workgroup-uniform: this tile is the single group's (p[1])
    GroupTile g;
    int tile_nt;
    const int tile_nsub = ts.nsub;
    if (second) {
        int mt;
        single_group_tile_at(smt, L.p[1].ntn, rs.first + o_rank, mt, tile_nt);
        g.expert = 0;
        g.row_begin = slo + mt * sbm + ts.sub * (sbm / ts.nsub);  // of this workgroup's part of the tile
        g.row_end = shi;
        if constexpr (BOTH) {
            const int b = mt * sbm / BM;
            link.mt = (ragged0 ? rmap.totalA + rmap.totalB : 0) + b;
            link.rows = shi - slo - b * BM;
        }
    } else {
        int a_rank = o_rank - n_s;
        if constexpr (BOTH && MODE == 1) {
            // The chunk of M-tiles that this XCD's share of the gate/up pass began inside of is finished by the XCD before, and
            // late: it comes last here, the first chunk that is all this XCD's own comes first.
            if (!is_b) {
                const int up_first = equal_range(rmap.totalA * link.up_ntn[0], xcd).first;
                const int skip = ragged_next_chunk(rmap, link.up_ntn[0], up_first) * L.p[0].ntn - ra.first;
                a_rank += skip > 0 && skip < ra.cnt ? skip : 0;
                if (a_rank >= ra.cnt) a_rank -= ra.cnt;
            }
        }
        const RaggedTile tr = is_b ? ragged_short_tile_at<BM>(rmap, L.p[0].ntn, rb.first + b_before)
                                   : ragged_full_tile_at<BM>(rmap, L.p[0].ntn, ra.first + a_rank);
        if (!tr.valid) return;
        if constexpr (BOTH) {
            link.mt = tr.mt;
            link.rows = tr.row_end - tr.row_begin;
        }
        g.expert = tr.expert;
        g.row_begin = tr.row_begin + ts.sub * (BM / ts.nsub);
        g.row_end = tr.row_end;
        tile_nt = tr.nt;
    }
    // the problem's arguments, uniform over the workgroup from here on
    const FfnProblemConst &P = L.p[second ? 1 : 0];  // (a scalar address: the fields are scalar loads)
    const uint16_t *__restrict__ A = P.A;
    const uint16_t *__restrict__ B0 = P.B0;
    const uint16_t *__restrict__ B1 = P.B1;
    uint16_t *__restrict__ out = P.out;
    const int32_t *__restrict__ gather = P.gather;
    const int lda = P.lda, N = P.N, Kdim = P.Kdim, ldo = P.ldo;
    const int zero_to = P.zero_to, gather_div = P.gather_div, gather_rows = P.gather_rows;
    const int n0 = tile_nt * BNF;
    int rows = g.row_end - g.row_begin;  // may exceed the tile (clamped by the row guards below)
    if (rows <= 0) return;
    const int part = (second ? sbm : BM) / tile_nsub;  // (a whole full tile's rows are clamped below)
    if (part < BM && rows > part) rows = part;
    const bool short_tile = rows <= LM;        // workgroup-uniform
    const bool tiny_tile = rows <= TM_T;
    if constexpr (BOTH) link.mt = link.mt < link.n_mtiles ? link.mt : link.n_mtiles - 1;  // (overlapping groups of a corrupt array)
    if constexpr (BOTH && MODE == 0) link.rows = rows < part ? rows : part;
    if constexpr (BOTH && MODE == 1) {
        if (!link.ready) {
            // Rows of h that another workgroup may still be writing.  The gate/up tiles have all been drawn by now, each by a workgroup
            // that is running and waits for nothing, so this ends.  The fence empties this CU's L1 and this XCD's L2 of what they may
            // hold of h; the other waves' loads come after the barrier.
            if (wave == 0) {
                const int need = (link.rows < BM ? link.rows : BM) * link.up_ntn[second ? 1 : 0];
                while (__builtin_amdgcn_readfirstlane(
                           __hip_atomic_load(&link.rows_done[link.mt * FFN_MTILE_INTS], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < need)
                    __builtin_amdgcn_s_sleep(16);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            lds_barrier();
        }
    }

    // ---- copy roles: one copy instruction fills 8 tile rows (1024 bytes); lane l lands on
    //      row l/8, chunk position l%8 and therefore fetches chunk (l%8) ^ key(row) ----
    const int lrow = lane >> 3, lpos = lane & 7;
    int chunkc[2];  // for even / odd 8-row groups (the key depends on row bits 0..3)
#pragma unroll
    for (int par = 0; par < 2; ++par) chunkc[par] = lpos ^ swz_key(par * 8 + lrow);
    // With `gather`, A is the un-permuted activation matrix and row p of the sorted order is
    // A[gather[p] / gather_div] (the dispatch gather folded into the copy addresses).
    const unsigned char *baseA =
        uniform_ptr(reinterpret_cast<const unsigned char *>(gather ? A : A + (size_t)g.row_begin * lda));
    const unsigned char *baseB0 = uniform_ptr(reinterpret_cast<const unsigned char *>(B0 + (size_t)g.expert * N * Kdim));
    const unsigned char *baseB1 =
        MODE == 0 ? uniform_ptr(reinterpret_cast<const unsigned char *>(B1 + (size_t)g.expert * N * Kdim)) : baseB0;
    uint32_t offA[GA], offB[GB], rowB[GB];
    int rowA[GA];
#pragma unroll
    for (int i = 0; i < GA; ++i) {
        const int rg = tiny_tile ? wave : short_tile ? wave * L_GA + (i < L_GA ? i : 0) : wave * GA + i;
        const int r = rg * 8 + lrow;
        rowA[i] = r < rows ? r : rows - 1;
    }
    if (gather) {
#pragma unroll
        for (int i = 0; i < GA; ++i) rowA[i] = gather[g.row_begin + rowA[i]];  // the index loads fly together
#pragma unroll
        for (int i = 0; i < GA; ++i) {
            const int r = rowA[i] > 0 ? (int)((uint32_t)rowA[i] / (uint32_t)gather_div) : 0;
            rowA[i] = r < gather_rows ? r : gather_rows - 1;  // an out-of-range entry cannot leave A
        }
    }
#pragma unroll
    for (int i = 0; i < GA; ++i) {
        const int rg = tiny_tile ? wave : short_tile ? wave * L_GA + (i < L_GA ? i : 0) : wave * GA + i;
        offA[i] = (uint32_t)rowA[i] * (uint32_t)lda * 2u + (uint32_t)chunkc[rg & 1] * 16u;
    }
#pragma unroll
    for (int i = 0; i < GB; ++i) {
        const int rg = wave * GB + i;
        int r = rg * 8 + lrow;
        if (MODE == 0 && r >= BN / 2) r -= BN / 2;
        int c = n0 + r;
        c = c < N ? c : N - 1;
        rowB[i] = (uint32_t)c * (uint32_t)Kdim * 2u;
        offB[i] = rowB[i] + (uint32_t)chunkc[rg & 1] * 16u;
    }
    // GB*8 rows per wave divide BN/2, so a wave's B rows are all gate rows or all up rows
    const unsigned char *baseB = (MODE == 0 && wave * GB * 8 >= BN / 2) ? baseB1 : baseB0;

    const int nk = (Kdim + BK - 1) / BK;
    const bool ktail = (Kdim % BK) != 0;
    // Piece p of a slice's copy: p < GA are this wave's A row groups, the rest its B groups.
    // Copies are issued one at a time between MFMAs (see slice_step): the texture-address
    // unit takes one 64-lane x 16-byte request per ~16 cycles, so a burst of all of a
    // workgroup's copies would hold every wave at its copy instructions for ~1000 cycles
    // with the matrix pipe idle.
    // `inner`: kt is known not to be the last slice (no k tail to clamp).
    auto copy_piece = [&](int kt, unsigned char *stage, int p, bool inner = false) {
        const uint32_t kb = (uint32_t)kt * ROWB;  // the slice's byte offset goes into the scalar base
        if (p < GA) {
            copy16_to_lds(baseA + kb, offA[p], stage + (wave * GA + p) * 1024);
        } else if (inner) {
            const int i = p - GA, rg = wave * GB + i;
            copy16_to_lds(baseB + kb, offB[i], stage + A_BYTES + rg * 1024);
        } else {  // a B chunk past K is taken from chunk 0: it meets A's zero padding
            const int i = p - GA, rg = wave * GB + i;
            const bool clampB = ktail && kt == nk - 1 && kt * BK + chunkc[rg & 1] * 8 >= Kdim;
            copy16_to_lds(baseB, clampB ? rowB[i] : offB[i] + kb, stage + A_BYTES + rg * 1024);
        }
    };
    constexpr int NPIECE = GA + GB;

    // v_mfma_f32_16x16x32_bf16: 16 x 16 output fragments, 32 k per instruction.  A wave owns
    // 8 x 4 of them (128 x 64 outputs); a k-step is one 32-wide k range x one 64-row half.
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int FM16 = TM / 16, FN16 = TN / 16;
    static_assert(FM16 == 8 && FN16 == 4, "k-step macros below");
    f32x4 acc[FM16][FN16];
#pragma unroll
    for (int i = 0; i < FM16; ++i)
#pragma unroll
        for (int j = 0; j < FN16; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;

    const int fr = lane & 15, fq = lane >> 4;
    uint32_t rdA[FM16], rdB[FN16];
#pragma unroll
    for (int i = 0; i < FM16; ++i) rdA[i] = (uint32_t)(wm * TM + i * 16 + fr) * ROWB;
#pragma unroll
    for (int j = 0; j < FN16; ++j) {
        int r;
        if (MODE == 0)
            r = (j < FN16 / 2) ? wn * (TN / 2) + j * 16 : BN / 2 + wn * (TN / 2) + (j - FN16 / 2) * 16;
        else
            r = wn * TN + j * 16;
        rdB[j] = (uint32_t)(tiny_tile ? T_A_BYTES : short_tile ? L_A_BYTES : A_BYTES) + (uint32_t)(r + fr) * ROWB;
    }
    const int sw = swz_key(fr);
    // waves whose whole M range lies past the group's end, or whose output columns all lie past N (the
    // last N-tile of a width that is not a multiple of the tile: 688 = 5 x 128 + 48), only help with
    // the copies: their results would be thrown away, and under the chip's power limit matrix
    // instructions on padding cost the other waves clock
    const bool cols_exist = n0 + (MODE == 0 ? wn * (TN / 2) : wn * TN) < N;  // (uniform per wave)
    const bool active = __builtin_amdgcn_readfirstlane(rows - wm * TM) > 0 && cols_exist;

    bf16x8 aset[2][4], bset[2][4];
    // A fragments of k range kq (0, 1) and 64-row half `half` into set `set`
    auto read_a = [&](const unsigned char *stage, int kq, int half, int set) {
        const uint32_t ch = (uint32_t)(((kq * 4 + fq) ^ sw) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) aset[set][i] = *reinterpret_cast<const bf16x8 *>(stage + rdA[half * 4 + i] + ch);
    };
    // the first n (wave-uniform, 1..4) of them only
    auto read_a_first = [&](const unsigned char *stage, int kq, int half, int set, int n) {
        const uint32_t ch = (uint32_t)(((kq * 4 + fq) ^ sw) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < n) aset[set][i] = *reinterpret_cast<const bf16x8 *>(stage + rdA[half * 4 + i] + ch);
    };
    auto read_b = [&](const unsigned char *stage, int kq, int set) {
        const uint32_t ch = (uint32_t)(((kq * 4 + fq) ^ sw) * 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) bset[set][j] = *reinterpret_cast<const bf16x8 *>(stage + rdB[j] + ch);
    };
    static_assert(NPIECE == 8, "copy schedule below: the A pieces in one k-step, the B pieces in another");
    // MFMAs of one k-step (operands swapped: the lane's 4 results lie along n) with up to
    // eight copy pieces P0.. of slice CKT slipped in after every second MFMA.  Macros, so that
    // every fragment and piece index is a literal and the arrays stay in registers.
#define C2R_MFMA(AS, BS, H, I, J)                                                                 \
    acc[(H) * 4 + (I)][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bset[BS][J], aset[AS][I],     \
                                                                    acc[(H) * 4 + (I)][J], 0, 0, 0)
#define C2R_MFMA_ROW(AS, BS, H, I) \
    C2R_MFMA(AS, BS, H, I, 0);     \
    C2R_MFMA(AS, BS, H, I, 1);     \
    C2R_MFMA(AS, BS, H, I, 2);     \
    C2R_MFMA(AS, BS, H, I, 3)
#define C2R_COPY_IF(Q, NCP, CKT, CST, P0)           \
    if ((Q) < (NCP)) {                              \
        __builtin_amdgcn_sched_barrier(0);          \
        copy_piece(CKT, CST, (P0) + (Q), STEADY);   \
        __builtin_amdgcn_sched_barrier(0);          \
    }
// (odd rows of fragments run through the columns backwards, so that two instructions in a row always share an operand.  It is worth little:
// layer call, every row forwards / so, 25 times in turn: 60 experts + shared, 8192 tokens 1032.4 / 1028.7 us, 1000 tokens 228.2 / 227.1, 15 of 60 experts,
// 32768 tokens 431.1 / 430.6, 16 experts of d 4096, 4096 tokens 320.8 / 320.5; the launch of 8192 tokens under counters 909.7 / 907.8, at 1.971 / 1.970 GHz with
// the matrix pipe busy 0.614 of the time either way.  Columns of fragments instead of rows: as forwards)
#define C2R_MFMA_HALF(AS, BS, H, I, J0)                  \
    C2R_MFMA(AS, BS, H, I, (J0) + ((I) & 1));            \
    C2R_MFMA(AS, BS, H, I, (J0) + 1 - ((I) & 1))
#define C2R_KSTEP(AS, BS, H, CKT, CST, P0, NCP, EARLY) \
    do {                                            \
        __builtin_amdgcn_sched_barrier(0);          \
        C2R_MFMA_HALF(AS, BS, H, 0, 0);             \
        __builtin_amdgcn_sched_barrier(0);          \
        EARLY;                                      \
        __builtin_amdgcn_sched_barrier(0);          \
        C2R_COPY_IF(0, NCP, CKT, CST, P0)           \
        C2R_MFMA_HALF(AS, BS, H, 0, 2);             \
        C2R_COPY_IF(1, NCP, CKT, CST, P0)           \
        C2R_MFMA_HALF(AS, BS, H, 1, 2);             \
        C2R_COPY_IF(2, NCP, CKT, CST, P0)           \
        C2R_MFMA_HALF(AS, BS, H, 1, 0);             \
        C2R_COPY_IF(3, NCP, CKT, CST, P0)           \
        C2R_MFMA_HALF(AS, BS, H, 2, 0);             \
        C2R_COPY_IF(4, NCP, CKT, CST, P0)           \
        C2R_MFMA_HALF(AS, BS, H, 2, 2);             \
        C2R_COPY_IF(5, NCP, CKT, CST, P0)           \
        C2R_MFMA_HALF(AS, BS, H, 3, 2);             \
        C2R_COPY_IF(6, NCP, CKT, CST, P0)           \
        C2R_MFMA_HALF(AS, BS, H, 3, 0);             \
        C2R_COPY_IF(7, NCP, CKT, CST, P0)           \
        __builtin_amdgcn_sched_barrier(0);          \
    } while (0)

    // One 64-wide slice = four k-steps.  The hand-over barrier sits before the LAST k-step:
    // by then the copy of the next slice has landed and every wave has finished reading this
    // slice's stages.  After it, the A tile of the slice after next starts going into the A
    // stage just handed over (the wave's 4 A pieces in the last k-step, one after every second
    // MFMA: as early as the stage allows, they have one slice to land in), and the first
    // fragments of the next slice are read while the last k-step's MFMAs run, so the MFMA
    // stream never starts a slice by waiting on LDS.  The B tile of the slice after next goes
    // into the ring slot that the slice BEFORE this one used, free since the previous
    // hand-over (the wave's 4 B pieces in one of the first three k-steps).
    // `steady` (a compile-time flag): kt + 3 < nk, i.e. both following slices exist and neither
    // is the last, so every copy is unconditional and unclamped: the instruction stream
    // between the MFMAs is what limits a wave that has a SIMD nearly to itself.
    auto slice_step = [&](int kt, unsigned char *cur, unsigned char *nxt, auto steady) {
        constexpr bool STEADY = decltype(steady)::value;
        static_assert(GA == 4 && GB == 4, "pieces 0..3 are the wave's A groups, 4..7 its B groups");
        const bool c1 = STEADY || kt + 1 < nk;
        const int nb = STEADY || kt + 2 < nk ? GB : 0;  // B pieces of slice kt+2, before the hand-over
        const int na = nb ? GA : 0;                      // A pieces of slice kt+2, after the hand-over
        if (active) {
            // (the first reads of a slice go out after its first two MFMAs: the compiler's wait
            // at the top of the loop body covers every LDS read in flight, and there the only
            // ones in flight should be those the first MFMAs need anyway)
            // (the B pieces have two slices to land in, so their place is free: measured, the
            // down pass likes them in the third k-step - away from the A pieces, which follow
            // the hand-over - by 2-3 %, the gate/up pass in the first by 1 %)
            constexpr int BSTEP = MODE == 1 ? 2 : 0;
            C2R_KSTEP(0, 0, 0, kt + 2, bwr, GA, (BSTEP == 0 ? nb : 0), read_a(cur, 0, 1, 1));
            read_a(cur, 1, 0, 0);
            read_b(bcur, 1, 1);
            C2R_KSTEP(1, 0, 1, kt + 2, bwr, GA, (BSTEP == 1 ? nb : 0), (void)0);
            read_a(cur, 1, 1, 1);
            C2R_KSTEP(0, 1, 0, kt + 2, bwr, GA, (BSTEP == 2 ? nb : 0), (void)0);
        } else if (nb) {
            copy_piece(kt + 2, bwr, 4, STEADY);
            copy_piece(kt + 2, bwr, 5, STEADY);
            copy_piece(kt + 2, bwr, 6, STEADY);
            copy_piece(kt + 2, bwr, 7, STEADY);
        }
        // my copies of slice kt+1 (A: issued after the previous hand-over, B: a slice earlier
        // still) have landed once at most the B pieces of slice kt+2 are outstanding; my reads of
        // this slice's stages have returned
        if (nb)
            wait_copies_but_and_lds<GB>();
        else
            wait_copies_and_lds();
        lds_barrier();
        if (active) {
            if (c1) {
                read_a(nxt, 0, 0, 0);
                read_b(bnxt, 0, 0);
            }
            C2R_KSTEP(1, 1, 1, kt + 2, cur, 0, na, (void)0);
        } else if (na) {
            copy_piece(kt + 2, cur, 0, STEADY);
            copy_piece(kt + 2, cur, 1, STEADY);
            copy_piece(kt + 2, cur, 2, STEADY);
            copy_piece(kt + 2, cur, 3, STEADY);
        }
        unsigned char *const freed = bcur;  // every wave has read it: the slot of slice kt+3
        bcur = bnxt;
        bnxt = bwr;
        bwr = freed;
    };

    if (tiny_tile) {
        // ---- tiny tile: four-stage ring, three slices in flight, one barrier per slice ----
        static_assert(GB == 4, "five copies per wave per slice below");
        auto tiny_copy = [&](int kt) {
            unsigned char *stage = smem + (kt & (T_NSTAGE - 1)) * T_STAGE_BYTES;
            const uint32_t kb = (uint32_t)kt * ROWB;
            copy16_to_lds(baseA + kb, offA[0], stage + wave * 1024);
            const bool last = ktail && kt == nk - 1;
            const bool clamp0 = last && kt * BK + chunkc[0] * 8 >= Kdim, clamp1 = last && kt * BK + chunkc[1] * 8 >= Kdim;
            unsigned char *sb = stage + T_A_BYTES + wave * GB * 1024;
            copy16_to_lds(baseB, clamp0 ? rowB[0] : offB[0] + kb, sb);
            copy16_to_lds(baseB, clamp1 ? rowB[1] : offB[1] + kb, sb + 1024);
            copy16_to_lds(baseB, clamp0 ? rowB[2] : offB[2] + kb, sb + 2048);
            copy16_to_lds(baseB, clamp1 ? rowB[3] : offB[3] + kb, sb + 3072);
        };
        const int nf = (rows + 15) >> 4;  // 1..4 fragments of 16 rows hold rows of the group
        tiny_copy(0);
        if (nk > 1) tiny_copy(1);
        if (nk > 2) tiny_copy(2);
        for (int kt = 0; kt < nk; ++kt) {
            // slice kt has landed once at most the copies of slices kt+1 and kt+2 are outstanding
            if (kt + 2 < nk)
                wait_copies_but_and_lds<10>();
            else if (kt + 1 < nk)
                wait_copies_but_and_lds<5>();
            else
                wait_copies_but_and_lds<0>();
            lds_barrier();  // every wave's reads of slice kt-1 have returned: its stage is free
            if (kt == 0) under_way();
            if (kt + 3 < nk) tiny_copy(kt + 3);
            if (wm == 0 && cols_exist) {
                const unsigned char *stage = smem + (kt & (T_NSTAGE - 1)) * T_STAGE_BYTES;
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) {
                    read_b(stage, kq, 0);
                    read_a_first(stage, kq, 0, 0, nf);
                    C2R_MFMA_ROW(0, 0, 0, 0);
                    if (nf > 1) { C2R_MFMA_ROW(0, 0, 0, 1); }
                    if (nf > 2) { C2R_MFMA_ROW(0, 0, 0, 2); }
                    if (nf > 3) { C2R_MFMA_ROW(0, 0, 0, 3); }
                }
            }
        }
    } else if (short_tile) {
        // ---- short tile: three-stage ring, two slices in flight, one barrier per slice ----
        static_assert(L_GA == 2 && GB == 4, "six copies per wave per slice below");
        auto short_copy = [&](int kt) {
            unsigned char *stage = smem + (kt % L_NSTAGE) * L_STAGE_BYTES;
            const uint32_t kb = (uint32_t)kt * ROWB;
            copy16_to_lds(baseA + kb, offA[0], stage + (wave * L_GA + 0) * 1024);
            copy16_to_lds(baseA + kb, offA[1], stage + (wave * L_GA + 1) * 1024);
            const bool last = ktail && kt == nk - 1;
            const bool clamp0 = last && kt * BK + chunkc[0] * 8 >= Kdim, clamp1 = last && kt * BK + chunkc[1] * 8 >= Kdim;
            unsigned char *sb = stage + L_A_BYTES + wave * GB * 1024;  // wave * GB is even: groups alternate parity
            copy16_to_lds(baseB, clamp0 ? rowB[0] : offB[0] + kb, sb);
            copy16_to_lds(baseB, clamp1 ? rowB[1] : offB[1] + kb, sb + 1024);
            copy16_to_lds(baseB, clamp0 ? rowB[2] : offB[2] + kb, sb + 2048);
            copy16_to_lds(baseB, clamp1 ? rowB[3] : offB[3] + kb, sb + 3072);
        };
        // Only the 16-row fragments that hold rows of the group are computed: most short tiles
        // belong to experts with a handful of tokens, the chip is power limited, and matrix
        // instructions on padding rows cost the other workgroups clock.
        const int nf = (rows + 15) >> 4;  // 1..8, workgroup-uniform
        short_copy(0);
        if (nk > 1) short_copy(1);
        for (int kt = 0; kt < nk; ++kt) {
            // slice kt has landed once at most the copies of slice kt+1 are outstanding; every
            // wave's reads of slice kt-1 have returned, so its stage may be refilled
            if (kt + 1 < nk)
                wait_copies_but_and_lds<6>();
            else
                wait_copies_but_and_lds<0>();
            lds_barrier();
            if (kt == 0) under_way();
            if (kt + 2 < nk) short_copy(kt + 2);
            if (wm == 0 && cols_exist) {
                const unsigned char *stage = smem + (kt % L_NSTAGE) * L_STAGE_BYTES;
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) {
                    read_b(stage, kq, 0);
                    read_a_first(stage, kq, 0, 0, nf);
                    C2R_MFMA_ROW(0, 0, 0, 0);
                    if (nf > 1) { C2R_MFMA_ROW(0, 0, 0, 1); }
                    if (nf > 2) { C2R_MFMA_ROW(0, 0, 0, 2); }
                    if (nf > 3) { C2R_MFMA_ROW(0, 0, 0, 3); }
                    if (nf > 4) {
                        read_a_first(stage, kq, 1, 1, nf - 4);
                        C2R_MFMA_ROW(1, 0, 1, 0);
                        if (nf > 5) { C2R_MFMA_ROW(1, 0, 1, 1); }
                        if (nf > 6) { C2R_MFMA_ROW(1, 0, 1, 2); }
                        if (nf > 7) { C2R_MFMA_ROW(1, 0, 1, 3); }
                    }
                }
            }
        }
    } else {
        copy_piece(0, st0, 0);
        copy_piece(0, st0, 1);
        copy_piece(0, st0, 2);
        copy_piece(0, st0, 3);
        copy_piece(0, bcur, 4);
        copy_piece(0, bcur, 5);
        copy_piece(0, bcur, 6);
        copy_piece(0, bcur, 7);
        // every stage is free at the start of a tile: slice 1 goes out right behind slice 0
        if (nk > 1) {
            copy_piece(1, st1, 0);
            copy_piece(1, st1, 1);
            copy_piece(1, st1, 2);
            copy_piece(1, st1, 3);
            copy_piece(1, bnxt, 4);
            copy_piece(1, bnxt, 5);
            copy_piece(1, bnxt, 6);
            copy_piece(1, bnxt, 7);
            wait_copies_but<8>();  // slice 0 has landed
        } else {
            wait_copies_but<0>();
        }
        lds_barrier();
        under_way();
        if (active) {
            read_a(st0, 0, 0, 0);
            read_b(bcur, 0, 0);
        }
        int kt = 0;
        for (; kt + 4 < nk; kt += 2) {  // both slices of the pair are followed by two inner slices
            slice_step(kt, st0, st1, std::true_type{});
            slice_step(kt + 1, st1, st0, std::true_type{});
        }
        for (; kt < nk; kt += 2) {
            slice_step(kt, st0, st1, std::false_type{});
            if (kt + 1 >= nk) break;
            slice_step(kt + 1, st1, st0, std::false_type{});
        }
        wait_copies_but<0>();
    }
#undef C2R_KSTEP
#undef C2R_COPY_IF
#undef C2R_MFMA_ROW
#undef C2R_MFMA

    before_epilogue();
    // ---- epilogue.  Fragment (i, j) holds C^T: lane (fr, fq), register v is
    //      row m = i*16 + fr, column n = j*16 + 4*fq + v.  Every wave of the workgroup is
    //      here at once with the matrix pipe idle, so the common case (all of the tile's
    //      columns exist) is kept short: hardware bf16 conversion, no per-element guards, and
    //      whole rows per store instruction (measured: routed down pass 227 -> 210 us against
    //      8-byte stores straight from the fragments). ----
    constexpr int FJ = MODE == 0 ? FN16 / 2 : FN16;
    const int col0 = n0 + (MODE == 0 ? wn * (TN / 2) : wn * TN);
    if (n0 + BNF <= N) {
        // The wave's 128 x (FJ*16) results go through a private piece of the (now idle) stage
        // memory so that they leave as whole rows: a lane's 8-byte fragment pieces would be
        // 16 separate 32-byte requests per store instruction, the rows read back are 8 (or
        // 4) lanes x 16 bytes = one contiguous 128 (64) bytes each.
        constexpr int ROW_BYTES = FJ * 16 * 2, PITCH = ROW_BYTES + 16;
        constexpr int LPR = ROW_BYTES / 16, RPI = 64 / LPR;  // lanes per row, rows per store instruction
        static_assert(NW * TM * PITCH <= SMEM_BYTES, "staging fits the stage memory");
        if (short_tile) {  // the ring may still be read by a slower wave
            wait_copies_but_and_lds<0>();
            lds_barrier();
        }
        unsigned char *stg = smem + wave * (TM * PITCH);
        const int rlim = rows - wm * TM;  // rows of this wave's M range that exist
#pragma unroll
        for (int i = 0; i < FM16; ++i) {
            if (i * 16 < rlim) {  // wave-uniform: skip fragment rows wholly past the end
#pragma unroll
                for (int j = 0; j < FJ; ++j) {
                    float v4[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        v4[u] = MODE == 0 ? silu_mul(acc[i][j][u], acc[i][j + FN16 / 2][u]) : acc[i][j][u];
                    *reinterpret_cast<uint2 *>(stg + (i * 16 + fr) * PITCH + (j * 16 + fq * 4) * 2) =
                        make_uint2(pack_bf16x2(v4[0], v4[1]), pack_bf16x2(v4[2], v4[3]));
                }
            }
        }
        const int srow = lane / LPR, chunk = lane % LPR;
        uint16_t *o = out + ((size_t)g.row_begin + wm * TM + srow) * ldo + col0 + chunk * 8;
#pragma unroll
        for (int r0 = 0; r0 < TM; r0 += RPI) {
            if (r0 + srow < rlim) {
                const uint4 q = *reinterpret_cast<const uint4 *>(stg + (r0 + srow) * PITCH + chunk * 16);
                if constexpr (BOTH && MODE == 0)
                    store16_through(o, q);
                else
                    *reinterpret_cast<uint4 *>(o) = q;
            }
            o += (size_t)RPI * ldo;
        }
        return;
    }
    uint16_t *outb = out + (size_t)g.row_begin * ldo;
#pragma unroll
    for (int i = 0; i < FM16; ++i) {
        const int r = wm * TM + i * 16 + fr;
        if (r >= rows) continue;
#pragma unroll
        for (int j = 0; j < FJ; ++j) {
            const int col = col0 + j * 16 + fq * 4;
            uint2 pk = make_uint2(0, 0);
            auto store = [&]() __attribute__((always_inline)) {
                uint16_t *o = outb + (size_t)r * ldo + col;
                if constexpr (BOTH && MODE == 0)
                    __hip_atomic_store(reinterpret_cast<uint64_t *>(o), (uint64_t)pk.x | ((uint64_t)pk.y << 32), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                else
                    *reinterpret_cast<uint2 *>(o) = pk;
            };
            if (col >= N) {
                // pass 0 keeps the padding columns of h at zero for pass 1's k tail
                if (col < zero_to) store();
                continue;
            }
            float v4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v4[u] = MODE == 0 ? silu_mul(acc[i][j][u], acc[i][j + FN16 / 2][u]) : acc[i][j][u];
            pk.x = pack_bf16x2(v4[0], v4[1]);
            pk.y = pack_bf16x2(v4[2], v4[3]);
            store();
        }
    }
}

// Work queues of the launches in flight: per launch one set of 8 ticket counters (one per XCD)
// and a count of the workgroups that have left.  All zero between launches: the last workgroup
// to leave a launch clears the set it used.  The host hands the sets out round-robin, so up to
// FFN_QUEUE_SETS launches of this kernel may be in flight on a GPU at once (on any streams).
// A launch of both passes has 8 more ticket counters for the second, the number of gate/up tiles that are finished, and per M-tile
// the rows of h that are, summed over its N-tiles.
// Every counter that the workgroups of one XCD use most has a 128-byte line of its own: atomics of several XCDs on one line wait for each
// other, and a workgroup's next tile for them.  (M-tiles next to each other are mostly one XCD's: four to a line.)  Microseconds, all in one line
// and its neighbours / so, one after the other in one process: the joint launch, 60 experts + shared, 420 tokens 166.4 / 161.0, 1000 tokens 210.3 /
// 203.4; 16 experts of d 4096, 4096 tokens 278.0 / 267.2; 8 experts, 2000 tokens 162.4 / 153.1; the layer call of the four 182.3 / 175.0, 226.1 / 222.0,
// 325.2 / 318.9, 187.8 / 175.6, 8192 tokens of the first 1045 / 1035.
constexpr int FFN_MTILES = 1024;
constexpr int FFN_LEFT = 8 * FFN_LINE, FFN_FINISHED = 9 * FFN_LINE, FFN_DOWN = 10 * FFN_LINE, FFN_ROWS_DONE = 18 * FFN_LINE;
constexpr int FFN_QUEUE_SETS = 64, FFN_QUEUE_INTS = 9 * FFN_LINE, FFN_BOTH_INTS = FFN_ROWS_DONE + FFN_MTILES * FFN_MTILE_INTS;
__device__ __attribute__((aligned(128))) int ffn_queues[FFN_QUEUE_SETS * (FFN_QUEUE_INTS + FFN_BOTH_INTS)];  // those of one pass, then those of both

// What stays the same for a workgroup while it walks the lists of one pass, or of both.
struct FfnWalk {
    unsigned char *smem;
    int *queues;
    // every wave keeps the row range of "its lane's" expert of the ragged problem (the tile
    // lookup is wave-wide arithmetic on them; they do not change during the launch)
    int grp_lo, grp_hi;
    int sg_lo, sg_hi;  // the single group's row range (two scalars)
    int up_slots;      // both passes: positions of all the lists of the first
    int ticket;        // and (lane 0 of the first wave) the first ticket of the workgroup's own list of the pass
    int n_mtiles;      // and the M-tiles that there are counters for
    int early;         // EARLY: the position of a down tile that comes before the gate/up tiles that are left; -1: none is left
    bool holds;        // EARLY: `ticket` is of the second pass already
};

__device__ __forceinline__ void ffn_walk_init(FfnWalk &w, const FfnLaunch &L) {
    w.grp_lo = w.grp_hi = w.sg_lo = w.sg_hi = w.up_slots = 0;
    if (L.has_ragged) load_group_range(L.p[0].offsets, L.p[0].E_local, L.p[0].A_cap, w.grp_lo, w.grp_hi);
    if (L.has_single) {
        int lo = L.p[1].offsets ? L.p[1].offsets[0] : L.p[1].row_lo;
        int hi = L.p[1].offsets ? L.p[1].offsets[1] : L.p[1].row_hi;
        lo = lo < 0 ? 0 : (lo > L.p[1].A_cap ? L.p[1].A_cap : lo);
        hi = hi < lo ? lo : (hi > L.p[1].A_cap ? L.p[1].A_cap : hi);
        w.sg_lo = __builtin_amdgcn_readfirstlane(lo);
        w.sg_hi = __builtin_amdgcn_readfirstlane(hi);
    }
}

// One workgroup's way through the lists of a pass: tiles until none are left.
// KERNARG: where the pass's FfnLaunch lies in the kernel-argument segment.
// EARLY: the first pass ends (for now) as well where a down tile of the single group comes next, and the second walks that one alone.
// down_single: the single group's tiles in the down pass; begin: the first pass is entered for the first time.
constexpr int FFN_NEVER = 0x7fffffff;
template <int MODE, int WM, int WN, bool BOTH, bool EARLY, int KERNARG>
__device__ __forceinline__ void ffn_walk_lists(FfnWalk &W, const FfnLaunch &L, const int up_ntn_ragged, const int up_ntn_single,
                                               const int down_single, const bool begin) {
    typedef FfnShape<WM, WN> S;
    int *const queues = W.queues + (BOTH && MODE == 1 ? FFN_DOWN : 0);
    // The claimed position (XCD of the list, slot; -1: nothing left) is handed to the waves in
    // the last bytes of the stage memory, which is all of the CU's LDS: every layout of a tile
    // writes them only after its first hand-over barrier (the third weight stage of a full
    // tile, the fourth ring stage of a tiny one; a short tile never does), and no wave gets
    // there before every wave has read the claim.
    int *const claim = reinterpret_cast<int *>(W.smem + S::SMEM_BYTES - 64);
    const int tid = threadIdx.x, lane = tid & 63;
    const int home = (int)(blockIdx.x & 7);
    // the first wave works the queues; its lane x < 8 keeps the number of slots of XCD x's list
    int my_len = 0, my_single = 0;
    // EARLY: the position of its own list from which on a workgroup takes the single group's down tiles, of which its XCD has n_early:
    // all positions that start along with the last round of that group's gate/up tiles are handed out then, and those tiles nearly finished
    int early_from = FFN_NEVER, n_early = 0;
    if (tid < 64) {
        const int n_s = (W.sg_hi - W.sg_lo + L.single_rows - 1) / L.single_rows * (L.has_single ? L.p[1].ntn : 0);
        int totA = 0, totB = 0;
        if (L.has_ragged) {
            const RaggedMap m = ragged_map_of<S::BM>(W.grp_lo, W.grp_hi);
            totA = m.totalA * L.p[0].ntn;
            totB = m.totalB * L.p[0].ntn;
        }
        const int x = lane & 7;
        my_single = equal_range(n_s, x).cnt;
        const int my_tiles = my_single + equal_range(totA, x).cnt + equal_range(totB, x).cnt;
        my_len = xcd_list_slots<BOTH && MODE == 0>(my_tiles);
        if (BOTH && MODE == 0) {
            W.up_slots = 0;
            for (int i = 0; i < 8; ++i) W.up_slots += __builtin_amdgcn_readlane(my_len, i);
        }
        if (EARLY && MODE == 0) {
            const int n = __builtin_amdgcn_readlane(my_single, home);
            const int from = 2 * ((n + CUS_PER_XCD - 1) / CUS_PER_XCD * CUS_PER_XCD) - n;
            n_early = equal_range(down_single, home).cnt;
            if (n_early > 0 && from < __builtin_amdgcn_readlane(my_len, home)) early_from = from;
            if (my_single > my_tiles / CUS_PER_XCD * CUS_PER_XCD) my_single = my_len;  // (some of them are cut into parts)
        }
    }
    // The first position of every workgroup is its own number in its XCD (no trip to the counter
    // before the first tile); the counters hand out what lies beyond those.  Not so where a pass waits for the other:
    // there a position must never be one's whose workgroup has not started (two such launches on two streams, each holding the
    // CUs that the other's last workgroups need, would wait for ever).  Its first tickets are drawn while the groups' ranges
    // are loaded, and while the last stores of the gate/up pass are under way.
    constexpr bool OWN_FIRST = !BOTH;
    auto beyond = [](int x) { return OWN_FIRST ? ((int)gridDim.x - x + 7) >> 3 : 0; };
    int q = home;        // the queue this workgroup draws from: its own XCD's until that is empty
    // (lane 0 of the first wave) a ticket of queue q drawn ahead
    int ticket = OWN_FIRST ? (int)(blockIdx.x >> 3) : EARLY && MODE == 1 && W.early >= 0 ? W.early : W.ticket;
    bool drawn = !(EARLY && MODE == 0) || begin;  // such a ticket is at hand
    bool first = true;
    FfnTileLink link;
    link.ready = false;
    link.up_ntn[0] = up_ntn_ragged;
    link.up_ntn[1] = up_ntn_single;
    link.n_mtiles = W.n_mtiles;
    link.rows_done = W.queues + FFN_ROWS_DONE;
    // gate/up beside down: the tile whose stores are under way, and the positions that are done with since the last post
    int done_mt = -1, done_rows = 0, done_slots = 0;
    auto post = [&]() {
        if constexpr (BOTH && MODE == 0) {
            asm volatile("" ::: "memory");
            if (tid == 0 && done_slots > 0) {
                if (done_mt >= 0) atomicAdd(&W.queues[FFN_ROWS_DONE + done_mt * FFN_MTILE_INTS], done_rows);
                atomicAdd(&W.queues[FFN_FINISHED], done_slots);
            }
            done_mt = -1;
            done_slots = 0;
        }
    };
    for (;;) {
        if (tid < 64) {
            // Every trip ends by checking the ticket it holds, so no valid ticket is ever dropped.
            // A ticket that comes back past the end of its list (another workgroup was faster) makes
            // that list look empty from then on, so at most one draw per list fails: 9 trips at most.
            int t = -1, early = -1;
            bool have = drawn;  // the ticket drawn during the last epilogue, or the static first one
            drawn = false;
            for (int tries = 0; tries < 16; ++tries) {
                if (!have) {
                    // Look before drawing: one coherent read of the eight counters tells which lists
                    // still hold something (counters only grow, so "empty" is final), and a workgroup
                    // that finds them all empty leaves at once - drawing from eight empty queues one
                    // after the other cost 15 us at the end of every launch.
                    const int x = lane & 7;
                    const int *counter = &queues[x * FFN_LINE];
                    if (EARLY && MODE == 0 && lane >= 8) counter = &queues[FFN_DOWN + home * FFN_LINE];
                    const int seen = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + beyond(x);
                    if (EARLY && MODE == 0 && early_from != FFN_NEVER) {
                        // A down tile may wait for the single group's gate/up tiles once all of those are drawn, each by a workgroup that
                        // runs and waits for nothing before it has finished them.
                        if (__builtin_amdgcn_readlane(seen, 8) >= n_early) {
                            early_from = FFN_NEVER;
                        } else if (__builtin_amdgcn_readlane(seen, home) >= early_from && __ballot(lane < 8 && seen < my_single) == 0) {
                            if (lane == 0) ticket = atomicAdd(&queues[FFN_DOWN + home * FFN_LINE], 1);
                            early = __builtin_amdgcn_readfirstlane(ticket);
                            if (early < n_early) break;
                            W.ticket = early;  // (another workgroup was faster: it is this one's first of the down pass)
                            W.holds = true;
                            early = -1;
                            early_from = FFN_NEVER;
                        }
                    }
                    const uint32_t avail = (uint32_t)__ballot(lane < 8 && seen < my_len) & 0xffu;
                    if (avail == 0) break;  // (t is -1)
                    // own XCD's list first, then the next one (cyclically) that holds something
                    const uint32_t rot = ((avail >> q) | (avail << (8 - q))) & 0xffu;
                    q = (q + __builtin_ctz(rot)) & 7;
                    if (lane == 0) ticket = atomicAdd(&queues[q * FFN_LINE], 1) + beyond(q);
                }
                have = false;
                t = __builtin_amdgcn_readfirstlane(ticket);
                if (t < __builtin_amdgcn_readlane(my_len, q)) break;
                t = -1;
            }
            if (BOTH && MODE == 1 && !link.ready && !first && t >= 0) {  // (it seldom is at the first: one trip less)
                const int n = __hip_atomic_load(&W.queues[FFN_FINISHED], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                link.ready = __builtin_amdgcn_readfirstlane(n) >= W.up_slots;
                if (link.ready) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            first = false;
            if (lane == 0) {
                claim[0] = q;
                claim[1] = t;
                if (EARLY && MODE == 0) claim[2] = early;
                if (BOTH && MODE == 1) claim[2] = link.ready ? 1 : 0;
            }
        }
        wait_lds_only();
        lds_barrier();  // the claim is visible
        q = __builtin_amdgcn_readfirstlane(claim[0]);
        const int slot = __builtin_amdgcn_readfirstlane(claim[1]);
        if (slot < 0) {  // every queue is empty, or a down tile comes first
            if (EARLY && MODE == 0) W.early = __builtin_amdgcn_readfirstlane(claim[2]);
            if (BOTH && MODE == 0 && tid == 0 && !(EARLY && (W.early >= 0 || W.holds)))
                W.ticket = atomicAdd(&W.queues[FFN_DOWN + home * FFN_LINE], 1);
            break;
        }
        if (BOTH && MODE == 1) link.ready = __builtin_amdgcn_readfirstlane(claim[2]) != 0;
        // The launch arguments are re-read per tile through a pointer the compiler cannot see
        // through: held in registers across the tile they are ~50 scalars too many.
        FfnLaunchArgs Lp = (FfnLaunchArgs)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + KERNARG);
        asm volatile("" : "+s"(Lp));
        drawn = false;
        link.mt = -1;
        bool begun = false;
        ffn_tile<MODE, WM, WN, BOTH, EARLY>(
            Lp, W.smem, q, slot, W.grp_lo, W.grp_hi, W.sg_lo, W.sg_hi, link, post,
            [&]() {
                // the next ticket of the same queue, drawn while the epilogue runs (but none where a down tile may come first)
                begun = true;
                drawn = !EARLY || (MODE == 0 ? q != home || slot + CUS_PER_XCD < early_from : W.early < 0);
                if (tid == 0 && drawn) ticket = atomicAdd(&queues[q * FFN_LINE], 1) + beyond(q);
            });
        if (BOTH && MODE == 0) {
            if (begun) {  // (else the position held nothing, and what was to be posted still is)
                done_mt = link.mt;
                done_rows = link.rows;
            }
            ++done_slots;
        }
        // This wave's LDS reads have returned; then every wave's: the next claim and the next tile's
        // copies may overwrite the stages.  The epilogue's stores are NOT waited for (a workgroup
        // that ends does not wait for its stores either): they drain while the next tile is looked
        // up and its first slices are requested.  The copy waits of the next tile stay correct with
        // stores in flight: they ask for "at most N operations outstanding", and what is older completes
        // first, so stores still in flight only make a wait longer.  Beside the down pass more rests on that
        // order: the first slice's wait is what the stores of h are known to be complete by (see ffn_tile).
        wait_lds_only();
        lds_barrier();
        if (EARLY && MODE == 1 && W.early >= 0) break;
    }
    if (BOTH && MODE == 0) {  // no tile follows whose first slice the last stores could be posted behind
        wait_copies_but<0>();
        lds_barrier();
        post();
    }
}

// The last workgroup to leave clears the set for the launch that gets it next
// (this workgroup's draws have all returned - their values were used - so they precede the
// count below; no fence: a device-scope release would write the XCD's whole L2 back)
__device__ __forceinline__ bool ffn_last_to_leave(int *queues) {
    return atomicAdd(&queues[FFN_LEFT], 1) == (int)gridDim.x - 1;
}

// The kernel: one workgroup per CU, each pulling tiles until none are left.  The hardware hands
// workgroups out strictly in order, the k-th of an XCD to shader engine k mod 4 - measured: a CU
// freed early by a short tile stayed empty for 100 us behind a workgroup that waited for a CU
// of ANOTHER engine - so with one workgroup per tile every tile shorter than its neighbours
// left a bubble, and the ragged groups' tiles differ by a factor of six.  Here the list of an
// XCD (ffn_common.h) is a queue: a ticket counter in device memory that the workgroups of that
// XCD draw from (the L2 locality of the list is kept), and a workgroup whose own XCD has
// nothing left draws from the others'.
template <int MODE, int WM, int WN>
__global__ __launch_bounds__(WM *WN * 64) void ffn_bf16_dma_kernel(const FfnLaunch L, int *__restrict__ queues) {
    typedef FfnShape<WM, WN> S;
    static_assert(S::SMEM_BYTES <= 160 * 1024, "one workgroup per CU owns all of its LDS");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[S::SMEM_BYTES];
    FfnWalk W;
    W.smem = smem;
    W.queues = queues;
    W.n_mtiles = W.ticket = 0;
    W.early = -1;
    W.holds = false;
    ffn_walk_init(W, L);
    ffn_walk_lists<MODE, WM, WN, false, false, 0>(W, L, 0, 0, 0, true);
    if (threadIdx.x == 0 && ffn_last_to_leave(queues))
        for (int i = 0; i <= FFN_LEFT; i += FFN_LINE) atomicExch(&queues[i], 0);
}

// Both passes in one launch: a workgroup that finds no gate/up tile left goes on with the down pass instead of idling until the
// last one is finished.  With tiles as long as a third of a pass the workgroups of a pass end up to a tile apart (idle per CU at the end of the
// gate/up pass, microseconds: 60 experts + shared, 1000 tokens 21 of 129, 16 experts of d 4096, 4096 tokens 28 of 170, 15 of 60 experts, 32768
// tokens 21 of 202), and a launch begins with all of them at once.  A down tile waits until all the gate/up tiles of its rows are
// finished; the order of the lists makes that rare (1 to 5 us per CU).  h is written through to the memory that all XCDs share (store16_through),
// counted per M-tile once a barrier behind the stores' completion has been passed, and read after the reader's caches are emptied.
// Layer call of the three, two launches / this: 254 / 231, 360 / 331, 469 / 439; 8192 tokens of the first, which the power limit bounds,
// are even.  Starting the down lists where the share begins instead of at the XCD's first own chunk: 230.3 against 228.2, 336 against 330.5, 446
// against 435; short gate/up tiles last, as in a launch of their own: 334.9 against 330.5 for the second.
//
// EARLY: a shared expert's down tiles (88 k-slices, three to five times the others' length) are what the launch ends with if they come after all
// gate/up tiles.  Here they come after its own gate/up tiles, which are the first of all, and the routed gate/up tiles beside and after them.
// Traced at 420 tokens of 60 experts + shared: they ran from 64-97 us to 171-174, the workgroups' ends 127 to 174, 144 on average; so from 56-78 to
// 144-148, the ends 119 to 150, 132 on average.
template <int WM, int WN, bool EARLY>
__global__ __launch_bounds__(WM *WN * 64) void ffn_bf16_dma_both_kernel(const FfnBothLaunch L, int *__restrict__ queues, int n_mtiles) {
    typedef FfnShape<WM, WN> S;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[S::SMEM_BYTES];
    FfnWalk W;
    W.smem = smem;
    W.queues = queues;
    W.n_mtiles = n_mtiles;
    W.ticket = 0;
    W.early = -1;
    W.holds = false;
    if (threadIdx.x == 0) W.ticket = atomicAdd(&queues[(blockIdx.x & 7) * FFN_LINE], 1);
    ffn_walk_init(W, L.pass[0]);
    const FfnLaunch &D = L.pass[1];
    const int down_single = EARLY && D.has_single ? (W.sg_hi - W.sg_lo + D.single_rows - 1) / D.single_rows * D.p[1].ntn : 0;
    bool begin = true;
    do {
        ffn_walk_lists<0, WM, WN, true, EARLY, 0>(W, L.pass[0], 0, 0, down_single, begin);
        ffn_walk_lists<1, WM, WN, true, EARLY, (int)sizeof(FfnLaunch)>(W, D, L.pass[0].p[0].ntn, L.pass[0].p[1].ntn, 0, false);
        begin = false;
    } while (EARLY && W.early >= 0);
    if (threadIdx.x < 64) {
        wait_copies_but<0>();  // (what this workgroup posted has arrived)
        int last = 0;
        if (threadIdx.x == 0) last = ffn_last_to_leave(queues) ? 1 : 0;
        if (__builtin_amdgcn_readfirstlane(last))
            for (int i = threadIdx.x * FFN_MTILE_INTS; i < FFN_ROWS_DONE + n_mtiles * FFN_MTILE_INTS; i += 64 * FFN_MTILE_INTS)
                __hip_atomic_store(&queues[i], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// One problem of a pass.  pass 0: a = x_perm [A_cap, d] (d % 64 == 0) or, with gather, x [T, d];
// out = h with row pitch ldo >= F, columns [F, ldo) zeroed.  pass 1: a = h (pitch lda, zero
// padded to 64), out = y_perm.  offsets == nullptr: one group, rows [0, A_cap).
FfnProblem ffn_bf16_dma_problem(int pass, const uint16_t *a, int lda, const int32_t *offsets, int E_local,
                                int64_t A_cap, int d, int F, const uint16_t *b0, const uint16_t *b1, uint16_t *out,
                                int ldo, const int32_t *gather, int gather_div, int gather_rows) {
    constexpr int BN = 256;
    FfnProblem P;
    P.A = a;
    P.offsets = offsets;
    P.B0 = b0;
    P.B1 = pass == 0 ? b1 : nullptr;
    P.out = out;
    P.gather = pass == 0 ? gather : nullptr;
    P.lda = lda;
    P.E_local = E_local;
    P.A_cap = (int)A_cap;
    P.N = pass == 0 ? F : d;
    P.Kdim = pass == 0 ? d : F;
    P.ldo = ldo;
    P.ntn = pass == 0 ? (ldo + BN / 2 - 1) / (BN / 2) : (d + BN - 1) / BN;
    P.zero_to = pass == 0 ? ldo : 0;
    P.gather_div = pass == 0 ? gather_div : 1;
    P.gather_rows = pass == 0 ? gather_rows : 1;
    P.row_lo = 0;
    P.row_hi = (int)A_cap;
    return P;
}

bool ffn_skinny_takes(int pass, const FfnLaunch &L);
bool ffn_skinny_takes_few(FfnLaunch L);
int launch_ffn_skinny(int pass, const FfnLaunch &L, const FewRoute *few, hipStream_t st);
bool ffn_mid_rows(int pass, const FfnLaunch &L, int likely, int (&rows)[2]);
bool ffn_mid_in_one_round(const FfnProblem &down, int rows);
int launch_ffn_mid(int pass, const int (&tile_rows)[2], FfnLaunch L, hipStream_t st);

// Rows of the single group's tiles.  Fewer tiles than a quarter of the CUs, each a chain of k-slices much longer than those
// beside it, are what a launch then waits for (a shared expert's down pass: 88 slices, 120 us, against 22): cut lower, the
// same tiles are more, and shorter too (a 64-row tile has three slices in flight instead of one).  Microseconds of a layer
// call with 256 / 128 / 64 rows in the down pass (60 experts + shared, d 2048, F 1408 / 5632): 600 tokens 261 / 248 / 217,
// 1000 tokens 290 / 270 / 255, 1300 tokens 316 / 301 / 311, 1600 tokens 340 / 320 / 347, 2000 tokens 379 / 374 / 399, 2500
// tokens 416 / 431 / 456 (every part reads the weights again).  In the gate/up pass, whose chains are alike, it only costs:
// 1000 tokens 290 -> 304 with 128 rows.  A group that runs alone gains from the cut in either pass if its own contraction is
// long: with 256 rows / by this rule, gate/up of d 4096, F 1344: 256 rows 50.7 / 42.1, 600 rows 52.0 / 45.6, 1000 rows 53.8 / 53.9;
// d 2048, F 1408: 256 rows 29.0 / 26.2; d 1024, F 512: 256 rows 18.0 / 15.3, 600 rows 18.3 / 17.8, 1000 rows 18.9 / 20.1; down, d 2048: F
// 5632: 600 rows 64.3 / 54.5; F 1408: 600 rows 22.4 / 21.4.  Below 1024 it does not: down of d 1024, F 512: 600 rows 12.8 / 13.9, 1000 rows
// 13.0 / 16.5.
static int single_tile_rows(const FfnProblem *ragged, const FfnProblem *single) {
    constexpr int BM = 256;
    if (!single || single->Kdim < (ragged ? 2 * ragged->Kdim : 1024)) return BM;
    const int64_t tiles = ((int64_t)single->A_cap + BM - 1) / BM * single->ntn;
    return tiles <= 40 ? BM / 4 : (tiles < 64 ? BM / 2 : BM);
}

// The kernel expects the ragged problem (more than one group) in p[0], a single group in p[1].
static FfnLaunch ffn_launch_of(const FfnProblem &first, const FfnProblem *second) {
    FfnLaunch L;
    const FfnProblem *single = second ? second : (first.E_local == 1 ? &first : nullptr);
    const FfnProblem *ragged = first.E_local != 1 ? &first : nullptr;
    L.p[0] = ragged ? *ragged : *single;
    L.p[1] = single ? *single : *ragged;
    L.has_ragged = ragged ? 1 : 0;
    L.has_single = single ? 1 : 0;
    L.single_rows = single_tile_rows(ragged, single);
    return L;
}

// One workgroup per CU (fewer if the bound on the tiles is smaller), whatever the number of tiles.
static int64_t ffn_grid_of(const FfnLaunch &L) {
    constexpr int BM = 256;
    int64_t tiles = 0;
    if (L.has_ragged)
        tiles += 8 * ragged_per_xcd_bound(((int64_t)L.p[0].A_cap + BM - 1) / BM + L.p[0].E_local, L.p[0].E_local, L.p[0].ntn);
    if (L.has_single)
        tiles += 8 * single_per_xcd_bound(((int64_t)L.p[1].A_cap + L.single_rows - 1) / L.single_rows + 1, L.p[1].ntn);
    tiles += 8 * CUS_PER_XCD;  // (row parts of the last rounds)
    return tiles < 8 * CUS_PER_XCD ? tiles : 8 * CUS_PER_XCD;
}

// A set of queues for one launch, of one pass or of both; nullptr: none to be had.
static int *ffn_next_queues(bool both) {
    static std::atomic<unsigned> next_set[2];
    static std::atomic<int *> queue_base[64];  // per device: the address of that device's copy of ffn_queues
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    int *base = queue_base[dev].load();
    if (!base) {  // (in host code the array's name is only a handle for this query)
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(ffn_queues)) != hipSuccess || !p) return nullptr;
        base = static_cast<int *>(p);
        queue_base[dev].store(base);
    }
    const unsigned set = next_set[both ? 1 : 0].fetch_add(1) % FFN_QUEUE_SETS;
    return both ? base + FFN_QUEUE_SETS * FFN_QUEUE_INTS + set * FFN_BOTH_INTS : base + set * FFN_QUEUE_INTS;
}

// Launches one pass over one problem (second == nullptr) or over two: the second must be a single
// group (E_local == 1).  Two go into ONE grid unless the first is a single group as well.
// likely: rows of the first that are likely (<= its A_cap): what the choice of a kernel goes by, and nothing else.
int launch_ffn_bf16_dma(int pass, const FfnProblem &first, const FfnProblem *second, int likely, hipStream_t st) {
    drop_stale_error();
    constexpr int WM = 2, WN = 4;
    if (second && second->E_local != 1) return C2R_ERR_INVALID_ARG;
    if (second && first.E_local == 1) {  // (a launch holds one single group)
        const int rc = launch_ffn_bf16_dma(pass, first, nullptr, likely, st);
        return rc != C2R_OK ? rc : launch_ffn_bf16_dma(pass, *second, nullptr, second->A_cap, st);
    }
    const FfnLaunch L = ffn_launch_of(first, second);
    // Few rows: the kernel of ffn_skinny.hip.  More, but not enough to fill the chip with 256 x 256 tiles: that of ffn_mid.hip.
    // Every output is the same chain of the same matrix instructions in all three, so a row's bits do not depend on the choice.
    if (ffn_skinny_takes(pass, L)) return launch_ffn_skinny(pass, L, nullptr, st);
    int tile_rows[2];
    if (ffn_mid_rows(pass, L, likely, tile_rows)) return launch_ffn_mid(pass, tile_rows, L, st);
    int *queues = ffn_next_queues(false);
    if (!queues) return C2R_ERR_LAUNCH;
    const dim3 g((unsigned)ffn_grid_of(L)), b(WM * WN * 64);
    if (pass == 0)
        ffn_bf16_dma_kernel<0, WM, WN><<<g, b, 0, st>>>(L, queues);
    else
        ffn_bf16_dma_kernel<1, WM, WN><<<g, b, 0, st>>>(L, queues);
    return launch_status();
}

// Whether one launch of the tile kernel takes both passes.  Microseconds of a layer call, a kernel per pass / so:
//   gate/up in tiles (more than 179 rows of a shared expert), down in ffn_mid / one launch, the shared expert's down tiles early (ffn_down_early): 60
//     experts + shared, F 1408 / 5632, 220 tokens 171.5 / 175.5, 241 tokens 173 / 178 (one M-tile of the shared expert), 260 tokens 175.9 / 163.8, 320
//     tokens 172.5 / 165.2, 390 tokens 175.5 / 162.0 (see both_fills for the narrow models); shared experts of 704 to 2816, 260 tokens 156.8 / 151.3 to 155.9 / 135.1, 320 tokens 156 / 154 to 175 /
//     159, 390 tokens 155 / 150 to 182 / 163; 8 experts of d 4096, F 2816 / 8192, 260 tokens 242 / 215, 320 tokens 273 / 220;
//   gate/up in ffn_mid, routed groups alone, r rows per expert: 16 experts of d 4096, r = 92 122.5 / 122.4, r = 125 128.4 / 132.6, r = 130
//     144.7 / 134.0 (a chunk more per group), r = 147 152.8 / 138.0; 8 experts, r = 100 120 / 128, r = 125 141.7 / 135.2, r = 147 155.2 / 141.9.
//   both in tiles, n gate/up tiles if the load is even: 16 experts of d 4096, n = 132 155 / 162, n = 188 184 / 179; 8 experts, n = 215 189 / 189:
//     under a round of tiles there is little to go on with, and what there is waits;
//   so with a part of the experts, whose rows are 0.5 to 2.1 times n's (skewed load): 15 of 60 experts, three light quarters and the heaviest,
//     n = 385 170 / 173, 166 / 166, 190 / 193, 319 / 294, n = 429 181 / 183, 173 / 175, 205 / 201, 356 / 328, n = 462 201 / 201, 194 / 193, 231 / 225;
//     30 of 60, the light half n = 385 167 / 172, n = 407 170 / 174, n = 440 174 / 163, the heavy one n = 385 211 / 210, n = 506 269 / 257.
//   one group alone, gate/up in tiles, by the items of ffn_mid's down pass (64 rows x 64 columns) for its 512 workgroups: up to one each, d 2048, F 12288,
//     300 rows 106.8 / 148.9, 511 rows 108.8 / 152.3; d 4096, F 14336, 300 rows 209 / 235, 511 rows (512 items) 222 / 249; d 5120, F 13824, 384 rows
//     232 / 254; more: 385 rows (560) 272.7 / 271.5, 511 rows 292 / 278; d 6144, F 12288, 320 rows (480) 241 / 273, 321 rows (576) 283 / 273; d 8192, F
//     12288, 257 rows (640) 343 / 329.
constexpr int BOTH_BESIDE = 256, BOTH_PER_GROUP = 125, BOTH_TILES = 180, BOTH_TILES_OF_PART = 435;

// Whether routed groups and a shared expert, of as many rows as ffn_mid takes, give one launch work enough.  Its down tiles are 256
// columns wide, ffn_mid's items 64: a narrow model has few of them, and chains as long as the rest of the launch leave most CUs idle behind them.  So
// there have to be down tiles for half of the CUs, and the k-slices of all tiles, per CU, have to be 0.7 of the longest down chain.  Microseconds of a
// layer call, a launch per pass / one (slices per CU to the longest chain, down tiles): E 8, K 1, d 512, F 4096 / 2048, 363 tokens 62 / 86 (0.14, 14);
// E 24, K 1, d 1024, F 2048 / 10240, 397 tokens 106 / 145 (0.29, 80); E 16, K 2, d 2048, F 4096 / 20480, 486 tokens 335 / 434 (0.58, 152); E 16, K 4, d 2048,
// F 1408 / 4224, 288 tokens 120 / 129 (0.66, 136); E 24, K 4, d 2048, F 1408 / 4224, 288 tokens 156 / 144 (0.78, 168); E 24, K 4, d 4096, F 1536 / 7680, 280 tokens
// 335 / 260 (1.16, 336).  Of 2146 drawn shapes with 257 to 511 tokens (d 512 to 5120, even and skewed loads), by this rule one launch is more than 3 % behind
// in 71 (nearly all skewed, whose experts in use nobody knows here), a launch per pass in 68; one launch for all would be in 552.
constexpr int BOTH_DOWN_TILES = 128;
static bool both_fills(const FfnLaunch &up, const FfnLaunch &down, int routed_mtiles) {
    const FfnProblem &R = down.p[0], &S = down.p[1];
    const int64_t cus = 8 * CUS_PER_XCD, up_slices = (up.p[0].Kdim + 63) / 64, routed = (R.Kdim + 63) / 64, shared = (S.Kdim + 63) / 64;
    const int64_t up_tiles = (int64_t)routed_mtiles * up.p[0].ntn + (int64_t)(up.p[1].A_cap + 255) / 256 * up.p[1].ntn;
    const int64_t routed_tiles = (int64_t)routed_mtiles * R.ntn, shared_tiles = (int64_t)(S.A_cap + down.single_rows - 1) / down.single_rows * S.ntn;
    return routed_tiles + shared_tiles >= BOTH_DOWN_TILES &&
           10 * (up_tiles * up_slices + routed_tiles * routed + shared_tiles * shared) >= 7 * cus * (routed > shared ? routed : shared);
}
static bool both_in_tiles(const FfnLaunch &up, const FfnLaunch &down, int likely) {
    int rows[2];
    if (ffn_skinny_takes(0, up) || ffn_skinny_takes(1, down)) return false;
    const FfnProblem &R = up.p[0], &S = up.p[1];
    if (ffn_mid_rows(0, up, likely, rows)) return !up.has_single && likely / R.E_local > BOTH_PER_GROUP;
    const int routed_mtiles = up.has_ragged ? likely / 256 + (R.E_local < likely ? R.E_local : likely) / 2 : 0;
    if (up.has_single && ffn_mid_rows(1, down, likely, rows) &&
        (up.has_ragged ? S.A_cap <= BOTH_BESIDE || !both_fills(up, down, routed_mtiles) : ffn_mid_in_one_round(down.p[1], rows[1])))
        return false;
    int64_t tiles = up.has_single ? (int64_t)(S.A_cap + 255) / 256 * S.ntn : 0;
    tiles += (int64_t)routed_mtiles * R.ntn;
    return tiles >= (up.has_ragged && likely < R.A_cap ? BOTH_TILES_OF_PART : BOTH_TILES);
}

// Whether a launch of both passes takes the single group's down tiles early.  They gain where they are longer than what else is there to fill the end
// of the launch with, and few; the rows of h that the routed down tiles wait for come later by it.  Microseconds of a layer call, after all gate/up
// tiles / early, by the ratio of the two contractions:
//   4, 60 experts, F 1408 / 5632, four draws of the weights: 420 tokens 185 / 171, 186 / 172, 199 / 181, 190 / 174, 512 tokens 188 / 177, 188 / 176, 204 / 191,
//     181 / 176, 560 tokens 189 / 192, 190 / 196, 204 / 199, 198 / 192, 600 tokens 196 / 197, 185 / 187, 204 / 202, 640 tokens 186 / 192, 194 / 201, 197 / 199,
//     195 / 195, 1000 tokens 226 / 248; 32 experts 520 tokens 179 / 172, 560 tokens 176 / 165; 16 of d 4096, F 2048 / 8192, 450 tokens 291 / 285, 520 tokens
//     314 / 303, 640 tokens 338 / 341;
//   3 and 2.5, 60 experts, F 1408 / 4224 and 3520: 300 tokens 165 / 157, 155.6 / 154, 390 tokens 159 / 160, 158 / 161, 420 tokens 159 / 161, 152.5 / 157, 512
//     tokens 163 / 166, 160 / 164; 32 experts, K 2, F 1408 / 4224, 409 tokens 189 / 168, 494 tokens 179 / 159;
//   2 and less: 260 tokens 148 / 145.5 (F 1408 / 2816), 151 / 135 (1408 / 1408), 390 tokens 156 / 158, 153 / 153, 480 tokens 156 / 158, 640 tokens 196 / 200.
// Of drawn shapes (as in both_fills) early is ahead / behind by more than 3 %, ratio 3, 391 to 600 tokens, in 30 / 7 of 80, ratio 4 in 28 / 3 of 110, ratio 2 in
// 13 / 12 of 91; 601 to 640 tokens, ratio 3, in 1 / 1 of 15, ratio 4 in 10 / 3 of 27, ratio 5 in 15 / 0 of 26.  (Where both_fills, either way is ahead of a launch
// per pass up to 390 rows.)
constexpr int BOTH_EARLY_UP_TO = 390, BOTH_EARLY_LONG_UP_TO = 600, BOTH_EARLY_LONGEST_UP_TO = 640;
static bool ffn_down_early(const FfnLaunch &down) {
    if (!down.has_single || !down.has_ragged) return false;
    const FfnProblem &R = down.p[0], &S = down.p[1];
    return S.A_cap <= (S.Kdim > 4 * R.Kdim ? BOTH_EARLY_LONGEST_UP_TO : S.Kdim >= 3 * R.Kdim ? BOTH_EARLY_LONG_UP_TO : BOTH_EARLY_UP_TO);
}

// Whether the down pass may write while the gate/up pass still reads: its outputs meet nothing else of the two (but for one in the place of
// its own problem's rows, not gathered: a tile waits until the gate/up tiles of its rows, the only ones that read them, are finished).
static bool ffn_both_apart(const FfnBothLaunch &L) {
    const MemRange none = {nullptr, 0};
    MemRange y[2], h[2], read[2][6];
    for (int q = 0; q < 2; ++q) {
        const FfnProblem &U = L.pass[0].p[q], &D = L.pass[1].p[q];
        y[q] = h[q] = none;
        for (MemRange &r : read[q]) r = none;
        if (!(q == 0 ? L.pass[0].has_ragged : L.pass[0].has_single)) continue;
        const size_t weights = (size_t)U.E_local * U.N * U.Kdim * 2;
        y[q] = {D.out, (size_t)D.A_cap * D.ldo * 2};
        h[q] = {U.out, (size_t)U.A_cap * U.ldo * 2};
        read[q][0] = {U.A, (size_t)(U.gather ? U.gather_rows : U.A_cap) * U.lda * 2};
        read[q][1] = {U.B0, weights};
        read[q][2] = {U.B1, weights};
        read[q][3] = {D.B0, weights};
        read[q][4] = {U.gather, (size_t)U.A_cap * 4};
        read[q][5] = {U.offsets, (size_t)(U.E_local + 1) * 4};
    }
    for (int q = 0; q < 2; ++q) {
        if (!apart(y[q], y[1 - q]) || !apart(y[q], h[0]) || !apart(y[q], h[1])) return false;
        for (int o = 0; o < 2; ++o)
            for (int i = 0; i < 6; ++i) {
                const FfnProblem &U = L.pass[0].p[q], &D = L.pass[1].p[q];
                const bool in_place = o == q && i == 0 && !U.gather && D.out == U.A && D.ldo == U.lda;
                if (!in_place && !apart(y[q], read[o][i])) return false;
            }
    }
    return true;
}

// Both passes over one problem or two (first[pass], second[pass] as above; pass 1 reads the rows that pass 0 writes): one launch where
// the tile kernel takes both, their buffers are apart, h has whole 128-byte lines and there are counters for all M-tiles (260000 rows: the
// idle end of a pass is under 1 % of it there).
int launch_ffn_bf16_dma_both(const FfnProblem (&first)[2], const FfnProblem *const (&second)[2], int likely, hipStream_t st) {
    constexpr int BM = 256, WM = 2, WN = 4;
    const bool two_single = second[0] && first[0].E_local == 1;
    if (!two_single && (!second[0] || second[0]->E_local == 1)) {
        FfnBothLaunch L;
        int64_t mtiles = 0;
        for (int pass = 0; pass < 2; ++pass) L.pass[pass] = ffn_launch_of(first[pass], second[pass]);
        bool tiles = both_in_tiles(L.pass[0], L.pass[1], likely);
        // An XCD writes whole lines of h: no line is in two XCDs' L2.
        for (int q = 0; q < 2; ++q) {
            const FfnProblem &P = L.pass[0].p[q];
            if (!(q == 0 ? L.pass[0].has_ragged : L.pass[0].has_single)) continue;
            tiles = tiles && aligned(P.out, 128) && P.ldo % 64 == 0;
            mtiles += P.A_cap / BM + P.E_local;
        }
        if (tiles && mtiles <= FFN_MTILES && ffn_both_apart(L)) {
            drop_stale_error();
            int *queues = ffn_next_queues(true);
            if (!queues) return C2R_ERR_LAUNCH;
            const int64_t g0 = ffn_grid_of(L.pass[0]), g1 = ffn_grid_of(L.pass[1]);
            const dim3 g((unsigned)(g0 > g1 ? g0 : g1)), b(WM * WN * 64);
            if (ffn_down_early(L.pass[1]))
                ffn_bf16_dma_both_kernel<WM, WN, true><<<g, b, 0, st>>>(L, queues, (int)mtiles);
            else
                ffn_bf16_dma_both_kernel<WM, WN, false><<<g, b, 0, st>>>(L, queues, (int)mtiles);
            return launch_status();
        }
    }
    const int rc = launch_ffn_bf16_dma(0, first[0], second[0], likely, st);
    return rc != C2R_OK ? rc : launch_ffn_bf16_dma(1, first[1], second[1], likely, st);
}

// Whether the gate/up pass of a few tokens does their selection and index at its start.
bool ffn_few_takes(const FfnProblem &routed, const FfnProblem *shared) {
    return routed.E_local != 1 && ffn_skinny_takes_few(ffn_launch_of(routed, shared));
}

// The gate/up pass that does so.
int launch_ffn_few(const FfnProblem &routed, const FfnProblem *shared, const FewRoute &few, hipStream_t st) {
    return launch_ffn_skinny(0, ffn_launch_of(routed, shared), &few, st);
}

int launch_ffn_bf16_dma_pass(int pass, const uint16_t *a, int lda, const int32_t *offsets, int E_local,
                             int64_t A_cap, int d, int F, const uint16_t *b0, const uint16_t *b1,
                             uint16_t *out, int ldo, const int32_t *gather, int gather_div, int gather_rows,
                             hipStream_t st) {
    const FfnProblem P = ffn_bf16_dma_problem(pass, a, lda, offsets, E_local, A_cap, d, F, b0, b1, out, ldo, gather,
                                              gather_div, gather_rows);
    return launch_ffn_bf16_dma(pass, P, nullptr, P.A_cap, st);
}

}  // namespace c2r
