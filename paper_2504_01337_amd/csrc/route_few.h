// Selection and dispatch index of a few tokens by one workgroup: route.hip runs it as a kernel of its own, the expert-FFN kernels of the
// smallest batches at their start.
#pragma once
#include <type_traits>

#include "c2r_internal.h"

namespace c2r {

// One merge step of a selection spread over neighbouring lanes: the partner's candidate (fetched by a data-parallel-primitive
// move, a tenth of an LDS shuffle's latency: one token's selection and index 8.6 -> 7.8 us) against this lane's, the part
// with the lower expert indices first; a later one only if it is strictly larger.  upper: this lane's part is the later one.
template <int DPP>
__device__ __forceinline__ void merge_lower(int upper, int &bi, float &bv) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int obi = __builtin_amdgcn_mov_dpp(bi, DPP, 0xf, 0xf, true);
    const float obv = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(bv), DPP, 0xf, 0xf, true));
    const int abi = upper ? obi : bi, bbi = upper ? bi : obi;
    const float abv = upper ? obv : bv, bbv = upper ? bv : obv;
    const bool later = abi < 0 || (bbi >= 0 && bbv > abv);
    bi = later ? bbi : abi;
    bv = later ? bbv : abv;
#endif
}

// The bitwise or of the values of a quad of lanes (N 4) or of a row of sixteen, in each of them.
template <int N>
__device__ __forceinline__ uint64_t or_of_lanes(uint64_t m) {
    int half[2] = {(int)(uint32_t)m, (int)(uint32_t)(m >> 32)};
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int &h : half) {
        h |= __builtin_amdgcn_mov_dpp(h, 0xB1, 0xf, 0xf, true);  // quad_perm 1,0,3,2
        h |= __builtin_amdgcn_mov_dpp(h, 0x4E, 0xf, 0xf, true);  // quad_perm 2,3,0,1
        if (N == 16) {
            h |= __builtin_amdgcn_mov_dpp(h, 0x141, 0xf, 0xf, true);  // row_half_mirror
            h |= __builtin_amdgcn_mov_dpp(h, 0x140, 0xf, 0xf, true);  // row_mirror
        }
    }
#endif
    return (uint64_t)(uint32_t)half[0] | ((uint64_t)(uint32_t)half[1] << 32);
}

// The best allowed expert of one token (see route_select_kernel for the rule), by the token's sixteen lanes: lane sub holds
// the logits l of experts 4 sub .. 4 sub + 3, row is the token's logits in LDS, m the allowed experts.
// NANS: there may be NaNs among them (else what keeps the rule for those is left out).
template <bool NANS = true>
__device__ __forceinline__ void pick_by_sixteen(const float (&l)[4], const float *row, uint64_t m, int sub, int &bi, float &bv) {
    const uint32_t mloc = (uint32_t)(m >> (sub * 4));
    bi = -1;
    bv = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool take = ((mloc >> j) & 1u) != 0 && (l[j] > bv || (bi < 0 && (!NANS || l[j] == l[j])));
        bv = take ? l[j] : bv;
        bi = take ? sub * 4 + j : bi;
    }
    merge_lower<0xB1>(sub & 1, bi, bv);   // quad_perm 1,0,3,2
    merge_lower<0x4E>(sub & 2, bi, bv);   // quad_perm 2,3,0,1
    merge_lower<0x141>(sub & 4, bi, bv);  // row_half_mirror: the other quad, whose lanes agree by now
    merge_lower<0x140>(sub & 8, bi, bv);  // row_mirror: the other eight lanes
    if (NANS && m != 0) {  // a NaN stands only as the first allowed expert
        const int f = __ffsll((unsigned long long)m) - 1;
        const float lf = row[f];
        if (lf != lf) {
            bi = f;
            bv = lf;
        }
    }
}

// What the selection and the index of a batch need and write.
struct FewRoute {
    const float *part;  // chunk results of the logits, [nchunk, ep, 64] for up to 64 tokens
    int ep, nchunk;
    const float *bias;
    int T, E, K;
    const int32_t *collab_idx;
    int Tc;
    const int32_t *local_slot;
    int E_local;
    int32_t *topk_idx;
    float *gates;
    int32_t *counts, *offsets, *perm, *inv_perm;
};

template <int THREADS, int ASSIGNMENTS>
struct FewScratch {
    float tile[THREADS / 16 * (C2R_MAX_E + 1)];
    uint64_t mask_tab[C2R_MAX_E];
    int32_t slot_tab[C2R_MAX_E], n_of[C2R_MAX_E];
    int32_t slots[ASSIGNMENTS];
    float gbuf[ASSIGNMENTS], den_of[THREADS / 16];
    int32_t by_wave[THREADS / 64][ASSIGNMENTS <= 64 ? 64 : 128];
};

// At most THREADS / 16 tokens and ASSIGNMENTS assignments.  Every thread of the workgroup calls it; sixteen lanes per token scan its
// experts.  lo, hi: the rows of the lane's slot (empty past E_local) in the sorted order; row_of (LDS, may be null, and is there after the
// caller's next barrier): the token of every sorted row.  Without it only the first wave leaves with the rows.
// `write`: this workgroup writes the results to memory.
template <int THREADS, int ASSIGNMENTS>
__device__ __forceinline__ void route_few(const FewRoute &R, FewScratch<THREADS, ASSIGNMENTS> &S, const bool write, int &lo, int &hi,
                                          uint16_t *row_of) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int LP = C2R_MAX_E + 1, WAVES = THREADS / 64, PER = THREADS / C2R_MAX_E;  // threads per expert
    constexpr int AHEAD = PER == 16 ? 2 : 8, DEEP = PER == 16 ? 8 : 16;  // a thread's list entries and chunk results in flight
    static_assert(PER == 4 || PER == 16, "lists are merged in quads or rows of lanes");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = R.T, E = R.E, K = R.K, Tc = R.Tc, E_local = R.E_local, ep = R.ep, nchunk = R.nchunk;
    const int32_t *__restrict__ collab_idx = R.collab_idx;
    const uint64_t all = E >= 64 ? ~0ull : ((1ull << E) - 1ull);

    // ---- logits: a thread adds up the chunk results (left to right) of one expert and four tokens, and walks a part of the expert's list.
    //      Everything that memory has to bring is requested before anything is waited for, from clamped addresses where it is not
    //      used: one trip instead of one each for the lists, the bias, the slots and the partial sums ----
    const int e_of = tid / PER, part_of = tid % PER, last = E * Tc - 1;
    int32_t listed[AHEAD];
    if (collab_idx) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) listed[u] = collab_idx[min(e_of * Tc + part_of + PER * u, last)];
    }
    int own_slot = tid;
    if (R.local_slot) own_slot = R.local_slot[min(tid, E - 1)];
    float bias = 0.0f;
    if (R.bias) bias = R.bias[min(e_of, E - 1)];
    {
        const float *p = R.part + (size_t)min(e_of, ep - 1) * 64 + min(part_of, (T - 1) >> 2) * 4;
        f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int c0 = 0; c0 < nchunk; c0 += DEEP) {
            f32x4 v[DEEP];
#pragma unroll
            for (int u = 0; u < DEEP; ++u) v[u] = *reinterpret_cast<const f32x4 *>(p + (size_t)min(c0 + u, nchunk - 1) * ep * 64);
#pragma unroll
            for (int u = 0; u < DEEP; ++u)
                if (c0 + u < nchunk) sum = c0 + u == 0 ? v[u] : sum + v[u];
        }
        if (R.bias && e_of < E) sum = sum + bias;
        if (e_of < ep && part_of * 4 < T) {
#pragma unroll
            for (int j = 0; j < 4; ++j) S.tile[(part_of * 4 + j) * LP + e_of] = sum[j];
        }
    }
    // ---- collaborator masks and the slot of every expert ----
    {
        uint64_t m = collab_idx ? 0ull : all;
        if (collab_idx) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
                if (part_of + PER * u < Tc && listed[u] >= 0 && listed[u] < E) m |= 1ull << listed[u];
            for (int i = part_of + PER * AHEAD; i < Tc; i += PER) {
                const int v = e_of < E ? collab_idx[e_of * Tc + i] : -1;
                if (v >= 0 && v < E) m |= 1ull << v;
            }
            m = or_of_lanes<PER>(m);
        }
        if (part_of == 0) S.mask_tab[e_of] = m & ~(1ull << e_of);
    }
    if (tid < C2R_MAX_E) {
        const int s = tid < E ? own_slot : -1;
        S.slot_tab[tid] = s >= 0 && s < E_local ? s : -1;
    }
    __syncthreads();

    // ---- selection: sixteen lanes per token, four experts each; see route_select_kernel for the rule ----
    const int t = tid >> 4, sub = tid & 15;
    const float *row = &S.tile[min(t, T - 1) * LP];
    float l[4];
    bool nan = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        l[j] = sub * 4 + j < E ? row[sub * 4 + j] : 0.0f;
        nan = nan || l[j] != l[j];
    }
    auto select = [&](auto nans) __attribute__((always_inline)) {
        int e;
        float v, v0 = 0.0f, den = 0.0f;
        uint64_t m = all;
        for (int s = 0; s < K; ++s) {
            pick_by_sixteen<decltype(nans)::value>(l, row, m, sub, e, v);
            float g = 0.0f;
            if (s == 0) {
                v0 = v;
                m = S.mask_tab[e];
                g = expf(v0 - v0);  // 1, or NaN when the largest logit is infinite or a NaN
            } else if (e >= 0) {
                m &= ~(1ull << e);
                g = expf(v - v0);
            }
            den = s == 0 ? g : den + g;
            if (sub == 0) {
                if (write) R.topk_idx[t * K + s] = e;
                S.slots[t * K + s] = e >= 0 ? S.slot_tab[e] : -1;
                S.gbuf[t * K + s] = g;
            }
        }
        if (sub == 0) S.den_of[t] = den;
    };
    if (t < T) {  // (the sixteen lanes of a token stay together)
        if (__ballot(nan) == 0)
            select(std::false_type{});
        else
            select(std::true_type{});
    }
    __syncthreads();

    // ---- dispatch index ----
    const int A = T * K;
    if (write && tid < A) R.gates[tid] = S.gbuf[tid] / S.den_of[tid / K];
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    if (ASSIGNMENTS <= 128 || A <= 128) {
        if (!row_of && wave != 0) return;  // (one wave writes it)
        // By every wave for itself, a lane per assignment and per slot: the lanes of the same slot find each other with ballots of the
        // slots' bits, the first of them leaves their number for the lane of that slot, and the scan of the numbers comes back the same
        // way.  (A loop in which a wave counts every fourth slot took 2 us in a workgroup of four waves.)
        constexpr int GROUPS = ASSIGNMENTS <= 64 ? 1 : 2;
        int32_t *const tab = S.by_wave[wave];
        int slot[GROUPS], rank[GROUPS];
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            slot[g] = g * 64 + lane < A ? S.slots[g * 64 + lane] : -1;
            tab[g * 64 + lane] = 0;
        }
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            uint64_t same = __ballot(slot[g] >= 0);
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const bool bit = (slot[g] >> b) & 1;
                const uint64_t set = __ballot(bit);
                same &= bit ? set : ~set;
            }
            rank[g] = __popcll(same & lt);
            if (slot[g] >= 0 && rank[g] == 0) tab[g * 64 + slot[g]] = __popcll(same);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int n0 = tab[lane], n = GROUPS == 1 ? n0 : n0 + tab[(GROUPS - 1) * 64 + lane];
        const int incl = wave_inclusive_scan(n);
        tab[lane] = incl - n;
        if (GROUPS == 2) tab[(GROUPS - 1) * 64 + lane] = incl - n + n0;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        lo = lane < E_local ? incl - n : 0;
        hi = lane < E_local ? incl : 0;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const int a = g * 64 + lane, pos = tab[g * 64 + max(slot[g], 0)] + rank[g];
            if (wave != 0 || a >= A) continue;
            if (row_of && slot[g] >= 0) row_of[pos] = (uint16_t)(a / K);
            if (write) {
                if (slot[g] >= 0) R.perm[pos] = a;
                R.inv_perm[a] = slot[g] >= 0 ? pos : -1;
            }
        }
        if (write && wave == 0 && lane < E_local) {
            R.counts[lane] = n;
            R.offsets[lane] = incl - n;
            if (lane == E_local - 1) R.offsets[E_local] = incl;
        }
        return;
    }
    // a wave counts the assignments of slots wave, wave + WAVES, ..., then hands out their positions in order (the stable order of
    // a = t * K + s)
    for (int s = wave; s < E_local; s += WAVES) {
        int n = 0;
        for (int a0 = 0; a0 < A; a0 += 64) n += __popcll(__ballot(a0 + lane < A && S.slots[a0 + lane] == s));
        if (lane == 0) S.n_of[s] = n;
    }
    __syncthreads();
    const int n = lane < E_local ? S.n_of[lane] : 0;
    int incl = n;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    lo = incl - n;
    hi = incl;
    if (write && wave == 0 && lane < E_local) {
        R.counts[lane] = n;
        R.offsets[lane] = incl - n;
        if (lane == E_local - 1) R.offsets[E_local] = incl;
    }
    for (int s = wave; s < E_local; s += WAVES) {
        int run = __shfl(incl - n, s);
        for (int a0 = 0; a0 < A; a0 += 64) {
            const bool mine = a0 + lane < A && S.slots[a0 + lane] == s;
            const uint64_t b = __ballot(mine);
            if (mine) {
                const int p = run + __popcll(b & lt);
                if (row_of) row_of[p] = (uint16_t)((a0 + lane) / K);
                if (write) {
                    R.perm[p] = a0 + lane;
                    R.inv_perm[a0 + lane] = p;
                }
            }
            run += __popcll(b);
        }
    }
    if (write && tid < A && S.slots[tid] < 0) R.inv_perm[tid] = -1;
}

}  // namespace c2r
