// Gate-weighted sums of rows, a wave per 2 KB piece of the result (combine.hip, dedup.hip).
#pragma once
#include "c2r_internal.h"

namespace c2r {

constexpr int ROW_NV = 2;  // 16-byte vectors per lane

// Adds rows in the order of the calls, fp32, and rounds once.  `row` and `out` are this lane's first vector of the piece.
template <bool BF16>
struct RowSum {
    static constexpr int N = BF16 ? 8 : 4;
    float acc[ROW_NV][N];
    __device__ __forceinline__ RowSum() {
#pragma unroll
        for (int i = 0; i < ROW_NV; ++i)
#pragma unroll
            for (int j = 0; j < N; ++j) acc[i][j] = 0.0f;
    }
    __device__ __forceinline__ void add(const uint4 *row, float g) {
        uint4 q[ROW_NV];
#pragma unroll
        for (int i = 0; i < ROW_NV; ++i) q[i] = row[i * 64];
#pragma unroll
        for (int i = 0; i < ROW_NV; ++i) {
            const uint32_t u[4] = {q[i].x, q[i].y, q[i].z, q[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (BF16) {
                    acc[i][2 * j] = __builtin_fmaf(g, __uint_as_float(u[j] << 16), acc[i][2 * j]);
                    acc[i][2 * j + 1] = __builtin_fmaf(g, __uint_as_float(u[j] & 0xffff0000u), acc[i][2 * j + 1]);
                } else {
                    acc[i][j] = __builtin_fmaf(g, __uint_as_float(u[j]), acc[i][j]);
                }
            }
        }
    }
    __device__ __forceinline__ void store(uint4 *out) const {
#pragma unroll
        for (int i = 0; i < ROW_NV; ++i) {
            if constexpr (BF16)
                out[i * 64] = make_uint4(pack_bf16x2(acc[i][0], acc[i][1]), pack_bf16x2(acc[i][2], acc[i][3]),
                                         pack_bf16x2(acc[i][4], acc[i][5]), pack_bf16x2(acc[i][6], acc[i][7]));
            else
                out[i * 64] = make_uint4(__float_as_uint(acc[i][0]), __float_as_uint(acc[i][1]), __float_as_uint(acc[i][2]),
                                         __float_as_uint(acc[i][3]));
        }
    }
};

// Whether rows of row_vecs 16-byte vectors are whole pieces, with a lane per slot.
static inline bool row_pieces(int row_vecs, int K) { return row_vecs % (64 * ROW_NV) == 0 && K <= 64; }

}  // namespace c2r
