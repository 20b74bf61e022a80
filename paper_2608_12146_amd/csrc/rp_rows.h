// Sums of q rows by one wave, shared by the scoring, the packing and the
// annealing build: a wave takes a piece of the row (whole layers, at most 256
// entries), a lane four ranks of one layer (one 16-byte load per row), with
// eight rows in flight.  A piece narrower than 33 lanes is read by several
// groups of lanes (ONE false), each taking every ng-th row.
#pragma once

#include "rp_device.h"

namespace rp {

// Split of L layers of P ranks (P a power of two from 4 to 64) into pieces.
struct RowPieces {
    int32_t lay_piece, n_pieces;  // layers per piece, pieces
    bool one;                     // a piece takes more than half a wave
    // Consecutive work items take different pieces: workgroups go round the 8
    // XCDs, so with 2, 4 or 8 pieces an XCD reads only its piece's slice of q.
    bool spread;
};

// Few-megabyte q (spread): pieces whose slice of q stays in a 4 MiB L2 (up to
// 2 MiB of it); larger q: the widest pieces, one after the other, each slice
// shared by all XCDs in the last level cache.  The first only with 1, 2, 4 or
// 8 pieces: with 3, 5, 6 or 7, as whole layers may leave, consecutive
// workgroups bring an XCD several pieces in turn and its L2 holds none of them
// (512 layouts of 8192 samples of 16 ranks: 20 layers in 7 pieces 0.68 ms a
// call, in 2 wide ones 0.35; 17 layers in 6: 0.44 and 0.34 ms).
inline RowPieces row_pieces(int64_t N, int64_t L, int64_t P) {
    RowPieces r;
    const int64_t most = 256 / P;
    int64_t np = 1;
    while (np <= 8 && ((L + np - 1) / np > most || N * ((L + np - 1) / np) * P * 4 > (int64_t)2 << 20)) np *= 2;
    const int64_t lay = (L + np - 1) / np, got = (L + lay - 1) / lay;
    r.spread = np <= 8 && (got & (got - 1)) == 0;
    if (!r.spread) np = (L + most - 1) / most;
    r.lay_piece = (int32_t)((L + np - 1) / np);
    r.n_pieces = (int32_t)((L + r.lay_piece - 1) / r.lay_piece);
    r.one = r.lay_piece * P > 128;
    return r;
}

// A lane's place in a piece.
template <bool ONE>
struct RowLane {
    int32_t l0, nl, g4, w4;  // first layer, layers, 16-byte words of a layer, of the piece
    int32_t ng, grp, col;
    bool act;
    __device__ inline RowLane(int32_t piece, int32_t lay_piece, int32_t L, int32_t P) {
        const int lane = lane_id();
        l0 = piece * lay_piece;
        nl = lay_piece < L - l0 ? lay_piece : L - l0;
        g4 = P >> 2;
        w4 = nl * g4;
        ng = ONE ? 1 : kWave / w4;
        grp = ONE ? 0 : lane / w4;
        col = lane - grp * w4;
        act = ONE ? lane < w4 : grp < ng;
        if (!act) col = 0;
    }
    // The lane's layer and the first of its ranks (lanes below w4).
    __device__ inline int32_t layer() const { return l0 + col / g4; }
    __device__ inline int32_t rank() const { return (col & (g4 - 1)) * 4; }

    // acc += the lane's four entries of rows ids[0 .. n) (of its group's share).
    template <typename Sum>
    __device__ inline void add(const int32_t *q, int64_t stride, int32_t P, const int32_t *ids_p, int32_t n,
                               Sum *acc) const {
        const int lane = lane_id();
        const int32_t *base = q + (int64_t)l0 * P + 4 * col;
        constexpr int U = 8;
        for (int32_t mb = 0; mb < n; mb += kWave) {
            const int32_t lim = n - mb < kWave ? n - mb : kWave;
            const int32_t ids = ids_p[mb + lane < n ? mb + lane : 0];
            for (int32_t m = 0; m < lim; m += U * ng) {
                int4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t x = m + u * ng + grp;
                    int32_t i;
                    if (ONE) i = __builtin_amdgcn_readlane(ids, x < lim ? x : 0);
                    else i = __shfl(ids, x < lim ? x : 0, kWave);
                    v[u] = *reinterpret_cast<const int4 *>(base + i * stride);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (m + u * ng + grp < lim) {
                        acc[0] += (Sum)v[u].x;
                        acc[1] += (Sum)v[u].y;
                        acc[2] += (Sum)v[u].z;
                        acc[3] += (Sum)v[u].w;
                    }
                }
            }
        }
    }

    // The groups' sums into the first group's lanes.
    template <typename Sum>
    __device__ inline void fold(Sum *acc) const {
        if (ONE) return;
        const int lane = lane_id();
        Sum part[4] = {acc[0], acc[1], acc[2], acc[3]};
        for (int32_t k = 1; k < ng; ++k) {
            const int src = lane + k * w4;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const Sum o = __shfl(part[c], src < kWave ? src : lane, kWave);
                acc[c] += lane < w4 ? o : 0;
            }
        }
    }

    // Maximum over the four entries and over the layer's lanes; the lane that
    // stands for the layer is the first one (head).
    __device__ inline bool head() const { return lane_id() < w4 && (lane_id() & (g4 - 1)) == 0; }
    template <typename T>
    __device__ inline int64_t layer_max(const T *v) const {
        int64_t mx = (int64_t)v[0];
#pragma unroll
        for (int c = 1; c < 4; ++c) mx = (int64_t)v[c] > mx ? (int64_t)v[c] : mx;
        int64_t o;
        if (g4 >= 2) { o = dpp64<kDppXor1>(mx, mx); mx = o > mx ? o : mx; }
        if (g4 >= 4) { o = dpp64<kDppXor2>(mx, mx); mx = o > mx ? o : mx; }
        if (g4 >= 8) { o = dpp64<kDppHalfMirror>(mx, mx); mx = o > mx ? o : mx; }
        if (g4 >= 16) { o = dpp64<kDppMirror>(mx, mx); mx = o > mx ? o : mx; }
        return mx;
    }
    template <typename T>
    __device__ inline int64_t layer_sum(const T *v) const {
        int64_t sm = (int64_t)v[0] + (int64_t)v[1] + (int64_t)v[2] + (int64_t)v[3];
        if (g4 >= 2) sm += dpp64<kDppXor1>(sm, 0);
        if (g4 >= 4) sm += dpp64<kDppXor2>(sm, 0);
        if (g4 >= 8) sm += dpp64<kDppHalfMirror>(sm, 0);
        if (g4 >= 16) sm += dpp64<kDppMirror>(sm, 0);
        return sm;
    }
};

}  // namespace rp
