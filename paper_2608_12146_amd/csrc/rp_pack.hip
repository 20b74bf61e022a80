// Row-count search, FixedRowFFD and the feasible seed population (Sec. 3.2,
// Sec. 4.1.1, Alg. 2) on gfx950.
//
//  k_rank_*        sigma = samples ordered by (-t, i): the rank of sample i is
//                  the number of samples that precede it (exact, parallel).
//  k_ffd           FixedRowFFD for K = R*D cells, one wave: the K longest
//                  samples open the cells; every later sample goes to the
//                  lowest-index cell with room, found with a two-level ballot
//                  (per-64-cell maximum room, then the cells of that chunk).
//  k_seed_words    Philox4x64-10 words of every randomized draw, in parallel.
//  k_pack_fit*, k_pack_cell*, k_pair_*  the seed trials in stages: best fit,
//                  cell sums, pairing (block 0 pairs x_length's cells with
//                  width 1; block b >= 1 runs trial b: WindowShuffle,
//                  RandomizedBestFit, EDPAwarePair with width w); below.
//  k_pack_trials   the same trials in one kernel, one wave per candidate, for
//                  the shapes and sizes the stages do not take.
//  k_canonical     canonical form of every candidate: cells are disjoint, so
//                  ordering the cells of a row-shard by their sorted id tuples
//                  is ordering them by smallest id, and ordering rows by their
//                  tuple of cell tuples is ordering them by the smallest id of
//                  the cell in slot 0.
//  k_pack_select   keep x_length, x_paired (if strictly better), and every
//                  successful trial; drop canonical duplicates (first kept);
//                  order by (score, discovery); fill the population cyclically.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>
#include <vector>

#include "rp_device.h"
#include "rp_internal.h"
#include "rp_rows.h"

namespace rp {

int eval_layouts(const routepack_problem *p, const Topology &topo, const DeviceProblem &dp,
                 const int32_t *t, const int32_t *q, int32_t R, int64_t n, const int32_t *layouts,
                 int64_t *scores, int32_t *status, int64_t *J, double *diag,
                 const int64_t *rank_load, bool sum32, hipStream_t stream);
__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v);

constexpr int kMaxCells = 4096;

// Ranks by counting: a workgroup counts, for 256 samples, those that precede
// them among a slice of the others (tiles of 256; a whole tile of earlier
// samples precedes at equal lengths too, a tile of later ones does not), and
// adds its counts to rank (zero on entry).  N^2 compares: slices as well as
// samples are spread over workgroups, about 2048 of them, since 128 or 16
// workgroups left most of the chip idle (32768 samples: 0.86 ms, now 73 us;
// 4096: 108 us, now 11 us).
__global__ void __launch_bounds__(256) k_rank_count(const int32_t *__restrict__ t, int32_t N, int32_t tiles,
                                                    int32_t *__restrict__ rank) {
    __shared__ __align__(16) int32_t tile[256];
    const int32_t ib = blockIdx.x, tid = threadIdx.x, i = ib * 256 + tid;
    const int32_t ti = i < N ? t[i] : 0;
    int32_t n = 0;
    const int32_t nt = (N + 255) / 256, j1 = ((int32_t)blockIdx.y + 1) * tiles < nt ? ((int32_t)blockIdx.y + 1) * tiles : nt;
    for (int32_t jb = blockIdx.y * tiles; jb < j1; ++jb) {
        __syncthreads();
        // (past the end: below every length, so counted nowhere)
        tile[tid] = jb * 256 + tid < N ? t[jb * 256 + tid] : INT32_MIN;
        __syncthreads();
        const int4 *t4 = reinterpret_cast<const int4 *>(tile);
        if (jb < ib) {
#pragma unroll 8
            for (int x = 0; x < 64; ++x) {
                const int4 v = t4[x];
                n += (v.x >= ti) + (v.y >= ti) + (v.z >= ti) + (v.w >= ti);
            }
        } else if (jb > ib) {
#pragma unroll 8
            for (int x = 0; x < 64; ++x) {
                const int4 v = t4[x];
                n += (v.x > ti) + (v.y > ti) + (v.z > ti) + (v.w > ti);
            }
        } else {
#pragma unroll 4
            for (int x = 0; x < 256; ++x) n += tile[x] > ti || (tile[x] == ti && x < tid);
        }
    }
    if (i < N && n) atomicAdd(&rank[i], n);
}

__global__ void __launch_bounds__(256) k_rank_place(const int32_t *__restrict__ rank, int32_t N,
                                                    int32_t *__restrict__ sigma) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < N) sigma[rank[i]] = i;
}

// FixedRowFFD (one wave).  ok = 1 and cell_of filled on success.  The N - K
// steps are one serial chain, bound by its length in cycles.  Lane x keeps the
// largest room of chunk x (cells 64x .. 64x + 63), and the rooms of the chunk
// that took the last sample stay in the lanes: samples come longest first, so
// the next one usually goes to the same chunk, and a step is then two compares
// (an earlier chunk with room, a cell of this one) and a lane update.  Leaving
// a chunk stores its rooms and forms its largest one.  4096 samples in 400
// cells took 1.3 ms and 32768 in 1984 took 10.7 ms with the rooms in LDS and a
// wave maximum per step; now 0.56 ms and 4.5 ms.  Room is int32 when the cap
// fits.
template <typename Room>
__global__ void __launch_bounds__(64) k_ffd(const int32_t *__restrict__ t, const int32_t *__restrict__ sigma,
                                            int32_t N, int64_t C, int32_t K, int32_t *cell_of, int32_t *ok) {
    extern __shared__ __align__(8) char sffd[];
    Room *room = reinterpret_cast<Room *>(sffd);  // [K]
    const int lane = lane_id();
    const int nchunk = (K + kWave - 1) / kWave;
    for (int c = lane; c < K; c += kWave) {
        const int32_t i = sigma[c];
        room[c] = (Room)(C - t[i]);
        cell_of[i] = c;
    }
    wave_sync();
    auto largest = [](Room v) -> Room {
        if constexpr (sizeof(Room) == 4) return wave_max32(v);
        else return wave_max(v);
    };
    auto chunk_rooms = [&](int x) -> Room { return x * kWave + lane < K ? room[x * kWave + lane] : -1; };
    Room cmax = -1;
    for (int x = 0; x < nchunk; ++x) {
        const Room v = largest(chunk_rooms(x));
        if (lane == x) cmax = v;
    }
    int cur = 0;
    Room row = chunk_rooms(0);
    // Items after the first K: this block's items and lengths (s0, t0), the
    // next block's (s1, t1) and the items of the one after (s2), loaded a
    // block of 64 ahead; item hb + x's cell stays in lane x until its block
    // is stored, so no step waits on memory.
    int32_t hb = K;
    const int32_t i0 = hb + lane, i1 = i0 + kWave, i2 = i1 + kWave;
    int32_t s0 = i0 < N ? sigma[i0] : 0, s1 = i1 < N ? sigma[i1] : 0, s2 = i2 < N ? sigma[i2] : 0;
    int32_t t0 = i0 < N ? t[s0] : 0, t1 = i1 < N ? t[s1] : 0;
    int32_t good = 1;
    while (hb < N && good) {
        const int32_t cnt = N - hb < kWave ? N - hb : kWave;
        int32_t p_cell = -1;
        for (int32_t x = 0; x < cnt; ++x) {
            const Room ti = (Room)__builtin_amdgcn_readlane(t0, x);
            const uint64_t before = __ballot(cmax >= ti) & low_lanes(cur);
            uint64_t m = before ? 0 : __ballot(row >= ti);
            if (!m) {
                if (cur * kWave + lane < K) room[cur * kWave + lane] = row;
                const Room mx = largest(row);
                cmax = lane == cur ? mx : cmax;
                const uint64_t any = __ballot(cmax >= ti);  // (lengths are at least 1)
                if (!any) {
                    good = 0;
                    break;
                }
                cur = first_lane(any);
                wave_sync();
                row = chunk_rooms(cur);
                m = __ballot(row >= ti);
            }
            const int at = first_lane(m);
            row = lane_in((uint64_t)1 << at) ? (Room)(row - ti) : row;
            p_cell = lane_in((uint64_t)1 << x) ? cur * kWave + at : p_cell;
        }
        if (p_cell >= 0) cell_of[s0] = p_cell;
        hb += kWave;
        s0 = s1;
        t0 = t1;
        s1 = s2;
        const int32_t j1 = hb + kWave + lane, j2 = j1 + kWave;
        t1 = j1 < N ? t[s1] : 0;
        s2 = j2 < N ? sigma[j2] : 0;
    }
    if (lane == 0) *ok = good;
}

// words[b][0][h] shuffle draws, words[b][1][h] best-fit draws (h < N),
// words[b][2][pos] pairing draws (pos < K), for trial b = 1 .. M-2.
__global__ void k_seed_words(uint64_t seed, int32_t n_trials, int32_t N, int32_t K, uint64_t *words) {
    const int64_t per = 2 * (int64_t)N + K;
    const int64_t total = (int64_t)(n_trials - 2) * per;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < total;
         x += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = x / per + 1, r = x % per;
        uint64_t draw, phase;
        if (r < N) { draw = r; phase = 0; }
        else if (r < 2 * (int64_t)N) { draw = r - N; phase = 1; }
        else { draw = r - 2 * (int64_t)N; phase = 2; }
        words[(b - 1) * per + r] = philox4x64_10(draw, (uint64_t)b, phase, 3, seed, 0).v[0];
    }
}

struct TrialArgs {
    const int32_t *t, *q, *sigma, *x_length;
    int32_t N, L, P, D, G, R, K, RG, LP, w;
    int64_t C;
    const int32_t *slots, *count;
    const uint64_t *words;   // [M-2][2N+K]
    // per-block scratch
    int32_t *cellk;          // [M-1][N]
    int32_t *Qc;             // [M-1][K][LP] (int64_t for k_pack_trials<int64_t>)
    int64_t *peak;           // [M-1][K]
    int32_t *order;          // [M-1][K]
    int32_t *Wt;             // [M-1][RG][LP] (as Qc)
    int64_t *base, *after, *pkv;  // [M-1][RG]
    int32_t *filled;         // [M-1][RG]
    int32_t *cell_to;        // [M-1][K]
    int32_t *out;            // [M-1][N] candidate layouts
    int32_t *ok;             // [M-1]
};

// (a before b) in RandomizedBestFit order: decreasing occupancy, then
// cardinality, then index.
__device__ inline bool fit_before(int64_t Ta, int32_t na, int32_t ca, int64_t Tb, int32_t nb, int32_t cb) {
    if (Ta != Tb) return Ta > Tb;
    if (na != nb) return na < nb;
    return ca < cb;
}
// (a before b) in EDPAwarePair insertion order.
__device__ inline bool pair_before(int64_t ia, int64_t pa, int32_t ha, int64_t ib, int64_t pb, int32_t hb) {
    if (ia != ib) return ia < ib;
    if (pa != pb) return pa < pb;
    return ha < hb;
}

// Sum: the type of the cell sums Qc and the row-shard loads Wt; int64_t when a
// load may reach 2^31 (the only kernel that then runs; its buffers hold
// int64_t).
template <typename Sum>
__global__ void __launch_bounds__(64) k_pack_trials(TrialArgs a) {
    __shared__ int64_t sT[kMaxCells];
    __shared__ int32_t sN[kMaxCells];
    const int lane = lane_id();
    const int b = blockIdx.x;  // 0: x_paired; >= 1: trial b
    const int32_t N = a.N, K = a.K, RG = a.RG, LP = a.LP, L = a.L, P = a.P, G = a.G, D = a.D;
    int32_t *cellk = a.cellk + (int64_t)b * N;
    Sum *Qc = reinterpret_cast<Sum *>(a.Qc) + (int64_t)b * K * LP;
    int64_t *peak = a.peak + (int64_t)b * K;
    int32_t *order = a.order + (int64_t)b * K;
    Sum *Wt = reinterpret_cast<Sum *>(a.Wt) + (int64_t)b * RG * LP;
    int64_t *base = a.base + (int64_t)b * RG, *after = a.after + (int64_t)b * RG, *pkv = a.pkv + (int64_t)b * RG;
    int32_t *filled = a.filled + (int64_t)b * RG;
    int32_t *cell_to = a.cell_to + (int64_t)b * K;
    int32_t *out = a.out + (int64_t)b * N;
    const int32_t w = b == 0 ? 1 : a.w;
    const uint64_t *wd = b == 0 ? nullptr : a.words + (int64_t)(b - 1) * (2 * (int64_t)N + K);

    if (b == 0) {
        for (int32_t i = lane; i < N; i += kWave) cellk[i] = a.x_length[i];
    } else {
        // WindowShuffle: the window holds the first min(w, remaining) items of
        // the remaining (-t, i) order; item h is window[bounded(word, |window|)].
        int32_t win = lane < w && lane < N ? a.sigma[lane] : -1;
        int32_t next = w < N ? w : N;
        int32_t wsize = next;
        for (int32_t c = lane; c < K; c += kWave) {
            sT[c] = 0;
            sN[c] = 0;
        }
        __syncthreads();
        int32_t good = 1;
        for (int32_t h = 0; h < N; ++h) {
            const int32_t pos = (int32_t)bounded(wd[h], (uint64_t)wsize);
            const int32_t item = __shfl(win, pos, kWave);
            // remove position pos, append the next sigma item
            const int32_t up = __shfl(win, lane + 1 < kWave ? lane + 1 : lane, kWave);
            if (lane >= pos && lane < wsize - 1) win = up;
            if (next < N) {
                if (lane == wsize - 1) win = a.sigma[next];
                ++next;
            } else {
                if (lane == wsize - 1) win = -1;
                --wsize;
            }
            const int64_t ti = a.t[item];
            int32_t c;
            if (h < K) {
                c = h;
            } else {
                // RandomizedBestFit: rank the feasible cells and take the
                // rho-th of the leading min(w, |F|).
                // (uniform trip count: every lane takes part in each ballot)
                int32_t nf = 0;
                int64_t bT = -1; int32_t bn = 0, bc = -1;
                for (int32_t cb = 0; cb < K; cb += kWave) {
                    const int32_t cc = cb + lane;
                    const bool f = cc < K && sT[cc] + ti <= a.C;
                    if (f && (bc < 0 || fit_before(sT[cc], sN[cc], cc, bT, bn, bc))) {
                        bT = sT[cc]; bn = sN[cc]; bc = cc;
                    }
                    nf += __popcll(__ballot(f));
                }
                if (nf == 0) {
                    good = 0;
                    break;
                }
                const int32_t wp = w < nf ? w : nf;
                const int32_t rho = (int32_t)bounded(wd[N + h], (uint64_t)wp);
                int64_t pT = 0; int32_t pn = 0, pc = -1;
                for (int32_t pass = 0; pass <= rho; ++pass) {
                    if (pass > 0) {
                        // first feasible cell strictly after the previous pick
                        bT = -1; bn = 0; bc = -1;
                        for (int32_t cc = lane; cc < K; cc += kWave) {
                            const bool f = sT[cc] + ti <= a.C && fit_before(pT, pn, pc, sT[cc], sN[cc], cc);
                            if (f && (bc < 0 || fit_before(sT[cc], sN[cc], cc, bT, bn, bc))) {
                                bT = sT[cc]; bn = sN[cc]; bc = cc;
                            }
                        }
                    }
#pragma unroll
                    for (int d = 32; d >= 1; d >>= 1) {
                        const int64_t oT = __shfl_xor(bT, d, kWave);
                        const int32_t on = __shfl_xor(bn, d, kWave), oc = __shfl_xor(bc, d, kWave);
                        if (oc >= 0 && (bc < 0 || fit_before(oT, on, oc, bT, bn, bc))) {
                            bT = oT; bn = on; bc = oc;
                        }
                    }
                    pT = bT; pn = bn; pc = bc;
                }
                c = pc;
            }
            if (lane == 0) {
                sT[c] += ti;
                sN[c] += 1;
                cellk[item] = c;
            }
            __syncthreads();
        }
        if (!good) {
            if (lane == 0) a.ok[b] = 0;
            return;
        }
    }
    __syncthreads();
    // EDPAwarePair.  Q_k = sum of member rows; peak_k = sum_l max_p Q_k.
    for (int64_t x = lane; x < (int64_t)K * LP; x += kWave) Qc[x] = 0;
    __syncthreads();
    for (int32_t i = 0; i < N; ++i) {
        const int32_t k = cellk[i];
        const int32_t *qi = a.q + (int64_t)i * LP;
        for (int32_t e = lane; e < LP; e += kWave) Qc[(int64_t)k * LP + e] += qi[e];
    }
    __syncthreads();
    for (int32_t k = lane; k < K; k += kWave) {
        int64_t pk = 0;
        for (int l = 0; l < L; ++l) {
            Sum mx = Qc[(int64_t)k * LP + l * P];
            for (int p = 1; p < P; ++p) mx = max(mx, Qc[(int64_t)k * LP + l * P + p]);
            pk += mx;
        }
        peak[k] = pk;
    }
    __syncthreads();
    for (int32_t k = lane; k < K; k += kWave) {
        const int64_t v = peak[k];
        int32_t rank = 0;
        for (int32_t f = 0; f < K; ++f) {
            const int64_t u = peak[f];
            rank += (u > v) || (u == v && f < k);
        }
        order[rank] = k;
    }
    for (int64_t x = lane; x < (int64_t)RG * LP; x += kWave) Wt[x] = 0;
    for (int32_t h = lane; h < RG; h += kWave) {
        base[h] = 0;
        filled[h] = 0;
    }
    __syncthreads();
    for (int32_t pos = 0; pos < K; ++pos) {
        const int32_t k = order[pos];
        const Sum *Qk = Qc + (int64_t)k * LP;
        int32_t cnt = 0;
        for (int32_t hb = 0; hb < RG; hb += kWave) {
            const int32_t h = hb + lane;
            const bool cand = h < RG && filled[h] < a.count[h % G];
            int64_t af = 0, pk = 0;
            if (cand) {
                const Sum *Wh = Wt + (int64_t)h * LP;
                for (int l = 0; l < L; ++l) {
                    Sum mx = Wh[l * P] + Qk[l * P];
                    for (int p = 1; p < P; ++p) mx = max(mx, Wh[l * P + p] + Qk[l * P + p]);
                    af += mx;
                    pk = mx > pk ? mx : pk;
                }
            }
            if (h < RG) {
                after[h] = af;
                pkv[h] = pk;
            }
            cnt += __popcll(__ballot(cand));
        }
        __syncthreads();
        const int32_t wp = w < cnt ? w : cnt;
        int32_t rho = 0;
        if (wp > 1) {
            const uint64_t total = (((uint64_t)1) << wp) - 1;
            const uint64_t pick = bounded(wd[2 * (int64_t)N + pos], total);
            uint64_t pref = 0;
            for (rho = 0; rho < wp; ++rho) {
                pref += ((uint64_t)1) << (wp - 1 - rho);
                if (pref > pick) break;
            }
        }
        int64_t pI = 0, pP = 0;
        int32_t pH = -1;
        for (int32_t pass = 0; pass <= rho; ++pass) {
            int64_t bI = 0, bP = 0;
            int32_t bH = -1;
            for (int32_t h = lane; h < RG; h += kWave) {
                if (filled[h] >= a.count[h % G]) continue;
                const int64_t ih = after[h] - base[h], ph = pkv[h];
                if (pass > 0 && !pair_before(pI, pP, pH, ih, ph, h)) continue;
                if (bH < 0 || pair_before(ih, ph, h, bI, bP, bH)) {
                    bI = ih; bP = ph; bH = h;
                }
            }
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                const int64_t oI = __shfl_xor(bI, d, kWave), oP = __shfl_xor(bP, d, kWave);
                const int32_t oH = __shfl_xor(bH, d, kWave);
                if (oH >= 0 && (bH < 0 || pair_before(oI, oP, oH, bI, bP, bH))) {
                    bI = oI; bP = oP; bH = oH;
                }
            }
            pI = bI; pP = bP; pH = bH;
        }
        const int32_t h = pH;
        const int32_t r = h / G, g = h % G;
        const int32_t d = a.slots[g * D + filled[h]];
        Sum *Wh = Wt + (int64_t)h * LP;
        for (int32_t e = lane; e < LP; e += kWave) Wh[e] += Qk[e];
        __syncthreads();
        if (lane == 0) {
            base[h] = after[h];
            filled[h] += 1;
            cell_to[k] = r * D + d;
        }
        __syncthreads();
    }
    for (int32_t i = lane; i < N; i += kWave) out[i] = cell_to[cellk[i]];
    if (lane == 0) a.ok[b] = 1;
}

// ---------------------------------------------------------------------------
// Seed trials in stages for the common shapes (C < 2^31, N and K below 2^16,
// every row-shard load below 2^31, the pairing's tables other than W within
// LDS); the single-kernel path above covers the rest.  Same draws, same
// decisions.
//
//  k_pack_fit      one wave per candidate: WindowShuffle and
//                  RandomizedBestFit with the draws, window items and their
//                  lengths prefetched 64 steps ahead into lane registers; the
//                  ranked pick compares 64-bit keys (load, then fewer
//                  members, then lower index) with DPP maxima.  Ends with the
//                  member list of every cell.  Up to 2048 cells
//                  k_pack_fit_sorted keeps the keys sorted instead.
//  k_pack_cellsum  one workgroup per (candidate, cell): Q_k = sum of the
//                  member rows and peak_k = sum_l max_p Q_k.
//  k_pair_*        EDPAwarePair in batches of cells (see there);
//  k_pack_pair     the shapes those do not take, one workgroup per candidate:
//                  EDPAwarePair with the W table
//                  in LDS when it fits (else in the trial's slice of HBM),
//                  threads over 4 consecutive entries of W + Q_k and a DPP
//                  maximum over each layer's ranks, and the next cell's Q
//                  row prefetched during each step.

struct PackFast {
    int32_t *mstart;  // [M-1][K+1] member list offsets
    int32_t *mlist;   // [M-1][N] members, grouped by cell
};

// RandomizedBestFit key of a cell: a larger key comes first.
__device__ inline uint64_t fit_key(int64_t T, int32_t n, int32_t c) {
    return ((uint64_t)T << 32) | ((uint64_t)(0xFFFF - n) << 16) | (uint64_t)(0xFFFF - c);
}

__global__ void __launch_bounds__(64) k_pack_fit(TrialArgs a, PackFast pf) {
    extern __shared__ int64_t sfit[];
    const int lane = lane_id();
    const int b = blockIdx.x;
    const int32_t N = a.N, K = a.K;
    int64_t *sT = sfit;
    int32_t *sN = reinterpret_cast<int32_t *>(sT + K);
    int32_t *cur = sN + K;
    int32_t *cellk = a.cellk + (int64_t)b * N;
    for (int32_t c = lane; c < K; c += kWave) {
        sT[c] = 0;
        sN[c] = 0;
    }
    __syncthreads();
    int32_t good = 1;
    if (b == 0) {
        for (int32_t i = lane; i < N; i += kWave) {
            const int32_t c = a.x_length[i];
            cellk[i] = c;
            atomicAdd(&sN[c], 1);
        }
    } else {
        const int32_t w = a.w;
        const uint64_t *wd = a.words + (int64_t)(b - 1) * (2 * (int64_t)N + K);
        // window: lane x < wsize holds item x and its length
        int32_t win = -1, wint = 0;
        if (lane < w && lane < N) {
            win = a.sigma[lane];
            wint = a.t[win];
        }
        int32_t next = w < N ? w : N, wsize = next;
        // prefetched sigma items entering the window, with their lengths
        int32_t sbase = next;
        int32_t sreg = sbase + lane < N ? a.sigma[sbase + lane] : 0;
        int32_t streg = sbase + lane < N ? a.t[sreg] : 0;
        // prefetched draws: shuffle word h and best-fit word h
        int32_t hbase = 0;
        uint64_t wr1 = lane < N ? wd[lane] : 0, wr2 = lane < N ? wd[N + lane] : 0;
        for (int32_t h = 0; h < N; ++h) {
            if (h - hbase == kWave) {
                hbase += kWave;
                wr1 = hbase + lane < N ? wd[hbase + lane] : 0;
                wr2 = hbase + lane < N ? wd[N + hbase + lane] : 0;
            }
            const int32_t pos = (int32_t)bounded(readlane64(wr1, h - hbase), (uint64_t)wsize);
            const int32_t item = __builtin_amdgcn_readlane(win, pos);
            const int64_t ti = __builtin_amdgcn_readlane(wint, pos);
            // remove position pos, append the next sigma item
            int32_t up, upt;
            if (w <= 16) {  // row_shl:1 -- lane i reads lane i + 1 of its 16-lane row
                up = __builtin_amdgcn_update_dpp(win, win, 0x101, 0xF, 0xF, false);
                upt = __builtin_amdgcn_update_dpp(wint, wint, 0x101, 0xF, 0xF, false);
            } else {
                up = __shfl_down(win, 1, kWave);
                upt = __shfl_down(wint, 1, kWave);
            }
            if (lane >= pos && lane < wsize - 1) {
                win = up;
                wint = upt;
            }
            if (next < N) {
                if (next - sbase == kWave) {
                    sbase += kWave;
                    sreg = sbase + lane < N ? a.sigma[sbase + lane] : 0;
                    streg = sbase + lane < N ? a.t[sreg] : 0;
                }
                const int32_t ni = __builtin_amdgcn_readlane(sreg, next - sbase);
                const int32_t nt = __builtin_amdgcn_readlane(streg, next - sbase);
                if (lane == wsize - 1) {
                    win = ni;
                    wint = nt;
                }
                ++next;
            } else {
                if (lane == wsize - 1) {
                    win = -1;
                    wint = 0;
                }
                --wsize;
            }
            int32_t c;
            if (h < K) {
                c = h;
            } else {
                uint64_t best = 0;
                int32_t nf = 0;
                for (int32_t cb = 0; cb < K; cb += kWave) {
                    const int32_t cc = cb + lane;
                    const bool f = cc < K && sT[cc] + ti <= a.C;
                    nf += __popcll(__ballot(f));
                    if (f) {
                        const uint64_t k = fit_key(sT[cc], sN[cc], cc);
                        best = k > best ? k : best;
                    }
                }
                if (nf == 0) {
                    good = 0;
                    break;
                }
                best = wave_max_u64(best);
                const int32_t wp = w < nf ? w : nf;
                const int32_t rho = (int32_t)bounded(readlane64(wr2, h - hbase), (uint64_t)wp);
                for (int32_t pass = 1; pass <= rho; ++pass) {
                    const uint64_t prev = best;
                    best = 0;
                    for (int32_t cb = 0; cb < K; cb += kWave) {
                        const int32_t cc = cb + lane;
                        if (cc < K && sT[cc] + ti <= a.C) {
                            const uint64_t k = fit_key(sT[cc], sN[cc], cc);
                            if (k < prev && k > best) best = k;
                        }
                    }
                    best = wave_max_u64(best);
                }
                c = 0xFFFF - (int32_t)(best & 0xFFFF);
            }
            if (lane == 0) {
                sT[c] += ti;
                sN[c] += 1;
                cellk[item] = c;
            }
            __syncthreads();
        }
    }
    if (lane == 0) a.ok[b] = good;
    if (!good) return;
    __syncthreads();
    // member lists: offsets by an exclusive scan of the counts, then a scatter
    int32_t *ms = pf.mstart + (int64_t)b * (K + 1);
    int32_t *ml = pf.mlist + (int64_t)b * N;
    int64_t carry = 0;
    for (int32_t cb = 0; cb < K; cb += kWave) {
        const int32_t cc = cb + lane;
        const int64_t v = cc < K ? sN[cc] : 0;
        const int64_t incl = wave_incl_scan(v);
        if (cc < K) {
            ms[cc] = (int32_t)(carry + incl - v);
            cur[cc] = (int32_t)(carry + incl - v);
        }
        carry += (int64_t)readlane64((uint64_t)incl, kWave - 1);
    }
    if (lane == 0) ms[K] = N;
    __syncthreads();
    for (int32_t i = lane; i < N; i += kWave) {
        const int32_t c = cellk[i];
        ml[atomicAdd(&cur[c], 1)] = i;
    }
}

// WindowShuffle of one trial, one wave: lane x < wsize of (win, wint) holds
// the x-th item of the window and its length; the items that enter it are
// loaded one block of 64 ahead.
struct Shuffle {
    const int32_t *sigma, *t;
    const uint64_t *wd;  // [N] draws
    int32_t N, w, win, wint, next, wsize, sbase, s0, s1, s2, t0, t1, hbase;
    uint64_t word;       // the draws of the next block
    __device__ inline void init(const int32_t *sigma_, const int32_t *t_, const uint64_t *wd_, int32_t N_, int32_t w_) {
        const int lane = lane_id();
        sigma = sigma_; t = t_; wd = wd_; N = N_; w = w_;
        win = -1;
        wint = 0;
        if (lane < w && lane < N) {
            win = sigma[lane];
            wint = t[win];
        }
        next = w < N ? w : N;
        wsize = next;
        sbase = next;
        const int32_t i0 = sbase + lane, i1 = i0 + kWave, i2 = i1 + kWave;
        s0 = i0 < N ? sigma[i0] : 0;
        s1 = i1 < N ? sigma[i1] : 0;
        s2 = i2 < N ? sigma[i2] : 0;
        t0 = i0 < N ? t[s0] : 0;
        t1 = i1 < N ? t[s1] : 0;
        hbase = 0;
        word = lane < N ? wd[lane] : 0;
    }
    // The next up to 64 items of the order, lane x the x-th, with lengths.
    __device__ inline void block(int32_t &item_l, int32_t &t_l) {
        const int lane = lane_id();
        const int32_t hh = hbase + lane, ws = w < N - hh ? w : N - hh;
        const int32_t pos_l = hh < N ? (int32_t)bounded(word, (uint64_t)ws) : 0;
        const int32_t hn = hh + kWave;
        word = hn < N ? wd[hn] : 0;
        const int32_t cnt = N - hbase < kWave ? N - hbase : kWave;
        item_l = 0;
        t_l = 0;
        for (int32_t x = 0; x < cnt; ++x) {
            const int32_t pos = __builtin_amdgcn_readlane(pos_l, x);
            const int32_t item = __builtin_amdgcn_readlane(win, pos);
            const int32_t ti = __builtin_amdgcn_readlane(wint, pos);
            const bool mine = lane_in((uint64_t)1 << x);
            item_l = mine ? item : item_l;
            t_l = mine ? ti : t_l;
            const int32_t up = lane_up(win), upt = lane_up(wint);
            const bool sh = lane >= pos;  // (lanes past the window hold nothing that is read)
            win = sh ? up : win;
            wint = sh ? upt : wint;
            if (next < N) {
                if (next - sbase == kWave) {
                    sbase += kWave;
                    s0 = s1;
                    t0 = t1;
                    s1 = s2;
                    const int32_t j1 = sbase + kWave + lane, j2 = j1 + kWave;
                    t1 = j1 < N ? t[s1] : 0;
                    s2 = j2 < N ? sigma[j2] : 0;
                }
                const int32_t ni = __builtin_amdgcn_readlane(s0, next - sbase);
                const int32_t nt = __builtin_amdgcn_readlane(t0, next - sbase);
                const bool last = lane == wsize - 1;
                win = last ? ni : win;
                wint = last ? nt : wint;
                ++next;
            } else {
                --wsize;
            }
        }
        hbase += kWave;
    }
};

constexpr int kFitThreads = 256;
constexpr int kFitRow = 64, kFitFill = 32;          // keys a row can hold, and after a rebuild
constexpr int kFitSortedCells = kWave * kFitFill;   // 2048

// LDS of k_pack_fit_sorted: the rows, a linear copy of the keys (later the
// member lists' counts and cursors), two blocks of items, a flag.
__host__ __device__ inline int fit_rows(int32_t K) { return (K + kFitFill - 1) / kFitFill; }
__host__ __device__ inline size_t fit_sorted_lds(int32_t K) {
    return (size_t)fit_rows(K) * kFitRow * 8 + (size_t)K * 8 + 2 * kWave * 8 + 16;
}

// k_pack_fit for up to 2048 cells.  The N - K best-fit steps are one serial
// chain, so its length in cycles bounds the kernel.  The cells' keys
//   (2^32 - 1 - T) << 32 | members << 16 | cell
// (ascending = RandomizedBestFit order; t fits iff key >= (2^32 - 1 - (C - t))
// << 32) are kept sorted in up to 64 rows of at most 64 keys in LDS, lane r
// holding row r's first key when built and its count.  A step finds the row
// (one compare and a ballot), the first fitting key in it (one row read, one
// ballot), takes the key rho places on, shifts it out, and shifts its new
// value, which comes earlier, into its row; a row that fills up has the keys
// spread over the rows again.  A second wave runs the shuffle, which does not
// depend on the cells, one block of 64 items ahead.  Keeping the keys unsorted
// in registers (each step a wave maximum per rank over all cells) took
// 4.5 ms for 4096 samples in 400 cells and 90 ms for 32768 in 1984; now
// 1.7 ms and 14.7 ms.
__global__ void __launch_bounds__(kFitThreads) k_pack_fit_sorted(TrialArgs a, PackFast pf) {
    extern __shared__ __align__(16) uint64_t sfs[];
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id()), tid = threadIdx.x;
    const int b = blockIdx.x;
    const int32_t N = a.N, K = a.K, w = a.w;
    const int32_t nrow = fit_rows(K);
    uint64_t *rows = sfs, *lin = rows + nrow * kFitRow;
    int2 *ring = reinterpret_cast<int2 *>(lin + K);  // [2][64] items and lengths
    // cleared by wave 0 when a step finds no cell; iteration j writes entry
    // (j + 1) & 1 and reads entry j & 1, so no wave reads what is being written
    int32_t *s_good = reinterpret_cast<int32_t *>(ring + 2 * kWave);
    int32_t *cellk = a.cellk + (int64_t)b * N;
    int32_t *cnt_s = reinterpret_cast<int32_t *>(lin), *cur = cnt_s + K;
    if (tid < 2) s_good[tid] = 1;
    if (b == 0) {
        for (int32_t c = tid; c < K; c += kFitThreads) cnt_s[c] = 0;
        __syncthreads();
        for (int32_t i = tid; i < N; i += kFitThreads) {
            const int32_t c = a.x_length[i];
            cellk[i] = c;
            atomicAdd(&cnt_s[c], 1);
        }
    } else {
        const uint64_t *wd = a.words + (int64_t)(b - 1) * (2 * (int64_t)N + K);
        const uint32_t Cu = 0xFFFFFFFFu - (uint32_t)a.C;
        Shuffle sh;
        if (wv == 1) {
            sh.init(a.sigma, a.t, wd, N, w);
            int32_t it, tt;
            sh.block(it, tt);
            ring[lane] = make_int2(it, tt);
        }
        uint64_t word = wv == 0 && lane < N ? wd[N + lane] : 0;  // wave 0: this block's best-fit draws
        uint64_t sep = 0;  // wave 0, lane r: row r holds the keys from sep on, below row r + 1's
        int32_t cnt = 0;   // and its number of keys
        const int32_t nblk = (N + kWave - 1) / kWave, jsort = (K - 1) / kWave;
        for (int32_t j = 0; j < nblk; ++j) {
            __syncthreads();
            if (!s_good[j & 1]) break;
            const int32_t h0 = j * kWave, hn = h0 + kWave;
            if (wv == 1 && j + 1 < nblk) {
                int32_t it, tt;
                sh.block(it, tt);
                ring[((j + 1) & 1) * kWave + lane] = make_int2(it, tt);
            }
            int32_t item_l = 0, t_l = 0, cell_l = 0, rho_l = 0;
            uint64_t nword = 0;
            if (wv == 0) {
                const int2 v = ring[(j & 1) * kWave + lane];
                item_l = v.x;
                t_l = v.y;
                cell_l = h0 + lane;  // the first K items open the cells
                if (h0 + lane < K && h0 + lane < N)
                    lin[h0 + lane] = ((uint64_t)(0xFFFFFFFFu - (uint32_t)t_l) << 32) | (1u << 16) | (uint32_t)(h0 + lane);
                rho_l = (int32_t)bounded(word, (uint64_t)w);
                nword = hn + lane < N ? wd[N + hn + lane] : 0;
            }
            if (j == jsort) {  // every cell is open: rank the keys by counting
                __syncthreads();
                for (int32_t c = tid; c < K; c += kFitThreads) {
                    const uint64_t v = lin[c];
                    int32_t rank = 0;
#pragma unroll 8
                    for (int32_t f = 0; f < K; ++f) rank += lin[f] < v ? 1 : 0;
                    rows[rank / kFitFill * kFitRow + rank % kFitFill] = v;
                }
                __syncthreads();
                if (wv == 0) {
                    const int32_t left = K - lane * kFitFill;
                    cnt = left < 0 ? 0 : (left < kFitFill ? left : kFitFill);
                    sep = lane == 0 ? 0 : (cnt > 0 ? rows[lane * kFitRow] : ~(uint64_t)0);
                }
            }
            if (wv == 0 && hn > K) {
                const int32_t x0 = K > h0 ? K - h0 : 0, x1 = N - h0 < kWave ? N - h0 : kWave;
                for (int32_t x = x0; x < x1; ++x) {
                    const int32_t ti = __builtin_amdgcn_readlane(t_l, x);
                    const uint64_t lim = (uint64_t)(Cu + (uint32_t)ti) << 32;
                    int32_t r = __popcll(__ballot(sep <= lim)) - 1;
                    uint64_t e = rows[r * kFitRow + lane];
                    int32_t n = __builtin_amdgcn_readlane(cnt, r);
                    int32_t p = __popcll(__ballot(e < lim) & low_lanes(n));
                    int32_t rho = __builtin_amdgcn_readlane(rho_l, x);
                    if (n - p < w) {
                        // fewer than w left in the row: the draw is over the
                        // min(w, fitting) first, which may be in later rows
                        const int32_t nf = n - p + (int32_t)wave_sum((int64_t)(lane > r ? cnt : 0));
                        if (nf == 0) {
                            if (lane == 0) s_good[(j + 1) & 1] = 0;
                            break;
                        }
                        if (nf < w) rho = (int32_t)bounded(readlane64(word, x), (uint64_t)nf);
                        if (rho >= n - p) {
                            rho -= n - p;
                            p = 0;
                            n = __builtin_amdgcn_readlane(cnt, ++r);
                            while (rho >= n) {  // (rho < nf: a later row holds it)
                                rho -= n;
                                n = __builtin_amdgcn_readlane(cnt, ++r);
                            }
                            e = rows[r * kFitRow + lane];
                        }
                    }
                    const int32_t at = p + rho;
                    const uint64_t key = readlane64(e, at);
                    const uint64_t nk = key - ((uint64_t)(uint32_t)ti << 32) + (1u << 16);
                    cell_l = lane_in((uint64_t)1 << x) ? (int32_t)(key & 0xFFFF) : cell_l;
                    int32_t r2 = __popcll(__ballot(sep <= nk)) - 1;
                    const uint64_t up = lane_up64(e);
                    e = lane_in(~low_lanes(at)) ? up : e;
                    if (r2 != r) {
                        rows[r * kFitRow + lane] = e;
                        cnt -= lane_in((uint64_t)1 << r) ? 1 : 0;
                        wave_sync();
                        if (__builtin_amdgcn_readlane(cnt, r2) == kFitRow) {
                            // spread the K - 1 keys over the rows again
                            const int32_t pre = (int32_t)wave_incl_scan((int64_t)cnt) - cnt;
                            for (int32_t k = 0; k < nrow; ++k) {
                                const int32_t nk_ = __builtin_amdgcn_readlane(cnt, k), ok_ = __builtin_amdgcn_readlane(pre, k);
                                if (lane < nk_) lin[ok_ + lane] = rows[k * kFitRow + lane];
                            }
                            wave_sync();
                            for (int32_t k = lane; k < K - 1; k += kWave) rows[k / kFitFill * kFitRow + k % kFitFill] = lin[k];
                            const int32_t left = K - 1 - lane * kFitFill;
                            cnt = left < 0 ? 0 : (left < kFitFill ? left : kFitFill);
                            sep = lane == 0 ? 0 : (cnt > 0 ? lin[lane * kFitFill] : ~(uint64_t)0);
                            wave_sync();
                            r2 = __popcll(__ballot(sep <= nk)) - 1;
                        }
                        e = rows[r2 * kFitRow + lane];
                        n = __builtin_amdgcn_readlane(cnt, r2);
                        cnt += lane_in((uint64_t)1 << r2) ? 1 : 0;
                    } else {
                        --n;
                    }
                    const int32_t p2 = __popcll(__ballot(e < nk) & low_lanes(n));
                    const uint64_t down = lane_down64(e);
                    e = lane_in(~low_lanes(p2)) ? down : e;
                    e = lane_in((uint64_t)1 << p2) ? nk : e;
                    rows[r2 * kFitRow + lane] = e;
                    wave_sync();
                }
            }
            if (wv == 0) {
                if (h0 + lane < N) cellk[item_l] = cell_l;
                word = nword;
            }
        }
        __syncthreads();
        const int32_t good = s_good[0] & s_good[1];
        if (tid == 0) a.ok[b] = good;
        if (!good) return;
        // member counts by cell (the keys' linear copy is no longer used)
        if (wv == 0)
            for (int32_t r = 0; r < nrow; ++r) {
                const uint64_t e = rows[r * kFitRow + lane];
                if (lane < __builtin_amdgcn_readlane(cnt, r)) cnt_s[e & 0xFFFF] = (int32_t)((e >> 16) & 0xFFFF);
            }
    }
    if (b == 0 && tid == 0) a.ok[b] = 1;
    __syncthreads();
    int32_t *ms = pf.mstart + (int64_t)b * (K + 1);
    int32_t *ml = pf.mlist + (int64_t)b * N;
    if (wv == 0) {
        int32_t carry = 0;
        for (int32_t cb = 0; cb < K; cb += kWave) {
            const int32_t cc = cb + lane;
            const int32_t v = cc < K ? cnt_s[cc] : 0;
            const int32_t incl = (int32_t)wave_incl_scan((int64_t)v);
            if (cc < K) {
                ms[cc] = carry + incl - v;
                cur[cc] = carry + incl - v;
            }
            carry += __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        if (lane == 0) ms[K] = N;
    }
    __syncthreads();
    for (int32_t i = tid; i < N; i += kFitThreads) {
        const int32_t c = cellk[i];
        ml[atomicAdd(&cur[c], 1)] = i;
    }
}

// Q_k and peak_k of cell k = blockIdx.x of candidate b = blockIdx.y; chunked:
// Q_k as [P/4][L][4] instead of [L][P].
__global__ void __launch_bounds__(128) k_pack_cellsum(TrialArgs a, PackFast pf, bool chunked) {
    extern __shared__ int32_t sq[];
    __shared__ int64_t spart[4];
    const int b = blockIdx.y, k = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    if (!a.ok[b]) return;  // uniform: a failed trial has no layout
    const int32_t K = a.K, LP = a.LP, L = a.L, P = a.P;
    const int32_t *ms = pf.mstart + (int64_t)b * (K + 1);
    const int32_t *ml = pf.mlist + (int64_t)b * a.N;
    const int32_t lo = ms[k], hi = ms[k + 1];
    int32_t *Qk = a.Qc + ((int64_t)b * K + k) * LP;
    for (int32_t e = tid; e < LP; e += nt) {
        int32_t acc = 0;
        for (int32_t x = lo; x < hi; ++x) acc += a.q[(int64_t)ml[x] * LP + e];
        const int32_t l = e / P, r = e - l * P;
        Qk[chunked ? ((r >> 2) * L + l) * 4 + (r & 3) : e] = acc;
        sq[e] = acc;
    }
    __syncthreads();
    int64_t part = 0;
    for (int32_t l = tid; l < L; l += nt) {
        int32_t mx = sq[l * P];
        for (int32_t p = 1; p < P; ++p) mx = max(mx, sq[l * P + p]);
        part += mx;
    }
    part = wave_sum(part);
    if (lane_id() == 0) spart[wave_id()] = part;
    __syncthreads();
    if (tid == 0) {
        int64_t tot = 0;
        for (int w = 0; w < nt / kWave; ++w) tot += spart[w];
        a.peak[(int64_t)b * K + k] = tot;
    }
}

// k_pack_cellsum by waves, for ranks a power of two from 4 to 64 (rp_rows.h):
// item (candidate, cell) x piece; peak starts at zero.  Every candidate reads
// all of q once, so this is bound by where the pieces' slices of q are kept:
// 15 candidates of 32768 samples (64 x 64, 512 MiB of q) take 8.2 ms with a
// workgroup per cell and scalar loads in member order, 0.99 ms in pieces.
template <bool ONE>
__global__ void __launch_bounds__(256) k_pack_cellrows(TrialArgs a, PackFast pf, RowPieces pc, int32_t items,
                                                       bool chunked) {
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const uint32_t per = (uint32_t)(items + 3) / 4, b = blockIdx.x, np = (uint32_t)pc.n_pieces;
    const int32_t piece = (int32_t)(pc.spread ? b % np : b / per);
    const int32_t it = (int32_t)((pc.spread ? b / np : b % per) * 4 + wv);
    if (it >= items) return;
    const int32_t K = a.K, L = a.L, tr = it / K, k = it - tr * K;
    if (!a.ok[tr]) return;  // a failed trial has no layout
    const int32_t *ms = pf.mstart + (int64_t)tr * (K + 1) + k;
    const int32_t lo = ms[0], n = ms[1] - lo;
    const RowLane<ONE> rl(piece, pc.lay_piece, L, a.P);
    int32_t acc[4] = {0, 0, 0, 0};
    rl.add(a.q, (int64_t)a.LP, a.P, pf.mlist + (int64_t)tr * a.N + lo, n, acc);
    rl.fold(acc);
    if (lane < rl.w4) {
        int32_t *Qk = a.Qc + (int64_t)it * a.LP;
        const int32_t l = rl.layer(), p = rl.rank();
        *reinterpret_cast<int4 *>(Qk + (chunked ? p * L + l * 4 : l * a.P + p)) = make_int4(acc[0], acc[1], acc[2], acc[3]);
    }
    const int64_t mx = rl.layer_max(acc);  // (every lane takes part)
    const int64_t part = wave_sum(rl.head() ? mx : 0);
    if (lane == 0) atomicAdd(reinterpret_cast<unsigned long long *>(a.peak + it), (unsigned long long)part);
}

// ---------------------------------------------------------------------------
// EDPAwarePair in batches of kPairBatch cells, for up to 64 layers and 64
// ranks (a multiple of 4).  A step's choice needs sum_l max_p (W_h + Q_k) and
// the largest entry of every open row-shard h, but it changes one W_h only:
//  k_pair_start    the cell order, zero W;
//  k_pair_table    those two numbers for every row-shard and each cell of
//                  the next batch on W as it stands, on the whole chip;
//  k_pair_resolve  the batch's choices in order, one workgroup per trial:
//                  after each one the chosen row-shard's numbers are formed
//                  again for the batch's remaining cells, one wave per cell
//                  with its Q row in registers.
// The chain of K choices bounds it (one workgroup streaming every W row in
// every step took 3.4 ms for 400 cells of 24 x 16 on 50 row-shards and 79 ms
// for 1984 of 64 x 64 on 62; now 0.75 ms and 8.4 ms).  A lane holds a
// layer (two row-shards per wave up to 32 layers), so W and Q rows are
// chunk-major, [P/4][L][4], the maximum over ranks is in-lane, and only the
// sum and the maximum over layers cross lanes.

constexpr int kPairBatch = 16;       // cells per batch: a wave of k_pair_resolve each
constexpr int kPairMaxShards = 512;  // row-shards (k_pair_resolve's tables in LDS)

struct PairArgs {
    int64_t *after;   // [M-1][kPairBatch][RG] sum_l max_p (W_h + Q_k)
    int32_t *pk;      // [M-1][kPairBatch][RG] the largest entry
};

// Sum and maximum over each half of the wave, in lanes 31 and 63; with FULL
// over the wave, in lane 63.  The sum is of signed 32-bit values (split in 16
// bits so that 64 of them fit), the maximum is of values >= 0.
template <bool FULL>
__device__ inline void layer_reduce(int32_t v, int64_t &sum, int32_t &mx) {
    int32_t lo = v & 0xFFFF, hi = v >> 16;
    mx = v > 0 ? v : 0;
    auto step = [&](auto ctrl, auto rows) {
        lo += dpp32<decltype(ctrl)::value, decltype(rows)::value>(lo, 0);
        hi += dpp32<decltype(ctrl)::value, decltype(rows)::value>(hi, 0);
        const int32_t o = dpp32<decltype(ctrl)::value, decltype(rows)::value>(mx, 0);
        mx = o > mx ? o : mx;
    };
    using All = std::integral_constant<int, 0xF>;
    step(std::integral_constant<int, kDppRowShr1>{}, All{});
    step(std::integral_constant<int, kDppRowShr1 + 1>{}, All{});
    step(std::integral_constant<int, kDppRowShr1 + 3>{}, All{});
    step(std::integral_constant<int, kDppRowShr1 + 7>{}, All{});
    step(std::integral_constant<int, kDppRowBcast15>{}, std::integral_constant<int, 0xA>{});
    if (FULL) step(std::integral_constant<int, kDppRowBcast31>{}, std::integral_constant<int, 0xC>{});
    sum = (int64_t)hi * 65536 + lo;
}

__device__ inline int32_t max4_sum(int32_t m, const int4 &w, const int4 &q) {
    m = max(m, max(w.x + q.x, w.y + q.y));
    return max(m, max(w.z + q.z, w.w + q.w));
}

// The cell order of each trial (decreasing peak, then index), W, base and
// filled at zero.
__global__ void __launch_bounds__(1024) k_pair_start(TrialArgs a) {
    extern __shared__ __align__(16) int64_t spk[];  // [K]
    const int b = blockIdx.x, tid = threadIdx.x;
    const int32_t K = a.K, RG = a.RG;
    if (!a.ok[b]) return;  // uniform
    for (int32_t k = tid; k < K; k += 1024) spk[k] = a.peak[(int64_t)b * K + k];
    for (int32_t h = tid; h < RG; h += 1024) {
        a.base[(int64_t)b * RG + h] = 0;
        a.filled[(int64_t)b * RG + h] = 0;
    }
    int4 *W = reinterpret_cast<int4 *>(a.Wt + (int64_t)b * RG * a.LP);
    for (int64_t x = tid; x < (int64_t)RG * a.LP / 4; x += 1024) W[x] = make_int4(0, 0, 0, 0);
    __syncthreads();
    for (int32_t k = tid; k < K; k += 1024) {
        const int64_t v = spk[k];
        int32_t rank = 0;
#pragma unroll 8
        for (int32_t f = 0; f < K; ++f) rank += (spk[f] > v) || (spk[f] == v && f < k);
        a.order[(int64_t)b * K + rank] = k;
    }
}

// A wave: two row-shards (four up to 32 layers, two in each half) and eight
// cells of the batch.  A chunk of each Q row is reused for the row-shards and
// a chunk of each W row for the cells.
template <bool HALF>
__global__ void __launch_bounds__(256) k_pair_table(TrialArgs a, PairArgs pa, int32_t pos0) {
    constexpr int CM = kPairBatch / 2, HS = 2;
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int b = blockIdx.z;
    if (!a.ok[b]) return;
    const int32_t RG = a.RG, L = a.L, LP = a.LP, K = a.K, p4 = a.P >> 2;
    const int32_t c0 = (int32_t)blockIdx.y * CM;  // first cell of the batch
    const int32_t nc = K - pos0 - c0;             // cells from there on
    const int32_t s0 = ((int32_t)blockIdx.x * 4 + wv) * HS;  // first row-shard slot of the wave
    if (nc <= 0 || (HALF ? 2 * s0 : s0) >= RG) return;
    const int half = HALF ? lane >> 5 : 0, hl = HALF ? lane & 31 : lane;
    const bool act = hl < L;
    const int32_t ll = act ? hl : L - 1;
    const int4 *wp[HS], *qp[CM];
#pragma unroll
    for (int u = 0; u < HS; ++u) {
        const int32_t h = HALF ? 2 * (s0 + u) + half : s0 + u;
        wp[u] = reinterpret_cast<const int4 *>(a.Wt + ((int64_t)b * RG + (h < RG ? h : RG - 1)) * LP) + ll;
    }
#pragma unroll
    for (int c = 0; c < CM; ++c) {
        const int32_t k = a.order[(int64_t)b * K + pos0 + c0 + (c < nc ? c : 0)];
        qp[c] = reinterpret_cast<const int4 *>(a.Qc + ((int64_t)b * K + k) * LP) + ll;
    }
    int32_t mx[HS][CM];
#pragma unroll
    for (int u = 0; u < HS; ++u)
#pragma unroll
        for (int c = 0; c < CM; ++c) mx[u][c] = INT32_MIN;
    for (int32_t x = 0; x < p4; ++x) {
        int4 w[HS], q[CM];
#pragma unroll
        for (int u = 0; u < HS; ++u) w[u] = wp[u][x * L];
#pragma unroll
        for (int c = 0; c < CM; ++c) q[c] = qp[c][x * L];
#pragma unroll
        for (int u = 0; u < HS; ++u)
#pragma unroll
            for (int c = 0; c < CM; ++c) mx[u][c] = max4_sum(mx[u][c], w[u], q[c]);
    }
#pragma unroll
    for (int u = 0; u < HS; ++u) {
        const int32_t h = HALF ? 2 * (s0 + u) + half : s0 + u;
#pragma unroll
        for (int c = 0; c < CM; ++c) {
            int64_t sum;
            int32_t m;
            layer_reduce<!HALF>(act ? mx[u][c] : 0, sum, m);
            if (lane == 63 || (HALF && lane == 31)) {
                if (h < RG && c < nc) {
                    const int64_t at = ((int64_t)b * kPairBatch + c0 + c) * RG + h;
                    pa.after[at] = sum;
                    pa.pk[at] = m;
                }
            }
        }
    }
}

__host__ __device__ inline size_t pair_resolve_lds(int64_t RG, int64_t LP, bool wl) {
    return (size_t)(kPairBatch * RG * 12 + RG * 16 + (wl ? RG + 2 : 2) * LP * 4 + 4 + kPairBatch * 8);
}

// A workgroup barrier for LDS only: __syncthreads also waits for the global
// stores before it, a trip to memory and back that nothing here needs.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The rank drawn among wp candidates with weights 2^(wp - 1 - rho): the
// prefix up to rho is 2^wp - 2^(wp - 1 - rho), and rho is the first whose
// prefix exceeds floor(word (2^wp - 1) / 2^64).
__device__ inline int32_t pair_rho(uint64_t word, int32_t wp) {
    if (wp <= 1) return 0;
    const uint64_t all = ((uint64_t)1 << wp) - 1;
    return wp - 64 + __clzll((long long)(all - bounded(word, all)));
}

// Unsigned minimum over the wave; uniform.
__device__ inline uint32_t wave_min_u32(uint32_t v) {
    auto step = [&](uint32_t o) { v = o < v ? o : v; };
    step((uint32_t)dpp32<kDppXor1>((int32_t)v, (int32_t)v));
    step((uint32_t)dpp32<kDppXor2>((int32_t)v, (int32_t)v));
    step((uint32_t)dpp32<kDppHalfMirror>((int32_t)v, (int32_t)v));
    step((uint32_t)dpp32<kDppMirror>((int32_t)v, (int32_t)v));
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int32_t)v, 48);
    const uint32_t x = a < b ? a : b, y = c < d ? c : d;
    return x < y ? x : y;
}

// EDPAwarePair's choice (one wave): the rho-th open row-shard in the order
// (increase, peak, index), drawn from the leading min(w, open).
__device__ inline int32_t pair_choice(const int64_t *after, const int32_t *pk, const int64_t *base,
                                      const int32_t *filled, const int32_t *hcnt, int32_t RG, int32_t w,
                                      uint64_t word, int32_t rho_w) {
    const int lane = lane_id();
    if (RG <= kWave) {
        const int32_t at = lane < RG ? lane : 0;
        const int64_t inc = after[at] - base[at];
        const int32_t peak = pk[at], fl = filled[at], hc = hcnt[at];
        uint64_t open = __ballot(lane < RG && fl < hc);
        if ((open & __ballot((uint64_t)inc >= 0xFFFFFFFFull)) == 0) {  // increases below 2^32 - 1, as all but always
            const int32_t cnt = __popcll(open);
            const int32_t rho = cnt >= w ? rho_w : pair_rho(word, cnt);
            for (int32_t pass = 0;; ++pass) {
                const uint32_t v = lane_in(open) ? (uint32_t)inc : 0xFFFFFFFFu;
                uint64_t eq = __ballot(v == wave_min_u32(v));
                if (__popcll(eq) > 1) {  // (lanes are in index order)
                    const uint32_t p = lane_in(eq) ? (uint32_t)peak : 0xFFFFFFFFu;
                    eq = __ballot(p == wave_min_u32(p));
                }
                const int src = first_lane(eq);
                if (pass == rho) return src;
                open &= ~((uint64_t)1 << src);
            }
        }
    }
    int32_t cnt = 0;
    for (int32_t hb = 0; hb < RG; hb += kWave)
        cnt += __popcll(__ballot(hb + lane < RG && filled[hb + lane] < hcnt[hb + lane]));
    const int32_t rho = cnt >= w ? rho_w : pair_rho(word, cnt);
    uint32_t taken = 0;  // bit x: this lane's row-shard lane + 64 x was an earlier choice
    int32_t h = 0;
    for (int32_t pass = 0; pass <= rho; ++pass) {
        int64_t k0 = LLONG_MAX;
        int32_t k1 = INT32_MAX, k2 = INT32_MAX;
        for (int32_t hb = 0, x = 0; hb < RG; hb += kWave, ++x) {
            const int32_t hh = hb + lane;
            if (hh < RG && filled[hh] < hcnt[hh] && !((taken >> x) & 1)) {
                const int64_t v0 = after[hh] - base[hh];
                const int32_t v1 = pk[hh];
                if (k2 == INT32_MAX || v0 < k0 || (v0 == k0 && v1 < k1)) {  // (ascending index)
                    k0 = v0;
                    k1 = v1;
                    k2 = hh;
                }
            }
        }
        const int64_t m0 = wave_min(k0);
        uint64_t eq = __ballot(k2 != INT32_MAX && k0 == m0);
        if (__popcll(eq) > 1) {
            const uint32_t p = lane_in(eq) ? (uint32_t)k1 : 0xFFFFFFFFu;
            eq = __ballot(p == wave_min_u32(p));
            if (__popcll(eq) > 1) {
                const uint32_t i = lane_in(eq) ? (uint32_t)k2 : 0xFFFFFFFFu;
                eq = __ballot(i == wave_min_u32(i));
            }
        }
        const int src = first_lane(eq);
        h = __builtin_amdgcn_readlane(k2, src);
        if (lane == src) taken |= 1u << (h >> 6);
    }
    return h;
}

// The choices of cells pos0 .. pos0 + kPairBatch - 1.  PV: the ranks rounded
// up to a compiled size.  WL: the trial's W is loaded into LDS first (when it
// fits): a launch finds it in the last level cache only, 1.5 to 2 us away, so
// a step that reads the chosen row from there takes that long.
template <int PV, bool WL>
__global__ void __launch_bounds__(kPairBatch *kWave) k_pair_resolve(TrialArgs a, PairArgs pa, int32_t pos0) {
    extern __shared__ __align__(16) char sres[];
    const int b = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    if (!a.ok[b]) return;  // uniform
    const int32_t RG = a.RG, L = a.L, LP = a.LP, K = a.K, D = a.D, G = a.G, p4 = a.P >> 2;
    const int32_t m = K - pos0 < kPairBatch ? K - pos0 : kPairBatch;
    const int32_t n4 = LP >> 2;
    int4 *qcur = reinterpret_cast<int4 *>(sres);                    // [n4] Q of the current cell (WL: [2][n4], by parity)
    int4 *wl = qcur + (WL ? 2 : 1) * n4;                            // [n4] the chosen row's new W (WL: [RG][n4], W)
    int64_t *after = reinterpret_cast<int64_t *>(wl + (WL ? RG : 1) * n4);  // [kPairBatch][RG]
    int64_t *base = after + kPairBatch * RG;                        // [RG]
    int32_t *pk = reinterpret_cast<int32_t *>(base + RG);           // [kPairBatch][RG]
    int32_t *filled = pk + kPairBatch * RG, *hcnt = filled + RG;    // [RG], [RG]
    int32_t *s_h = hcnt + RG;                                       // [1]
    int32_t *pick_h = s_h + 1, *pick_f = pick_h + kPairBatch;       // [kPairBatch] choices, their fill before
    for (int32_t x = tid; x < m * RG; x += kPairBatch * kWave) {
        after[x] = pa.after[(int64_t)b * kPairBatch * RG + x];
        pk[x] = pa.pk[(int64_t)b * kPairBatch * RG + x];
    }
    for (int32_t h = tid; h < RG; h += kPairBatch * kWave) {
        base[h] = a.base[(int64_t)b * RG + h];
        filled[h] = a.filled[(int64_t)b * RG + h];
        hcnt[h] = a.count[h % G];
    }
    // wave j: Q of the batch's j-th cell, lane = layer
    const bool act = lane < L;
    const int32_t ll = act ? lane : L - 1;
    int4 q[PV / 4];
    int32_t kl = 0;  // lane j: the batch's j-th cell
    if (lane < m) kl = a.order[(int64_t)b * K + pos0 + lane];
    const int32_t w = b == 0 ? 1 : a.w;
    uint64_t word = 0;  // lane j: the j-th cell's draw
    if (b > 0 && lane < m) word = a.words[(int64_t)(b - 1) * (2 * (int64_t)a.N + K) + 2 * (int64_t)a.N + pos0 + lane];
    const int32_t rho_w = pair_rho(word, w);  // its rank when w or more row-shards are open
    {
        const int32_t k = __builtin_amdgcn_readlane(kl, wv < m ? wv : 0);
        const int4 *qp = reinterpret_cast<const int4 *>(a.Qc + ((int64_t)b * K + k) * LP) + ll;
#pragma unroll
        for (int x = 0; x < PV / 4; ++x) q[x] = x < p4 ? qp[x * L] : make_int4(0, 0, 0, 0);
    }
    int4 *W = reinterpret_cast<int4 *>(a.Wt + (int64_t)b * RG * LP);
    if (WL)
        for (int32_t x = tid; x < RG * n4; x += kPairBatch * kWave) wl[x] = W[x];
    auto share_q = [&](int4 *to) {
#pragma unroll
        for (int x = 0; x < PV / 4; ++x)
            if (x < p4 && act) to[x * L + ll] = q[x];
    };
    auto choose = [&](int32_t i) {  // (wave 0)
        const int32_t h = pair_choice(after + i * RG, pk + i * RG, base, filled, hcnt, RG, w, readlane64(word, i),
                                      __builtin_amdgcn_readlane(rho_w, i));
        if (lane == 0) {
            *s_h = h;
            base[h] = after[i * RG + h];
            pick_h[i] = h;
            pick_f[i] = filled[h];
            filled[h] += 1;
        }
    };
    // row h of W takes the cell of qv; waves from w0 on (the same threads for
    // a row in every step, so its stores to global memory stay in order
    // without a barrier that waits for them)
    auto apply = [&](int32_t h, const int4 *qv, int4 *to, int32_t w0) {
        for (int32_t x = tid - w0 * kWave; x < n4; x += (kPairBatch - w0) * kWave) {
            const int4 v = WL ? wl[h * n4 + x] : W[(int64_t)h * n4 + x], c = qv[x];
            const int4 s = make_int4(v.x + c.x, v.y + c.y, v.z + c.z, v.w + c.w);
            to[x] = s;
            W[(int64_t)h * n4 + x] = s;
        }
    };
    auto refresh = [&](int32_t h, int32_t mx) {
        int64_t sum;
        int32_t most;
        layer_reduce<true>(act ? mx : 0, sum, most);
        if (lane == 63) {
            after[wv * RG + h] = sum;
            pk[wv * RG + h] = most;
        }
    };
    if (WL) {
        // wave 0 chooses while the others add the previous cell to its row;
        // then the later cells' waves form their numbers from the row and the
        // current cell's Q
        int32_t hp = 0;
        for (int32_t i = 0; i < m; ++i) {
            lds_barrier();
            if (wv == i) share_q(qcur + (i & 1) * n4);
            if (wv == 0) choose(i);
            else if (i > 0) apply(hp, qcur + ((i - 1) & 1) * n4, wl + hp * n4, 1);
            lds_barrier();
            const int32_t h = hp = *s_h;
            if (wv > i && wv < m) {
                const int4 *row = wl + h * n4 + ll, *qv = qcur + (i & 1) * n4 + ll;
                int32_t mx = INT32_MIN;
#pragma unroll
                for (int x = 0; x < PV / 4; ++x)
                    if (x < p4) {
                        const int4 v = row[x * L], c = qv[x * L];
                        mx = max4_sum(mx, make_int4(v.x + c.x, v.y + c.y, v.z + c.z, v.w + c.w), q[x]);
                    }
                refresh(h, mx);
            }
        }
        lds_barrier();
        if (wv > 0) apply(hp, qcur + ((m - 1) & 1) * n4, wl + hp * n4, 1);
    } else {
        if (wv == 0) share_q(qcur);
        for (int32_t i = 0; i < m; ++i) {
            lds_barrier();
            if (wv == 0) choose(i);
            lds_barrier();
            const int32_t h = *s_h;
            apply(h, qcur, wl, 0);
            lds_barrier();
            if (wv == i + 1) share_q(qcur);
            if (wv > i && wv < m) {
                int32_t mx = INT32_MIN;
#pragma unroll
                for (int x = 0; x < PV / 4; ++x)
                    if (x < p4) mx = max4_sum(mx, wl[x * L + ll], q[x]);
                refresh(h, mx);
            }
        }
    }
    lds_barrier();
    if (tid < m) {
        const int32_t h = pick_h[tid], r = h / G, g = h - r * G;
        a.cell_to[(int64_t)b * K + kl] = r * D + a.slots[g * D + pick_f[tid]];
    }
    for (int32_t h = tid; h < RG; h += kPairBatch * kWave) {
        a.base[(int64_t)b * RG + h] = base[h];
        a.filled[(int64_t)b * RG + h] = filled[h];
    }
}

// The layouts of the paired trials (workgroups of a trial in blockIdx.x).
__global__ void __launch_bounds__(256) k_pair_out(TrialArgs a) {
    const int b = blockIdx.y;
    if (!a.ok[b]) return;
    for (int32_t i = blockIdx.x * 256 + threadIdx.x; i < a.N; i += gridDim.x * 256)
        a.out[(int64_t)b * a.N + i] = a.cell_to[(int64_t)b * a.K + a.cellk[(int64_t)b * a.N + i]];
}

// EDPAwarePair of candidate b (block per candidate).
// WG: the trial's row-shard loads W stay in its slice of a.Wt in HBM (when
// they do not fit LDS next to the rest); every W access is a coalesced
// 16-byte read or an update of one row by the whole workgroup.
template <bool WG>
__global__ void __launch_bounds__(1024) k_pack_pair(TrialArgs a, PackFast pf) {
    extern __shared__ __align__(16) char spair[];
    __shared__ int32_t s_h;
    const int b = blockIdx.x, tid = threadIdx.x, nt = blockDim.x, lane = lane_id(), wv = wave_id();
    if (!a.ok[b]) return;  // uniform
    const int32_t N = a.N, K = a.K, RG = a.RG, LP = a.LP, L = a.L, P = a.P, G = a.G, D = a.D;
    const int32_t w = b == 0 ? 1 : a.w;
    const uint64_t *wd = b == 0 ? nullptr : a.words + (int64_t)(b - 1) * (2 * (int64_t)N + K);
    int64_t *after = reinterpret_cast<int64_t *>(spair);            // [RG]
    int64_t *pkv = after + RG, *base = pkv + RG;                    // [RG], [RG]
    int64_t *speak = base + RG;                                     // [K]
    int32_t *lds_next = reinterpret_cast<int32_t *>(speak + K + ((3 * RG + K) & 1));  // 16-byte aligned
    int32_t *Wl = WG ? a.Wt + (int64_t)b * RG * LP : lds_next;      // [RG][LP]
    int32_t *qb = WG ? lds_next : Wl + (int64_t)RG * LP;            // [2][LP]
    int32_t *mxs = qb + 2 * LP;                                     // [RG][L]
    int32_t *filled = mxs + RG * L;                                 // [RG]
    int32_t *hcnt = filled + RG;                                    // [RG]
    int32_t *order = hcnt + RG;                                     // [K]
    int32_t *cell_to = order + K;                                   // [K]
    const int32_t *Qc = a.Qc + (int64_t)b * K * LP;
    for (int32_t k = tid; k < K; k += nt) speak[k] = a.peak[(int64_t)b * K + k];
    for (int64_t x = tid; x < (int64_t)RG * LP; x += nt) Wl[x] = 0;
    for (int32_t h = tid; h < RG; h += nt) {
        base[h] = 0;
        filled[h] = 0;
        hcnt[h] = a.count[h % G];
    }
    __syncthreads();
    // order: cells by decreasing peak, then index
    for (int32_t k = tid; k < K; k += nt) {
        const int64_t v = speak[k];
        int32_t rank = 0;
        for (int32_t f = 0; f < K; ++f) {
            const int64_t u = speak[f];
            rank += (u > v) || (u == v && f < k);
        }
        order[rank] = k;
    }
    __syncthreads();
    for (int32_t e = tid; e < LP; e += nt) qb[e] = Qc[(int64_t)order[0] * LP + e];
    __syncthreads();
    constexpr int kPre = 16;  // Q entries per thread held for the next step (LP <= 16 * 1024)
    uint64_t wpair = 0;       // wave 0: pairing draws of steps pbase .. pbase + 63, one per lane
    int32_t pbase = -kWave;
    for (int32_t pos = 0; pos < K; ++pos) {
        if (wv == 0 && wd && pos - pbase == kWave) {
            pbase = pos;
            wpair = pos + lane < K ? wd[2 * (int64_t)N + pos + lane] : 0;
        }
        const int32_t k = order[pos];
        const int32_t *qk = qb + (pos & 1) * LP;
        // next cell's Q row into registers while this step runs
        int32_t nq[kPre];
        const bool more = pos + 1 < K;
        const int64_t nrow = more ? (int64_t)order[pos + 1] * LP : 0;
#pragma unroll
        for (int u = 0; u < kPre; ++u) {
            const int32_t e = tid + u * nt;
            nq[u] = more && e < LP ? Qc[nrow + e] : 0;
        }
        // per (row-shard, layer): max over ranks of W + Q_k; a thread holds 4
        // consecutive entries, a layer's ranks span P / 4 adjacent threads.
        // Every thread runs the same number of iterations, so the DPP maximum
        // always sees its whole group.
        {
            const int32_t c4 = LP >> 2, g4 = P >> 2;
            const int32_t iters = (RG * c4 + nt - 1) / nt;
            int32_t y = tid, h = 0;
            while (y >= c4) {
                y -= c4;
                ++h;
            }
            for (int32_t it = 0; it < iters; ++it) {
                const bool cand = h < RG && filled[h] < hcnt[h];
                int32_t mx = INT32_MIN;
                if (cand) {
                    const int4 wv4 = reinterpret_cast<const int4 *>(Wl + (int64_t)h * LP)[y];
                    const int4 qv4 = reinterpret_cast<const int4 *>(qk)[y];
                    mx = max(max(wv4.x + qv4.x, wv4.y + qv4.y), max(wv4.z + qv4.z, wv4.w + qv4.w));
                }
                mx = seg_max32(mx, g4);
                if (cand && (y & (g4 - 1)) == 0) mxs[h * L + y / g4] = mx;
                y += nt;
                while (y >= c4) {
                    y -= c4;
                    ++h;
                }
            }
        }
        __syncthreads();
        for (int32_t h = tid; h < RG; h += nt) {
            int64_t af = 0, pk = 0;
            if (filled[h] < hcnt[h]) {
                if ((L & 3) == 0) {  // the row's maxima as 16-byte reads (mxs is 16-byte aligned)
                    const int4 *m4 = reinterpret_cast<const int4 *>(mxs + h * L);
                    for (int32_t l4 = 0; l4 < (L >> 2); ++l4) {
                        const int4 v = m4[l4];
                        af += (int64_t)v.x + v.y + v.z + v.w;
                        const int32_t m = max(max(v.x, v.y), max(v.z, v.w));
                        pk = m > pk ? m : pk;
                    }
                } else {
                    for (int32_t l = 0; l < L; ++l) {
                        const int32_t mx = mxs[h * L + l];
                        af += mx;
                        pk = mx > pk ? mx : pk;
                    }
                }
            }
            after[h] = af;
            pkv[h] = pk;
        }
        __syncthreads();
        if (wv == 0) {
            // candidates in EDPAwarePair order (increase, peak, index); the
            // rho-th of the leading min(w, |candidates|)
            int32_t cnt = 0;
            for (int32_t hb = 0; hb < RG; hb += kWave)
                cnt += __popcll(__ballot(hb + lane < RG && filled[hb + lane] < hcnt[hb + lane]));
            const int32_t wp = w < cnt ? w : cnt;
            int32_t rho = 0;
            if (wp > 1) {
                const uint64_t total = (((uint64_t)1) << wp) - 1;
                const uint64_t pick = bounded(readlane64(wpair, pos - pbase), total);
                uint64_t pref = 0;
                for (rho = 0; rho < wp; ++rho) {
                    pref += ((uint64_t)1) << (wp - 1 - rho);
                    if (pref > pick) break;
                }
            }
            int64_t p0 = LLONG_MIN, p1 = LLONG_MIN, p2 = LLONG_MIN;
            for (int32_t pass = 0; pass <= rho; ++pass) {
                int64_t k0 = LLONG_MAX, k1 = LLONG_MAX, k2 = LLONG_MAX, kj = LLONG_MAX;
                for (int32_t hb = 0; hb < RG; hb += kWave) {
                    const int32_t h = hb + lane;
                    if (h < RG && filled[h] < hcnt[h]) {
                        const int64_t v0 = after[h] - base[h], v1 = pkv[h], v2 = h;
                        if ((pass == 0 || lex_less(p0, p1, p2, v0, v1, v2)) && lex_less(v0, v1, v2, k0, k1, k2)) {
                            k0 = v0; k1 = v1; k2 = v2; kj = v2;
                        }
                    }
                }
                wave_lexmin(k0, k1, k2, kj);
                p0 = k0; p1 = k1; p2 = k2;
            }
            if (lane == 0) s_h = (int32_t)p2;
        }
        __syncthreads();
        const int32_t h = s_h;
        for (int32_t e = tid; e < LP; e += nt) Wl[(int64_t)h * LP + e] += qk[e];
        if (tid == 0) {
            const int32_t r = h / G, g = h - r * G;
            base[h] = after[h];
            cell_to[k] = r * D + a.slots[g * D + filled[h]];
            filled[h] += 1;
        }
        int32_t *qn = qb + ((pos + 1) & 1) * LP;
#pragma unroll
        for (int u = 0; u < kPre; ++u) {
            const int32_t e = tid + u * nt;
            if (more && e < LP) qn[e] = nq[u];
        }
        __syncthreads();
    }
    const int32_t *cellk = a.cellk + (int64_t)b * N;
    int32_t *out = a.out + (int64_t)b * N;
    for (int32_t i = tid; i < N; i += nt) out[i] = cell_to[cellk[i]];
}

// Canonical form of layouts[b] (b < n) into canon[b], with an order-free hash
// of it.  One workgroup per layout, cell tables in LDS; bound by the two
// passes over the layout (a quarter of the threads and tables in global
// memory: 168 us for 16 layouts of 32768 samples, now 35 us).
__global__ void __launch_bounds__(1024) k_canonical(const int32_t *layouts, int32_t N, int32_t R, int32_t D,
                                                    const int32_t *slots, const int32_t *count,
                                                    const int32_t *slot_shard, int32_t *canon, uint64_t *hash) {
    extern __shared__ __align__(16) int32_t scan_lds[];
    __shared__ uint64_t part[16];
    const int b = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int32_t B = R * D;
    const int32_t *lay = layouts + (int64_t)b * N;
    int32_t *cmin = scan_lds, *newd = cmin + B, *rkey = newd + B;  // [B], [B], [R]
    for (int32_t c = tid; c < B; c += nt) cmin[c] = INT32_MAX;
    __syncthreads();
    for (int32_t i = tid; i < N; i += nt) {
        const int32_t c = lay[i];
        if (c >= 0 && c < B) atomicMin(&cmin[c], i);
    }
    __syncthreads();
    // slot of each cell within its row-shard after ordering by smallest id
    for (int32_t c = tid; c < B; c += nt) {
        const int32_t r = c / D, d = c % D, g = slot_shard[d];
        const int32_t v = cmin[c];
        int32_t rank = 0;
        for (int32_t x = 0; x < count[g]; ++x) rank += cmin[r * D + slots[g * D + x]] < v;
        newd[c] = slots[g * D + rank];
    }
    // row key: smallest id of the cell that lands in slot 0
    for (int32_t r = tid; r < R; r += nt) rkey[r] = INT32_MAX;
    __syncthreads();
    for (int32_t c = tid; c < B; c += nt)
        if (newd[c] == 0) rkey[c / D] = cmin[c];
    __syncthreads();
    for (int32_t c = tid; c < B; c += nt) {
        const int32_t v = rkey[c / D];
        int32_t rank = 0;
        for (int32_t x = 0; x < R; ++x) rank += rkey[x] < v;
        newd[c] = rank * D + newd[c];
    }
    __syncthreads();
    uint64_t h = 0;
    for (int32_t i = tid; i < N; i += nt) {
        const int32_t c = lay[i];
        const int32_t v = (c >= 0 && c < B) ? newd[c] : -1;
        canon[(int64_t)b * N + i] = v;
        h += mix64(((uint64_t)(uint32_t)i << 32) | (uint32_t)v);
    }
    h = (uint64_t)wave_sum((int64_t)h);
    if (lane_id() == 0) part[wave_id()] = h;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < nt / kWave; ++w) h += part[w];
        hash[b] = h;
    }
}

// Selection and cyclic fill.  cand m: 0 x_length, 1 x_paired (kept when
// strictly better than x_length), m >= 2 trial m-1 (kept when it succeeded).
// Layouts are compared only when their hashes are equal (every pair, element
// by element in one workgroup: 316 us for 15 layouts of 4096 samples and
// 2.2 ms for 32768, now 32 us and 34 us).
__global__ void __launch_bounds__(1024) k_pack_select(const int32_t *canon, const uint64_t *hash, const int64_t *scores,
                                                     const int32_t *ok, const int32_t *status,
                                                     int32_t M, int32_t N,
                                                     int32_t *keep_order, int32_t *meta) {
    __shared__ int32_t valid[64], kept[64], order[64];
    __shared__ int32_t differ;
    const int tid = threadIdx.x;
    if (tid < M) {
        int32_t v = 1;
        if (tid == 1) {
            const int64_t *a = scores + 3, *x = scores;
            v = ok[0] && status[1] == 0 && lex_less(a[0], a[1], a[2], x[0], x[1], x[2]);
        } else if (tid >= 2) {
            v = ok[tid - 1] && status[tid] == 0;
        }
        valid[tid] = v;
        kept[tid] = 0;
    }
    __syncthreads();
    for (int m = 0; m < M; ++m) {
        if (!valid[m]) continue;
        bool dup = false;
        for (int u = 0; u < m && !dup; ++u) {
            if (!kept[u] || hash[u] != hash[m]) continue;  // (uniform)
            if (tid == 0) differ = 0;
            __syncthreads();
            for (int32_t i = tid; i < N; i += blockDim.x)
                if (canon[(int64_t)m * N + i] != canon[(int64_t)u * N + i]) differ = 1;
            __syncthreads();
            dup = differ == 0;
            __syncthreads();
        }
        if (tid == 0) kept[m] = dup ? 0 : 1;
        __syncthreads();
    }
    if (tid == 0) {
        int32_t n = 0;
        for (int m = 0; m < M; ++m)
            if (kept[m]) order[n++] = m;
        // insertion sort by (score, discovery)
        for (int x = 1; x < n; ++x) {
            const int32_t v = order[x];
            int y = x - 1;
            while (y >= 0) {
                const int64_t *a = scores + 3 * (int64_t)order[y], *c = scores + 3 * (int64_t)v;
                if (lex_less(c[0], c[1], c[2], a[0], a[1], a[2])) {
                    order[y + 1] = order[y];
                    --y;
                } else {
                    break;
                }
            }
            order[y + 1] = v;
        }
        for (int x = 0; x < n; ++x) keep_order[x] = order[x];
        int32_t ntr = 0;
        for (int m = 2; m < M; ++m) ntr += ok[m - 1] && status[m] == 0;
        meta[0] = n;
        meta[1] = ntr;
    }
}

__global__ void k_pack_fill(const int32_t *canon, const int64_t *scores, const int32_t *keep_order,
                            const int32_t *meta, int32_t N, int32_t *population, int64_t *pop_scores) {
    const int m = blockIdx.x;
    const int32_t src = keep_order[m % meta[0]];
    for (int32_t i = threadIdx.x; i < N; i += blockDim.x)
        population[(int64_t)m * N + i] = canon[(int64_t)src * N + i];
    if (threadIdx.x < 3) pop_scores[(int64_t)m * 3 + threadIdx.x] = scores[(int64_t)src * 3 + threadIdx.x];
}

}  // namespace rp

namespace rp {
int rank_sort_desc(const int32_t *lengths, int32_t N, int32_t *sigma, Scratch &scr, hipStream_t stream) {
    int32_t *rank = scr.get<int32_t>(N);
    if (scr.failed()) return ROUTEPACK_E_DEVICE;
    const int32_t nt = (N + 255) / 256;
    int32_t slices = 2048 / nt;
    slices = slices < 1 ? 1 : (slices > nt ? nt : slices);
    const int32_t tiles = (nt + slices - 1) / slices;
    slices = (nt + tiles - 1) / tiles;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)(nt < 64 ? nt : 64)), dim3(256), 0, stream, rank, (int64_t)N, 0);
    hipLaunchKernelGGL(k_rank_count, dim3((unsigned)nt, (unsigned)slices), dim3(256), 0, stream, lengths, N, tiles, rank);
    hipLaunchKernelGGL(k_rank_place, dim3((unsigned)nt), dim3(256), 0, stream, (const int32_t *)rank, N, sigma);
    return hipGetLastError() == hipSuccess ? ROUTEPACK_OK : ROUTEPACK_E_DEVICE;
}
}  // namespace rp

using namespace rp;

extern "C" int routepack_pack_rows(const routepack_problem *prob, const int32_t *lengths,
                                   const int32_t *q, uint64_t seed, int32_t n_trials,
                                   int32_t choice_width, int32_t pop_size, int32_t *r_star,
                                   int32_t *certified, int32_t *population, int64_t *scores,
                                   int32_t *info, hipStream_t stream) {
    Topology topo;
    RP_TRY(check_problem(prob, &topo));
    if (!lengths || (!q && prob->n_layers > 0) || !r_star || !certified || !population || !scores)
        return ROUTEPACK_E_INVALID;
    if (n_trials < 2 || n_trials > 64 || choice_width < 1 || choice_width > 62 || pop_size < 1)
        return ROUTEPACK_E_INVALID;
    const int32_t N = prob->n_samples, D = topo.D, G = topo.G;
    const int64_t C = prob->capacity;
    const int64_t LP = (int64_t)prob->n_layers * prob->n_ranks;
    if (LP > 4096) return ROUTEPACK_E_UNSUPPORTED;
    WindowStats ws;
    RP_TRY(window_stats(prob, lengths, q, &ws, stream));
    if (ws.q_negative) return ROUTEPACK_E_INVALID;
    if (ws.min_t < 1 || ws.max_t > C) return ROUTEPACK_E_INFEASIBLE;
    int64_t r_lb = prob->min_rows > 1 ? prob->min_rows : 1;
    const int64_t a1 = (ws.sum_t + C * D - 1) / (C * D);
    const int64_t a2 = (ws.n_big + D - 1) / D;
    r_lb = a1 > r_lb ? a1 : r_lb;
    r_lb = a2 > r_lb ? a2 : r_lb;
    const int64_t r_max = N / D;
    if (r_lb > r_max) return ROUTEPACK_E_INFEASIBLE;

    Scratch scr(stream);
    DeviceProblem dp;
    RP_TRY(upload_problem(prob, topo, scr, &dp, stream));
    int32_t *sigma = scr.get<int32_t>(N);
    int32_t *x_len = scr.get<int32_t>(N);
    int32_t *flag = scr.get<int32_t>(4);
    if (scr.failed()) return ROUTEPACK_E_DEVICE;
    RP_TRY(rank_sort_desc(lengths, N, sigma, scr, stream));
    int64_t R = -1;
    for (int64_t r = r_lb; r <= r_max; ++r) {
        if (r * D > kMaxCells) return ROUTEPACK_E_UNSUPPORTED;
        if (C < ((int64_t)1 << 31))
            hipLaunchKernelGGL(k_ffd<int32_t>, dim3(1), dim3(64), (size_t)(4 * r * D), stream, lengths, sigma, N, C,
                               (int32_t)(r * D), x_len, flag);
        else
            hipLaunchKernelGGL(k_ffd<int64_t>, dim3(1), dim3(64), (size_t)(8 * r * D), stream, lengths, sigma, N, C,
                               (int32_t)(r * D), x_len, flag);
        int32_t ok = 0;
        RP_HIP(hipMemcpyAsync(&ok, flag, sizeof(ok), hipMemcpyDeviceToHost, stream));
        RP_HIP(hipStreamSynchronize(stream));
        if (ok) {
            R = r;
            break;
        }
    }
    if (R < 0) return ROUTEPACK_E_HEURISTIC;
    RP_TRY(overflow_check(prob, R, ws, false));
    const int32_t K = (int32_t)(R * D), RG = (int32_t)(R * G), M = n_trials;
    const int32_t nb = M - 1;  // blocks: x_paired + trials 1..M-2
    uint64_t *words = scr.get<uint64_t>((size_t)(M - 2 > 0 ? M - 2 : 1) * (2 * (size_t)N + K));
    TrialArgs ta;
    memset(&ta, 0, sizeof(ta));
    ta.t = lengths; ta.q = q; ta.sigma = sigma; ta.x_length = x_len;
    ta.N = N; ta.L = prob->n_layers; ta.P = prob->n_ranks; ta.D = D; ta.G = G; ta.R = (int32_t)R;
    ta.K = K; ta.RG = RG; ta.LP = (int32_t)LP; ta.w = choice_width; ta.C = C;
    ta.slots = dp.slots; ta.count = dp.count; ta.words = words;
    ta.cellk = scr.get<int32_t>((size_t)nb * N);
    // Cell sums and row-shard loads are int32 while every load stays below 2^31.
    const bool wide = w_entry_bound(prob, ws) > INT32_MAX;
    const size_t per_sum = wide ? 2 : 1;
    ta.Qc = scr.get<int32_t>(per_sum * nb * K * (LP ? LP : 1));
    ta.peak = scr.get<int64_t>((size_t)nb * K);
    ta.order = scr.get<int32_t>((size_t)nb * K);
    ta.Wt = scr.get<int32_t>(per_sum * nb * RG * (LP ? LP : 1));
    ta.base = scr.get<int64_t>((size_t)nb * RG);
    ta.after = scr.get<int64_t>((size_t)nb * RG);
    ta.pkv = scr.get<int64_t>((size_t)nb * RG);
    ta.filled = scr.get<int32_t>((size_t)nb * RG);
    ta.cell_to = scr.get<int32_t>((size_t)nb * K);
    // candidates: [0] x_length, [1..M-1] the blocks' layouts
    int32_t *cand = scr.get<int32_t>((size_t)M * N);
    int32_t *canon = scr.get<int32_t>((size_t)M * N);
    int64_t *cscore = scr.get<int64_t>((size_t)M * 3);
    int32_t *cstat = scr.get<int32_t>(M);
    int32_t *okv = scr.get<int32_t>(M);
    uint64_t *chash = scr.get<uint64_t>(M);
    int32_t *keep = scr.get<int32_t>(64);
    int32_t *meta = scr.get<int32_t>(2);
    if (scr.failed()) return ROUTEPACK_E_DEVICE;
    ta.out = cand + N;
    ta.ok = okv;
    if (M > 2)
        hipLaunchKernelGGL(k_seed_words, dim3(1024), dim3(256), 0, stream, seed, M, N, K, words);
    // every candidate slot starts as a valid layout (all samples in cell 0),
    // so a failed trial never leaves indices outside [0, R*D)
    hipLaunchKernelGGL(k_fill_i32, dim3(256), dim3(256), 0, stream, cand, (int64_t)M * N, 0);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, stream, okv, (int64_t)M, 0);
    RP_HIP(hipMemcpyAsync(cand, x_len, sizeof(int32_t) * N, hipMemcpyDeviceToDevice, stream));
    // Seed trials in stages for the common shapes, else k_pack_trials.
    // ROUTEPACK_PACK_KERNEL=single requests the latter.
    const char *pk_force = getenv("ROUTEPACK_PACK_KERNEL");
    // Batched pairing (k_pair_*) for layers that fit a wave and ranks that a
    // lane holds.  k_pack_pair beyond 64 layers or ranks or 512 row-shards,
    // for power-of-two ranks whose tables fit LDS: W there too when it fits,
    // else in HBM.  ROUTEPACK_PACK_W=hbm requests k_pack_pair with W in HBM.
    const int64_t pair_rest = 8 * (3 * (int64_t)RG + K + 1) +
                              4 * (2 * LP + (int64_t)RG * prob->n_layers + 2 * (int64_t)RG + 2 * (int64_t)K);
    const char *pw_force = getenv("ROUTEPACK_PACK_W");
    const bool force_hbm = pw_force && strcmp(pw_force, "hbm") == 0;
    const bool w_hbm = force_hbm || pair_rest + 4 * (int64_t)RG * LP > 150 * 1024;
    const int64_t pair_lds = pair_rest + (w_hbm ? 0 : 4 * (int64_t)RG * LP);
    const int32_t P = prob->n_ranks, L = prob->n_layers;
    const bool batched = !force_hbm && L <= kWave && P % 4 == 0 && P <= 64 && RG <= kPairMaxShards;
    const bool one_wg = P >= 4 && P <= 256 && (P & (P - 1)) == 0 && pair_lds <= 150 * 1024;
    const bool fast = !(pk_force && strcmp(pk_force, "single") == 0) && C < ((int64_t)1 << 31) && N < 65536 &&
                      LP > 0 && !wide && (batched || one_wg);
    if (fast) {
        PackFast pf;
        pf.mstart = scr.get<int32_t>((size_t)nb * (K + 1));
        pf.mlist = scr.get<int32_t>((size_t)nb * N);
        if (scr.failed()) return ROUTEPACK_E_DEVICE;
        const size_t fit_lds = (size_t)16 * K;
        RP_HIP(hipFuncSetAttribute((const void *)k_pack_fit, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fit_lds));
        if (K <= kFitSortedCells) {
            hipLaunchKernelGGL(k_pack_fit_sorted, dim3(nb), dim3(kFitThreads), fit_sorted_lds(K), stream, ta, pf);
        } else {
            hipLaunchKernelGGL(k_pack_fit, dim3(nb), dim3(64), fit_lds, stream, ta, pf);
        }
        if (P >= 4 && P <= 64 && (P & (P - 1)) == 0 && ((uintptr_t)q & 15) == 0) {
            const RowPieces pc = row_pieces(N, L, P);
            const int32_t items = nb * K;
            const unsigned wgs = (unsigned)((items + 3) / 4 * pc.n_pieces);
            hipLaunchKernelGGL(k_fill_i32, dim3(64), dim3(256), 0, stream, reinterpret_cast<int32_t *>(ta.peak),
                               (int64_t)2 * items, 0);
            hipLaunchKernelGGL(pc.one ? k_pack_cellrows<true> : k_pack_cellrows<false>, dim3(wgs), dim3(256), 0, stream,
                               ta, pf, pc, items, batched);
        } else {
            hipLaunchKernelGGL(k_pack_cellsum, dim3(K, nb), dim3(128), (size_t)4 * LP, stream, ta, pf, batched);
        }
        if (batched) {
            PairArgs pa;
            pa.after = scr.get<int64_t>((size_t)nb * kPairBatch * RG);
            pa.pk = scr.get<int32_t>((size_t)nb * kPairBatch * RG);
            if (scr.failed()) return ROUTEPACK_E_DEVICE;
            const bool wl = pair_resolve_lds(RG, LP, true) <= 150 * 1024;
            const size_t res_lds = pair_resolve_lds(RG, LP, wl);
            auto pick = [&](auto with, auto without) { return wl ? with : without; };
            auto resolve = P <= 8    ? pick(k_pair_resolve<8, true>, k_pair_resolve<8, false>)
                           : P <= 16 ? pick(k_pair_resolve<16, true>, k_pair_resolve<16, false>)
                           : P <= 32 ? pick(k_pair_resolve<32, true>, k_pair_resolve<32, false>)
                                     : pick(k_pair_resolve<64, true>, k_pair_resolve<64, false>);
            if (res_lds > 64 * 1024)
                RP_HIP(hipFuncSetAttribute((const void *)resolve, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)res_lds));
            const bool half = L <= 32;  // two row-shards per wave
            const int32_t slots = half ? (RG + 1) / 2 : RG;
            hipLaunchKernelGGL(k_pair_start, dim3(nb), dim3(1024), (size_t)8 * K, stream, ta);
            for (int32_t pos = 0; pos < K; pos += kPairBatch) {
                const dim3 grid((unsigned)((slots + 7) / 8), 2, (unsigned)nb);
                if (half) hipLaunchKernelGGL(k_pair_table<true>, grid, dim3(256), 0, stream, ta, pa, pos);
                else hipLaunchKernelGGL(k_pair_table<false>, grid, dim3(256), 0, stream, ta, pa, pos);
                hipLaunchKernelGGL(resolve, dim3(nb), dim3(kPairBatch * kWave), res_lds, stream, ta, pa, pos);
            }
            hipLaunchKernelGGL(k_pair_out, dim3((unsigned)(N < 65536 / 4 ? 8 : 32), (unsigned)nb), dim3(256), 0, stream,
                               ta);
        } else {
            const void *pair_fn = w_hbm ? (const void *)k_pack_pair<true> : (const void *)k_pack_pair<false>;
            RP_HIP(hipFuncSetAttribute(pair_fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pair_lds));
            if (w_hbm) hipLaunchKernelGGL(k_pack_pair<true>, dim3(nb), dim3(1024), (size_t)pair_lds, stream, ta, pf);
            else hipLaunchKernelGGL(k_pack_pair<false>, dim3(nb), dim3(1024), (size_t)pair_lds, stream, ta, pf);
        }
    } else {
        hipLaunchKernelGGL(wide ? k_pack_trials<int64_t> : k_pack_trials<int32_t>, dim3(nb), dim3(64), 0, stream, ta);
    }
    RP_HIP(hipGetLastError());
    // Score every candidate (failed trials leave garbage layouts: their
    // status is nonzero or they are ignored by the selection).
    RP_TRY(eval_layouts(prob, topo, dp, lengths, q, (int32_t)R, M, cand, cscore, cstat, nullptr,
                        nullptr, nullptr, sums_fit32(ws), stream));
    const int threads = N > 1024 ? 1024 : 256;
    hipLaunchKernelGGL(k_canonical, dim3(M), dim3(threads), (size_t)4 * (2 * K + R), stream, cand, N, (int32_t)R, D,
                       dp.slots, dp.count, dp.slot_shard, canon, chash);
    hipLaunchKernelGGL(k_pack_select, dim3(1), dim3(threads), 0, stream, canon, chash, cscore, okv, cstat, M, N, keep,
                       meta);
    hipLaunchKernelGGL(k_pack_fill, dim3(pop_size), dim3(256), 0, stream, canon, cscore, keep, meta, N,
                       population, scores);
    RP_HIP(hipGetLastError());
    int32_t hmeta[2] = {0, 0};
    RP_HIP(hipMemcpyAsync(hmeta, meta, sizeof(hmeta), hipMemcpyDeviceToHost, stream));
    RP_HIP(hipStreamSynchronize(stream));
    *r_star = (int32_t)R;
    *certified = (R == r_lb) ? 1 : 0;
    if (info) {
        info[0] = (int32_t)r_lb;
        info[1] = hmeta[0];
        info[2] = hmeta[1];
    }
    return ROUTEPACK_OK;
}
