// Exact objective of layouts (Eqs. cell-token-statistics, stage-aware-
// attention, row-expert-load, row-expert-cost, lexicographic-score) with
// feasibility status (Eqs. sample-bijection .. token-capacity) and the online
// load diagnostics (Eqs. global-ep-cv and ep-efficiency).
//
// k_eval_lists, one workgroup per layout: the cell statistics in LDS, from
// them A of every row-shard h = r*G + g and the status, and the samples
// grouped by row-shard.  k_eval_rows, one wave per (layout, row-shard, up to
// 256 entries of whole layers): adds the members' q rows into W_h, then
// J(h) = A(h) + 2^F sum_l max_p W_h and the per-layer max/sum of W_h for the
// diagnostics.  k_eval_finalize, one workgroup per layout: the score tuple,
// status and diagnostics.  k_eval_rowshard does the first two steps for the
// remaining shapes (see eval_layouts).
#include <math.h>

#include "rp_device.h"
#include "rp_internal.h"
#include "rp_rows.h"

namespace rp {

struct EvalArgs {
    const int32_t *t;        // [N]
    const int32_t *q;        // [N][L][P]
    const int32_t *layouts;  // [n][N]
    int32_t N, L, P, D, G, R, S, F;
    int64_t C;
    const int32_t *slots, *count, *slot_shard;
    const int64_t *alpha, *beta;
    int32_t *status;                        // [n]
    int64_t *Jbuf, *Abuf;                   // [n][R*G]
    int64_t *wmax, *wsum;                   // [n][R*G][L] or null
    int64_t items;                          // n * R*G
};

__global__ void __launch_bounds__(256) k_eval_rowshard(EvalArgs a) {
    extern __shared__ char smem[];
    const int64_t LP = (int64_t)a.L * a.P;
    const int64_t RG = (int64_t)a.R * a.G;
    int64_t *W = reinterpret_cast<int64_t *>(smem);     // [LP]
    int64_t *cT = W + LP;                               // [D] (only shard slots used)
    int64_t *cQ = cT + a.D;                             // [D]
    int32_t *cN = reinterpret_cast<int32_t *>(cQ + a.D);  // [D]
    int32_t *mem = cN + a.D;                            // [256]
    int32_t *nmem = mem + 256;                          // [1]
    int32_t *stat = nmem + 1;                           // [1]
    int64_t *red = reinterpret_cast<int64_t *>(((uintptr_t)(stat + 1) + 7) & ~(uintptr_t)7);  // [4]

    const int64_t item = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (item >= a.items) return;
    const int64_t lay_idx = item / RG;
    const int64_t h = item % RG;
    const int32_t r = (int32_t)(h / a.G), g = (int32_t)(h % a.G);
    const int32_t *lay = a.layouts + lay_idx * a.N;
    const int64_t B = (int64_t)a.R * a.D;
    const int tid = threadIdx.x;

    for (int64_t e = tid; e < LP; e += blockDim.x) W[e] = 0;
    for (int d = tid; d < a.D; d += blockDim.x) {
        cT[d] = 0;
        cQ[d] = 0;
        cN[d] = 0;
    }
    if (tid == 0) {
        *nmem = 0;
        *stat = 0;
    }
    __syncthreads();
    for (int64_t base = 0; base < a.N; base += blockDim.x) {
        const int64_t i = base + tid;
        if (i < a.N) {
            const int32_t c = lay[i];
            if (c < 0 || c >= B) {
                if (h == 0) atomicOr(stat, 1);
            } else if (c / a.D == r && a.slot_shard[c % a.D] == g) {
                const int d = c % a.D;
                const int64_t ti = a.t[i];
                atomicAdd(reinterpret_cast<unsigned long long *>(&cT[d]), (unsigned long long)ti);
                atomicAdd(reinterpret_cast<unsigned long long *>(&cQ[d]), (unsigned long long)(ti * ti));
                atomicAdd(&cN[d], 1);
                mem[atomicAdd(nmem, 1)] = (int32_t)i;
            }
        }
        __syncthreads();
        const int32_t nm = *nmem;
        for (int32_t m = 0; m < nm; ++m) {
            const int32_t *qi = a.q + (int64_t)mem[m] * LP;
            for (int64_t e = tid; e < LP; e += blockDim.x) W[e] += qi[e];
        }
        __syncthreads();
        if (tid == 0) *nmem = 0;
        __syncthreads();
    }
    // Per-layer max and sum of W_h; E = 2^F sum_l max_p W.
    int64_t esum = 0;
    for (int l = tid; l < a.L; l += blockDim.x) {
        int64_t mx = W[(int64_t)l * a.P], sm = 0;
        for (int p = 0; p < a.P; ++p) {
            const int64_t v = W[(int64_t)l * a.P + p];
            mx = v > mx ? v : mx;
            sm += v;
        }
        esum += mx;
        if (a.wmax) {
            const int64_t o = (lay_idx * RG + h) * a.L + l;
            a.wmax[o] = mx;
            a.wsum[o] = sm;
        }
    }
    esum = wave_sum(esum);
    if (lane_id() == 0) red[wave_id()] = esum;
    __syncthreads();
    if (tid == 0) {
        int64_t e = 0;
        for (int w = 0; w < (int)(blockDim.x / kWave); ++w) e += red[w];
        int32_t st = *stat;
        int64_t A = 0;
        const int32_t m = a.count[g];
        for (int s = 0; s < a.S; ++s) {
            int64_t mx = 0;
            for (int x = 0; x < m; ++x) {
                const int d = a.slots[g * a.D + x];
                const int64_t cost = a.alpha[s] * cT[d] + a.beta[s] * cQ[d];
                if (x == 0 || cost > mx) mx = cost;
            }
            A += mx;
        }
        for (int x = 0; x < m; ++x) {
            const int d = a.slots[g * a.D + x];
            if (cT[d] > a.C) st |= 2;
            if (cN[d] == 0) st |= 4;
        }
        if (st) atomicOr(&a.status[lay_idx], st);
        a.Abuf[lay_idx * RG + h] = A;
        a.Jbuf[lay_idx * RG + h] = A + (e << a.F);
    }
}

struct ListArgs {
    const int32_t *t, *layouts;
    int32_t N, D, G, R, S;
    int64_t C;
    const int32_t *slots, *count, *slot_shard;
    const int64_t *alpha, *beta;
    int32_t *status;       // [n]
    int64_t *Jbuf, *Abuf;  // [n][R*G], both set to A
    int32_t *list;         // [n][N] samples grouped by row-shard
    int32_t *hstart;       // [n][R*G + 1] where each row-shard's samples begin
};

// LDS of k_eval_lists: sum t, sum t^2 and member count of every cell, member
// count of every row-shard, the status.
__host__ __device__ inline size_t eval_lists_lds(int64_t B, int64_t RG) { return (size_t)(B * 20 + RG * 4 + 4); }

__global__ void __launch_bounds__(1024) k_eval_lists(ListArgs a) {
    // (a name of its own: every declaration of one name shares its alignment,
    // and the 64-bit LDS atomics need theirs)
    extern __shared__ __align__(16) char slists[];
    const int32_t B = a.R * a.D, RG = a.R * a.G, N = a.N, D = a.D, G = a.G;
    int64_t *cT = reinterpret_cast<int64_t *>(slists);  // [B]
    int64_t *cQ = cT + B;                             // [B]
    int32_t *cN = reinterpret_cast<int32_t *>(cQ + B);  // [B]
    int32_t *hc = cN + B;                             // [RG] counts, then the next free place
    int32_t *s_stat = hc + RG;                        // [1]
    const int tid = threadIdx.x, nt = blockDim.x, lane = lane_id();
    const int64_t lay = blockIdx.x;
    const int32_t *cells = a.layouts + lay * N;
    int32_t *list = a.list + lay * N, *hstart = a.hstart + lay * (RG + 1);
    for (int32_t c = tid; c < B; c += nt) {
        cT[c] = 0;
        cQ[c] = 0;
        cN[c] = 0;
    }
    for (int32_t h = tid; h < RG; h += nt) hc[h] = 0;
    if (tid == 0) *s_stat = 0;
    __syncthreads();
    int32_t st = 0;
    for (int32_t i = tid; i < N; i += nt) {
        const int32_t c = cells[i];
        if (c < 0 || c >= B) {
            st = 1;
            continue;
        }
        const int64_t ti = a.t[i];
        const int32_t r = c / D;
        atomicAdd(reinterpret_cast<unsigned long long *>(&cT[c]), (unsigned long long)ti);
        atomicAdd(reinterpret_cast<unsigned long long *>(&cQ[c]), (unsigned long long)(ti * ti));
        atomicAdd(&cN[c], 1);
        atomicAdd(&hc[r * G + (G == 1 ? 0 : a.slot_shard[c - r * D])], 1);
    }
    __syncthreads();
    // where each row-shard's list begins (first wave), A and the status (all)
    if (tid < kWave) {
        int32_t carry = 0;
        for (int32_t hb = 0; hb < RG; hb += kWave) {
            const int32_t h = hb + lane;
            const int32_t v = h < RG ? hc[h] : 0;
            const int32_t incl = (int32_t)wave_incl_scan(v);
            if (h < RG) {
                hc[h] = carry + incl - v;
                hstart[h] = carry + incl - v;
            }
            carry += __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        if (lane == 0) hstart[RG] = carry;
    }
    for (int32_t c = tid; c < B; c += nt) st |= (cT[c] > a.C ? 2 : 0) | (cN[c] == 0 ? 4 : 0);
    for (int32_t h = tid; h < RG; h += nt) {
        const int32_t r = h / G, g = h - r * G, m = a.count[g];
        int64_t A = 0;
        for (int s = 0; s < a.S; ++s) {
            int64_t mx = 0;
            for (int x = 0; x < m; ++x) {
                const int32_t c = r * D + a.slots[g * D + x];
                const int64_t cost = a.alpha[s] * cT[c] + a.beta[s] * cQ[c];
                if (x == 0 || cost > mx) mx = cost;
            }
            A += mx;
        }
        a.Abuf[lay * RG + h] = A;
        a.Jbuf[lay * RG + h] = A;
    }
    if (st) atomicOr(s_stat, st);
    __syncthreads();
    if (tid == 0) a.status[lay] = *s_stat;
    for (int32_t i = tid; i < N; i += nt) {
        const int32_t c = cells[i];
        if (c < 0 || c >= B) continue;
        const int32_t r = c / D;
        list[atomicAdd(&hc[r * G + (G == 1 ? 0 : a.slot_shard[c - r * D])], 1)] = i;
    }
}

struct RowArgs {
    const int32_t *q, *list, *hstart;
    int32_t N, L, P, RG, F;
    int32_t lay_piece, n_pieces;  // whole layers per piece, at most 256 entries
    int32_t spread;               // consecutive workgroups take different pieces
    int64_t items;                // layouts * row-shards
    int64_t *Jbuf;                // [n][RG], holds A on entry
    int64_t *wmax, *wsum;         // [n][RG][L] or null
};

constexpr int kEvalWaves = 4;

// Bound by reading q rows (each of the n layouts reads all of q) from
// wherever they are kept: the pieces are laid out so that the slice of q that
// an XCD reads stays in its L2 when it fits, and in the last level cache
// otherwise (row_pieces).  Sum is uint32_t when no sum of q entries passes
// 2^32.
template <bool ONE, typename Sum>
__global__ void __launch_bounds__(kEvalWaves *kWave) k_eval_rows(RowArgs a) {
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const uint32_t per = (uint32_t)((a.items + kEvalWaves - 1) / kEvalWaves);  // workgroups per piece
    const uint32_t b = blockIdx.x, np = (uint32_t)a.n_pieces;
    const int32_t piece = (int32_t)(a.spread ? b % np : b / per);
    const uint32_t it = (a.spread ? b / np : b % per) * kEvalWaves + wv;
    if (it >= (uint32_t)a.items) return;
    const uint32_t lay = it / (uint32_t)a.RG;
    const int32_t h = (int32_t)(it - lay * (uint32_t)a.RG);
    const int32_t *list = a.list + (int64_t)lay * a.N, *hs = a.hstart + (int64_t)lay * (a.RG + 1) + h;
    const int32_t lo = hs[0], n = hs[1] - lo;
    const RowLane<ONE> rl(piece, a.lay_piece, a.L, a.P);
    Sum acc[4] = {0, 0, 0, 0};
    rl.add(a.q, (int64_t)a.L * a.P, a.P, list + lo, n, acc);
    int64_t s4[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) s4[c] = (int64_t)acc[c];
    rl.fold(s4);
    const int64_t mx = rl.layer_max(s4), sm = rl.layer_sum(s4);
    const bool head = rl.head();
    if (a.wmax && head) {
        const int64_t at = (int64_t)it * a.L + rl.layer();
        a.wmax[at] = mx;
        a.wsum[at] = sm;
    }
    const int64_t esum = wave_sum(head ? mx : 0);
    if (lane == 0)
        atomicAdd(reinterpret_cast<unsigned long long *>(a.Jbuf + it), (unsigned long long)esum << a.F);
}

__device__ inline double wave_sum_d(double v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}
__device__ inline double wave_max_d(double v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const double o = __shfl_xor(v, d, kWave);
        v = o > v ? o : v;
    }
    return v;
}

struct FinalArgs {
    int32_t L, P, G, R;
    double scale;
    const int32_t *status;
    const int64_t *Jbuf, *Abuf, *wmax, *wsum;
    const int64_t *rank_load;  // [L][P] or null
    int64_t *scores;           // [n][3]
    int64_t *J;                // [n][RG] or null
    double *diag;              // [n][8] or null
};

__global__ void __launch_bounds__(256) k_eval_finalize(FinalArgs a) {
    __shared__ int64_t ri[3][4];
    __shared__ double rd[4][4];
    const int64_t lay = blockIdx.x;
    const int64_t RG = (int64_t)a.R * a.G;
    const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int64_t *Jl = a.Jbuf + lay * RG;
    const int32_t st = a.status[lay];
    // U_g = sum_r J(r, g): s0 = max_g U, s1 = sum_g U; s2 = max J.
    int64_t umax = LLONG_MIN, usum = 0, jmax = LLONG_MIN;
    for (int g = tid; g < a.G; g += blockDim.x) {
        int64_t U = 0;
        for (int r = 0; r < a.R; ++r) U += Jl[(int64_t)r * a.G + g];
        umax = U > umax ? U : umax;
        usum += U;
    }
    for (int64_t h = tid; h < RG; h += blockDim.x) jmax = Jl[h] > jmax ? Jl[h] : jmax;
    umax = wave_max(umax);
    usum = wave_sum(usum);
    jmax = wave_max(jmax);
    if (lane == 0) {
        ri[0][wv] = umax;
        ri[1][wv] = usum;
        ri[2][wv] = jmax;
    }
    // Diagnostics partials.
    double cv = 0.0, sep = 0.0, tep = 0.0, ideal = 0.0, att = 0.0;
    if (a.diag) {
        if (a.rank_load) {
            for (int l = tid; l < a.L; l += blockDim.x) {
                double mean = 0.0;
                for (int p = 0; p < a.P; ++p) mean += (double)a.rank_load[(int64_t)l * a.P + p];
                mean /= (double)a.P;
                double var = 0.0;
                for (int p = 0; p < a.P; ++p) {
                    const double dv = (double)a.rank_load[(int64_t)l * a.P + p] - mean;
                    var += dv * dv;
                }
                var /= (double)a.P;
                cv += mean > 0.0 ? sqrt(var) / mean : 0.0;
            }
        }
        for (int64_t x = tid; x < (int64_t)a.R * a.L; x += blockDim.x) {
            const int64_t r = x / a.L, l = x % a.L;
            int64_t mx = 0;
            double best_mean = 0.0;
            for (int g = 0; g < a.G; ++g) {
                const int64_t o = ((lay * RG) + r * a.G + g) * a.L + l;
                mx = a.wmax[o] > mx ? a.wmax[o] : mx;
                const double mean = (double)a.wsum[o] / (double)a.P;
                best_mean = mean > best_mean ? mean : best_mean;
            }
            sep += (double)mx;
            tep = (double)mx > tep ? (double)mx : tep;
            ideal += best_mean;
        }
        for (int64_t h = tid; h < RG; h += blockDim.x) att += (double)a.Abuf[lay * RG + h] / a.scale;
        cv = wave_sum_d(cv);
        sep = wave_sum_d(sep);
        tep = wave_max_d(tep);
        ideal = wave_sum_d(ideal);
        att = wave_sum_d(att);
        if (lane == 0) {
            rd[0][wv] = cv;
            rd[1][wv] = sep;
            rd[2][wv] = tep;
            rd[3][wv] = ideal;
        }
        __shared__ double ra[4];
        if (lane == 0) ra[wv] = att;
        __syncthreads();
        if (tid == 0) {
            double s_cv = 0, s_sep = 0, s_tep = 0, s_ideal = 0, s_att = 0;
            for (int w = 0; w < (int)(blockDim.x / kWave); ++w) {
                s_cv += rd[0][w];
                s_sep += rd[1][w];
                s_tep = rd[2][w] > s_tep ? rd[2][w] : s_tep;
                s_ideal += rd[3][w];
                s_att += ra[w];
            }
            int64_t s0 = LLONG_MIN, s1 = 0, s2 = LLONG_MIN;
            for (int w = 0; w < (int)(blockDim.x / kWave); ++w) {
                s0 = ri[0][w] > s0 ? ri[0][w] : s0;
                s1 += ri[1][w];
                s2 = ri[2][w] > s2 ? ri[2][w] : s2;
            }
            double *dg = a.diag + lay * 8;
            if (st) {
                for (int k = 0; k < 8; ++k) dg[k] = __builtin_nan("");
            } else {
                dg[0] = a.rank_load ? (a.L > 0 ? s_cv / (double)a.L : 0.0) : __builtin_nan("");
                dg[1] = s_sep;
                dg[2] = s_tep;
                dg[3] = s_sep > 0.0 ? s_ideal / s_sep : 1.0;
                dg[4] = s_att;
                dg[5] = (double)s0 / a.scale;
                dg[6] = (double)s1 / a.scale;
                dg[7] = energy(s0, s1, s2, a.scale);
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        int64_t s0 = LLONG_MIN, s1 = 0, s2 = LLONG_MIN;
        for (int w = 0; w < (int)(blockDim.x / kWave); ++w) {
            s0 = ri[0][w] > s0 ? ri[0][w] : s0;
            s1 += ri[1][w];
            s2 = ri[2][w] > s2 ? ri[2][w] : s2;
        }
        int64_t *so = a.scores + lay * 3;
        if (st) {
            so[0] = so[1] = so[2] = LLONG_MAX;
        } else {
            so[0] = s0;
            so[1] = s1;
            so[2] = s2;
        }
    }
    if (a.J)
        for (int64_t h = tid; h < RG; h += blockDim.x) a.J[lay * RG + h] = st ? LLONG_MAX : Jl[h];
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Scores `n` layouts already on the device; used by the public entry point
// and by the packing and annealing paths.  status must hold n int32; sum32:
// every layer's total of q is below 2^32 (so is any sum of its entries).
int eval_layouts(const routepack_problem *p, const Topology &topo, const DeviceProblem &dp,
                 const int32_t *t, const int32_t *q, int32_t R, int64_t n, const int32_t *layouts,
                 int64_t *scores, int32_t *status, int64_t *J, double *diag,
                 const int64_t *rank_load, bool sum32, hipStream_t stream) {
    if (n == 0) return ROUTEPACK_OK;
    const int64_t RG = (int64_t)R * topo.G, LP = (int64_t)p->n_layers * p->n_ranks;
    if (LP > 16384) return ROUTEPACK_E_UNSUPPORTED;
    const int64_t B = (int64_t)R * topo.D, L = p->n_layers, P = p->n_ranks, N = p->n_samples;
    // The list path: a power-of-two rank count from 4 to 64 (a layer's ranks
    // on up to 16 adjacent lanes), 16-byte rows and cell statistics that fit
    // LDS next to a second workgroup's.  1024 layouts of 3971 samples (24 x
    // 16, 112 row-shards): 2.3 ms with a scan of the layout per row-shard,
    // 0.62 ms with lists; 16 layouts of 32768 samples (64 x 64, 62): 21.5 ms
    // and 2.1 ms.
    const bool lists = L > 0 && P >= 4 && P <= 64 && (P & (P - 1)) == 0 && ((uintptr_t)q & 15) == 0 &&
                       eval_lists_lds(B, RG) <= 60 * 1024;
    const RowPieces pc = lists ? row_pieces(N, L, P) : RowPieces{};
    // Layouts per pass.  A launch of 2^32 threads and more is cut short
    // without an error, so every kernel's grid stays below 2^24 workgroups of
    // 256; sample lists of at most 64 Mi entries.
    constexpr int64_t kMostWgs = ((int64_t)1 << 24) - 1;
    int64_t nb = n < kMostWgs ? n : kMostWgs;
    if (lists) {
        const int64_t by_list = ((int64_t)64 << 20) / N, by_rows = kMostWgs / pc.n_pieces * kEvalWaves / RG;
        nb = by_list < nb ? by_list : nb;
        nb = by_rows < nb ? by_rows : nb;
        nb = nb < 1 ? 1 : nb;
    }
    Scratch scr(stream);
    int64_t *Jbuf = scr.get<int64_t>(nb * RG);
    int64_t *Abuf = scr.get<int64_t>(nb * RG);
    int64_t *wmax = diag ? scr.get<int64_t>(nb * RG * (L ? L : 1)) : nullptr;
    int64_t *wsum = diag ? scr.get<int64_t>(nb * RG * (L ? L : 1)) : nullptr;
    int32_t *list = lists ? scr.get<int32_t>((size_t)(nb * N)) : nullptr;
    int32_t *hstart = lists ? scr.get<int32_t>((size_t)(nb * (RG + 1))) : nullptr;
    if (scr.failed()) return ROUTEPACK_E_DEVICE;
    for (int64_t l0 = 0; l0 < n; l0 += nb) {
        const int64_t m = nb < n - l0 ? nb : n - l0;
        if (lists) {
            ListArgs la;
            la.t = t; la.layouts = layouts + l0 * N;
            la.N = (int32_t)N; la.D = topo.D; la.G = topo.G; la.R = R; la.S = p->n_stages; la.C = p->capacity;
            la.slots = dp.slots; la.count = dp.count; la.slot_shard = dp.slot_shard;
            la.alpha = dp.alpha; la.beta = dp.beta;
            la.status = status + l0; la.Jbuf = Jbuf; la.Abuf = Abuf; la.list = list; la.hstart = hstart;
            // few layouts: more threads for each
            const int threads = m >= 512 || N <= 1024 ? 256 : 1024;
            hipLaunchKernelGGL(k_eval_lists, dim3((unsigned)m), dim3(threads), eval_lists_lds(B, RG), stream, la);
            RowArgs ra;
            ra.q = q; ra.list = list; ra.hstart = hstart;
            ra.N = (int32_t)N; ra.L = (int32_t)L; ra.P = (int32_t)P; ra.RG = (int32_t)RG; ra.F = p->frac_bits;
            ra.lay_piece = pc.lay_piece;
            ra.n_pieces = pc.n_pieces;
            ra.spread = pc.spread ? 1 : 0;
            ra.items = m * RG;
            ra.Jbuf = Jbuf; ra.wmax = wmax; ra.wsum = wsum;
            const int64_t wgs = (ra.items + kEvalWaves - 1) / kEvalWaves * ra.n_pieces;
            auto rows = pc.one ? (sum32 ? k_eval_rows<true, uint32_t> : k_eval_rows<true, int64_t>)
                               : (sum32 ? k_eval_rows<false, uint32_t> : k_eval_rows<false, int64_t>);
            hipLaunchKernelGGL(rows, dim3((unsigned)wgs), dim3(kEvalWaves * kWave), 0, stream, ra);
        } else {
            hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((m + 255) / 256 < 1024 ? (m + 255) / 256 : 1024)),
                               dim3(256), 0, stream, status + l0, m, 0);
            EvalArgs a;
            a.t = t; a.q = q; a.layouts = layouts + l0 * N;
            a.N = p->n_samples; a.L = p->n_layers; a.P = p->n_ranks; a.D = topo.D; a.G = topo.G; a.R = R;
            a.S = p->n_stages; a.F = p->frac_bits; a.C = p->capacity; a.items = m * RG;
            a.slots = dp.slots; a.count = dp.count; a.slot_shard = dp.slot_shard;
            a.alpha = dp.alpha; a.beta = dp.beta;
            a.status = status + l0; a.Jbuf = Jbuf; a.Abuf = Abuf; a.wmax = wmax; a.wsum = wsum;
            const size_t lds = (size_t)LP * 8 + (size_t)topo.D * 20 + 256 * 4 + 64 + 64;
            if (lds > 160 * 1024) return ROUTEPACK_E_UNSUPPORTED;
            hipLaunchKernelGGL(k_eval_rowshard, grid_of(a.items), dim3(256), lds, stream, a);
        }
        FinalArgs f;
        f.L = p->n_layers; f.P = p->n_ranks; f.G = topo.G; f.R = R;
        f.scale = ldexp((double)p->capacity, p->frac_bits);
        f.status = status + l0; f.Jbuf = Jbuf; f.Abuf = Abuf; f.wmax = wmax; f.wsum = wsum;
        f.rank_load = rank_load; f.scores = scores + l0 * 3; f.J = J ? J + l0 * RG : nullptr;
        f.diag = diag ? diag + l0 * 8 : nullptr;
        hipLaunchKernelGGL(k_eval_finalize, dim3((unsigned)m), dim3(256), 0, stream, f);
        RP_HIP(hipGetLastError());
    }
    return ROUTEPACK_OK;
}

}  // namespace rp

using namespace rp;

extern "C" int routepack_eval_objective(const routepack_problem *prob, const int32_t *lengths,
                                        const int32_t *q, int32_t n_rows, int32_t n_layouts,
                                        const int32_t *layouts, int64_t *scores, int32_t *status,
                                        int64_t *J, double *diag, const int64_t *rank_load,
                                        hipStream_t stream) {
    Topology topo;
    RP_TRY(check_problem(prob, &topo));
    if (n_rows < 1 || n_layouts < 0) return ROUTEPACK_E_INVALID;
    if (!lengths || (!q && prob->n_layers > 0) || !scores || !status || (!layouts && n_layouts > 0))
        return ROUTEPACK_E_INVALID;
    WindowStats ws;
    RP_TRY(window_stats(prob, lengths, q, &ws, stream));
    if (ws.min_t < 1 || ws.q_negative) return ROUTEPACK_E_INVALID;
    RP_TRY(overflow_check(prob, n_rows, ws, false));
    Scratch scr(stream);
    DeviceProblem dp;
    RP_TRY(upload_problem(prob, topo, scr, &dp, stream));
    RP_TRY(eval_layouts(prob, topo, dp, lengths, q, n_rows, n_layouts, layouts, scores, status, J,
                        diag, rank_load, sums_fit32(ws), stream));
    RP_HIP(hipStreamSynchronize(stream));
    return ROUTEPACK_OK;
}
