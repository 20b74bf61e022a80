// Validation, scratch, window bounds and status strings for the RoutePack
// C-ABI library.
#include <atomic>
#include <map>
#include <math.h>
#include <mutex>
#include <string.h>
#include <thread>
#include <utility>

#include "rp_device.h"
#include "rp_internal.h"

namespace rp {

int check_problem(const routepack_problem *p, Topology *topo) {
    if (!p) return ROUTEPACK_E_INVALID;
    if (p->n_samples < 1 || p->n_layers < 0 || p->n_experts < 1 || p->n_ranks < 1)
        return ROUTEPACK_E_INVALID;
    if (p->n_experts % p->n_ranks != 0) return ROUTEPACK_E_INVALID;
    if (p->n_dp < 1 || p->n_edp < 1 || p->n_edp > p->n_dp) return ROUTEPACK_E_INVALID;
    if (p->capacity < 1 || p->n_stages < 1 || p->frac_bits < 0 || p->frac_bits > 30)
        return ROUTEPACK_E_INVALID;
    if (p->min_rows < 1 || !p->dp_to_edp || !p->alpha_fp || !p->beta_fp) return ROUTEPACK_E_INVALID;
    for (int s = 0; s < p->n_stages; ++s)
        if (p->alpha_fp[s] < 0 || p->beta_fp[s] < 0) return ROUTEPACK_E_INVALID;
    Topology t;
    t.D = p->n_dp;
    t.G = p->n_edp;
    t.count.assign(t.G, 0);
    t.slots.assign((size_t)t.G * t.D, 0);
    for (int d = 0; d < t.D; ++d) {
        const int g = p->dp_to_edp[d];
        if (g < 0 || g >= t.G) return ROUTEPACK_E_INVALID;
        t.slots[(size_t)g * t.D + t.count[g]++] = d;
    }
    for (int g = 0; g < t.G; ++g) {
        if (t.count[g] == 0) return ROUTEPACK_E_INVALID;
        if (t.count[g] > t.max_count) t.max_count = t.count[g];
    }
    if (topo) *topo = t;
    return ROUTEPACK_OK;
}

// The device's default stream-ordered pool keeps the memory freed into it
// (release threshold: unlimited), set once per device: otherwise every
// synchronisation hands the pool's memory back and the next call maps it
// again, which costs milliseconds for the annealing state.
static void keep_pool_memory() {
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
    if (done.fetch_or(1ull << dev) & (1ull << dev)) return;
    hipMemPool_t pool = nullptr;
    if (hipDeviceGetDefaultMemPool(&pool, dev) != hipSuccess || !pool) return;
    uint64_t threshold = UINT64_MAX;
    (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &threshold);
}

// One stream's scratch arena: [0, top) is held by the live Scratch objects
// on it (nested calls stack), want is the largest extent a call has needed.
struct Arena {
    char *base = nullptr;
    size_t cap = 0, top = 0, want = 0;
    int depth = 0;
    std::thread::id owner;
};

static std::mutex g_arena_mu;
static std::map<std::pair<int, hipStream_t>, Arena> g_arenas;  // (device, stream); never erased

Scratch::Scratch(hipStream_t s) : stream_(s) {
    keep_pool_memory();
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    std::lock_guard<std::mutex> lock(g_arena_mu);
    Arena &a = g_arenas[std::make_pair(dev, s)];
    if (a.depth > 0 && a.owner != std::this_thread::get_id()) return;  // another thread's call: pool only
    a.owner = std::this_thread::get_id();
    depth_ = ++a.depth;
    start_ = a.top;
    arena_ = &a;
}

Scratch::~Scratch() {
    for (void *q : ptrs_) (void)hipFreeAsync(q, stream_);
    if (!arena_) return;
    std::lock_guard<std::mutex> lock(g_arena_mu);
    Arena &a = *arena_;
    constexpr size_t kGrain = (size_t)2 << 20;
    const size_t peak = (start_ + need_ + kGrain - 1) & ~(kGrain - 1);
    if (peak > a.want) a.want = peak;
    a.top = start_;
    --a.depth;
}

void *Scratch::alloc(size_t n) {
    n = (n + 255) & ~(size_t)255;
    if (arena_) {
        std::lock_guard<std::mutex> lock(g_arena_mu);
        Arena &a = *arena_;
        need_ += n;
        if (depth_ == a.depth) {  // the innermost live Scratch: the top of the arena is its own
            if (depth_ == 1 && a.top == 0 && a.want > a.cap) {
                // grow before the outermost call's first piece; the old arena
                // goes back to the pool in stream order
                if (a.base) (void)hipFreeAsync(a.base, stream_);
                a.base = nullptr;
                a.cap = 0;
                void *q = nullptr;
                if (hipMallocAsync(&q, a.want, stream_) == hipSuccess) {
                    a.base = static_cast<char *>(q);
                    a.cap = a.want;
                }
            }
            if (a.top + n <= a.cap) {
                void *q = a.base + a.top;
                a.top += n;
                return q;
            }
        }
    }
    void *q = nullptr;
    if (hipMallocAsync(&q, n, stream_) != hipSuccess) {
        failed_ = true;
        return nullptr;
    }
    ptrs_.push_back(q);
    return q;
}

// What window_stats reads back, in int64 units.
enum { kStatSum, kStatBig, kStatMax, kStatMin, kStatBound, kStatRate, kStatNeg, kStats };

struct StatArgs {
    const int32_t *t, *q;
    int32_t N, L, P;
    int64_t C;
    int32_t band, lay_wg;  // samples and layers per workgroup
    int64_t *tot;          // [gridDim.y][L] sums of q
    int64_t *part;         // [gridDim.y][gridDim.x][kStats]
};

constexpr int kStatThreads = 256;

// One band of samples and a group of whole layers per workgroup: the sum of
// each layer's q, the largest ceil(max q / t_i), any negative q, and (first
// layer group) the length statistics.  Bound by reading q once: a thread
// keeps the same ranks for every sample of the band and sums in registers
// with eight samples' loads in flight, so only one sum per workgroup and
// layer leaves it (a device atomic per (sample, layer) on L addresses took
// 122 us for 4096 x 24 x 16 and 1.97 ms for 32768 x 64 x 64; now 6 us and
// 0.11 ms).  VEC = 4 takes 16-byte loads (P % 4 == 0, q aligned).
template <int VEC>
__global__ void __launch_bounds__(kStatThreads) k_window_bands(StatArgs a) {
    extern __shared__ __align__(16) unsigned long long stot[];  // [lay_wg]
    __shared__ long long sred[4][kStats];
    const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int32_t r0 = (int32_t)blockIdx.y * a.band, r1 = r0 + a.band < a.N ? r0 + a.band : a.N;
    const int32_t l0 = (int32_t)blockIdx.x * a.lay_wg, nl = a.lay_wg < a.L - l0 ? a.lay_wg : a.L - l0;
    int64_t v[kStats] = {0, 0, LLONG_MIN, LLONG_MAX, 0, 0, 0};
    if (blockIdx.x == 0)
        for (int32_t i = r0 + tid; i < r1; i += kStatThreads) {
            const int64_t x = a.t[i];
            v[kStatSum] += x;
            v[kStatBig] += 2 * x > a.C ? 1 : 0;
            v[kStatMax] = x > v[kStatMax] ? x : v[kStatMax];
            v[kStatMin] = x < v[kStatMin] ? x : v[kStatMin];
        }
    if (nl > 0) {
        for (int32_t l = tid; l < nl; l += kStatThreads) stot[l] = 0;
        __syncthreads();
        const int32_t pv = a.P / VEC, cols = nl * pv;
        const int64_t stride = (int64_t)a.L * a.P;
        const int32_t ng = cols < kStatThreads ? kStatThreads / cols : 1;
        const int32_t grp = cols < kStatThreads ? tid / cols : 0;
        int64_t rate = 0;
        int32_t any = 0;
        if (grp < ng)
            for (int32_t c = tid - grp * cols; c < cols; c += kStatThreads) {
                const int32_t *src = a.q + (int64_t)l0 * a.P + (int64_t)c * VEC;
                int64_t sum = 0;
                constexpr int U = 8;
                for (int32_t i = r0 + grp; i < r1; i += U * ng) {
                    int32_t x[U][VEC], ti[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int32_t k = i + u * ng < r1 ? i + u * ng : r1 - 1;
                        ti[u] = a.t[k];
                        if (VEC == 4) {
                            const int4 w = *reinterpret_cast<const int4 *>(src + k * stride);
                            x[u][0] = w.x;
                            x[u][1 % VEC] = w.y;
                            x[u][2 % VEC] = w.z;
                            x[u][3 % VEC] = w.w;
                        } else {
                            x[u][0] = src[k * stride];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        int32_t mx = 0;
                        int64_t s = 0;
#pragma unroll
                        for (int e = 0; e < VEC; ++e) {
                            any |= x[u][e];
                            mx = x[u][e] > mx ? x[u][e] : mx;
                            s += x[u][e];
                        }
                        sum += i + u * ng < r1 ? s : 0;
                        // (a repeated last sample changes neither maximum nor sign)
                        if (ti[u] <= 0) rate = mx > rate ? mx : rate;
                        else if (mx > rate * ti[u]) rate = ((int64_t)mx + ti[u] - 1) / ti[u];
                    }
                }
                atomicAdd(&stot[c / pv], (unsigned long long)sum);
            }
        v[kStatRate] = rate;
        v[kStatNeg] = any < 0 ? 1 : 0;
        __syncthreads();
        for (int32_t l = tid; l < nl; l += kStatThreads)
            a.tot[(int64_t)blockIdx.y * a.L + l0 + l] = (int64_t)stot[l];
    }
    v[kStatSum] = wave_sum(v[kStatSum]);
    v[kStatBig] = wave_sum(v[kStatBig]);
    v[kStatMax] = wave_max(v[kStatMax]);
    v[kStatMin] = wave_min(v[kStatMin]);
    v[kStatRate] = wave_max(v[kStatRate]);
    v[kStatNeg] = wave_max(v[kStatNeg]);
    if (lane == 0)
        for (int k = 0; k < kStats; ++k) sred[wv][k] = v[k];
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kStatThreads / kWave; ++w) {
            v[kStatSum] += sred[w][kStatSum];
            v[kStatBig] += sred[w][kStatBig];
            v[kStatMax] = sred[w][kStatMax] > v[kStatMax] ? sred[w][kStatMax] : v[kStatMax];
            v[kStatMin] = sred[w][kStatMin] < v[kStatMin] ? sred[w][kStatMin] : v[kStatMin];
            v[kStatRate] = sred[w][kStatRate] > v[kStatRate] ? sred[w][kStatRate] : v[kStatRate];
            v[kStatNeg] |= sred[w][kStatNeg];
        }
        int64_t *out = a.part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kStats;
        for (int k = 0; k < kStats; ++k) out[k] = v[k];
    }
}

// The bands' sums and statistics into one record (one workgroup).
__global__ void __launch_bounds__(1024) k_window_finish(const int64_t *tot, const int64_t *part, int32_t bands,
                                                        int32_t parts, int32_t L, int64_t *out) {
    __shared__ long long sred[16][kStats];
    const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    int64_t v[kStats] = {0, 0, LLONG_MIN, LLONG_MAX, 0, 0, 0};
    for (int32_t x = tid; x < parts; x += 1024) {
        const int64_t *p = part + (int64_t)x * kStats;
        v[kStatSum] += p[kStatSum];
        v[kStatBig] += p[kStatBig];
        v[kStatMax] = p[kStatMax] > v[kStatMax] ? p[kStatMax] : v[kStatMax];
        v[kStatMin] = p[kStatMin] < v[kStatMin] ? p[kStatMin] : v[kStatMin];
        v[kStatRate] = p[kStatRate] > v[kStatRate] ? p[kStatRate] : v[kStatRate];
        v[kStatNeg] |= p[kStatNeg];
    }
    // a wave per layer, lanes over the bands
    for (int32_t l = wv; l < L; l += 16) {
        int64_t s = 0;
        for (int32_t b = lane; b < bands; b += kWave) s += tot[(int64_t)b * L + l];
        s = wave_sum(s);
        v[kStatBound] = s > v[kStatBound] ? s : v[kStatBound];
    }
    v[kStatSum] = wave_sum(v[kStatSum]);
    v[kStatBig] = wave_sum(v[kStatBig]);
    v[kStatMax] = wave_max(v[kStatMax]);
    v[kStatMin] = wave_min(v[kStatMin]);
    v[kStatRate] = wave_max(v[kStatRate]);
    v[kStatNeg] = wave_max(v[kStatNeg]);
    if (lane == 0)
        for (int k = 0; k < kStats; ++k) sred[wv][k] = v[k];
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 16; ++w) {
            v[kStatSum] += sred[w][kStatSum];
            v[kStatBig] += sred[w][kStatBig];
            v[kStatMax] = sred[w][kStatMax] > v[kStatMax] ? sred[w][kStatMax] : v[kStatMax];
            v[kStatMin] = sred[w][kStatMin] < v[kStatMin] ? sred[w][kStatMin] : v[kStatMin];
            v[kStatBound] = sred[w][kStatBound] > v[kStatBound] ? sred[w][kStatBound] : v[kStatBound];
            v[kStatRate] = sred[w][kStatRate] > v[kStatRate] ? sred[w][kStatRate] : v[kStatRate];
            v[kStatNeg] |= sred[w][kStatNeg];
        }
        for (int k = 0; k < kStats; ++k) out[k] = v[k];
    }
}

int window_stats(const routepack_problem *p, const int32_t *lengths, const int32_t *q,
                 WindowStats *out, hipStream_t stream) {
    const int32_t L = q ? p->n_layers : 0, P = p->n_ranks, N = p->n_samples;
    StatArgs a;
    a.t = lengths; a.q = q; a.N = N; a.L = L; a.P = P; a.C = p->capacity;
    const bool vec = P % 4 == 0 && ((uintptr_t)q & 15) == 0;
    // whole layers per workgroup, about one 16-byte word per thread
    const int32_t most = 4 * kStatThreads / P;  // (at most 8 KiB of sums)
    a.lay_wg = L == 0 ? 1 : (most < 1 ? 1 : (most < L ? most : L));
    const int32_t gx = L == 0 ? 1 : (L + a.lay_wg - 1) / a.lay_wg;
    // bands of at least 16 samples, about 2048 workgroups (8 per CU)
    int32_t gy = 2048 / gx;
    gy = gy < 1 ? 1 : (gy > 512 ? 512 : gy);
    if (gy > (N + 15) / 16) gy = (N + 15) / 16;
    a.band = (N + gy - 1) / gy;
    gy = (N + a.band - 1) / a.band;
    Scratch scr(stream);
    a.tot = scr.get<int64_t>((size_t)gy * (L ? L : 1));
    a.part = scr.get<int64_t>((size_t)gy * gx * kStats);
    int64_t *rec = scr.get<int64_t>(kStats);
    if (scr.failed()) return ROUTEPACK_E_DEVICE;
    auto bands = vec ? k_window_bands<4> : k_window_bands<1>;
    hipLaunchKernelGGL(bands, dim3((unsigned)gx, (unsigned)gy), dim3(kStatThreads), (size_t)8 * a.lay_wg, stream, a);
    hipLaunchKernelGGL(k_window_finish, dim3(1), dim3(1024), 0, stream, a.tot, a.part, gy, gx * gy, L, rec);
    RP_HIP(hipGetLastError());
    int64_t h[kStats];
    RP_HIP(hipMemcpyAsync(h, rec, sizeof(h), hipMemcpyDeviceToHost, stream));
    RP_HIP(hipStreamSynchronize(stream));
    out->sum_t = h[kStatSum];
    out->n_big = h[kStatBig];
    out->max_t = h[kStatMax];
    out->min_t = h[kStatMin];
    out->w_bound = h[kStatBound];
    out->q_negative = h[kStatNeg] != 0;
    out->q_rate = h[kStatRate];
    return ROUTEPACK_OK;
}

int64_t w_entry_bound(const routepack_problem *p, const WindowStats &ws) {
    // A row-shard holds at most maxD * C tokens and q[i][l][p] <= rate * t_i.
    int32_t maxd = 0;
    {
        std::vector<int32_t> cnt(p->n_edp, 0);
        for (int d = 0; d < p->n_dp; ++d) cnt[p->dp_to_edp[d]]++;
        for (int g = 0; g < p->n_edp; ++g) maxd = cnt[g] > maxd ? cnt[g] : maxd;
    }
    const long double wcap = (long double)ws.q_rate * (long double)maxd * (long double)p->capacity;
    return wcap < (long double)ws.w_bound ? (int64_t)wcap : ws.w_bound;
}

int overflow_check(const routepack_problem *p, int64_t n_rows, const WindowStats &ws,
                   bool w_as_int32) {
    const long double lim = 9007199254740992.0L;  // 2^53
    const long double C = (long double)p->capacity;
    const int64_t wb = w_entry_bound(p, ws);
    long double a_max = 0.0L;
    for (int s = 0; s < p->n_stages; ++s)
        a_max += (long double)p->alpha_fp[s] * C + (long double)p->beta_fp[s] * C * C;
    const long double e_max = ldexpl((long double)p->n_layers * (long double)wb, p->frac_bits);
    const long double total = (long double)n_rows * (long double)p->n_edp * (a_max + e_max + 1.0L);
    if (!(total < lim)) return ROUTEPACK_E_OVERFLOW;
    if (!(ldexpl(C, p->frac_bits) < lim)) return ROUTEPACK_E_OVERFLOW;
    if (w_as_int32 && wb > 2147483647LL) return ROUTEPACK_E_OVERFLOW;
    return ROUTEPACK_OK;
}

int upload_problem(const routepack_problem *p, const Topology &topo, Scratch &scr,
                   DeviceProblem *dp, hipStream_t stream) {
    const size_t D = topo.D, G = topo.G, S = p->n_stages;
    // one record, one copy: alpha, beta, slots, count, slot_shard
    const size_t n = 16 * S + 4 * (G * D + G + D);
    char *dev = scr.get<char>(n);
    if (scr.failed()) return ROUTEPACK_E_DEVICE;
    dp->host.resize(n);
    size_t at = 0;
    auto put = [&](const void *src, size_t bytes) {
        memcpy(dp->host.data() + at, src, bytes);
        at += bytes;
        return dev + at - bytes;
    };
    dp->alpha = reinterpret_cast<int64_t *>(put(p->alpha_fp, 8 * S));
    dp->beta = reinterpret_cast<int64_t *>(put(p->beta_fp, 8 * S));
    dp->slots = reinterpret_cast<int32_t *>(put(topo.slots.data(), 4 * G * D));
    dp->count = reinterpret_cast<int32_t *>(put(topo.count.data(), 4 * G));
    dp->slot_shard = reinterpret_cast<int32_t *>(put(p->dp_to_edp, 4 * D));
    RP_HIP(hipMemcpyAsync(dev, dp->host.data(), n, hipMemcpyHostToDevice, stream));
    return ROUTEPACK_OK;
}

}  // namespace rp

extern "C" const char *routepack_strerror(int code) {
    switch (code) {
        case ROUTEPACK_OK: return "ok";
        case ROUTEPACK_E_INVALID: return "invalid argument";
        case ROUTEPACK_E_INFEASIBLE: return "infeasible window (t_i > C or too few samples for the row bound)";
        case ROUTEPACK_E_HEURISTIC: return "FixedRowFFD found no feasible row count";
        case ROUTEPACK_E_LAYOUT: return "layout violates coverage, capacity or non-empty cells";
        case ROUTEPACK_E_OVERFLOW: return "fixed-point score bound exceeds 2^53";
        case ROUTEPACK_E_DEVICE: return "HIP runtime error";
        case ROUTEPACK_E_INTERNAL: return "postcondition failed";
        case ROUTEPACK_E_UNSUPPORTED: return "size not supported by these kernels";
        default: return "unknown status";
    }
}
