// Exact T(lambda) screening (Pseudocode section): T = Mean + lambda (Max - Mean)
// over the generation's M objective values, pass iff f > T, decided in 128-bit
// integers as  den*M*f > (den - num)*Sum + num*M*Max  (lambda = num/den).
// Passer indices are compacted in ascending order.
//
// Three HBM-bound passes over f (8 B/candidate each): block partial Sum/Max,
// per-block passer counts, and an order-preserving scatter.  No atomics, so the
// output is the same on every run.
#include <mutex>

#include "ubqp_internal.h"

namespace {

constexpr int THR = 256;
constexpr int PER = 8;
constexpr int64_t CH = THR * PER;  // candidates per block

__device__ inline int64_t wave_sum(int64_t v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ inline int64_t wave_max(int64_t v)
{
    for (int o = 32; o > 0; o >>= 1) {
        int64_t u = __shfl_xor(v, o);
        v = u > v ? u : v;
    }
    return v;
}

// Block-wide sum and max; every thread gets the result.
__device__ void block_sum_max(int64_t &s, int64_t &m)
{
    __shared__ int64_t ss[THR / 64], sm[THR / 64];
    s = wave_sum(s);
    m = wave_max(m);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { ss[wv] = s; sm[wv] = m; }
    __syncthreads();
    s = ss[0];
    m = sm[0];
    for (int i = 1; i < THR / 64; i++) { s += ss[i]; m = sm[i] > m ? sm[i] : m; }
    __syncthreads();
}

__device__ inline bool passes(int64_t f, int64_t M, int32_t den, __int128 rhs) { return (__int128)den * M * f > rhs; }

__device__ void reduce_body(const ScreenArgs &a, int64_t bid)
{
    const int64_t base = bid * CH;
    int64_t s = 0, m = INT64_MIN;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int64_t c = base + i * THR + threadIdx.x;
        if (c < a.M) { const int64_t v = a.f[c]; s += v; m = v > m ? v : m; }
    }
    block_sum_max(s, m);
    if (threadIdx.x == 0) { a.psum[bid] = s; a.pmax[bid] = m; }
}

// Sum and Max of the whole population from the block partials.
__device__ void total_sum_max(const ScreenArgs &a, int64_t &s, int64_t &m)
{
    s = 0;
    m = INT64_MIN;
    for (int b = threadIdx.x; b < a.nblk; b += THR) { s += a.psum[b]; m = a.pmax[b] > m ? a.pmax[b] : m; }
    block_sum_max(s, m);
}

__device__ void count_body(const ScreenArgs &a, int64_t bid)
{
    int64_t S, Mx;
    total_sum_max(a, S, Mx);
    const __int128 rhs = (__int128)(a.lam_den - a.lam_num) * S + (__int128)a.lam_num * a.M * Mx;
    const int64_t base = bid * CH;
    int64_t k = 0;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int64_t c = base + i * THR + threadIdx.x;
        if (c < a.M && passes(a.f[c], a.M, a.lam_den, rhs)) k++;
    }
    int64_t dummy = 0;
    block_sum_max(k, dummy);
    if (threadIdx.x == 0) {
        a.cnt[bid] = k;
        if (bid == 0) { a.sum_max[0] = S; a.sum_max[1] = Mx; }
    }
}

__device__ void scatter_body(const ScreenArgs &a, int64_t bid)
{
    __shared__ int64_t wtot[THR / 64];
    // passers in earlier blocks
    int64_t off = 0, dummy = 0;
    for (int b = threadIdx.x; b < (int)bid; b += THR) off += a.cnt[b];
    block_sum_max(off, dummy);
    const __int128 rhs = (__int128)(a.lam_den - a.lam_num) * a.sum_max[0] + (__int128)a.lam_num * a.M * a.sum_max[1];
    // each thread owns PER consecutive candidates, so thread order is index order
    const int64_t c0 = bid * CH + (int64_t)threadIdx.x * PER;
    uint32_t bits = 0;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int64_t c = c0 + i;
        if (c < a.M && passes(a.f[c], a.M, a.lam_den, rhs)) bits |= 1u << i;
    }
    const int mine = __popc(bits);
    // exclusive scan of `mine` over the block
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wtot[wv] = incl;
    __syncthreads();
    int64_t pos = off + incl - mine;
    for (int i = 0; i < wv; i++) pos += wtot[i];
    for (int i = 0; i < PER; i++)
        if (bits & (1u << i)) a.idx[pos++] = (int32_t)(c0 + i);
    if (bid == a.nblk - 1 && threadIdx.x == THR - 1) *a.npass = pos;
}

__global__ __launch_bounds__(THR) void screen_reduce(ScreenArgs a) { reduce_body(a, blockIdx.x); }
__global__ __launch_bounds__(THR) void screen_count(ScreenArgs a) { count_body(a, blockIdx.x); }
__global__ __launch_bounds__(THR) void screen_scatter(ScreenArgs a) { scatter_body(a, blockIdx.x); }

__global__ __launch_bounds__(THR) void screen_reduce_b(const ScreenArgs *args, const int64_t *prefix, int count)
{
    const int i = ubqp_find_inst(prefix, count, blockIdx.x);
    const ScreenArgs a = args[i];
    reduce_body(a, blockIdx.x - prefix[i]);
}
__global__ __launch_bounds__(THR) void screen_count_b(const ScreenArgs *args, const int64_t *prefix, int count)
{
    const int i = ubqp_find_inst(prefix, count, blockIdx.x);
    const ScreenArgs a = args[i];
    count_body(a, blockIdx.x - prefix[i]);
}
__global__ __launch_bounds__(THR) void screen_scatter_b(const ScreenArgs *args, const int64_t *prefix, int count)
{
    const int i = ubqp_find_inst(prefix, count, blockIdx.x);
    const ScreenArgs a = args[i];
    scatter_body(a, blockIdx.x - prefix[i]);
}

// Ascent order of the passers: lowest objective first, in power-of-two-wide
// buckets of the objective range, so that the candidates furthest below a local
// optimum (the longest flip chains) are taken first and short chains fill in
// behind them.  Only the order in which the ascent's waves take candidates
// changes; every candidate's result is the same in any order.
constexpr int ORD_THR = 1024, ORD_WAVES = ORD_THR / 64;
constexpr int ORD_BUCKETS = 1024;
constexpr int ORD_PER = 16;  // objectives a thread holds in registers
static_assert(ORD_THR == ORD_BUCKETS, "one bucket per thread: zeroing and the scan assume it");
static_assert(ORD_THR * ORD_PER == UBQP_SCREEN_BLOCK_MAX_M, "the one-block screen's largest population");

struct OrderLds {
    int32_t start[ORD_BUCKETS];
    int64_t lo[ORD_WAVES], hi[ORD_WAVES];
    int32_t wsum[ORD_WAVES];
};

// Smallest and largest v over the block (start[] cleared on the way).
__device__ void order_range(OrderLds &l, int64_t &lo, int64_t &hi)
{
    for (int o = 32; o > 0; o >>= 1) {
        const int64_t l2 = __shfl_xor(lo, o), h2 = __shfl_xor(hi, o);
        lo = l2 < lo ? l2 : lo;
        hi = h2 > hi ? h2 : hi;
    }
    if ((threadIdx.x & 63) == 0) { l.lo[threadIdx.x >> 6] = lo; l.hi[threadIdx.x >> 6] = hi; }
    l.start[threadIdx.x] = 0;  // ORD_THR == ORD_BUCKETS
    __syncthreads();
    for (int i = 0; i < ORD_WAVES; i++) {
        lo = l.lo[i] < lo ? l.lo[i] : lo;
        hi = l.hi[i] > hi ? l.hi[i] : hi;
    }
}

// bucket = (v - lo) >> shift, with (hi - lo) >> shift < ORD_BUCKETS
__device__ inline int order_shift(int64_t lo, int64_t hi)
{
    const uint64_t span = (uint64_t)(hi - lo);
    const int bits = 64 - __clzll((long long)span);  // 64 - 64 when the span is 0
    return bits > 10 ? bits - 10 : 0;
}
static_assert(ORD_BUCKETS == 1 << 10, "order_shift");

// Bucket counts -> first position of each bucket (one bucket per thread).
__device__ void order_scan(OrderLds &l)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    const int cnt = l.start[threadIdx.x];
    int incl = cnt;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    if (lane == 63) l.wsum[wv] = incl;
    __syncthreads();
    int before = 0;
    for (int i = 0; i < wv; i++) before += l.wsum[i];
    l.start[threadIdx.x] = before + incl - cnt;
    __syncthreads();
}

// One block per instance, after the multi-block screen (more than
// UBQP_SCREEN_BLOCK_MAX_M candidates).  Each pass over the passers is a gather of
// their objectives, bound by its latency: up to 16 x 1024 passers are gathered once,
// 16 independent loads per thread, and kept in registers for the three passes.
__global__ __launch_bounds__(ORD_THR) void order_batched(const OrdArgs *args, int count)
{
    __shared__ OrderLds l;
    if ((int)blockIdx.x >= count) return;
    const OrdArgs a = args[blockIdx.x];
    const int64_t P = *a.npass;
    if (P <= 0) return;
    int64_t lo = INT64_MAX, hi = INT64_MIN;
    if (P <= ORD_THR * ORD_PER) {
        int32_t c[ORD_PER];
        int64_t v[ORD_PER];
#pragma unroll
        for (int i = 0; i < ORD_PER; i++) {
            const int p = i * ORD_THR + threadIdx.x;
            c[i] = p < P ? a.idx[p] : 0;
        }
#pragma unroll
        for (int i = 0; i < ORD_PER; i++) {
            const int p = i * ORD_THR + threadIdx.x;
            v[i] = p < P ? a.f[c[i]] : 0;
        }
#pragma unroll
        for (int i = 0; i < ORD_PER; i++) {
            const int p = i * ORD_THR + threadIdx.x;
            if (p < P) {
                lo = v[i] < lo ? v[i] : lo;
                hi = v[i] > hi ? v[i] : hi;
                a.rank[p] = 0;
            }
        }
        order_range(l, lo, hi);
        const int shift = order_shift(lo, hi);
#pragma unroll
        for (int i = 0; i < ORD_PER; i++)
            if (i * ORD_THR + (int)threadIdx.x < P) atomicAdd(&l.start[(int)((uint64_t)(v[i] - lo) >> shift)], 1);
        order_scan(l);
#pragma unroll
        for (int i = 0; i < ORD_PER; i++)
            if (i * ORD_THR + (int)threadIdx.x < P)
                a.oidx[atomicAdd(&l.start[(int)((uint64_t)(v[i] - lo) >> shift)], 1)] = c[i];
        return;
    }
    for (int64_t p = threadIdx.x; p < P; p += ORD_THR) {
        const int64_t v = a.f[a.idx[p]];
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
        a.rank[p] = 0;
    }
    order_range(l, lo, hi);
    const int shift = order_shift(lo, hi);
    for (int64_t p = threadIdx.x; p < P; p += ORD_THR)
        atomicAdd(&l.start[(int)((uint64_t)(a.f[a.idx[p]] - lo) >> shift)], 1);
    order_scan(l);
    for (int64_t p = threadIdx.x; p < P; p += ORD_THR) {
        const int32_t c = a.idx[p];
        a.oidx[atomicAdd(&l.start[(int)((uint64_t)(a.f[c] - lo) >> shift)], 1)] = c;
    }
}

// Screening, ascent order and the clearing of the ranks by one block per instance
// (at most UBQP_SCREEN_BLOCK_MAX_M candidates).  At these sizes the three screening
// launches and the order launch are bound by launch and load latency, not by the
// 8 B per candidate they read: here f is read once into registers (PER objectives
// per thread, candidate 1024 i + thread) and every later pass works on chip.
// The passers' ascending positions come from one ballot per wave and i, scanned over
// the (i, wave) pairs in LDS.
template <int PER> __device__ void screen_order_body(const ScrOrdArgs &a)
{
    __shared__ OrderLds l;
    __shared__ int64_t ws[ORD_WAVES], wm[ORD_WAVES];
    __shared__ int32_t cnt[ORD_WAVES * PER];
    __shared__ int32_t total;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int M = (int)a.s.M;
    int64_t v[PER];
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int c = i * ORD_THR + threadIdx.x;
        v[i] = c < M ? a.s.f[c] : 0;
    }
    int64_t sum = 0, mx = INT64_MIN;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int c = i * ORD_THR + threadIdx.x;
        if (c < M) { sum += v[i]; mx = v[i] > mx ? v[i] : mx; }
    }
    sum = wave_sum(sum);
    mx = wave_max(mx);
    if (lane == 0) { ws[wv] = sum; wm[wv] = mx; }
    __syncthreads();
    sum = ws[0];
    mx = wm[0];
    for (int i = 1; i < ORD_WAVES; i++) { sum += ws[i]; mx = wm[i] > mx ? wm[i] : mx; }
    const __int128 rhs = (__int128)(a.s.lam_den - a.s.lam_num) * sum + (__int128)a.s.lam_num * M * mx;
    uint64_t ball[PER];
    int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int c = i * ORD_THR + threadIdx.x;
        const bool ok = c < M && passes(v[i], M, a.s.lam_den, rhs);
        ball[i] = __ballot(ok);
        if (lane == 0) cnt[i * ORD_WAVES + wv] = __popcll(ball[i]);
        if (ok) {
            lo = v[i] < lo ? v[i] : lo;
            hi = v[i] > hi ? v[i] : hi;
        }
    }
    order_range(l, lo, hi);  // its barrier also covers cnt
    if (wv == 0) {
        // exclusive scan of the 16 PER counts: lane k takes PER / 4 (or one) of them
        constexpr int N = ORD_WAVES * PER, Q = N > 64 ? N / 64 : 1;
        int own[Q], s = 0;
#pragma unroll
        for (int k = 0; k < Q; k++) {
            const int j = lane * Q + k;
            own[k] = j < N ? cnt[j] : 0;
            s += own[k];
        }
        int incl = s;
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        int run = incl - s;
#pragma unroll
        for (int k = 0; k < Q; k++) {
            const int j = lane * Q + k;
            if (j < N) cnt[j] = run;
            run += own[k];
        }
        if (lane == 63) {
            total = incl;
            *a.s.npass = incl;
            a.s.sum_max[0] = sum;
            a.s.sum_max[1] = mx;
        }
    }
    __syncthreads();
    if (total == 0) return;
    const int shift = order_shift(lo, hi);
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        if ((ball[i] >> lane) & 1ull) {
            const int pos = cnt[i * ORD_WAVES + wv] + __popcll(ball[i] & below);
            a.s.idx[pos] = i * ORD_THR + threadIdx.x;
            a.rank[pos] = 0;
            atomicAdd(&l.start[(int)((uint64_t)(v[i] - lo) >> shift)], 1);
        }
    }
    order_scan(l);
#pragma unroll
    for (int i = 0; i < PER; i++)
        if ((ball[i] >> lane) & 1ull)
            a.oidx[atomicAdd(&l.start[(int)((uint64_t)(v[i] - lo) >> shift)], 1)] = i * ORD_THR + threadIdx.x;
}

__global__ __launch_bounds__(ORD_THR) void screen_order_b(const ScrOrdArgs *args, int count)
{
    if ((int)blockIdx.x >= count) return;
    const ScrOrdArgs a = args[blockIdx.x];
    if (a.s.M <= ORD_THR) screen_order_body<1>(a);
    else if (a.s.M <= 4 * ORD_THR) screen_order_body<4>(a);
    else screen_order_body<ORD_PER>(a);
}

}  // namespace

hipError_t ubqp_launch_order_batch(hipStream_t st, const OrdArgs *args, int count)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(order_batched, dim3((unsigned)count), dim3(ORD_THR), 0, st, args, count);
    return hipGetLastError();
}

hipError_t ubqp_launch_screen_order_batch(hipStream_t st, const ScrOrdArgs *args, int count)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(screen_order_b, dim3((unsigned)count), dim3(ORD_THR), 0, st, args, count);
    return hipGetLastError();
}

int32_t ubqp_screen_blocks(int64_t M) { return (int32_t)((M + CH - 1) / CH); }
size_t ubqp_screen_partials_bytes(int64_t M) { return (size_t)ubqp_screen_blocks(M) * 3 * sizeof(int64_t); }

ScreenArgs ubqp_screen_args(const int64_t *f, int64_t M, int32_t lam_num, int32_t lam_den, int32_t *idx,
                            int64_t *npass, int64_t *sum_max, void *partials)
{
    ScreenArgs a{};
    a.f = f;
    a.M = M;
    a.lam_num = lam_num;
    a.lam_den = lam_den;
    a.idx = idx;
    a.npass = npass;
    a.sum_max = sum_max;
    a.nblk = ubqp_screen_blocks(M);
    a.psum = (int64_t *)partials;
    a.pmax = a.psum + a.nblk;
    a.cnt = a.pmax + a.nblk;
    return a;
}

hipError_t ubqp_launch_screen(hipStream_t st, const ScreenArgs &a)
{
    hipLaunchKernelGGL(screen_reduce, dim3(a.nblk), dim3(THR), 0, st, a);
    hipLaunchKernelGGL(screen_count, dim3(a.nblk), dim3(THR), 0, st, a);
    hipLaunchKernelGGL(screen_scatter, dim3(a.nblk), dim3(THR), 0, st, a);
    return hipGetLastError();
}

hipError_t ubqp_launch_screen_batch(hipStream_t st, const ScreenArgs *args, const int64_t *prefix, int count,
                                    int64_t blocks)
{
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(screen_reduce_b, dim3((unsigned)blocks), dim3(THR), 0, st, args, prefix, count);
    hipLaunchKernelGGL(screen_count_b, dim3((unsigned)blocks), dim3(THR), 0, st, args, prefix, count);
    hipLaunchKernelGGL(screen_scatter_b, dim3((unsigned)blocks), dim3(THR), 0, st, args, prefix, count);
    return hipGetLastError();
}

// ---- screening without allocation ----------------------------------------------
// The block partials of ubqp_screen_noalloc live in one file-scope device array per
// GPU.  Host code never passes the array's name to a kernel (on the host it is only
// a stand-in): the device address of each GPU's copy is looked up once, with that
// GPU current, when the first context on it is created, and kept per device.
static constexpr int64_t STATIC_BLOCKS = (UBQP_SCREEN_NOALLOC_MAX_M + CH - 1) / CH;
static __device__ __align__(256) int64_t scratch[3 * STATIC_BLOCKS];  // psum, pmax, cnt: 48 KiB

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
void *scratch_ptr[MAX_DEVICES] = {};

}  // namespace

int ubqp_screen_scratch_init(ubqp_ctx *ctx)
{
    if (ctx->device < 0 || ctx->device >= MAX_DEVICES)
        return ubqp_fail(ctx, UBQP_EDEVICE, "device %d beyond the %d the static screen scratch tracks", ctx->device,
                         MAX_DEVICES);
    std::lock_guard<std::mutex> lk(scratch_mu);
    if (scratch_ptr[ctx->device]) return UBQP_OK;
    void *ptr = nullptr;
    UBQP_HIP_TRY(ctx, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return ubqp_fail(ctx, UBQP_EDEVICE, "hipGetSymbolAddress returned a null address for the screen scratch");
    scratch_ptr[ctx->device] = ptr;
    return UBQP_OK;
}

extern "C" int ubqp_screen_noalloc(ubqp_ctx *ctx, const int64_t *f_d, int64_t M, int32_t lam_num, int32_t lam_den,
                                   int32_t *pass_idx_d, int64_t *n_pass_d, int64_t *sum_max_d)
{
    if (!ctx || !f_d || !pass_idx_d || !n_pass_d || !sum_max_d) return ubqp_fail(ctx, UBQP_EINVAL, "null argument");
    if (M < 1 || M > UBQP_SCREEN_NOALLOC_MAX_M)
        return ubqp_fail(ctx, UBQP_EINVAL, "M=%lld outside [1, %lld], the size of the static screen scratch",
                         (long long)M, (long long)UBQP_SCREEN_NOALLOC_MAX_M);
    if (lam_den < 1 || lam_num < 0 || lam_num > lam_den)
        return ubqp_fail(ctx, UBQP_EINVAL, "lambda=%d/%d outside [0, 1]", lam_num, lam_den);
    UBQP_TRY(ubqp_set_device(ctx));
    void *part = nullptr;
    {
        std::lock_guard<std::mutex> lk(scratch_mu);
        if (ctx->device >= 0 && ctx->device < MAX_DEVICES) part = scratch_ptr[ctx->device];
    }
    if (!part) return ubqp_fail(ctx, UBQP_EDEVICE, "the static screen scratch of device %d was not set up", ctx->device);
    // every partial is written (reduce: psum, pmax; count: cnt) before it is read
    UBQP_HIP_TRY(ctx, ubqp_launch_screen(ctx->stream, ubqp_screen_args(f_d, M, lam_num, lam_den, pass_idx_d, n_pass_d,
                                                                       sum_max_d, part)));
    return UBQP_OK;
}
