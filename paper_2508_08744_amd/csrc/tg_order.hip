// An order of the nodes in which neighbours come together: the joins from the fourth round on, the rounds of phase 2 and finalize
// take the nodes in it, so that the rows they gather at one time are few and stay in an XCD's L2 (those steps wait for rows that
// come from everywhere).  Nothing but the order of independent work depends on it, so the graph is the same.
// A node's label is the smallest node number it can reach in a few steps over the first entries of the lists (a step takes the smallest label of
// the node and of its closest neighbours, and the label's own label): nodes of one dense region share it.  The nodes are
// then brought together by a hash of their label, in buckets of about a thousand.
// 10M x 96 (cosine, 4 + 1 rounds): 5 ms for the order; fourth round's joins 58.9 -> 53.5 ms, phase 2 40.5 -> 29.5, finalize 24.8 -> 13.4, the build
// 526 -> 506.  200 000 x 960 (4 + 4): 0.07 ms; a phase-2 round 2.55 -> 1.66, finalize 3.6 -> 1.5, the build 61.3 -> 55.7.  With ids sorted by the clusters
// the points were drawn from, which is as good as an order gets: phase 2 and finalize 23 and 11 ms, 1.45 and 1.3.
// Measured choices (10M x 96: phase 2 / finalize): three steps over 4 entries 32.6 / 15.6, four over 4 31.1 / 14.2, six over 4 30.1 / 13.2 (200 000 x 960: 1.6 / 1.43),
// three over 8 31.0 / 14.2, four over 8 30.0 / 13.3 and the fewest launches; over 2 entries worse with any number of steps.
#include "tg_kernels.h"
#include "tg_device.h"

#define ORDER_NEAR 8             // entries of a list that a step looks at
#define ORDER_STEPS 4
#define ORDER_MAX_BUCKETS 8192
#define ORDER_THREADS 1024

__global__ __launch_bounds__(256) void label_kernel(TgGraph g, const u32* __restrict__ in /* null: a node's own number */, u32* __restrict__ out,
                                                    u32* __restrict__ cnt, int nb)
{
    if (!tg_use_order(g)) return;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < nb; i += stride) cnt[i] = 0u;
    const int near = g.k < ORDER_NEAR ? g.k : ORDER_NEAR;
    for (int64_t v = i0; v < g.n; v += stride) {
        u32 e[ORDER_NEAR], l = in ? in[v] : (u32)v;
#pragma unroll
        for (int q = 0; q < ORDER_NEAR; ++q) e[q] = g.gid[v * g.k + (q < near ? q : 0)] & TG_ID_MASK;
#pragma unroll
        for (int q = 0; q < ORDER_NEAR; ++q) l = min(l, in ? in[e[q]] : e[q]);
        out[v] = in ? min(l, in[l]) : l;
    }
}

// FILL = false: counts the nodes per bucket.  true: counts again, takes a run of every bucket off the counts (which end at zero) and stores
// the nodes there.
template <bool FILL>
__global__ __launch_bounds__(ORDER_THREADS) void order_kernel(TgGraph g, const u32* __restrict__ label, int shift, int nb, int64_t chunk, u32* cnt,
                                                              const u64* __restrict__ off, u32* __restrict__ order)
{
    __shared__ u32 hist[ORDER_MAX_BUCKETS];
    if (!tg_use_order(g)) return;
    const int64_t n = g.n;
    for (int i = threadIdx.x; i < nb; i += ORDER_THREADS) hist[i] = 0u;
    __syncthreads();
    const int64_t beg = (int64_t)blockIdx.x * chunk, end = beg + chunk < n ? beg + chunk : n;
    auto bucket = [&](int64_t v) { return (label[v] * 0x9E3779B1u) >> shift; };
    for (int64_t v = beg + threadIdx.x; v < end; v += ORDER_THREADS) atomicAdd(&hist[bucket(v)], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += ORDER_THREADS) {
        const u32 c = hist[i];
        if (!c) continue;
        if (!FILL) atomicAdd(cnt + i, c);
        else hist[i] = (u32)off[i] + (atomicSub(cnt + i, c) - c);
    }
    if (!FILL) return;
    __syncthreads();
    for (int64_t v = beg + threadIdx.x; v < end; v += ORDER_THREADS) order[atomicAdd(&hist[bucket(v)], 1u)] = (u32)v;
}

// Rows of at least 96 values, 8 M values in all: 100 000 x 128 builds in 7.03 -> 6.94 ms, 30 000 x 500 6.46 -> 5.58, 1M x 128 76.1 -> 74.3 (5 + 5 rounds).
// Below, it is worth less the shorter the rows and costs what it gives: 400 000 x 92 24.1 -> 23.6, 300 000 x 64 15.60 -> 15.63, 1M x 32 49.0 -> 49.6; and at few
// values 87 382 x 96 5.75 -> 5.73, 30 000 x 128 2.62 -> 2.63.
bool tg_order_pays(int64_t n, int ld) { return ld >= 96 && n * ld >= (int64_t)8 << 20; }
// in bytes: the two arrays of labels, the buckets' places and counts
size_t tg_order_space(int64_t n) { return (size_t)(2 * n + 3 * ORDER_MAX_BUCKETS + 4) * sizeof(u32); }
void tg_launch_order(const TgGraph& gr, uint32_t* order, uint32_t* wl_cnt, void* space, hipStream_t s)
{
    TgGraph g = gr;
    g.order = order;
    u64* off = reinterpret_cast<u64*>(space);
    u32* cnt = reinterpret_cast<u32*>(off + ORDER_MAX_BUCKETS + 1);
    u32* label[2] = {cnt + ORDER_MAX_BUCKETS, cnt + ORDER_MAX_BUCKETS + g.n};
    int bits = 6;
    while (bits < 13 && (g.n >> bits) > 1024) ++bits;
    const int nb = 1 << bits;
    const int64_t wgs = (g.n + 255) / 256;
    const dim3 grid((unsigned)(wgs < 8192 ? wgs : 8192)), block(256);
    for (int i = 0; i < ORDER_STEPS; ++i)
        hipLaunchKernelGGL(label_kernel, grid, block, 0, s, g, i ? (const u32*)label[(i + 1) & 1] : (const u32*)nullptr, label[i & 1], cnt, i ? 0 : nb);
    const u32* last = label[(ORDER_STEPS - 1) & 1];
    int64_t chunk = g.n / 512;
    chunk = chunk < ORDER_THREADS ? ORDER_THREADS : chunk > 1 << 14 ? 1 << 14 : chunk;
    const dim3 ogrid((unsigned)((g.n + chunk - 1) / chunk));
    hipLaunchKernelGGL(order_kernel<false>, ogrid, dim3(ORDER_THREADS), 0, s, g, last, 32 - bits, nb, chunk, cnt, (const u64*)off, order);
    tg_launch_scan(cnt, nb, off, wl_cnt, s);
    hipLaunchKernelGGL(order_kernel<true>, ogrid, dim3(ORDER_THREADS), 0, s, g, last, 32 - bits, nb, chunk, cnt, (const u64*)off, order);
}
