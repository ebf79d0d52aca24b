// Merge of a local index into the global neighbour lists (section 6.1: every node belongs to
// its closest clusters, each cluster gets a local index, and a node's list becomes
// merge(list so far, its list in the local index)).  The paper merges on the CPU because two
// indexes would not fit a 24 GB card beside the construction; 288 GB of HBM hold both.
//
// W lanes per node of the local index: 32 where both rows have at most 32 entries, so that a wave serves two
// nodes, else the whole wave.  The kernel is bound by the instructions of the map and the merge, not by its
// bytes (0.75 KB per node read or written): eight clusters of 125 000 nodes into 500 000 lists, k = k_local = 32, took 63 us
// a cluster with a wave per node (1.5 TB/s), 44 us with two nodes to a wave and a row without gaps left as it is.
// The node's global row (one entry per lane) and its local row, ids translated to global numbering through the
// cluster's id table, go into an id map in LDS that keeps for every id the first entry that brought it (global
// entries come first); the survivors of both rows are sorted as (distance, id) keys with a bitonic network over the
// W lanes, merged, and the first k are written back.  Rows shorter than k end in id -1, distance +inf.
#include "tg_kernels.h"
#include "tg_device.h"

#define MERGE_MAP_WORDS 256          // of a wave: 4 W entries for the at most 2 W ids of each of its 64 / W nodes
#define MERGE_FREE 0xFFFFFFFFu
#define MERGE_GRID 16384

template <int W>
__device__ inline u32 merge_map_insert(u32* keys, u32* owner, u32 id, u32 entry, bool active)
{
    bool pending = active;
    u32 h = (id * 0x9E3779B1u) >> (W == 32 ? 25 : 24);
    while (__ballot(pending)) {
        if (pending) {
            const u32 old = atomicCAS(keys + h, MERGE_FREE, id);
            if (old == MERGE_FREE || old == id) { atomicMin(owner + h, entry); pending = false; }
            else h = (h + 1) & (4 * W - 1);
        }
    }
    return h;
}

__device__ inline void merge_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// the node's lanes of a ballot
template <int W>
__device__ inline u64 merge_lanes(u64 mask, int lane) { return W == 64 ? mask : (mask >> (lane & 32)) & 0xFFFFFFFFull; }

// the keys of a node that are not empty move to its first lanes, order kept (tmp: W words of 8 bytes private to the node)
template <int W>
__device__ inline u64 merge_close_up(u64 key, u64* tmp, int lane)
{
    const bool has = key != TG_EMPTY_KEY;
    const u64 mask = merge_lanes<W>(__ballot(has), lane);
    if (__ballot((mask & (mask + 1ull)) != 0ull) == 0ull) return key;          // no gaps
    const int r = lane & (W - 1);
    merge_sync();
    if (has) tmp[__popcll(mask & ((1ull << r) - 1ull))] = key;
    merge_sync();
    return r < __popcll(mask) ? tmp[r] : TG_EMPTY_KEY;
}
// true when the keys of every node ascend across its lanes (uniform)
template <int W>
__device__ inline bool merge_ascending(u64 key, int lane)
{
    const u64 prev = tg_shfl64(key, lane > 0 ? lane - 1 : 0);
    return __ballot((lane & (W - 1)) > 0 && prev > key) == 0ull;
}
template <int W>
__device__ inline u64 merge_sort(u64 key) { return W == 64 ? tg_wave_sort(key) : tg_half_sort(key); }
// a and b ascend across the node's lanes: the W smallest keys of their union, ascending
template <int W>
__device__ inline u64 merge_low(u64 a, u64 b)
{
    return W == 64 ? tg_wave_merge_low(a, b) : tg_half_merge_low(a, b);
}

template <int W>
__global__ __launch_bounds__(256) void merge_local_kernel(int32_t* __restrict__ g_ids, float* __restrict__ g_dist, int64_t n, int k,
                                                          const int32_t* __restrict__ l_ids, const float* __restrict__ l_dist,
                                                          int64_t n_local, int k_local, const int32_t* __restrict__ l2g)
{
    constexpr int NODES = 64 / W;
    __shared__ __align__(16) u32 s_keys[4][MERGE_MAP_WORDS];
    __shared__ __align__(16) u32 s_owner[4][MERGE_MAP_WORDS];
    const int wave = threadIdx.x >> 6, lane = tg_lane(), r = lane & (W - 1);
    u32* keys = s_keys[wave] + (lane / W) * 4 * W;
    u32* owner = s_owner[wave] + (lane / W) * 4 * W;
    for (int64_t i0 = ((int64_t)blockIdx.x * 4 + wave) * NODES; i0 < n_local; i0 += (int64_t)gridDim.x * 4 * NODES) {
        const int64_t i = i0 + lane / W;
        const int64_t v = i < n_local ? l2g[i] : -1;
        const bool real = v >= 0 && v < n;                   // else a node without a global row
        if (__ballot(real) == 0ull) continue;
        const uint4 none4 = make_uint4(MERGE_FREE, MERGE_FREE, MERGE_FREE, MERGE_FREE);
        reinterpret_cast<uint4*>(s_keys[wave])[lane] = none4;
        reinterpret_cast<uint4*>(s_owner[wave])[lane] = none4;
        const bool a_on = real && r < k, b_on = real && r < k_local;
        const int32_t a_id = a_on ? g_ids[v * k + r] : -1;
        const float a_dist = a_on ? g_dist[v * k + r] : 0.f;
        const int32_t c = b_on ? l_ids[i * k_local + r] : -1;
        const float b_dist = b_on ? l_dist[i * k_local + r] : 0.f;
        const int32_t b_id = (c >= 0 && c < n_local) ? l2g[c] : -1;
        const bool a_ok = a_id >= 0 && a_id < n && a_id != v;
        const bool b_ok = b_id >= 0 && b_id < n && b_id != v;
        merge_sync();
        // an id counts once: the first entry that brought it, global entries in front of local ones
        const u32 ha = merge_map_insert<W>(keys, owner, (u32)a_id, (u32)r, a_ok);
        const u32 hb = merge_map_insert<W>(keys, owner, (u32)b_id, (u32)(W + r), b_ok);
        merge_sync();
        const bool a_in = a_ok && owner[ha] == (u32)r;
        const bool b_in = b_ok && owner[hb] == (u32)(W + r);
        u64 ka = a_in ? tg_key(a_dist, (u32)a_id, 0u) : TG_EMPTY_KEY;
        u64 kb = b_in ? tg_key(b_dist, (u32)b_id, 0u) : TG_EMPTY_KEY;
        // Rows that tg_knn_build wrote are ascending already; an entry that fell out above leaves a
        // gap.  Closing the gaps (through the map's words, free again by now) keeps the order, and a
        // row whose neighbours in lanes are then in order needs no sorting network.
        ka = merge_close_up<W>(ka, reinterpret_cast<u64*>(keys), lane);
        kb = merge_close_up<W>(kb, reinterpret_cast<u64*>(keys) + W, lane);
        if (!merge_ascending<W>(ka, lane)) ka = merge_sort<W>(ka);
        if (!merge_ascending<W>(kb, lane)) kb = merge_sort<W>(kb);
        const u64 m = merge_low<W>(ka, kb);
        if (a_on) {
            const bool none = m == TG_EMPTY_KEY;
            g_ids[v * k + r] = none ? -1 : (int32_t)tg_key_id(m);
            g_dist[v * k + r] = none ? __builtin_inff() : tg_key_dist(m);
        }
        merge_sync();
    }
}

template <int W>
static void launch_merge(int32_t* g_ids, float* g_dist, int64_t n, int k, const int32_t* l_ids, const float* l_dist, int64_t n_local,
                         int k_local, const int32_t* l2g, hipStream_t s)
{
    const int64_t per = 4 * (64 / W);
    int64_t wgs = (n_local + per - 1) / per;
    if (wgs > MERGE_GRID) wgs = MERGE_GRID;
    hipLaunchKernelGGL(merge_local_kernel<W>, dim3((unsigned)wgs), dim3(256), 0, s, g_ids, g_dist, n, k, l_ids, l_dist, n_local,
                       k_local, l2g);
}
void tg_launch_merge_local(int32_t* g_ids, float* g_dist, int64_t n, int k, const int32_t* l_ids, const float* l_dist,
                           int64_t n_local, int k_local, const int32_t* l2g, hipStream_t s)
{
    if (n_local == 0) return;
    if (k <= 32 && k_local <= 32) launch_merge<32>(g_ids, g_dist, n, k, l_ids, l_dist, n_local, k_local, l2g, s);
    else launch_merge<64>(g_ids, g_dist, n, k, l_ids, l_dist, n_local, k_local, l2g, s);
}
