// Rank-based pruning of a k-NN graph by detourable routes (section 3.2, the CAGRA row of the
// table of pruning strategies; computing paradigm of section 5.2).  The position of a neighbour
// in a row stands for its distance.  For node A and its neighbour F at position p, a node D is
// a detour of the edge (A, F) when both its position in A's row and its position in F's row
// are below p; neighbours with more detours go first: the d_out neighbours with the smallest
// (count, position) stay.
//
// One wave per node A.  A's row goes into an id -> position map in LDS; the rows of the
// neighbours F are read 64 / k' at a time (k' = k rounded up to a power of two), one entry D
// per lane and only the entries in front of F's own position in A's row, and each lane looks
// its D up in the map.  A ballot per row gives the count.  Rows of different useful length are
// balanced as in the paper, by pairing positions q and k - 1 - q inside one group of lanes.
#include "tg_kernels.h"
#include "tg_device.h"

#define PRUNE_ENTRIES 256       // 128 buckets of two (id, position) entries for the at most 64 ids of a row
#define PRUNE_FREE 0xFFFFFFFFu
#define PRUNE_NOPOS 0xFFFFu
#define PRUNE_PAST 0x80000000u  // in the position of a bucket's second entry: an id whose place would have been here is further on
#define PRUNE_GRID 8192
#define PRUNE_PASSES 8

// What a lane does in pass t of a round of eight passes that starts at pair p0 depends only on the
// lane, t, p0 and k: which neighbour F of A it reads (the lane of A's row that holds F, which is F's
// own position) and which entry of F's row.  A lane with nothing to read has position 0: no position is
// below 0, so it never reports a hit.  Positions are kept times four throughout, in the map too: the byte
// address ds_bpermute wants.
struct PruneLaneTable {
    u32 pos4[PRUNE_PASSES];     // 4 x F's position in A's row, 0 if idle
    u32 rr4[PRUNE_PASSES];      // 4 x entry of F's row
};

__device__ inline void prune_fill_table(PruneLaneTable& T, int p0, int k, int kp, int per, int npairs, int my_row, int r)
{
#pragma unroll
    for (int t = 0; t < PRUNE_PASSES; ++t) {
        const int q = p0 + t * per + my_row;
        const int jlo = q, jhi = k - 1 - q;
        const bool lo = r < jlo;
        const int j = lo ? jlo : jhi;
        const int rr = lo ? r : r - jlo;
        const bool on = my_row < per && q < npairs && (lo || (jhi != jlo && rr < jhi));
        T.pos4[t] = on ? (u32)(4 * j) : 0u;
        T.rr4[t] = on ? (u32)(4 * rr) : 0u;
    }
}

// A look-up goes on beyond its home bucket only where an id went past that when the map was built, which the bucket's second entry says: a full
// bucket alone, which every other pass meets, used to start a loop of the whole wave.  1M lists of 32: 868 -> 670 us, 100 000 of 64: 594 -> 470,
// 200 000 of 48: 659 -> 497, 300 000 of 16: 139 -> 120, 10 000 of 32: 20.1 -> 17.9.
// ONE (all pairs in one round of eight passes: k <= 32, the lane table never changes): the neighbours' entries are asked for before
// the map is built, the next node's row before this one is looked up.  What bounds the kernel is instructions and the latency of the
// entries; without and with ONE, kernels under the profiler: 1M lists of 32: 871 / 760 us, of 16: 521 / 399, 300 000 of 24: 228 / 191.
// NEAR: the lists are less than 4 GiB, so an entry's byte offset has 32 bits (half the address registers).
// LONE (with ONE and NEAR): every wave serves one node.  No next row to ask for, the entries are asked for behind the map, which takes
// 44 registers instead of 76 and leaves eight waves per SIMD to cover them; passes without a pair are left out, and idle lanes read one row that
// is there already instead of the first neighbour's.  Without and with it: 30 000 lists of 16: 24.2 / 21.0 us, 14 448: 13.4 / 12.1,
// 30 000 of 32: 34.4 / 34.4, 5000 of 32: 11.4 / 11.5.
template <bool ONE, bool NEAR, bool LONE>
__global__ __launch_bounds__(256) void prune_rank_kernel(const int32_t* __restrict__ ids, int64_t n, int k, int kp, int d_out,
                                                         int32_t* __restrict__ out_ids, int32_t* __restrict__ counts)
{
    __shared__ __align__(16) u32 maps[4][2 * PRUNE_ENTRIES];      // entry e: word 2e = id, word 2e + 1 = position x 4
    const int wave = threadIdx.x >> 6, lane = tg_lane();
    u32* map = maps[wave];
    const int per = 64 / kp;                         // rows of neighbours per pass
    const int my_row = lane / kp, r = lane - my_row * kp;
    const int npairs = (k + 1) >> 1;
    PruneLaneTable T;
    prune_fill_table(T, 0, k, kp, per, npairs, my_row, r);
    // the count of position P = lane comes out of the pass that serves pair q = min(P, k - 1 - P):
    // in that pass's ballot its hits start at bit (row of the pair) x k' (+ q for the far partner), P bits long
    const int myq = min(lane, k - 1 - lane);
    const int lp = 31 - __clz(per);                  // per is a power of two
    const u32 n32 = (u32)n;                          // n < 2^30
    const int64_t A0 = (int64_t)blockIdx.x * 4 + wave, step = (int64_t)gridDim.x * 4;
    if (A0 >= n) return;                             // (no workgroup barrier below)
    auto row_of = [&](int64_t A) __attribute__((always_inline)) -> int32_t {          // past the end: the last node's, never used
        const int32_t got = ids[min(A, n - 1) * k + (lane < k ? lane : 0)];
        return lane < k ? got : -1;
    };
    auto gather = [&](int32_t a, int32_t (&D)[PRUNE_PASSES]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < PRUNE_PASSES; ++t) {
            if (LONE && t * per >= npairs) break;            // uniform
            const int32_t F = __builtin_amdgcn_ds_bpermute((int)T.pos4[t], a);
            // row 0 where F is no node (one unsigned compare also rejects negative ids): what is found there is counted for F alone,
            // and F's count is left out at the end
            const u32 row = ((u32)F < n32) & (!LONE | (T.pos4[t] != 0u)) ? (u32)F : 0u;
            if (NEAR) D[t] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(ids) + (row * (4u * (u32)k) + T.rr4[t]));
            else D[t] = ids[(u64)row * (u32)k + (T.rr4[t] >> 2)];
        }
    };
    int32_t a = ONE ? row_of(A0) : -1, a_after = -1;
    int32_t D[PRUNE_PASSES];
    for (int64_t A = A0; A < n; A += step) {
        if (ONE && !LONE) {
            a_after = row_of(A + step);
            gather(a, D);
        }
        if (!ONE) a = row_of(A);
        const bool a_ok = (u32)a < n32;
        for (int i = lane; i < PRUNE_ENTRIES; i += 64) *reinterpret_cast<uint2*>(map + 2 * i) = make_uint2(PRUNE_FREE, PRUNE_NOPOS);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // A's row into the map (a bucket is read with one 16-byte load later); an id listed twice
        // keeps its first position (its lanes walk in step, so all of them find it in the same turn, before that turn's marks)
        {
            bool pending = a_ok;
            u32 e = (((u32)a * 0x9E3779B1u) >> 25) << 1;
            while (__ballot(pending)) {
                if (pending) {
                    const u32 old = atomicCAS(map + 2 * e, PRUNE_FREE, (u32)a);
                    if (old == PRUNE_FREE || old == (u32)a) { atomicMin(map + 2 * e + 1, (u32)lane << 2); pending = false; }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (pending) {
                    if (e & 1u) atomicOr(map + 2 * e + 1, PRUNE_PAST);
                    e = (e + 1) & (PRUNE_ENTRIES - 1);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // Rows are taken in pairs (positions q and k - 1 - q): the first needs its q entries in
        // front, the second k - 1 - q, together k - 1 lanes of a group of k' (the balanced
        // pairing of section 5.2).  64 / k' pairs per pass; the loads of eight passes are in
        // flight before the first look-up.
        u32 c = 0u;
        for (int p0 = 0; p0 < npairs; p0 += PRUNE_PASSES * per) {
            if (!ONE) {
                prune_fill_table(T, p0, k, kp, per, npairs, my_row, r);
                gather(a, D);
            }
            if (LONE) gather(a, D);
            u64 mine = 0ull;                      // the ballot of the pass that serves this lane's position
#pragma unroll
            for (int t = 0; t < PRUNE_PASSES; ++t) {
                if (p0 + t * per >= npairs) break;           // uniform
                // look D up: its home bucket, then, if ids went past that (3 targets in 10 have such a bucket), entry by entry.
                // -1 matches a free entry, whose position is below nothing.
                const u32 d = (u32)D[t];
                u32 e = ((d * 0x9E3779B1u) >> 25) << 1;
                const uint4 b = *reinterpret_cast<const uint4*>(map + 2 * e);
                // (no short cuts: every lane evaluates everything, nothing branches)
                const bool e0 = b.x == d, e1 = b.z == d;
                bool hit = (e0 & (b.y < T.pos4[t])) | (e1 & ((b.w & ~PRUNE_PAST) < T.pos4[t]));
                bool pending = !e0 & !e1 & ((b.w & PRUNE_PAST) != 0u);
                e = (e + 2) & (PRUNE_ENTRIES - 1);
                while (__ballot(pending)) {
                    if (pending) {
                        const uint2 w = *reinterpret_cast<const uint2*>(map + 2 * e);
                        if (w.x == d) { hit = (w.y & ~PRUNE_PAST) < T.pos4[t]; pending = false; }
                        else if (w.x == PRUNE_FREE) pending = false;
                        else e = (e + 1) & (PRUNE_ENTRIES - 1);
                    }
                }
                const u64 hits = __ballot(hit);
                if (((myq - p0) >> lp) == t) mine = hits;          // (a pair of an earlier round gives a negative number)
            }
            const int rel = myq - p0;
            if (lane < k && rel >= 0 && rel < PRUNE_PASSES * per) {
                const int row = rel & (per - 1);
                const int shift = row * kp + (lane == myq ? 0 : myq);       // the near partner's hits come first
                c = a_ok ? (u32)__popcll((mine >> shift) & ((1ull << lane) - 1ull)) : 0u;
            }
        }
        if (counts && lane < k) counts[A * k + lane] = (int32_t)c;
        // smallest (count, position) first
        u32 key = lane < k ? ((c << 8) | (u32)lane) : 0xFFFFFFFFu;
        key = tg_wave_sort32(key);
        const int32_t keep = __shfl(a, (int)(key & 63u));
        if (lane < d_out) out_ids[A * d_out + lane] = keep;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (LONE) return;
        if (ONE) a = a_after;
    }
}

void tg_launch_prune_rank(const int32_t* ids, int64_t n, int k, int d_out, int32_t* out_ids, int32_t* counts, hipStream_t s)
{
    int kp = 1;
    while (kp < k) kp <<= 1;
    int64_t wgs = (n + 3) / 4;
    if (wgs > PRUNE_GRID) wgs = PRUNE_GRID;
    const bool one_round = (k + 1) / 2 <= PRUNE_PASSES * (64 / kp);
    const bool near = (uint64_t)n * (uint64_t)k * 4u < (1ull << 32);
    const bool lone = one_round && near && n <= 4 * wgs;
    auto kernel = lone ? prune_rank_kernel<true, true, true>
                  : one_round ? (near ? prune_rank_kernel<true, true, false> : prune_rank_kernel<true, false, false>)
                              : (near ? prune_rank_kernel<false, true, false> : prune_rank_kernel<false, false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(256), 0, s, ids, n, k, kp, d_out, out_ids, counts);
}
