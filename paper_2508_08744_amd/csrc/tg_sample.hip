// Phase-1 sampling (step (1) of section 3.1.1): forward samples are read straight from
// the lists (first S new and first S old entries in list order); this file builds the
// bounded reverse samples.  The sampled edges v -> u are brought together by target in two
// steps that write runs, not single words: the targets are cut into buckets of 2^bshift
// consecutive nodes; a workgroup walks a chunk of lists, counts its edges per bucket in LDS,
// takes one run per bucket with one atomic and stores its edges there (bucket step); then one
// workgroup per bucket counts the bucket's edges per target in LDS, stores them grouped by target
// and, a wave per target, keeps per class the R arrivals with the smallest
// (hash(round, source, u), source): a uniform subset that does not depend on arrival order.
// The same wave then assembles the anchor's block and stores it for the join.
#include "tg_kernels.h"
#include "tg_device.h"

// ---- walk of a workgroup over the sampled edges of the lists [vbeg, vend): each group of KP lanes
// (KP = power of two >= k) owns one list at a time
template <class F>
__device__ inline void for_chunk_edges(const TgGraph& g, int S, int kp, int64_t vbeg, int64_t vend, F f)
{
    const int lane = tg_lane(), wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int per_wave = 64 / kp;
    const int sub = lane & (kp - 1), grp = lane / kp;
    const u64 gmask = (kp == 64 ? ~0ull : ((1ull << kp) - 1ull)) << (grp * kp);
    const u64 below = tg_lanemask_lt() & gmask;
    for (int64_t base = vbeg + (int64_t)wave * per_wave; base < vend; base += (int64_t)nwaves * per_wave) {
        const int64_t v = base + grp;
        const bool live = v < vend && sub < g.k;
        const u32 w = live ? g.gid[v * g.k + sub] : 0u;
        const bool fresh = live && (w >> 31);
        const bool old = live && !(w >> 31);
        const u64 mf = __ballot(fresh), mo = __ballot(old);
        const bool take_new = fresh && __popcll(mf & below) < S;
        const bool take_old = old && __popcll(mo & below) < S;
        if (take_new || take_old) f((u32)v, w & TG_ID_MASK, take_old ? 1u : 0u);
    }
}

// Bucket step.  Both kernels count the chunk's edges per bucket in LDS (buckets b0 .. b0 + nb of this launch;
// edges to other buckets belong to another launch).  The first adds the counts to bcnt; once a prefix sum has
// turned bcnt into the buckets' places (boff), the second takes its runs off bcnt again (which so ends at zero,
// ready for the next round) and stores every edge as target % 2^bshift << 32 | class << 31 | source.
#define REV_BUCKET_THREADS 1024      // many waves on one table of counters: the walk is a chain of dependent accesses
template <bool FILL>
__global__ __launch_bounds__(REV_BUCKET_THREADS) void rev_bucket_kernel(TgGraph g, int S, int kp, int bshift, int64_t b0, int nb, int64_t chunk,
                                                         u32* bcnt, const u64* __restrict__ boff, u64* __restrict__ ebuf)
{
    extern __shared__ u32 hist[];            // nb words
    for (int i = threadIdx.x; i < nb; i += REV_BUCKET_THREADS) hist[i] = 0u;
    __syncthreads();
    const int64_t vbeg = (int64_t)blockIdx.x * chunk, vend = vbeg + chunk < g.n ? vbeg + chunk : g.n;
    for_chunk_edges(g, S, kp, vbeg, vend, [&](u32, u32 u, u32) {
        const int64_t b = (int64_t)(u >> bshift) - b0;
        if (b >= 0 && b < nb) atomicAdd(&hist[b], 1u);
    });
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += REV_BUCKET_THREADS) {
        const u32 c = hist[i];
        if (!FILL) {
            if (c) atomicAdd(bcnt + b0 + i, c);
        } else if (c) {
            hist[i] = atomicSub(bcnt + b0 + i, c) - c;       // where this workgroup's run begins inside the bucket
        }
    }
    if (!FILL) return;
    __syncthreads();
    const u32 tmask = (1u << bshift) - 1u;
    for_chunk_edges(g, S, kp, vbeg, vend, [&](u32 v, u32 u, u32 cls) {
        const int64_t b = (int64_t)(u >> bshift) - b0;
        if (b >= 0 && b < nb) {
            const u32 pos = atomicAdd(&hist[b], 1u);
            ebuf[boff[b0 + b] + pos] = ((u64)(u & tmask) << 32) | (u64)(v | (cls << 31));
        }
    });
}

// ---- exclusive prefix sum of the buckets' counts (cnt stays), off[n] = their sum; one workgroup, which also empties the round's work lists.
// (Three launches over the same words, as it was, took 13 us whatever n; this takes 5 for up to 8192 buckets.)
#define SCAN_THREADS 1024
#define SCAN_EACH 8
__global__ __launch_bounds__(SCAN_THREADS) void scan_kernel(const u32* __restrict__ cnt, int64_t n, u64* __restrict__ off, u32* __restrict__ wl_cnt)
{
    __shared__ u64 wsum[SCAN_THREADS / 64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tg_lane();
    if (tid < TG_WL_LISTS) wl_cnt[tid] = 0u;
    u64 carry = 0;
    for (int64_t base = 0; base < n; base += SCAN_THREADS * SCAN_EACH) {
        const int64_t i0 = base + (int64_t)tid * SCAN_EACH;
        u32 x[SCAN_EACH];
        u64 sum = 0;
#pragma unroll
        for (int i = 0; i < SCAN_EACH; ++i) { x[i] = i0 + i < n ? cnt[i0 + i] : 0u; sum += x[i]; }
        u64 incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const u64 y = tg_shfl64(incl, max(lane - o, 0));
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        u64 before = carry, all = 0;
        for (int w = 0; w < SCAN_THREADS / 64; ++w) {
            if (w < wave) before += wsum[w];
            all += wsum[w];
        }
        u64 run = before + incl - sum;
#pragma unroll
        for (int i = 0; i < SCAN_EACH; ++i) {
            if (i0 + i < n) off[i0 + i] = run;
            run += x[i];
        }
        carry += all;
        __syncthreads();
    }
    if (tid == 0) off[n] = carry;
}

// ---- per node: keep the R smallest (priority, source) of each class, then assemble the block --
// Block of anchor v:  NEW = new_fwd ++ (new_rev not yet there),
//                     OLD = (old_fwd not in NEW) ++ (old_rev in neither).
// fwd entries sit one per lane (lanes < k); rid: the kept reverse arrivals (where `has`), ascending
// by (priority, source), the new ones in the lanes from 0, the old ones in those from 32 (at most 32 of either: R is no more).
// A small id -> tag map in LDS for the cross checks between the forward and the reverse samples
// (open addressing, 256 words for at most 64 ids; ids inside one list are distinct).
#define ASM_WORDS 256
#define ASM_FREE 0xFFFFFFFFu
#define ASM_PAST 0x80000000u      // of a taken place (ids have 30 bits): an id whose place it would have been is further on
__device__ inline int asm_insert(u32* keys, u32 id, bool active)
{
    int slot = -1;
    bool pending = active;
    u32 h = (id * 0x9E3779B1u) >> 24;
    while (__ballot(pending)) {
        if (pending) {
            const u32 old = atomicCAS(keys + h, ASM_FREE, id);
            if (old == ASM_FREE) { slot = (int)h; pending = false; }
            else { atomicOr(keys + h, ASM_PAST); h = (h + 1) & (ASM_WORDS - 1); }
        }
    }
    return slot;
}
// (one look, and a walk only from a place that an id went past)
__device__ inline int asm_find(const u32* keys, u32 id, bool active)
{
    u32 h = (id * 0x9E3779B1u) >> 24;
    u32 t = keys[h];
    bool pending = active && t != ASM_FREE && (t & ASM_PAST) && (t & ~ASM_PAST) != id;
    while (__ballot(pending)) {
        if (pending) {
            h = (h + 1) & (ASM_WORDS - 1);
            t = keys[h];
            pending = t != ASM_FREE && (t & ASM_PAST) && (t & ~ASM_PAST) != id;
        }
    }
    return active && (t & ~ASM_PAST) == id ? (int)h : -1;
}
__device__ inline void assemble_block(const TgGraph& g, const TgSample& sm, int64_t v, u32 w /* list entry of lane < k */, u32 rid, bool has,
                                      u32* keys, u32* tags)
{
    const int lane = tg_lane();
    const int k = g.k, S = sm.S;
    const u64 lt = tg_lanemask_lt();
    const bool fr = lane < k && (w >> 31);
    const bool ol = lane < k && !(w >> 31);
    const u64 mf = __ballot(fr), mo = __ballot(ol);
    const bool is_nf = fr && __popcll(mf & lt) < S;     // sampled new forward entry
    const bool is_of = ol && __popcll(mo & lt) < S;     // sampled old forward entry
    const u32 fid = w & TG_ID_MASK;
    const u64 m_nf = __ballot(is_nf);
    // forward samples into the map: tag 1 = new, 2 = old (4 is added when a reverse-new arrival repeats it)
    reinterpret_cast<uint4*>(keys)[lane] = make_uint4(ASM_FREE, ASM_FREE, ASM_FREE, ASM_FREE);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int fslot = asm_insert(keys, fid, is_nf || is_of);
    if (fslot >= 0) tags[fslot] = is_nf ? 1u : 2u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const bool rev_new = lane < 32;
    const int rslot = asm_find(keys, rid, has);
    const u32 tag = rslot >= 0 ? tags[rslot] : 0u;
    // a new arrival is there already as a new forward sample, an old one as a forward sample of either class
    const bool keep_r = has && (rev_new ? tag != 1u : rslot < 0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (rev_new && tag == 2u) tags[rslot] = 6u;         // the old forward sample is NEW through the reverse side
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const bool of_drop = is_of && (tags[fslot >= 0 ? fslot : 0] & 4u);
    const bool keep_of = is_of && !of_drop;
    const u64 m_kr = __ballot(keep_r), m_kof = __ballot(keep_of);
    const int n_nf = __popcll(m_nf), n_krn = __popc((u32)m_kr);
    const int nN = n_nf + n_krn;
    const int n_kof = __popcll(m_kof);
    const int nT = nN + n_kof + __popcll(m_kr >> 32);
    u32* ids = sm.blk + v * (int64_t)sm.BC;
    if (is_nf) ids[__popcll(m_nf & lt)] = fid;
    if (keep_of) ids[nN + __popcll(m_kof & lt)] = fid;
    if (keep_r) ids[__popcll(m_kr & lt) + (rev_new ? n_nf : nN + n_kof - n_krn)] = rid;
    if (lane == 0) sm.bsz[v] = (u32)nN | ((u32)nT << 8);
}

// the work list that takes anchor v's block, -1: nothing to join
__device__ inline int work_list(const TgSample& sm, int64_t v, int nN, int nT)
{
    if (nN == 0 || nT < 2) return -1;
    const int NT = (nT + 15) >> 4;
    return ((int)v & (sm.parts - 1)) * 3 + (NT > 4 ? 2 : (NT == 4 || !sm.wave_ok) ? 1 : 0);
}

// One workgroup per bucket: its edges are counted per target in LDS, stored grouped by target (csr, at the
// bucket's own place: one workgroup writes and reads it, so it stays in that workgroup's cache), and every
// target's arrivals are then cut down to its reverse samples by one wave, which also assembles its block.
__global__ __launch_bounds__(256) void rev_select_kernel(TgGraph g, TgSample sm, u64 hs_rev, int64_t bfirst)
{
    __shared__ u32 tpos[TG_REV_MAX_W];
    __shared__ u64 part[4][2][64];
    __shared__ __align__(16) u32 asm_keys[4][ASM_WORDS];
    __shared__ u32 asm_tags[4][ASM_WORDS];
    __shared__ u32 lcnt[TG_WL_LISTS], lbase[TG_WL_LISTS];
    const int lane = tg_lane(), wave = threadIdx.x >> 6;
    const int64_t b = bfirst + blockIdx.x;
    if (b >= sm.nbuckets) return;
    const int W = 1 << sm.bshift;
    const u64 beg = sm.boff[b], end = sm.boff[b + 1];
    const u64* eb = sm.ebuf;
    for (int i = threadIdx.x; i < W; i += 256) tpos[i] = 0u;
    __syncthreads();
    for (u64 e0 = beg + threadIdx.x; e0 < end; e0 += 4 * 256) {       // four loads on their way at a time
        u64 rec[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) rec[j] = e0 + 256 * j < end ? eb[e0 + 256 * j] : ~0ull;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (e0 + 256 * j < end) atomicAdd(&tpos[(u32)(rec[j] >> 32) & (u32)(W - 1)], 1u);
    }
    __syncthreads();
    if (wave == 0) {
        // exclusive prefix sum over the W targets: a lane takes W / 64 neighbouring ones (fewer targets than lanes: the first W lanes one each)
        const int per = W < 64 ? (lane < W ? 1 : 0) : W >> 6;
        u32 sum = 0;
        for (int i = 0; i < per; ++i) sum += tpos[lane * per + i];
        u32 incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const u32 y = (u32)__shfl((int)incl, max(lane - o, 0));
            if (lane >= o) incl += y;
        }
        u32 run = incl - sum;
        for (int i = 0; i < per; ++i) {
            const u32 c = tpos[lane * per + i];
            tpos[lane * per + i] = run;
            run += c;
        }
    }
    __syncthreads();
    for (u64 e0 = beg + threadIdx.x; e0 < end; e0 += 4 * 256) {
        u64 rec[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) rec[j] = e0 + 256 * j < end ? eb[e0 + 256 * j] : ~0ull;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (e0 + 256 * j < end) {
                const u32 pos = atomicAdd(&tpos[(u32)(rec[j] >> 32) & (u32)(W - 1)], 1u);
                sm.csr[beg + pos] = (u32)rec[j];
            }
    }
    __syncthreads();          // (the stores above are waited for and seen by the whole workgroup)
    // now tpos[t] is where the arrivals of target t end, and those of t + 1 begin
    const u64 lt = tg_lanemask_lt();
    // a wave's targets one after the other; the first arrivals and the list of the next target travel while this one is worked on
    const int k = g.k;
    auto arrivals_of = [&](int t, u64& abeg, u64& aend) {
        abeg = beg + (t ? tpos[t - 1] : 0u);
        aend = beg + tpos[t];
    };
    auto target_ok = [&](int t) { return t < W && (b << sm.bshift) + t < g.n; };
    u64 abeg = 0, aend = 0;
    u32 e_first = 0u, w_list = 0u;
    if (target_ok(wave)) {
        arrivals_of(wave, abeg, aend);
        e_first = abeg + lane < aend ? sm.csr[abeg + lane] : 0u;
        w_list = lane < k ? g.gid[((b << sm.bshift) + wave) * k + lane] : 0u;
    }
    for (int t = wave; target_ok(t); t += 4) {
        const int64_t u = (b << sm.bshift) + t;
        u64 nbeg = 0, nend = 0;
        u32 e_next = 0u, w_next = 0u;
        if (target_ok(t + 4)) {
            arrivals_of(t + 4, nbeg, nend);
            e_next = nbeg + lane < nend ? sm.csr[nbeg + lane] : 0u;
            w_next = lane < k ? g.gid[(u + 4) * k + lane] : 0u;
        }
        // Up to 64 arrivals, the usual case: sorted by class, then the upper 25 bits of their priority, in one network on 32-bit keys.
        u32 rid = 0u;
        int cn = 0, co = 0;
        bool settled = false;
        const int count = (int)min(aend - abeg, (u64)65);
        if (count <= 64) {
            const u32 prio = (u32)(tg_hash_xy(hs_rev, (u64)(e_first & TG_ID_MASK), (u64)u) >> 32);
            u32 order = lane < count ? (e_first & 0x80000000u) | ((prio >> 7) << 6) | (u32)lane : 0xFFFFFFFFu;
            order = tg_wave_sort32_first(order, count);
            const u32 before = (u32)__builtin_amdgcn_update_dpp(-1, (int)order, 0x138, 0xF, 0xF, false);
            // two that agree in those bits (1 target in 60 000): the lower ones decide, below
            if (__ballot(lane > 0 && lane < count && ((order ^ before) >> 6) == 0u) == 0ull) {
                const u32 e = (u32)__builtin_amdgcn_ds_bpermute((int)(order << 2) & 252, (int)e_first);
                co = __popcll(__ballot(lane < count && (e >> 31)));
                cn = count - co;
                const int from = lane < 32 ? lane : cn + lane - 32;
                rid = (u32)__builtin_amdgcn_ds_bpermute(4 * from, (int)e) & TG_ID_MASK;
                settled = true;
            }
        }
        if (!settled) {
            u64 best_new = TG_EMPTY_KEY, best_old = TG_EMPTY_KEY;   // ascending across the wave
            int tot_new = 0, tot_old = 0;
            for (u64 base = abeg; base < aend; base += 64) {
                // key = priority | class << 31 | source: one sort orders both classes; the class bit sits
                // below the priority, so inside a class the order is (priority, source)
                u64 key = TG_EMPTY_KEY;
                if (base + lane < aend) {
                    const u32 e = base == abeg ? e_first : sm.csr[base + lane];
                    const u32 v = e & TG_ID_MASK;
                    key = (tg_hash_xy(hs_rev, (u64)v, (u64)u) & 0xFFFFFFFF00000000ull) | (u64)e;
                }
                key = tg_wave_sort_first(key, (int)(aend - base < 64 ? aend - base : 64));
                const bool is_old = key != TG_EMPTY_KEY && (((u32)key) >> 31);
                const bool is_new = key != TG_EMPTY_KEY && !(((u32)key) >> 31);
                const u64 mn = __ballot(is_new), mo = __ballot(is_old);
                const int mine_new = __popcll(mn), mine_old = __popcll(mo);
                // split into two ascending runs through LDS
                if (is_new) part[wave][0][__popcll(mn & lt)] = key;
                if (is_old) part[wave][1][__popcll(mo & lt)] = key & ~0x80000000ull;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const u64 kn = lane < mine_new ? part[wave][0][lane] : TG_EMPTY_KEY;
                const u64 ko = lane < mine_old ? part[wave][1][lane] : TG_EMPTY_KEY;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (base == abeg) {
                    best_new = kn;
                    best_old = ko;
                } else {
                    if (mine_new) best_new = tg_wave_merge_low(best_new, kn);
                    if (mine_old) best_old = tg_wave_merge_low(best_old, ko);
                }
                tot_new += mine_new;
                tot_old += mine_old;
            }
            const u32 old_id = (u32)__shfl((int)(u32)best_old, lane & 31);       // (every lane takes part)
            rid = lane < 32 ? (u32)best_new : old_id;
            cn = tot_new;
            co = tot_old;
        }
        const bool has = lane < 32 ? lane < min(cn, sm.R) : lane - 32 < min(co, sm.R);
        assemble_block(g, sm, u, w_list, rid, has, asm_keys[wave], asm_tags[wave]);
        abeg = nbeg; aend = nend; e_first = e_next; w_list = w_next;
    }
    if (tg_use_order(g)) return;        // wl_order_kernel writes the work lists
    // Work lists of the join: the bucket's anchors with something to join, by part of the round (v mod parts) and by block size.
    // List 0: at most 3 row groups, list 1: exactly 4, list 2: more.  Without the register-resident join (longer rows)
    // list 1 takes every block of at most 4 row groups and list 0 stays empty.  The list of (part, size class) is
    // wl + (part * 3 + class) * cap with cap = ceil(n / parts) records.  One global atomic per workgroup and list.
    if (threadIdx.x < TG_WL_LISTS) lcnt[threadIdx.x] = 0u;
    __syncthreads();                    // (and every block of the bucket is stored)
    const int64_t cap = (g.n + sm.parts - 1) / sm.parts;
    for (int t0 = 0; t0 < W; t0 += 256) {
        const int t = t0 + (int)threadIdx.x;
        const int64_t v = (b << sm.bshift) + t;
        int list = -1, nN = 0, nT = 0;
        if (t < W && v < g.n) {
            const u32 z = sm.bsz[v];
            nN = (int)(z & 0xFFu);
            nT = (int)(z >> 8);
            list = work_list(sm, v, nN, nT);
        }
        const u32 mypos = list >= 0 ? atomicAdd(lcnt + list, 1u) : 0u;
        __syncthreads();
        if (threadIdx.x < TG_WL_LISTS) lbase[threadIdx.x] = lcnt[threadIdx.x] ? atomicAdd(sm.wl_cnt + threadIdx.x, lcnt[threadIdx.x]) : 0u;
        __syncthreads();
        if (list >= 0 && (int64_t)lbase[list] + mypos < cap) sm.wl[(int64_t)list * cap + lbase[list] + mypos] = tg_pack_rec((u32)v, nN, nT);
        if (threadIdx.x < TG_WL_LISTS) lcnt[threadIdx.x] = 0u;
        __syncthreads();
    }
}

// The work lists in the nodes' order: a workgroup takes 1024 nodes of it and a run of every list.
#define WLO_EACH 4
__global__ __launch_bounds__(256) void wl_order_kernel(TgGraph g, TgSample sm)
{
    __shared__ u32 lcnt[TG_WL_LISTS], lbase[TG_WL_LISTS];
    if (!tg_use_order(g)) return;
    if (threadIdx.x < TG_WL_LISTS) lcnt[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t cap = (g.n + sm.parts - 1) / sm.parts;
    u32 v[WLO_EACH], z[WLO_EACH], pos[WLO_EACH];
    int list[WLO_EACH];
#pragma unroll
    for (int j = 0; j < WLO_EACH; ++j) {
        const int64_t i = ((int64_t)blockIdx.x * WLO_EACH + j) * 256 + threadIdx.x;
        v[j] = i < g.n ? g.order[i] : 0u;
        z[j] = i < g.n ? sm.bsz[v[j]] : 0u;
    }
#pragma unroll
    for (int j = 0; j < WLO_EACH; ++j) {
        list[j] = work_list(sm, v[j], (int)(z[j] & 0xFFu), (int)(z[j] >> 8));
        pos[j] = list[j] >= 0 ? atomicAdd(lcnt + list[j], 1u) : 0u;
    }
    __syncthreads();
    if (threadIdx.x < TG_WL_LISTS) lbase[threadIdx.x] = lcnt[threadIdx.x] ? atomicAdd(sm.wl_cnt + threadIdx.x, lcnt[threadIdx.x]) : 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < WLO_EACH; ++j)
        if (list[j] >= 0 && (int64_t)lbase[list[j]] + pos[j] < cap)
            sm.wl[(int64_t)list[j] * cap + lbase[list[j]] + pos[j]] = tg_pack_rec(v[j], (int)(z[j] & 0xFFu), (int)(z[j] >> 8));
}

// blocks as stored -> the boundary's fixed n x 128 layout (padding -1) and (|NEW|, |OLD|)
__global__ void dump_blocks_kernel(TgGraph g, TgSample sm, int32_t* blk, int32_t* sizes)
{
    size_t total = (size_t)g.n * TG_BLOCK_COLS;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < total; i += stride) {
        const size_t v = i / TG_BLOCK_COLS;
        const int c = (int)(i % TG_BLOCK_COLS);
        const u32 z = sm.bsz[v];
        const int nN = (int)(z & 0xFFu), nT = (int)(z >> 8);
        blk[i] = c < nT ? (int32_t)sm.blk[v * sm.BC + c] : -1;
        if (c == 0) { sizes[v * 2] = nN; sizes[v * 2 + 1] = nT - nN; }
    }
}
void tg_launch_dump_blocks(const TgGraph& g, const TgSample& sm, int32_t* blk, int32_t* sizes, hipStream_t s)
{
    size_t total = (size_t)g.n * TG_BLOCK_COLS;
    size_t grid = (total + 255) / 256;
    if (grid > 65536) grid = 65536;
    hipLaunchKernelGGL(dump_blocks_kernel, dim3((unsigned)grid), dim3(256), 0, s, g, sm, blk, sizes);
}

void tg_launch_scan(const uint32_t* cnt, int64_t n, unsigned long long* off, uint32_t* wl_cnt, hipStream_t s)
{
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(SCAN_THREADS), 0, s, cnt, n, off, wl_cnt);
}

void tg_launch_reverse(const TgGraph& g, const TgSample& sm, uint64_t hs_rev, hipStream_t s)
{
    int kp = 1;
    while (kp < g.k) kp <<= 1;
    const int per_step = (REV_BUCKET_THREADS / 64) * (64 / kp);   // lists a workgroup reads at a time
    // about 2^14 edges per workgroup (measured at 1M x 32: many short walks beat long runs per bucket), fewer where that would leave CUs without
    // one (10 000 x 16: 18 + 9 us for the two walks with 10 workgroups)
    int64_t chunk = (1 << 14) / g.k;
    if (chunk > (g.n + 255) / 256) chunk = (g.n + 255) / 256;
    chunk = (chunk + per_step - 1) / per_step * per_step;
    const unsigned grid = (unsigned)((g.n + chunk - 1) / chunk);
    if (sm.nbuckets * sizeof(u32) > 65536) {
        tg_allow_lds<rev_bucket_kernel<false>>(TG_REV_BUCKETS * sizeof(u32));
        tg_allow_lds<rev_bucket_kernel<true>>(TG_REV_BUCKETS * sizeof(u32));
    }
    for (int pass = 0; pass < 2; ++pass) {
        for (int64_t b0 = 0; b0 < sm.nbuckets; b0 += TG_REV_BUCKETS) {
            const int nb = (int)(sm.nbuckets - b0 < TG_REV_BUCKETS ? sm.nbuckets - b0 : TG_REV_BUCKETS);
            if (pass == 0)
                hipLaunchKernelGGL(rev_bucket_kernel<false>, dim3(grid), dim3(REV_BUCKET_THREADS), nb * sizeof(u32), s, g, sm.S, kp, sm.bshift, b0, nb, chunk, sm.bcnt,
                                   (const u64*)sm.boff, sm.ebuf);
            else
                hipLaunchKernelGGL(rev_bucket_kernel<true>, dim3(grid), dim3(REV_BUCKET_THREADS), nb * sizeof(u32), s, g, sm.S, kp, sm.bshift, b0, nb, chunk, sm.bcnt,
                                   (const u64*)sm.boff, sm.ebuf);
        }
        if (pass == 0) tg_launch_scan(sm.bcnt, sm.nbuckets, sm.boff, sm.wl_cnt, s);
    }
    for (int64_t bf = 0; bf < sm.nbuckets; bf += (1 << 20))
        hipLaunchKernelGGL(rev_select_kernel, dim3((unsigned)(sm.nbuckets - bf < (1 << 20) ? sm.nbuckets - bf : (1 << 20))), dim3(256), 0, s, g, sm,
                           hs_rev, bf);
    if (g.order) hipLaunchKernelGGL(wl_order_kernel, dim3((unsigned)((g.n + 256 * WLO_EACH - 1) / (256 * WLO_EACH))), dim3(256), 0, s, g, sm);
}
// Buckets of 2^shift targets: the smallest (16 at least) of which one launch of the bucket step takes all, because a workgroup of
// the selection serves a bucket and n / 2^shift of them have to fill the chip; at 1M nodes that is 128.  More where one launch of the
// bucket step could not take them (n > 2.6 M): a second one reads every list again.  A round's samples and blocks, against buckets half as wide in two
// launches: 3M nodes, k = 32: 4.6 / 5.1 ms; 4M, k = 16: 3.65 / 4.2; 6M, k = 32: 9.45 / 10.4; 8M, k = 16: 7.5 / 8.2.
int tg_rev_bucket_shift(int64_t n)
{
    int sh = 4;
    while (sh < 7 && ((n + (1ll << sh) - 1) >> sh) > TG_REV_FINE) ++sh;
    while (sh < TG_REV_MAX_SHIFT && ((n + (1ll << sh) - 1) >> sh) > TG_REV_BUCKETS) ++sh;
    return sh;
}
