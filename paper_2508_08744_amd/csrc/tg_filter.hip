// Distance-based and angle-based pruning of a k-NN graph in the Collect-Filter-Store procedure
// (section 5.1; the NSG, Vamana and NSSG rows of the table of pruning strategies, section 3.2).
// For node p the candidates are its neighbours (hops = 1) or those and their neighbours
// (hops = 2), ordered by (dis(p, c), id) and cut to cand_size; they are taken closest first and
// p' is inserted iff, for every p* inserted before,
//   distance rule:  dis(p, p') < alpha dis(p*, p')   (distances are squared here: alpha^2), or
//   angle rule:     the angle between p -> p* and p -> p' exceeds gamma; with the squared
//                   lengths a = |p p*|^2, b = |p p'|^2, c = |p* p'|^2 and t = a + b - c that is
//                   t < 0 or t^2 < 4 cos^2(gamma) a b   (no square root, no division),
// until d_out are in.  The dispersion rule (DPG) has no threshold: the nearest candidate is
// inserted first, then again and again the candidate whose angles at p to the inserted nodes add
// up to the most (equal sums: the nearer one), until d_out are in or none is left.
//
// One wave per node.  Section 5.2 evaluates a batch of candidates against the neighbour that
// was inserted last, one batch per insertion.  Here the candidate rows (at most 64) are loaded
// once into registers in matrix-core operand layout and ALL their pairwise products are
// formed at once (a Gram matrix on v_mfma_f32_16x16x4_f32, upper triangle of 16 x 16 tiles);
// what remains of the serial rule is bit arithmetic: every candidate gets the 64-bit set of
// the candidates in front of it that would occlude it, and the set of inserted candidates is the
// fixed point of "inserted iff no inserted candidate occludes me", found in a few passes.  The rows are the only large HBM traffic
// (4 d bytes per candidate); the products are cheap next to it.
//
// Lane (r, q) = (lane % 16, lane / 16) holds, for row group t and column step s, columns
// 16 s + 4 q .. + 3 of the current chunk of columns of candidate 16 t + r: one load instruction
// reads 64 contiguous bytes of each of 16 rows.  dis(p, c) is summed in difference form from
// the same registers.
#include "tg_kernels.h"
#include "tg_device.h"

// Collect: the neighbours; those and theirs for rows of at most 32 ids; the same for rows of up to 64 ids
// (a larger id set and queue per wave)
#define FILTER_ONE_HOP 1
#define FILTER_TWO_HOPS 2
#define FILTER_TWO_HOPS_WIDE 3
// 2-hop collection of at most k + k * k ids: places of the id set (a power of two, at most half of them taken) and words of the queue
__host__ __device__ constexpr int filter_set_places(int collect) { return collect == FILTER_TWO_HOPS_WIDE ? 8192 : 2048; }
__host__ __device__ constexpr int filter_queue_words(int collect) { return collect == FILTER_TWO_HOPS_WIDE ? 4224 : 1088; }
#define FILTER_WAVES 4
// Rows of second-hop ids on their way at a time.  Rows of X that are no multiple of 16 bytes come value by value, four times the loads, and
// eight rows of ids before them only hold registers (18 595 x 279, k = 12: 1280 us with eight, 1264 with two; 18 595 x 280 in
// 16-byte pieces: 460 us with eight, 474 with two).
__host__ __device__ constexpr int filter_loads(bool vec) { return vec ? 8 : 2; }
#define FILTER_NOWHERE 0xFFFFu  // a free place of the id set
#define FILTER_GRID 16384
#define FILTER_FREE 0xFFFFFFFFu

typedef float floatx4 __attribute__((ext_vector_type(4)));

struct FilterArgs {
    const float* X;
    int64_t n;
    int32_t d;
    const int32_t* ids;
    int32_t k, kp;          // kp: k rounded up to a power of two
    int32_t hops, cand_size;
    float thr;              // alpha^2 (distance rule) or 4 cos^2(gamma) (angle rule)
    int32_t d_out;
    int32_t* out_ids;
    int32_t* out_deg;
};

__device__ inline float4 filter_load4(const float* row, int col, int d, bool full, bool vec)
{
    if (full) return *reinterpret_cast<const float4*>(row + col);
    if (vec) return col < d ? *reinterpret_cast<const float4*>(row + col) : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 v;
    v.x = col + 0 < d ? row[col + 0] : 0.f;
    v.y = col + 1 < d ? row[col + 1] : 0.f;
    v.z = col + 2 < d ? row[col + 2] : 0.f;
    v.w = col + 3 < d ? row[col + 3] : 0.f;
    return v;
}

// Loads the chunk [c0, c0 + 16 KS) of the rows cid[0 .. cnt) (16 NG >= cnt; rows past cnt repeat
// row 0) and adds this lane's share of the squared differences to node p's row into dp[t].
template <int NG, int KS, bool FULL, bool VEC>
__device__ inline void filter_load_chunk(const FilterArgs& A, const float* xp, const int* cid, int cnt, int c0,
                                         float4 (&X)[NG][KS], float (&dp)[NG])
{
    const int lane = tg_lane(), r16 = lane & 15, q4 = lane >> 4;
    const float* rp[NG];
#pragma unroll
    for (int t = 0; t < NG; ++t) {
        const int row = 16 * t + r16;
        rp[t] = A.X + (int64_t)cid[row < cnt ? row : 0] * A.d;
    }
#pragma unroll
    for (int t = 0; t < NG; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s) X[t][s] = filter_load4(rp[t], c0 + 16 * s + 4 * q4, A.d, FULL, VEC);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const float4 a = filter_load4(xp, c0 + 16 * s + 4 * q4, A.d, FULL, VEC);
#pragma unroll
        for (int t = 0; t < NG; ++t) {
            const float t0 = a.x - X[t][s].x, t1 = a.y - X[t][s].y, t2 = a.z - X[t][s].z, t3 = a.w - X[t][s].w;
            dp[t] += t0 * t0 + t1 * t1 + t2 * t2 + t3 * t3;
        }
    }
}

// the four quarter sums of a row meet: afterwards every lane (r, q) holds the whole sum of row 16 t + r
template <int NG>
__device__ inline void filter_reduce_quarters(float (&dp)[NG])
{
#pragma unroll
    for (int t = 0; t < NG; ++t) {
        dp[t] += __shfl_xor(dp[t], 16);
        dp[t] += __shfl_xor(dp[t], 32);
    }
}

template <int NG>
__device__ inline float filter_own(const float (&dp)[NG], int q4)
{
    // lane 16 q + r speaks for row 16 q + r (values are picked from copies: an indexed read would go through scratch); rows
    // past 16 NG are none
    const float d0 = dp[0], d1 = dp[NG > 1 ? 1 : 0], d2 = dp[NG > 2 ? 2 : 0], d3 = dp[NG > 3 ? 3 : 0];
    const float lo = (q4 & 1) ? d1 : d0;
    const float hi = (q4 & 1) ? d3 : d2;
    return (NG > 2 && (q4 & 2)) ? hi : lo;
}

__device__ inline void filter_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Appends the ids of the lanes that are `active` to the queue, each id once and only if it is not there already; returns the
// queue's new length.  A place of the set holds where in the queue its id is (two bytes instead of the id's four: the set is
// most of what a wave needs of LDS), or, while the ids of one call meet, 0x8000 | lane, the id being in batch[lane].  Lanes that
// find the same place free all write it and read back who got it, so the accesses are volatile.  The set is at most half
// full, so every search ends.
template <int PLACES>
__device__ inline int filter_collect(unsigned short* set, int* queue, int* batch, int Q, int id, bool active)
{
    volatile unsigned short* T = set;
    const int lane = tg_lane();
    const unsigned short mine = (unsigned short)(0x8000 | lane);
    bool pending = active, fresh = false;
    u32 h = ((u32)id * 0x9E3779B1u) >> (PLACES == 8192 ? 19 : 21);          // the top log2(PLACES) bits
    batch[lane] = id;
    filter_wave_sync();
    while (__ballot(pending)) {
        if (pending && T[h] == FILTER_NOWHERE) T[h] = mine;
        filter_wave_sync();
        if (pending) {
            const u32 e = T[h];
            const int there = (e & 0x8000u) ? batch[e & 63u] : queue[e];
            if (e == mine) { fresh = true; pending = false; }
            else if (there == id) pending = false;
            else h = (h + 1) & (PLACES - 1);
        }
        filter_wave_sync();
    }
    const u64 mask = __ballot(fresh);
    const int at = Q + __popcll(mask & tg_lanemask_lt());
    if (fresh) { queue[at] = id; T[h] = (unsigned short)at; }
    filter_wave_sync();
    return Q + __popcll(mask);
}

// The same on a set that holds the ids themselves (four bytes a place, free: FILTER_FREE): one atomic per step of a search, where the
// above takes a read, a write, a read back and the waits between them.
template <int PLACES>
__device__ inline int filter_collect_ids(u32* set, int* queue, int Q, int id, bool active)
{
    bool pending = active, fresh = false;
    u32 h = ((u32)id * 0x9E3779B1u) >> (PLACES == 8192 ? 19 : 21);          // the top log2(PLACES) bits
    while (__ballot(pending)) {
        if (pending) {
            const u32 old = atomicCAS(set + h, FILTER_FREE, (u32)id);
            if (old == FILTER_FREE) { fresh = true; pending = false; }
            else if (old == (u32)id) pending = false;
            else h = (h + 1) & (PLACES - 1);
        }
    }
    const u64 mask = __ballot(fresh);
    if (fresh) queue[Q + __popcll(mask & tg_lanemask_lt())] = id;
    return Q + __popcll(mask);
}

// Square root and quotient rounded once, for arguments whose exponents leave every step room: the hardware's approximation, a step of
// Newton's method on it, and the remainder, taken exactly by a fused multiply-add, times it (Markstein, "Computation of elementary functions on
// the IBM RISC System/6000 processor", 1990).  8 and 6 instructions where the general ones, which scale and sort out the special values, take
// 16 and 12.  Checked against sqrtf for every float of 2^-92 .. 2^92 and against / for 2e10 pairs of the range below: the same bits.
__device__ inline float filter_sqrt(float x)
{
#pragma clang fp contract(off)
    const float y = __builtin_amdgcn_rsqf(x);
    float g = x * y, h = 0.5f * y;
    const float r = fmaf(-h, g, 0.5f);
    g = fmaf(g, r, g);
    h = fmaf(h, r, h);
    return fmaf(fmaf(-g, g, x), h, g);
}
__device__ inline float filter_quotient(float t, float d)
{
#pragma clang fp contract(off)
    float r = __builtin_amdgcn_rcpf(d);
    r = fmaf(fmaf(-d, r, 1.0f), r, r);
    const float q = t * r;
    return fmaf(fmaf(-d, q, t), r, q);
}
// Squared lengths a and b for which the above serve: 0 (the angle is 0 whatever comes out) or 2^-45 .. 2^45.  Then a b is 0 or within 2^+-90, and
// t, a multiple of 2^-70 unless it is larger than 2^-46, is 0 or large enough for the remainder to be exact.  Nothing is asked of c, which bounds t
// from above: a t beyond the divisor is taken for it before the division, not the quotient for 1 behind it.
__device__ inline bool filter_plain_length(float v) { return v == 0.0f || (v >= 2.842170943e-14f && v <= 3.518437209e13f); }

// Angle at p between p -> r and p -> c from the squared lengths a = |p r|^2, b = |p c|^2, c = |r c|^2:
// acos((a + b - c) / (2 sqrt(a b))), the arc cosine from the eight-term polynomial of Abramowitz and
// Stegun 4.4.46 (acos x = sqrt(1 - x) (a0 + .. + a7 x^7) on [0, 1], pi - acos(-x) below 0).  Every
// operation is rounded once, in this order, so that a host program can follow it bit for bit.
// A node at p's position (a b = 0) has no direction: angle 0.  PLAIN: a and b are filter_plain_length.
template <bool PLAIN>
__device__ inline float filter_angle_at(float a, float b, float c)
{
#pragma clang fp contract(off)
    const float ab = a * b;
    const float den = 2.0f * (PLAIN ? filter_sqrt(ab) : sqrtf(ab));
    float t = (a + b) - c, x;
    if (PLAIN) {
        // (the quotient of an infinite or huge t would be infinity less infinity; a rounded quotient is beyond 1 exactly where t is beyond den)
        t = t > den ? den : t;
        t = t < -den ? -den : t;
        x = filter_quotient(t, den);
    } else {
        x = t / den;
        x = x > 1.0f ? 1.0f : x;
        x = x < -1.0f ? -1.0f : x;
    }
    const float ax = fabsf(x);
    float pol = -0.0012624911f;
    pol = fmaf(pol, ax, 0.0066700901f);
    pol = fmaf(pol, ax, -0.0170881256f);
    pol = fmaf(pol, ax, 0.0308918810f);
    pol = fmaf(pol, ax, -0.0501743046f);
    pol = fmaf(pol, ax, 0.0889789874f);
    pol = fmaf(pol, ax, -0.2145988016f);
    pol = fmaf(pol, ax, 1.5707963050f);
    const float u = 1.0f - ax;                      // 0, or 2^-24 and more
    const float root = !PLAIN ? sqrtf(u) : u == 0.0f ? 0.0f : filter_sqrt(u);
    const float r = root * pol;
    const float th = x < 0.0f ? 3.14159265358979323846f - r : r;
    return ab > 0.0f ? th : 0.0f;
}

__global__ void angle_at_kernel(const float* a, const float* b, const float* c, float* out, int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    // (as the filter does: a wave takes the short way where all its lengths allow it)
    if (__ballot(!(filter_plain_length(a[i]) && filter_plain_length(b[i]))) == 0ull) out[i] = filter_angle_at<true>(a[i], b[i], c[i]);
    else out[i] = filter_angle_at<false>(a[i], b[i], c[i]);
}
void tg_launch_angle_at(const float* a, const float* b, const float* c, float* out, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(angle_at_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, a, b, c, out, count);
}

// maximum over the wave: xor butterfly by DPP inside each row of 16 lanes, then the four rows meet in scalar registers
__device__ inline u32 filter_wave_max(u32 x)
{
    x = max(x, tg_partner32<1>(x));
    x = max(x, tg_partner32<2>(x));
    x = max(x, tg_partner32<7>(x));
    x = max(x, tg_partner32<15>(x));
    const u32 r0 = (u32)__builtin_amdgcn_readlane((int)x, 0), r1 = (u32)__builtin_amdgcn_readlane((int)x, 16);
    const u32 r2 = (u32)__builtin_amdgcn_readlane((int)x, 32), r3 = (u32)__builtin_amdgcn_readlane((int)x, 48);
    return max(max(r0, r1), max(r2, r3));
}

#define FILTER_RULE_DIST 0
#define FILTER_RULE_ANGLE 1
#define FILTER_RULE_DISPERSION 2
// The neighbours under a threshold rule: 2.75 KB of LDS a wave are enough for arrays of their own, registers (three or four waves per
// SIMD) are what limits the waves, and a wait before the keys replace the distances is saved: 100 000 x 300, k = 32: 680 -> 671 us,
// 60 000 x 37, k = 64: 348 -> 344 us.
__host__ __device__ constexpr bool filter_apart(int collect, int rule) { return collect == FILTER_ONE_HOP && rule != FILTER_RULE_DISPERSION; }

// Rows of at most 32 ids within two hops under the dispersion rule: the matrix of angles (16.6 KB a wave, two workgroups a CU) is larger
// than a set of ids, so nothing is saved by two-byte places, and two waves per SIMD do not cover their waits: 30 000 x 64, k = 32:
// 883 -> 779 us, 30 000 x 128: 1242 -> 1138 us.  Where the set sets the number of workgroups two bytes are better (k = 48: 3.29 ms with
// ids, 2.44 with two bytes).
__host__ __device__ constexpr bool filter_set_of_ids(int collect, int rule) { return collect == FILTER_TWO_HOPS && rule == FILTER_RULE_DISPERSION; }

// Words of dynamic LDS per wave.  While ids are collected: the id -> first lane table of one hop (256 words behind the candidates' ids),
// or the set, queue and batch of two hops.  Afterwards, in the same words: the candidates' ids (64), their distances to p and
// norms and then their keys (128), and the sets of occluding candidates (128) or the matrix of angles (rows of 16 NG + 1 words).
// With this a workgroup of the dispersion rule for k in 33..48 takes 40 704 bytes and one of the 2-hop collection 35 072, four a
// CU (as separate arrays, with ids in the set: 78 and 62 KB, two a CU).
__host__ __device__ constexpr int filter_lds_words(int ng, int collect, int rule)
{
    if (filter_apart(collect, rule)) return 0;
    const int set = filter_set_of_ids(collect, rule) ? filter_set_places(collect) : filter_set_places(collect) / 2 + 64;
    const int ids = collect == FILTER_ONE_HOP ? 64 + 256 : set + filter_queue_words(collect);
    const int rows = 64 + 128 + (rule == FILTER_RULE_DISPERSION ? 16 * ng * (16 * ng + 1) : 128);
    return ((ids > rows ? ids : rows) + 3) & ~3;
}

// Waves per SIMD that the compiler must leave room for.  Four for the neighbours under the dispersion rule, which is bound by what a
// wave does in sequence (products, angles, the greedy): 200 000 x 200, k = 40, d_out = 20: 2.65 ms with 64 rows and two waves, 1.85 ms
// with 48 rows and four (two for 49..64 neighbours, whose matrices of angles leave room for no more); and for 33..48 neighbours under the others, which have the registers (111) anyway.  No demand on the other
// threshold instances, which wait for rows: asked for four, that of up to 32 neighbours gets fewer loads on their way (100 000 x 128,
// k = 32: 310 us against 274) and that of 49..64 spills (60 000 x 37, k = 64: 353 against 344 us).  Three for two hops, which wait for
// rows too (4 d bytes per distinct id, 5.5 TB/s): with four the compiler spills, 250 000 x 128, k = 32: 8.62 against 8.45 ms (9.17 with
// two waves and the rows of ids read one at a time), and none where rows come value by value (18 595 x 279, k = 12: 1298 -> 1280 us).
__host__ __device__ constexpr int filter_least_waves(int ng, int collect, int rule, bool vec)
{
    if (collect != FILTER_ONE_HOP) return vec ? 3 : 1;
    if (rule == FILTER_RULE_DISPERSION && ng == 4) return 2;
    return rule == FILTER_RULE_DISPERSION || ng == 3 ? 4 : 1;
}

// The angle at p of every pair of candidates into the matrix `ang` (rows of 16 NG + 1 words), both ways round, from the products of their rows
// (tile (i, j), j >= i), their distances to p (dp: of row 16 t + r; dpc: of all) and squared norms.  A tile on the diagonal holds each pair
// twice, so two of them are worked through as one: the upper half of the first, the lower half of the second.  (An entry on the
// diagonal is nobody's angle and is not read.)
template <int NG, bool PLAIN>
__device__ __forceinline__ void filter_angles(const floatx4 (&acc)[NG][NG], const float (&dp)[NG], const float* nrm, const float* dpc, int groups,
                                              float* ang)
{
    constexpr int AS = 16 * NG + 1;
    const int lane = tg_lane(), r16 = lane & 15, q4 = lane >> 4;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        if (i >= groups) break;
        const float4 nRv = *reinterpret_cast<const float4*>(nrm + 16 * i + 4 * q4);
        const float4 dRv = *reinterpret_cast<const float4*>(dpc + 16 * i + 4 * q4);
        const float nR[4] = {nRv.x, nRv.y, nRv.z, nRv.w}, dR[4] = {dRv.x, dRv.y, dRv.z, dRv.w};
        const bool first = (i & 1) == 0, two = i + 1 < NG && i + 1 < groups;       // of two diagonal tiles that go together; both there
#pragma unroll
        for (int j = i; j < NG; ++j) {
            if (j >= groups) break;
            if (j == i && (!first || two)) continue;                    // (with the other one, below)
            const float nC = nrm[16 * j + r16];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int R = 16 * i + 4 * q4 + e, C = 16 * j + r16;
                const float rc = (nR[e] + nC) - 2.0f * acc[i][j][e];        // dis(R, C)
                const float th = filter_angle_at<PLAIN>(dR[e], dp[j], rc);
                ang[R * AS + C] = th;
                ang[C * AS + R] = th;
            }
        }
        if (!first || !two) continue;
        constexpr int LAST = NG - 1;
        const int h = i < LAST ? i + 1 : LAST;
        const float nC1 = nrm[16 * i + r16], nC2 = nrm[16 * h + r16];
        const float4 nR2v = *reinterpret_cast<const float4*>(nrm + 16 * h + 4 * q4);
        const float4 dR2v = *reinterpret_cast<const float4*>(dpc + 16 * h + 4 * q4);
        const float nR2[4] = {nR2v.x, nR2v.y, nR2v.z, nR2v.w}, dR2[4] = {dR2v.x, dR2v.y, dR2v.z, dR2v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int R = 4 * q4 + e;
            const bool up = r16 > R;                                        // the pair of tile i, else that of tile i + 1
            const float rc = (up ? nR[e] + nC1 : nR2[e] + nC2) - 2.0f * (up ? acc[i][i][e] : acc[h][h][e]);
            const float th = filter_angle_at<PLAIN>(up ? dR[e] : dR2[e], up ? dp[i] : dp[h], rc);
            const int at = (AS + 1) * 16 * (up ? i : h);
            ang[at + R * AS + r16] = th;
            ang[at + r16 * AS + R] = th;
        }
    }
}

template <int NG, int KS, bool FULL, bool VEC, int COLLECT, int RULE>
__global__ __launch_bounds__(256, filter_least_waves(NG, COLLECT, RULE, VEC)) void filter_dist_kernel(FilterArgs A)
{
    constexpr bool TWO_HOPS = COLLECT != FILTER_ONE_HOP;
    constexpr int PLACES = filter_set_places(COLLECT);
    constexpr int LOADS = filter_loads(VEC);
    constexpr bool ANGLE = RULE == FILTER_RULE_ANGLE;
    constexpr bool APART = filter_apart(COLLECT, RULE);
    constexpr bool ID_SET = filter_set_of_ids(COLLECT, RULE);
    constexpr int LDS_WORDS = filter_lds_words(NG, COLLECT, RULE);
    [[maybe_unused]] constexpr int AS = 16 * NG + 1;      // row stride of the matrix of angles
    constexpr int AW = APART ? FILTER_WAVES : 1;
    extern __shared__ __align__(16) u32 lds[];
    __shared__ int s_cid[AW][64];                       // (these six: unused and not allocated unless APART)
    __shared__ __align__(16) float s_dpc[AW][64];
    __shared__ __align__(16) float s_nrm[AW][64];
    __shared__ u32 s_occ[AW][128];
    __shared__ __align__(16) u64 s_key[AW][64];
    __shared__ u32 s_twin[AW][256];
    const int wave = threadIdx.x >> 6, lane = tg_lane();
    const int r16 = lane & 15, q4 = lane >> 4;
    u32* own_lds = lds + wave * LDS_WORDS;
    int* cid = APART ? s_cid[wave] : reinterpret_cast<int*>(own_lds);
    float* dpc = APART ? s_dpc[wave] : reinterpret_cast<float*>(own_lds + 64);
    float* nrm = APART ? s_nrm[wave] : reinterpret_cast<float*>(own_lds + 128);
    u64* skey = APART ? s_key[wave] : reinterpret_cast<u64*>(own_lds + 64);           // the candidates' (distance, id) keys, read by every lane
    u32* occ = APART ? s_occ[wave] : own_lds + 192;
    float* ang = reinterpret_cast<float*>(own_lds + 192);
    const int k = A.k;
    const int nchunks = (A.d + 16 * KS - 1) / (16 * KS);

    for (int64_t p = (int64_t)blockIdx.x * FILTER_WAVES + wave; p < A.n; p += (int64_t)gridDim.x * FILTER_WAVES) {
        const float* xp = A.X + p * A.d;
        int m = 0;
        // ---- Collect ----
        const int32_t u = lane < k ? A.ids[p * k + lane] : -1;
        bool u_ok = u >= 0 && u < A.n && u != p;
        if (!TWO_HOPS) {
            // candidate l is entry l of the row; an entry that is no candidate (padding, p itself, an
            // id that an earlier entry lists already) keeps its place as a dead one and reads p's own row
            m = k;
            u32* tw = APART ? s_twin[wave] : own_lds + 64;
            for (int i = lane; i < 256; i += 64) tw[i] = FILTER_FREE;
            filter_wave_sync();
            {
                bool pending = u_ok;
                u32 h = ((u32)u * 0x9E3779B1u) >> 25;
                while (__ballot(pending)) {
                    if (pending) {
                        const u32 old = atomicCAS(tw + h, FILTER_FREE, (u32)u);
                        if (old == FILTER_FREE || old == (u32)u) { atomicMin(tw + 128 + h, (u32)lane); pending = false; }
                        else h = (h + 1) & 127u;
                    }
                }
                filter_wave_sync();
                u_ok = u_ok && tw[128 + h] == (u32)lane;
            }
            cid[lane] = u_ok ? u : (int)p;
            filter_wave_sync();
        } else {
            constexpr int SET_WORDS = ID_SET ? PLACES : PLACES / 2;          // (a free place is all ones in either set)
            int* queue = reinterpret_cast<int*>(own_lds + SET_WORDS);
            auto collect = [&](int Q, int id, bool active) __attribute__((always_inline)) {
                if (ID_SET) return filter_collect_ids<PLACES>(own_lds, queue, Q, id, active);
                return filter_collect<PLACES>(reinterpret_cast<unsigned short*>(own_lds), queue, queue + filter_queue_words(COLLECT), Q, id, active);
            };
            for (int i = lane; i < SET_WORDS / 4; i += 64) reinterpret_cast<uint4*>(own_lds)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
            filter_wave_sync();
            int Q = collect(0, u, u_ok);
            const int per = 64 / A.kp;
            const int my_row = lane / A.kp, r = lane - my_row * A.kp;
            for (int j0 = 0; j0 < k; j0 += LOADS * per) {
                int32_t w[LOADS];
#pragma unroll
                for (int t = 0; t < LOADS; ++t) {
                    const int j = j0 + t * per + my_row;
                    const bool on = my_row < per && j < k && r < k;
                    const int32_t uj = __shfl(u, on ? j : 0);
                    const bool uj_ok = __shfl((int)u_ok, on ? j : 0) != 0;
                    w[t] = (on && uj_ok) ? A.ids[(int64_t)uj * k + r] : -1;
                }
#pragma unroll
                for (int t = 0; t < LOADS; ++t) {
                    if (j0 + t * per >= k) break;                 // uniform
                    Q = collect(Q, w[t], w[t] >= 0 && w[t] < A.n && w[t] != p);
                }
            }
            filter_wave_sync();
            // distance to p of everything collected, 64 at a time; the 64 closest stay, in order
            u64 best = TG_EMPTY_KEY;
            for (int b0 = 0; b0 < Q; b0 += 64) {
                const int cnt = min(64, Q - b0);
                float dp[4] = {0.f, 0.f, 0.f, 0.f};
                for (int c = 0; c < nchunks; ++c) {
                    float4 X[4][KS];
                    filter_load_chunk<4, KS, FULL, VEC>(A, xp, queue + b0, cnt, c * 16 * KS, X, dp);
                }
                filter_reduce_quarters<4>(dp);
                const float own = filter_own<4>(dp, q4);
                u64 key = lane < cnt ? tg_key(own, (u32)queue[b0 + lane], 0u) : TG_EMPTY_KEY;
                key = tg_wave_sort(key);
                best = b0 == 0 ? key : tg_wave_merge_low(best, key);
            }
            m = min(min(Q, 64), A.cand_size);
            filter_wave_sync();                // the queue's words hold the candidates' rows from here on
            if (lane < m) cid[lane] = (int)tg_key_id(best);
            filter_wave_sync();
        }
        if (m > 16 * NG) m = 16 * NG;          // never true: the launcher sizes NG for the largest candidate set
        if (m == 0) {
            if (lane < A.d_out) A.out_ids[p * A.d_out + lane] = -1;
            if (A.out_deg && lane == 0) A.out_deg[p] = 0;
            filter_wave_sync();
            continue;
        }

        // ---- Filter: rows into registers, dis(p, c) and the Gram matrix of the candidates ----
        floatx4 acc[NG][NG];
#pragma unroll
        for (int i = 0; i < NG; ++i)
#pragma unroll
            for (int j = 0; j < NG; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        float dp[NG];
#pragma unroll
        for (int t = 0; t < NG; ++t) dp[t] = 0.f;
        const int groups = (m + 15) >> 4;
        for (int c = 0; c < nchunks; ++c) {
            float4 X[NG][KS];
            filter_load_chunk<NG, KS, FULL, VEC>(A, xp, cid, m, c * 16 * KS, X, dp);
            auto multiply = [&](int i, int j, int s) __attribute__((always_inline)) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(X[i][s].x, X[j][s].x, acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(X[i][s].y, X[j][s].y, acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(X[i][s].z, X[j][s].z, acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(X[i][s].w, X[j][s].w, acc[i][j], 0, 0, 0);
            };
            // Steps beyond the row hold nothing but zeros and are left out (500 000 x 16, k = 32: 767 -> 522 us, 100 000 x 101, k = 32: 594 -> 501),
            // so they come outermost: one test each.  Whole chunks take a tile at a time (300 000 x 64, k = 24: 488 us, steps outermost 500).
            // A tile's sum takes its columns in the same order either way.
            if (FULL) {
#pragma unroll
                for (int i = 0; i < NG; ++i) {
                    if (i >= groups) break;                           // uniform
#pragma unroll
                    for (int j = i; j < NG; ++j) {
                        if (j >= groups) break;
#pragma unroll
                        for (int s = 0; s < KS; ++s) multiply(i, j, s);
                    }
                }
            } else {
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    if (c * 16 * KS + 16 * s >= A.d) break;           // uniform
#pragma unroll
                    for (int i = 0; i < NG; ++i) {
                        if (i >= groups) break;
#pragma unroll
                        for (int j = i; j < NG; ++j) {
                            if (j >= groups) break;
                            multiply(i, j, s);
                        }
                    }
                }
            }
        }
        filter_reduce_quarters<NG>(dp);
        // accumulator register e of lane (r, q) in tile (i, j) is the product of rows 16 i + 4 q + e
        // and 16 j + r; the diagonal of tile (t, t) gives the squared norms
#pragma unroll
        for (int t = 0; t < NG; ++t) {
            const floatx4 a = acc[t][t];
            const float lo = (r16 & 1) ? a.y : a.x, hi = (r16 & 1) ? a.w : a.z;
            if (q4 == (r16 >> 2)) nrm[16 * t + r16] = (r16 & 2) ? hi : lo;
            if (q4 == 0) dpc[16 * t + r16] = dp[t];
        }
        if (RULE != FILTER_RULE_DISPERSION) {
            occ[lane] = 0u;
            occ[lane + 64] = 0u;
        }
        filter_wave_sync();
        if constexpr (RULE == FILTER_RULE_DISPERSION) {
            // Where no length is out of the ordinary the short square root and quotient serve.
            bool plain = true;
#pragma unroll
            for (int t = 0; t < NG; ++t) plain &= filter_plain_length(dp[t]);
            if (__ballot(!plain) == 0ull) filter_angles<NG, true>(acc, dp, nrm, dpc, groups, ang);
            else filter_angles<NG, false>(acc, dp, nrm, dpc, groups, ang);
        } else {
            // occ[C] = the candidates R that would occlude C: not dis(p, C) < alpha^2 dis(R, C), or an angle
            // at p of at most gamma (that relation is symmetric in R and C).  The lane holds its column's
            // four rows as a nibble; the mirrored pairs (rows and columns exchanged) of a tile off the
            // diagonal come out of ballots.
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                if (i >= groups) break;
                const float4 nR = *reinterpret_cast<const float4*>(nrm + 16 * i + 4 * q4);
                const float4 dR = *reinterpret_cast<const float4*>(dpc + 16 * i + 4 * q4);
#pragma unroll
                for (int j = i; j < NG; ++j) {
                    if (j >= groups) break;
                    const float nC = nrm[16 * j + r16];
                    const float dC = dp[j];
                    const floatx4 g = acc[i][j];
                    const float rc0 = (nR.x + nC) - 2.0f * g.x;        // dis(R, C)
                    const float rc1 = (nR.y + nC) - 2.0f * g.y;
                    const float rc2 = (nR.z + nC) - 2.0f * g.z;
                    const float rc3 = (nR.w + nC) - 2.0f * g.w;
                    bool o0, o1, o2, o3, m0, m1, m2, m3;               // R occludes C; C occludes R
                    if (ANGLE) {
                        const float t0 = (dR.x + dC) - rc0, t1 = (dR.y + dC) - rc1, t2 = (dR.z + dC) - rc2, t3 = (dR.w + dC) - rc3;
                        o0 = m0 = !((t0 < 0.0f) | (t0 * t0 < A.thr * (dR.x * dC)));
                        o1 = m1 = !((t1 < 0.0f) | (t1 * t1 < A.thr * (dR.y * dC)));
                        o2 = m2 = !((t2 < 0.0f) | (t2 * t2 < A.thr * (dR.z * dC)));
                        o3 = m3 = !((t3 < 0.0f) | (t3 * t3 < A.thr * (dR.w * dC)));
                    } else {
                        const float rhs0 = A.thr * rc0, rhs1 = A.thr * rc1, rhs2 = A.thr * rc2, rhs3 = A.thr * rc3;
                        o0 = !(dC < rhs0); o1 = !(dC < rhs1); o2 = !(dC < rhs2); o3 = !(dC < rhs3);
                        m0 = !(dR.x < rhs0); m1 = !(dR.y < rhs1); m2 = !(dR.z < rhs2); m3 = !(dR.w < rhs3);
                    }
                    const u32 nib = (u32)o0 | ((u32)o1 << 1) | ((u32)o2 << 2) | ((u32)o3 << 3);
                    atomicOr(occ + 2 * (16 * j + r16) + (i >> 1), nib << (16 * (i & 1) + 4 * q4));
                    if (j > i) {
                        const u64 b0 = __ballot(m0);
                        const u64 b1 = __ballot(m1);
                        const u64 b2 = __ballot(m2);
                        const u64 b3 = __ballot(m3);
                        if (r16 == 0) {
                            const int R = 16 * i + 4 * q4, sh = 16 * q4, word = j >> 1, up = 16 * (j & 1);
                            atomicOr(occ + 2 * (R + 0) + word, (u32)((b0 >> sh) & 0xFFFFull) << up);
                            atomicOr(occ + 2 * (R + 1) + word, (u32)((b1 >> sh) & 0xFFFFull) << up);
                            atomicOr(occ + 2 * (R + 2) + word, (u32)((b2 >> sh) & 0xFFFFull) << up);
                            atomicOr(occ + 2 * (R + 3) + word, (u32)((b3 >> sh) & 0xFFFFull) << up);
                        }
                    }
                }
            }
        }
        // before = the candidates in front of this lane's under (dis(p, c), id); dead entries have the
        // largest key and are in front of nothing
        const float own = filter_own<NG>(dp, q4);
        const int my_id = lane < m ? cid[lane] : 0;
        const bool dead = TWO_HOPS ? lane >= m : !u_ok;
        const u64 key = dead ? TG_EMPTY_KEY : tg_key(own, (u32)my_id, 0u);
        if (!APART) filter_wave_sync();        // (over the distances and norms)
        skey[lane] = key;
        filter_wave_sync();
        // one bit per other candidate, shifted in from below: after J steps candidate j sits at bit J - 1 - j
        u32 lt_lo = 0u, lt_hi = 0u;
        const int J = (m + 7) & ~7, J_lo = min(J, 32);
        for (int j0 = 0; j0 < J_lo; j0 += 8) {
#pragma unroll
            for (int j = 0; j < 8; ++j) lt_lo = lt_lo + lt_lo + (skey[j0 + j] < key ? 1u : 0u);
        }
        for (int j0 = 32; j0 < J; j0 += 8) {
#pragma unroll
            for (int j = 0; j < 8; ++j) lt_hi = lt_hi + lt_hi + (skey[j0 + j] < key ? 1u : 0u);
        }
        lt_lo = __brev(lt_lo) >> (32 - J_lo);
        lt_hi = J > 32 ? __brev(lt_hi) >> (64 - J) : 0u;
        const u64 live = ~__ballot(dead);
        const u64 before = (((u64)lt_hi << 32) | lt_lo) & live;
        filter_wave_sync();
        // ---- the serial rule as a fixed point ----
        // c is inserted iff no inserted candidate in front of it occludes it.  Starting from "all
        // inserted", every pass settles at least the next candidate in order, so the set stops
        // changing after at most m passes, and what it then holds obeys the rule.
        const bool in_cut = !dead && __popcll(before) < A.cand_size;       // the cut to cand_size counts candidates only
        if (RULE == FILTER_RULE_DISPERSION) {
            // ---- greedy insertion: one candidate per pass ----
            const int want = min(A.d_out, __popcll(__ballot(in_cut)));
            const u32 rnk = (u32)__popcll(before);                  // place among the candidates, nearest first
            float score = 0.0f;                                     // sum of the angles to the inserted nodes
            bool open = in_cut;
            int my_pos = -1;
            u64 pick = __ballot(in_cut && rnk == 0u);               // the nearest candidate goes first
            for (int it = 0; it < want && pick != 0ull; ++it) {
                const int r_new = __ffsll((unsigned long long)pick) - 1;
                if (lane == r_new) { my_pos = it; open = false; }
                if (it + 1 >= want) break;
                score += lane < 16 * NG ? ang[r_new * AS + lane] : 0.0f;
                // sums are no less than +0, so their bit patterns order them; + 1 puts every open lane above the rest
                const u32 sb = open ? __float_as_uint(score) + 1u : 0u;
                const u32 top = filter_wave_max(sb);
                const bool first = open && sb == top;
                pick = __ballot(first);
                if (__popcll(pick) > 1) {                           // (uniform) equal sums
                    const u32 near = 64u - filter_wave_max(first ? 64u - rnk : 0u);
                    pick = __ballot(first && rnk == near);
                }
            }
            if (my_pos >= 0) A.out_ids[p * A.d_out + my_pos] = my_id;
            if (lane >= want && lane < A.d_out) A.out_ids[p * A.d_out + lane] = -1;
            if (A.out_deg && lane == 0) A.out_deg[p] = want;
            filter_wave_sync();
            continue;
        }
        const u64 occ_by = (((u64)occ[2 * lane + 1] << 32) | occ[2 * lane]) & before;
        u64 K = __ballot(in_cut);
        for (int pass = 0; pass < 65; ++pass) {
            const u64 Kn = __ballot(in_cut && (occ_by & K) == 0ull);
            if (Kn == K) break;
            K = Kn;
        }
        // ---- Store: insertion order is the order of the candidates; the first d_out are in ----
        const bool kept = (K >> lane) & 1ull;
        const int pos = __popcll(K & before);
        const int deg = min(__popcll(K), A.d_out);
        if (kept && pos < A.d_out) A.out_ids[p * A.d_out + pos] = my_id;
        if (lane >= deg && lane < A.d_out) A.out_ids[p * A.d_out + lane] = -1;
        if (A.out_deg && lane == 0) A.out_deg[p] = deg;
        filter_wave_sync();
    }
}

template <class K>
static void filter_launch(K kernel, const FilterArgs& A, size_t shm, hipStream_t s)
{
    // more than 64 KB of dynamic LDS has to be asked for
    if (shm > 65536) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    int64_t wgs = (A.n + FILTER_WAVES - 1) / FILTER_WAVES;        // a wave per node; workgroups beyond the grid walk on
    if (wgs > FILTER_GRID) wgs = FILTER_GRID;
    hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(64 * FILTER_WAVES), shm, s, A);
}

template <int NG, int COLLECT, int RULE>
static void launch_filter(const FilterArgs& A, bool vec, hipStream_t s)
{
    const size_t shm = (size_t)FILTER_WAVES * filter_lds_words(NG, COLLECT, RULE) * sizeof(u32);
    // two row groups take their columns in chunks of 64, four in chunks of 32: few registers, so that
    // four (three) waves per SIMD cover each other's loads
    constexpr int KS = NG > 2 ? 2 : 4;
    const bool full = vec && (A.d % (16 * KS) == 0);         // no column guards needed
    if (full) filter_launch(filter_dist_kernel<NG, KS, true, true, COLLECT, RULE>, A, shm, s);
    else if (vec) filter_launch(filter_dist_kernel<NG, KS, false, true, COLLECT, RULE>, A, shm, s);
    else filter_launch(filter_dist_kernel<NG, KS, false, false, COLLECT, RULE>, A, shm, s);
}

template <int RULE>
static void launch_filter_rule(const FilterArgs& A, bool vec, int most, hipStream_t s)
{
    // the 2-hop collection measures 64 candidates at a time, which needs the four-group instance
    if (A.hops == 2 && A.k > 32) launch_filter<4, FILTER_TWO_HOPS_WIDE, RULE>(A, vec, s);
    else if (A.hops == 2) launch_filter<4, FILTER_TWO_HOPS, RULE>(A, vec, s);
    else if (most <= 32) launch_filter<2, FILTER_ONE_HOP, RULE>(A, vec, s);
    else if (most <= 48) launch_filter<3, FILTER_ONE_HOP, RULE>(A, vec, s);
    else launch_filter<4, FILTER_ONE_HOP, RULE>(A, vec, s);
}

void tg_launch_filter(const float* X, int64_t n, int d, const int32_t* ids, int k, int hops, int cand_size, int rule, float thr,
                      int d_out, int32_t* out_ids, int32_t* out_deg, hipStream_t s)
{
    FilterArgs A;
    A.X = X; A.n = n; A.d = d; A.ids = ids; A.k = k;
    A.kp = 1;
    while (A.kp < k) A.kp <<= 1;
    A.hops = hops; A.cand_size = cand_size;
    A.thr = thr;
    A.d_out = d_out; A.out_ids = out_ids; A.out_deg = out_deg;
    const bool vec = (d % 4 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0);
    const int most = hops == 1 ? k : (cand_size < 64 ? cand_size : 64);      // candidates that reach the filter
    if (rule == FILTER_RULE_DISPERSION) launch_filter_rule<FILTER_RULE_DISPERSION>(A, vec, most, s);
    else if (rule == FILTER_RULE_ANGLE) launch_filter_rule<FILTER_RULE_ANGLE>(A, vec, most, s);
    else launch_filter_rule<FILTER_RULE_DIST>(A, vec, most, s);
}
