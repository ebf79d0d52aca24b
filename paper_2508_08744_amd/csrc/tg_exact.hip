// Exhaustive exact k-NN of selected rows (the ground truth of the recall definition, section 7.1): the k
// rows with the smallest (distance, id), distances computed directly from the vectors in fp32.
//
// Measuring every pair that way is bound by the vector units (245 ms for 10 000 queries against 1M x 128, k = 32:
// 10.5 TFLOP/s; this search takes 3.9 ms).  Here the matrix cores bound every pair from both sides first, and only pairs that may be
// among the k nearest are measured directly:
//   w(q, r) = |r|^2 / 2 - <q, r>  (squared L2; -<q, r> for the inner product, the same on unit vectors for the
//   cosine) orders the rows for query q.  A tile of w is formed on the matrix cores, either from the rows
//   rounded to fp16 (scaled by a power of two and, for L2, centred) or from the fp32 rows; m(q, r) bounds
//   |w - the directly computed value| (ex_margin), so the pair matters only if w - m <= tau, tau being an
//   upper bound of the k-th smallest value.
//   1. tau comes from samples: all pairs with 2048 rows spread over X, the k-th smallest w + m of each query;
//      larger samples then go through the same scan with that tau (each level as much larger as EX_CAP places allow).
//   2. The scan of all rows appends the pairs that pass to a list of EX_CAP places per query (about k n / sample).
//   3. The list is cut by its own k-th smallest w + m, what is left is measured directly and sorted.
// A query whose list overflows (masses of equal distances, or rounding coarser than the distances) is measured
// against every row directly instead (exact_scan_kernel).
#include "tg_kernels.h"
#include "tg_device.h"
#include "tg_exact.h"

#include <cmath>

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));

#define EXQ 4            // direct measurement: queries per wave
#define EX_BUF 64        // direct measurement: buffered survivors per query
#define EX_FULL 0
#define EX_SAMPLE 1
#define EX_FIRST 2
#define EX_ALWAYS 3e38f  // -w of a row without a defined norm on the fp16 side (whose products are finite): above every threshold
#define EX_QUEUE 128     // pairs a wave of the scan collects before they go to the lists
#define EX_RT 128        // rows per tile of the scan
#define EX_CHUNK 128     // bytes of a row per step of the scan (64 fp16 or 32 fp32 columns)

__device__ inline void ex_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------------------
// Direct measurement of whole queries.  One wave serves EXQ queries over one slice of the rows: 16 lanes
// share a row, each row chunk is loaded once and used for all EXQ queries, survivors of the running
// threshold are appended to a small LDS buffer per query and folded into the wave-wide sorted top list by
// a sort + merge when the buffer fills.  Slices are merged by a second kernel.
// list / list_n: the queries to measure (indices into rows), or null for all nq of them.  How many a list holds is known on the device
// only, so the waves of the launch, as many as all nq queries would take, are shared out among the listed ones there.  (With
// the slices of a full batch ten listed queries of 10 000 against 1M x 128 kept twelve waves busy, each walking 250 000 rows: 132 ms for
// the call, 10.6 now; one of 1000 against 100 000 x 128: 1.84 ms, 0.82 now.)
// ---------------------------------------------------------------------------------------
#define EX_LIST_SLICES 512       // at most: one wave merges a query's slices one after another
#define EX_LIST_ROWS 256         // rows of a slice, at least
#define EX_LIST_WAVES 2048       // waves of a launch over a list, at least (64 listed queries against 50 000 x 96: 768 waves otherwise)
__device__ inline int ex_list_slices(int64_t waves, int64_t listed, int64_t nq, int64_t n, int k)
{
    int64_t s = waves / ((listed + EXQ - 1) / EXQ);
    const int64_t room = nq * EX_CAP / (listed * k);                  // partial holds nq x EX_CAP keys
    if (s > room) s = room;
    if (s > (n + EX_LIST_ROWS - 1) / EX_LIST_ROWS) s = (n + EX_LIST_ROWS - 1) / EX_LIST_ROWS;
    if (s > EX_LIST_SLICES) s = EX_LIST_SLICES;
    return s < 1 ? 1 : (int)s;
}
__global__ __launch_bounds__(256) void exact_scan_kernel(const float* __restrict__ X, int ld, const float* __restrict__ rnorm,
                                                                  int64_t n, int k, int metric, const int64_t* __restrict__ rows,
                                                                  int64_t nq, int64_t q_first, const u32* __restrict__ list,
                                                                  const u32* __restrict__ list_n, int nslices, u64* __restrict__ partial)
{
    extern __shared__ __align__(16) unsigned char ex_smem[];
    const int wave = threadIdx.x >> 6, lane = tg_lane();
    const int grp = lane >> 4, sub = lane & 15;
    int64_t qgroup = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    int slice = blockIdx.y;
    if (list) {
        const int64_t listed = (int64_t)*list_n;
        if (listed == 0) return;
        const int64_t waves = (int64_t)gridDim.x * gridDim.y * (blockDim.x >> 6), groups = (listed + EXQ - 1) / EXQ;
        const int64_t w = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (blockDim.x >> 6) + wave;
        nslices = ex_list_slices(waves, listed, nq, n, k);
        nq = listed;
        slice = (int)(w / groups);                                    // neighbouring waves read the same rows
        qgroup = w - slice * groups;
        if (slice >= nslices) return;
    }
    if (qgroup * EXQ >= nq) return;
    // per-wave LDS: EXQ query vectors, EXQ survivor buffers
    const size_t per_wave = (size_t)EXQ * ld * sizeof(float) + (size_t)EXQ * EX_BUF * sizeof(u64);
    float* qs = reinterpret_cast<float*>(ex_smem + wave * per_wave);
    u64* buf = reinterpret_cast<u64*>(ex_smem + wave * per_wave + (size_t)EXQ * ld * sizeof(float));

    int64_t qrow[EXQ];
    float qrn[EXQ];
#pragma unroll
    for (int q = 0; q < EXQ; ++q) {
        int64_t qi = qgroup * EXQ + q;
        if (list && qi < nq) qi = (int64_t)list[qi];
        const int64_t asked = qgroup * EXQ + q < nq ? (rows ? rows[q_first + qi] : q_first + qi) : -1;
        qrow[q] = asked < n ? asked : -1;               // a row index outside [0, n) is no query: its output stays empty
        qrn[q] = (metric == 2 && qrow[q] >= 0) ? rnorm[qrow[q]] : 1.0f;
        for (int col = lane * 4; col < ld; col += 256) {
            float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            if (qrow[q] >= 0) z = *reinterpret_cast<const float4*>(X + qrow[q] * (int64_t)ld + col);
            *reinterpret_cast<float4*>(qs + (size_t)q * ld + col) = z;
        }
    }
    ex_sync();

    u64 top[EXQ];       // ascending across lanes, lanes >= k hold TG_EMPTY_KEY
    u64 tau[EXQ];       // key of the k-th best so far
    int cnt[EXQ];
#pragma unroll
    for (int q = 0; q < EXQ; ++q) { top[q] = TG_EMPTY_KEY; tau[q] = TG_EMPTY_KEY; cnt[q] = 0; }

    const int64_t per_slice = (n + nslices - 1) / nslices;
    const int64_t r0 = (int64_t)slice * per_slice;
    const int64_t r1 = min(n, r0 + per_slice);
    for (int64_t base = r0; base < r1; base += 4) {
        const int64_t row = base + grp;
        const bool live = row < r1;
        float acc[EXQ];
#pragma unroll
        for (int q = 0; q < EXQ; ++q) acc[q] = 0.0f;
        if (live) {
            const float* y = X + row * (int64_t)ld;
            for (int col = sub * 4; col < ld; col += 64) {
                const float4 b = *reinterpret_cast<const float4*>(y + col);
#pragma unroll
                for (int q = 0; q < EXQ; ++q) {
                    const float4 a = *reinterpret_cast<const float4*>(qs + (size_t)q * ld + col);
                    if (metric == 0) {
                        const float t0 = a.x - b.x, t1 = a.y - b.y, t2 = a.z - b.z, t3 = a.w - b.w;
                        acc[q] += t0 * t0 + t1 * t1 + t2 * t2 + t3 * t3;
                    } else {
                        acc[q] += a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
                    }
                }
            }
        }
        const float rn_row = (metric == 2 && live) ? rnorm[row] : 1.0f;
#pragma unroll
        for (int q = 0; q < EXQ; ++q) {
            float s = acc[q];
            s += __shfl_xor(s, 1);
            s += __shfl_xor(s, 2);
            s += __shfl_xor(s, 4);
            s += __shfl_xor(s, 8);
            float dist = s;
            if (metric == 1) dist = -s;
            else if (metric == 2) dist = 1.0f - s * qrn[q] * rn_row;
            const u64 key = tg_key(dist, (u32)row, 0u);
            const bool pass = live && sub == 0 && qrow[q] >= 0 && row != qrow[q] && key < tau[q];
            const u64 m = __ballot(pass);
            if (m) {
                if (pass) buf[q * EX_BUF + cnt[q] + __popcll(m & tg_lanemask_lt())] = key;
                cnt[q] += __popcll(m);
                if (cnt[q] > EX_BUF - 4) {
                    ex_sync();
                    u64 c = lane < cnt[q] ? buf[q * EX_BUF + lane] : TG_EMPTY_KEY;
                    ex_sync();
                    top[q] = tg_wave_merge_low(top[q], tg_wave_sort(c));
                    if (lane >= k) top[q] = TG_EMPTY_KEY;
                    tau[q] = tg_shfl64(top[q], k - 1);
                    cnt[q] = 0;
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < EXQ; ++q) {
        ex_sync();
        u64 c = lane < cnt[q] ? buf[q * EX_BUF + lane] : TG_EMPTY_KEY;
        top[q] = tg_wave_merge_low(top[q], tg_wave_sort(c));
        const int64_t qi = qgroup * EXQ + q;
        if (qi < nq && lane < k) partial[(qi * nslices + slice) * k + lane] = top[q];
    }
}

__device__ inline void ex_write_row(u64 top, int k, int64_t qi, int32_t* __restrict__ out_ids, float* __restrict__ out_dist)
{
    const int lane = tg_lane();
    if (lane < k) {
        const bool none = top == TG_EMPTY_KEY;
        out_ids[qi * k + lane] = none ? -1 : (int32_t)tg_key_id(top);
        if (out_dist) out_dist[qi * k + lane] = none ? __builtin_inff() : tg_key_dist(top);
    }
}
__global__ __launch_bounds__(256) void exact_merge_kernel(const u64* __restrict__ partial, int64_t nq, int k, int nslices,
                                                          const u32* __restrict__ list, const u32* __restrict__ list_n, int64_t waves, int64_t n,
                                                          int32_t* __restrict__ out_ids, float* __restrict__ out_dist)
{
    const int lane = tg_lane();
    const int64_t qi = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (list) {
        const int64_t listed = (int64_t)*list_n;
        if (listed == 0) return;
        nslices = ex_list_slices(waves, listed, nq, n, k);
        nq = listed;
    }
    if (qi >= nq) return;
    u64 top = TG_EMPTY_KEY;
    for (int s = 0; s < nslices; ++s) {
        u64 c = lane < k ? partial[(qi * nslices + s) * k + lane] : TG_EMPTY_KEY;
        top = tg_wave_merge_low(top, c);
        if (lane >= k) top = TG_EMPTY_KEY;
    }
    ex_write_row(top, k, list ? (int64_t)list[qi] : qi, out_ids, out_dist);
}

// partial must hold nq * nslices * k keys (with a list: nq * EX_CAP); returns the slice count used for (n, nq)
int tg_exact_slices(int64_t n, int64_t nq)
{
    const int64_t groups = (nq + EXQ - 1) / EXQ;
    int64_t s = (8192 + groups - 1) / groups;
    if (s > 64) s = 64;
    if (s < 1) s = 1;
    while (s > 1 && (n + s - 1) / s < 1024) --s;
    return (int)s;
}

void tg_launch_exact_knn(const float* X, int ld, const float* rnorm, int64_t n, int k, int metric, const int64_t* rows, int64_t nq,
                         int64_t q_first, const u32* list, const u32* list_n, int32_t* out_ids, float* out_dist, u64* partial,
                         int nslices, hipStream_t s)
{
    const int64_t groups = (nq + EXQ - 1) / EXQ;
    const int waves = ld <= 1024 ? 4 : ld <= 2048 ? 2 : 1;     // independent waves per workgroup, bounded by LDS
    const size_t shm = (size_t)waves * ((size_t)EXQ * ld * sizeof(float) + (size_t)EXQ * EX_BUF * sizeof(u64));
    tg_allow_lds<exact_scan_kernel>(160 * 1024 - 256);
    const int64_t across = (groups + waves - 1) / waves;
    if (list && across * waves * nslices < EX_LIST_WAVES) nslices = (int)((EX_LIST_WAVES / waves + across - 1) / across);
    const dim3 grid((unsigned)across, (unsigned)nslices);
    hipLaunchKernelGGL(exact_scan_kernel, grid, dim3(64 * waves), shm, s, X, ld, rnorm, n, k, metric, rows, nq, q_first, list, list_n, nslices,
                       partial);
    hipLaunchKernelGGL(exact_merge_kernel, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, s, partial, nq, k, nslices, list, list_n,
                       (int64_t)grid.x * grid.y * waves, n, out_ids, out_dist);
}

// ---------------------------------------------------------------------------------------
// fp16 rows.  ex_stat_kernel looks at up to 512 rows spread over X: the mean of every column (L2: the
// centre, any vector would do) and the largest |x - centre| of those rows, from which ex_half_kernel takes the
// power of two that brings it to 128..256, where fp16 has 2^8 of room above and 2^21 below.  A value that
// leaves the range all the same is clipped: what a row loses in any way is in its residual norm, which
// the margin is made of.
// ---------------------------------------------------------------------------------------
#define EX_STAT_ROWS 512
__global__ __launch_bounds__(1024) void ex_stat_kernel(const float* __restrict__ X, int64_t n, int d, int ld, int centre_it, float* centre,
                                                       u32* top_bits)
{
    __shared__ float s_part[16][64];
    const int c = (int)blockIdx.x * 64 + (threadIdx.x & 63), g = threadIdx.x >> 6;
    const int64_t m = n < EX_STAT_ROWS ? n : EX_STAT_ROWS;
    const int64_t apart = n / m;
    const int cc = c < d ? c : 0;
    float v[EX_STAT_ROWS / 16];
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < EX_STAT_ROWS / 16; ++i) {
        const int64_t j = g + 16 * i;
        v[i] = j < m ? X[j * apart * ld + cc] : 0.0f;
        sum += v[i];
    }
    s_part[g][threadIdx.x & 63] = sum;
    __syncthreads();
    float mean = 0.0f;
    if (centre_it) {
        for (int i = 0; i < 16; ++i) mean += s_part[i][threadIdx.x & 63];
        mean /= (float)m;
        if (!(fabsf(mean) < 1e30f)) mean = 0.0f;
    }
    float top = 0.0f;
#pragma unroll
    for (int i = 0; i < EX_STAT_ROWS / 16; ++i)
        if (g + 16 * i < m) top = fmaxf(top, fabsf(v[i] - mean));
    if (c >= d) { mean = 0.0f; top = 0.0f; }
    if (g == 0 && c < ld) centre[c] = mean;
    for (int o = 1; o < 64; o <<= 1) top = fmaxf(top, __shfl_xor(top, o));
    if ((threadIdx.x & 63) == 0 && top < __builtin_inff()) atomicMax(top_bits, __float_as_uint(top));
}
__device__ inline float ex_scale(u32 top_bits, int metric)
{
    if (metric == 2) return 256.0f;                          // unit rows
    const int e = (int)(top_bits >> 23);                     // 2^(e - 127) <= top < 2^(e - 126)
    return e < 20 || e > 234 ? 1.0f : __uint_as_float((u32)(127 + 7 - (e - 127)) << 23);
}
// One row per 16 lanes: the fp16 row (zero beyond column d), its squared norm and the norm of what rounding took
// from it (both in the scaled units), and for the cosine 1 / |x| as norms_kernel forms it.
__global__ __launch_bounds__(256) void ex_half_kernel(const float* __restrict__ X, int64_t n, int d, int ld, int metric,
                                                      const float* __restrict__ centre, const u32* __restrict__ top_bits,
                                                      uint16_t* __restrict__ Xh, int ldh, float* __restrict__ rn, float* __restrict__ er,
                                                      float* __restrict__ rnorm)
{
    const int sub = threadIdx.x & 15;
    const float scale = ex_scale(*top_bits, metric);
    for (int64_t row = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); row < n; row += (int64_t)gridDim.x * 16) {
        const float* x = X + row * (int64_t)ld;
        float s = scale;
        if (metric == 2) {
            float acc = 0.0f;
            for (int c = sub * 4; c < ld; c += 64) {
                const float4 v = *reinterpret_cast<const float4*>(x + c);
                acc += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
            }
            acc += __shfl_xor(acc, 1);
            acc += __shfl_xor(acc, 2);
            acc += __shfl_xor(acc, 4);
            acc += __shfl_xor(acc, 8);
            const float r = 1.0f / sqrtf(acc);
            if (sub == 0) rnorm[row] = r;
            s = scale * r;
        }
        float nn = 0.0f, ee = 0.0f;
        for (int c = sub * 4; c < ldh; c += 64) {
            halfx4 h = {};
            if (c < ld) {
                const float4 v = *reinterpret_cast<const float4*>(x + c);
                const float4 m = metric == 0 ? *reinterpret_cast<const float4*>(centre + c) : make_float4(0.f, 0.f, 0.f, 0.f);
                const float e[4] = {(v.x - m.x) * s, (v.y - m.y) * s, (v.z - m.z) * s, (v.w - m.w) * s};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float t = fminf(65504.0f, fmaxf(-65504.0f, e[i]));
                    if (fabsf(t) < 6.103515625e-05f) t = 0.0f;           // no subnormal fp16 numbers: whether the matrix unit keeps them is not relied on
                    h[i] = (_Float16)t;
                    const float back = (float)h[i];
                    nn = fmaf(e[i], e[i], nn);
                    ee = fmaf(e[i] - back, e[i] - back, ee);
                }
            }
            *reinterpret_cast<halfx4*>(Xh + row * (int64_t)ldh + c) = h;
        }
        nn += __shfl_xor(nn, 1);
        nn += __shfl_xor(nn, 2);
        nn += __shfl_xor(nn, 4);
        nn += __shfl_xor(nn, 8);
        ee += __shfl_xor(ee, 1);
        ee += __shfl_xor(ee, 2);
        ee += __shfl_xor(ee, 4);
        ee += __shfl_xor(ee, 8);
        if (sub == 0) {
            rn[row] = nn;
            er[row] = sqrtf(ee) * 1.001f;
        }
    }
}

// ---------------------------------------------------------------------------------------
// The queries of this batch, packed: rows of whole chunks, zero padded (so that what the scan reads beyond the
// end of a row of X counts for nothing), zero rows up to a multiple of the tile.  One wave per query.
// qmeta: |q|, residual norm, squared norm; qrow: its row of X (-1: no query); the query's counter is cleared.
// Where the scan is on the fp32 rows a query's norm is formed here, as norms_kernel forms it, and the workgroups behind those of the
// queries form the norms of all rows (first batch): one launch, not two (64 queries against 50 000 x 96: 54.1 -> 51.2 us).
// ---------------------------------------------------------------------------------------
// |x|^2 of a row by each 16 lanes of a wave
__device__ inline float ex_row_norm(const float* __restrict__ x, int ld)
{
    float acc = 0.0f;
    for (int c = (threadIdx.x & 15) * 4; c < ld; c += 64) {
        const float4 v = *reinterpret_cast<const float4*>(x + c);
        acc += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
    acc += __shfl_xor(acc, 1);
    acc += __shfl_xor(acc, 2);
    acc += __shfl_xor(acc, 4);
    acc += __shfl_xor(acc, 8);
    return acc;
}
__global__ __launch_bounds__(256) void ex_query_kernel(ExScanArgs a, int f16, const int64_t* __restrict__ rows, int64_t q_first, int64_t nqpad,
                                                       int ld, float* __restrict__ nrm, float* __restrict__ rnorm)
{
    const int lane = tg_lane();
    if ((int64_t)blockIdx.x * 4 >= nqpad) {
        const int64_t groups = gridDim.x - nqpad / 4, group = blockIdx.x - nqpad / 4;
        for (int64_t row = group * 16 + (threadIdx.x >> 4); row < a.n; row += groups * 16) {
            const float acc = ex_row_norm(reinterpret_cast<const float*>(a.rows) + row * (int64_t)ld, ld);
            if ((threadIdx.x & 15) == 0) {
                nrm[row] = acc;
                if (a.metric == 2) rnorm[row] = 1.0f / sqrtf(acc);
            }
        }
        return;
    }
    const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (q == 0 && lane == 0) *a.fb_n = 0u;
    int64_t row = -1;
    if (q < a.nq) row = rows ? rows[q_first + q] : q_first + q;
    if (row >= a.n || row < 0) row = -1;
    float qn = 0.0f;
    if (row >= 0) qn = f16 ? a.rn[row] : ex_row_norm(reinterpret_cast<const float*>(a.rows) + row * (int64_t)ld, ld);
    const int words = a.qbytes >> 4;
    const float s = (!f16 && a.metric == 2 && row >= 0) ? 1.0f / sqrtf(qn) : 1.0f;
    for (int c = lane; c < words; c += 64) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (row >= 0 && c * 16 < a.rowbytes) {
            v = *reinterpret_cast<const uint4*>(a.rows + row * (int64_t)a.rowbytes + c * 16);
            if (!f16 && a.metric == 2) {
                v.x = __float_as_uint(__uint_as_float(v.x) * s);
                v.y = __float_as_uint(__uint_as_float(v.y) * s);
                v.z = __float_as_uint(__uint_as_float(v.z) * s);
                v.w = __float_as_uint(__uint_as_float(v.w) * s);
            }
        }
        *reinterpret_cast<uint4*>(a.Q + q * (int64_t)a.qbytes + c * 16) = v;
    }
    if (lane == 0) {
        if (!f16 && a.metric == 2 && row >= 0) qn = 1.0f;
        a.qmeta[q] = make_float4(sqrtf(qn), row >= 0 && a.er ? a.er[row] : 0.0f, qn, 0.0f);
        a.qrow[q] = (int32_t)row;
        if (q < a.nq) a.cnt[q * EX_CSTRIDE] = 0u;
    }
}

// Bound of |w(q, r) - (the directly computed distance, in the same units)|, for |r| <= R and a residual of at most E:
// |q| E + (R + E) e_q for what rounding to fp16 took; (2 d + 32) 2^-24 times both squared norms for every fp32
// rounding on either side (products and their sum here: at most d + 3 half ulps of |q| |r| + |r|^2 / 2; the direct
// form: d / 16 + 14 of twice the squared norms).
__device__ inline float ex_margin(float q, float eq, float kq, float R, float E, float c1)
{
    return fmaf(q, E, fmaf(eq, R + E, fmaf(c1 * R, R, kq)));
}
// Row number of the j-th visited row: j itself in the full scan, j * step mod n (step coprime to n) in a sample.  The quotient
// comes from a double (j, step, n < 2^30: it is off by one at most).
template <bool SAMPLE>
__device__ inline u32 ex_row(const ExScanArgs& a, u32 j)
{
    if (!SAMPLE) return j;
    const u32 n = (u32)a.n;
    const u64 quo = (u64)((double)j * a.step_by_n);
    const int64_t rem = (int64_t)((u64)j * a.step - quo * n);
    return (u32)(rem < 0 ? rem + n : rem >= (int64_t)n ? rem - n : rem);
}

// ---------------------------------------------------------------------------------------
// The scan.  A workgroup takes QT queries against a slice of the visited rows, 128 rows per tile, 128 bytes of
// every row per step.  Eight waves: QT = 128: each 64 queries x 32 rows; QT = 64: each 64 queries x 16 rows.  Rows
// and queries are staged in LDS, a row's eight 16-byte pieces permuted by (row mod 8) so that neither the
// stores nor the operand reads meet in a bank; while a step is multiplied, the next one's rows travel.
// Queries that fit (RES: at most 256 bytes each) stay in LDS for the whole slice, longer ones come again with
// every tile.  Lane (r, q) of a 16 x 16 tile holds query r against rows 4 q .. 4 q + 3: the query's threshold
// is a register, and -|r|^2 / 2 is where the accumulator starts, so a tile costs three maxima, one compare and a
// ballot unless something passes.  MODE: all rows (EX_FULL), a sample (EX_SAMPLE), or the first sample, of which everything
// is kept (EX_FIRST: place = number of the visit).
// What bounds it is the vector work of a tile (bounds, maxima, the pairs that pass; about as long as its matrix instructions twice over) and
// waits for rows, which sixteen waves on a CU cover better than eight with twice the tile each: 1M x 128 against 10 000 queries, fp16 (which
// ex_scan_wave_kernel takes now): 7.15 -> 5.0 ms; 50 000 x 96 against 64 (fp32): 66 -> 62 us.  Where the queries come again (not RES, 128 of them) three to
// seven registers spill at four waves per SIMD, which still is the better side: whole searches with four waves a workgroup / eight / eight, two per SIMD
// and no spill: 200 000 x 960 against 2000 (fp16): 2.33 / 2.19 / 2.81 ms; 200 000 x 200 against 4000: 1.83 / 1.54 / 2.08; 1M x 96 against 100 (fp32): 543 / 531 / 571 us.
// ---------------------------------------------------------------------------------------
#define EX_WAVES 8
template <bool F16, int QT, bool RES, int MODE>
__global__ __launch_bounds__(64 * EX_WAVES, 4) void ex_scan_kernel(ExScanArgs a)
{
    constexpr int WAVES = EX_WAVES, THREADS = 64 * WAVES;
    constexpr bool ALL = MODE == EX_FIRST;
    constexpr bool SAMPLE = MODE != EX_FULL;
    extern __shared__ __align__(16) unsigned char ex_lds[];
    __shared__ __align__(16) float s_c0[2][EX_RT], s_c1[2][EX_RT];      // -|r|^2 / 2 (or 0; -inf past the end) and, fp32 cosine, 1 / |r|
    __shared__ float s_E[2][EX_RT / 16], s_R[2][EX_RT / 16];            // largest residual and norm of every 16 rows
    __shared__ u64 s_queue[ALL ? 1 : WAVES][EX_QUEUE];                      // pairs on their way to the lists: ordered w << 32 | row of X ...
    __shared__ u32 s_qof[ALL ? 1 : WAVES][EX_QUEUE];                        // ... and the query within the tile
    __shared__ u32 s_full[QT];                                          // the query's list is full: it is measured another way
    __shared__ u32 s_row[ALL ? 2 : 1][ALL ? EX_RT : 1];                 // the rows' numbers in X
    constexpr int WQ = QT / 64;                                         // waves side by side over the queries
    constexpr int WI = EX_RT / 16 / (WAVES / WQ);                       // 16-row tiles per wave
    constexpr int RP = THREADS / 8;                                     // rows whose step the threads fetch at once, a 16-byte piece each
    constexpr int BP = EX_RT / RP, AP = QT / RP;                        // pieces of a step of the rows and of the queries per thread
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int r16 = lane & 15, q4 = lane >> 4;
    const int wq = wave % WQ, wr = wave / WQ;
    const int qb = (int)(blockIdx.x % (unsigned)a.nqb);
    const int slice = (int)(blockIdx.x / (unsigned)a.nqb);
    const int tiles = (int)((a.nvisit + EX_RT - 1) / EX_RT);
    const int per = (tiles + a.nslices - 1) / a.nslices;
    const int t0 = slice * per, t1 = min(tiles, t0 + per);
    if (t0 >= t1) return;
    const int nch = a.qbytes / EX_CHUNK;
    unsigned char* lA = ex_lds;                                         // RES: nch steps, else two
    unsigned char* lB = ex_lds + (size_t)(RES ? nch : 2) * QT * EX_CHUNK;
    const unsigned char* qbase = a.Q + (int64_t)qb * QT * a.qbytes;

    // this lane's queries
    float ntau[4], qa[4], qe[4], kq[4];
    int qself[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t q = (int64_t)qb * QT + wq * 64 + 16 * j + r16;
        const float4 m = a.qmeta[q];
        qself[j] = a.qrow[q];
        qa[j] = m.x; qe[j] = m.y; kq[j] = a.c1 * m.z;
        ntau[j] = -__builtin_inff();
        if (F16 && !(m.z < __builtin_inff())) qa[j] = qe[j] = kq[j] = 0.0f;    // a query without a defined norm: everything passes
        else if (!ALL) ntau[j] = -a.tau[q];
        if (q >= a.nq || qself[j] < 0) ntau[j] = __builtin_inff();      // no query: nothing passes
    }

    floatx4 preB[BP], preA[AP];
    float pre_rn = 0.0f, pre_er = 0.0f, pre_c1 = 1.0f;
    u32 pre_row = 0u;
    const unsigned char* rp[BP];
    const int nvisit = (int)a.nvisit;
    const int piece = tid & 7, prow = tid >> 3;
    auto fetch = [&](int t, int ch) __attribute__((always_inline)) {
        if (ch == 0) {
#pragma unroll
            for (int it = 0; it < BP; ++it) rp[it] = a.rows + (int64_t)ex_row<SAMPLE>(a, (u32)min(t * EX_RT + prow + RP * it, nvisit - 1)) * a.rowbytes;
            if (tid < EX_RT) {
                const u32 r = ex_row<SAMPLE>(a, (u32)min(t * EX_RT + tid, nvisit - 1));
                pre_row = r;
                pre_rn = a.rn[r];
                pre_er = F16 ? a.er[r] : 0.0f;
                if (!F16 && a.metric == 2) pre_c1 = a.rnorm[r];
            }
        }
        const int off = ch * EX_CHUNK + piece * 16;
        const int offc = off < a.rowbytes ? off : 0;                    // beyond the row: any of its own values (the query is zero there)
#pragma unroll
        for (int it = 0; it < BP; ++it) preB[it] = *reinterpret_cast<const floatx4*>(rp[it] + offc);
        if (!RES) {
#pragma unroll
            for (int it = 0; it < AP; ++it) preA[it] = *reinterpret_cast<const floatx4*>(qbase + (int64_t)(prow + RP * it) * a.qbytes + off);
        }
    };
    auto store = [&](int t, int ch, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < BP; ++it) {
            const int row = prow + RP * it;
            *reinterpret_cast<floatx4*>(lB + (size_t)buf * EX_RT * EX_CHUNK + row * EX_CHUNK + ((piece ^ (row & 7)) << 4)) = preB[it];
        }
        if (!RES) {
#pragma unroll
            for (int it = 0; it < AP; ++it) {
                const int row = prow + RP * it;
                *reinterpret_cast<floatx4*>(lA + (size_t)buf * QT * EX_CHUNK + row * EX_CHUNK + ((piece ^ (row & 7)) << 4)) = preA[it];
            }
        }
        if (ch == 0 && tid < EX_RT) {
            const int par = (t - t0) & 1;
            const bool real = t * EX_RT + tid < nvisit;
            const bool undefined = !(pre_rn < __builtin_inff()) || !(pre_c1 < __builtin_inff());
            s_c0[par][tid] = !real ? -__builtin_inff() : F16 && undefined ? EX_ALWAYS : a.metric == 0 ? -0.5f * pre_rn : 0.0f;
            if (!F16) s_c1[par][tid] = pre_c1;
            if (ALL) s_row[ALL ? par : 0][ALL ? tid : 0] = pre_row;
            float R = (!F16 && a.metric == 2) ? 1.0f : sqrtf(pre_rn), E = pre_er;
            // A row without a defined norm is bounded by nothing.  fp32: nor are its neighbours in the tile then (a maximum alone would pass
            // over a NaN).  fp16: EX_ALWAYS takes it past any threshold, and its neighbours keep theirs (with an infinite norm among the
            // maxima a threshold would be 0 x infinity for queries that rounding took nothing from: no number, and no pair passes that).
            if (undefined) R = F16 ? 0.0f : __builtin_inff();
            if (F16 && undefined) E = 0.0f;
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) {
                R = fmaxf(R, __shfl_xor(R, o));
                E = fmaxf(E, __shfl_xor(E, o));
            }
            if ((tid & 15) == 0) { s_R[par][tid >> 4] = R * 1.0001f; s_E[par][tid >> 4] = E; }
        }
    };

    if (RES) {
        for (int e = tid; e < QT * nch * 8; e += THREADS) {
            const int c = e & 7, row = (e >> 3) % QT, ch = (e >> 3) / QT;
            *reinterpret_cast<float4*>(lA + ((size_t)ch * QT + row) * EX_CHUNK + ((c ^ (row & 7)) << 4)) =
                *reinterpret_cast<const float4*>(qbase + (int64_t)row * a.qbytes + ch * EX_CHUNK + c * 16);
        }
    }
    if (!ALL) {
        for (int i = tid; i < QT; i += THREADS) s_full[i] = 0u;             // (seen by everyone behind the first barrier of the loop)
    }
    // Pairs that pass wait in a queue of the wave's own and go to the lists up to 64 at a time: their places come from
    // one atomic per pair, and a wave that waited for those pair by pair did little else (the scan of 1M x 128 for 10 000
    // queries took 13.4 ms with its sample so, 11.3 with the queue).
    int nqueue = 0;
    auto flush = [&]() {
        ex_sync();
        for (int b = 0; b < nqueue; b += 64) {
            if (b + lane < nqueue) {
                const u32 ql = s_qof[wave][b + lane];
                const int64_t q = (int64_t)qb * QT + ql;
                const u32 pos = atomicAdd(a.cnt + q * EX_CSTRIDE, 1u);
                if (pos < EX_CAP) a.buf[q * EX_CAP + pos] = s_queue[wave][b + lane];
                else s_full[ql] = 1u;
            }
        }
        nqueue = 0;
        ex_sync();
    };
    floatx4 acc[WI][4];
    fetch(t0, 0);
    int buf = 0;
    for (int t = t0; t < t1; ++t) {
        const int par = (t - t0) & 1;
        for (int ch = 0; ch < nch; ++ch) {
            store(t, ch, buf);
            __syncthreads();
            {
                const bool more = ch + 1 < nch;
                if (more || t + 1 < t1) fetch(more ? t : t + 1, more ? ch + 1 : 0);
            }
            if (ch == 0) {
#pragma unroll
                for (int i = 0; i < WI; ++i) {
                    floatx4 c0 = (floatx4){0.f, 0.f, 0.f, 0.f};
                    if (F16) c0 = *reinterpret_cast<const floatx4*>(&s_c0[par][wr * 16 * WI + 16 * i + 4 * q4]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] = c0;
                }
            }
            const unsigned char* pB = lB + (size_t)buf * EX_RT * EX_CHUNK + (size_t)wr * 16 * WI * EX_CHUNK;
            const unsigned char* pA = lA + (size_t)(RES ? ch : buf) * QT * EX_CHUNK + (size_t)wq * 64 * EX_CHUNK;
            const int ksteps = a.rowbytes - ch * EX_CHUNK > 64 ? 2 : 1;
            for (int ks = 0; ks < ksteps; ++ks) {
                const int slot = ((4 * ks + q4) ^ (r16 & 7)) << 4;
                float4 fr[WI], fq[4];
#pragma unroll
                for (int i = 0; i < WI; ++i) fr[i] = *reinterpret_cast<const float4*>(pB + (16 * i + r16) * EX_CHUNK + slot);
#pragma unroll
                for (int j = 0; j < 4; ++j) fq[j] = *reinterpret_cast<const float4*>(pA + (16 * j + r16) * EX_CHUNK + slot);
#pragma unroll
                for (int i = 0; i < WI; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (F16) {
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, fr[i]), __builtin_bit_cast(halfx8, fq[j]),
                                                                                acc[i][j], 0, 0, 0);
                        } else {
                            // the same permutation of the columns on both sides: the sum is the full dot product
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fr[i].x, fq[j].x, acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fr[i].y, fq[j].y, acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fr[i].z, fq[j].z, acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fr[i].w, fq[j].w, acc[i][j], 0, 0, 0);
                        }
                    }
            }
            buf ^= 1;
        }
        // -w of every pair of the tile against -tau - m: which of the wave's 16 x 16 tiles hold a pair that passes ...
        u32 hits = 0u;
        auto threshold = [&](int i, int j) {
            const float R = s_R[par][wr * WI + i], E = s_E[par][wr * WI + i];
            return ntau[j] - ex_margin(qa[j], qe[j], kq[j], R, E, a.c1);
        };
        auto value = [&](int i, int j) {
            floatx4 v = acc[i][j];
            if (!F16) {
                const floatx4 c0 = *reinterpret_cast<const floatx4*>(&s_c0[par][16 * (wr * WI + i) + 4 * q4]);
                const floatx4 c1 = *reinterpret_cast<const floatx4*>(&s_c1[par][16 * (wr * WI + i) + 4 * q4]);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = fmaf(v[e], c1[e], c0[e]);
            }
            return v;
        };
        if (ALL) {
            // every value is kept, at the number of its visit
#pragma unroll
            for (int i = 0; i < WI; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const floatx4 v = value(i, j);
                    const int at = 16 * (wr * WI + i) + 4 * q4;
                    if (ntau[j] > 0.0f) continue;                               // no query
                    u64* out = a.buf + ((int64_t)qb * QT + wq * 64 + 16 * j + r16) * EX_CAP + t * EX_RT + at;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const u32 row = s_row[ALL ? par : 0][ALL ? at + e : 0];
                        if (t * EX_RT + at + e < nvisit) out[e] = row == (u32)qself[j] ? TG_EMPTY_KEY : ((u64)tg_ord(-v[e]) << 32) | row;
                    }
                }
            continue;
        }
#pragma unroll
        for (int i = 0; i < WI; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const floatx4 v = value(i, j);
                const float best = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
                hits |= __ballot(F16 ? best >= threshold(i, j) : !(best < threshold(i, j))) != 0ull ? 1u << (4 * i + j) : 0u;
            }
        // ... and those tiles one by one (one copy of the code for all of them: unrolled it drowned the loop above)
        while (hits) {
            const int at = __builtin_amdgcn_readfirstlane(__ffs(hits) - 1);
            hits &= hits - 1u;
            floatx4 v = (floatx4){0.f, 0.f, 0.f, 0.f};
            float thr = 0.0f;
            int self = -1;
            bool live = false;                                              // a query whose list still has places
#pragma unroll
            for (int i = 0; i < WI; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (at == 4 * i + j) { v = value(i, j); thr = threshold(i, j); self = qself[j]; live = ntau[j] < __builtin_inff(); }
            const int ql = wq * 64 + 16 * (at & 3) + r16;
#pragma unroll 1
            for (int e = 0; e < 4; ++e) {
                const float ve = e == 0 ? v[0] : e == 1 ? v[1] : e == 2 ? v[2] : v[3];
                const int jv = t * EX_RT + 16 * (wr * WI + (at >> 2)) + 4 * q4 + e;
                const u64 key_hi = (u64)tg_ord(-ve) << 32;
                bool pass = (F16 ? ve >= thr : !(ve < thr) && live) && jv < nvisit;     // fp32: an undefined bound rules nothing out
                if (__ballot(pass) == 0ull) continue;
                const u32 row = ex_row<SAMPLE>(a, (u32)jv);
                pass = pass && row != (u32)self;
                const u64 m = __ballot(pass);
                const int more = __popcll(m);
                if (nqueue + more > EX_QUEUE) flush();
                if (pass) {
                    const int put = nqueue + __popcll(m & tg_lanemask_lt());
                    s_queue[wave][put] = key_hi | row;
                    s_qof[wave][put] = (u32)ql;
                }
                nqueue += more;
            }
        }
        if (!ALL) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (s_full[wq * 64 + 16 * j + r16]) ntau[j] = __builtin_inff();
        }
    }
    if (!ALL) flush();
}

// ---------------------------------------------------------------------------------------
// The scan of fp16 rows of at most 256 bytes, all rows (EX_FULL) or a sample of them.  A wave keeps 64 queries in registers, in matrix
// operand layout (lane (r, q) holds piece 4 s + q of query 16 j + r: 16 KS registers), and meets one group of 16 rows after the other;
// only the rows go through LDS, 64 at a time in two buffers, a row's 16-byte pieces permuted so that neither the stores nor the
// operand reads meet in a bank.  The four waves of a workgroup stand side by side over the queries, or over two or four shares of the
// rows of a tile where there are fewer queries (a.wqs: waves over the queries).
// A group of 16 x 64 pairs costs 4 KS matrix instructions, KS operand reads, and on the vector units two maxima and a compare for each
// 16 queries: the thresholds are taken for the 64 rows of a tile (the bound of a pair is made of the largest norm and the largest
// residual among them: a little looser than a row's own, no pair is lost), or for each group where those of the groups differ (EXG_UNEVEN): one row
// far from the others would loosen the bounds of 63, pairs pass that need not, lists fill up and their queries are measured directly.  300 000 x 128
// against 2000, one row of a hundred times the norm in every 64: 4.34 ms by the tile, 1.09 by the group (1.24 in ex_scan_kernel, by 16 rows); 500 000 x 96
// against 4000, norms spread over e^+-1: 7.3, 1.98 (2.55).  By the group always this kernel takes 3.1 ms for the
// 2.83 below, with the choice 2.83 still: the maxima by DPP and in scalar registers pay for it.
// Pairs that pass wait in a queue of the wave's own and go to the lists up to 64 at a time and more (see ex_scan_kernel).
// 1M x 128 against 10 000 queries: 5.75 ms with the queries in LDS and each row read for 128 of them, 0.73 its sample; now 2.83 and 0.37, of
// which about 1.2 go to the pairs that pass (700 a query in either); without those the scan runs at 1.0 PFLOP/s (a library product of
// 8192 cubed: 1.15).  Rows 128 at a time with two waves per SIMD: 0.2 ms more; the next group's operands asked for ahead: no
// gain with two waves, spills with three.
// ---------------------------------------------------------------------------------------
#define EXG_RT 64            // rows of a tile
#define EXG_UNEVEN 1.5f      // a tile whose largest norm or residual is more than this many times the largest of one of its groups takes thresholds by the group
#define EXG_QUEUE 320        // pairs a wave collects before they go to the lists: 64 and the 256 of a 16 x 16 tile
template <int KS, bool SAMPLE>
__global__ __launch_bounds__(256, 3) void ex_scan_wave_kernel(ExScanArgs a)
{
    constexpr int PIECES = 4 * KS;                                      // of a row
    constexpr int UNITS = EXG_RT * PIECES / 256;                        // pieces of a tile per thread
    __shared__ floatx4 s_tile[2][EXG_RT * PIECES];
    __shared__ __align__(16) float s_c0[2][EXG_RT];                     // where a row's sums start: -|r|^2 / 2 (or 0; -inf past the end)
    __shared__ float s_R[2][5], s_E[2][5];                              // largest norm and residual of every 16 rows, and of the tile
    __shared__ u32 s_uneven[2];
    __shared__ u64 s_queue[4][EXG_QUEUE];                               // ordered w << 32 | visit within the slice << 6 | query within the wave's
    __shared__ u32 s_full[256];                                         // the query's list is full: it is measured another way
    __shared__ int s_self[256];                                         // the query's own row
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int r16 = lane & 15, q4 = lane >> 4;
    const int wqs = a.wqs, wq = wave & (wqs - 1), wr = wave / wqs;
    const int qb = (int)(blockIdx.x % (unsigned)a.nqb), slice = (int)(blockIdx.x / (unsigned)a.nqb);
    const int tiles = (int)((a.nvisit + EXG_RT - 1) / EXG_RT);
    const int per = (tiles + a.nslices - 1) / a.nslices;
    const int t0 = slice * per, t1 = min(tiles, t0 + per);
    if (t0 >= t1) return;
    const int nvisit = (int)a.nvisit;
    const int64_t q0 = (int64_t)qb * (64 * wqs);                        // the workgroup's first query, and this wave's first among them
    const int qw = wq * 64;

    halfx8 fq[4][KS];
    // A pair passes where -w >= -tau - m, m as in ex_margin: of a query, -tau less its own share of m, |q| + e_q, e_q.  (Four roundings more than
    // ex_margin has are in c1; |tau| counts for no more than the pair's norms do, since nothing but a w about as large is near it.)
    const float c1 = a.c1 + 2.4e-7f;
    float base[4], qs[4], qe[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t q = q0 + qw + 16 * j + r16;
        const bool some = q < a.nq;
        const int64_t qc = some ? q : 0;
        const float4 m = a.qmeta[qc];
        base[j] = -__builtin_inff();                                    // a query without a defined norm: everything passes
        qs[j] = qe[j] = 0.0f;
        if (m.z < __builtin_inff()) { base[j] = -a.tau[qc] - c1 * m.z; qs[j] = m.x + m.y; qe[j] = m.y; }
        if (!some || a.qrow[qc] < 0) base[j] = __builtin_inff();        // no query: nothing passes
        const unsigned char* src = a.Q + qc * (int64_t)a.qbytes + q4 * 16;
#pragma unroll
        for (int s = 0; s < KS; ++s) fq[j][s] = *reinterpret_cast<const halfx8*>(src + 64 * s);
    }

    // the rows of the next tile: registers first, LDS once the tile before the last is done with
    floatx4 pre[UNITS];
    float pre_rn = 0.0f, pre_er = 0.0f;
    auto row_of = [&](int j) __attribute__((always_inline)) { return ex_row<SAMPLE>(a, (u32)min(j, nvisit - 1)); };
    // sixteen rows' pieces of one number lie in the sixteen 16-byte columns of the 64 banks
    auto swizzle = [](int row) __attribute__((always_inline)) { return KS == 4 ? row & 15 : KS == 2 ? (row >> 1) & 7 : (row >> 2) & 3; };
    auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < UNITS; ++it) {
            const int u = tid + 256 * it, row = u / PIECES, off = ((u - row * PIECES) ^ swizzle(row)) * 16;
            pre[it] = *reinterpret_cast<const floatx4*>(a.rows + (int64_t)row_of(t * EXG_RT + row) * (64 * KS) + off);
        }
        if (tid < EXG_RT) {
            const u32 r = row_of(t * EXG_RT + tid);
            pre_rn = a.rn[r];
            pre_er = a.er[r];
        }
    };
    auto store = [&](int t, int par) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < UNITS; ++it) s_tile[par][tid + 256 * it] = pre[it];
        if (tid < EXG_RT) {
            const bool real = t * EXG_RT + tid < nvisit;
            // a row without a defined norm: EX_ALWAYS takes it past any threshold, and its neighbours keep theirs (see ex_scan_kernel)
            const bool undefined = !(pre_rn < __builtin_inff());
            s_c0[par][tid] = !real ? -__builtin_inff() : undefined ? EX_ALWAYS : a.metric == 0 ? -0.5f * pre_rn : 0.0f;
            const float R = undefined ? 0.0f : sqrtf(pre_rn), E = undefined ? 0.0f : pre_er;
            // (as bits, which order them: neither is negative)
            u32 r = __float_as_uint(R), e = __float_as_uint(E);
            r = max(r, tg_partner32<1>(r));   e = max(e, tg_partner32<1>(e));
            r = max(r, tg_partner32<2>(r));   e = max(e, tg_partner32<2>(e));
            r = max(r, tg_partner32<7>(r));   e = max(e, tg_partner32<7>(e));
            r = max(r, tg_partner32<15>(r));  e = max(e, tg_partner32<15>(e));
            if ((tid & 15) == 0) { s_R[par][tid >> 4] = __uint_as_float(r) * 1.0001f; s_E[par][tid >> 4] = __uint_as_float(e); }
            auto of = [](u32 x, int group) __attribute__((always_inline)) { return (u32)__builtin_amdgcn_readlane((int)x, 16 * group); };
            const u32 r_most = max(max(of(r, 0), of(r, 1)), max(of(r, 2), of(r, 3))), r_least = min(min(of(r, 0), of(r, 1)), min(of(r, 2), of(r, 3)));
            const u32 e_most = max(max(of(e, 0), of(e, 1)), max(of(e, 2), of(e, 3))), e_least = min(min(of(e, 0), of(e, 1)), min(of(e, 2), of(e, 3)));
            if (tid == 0) {
                s_R[par][4] = __uint_as_float(r_most) * 1.0001f;
                s_E[par][4] = __uint_as_float(e_most);
                s_uneven[par] = __uint_as_float(r_most) > EXG_UNEVEN * __uint_as_float(r_least) || __uint_as_float(e_most) > EXG_UNEVEN * __uint_as_float(e_least);
            }
        }
    };

    s_full[tid] = 0u;                                                   // (seen by everyone behind the first barrier of the loop)
    s_self[tid] = tid < 64 * wqs && q0 + tid < a.nq ? a.qrow[q0 + tid] : -1;
    int nqueue = 0;
    auto flush = [&]() __attribute__((always_inline)) {
        ex_sync();
        for (int b = 0; b < nqueue; b += 64) {
            if (b + lane < nqueue) {
                const u64 e = s_queue[wave][b + lane];
                const u32 ql = (u32)qw + ((u32)e & 63u), visit = (u32)(t0 * EXG_RT) + ((u32)e >> 6);
                const int64_t q = q0 + ql;
                const u32 r = row_of((int)visit);
                if (visit < (u32)nvisit && r != (u32)s_self[ql]) {
                    const u32 pos = atomicAdd(a.cnt + q * EX_CSTRIDE, 1u);
                    if (pos < EX_CAP) a.buf[q * EX_CAP + pos] = (e & 0xFFFFFFFF00000000ull) | r;
                    else s_full[ql] = 1u;
                }
            }
        }
        nqueue = 0;
        ex_sync();
    };

    const u64 below = tg_lanemask_lt();
    fetch(t0);
    for (int t = t0; t < t1; ++t) {
        const int par = (t - t0) & 1;
        store(t, par);
        __syncthreads();
        if (t + 1 < t1) fetch(t + 1);
        float thr[4];
        auto bound_by = [&](int group) __attribute__((always_inline)) {
            const float R = s_R[par][group], E = s_E[par][group], own = c1 * R * R;
#pragma unroll
            for (int j = 0; j < 4; ++j) thr[j] = fmaf(-qs[j], E, fmaf(-qe[j], R, base[j] - own));
        };
        auto meet = [&](int i) __attribute__((always_inline)) {
            const int row = 16 * i + r16;
            halfx8 fr[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) fr[s] = __builtin_bit_cast(halfx8, s_tile[par][row * PIECES + ((4 * s + q4) ^ swizzle(row))]);
            const floatx4 c0 = *reinterpret_cast<const floatx4*>(&s_c0[par][16 * i + 4 * q4]);
            floatx4 acc[4];
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fr[s], fq[j][s], s ? acc[j] : c0, 0, 0, 0);
            // -w of every pair against -tau - m
            u64 hit[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) hit[j] = __ballot(fmaxf(fmaxf(acc[j][0], acc[j][1]), fmaxf(acc[j][2], acc[j][3])) >= thr[j]);
            if ((hit[0] | hit[1] | hit[2] | hit[3]) == 0ull) return;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (hit[j] == 0ull) continue;
                if (nqueue > EXG_QUEUE - 256) flush();
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool pass = acc[j][e] >= thr[j];
                    const u64 m = __ballot(pass);
                    if (m == 0ull) continue;
                    const u32 tag = (u32)(((t - t0) * EXG_RT + 16 * i + 4 * q4 + e) << 6) | (u32)(16 * j + r16);
                    if (pass) s_queue[wave][nqueue + __popcll(m & below)] = ((u64)tg_ord(-acc[j][e]) << 32) | tag;
                    nqueue += __popcll(m);
                }
            }
        };
        // (64 rows are four groups: wqs of them for each of the 4 / wqs shares)
        const bool uneven = __builtin_amdgcn_readfirstlane((int)s_uneven[par]) != 0;
        const int last = (wr + 1) * wqs;
#pragma unroll 1
        for (int i = wr * wqs; i < last;) {
            bound_by(uneven ? i : 4);
            const int upto = uneven ? i + 1 : last;
#pragma unroll 1
            for (; i < upto; ++i) meet(i);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (s_full[qw + 16 * j + r16]) base[j] = __builtin_inff();
    }
    flush();
}

// The waves' lists of 64 keys, ascending, become one, in wave 0 (the others return what they have): halves of the waves that are left meet
// until one is.  s_top: WAVES / 2 x 64 words.
template <int WAVES>
__device__ inline u64 ex_waves_merge(u64 top, u64 (*s_top)[64])
{
    const int wave = threadIdx.x >> 6, lane = tg_lane();
#pragma unroll
    for (int h = WAVES / 2; h > 0; h /= 2) {
        __syncthreads();
        if (wave >= h && wave < 2 * h) s_top[wave - h][lane] = top;
        __syncthreads();
        if (wave < h) top = tg_wave_merge_low(top, s_top[wave][lane]);
    }
    return top;
}
// The k-th smallest of count keys key_of(i), found by the waves of a workgroup: waves take a batch of
// 64 in turn, batches without a key below the wave's k-th so far are passed over, the sorted lists are merged.
// Wave 0 returns the 64 smallest keys, ascending.
template <int WAVES, class F>
__device__ inline u64 ex_block_smallest(int count, int k, u64 (*s_top)[64], F key_of)
{
    const int wave = threadIdx.x >> 6, lane = tg_lane();
    u64 top = TG_EMPTY_KEY, last = TG_EMPTY_KEY;
    for (int b = wave * 64; b < count; b += 64 * WAVES) {
        u64 key = b + lane < count ? key_of(b + lane) : TG_EMPTY_KEY;
        if (__ballot(key < last) == 0ull) continue;
        key = tg_wave_sort(key);
        top = b == wave * 64 ? key : tg_wave_merge_low(top, key);
        last = tg_shfl64(top, k - 1);
    }
    return ex_waves_merge<WAVES>(top, s_top);
}
// upper bound of an entry's value: w + m with the row's own norm and residual (unit rows in the fp32 cosine scan)
__device__ inline u64 ex_upper_key(const ExScanArgs& a, u64 e, float4 qm, float kq, bool unit)
{
    if (e == TG_EMPTY_KEY) return e;
    const u32 row = (u32)e;
    const float R = unit ? 1.0f : sqrtf(a.rn[row]) * 1.0001f, E = a.er ? a.er[row] : 0.0f;
    const float m = ex_margin(qm.x, qm.y, kq, R, E, a.c1);
    const float up = tg_unord((u32)(e >> 32)) + m;
    if (up != up) return TG_EMPTY_KEY;                                  // an undefined distance bounds no other
    return ((u64)tg_ord(up) << 32) | row;
}
// tau of every query from the entries of a sample: one workgroup per query, of sixteen waves where there are few queries and the time of
// one is the time of all (64 queries: 9.5 -> 5.9 us; the answers below got no faster, 11.1 -> 12.3), of four where they fill the chip.
#define EX_FEW 512
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void ex_select_kernel(ExScanArgs a, int k, int fixed_count, int unit)
{
    __shared__ u64 s_top[WAVES / 2][64];
    const int64_t q = blockIdx.x;
    if (a.qrow[q] < 0) return;
    const int count = fixed_count ? fixed_count : (int)min(a.cnt[q * EX_CSTRIDE], (u32)EX_CAP);
    const float4 qm = a.qmeta[q];
    const u64* e = a.buf + q * EX_CAP;
    const u64 top = ex_block_smallest<WAVES>(count, k, s_top, [&](int i) { return ex_upper_key(a, e[i], qm, a.c1 * qm.z, unit != 0); });
    if (threadIdx.x < 64) {
        const u64 kth = tg_shfl64(top, k - 1);
        if (threadIdx.x == 0) {
            // the next scan's rows come on top of none: fewer than k entries (rows without a defined distance) bound nothing
            a.tau[q] = kth == TG_EMPTY_KEY ? __builtin_inff() : tg_unord((u32)(kth >> 32));
            a.cnt[q * EX_CSTRIDE] = 0u;
        }
    }
}

// The answer of a query from its list: entries that cannot be among the k nearest by the list's own k-th smallest upper
// bound fall out, the others are measured directly (16 lanes per row, the sum taken as exact_scan_kernel takes it), sorted, written.
#define EX_ANSWER_WAVES 4
__global__ __launch_bounds__(64 * EX_ANSWER_WAVES) void ex_answer_kernel(ExScanArgs a, const float* __restrict__ X, int ld, const float* __restrict__ rnorm, int k,
                                                        int fixed_count, int unit, int32_t* __restrict__ out_ids, float* __restrict__ out_dist)
{
    extern __shared__ __align__(16) float s_q[];
    __shared__ u64 s_top[EX_ANSWER_WAVES / 2][64];
    __shared__ u64 s_key[64 * EX_ANSWER_WAVES];
    __shared__ u32 s_row[EX_CAP];
    __shared__ float s_tau;
    __shared__ u32 s_n;
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tg_lane(), grp = lane >> 4, sub = lane & 15;
    const int qrow = a.qrow[q];
    const u32 cnt = fixed_count ? (u32)fixed_count : a.cnt[q * EX_CSTRIDE];
    if (qrow >= 0 && cnt > (u32)EX_CAP) {
        if (tid == 0) a.fb_list[atomicAdd(a.fb_n, 1u)] = (u32)q;
        return;
    }
    if (qrow < 0) {
        if (wave == 0) ex_write_row(TG_EMPTY_KEY, k, q, out_ids, out_dist);
        return;
    }
    const float* xq = X + (int64_t)qrow * ld;
    for (int c = tid * 4; c < ld; c += 256 * EX_ANSWER_WAVES) *reinterpret_cast<float4*>(s_q + c) = *reinterpret_cast<const float4*>(xq + c);
    const int count = (int)cnt;
    const float4 qm = a.qmeta[q];
    const float kq = a.c1 * qm.z;
    const u64* ent = a.buf + q * EX_CAP;
    if (tid == 0) s_n = 0u;
    u64 top = TG_EMPTY_KEY;
    float tau = __builtin_inff();
    if (count > k) {
        top = ex_block_smallest<EX_ANSWER_WAVES>(count, k, s_top, [&](int i) { return ex_upper_key(a, ent[i], qm, kq, unit != 0); });
        if (wave == 0) {
            const u64 kth = tg_shfl64(top, k - 1);
            if (lane == 0) s_tau = kth == TG_EMPTY_KEY ? __builtin_inff() : tg_unord((u32)(kth >> 32));
        }
        __syncthreads();
        tau = s_tau;
    } else {
        __syncthreads();
    }
    for (int i = tid; i < count; i += 64 * EX_ANSWER_WAVES) {
        const u64 e = ent[i];
        if (e == TG_EMPTY_KEY) continue;
        const u32 row = (u32)e;
        const float R = unit ? 1.0f : sqrtf(a.rn[row]) * 1.0001f, E = a.er ? a.er[row] : 0.0f;
        const float low = tg_unord((u32)(e >> 32)) - ex_margin(qm.x, qm.y, kq, R, E, a.c1);
        if (!(low > tau)) s_row[atomicAdd(&s_n, 1u)] = row;
    }
    __syncthreads();
    const int m = (int)s_n;
    const float qrn = a.metric == 2 ? rnorm[qrow] : 1.0f;
    top = TG_EMPTY_KEY;
    u64 last = TG_EMPTY_KEY;
    // a wave measures 64 rows (16 per quarter, four of them on their way at a time), then folds them into its list
    u64* mine = s_key + wave * 64;
    for (int b = wave * 64; b < m; b += 64 * EX_ANSWER_WAVES) {
        mine[lane] = TG_EMPTY_KEY;
        ex_sync();
        for (int p0 = 0; p0 < 64 && b + p0 < m; p0 += 16) {
            const float* y[4];
            u32 row[4];
            float acc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = b + p0 + 4 * i + grp;
                row[i] = s_row[p < m ? p : m - 1];
                y[i] = X + (int64_t)row[i] * ld;
                acc[i] = 0.0f;
            }
            for (int col = sub * 4; col < ld; col += 64) {
                const float4 z = *reinterpret_cast<const float4*>(s_q + col);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 v = *reinterpret_cast<const float4*>(y[i] + col);
                    if (a.metric == 0) {
                        const float t0 = z.x - v.x, t1 = z.y - v.y, t2 = z.z - v.z, t3 = z.w - v.w;
                        acc[i] += t0 * t0 + t1 * t1 + t2 * t2 + t3 * t3;
                    } else {
                        acc[i] += z.x * v.x + z.y * v.y + z.z * v.z + z.w * v.w;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float s = acc[i];
                s += __shfl_xor(s, 1);
                s += __shfl_xor(s, 2);
                s += __shfl_xor(s, 4);
                s += __shfl_xor(s, 8);
                float dist = s;
                if (a.metric == 1) dist = -s;
                else if (a.metric == 2) dist = 1.0f - s * qrn * rnorm[row[i]];
                if (sub == 0 && b + p0 + 4 * i + grp < m) mine[p0 + 4 * i + grp] = tg_key(dist, row[i], 0u);
            }
        }
        ex_sync();
        u64 key = mine[lane];
        ex_sync();
        if (__ballot(key < last) == 0ull) continue;
        key = tg_wave_sort(key);
        top = b == wave * 64 ? key : tg_wave_merge_low(top, key);
        last = tg_shfl64(top, k - 1);
    }
    top = ex_waves_merge<EX_ANSWER_WAVES>(top, s_top);
    if (wave == 0) ex_write_row(top, k, q, out_ids, out_dist);
}

// ---------------------------------------------------------------------------------------
// Host side of the screened search
// ---------------------------------------------------------------------------------------
static size_t ex_up(size_t b) { return (b + 255) & ~(size_t)255; }
static int ex_qbytes(int ld, bool f16)
{
    const int b = f16 ? 2 * ((ld + 31) & ~31) : 4 * ld;
    return (b + EX_CHUNK - 1) / EX_CHUNK * EX_CHUNK;
}
// Rounding X to fp16 costs a read of X and half a write before anything is gained; multiplying in fp32 takes 1 / 16 of the
// rate.  Whole calls, fp16 / fp32, us: 1M x 128, k = 32: 750 / 485 at 64 queries, 805 / 654 at 128, 870 / 1014 at 192, 3764 / 11329
// at 4000; 50 000 x 400: 259 / 275 at 128, 271 / 351 at 192; 20 000 x 32: 189 / 180 at 512, 218 / 207 at 1024.
bool tg_exact_use_f16(int64_t n, int ld, int64_t nq) { return nq > 128 && (double)n * ld * nq >= 2e9; }

size_t tg_exact_fixed_bytes(int64_t n, int ld, int metric, bool f16)
{
    size_t b = ex_up((size_t)n * 4);                                   // squared norms
    if (metric == 2 || !f16) b += ex_up((size_t)n * 4);                // 1 / |x|
    if (f16) b += ex_up((size_t)n * 2 * ((ld + 31) & ~31)) + ex_up((size_t)n * 4) + ex_up((size_t)ld * 4 + 64) + 256;
    return b + 256;
}
size_t tg_exact_query_bytes(int64_t nq, int ld, bool f16)
{
    const int64_t pad = (nq + 127) / 128 * 128;
    return ex_up((size_t)nq * EX_CAP * 8) + ex_up((size_t)pad * ex_qbytes(ld, f16)) + ex_up((size_t)pad * 16) + ex_up((size_t)pad * 4 * EX_CSTRIDE) + 3 * ex_up((size_t)pad * 4 + 4);
}

bool tg_exact_plan(int64_t n, int ld, int metric, int64_t nq, size_t padded, int attempt, TgExactPlan* plan)
{
    // fp16 rows where they are faster, the fp32 rows as they are, then fewer queries at a time: 16384, 4096, 1024, 256, 64
    const bool half = tg_exact_use_f16(n, ld, nq);
    const int step = half && attempt > 0 ? attempt - 1 : attempt;
    if (step > 4) return false;
    plan->f16 = half && attempt == 0;
    plan->fixed = tg_exact_fixed_bytes(n, ld, metric, plan->f16 != 0);
    const int64_t most = 16384 >> (2 * step);
    int64_t batch = nq < most ? nq : most;
    // An allocation of 64 MiB or more costs 0.35 ms to give back (65 us below that): where the lists are what makes it so large,
    // the queries go in several batches (about 60 us each).
    if (padded + plan->fixed < (32u << 20) && nq <= 16384)
        for (int64_t parts = 1; padded + plan->fixed + tg_exact_query_bytes(batch, ld, plan->f16 != 0) >= (64u << 20); ++parts)
            batch = ((nq + parts - 1) / parts + 127) & ~127ll;
    if (batch > most) batch = most;
    plan->batch = batch > nq ? nq : batch;
    plan->bytes = padded + plan->fixed + tg_exact_query_bytes(plan->batch, ld, plan->f16 != 0);
    return true;
}

template <bool F16, int QT, bool RES, int MODE>
static void ex_launch_scan_t(const ExScanArgs& a, hipStream_t s)
{
    const int nch = a.qbytes / EX_CHUNK;
    const size_t shm = (size_t)(RES ? nch : 2) * QT * EX_CHUNK + 2 * EX_RT * EX_CHUNK;
    tg_allow_lds<ex_scan_kernel<F16, QT, RES, MODE>>(64 * 1024);
    hipLaunchKernelGGL((ex_scan_kernel<F16, QT, RES, MODE>), dim3((unsigned)(a.nqb * a.nslices)), dim3(64 * EX_WAVES), shm, s, a);
}
template <bool SAMPLE>
static void ex_launch_scan_wave(ExScanArgs a, hipStream_t s)
{
    // 256, 128 or 64 queries to a workgroup (rows are fetched once for all of them): the most that need at most a fifteenth more places
    auto padded = [&](int wqs) { return (a.nq + 64 * wqs - 1) / (64 * wqs) * (64 * wqs); };
    a.wqs = 4;
    while (padded(a.wqs) * 15 > padded(1) * 16) a.wqs /= 2;
    a.nqb = (int)(padded(a.wqs) / (64 * a.wqs));
    const int64_t tiles = (a.nvisit + EXG_RT - 1) / EXG_RT;
    // three workgroups per CU at a time, three times over; a place in a slice has 26 bits in the queue, and 16384 queries leave 36 slices
    int64_t slices = 2304 / a.nqb;
    if (slices < 1) slices = 1;
    a.nslices = (int)(slices < tiles ? slices : tiles);
    const dim3 grid((unsigned)(a.nqb * a.nslices)), block(256);
    switch (a.rowbytes >> 6) {
    case 1: hipLaunchKernelGGL((ex_scan_wave_kernel<1, SAMPLE>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((ex_scan_wave_kernel<2, SAMPLE>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((ex_scan_wave_kernel<3, SAMPLE>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((ex_scan_wave_kernel<4, SAMPLE>), grid, block, 0, s, a); break;
    }
}
template <bool F16, int MODE>
static void ex_launch_scan_m(ExScanArgs a, hipStream_t s)
{
    if constexpr (F16 && MODE != EX_FIRST) {
        if (a.qbytes <= 2 * EX_CHUNK) {
            ex_launch_scan_wave<MODE == EX_SAMPLE>(a, s);
            return;
        }
    }
    const bool wide = a.nq > 64;
    const int qt = wide ? 128 : 64;
    a.nqb = (int)((a.nq + qt - 1) / qt);
    const int64_t tiles = (a.nvisit + EX_RT - 1) / EX_RT;
    int64_t slices = (2048 + a.nqb - 1) / a.nqb;                       // two workgroups per CU at a time, a few times over
    a.nslices = (int)(slices < tiles ? slices : tiles);
    if (a.nslices < 1) a.nslices = 1;
    if constexpr (!F16 || MODE == EX_FIRST) {
        if (a.qbytes <= 2 * EX_CHUNK) {
            if (wide) ex_launch_scan_t<F16, 128, true, MODE>(a, s);
            else ex_launch_scan_t<F16, 64, true, MODE>(a, s);
            return;
        }
    }
    if (wide) ex_launch_scan_t<F16, 128, false, MODE>(a, s);
    else ex_launch_scan_t<F16, 64, false, MODE>(a, s);
}
template <bool F16>
static void ex_launch_scan_f(const ExScanArgs& a, int mode, hipStream_t s)
{
    if (mode == EX_FIRST) ex_launch_scan_m<F16, EX_FIRST>(a, s);
    else if (mode == EX_SAMPLE) ex_launch_scan_m<F16, EX_SAMPLE>(a, s);
    else ex_launch_scan_m<F16, EX_FULL>(a, s);
}
static void ex_launch_scan(const ExScanArgs& a, bool f16, int mode, hipStream_t s)
{
    if (f16) ex_launch_scan_f<true>(a, mode, s);
    else ex_launch_scan_f<false>(a, mode, s);
}
static u64 ex_gcd(u64 a, u64 b) { while (b) { const u64 t = a % b; a = b; b = t; } return a; }

// fixed: tg_exact_fixed_bytes, per_batch: tg_exact_query_bytes of `batch` queries; both 256-byte aligned
void tg_launch_exact_screened(const float* X, int ld, int64_t n, int d, int k, int metric, const int64_t* rows, int64_t nq, bool f16,
                              void* fixed, void* per_batch, int64_t batch, int32_t* out_ids, float* out_dist, hipStream_t s)
{
    unsigned char* f = static_cast<unsigned char*>(fixed);
    auto take = [&](size_t b) { unsigned char* p = f; f += ex_up(b); return p; };
    ExScanArgs a = {};
    a.n = n; a.metric = metric;
    float* rn = reinterpret_cast<float*>(take((size_t)n * 4));
    float* rnorm = (metric == 2 || !f16) ? reinterpret_cast<float*>(take((size_t)n * 4)) : nullptr;
    a.rn = rn;
    a.c1 = (float)(2 * d + 32) * 5.9604645e-08f;
    if (f16) {
        const int ldh = (ld + 31) & ~31;
        uint16_t* Xh = reinterpret_cast<uint16_t*>(take((size_t)n * 2 * ldh));
        float* er = reinterpret_cast<float*>(take((size_t)n * 4));
        float* centre = reinterpret_cast<float*>(take((size_t)ld * 4 + 64));
        u32* top = reinterpret_cast<u32*>(take(4));
        tg_launch_fill_u32(top, 1, 0u, s);
        hipLaunchKernelGGL(ex_stat_kernel, dim3((unsigned)((ld + 63) / 64)), dim3(1024), 0, s, X, n, d, ld, metric == 0 ? 1 : 0, centre, top);
        const int64_t wgs = (n + 15) / 16;
        hipLaunchKernelGGL(ex_half_kernel, dim3((unsigned)(wgs < 4096 ? wgs : 4096)), dim3(256), 0, s, X, n, d, ld, metric, (const float*)centre,
                           (const u32*)top, Xh, ldh, rn, er, rnorm);
        a.rows = reinterpret_cast<const unsigned char*>(Xh);
        a.rowbytes = 2 * ldh;
        a.er = er;
    } else {
        a.rows = reinterpret_cast<const unsigned char*>(X);
        a.rowbytes = 4 * ld;
    }
    a.rnorm = rnorm;
    a.qbytes = ex_qbytes(ld, f16);
    const int unit = !f16 && metric == 2 ? 1 : 0;
    // a step through the rows that meets each once in n steps and spreads any run of them evenly
    u64 step = (u64)((double)n * 0.6180339887498949);
    if (step < 1) step = 1;
    while (ex_gcd(step, (u64)n) != 1) ++step;
    // Sample sizes: from one level to the next the rows may grow by a factor f so that k f pairs per query, give or take
    // sqrt(k) f, pass and never more than EX_CAP do (7 deviations, and the exponential tail of small k).
    const double grow = (double)EX_CAP / (k + 7.0 * sqrt((double)k) + 10.0);
    int64_t level[16];
    int levels = 0;
    if (n > EX_CAP) {
        const int steps = (int)ceil(log((double)n / EX_CAP) / log(grow) - 1e-9);
        const double by = exp(log((double)n / EX_CAP) / (steps < 1 ? 1 : steps));
        double size = EX_CAP;
        for (int i = 1; i < steps && levels < 15; ++i) { size *= by; level[levels++] = (int64_t)size; }
    }
    const int shm_q = ld * 4;
    for (int64_t q0 = 0; q0 < nq; q0 += batch) {
        a.nq = nq - q0 < batch ? nq - q0 : batch;
        const int64_t pad = (a.nq + 127) / 128 * 128;
        unsigned char* p = static_cast<unsigned char*>(per_batch);
        auto tb = [&](size_t b) { unsigned char* r = p; p += ex_up(b); return r; };
        a.buf = reinterpret_cast<u64*>(tb((size_t)a.nq * EX_CAP * 8));
        a.Q = tb((size_t)pad * a.qbytes);
        a.qmeta = reinterpret_cast<float4*>(tb((size_t)pad * 16));
        a.qrow = reinterpret_cast<int32_t*>(tb((size_t)pad * 4));
        a.cnt = reinterpret_cast<u32*>(tb((size_t)pad * 4 * EX_CSTRIDE));
        a.tau = reinterpret_cast<float*>(tb((size_t)pad * 4));
        a.fb_list = reinterpret_cast<u32*>(tb((size_t)pad * 4 + 4));
        a.fb_n = a.fb_list + a.nq;
        const int64_t norm_wgs = f16 || q0 ? 0 : (n + 15) / 16 < 2048 ? (n + 15) / 16 : 2048;
        hipLaunchKernelGGL(ex_query_kernel, dim3((unsigned)(pad / 4 + norm_wgs)), dim3(256), 0, s, a, f16 ? 1 : 0, rows, q0, pad, ld, rn, rnorm);
        const int first = (int)(n < EX_CAP ? n : EX_CAP);
        const bool few = a.nq <= EX_FEW;
        auto select = [&](int fixed) {
            hipLaunchKernelGGL((few ? ex_select_kernel<16> : ex_select_kernel<4>), dim3((unsigned)a.nq), dim3(few ? 1024 : 256), 0, s, a, k, fixed, unit);
        };
        a.nvisit = first;
        a.step = n > EX_CAP ? step : 1;                                // (fewer rows than places: all of them in order)
        a.step_by_n = (double)a.step / (double)n;
        ex_launch_scan(a, f16, EX_FIRST, s);
        if (n > EX_CAP) {
            select(first);
            for (int i = 0; i < levels; ++i) {
                a.nvisit = level[i];
                ex_launch_scan(a, f16, EX_SAMPLE, s);
                select(0);
            }
            a.nvisit = n;
            ex_launch_scan(a, f16, EX_FULL, s);
        }
        hipLaunchKernelGGL(ex_answer_kernel, dim3((unsigned)a.nq), dim3(64 * EX_ANSWER_WAVES), shm_q, s, a, X, ld, (const float*)rnorm, k, n > EX_CAP ? 0 : first, unit,
                           out_ids + q0 * k, out_dist ? out_dist + q0 * k : nullptr);
        if (n > EX_CAP) {
            // queries whose list overflowed, if any (the lists are free by now: they take the partial results)
            int slices = tg_exact_slices(n, a.nq);
            while (slices > 1 && (int64_t)slices * k > EX_CAP) --slices;
            tg_launch_exact_knn(X, ld, rnorm, n, k, metric, rows, a.nq, q0, a.fb_list, a.fb_n, out_ids + q0 * k,
                                out_dist ? out_dist + q0 * k : nullptr, a.buf, slices, s);
        }
    }
}
