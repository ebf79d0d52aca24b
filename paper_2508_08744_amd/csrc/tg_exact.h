// Exact k-NN: what the kernels and the host side of the screened search share (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define EX_CAP 2048      // places per query for pairs that passed the screen; also the rows of the first sample

#define EX_CSTRIDE 16     // a query's counter has a 64-byte line of its own: atomics on one line take turns (64 queries against
                         // 50 000 x 96: the scan takes 19 us so, 45 with the counters side by side)

struct ExScanArgs {
    int64_t n;                       // rows of X
    int64_t nvisit;                  // rows this scan visits
    unsigned long long step;         // the j-th row of a sample is j * step mod n
    double step_by_n;                // step / n
    int64_t nq;                      // queries of this batch
    int32_t metric;
    int32_t rowbytes, qbytes;        // bytes of a stored row; of a packed query (whole chunks)
    int32_t nqb, nslices;            // query tiles and row slices of the launch
    int32_t wqs;                     // ex_scan_wave_kernel: waves of a workgroup side by side over the queries
    float c1;                        // see ex_margin
    const unsigned char* rows;       // fp16 or fp32 rows
    const float* rn;                 // squared norm of every row, in the units of `rows`
    const float* er;                 // norm of what rounding took from a row, or null
    const float* rnorm;              // 1 / |x| (cosine)
    unsigned char* Q;                // packed queries
    float4* qmeta;                   // |q|, residual, |q|^2
    int32_t* qrow;                   // row of X, -1: no query
    float* tau;                      // upper bound of the k-th smallest value
    uint32_t* cnt;                   // entries so far, EX_CSTRIDE words apart
    unsigned long long* buf;         // nq x EX_CAP entries: ordered w << 32 | row
    uint32_t* fb_list;               // queries that overflowed
    uint32_t* fb_n;
};

// list / list_n: only these queries (device), or null; with a list the slices are chosen on the device, and partial holds nq x EX_CAP keys
void tg_launch_exact_knn(const float* X, int ld, const float* rnorm, int64_t n, int k, int metric, const int64_t* rows, int64_t nq,
                         int64_t q_first, const uint32_t* list, const uint32_t* list_n, int32_t* out_ids, float* out_dist,
                         unsigned long long* partial /* nq x slices x k */, int nslices, hipStream_t s);
int tg_exact_slices(int64_t n, int64_t nq);
bool tg_exact_use_f16(int64_t n, int ld, int64_t nq);
size_t tg_exact_fixed_bytes(int64_t n, int ld, int metric, bool f16);
size_t tg_exact_query_bytes(int64_t nq, int ld, bool f16);
// what tg_exact_knn allocates: `padded` bytes for its own copy of X, tg_exact_fixed_bytes, tg_exact_query_bytes of `batch` queries
struct TgExactPlan {
    int32_t f16;
    int64_t batch;
    size_t fixed, bytes;
};
// attempt 0 is the fastest, the later ones take less memory; false (and the plan as it was) when there is no such attempt
bool tg_exact_plan(int64_t n, int ld, int metric, int64_t nq, size_t padded, int attempt, TgExactPlan* plan);
void tg_launch_exact_screened(const float* X, int ld, int64_t n, int d, int k, int metric, const int64_t* rows, int64_t nq, bool f16,
                              void* fixed, void* per_batch, int64_t batch, int32_t* out_ids, float* out_dist, hipStream_t s);
