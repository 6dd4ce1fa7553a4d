// svm_kernels.hip -- set-up and support kernels of libsvmhip.so for gfx950:
// input validation, dense packing, state initialisation, the initial and
// post-reconstruction selection, stable compaction of id lists, the kernel
// sums behind gradient reconstruction (Alg. 6) and the classifier
// (eq:classi), and the closing reductions (threshold, dual objective).
// The persistent SMO loop itself is in svm_step.hip.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "svm_device.h"
#include "svm_internal.h"

namespace svm {

int device_cu_count() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

// ------------------------------------------------------------------ set-up kernels

// Labels +-1 (both counted), finite values and, for CSR, row pointers from 0 that never fall and
// strictly increasing columns in [0, d); the longest row and whether a value differs from 1.0.  A
// workgroup checks a contiguous share of the rows (dense rows element by element, CSR rows by 16
// lanes each, so the loads coalesce) and stores one part; the host adds the parts.  Bound by the
// read of the samples.  Atomic counters in one place cost about 250 ns per wave that adds to them:
// 3.86 ms for 500,000 x 28 dense rows.
// One instance per form of the rows (VAL_*_ROWS), so that each takes at most 16 registers, which is what
// a serving loop leaves free on its compute units: workgroups of 256 threads then run beside it wherever
// the hardware places them, where a grid of more workgroups than the eight free units would wait for the
// loop to stop (2 s, and as long as it is busy).
enum : int { VAL_CSR_ROWS, VAL_FEATURE_MAJOR, VAL_PACKED_ROWS, VAL_STRIDED_ROWS };
template <int BLOCK, int ROWS>
__global__ __launch_bounds__(BLOCK) void validate_kernel(int n, int d, const float* __restrict__ x, int64_t ldx,
                                                         const int32_t* __restrict__ rp,
                                                         const int32_t* __restrict__ col,
                                                         const float* __restrict__ val,
                                                         const int8_t* __restrict__ y, ValPart* part) {
    __shared__ ValPart s_p[BLOCK / 64];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int r0 = (int)((long long)n * blockIdx.x / gridDim.x);
    const int r1 = (int)((long long)n * (blockIdx.x + 1) / gridDim.x);
    int flags = 0;
    if constexpr (ROWS == VAL_CSR_ROWS) {
        const int nnz = rp[n];
        for (int i = r0 + (tid >> 4); i < r1; i += BLOCK / 16) {
            int p = rp[i];
            const int p1 = rp[i + 1];
            // (a row beyond the nonzeros means that a later pointer falls)
            const bool bad = p1 < p || p < 0 || p1 > nnz || (i == 0 && p != 0);
            if (bad) {
                flags |= VAL_MALFORMED;
                continue;
            }
            const int first = p;
            for (p += tid & 15; p < p1; p += 16) {
                const int cp = p > first ? col[p - 1] : -1, c = col[p];
                const float v = val[p];
                if (c < 0 || c >= d || c <= cp) flags |= VAL_MALFORMED;
                if (!isfinite(v)) flags |= VAL_NONFINITE;
                if (v != 1.0f) flags |= VAL_NOT_ONES;
            }
        }
    } else if constexpr (ROWS == VAL_FEATURE_MAJOR) {
        // (a thread's features several at a time: with few rows of many features the chain of loads is all
        // there is, 300 rows of 2000 features 1,024 us a classifier call one by one; four take 18 registers)
        for (int i = r0 + tid; i < r1; i += BLOCK) {
#pragma unroll 3
            for (int k = 0; k < d; ++k)
                if (!isfinite(x[(size_t)k * ldx + i])) flags |= VAL_NONFINITE;
        }
    } else if constexpr (ROWS == VAL_PACKED_ROWS) {
        const float* xb = x + (size_t)r0 * d;
        const size_t m = (size_t)(r1 - r0) * d;
#pragma unroll 4
        for (size_t e = tid; e < m; e += BLOCK)
            if (!isfinite(xb[e])) flags |= VAL_NONFINITE;
    } else {
        for (int i = r0 + wid; i < r1; i += BLOCK / 64)
            for (int k = lane; k < d; k += 64)
                if (!isfinite(x[(size_t)i * ldx + k])) flags |= VAL_NONFINITE;
    }
    // (labels and row lengths in loops of their own: their sums would take registers in the one above)
    int npos = 0, nneg = 0, maxn = 0;
    if constexpr (ROWS == VAL_CSR_ROWS)
        for (int i = r0 + tid; i < r1; i += BLOCK) maxn = max(maxn, rp[i + 1] - rp[i]);
    if (y)
        for (int i = r0 + tid; i < r1; i += BLOCK) {
            const int8_t v = y[i];
            npos += v == 1;
            nneg += v == -1;
            if (v != 1 && v != -1) flags |= VAL_MALFORMED;
        }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        flags |= __shfl_xor(flags, off);
        npos += __shfl_xor(npos, off);
        nneg += __shfl_xor(nneg, off);
        maxn = max(maxn, __shfl_xor(maxn, off));
    }
    if (lane == 0) s_p[wid] = ValPart{flags, npos, nneg, maxn, ROWS == VAL_CSR_ROWS ? rp[n] : 0};
    __syncthreads();
    if (tid == 0) {
        ValPart t = s_p[0];
        for (int w = 1; w < BLOCK / 64; ++w) {
            t.flags |= s_p[w].flags;
            t.n_pos += s_p[w].n_pos;
            t.n_neg += s_p[w].n_neg;
            t.max_row_nnz = max(t.max_row_nnz, s_p[w].max_row_nnz);
        }
        part[blockIdx.x] = t;
    }
}

template <int ROWS>
static void validate_rows(int n, int d, const float* x, int64_t ldx, const int32_t* rp, const int32_t* col,
                          const float* val, const int8_t* y, ValPart* part, hipStream_t s) {
    const int nb = val_blocks(n);
    if (n <= VAL_SMALL) validate_kernel<256, ROWS><<<nb, 256, 0, s>>>(n, d, x, ldx, rp, col, val, y, part);
    else validate_kernel<1024, ROWS><<<nb, 1024, 0, s>>>(n, d, x, ldx, rp, col, val, y, part);
}

hipError_t launch_validate(int n, int d, int lay, const float* x, int64_t ldx, int feature_major, const int32_t* rp,
                           const int32_t* col, const float* val, const int8_t* y, ValPart* part, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (lay == SVM_CSR) validate_rows<VAL_CSR_ROWS>(n, d, x, ldx, rp, col, val, y, part, s);
    else if (feature_major) validate_rows<VAL_FEATURE_MAJOR>(n, d, x, ldx, rp, col, val, y, part, s);
    else if (ldx == d) validate_rows<VAL_PACKED_ROWS>(n, d, x, ldx, rp, col, val, y, part, s);
    else validate_rows<VAL_STRIDED_ROWS>(n, d, x, ldx, rp, col, val, y, part, s);
    return hipGetLastError();
}

// Rows to [n][dpad] (zeros beyond d).  With a list, row r of the output is sample list[r], for the first
// *count of them (in device memory; n is the most there can be).
__global__ void pack_dense_kernel(int n, int d, int dpad, const float* __restrict__ x, int64_t ldx, int feature_major,
                                  float* __restrict__ out, const int32_t* __restrict__ list,
                                  const int32_t* __restrict__ count) {
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (size_t)n * dpad) return;
    const int r = (int)(e / dpad), k = (int)(e % dpad);
    if (list && r >= *count) return;
    const int i = list ? list[r] : r;
    float v = 0.f;
    if (k < d) v = feature_major ? x[(size_t)k * ldx + i] : x[(size_t)i * ldx + k];
    out[e] = v;
}

hipError_t launch_pack_dense(int n, int d, int dpad, const float* x, int64_t ldx, int feature_major, float* out,
                             hipStream_t s, const int32_t* list, const int32_t* count) {
    size_t tot = (size_t)n * dpad;
    if (!tot) return hipSuccess;
    pack_dense_kernel<<<(unsigned)((tot + 255) / 256), 256, 0, s>>>(n, d, dpad, x, ldx, feature_major, out, list,
                                                                    count);
    return hipGetLastError();
}

__global__ void init_state_kernel(int n, const int8_t* __restrict__ y, double C, int warm, double* alpha, double* f,
                                  uint8_t* status) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const bool yp = y[i] > 0;
    double a = 0.0;
    if (warm) a = alpha[i];
    else {
        alpha[i] = 0.0;
        f[i] = yp ? -1.0 : 1.0;
    }
    status[i] = st_make(yp, a, C);
}

hipError_t launch_init_state(int n, const int8_t* y, double C, int warm, double* alpha, double* f, uint8_t* status,
                             hipStream_t s) {
    init_state_kernel<<<(n + 255) / 256, 256, 0, s>>>(n, y, C, warm, alpha, f, status);
    return hipGetLastError();
}

__global__ void refresh_status_kernel(int n, const double* __restrict__ alpha, const int8_t* __restrict__ y, double C,
                                      uint8_t* status) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) status[i] = st_make(y[i] > 0, alpha[i], C);
}

hipError_t launch_refresh_status(int n, const double* alpha, const int8_t* y, double C, uint8_t* status,
                                 hipStream_t s) {
    refresh_status_kernel<<<(n + 255) / 256, 256, 0, s>>>(n, alpha, y, C, status);
    return hipGetLastError();
}

__global__ void reset_active_kernel(int n, int G, int32_t* seg_start, int32_t* cnt, int32_t* act) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) act[i] = i;
    if (i <= G) {
        const int s = (int)(((long long)n * i) / G);
        seg_start[i] = s;
        if (i < G) cnt[i] = (int)(((long long)n * (i + 1)) / G) - s;
    }
}

__global__ void iota_kernel(int n, int32_t* out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = i;
}

hipError_t launch_iota(int n, int32_t* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    iota_kernel<<<(n + 255) / 256, 256, 0, s>>>(n, out);
    return hipGetLastError();
}

hipError_t launch_reset_active(int n, int G, int32_t* seg_start, int32_t* cnt, int32_t* act, hipStream_t s) {
    int m = n > G + 1 ? n : G + 1;
    reset_active_kernel<<<(m + 255) / 256, 256, 0, s>>>(n, G, seg_start, cnt, act);
    return hipGetLastError();
}

__global__ void mark_active_kernel(int G, const int32_t* seg_start, const int32_t* cnt, const int32_t* act,
                                   uint8_t* mask) {
    const int b = blockIdx.x;
    const int s0 = seg_start[b], c = cnt[b];
    for (int t = threadIdx.x; t < c; t += blockDim.x) mask[act[s0 + t]] = 1;
}

hipError_t launch_mark_active(int n, int G, const int32_t* seg_start, const int32_t* cnt, const int32_t* act,
                              uint8_t* mask, hipStream_t s) {
    hipError_t e = hipMemsetAsync(mask, 0, (size_t)n, s);
    if (e != hipSuccess) return e;
    mark_active_kernel<<<G, 256, 0, s>>>(G, seg_start, cnt, act, mask);
    return hipGetLastError();
}

// ------------------------------------------------------------------ selection (set-up and test hook)

// Each workgroup reduces one segment of the active lists to a record; a
// second one-workgroup kernel merges the records into ctl.  Membership comes
// from (alpha, y, C) directly.
__global__ __launch_bounds__(256) void select_partial_kernel(const int32_t* seg_start, const int32_t* cnt,
                                                             const int32_t* act, const double* __restrict__ f,
                                                             const double* __restrict__ alpha,
                                                             const int8_t* __restrict__ y, double C, Rec* rec) {
    __shared__ double s_v[SEL_LDS(256)];
    __shared__ int s_i[SEL_LDS(256)];
    const int b = blockIdx.x;
    const int s0 = seg_start[b], c = cnt[b];
    double bu = INFINITY, bl = -INFINITY;
    int iu = IDX_NONE, il = IDX_NONE;
    for (int t = threadIdx.x; t < c; t += blockDim.x) {
        const int i = act[s0 + t];
        const uint8_t st = st_make(y[i] > 0, alpha[i], C);
        const double fi = f[i];
        if (st_in_up(st) && better_up(fi, i, bu, iu)) { bu = fi; iu = i; }
        if (st_in_low(st) && better_low(fi, i, bl, il)) { bl = fi; il = i; }
    }
    block_reduce_sel<256>(bu, iu, bl, il, s_v, s_i);
    if (threadIdx.x == 0) {
        rec[b].w[0] = (unsigned long long)__double_as_longlong(bu);
        rec[b].w[1] = (unsigned long long)__double_as_longlong(bl);
        rec[b].w[2] = (unsigned long long)(unsigned)iu | ((unsigned long long)(unsigned)il << 32);
        rec[b].w[3] = (unsigned long long)(unsigned)c;
    }
}

__global__ __launch_bounds__(1024) void select_merge_kernel(int G, const Rec* rec, const double* alpha, Ctl* ctl) {
    __shared__ double s_v[SEL_LDS(1024)];
    __shared__ int s_i[SEL_LDS(1024)];
    __shared__ long long s_c[16];
    double bu = INFINITY, bl = -INFINITY;
    int iu = IDX_NONE, il = IDX_NONE;
    long long c = 0;
    for (int t = threadIdx.x; t < G; t += blockDim.x) {
        double v = __longlong_as_double((long long)rec[t].w[0]);
        double w = __longlong_as_double((long long)rec[t].w[1]);
        int a = (int)(unsigned)(rec[t].w[2] & 0xffffffffull);
        int b2 = (int)(unsigned)(rec[t].w[2] >> 32);
        if (better_up(v, a, bu, iu)) { bu = v; iu = a; }
        if (better_low(w, b2, bl, il)) { bl = w; il = b2; }
        c += (long long)rec[t].w[3];
    }
    c = wave_sum(c);
    if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = c;
    block_reduce_sel<1024>(bu, iu, bl, il, s_v, s_i);
    if (threadIdx.x == 0) {
        long long tot = 0;
        for (int w = 0; w < 16; ++w) tot += s_c[w];
        ctl->b_up = bu; ctl->b_low = bl;
        ctl->i_up = iu == IDX_NONE ? -1 : iu;
        ctl->i_low = il == IDX_NONE ? -1 : il;
        ctl->a_up = iu == IDX_NONE ? 0.0 : alpha[iu];
        ctl->a_low = il == IDX_NONE ? 0.0 : alpha[il];
        ctl->n_active = tot;
    }
}

hipError_t launch_select(int G, const int32_t* seg_start, const int32_t* cnt, const int32_t* act, const double* f,
                         const double* alpha, const int8_t* y, double C, Rec* rec, Ctl* ctl, hipStream_t s) {
    select_partial_kernel<<<G, 256, 0, s>>>(seg_start, cnt, act, f, alpha, y, C, rec);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    select_merge_kernel<<<1, 1024, 0, s>>>(G, rec, alpha, ctl);
    return hipGetLastError();
}

// ------------------------------------------------------------------ stable compaction (flags -> sorted id list)

template <int PRED>
DEV bool pred_at(int i, const uint8_t* mask, const double* alpha) {
    if (PRED == 0) return mask[i] == 0;
    if (PRED == 1) return alpha[i] > 0.0;
    return true;
}

constexpr int CMP_BLOCK = 1024;

template <int PRED>
__global__ __launch_bounds__(CMP_BLOCK) void compact_count_kernel(int n, const uint8_t* mask, const double* alpha,
                                                                  int32_t* blk_cnt) {
    __shared__ int s_c[CMP_BLOCK / 64];
    const int i = blockIdx.x * CMP_BLOCK + threadIdx.x;
    const bool p = i < n && pred_at<PRED>(i, mask, alpha);
    const unsigned long long m = __ballot(p);
    if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = __popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < CMP_BLOCK / 64; ++w) t += s_c[w];
        blk_cnt[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(1024) void compact_scan_kernel(int nb, int32_t* blk_cnt, int32_t* count_out) {
    // exclusive scan of nb block counts by one workgroup, in chunks of 1024
    __shared__ int s_w[16];
    __shared__ int s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int base = 0; base < nb; base += 1024) {
        const int t = base + threadIdx.x;
        const int v = t < nb ? blk_cnt[t] : 0;
        // inclusive scan within the wave
        int x = v;
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            int o = __shfl_up(x, off);
            if (lane >= off) x += o;
        }
        if (lane == 63) s_w[wid] = x;
        __syncthreads();
        int woff = 0, tot = 0;
        for (int w = 0; w < 16; ++w) {
            woff += (w < wid) ? s_w[w] : 0;
            tot += s_w[w];
        }
        const int carry = s_carry;
        if (t < nb) blk_cnt[t] = carry + woff + x - v;
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) *count_out = s_carry;
}

template <int PRED>
__global__ __launch_bounds__(CMP_BLOCK) void compact_write_kernel(int n, const uint8_t* mask, const double* alpha,
                                                                  const int8_t* y, const int32_t* blk_off,
                                                                  int32_t* list, double* coef) {
    __shared__ int s_c[CMP_BLOCK / 64];
    const int i = blockIdx.x * CMP_BLOCK + threadIdx.x;
    const bool p = i < n && pred_at<PRED>(i, mask, alpha);
    const unsigned long long m = __ballot(p);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) s_c[wid] = __popcll(m);
    __syncthreads();
    int off = blk_off[blockIdx.x];
    for (int w = 0; w < wid; ++w) off += s_c[w];
    off += __popcll(m & ((1ull << lane) - 1ull));
    if (p) {
        list[off] = i;
        if (coef) coef[off] = alpha[i] * (y[i] > 0 ? 1.0 : -1.0);
    }
}

// Up to CMP_SMALL rows a thread in one workgroup: count, offsets and list in one launch instead of three,
// which for so few rows is all that their time is; with more, the three use more than one CU's loads.
constexpr int CMP_SMALL = 4;
template <int PRED>
__global__ __launch_bounds__(CMP_BLOCK) void compact_small_kernel(int n, const uint8_t* mask, const double* alpha,
                                                                  const int8_t* y, int32_t* list, double* coef,
                                                                  int32_t* count_out) {
    constexpr int NW = CMP_BLOCK / 64;
    __shared__ int s_c[CMP_SMALL][NW];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    unsigned long long m[CMP_SMALL];
#pragma unroll
    for (int k = 0; k < CMP_SMALL; ++k) {
        const int i = k * CMP_BLOCK + threadIdx.x;
        m[k] = __ballot(i < n && pred_at<PRED>(i, mask, alpha));
        if (lane == 0) s_c[k][wid] = __popcll(m[k]);
    }
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int k = 0; k < CMP_SMALL; ++k) {
        const int i = k * CMP_BLOCK + threadIdx.x;
        int off = base;
        for (int w = 0; w < NW; ++w) {
            off += w < wid ? s_c[k][w] : 0;
            base += s_c[k][w];
        }
        if ((m[k] >> lane) & 1) {
            off += __popcll(m[k] & ((1ull << lane) - 1ull));
            list[off] = i;
            if (coef) coef[off] = alpha[i] * (y[i] > 0 ? 1.0 : -1.0);
        }
    }
    if (threadIdx.x == 0) *count_out = base;
}

hipError_t launch_compact(int n, int pred, const uint8_t* mask, const double* alpha, const int8_t* y,
                          int32_t* blk_cnt, int32_t* list, double* coef, int32_t* count_out, hipStream_t s) {
    const int nb = (n + CMP_BLOCK - 1) / CMP_BLOCK;
    if (nb == 0) return hipMemsetAsync(count_out, 0, sizeof(int32_t), s);
    if (nb <= CMP_SMALL) {
        if (pred == 0) compact_small_kernel<0><<<1, CMP_BLOCK, 0, s>>>(n, mask, alpha, y, list, coef, count_out);
        else if (pred == 1) compact_small_kernel<1><<<1, CMP_BLOCK, 0, s>>>(n, mask, alpha, y, list, coef, count_out);
        else compact_small_kernel<2><<<1, CMP_BLOCK, 0, s>>>(n, mask, alpha, y, list, coef, count_out);
        return hipGetLastError();
    }
    if (pred == 0) compact_count_kernel<0><<<nb, CMP_BLOCK, 0, s>>>(n, mask, alpha, blk_cnt);
    else if (pred == 1) compact_count_kernel<1><<<nb, CMP_BLOCK, 0, s>>>(n, mask, alpha, blk_cnt);
    else compact_count_kernel<2><<<nb, CMP_BLOCK, 0, s>>>(n, mask, alpha, blk_cnt);
    compact_scan_kernel<<<1, 1024, 0, s>>>(nb, blk_cnt, count_out);
    if (pred == 0) compact_write_kernel<0><<<nb, CMP_BLOCK, 0, s>>>(n, mask, alpha, y, blk_cnt, list, coef);
    else if (pred == 1) compact_write_kernel<1><<<nb, CMP_BLOCK, 0, s>>>(n, mask, alpha, y, blk_cnt, list, coef);
    else compact_write_kernel<2><<<nb, CMP_BLOCK, 0, s>>>(n, mask, alpha, y, blk_cnt, list, coef);
    return hipGetLastError();
}

// ------------------------------------------------------------------ kernel sums (reconstruction, decision)

// Workgroup = 256 threads, holding R rows of A in LDS (dense: [R][dpad];
// CSR: densified [R][d]).  Threads stride over this split's part of the B
// list; each keeps R distances and R FP64 partial sums.  Partial sums per
// split go to part[split][a]; launch_finish_sum adds the splits in order.
constexpr int SUM_BLOCK = 256;
constexpr int SUM_RMAX = 16;
constexpr int SLOT_R_MAX = 8;

template <int LAY, typename KT>
__global__ __launch_bounds__(SUM_BLOCK) void kernel_sum_kernel(SumArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_red[SUM_BLOCK / 64][SUM_RMAX];
    __shared__ double s_na[SUM_RMAX];
    float* at = reinterpret_cast<float*>(smem);
    const int R = A.rows_per_block;
    const int r0 = blockIdx.x * R;
    const int nr = min(R, A.na - r0);
    const int W = (LAY == LAY_DENSE) ? A.dpad : A.d;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;

    // stage the A rows
    for (int e = tid; e < R * W; e += SUM_BLOCK) at[e] = 0.f;
    __syncthreads();
    if (LAY == LAY_DENSE) {
        for (int e = tid; e < nr * W; e += SUM_BLOCK) {
            const int r = e / W, k = e % W;
            const int a = A.alist ? A.alist[r0 + r] : r0 + r;
            at[e] = A.ax[(size_t)a * A.dpad + k];
        }
    } else {
        for (int r = 0; r < nr; ++r) {
            const int a = A.alist ? A.alist[r0 + r] : r0 + r;
            const int p0 = A.arp[a], p1 = A.arp[a + 1];
            for (int p = p0 + tid; p < p1; p += SUM_BLOCK) at[r * W + A.acol[p]] = A.aval[p];
        }
    }
    __syncthreads();
    if (LAY != LAY_DENSE) {
        // |a|^2 of each staged row
        for (int r = wid; r < nr; r += SUM_BLOCK / 64) {
            KT s = 0;
            for (int k = lane; k < W; k += 64) {
                KT v = (KT)at[r * W + k];
                s += v * v;
            }
            s = wave_sum(s);
            if (lane == 0) s_na[r] = (double)s;
        }
        __syncthreads();
    }

    double acc[SUM_RMAX];
#pragma unroll
    for (int r = 0; r < SUM_RMAX; ++r) acc[r] = 0.0;
    const KT gam = (KT)A.gamma;
    const int nb = A.nb;
    const int per = (nb + A.nsplit - 1) / A.nsplit;
    const int b0 = blockIdx.y * per, b1 = min(nb, b0 + per);
    for (int jb = b0 + tid; jb < b1; jb += SUM_BLOCK) {
        const int j = A.blist[jb];
        const double cj = A.coef[jb];
        KT dist[SUM_RMAX];
#pragma unroll
        for (int r = 0; r < SUM_RMAX; ++r) dist[r] = 0;
        if (LAY == LAY_DENSE) {
            const float4* xb = reinterpret_cast<const float4*>(A.bx + (size_t)j * A.dpad);
            for (int k4 = 0; k4 < A.dpad / 4; ++k4) {
                const float4 v = xb[k4];
#pragma unroll
                for (int r = 0; r < SUM_RMAX; ++r) {
                    if (r < nr) {
                        const float4 q = reinterpret_cast<const float4*>(at + r * W)[k4];
                        if constexpr (std::is_same<KT, double>::value) {
#pragma clang fp contract(off)
                            double t, s = dist[r];
                            t = (double)q.x - (double)v.x; s = s + t * t;
                            t = (double)q.y - (double)v.y; s = s + t * t;
                            t = (double)q.z - (double)v.z; s = s + t * t;
                            t = (double)q.w - (double)v.w; s = s + t * t;
                            dist[r] = s;
                        } else {
                            float t, s = dist[r];
                            t = q.x - v.x; s = fmaf(t, t, s);
                            t = q.y - v.y; s = fmaf(t, t, s);
                            t = q.z - v.z; s = fmaf(t, t, s);
                            t = q.w - v.w; s = fmaf(t, t, s);
                            dist[r] = s;
                        }
                    }
                }
            }
        } else {
            const int p0 = A.brp[j], p1 = A.brp[j + 1];
            KT nbn = 0;
            for (int p = p0; p < p1; ++p) {
                const int c = A.bcol[p];
                const KT v = (KT)A.bval[p];
                nbn += v * v;
#pragma unroll
                for (int r = 0; r < SUM_RMAX; ++r)
                    if (r < nr) dist[r] += v * (KT)at[r * W + c];
            }
#pragma unroll
            for (int r = 0; r < SUM_RMAX; ++r) {
                KT d2 = (KT)s_na[r < nr ? r : 0] + nbn - (KT)2 * dist[r];
                dist[r] = d2 < (KT)0 ? (KT)0 : d2;
            }
        }
#pragma unroll
        for (int r = 0; r < SUM_RMAX; ++r) {
            if (r < nr) {
                const double k = (double)kexp(-gam * dist[r]);
                acc[r] += cj * k;
            }
        }
    }
    // reduce acc[r] over the workgroup
#pragma unroll
    for (int r = 0; r < SUM_RMAX; ++r) {
        double v = wave_sum(acc[r]);
        if (lane == 0) s_red[wid][r] = v;
    }
    __syncthreads();
    if (tid < nr) {
        double v = 0.0;
        for (int w = 0; w < SUM_BLOCK / 64; ++w) v += s_red[w][tid];
        A.part[(size_t)blockIdx.y * A.na + r0 + tid] = v;
    }
}

// Large-d CSR: a few A rows at a time per workgroup, densified through a u16 slot map over
// the d columns (zeroed once, cleared sparsely after each group).
template <typename KT>
__global__ __launch_bounds__(SUM_BLOCK) void kernel_sum_slot_kernel(SumArgs A) {
    // R = A.slot_rows target rows at a time: slot[c] numbers the columns of their union
    // (1-based; 0 = in none of them) and tab[slot][r] holds row r's value there, so one pass
    // over a support vector's nonzeros serves all R rows
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_red[SUM_BLOCK / 64][SLOT_R_MAX];
    __shared__ double s_na[SLOT_R_MAX];
    __shared__ int s_u;
    const int R = A.slot_rows;
    uint16_t* slot = reinterpret_cast<uint16_t*>(smem);
    float* tab = reinterpret_cast<float*>(smem + ((sizeof(uint16_t) * (size_t)A.d + 15) & ~(size_t)15));
    const int tab_rows = 1 + R * A.rows_per_block;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    for (int k = tid; k < A.d; k += SUM_BLOCK) slot[k] = 0;
    for (int e = tid; e < tab_rows * R; e += SUM_BLOCK) tab[e] = 0.f;
    __syncthreads();
    const KT gam = (KT)A.gamma;
    const int per = (A.nb + A.nsplit - 1) / A.nsplit;
    const int b0 = blockIdx.y * per, b1 = min(A.nb, b0 + per);
    const int ngroups = (A.na + R - 1) / R;
    for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
        const int r0 = grp * R, nr = min(R, A.na - r0);
        // union of the group's columns: one thread per row claims slots in row order
        if (tid == 0) {
            int u = 0;
            for (int r = 0; r < nr; ++r) {
                const int a = A.alist ? A.alist[r0 + r] : r0 + r;
                for (int p = A.arp[a]; p < A.arp[a + 1]; ++p) {
                    const int c = A.acol[p];
                    int sl = slot[c];
                    if (!sl) { sl = ++u; slot[c] = (uint16_t)sl; }
                    tab[sl * R + r] = A.aval[p];
                }
            }
            s_u = u;
        }
        __syncthreads();
        if (tid < nr) {
            const int a = A.alist ? A.alist[r0 + tid] : r0 + tid;
            KT nn = 0;
            for (int p = A.arp[a]; p < A.arp[a + 1]; ++p) {
                const KT v = (KT)A.aval[p];
                nn += v * v;
            }
            s_na[tid] = (double)nn;
        }
        __syncthreads();
        double acc[SLOT_R_MAX];
#pragma unroll
        for (int r = 0; r < SLOT_R_MAX; ++r) acc[r] = 0.0;
        for (int jb = b0 + tid; jb < b1; jb += SUM_BLOCK) {
            const int j = A.blist[jb];
            const int q0 = A.brp[j], q1 = A.brp[j + 1];
            KT nb = 0, dot[SLOT_R_MAX];
#pragma unroll
            for (int r = 0; r < SLOT_R_MAX; ++r) dot[r] = 0;
            for (int q = q0; q < q1; ++q) {
                const KT v = (KT)A.bval[q];
                nb += v * v;
                const float* t = tab + (int)slot[A.bcol[q]] * R;
#pragma unroll
                for (int r = 0; r < SLOT_R_MAX; ++r)
                    if (r < R) dot[r] += v * (KT)t[r];
            }
#pragma unroll
            for (int r = 0; r < SLOT_R_MAX; ++r) {
                if (r < nr) {
                    KT d2 = (KT)s_na[r] + nb - (KT)2 * dot[r];
                    if (d2 < (KT)0) d2 = (KT)0;
                    acc[r] += A.coef[jb] * (double)kexp(-gam * d2);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < SLOT_R_MAX; ++r) {
            const double v = wave_sum(acc[r]);
            if (lane == 0) s_red[wid][r] = v;
        }
        __syncthreads();
        if (tid < nr) {
            double t = 0.0;
            for (int w = 0; w < SUM_BLOCK / 64; ++w) t += s_red[w][tid];
            A.part[(size_t)blockIdx.y * A.na + r0 + tid] = t;
        }
        // clear the group's slots and table rows for the next group
        if (tid == 0) {
            for (int r = 0; r < nr; ++r) {
                const int a = A.alist ? A.alist[r0 + r] : r0 + r;
                for (int p = A.arp[a]; p < A.arp[a + 1]; ++p) slot[A.acol[p]] = 0;
            }
        }
        for (int e = tid; e < (1 + s_u) * R; e += SUM_BLOCK) tab[e] = 0.f;
        __syncthreads();
    }
}

// Dense rows of up to 128 features, FP32 kernel values, on the matrix cores.  A workgroup (4 waves)
// takes 64 rows of A, 16 a wave, whose values stay in registers (K4 a lane and 16 rows), and
// sweeps its split of the B rows 64 at a time: the chunk goes to LDS (double-buffered, loaded one
// chunk ahead; [k / 4][row][4], so that a matrix operand is 64 consecutive words) with its norms and
// coefficients, each wave forms 16 x 16 blocks of dot products by v_mfma_f32_16x16x4f32 and applies
// d2 = |a|^2 + |b|^2 - 2 a.b (clamped at 0), exp(-gamma d2) and coef_b K into FP64 row sums.  Operand
// lanes: A[row][k] and B[k][col] sit in lane (row or col) + 16 k; output C[row][col] in lane
// col + 16 (row / 4), register row % 4.
// The products need 32 K4 cycles of a matrix core per 256 pairs and the epilogue about 51 vector
// instructions (280 cycles with the exponential and the conversions); the counters show the two adding up
// rather than overlapping, so what helps is less of either: norms come from a pass of their own (in the
// sweep they cost two barriers a chunk and 64 of 256 threads summing) and the rows' values from registers.
// 10,000 x 95,000 pairs, d = 28: 0.77 ms, against 1.33 with both tiles in LDS and the norms in the
// sweep; two 16-row blocks a wave, 0.85 (three waves a SIMD instead of five).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int MD_K4_MAX = 32;
constexpr int MD_CHUNK = 64;

template <int K4>
__global__ __launch_bounds__(SUM_BLOCK) void kernel_sum_dense_kernel(SumArgs A) {
    constexpr int NV = (K4 * MD_CHUNK + SUM_BLOCK - 1) / SUM_BLOCK;   // float4 of a chunk per thread
    __shared__ __align__(16) f32x4 s_b[2][K4][MD_CHUNK];
    __shared__ float s_nb[2][MD_CHUNK];
    __shared__ double s_cb[2][MD_CHUNK];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int m16 = lane & 15, mk = lane >> 4;
    const int n4 = A.dpad >> 2;
    const int r0 = blockIdx.x * KSUM_DENSE_ROWS + 16 * wid;   // the wave's first row
    float ar[K4], na[4];
    {
        const int r = r0 + m16;
        const float* src = r < A.na ? A.ax + (size_t)(A.alist ? A.alist[r] : r) * A.dpad : nullptr;
#pragma unroll
        for (int k = 0; k < K4; ++k) ar[k] = src && k < n4 ? src[4 * k + mk] : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = r0 + 4 * mk + i;
            na[i] = q < A.na ? A.anrm[A.alist ? A.alist[q] : q] : 0.f;
        }
    }
    const float gam = (float)A.gamma;
    // splits are whole chunks
    const int per = (A.nb + A.nsplit * MD_CHUNK - 1) / (A.nsplit * MD_CHUNK) * MD_CHUNK;
    const int b0 = min(A.nb, (int)blockIdx.y * per), b1 = min(A.nb, b0 + per);
    f32x4 hv[NV];
    float pn = 0.f;
    double pc = 0.0;
    auto load = [&](int c0) {   // chunk c0 into registers: lane l of a quad of waves takes row l
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int e = tid + SUM_BLOCK * v, k = e / MD_CHUNK, j = c0 + e % MD_CHUNK;
            hv[v] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (k < n4 && j < b1)
                hv[v] = reinterpret_cast<const f32x4*>(A.bx + (size_t)(A.blist ? A.blist[j] : j) * A.dpad)[k];
        }
        if (tid < MD_CHUNK) {
            const int j = c0 + tid;
            const bool in = j < b1;
            // (rows beyond the split: distance 0 would be NaN where gamma is infinite in FP32)
            pn = in ? A.bnrm[A.blist ? A.blist[j] : j] : 1.f;
            pc = in ? A.coef[j] : 0.0;
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int e = tid + SUM_BLOCK * v, k = e / MD_CHUNK;
            if (k < K4) s_b[buf][k][e % MD_CHUNK] = hv[v];
        }
        if (tid < MD_CHUNK) {
            s_nb[buf][tid] = pn;
            s_cb[buf][tid] = pc;
        }
    };
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (b0 < b1) {
        load(b0);
        store(0);
    }
    __syncthreads();
    int buf = 0;
    for (int c0 = b0; c0 < b1; c0 += MD_CHUNK, buf ^= 1) {
        const bool more = c0 + MD_CHUNK < b1;
        if (more) load(c0 + MD_CHUNK);
        auto block = [&](int cb) {   // 16 rows by columns 16 cb .. of the chunk
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < K4; ++k)
                d = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    ar[k], reinterpret_cast<const float*>(&s_b[buf][k][16 * cb + m16])[mk], d, 0, 0, 0);
            return d;
        };
        // a block's products run on the matrix core while the one before is reduced
        f32x4 d = block(0);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const f32x4 cur = d;
            if (cb < 3) d = block(cb + 1);
            const float nbc = s_nb[buf][16 * cb + m16];
            const double cbv = s_cb[buf][16 * cb + m16];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float d2 = na[i] + nbc - 2.f * cur[i];
                d2 = d2 < 0.f ? 0.f : d2;
                acc[i] += cbv * (double)kexp(-gam * d2);
            }
            if (cb < 3) {
#pragma unroll
                for (int k = 0; k < K4; ++k) {
                    __builtin_amdgcn_sched_group_barrier(0x008 /* matrix */, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002 /* vector ALU */, (48 + K4 - 1) / K4, 0);
                }
            }
        }
        if (more) store(buf ^ 1);
        __syncthreads();
    }
    // rows 4 mk + i of the wave: add the 16 lanes (columns) that share mk
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        double v = acc[i];
        v = xor_add<1>(v);
        v = xor_add<2>(v);
        v = xor_add<4>(v);
        v = xor_add<8>(v);
        const int r = r0 + 4 * mk + i;
        if (m16 == 0 && r < A.na) A.part[(size_t)blockIdx.y * A.na + r] = v;
    }
}

// |x|^2 of packed dense rows in feature order (FP32): two sets in one launch (n2 may be 0).
__global__ __launch_bounds__(256) void dense_norms_kernel(int n1, const float* __restrict__ x1, float* o1, int n2,
                                                          const float* __restrict__ x2, float* o2, int dpad) {
    int i = blockIdx.x * 256 + threadIdx.x;
    const float* x = x1;
    float* o = o1;
    if (i >= n1) {
        i -= n1;
        if (i >= n2) return;
        x = x2;
        o = o2;
    }
    const float4* r = reinterpret_cast<const float4*>(x + (size_t)i * dpad);
    float s = 0.f;
    for (int k = 0; k < dpad / 4; ++k) {
        const float4 v = r[k];
        s = fmaf(v.x, v.x, s);
        s = fmaf(v.y, v.y, s);
        s = fmaf(v.z, v.z, s);
        s = fmaf(v.w, v.w, s);
    }
    o[i] = s;
}

hipError_t launch_dense_norms(int n1, const float* x1, float* o1, int n2, const float* x2, float* o2, int dpad,
                              hipStream_t s) {
    const int64_t n = (int64_t)n1 + n2;
    if (n <= 0) return hipSuccess;
    dense_norms_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n1, x1, o1, n2, x2, o2, dpad);
    return hipGetLastError();
}

// Row width (in float4) of the instance for rows of dpad floats; 0: none
static int dense_sum_width(int dpad) {
    static const int w[] = {1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 24, 32};
    for (int k : w)
        if (4 * k >= dpad) return k;
    return 0;
}
static const void* dense_sum_pick(int k4) {
    switch (k4) {
        case 1: return (const void*)kernel_sum_dense_kernel<1>;
        case 2: return (const void*)kernel_sum_dense_kernel<2>;
        case 3: return (const void*)kernel_sum_dense_kernel<3>;
        case 4: return (const void*)kernel_sum_dense_kernel<4>;
        case 5: return (const void*)kernel_sum_dense_kernel<5>;
        case 6: return (const void*)kernel_sum_dense_kernel<6>;
        case 7: return (const void*)kernel_sum_dense_kernel<7>;
        case 8: return (const void*)kernel_sum_dense_kernel<8>;
        case 12: return (const void*)kernel_sum_dense_kernel<12>;
        case 16: return (const void*)kernel_sum_dense_kernel<16>;
        case 24: return (const void*)kernel_sum_dense_kernel<24>;
        case 32: return (const void*)kernel_sum_dense_kernel<32>;
        default: return nullptr;
    }
}

bool kernel_sum_uses_norms(int lay, int dpad, int kprec) {
    return lay == LAY_DENSE && kprec == SVM_KERNEL_FP32 && dpad <= 4 * MD_K4_MAX;
}
// Dense rows beyond that, FP32 kernel values: both sides' tiles in LDS.  A
// workgroup (4 waves) holds 64 A rows in LDS and sweeps its split of the B list 64 rows at a
// time; wave w forms the 16 x 64 block of dot products of A rows 16w.. with the chunk through
// v_mfma_f32_16x16x4f32 (a 16x4 by 4x16 product per instruction, K = dpad in steps of 4), then
// applies the epilogue d2 = |a|^2 + |b|^2 - 2 a.b (clamped at 0), exp(-gamma d2), and adds
// coef_b * K into FP64 row sums.
constexpr int MF_T = 64;              // A rows per workgroup, B rows per chunk
constexpr int MF_MAX_DPAD = 240;      // LDS: 2 x 64 rows x (dpad + 1) floats

__global__ __launch_bounds__(SUM_BLOCK) void kernel_sum_mfma_kernel(SumArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float s_na[MF_T], s_nb[MF_T];
    __shared__ double s_cb[MF_T];
    const int dpad = A.dpad, S = dpad + 1;       // odd row stride: column reads hit distinct banks
    float* at = reinterpret_cast<float*>(smem);
    float* bt = at + MF_T * S;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int r0 = blockIdx.x * MF_T;
    const int nr = min(MF_T, A.na - r0);
    for (int e = tid; e < MF_T * dpad; e += SUM_BLOCK) {
        const int r = e / dpad, k = e % dpad;
        float v = 0.f;
        if (r < nr) v = A.ax[(size_t)(A.alist ? A.alist[r0 + r] : r0 + r) * dpad + k];
        at[r * S + k] = v;
    }
    __syncthreads();
    if (tid < MF_T) {
        float sq = 0.f;
        for (int k = 0; k < dpad; ++k) sq = fmaf(at[tid * S + k], at[tid * S + k], sq);
        s_na[tid] = sq;
    }
    const float gam = (float)A.gamma;
    const int per = (A.nb + A.nsplit - 1) / A.nsplit;
    const int b0 = blockIdx.y * per, b1 = min(A.nb, b0 + per);
    const int mrow = lane & 15, mk = lane >> 4;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int c0 = b0; c0 < b1; c0 += MF_T) {
        const int nc = min(MF_T, b1 - c0);
        __syncthreads();                          // the previous chunk is no longer read
        for (int e = tid; e < MF_T * dpad; e += SUM_BLOCK) {
            const int c = e / dpad, k = e % dpad;
            bt[c * S + k] = c < nc ? A.bx[(size_t)A.blist[c0 + c] * dpad + k] : 0.f;
        }
        if (tid < MF_T) s_cb[tid] = tid < nc ? A.coef[c0 + tid] : 0.0;
        __syncthreads();
        if (tid < MF_T) {
            float sq = 0.f;
            for (int k = 0; k < dpad; ++k) sq = fmaf(bt[tid * S + k], bt[tid * S + k], sq);
            s_nb[tid] = tid < nc ? sq : 1.f;   // (rows beyond the end: as in kernel_sum_dense_kernel)
        }
        __syncthreads();
        const float* arow = at + (16 * wid + mrow) * S + mk;
        for (int cb = 0; cb < 4; ++cb) {
            const float* brow = bt + (16 * cb + mrow) * S + mk;
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
            for (int k4 = 0; k4 < dpad; k4 += 4)
                d = __builtin_amdgcn_mfma_f32_16x16x4f32(arow[k4], brow[k4], d, 0, 0, 0);
            const int col = 16 * cb + mrow;
            const float nbc = s_nb[col];
            const double cbv = s_cb[col];
            const float dv[4] = {d[0], d[1], d[2], d[3]};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * wid + 4 * mk + i;
                float d2 = s_na[row] + nbc - 2.f * dv[i];
                d2 = d2 < 0.f ? 0.f : d2;
                acc[i] += cbv * (double)kexp(-gam * d2);
            }
        }
    }
    // rows 16 wid + 4 mk + i: add the 16 lanes (columns) that share mk
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        double v = acc[i];
        for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o);
        const int row = 16 * wid + 4 * mk + i;
        if (mrow == 0 && row < nr) A.part[(size_t)blockIdx.y * A.na + r0 + row] = v;
    }
}

// Binary rows as bitsets (LAY_BITS): the intersections |a & b| are products of 0/1 bytes on the matrix
// cores (v_mfma_i32_16x16x64_i8, exact), the squared distance |a| + |b| - 2 |a & b| = |a ^ b| is a whole
// number of at most d, and the kernel value comes from a table over those, formed once per workgroup by the
// expression the other kernels use: no exponential per pair, in FP64 none of its 40 instructions either.
// A workgroup (4 waves) takes 64 RT rows of A, whose bytes stay in registers (lane (row, g) holds bits
// 64 s + 16 g .. of its row for step s; B alike, so the order of the columns does not matter), and sweeps
// its split of the B rows 64 at a time through LDS, expanded to bytes there ([step][g][row] in 16-byte
// words, four threads a row, which also count its bits), double-buffered and loaded one chunk ahead.
// Output lanes as in kernel_sum_dense_kernel.  What bounds it is the table read and the FP64 sum of each
// pair.  10,000 x 24,000 pairs, d = 300: 146 us, against 315 with popcounts and an exponential per pair.
constexpr int MB_CHUNK = 64;
typedef int i32x4 __attribute__((ext_vector_type(4)));

// 16 bits to 16 bytes of 0 or 1
DEV i32x4 bits_to_bytes(uint32_t h) {
    i32x4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = (int)(__umul24((h >> (4 * q)) & 15u, 0x204081u) & 0x01010101u);
    return r;
}

// dynamic LDS: the table, then two buffers of a chunk's bytes, bit counts and coefficients
// (distances 0 .. d; rows beyond the split have one bit and no column: up to d + 1)
__host__ __device__ constexpr int mb_table_entries(int d) { return d + 2; }
constexpr size_t mb_table_bytes(int d) { return ((size_t)mb_table_entries(d) * sizeof(double) + 15) & ~(size_t)15; }
constexpr size_t mb_buffer_bytes(int NS) {
    return (size_t)NS * 4 * MB_CHUNK * 16 + MB_CHUNK * (sizeof(int) + sizeof(double));
}

template <typename KT, int NS, int RT>
__global__ __launch_bounds__(SUM_BLOCK) void kernel_sum_bits_kernel(SumArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* tab = reinterpret_cast<double*>(smem);
    const size_t tb = mb_table_bytes(A.d);
    auto bytes = [&](int buf) { return reinterpret_cast<i32x4*>(smem + tb + buf * mb_buffer_bytes(NS)); };
    auto coefs = [&](int buf) { return reinterpret_cast<double*>(bytes(buf) + NS * 4 * MB_CHUNK); };
    auto counts = [&](int buf) { return reinterpret_cast<int*>(coefs(buf) + MB_CHUNK); };
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int m16 = lane & 15, mk = lane >> 4;
    const int wpr = A.wpr;
    const KT gam = (KT)A.gamma;
    for (int k = tid; k < mb_table_entries(A.d); k += SUM_BLOCK) tab[k] = (double)kexp((KT)(-gam * (KT)k));
    const int r0 = blockIdx.x * 64 * RT + 16 * RT * wid;   // the wave's first row
    i32x4 ar[RT][NS];
    int na[RT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int r = r0 + 16 * t + m16;
        const bool in = r < A.na;
        const uint32_t* row = A.abits + (size_t)(in ? (A.alist ? A.alist[r] : r) : 0) * wpr;
        int c = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int w = 2 * s + (mk >> 1);
            const uint32_t h = in && w < wpr ? (row[w] >> (16 * (mk & 1))) & 0xffffu : 0u;
            c += __popc(h);
            ar[t][s] = bits_to_bytes(h);
        }
        c = xor_add<16>(c);
        c = xor_add<32>(c);   // |a| of row m16, in every lane of that row
#pragma unroll
        for (int i = 0; i < 4; ++i) na[t][i] = __shfl(c, 4 * mk + i);
    }
    // splits are whole chunks
    const int per = (A.nb + A.nsplit * MB_CHUNK - 1) / (A.nsplit * MB_CHUNK) * MB_CHUNK;
    const int b0 = min(A.nb, (int)blockIdx.y * per), b1 = min(A.nb, b0 + per);
    constexpr int NW = (2 * NS + 3) / 4;   // words of a row per thread
    const int brow = tid >> 2, bsub = tid & 3;
    uint32_t hw[NW];
    double pc = 0.0;
    int pad = 0;   // rows beyond the split count one bit: distance 0 is NaN where gamma is infinite in FP32
    auto load = [&](int c0) {
        const int j = c0 + brow;
        const bool in = j < b1;
        const uint32_t* row = A.bbits + (size_t)(in ? A.blist[j] : 0) * wpr;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int w = bsub + 4 * k;
            hw[k] = in && w < wpr ? row[w] : 0u;
        }
        pad = in ? 0 : 1;
        pc = in ? A.coef[j] : 0.0;
    };
    auto store = [&](int buf) {
        int c = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int w = bsub + 4 * k;
            if (w < 2 * NS) {
                i32x4* dst = bytes(buf) + (size_t)(2 * w) * MB_CHUNK + brow;
                dst[0] = bits_to_bytes(hw[k] & 0xffffu);
                dst[MB_CHUNK] = bits_to_bytes(hw[k] >> 16);
            }
            c += __popc(hw[k]);
        }
        c = xor_add<1>(c);
        c = xor_add<2>(c);
        if (bsub == 0) {
            counts(buf)[brow] = c + pad;
            coefs(buf)[brow] = pc;
        }
    };
    double acc[RT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][i] = 0.0;
    if (b0 < b1) {
        load(b0);
        store(0);
    }
    __syncthreads();
    int buf = 0;
    for (int c0 = b0; c0 < b1; c0 += MB_CHUNK, buf ^= 1) {
        const bool more = c0 + MB_CHUNK < b1;
        if (more) load(c0 + MB_CHUNK);
        const i32x4* by = bytes(buf);
        const int* cn = counts(buf);
        const double* cf = coefs(buf);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const int col = 16 * cb + m16;
            i32x4 d[RT];
#pragma unroll
            for (int t = 0; t < RT; ++t) d[t] = i32x4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const i32x4 bv = by[(size_t)(4 * s + mk) * MB_CHUNK + col];
#pragma unroll
                for (int t = 0; t < RT; ++t) d[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[t][s], bv, d[t], 0, 0, 0);
            }
            const int nbc = cn[col];
            const double cbv = cf[col];   // (0 beyond the split's rows)
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[t][i] += cbv * tab[na[t][i] + nbc - 2 * d[t][i]];
        }
        if (more) store(buf ^ 1);
        __syncthreads();
    }
    // rows 16 t + 4 mk + i of the wave: add the 16 lanes (columns) that share mk
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = acc[t][i];
            v = xor_add<1>(v);
            v = xor_add<2>(v);
            v = xor_add<4>(v);
            v = xor_add<8>(v);
            const int r = r0 + 16 * t + 4 * mk + i;
            if (m16 == 0 && r < A.na) A.part[(size_t)blockIdx.y * A.na + r] = v;
        }
}

// Steps of 64 columns of the instance for d columns, and rows of A per workgroup
static int bits_sum_steps(int d) {
    static const int n[] = {1, 2, 3, 4, 5, 6, 8, 12, 16};
    for (int k : n)
        if (64 * k >= d) return k;
    return 0;
}
// (two 16-row blocks a wave share the reads of B: 146 us against 173 with one; beyond 384 columns their
// bytes would take the registers of a second wave per SIMD)
int kernel_sum_bits_rows(int d) { return bits_sum_steps(d) <= 6 ? 128 : 64; }
template <typename KT>
static const void* bits_sum_pick(int ns) {
    switch (ns) {
        case 1: return (const void*)kernel_sum_bits_kernel<KT, 1, 2>;
        case 2: return (const void*)kernel_sum_bits_kernel<KT, 2, 2>;
        case 3: return (const void*)kernel_sum_bits_kernel<KT, 3, 2>;
        case 4: return (const void*)kernel_sum_bits_kernel<KT, 4, 2>;
        case 5: return (const void*)kernel_sum_bits_kernel<KT, 5, 2>;
        case 6: return (const void*)kernel_sum_bits_kernel<KT, 6, 2>;
        case 8: return (const void*)kernel_sum_bits_kernel<KT, 8, 1>;
        case 12: return (const void*)kernel_sum_bits_kernel<KT, 12, 1>;
        case 16: return (const void*)kernel_sum_bits_kernel<KT, 16, 1>;
        default: return nullptr;
    }
}

int slot_rows_for(int d, int max_nnz) {
    const size_t budget = 150 * 1024;
    const size_t base = (sizeof(uint16_t) * (size_t)d + 15) & ~(size_t)15;
    for (int r = SLOT_R_MAX; r > 1; r /= 2)
        if (base + sizeof(float) * (size_t)(1 + r * max_nnz) * r <= budget) return r;
    return 1;
}

bool kernel_sum_uses_mfma(int lay, int dpad, int kprec) {
    return lay == LAY_DENSE && kprec == SVM_KERNEL_FP32 && dpad <= MF_MAX_DPAD;
}

hipError_t launch_kernel_sum(const SumArgs& a, int kprec, hipStream_t s) {
    if (a.na <= 0) return hipSuccess;
    if (a.lay == LAY_BITS) {
        const int ns = bits_sum_steps(a.d);
        const void* fn = kprec == SVM_KERNEL_FP64 ? bits_sum_pick<double>(ns) : bits_sum_pick<float>(ns);
        if (!fn || a.wpr != bits_wpr(a.d)) return hipErrorInvalidValue;
        const size_t lds = mb_table_bytes(a.d) + 2 * mb_buffer_bytes(ns);
        if (lds > 64 * 1024) {
            const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        const int rows = kernel_sum_bits_rows(a.d);
        SumArgs c = a;
        void* args[] = {&c};
        return hipLaunchKernel(fn, dim3((a.na + rows - 1) / rows, a.nsplit), dim3(SUM_BLOCK), args, lds, s);
    }
    if (kernel_sum_uses_norms(a.lay, a.dpad, kprec)) {
        const void* fn = dense_sum_pick(dense_sum_width(a.dpad));
        if (!fn || !a.anrm || !a.bnrm) return hipErrorInvalidValue;
        SumArgs c = a;
        void* args[] = {&c};
        return hipLaunchKernel(fn, dim3((a.na + a.rows_per_block - 1) / a.rows_per_block, a.nsplit), dim3(SUM_BLOCK),
                               args, 0, s);
    }
    if (kernel_sum_uses_mfma(a.lay, a.dpad, kprec)) {
        const size_t lds = sizeof(float) * 2 * MF_T * (size_t)(a.dpad + 1);
        dim3 grid((a.na + MF_T - 1) / MF_T, a.nsplit);
        SumArgs c = a;
        (void)hipFuncSetAttribute((const void*)kernel_sum_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        kernel_sum_mfma_kernel<<<grid, SUM_BLOCK, lds, s>>>(c);
        return hipGetLastError();
    }
    if (a.lay == LAY_CSR_SLOT) {
        // rows_per_block carries the longest A row here, slot_rows the rows per group
        const size_t lds = ((sizeof(uint16_t) * (size_t)a.d + 15) & ~(size_t)15) +
                           sizeof(float) * (size_t)(1 + a.slot_rows * a.rows_per_block) * a.slot_rows;
        dim3 grid(std::min((a.na + a.slot_rows - 1) / a.slot_rows, 2048), a.nsplit);
        SumArgs c = a;
        if (kprec == SVM_KERNEL_FP64) {
            (void)hipFuncSetAttribute((const void*)kernel_sum_slot_kernel<double>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_slot_kernel<double><<<grid, SUM_BLOCK, lds, s>>>(c);
        } else {
            (void)hipFuncSetAttribute((const void*)kernel_sum_slot_kernel<float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_slot_kernel<float><<<grid, SUM_BLOCK, lds, s>>>(c);
        }
        return hipGetLastError();
    }
    const int W = a.lay == LAY_DENSE ? a.dpad : a.d;
    const size_t lds = sizeof(float) * (size_t)a.rows_per_block * W;
    dim3 grid((a.na + a.rows_per_block - 1) / a.rows_per_block, a.nsplit);
    SumArgs c = a;
    if (kprec == SVM_KERNEL_FP64) {
        if (a.lay == LAY_DENSE) {
            if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kernel_sum_kernel<LAY_DENSE, double>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_kernel<LAY_DENSE, double><<<grid, SUM_BLOCK, lds, s>>>(c);
        } else {
            if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kernel_sum_kernel<LAY_CSR_TABLE, double>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_kernel<LAY_CSR_TABLE, double><<<grid, SUM_BLOCK, lds, s>>>(c);
        }
    } else {
        if (a.lay == LAY_DENSE) {
            if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kernel_sum_kernel<LAY_DENSE, float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_kernel<LAY_DENSE, float><<<grid, SUM_BLOCK, lds, s>>>(c);
        } else {
            if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kernel_sum_kernel<LAY_CSR_TABLE, float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_kernel<LAY_CSR_TABLE, float><<<grid, SUM_BLOCK, lds, s>>>(c);
        }
    }
    return hipGetLastError();
}

// Kernel sums from the whole kernel matrix in memory (K(b, a) at kmat[b * ldk + a]): one thread
// per target row a, its split of the B list in order, eight matrix rows in flight per thread.
// The rows of B are read contiguously along a, so a workgroup reads 1 KB per support vector.
__global__ __launch_bounds__(256) void kmat_sum_kernel(int na, const int32_t* __restrict__ alist, int nb,
                                                       const int32_t* __restrict__ blist,
                                                       const double* __restrict__ coef,
                                                       const float* __restrict__ kmat, long long ldk, double* part) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    const int per = (nb + gridDim.y - 1) / gridDim.y;
    const int b0 = blockIdx.y * per, b1 = min(nb, b0 + per);
    if (r >= na) return;
    const int a = alist ? alist[r] : r;
    double acc = 0.0;
    int j = b0;
    for (; j + 8 <= b1; j += 8) {
        float k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) k[u] = kmat[(size_t)blist[j + u] * ldk + a];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += coef[j + u] * (double)k[u];
    }
    for (; j < b1; ++j) acc += coef[j] * (double)kmat[(size_t)blist[j] * ldk + a];
    part[(size_t)blockIdx.y * na + r] = acc;
}

hipError_t launch_kmat_sum(int na, const int32_t* alist, int nb, const int32_t* blist, const double* coef,
                           const float* kmat, long long ldk, int nsplit, double* part, hipStream_t s) {
    if (na <= 0) return hipSuccess;
    const dim3 grid((na + 255) / 256, nsplit);
    kmat_sum_kernel<<<grid, 256, 0, s>>>(na, alist, nb, blist, coef, kmat, ldk, part);
    return hipGetLastError();
}

__global__ void finish_sum_kernel(int na, int nsplit, const double* __restrict__ part, const int32_t* __restrict__ alist,
                                  const int8_t* __restrict__ y, double beta, double* out) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= na) return;
    double v = 0.0;
    for (int s = 0; s < nsplit; ++s) v += part[(size_t)s * na + r];
    const int a = alist ? alist[r] : r;
    out[a] = v - (y ? (y[a] > 0 ? 1.0 : -1.0) : beta);
}

hipError_t launch_finish_sum(int na, int nsplit, const double* part, const int32_t* alist, const int8_t* y, double beta,
                             double* out, hipStream_t s) {
    if (na <= 0) return hipSuccess;
    finish_sum_kernel<<<(na + 255) / 256, 256, 0, s>>>(na, nsplit, part, alist, y, beta, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ closing reductions

__global__ __launch_bounds__(256) void summary_partial_kernel(int n, const double* __restrict__ alpha,
                                                              const double* __restrict__ f,
                                                              const int8_t* __restrict__ y, double C, double* blk) {
    __shared__ double s[6][4];
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const double a = alpha[i];
        const double yi = y[i] > 0 ? 1.0 : -1.0;
        if (a > 0.0 && a < C) { v[0] += f[i]; v[1] += 1.0; }
        v[2] += a;
        v[3] += a * yi * (f[i] + yi);
        if (a > 0.0) v[4] += 1.0;
        if (a >= C) v[5] += 1.0;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        double t = wave_sum(v[k]);
        if (lane == 0) s[k][wid] = t;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        double t = 0.0;
        for (int w = 0; w < 4; ++w) t += s[threadIdx.x][w];
        blk[blockIdx.x * 6 + threadIdx.x] = t;
    }
}

// The parts come into LDS side by side and are added in their order from there: 34.6 us when each of six
// threads loaded and added its 256 parts one behind the other.
constexpr int SUMMARY_BLOCKS = 256;
__global__ __launch_bounds__(SUMMARY_BLOCKS) void summary_final_kernel(const double* __restrict__ blk, double* out6) {
    __shared__ double s[6 * SUMMARY_BLOCKS];
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k * SUMMARY_BLOCKS + threadIdx.x] = blk[k * SUMMARY_BLOCKS + threadIdx.x];
    __syncthreads();
    if (threadIdx.x < 6) {
        double t = 0.0;
#pragma unroll 16
        for (int b = 0; b < SUMMARY_BLOCKS; ++b) t += s[b * 6 + threadIdx.x];
        out6[threadIdx.x] = t;
    }
}

hipError_t launch_summary(int n, const double* alpha, const double* f, const int8_t* y, double C, double* blk,
                          double* out6, hipStream_t s) {
    summary_partial_kernel<<<SUMMARY_BLOCKS, 256, 0, s>>>(n, alpha, f, y, C, blk);
    summary_final_kernel<<<1, SUMMARY_BLOCKS, 0, s>>>(blk, out6);
    return hipGetLastError();
}

__global__ void check_pattern_kernel(int nnz, const float* __restrict__ val, int32_t* flag) {
    int bad = 0;
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += gridDim.x * blockDim.x)
        if (val[p] != 1.0f) bad = 1;
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

hipError_t launch_check_pattern(int nnz, const float* val, int32_t* flag, hipStream_t s) {
    hipError_t e = hipMemsetAsync(flag, 0, sizeof(int32_t), s);
    if (e != hipSuccess || nnz <= 0) return e;
    check_pattern_kernel<<<512, 256, 0, s>>>(nnz, val, flag);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void pack_pairs_kernel(int n, const int32_t* __restrict__ rp,
                                                         const int32_t* __restrict__ prp,
                                                         const int32_t* __restrict__ col,
                                                         const float* __restrict__ val, int pattern_only,
                                                         uint16_t* col16, float* val2) {
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4), sub = threadIdx.x & 15;   // 16 threads per row
    if (i >= n) return;
    const int p0 = rp[i], len = rp[i + 1] - p0;
    const int64_t o = 2 * (int64_t)prp[i];
    for (int k = sub; k < len; k += 16) {
        col16[o + k] = (uint16_t)col[p0 + k];
        val2[o + k] = pattern_only ? 1.f : val[p0 + k];
    }
    if ((len & 1) && sub == 0) {
        col16[o + len] = (uint16_t)0;
        val2[o + len] = 0.f;
    }
}

hipError_t launch_pack_pairs(int n, const int32_t* rp, const int32_t* prp, const int32_t* col, const float* val,
                             int pattern_only, uint16_t* col16, float* val2, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    pack_pairs_kernel<<<(n + 15) / 16, 256, 0, s>>>(n, rp, prp, col, val, pattern_only, col16, val2);
    return hipGetLastError();
}

}  // namespace svm
