// svm_ksum_ht.hip -- kernel sums over wide sparse rows (Alg. 6 gradient reconstruction, the
// closing recompute and the classifier of eq:classi) with the dot products split by column
// frequency: the H most frequent columns of the training set form a dense "head" row per
// sample, multiplied on the matrix cores; the remaining "tail" nonzeros are matched through a
// bitmap of the target rows' tail columns in LDS.  Both parts are sums of FP32 products:
// the head on the matrix cores, the tail exactly in 64-bit fixed point (so its sum does not
// depend on the order in which threads add); the squared distance is
// |a|^2 + |b|^2 - 2 (a_h.b_h + a_t.b_t) as in the other FP32 kernel sums.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "svm_device.h"
#include "svm_internal.h"

namespace svm {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ preparation

// Occurrences of every column over the nonzeros of a CSR matrix (cnt zeroed by the caller).  Each
// workgroup counts its share in LDS, 16 bits a column (a share has fewer elements than that holds), and
// adds what it found, from a place of its own on: the frequent columns come up in every row, and an
// atomic in memory for each of 3.75 million text-like nonzeros took 631 us (now 35).
constexpr int COUNT_SHARE = 65535;
constexpr int COUNT_BLOCK = 1024;
__global__ __launch_bounds__(COUNT_BLOCK) void col_count_kernel(int64_t nnz, int d, const int32_t* __restrict__ col,
                                                                int32_t* cnt) {
    extern __shared__ uint32_t s_half[];   // two columns a word
    const int words = (d + 1) >> 1;
    for (int k = threadIdx.x; k < words; k += COUNT_BLOCK) s_half[k] = 0u;
    __syncthreads();
    const int64_t p0 = (int64_t)blockIdx.x * COUNT_SHARE;
    const int m = (int)min((int64_t)COUNT_SHARE, nnz - p0);
#pragma unroll 4
    for (int k = threadIdx.x; k < m; k += COUNT_BLOCK) {
        const int c = col[p0 + k];
        atomicAdd(&s_half[c >> 1], 1u << (16 * (c & 1)));
    }
    __syncthreads();
    const int turn = (int)((long long)words * blockIdx.x / gridDim.x);
    for (int j = threadIdx.x; j < words; j += COUNT_BLOCK) {
        const int k = j + turn < words ? j + turn : j + turn - words;
        const uint32_t v = s_half[k];
        if (v & 0xffffu) atomicAdd(&cnt[2 * k], (int)(v & 0xffffu));
        if (v >> 16) atomicAdd(&cnt[2 * k + 1], (int)(v >> 16));
    }
}

hipError_t launch_col_count(int64_t nnz, int d, const int32_t* col, int32_t* cnt, hipStream_t s) {
    if (nnz <= 0) return hipSuccess;
    const size_t lds = sizeof(uint32_t) * (size_t)((d + 1) / 2);   // d <= HT_MAX_D: at most 128 KB
    if (d < 1 || d > HT_MAX_D) return hipErrorInvalidValue;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)col_count_kernel,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    col_count_kernel<<<(unsigned)((nnz + COUNT_SHARE - 1) / COUNT_SHARE), COUNT_BLOCK, lds, s>>>(nnz, d, col, cnt);
    return hipGetLastError();
}

// The h most frequent of the d columns (ties to the lower id) become the head, in that order: hmap[c] =
// position of column c, -1 for the tail; hbits as a bitmap.  One workgroup, 64 counts a thread (63 of them
// in scratch memory, as a lane of 1024 threads has 128 registers; each step of the bisections reads them
// again: 94 us for 47,000 columns): the h-th largest count by bisection, of the columns that have it the
// lowest ids by another one, and each of the h selected finds its place among them.
constexpr int HEAD_BLOCK = 1024;
__global__ __launch_bounds__(HEAD_BLOCK) void ht_choose_kernel(int d, int h, const int32_t* __restrict__ cnt,
                                                               int32_t* hmap, uint32_t* hbits) {
    constexpr int PER = (HT_MAX_D + HEAD_BLOCK) / HEAD_BLOCK;
    __shared__ int s_w[HEAD_BLOCK / 64];
    __shared__ int s_id[HT_H_MAX], s_cnt[HT_H_MAX], s_n;
    __shared__ uint32_t s_bits[HT_MAX_WORDS];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int v[PER];
    int top = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int c = k * HEAD_BLOCK + tid;
        v[k] = c < d ? cnt[c] : -1;
        top = max(top, v[k]);
    }
    for (int k = tid; k < HT_MAX_WORDS; k += HEAD_BLOCK) s_bits[k] = 0u;
    if (tid == 0) s_n = 0;
    auto total = [&](int x) -> int {   // over the workgroup
        const int t = wave_sum(x);
        __syncthreads();
        if (lane == 0) s_w[wid] = t;
        __syncthreads();
        int r = 0;
#pragma unroll
        for (int w = 0; w < HEAD_BLOCK / 64; ++w) r += s_w[w];
        return r;
    };
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) top = max(top, __shfl_xor(top, off));
    if (lane == 0) s_w[wid] = top;
    __syncthreads();
    for (int w = 0; w < HEAD_BLOCK / 64; ++w) top = max(top, s_w[w]);
    // the largest count T that at least h columns reach (every column reaches 0)
    int lo = 0, hi = top;
    while (lo < hi) {
        const int mid = lo + (hi - lo + 1) / 2;
        int n = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) n += v[k] >= mid ? 1 : 0;
        if (total(n) >= h) lo = mid;
        else hi = mid - 1;
    }
    const int T = lo;
    int n = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) n += v[k] > T ? 1 : 0;
    const int want = h - total(n);   // columns with count T, the lowest ids: those up to B
    int bl = 0, bh = d - 1;
    while (bl < bh) {
        const int mid = (bl + bh) / 2;
        n = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) n += v[k] == T && k * HEAD_BLOCK + tid <= mid ? 1 : 0;
        if (total(n) >= want) bh = mid;
        else bl = mid + 1;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int c = k * HEAD_BLOCK + tid;
        if (v[k] > T || (want > 0 && v[k] == T && c <= bl)) {
            const int at = atomicAdd(&s_n, 1);
            s_id[at] = c;
            s_cnt[at] = v[k];
            atomicOr(&s_bits[c >> 5], 1u << (c & 31));
        }
        if (c < d) hmap[c] = -1;
    }
    __syncthreads();
    if (tid < h) {
        const int id = s_id[tid], ct = s_cnt[tid];
        int at = 0;
        for (int j = 0; j < h; ++j) at += s_cnt[j] > ct || (s_cnt[j] == ct && s_id[j] < id) ? 1 : 0;
        hmap[id] = at;
    }
    for (int k = tid; k < HT_MAX_WORDS; k += HEAD_BLOCK) hbits[k] = s_bits[k];
}

hipError_t launch_ht_choose(int d, int H, const int32_t* cnt, int32_t* hmap, uint32_t* hbits, hipStream_t s) {
    if (d < 1 || d > HT_MAX_D || H > HT_H_MAX) return hipErrorInvalidValue;
    ht_choose_kernel<<<1, HEAD_BLOCK, 0, s>>>(d, H < d ? H : d, cnt, hmap, hbits);
    return hipGetLastError();
}

// Value of lane k of each row of 16 lanes.
template <int K>
DEV float row_lane(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 /* row_newbcast:0 */ + K,
                                                                 0xF, 0xF, false));
}

// Per row i (16 threads): head[i][0..H) = the row's values in the head columns (hmap[c] >= 0
// gives the position), zero elsewhere; nrm[i] = |x_i|^2 summed in CSR order in FP32 (the 16 lanes hold
// 16 elements, broadcast one after the other); tcnt[i] = its tail nonzeros.  maxn2 receives the largest
// |x_i|^2 (bits of a non-negative float).  50,000 and 10,000 text-like rows 38 against 246 us with the sum
// and the atomic in one lane of each row.
__global__ __launch_bounds__(256) void ht_split_kernel(int n, int H, const int32_t* __restrict__ rp,
                                                       const int32_t* __restrict__ col,
                                                       const float* __restrict__ val,
                                                       const int32_t* __restrict__ hmap, float* head, float* nrm,
                                                       int32_t* tcnt, unsigned* maxn2) {
    __shared__ unsigned s_max;
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4), sub = threadIdx.x & 15;
    const bool ok = i < n;
    float* h = head + (size_t)i * H;
    if (threadIdx.x == 0) s_max = 0u;
    if (ok)
        for (int k = sub; k < H; k += 16) h[k] = 0.f;
    __syncthreads();   // zeros before values
    const int p0 = ok ? rp[i] : 0, p1 = ok ? rp[i + 1] : 0;
    float s = 0.f;
    int t = 0;
    for (int pb = p0; pb < p1; pb += 16) {
        const int p = pb + sub;
        const bool in = p < p1;
        const float v = in ? val[p] : 0.f;   // zeros beyond the row add nothing
        if (in) {
            const int k = hmap[col[p]];
            if (k >= 0) h[k] = v;
            else ++t;
        }
        auto add = [&](float x) { s = fmaf(x, x, s); };
        add(row_lane<0>(v)); add(row_lane<1>(v)); add(row_lane<2>(v)); add(row_lane<3>(v));
        add(row_lane<4>(v)); add(row_lane<5>(v)); add(row_lane<6>(v)); add(row_lane<7>(v));
        add(row_lane<8>(v)); add(row_lane<9>(v)); add(row_lane<10>(v)); add(row_lane<11>(v));
        add(row_lane<12>(v)); add(row_lane<13>(v)); add(row_lane<14>(v)); add(row_lane<15>(v));
    }
    t = lanes_sum<16>(t);
    if (ok && sub == 0) {
        nrm[i] = s;
        tcnt[i] = t;
        atomicMax(&s_max, __float_as_uint(s));
    }
    __syncthreads();
    // (an atomic in one place only where it can raise it)
    if (threadIdx.x == 0 && s_max > __hip_atomic_load(maxn2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(maxn2, s_max);
}

hipError_t launch_ht_split(int n, int H, const int32_t* rp, const int32_t* col, const float* val,
                           const int32_t* hmap, float* head, float* nrm, int32_t* tcnt, unsigned* maxn2,
                           hipStream_t s) {
    if (n <= 0) return hipSuccess;
    ht_split_kernel<<<(n + 15) / 16, 256, 0, s>>>(n, H, rp, col, val, hmap, head, nrm, tcnt, maxn2);
    return hipGetLastError();
}

// Largest number of tail nonzeros in any tile of 64, 32 and 16 consecutive target rows
// (out3[0..2], zeroed by the caller): the host takes the largest tile whose tail fits the
// kernel's LDS table.
__global__ __launch_bounds__(256) void ht_tiles_kernel(int na, const int32_t* __restrict__ alist,
                                                       const int32_t* __restrict__ tcnt, int32_t* out3) {
    const int lane = threadIdx.x & 63;
    int m64 = 0, m32 = 0, m16 = 0;
    // one wave per tile of 64 rows
    for (int t = blockIdx.x * 4 + (threadIdx.x >> 6); t * 64 < na; t += gridDim.x * 4) {
        const int k = t * 64 + lane;
        const int s16 = lanes_sum<16>(k < na ? tcnt[alist ? alist[k] : k] : 0);
        const int s32 = xor_add<16>(s16), s64 = xor_add<32>(s32);
        m16 = max(m16, s16);
        m32 = max(m32, s32);
        m64 = max(m64, s64);
    }
#pragma unroll
    for (int off = 32; off > 8; off >>= 1) {
        m16 = max(m16, __shfl_xor(m16, off));
        m32 = max(m32, __shfl_xor(m32, off));
    }
    if (lane == 0) {
        atomicMax(&out3[0], m64);
        atomicMax(&out3[1], m32);
        atomicMax(&out3[2], m16);
    }
}

hipError_t launch_ht_tiles(int na, const int32_t* alist, const int32_t* tcnt, int32_t* out3, hipStream_t s) {
    if (na <= 0) return hipSuccess;
    const int tiles = (na + 63) / 64;
    ht_tiles_kernel<<<std::min((tiles + 3) / 4, 64), 256, 0, s>>>(na, alist, tcnt, out3);
    return hipGetLastError();
}

// The support vectors in sweep order, packed once per kernel sum so the sweep reads them
// contiguously: head rows [nbp][H] and |x|^2 (rows nb..nbp-1 zero), and the tail nonzeros of
// support vector j (in its column order) as (column << 6 | j % 64, value bits) from toff[j].
// toff is the exclusive scan of the tail counts, by one workgroup in chunks of 8 * 1024.
__global__ __launch_bounds__(1024) void ht_tail_offsets_kernel(int nb, const int32_t* __restrict__ blist,
                                                               const int32_t* __restrict__ tcnt, int32_t* toff) {
    constexpr int PER = 8;
    __shared__ int s_w[16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int carry = 0;
    for (int base = 0; base < nb; base += 1024 * PER) {
        const int t0 = base + (int)threadIdx.x * PER;
        int v[PER], mine = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) v[k] = t0 + k < nb ? blist[t0 + k] : -1;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            v[k] = v[k] >= 0 ? tcnt[v[k]] : 0;
            mine += v[k];
        }
        const int x = wave_scan(mine);
        if (lane == 63) s_w[wid] = x;
        __syncthreads();
        int run = carry + x - mine;
        for (int w = 0; w < 16; ++w) {
            const int c = s_w[w];
            run += (w < wid) ? c : 0;
            carry += c;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (t0 + k < nb) toff[t0 + k] = run;
            run += v[k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) toff[nb] = carry;
}

__global__ __launch_bounds__(256) void ht_pack_kernel(int nb, int nbp, int H, const int32_t* __restrict__ blist,
                                                      const float* __restrict__ head, const float* __restrict__ nrm,
                                                      const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                      const float* __restrict__ val, const int32_t* __restrict__ hmap,
                                                      const int32_t* __restrict__ toff, float* bhead, float* bnrm,
                                                      uint2* tent) {
    const int j = blockIdx.x * 16 + (threadIdx.x >> 4), sub = threadIdx.x & 15;
    if (j >= nbp) return;
    float* dst = bhead + (size_t)j * H;
    if (j >= nb) {
        for (int k = sub; k < H; k += 16) dst[k] = 0.f;
        if (sub == 0) bnrm[j] = 0.f;
        return;
    }
    const int a = blist[j];
    const float* src = head + (size_t)a * H;
    for (int k = sub; k < H; k += 16) dst[k] = src[k];
    if (sub == 0) bnrm[j] = nrm[a];
    // tail nonzeros in column order: each lane's place is the number of them before it in its row's 16
    int e = toff[j];
    const unsigned tag = (unsigned)(j & 63);
    const int p1 = rp[a + 1];
    for (int pb = rp[a]; pb < p1; pb += 16) {
        const int p = pb + sub;
        const int c = p < p1 ? col[p] : 0;
        const bool t = p < p1 && hmap[c] < 0;
        const unsigned m = (unsigned)(__ballot(t) >> (threadIdx.x & 48)) & 0xffffu;
        if (t) tent[e + __popc(m & ((1u << sub) - 1u))] = make_uint2(((unsigned)c << 6) | tag, __float_as_uint(val[p]));
        e += __popc(m);
    }
}

hipError_t launch_ht_pack(int nb, int H, const int32_t* blist, const float* head, const float* nrm, const int32_t* rp,
                          const int32_t* col, const float* val, const int32_t* hmap, const int32_t* tcnt,
                          int32_t* toff, float* bhead, float* bnrm, uint2* tent, hipStream_t s) {
    const int nbp = (nb + HT_CHUNK - 1) / HT_CHUNK * HT_CHUNK;
    ht_tail_offsets_kernel<<<1, 1024, 0, s>>>(nb, blist, tcnt, toff);
    if (nbp > 0)
        ht_pack_kernel<<<(nbp + 15) / 16, 256, 0, s>>>(nb, nbp, H, blist, head, nrm, rp, col, val, hmap, toff, bhead,
                                                         bnrm, tent);
    return hipGetLastError();
}

// ------------------------------------------------------------------ the kernel sum

// LDS table of the tile's tail nonzeros grouped by column: a bitmap of the columns with, beside every
// word, the number of columns before it, so a lookup is one 8-byte read and a bit count (a hash table's
// chains end when the longest of a wave's 64 does: about 0.9 us per 128 lookups, and most columns are in
// none of the rows); per column, in that order, its first entry and their number; and the entries
// (target row, value), those of one column contiguous.
constexpr int HT_LK = 2;                // tail entries a lane looks up per step
constexpr int HT_HITS = 64 * HT_LK;     // of a wave
// a hit: first entry in the table, support vector (of the chunk), first place among the step's matches
static_assert(HT_ENTRIES <= 1 << 13 && HT_CHUNK <= 1 << 6 && HT_HITS * HT_TILE_MAX <= 1 << 13, "hit word");
static_assert(HT_TILE_MAX <= 255, "row byte");
static_assert(HT_MAX_WORDS % HT_BLOCK == 0 && HT_ENTRIES % HT_BLOCK == 0, "scans");

template <int H>
struct HtLds {
    static constexpr int HS = H + 4;   // row stride of the staged head rows (b128 reads without conflicts)
    // tail-dot tile, support vector major: the atomics of one support vector's nonzeros go to
    // consecutive target rows (distinct banks); the odd stride spreads the epilogue's reads
    static constexpr int CS = HT_TILE_MAX + 1;
    static constexpr size_t map = 0;                                        // uint2: bits, columns before
    static constexpr size_t ent = map + sizeof(uint2) * HT_MAX_WORDS;       // per column: first | number << 13
    static constexpr size_t erow = ent + sizeof(uint32_t) * HT_ENTRIES;
    static constexpr size_t eval = erow + sizeof(uint8_t) * HT_ENTRIES;
    static constexpr size_t bt = eval + sizeof(float) * HT_ENTRIES;
    static constexpr size_t corr = bt + sizeof(float) * HT_CHUNK * HS;
    static constexpr size_t cb = corr + sizeof(unsigned long long) * HT_CHUNK * CS;
    static constexpr size_t nb = cb + sizeof(double) * HT_CHUNK;
    static constexpr size_t na = nb + sizeof(float) * HT_CHUNK;
    static constexpr size_t red = na + sizeof(float) * HT_TILE_MAX;
    static constexpr size_t misc = red + sizeof(double) * 4 * HT_TILE_MAX;
    static constexpr size_t desc = misc + 64;   // per wave: the hits of one step of its tail entries
    static constexpr size_t marks = desc + sizeof(uint2) * HT_HITS * (HT_BLOCK / 64);
    static constexpr size_t total = marks + sizeof(uint64_t) * HT_HITS * (HT_BLOCK / 64);
    // the tail-dot tile doubles as the table builder's head bitmap and per-column counters
    static_assert(sizeof(unsigned long long) * HT_CHUNK * CS >=
                      sizeof(uint32_t) * HT_MAX_WORDS + sizeof(uint32_t) * HT_ENTRIES, "builder scratch");
    static_assert(total <= 160 * 1024, "LDS");
};

// Workgroup = 8 waves and one tile of R (16, 32 or 64) target rows; it sweeps its split (whole
// chunks) of the packed support vectors HT_CHUNK at a time.  Per chunk: the head rows are
// staged in LDS, and the chunk's tail nonzeros, spread evenly over the threads, are looked up
// in the tile's column table; each match adds a value product into a 64 x 64 tile of 64-bit
// fixed-point tail dots (stored support vector major, so the adds of one support vector's
// nonzeros fall in distinct LDS banks).  A column of the tail is in none of the tile's rows or in
// up to ten (text-like rows, H = 128: 0.5 matches an entry), so walking an entry's matches in its
// own lane leaves 19 of 20 lanes idle in a chain of dependent LDS reads and atomics; instead a
// wave lays the matches of its 128 entries out one after the other and its lanes take 64 at a time
// (a scan gives every hit its first place, a bit there marks it, and the lane at place p finds its hit
// as the number of marks up to p).  10,000 x 39,000 text-like pairs: 2.4 ms, against 5.96 with
// a hash table and lane by lane.  The next chunk's data are loaded into registers meanwhile.
// Then the waves form the head dots of their 16 x 16 blocks on the matrix cores
// (v_mfma_f32_16x16x4f32; K = H, where for instruction t lane q of a 16-lane group supplies
// column (H/4) q + t of both operands, so each lane reads H/4 consecutive values), add the tail
// dot, and apply d2 = |a|^2 + |b|^2 - 2 dot (clamped at 0), exp(-gamma d2), coef_b K into FP64
// row sums.  Block k of the tile is (row block k % RB, column block k / RB), RB = R / 16, and
// wave w takes blocks w and w + 8, so its row block is fixed for the whole sweep and its A
// operands stay in registers.
template <int H>
__global__ __launch_bounds__(HT_BLOCK) void kernel_sum_ht_kernel(HtArgs A) {
    using L = HtLds<H>;
    constexpr int KQ = H / 4;
    extern __shared__ __align__(16) unsigned char smem[];
    uint2* s_map = reinterpret_cast<uint2*>(smem + L::map);
    uint32_t* s_ent = reinterpret_cast<uint32_t*>(smem + L::ent);
    uint8_t* s_erow = reinterpret_cast<uint8_t*>(smem + L::erow);
    float* s_eval = reinterpret_cast<float*>(smem + L::eval);
    float* s_bt = reinterpret_cast<float*>(smem + L::bt);
    unsigned long long* s_corr = reinterpret_cast<unsigned long long*>(smem + L::corr);
    uint32_t* s_hb = reinterpret_cast<uint32_t*>(smem + L::corr);           // builder: head columns
    uint32_t* s_cnt = s_hb + HT_MAX_WORDS;                                  // builder: entries of a column
    double* s_cb = reinterpret_cast<double*>(smem + L::cb);
    float* s_nb = reinterpret_cast<float*>(smem + L::nb);
    float* s_na = reinterpret_cast<float*>(smem + L::na);
    double* s_red = reinterpret_cast<double*>(smem + L::red);
    int* s_scan = reinterpret_cast<int*>(smem + L::misc);               // [HT_BLOCK / 64]

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int R = A.tile_rows, RB = R >> 4;
    const int r0 = blockIdx.x * R;
    const int nr = min(R, A.na - r0);
    const int nwords = (A.d + 31) >> 5;
    for (int k = tid; k < HT_MAX_WORDS; k += HT_BLOCK) {
        s_hb[k] = k < nwords ? A.hbits[k] : 0u;
        s_map[k] = make_uint2(0u, 0u);
    }
    for (int k = tid; k < HT_ENTRIES; k += HT_BLOCK) s_cnt[k] = 0u;
    __syncthreads();

    // the tile's rows (8 threads per row): norms; the columns of their tail nonzeros
    const int tr = tid >> 3, tsub = tid & 7;
    const int ta = tr < nr ? (A.alist ? A.alist[r0 + tr] : r0 + tr) : 0;
    const int tp0 = tr < nr ? A.a_rp[ta] + tsub : 0, tp1 = tr < nr ? A.a_rp[ta + 1] : 0;
    auto in_tail = [&](int c) { return !((s_hb[c >> 5] >> (c & 31)) & 1u); };
    auto rank_of = [&](int c) {   // of a column in the bitmap
        const uint2 w = s_map[c >> 5];
        return (int)w.y + __popc(w.x & ((1u << (c & 31)) - 1u));
    };
    if (tr < nr && tsub == 0) s_na[tr] = A.a_nrm[ta];
    for (int p = tp0; p < tp1; p += 8) {
        const int c = A.a_col[p];
        if (in_tail(c)) atomicOr(&s_map[c >> 5].x, 1u << (c & 31));
    }
    __syncthreads();
    // exclusive scan over the workgroup of one number per thread
    auto block_scan = [&](int v) -> int {
        const int x = wave_scan(v);
        if (lane == 63) s_scan[wid] = x;
        __syncthreads();
        int run = x - v;
        for (int w = 0; w < wid; ++w) run += s_scan[w];
        return run;
    };
    {
        constexpr int PER = HT_MAX_WORDS / HT_BLOCK;
        int loc = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) loc += __popc(s_map[tid * PER + k].x);
        int run = block_scan(loc);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            s_map[tid * PER + k].y = (uint32_t)run;
            run += __popc(s_map[tid * PER + k].x);
        }
    }
    __syncthreads();
    for (int p = tp0; p < tp1; p += 8) {
        const int c = A.a_col[p];
        if (in_tail(c)) atomicAdd(&s_cnt[rank_of(c)], 1u);
    }
    __syncthreads();
    {
        constexpr int PER = HT_ENTRIES / HT_BLOCK;
        int loc = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) loc += (int)s_cnt[tid * PER + k];
        int run = block_scan(loc);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t cnt = s_cnt[tid * PER + k];
            s_ent[tid * PER + k] = ((uint32_t)run & 0x1FFFu) | cnt << 13;
            run += (int)cnt;
            s_cnt[tid * PER + k] = 0u;   // from here on the fill cursor of the column
        }
    }
    __syncthreads();
    // the entries themselves, contiguous per column (their order within a column is free:
    // the tail dots are exact fixed-point sums)
    for (int p = tp0; p < tp1; p += 8) {
        const int c = A.a_col[p];
        if (!in_tail(c)) continue;
        const int k = rank_of(c);
        const int e = (int)(s_ent[k] & 0x1FFFu) + (int)atomicAdd(&s_cnt[k], 1u);
        s_erow[e] = (uint8_t)tr;
        s_eval[e] = A.a_val[p];
    }
    __syncthreads();
    for (int k = tid; k < HT_CHUNK * L::CS; k += HT_BLOCK) s_corr[k] = 0ull;
    // head values of this wave's 16 target rows: lane (row + 16 q) holds columns (H/4) q ..
    const int rb = wid % RB;
    const int q = lane >> 4, l16 = lane & 15;
    const bool mwave = wid < 4 * RB;
    float areg[KQ];
    {
        const int r = 16 * rb + l16;
#pragma unroll
        for (int t = 0; t < KQ; ++t) areg[t] = 0.f;
        if (mwave && r < nr) {
            const int a = A.alist ? A.alist[r0 + r] : r0 + r;
            const float4* src = reinterpret_cast<const float4*>(A.a_head + (size_t)a * H + KQ * q);
#pragma unroll
            for (int t4 = 0; t4 < KQ / 4; ++t4) {
                const float4 v = src[t4];
                areg[4 * t4] = v.x; areg[4 * t4 + 1] = v.y; areg[4 * t4 + 2] = v.z; areg[4 * t4 + 3] = v.w;
            }
        }
    }
    __syncthreads();   // table and entries complete

    uint2* desc = reinterpret_cast<uint2*>(smem + L::desc) + HT_HITS * wid;
    unsigned long long* marks = reinterpret_cast<unsigned long long*>(smem + L::marks) + HT_HITS * wid;
    const float gam = (float)A.gamma;
    const double fx_scale = A.fx_scale, fx_inv = A.fx_inv;
    // splits are whole chunks, so chunk rows are support-vector ordinals modulo 64
    const int per = (A.nb + A.nsplit * HT_CHUNK - 1) / (A.nsplit * HT_CHUNK) * HT_CHUNK;
    const int b0 = blockIdx.y * per, b1 = min(A.nb, b0 + per);
    constexpr int HV = HT_CHUNK * (H / 4) / HT_BLOCK;   // float4 of head rows per thread and chunk
    constexpr int PE = 8;                               // tail entries per thread held ahead
    static_assert(HV >= 1, "head tile");
    double racc[4] = {0.0, 0.0, 0.0, 0.0};
    // the next chunk's head values, tail entries, norm and coefficient are loaded one chunk
    // ahead into registers (the end offset of its tail two chunks ahead)
    f32x4 hv[HV];   // (a native vector: an array of float4 stays in scratch memory, and the loads with it)
    uint2 pe[PE];
    float pnrm = 0.f;
    double pcf = 0.0;
    int e_lo = 0, e_hi = 0, e_next = 0;
    auto prefetch = [&](int c0, int lo, int hi) {
        const f32x4* src = reinterpret_cast<const f32x4*>(A.b_head + (size_t)c0 * H);
#pragma unroll
        for (int v = 0; v < HV; ++v) hv[v] = src[tid + HT_BLOCK * v];
#pragma unroll
        for (int m = 0; m < PE; ++m) {
            const int e = lo + tid + HT_BLOCK * m;
            pe[m] = e < hi ? A.b_tent[e] : make_uint2(0xffffffffu, 0u);
        }
        if (tid < HT_CHUNK) {
            pnrm = A.b_nrm[c0 + tid];
            pcf = c0 + tid < b1 ? A.coef[c0 + tid] : 0.0;
        }
    };
    if (b0 < b1) {
        e_lo = A.b_toff[b0];
        e_hi = A.b_toff[min(b0 + HT_CHUNK, b1)];
        e_next = A.b_toff[min(b0 + 2 * HT_CHUNK, b1)];
        prefetch(b0, e_lo, e_hi);
    }
    for (int c0 = b0; c0 < b1; c0 += HT_CHUNK) {
        const int nc = min(HT_CHUNK, b1 - c0);
        // this chunk: head rows into LDS, norms and coefficients, tail products into the tile
#pragma unroll
        for (int v = 0; v < HV; ++v) {
            const int e = tid + HT_BLOCK * v;
            *reinterpret_cast<f32x4*>(s_bt + (e / (H / 4)) * L::HS + 4 * (e % (H / 4))) = hv[v];
        }
        if (tid < HT_CHUNK) {
            s_nb[tid] = pnrm;
            s_cb[tid] = pcf;
        }
        // HT_LK support-vector tail nonzeros per lane: each entry that the table holds in one of their
        // columns adds the value product as a 64-bit integer (the product of two FP32 values is exact
        // in FP64, the scale a power of two, the conversion rounds to nearest)
        auto tail = [&](const uint2 (&t)[HT_LK]) __attribute__((always_inline)) {
            uint2 w[HT_LK];
            uint32_t en[HT_LK];
#pragma unroll
            for (int u = 0; u < HT_LK; ++u) w[u] = s_map[min(t[u].x >> 11, (uint32_t)HT_MAX_WORDS - 1u)];
#pragma unroll
            for (int u = 0; u < HT_LK; ++u) {
                const uint32_t bit = (t[u].x >> 6) & 31u;
                const bool in = t[u].x != 0xffffffffu && ((w[u].x >> bit) & 1u);
                en[u] = in ? s_ent[w[u].y + __popc(w[u].x & ((1u << bit) - 1u))] : 0u;
            }
            // matches before this lane (low half; at most 64 * HT_HITS = 8,192) and hits before it
            int mine = 0;
#pragma unroll
            for (int u = 0; u < HT_LK; ++u) mine += (int)(en[u] >> 13) + (en[u] ? 1 << 16 : 0);
            const int incl = wave_scan(mine);
            const int T = __builtin_amdgcn_readlane(incl, 63) & 0xffff;
            if (!T) return;
            int hit = (incl - mine) >> 16, at = (incl - mine) & 0xffff;
            for (int k = lane; 64 * k < T; k += 64) marks[k] = 0ull;
            wave_lds_fence();
#pragma unroll
            for (int u = 0; u < HT_LK; ++u) {
                if (en[u]) {
                    desc[hit++] = make_uint2((en[u] & 0x1FFFu) | (t[u].x & 63u) << 13 | (uint32_t)at << 19, t[u].y);
                    atomicOr(&marks[at >> 6], 1ull << (at & 63));
                    at += (int)(en[u] >> 13);
                }
            }
            wave_lds_fence();
            int before = -1;
            for (int p0 = 0; p0 < T; p0 += 64) {
                const unsigned long long m = marks[p0 >> 6];
                const int h = before + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)) +
                              (int)((m >> lane) & 1ull);
                if (p0 + lane < T) {
                    const uint2 q = desc[h];
                    const int e = (int)(q.x & 0x1FFFu) + (p0 + lane - (int)(q.x >> 19));
                    const double vb = (double)__uint_as_float(q.y) * fx_scale;
                    const long long v = __double2ll_rn((double)s_eval[e] * vb);
                    atomicAdd(&s_corr[(int)((q.x >> 13) & 63u) * L::CS + s_erow[e]], (unsigned long long)v);
                }
                before += __popcll(m);
            }
        };
#pragma unroll
        for (int m = 0; m < PE; m += HT_LK)
            if (e_lo + HT_BLOCK * m < e_hi) {
                const uint2 t[HT_LK] = {pe[m], pe[m + 1]};
                tail(t);
            }
        for (int e = e_lo + HT_BLOCK * PE; e < e_hi; e += HT_LK * HT_BLOCK) {
            uint2 t[HT_LK];
#pragma unroll
            for (int u = 0; u < HT_LK; ++u) {
                const int k = e + HT_BLOCK * u + tid;
                t[u] = k < e_hi ? A.b_tent[k] : make_uint2(0xffffffffu, 0u);
            }
            tail(t);
        }
        // the next chunk's loads are in flight while this one is reduced
        if (c0 + HT_CHUNK < b1) {
            const int c2 = c0 + HT_CHUNK;
            const int lo = e_hi, hi = e_next;
            e_lo = lo;
            e_hi = hi;
            prefetch(c2, lo, hi);
            e_next = A.b_toff[min(c2 + 2 * HT_CHUNK, b1)];
        }
        __syncthreads();
        if (mwave) {
            for (int k = wid; k < 4 * RB; k += 8) {
                const int cbk = k / RB;
                const int col = 16 * cbk + l16;
                const float* brow = s_bt + col * L::HS + KQ * q;
                float bv[KQ];
#pragma unroll
                for (int t4 = 0; t4 < KQ / 4; ++t4) {
                    const float4 v = *reinterpret_cast<const float4*>(brow + 4 * t4);
                    bv[4 * t4] = v.x; bv[4 * t4 + 1] = v.y; bv[4 * t4 + 2] = v.z; bv[4 * t4 + 3] = v.w;
                }
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int t = 0; t < KQ; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(areg[t], bv[t], acc, 0, 0, 0);
                const float nbc = s_nb[col];
                const double cbv = s_cb[col];
                const float dv[4] = {acc[0], acc[1], acc[2], acc[3]};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 16 * rb + 4 * q + i;
                    unsigned long long* cell = &s_corr[col * L::CS + row];
                    const long long tv = (long long)*cell;
                    *cell = 0ull;
                    if (row < nr && col < nc) {
                        const float dot = dv[i] + (float)((double)tv * fx_inv);
                        float d2 = s_na[row] + nbc - 2.f * dot;
                        d2 = d2 < 0.f ? 0.f : d2;
                        const float kv = kexp(-gam * d2);
                        racc[i] += cbv * (double)kv;
                        if (A.kout) {
                            const int a = A.alist ? A.alist[r0 + row] : r0 + row;
                            const int b = c0 + col;
                            A.kout[(size_t)b * A.ldk + a] = a == b ? 1.f : kv;
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    // rows 16 rb + 4 q + i: add the 16 lanes (columns) of each q, then the waves of each row block
    if (mwave) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = racc[i];
            for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o);
            if (l16 == 0) s_red[(wid / RB) * HT_TILE_MAX + 16 * rb + 4 * q + i] = v;
        }
    }
    __syncthreads();
    if (tid < nr) {
        const int groups = RB == 4 ? 2 : 4;
        double v = 0.0;
        for (int g = 0; g < groups; ++g) v += s_red[g * HT_TILE_MAX + tid];
        A.part[(size_t)blockIdx.y * A.na + r0 + tid] = v;
    }
}

size_t ht_lds_bytes(int H) {
    switch (H) {
        case 32: return HtLds<32>::total;
        case 64: return HtLds<64>::total;
        case 128: return HtLds<128>::total;
        default: return 0;
    }
}

hipError_t launch_kernel_sum_ht(const HtArgs& a, hipStream_t s) {
    if (a.na <= 0) return hipSuccess;
    const size_t lds = ht_lds_bytes(a.H);
    if (!lds || (a.tile_rows != 16 && a.tile_rows != 32 && a.tile_rows != 64)) return hipErrorInvalidValue;
    dim3 grid((a.na + a.tile_rows - 1) / a.tile_rows, a.nsplit);
    HtArgs c = a;
    switch (a.H) {
        case 32:
            (void)hipFuncSetAttribute((const void*)kernel_sum_ht_kernel<32>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_ht_kernel<32><<<grid, HT_BLOCK, lds, s>>>(c);
            break;
        case 64:
            (void)hipFuncSetAttribute((const void*)kernel_sum_ht_kernel<64>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_ht_kernel<64><<<grid, HT_BLOCK, lds, s>>>(c);
            break;
        default:
            (void)hipFuncSetAttribute((const void*)kernel_sum_ht_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kernel_sum_ht_kernel<128><<<grid, HT_BLOCK, lds, s>>>(c);
            break;
    }
    return hipGetLastError();
}

}  // namespace svm
