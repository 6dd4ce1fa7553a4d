// svm_regloop.h -- the persistent SMO loop (see svm_step.hip) for dense rows and bitset rows
// that fit the register file: included by svm_reg_dense.hip and svm_reg_bits.hip, one kernel
// instance per row width, rows per thread and kernel precision.
//
// A CU holds 512 KB of vector registers against 160 KB of LDS, so the 56 MB of the dense mixture
// (500,000 x 28 floats) fit the chip: a thread keeps R rows of its workgroup's segment, their f
// and their status in registers for the whole launch, and an iteration reads memory only for
// the two pair rows and the records.  A shrunk row stays where it is with its active bit cleared:
// there is no list to compact.  What bounds an iteration is the chain pair rows -> kernel values ->
// block reduction -> exchange -> merge, so the rest is built to shorten it:
//  * 512 threads (two waves per SIMD, 256 registers a lane), because the reductions and the merge
//    are instruction-bound per wave and barriers cost by the wave;
//  * every wave stages the pair for itself in its own LDS, so the stage needs no barrier: an
//    iteration has two barriers (three beyond 8 workgroups) where svm_step.hip has four;
//  * records of one 64-byte line (eight words of 48 payload bits and a 16-bit tag), read eight per
//    load instruction: the exchange and its reductions alone take 2.9 / 3.4 / 4.3 us at 29 / 128 /
//    256 workgroups, against 3.2 / 4.0 / 4.8 with the 128-byte records of svm_step.hip on 1024
//    threads (a record spread over word arrays, so that a lane reads a whole one, took 5.6 / 5.6 / 6.3);
//  * up to 8 workgroups, wave 0 alone reads and merges the records.
// A launch runs up to 8 problems of one sample set side by side (svm_train_shared), each on a row of
// the grid (blockIdx.y) with its own records and state: their chains overlap, and nothing is shared.
// Kernel values, the f update and the selection are those of svm_step.hip operation for operation,
// so results are equal bit for bit.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "svm_device.h"
#include "svm_internal.h"

namespace svm {

constexpr int REG_NW = REG_BLOCK / 64;
// active / selection bits kept with the status byte of a row
enum : int { RST_ACTIVE = 8, RST_UP = 16, RST_LOW = 32 };
DEV int rst_make(int st, bool active) {
    const uint8_t s = (uint8_t)st;
    return st | (active ? RST_ACTIVE : 0) | (st_in_up(s) ? RST_UP : 0) | (st_in_low(s) ? RST_LOW : 0);
}

// A value that the compiler takes as formed at this place and unknown from here on.
template <typename T>
DEV void pin(T& v) { asm volatile("" : "+v"(v)); }

// BITS: rows of 4 * W4 words; else rows of 4 * W4 floats (zeros beyond dpad).
template <bool BITS, typename KT, int W4, int R>
__global__ __launch_bounds__(REG_BLOCK) void smo_reg_kernel(RegLaunch L) {
    const RegArgs& A = L.a[blockIdx.y];
    constexpr int NT = REG_BLOCK, NW = REG_NW, W = 4 * W4;
    typedef typename std::conditional<BITS, uint4, float4>::type V4;
    __shared__ double s_al[R * NT];                               // alpha of the segment's rows
    __shared__ uint8_t s_lab[R * NT];      // bit 0: label +1; bit 1: on the active list at launch
    __shared__ __align__(16) uint32_t s_pair[NW][2 * W];          // a wave's copy of the pair rows
    __shared__ unsigned long long s_rec[REG_GRID_MAX * 9];        // records (odd stride in 8-byte words)
    __shared__ double s_v[2 * NW], m_v[8], m_a[8];
    __shared__ int s_i[2 * NW], m_i[8], s_wc[NW], m_c[4];
    __shared__ int s_abort;
    __shared__ unsigned long long s_pt[PROF_SLOTS + 1];

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int blk = blockIdx.x, G = gridDim.x;
    const double C = A.C;
    const KT gam = (KT)A.gamma;
    const int seg0 = A.seg_start[blk], nseg = A.seg_start[blk + 1] - seg0;
    int nrows = A.cnt[blk];

    // ---- this thread's rows: segment row r * NT + tid
    V4 X[R][W4];
    double F[R];
    int ST[R];
    int nn[R];                                                    // bitset rows: bits set
    for (int li = tid; li < nseg; li += NT) {
        s_lab[li] = A.y[seg0 + li] > 0 ? 1 : 0;
        s_al[li] = A.alpha[seg0 + li];
    }
    if (tid == 0) s_abort = 0;
    if (tid < 8) {
        m_v[tid] = tid < 4 ? INFINITY : -INFINITY;
        m_a[tid] = 0.0;
        m_i[tid] = IDX_NONE;
        m_c[tid & 3] = 0;
    }
    __syncthreads();
    for (int t = tid; t < nrows; t += NT) s_lab[A.act[seg0 + t] - seg0] |= 2;   // (each id once)
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int li = r * NT + tid, i = seg0 + li;
        const bool in = li < nseg;
        const V4* src = BITS ? reinterpret_cast<const V4*>(A.bits + (size_t)i * A.stride)
                             : reinterpret_cast<const V4*>(A.x + (size_t)i * A.stride);
        nn[r] = 0;
#pragma unroll
        for (int k = 0; k < W4; ++k) {
            X[r][k] = V4{0, 0, 0, 0};
            if (in && 4 * k < A.stride) X[r][k] = src[k];
            if constexpr (BITS) nn[r] += __popc(X[r][k].x) + __popc(X[r][k].y) + __popc(X[r][k].z) + __popc(X[r][k].w);
        }
        F[r] = in ? A.f[i] : 0.0;
        ST[r] = in ? rst_make(A.status[i], (s_lab[li] & 2) != 0) : 0;
    }

    // ---- solver state (identical in every workgroup)
    Ctl* ctl = A.ctl;
    double bu = ctl->b_up, bl = ctl->b_low, au = ctl->a_up, al = ctl->a_low;
    int iu = ctl->i_up, il = ctl->i_low;
    int yu = iu >= 0 && A.y[iu] > 0 ? 1 : -1, yl = il >= 0 && A.y[il] > 0 ? 1 : -1;
    long long iter = ctl->iter, counter = ctl->counter, n_act_total = ctl->n_active;
    long long passes = ctl->shrink_passes, shrunk = ctl->shrunk_total;
    int exit_reason = EXIT_NONE;
    unsigned long long work_rows = 0, work_nnz = 0;
    const bool dbg_on = A.dbg != nullptr && blk == 0 && tid == 0;
    const bool prof_on = dbg_on && A.dbg->prof != nullptr;
    if (prof_on) {
        for (int k = 0; k < PROF_SLOTS; ++k) s_pt[k] = 0;
        s_pt[PROF_SLOTS] = wall_clock64();
    }
    auto lap = [&](int k) {
        if (A.dbg != nullptr && prof_on) {
            const unsigned long long t = wall_clock64();
            s_pt[k] += t - s_pt[PROF_SLOTS];
            s_pt[PROF_SLOTS] = t;
        }
    };
    __syncthreads();
    lap(6);

    for (;;) {
        if (!(bl - bu > A.thr)) { exit_reason = EXIT_CONVERGED; break; }
        if (iter >= A.max_iter) { exit_reason = EXIT_MAXITER; break; }
        if (dbg_on && iter < A.dbg->trace_cap) {
            A.dbg->tr_iu[iter] = iu; A.dbg->tr_il[iter] = il; A.dbg->tr_bu[iter] = bu; A.dbg->tr_bl[iter] = bl;
        }
        // ---- 1. the working pair, by every wave for itself: rows into the wave's LDS, K(up, low)
        uint32_t* pw = s_pair[wid];
        double kul;
        KT nuu = (KT)0, nll = (KT)0;
        if constexpr (BITS) {
            uint32_t wu = 0, wl = 0;
            if (lane < A.stride) {
                wu = A.bits[(size_t)iu * A.stride + lane];
                wl = A.bits[(size_t)il * A.stride + lane];
            }
            if (lane < W) {
                pw[lane] = wu;
                pw[W + lane] = wl;
            }
            int c2 = __popc(wu) | (__popc(wl) << 16), cd = __popc(wu & wl);
            sum2_lanes32(c2, cd);
            const int cu = c2 & 0xffff, cl = c2 >> 16;
            KT d2 = (KT)cu + (KT)cl - (KT)2 * (KT)cd;
            if (d2 < (KT)0) d2 = (KT)0;
            kul = (double)kexp((KT)(-gam * d2));
            nuu = (KT)cu;
            nll = (KT)cl;
        } else {
            const float* xu = A.x + (size_t)iu * A.stride;
            const float* xl = A.x + (size_t)il * A.stride;
            float a = 0.f;
#pragma unroll
            for (int k0 = 0; k0 < W; k0 += 64) {
                const int k = k0 + lane;
                if (k < W) {
                    const bool in = k < A.stride;
                    const float u = in ? xu[k] : 0.f, l = in ? xl[k] : 0.f;
                    reinterpret_cast<float2*>(pw)[k] = make_float2(u, l);
                    const float t = u - l;
                    a = fmaf(t, t, a);
                }
            }
            if constexpr (std::is_same<KT, float>::value) {
                a = wave_sum_dpp(a);
                kul = (double)kexp(-gam * a);
            } else {
                // sequential in k: the same rounding as the FP64 reference
                wave_lds_fence();
                double s = 0.0;
                {
#pragma clang fp contract(off)
#pragma unroll
                    for (int k = 0; k < W / 2; ++k) {
                        const float4 e = reinterpret_cast<const float4*>(pw)[k];   // (u0 l0 u1 l1)
                        double t = (double)e.x - (double)e.y;
                        s = s + t * t;
                        t = (double)e.z - (double)e.w;
                        s = s + t * t;
                        if (k % 8 == 7) {
                            pin(s);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
                kul = exp(-A.gamma * s);
            }
        }
        wave_lds_fence();
        const PairNew pn = pair_update(au, al, yu, yl, bu, bl, kul, C);
        bool do_shrink = false;
        if (A.H > 0) {
            --counter;
            do_shrink = counter == 0;
        }
        lap(0);

        // ---- 2. f update over this thread's rows, candidates, shrink rule
        double cbu = INFINITY, cbl = -INFINITY;
        int ciu = IDX_NONE, cil = IDX_NONE;
        work_rows += (unsigned long long)nrows;
        KT du[R], dl[R];
        if constexpr (BITS) {
            int su[R], sl[R];
#pragma unroll
            for (int r = 0; r < R; ++r) { su[r] = 0; sl[r] = 0; }
            const uint4* pu = reinterpret_cast<const uint4*>(pw);
            const uint4* pl = reinterpret_cast<const uint4*>(pw + W);
#pragma unroll
            for (int k = 0; k < W4; ++k) {
                const uint4 a = pu[k], b = pl[k];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint4 v = X[r][k];
                    su[r] += __popc(v.x & a.x) + __popc(v.y & a.y) + __popc(v.z & a.z) + __popc(v.w & a.w);
                    sl[r] += __popc(v.x & b.x) + __popc(v.y & b.y) + __popc(v.z & b.z) + __popc(v.w & b.w);
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                du[r] = (KT)nn[r] + nuu - (KT)2 * (KT)su[r];
                dl[r] = (KT)nn[r] + nll - (KT)2 * (KT)sl[r];
                if (du[r] < (KT)0) du[r] = (KT)0;
                if (dl[r] < (KT)0) dl[r] = (KT)0;
                if (ST[r] & RST_ACTIVE) work_nnz += (unsigned long long)nn[r];
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) { du[r] = (KT)0; dl[r] = (KT)0; }
            const float4* p4 = reinterpret_cast<const float4*>(pw);
#pragma unroll
            for (int k = 0; k < W4; ++k) {
                const float4 q0 = p4[2 * k], q1 = p4[2 * k + 1];   // (u0 l0 u1 l1) (u2 l2 u3 l3)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if constexpr (std::is_same<KT, double>::value) {
                        // (the rows stay floats: without this their conversions leave the loop, in twice
                        // the registers)
                        pin(X[r][k].x); pin(X[r][k].y); pin(X[r][k].z); pin(X[r][k].w);
                    }
                    const float4 v = X[r][k];
                    KT a = du[r], b = dl[r];
                    if constexpr (std::is_same<KT, double>::value) {
#pragma clang fp contract(off)
                        double t;
                        t = (double)v.x - (double)q0.x; a = a + t * t;
                        t = (double)v.x - (double)q0.y; b = b + t * t;
                        t = (double)v.y - (double)q0.z; a = a + t * t;
                        t = (double)v.y - (double)q0.w; b = b + t * t;
                        t = (double)v.z - (double)q1.x; a = a + t * t;
                        t = (double)v.z - (double)q1.y; b = b + t * t;
                        t = (double)v.w - (double)q1.z; a = a + t * t;
                        t = (double)v.w - (double)q1.w; b = b + t * t;
                    } else {
                        float t;
                        t = v.x - q0.x; a = fmaf(t, t, a);
                        t = v.x - q0.y; b = fmaf(t, t, b);
                        t = v.y - q0.z; a = fmaf(t, t, a);
                        t = v.y - q0.w; b = fmaf(t, t, b);
                        t = v.z - q1.x; a = fmaf(t, t, a);
                        t = v.z - q1.y; b = fmaf(t, t, b);
                        t = v.w - q1.z; a = fmaf(t, t, a);
                        t = v.w - q1.w; b = fmaf(t, t, b);
                    }
                    du[r] = a;
                    dl[r] = b;
                    // (the sums are formed here, not where they are used, and the pair rows read as
                    // they are needed: reading all of them ahead takes 8 registers a word)
                    if (k % 2 == 1) { pin(du[r]); pin(dl[r]); }
                }
                if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!(ST[r] & RST_ACTIVE)) continue;
            const int li = r * NT + tid, i = seg0 + li;
            const double ku = (i == iu) ? 1.0 : (double)kexp(-gam * du[r]);
            const double kl = (i == il) ? 1.0 : (double)kexp(-gam * dl[r]);
            double fi;
            {
#pragma clang fp contract(off)
                fi = F[r] + (pn.cu * ku + pn.cl * kl);
            }
            F[r] = fi;
            if (i == iu) {
                ST[r] = rst_make(st_make(yu > 0, pn.au, C), true);
                s_al[li] = pn.au;
            } else if (i == il) {
                ST[r] = rst_make(st_make(yl > 0, pn.al, C), true);
                s_al[li] = pn.al;
            }
            int sel = ST[r];
            if (do_shrink && shrink_rule((uint8_t)(sel & 7), fi, bu, bl)) {
                ST[r] &= ~RST_ACTIVE;
                sel = 0;
            }
            const bool tu = (sel & RST_UP) && better_up(fi, i, cbu, ciu);
            const bool tl = (sel & RST_LOW) && better_low(fi, i, cbl, cil);
            cbu = tu ? fi : cbu;
            ciu = tu ? i : ciu;
            cbl = tl ? fi : cbl;
            cil = tl ? i : cil;
        }
        if (do_shrink) {
            int c = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) c += __popcll(__ballot(ST[r] & RST_ACTIVE));
            if (lane == 0) s_wc[wid] = c;
        }
        lap(1);
        waves_to_lds<NT>(cbu, ciu, cbl, cil, s_v, s_i);
        __syncthreads();
        if (do_shrink) {
            nrows = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) nrows += s_wc[w];
        }
        // ---- 3. this workgroup's candidates with their alpha and label, by wave 0
        double cau = 0.0, cal = 0.0;
        int eu = IDX_NONE, el = IDX_NONE;   // sample id, bit 31: label +1
        if (wid == 0) {
            // the alpha and label of every wave's winners are read while they are reduced
            const bool in = lane < NW;
            cbu = in ? s_v[lane] : INFINITY;
            ciu = in ? s_i[lane] : IDX_NONE;
            cbl = in ? s_v[NW + lane] : -INFINITY;
            cil = in ? s_i[NW + lane] : IDX_NONE;
            if (ciu != IDX_NONE) {
                cau = s_al[ciu - seg0];
                eu = ciu | (int)((unsigned)s_lab[ciu - seg0] << 31);
            }
            if (cil != IDX_NONE) {
                cal = s_al[cil - seg0];
                el = cil | (int)((unsigned)s_lab[cil - seg0] << 31);
            }
            int wu, wl;
            wave_reduce_sel<16>(cbu, ciu, cbl, cil, wu, wl);
            cau = readlane_d(cau, wu);
            cal = readlane_d(cal, wl);
            eu = __builtin_amdgcn_readlane(eu, wu);
            el = __builtin_amdgcn_readlane(el, wl);
        }
        // ---- 4. exchange and merge (the records as in svm_step.hip, eight words each)
        int ncnt = nrows;
        if (G > 1) {
            const int par = (int)(iter & 1);
            const unsigned tg = rec_tag(iter);
            unsigned long long* rec = A.rec + (size_t)par * G * 8;
            if (wid == 0 && lane < 8) {
                const unsigned long long bub = (unsigned long long)__double_as_longlong(cbu);
                const unsigned long long blb = (unsigned long long)__double_as_longlong(cbl);
                const unsigned long long aub = (unsigned long long)__double_as_longlong(cau);
                const unsigned long long alb = (unsigned long long)__double_as_longlong(cal);
                unsigned long long x;
                switch (lane) {
                    case 0: x = bub & REC8_MASK; break;
                    case 1: x = blb & REC8_MASK; break;
                    case 2: x = aub & REC8_MASK; break;
                    case 3: x = alb & REC8_MASK; break;
                    case 4: x = (bub >> 48) | ((unsigned long long)(unsigned)eu << 16); break;
                    case 5: x = (blb >> 48) | ((unsigned long long)(unsigned)el << 16); break;
                    case 6: x = (aub >> 48) | ((unsigned long long)(unsigned)nrows << 16); break;
                    default: x = alb >> 48; break;
                }
                st_agent(rec + 8 * blk + lane, ((unsigned long long)tg << 48) | x);
            }
            lap(2);
            // up to 8 workgroups wave 0 reads all the records, beyond that every wave its share
            const int readers = G <= 8 ? 1 : NW;
            if (wid < readers) {
                constexpr int QW = 4;
                const int sub = lane >> 3, wd = lane & 7;
                const unsigned long long t0 = wall_clock64();
                bool ab = false;
                for (int q0 = wid; 8 * q0 < G && !ab; q0 += readers * QW) {
                    unsigned long long x[QW];
                    bool ok[QW];
#pragma unroll
                    for (int j = 0; j < QW; ++j) {
                        ok[j] = 8 * (q0 + readers * j) + sub >= G;
                        x[j] = 0;
                    }
                    for (;;) {
                        bool all = true;
#pragma unroll
                        for (int j = 0; j < QW; ++j) {
                            if (!ok[j]) {
                                x[j] = ld_agent(rec + 64 * (size_t)(q0 + readers * j) + lane);
                                ok[j] = (unsigned)(x[j] >> 48) == tg;
                            }
                            all = all && ok[j];
                        }
                        if (__all(all)) break;
                        if (wait_expired(t0, A.spin_limit, ctl, iter)) { ab = true; break; }
                    }
#pragma unroll
                    for (int j = 0; j < QW; ++j) {
                        const int rr = 8 * (q0 + readers * j) + sub;
                        if (rr < G) s_rec[rr * 9 + wd] = x[j] & REC8_MASK;
                    }
                }
                if (__any(ab) && lane == 0) s_abort = 1;
            }
            if (G > 8) __syncthreads();
            else wave_lds_fence();
            lap(3);
            // 64 records per wave; the lane that holds a winner publishes its alpha
            const int NR = (G + 63) / 64;
            if (wid < NR) {
                double rbu = INFINITY, rbl = -INFINITY, rau = 0.0, ral = 0.0;
                int riu = IDX_NONE, ril = IDX_NONE, yb = 0, rc = 0;
                if (tid < G) {
                    const unsigned long long* w = s_rec + tid * 9;
                    const unsigned long long w4 = w[4], w5 = w[5], w6 = w[6], w7 = w[7];
                    rbu = rec8_double(w[0], w4);
                    rbl = rec8_double(w[1], w5);
                    rau = rec8_double(w[2], w6);
                    ral = rec8_double(w[3], w7);
                    const unsigned qu = (unsigned)(w4 >> 16), ql = (unsigned)(w5 >> 16);
                    riu = (int)(qu & 0x7fffffffu);
                    ril = (int)(ql & 0x7fffffffu);
                    yb = (int)(qu >> 31) | (int)(ql >> 31) << 1;
                    rc = (int)(unsigned)(w6 >> 16);
                }
                const long long csum = do_shrink ? wave_sum((long long)rc) : 0;
                int wu, wl;
                wave_reduce_sel(rbu, riu, rbl, ril, wu, wl);
                // (bit 31 of the ids published in LDS: the label)
                const int yu1 = __builtin_amdgcn_readlane(yb, wu) & 1, yl1 = __builtin_amdgcn_readlane(yb, wl) & 2;
                rau = readlane_d(rau, wu);
                ral = readlane_d(ral, wl);
                if (lane == 0) {
                    m_v[wid] = rbu;
                    m_v[4 + wid] = rbl;
                    m_a[wid] = rau;
                    m_a[4 + wid] = ral;
                    m_i[wid] = riu | (yu1 ? (int)0x80000000 : 0);
                    m_i[4 + wid] = ril | (yl1 ? (int)0x80000000 : 0);
                    m_c[wid] = (int)csum;
                }
            }
            __syncthreads();
            if (s_abort) {
                if (tid == 0) __hip_atomic_store(&ctl->abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                exit_reason = EXIT_ABORT;
                break;
            }
            bu = m_v[0]; au = m_a[0]; eu = m_i[0];
            bl = m_v[4]; al = m_a[4]; el = m_i[4];
            ncnt = m_c[0];
            if (NR > 1) {   // the entries of waves beyond NR are empty
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const double vu = m_v[w], vl = m_v[4 + w], qu = m_a[w], ql = m_a[4 + w];
                    const int xu = m_i[w], xl = m_i[4 + w];
                    const bool tu = better_up(vu, xu & 0x7fffffff, bu, eu & 0x7fffffff);
                    const bool tl = better_low(vl, xl & 0x7fffffff, bl, el & 0x7fffffff);
                    bu = tu ? vu : bu;
                    au = tu ? qu : au;
                    eu = tu ? xu : eu;
                    bl = tl ? vl : bl;
                    al = tl ? ql : al;
                    el = tl ? xl : el;
                    ncnt += m_c[w];
                }
            }
        } else {
            if (tid == 0) {
                m_v[0] = cbu; m_v[4] = cbl; m_a[0] = cau; m_a[4] = cal;
                m_i[0] = eu; m_i[4] = el;
            }
            lap(2);
            __syncthreads();
            bu = m_v[0]; au = m_a[0]; eu = m_i[0];
            bl = m_v[4]; al = m_a[4]; el = m_i[4];
        }
        // (uniform: into scalar registers)
        eu = __builtin_amdgcn_readfirstlane(eu);
        el = __builtin_amdgcn_readfirstlane(el);
        iu = eu & 0x7fffffff;
        il = el & 0x7fffffff;
        yu = eu < 0 ? 1 : -1;
        yl = el < 0 ? 1 : -1;
        if (iu == IDX_NONE) iu = -1;
        if (il == IDX_NONE) il = -1;
        if (do_shrink) {
            shrunk += n_act_total - ncnt;
            n_act_total = ncnt;
            ++passes;
            counter = ncnt < A.H ? ncnt : A.H;
            if (counter < 1) counter = 1;
        }
        ++iter;
        lap(4);
        if (prof_on) s_pt[5] += 1;
    }

    // ---- write the segment back for the host-side phases (reconstruction, selection)
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int li = r * NT + tid, i = seg0 + li;
        const bool in = li < nseg, act = (ST[r] & RST_ACTIVE) != 0;
        if (in) {
            A.f[i] = F[r];
            A.alpha[i] = s_al[li];
            A.status[i] = (uint8_t)(ST[r] & 7);
        }
        const unsigned long long m = __ballot(act);
        if (lane == 0) s_wc[wid] = __popcll(m);
        __syncthreads();
        int off = base;
        for (int w = 0; w < NW; ++w) {
            const int c = s_wc[w];
            off += w < wid ? c : 0;
            base += c;
        }
        if (act) A.act[seg0 + off + __popcll(m & ((1ull << lane) - 1ull))] = i;
        __syncthreads();
    }
    if (tid == 0) A.cnt[blk] = base;
    if (A.work) {
        const unsigned long long wn = wave_sum(work_nnz);
        if (lane == 0) s_v[wid] = __longlong_as_double((long long)wn);
        __syncthreads();
        if (tid == 0) {
            unsigned long long t = 0;
            for (int w = 0; w < NW; ++w) t += (unsigned long long)__double_as_longlong(s_v[w]);
            A.work[4 * blk] = work_rows;
            A.work[4 * blk + 1] = t;
            A.work[4 * blk + 2] = work_rows;
            A.work[4 * blk + 3] = 0;
        }
    }
    if (prof_on) {
        lap(7);
        for (int k = 0; k < PROF_SLOTS; ++k) A.dbg->prof[k] += s_pt[k];
    }
    if (blk == 0 && tid == 0) {
        ctl->b_up = bu; ctl->b_low = bl; ctl->i_up = iu; ctl->i_low = il;
        ctl->a_up = au; ctl->a_low = al;
        ctl->iter = iter; ctl->counter = counter; ctl->n_active = n_act_total;
        ctl->shrink_passes = passes; ctl->shrunk_total = shrunk;
        ctl->exit_reason = exit_reason;
    }
}

template <bool BITS, typename KT, int W4>
static const void* reg_pick_rows(int R) {
    constexpr int RM = reg_rows_max(std::is_same<KT, double>::value, W4);
    if (R == 1) return (const void*)smo_reg_kernel<BITS, KT, W4, 1>;
    if constexpr (RM >= 2)
        if (R == 2) return (const void*)smo_reg_kernel<BITS, KT, W4, 2>;
    if constexpr (RM >= 4)
        if (R == 4) return (const void*)smo_reg_kernel<BITS, KT, W4, 4>;
    return nullptr;
}

}  // namespace svm
