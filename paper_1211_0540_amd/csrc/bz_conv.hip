// Weighted convolution of Sec. 3.2,
//   Qhat_k = sum_m Ghat(xi_m, zeta_k) fhat_m fhat_{k-m+N/2} dzeta^3,
// the O(N^6) step where the method spends its time (Sec. 3.2, Sec. 4).
//
// Two schedules:
//
// * Batched (lane = cell).  64 cells of one mesh share a wavefront, so every
//   weight is wavefront-uniform and is read once per 64 cells.  The weights of
//   a step are contiguous; while a step runs, the next step's weights are
//   copied HBM -> LDS by one coalesced direct-to-LDS load per 1 KiB
//   (global_load_lds_dwordx4) into the other half of a per-wave double buffer,
//   and the running step reads its weights with broadcast LDS reads; from N = 28
//   on the one-launch kernel reads them through the scalar cache instead, with
//   the next step's weights pulled into L2 (cells_step_scalar).  A work item is a range of
//   steps of one output row (k1, k2, 0..N-1) of 64 cells; it keeps
//   the row's N accumulators and, per step (m1, m2), the rows fhat(m1, m2, .)
//   and fhat(j1, j2, .) of its own cell in registers (cell-interleaved layout,
//   coalesced 512-byte loads).  Each unordered pair {m, j} is visited once
//   with the symmetrised weight (see bz_internal.h), so a step costs 6 VALU
//   operations per visited pair: 4 for the complex product fhat_m fhat_j and 2
//   FMAs that add its weighted parts to a fresh per-output partial of the step,
//   plus 2 additions per output and step into the running sums (and 2 more that
//   combine two interleaved partials, where a variant keeps two).  Work items are popped from
//   atomic queues ordered longest first, so the launch is persistent.  Every item names
//   its pass of the conjugate-symmetric schedule (bz_internal.h): which fhat
//   copy it reads, which weight stream and which output buffer it writes; the
//   full-sum schedule uses pass A only.  Steps of pass A whose rows lie on a
//   zeroed plane of its fhat copy (N = 32: 4.5% of them) are left out; of the narrow items
//   (narrow_item) the FP64 ones of N = 20 to 28 leave them out.
//
//   FP32 variant: products, per-step partials and a running sum over FOLD
//   steps in FP32 (the running sum takes one rounding per output and step);
//   every FOLD steps the running sum is folded into a compensated total:
//   an FP64 total in registers (COMP = 0), an FP32 (hi, lo) pair updated with
//   Knuth's error-free TwoSum (COMP = 1, Kahan-style compensation), or an FP64
//   total kept in the item's own output slot and updated by read-modify-write
//   (COMP = 2), which leaves the registers to fit two wavefronts per SIMD at
//   N = 32.  FP64 variant: everything FP64.
//
// * Plain (lane = output), one cell per launch: the lanes of a wavefront are R
//   output rows of one k1 plane; all lanes walk the same m, the weight of each
//   (lane, m) is streamed from HBM in a coalesced layout, fhat_m is uniform and
//   fhat_j is a per-lane read.  This is the paper's precompute-and-store
//   organisation; it is bound by the weight stream.
#include <type_traits>
#include <utility>

#include "bz_internal.h"

// The file is compiled in four units side by side (BZ_CONV_UNIT): 0 the one launch, the cores and the
// dispatch, 1 and 2 the per-mesh FP32 variants of the small and large meshes, 3 FP64 and plain; in
// one unit it takes ten minutes.
#ifndef BZ_CONV_UNIT
#error "compile with -DBZ_CONV_UNIT=0 .. 3"
#endif

namespace bz {
namespace {

template <typename T>
struct cplx;
template <>
struct cplx<float> {
    using t = float2;
};
template <>
struct cplx<double> {
    using t = double2;
};

// TwoSum: hi + lo += p without losing the rounding error of the addition.
__device__ inline void two_sum_acc(float &hi, float &lo, float p) {
    const float s = hi + p;
    const float bp = s - hi;
    const float e = (hi - (s - bp)) + (p - bp);
    hi = s;
    lo += e;
}

// One step of the batched schedule for one row: for each output k3 its terms
// of the step are summed into fresh partials (SPLIT interleaved accumulators,
// combined pairwise), which are then added to the running sum once (one
// rounding of the running sum per output and step).
template <typename T, int N, int SPLIT, typename WP>
__device__ __forceinline__ void cells_step(const typename cplx<T>::t (&mv)[N], const typename cplx<T>::t (&jv)[N],
                                           WP w, T (&pr)[N], T (&pi)[N]) {
    constexpr int h = N / 2;
#pragma unroll
    for (int k3 = 0; k3 < N; ++k3) {
        const int mlo = k3 - h + 1 > 0 ? k3 - h + 1 : 0;
        const int mhi = k3 + h < N - 1 ? k3 + h : N - 1;
        T sr[SPLIT], si[SPLIT];
#pragma unroll
        for (int a = 0; a < SPLIT; ++a) sr[a] = si[a] = 0;
#pragma unroll
        for (int m3 = mlo; m3 <= mhi; ++m3) {
            const int j3 = k3 - m3 + h;
            const int a = (m3 - mlo) % SPLIT;
            const T wt = w[step_koff(N, k3) + (m3 - mlo)];
            // product fhat_m fhat_j first, then one rounding into a partial per term
            const T px = fma(mv[m3].x, jv[j3].x, -(mv[m3].y * jv[j3].y));
            const T py = fma(mv[m3].x, jv[j3].y, mv[m3].y * jv[j3].x);
            sr[a] = fma(wt, px, sr[a]);
            si[a] = fma(wt, py, si[a]);
        }
#pragma unroll
        for (int st = 1; st < SPLIT; st *= 2)
#pragma unroll
            for (int a = 0; a + st < SPLIT; a += 2 * st) {
                sr[a] += sr[a + st];
                si[a] += si[a + st];
            }
        pr[k3] += sr[0];
        pi[k3] += si[0];
    }
}

// Weights through scalar registers.  A VALU instruction takes a scalar operand for free, while a
// broadcast LDS read returns its weights to every lane: 16 bytes to 64 lanes take 16 cycles of the
// CU's LDS, which feed 24 operations, and the four SIMDs issue those in 13 (two wavefronts of a
// SIMD issue one operation per 2 cycles together; one alone, one per 4).  The step's weights come
// in chunks of CW by scalar loads, two chunks in registers: the next one is requested when the
// current one has arrived (scalar loads return in any order, so a wait is a wait for all).
template <typename T, int N>
constexpr int weight_chunk() {
    constexpr int PS = 3 * N * N / 4;
    if (sizeof(T) == 8) return PS % 16 == 0 ? 16 : PS % 12 == 0 ? 12 : 4;
    return PS % 32 == 0 ? 32 : PS % 24 == 0 ? 24 : PS % 28 == 0 ? 28 : PS % 20 == 0 ? 20 : 12;
}
template <typename T, int CW>
struct WeightChunk {
    T v[CW];
};
template <typename T, int CW>
__device__ __forceinline__ WeightChunk<T, CW> load_chunk(const T *w) {
    WeightChunk<T, CW> c;
    const auto *p = (const __attribute__((address_space(4))) T *)w;
#pragma unroll
    for (int i = 0; i < CW; ++i) c.v[i] = p[i];
    return c;
}
// a wavefront-uniform pointer, in scalar registers
template <typename T>
__device__ __forceinline__ const T *uniform_ptr(const T *p) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return (const T *)(((unsigned long long)hi << 32) | lo);
}
template <int... I, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}

// cells_step with the weights of the step at w (global memory, wavefront-uniform) through scalar
// registers; `cur` holds the first chunk of the step and, on return, that of the next, whose weights are at wn
template <typename T, int N, int SPLIT, int CW>
__device__ __forceinline__ void cells_step_scalar(const typename cplx<T>::t (&mv)[N], const typename cplx<T>::t (&jv)[N],
                                                  const T *w, const T *wn, WeightChunk<T, CW> &cur, T (&pr)[N], T (&pi)[N]) {
    constexpr int h = N / 2, PS = 3 * N * N / 4;
    WeightChunk<T, CW> nxt;
    static_for(std::make_integer_sequence<int, N>{}, [&](auto K) {
        constexpr int k3 = K;
        constexpr int mlo = k3 - h + 1 > 0 ? k3 - h + 1 : 0;
        constexpr int mhi = k3 + h < N - 1 ? k3 + h : N - 1;
        T sr[SPLIT], si[SPLIT];
#pragma unroll
        for (int a = 0; a < SPLIT; ++a) sr[a] = si[a] = 0;
        static_for(std::make_integer_sequence<int, mhi - mlo + 1>{}, [&](auto I) {
            constexpr int m3 = mlo + I, j3 = k3 - m3 + h, a = I % SPLIT, t = step_koff(N, k3) + I;
            if constexpr (t % CW == 0) {
                if (t > 0) cur = nxt;
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the current chunk is here
                nxt = load_chunk<T, CW>(t + CW < PS ? w + t + CW : wn);
                __builtin_amdgcn_sched_barrier(0);
            }
            const T wt = cur.v[t % CW];
            const T px = fma(mv[m3].x, jv[j3].x, -(mv[m3].y * jv[j3].y));
            const T py = fma(mv[m3].x, jv[j3].y, mv[m3].y * jv[j3].x);
            sr[a] = fma(wt, px, sr[a]);
            si[a] = fma(wt, py, si[a]);
        });
#pragma unroll
        for (int st = 1; st < SPLIT; st *= 2)
#pragma unroll
            for (int a = 0; a + st < SPLIT; a += 2 * st) {
                sr[a] += sr[a + st];
                si[a] += si[a + st];
            }
        pr[k3] += sr[0];
        pi[k3] += si[0];
    });
    cur = nxt;
}

template <typename T, int N>
__device__ __forceinline__ void load_row(const typename cplx<T>::t *__restrict__ p, typename cplx<T>::t (&v)[N]) {
#pragma unroll
    for (int t = 0; t < N; ++t) v[t] = p[t * kWave];
}

// Copy `chunks` KiB of a step's weights from global memory to LDS: each lane
// moves 16 bytes per chunk, the wave 1 KiB, landing contiguously at dst.
typedef __attribute__((address_space(3))) char lds_char;

// LDS address of a __shared__ object, taken directly so that no generic-to-LDS
// conversion of a computed pointer is needed.
template <typename T>
__device__ __forceinline__ lds_char *lds_ptr(T *shared_obj) {
    return (lds_char *)shared_obj;
}

template <int CHUNKS>
__device__ __forceinline__ void prefetch_weights(const void *src, lds_char *dst) {
    const char *g = (const char *)src + threadIdx.x * 16;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c)
        __builtin_amdgcn_global_load_lds((const void *)(g + c * 1024), (void __attribute__((address_space(3))) *)(dst + c * 1024),
                                         16, 0, 0);
}

// Position (m1, m2) of step index s0 in the row's step enumeration.
template <int N>
__device__ __forceinline__ void seek_step(int k1, int k2, int s0, int &m1, int &m2) {
    const int lo2 = axis_lo(N, k2);
    m1 = axis_lo(N, k1);
    for (;;) {
        const int cnt = cells_m2_last(N, k1, k2, m1) - lo2 + 1;
        if (s0 < cnt) break;
        s0 -= cnt;
        ++m1;
    }
    m2 = lo2 + s0;
}

// The steps of a row from step s0 on.  With `cut` (pass A on the plane-zeroed copy, rows k2 < N/2)
// those with m2 = 0 or j2 = 0, whose products are all zero, are left out: per m1 the first and, below the
// diagonal, the last (evaluations with / without them: FP32 N = 32 128 cells 2.75 / 2.71 ms, 190 4.09 / 4.00, N = 28 128 1.475 / 1.433;
// FP64 N = 24 128 1.291 / 1.245, N = 32 190 8.41 / 8.20).
template <int N>
struct StepWalk {
    int k1, k2, lo2, m1, m2, s;
    bool cut;
    __device__ StepWalk(int k1_, int k2_, int s0, bool cut_) : k1(k1_), k2(k2_), lo2(axis_lo(N, k2_)), s(s0), cut(cut_) {
        seek_step<N>(k1, k2, s0, m1, m2);
        skip();
    }
    __device__ void next() {
        ++s;
        if (++m2 > cells_m2_last(N, k1, k2, m1)) {
            ++m1;
            m2 = lo2;
        }
        skip();
    }

  private:
    __device__ void skip() {
        if (!cut) return;
        if (m2 == k2 + N / 2) {
            ++m1;
            m2 = 0;
            ++s;
        }
        if (m2 == 0) {
            m2 = 1;
            ++s;
        }
    }
};

// The pass of an item (wavefront-uniform): its fhat copy, weights and output buffer.
__device__ __forceinline__ ConvPass pick_pass(const ConvPasses &ps, int pass) {
    ConvPass c = ps.p[0];
    if (pass == kPassE1) c = ps.p[kPassE1];
    if (pass == kPassE2) c = ps.p[kPassE2];
    if (pass == kPassE3) c = ps.p[kPassE3];
    if (pass == kPassZ) c = ps.p[kPassZ];
    return c;
}

__device__ inline int pop_item(unsigned *counter) {
    unsigned it = 0;
    if (threadIdx.x == 0) it = atomicAdd(counter, 1u);
    return (int)__builtin_amdgcn_readfirstlane(it);
}

// ---------------------------------------------------------------------------
// Batched FP32 with compensated accumulation.  One work item: the body is
// shared by the one-mesh kernel and by the kernel whose queue holds the items
// of several meshes (an item names its mesh; N is wavefront-uniform).
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) double lds_double;

template <int N, int FOLD, int COMP, int WP, int RP, int SPLIT>
__device__ __forceinline__ void cells_f32_item(const float2 *__restrict__ fh, double2 *__restrict__ qh,
                                               const unsigned char *__restrict__ skip, const ConvPass &cp,
                                               const int4 item, lds_char *const wl, lds_char *const rl) {
    constexpr int h = N / 2, M = N * N * N, PS = 3 * N * N / 4;
    constexpr int CH = (PS * 4 + 1023) / 1024;       // KiB per step of weights
    constexpr int RCH = N * kWave * 8 / 1024;        // KiB per fhat row of 64 cells
    const int lane = threadIdx.x;
    const int g = item.x, r = item.y & 0xffff, part = (item.y >> 16) & 0xf, s0 = item.z, s1 = item.w;
    const int k1 = r / N, k2 = r - k1 * N;
    double2 *const out = qh + cp.out_off + part * cp.pstride + g * cp.gstride + (size_t)(r - cp.row0) * N * kWave + lane;
    if (skip && skip[g]) {
        // every cell of the group is served elsewhere: leave zeros in this item's outputs
#pragma unroll
        for (int t = 0; t < N; ++t) out[t * kWave] = make_double2(0.0, 0.0);
        return;
    }
    StepWalk<N> at(k1, k2, s0, WP == 3 && cp.zero_planes && k2 < h);
    const float *w = (const float *)cp.w + cp.row_woff[r] + (long long)(at.s < s1 ? at.s : s0) * PS;
    if constexpr (WP == 3) w = uniform_ptr(w);
    const float2 *G = fh + cp.fh_off + (size_t)g * M * kWave;   // this group's fhat (copy of the pass)
    const float2 *F = G + lane;
    const lds_float *const rbuf = (const lds_float *)rl;   // rows as (re, im) float pairs

    float pr[N], pi[N];
    float hr[N], hi[N], lr[N], li[N];
    double dr[N], di[N];
#pragma unroll
    for (int t = 0; t < N; ++t) {
        pr[t] = pi[t] = 0.f;
        if (COMP == 1) hr[t] = hi[t] = lr[t] = li[t] = 0.f;
        else if (COMP == 0) dr[t] = di[t] = 0.0;
    }
    bool first = true;
    auto fold = [&]() {
        if (COMP == 2) {
            // the FP64 total lives in this item's own output slot (no other item writes it)
#pragma unroll
            for (int t = 0; t < N; ++t) {
                double2 o = make_double2(0.0, 0.0);
                if (!first) o = out[t * kWave];
                o.x += (double)pr[t];
                o.y += (double)pi[t];
                out[t * kWave] = o;
                pr[t] = pi[t] = 0.f;
            }
            first = false;
            return;
        }
#pragma unroll
        for (int t = 0; t < N; ++t) {
            if (COMP == 1) {
                two_sum_acc(hr[t], lr[t], pr[t]);
                two_sum_acc(hi[t], li[t], pi[t]);
            } else {
                dr[t] += (double)pr[t];
                di[t] += (double)pi[t];
            }
            pr[t] = pi[t] = 0.f;
        }
    };
    // rows of step (m1, m2): fhat(m1, m2, .) and fhat(j1, j2, .) of the 64 cells, N/2 KiB each
    auto prefetch_rows = [&](int a1, int a2) {
        prefetch_weights<RCH>(G + (size_t)((a1 * N + a2) * N) * kWave, rl);
        prefetch_weights<RCH>(G + (size_t)(((k1 + h - a1) * N + (k2 + h - a2)) * N) * kWave, rl + RCH * 1024);
    };

    constexpr int CW = weight_chunk<float, N>();
    WeightChunk<float, CW> wc;
    if constexpr (WP == 3) wc = load_chunk<float, CW>(w);
    else prefetch_weights<CH>(w, wl);
    if (RP && s0 < s1) prefetch_rows(at.m1, at.m2);
    if (WP != 3) __builtin_amdgcn_s_waitcnt(0);
    int buf = 0, nst = at.s - s0;
    while (at.s < s1) {
        const int m1 = at.m1, m2 = at.m2, j1 = k1 + h - m1, j2 = k2 + h - m2;
        // on a plane-zeroed copy a step with m2 = 0 or j2 = 0 has only zero products (the scalar
        // weights leave it out, the others its arithmetic)
        const bool live = WP == 3 || !cp.zero_planes || (m2 != 0 && j2 != 0);
        StepWalk<N> nx = at;
        nx.next();
        float2 mv[N], jv[N];
        if (RP) {
#pragma unroll
            for (int t = 0; t < N; ++t) {
                const int a = 2 * (t * kWave + lane), b = 2 * (N * kWave + t * kWave + lane);
                mv[t] = make_float2(rbuf[a], rbuf[a + 1]);
                jv[t] = make_float2(rbuf[b], rbuf[b + 1]);
            }
            __builtin_amdgcn_s_waitcnt(0);        // rows are in registers: the buffer is free
            if (nx.s < s1) prefetch_rows(nx.m1, nx.m2);
        } else {
            load_row<float, N>(F + (size_t)((m1 * N + m2) * N) * kWave, mv);
            load_row<float, N>(F + (size_t)((j1 * N + j2) * N) * kWave, jv);
        }
        if (WP == 0) {
            // next step's weights into the other LDS half; this step reads its half
            prefetch_weights<CH>(w + PS, wl + (buf ^ 1) * CH * 1024);
            if (live) cells_step<float, N, SPLIT>(mv, jv, (const lds_float *)(wl + buf * CH * 1024), pr, pi);
        } else if (WP == 3) {
            // the next step's weights pulled into L2 (64 bytes a lane, the LDS copy is discarded)
            constexpr int WL = (PS * 4 + 4095) / 4096;
            const float *const wn = w + (nx.s < s1 ? nx.s - at.s : 1) * PS;
#pragma unroll
            for (int c = 0; c < WL; ++c)
                __builtin_amdgcn_global_load_lds((const void *)((const char *)wn + lane * 64 + c * 4096),
                                                 (void __attribute__((address_space(3))) *)rl, 4, 0, 0);
            cells_step_scalar<float, N, SPLIT, CW>(mv, jv, w, wn, wc, pr, pi);
            w = wn;
        } else if (WP == 1) {
            // next step's weights pulled into L2 (the LDS copy is discarded); this
            // step's weights, pulled last step, are read through the scalar cache
            prefetch_weights<CH>(w + PS, wl + CH * 1024);
            if (live)
                cells_step<float, N, SPLIT>(mv, jv, (const __attribute__((address_space(4))) float *)w, pr, pi);
        } else {
            // as 1, but the weights are read by uniform-address vector loads
            prefetch_weights<CH>(w + PS, wl + CH * 1024);
            if (live) cells_step<float, N, SPLIT>(mv, jv, w, pr, pi);
        }
        if (WP != 3) w += PS;
        buf ^= 1;
        // steps left out count, so that a sum is folded where it is without
        nst += nx.s - at.s;
        if (nst >= FOLD) {
            fold();
            nst -= FOLD;
        }
        at = nx;
        if (WP != 3) __builtin_amdgcn_s_waitcnt(0);
    }
    fold();
    if (COMP == 2) return;
#pragma unroll
    for (int t = 0; t < N; ++t) {
        if (COMP == 1)
            out[t * kWave] = make_double2((double)hr[t] + (double)lr[t], (double)hi[t] + (double)li[t]);
        else
            out[t * kWave] = make_double2(dr[t], di[t]);
    }
}

template <int N, int FOLD, int COMP, int WP, int RP, int SPLIT>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(COMP == 2 ? 2 : 1)))
k_conv_cells_f32(const float2 *__restrict__ fh, const int4 *__restrict__ items, int n_items,
                 unsigned *__restrict__ counter, double2 *__restrict__ qh,
                 const unsigned char *__restrict__ skip, const ConvPasses ps) {
    constexpr int PS = 3 * N * N / 4;
    constexpr int CH = (PS * 4 + 1023) / 1024;
    __shared__ __attribute__((aligned(16))) float wbuf[2][CH * 256];
    __shared__ __attribute__((aligned(16))) float2 rbuf[RP ? 2 * N * kWave : 2];
    lds_char *const wl = lds_ptr(&wbuf[0][0]);
    lds_char *const rl = lds_ptr(&rbuf[0]);
    for (;;) {
        const int it = pop_item(counter);
        if (it >= n_items) break;
        const int4 item = items[it];
        const ConvPass cp = pick_pass(ps, (item.y >> 20) & 0xf);
        cells_f32_item<N, FOLD, COMP, WP, RP, SPLIT>(fh, qh, skip, cp, item, wl, rl);
    }
}

// One item of a narrow group (NarrowTail: W = 2^lw cells).  The 64 lanes take W cells times
// S = 64 / W consecutive steps of the row: lane l computes the per-output partials of step
// s + l / W for cell l % W, with that step's weights, so the row's steps take 1/S as many
// passes as with one cell on every lane and the other lanes idle (one
// N=32 cell: 0.30 against 1.41 ms).  The partials go to LDS, half a row at a time, and are then added
// to the running sums in step order, so the sums are bitwise those of a 64-cell group: a cell's
// result does not depend on the width of its group.  The weights are read from memory once per
// 16 bytes and lane (a step's weights are contiguous), kRing reads ahead of their use.  These reads take 16
// cycles of the CU's L1 per 24 operations, as the broadcasts of LDS: 56 of the 316 us of a launch for one
// N = 32 cell, so a pass is bound by its latencies (the row loads before it, the two flushes through
// LDS in it, at W = 4 a fold in every pass) rather than by a rate.
// LDS: [N values][64 lanes] partials, [2N values][W cells] running sums (W <= 32).  FP64 items (one partial per output and step, no fold) take the same
// form at half the read-ahead (one N = 32 cell: 0.97 against
// 2.9 ms an evaluation).
// CUT: the steps on a zeroed plane are left out as in the wide items (StepWalk), in FP64 from N = 20 to 28 (evaluations of
// 16 cells: N = 20 190 -> 188 us, N = 24 388 -> 379, N = 28 1207 -> 1158).  At N = 32, short of registers, it cost
// 5%, below N = 20 it gave nothing, and in FP32, whose totals are folded by the steps' indices, up to 2% at
// W = 4 against 2% lost at W = 32 and 1% in the wide items of the launch.
// REMAT: what is the same in every pass (LDS addresses, row strides) is computed again in each: kept
// live it takes registers that the wide body of the same kernel is short of (FP64, N = 32: 16
// cells 2.77 -> 2.34 ms an evaluation).
template <typename T>
constexpr int narrow_lds_bytes(int N) {
    return (int)sizeof(T) * N * (kWave + 2 * (kWave / 2));
}
template <typename T>
struct vec4;
template <>
struct vec4<float> {
    using t = float4;
};
template <>
struct vec4<double> {
    using t = double4;
};
template <typename T, int N, bool REMAT, bool CUT>
__device__ __forceinline__ void narrow_item(const typename cplx<T>::t *fh, double2 *qh, const ConvPass &cp, const int4 item,
                                            const int lw, lds_char *lds, lds_char *sink) {
    using C = typename cplx<T>::t;
    using T4 = typename vec4<T>::t;
    typedef __attribute__((address_space(3))) T lds_t;
    constexpr bool f32 = sizeof(T) == 4;
    constexpr int h = N / 2, M = N * N * N, PS = 3 * N * N / 4, FOLD = 16, kRing = f32 ? 14 : 7, SPLIT = f32 ? 2 : 1;
    constexpr int CB = (int)sizeof(C), CS = f32 ? 3 : 4;   // bytes of a complex value, and their log2
    const int W = 1 << lw, S = kWave >> lw;
    int lane = threadIdx.x;
    if constexpr (REMAT) asm volatile("" : "+v"(lane));
    const int cell = lane & (W - 1), slice = lane >> lw;
    const int g = item.x, r = item.y & 0xffff, part = (item.y >> 16) & 0xf, s0 = item.z, s1 = item.w;
    const int k1 = r / N, k2 = r - k1 * N, lo2 = axis_lo(N, k2);
    double *const out = (double *)(qh + cp.out_off + part * cp.pstride + g * cp.gstride) +
                        ((size_t)(r - cp.row0) * N << (lw + 1));
    lds_t *const part_l = (lds_t *)lds, *const run_l = part_l + N * kWave;
    for (int i = lane; i < 2 * N * W; i += kWave) run_l[i] = 0;
    if (s0 >= s1) {
        for (int i = lane; i < 2 * N * W; i += kWave) out[i] = 0.0;
        return;
    }
    const char *const wu = (const char *)uniform_ptr((const T *)cp.w + cp.row_woff[r] + (long long)s0 * PS);
    const char *const G = (const char *)uniform_ptr(fh + cp.fh_off + (size_t)g * M * kWave);
    // this lane's step, of index `at` in the row, or one of the item past its last step
    int m1, m2, at = slice < s1 - s0 ? s0 + slice : s1 - 1;
    const bool cut = CUT && __builtin_amdgcn_readfirstlane(cp.zero_planes) && k2 < h;
    const int lo = cut ? 1 : lo2;
    auto row_end = [&](int last) { return cut && last == k2 + h ? last - 1 : last; };
    int s = s0, next = s0 + S;   // the first slice's step of this pass and of the next (CUT: in turn)
    if constexpr (CUT) at = s0;
    seek_step<N>(k1, k2, at, m1, m2);
    // n steps on
    auto advance = [&](int n) {
        at += n;
        for (m2 += n;;) {
            const int last = cells_m2_last(N, k1, k2, m1), end = row_end(last);
            if (m2 <= end) break;
            m2 -= end - lo + 1;
            at += last - end + lo - lo2;
            ++m1;
        }
    };
    int m1_0 = 0, m2_0 = 0, at_0 = 0;
    if constexpr (CUT) {
        const int off = m2 < lo;
        m2 += off;
        at += off;
        advance(0);
        s = __builtin_amdgcn_readfirstlane(at);
        if (s >= s1) {
            for (int i = lane; i < 2 * N * W; i += kWave) out[i] = 0.0;
            return;
        }
        m1_0 = m1;
        m2_0 = m2;
        at_0 = at;
        advance(slice);
    }
    // weights of the pass at step s pulled into L2, one 128-byte line per lane and load (the copies
    // in LDS are discarded): a pass reads its S steps' weights far faster than memory answers
    // one line after the other
    auto touch = [&](int s) {
        int n = s1 - s < S ? s1 - s : S;
        if constexpr (CUT) {
            const int b = __builtin_amdgcn_readlane(at, kWave - 1);
            n = (b < s1 ? b + 1 : s1) - s;
        }
        const int bytes = n * (PS * (int)sizeof(T));
        for (int o = lane * 128; o < bytes; o += kWave * 128)
            __builtin_amdgcn_global_load_lds((const void *)(wu + (size_t)(s - s0) * (PS * sizeof(T)) + o),
                                             (void __attribute__((address_space(3))) *)sink, 4, 0, 0);
    };
    touch(s);
    bool first = true;
    for (; s < s1; s = next) {
        int left = s1 - s < S ? s1 - s : S;                   // steps of this pass
        int c1 = m1, c2 = m2, ca = at;
        if constexpr (CUT) {
            const bool in = at < s1;
            left = __builtin_popcountll(__ballot(in)) >> lw;
            c1 = in ? m1 : m1_0;
            c2 = in ? m2 : m2_0;
            ca = in ? at : at_0;
            advance(S);
            next = __builtin_amdgcn_readfirstlane(at);
        } else {
            next = s + S;
        }
        int pl = lane, plw = lw;                              // this pass's copies
        if constexpr (REMAT) asm volatile("" : "+v"(pl), "+s"(plw));
        const bool fold = (f32 && (next - s0) % FOLD == 0) || next >= s1;
        const unsigned um = (unsigned)((((c1 * N + c2) * N) << lw) + cell) * (unsigned)CB;
        const unsigned uj = (unsigned)(((((k1 + h - c1) * N + (k2 + h - c2)) * N) << lw) + cell) * (unsigned)CB;
        const unsigned uw = (unsigned)(ca - s0) * (unsigned)(PS * sizeof(T));
        C mv[N], jv[N];
#pragma unroll
        for (int t = 0; t < N; ++t) {
            mv[t] = *(const C *)(G + (t << (plw + CS)) + um);
            jv[t] = *(const C *)(G + (t << (plw + CS)) + uj);
        }
        if (next < s1) touch(next);
        T4 ring[kRing];
#pragma unroll
        for (int i = 0; i < kRing; ++i) ring[i] = *(const T4 *)(wu + uw + i * (4 * sizeof(T)));
        // the running sums of outputs k3 = K h .. K h + h - 1 from the partials in LDS
        auto flush = [&](int half) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int i = lane; i < N * W; i += kWave) {
                const int v = i >> lw, c = i & (W - 1), sw = (v << lw) & (kWave - 1), o = half * N * W + i;
                T run = run_l[o];
                for (int q = 0; q < left; ++q) run += part_l[v * kWave + (((q << lw) + c) ^ sw)];
                if (fold) {
                    // value v is component v % 2 of output k3 = half h + v / 2
                    double *const p = out + (((size_t)(half * h + (v >> 1)) << lw) + c) * 2 + (v & 1);
                    *p = (first ? 0.0 : *p) + (double)run;
                    run = 0;
                }
                run_l[o] = run;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        static_for(std::make_integer_sequence<int, N>{}, [&](auto K) {
            constexpr int k3 = K;
            constexpr int mlo = k3 - h + 1 > 0 ? k3 - h + 1 : 0;
            constexpr int mhi = k3 + h < N - 1 ? k3 + h : N - 1;
            T sr[SPLIT], si[SPLIT];
#pragma unroll
            for (int a = 0; a < SPLIT; ++a) sr[a] = si[a] = 0;
            static_for(std::make_integer_sequence<int, mhi - mlo + 1>{}, [&](auto I) {
                constexpr int m3 = mlo + I, j3 = k3 - m3 + h, a = I % SPLIT, t = step_koff(N, k3) + I, c = t / 4;
                const T4 q = ring[c % kRing];
                const T wt = t % 4 == 0 ? q.x : t % 4 == 1 ? q.y : t % 4 == 2 ? q.z : q.w;
                const T px = fma(mv[m3].x, jv[j3].x, -(mv[m3].y * jv[j3].y));
                const T py = fma(mv[m3].x, jv[j3].y, mv[m3].y * jv[j3].x);
                sr[a] = fma(wt, px, sr[a]);
                si[a] = fma(wt, py, si[a]);
                if constexpr (t % 4 == 3 && c + kRing < PS / 4)
                    ring[c % kRing] = *(const T4 *)(wu + uw + (c + kRing) * (4 * sizeof(T)));
            });
            // lane positions rotated by value, so that lanes reading different values hit different banks
            constexpr int v = 2 * (k3 % h);
            part_l[v * kWave + (pl ^ ((v << plw) & (kWave - 1)))] = f32 ? sr[0] + sr[SPLIT - 1] : sr[0];
            part_l[(v + 1) * kWave + (pl ^ (((v + 1) << plw) & (kWave - 1)))] = f32 ? si[0] + si[SPLIT - 1] : si[0];
            if constexpr (k3 % h == h - 1) flush(k3 / h);
        });
        if (fold) first = false;
        if constexpr (!CUT) {
            // this lane's next step
            const int nx = at + S < s1 ? at + S : s1 - 1;
            for (m2 += nx - at, at = nx;;) {
                const int last = cells_m2_last(N, k1, k2, m1);
                if (m2 <= last) break;
                m2 -= last - lo2 + 1;
                ++m1;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// FP64 core of the batched FP32 mode (CoreSched in bz_internal.h): the pairs
// whose two partners lie in the low-frequency ball carry the largest terms of
// the sum, so they are summed here in FP64 from FP64 fhat, with FP64 weights.
// Lane = cell, like the batched kernels; an item is one output row of one
// group.  A step loads its two rows (2R + 1 values each) and reads its
// (2R + 1)^2 weights by scalar loads.  Item
// kinds (bits 16..17 of the row word): 2 = every output of the row
// (k3 - N/2 in [-2R, 2R]); 0 = only k3 - N/2 in [-2R, 0] (rows whose other
// outputs follow from conjugate symmetry); 1 = only [1, 2R].  A full row
// loads each row value once for 2R + 1 products.
// ---------------------------------------------------------------------------
template <int R, int KIND>
struct CoreOut {
    static constexpr int lo = KIND == 1 ? 1 : -2 * R;
    static constexpr int hi = KIND == 0 ? 0 : 2 * R;
    static constexpr int n = hi - lo + 1;
};

// One core step: rows pm and pj of half-widths am and aj inside the ball (wavefront-uniform; entries
// beyond them are zero), weights at w, through scalar registers like the FP32 items': the row of S
// weights of the next m value is requested while the current one is used, and the m values are
// loaded kAhead before their use.  (Weights from LDS, each read waited for between the branches of
// its product, took 14 of the 18 us of a step: one N = 32 cell 915 us a launch, its FP32 items
// 330.)  m values outside the ball are skipped, and j values kTj at a time.
template <int R, int KIND>
__device__ __forceinline__ void core_step(const double2 *pm, const double2 *pj, int am, int aj, const double *w,
                                          double2 (&acc)[CoreOut<R, KIND>::n]) {
    constexpr int S = 2 * R + 1, LO = CoreOut<R, KIND>::lo, HI = CoreOut<R, KIND>::hi, kAhead = 3, kTj = 2;
    double2 jr[S], mr[kAhead];
#pragma unroll
    for (int t = 0; t < kAhead; ++t) mr[t] = pm[t * kWave];
#pragma unroll
    for (int t = 0; t < S; ++t) jr[t] = pj[t * kWave];
    WeightChunk<double, S> cur = load_chunk<double, S>(w), nxt;
    static_for(std::make_integer_sequence<int, S>{}, [&](auto T) {
        constexpr int tm = T;
        const double2 mv = mr[tm % kAhead];
        if constexpr (tm + kAhead < S) mr[tm % kAhead] = pm[(tm + kAhead) * kWave];
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
        if constexpr (tm + 1 < S) nxt = load_chunk<double, S>(w + (tm + 1) * S);
        constexpr int dm = tm < R ? R - tm : tm - R;
        if (dm <= am) {
            // j values R - a and R + a
            static_for(std::make_integer_sequence<int, (R + kTj) / kTj>{}, [&](auto B) {
                constexpr int a0 = B * kTj;
                if (a0 > aj) return;
                static_for(std::make_integer_sequence<int, 2 * kTj>{}, [&](auto I) {
                    constexpr int a = a0 + I / 2, tj = I % 2 ? R + a : R - a, e = tm + tj - 2 * R;   // k3 - N/2
                    if constexpr (a <= R && (a > 0 || I % 2) && e >= LO && e <= HI) {
                        const double wt = cur.v[tj];
                        const double px = fma(mv.x, jr[tj].x, -(mv.y * jr[tj].y));
                        const double py = fma(mv.x, jr[tj].y, mv.y * jr[tj].x);
                        acc[e - LO].x = fma(wt, px, acc[e - LO].x);
                        acc[e - LO].y = fma(wt, py, acc[e - LO].y);
                    }
                });
            });
        }
        cur = nxt;
    });
}

template <int R, int KIND>
__device__ __forceinline__ void core_rows(int N, const double2 *G, const int *steps, const int *ext, const double *ws,
                                          int s0, int s1, double2 *o, lds_char *sink) {
    constexpr int S = 2 * R + 1, WS = core_wstride(R), WL = (WS * 8 + 8191) / 8192;
    constexpr int LO = CoreOut<R, KIND>::lo, NO = CoreOut<R, KIND>::n;
    const int h = N / 2, lane = threadIdx.x;
    double2 acc[NO];
#pragma unroll
    for (int a = 0; a < NO; ++a) acc[a] = make_double2(0.0, 0.0);
    const double *w = uniform_ptr(ws);
    // a step's rows and their half-widths, read a step ahead
    int st = s0 < s1 ? steps[s0] : 0, em = ext[st & 0xffff], ej = ext[st >> 16];
    for (int s = s0; s < s1; ++s) {
        const int dm = __builtin_amdgcn_readfirstlane(st) & 0xffff, dj = __builtin_amdgcn_readfirstlane(st) >> 16;
        const int am = __builtin_amdgcn_readfirstlane(em), aj = __builtin_amdgcn_readfirstlane(ej);
        const int sn = steps[s + 1 < s1 ? s + 1 : s];
        // the next step's weights pulled into L2, a 128-byte line per lane (the copy in LDS is discarded)
#pragma unroll
        for (int c = 0; c < WL; ++c)
            if (lane * 128 + c * 8192 < WS * 8)
                __builtin_amdgcn_global_load_lds((const void *)((const char *)(w + WS) + lane * 128 + c * 8192),
                                                 (void __attribute__((address_space(3))) *)sink, 4, 0, 0);
        core_step<R, KIND>(G + (size_t)dm * S * kWave, G + (size_t)dj * S * kWave, am, aj, w, acc);
        w += WS;
        st = sn;
        em = ext[sn & 0xffff];
        ej = ext[sn >> 16];
    }
#pragma unroll
    for (int a = 0; a < NO; ++a) {
        const int k3 = h + LO + a;
        if (k3 >= 0 && k3 < N) o[k3 * kWave] = acc[a];
    }
}

// One core item: group g, output row, kind; rows of the group from cf, weights of
// step s at w + s * core_wstride(R), outputs into out [G][N^3][64].
template <int R>
__device__ __forceinline__ void core_item(int N, int nD, const double2 *cf, const int *steps, const int *ext,
                                          const double *w, double2 *out, long long pstride, const int4 item,
                                          lds_char *wl) {
    constexpr int S = 2 * R + 1, WS = core_wstride(R);
    const int lane = threadIdx.x;
    const int g = item.x, row = item.y & 0xffff, kind = (item.y >> 16) & 3, piece = (item.y >> 20) & 0xf;
    const int s0 = item.z, s1 = item.w;
    double2 *const o = out + (size_t)piece * pstride + ((size_t)g * N * N * N + (size_t)row * N) * kWave + lane;
    const double2 *const G = cf + (size_t)g * nD * S * kWave + lane;
    const double *ws = w + (size_t)s0 * WS;
    if (kind == 2) core_rows<R, 2>(N, G, steps, ext, ws, s0, s1, o, wl);
    else if (kind == 0) core_rows<R, 0>(N, G, steps, ext, ws, s0, s1, o, wl);
    else core_rows<R, 1>(N, G, steps, ext, ws, s0, s1, o, wl);
}

// One core item of a narrow group of W = 2^lw cells, W <= 8: the outputs of the row are spread over the
// lanes too.  With S = 2R + 1, lane l takes cell l % W and the residues rho = l / W, l / W + 64 / W, ...
// below S; for a residue each m value meets one j value, tj = rho - tm (mod S), whose product goes to output
// tm + tj = rho or rho + S.  A step is then S products and loads per residue, all independent, in place of
// S^2 products one after the other (one N = 32 cell: 490 us a launch with the wide item, whose longest
// row of 50 steps outlasted everything else by 200 us).  Each output takes its products in the
// same order as in the wide item (those left out there are zero), so the sums are bitwise equal.
template <int R>
__device__ __forceinline__ void narrow_core_item(int N, int nD, const double2 *cf, const int *steps, const double *w,
                                                 double2 *out, long long pstride, const int4 item, int lw) {
    constexpr int S = 2 * R + 1, WS = core_wstride(R);
    const int lane = threadIdx.x, cell = lane & ((1 << lw) - 1), h = N / 2;
    const int g = item.x, row = item.y & 0xffff, kind = (item.y >> 16) & 3, piece = (item.y >> 20) & 0xf;
    double2 *const o = out + (size_t)piece * pstride + ((size_t)g * N * N * N + (size_t)row * N) * kWave + cell;
    const double2 *const G = cf + (size_t)g * nD * S * kWave + cell;
    for (int rho = lane >> lw; rho < S; rho += kWave >> lw) {
        double2 lo = make_double2(0.0, 0.0), hi = lo;
        int st = item.z < item.w ? steps[item.z] : 0;
        for (int s = item.z; s < item.w; ++s) {
            const double2 *const pm = G + (size_t)(st & 0xffff) * S * kWave, *const pj = G + (size_t)(st >> 16) * S * kWave;
            const double *const ws = w + (size_t)s * WS;
            st = steps[s + 1 < item.w ? s + 1 : s];
            double2 mv[S], jv[S];
            double wt[S];
#pragma unroll
            for (int tm = 0; tm < S; ++tm) {
                const int tj = rho - tm + (tm > rho ? S : 0);
                mv[tm] = pm[tm * kWave];
                jv[tm] = pj[tj * kWave];
                wt[tm] = ws[tm * S + tj];
            }
#pragma unroll
            for (int tm = 0; tm < S; ++tm) {
                const double px = fma(mv[tm].x, jv[tm].x, -(mv[tm].y * jv[tm].y));
                const double py = fma(mv[tm].x, jv[tm].y, mv[tm].y * jv[tm].x);
                double2 &acc = tm > rho ? hi : lo;
                acc.x = fma(wt[tm], px, acc.x);
                acc.y = fma(wt[tm], py, acc.y);
            }
        }
        // outputs k3 - N/2 = rho - 2R and rho - 2R + S, within the item's kind and the mesh
        const int e0 = rho - 2 * R, e1 = e0 + S;
        if (kind != 1 && h + e0 >= 0) o[(h + e0) * kWave] = lo;
        if (rho < S - 1 && (e1 <= 0 ? kind != 1 : kind != 0) && h + e1 >= 0 && h + e1 < N) o[(h + e1) * kWave] = hi;
    }
}

template <int R>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_conv_core(int N, int nD, const double2 *__restrict__ cf, const int4 *__restrict__ items, int n_items,
            unsigned *__restrict__ counter, const int *__restrict__ steps, const int *__restrict__ ext,
            const double *__restrict__ w, double2 *__restrict__ out, long long pstride,
            const unsigned char *__restrict__ skip) {
    __shared__ __attribute__((aligned(16))) float sink[kWave];
    lds_char *const wl = lds_ptr(&sink[0]);
    for (;;) {
        const int it = pop_item(counter);
        if (it >= n_items) break;
        const int4 item = items[it];
        if (skip && skip[item.x]) continue;   // the closure serves every cell of the group
        core_item<R>(N, nD, cf, steps, ext, w, out, pstride, item, wl);
    }
}

// Items of several meshes in one persistent launch: the mesh index sits in bits 24..27
// of the item word; its descriptor (N, buffer offsets in the workspace, one ConvPass per
// pass, its FP64 core) is read from a device table with wavefront-uniform loads.  Every
// mesh runs the output-slot accumulation with FOLD 16 and two interleaved partials
// (tuning variant 12: with the FP64 core as accurate as four, and 1% faster), two
// wavefronts per SIMD.  Items with kCoreItemBit are rows of an
// FP64 core (core_item): spread through the queue, their row loads overlap the FP32
// arithmetic of the other wavefront on the SIMD.
// Weights by scalar loads from N = 28 on (N = 32, 190 cells: 3.9 against 4.2 ms a launch, whose
// LDS broadcasts return 64 bytes a cycle and CU, less than the four SIMDs consume); below, where
// a step is short (N = 16: 192 pairs, N = 32: 768), the wait for each chunk costs about what the broadcasts
// do: N = 16 72 to 521 cells within 1%, one cell 2% slower; N = 24 256 cells 2% faster by scalar loads (2.65
// against 2.71 ms a Strang step), 72 cells, of which 8 are narrow, 3% slower (1.06 against 1.03).
template <int N>
constexpr int multi_weight_path() {
    return N >= 28 ? 3 : 0;
}
template <int N>
__device__ __forceinline__ void multi_item(const MeshConvDesc &d, char *ws, int pass, const int4 item, lds_char *wl,
                                           lds_char *sink) {
    const ConvPass cp = d.ps.p[pass];
    cells_f32_item<N, 16, 2, multi_weight_path<N>(), 0, 2>((const float2 *)(ws + d.fh_bytes), (double2 *)(ws + d.qh_bytes), nullptr, cp,
                                      item, wl, sink);
}

// LDS of the one-launch kernel: a narrow item's (the FP32 steps' weights, N = 24 2 KiB double-buffered,
// take less), then 256 bytes that the prefetches into L2 write and nothing reads
constexpr int kMultiSink = narrow_lds_bytes<float>(kMaxN), kMultiLdsBytes = kMultiSink + 256;

template <int N>
__device__ __forceinline__ void fp32_item(const MeshConvDesc &d, char *ws, int pass, const int4 item, lds_char *lds) {
    lds_char *const sink = lds + kMultiSink;
    if (item.x == d.tail_g)
        narrow_item<float, N, false, false>((const float2 *)(ws + d.fh_bytes), (double2 *)(ws + d.qh_bytes), d.ps.p[pass], item, d.tail_lw, lds,
                              sink);
    else
        multi_item<N>(d, ws, pass, item, lds, sink);
}

template <int R>
__device__ __forceinline__ void multi_core(const MeshConvDesc &d, char *ws, const int4 item, lds_char *wl) {
    const double2 *const cf = (const double2 *)(ws + d.cf_bytes);
    double2 *const out = (double2 *)(ws + d.cq_bytes);
    if (item.x == d.tail_g && d.tail_lw <= 3)
        narrow_core_item<R>(d.N, d.nD, cf, d.core_steps, d.core_w, out, d.cq_pstride, item, d.tail_lw);
    else
        core_item<R>(d.N, d.nD, cf, d.core_steps, d.core_ext, d.core_w, out, d.cq_pstride, item, wl);
}

#if BZ_CONV_UNIT == 0
// The work queues of the one launch (MultiQueues): a wavefront takes items from its XCD's queue, then
// from the others in turn.
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_conv_cells_f32_multi(const int4 *__restrict__ items, const MultiQueues mq, unsigned *__restrict__ counter,
                       const MeshConvDesc *__restrict__ desc, char *__restrict__ ws,
                       const unsigned char *__restrict__ skip) {
    __shared__ __attribute__((aligned(16))) double wbuf[kMultiLdsBytes / 8];
    lds_char *const wl = lds_ptr(&wbuf[0]);
    constexpr int kXccId = 20 | (3 << 11);   // hardware register 20, XCC_ID, bits 0..3
    int q = mq.n > 1 ? (int)(__builtin_amdgcn_s_getreg(kXccId) % kMultiQueues) : 0, tried = 0;
    for (;;) {
        const int it = mq.start[q] + pop_item(counter + q * kQueueStride);
        if (it >= mq.start[q + 1]) {
            if (++tried >= mq.n) break;
            q = q + 1 < mq.n ? q + 1 : 0;
            continue;
        }
        const int4 item = items[it];
        // a group whose cells are all served elsewhere: nothing reads its outputs
        if (skip && skip[item.x]) continue;
        const int mi = (item.y >> 24) & 0xf, pass = (item.y >> 20) & 0xf;
        const MeshConvDesc &d = desc[mi];
        if (item.y & kCoreItemBit) {
            const int4 ci = make_int4(item.x, item.y & 0xffffff, item.z, item.w);
            switch (d.core_r) {
            case 1: multi_core<1>(d, ws, ci, wl + kMultiSink); break;
            case 2: multi_core<2>(d, ws, ci, wl + kMultiSink); break;
            case 3: multi_core<3>(d, ws, ci, wl + kMultiSink); break;
            case 4: multi_core<4>(d, ws, ci, wl + kMultiSink); break;
            case 5: multi_core<5>(d, ws, ci, wl + kMultiSink); break;
            case 6: multi_core<6>(d, ws, ci, wl + kMultiSink); break;
            case 7: multi_core<7>(d, ws, ci, wl + kMultiSink); break;
            default: multi_core<8>(d, ws, ci, wl + kMultiSink); break;
            }
            continue;
        }
        switch (d.N) {
        case 8: fp32_item<8>(d, ws, pass, item, wl); break;
        case 12: fp32_item<12>(d, ws, pass, item, wl); break;
        case 16: fp32_item<16>(d, ws, pass, item, wl); break;
        case 20: fp32_item<20>(d, ws, pass, item, wl); break;
        case 24: fp32_item<24>(d, ws, pass, item, wl); break;
        case 28: fp32_item<28>(d, ws, pass, item, wl); break;
        default: fp32_item<32>(d, ws, pass, item, wl); break;
        }
    }
}
#endif

// ---------------------------------------------------------------------------
// Batched FP64.
// ---------------------------------------------------------------------------
// The weights arrive by scalar loads from N = 24 on (190 N = 32 cells 10.0 -> 8.0 ms a launch, 200 N = 24
// cells 2.76 -> 2.41 ms an evaluation): with one wavefront per SIMD the broadcast LDS reads take 32 cycles per
// pair and CU, the FP64 operations of the four SIMDs 24.  Below, the steps are short and the
// wait for a chunk of 16 weights costs more (N = 20, one wavefront per SIMD too, 1.06 against 1.12 ms, N = 16 330 against 352 us).
// Forms of the kernel at N = 16, by the groups of the batch.  The wide body alone takes 250 of the 256 vector
// registers that leave two wavefronts on a SIMD, with the narrow body beside it 290 (256 cells 321 against 365 us): a batch
// of whole groups has a kernel without the narrow body.  With whole groups and a narrow one the two are
// held to 256, at twelve spills outside the products (80 cells 168 -> 146 us, 270 395 -> 357); a narrow group alone
// keeps its registers (32 cells 114 us, 129 at 256).  The other meshes have the mixed form alone: below, both
// bodies fit (N = 12: 243; N = 8 times the same at 132 and 170), above, the wide body has one wavefront per SIMD anyway.
enum { kMixedGroups = 0, kWholeGroups = 1, kNarrowGroup = 2 };
__host__ __device__ constexpr int f64_form(int N, int form) { return N == 16 ? form : kMixedGroups; }
template <int N, int FORM>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(
    N == 16 && FORM != kNarrowGroup ? 2 : 1, N == 16 && FORM == kNarrowGroup ? 1 : 8)))
k_conv_cells_f64(const double2 *__restrict__ fh, const int4 *__restrict__ items, int n_items,
                 unsigned *__restrict__ counter, double2 *__restrict__ qh, const unsigned char *__restrict__ skip,
                 const ConvPasses ps, const NarrowTail nt) {
    constexpr int h = N / 2, M = N * N * N, PS = 3 * N * N / 4;
    constexpr bool kScalar = N >= 24;
    constexpr int CH = (PS * 8 + 1023) / 1024, CW = weight_chunk<double, N>(), WL = (PS * 8 + 4095) / 4096;
    constexpr int kNarrowLds = FORM == kWholeGroups ? 0 : narrow_lds_bytes<double>(N);
    constexpr int kLds = 2 * CH * 1024 > kNarrowLds ? 2 * CH * 1024 : kNarrowLds;
    __shared__ __attribute__((aligned(16))) double wbuf[(kLds + 256) / 8];
    lds_char *const wl = lds_ptr(&wbuf[0]), *const sink = wl + kLds;   // sink: written by the prefetches into L2
    const int lane = threadIdx.x;
    for (;;) {
        const int it = pop_item(counter);
        if (it >= n_items) break;
        const int4 item = items[it];
        const int g = item.x, r = item.y & 0xffff, part = (item.y >> 16) & 0xf, s0 = item.z, s1 = item.w;
        const ConvPass cp = pick_pass(ps, (item.y >> 20) & 0xf);
        const int k1 = r / N, k2 = r - k1 * N;
        double2 *const out = qh + cp.out_off + part * cp.pstride + g * cp.gstride + (size_t)(r - cp.row0) * N * kWave + lane;
        if (skip && skip[g]) {
            // every cell of the group is served elsewhere: leave zeros in this item's outputs
#pragma unroll
            for (int t = 0; t < N; ++t) out[t * kWave] = make_double2(0.0, 0.0);
            continue;
        }
        if (FORM == kNarrowGroup || (FORM == kMixedGroups && g == nt.g)) {
            narrow_item<double, N, (N >= 16 && FORM == kMixedGroups), (N >= 20 && N < 32)>(fh, qh, cp, item, nt.lw, wl, sink);
            continue;
        }
        StepWalk<N> at(k1, k2, s0, kScalar && __builtin_amdgcn_readfirstlane(cp.zero_planes) && k2 < h);
        const double *w = (const double *)cp.w + cp.row_woff[r] + (long long)(at.s < s1 ? at.s : s0) * PS;
        const double2 *F = fh + cp.fh_off + (size_t)g * M * kWave + lane;
        double pr[N], pi[N];
#pragma unroll
        for (int t = 0; t < N; ++t) pr[t] = pi[t] = 0.0;
        WeightChunk<double, CW> wc;
        if constexpr (kScalar) {
            w = uniform_ptr(w);
            wc = load_chunk<double, CW>(w);
        } else {
            prefetch_weights<CH>(w, wl);
            __builtin_amdgcn_s_waitcnt(0);
        }
        int buf = 0;
        while (at.s < s1) {
            const int m1 = at.m1, m2 = at.m2, j1 = k1 + h - m1, j2 = k2 + h - m2;
            StepWalk<N> nx = at;
            nx.next();
            if constexpr (!kScalar) prefetch_weights<CH>(w + PS, wl + (buf ^ 1) * CH * 1024);
            double2 mv[N], jv[N];
            load_row<double, N>(F + (size_t)((m1 * N + m2) * N) * kWave, mv);
            load_row<double, N>(F + (size_t)((j1 * N + j2) * N) * kWave, jv);
            if constexpr (kScalar) {
                // the next step's weights pulled into L2 (64 bytes a lane, the LDS copy is discarded)
                const double *const wn = w + (nx.s < s1 ? nx.s - at.s : 1) * PS;
#pragma unroll
                for (int c = 0; c < WL; ++c)
                    __builtin_amdgcn_global_load_lds((const void *)((const char *)wn + lane * 64 + c * 4096),
                                                     (void __attribute__((address_space(3))) *)sink, 4, 0, 0);
                cells_step_scalar<double, N, 1, CW>(mv, jv, w, wn, wc, pr, pi);
                w = wn;
            } else if (!cp.zero_planes || (m2 != 0 && j2 != 0)) {
                cells_step<double, N, 1>(mv, jv, (const lds_double *)(wl + buf * CH * 1024), pr, pi);
            }
            if constexpr (!kScalar) w += PS;
            buf ^= 1;
            at = nx;
            if constexpr (!kScalar) __builtin_amdgcn_s_waitcnt(0);
        }
#pragma unroll
        for (int t = 0; t < N; ++t) out[t * kWave] = make_double2(pr[t], pi[t]);
    }
}

// ---------------------------------------------------------------------------
// Plain schedule, one cell.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int plain_rows_c(int N) {
    int R = kWave / N;
    while (R > 1 && N % R) --R;
    return R;
}

// A block's kPlainWaves wavefronts share the rows and split its (m1, m2) range, their sums added through LDS in
// order: with one wavefront per block two to three shared a SIMD, and the launch waited for its
// loads (one N = 24 cell in FP64 756 -> 309 us; its weights alone take 150 us at the rate of a large copy).
constexpr int kPlainWaves = 8;
template <typename T, int N>
__global__ void __launch_bounds__(64 * kPlainWaves) k_conv_plain(const typename cplx<T>::t *__restrict__ fh,
                                                   const T *__restrict__ W, const long long *__restrict__ blk_woff,
                                                   int nsplit, double2 *__restrict__ qh) {
    using C = typename cplx<T>::t;
    constexpr int h = N / 2, R = plain_rows_c(N), NB = N / R, LN = R * N, M = N * N * N;
    __shared__ double2 sum[kPlainWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.x, s = blockIdx.y;
    const int k1 = b / NB, kb = b - k1 * NB;
    const bool active = lane < LN;
    const int r = active ? lane / N : 0, k3 = active ? lane - (lane / N) * N : 0;
    const int k2 = kb * R + r;
    const int lo1 = axis_lo(N, k1), c1 = axis_cnt(N, k1);
    const int u2lo = plain_u2_lo(N, kb), U2 = plain_u2_hi(N, kb) - u2lo + 1;
    // this wavefront's range of the steps (m1 - lo1) U2 + (m2 - u2lo)
    const int steps = c1 * U2, part = s * kPlainWaves + wave, parts = nsplit * kPlainWaves;
    const int ta = (int)((long long)steps * part / parts), tb = (int)((long long)steps * (part + 1) / parts);
    const T *w = W + blk_woff[b] + (long long)ta * N * LN + (active ? lane : 0);
    int m1 = lo1 + ta / U2, m2 = u2lo + ta % U2;
    double ar = 0.0, ai = 0.0;
    for (int t = ta; t < tb; ++t) {
        const int j1 = k1 + h - m1;
        int j2 = k2 + h - m2;
        j2 = j2 < 0 ? 0 : (j2 > N - 1 ? N - 1 : j2);
        const C *rowm = fh + (m1 * N + m2) * N;
        const C *rowj = fh + (j1 * N + j2) * N;
        T pr = 0, pi = 0;
#pragma unroll
        for (int m3 = 0; m3 < N; ++m3) {
            int j3 = k3 + h - m3;
            j3 = j3 < 0 ? 0 : (j3 > N - 1 ? N - 1 : j3);
            const C a = rowm[m3];
            const C bb = rowj[j3];
            const T wt = w[m3 * LN];
            const T px = fma(a.x, bb.x, -(a.y * bb.y));
            const T py = fma(a.x, bb.y, a.y * bb.x);
            pr = fma(wt, px, pr);
            pi = fma(wt, py, pi);
        }
        w += N * LN;
        ar += (double)pr;
        ai += (double)pi;
        if (++m2 == u2lo + U2) {
            m2 = u2lo;
            ++m1;
        }
    }
    sum[wave][lane] = make_double2(ar, ai);
    __syncthreads();
    if (wave == 0 && active) {
        for (int v = 1; v < kPlainWaves; ++v) {
            ar += sum[v][lane].x;
            ai += sum[v][lane].y;
        }
        qh[(size_t)s * M + ((size_t)k1 * N + k2) * N + k3] = make_double2(ar, ai);
    }
}

// Tuning variants of the batched FP32 kernel: (fold interval, compensation, weight path, row path).
//   0: FOLD 2, FP64 total,   LDS double-buffered weights, rows prefetched to LDS   (default)
//   1: FOLD 2, TwoSum total, LDS double-buffered weights, rows prefetched to LDS
//   2: FOLD 2, FP64 total,   LDS double-buffered weights, rows loaded per step
//   3: FOLD 2, TwoSum total, LDS double-buffered weights, rows loaded per step
//   4: FOLD 2, FP64 total,   scalar weights + L2 prefetch, rows prefetched to LDS
//   5: FOLD 4, FP64 total,   LDS double-buffered weights, rows prefetched to LDS
//   6: FOLD 2, FP64 total kept in the output slot (read-modify-write per fold), LDS
//      double-buffered weights, rows loaded per step; fits two wavefronts per SIMD
//   7: as 6 with FOLD 4
//   8: as 6 with FOLD 8
//   9: as 6 with FOLD 16
//  10: as 9 with four interleaved partials per output and step (pairwise combined)
//  11: as 10 with FOLD 8
//  12: as 10 with two interleaved partials
//  13: as 5 with four interleaved partials
//  14: as 10 with FOLD 4
//  15: as 10 with FOLD 2
// Accumulation parameters of each variant (must match the switch below): the
// autotuner prefers more interleaved partials, then a shorter fold interval.
struct VariantAcc {
    int fold, split;
};
constexpr VariantAcc kVariantAcc[] = {{2, 1}, {2, 1}, {2, 1}, {2, 1}, {2, 1},  {4, 1},  {2, 1},
                                      {4, 1}, {8, 1}, {16, 1}, {16, 4}, {8, 4}, {16, 2}, {4, 4},
                                      {4, 4}, {2, 4}};

template <int N>
hipError_t cells_f32_variant(const CellsLaunch &p, unsigned grid, hipStream_t s) {
#define BZ_CELLS_F32(F, C, WPV, RPV, SP)                                                                    \
    hipLaunchKernelGGL((k_conv_cells_f32<N, F, C, WPV, RPV, SP>), dim3(grid), dim3(64), 0, s,               \
                       (const float2 *)p.fh, p.items, p.n_items, p.counter, p.qh, p.skip, p.passes)
    switch (p.variant) {
    case 1: BZ_CELLS_F32(2, 1, 0, 1, 1); break;
    case 2: BZ_CELLS_F32(2, 0, 0, 0, 1); break;
    case 3: BZ_CELLS_F32(2, 1, 0, 0, 1); break;
    case 4: BZ_CELLS_F32(2, 0, 1, 1, 1); break;
    case 5: BZ_CELLS_F32(4, 0, 0, 1, 1); break;
    case 6: BZ_CELLS_F32(2, 2, 0, 0, 1); break;
    case 7: BZ_CELLS_F32(4, 2, 0, 0, 1); break;
    case 8: BZ_CELLS_F32(8, 2, 0, 0, 1); break;
    case 9: BZ_CELLS_F32(16, 2, 0, 0, 1); break;
    case 10: BZ_CELLS_F32(16, 2, 0, 0, 4); break;
    case 11: BZ_CELLS_F32(8, 2, 0, 0, 4); break;
    case 12: BZ_CELLS_F32(16, 2, 0, 0, 2); break;
    case 13: BZ_CELLS_F32(4, 0, 0, 1, 4); break;
    case 14: BZ_CELLS_F32(4, 2, 0, 0, 4); break;
    case 15: BZ_CELLS_F32(2, 2, 0, 0, 4); break;
    default: BZ_CELLS_F32(2, 0, 0, 1, 1); break;
    }
#undef BZ_CELLS_F32
    return hipGetLastError();
}

template <int N>
hipError_t cells_f64_launch(const CellsLaunch &p, unsigned grid, hipStream_t s) {
    auto launch = [&](auto form) {
        hipLaunchKernelGGL((k_conv_cells_f64<N, f64_form(N, form)>), dim3(grid), dim3(64), 0, s, (const double2 *)p.fh,
                           p.items, p.n_items, p.counter, p.qh, p.skip, p.passes, p.tail);
    };
    // a narrow group is the last one: as group 0 it is the only one
    if (p.tail.g < 0) launch(std::integral_constant<int, kWholeGroups>{});
    else if (p.tail.g == 0) launch(std::integral_constant<int, kNarrowGroup>{});
    else launch(std::integral_constant<int, kMixedGroups>{});
    return hipGetLastError();
}

template <typename T, int N>
hipError_t plain_launch(const PlainLaunch &p, hipStream_t s) {
    const int nb = N * (N / plain_rows_c(N));
    hipLaunchKernelGGL((k_conv_plain<T, N>), dim3(nb, p.nsplit), dim3(64 * kPlainWaves), 0, s,
                       (const typename cplx<T>::t *)p.fh, (const T *)p.w, p.blk_woff, p.nsplit, p.qh);
    return hipGetLastError();
}

}  // namespace

#if BZ_CONV_UNIT == 0
int conv_variant_count() { return (int)(sizeof(kVariantAcc) / sizeof(kVariantAcc[0])); }

// The compensation form does not enter the rank: the FP64 total (in registers or in the
// output slot) and the TwoSum (hi, lo) pair both carry the folded total to at least 48
// bits, far below the FP32 rounding of the running sum between folds, which the fold
// interval and the interleaved partials set.
int conv_variant_accuracy_rank(int v) {
    if (v < 0 || v >= conv_variant_count()) return -1;
    return kVariantAcc[v].split * 1000 - kVariantAcc[v].fold;
}

// Persistent grid: enough single-wave workgroups to keep every SIMD busy.
static unsigned persistent_grid(int n_items) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    unsigned g = (unsigned)cus * 8u;
    return (unsigned)n_items < g ? (unsigned)n_items : g;
}

template <int R>
hipError_t core_launch(const CoreLaunch &p, unsigned grid, hipStream_t s) {
    hipLaunchKernelGGL(k_conv_core<R>, dim3(grid), dim3(64), 0, s, p.N, p.nD, p.cf, p.items, p.n_items, p.counter,
                       p.steps, p.ext, p.w, p.out, p.pstride, p.skip);
    return hipGetLastError();
}

hipError_t launch_conv_cells_multi(const MultiLaunch &p, hipStream_t s) {
    if (p.n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_conv_cells_f32_multi, dim3(persistent_grid(p.n_items)), dim3(64), 0, s, p.items, p.queues,
                       p.counter, p.desc, p.ws, p.skip);
    return hipGetLastError();
}

hipError_t launch_conv_core(const CoreLaunch &p, hipStream_t s) {
    if (p.n_items <= 0) return hipSuccess;
    if (p.r < 1 || p.r > kCoreMaxR) return hipErrorInvalidValue;
    hipError_t e = launch_fill_u32(p.counter, 1, 0u, s);
    if (e != hipSuccess) return e;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    const int want = p.waves > 0 ? p.waves : 8 * cus;
    const unsigned grid = (unsigned)(p.n_items < want ? p.n_items : want);
    switch (p.r) {
    case 1: return core_launch<1>(p, grid, s);
    case 2: return core_launch<2>(p, grid, s);
    case 3: return core_launch<3>(p, grid, s);
    case 4: return core_launch<4>(p, grid, s);
    case 5: return core_launch<5>(p, grid, s);
    case 6: return core_launch<6>(p, grid, s);
    case 7: return core_launch<7>(p, grid, s);
    default: return core_launch<8>(p, grid, s);
    }
}

hipError_t launch_conv_cells(const CellsLaunch &p, bool f64, hipStream_t s) {
    if (p.n_items <= 0) return hipSuccess;
    hipError_t e = launch_fill_u32(p.counter, 1, 0u, s);
    if (e != hipSuccess) return e;
    const unsigned grid = persistent_grid(p.n_items);
    if (f64) return launch_cells_f64(p, grid, s);
    return p.N <= 20 ? launch_cells_f32_small(p, grid, s) : launch_cells_f32_large(p, grid, s);
}
#endif

#if BZ_CONV_UNIT == 1
hipError_t launch_cells_f32_small(const CellsLaunch &p, unsigned grid, hipStream_t s) {
    switch (p.N) {
    case 8: return cells_f32_variant<8>(p, grid, s);
    case 12: return cells_f32_variant<12>(p, grid, s);
    case 16: return cells_f32_variant<16>(p, grid, s);
    case 20: return cells_f32_variant<20>(p, grid, s);
    default: return hipErrorInvalidValue;
    }
}
#endif

#if BZ_CONV_UNIT == 2
hipError_t launch_cells_f32_large(const CellsLaunch &p, unsigned grid, hipStream_t s) {
    switch (p.N) {
    case 24: return cells_f32_variant<24>(p, grid, s);
    case 28: return cells_f32_variant<28>(p, grid, s);
    case 32: return cells_f32_variant<32>(p, grid, s);
    default: return hipErrorInvalidValue;
    }
}
#endif

#if BZ_CONV_UNIT == 3
#define BZ_FOR_EACH_N(X) X(8) X(12) X(16) X(20) X(24) X(28) X(32)

hipError_t launch_cells_f64(const CellsLaunch &p, unsigned grid, hipStream_t s) {
#define CASE(NN) \
    case NN: return cells_f64_launch<NN>(p, grid, s);
    switch (p.N) {
        BZ_FOR_EACH_N(CASE)
    default:
        return hipErrorInvalidValue;
    }
#undef CASE
}

hipError_t launch_conv_plain(const PlainLaunch &p, bool f64, hipStream_t s) {
#define CASE(NN) \
    case NN:     \
        return f64 ? plain_launch<double, NN>(p, s) : plain_launch<float, NN>(p, s);
    switch (p.N) {
        BZ_FOR_EACH_N(CASE)
    default:
        return hipErrorInvalidValue;
    }
#undef CASE
}
#endif

}  // namespace bz
