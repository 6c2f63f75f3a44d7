// What goes before and after the step kernel's launches: the cut of padded batches, the last step's potentials, the solve of a
// problem whose chain has given up.
#pragma once
#include "ska_step.h"

namespace {

// The cut of a call with lengths: the shortest segments of which there are at most CUT_SEGS in all and CUT_HALF in either half of
// the problems (M blocks, the segments of a call without lengths, always do).  One workgroup; thread i tries the i-th length.
__global__ __launch_bounds__(NTHREADS) void step_cut_kernel(const CutArgs a)
{
    __shared__ int nb[CUT_ITEMS], total, best;
    const int tid = threadIdx.x, n0 = a.items * a.nh / 2;
    if (tid == 0) { total = 0; best = a.M; }
    __syncthreads();
    if (tid < a.items) {
        int Lq = a.L, Lk = a.L;
        if (a.len_q) Lq = min(max(a.len_q[tid], 0), a.L);
        if (a.len_k) Lk = min(max(a.len_k[tid], 0), a.L);
        nb[tid] = ((Lk > 0 ? min(Lq, Lk + a.W) : 0) + 32 * a.NF - 1) / (32 * a.NF);
        atomicAdd(&total, nb[tid] * a.nh);
    }
    __syncthreads();
    auto segments = [&](int b, int M) { return max((nb[b] + M - 1) / M, 1); };
    const int M = max((total + CUT_SEGS - 1) / CUT_SEGS, a.least) + tid;
    if (M < a.M) {
        int lo = 0, hi = 0;
        for (int b = 0; b < a.items; ++b) {
            const int s = segments(b, M), in_lo = min(max(n0 - b * a.nh, 0), a.nh);
            lo += s * in_lo;
            hi += s * (a.nh - in_lo);
        }
        // (a split call's halves share the CUs of each XCD; uneven ones that fill all 32 of them get in each other's way: 104 + 148
        // segments 1653 us, 112 + 144 longer ones 1424)
        const int xlo = (lo + 7) / 8, xhi = (hi + 7) / 8;
        const bool halves = lo <= CUT_HALF && hi <= CUT_HALF && (xlo == xhi || xlo + xhi < CUT_SEGS / 8);
        if (lo + hi <= CUT_SEGS && (n0 == 0 || halves)) atomicMin(&best, M);
    }
    __syncthreads();
    if (tid == 0) {
        const int SL = a.NF * best;
        a.cut[0] = SL; a.cut[1] = best;
        a.cut[2] = SL == 1 ? 0 : (int)(0xffffffffu / (unsigned)SL + 1u);
        int at = 0;
        for (int b = 0; b < a.items; ++b) {
            const int s = segments(b, best);
            a.cut[CUT_HEAD + b] = at;
            if (n0 >= b * a.nh && n0 < (b + 1) * a.nh) a.cut[3] = at + s * (n0 - b * a.nh);
            at += s * a.nh;
        }
        a.cut[CUT_HEAD + a.items] = a.cut[4] = at;
    }
}

// v from the column sums of a step that no step follows (v_out may be p.v), by workgroups of NTHR threads.  (The dustbin's shares are
// added up as by NTHREADS, so that its bits do not depend on who does it; more threads' sums are not used.)
template <int NTHR> __device__ __forceinline__ void final_columns(const StepArgs &p)
{
    __shared__ float red[32];
    const int nblk = (p.L + NTHR - 1) / NTHR, n = blockIdx.x / nblk, blk = blockIdx.x % nblk, t = blk * NTHR + threadIdx.x;
    const float *part = p.part_in + n * p.part_stride, *spr = p.spoke_r ? p.spoke_r + (long)n * p.sstride : nullptr;
    float *v_out = p.v_out + n * p.us;
    float uL = 0.f;
    if (p.dustbin) {
        const DustbinPair d = dustbin_pair<NTHREADS>(p, part, spr ? spr[p.L] : p.sdb, red);
        uL = d.u;
        if (blk == 0 && threadIdx.x == 0) {
            p.u_fin[n * p.us + p.L] = d.u;
            v_out[p.L] = d.v;
        }
    }
    if (t >= p.L) return;
    const StepLens ln = step_lens(p, n);
    float out = 0.f;
    if (t < ln.Lc) {
        const float v = p.v[n * p.us + t];
        const StepCut cut = step_cut(p);
        float sum = column_sum(p, cut, part, t, (ln.Le + 32 * cut.SL - 1) / (32 * cut.SL));
        if (p.dustbin) sum += fast_exp2(((p.spoke_c ? p.spoke_c[(long)n * p.sstride + t] : p.sdb) + uL + v) * LOG2E);
        out = column_update<true>(v, sum, ColumnTarget(p.log_b ? p.log_b[(long)n * p.lstride + t] : 0.f));
    }
    v_out[t] = out;
}
__global__ __launch_bounds__(NTHREADS) void vfinal_kernel(const StepArgs p) { final_columns<NTHREADS>(p); }

// One half-step of a problem by one workgroup: a wavefront takes 32 rows at a time and its band's tiles one after the other, a lane is
// a column, its registers are rows, each with a maximum and a sum of its own.  Nothing is assumed of the potentials.
// own, oth: valid rows and partners; mark: -inf where a token is inactive; olog: log targets; dustbin: edges to and from index L,
// scores of the owners' spokes and of the others' (null: sdb).  A sum without an entry: marks its token while it is not `settled` who
// is active (as the launched half-steps do with their running maximum), and is an error after that, as in the launched steps.
constexpr int SOLVE_THREADS = 512;
struct PlainSide { const float *mark, *olog, *spoke; int valid; };
template <typename T, int D>
__device__ __forceinline__ void plain_half_step(const StepArgs &p, const T *X, const T *Y, const PlainSide own, const PlainSide oth, bool settled, const float *y, float *x)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 31, h = lane >> 5, L = p.L, W = p.W;
    constexpr float NONE = -3e38f;   // (a number: a NaN stays in the sum, whatever comes before and after it)
    auto add = [](float &m, float &sum, float e, float times) {
        const float mn = fmaxf(m, e);
        sum = sum * fast_exp2(m - mn) + times * fast_exp2(e - mn);
        m = mn;
    };
    auto finish = [&](int o, float m, float sum) {
        if (m > NONE) x[o] = (own.olog ? own.olog[o] : 0.f) - LN2 * (m + fast_log2(sum));
        else x[o] = settled ? __builtin_nanf("") : -INFINITY;
    };
    for (int o0 = 32 * wave; o0 < own.valid; o0 += SOLVE_THREADS / 2) {
        float m[16], sum[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) { m[r] = NONE; sum[r] = 0.f; }
        const int first = max(o0 - W, 0) >> 5, last = min(o0 + 31 + W, oth.valid - 1) >> 5;
        constexpr bool AHEAD = D * sizeof(T) <= 256;   // (registers)
        OwnerFrag<T, D> xf, yf, next;
        xf.load(X, o0 + c, own.valid, h);
        if (AHEAD) next.load(Y, 32 * first + c, oth.valid, h);
        for (int k = first; k <= last; ++k) {
            if (AHEAD) yf = next;
            (AHEAD ? next : yf).load(Y, 32 * (k + AHEAD) + c, oth.valid, h);
            f32x16 e;
#pragma unroll
            for (int r = 0; r < 16; ++r) e[r] = 0.f;
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int ks = 0; ks < D / 16; ++ks) e = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf.v[ks], yf.v[ks], e, 0, 0, 0);
            } else {
#pragma unroll
                for (int ks = 0; ks < D / 2; ++ks) e = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.v[ks], yf.v[ks], e, 0, 0, 0);
            }
            const int t = 32 * k + c;
            const float yt = t < oth.valid ? y[t] * LOG2E : -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int o = o0 + 8 * (r >> 2) + (r & 3) + 4 * h;
                add(m[r], sum[r], t < oth.valid && abs(t - o) <= W ? fmaf(e[r], p.c2, yt) : -INFINITY, 1.f);
            }
        }
        float mr = NONE, sr = 0.f;   // lane c < 16: of its register c
#pragma unroll
        for (int r = 0; r < 16; ++r) {
#pragma unroll
            for (int s = 16; s >= 1; s >>= 1) {
                const float mo = __shfl_xor(m[r], s), so = __shfl_xor(sum[r], s);
                add(m[r], sum[r], mo, so);
            }
            if (c == r) { mr = m[r]; sr = sum[r]; }
        }
        const int o = o0 + 8 * (c >> 2) + (c & 3) + 4 * h;
        if (c < 16 && o < own.valid) {
            if (p.dustbin) add(mr, sr, ((own.spoke ? own.spoke[o] : p.sdb) + y[L]) * LOG2E, 1.f);
            if (own.mark[o] == -INFINITY) x[o] = -INFINITY;
            else finish(o, mr, sr);
        }
    }
    if (p.dustbin && wave == SOLVE_THREADS / 64 - 1) {
        float m = NONE, sum = 0.f;
        for (int t = lane; t <= L; t += 64) add(m, sum, ((oth.spoke ? oth.spoke[t] : p.sdb) + y[t]) * LOG2E, 1.f);
        for (int s = 32; s >= 1; s >>= 1) {
            const float mo = __shfl_xor(m, s), so = __shfl_xor(sum, s);
            add(m, sum, mo, so);
        }
        if (lane == 0) finish(L, m, sum);
    }
    for (int o = own.valid + threadIdx.x; o < L; o += SOLVE_THREADS) x[o] = 0.f;
    __syncthreads();
}
// After a chain: the last step's v.  If the chain has given up, one workgroup per problem does all its steps from the start (it asks
// nothing of the device).  That takes as long as one CU needs for a problem's tiles (2 (T + R) times), beside
// a spin limit of about 100 ms.  Whole forward in ms, T + R = 18, bf16, d = 64, rows dot by dot (a wavefront a row) -> so: 8 problems of
// L = 701, W = 64 24 -> 1.6; 16 of 3001, W = 100 130 -> 8; one of 16384, W = 64 580 -> 28; fp32, 8 of 4096, W = 128 350 -> 20.  The
// longest problems that chains take: one of 65536, W = 64 115; of 16000, W = 480, T + R = 22 134; fp32, of 14000, W = 128 69.
struct SolveArgs { int T, R, cold; };   // cold: half-steps until it is settled who is active
template <typename T, int D> __global__ __launch_bounds__(SOLVE_THREADS) void vfinish_kernel(const StepArgs p, const SolveArgs a)
{
    if (p.chain->failed != CHAIN_GAVE_UP) {   // (written by the launch before)
        final_columns<SOLVE_THREADS>(p);
        return;
    }
    const int nblk = (p.L + SOLVE_THREADS - 1) / SOLVE_THREADS, n = blockIdx.x / nblk;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        chain_given_up = p.seq;
        __hip_atomic_store(p.gate + 1, p.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (blockIdx.x % nblk) return;
    const T *X = reinterpret_cast<const T *>(p.X) + (long)n * p.L * D, *Y = reinterpret_cast<const T *>(p.Y) + (long)n * p.L * D;
    float *slots = p.slots + n * p.us;
    auto slot = [&](int k) { return slots + (long)k * p.Lp; };
    const StepLens ln = step_lens(p, n);
    const PlainSide rows{slot(0), p.log_a ? p.log_a + (long)n * p.lstride : nullptr, p.spoke_r ? p.spoke_r + (long)n * p.sstride : nullptr, ln.Le};
    const PlainSide cols{slot(1), p.log_b ? p.log_b + (long)n * p.lstride : nullptr, p.spoke_c ? p.spoke_c + (long)n * p.sstride : nullptr, ln.Lc};
    for (int i = threadIdx.x; i < p.Lp; i += SOLVE_THREADS)   // v = 0; inactive tokens keep their mark
        for (int k = 0; k < 2; ++k) slot(k)[i] = slot(k)[i] == -INFINITY ? -INFINITY : 0.f;
    __syncthreads();
    for (int st = 0; st < a.T + a.R; ++st) {
        const int to = st < a.T ? 0 : 2 * (st - a.T + 1), from = st < a.T ? 1 : to - 1;
        plain_half_step<T, D>(p, X, Y, rows, PlainSide{nullptr, nullptr, cols.spoke, ln.Lt}, 2 * st >= a.cold, slot(from), slot(to));
        plain_half_step<T, D>(p, Y, X, cols, PlainSide{nullptr, nullptr, rows.spoke, ln.Le}, 2 * st + 1 >= a.cold, slot(to), slot(to + 1));
    }
}

}  // namespace
