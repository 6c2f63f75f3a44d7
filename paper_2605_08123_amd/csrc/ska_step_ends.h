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

// v from the column sums of a step that no step follows (v_out may be p.v).
__device__ __forceinline__ void final_columns(const StepArgs &p)
{
    __shared__ float red[32];
    const int nblk = (p.L + NTHREADS - 1) / NTHREADS, n = blockIdx.x / nblk, blk = blockIdx.x % nblk, t = blk * NTHREADS + threadIdx.x;
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
__global__ __launch_bounds__(NTHREADS) void vfinal_kernel(const StepArgs p) { final_columns(p); }

// One half-step of problem n by one workgroup, a wavefront per row and a lane per partner; nothing is assumed of the potentials.
template <typename T, int D>
__device__ __forceinline__ void plain_half_step(const T *X, const T *Y, const float *y, float *x, int L, int W, int own, int oth, float c2)
{
    const int lane = threadIdx.x & 63;
    for (int o = threadIdx.x >> 6; o < L; o += NWAVES) {
        float m = -INFINITY, sum = 0.f;
        for (int t = max(o - W, 0) + lane; t <= min(o + W, oth - 1) && o < own; t += 64) {
            float dot = 0.f;
            for (int k = 0; k < D; k += 4) {
                float a[4], b[4];
                load4<T>(X + (long)o * D + k, a);
                load4<T>(Y + (long)t * D + k, b);
#pragma unroll
                for (int i = 0; i < 4; ++i) dot = fmaf(a[i], b[i], dot);
            }
            const float e = fmaf(dot, c2, y[t] * LOG2E), mn = fmaxf(m, e);
            sum = sum * fast_exp2(m - mn) + fast_exp2(e - mn);
            m = mn;
        }
        for (int s = 32; s >= 1; s >>= 1) {
            const float mo = __shfl_xor(m, s), so = __shfl_xor(sum, s), mn = fmaxf(m, mo);
            sum = mn > -INFINITY ? sum * fast_exp2(m - mn) + so * fast_exp2(mo - mn) : 0.f;
            m = mn;
        }
        if (lane == 0) x[o] = o < own ? -LN2 * (m + fast_log2(sum)) : 0.f;
    }
    __syncthreads();
}
// After a chain: the last step's v.  If the chain has given up, one workgroup per problem does all its steps from the start
// (milliseconds; it asks nothing of the device).
struct SolveArgs { int T, R; };
template <typename T, int D> __global__ __launch_bounds__(NTHREADS) void vfinish_kernel(const StepArgs p, const SolveArgs a)
{
    if (!p.chain->failed) {   // (written by the launch before)
        final_columns(p);
        return;
    }
    const int nblk = (p.L + NTHREADS - 1) / NTHREADS, n = blockIdx.x / nblk;
    if (blockIdx.x % nblk) return;
    const T *X = reinterpret_cast<const T *>(p.X) + (long)n * p.L * D, *Y = reinterpret_cast<const T *>(p.Y) + (long)n * p.L * D;
    float *slots = p.slots + n * p.us;
    auto slot = [&](int k) { return slots + (long)k * p.Lp; };
    const StepLens ln = step_lens(p, n);
    for (int i = threadIdx.x; i < p.L; i += NTHREADS) slot(0)[i] = slot(1)[i] = 0.f;
    __syncthreads();
    for (int st = 0; st < a.T + a.R; ++st) {
        const int to = st < a.T ? 0 : 2 * (st - a.T + 1), from = st < a.T ? 1 : to - 1;
        plain_half_step<T, D>(X, Y, slot(from), slot(to), p.L, p.W, ln.Le, ln.Lt, p.c2);
        plain_half_step<T, D>(Y, X, slot(to), slot(to + 1), p.L, p.W, ln.Lc, ln.Le, p.c2);
    }
}

}  // namespace
