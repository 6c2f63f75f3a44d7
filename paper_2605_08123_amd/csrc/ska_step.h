// A whole Sinkhorn step (row half-step and column half-step) from one evaluation of the scores.
#pragma once
#include "ska_common.h"
#include "ska_step_shape.h"

namespace {

// ------------------------------------------------------------------ one Sinkhorn step per launch
// From potentials (u, v) the row half-step needs r_i = sum_j E_ij with E_ij = exp(S_ij + u_i + v_j), u'_i = u_i - log r_i,
// and the column half-step the column sums of the same matrix with its rows rescaled, c_j = sum_i E_ij / r_i,
// v'_j = v_j - log c_j.  So E is evaluated once per step if it can be kept between the two sums: a wavefront
// keeps the 32 rows x 32 NTW columns it evaluates in registers (16 of them per 32 x 32 tile), where two half-steps
// evaluate every score and exponential twice.  The owner rows are the MFMA's A operand here: a lane is one
// column and its registers are rows, so both sums are in-lane (row sums: 16 accumulators, exchanged between the
// lanes once per wavefront; column sums: 16 multiply-adds per tile).
//   A workgroup of NF G wavefronts owns blocks of NF fragments (32 rows each); G wavefronts share a fragment, each with NTW
// of the 2 ceil(W / 32) + 1 tiles that its band meets.  The other side's rows that a block meets lie in LDS as
// a whole (written by LDS-direct loads, 16-byte chunks swizzled on the way), so the evaluation runs without a barrier.
// With MARCH a workgroup walks M blocks (a segment) on a ring of tiles: a block adds NF tiles, requested one block ahead.
//   Column sums are summed over the fragments of a block in LDS and over the blocks of a segment in registers (a thread keeps
// its places of the ring), and written per segment; a column has those of at most ceil(2 ceil(W / 32) / (NF M)) + 1
// segments, which the next launch adds up in a fixed order where it needs v' (vfinal_kernel where no step follows).
//   Every row and every column carries its own potential as stabiliser: after one step the row sums of a
// column-normalised plan lie between 1 / (2 W + 1) and 2 W + 1 (unit targets), and likewise the column sums.
//   What bounds it: the instructions of a SIMD's two wavefronts.  A step of two problems of L = 262144, W = 256 (256 segments of 16
// blocks, one per CU) takes 82 us; by counters the plain ALUs are busy for 72 % of its SIMD cycles, the matrix cores for 28 %, either for
// 85 %, with about 90 instructions a tile where its exponentials and two sums are 48.  When it took 88 us, leaving one thing out saved:
// the exponentials 20, the products of the scores 13, the request of the next block's tiles 7, the segment's column sums 7, the adds of
// the row sums 6, the masks 6, the exchange of row sums 4, the column sums 4, the LDS reads of the operands 2.  So what is not a product,
// an exponential or one of the two sums is kept short: LDS addresses advance by the instructions' offsets, the tiles that are not there are
// not evaluated and lie on all SIMDs evenly, fragments' column sums lie by column with zeros around, the reduction of row sums halves
// its registers on the way, and the column sums of a block are added up among the products of the next one: 91.4 -> 83.2 us, the
// one-call step of the same problems 2583 -> 2424, of four of 65536 1408 -> 1308.  Taking the column sums themselves from
// the registers while the next block is evaluated into them, with one barrier a block instead of two: 91.8 -> 95.7.
// Two independent workgroups of half the size per CU: W = 128 (4,1,9) 960 us instead of 990 at
// 524288 rows, but 588 instead of 577 at 262144; at W = 256 two windows fit LDS only if the fragments' column sums
// share their place by LDS atomics, which cost more than that (900 -> 1120).  Small calls are bound by latency from start to
// end: a launch of short blocks is 5 us, 2.3 of them until the first product.
//   Forward of T = 16, R = 2 steps, bf16, d = 64, us, by half-steps -> by a launch per step (short calls take less as chains, see
// below): 8 problems of L = 700, W = 64 210 -> 117; 4 of
// 3000, W = 128 266 -> 155; 32 of 4096, W = 128 460 -> 327; 4 of 65536, W = 64 702 -> 416, W = 256 1085 -> 900; 2 of 262144,
// W = 256 1900 -> 1676.  fp32: 8 of 4096, W = 128 607 -> 370 (matrix instructions: half as many).
//   The potentials enter through the products (potential_parts): as 16 adds per tile they took 6 % of a long call, and as
// the products' initial accumulator 16 registers.  The products of a tile are issued among the exponentials of the tile
// before it, in an order that scheduling barriers pin: left to itself the compiler puts all products first.
//   DUST: every segment also writes what the dustbin's row and its column get from it, and the next launch makes the dustbin's
// two potentials of them (dustbin_pair), each workgroup for itself.  A launch between the steps (the column sums and
// the dustbin's elements, one long workgroup each) took a fifth of the step: forward and backward of 8 problems of L = 16384,
// W = 256, T = 20 1022 -> 863 us, 8 of 5000, W = 128 with learned tokens 396 -> 357.  In segments a template parameter (DB),
// since its branches and registers cost calls without a dustbin 4 % (2 problems of 262144: 2730 -> 2650 us); single blocks
// have registers to spare and read a flag.
//   TARGETS: small marginal targets stay out of the exponents (ColumnTarget) and come in as weights of the two sums: one more
// factor where rows are summed (a multiply-add instead of an add).  With a row's and a column's target in them, the entries
// of a row of e^-80 next to ordinary ones lost all but the largest, and at e^-90 the row was empty; a mask of -100 or -1e4 on
// every sixteenth row gave NaN everywhere.  The block's largest potential, as the half-steps take it, would carry those, but
// not potentials that lie apart by their scores.  A template parameter as well: forward and backward of four problems of
// L = 65536, W = 256 1388 -> 1445 us, a forward of eight of 701, W = 64 113 -> 115; by half-steps 1674 and 211.
//   The arguments are a struct of their own, read as a whole at a kernel's start (take_args): fetched where they are first
// used they cost a short launch one wait of some hundred cycles after another.
struct StepArgs {
    const void *X, *Y;             // row (owner) and column operand
    const float *v, *u;            // potentials before the step (with part_in: v before the step before)
    float *u_out;                  // u'
    float *v_out;                  // part_in: where v goes (never p.v: other blocks read that)
    float *u_fin;                  // part_in and a dustbin: the step before's u', whose dustbin element is known only now
    const float *part_in;          // column sums of the step before, to be taken into v first (null: v is final)
    float *part_out;               // column sums of this step  [problem][segment][32 (NF M + 2 hw)]; with a dustbin, what its
                                   // row and its column got from each segment, and the potentials those refer to [2 nseg + 2]
    const float *log_a, *log_b;    // logs of the row and column targets (null: unit)
    const float *spoke_r, *spoke_c;   // learned dustbin token: scores of the spokes of the rows and of the columns (null: sdb)
    const int *len_q, *len_k;      // valid lengths per batch item (null: L)
    long us, part_stride;          // floats between problems: potentials; part_in, part_out
    int lstride, sstride;          // ... targets, spokes
    int L, W, NF, M, hw, nseg;     // fragments per block, blocks per segment, ceil(W / 32), segments per problem
    unsigned rcp;                  // segment_reciprocal(NF M)
    const int *cut;                // with lengths: how the problems are cut into segments (null: M blocks each, nseg of them)
    int items, np;                 // batch items of the call, problems of the launch
    int nb_total, rev, nh, n0, dustbin;   // (as in SweepArgs)
    float c2, sdb;                 // score scale in base 2 (fp32 storage); scalar dustbin score
    // fp32 storage: entries are evaluated 2^up times too large, about 2 W + 1, which their row's sum and weight take out again:
    // their exponents are then near zero, where fp32 is finest.  It goes into the rows' potentials, whose rounding a row's own
    // sum sees as a whole (in the columns' the row sums would be off by it).  Distance of O from 64 bits, rms over 40 problems
    // of L = 256, d = 32, W = 16: half-steps 2.61e-7, without 2.70e-7, with 2.52e-7; 16 of L = 4096, d = 64, W = 128: 5.44, 5.36,
    // 4.99e-7.
    float up;
    // Several steps in one launch (single blocks; see STEP_CHAIN in vstep_kernel)
    int nsteps;                    // 1: one step, as everything above says
    int base_left, tail;           // the first base_left end the base solve (slots 0 and 1), the others are the tail's from step `tail` on
    float *slots;                  // u_t in slot 2 t, v_t in slot 2 t + 1 of a problem, Lp floats each
    int Lp;
    StepChain *chain;
    unsigned long long *words;     // [2][problem][block][32 (NF + 2 hw)] column sums on their way, with the step's number
    long wstride, wbuf;            // words between problems, buffers
    unsigned *gate;                // host memory: [0] `seq` when all workgroups have started, [1] where the chain gives up (vfinish_kernel)
    unsigned seq, limit;           // the chain's number; polls of a wait before it gives up
};
__device__ __forceinline__ void take_args(const StepArgs &p)
{
    asm volatile("" ::"s"(p.X), "s"(p.Y), "s"(p.v), "s"(p.u), "s"(p.u_out), "s"(p.v_out), "s"(p.part_in), "s"(p.part_out),
                 "s"(p.log_a), "s"(p.log_b), "s"(p.len_q), "s"(p.len_k), "s"(p.spoke_c), "s"(p.us), "s"(p.part_stride), "s"(p.L),
                 "s"(p.W), "s"(p.M), "s"(p.hw), "s"(p.nseg), "s"(p.rcp), "s"(p.nb_total), "s"(p.rev), "s"(p.lstride), "s"(p.dustbin));
}
// Valid lengths of problem n: Lt columns, Le rows and Lc columns with at least one band edge.
struct StepLens { int Lt, Le, Lc; };
__device__ __forceinline__ StepLens step_lens(const StepArgs &p, int n)
{
    int Lq = p.L, Lk = p.L;
    if (p.len_q) Lq = min(max(p.len_q[(n + p.n0) / p.nh], 0), p.L);
    if (p.len_k) Lk = min(max(p.len_k[(n + p.n0) / p.nh], 0), p.L);
    return StepLens{Lk, Lk > 0 ? min(Lq, Lk + p.W) : 0, Lq > 0 ? min(Lk, Lq + p.W) : 0};
}

// x / SL (tiles per segment) as a multiplication: exact for x < 2^20 and SL <= 2^12, since x (SL - 1) < 2^32
inline unsigned segment_reciprocal(int SL) { return SL == 1 ? 0u : (unsigned)((0x100000000ull + SL - 1) / SL); }
// How a problem is cut into segments: SL tiles each, and 1 / SL as above.
struct StepCut { int SL; unsigned rcp; };
// With lengths the segments are cut from the valid rows of all problems (step_cut_kernel, once per call): as long as it takes to
// have one per CU, each problem as many as its rows need.  Cut for all L rows, most of them have nothing to do where a padded
// batch is short, and the longest item alone sets the time of a launch.  Forward of 32 problems of L = 16384, W = 200, us, cut for
// all rows / so / half-steps: lengths of L/2 .. L 1527 / 1401 / 1416, L/8 .. L 1518 / 1080 / 1239, one item of eight of L and the
// others L/10 1472 / 583 / 1129, all L/10 1220 / 385 / 734; all L the same 1605 / 1746.  In memory: CUT_HEAD words (tiles and blocks per
// segment, 1 / tiles, segments of the problems before the second half and of all), then the segments of the problems before each item.
constexpr int CUT_HEAD = 5, CUT_ITEMS = 128, CUT_SEGS = 256, CUT_HALF = 176;   // (at most so many segments in all, in either half)
struct CutArgs {
    const int *len_q, *len_k;
    int *cut;
    int items, nh, L, W, NF, M, least;   // M blocks per segment at most, at least `least`
};
__device__ __forceinline__ StepCut step_cut(const StepArgs &p)
{
    if (!p.cut) return StepCut{p.NF * p.M, p.rcp};
    return StepCut{p.cut[0], (unsigned)p.cut[2]};
}
// problem and segment of the launch's lb-th one (n < 0: there are no more); the problem's segments
struct CutPlace { int n, seg, nseg; };
__device__ __forceinline__ CutPlace cut_place(const StepArgs &p, int bx)
{
    const int lane = threadIdx.x & 63, half = p.cut[3], all = p.cut[4];
    // the launch's problems are all of the call's, or its first or second half
    const int first = p.n0 ? half : 0, count = (p.n0 ? all : p.np < p.items * p.nh ? half : all) - first;
    const int chunk = (count + 7) >> 3, k = bx >> 3, lb = (bx & 7) * chunk + (p.rev ? chunk - 1 - k : k);
    if (k >= chunk || lb >= count) return CutPlace{-1, 0, 0};
    const int g = first + lb;
    int item = -1;
#pragma unroll
    for (int q = 0; q < CUT_ITEMS / 64; ++q) {
        const int i = 64 * q + lane;
        item += __popcll(__ballot(i < p.items && p.cut[CUT_HEAD + min(i, p.items)] <= g));
    }
    const int before = p.cut[CUT_HEAD + item], nseg = (p.cut[CUT_HEAD + item + 1] - before) / p.nh, r = g - before;
    return CutPlace{item * p.nh + r / nseg - p.n0, r % nseg, nseg};
}
__device__ __forceinline__ int segment_of(const StepCut &cut, int x) { return cut.rcp ? (int)__umulhi((unsigned)x, cut.rcp) : x; }
// What x in base 2 lost by rounding, as the evaluation takes it (x * LOG2E in fp32): a whole row's or column's entries are
// off by it, and the update of its potential puts it right.  (Without: fp32 outputs 4 % further from their value.)
__device__ __forceinline__ float base2_rest(float x)
{
    const float y = x * LOG2E;
    return fmaf(x, LOG2E, -y) + x * 1.925963e-8f;   // (log2 e less its fp32 value)
}
// x in base 2 less `two`, and what that difference lost by rounding
struct Base2 { float x, lost; };
__device__ __forceinline__ Base2 base2_less(float x, float two)
{
#pragma clang fp contract(off)   // (the product rounded by itself, as base2_rest takes it)
    const float y = x * LOG2E, z = y - two;
    return Base2{z, (y - z) - two};
}
// A target's log split up so that a small target (below 2^-32) stays out of the exponents of its column's entries: exp2(score +
// u + v) would go down with the target until the column is empty, next to ordinary ones that need nothing of the kind.
// The entries are evaluated with the potential less `nat` (natural units), then less `two` (base 2); `rest` is what the
// target's log has beside the two.  Where rows are summed, a column's entries get the target back as the factor `weight`:
// a power of two, exact in bf16, or zero, which a target below 2^-126 is beside any other (and whose potential may be
// so large that base 2 loses it: less `nat` it is not).
struct ColumnTarget {
    float two, nat, rest, weight;
    __device__ __forceinline__ ColumnTarget(float log_t) : two(0.f), nat(0.f), rest(log_t), weight(1.f)
    {
        const float y = log_t * LOG2E;
        if (y < -126.f) {
            nat = log_t; rest = 0.f; weight = 0.f;
        } else if (y < -32.f) {
            two = rintf(y);
            rest = fmaf(-LN2, two, log_t);
            weight = __builtin_amdgcn_ldexpf(1.f, (int)two);
        }
    }
};
// The same of a row: its weight, which no product takes, need not be a power of two, so all of the target's log is left out.
__device__ __forceinline__ float row_target_nat(float log_t) { return log_t * LOG2E < -32.f ? log_t : 0.f; }
__device__ __forceinline__ float less_nat(float x, float nat) { return x == -INFINITY ? x : x - nat; }   // (a mark stays one)

// v' of a column from its old value and its column sum; the marks as in the half-steps' epilogue.  BASE2: the sum's entries
// were evaluated with v in base 2.
template <bool BASE2> __device__ __forceinline__ float column_update(float v, float sum, const ColumnTarget &t)
{
    if (v == -INFINITY) return -INFINITY;                       // inactive token: stays so
    if (!(sum > 0.f && sum < INFINITY)) return __builtin_nanf("");
    float x = v - t.nat, rest = BASE2 ? base2_rest(x) : 0.f;
    if (BASE2 && t.two != 0.f) rest += base2_less(x, t.two).lost;
    x += fmaf(-LN2, fast_log2(sum) + rest, t.rest);
    return t.nat != 0.f ? t.nat + x : x;
}
// where the sums of column t < L are: n segments from the first one that meets it
struct ColumnSegments {
    int n, step;
    long first;
    __device__ __forceinline__ ColumnSegments(const StepArgs &p, const StepCut &cut, int t, int nseg_valid)
    {
        const int tile = t >> 5, SL = cut.SL;
        const int lo = min(segment_of(cut, max(tile - p.hw, 0)), nseg_valid - 1), hi = min(segment_of(cut, tile + p.hw), nseg_valid - 1);
        n = hi - lo + 1;
        step = 64 * p.hw;   // (segments overlap by 2 hw tiles)
        first = (long)lo * (32 * (SL + 2 * p.hw)) + (t - 32 * (lo * SL - p.hw));
    }
    // past the last one: the last one again.  (No load is under a condition: it would be waited for at once.)
    __device__ __forceinline__ long at(int i) const { return first + (long)min(i, n - 1) * step; }
};
// their sum, in the order of the segments
__device__ __forceinline__ float column_sum(const StepArgs &p, const StepCut &cut, const float *part, int t, int nseg_valid)
{
    const ColumnSegments cg(p, cut, t, nseg_valid);
    float c = 0.f;
    for (int i0 = 0; i0 < cg.n; i0 += 4) {
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = part[cg.at(i0 + i)];
#pragma unroll
        for (int i = 0; i < 4; ++i) c += i0 + i < cg.n ? x[i] : 0.f;
    }
    return c;
}

// A potential (base 2) in three bf16 parts, which hold its 24 bits.  A column's operand row is (its parts, 0, 1, 1, 1, 0),
// a row's (1, 1, 1, 0, its parts, 0): their product is the sum of the two potentials.  An absent or inactive
// token (-inf) is a number whose exponential is zero, since -inf times an absent part would not be.
__device__ __forceinline__ bf16x4 potential_parts(float x)
{
    const float y = fmaxf(x, -1e30f), z = x == x ? y : x;
    const __bf16 hi = (__bf16)z, mid = (__bf16)(z - (float)hi), lo = (__bf16)(z - (float)hi - (float)mid);
    return bf16x4{hi, mid, lo, (__bf16)0.f};
}

// The dustbin's own potentials after the step before, from what its row and its column got from each segment (in the order
// of the segments, the same in every workgroup).  The column half-step follows the row half-step.  All threads call it;
// red: 2 * 16 floats of LDS.
struct DustbinPair { float u, v; };
// r, c: this thread's share of the sums; u0, v0: the potentials they refer to
template <int NTHR> __device__ __forceinline__ DustbinPair dustbin_from(float r, float c, float u0, float v0, float corner, float *red)
{
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) { r += __shfl_xor(r, s); c += __shfl_xor(c, s); }
    if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = r; red[16 + (threadIdx.x >> 6)] = c; }
    __syncthreads();
    r = c = 0.f;
#pragma unroll
    for (int i = 0; i < NTHR / 64; ++i) { r += red[i]; c += red[16 + i]; }
    const float u = column_update<false>(u0, r + fast_exp2((corner + v0 + u0) * LOG2E), ColumnTarget(0.f));
    return DustbinPair{u, column_update<false>(v0, c + fast_exp2((corner + u + v0) * LOG2E), ColumnTarget(0.f))};
}
template <int NTHR> __device__ __forceinline__ DustbinPair dustbin_pair(const StepArgs &p, const float *part, float corner, float *red)
{
    const float *q = part + (long)p.nseg * (32 * (p.NF * p.M + 2 * p.hw));
    float r = 0.f, c = 0.f;
    for (int i = threadIdx.x; i < p.nseg; i += NTHR) { r += q[i]; c += q[p.nseg + i]; }
    return dustbin_from<NTHR>(r, c, q[2 * p.nseg], q[2 * p.nseg + 1], corner, red);
}

template <int CTRL> __device__ __forceinline__ float dpp_add(float x)
{
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// a: in the lanes of the banks BANKS (quarters of a row of 16 lanes) the sum of b over a lane and its neighbour by CTRL, in the
// others that of a.  (Written out: the compiler makes a move and an add of it.  A DPP source needs the s_nop after a VALU write, here and after it.)
template <int CTRL, int BANKS> __device__ __forceinline__ void merge_add(float &a0, float &a1, float b0, float b1)
{
    a0 = dpp_add<CTRL>(a0); a1 = dpp_add<CTRL>(a1);
    if constexpr (CTRL == 0x128)
        asm("s_nop 1\n\tv_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:%4\n\tv_add_f32_dpp %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:%4\n\ts_nop 1"
            : "+v"(a0), "+v"(a1) : "v"(b0), "v"(b1), "n"(BANKS));
    else
        asm("s_nop 1\n\tv_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:%4\n\tv_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:%4\n\ts_nop 1"
            : "+v"(a0), "+v"(a1) : "v"(b0), "v"(b1), "n"(BANKS));
}
template <int CTRL, int BANKS> __device__ __forceinline__ void merge_add(float &a0, float &a1, float &a2, float &a3, float b0, float b1, float b2, float b3)
{
    merge_add<CTRL, BANKS>(a0, a1, b0, b1);
    merge_add<CTRL, BANKS>(a2, a3, b2, b3);
}
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
// lanes 0 .. 31: a over both halves of the wavefront; lanes 32 .. 63: b
__device__ __forceinline__ float halves_sum(float a, float b)
{
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// the same within each half, between its rows of 16 lanes
__device__ __forceinline__ float rows16_sum(float a, float b)
{
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Wavefronts per SIMD that the registers must allow: three short blocks of four wavefronts fit a CU's LDS (a chain of 16 problems of
// L = 3001, W = 100 needs them all).  Narrow blocks at d = 32: five (32 problems of L = 17853, W = 17, us per step: 26.1 -> 25.7,
// forward and backward 699 -> 685).
template <typename T, int D, int NF, int G, int NTW, int KIND, int FORM> constexpr bool step_narrow = sizeof(T) == 2 && D == 32 && NF * G == 4 && NTW <= 3 && KIND == STEP_BLOCK && FORM == STEP_ANY;
template <typename T, int D, int NF, int G, int NTW, int KIND, int FORM> constexpr int step_waves =
    KIND == STEP_CHAIN && FORM == STEP_DUSTBIN && NF * G == 4 && NTW <= 5 && StepTile<T, D>::BYTES <= 4096 && sizeof(T) == 2 ? 3
    : step_narrow<T, D, NF, G, NTW, KIND, FORM> ? 5 : 1;
template <typename T, int D, int NF, int G, int NTW, int KIND, int FORM>
__global__ __launch_bounds__(64 * NF * G, (step_waves<T, D, NF, G, NTW, KIND, FORM>)) void vstep_kernel(const StepArgs p)
{
    using ST = StepTile<T, D>;
    using LD = StepLds<T, D, NF, G, NTW, KIND, FORM>;
    constexpr bool TIGHT = KIND == STEP_TIGHT, MARCH = KIND == STEP_MARCH || TIGHT, CHAIN = KIND == STEP_CHAIN;
    constexpr bool PRE = (sizeof(T) == 2);
    constexpr int BM = 32 * NF, NTHR = 64 * NF * G;
    constexpr bool TARGETS = FORM == STEP_TARGETS, MAY_CUT = MARCH && (TARGETS || FORM == STEP_CUT);
    const bool DUST = FORM == STEP_ANY ? p.dustbin != 0 : FORM == STEP_DUSTBIN;
    extern __shared__ __align__(16) unsigned char smem[];
    take_args(p);
    const int bx = (int)blockIdx.x;
    int n, seg, nseg = p.nseg;
    if (MAY_CUT && p.cut) {
        const CutPlace at = cut_place(p, bx);
        if (at.n < 0) return;
        n = __builtin_amdgcn_readfirstlane(at.n); seg = __builtin_amdgcn_readfirstlane(at.seg); nseg = __builtin_amdgcn_readfirstlane(at.nseg);
    } else {
        const int chunk = (p.nb_total + 7) >> 3, lb = (bx & 7) * chunk + (p.rev ? chunk - 1 - (bx >> 3) : (bx >> 3));
        if (lb >= p.nb_total) return;
        n = lb / nseg; seg = lb % nseg;
    }
    const int hw = p.hw, NT = 2 * hw + 1, nwt = NF + 2 * hw;
    const LD lds(hw);
    const int RS = lds.rs;
    int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int f = wave / G, g = wave % G;
    const int L = p.L, W = p.W;
    const StepLens ln = step_lens(p, n);
    const int Lt = ln.Lt, Le = ln.Le, Lc = ln.Lc;
    const StepCut cut = MAY_CUT ? step_cut(p) : StepCut{MARCH ? NF * p.M : NF, p.rcp};
    const int M = MAY_CUT ? cut.SL / NF : MARCH ? p.M : 1, nseg_valid = (Le + BM * M - 1) / (BM * M), nblk = (L + BM - 1) / BM;
    // blocks (the last segment's go on to the end: the rows past the valid ones are its to clear); those with valid rows
    const int b0 = min(seg * M, nblk), b1 = seg + 1 == nseg ? nblk : min(b0 + M, nblk), bv = min(b1, (Le + BM - 1) / BM);

    unsigned char *vs = smem + lds.vs;
    const int cps = lds.cps, cp_own = f * (LD::PADDED ? cps + 32 : cps);   // column sums of a fragment (StepLds::PADDED); this one's first tile
    float *us = reinterpret_cast<float *>(smem + LD::US);
    float *rs = reinterpret_cast<float *>(smem + LD::RSUM), *cp0 = reinterpret_cast<float *>(smem + lds.cp);
    float *wsw = reinterpret_cast<float *>(smem + LD::WS) + 32 * wave;

    const float *vp = p.v + n * p.us, *xsp = p.u + n * p.us;
    float *u_out = p.u_out + n * p.us, *v_out = p.v_out + n * p.us;
    const float *part = p.part_in ? p.part_in + n * p.part_stride : nullptr;
    const float *lap = TARGETS && p.log_a ? p.log_a + (long)n * p.lstride : nullptr;
    const float *lbp = TARGETS && p.log_b ? p.log_b + (long)n * p.lstride : nullptr;
    const float *spr = p.spoke_r ? p.spoke_r + (long)n * p.sstride : nullptr, *spc = p.spoke_c ? p.spoke_c + (long)n * p.sstride : nullptr;
    // A chain: steps follow each other in the same workgroups.  What a block needs of others between two steps are their column sums
    // of its window, which go from hand to hand as 8-byte words of a sum and the step's number: a reader polls the words
    // themselves, so nothing has to be ordered or acknowledged (relaxed accesses of agent scope).  Two buffers do: a
    // block writes a step's words after it has read the step before's of every block that reads its own, and those have then read
    // the words of two steps before.  A hand-over by itself takes about 1 us (neighbours, 256 words; inside a step 1000 to 1600 cycles)
    // where a launch takes 5 (2.3 if it is empty).  The host sees to it that the workgroups fit the device together and that no other
    // launch of this process that waits is waiting for room (WaitGate); a wait that runs out all the same (other programs on the
    // device) ends the launch, and the problem is solved again by the launch that follows (vfinish_kernel).
    // (A kind of its own, since what it adds costs a launched step of a call with a dustbin 4 %, and forms of its own, since a flag that is
    // read costs a chain without a dustbin as much.)
    __shared__ int gave_up;
    float *slots = p.slots + n * p.us;
    if (CHAIN && tid == 0) {
        gave_up = 0;
        if (__hip_atomic_fetch_add(&p.chain->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == (unsigned)p.nb_total)
            __hip_atomic_store(p.gate, p.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // where step st leaves its potentials (-1: nowhere)
    auto slot_of = [&](int st) { return st + 1 < p.base_left ? -1 : st + 1 == p.base_left ? 0 : 2 * (p.tail + st - p.base_left); };
    if constexpr (CHAIN) {   // rows without an edge: zeros (v: from the last column with an edge on; the last block with rows has the others)
        for (int t = max(b0, bv) * BM + tid; t < min(b1 * BM, L); t += NTHR)
            for (int st = 0; st < p.nsteps; ++st) {
                const int sl = slot_of(st);
                if (sl < 0) continue;
                slots[(long)sl * p.Lp + t] = 0.f;
                if (t >= Lc && st + 1 < p.nsteps) slots[(long)(sl + 1) * p.Lp + t] = 0.f;
            }
        if (b0 >= bv) return;
    }
    // rows without an edge: zeros, and this segment's share of v there
    for (int t = max(b0, bv) * BM + tid; t < min(b1 * BM, L) && !CHAIN; t += NTHR) {
        u_out[t] = 0.f;
        if (part) v_out[t] = t < Lc ? column_update<true>(vp[t], column_sum(p, cut, part, t, nseg_valid), ColumnTarget(lbp ? lbp[t] : 0.f)) : 0.f;
    }
    if (b0 >= bv) return;
    const long moff = (long)n * L * D;
    const unsigned char *Xb = reinterpret_cast<const unsigned char *>(reinterpret_cast<const T *>(p.X) + moff);
    const unsigned char *Yb = reinterpret_cast<const unsigned char *>(reinterpret_cast<const T *>(p.Y) + moff);
    const int kseg = b0 * NF - hw;   // the segment's first tile, ring slot 0

    // LDS-direct loads of the other side's tiles: one instruction of a wavefront fills 1 KB, RPI rows.  Rows outside the
    // matrix repeat its first or last valid one; they are masked where they are used.
    constexpr int RPI = 64 / ST::CPR, IPT = 32 / RPI;
    const unsigned smem_at = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    auto dma_at = [&](long t, int lds_at, unsigned o) {   // (t uniform)
        // (written out, because the compiler takes every later LDS read for one of these bytes and waits at once; the
        // kernel waits where it needs them.  No register is written.)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(smem_at + lds_at), "v"(o), "s"(Yb + t * ST::ROWB)
                     : "memory", "m0");
    };
    auto dma_rows = [&](long t, int lds_at, bool whole) {   // rows t ... t + RPI - 1
        const int lrow = lane / ST::CPR;
        const unsigned col = ((lane % ST::CPR) ^ ST::swz((int)(t & 31) + lrow)) * 16;
        unsigned o = lrow * ST::ROWB + col;
        if (!whole) {
            const long last = Lt - 1, tb = min(max(t, 0L), last);
            o = (unsigned)(min(max(t + lrow, 0L), last) - tb) * ST::ROWB + col;
            t = tb;
        }
        dma_at(t, lds_at, o);
    };
    // `count` tiles from tile k on into the ring from `slot` on, by the whole workgroup
    auto dma = [&](int k, int count, int slot) {
        const bool whole = k >= 0 && 32 * (k + count) <= Lt;
        for (int i = wave; i < count * IPT; i += NF * G) {
            int sl = slot + i / IPT;
            if (sl >= RS) sl -= RS;
            dma_rows(32L * (k + i / IPT) + (i % IPT) * RPI, lds.y + sl * ST::BYTES + (i % IPT) * 1024, whole);
        }
    };
    // v of a column (and with targets its weight) into its place in LDS, as the evaluation takes it
    auto stage_v = [&](int at, int t, float v, float lb) {
        const ColumnTarget tg(TARGETS ? lb : 0.f);
        v = t >= 0 && t < Lt ? base2_less(less_nat(v, tg.nat), tg.two).x : -INFINITY;
        if constexpr (PRE) {
            bf16x4 parts = potential_parts(v);
            if constexpr (TARGETS) parts[3] = (__bf16)tg.weight;
            *reinterpret_cast<bf16x4 *>(vs + at * 8) = parts;
        } else if constexpr (TARGETS) {
            *reinterpret_cast<float2 *>(vs + at * 8) = make_float2(v, __builtin_amdgcn_ldexpf(tg.weight, -(int)p.up));
        } else {
            *reinterpret_cast<float *>(vs + at * 4) = v;
        }
    };
    // u of a row of a block, less its target, into its place in LDS
    auto stage_u = [&](int at, float u, float log_a) {
        if constexpr (TARGETS) u = less_nat(u, row_target_nat(log_a));
        us[at] = u;
        if constexpr (!PRE) us[(LD::UE - LD::US) / 4 + at] = base2_less(u, -p.up).x;
    };
    // Loads return in order: the vectors, which need work, are requested before the tiles and the owner rows.
    constexpr int NWIN = (32 * (NF + G * NTW) + NTHR - 1) / NTHR;   // columns of a window per thread
    constexpr int NSUM = MARCH ? 3 : (G * NTW - 1) / NF + 2;        // segments that a column can have sums from, at most
    const float u_first = tid < BM && b0 * BM + tid < Le ? xsp[b0 * BM + tid] : -INFINITY;
    const float la_first = lap ? lap[min(b0 * BM + min(tid, BM - 1), Le - 1)] : 0.f;
    float win_v[NWIN], win_sum[NWIN][NSUM], win_lb[NWIN], win_sp[NWIN];
#pragma unroll
    for (int k = 0; k < NWIN; ++k) {
        const int t = min(max(32 * kseg + tid + k * NTHR, 0), L - 1);
        win_v[k] = vp[t];
        win_lb[k] = 0.f;
        win_sp[k] = (DUST && spc ? spc : vp)[t];   // (v, which is requested anyway, where nobody asks)
        if (lbp) win_lb[k] = lbp[min(t, max(Lc - 1, 0))];
        if (part) {
            const ColumnSegments cg(p, cut, t, nseg_valid);
#pragma unroll
            for (int i = 0; i < NSUM; ++i) win_sum[k][i] = part[cg.at(i)];
        }
    }
    // Dustbin: its potentials as this step's rows see them (uL is a reference only: the row half-step replaces it)
    auto uniform = [](float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); };
    float uL = 0.f, vL = 0.f, to_row = 0.f, to_col = 0.f;   // this thread's share of what its row and its column get
    float *dust = p.part_out + n * p.part_stride + (long)p.nseg * (32 * (NF * M + 2 * hw));
    if (DUST) {
        const float corner = spr ? spr[L] : p.sdb;
        if (part) {
            const DustbinPair d = dustbin_pair<NTHR>(p, part, corner, rs);
            uL = uniform(d.u); vL = uniform(d.v);
        } else {
            uL = uniform(xsp[L]); vL = uniform(vp[L]);
        }
        if (seg == 0 && tid == 0) {
            dust[2 * p.nseg] = uL; dust[2 * p.nseg + 1] = vL;
            if (part) { p.u_fin[n * p.us + L] = uL; v_out[L] = vL; }
        }
    }
    // v of a column from its sums; what the dustbin's row gets from it
    auto finish_v = [&](int t, float v, float sum, float lb, float sp) {
        if (DUST && !spc) sp = p.sdb;
        if (part) {
            if (DUST) sum += fast_exp2((sp + uL + v) * LOG2E);
            v = t < Lc ? column_update<true>(v, sum, ColumnTarget(TARGETS ? lb : 0.f)) : 0.f;
        }
        if (t >= b0 * BM && t < min(bv * BM, L)) {
            if (part) v_out[t] = v;
            if (DUST) to_row += fast_exp2((sp + v + uL) * LOG2E);
        }
        return v;
    };
    OwnerFrag<T, D> xf;
    dma(kseg, nwt, 0);
    xf.load(reinterpret_cast<const T *>(Xb), min((b0 * NF + f) * 32 + (lane & 31), Le - 1), Le, lane >> 5);
    if constexpr (LD::PADDED)
        for (int i = tid; i < LD::TWO * NF * cps; i += NTHR) cp0[i] = 0.f;   // (while the loads are on their way)
#pragma unroll
    for (int k = 0; k < NWIN; ++k) {
        const int i = tid + k * NTHR, t = 32 * kseg + i;
        float sum = 0.f;
        if (part) {
            const ColumnSegments cg(p, cut, min(max(t, 0), L - 1), nseg_valid);
#pragma unroll
            for (int q = 0; q < NSUM; ++q) sum += q < cg.n ? win_sum[k][q] : 0.f;
        }
        if (i < 32 * nwt) {   // (later columns: with their block)
            win_v[k] = finish_v(t, win_v[k], sum, win_lb[k], win_sp[k]);
            stage_v(i, t, win_v[k], win_lb[k]);
        }
    }
    // a chain's rows' share is known here, before the evaluation
    __shared__ float dust_row[16];
    auto sum_row = [&]() {
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) to_row += __shfl_xor(to_row, s);
        if ((tid & 63) == 0) dust_row[wave] = to_row;
    };
    if (CHAIN && DUST) sum_row();
    if (tid < BM) stage_u(tid, u_first, la_first);
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0): the LDS-direct loads have arrived
    __syncthreads();

    const int klast = (Lt - 1) / TT;
    // This wavefront's tiles of the 2 hw + 1: j0 on, cnt of them.  Groups of a fragment that have one more than others are other
    // groups in its neighbour on the same SIMD, which has the wavefronts w and w + 4: the last of NTW is not evaluated where it is not
    // there.  (Others are, in bf16 storage, and masked: at half-bands of 257 to 480 a wavefront has 5 to 8 tiles and evaluates 8.)
    const int turn = G == 4 ? f : f >> 1;
    int j0 = g * (NT / G), cnt = NT / G;
#pragma unroll
    for (int i = 0; i < G; ++i)
        if ((i + turn) % G < NT % G) {
            if (i < g) ++j0;
            if (i == g) ++cnt;
        }
    int base = 0;   // ring slot of the block's first tile
    float *po = p.part_out + n * p.part_stride + (long)seg * (32 * (NF * M + 2 * hw));   // the segment's column sums

    // what block b + 1 adds (a thread below BM: one column, one row): requested while block b is worked on, stored after the
    // last use of the slots' old content
    struct Added { float v, u, sum[3], la, lb, spoke; };
    auto added_column = [&](int b) { return 32 * (b * NF - hw + nwt) + tid; };
    auto later_segments = [&](int t) { return min(segment_of(cut, (t >> 5) + hw), nseg_valid - 1) - seg; };   // that have summed column t too
    auto request = [&](int b) {
        Added a{0.f, 0.f, {0.f, 0.f, 0.f}, 0.f, 0.f, 0.f};
        if (64 * wave < BM) {   // (uniform: the other wavefronts have nothing to add)
            const int nt = added_column(b), tc = min(nt, L - 1), o = min((b + 1) * BM + tid, Le - 1);
            a.v = vp[tc];
            a.u = xsp[o];
            if (lap) a.la = lap[o];
            if (lbp) a.lb = lbp[min(tc, max(Lc - 1, 0))];
            if (DUST) a.spoke = (spc ? spc : vp)[tc];
            if (part) {   // the first segment is this one, and there are at most three: a segment is at least hw tiles long
                const float *pp = part + (long)seg * (32 * (NF * M + 2 * hw)) + (tc - 32 * kseg);
                const int nq = later_segments(nt);
#pragma unroll
                for (int i = 0; i < 3; ++i) a.sum[i] = pp[(long)min(i, nq) * (64 * hw)];
            }
        }
        return a;
    };
    auto request_tiles = [&](int b) {
        const int k = b * NF - hw + nwt;
        int sl = base + nwt;
        if (sl >= RS) sl -= RS;
        if constexpr (MARCH) {   // (its address work is most of this: a wavefront loads the same piece of every few tiles)
            static_assert(NF * G % IPT == 0 && NF * IPT % (NF * G) == 0, "whole tiles by all wavefronts");
            constexpr int STEP = NF * G / IPT;
            const int piece = wave % IPT, lrow = lane / ST::CPR;
            const bool whole = 32 * (k + NF) <= Lt;
            const unsigned o = lrow * ST::ROWB + ((lane % ST::CPR) ^ ST::swz(piece * RPI + lrow)) * 16;
#pragma unroll
            for (int i = 0; i < IPT / G; ++i) {
                const int tile = wave / IPT + i * STEP;
                int at = sl + tile;
                if (at >= RS) at -= RS;
                if (whole) dma_at(32L * (k + tile) + piece * RPI, lds.y + at * ST::BYTES + piece * 1024, o);
                else dma_rows(32L * (k + tile) + piece * RPI, lds.y + at * ST::BYTES + piece * 1024, false);
            }
        }
    };
    auto stage_added_v = [&](const Added &a, int b) {
        if (tid >= BM) return;
        const int nt = added_column(b), nq = later_segments(nt);
        const float v = finish_v(nt, a.v, a.sum[0] + (nq >= 1 ? a.sum[1] : 0.f) + (nq >= 2 ? a.sum[2] : 0.f), a.lb, a.spoke);
        int sl = 32 * (base + nwt) + tid;
        if (sl >= 32 * RS) sl -= 32 * RS;
        stage_v(sl, nt, v, a.lb);
    };
    auto stage_added_u = [&](const Added &a, int b, int us_buf) {
        if (tid < BM) stage_u(us_buf * BM + tid, (b + 1) * BM + tid < Le ? a.u : -INFINITY, a.la);
    };
    // a row of block b, this lane's: its potential (TARGETS: less nat), the score of its spoke, its target
    struct Row { float u, rest, spoke, la; };
    auto row_of = [&](int b, int us_buf) {
        const int c = lane & 31, o = (b * NF + f) * 32 + c;
        Row r;
        r.spoke = r.la = 0.f;
        if (DUST) r.spoke = spr ? spr[min(o, L - 1)] : p.sdb;
        if (lap) r.la = lap[min(o, Le - 1)];
        r.u = us[us_buf * BM + 32 * f + c];
        r.rest = PRE ? base2_rest(r.u) : base2_rest(r.u) + base2_less(r.u, -p.up).lost;
        return r;
    };

    // KEEP: a chain's scores stay in registers from step to step, since a tile's products take 2048 cycles at d = 64.  The plan
    // entries lie beside them where one workgroup fills a CU's LDS with four wavefronts, which may have 512 registers each, or
    // where both are few; elsewhere they are evaluated a second time for the column sums.
    // Chained steps, us each, products in every step -> kept: 8 problems of L = 4096, d = 64, W = 128 (4,1,9) 14.8 -> 6.4, of 8000 (8,1,9)
    // 25.6 -> 11.9; 4 of 4000, W = 256 (2,4,5) 15.5 -> 8.4; 8 of 2000, d = 32, W = 128 (2,2,5) 7.1 -> 6.2; one of 256, W = 16 3.5 -> 2.7.
    // (bf16: a tile's products take 160 cycles, which the exponentials partly hide.)
    constexpr bool KEEP = FORM == STEP_KEEP;
    constexpr bool STORE_E = !KEEP || NTW <= 3 || (NF * G <= 4 && ST::BYTES >= 8192 && NF + G * NTW > 9);
    f32x16 E[STORE_E ? NTW : 1], S[KEEP ? NTW : 1];   // plan entries, scores of a block: this wavefront's
    // KEEP: first, that the scores are not there yet; columns, that the entries are wanted again, by column(s, e).
    auto evaluate = [&](int b, int us_buf, float u_own, float (&rsum)[16], auto &&late, bool first, bool columns, auto &&column) {
        const int c = lane & 31, h = lane >> 5, k0 = b * NF - hw, o_f = (b * NF + f) * 32;
        [[maybe_unused]] f32x16 ci;   // fp32 storage: the rows' potentials
        if constexpr (!PRE) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v4 = *reinterpret_cast<const float4 *>(us + (LD::UE - LD::US) / 4 + us_buf * BM + 32 * f + 8 * q + 4 * h);
                ci[4 * q + 0] = v4.x; ci[4 * q + 1] = v4.y; ci[4 * q + 2] = v4.z; ci[4 * q + 3] = v4.w;
            }
        }
        if (!columns) {
#pragma unroll
            for (int r = 0; r < 16; ++r) rsum[r] = 0.f;
        }
        [[maybe_unused]] float bt[NTW];   // TARGETS: weight of this lane's column of each tile
        auto add_rows = [&](const f32x16 &e, int s, int r) {
            if constexpr (TARGETS) rsum[r] = fmaf(e[r], bt[s], rsum[r]);
            else rsum[r] += e[r];
        };
        // entries of an edge tile outside the band or the matrix become zero (whatever they are): with o = o_f + 4 h +
        // off_r and t = t0 + c, |t - o| <= W keeps lo <= off_r <= lo + 2 W.  As a bit per offset: two instructions an
        // entry, the first ones of eight entries together (one after the other they wait for each other).
        auto mask = [&](f32x16 &e, int t0, bool present) {
            const int lo = t0 + c - o_f - 4 * h - W, hi = min(min(lo + 2 * W, Le - 1 - o_f - 4 * h), 31);
            unsigned keep = (~0u << min(max(lo, 0), 31)) & (~0u >> (31 - max(hi, 0)));
            keep = lo <= 31 && hi >= 0 && present && t0 + c < Lt ? keep : 0u;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                int m[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) asm volatile("v_bfe_i32 %0, %1, %2, 1" : "=v"(m[i]) : "v"(keep), "n"(16 * q + 8 * (i >> 2) + (i & 3)));
#pragma unroll
                for (int i = 0; i < 8; ++i) e[8 * q + i] = __int_as_float(__float_as_int(e[8 * q + i]) & m[i]);
            }
        };
        const int kw = k0 + f + j0;   // this wavefront's first tile
        const int nj = min(cnt, klast + 1 - kw), sfirst = max(0, -kw);   // tiles [sfirst, nj) are there
        // [ilo, ilo + icnt): tiles wholly inside the matrix and, for all 32 rows, inside the band
        const int d0 = 32 * kw - o_f;
        const int ilo = max(sfirst, (62 - W - d0) >> 5), ihi = min(min((W - 31 - d0) >> 5, Lt / 32 - 1 - kw), nj - 1);
        const unsigned icnt = o_f + 32 <= Le ? max(ihi - ilo + 1, 0) : 0, pcnt = max(nj - sfirst, 0);
        const unsigned whole = icnt ? (2u << (ilo + icnt - 1)) - (1u << ilo) : 0u;   // (ilo + icnt <= NTW)
        auto interior = [&](int s) { return whole >> s & 1; };
        auto present = [&](int s) { return (unsigned)(s - sfirst) < pcnt; };
        int slot = lds.slot(base + f + j0);
        if constexpr (PRE) {
            // one wavefront's pipeline: the products of tile s + 1 are issued among the exponentials of tile s, and the
            // operand of tile s + 2 is requested as its registers come free
            constexpr int KS = D / 16;
            bf16x8 y[KS], yv, xv;
            {   // the rows' potentials, in the lanes that hold the first eight of the sixteen
                const bf16x4 u3 = potential_parts(u_own * LOG2E);
                const __bf16 one = (__bf16)1.f, no = (__bf16)0.f;
                xv = bf16x8{one, one, one, no, u3[0], u3[1], u3[2], no};
#pragma unroll
                for (int i = 0; i < 8; ++i) xv[i] = h ? no : xv[i];
            }
            f32x16 zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.f;
            // LDS addresses of tile s less s tiles: the instructions add those.  Where the ring ends (of a single block: where its
            // window does) they go back by as much.  (Narrow blocks make each address where it is used, which takes fewer registers.)
            constexpr bool ADVANCE = !step_narrow<T, D, NF, G, NTW, KIND, FORM>;
            typedef __attribute__((address_space(3))) const unsigned char *lds_ptr;
            typedef __attribute__((address_space(3))) const bf16x8 *lds_row;
            typedef __attribute__((address_space(3))) const bf16x4 *lds_parts;
            unsigned ya[KS], va = smem_at + lds.vs + (32 * slot + c) * 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) ya[ks] = smem_at + lds.y + slot * ST::BYTES + c * ST::ROWB + (((2 * ks + h) ^ ST::swz(c)) << 4);
            const unsigned char *ybase = smem + lds.y + c * ST::ROWB;
            auto rd = [&](int s, int ks) {
                if constexpr (ADVANCE) y[ks] = *(lds_row)((lds_ptr)(ya[ks] + 0u) + s * ST::BYTES);
                else y[ks] = *reinterpret_cast<const bf16x8 *>(ybase + slot * ST::BYTES + (((2 * ks + h) ^ ST::swz(c)) << 4));
            };
            auto rdv = [&](int s) {   // (the first read of tile s)
                if constexpr (!ADVANCE) {
                    if (s > 0) slot = lds.slot(slot + 1);
                } else if (s > 0 && (MARCH ? slot + s == RS : slot + s >= RS)) {
                    const int back = MARCH ? RS : 1;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) ya[ks] -= back * ST::BYTES;
                    va -= back * 256;
                }
                const bf16x4 v3 = ADVANCE ? *(lds_parts)((lds_ptr)(va + 0u) + s * 256) : *reinterpret_cast<const bf16x4 *>(vs + (32 * slot + c) * 8);
                // (a zero of the row's operand meets it; an absent tile's slot may hold anything, and its zero entries stay zero)
                if constexpr (TARGETS) bt[s] = present(s) ? (float)v3[3] : 0.f;
                const __bf16 one = (__bf16)1.f, no = (__bf16)0.f;
                yv = bf16x8{v3[0], v3[1], v3[2], v3[3], one, one, one, no};
            };
            rdv(0);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) rd(0, ks);
            E[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv, yv, zero, 0, 0, 0);
            if (NTW > 1) rdv(1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                E[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf.v[ks], y[ks], E[0], 0, 0, 0);
                if (NTW > 1) rd(1, ks);
            }
            constexpr int RPS = 16 / (KS + 1) + 1;   // entries per product: KS + 1 products and sixteen entries
            constexpr int SURE = G > 1 ? NTW - 1 : NTW;   // (with one group the last tile is there, or masked where the band is less)
#pragma unroll
            for (int s = 0; s < SURE; ++s) {
#pragma unroll
                for (int ks = 0; ks <= KS; ++ks) {
                    if (s + 1 < NTW) {
                        if (ks == 0) E[s + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv, yv, zero, 0, 0, 0);
                        else E[s + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf.v[ks - 1], y[ks - 1], E[s + 1], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (s + 2 < NTW) {
                            if (ks == 0) rdv(s + 2);
                            else rd(s + 2, ks - 1);
                        }
                    }
#pragma unroll
                    for (int r = ks * RPS; r < 16 && r < (ks + 1) * RPS; ++r) {
                        E[s][r] = fast_exp2(E[s][r]);
                        if (s > 0) add_rows(E[s - 1], s - 1, r);
                        asm volatile("" : "+v"(rsum[r]));   // the sums here, among the products, not for all tiles at the end
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (!interior(s)) mask(E[s], 32 * (kw + s), present(s));
                if (s == (NTW > 4 ? 3 : NTW - 2)) late();
            }
            if constexpr (SURE < NTW) {
                if constexpr (NTW > 1) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) add_rows(E[NTW - 2], NTW - 2, r);
                }
                if (NTW - 1 < cnt) {   // (uniform)
#pragma unroll
                    for (int r = 0; r < 16; ++r) E[NTW - 1][r] = fast_exp2(E[NTW - 1][r]);
                    if (!interior(NTW - 1)) mask(E[NTW - 1], 32 * (kw + NTW - 1), present(NTW - 1));
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) E[NTW - 1][r] = 0.f;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) add_rows(E[NTW - 1], NTW - 1, r);
        } else {
#pragma unroll
            for (int s = 0; s < NTW; ++s) {
                if (s == NTW / 2) late();
                f32x16 e;
                if (present(s)) {   // (uniform)
                    f32x16 &score = KEEP ? S[KEEP ? s : 0] : e;
                    if (!KEEP || first) {
                        const unsigned char *yr = smem + lds.y + slot * ST::BYTES + c * ST::ROWB;
                        f32x16 a;
#pragma unroll
                        for (int r = 0; r < 16; ++r) a[r] = 0.f;
#pragma unroll
                        for (int q = 0; q < D / 8; ++q) {
                            const float4 y = *reinterpret_cast<const float4 *>(yr + (((h * (D / 8) + q) ^ ST::swz(c)) << 4));
                            a = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.v[4 * q + 0], y.x, a, 0, 0, 0);
                            a = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.v[4 * q + 1], y.y, a, 0, 0, 0);
                            a = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.v[4 * q + 2], y.z, a, 0, 0, 0);
                            a = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.v[4 * q + 3], y.w, a, 0, 0, 0);
                        }
                        score = a;
                    }
                    const float vt = *reinterpret_cast<const float *>(vs + (32 * slot + c) * LD::VB);
                    if constexpr (TARGETS) bt[s] = *reinterpret_cast<const float *>(vs + (32 * slot + c) * LD::VB + 4);
#pragma unroll
                    for (int r = 0; r < 16; ++r) e[r] = fast_exp2(fmaf(score[r], p.c2, ci[r] + vt));
                    if (!interior(s)) mask(e, 32 * (kw + s), true);
                    if (!columns) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) add_rows(e, s, r);
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) e[r] = 0.f;
                }
                if constexpr (STORE_E) E[s] = e;
                else if (columns) column(s, e);
                slot = lds.slot(slot + 1);
            }
        }
    };
    // row sums over the 32 columns of a lane half: registers r, r + 8 to the two rows of 16 lanes, then within those
    auto write_row_sums = [&](const float (&rsum)[16], float *d) {
        float t[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) t[r] = rows16_sum(rsum[r], rsum[r + 8]);
        if constexpr (MARCH) {
            // two registers into one each time: one in the first half of a row of lanes and one in the second, then by quarters.  (Fewer
            // instructions, but each waits for the one before: with one block per workgroup, which has others beside it, the plain way is
            // 1 % faster.)
            merge_add<0x128, 0xc>(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7]);   // row_ror:8
            merge_add<0x141, 0xa>(t[0], t[1], t[2], t[3]);                           // row_half_mirror
#pragma unroll
            for (int r = 0; r < 2; ++r) t[r] = dpp_add<0xb1>(dpp_add<0x4e>(t[r]));   // quad_perm:[2,3,0,1], [1,0,3,2]
            // register r of quarter q of a row of lanes is the r + 2 (q & 1) + 4 (q >> 1)-th of eight, the second row's 8 further; the
            // i-th of sixteen is row 8 (i >> 2) + (i & 3) (+ 4 in the second half)
            if ((lane & 3) == 0) {
                const int q = lane >> 2;
                d += (f * G + g) * 32 + 16 * ((q >> 2) & 1) + 8 * ((q >> 1) & 1) + 4 * (lane >> 5) + 2 * (q & 1);
                *reinterpret_cast<float2 *>(d) = make_float2(t[0], t[1]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) t[r] = dpp_add<0x128>(t[r]);   // row_ror:8, 4, 2, 1
#pragma unroll
            for (int r = 0; r < 8; ++r) t[r] = dpp_add<0x124>(t[r]);
#pragma unroll
            for (int r = 0; r < 8; ++r) t[r] = dpp_add<0x122>(t[r]);
#pragma unroll
            for (int r = 0; r < 8; ++r) t[r] = dpp_add<0x121>(t[r]);
            if ((lane & 15) == 0) {   // register r of the second row of lanes is r + 8: rows 16 further
                d += (f * G + g) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane >> 5);
                *reinterpret_cast<float4 *>(d) = make_float4(t[0], t[1], t[2], t[3]);
                *reinterpret_cast<float4 *>(d + 8) = make_float4(t[4], t[5], t[6], t[7]);
            }
        }
    };
    // From the row sums of block b: u' of this lane's row, and the weights of the fragment's rows as the column sums take them.
    // exp: TARGETS, exponent that the weights are taken less of.
    struct Weights { f32x16 w; float u_new; int exp; };
    auto weights = [&](int b, const Row &row, const float *sums) {
        const int c = lane & 31, h = lane >> 5, o = (b * NF + f) * 32 + c;
        float tot = 0.f;
#pragma unroll
        for (int i = 0; i < G; ++i) tot += sums[(f * G + i) * 32 + c];
        if constexpr (!PRE && !TARGETS) tot = __builtin_amdgcn_ldexpf(tot, -(int)p.up);   // (TARGETS: in the columns' weights)
        const float edge = DUST ? fast_exp2((row.spoke + vL + row.u) * LOG2E) : 0.f;   // spoke (o, dustbin of the other side)
        tot += edge;
        float u_new = 0.f, w = 0.f;
        int wexp = 0;
        if (o < Le) {
            if (row.u == -INFINITY) {
                u_new = -INFINITY;   // inactive token: stays so
            } else if (!(tot > 0.f && tot < INFINITY)) {
                u_new = w = __builtin_nanf("");
            } else if constexpr (!TARGETS) {
                const float delta = fmaf(-LN2, fast_log2(tot) + row.rest, 0.f);
                u_new = row.u + delta;
                w = PRE ? __builtin_amdgcn_rcpf(tot) : 1.f / tot;
                w = fmaf(w, (u_new - row.u) - delta, w);   // as u' was rounded, so that v' makes up for it
            } else {
                const float nat = row_target_nat(row.la), delta = fmaf(-LN2, fast_log2(tot) + row.rest, row.la - nat), x = row.u + delta;
                u_new = nat + x;
                w = PRE ? __builtin_amdgcn_rcpf(tot) : 1.f / tot;
                w = fmaf(w, ((u_new - nat) - x) + ((x - row.u) - delta), w);
            }
        }
        if constexpr (TARGETS) {
            // the weight is target / sum.  Where a fragment's rows all weigh little (small targets over columns of ordinary ones),
            // their entries are as large as the weights are small: a common exponent is left out until the column sums are done
            const float lac = fmaxf(row.la, -1e5f), la2 = lac * LOG2E, q = rintf(la2);   // (a target below that weighs nothing either way)
            w *= fast_exp2((la2 - q) + base2_rest(lac));
            float top = w > 0.f ? q + fast_log2(w) : -INFINITY;
            if (!__any(top >= -40.f)) {
#pragma unroll
                for (int s = 16; s >= 1; s >>= 1) top = fmaxf(top, __shfl_xor(top, s));
                if (top > -INFINITY) wexp = (int)top;
            }
            w = __builtin_amdgcn_ldexpf(w, (int)q - wexp);
        }
        if (h == 0) wsw[c] = PRE ? w : __builtin_amdgcn_ldexpf(w, -(int)p.up);
        if (h == 0 && g == 0 && o < Le) to_col += edge * w;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        Weights wt;
        wt.u_new = u_new; wt.exp = wexp;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v4 = *reinterpret_cast<const float4 *>(wsw + 8 * q + 4 * h);
            wt.w[4 * q + 0] = v4.x; wt.w[4 * q + 1] = v4.y; wt.w[4 * q + 2] = v4.z; wt.w[4 * q + 3] = v4.w;
        }
        return wt;
    };
    auto column_of = [&](const f32x16 &e, const Weights &wt) {
        float x = 0.f, y = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) { x = fmaf(e[r], wt.w[r], x); y = fmaf(e[r + 1], wt.w[r + 1], y); }
        if constexpr (TARGETS) return __builtin_amdgcn_ldexpf(x + y, wt.exp);
        else return x + y;
    };
    // of tiles s and s + 1, if there is one (their columns' halves are in the two halves of the wavefront)
    auto store_columns = [&](float *cpw, int s, float x, float x1) {
        const float y = halves_sum(x, x1);
        if (lane < (s + 1 < NTW ? 64 : 32) && s + (lane >> 5) < cnt) cpw[32 * s + lane] = y;   // (tiles that are not there: zeros stay)
    };
    auto add_columns = [&](float *cpw, const Weights &wt) {   // of a fragment
        if constexpr (STORE_E) {
#pragma unroll
            for (int s = 0; s < NTW; s += 2) {
                const float x = column_of(E[s], wt);
                store_columns(cpw, s, x, s + 1 < NTW ? column_of(E[s + 1 < NTW ? s + 1 : s], wt) : x);
            }
        }
    };
    // the segment's last block: every thread has added its share of what the dustbin gets (wsw: its weights have been read)
    auto sum_dustbin = [&]() {
        if (!DUST) return;
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) {
            if constexpr (!CHAIN) to_row += __shfl_xor(to_row, s);
            to_col += __shfl_xor(to_col, s);
        }
        if (lane == 0) {
            if constexpr (!CHAIN) wsw[0] = to_row;
            wsw[1] = to_col;
        }
    };
    // (a chain's: as words behind the columns')
    auto dust_words = [&](int st) { return p.words + 2 * p.wbuf + ((long)(st & 1) * p.np + n) * (2 * p.nseg); };
    auto store_dustbin = [&](int st) {
        if (!DUST || tid >= 2) return;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NF * G; ++i) s += CHAIN && tid == 0 ? dust_row[i] : reinterpret_cast<const float *>(smem + LD::WS)[32 * i + tid];
        if (CHAIN && st + 1 < p.nsteps)
            __hip_atomic_store(dust_words(st) + tid * p.nseg + seg, (unsigned long long)(st + 1) << 32 | __float_as_uint(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else dust[tid * p.nseg + seg] = s;
    };
    // column sums of the block's fragments at column i of its window
    auto over_fragments = [&](const float *cp, int i, float s) {
        float x[NF];
        if constexpr (LD::PADDED) {
#pragma unroll
            for (int q = 0; q < NF; ++q) x[q] = cp[q * cps + i];
#pragma unroll
            for (int q = 0; q < NF; ++q) s += x[q];
        } else {
            const int wt = i >> 5;
#pragma unroll
            for (int q = 0; q < NF; ++q) x[q] = cp[q * cps + min(max(wt - q, 0), NT - 1) * 32 + (i & 31)];
#pragma unroll
            for (int q = 0; q < NF; ++q) s += (unsigned)(wt - q) < (unsigned)NT ? x[q] : 0.f;
        }
        return s;
    };
    constexpr int NPOS = (32 * ((TIGHT ? 1 : 2) * NF + G * NTW) + NTHR - 1) / NTHR;   // ring positions of a thread, always the same ones
    [[maybe_unused]] float acc[NPOS];   // MARCH: the segment's column sums there so far
    // a block's column sums onto the segment's; tiles that no later block of the segment meets are done (at: ring slot of its
    // first tile)
    auto add_to_segment = [&](const float *cp, int b, int at) {
#pragma unroll
        for (int k = 0; k < NPOS; ++k) {
            const int i = tid + k * NTHR;
            int wt = (i >> 5) - at;
            if (wt < 0) wt += RS;
            if (i >= 32 * RS || wt >= nwt) continue;
            const float s = over_fragments(cp, 32 * wt + (i & 31), b == b0 || wt >= nwt - NF ? 0.f : acc[k]);
            if (b + 1 == bv || wt < NF) po[32 * (b * NF - hw + wt - kseg) + (i & 31)] = s;
            acc[k] = s;
        }
    };
    float rsum[16];

    for (int b = b0, st = 0; MARCH ? b < bv : CHAIN || st == 0; MARCH ? ++b : ++st) {
        // what depends on the lane alone is computed again in every block: kept across the loop it would take the
        // registers that the plan entries need
        if constexpr (MARCH || CHAIN) asm volatile("" : "+v"(tid));
        lane = tid & 63;
        const int par = LD::TWO == 2 ? (b - b0) & 1 : 0, o = (b * NF + f) * 32 + (lane & 31);
        const bool more = MARCH && b + 1 < bv;
        Added next{};
        if (more) {
            next = request(b);
            if constexpr (!TIGHT) request_tiles(b);
        }
        if constexpr (CHAIN) to_col = 0.f;
        const Row row = row_of(b, par);
        evaluate(b, par, row.u, rsum, [&]() {
            if (MARCH && b > b0) add_to_segment(cp0 + (LD::TWO == 2 ? par ^ 1 : 0) * NF * cps, b - 1, base >= NF ? base - NF : base - NF + RS);
        }, st == 0, false, [](int, const f32x16 &) {});
        if (more) xf.load(reinterpret_cast<const T *>(Xb), min(((b + 1) * NF + f) * 32 + (lane & 31), Le - 1), Le, lane >> 5);
        write_row_sums(rsum, rs);
        if (KIND == STEP_MARCH && more) stage_added_v(next, b);   // (slots of their own)
        if constexpr (G > 1) __syncthreads();
        else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if constexpr (TIGHT)
            if (more) request_tiles(b);   // (every wavefront is done with this block's)
        const Weights wt = weights(b, row, rs);
        float *cp = cp0 + par * NF * cps;
        add_columns(cp + cp_own + j0 * 32, wt);
        if constexpr (!STORE_E) {
            float before = 0.f;
            evaluate(b, par, row.u, rsum, []() {}, false, true, [&](int s, const f32x16 &e) {
                const float x = column_of(e, wt);
                if (s & 1) store_columns(cp + cp_own + j0 * 32, s - 1, before, x);
                else if (s == NTW - 1) store_columns(cp + cp_own + j0 * 32, s, x, x);
                before = x;
            });
        }
        if (TIGHT && more) stage_added_v(next, b);
        if (more) stage_added_u(next, b, LD::TWO == 2 ? par ^ 1 : 0);
        else sum_dustbin();
        __builtin_amdgcn_s_waitcnt(0x0070);   // the next block's tiles
        __syncthreads();
        // rows' stores only now: the wait above would wait for them as well
        const int to = CHAIN ? slot_of(st) : 0;
        if (lane < 32 && g == 0 && o < L && to >= 0) (CHAIN ? slots + (long)to * p.Lp : u_out)[o] = wt.u_new;
        if (!more) store_dustbin(st);
        if constexpr (!MARCH) {
            float sum[NWIN];
#pragma unroll
            for (int k = 0; k < NWIN; ++k) sum[k] = over_fragments(cp, min(tid + k * NTHR, 32 * nwt - 1), 0.f);
            if (!CHAIN || st + 1 == p.nsteps) {
#pragma unroll
                for (int k = 0; k < NWIN; ++k)
                    if (tid + k * NTHR < 32 * nwt) po[tid + k * NTHR] = sum[k];
                return;
            }
            const unsigned tag = st + 1;
            unsigned long long *words = p.words + (st & 1) * p.wbuf + n * p.wstride;
#pragma unroll
            for (int k = 0; k < NWIN; ++k)
                if (tid + k * NTHR < 32 * nwt)
                    __hip_atomic_store(words + (long)seg * (32 * nwt) + tid + k * NTHR, (unsigned long long)tag << 32 | __float_as_uint(sum[k]),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane < 32 && g == 0) stage_u(32 * f + lane, o < Le ? wt.u_new : -INFINITY, row.la);
            unsigned polls = 0;
            // whether to give up waiting
            auto enough = [&]() {
                if (++polls < p.limit && ((polls & 63) || !__hip_atomic_load(&p.chain->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) return false;
                gave_up = 1;
                return true;
            };
            for (;;) {
                unsigned long long w[NWIN][NSUM];
                int cn[NWIN];
#pragma unroll
                for (int k = 0; k < NWIN; ++k) {
                    const ColumnSegments cg(p, cut, min(max(32 * kseg + min(tid + k * NTHR, 32 * nwt - 1), 0), L - 1), nseg_valid);
                    cn[k] = cg.n;
#pragma unroll
                    for (int i = 0; i < NSUM; ++i)
                        w[k][i] = __hip_atomic_load(words + cg.at(i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                bool ok = true;
#pragma unroll
                for (int k = 0; k < NWIN; ++k) {
                    sum[k] = 0.f;
#pragma unroll
                    for (int i = 0; i < NSUM; ++i) {
                        ok = ok && (unsigned)(w[k][i] >> 32) == tag;
                        sum[k] += i < cn[k] ? __uint_as_float((unsigned)w[k][i]) : 0.f;
                    }
                }
                if (__all(ok)) break;
                if (enough()) break;
            }
            if (DUST) {
                const unsigned long long *q = dust_words(st);
                float r = 0.f, c = 0.f;
                for (int i = tid; i < p.nseg; i += NTHR) {
                    unsigned long long a, b;
                    do {
                        a = __hip_atomic_load(q + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        b = __hip_atomic_load(q + p.nseg + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    } while (((unsigned)(a >> 32) != tag || (unsigned)(b >> 32) != tag) && !enough());
                    r += __uint_as_float((unsigned)a); c += __uint_as_float((unsigned)b);
                }
                const DustbinPair d = dustbin_from<NTHR>(r, c, uL, vL, spr ? spr[L] : p.sdb, rs);
                uL = uniform(d.u); vL = uniform(d.v);
                to_row = 0.f;
                if (seg == 0 && tid == 0) {
                    if (to >= 0) { slots[(long)to * p.Lp + L] = uL; slots[(long)(to + 1) * p.Lp + L] = vL; }
                    dust[2 * p.nseg] = uL; dust[2 * p.nseg + 1] = vL;   // (the last step's is what the launch after this one reads)
                }
            }
            // (the scores of the spokes are read again: kept over the evaluation they cost a workgroup per CU)
            float spoke_c[NWIN];
#pragma unroll
            for (int k = 0; k < NWIN; ++k) spoke_c[k] = DUST && spc ? spc[min(max(32 * kseg + tid + k * NTHR, 0), L - 1)] : p.sdb;
            const int own_end = b + 1 == nseg_valid ? max(bv * BM, Lc) : bv * BM;
#pragma unroll
            for (int k = 0; k < NWIN; ++k) {
                const int i = tid + k * NTHR, t = 32 * kseg + i;
                if (i >= 32 * nwt) continue;
                if (DUST) sum[k] += fast_exp2((spoke_c[k] + uL + win_v[k]) * LOG2E);
                win_v[k] = t < Lc ? column_update<true>(win_v[k], sum[k], ColumnTarget(TARGETS ? win_lb[k] : 0.f)) : 0.f;
                if (DUST && t >= b0 * BM && t < min(bv * BM, L)) to_row += fast_exp2((spoke_c[k] + win_v[k] + uL) * LOG2E);
                if (to >= 0 && t >= b0 * BM && t < min(own_end, L)) slots[(long)(to + 1) * p.Lp + t] = win_v[k];
                stage_v(i, t, win_v[k], win_lb[k]);
            }
            if (DUST) sum_row();
            __syncthreads();
            if (gave_up) {
                if (tid == 0) __hip_atomic_store(&p.chain->failed, CHAIN_GAVE_UP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
            continue;
        }
        if (!more) add_to_segment(cp, b, base);
        base += NF;
        if (base >= RS) base -= RS;
    }
}

}  // namespace
