// Block shapes of the step kernel (ska_step.h): which instances there are, what they take of LDS, which one a call takes.
// Plain C++ but for __host__ and __device__.
#pragma once

namespace {

template <typename T, int D> struct StepTile {
    static constexpr int ROWB = D * (int)sizeof(T), CPR = ROWB / 16, BYTES = 32 * ROWB;
    // position of a 16-byte chunk in its row: sixteen consecutive rows spread one chunk over all 64 banks
    static __host__ __device__ int swz(int row) { return CPR >= 16 ? (row & 15) : CPR == 8 ? ((row >> 1) & 7) : ((row >> 2) & 3); }
};
// How a workgroup goes over its rows: one block; a segment of blocks on a ring of tiles, the next block's requested at a
// block's start; the same on a ring that holds one block's window and no more (LDS): requested once a block's
// products are done, into the slots that it leaves.  (8 KB tiles: a forward of eight problems of L = 16384, d = 128,
// W = 256 1300 us block by block, 867 so, 1115 by half-steps.  Streams of tiles of each wavefront's own, which need no
// window, expose a tile's latency in every product: 1017, and 3358 -> 5301 at L = 262144, d = 64, W = 1024.)
// STEP_CHAIN: single blocks, several steps in one launch (not a choice of step_shape: the launch says so).
enum StepKind { STEP_BLOCK, STEP_MARCH, STEP_TIGHT, STEP_CHAIN };
// What a call's steps add to the plain ones: nothing, a dustbin, a dustbin if the arguments say so, targets of rows or columns
// (which go with no dustbin; a cut or none), segments cut from valid rows.
// STEP_KEEP: plain ones of a chain in fp32 storage.
enum StepForm { STEP_PLAIN, STEP_DUSTBIN, STEP_ANY, STEP_TARGETS, STEP_CUT, STEP_KEEP };
template <typename T, int D, int NF, int G, int NTW, int KIND, int FORM> struct StepLds {   // offsets in bytes
    static constexpr bool MARCH = KIND == STEP_MARCH || KIND == STEP_TIGHT;
    static_assert(KIND != STEP_TIGHT || G > 1, "the exchange of row sums says that the products are done");
    // With G > 1 that exchange lies between a wavefront's reads and its next block's writes; without it there are two buffers.
    static constexpr int TWO = MARCH && G == 1 ? 2 : 1;
    static constexpr int RSUM = 0;                              // [NF][G][32] row sums
    static constexpr int WS = RSUM + NF * G * 128;                // [wave][32] weights of the rows
    static constexpr int US = WS + NF * G * 128;                // [TWO][32 NF] potentials of the rows
    static constexpr int UE = US + TWO * NF * 128;              // fp32 storage: the same as the evaluation takes them
    static constexpr int CP = UE + (sizeof(T) == 4 ? TWO * NF * 128 : 0);
    static constexpr int VB = sizeof(T) == 2 || FORM == STEP_TARGETS ? 8 : 4;   // bytes of a column's potential (and weight)
    // Column sums of a fragment by column of the block's window, with zeros where its band does not reach; of a single launched block by
    // tile of the band, which is less (d = 128, W = 32: three workgroups fit a CU instead of two).
    static constexpr bool PADDED = KIND != STEP_BLOCK;
    int cp, cps, y, rs, vs, total;   // cp: [TWO][NF][cps] column sums of a fragment; y: ring of the other side's tiles
    __host__ __device__ StepLds(int hw)
    {
        rs = NF + 2 * hw + (KIND == STEP_MARCH ? NF : 0);   // ring slots: the window of a block (and the tiles the next one adds)
        cp = CP;
        cps = 32 * (G * NTW + (PADDED ? NF - 1 : 0));   // (the window, and tiles that the last fragment's wavefronts are short of)
        y = cp + TWO * NF * cps * 4;
        vs = y + rs * StepTile<T, D>::BYTES;   // [32 rs] potentials of the columns, base 2 (bf16 storage: an operand row each)
        total = vs + rs * 32 * VB;
    }
    // Ring slot of the tile `at` slots on from the ring's first.  A wavefront evaluates NTW tiles also where its band ends before:
    // of a single block, whose ring is its window, it takes the last slot for those (their entries are masked).
    __host__ __device__ int slot(int at) const { return MARCH ? (at >= rs ? at - rs : at) : (at < rs ? at : rs - 1); }
};

// Blocks of NF fragments of 32 rows, G wavefronts per fragment with NTW tiles each, M blocks per workgroup (a segment);
// hw = ceil(W / 32).  NF = 0: the half-steps run one by one.
struct StepShape { int NF, G, NTW, hw, M, kind; };
constexpr int STEP_LDS = 159 * 1024;
// The instances, by the bytes of a 32-row tile (TB).
#define SKA_STEP_SHAPES(X) \
    X(TB <= 16384, 2, 2, 2, STEP_BLOCK) X(TB <= 16384, 2, 2, 3, STEP_BLOCK) X(TB <= 8192, 2, 2, 4, STEP_BLOCK) X(TB <= 8192, 2, 2, 5, STEP_BLOCK) \
    X(TB <= 16384, 4, 1, 3, STEP_BLOCK) X(TB <= 16384, 4, 1, 5, STEP_BLOCK) X(TB == 8192, 4, 1, 7, STEP_BLOCK) X(TB == 8192, 4, 1, 9, STEP_BLOCK) \
    X(TB == 16384, 1, 2, 5, STEP_BLOCK) X(TB == 8192 && sizeof(T) == 4, 1, 4, 5, STEP_BLOCK) \
    X(TB <= 8192, 8, 1, 7, STEP_BLOCK) X(TB <= 8192, 8, 1, 9, STEP_BLOCK) X(TB <= 4096, 8, 1, 7, STEP_MARCH) X(TB <= 4096, 8, 1, 9, STEP_MARCH) \
    X(TB <= 8192, 2, 4, 3, STEP_BLOCK) X(TB <= 8192, 2, 4, 4, STEP_BLOCK) X(TB <= 8192, 2, 4, 5, STEP_BLOCK) X(TB <= 4096, 2, 4, 9, STEP_BLOCK) \
    X(TB == 8192, 2, 4, 3, STEP_TIGHT) X(TB == 8192, 2, 4, 4, STEP_TIGHT) X(TB == 8192, 2, 4, 5, STEP_TIGHT) \
    X(TB <= 4096, 4, 2, 6, STEP_MARCH) X(TB <= 4096, 4, 2, 7, STEP_MARCH) X(TB <= 4096, 4, 2, 8, STEP_MARCH) X(TB <= 4096, 4, 2, 9, STEP_MARCH) \
    X(TB <= 4096, 4, 2, 9, STEP_BLOCK) X(TB <= 4096, 4, 2, 7, STEP_BLOCK) X(TB <= 4096, 4, 2, 8, STEP_BLOCK)
template <typename T, int D> constexpr int step_tile_bytes = StepTile<T, D>::BYTES;
template <typename T, int D> int step_lds(const StepShape &sh)   // bytes (of the form that takes most); -1: no such instance
{
    constexpr int TB = step_tile_bytes<T, D>;
#define SKA_LDS(COND, NF_, G_, NTW_, KIND_) \
    if constexpr (COND) \
        if (sh.NF == NF_ && sh.G == G_ && sh.NTW == NTW_ && sh.kind == KIND_) return StepLds<T, D, NF_, G_, NTW_, KIND_, STEP_TARGETS>(sh.hw).total;
    SKA_STEP_SHAPES(SKA_LDS)
#undef SKA_LDS
    return -1;
}
// Which shape a call takes, from the rows of the whole call (not of a launch: results do not depend on how a call is cut).
// Short blocks while they leave CUs idle or barely fill them, large ones (less of the band read twice) beyond, one segment per
// CU where two buffers of tiles fit LDS.  Forward of T = 16, R = 2 steps, us, at the sizes next to each line, by a launch per step
// (chains take the shape that launches take, since a call's bits are the same either way):
//   bf16, d = 64, W = 64:  48000 rows (2,2,3) 155 (4,1,5) 159; 65536 rows 175 / 163; half-steps 255 / 253
//   W = 128: 48000 rows (2,2,5) 196 (8,1,9) 203, 65536 rows 262 / 203; 131072 rows (8,1,9) one block 364, segments 340
//   W = 200: 5600 rows (2,4,5) 176 (4,2,9) 206; 48000 rows 408 / 336 in segments; 524288 rows 1803, half-steps 1804
//   d = 32, W = 256: 131072 rows 464, half-steps 574; 262144 rows 805 / 742, as d = 32 half-steps have half the products
//   d = 128 or fp32 d = 64 (8 KB tiles), W = 128: 5600 rows (2,2,5) 195 (4,1,9) 222; 32768 rows (4,1,9) 229 (8,1,9) 247;
//   131072 rows (4,1,9) 702 (8,1,9) 539, half-steps 826.  W = 256 (2,4,5): 5600 rows 236, half-steps 481; 32768 rows block by
//   block 401, in segments 481, half-steps 481; 131072 rows 1321 / 916 / 1115; 262144 rows 2502 / 1625 / 1786.  fp32: 131072
//   rows 2701 / 2253 / 3181; 5600 rows (1,4,5) 381 (2,4,5) 436
//   fp32 d = 128 (16 KB tiles): W = 32 32768 rows (2,2,3) 393 (4,1,5) 329; W = 128 5600 rows 539, half-steps 989; 32768 rows
//   1532 / 995
//   NTW is the least that the band's tiles need up to W = 256 (absent ones cost as much as others): d = 64, W = 32: 262144 rows (4,1,5) 413
//   (4,1,3) 333; W = 96: (8,1,9) 576 (8,1,7) 507; W = 160: (4,2,9) 974 (4,2,6) 738, half-steps 974; W = 192: 933, (4,2,7) 794, 888;
//   W = 224: (4,2,9) 917 (4,2,8) 853; 16384 rows, W = 160: (2,4,5) 168 (2,4,3) 146; 32768 rows (2,4,3) 177 (4,2,7) 185, W = 192:
//   (2,4,4) 266 (4,2,7) 190.  d = 128, W = 160: 131072 rows (2,4,5) 850 (2,4,3) 715.  fp32 d = 64, 8000 rows, W = 160: (1,4,5) 324
//   (2,4,3) 311, W = 192: 343, (2,4,4) 372.  d = 32, W = 160: 262144 rows (4,2,6) 620, 524288 rows 1137, half-steps 656 / 935
//   W = 300 .. 480 (2,4,9): 16384 rows 244 .. 271, half-steps 469 .. 618; 32768 rows 414 .. 456 / 470 .. 619; beyond, the 36
//   tiles that a block of 64 rows reads are what bounds it
template <typename T, int D> StepShape step_choice(int N, int L, int W)
{
    constexpr int TB = step_tile_bytes<T, D>;
    const int hw = ((W < L ? W : L) + 31) / 32;
    const long rows = (long)N * L;
    StepShape sh{0, 0, 0, hw, 1, STEP_BLOCK};
    auto take = [&](int NF, int G, int NTW) { sh.NF = NF; sh.G = G; sh.NTW = NTW; };
    bool march = false;
    if (hw <= 2) {
        if (rows <= (TB <= 4096 ? 49152 : TB == 8192 ? 32768 : 16384)) take(2, 2, hw < 2 ? 2 : 3);
        else take(4, 1, hw < 2 ? 3 : 5);
    } else if (hw <= 4) {
        if (TB == 16384) {
            if (rows <= 8192) take(1, 2, 5);
        } else if (rows <= (TB <= 4096 ? 49152 : 16384)) {
            take(2, 2, hw + 1);
        } else if (TB == 8192 && rows <= 32768) {
            take(4, 1, 2 * hw + 1);
        } else {
            take(8, 1, 2 * hw + 1);
            march = TB <= 4096;
        }
    } else if (hw <= 8) {
        const int ntw = hw == 5 ? 3 : hw <= 7 ? 4 : 5;   // of four wavefronts
        if (TB <= 4096) {
            if (rows <= (hw == 5 ? 32768 : 16384)) {
                take(2, 4, ntw);
            } else if (TB == 4096 || rows <= 196608) {
                take(4, 2, hw + 1);
                march = true;
            }
        } else if (TB == 8192) {
            if (sizeof(T) == 4 && hw > 5 && rows <= 8192) take(1, 4, 5);
            else take(2, 4, ntw);
            march = rows > 32768;
        }
    } else if (hw <= 15 && TB <= 4096 && rows <= 32768) {
        take(2, 4, 9);
    }
    if (!sh.NF) return sh;
    if (march) {   // one segment per CU, of equal lengths and at least hw tiles
        const int nblk = (L + 32 * sh.NF - 1) / (32 * sh.NF);
        const long per = 256 / N > 1 ? 256 / N : 1;   // segments per problem
        int M = (int)((nblk + per - 1) / per);
        if (M > 4096 / sh.NF) M = 4096 / sh.NF;   // (segment_reciprocal)
        if (M > 1 && M * sh.NF < hw) M = (hw + sh.NF - 1) / sh.NF;
        sh.M = M;
        if (M > 1) sh.kind = TB <= 4096 ? STEP_MARCH : STEP_TIGHT;
    }
    return sh;
}
// Every choice has an instance that fits LDS (a test goes over them).  (4,2,6) needs none for single blocks: beyond 32768 rows
// there are more blocks of 128 than segments, so that a segment has at least two.
template <typename T, int D> StepShape step_shape(int N, int L, int W)
{
    StepShape sh = step_choice<T, D>(N, L, W);
    const int lds = sh.NF ? step_lds<T, D>(sh) : 0;
    if (lds < 0 || lds > STEP_LDS) sh.NF = 0;
    return sh;
}
inline long step_segments(const StepShape &sh, int L) { return (L + 32L * sh.NF * sh.M - 1) / (32L * sh.NF * sh.M); }
inline int step_least(const StepShape &sh) { return sh.hw > sh.NF ? (sh.hw + sh.NF - 1) / sh.NF : 1; }   // blocks of a segment, at least
// floats of column sums per problem; cut: segments of any length from step_least to M blocks
inline long step_part_stride(const StepShape &sh, int L, bool dustbin, bool cut)
{
    const long nseg = step_segments(sh, L);
    if (cut) {   // (blocks / m + 1) (NF m + 2 hw) tiles with m blocks each: convex in m
        const long nblk = (L + 32L * sh.NF - 1) / (32L * sh.NF), least = step_least(sh);
        const long a = sh.NF * least + 2 * sh.hw * (nblk / least + 1), b = sh.NF * sh.M + 2 * sh.hw * (nblk / sh.M + 1);
        return 32 * (sh.NF * nblk + 2 * sh.hw + (a > b ? a : b));
    }
    return nseg * 32 * (sh.NF * sh.M + 2 * sh.hw) + (dustbin ? 2 * nseg + 2 : 0);
}

}  // namespace
