// Block shapes of the step kernel over sizes and types, on the host: every shape that the rule takes has an instance and fits
// LDS, and every tile that a wavefront reads lies inside the launch's ring.  Prints the first violation and returns 1.
#include "ska_step_shape.h"

#include <cstdio>

namespace {
struct half_word { short x; };   // (of a bf16's size; nothing else of the type is asked)
long shapes = 0, clamped = 0;

// the slots that the kernel's wavefronts go through in a block whose first tile lies in slot `base`
template <typename T, int D, int NF, int G, int NTW, int KIND> bool reads_inside(const StepShape &sh)
{
    const StepLds<T, D, NF, G, NTW, KIND, STEP_TARGETS> lds(sh.hw);   // (the form that takes most)
    const int window = NF + 2 * sh.hw, NT = 2 * sh.hw + 1;
    if (G * NTW < NT || lds.total > STEP_LDS || lds.rs < window) return false;
    for (int base = 0; base < (KIND == STEP_BLOCK ? 1 : lds.rs); ++base)
        for (int f = 0; f < NF; ++f)
            for (int g = 0; g < G; ++g) {
                int slot = lds.slot(base + f + g * NTW);
                for (int s = 0; s < NTW; ++s, slot = lds.slot(slot + 1)) {
                    const int tile = f + g * NTW + s;   // of the block's window
                    const bool present = g * NTW + s < NT;
                    clamped += tile >= window;
                    if (slot < 0 || slot >= lds.rs || (present && slot != (base + tile) % lds.rs)) return false;
                }
            }
    return true;
}
template <typename T, int D> bool check(int N, int L, int W)
{
    const StepShape sh = step_choice<T, D>(N, L, W);
    if (!sh.NF) return true;
    const int lds = step_lds<T, D>(sh);
    constexpr int TB = step_tile_bytes<T, D>;
    bool ok = lds >= 0 && lds <= STEP_LDS && step_shape<T, D>(N, L, W).NF == sh.NF, instance = false;
#define CHECK(COND, NF_, G_, NTW_, KIND_) \
    if constexpr (COND) \
        if (sh.NF == NF_ && sh.G == G_ && sh.NTW == NTW_ && sh.kind == KIND_) instance = reads_inside<T, D, NF_, G_, NTW_, KIND_>(sh);
    SKA_STEP_SHAPES(CHECK)
#undef CHECK
    ++shapes;
    if (ok && instance) return true;
    std::printf("%d-byte d = %d, N = %d, L = %d, W = %d: (%d, %d, %d) kind %d, %d blocks, %d bytes of LDS\n", (int)sizeof(T), D, N, L, W,
                sh.NF, sh.G, sh.NTW, sh.kind, sh.M, lds);
    return false;
}
}  // namespace

int main()
{
    const int Ns[] = {1, 2, 3, 8, 32, 100, 300, 600, 5000}, Ls[] = {1, 31, 33, 100, 300, 500, 700, 1000, 3001, 5000, 9000, 17000, 33000, 50001, 70001, 262144};
    for (int N : Ns)
        for (int L : Ls)
            for (int W = 0; W <= 520; W += W < 40 || W % 32 > 28 || W % 32 < 2 ? 1 : 9)
                if ((long)N * L <= 1L << 22 &&
                    !(check<half_word, 32>(N, L, W) && check<half_word, 64>(N, L, W) && check<half_word, 128>(N, L, W) &&
                      check<float, 32>(N, L, W) && check<float, 64>(N, L, W) && check<float, 128>(N, L, W)))
                    return 1;
    std::printf("%ld shapes, %ld tiles beyond a window\n", shapes, clamped);
    return shapes > 1000 && clamped > 0 ? 0 : 1;
}
