// The step kernel's instances for one storage type and head dimension (SKA_T, SKA_D; the function's name: SKA_NAME).
#include "sinkhorn_attn.h"
#include "ska_step.h"
#include "ska_step_launch.h"

namespace {

template <typename T, int D, int NF, int G, int NTW, int KIND, int FORM> int launch_vstep_n(StepArgs p, int N, hipStream_t st, int dev)
{
    p.nb_total = p.cut ? (N < p.items * p.nh ? CUT_HALF : CUT_SEGS) : p.nseg * N;
    const int lds = StepLds<T, D, NF, G, NTW, KIND, FORM>(p.hw).total;
    static bool raised[MAX_DEVICES];
    if (!raised[dev]) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(&vstep_kernel<T, D, NF, G, NTW, KIND, FORM>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, STEP_LDS) != hipSuccess)
            return SKA_EHIP;
        raised[dev] = true;
    }
    if constexpr (KIND == STEP_CHAIN) {   // a chain's workgroups wait for each other: they must fit the device together
        static int caps[MAX_DEVICES], caps_lds[MAX_DEVICES];   // what it holds, at which LDS size (0: not asked yet; g_mutex held)
        if (caps_lds[dev] != lds) {
            int per_cu = 0, cus = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(&vstep_kernel<T, D, NF, G, NTW, KIND, FORM>),
                                                             64 * NF * G, lds) != hipSuccess ||
                hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
                return SKA_EHIP;
            caps[dev] = per_cu * cus;
            caps_lds[dev] = lds;
        }
        if ((p.nb_total + 7) / 8 * 8 > caps[dev]) return SKA_EUNSUPPORTED;   // (nothing has been launched)
        // with a dustbin every step waits for the slowest block of its problem (bounded by all problems' blocks, as measured): forward of 4 problems of L = 6000, W = 64 (376 blocks) 164 us by launches,
        // 133 as a chain; 8 of 4000, W = 128 (504) 201 / 173; 8 of 5000 (632) 200 / 208
        if (p.dustbin && p.nb_total > 512) return SKA_EUNSUPPORTED;
    }
    hipLaunchKernelGGL((vstep_kernel<T, D, NF, G, NTW, KIND, FORM>), dim3((p.nb_total + 7) / 8 * 8), dim3(64 * NF * G), lds, st, p);
    return hipGetLastError() == hipSuccess ? SKA_OK : SKA_EHIP;
}
template <typename T, int D> int launch_vstep(const StepArgs &p, const StepShape &sh, int N, hipStream_t st, int dev)
{
    constexpr int TB = step_tile_bytes<T, D>;
#define SKA_LAUNCH(COND, NF_, G_, NTW_, KIND_) \
    if constexpr (COND) \
        if (sh.NF == NF_ && sh.G == G_ && sh.NTW == NTW_ && sh.kind == KIND_) { \
            constexpr bool ANY = KIND_ == STEP_BLOCK; \
            if constexpr (ANY) { \
                if (p.nsteps > 1) { \
                    if (p.log_a || p.log_b) return launch_vstep_n<T, D, NF_, G_, NTW_, STEP_CHAIN, STEP_TARGETS>(p, N, st, dev); \
                    if (p.dustbin) return launch_vstep_n<T, D, NF_, G_, NTW_, STEP_CHAIN, STEP_DUSTBIN>(p, N, st, dev); \
                    if constexpr (sizeof(T) == 4) { /* (more registers: fewer workgroups fit) */ \
                        const int rc = launch_vstep_n<T, D, NF_, G_, NTW_, STEP_CHAIN, STEP_KEEP>(p, N, st, dev); \
                        if (rc != SKA_EUNSUPPORTED) return rc; \
                    } \
                    return launch_vstep_n<T, D, NF_, G_, NTW_, STEP_CHAIN, STEP_PLAIN>(p, N, st, dev); \
                } \
            } \
            if (p.log_a || p.log_b) return launch_vstep_n<T, D, NF_, G_, NTW_, KIND_, STEP_TARGETS>(p, N, st, dev); \
            if constexpr (!ANY) \
                if (p.cut) return launch_vstep_n<T, D, NF_, G_, NTW_, KIND_, STEP_CUT>(p, N, st, dev); \
            if (!ANY && p.dustbin) return launch_vstep_n<T, D, NF_, G_, NTW_, KIND_, ANY ? STEP_ANY : STEP_DUSTBIN>(p, N, st, dev); \
            return launch_vstep_n<T, D, NF_, G_, NTW_, KIND_, ANY ? STEP_ANY : STEP_PLAIN>(p, N, st, dev); \
        }
    SKA_STEP_SHAPES(SKA_LAUNCH)
#undef SKA_LAUNCH
    return SKA_EUNSUPPORTED;
}
}  // namespace

SKA_DECLARE_STEPS(SKA_NAME)
{
    return launch_vstep<SKA_T, SKA_D>(*static_cast<const StepArgs *>(args), *static_cast<const StepShape *>(shape), N, st, dev);
}
