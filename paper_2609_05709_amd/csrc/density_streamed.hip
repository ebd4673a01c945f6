// Host side of the streamed density kernel k_djs (soap_device.h): variants,
// on-chip plan and launch.  Its own translation unit, so that its variants
// compile beside the other kernels.
#include "soap_device.h"

namespace soap {
using namespace dev;

// variants: QT (radial pair, lm) tasks per thread
template <typename T, typename ST>
static const void *djs_kernel_t(int qt) {
    switch (qt) {
    case 1: return (const void *)k_djs<T, ST, 1>;
    case 2: return (const void *)k_djs<T, ST, 2>;
    case 3: return (const void *)k_djs<T, ST, 3>;
    case 4: return (const void *)k_djs<T, ST, 4>;
    default: return nullptr;
    }
}
static const void *djs_kernel(bool f64, bool ar64, int qt) {
    if (f64) return djs_kernel_t<double, double>(qt);
    return ar64 ? djs_kernel_t<float, double>(qt) : djs_kernel_t<float, float>(qt);
}

bool djs_shape(const Params &P, int *qt) {
    const int t = djs_tasks(P);
    *qt = t < 1 ? 1 : t;
    return t <= 4;
}

size_t djs_lds_bytes(const Params &P, int W, bool st64) { return 8 * djs_lds_doubles(P, W, st64 ? 8 : 4); }

int djs_blocks_per_cu(bool f64, bool ar64, int qt, size_t lds) {
    int nb = 0;
    const void *k = djs_kernel(f64, ar64, qt);
    if (!k) return 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, BSC, lds);
    return (e == hipSuccess && nb > 0) ? nb : 0;
}

// dynamic LDS above the default limit for every variant (set_lds_limits)
hipError_t djs_set_lds_limit(int lim) {
    hipError_t e = hipSuccess;
    for (int f64 = 0; f64 < 2; ++f64)
        for (int ar64 = 0; ar64 < 2; ++ar64)
            for (int qt = 1; qt <= 4; ++qt)
                if (e == hipSuccess)
                    e = hipFuncSetAttribute(djs_kernel(f64 != 0, ar64 != 0, qt),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, lim);
    return e;
}

hipError_t launch_djs(const Params &P, const Rows &R, const void *pos, bool f64, bool ar64, const DjsLaunch &cfg,
                      void *c_scratch, hipStream_t st) {
    if (R.nc <= 0) return hipSuccess;
    Params Pk = P;
    Rows Rk = R;
    int W = cfg.W;
    void *args[] = {&Pk, &Rk, &pos, &W, &c_scratch};
    // persistent: as many workgroups as stay resident, each striding over the centers
    const int64_t blocks = std::min<int64_t>(R.nc, (int64_t)cfg.blocks);
    return hipLaunchKernel(djs_kernel(f64, ar64, cfg.qt), dim3((unsigned)blocks), dim3(BSC), args,
                           cfg.lds, st);
}

} // namespace soap
