// FFT length classes for FP64 tiles.  2^12 .. 2^13: one kernel per tile, the
// whole length in one workgroup (tile_fused.hpp).  2^14: 128 x 128, workgroup-wide
// Stockham stages (conv_kernels.hpp).  2^15 .. 2^19: n1 = 512; 2^20 .. 2^24: n1 =
// 4096; wave-level transforms (conv_v2.hpp; pass 3 of 2^24 workgroup-wide).
#include "conv_kernels.hpp"
#include "conv_v2.hpp"
#include "tile_fused.hpp"

namespace pa {

#define PA_CLASS(LOGL, N1, N2) \
    {ClassCfg{64, LOGL, N1, N2, 4, 8, 16}, &ClassImpl<double, N1, N2, 4, 8, 16, 16>::pass1, \
     &ClassImpl<double, N1, N2, 4, 8, 16, 16>::pass2, &ClassImpl<double, N1, N2, 4, 8, 16, 16>::pass3}
#define PA_CLASS2(LOGL, N1, N2) \
    {ClassCfg{64, LOGL, N1, N2, ClassImpl2<double, N1, N2>::C1, ClassImpl2<double, N1, N2>::C3, 16, \
              ClassImpl2<double, N1, N2>::kWsExtra, true}, \
     &ClassImpl2<double, N1, N2>::pass1, &ClassImpl2<double, N1, N2>::pass2, &ClassImpl2<double, N1, N2>::pass3}
#define PA_FUSED(LOGL) \
    {ClassCfg{64, LOGL, 1 << LOGL, 1, 1 << LOGL, 1 << LOGL, 16}, &ClassImplF<double, 1 << LOGL>::pass1, \
     &ClassImplF<double, 1 << LOGL>::pass2, &ClassImplF<double, 1 << LOGL>::pass3}

static const ClassKernels kClasses64[] = {
    PA_FUSED(12),
    PA_FUSED(13),
    PA_CLASS(14, 128, 128),
    PA_CLASS2(15, 512, 64),
    PA_CLASS2(16, 512, 128),
    PA_CLASS2(17, 512, 256),
    PA_CLASS2(18, 512, 512),
    PA_CLASS2(19, 512, 1024),
    PA_CLASS2(20, 4096, 256),
    PA_CLASS2(21, 4096, 512),
    PA_CLASS2(22, 4096, 1024),
    PA_CLASS2(23, 4096, 2048),
    // columns of 4096 points: split columns in pass 1, a workgroup-wide Stockham
    // pass 3 with the split exchange
    {ClassCfg{64, 24, 4096, 4096, ClassImplS<double, 4096, 8, 16>::C1, 8, 16, ClassImplS<double, 4096, 8, 16>::kWsExtra,
              true},
     &ClassImplS<double, 4096, 8, 16>::pass1, &ClassImplS<double, 4096, 8, 16>::pass2,
     &ClassImplS<double, 4096, 8, 16>::pass3},
};

const ClassKernels* class_kernels64(int cls) {
    for (const ClassKernels& k : kClasses64)
        if (k.cfg.cls == cls) return &k;
    return nullptr;
}

}  // namespace pa
