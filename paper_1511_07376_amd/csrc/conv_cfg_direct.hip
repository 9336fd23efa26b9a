// The direct convolution kernels (configurations 22 to 24).
#include "conv_direct_kernel.h"

namespace cnn {
namespace conv {
namespace {

template <int FM, int FN, int KW>
int launch_direct(const ConvParams& prm, bool vec_w, hipStream_t st) {
    const dim3 grid(ceil_div(prm.M, FN * 32), ceil_div(prm.Kg, FM * 32), prm.G * prm.splits), block(64 * KW);
    const int window = direct_window(prm);
    const size_t shm = (size_t)direct_table_entries(prm.kchunk, KW) * 4 * (window == kWindowAny ? 2 : 1);
    if (shm > kDirectTableBytes) return fail(CNN_ERR_UNSUPPORTED, "conv: tap table of %zu bytes", shm);
#define GO(V, M) enqueue((conv2d_direct_f32<FM, FN, KW, V, M>), grid, block, shm, st, prm)
    if (vec_w) {
        if (window == kWindowNoPad) GO(true, kWindowNoPad);
        else if (window == kWindowMask) GO(true, kWindowMask);
        else GO(true, kWindowAny);
    } else {
        if (window == kWindowNoPad) GO(false, kWindowNoPad);
        else if (window == kWindowMask) GO(false, kWindowMask);
        else GO(false, kWindowAny);
    }
#undef GO
    return check_launch("conv2d_direct_f32");
}

}  // namespace

#define CNN_DIRECT_DEFINE(I, FM, FN, KW) \
    int launch_c##I(const ConvParams& prm, bool vec_w, hipStream_t st) { return launch_direct<FM, FN, KW>(prm, vec_w, st); }
CNN_DIRECT_CONFIGS(CNN_DIRECT_DEFINE)

}  // namespace conv
}  // namespace cnn
