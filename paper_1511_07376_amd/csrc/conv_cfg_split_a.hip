// Instantiations of the split convolution kernel for configurations 16 and 17.
#include "conv_split_kernel.h"

namespace cnn {
namespace conv {

CNN_SPLIT_DEFINE(16, 2, 2, 2, 2, 16)
CNN_SPLIT_DEFINE(17, 4, 1, 1, 2, 16)

}  // namespace conv
}  // namespace cnn
