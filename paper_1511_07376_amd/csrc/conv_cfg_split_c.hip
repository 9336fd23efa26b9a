// Instantiations of the split convolution kernel for configurations 20 and 21.
#include "conv_split_kernel.h"

namespace cnn {
namespace conv {

CNN_SPLIT_DEFINE(20, 2, 2, 1, 1, 16)
CNN_SPLIT_DEFINE(21, 2, 2, 1, 1, 32)

}  // namespace conv
}  // namespace cnn
