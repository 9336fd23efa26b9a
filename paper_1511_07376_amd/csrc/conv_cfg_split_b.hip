// Instantiations of the split convolution kernel for configurations 18 and 19.
#include "conv_split_kernel.h"

namespace cnn {
namespace conv {

CNN_SPLIT_DEFINE(18, 1, 4, 2, 1, 16)
CNN_SPLIT_DEFINE(19, 1, 4, 3, 1, 16)

}  // namespace conv
}  // namespace cnn
