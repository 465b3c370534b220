// The convolution kernel: its register-staged bf16 tiles.
#include "conv_launch.h"

namespace ftcnn {
namespace convk {

FTCNN_CONV_TILE(BF16_M32)
FTCNN_CONV_TILE(BF16_M64)
FTCNN_CONV_TILE(BF16_128x128_K64)
FTCNN_CONV_TILE(BF16_256x256)

}  // namespace convk
}  // namespace ftcnn
