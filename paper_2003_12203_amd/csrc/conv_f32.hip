// The convolution kernel: its fp32 tiles.
#include "conv_launch.h"

namespace ftcnn {
namespace convk {

FTCNN_CONV_TILE(F32_M32)
FTCNN_CONV_TILE(F32_M64)
FTCNN_CONV_TILE(F32_64x256)
FTCNN_CONV_TILE(F32_M96)
FTCNN_CONV_TILE(F32_128x128)
FTCNN_CONV_TILE(F32_128x64)
FTCNN_CONV_TILE(F32_64x64)

}  // namespace convk
}  // namespace ftcnn
