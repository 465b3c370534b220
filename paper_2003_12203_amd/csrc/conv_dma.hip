// The convolution kernel: its direct-to-LDS bf16 tiles.
#include "conv_launch.h"

namespace ftcnn {
namespace convk {

FTCNN_CONV_TILE(BF16_DMA_128x128)
FTCNN_CONV_TILE(BF16_DMA_128x128_3)
FTCNN_CONV_TILE(BF16_DMA_64x64_3)
FTCNN_CONV_TILE(BF16_DMA_64x128)
FTCNN_CONV_TILE(BF16_DMA_256x256)
FTCNN_CONV_TILE(BF16W_64x128)
FTCNN_CONV_TILE(BF16W_128x128)

}  // namespace convk
}  // namespace ftcnn
