// The convolution kernel: its tiles on packed copies.
#include "conv_launch.h"

namespace ftcnn {
namespace convk {

FTCNN_CONV_TILE(S3P_32x128)
FTCNN_CONV_TILE(S3P_64x128)
FTCNN_CONV_TILE(S3P_96x256)
FTCNN_CONV_TILE(S3P_128x128)
FTCNN_CONV_TILE(S3P_64x64)
FTCNN_CONV_TILE(BF16P_64x128)
FTCNN_CONV_TILE(BF16P_64x256)
FTCNN_CONV_TILE(BF16P_128x128)
FTCNN_CONV_TILE(BF16P_64x64)

}  // namespace convk
}  // namespace ftcnn
