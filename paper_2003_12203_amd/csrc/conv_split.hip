// The convolution kernel: its fp32 tiles on split copies.
#include "conv_launch.h"

namespace ftcnn {
namespace convk {

FTCNN_CONV_TILE(S3_128x256)
FTCNN_CONV_TILE(S3_128x128)
FTCNN_CONV_TILE(S3_64x64)
FTCNN_CONV_TILE(S3_64x128)
FTCNN_CONV_TILE(S3_32x128)
FTCNN_CONV_TILE(S3W_64x128)
FTCNN_CONV_TILE(S3W_128x128)

}  // namespace convk
}  // namespace ftcnn
