// Scales that bring the FP32 network's operands into FP16's range
// (qnet_split.hip).  Host only.
#pragma once
#include <vector>

namespace bcts {

// Per layer conv1..fc1, powers of two unless said otherwise: of its rows of
// weights, of its weights on each input channel (conv1: all 256 of a row), of
// its accumulators on the way out (conv1: times 1/255), and its biases as the
// outputs are scaled.
struct SplitScales {
  std::vector<float> row[4], col[4], out[4], bias[4];
};

// W[4]: [N][K] with the input channel innermost (weight k of a row is on
// channel k % 32 in conv2, k % 64 in conv3 and fc1; conv1 reads pixels), B[4]:
// [N].  False where the split form would hold fewer bits than FP32 needs: the
// FP32 instruction runs then.
bool split_scales(const std::vector<float>* W, const std::vector<float>* B, SplitScales* sp);

}  // namespace bcts
