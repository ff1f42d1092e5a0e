// C entry point around the scales of the FP32 network's split form, for
// tests/test_split_scales.py (built together with csrc/split_scales.cpp).
// w: conv1..fc1 in the order split_scales reads them, one after another, b
// their biases; row, out and bias are laid out like b, col holds 256 + 32 + 64 + 64.
#include <algorithm>

#include "../../paper_2107_01715_amd/csrc/split_scales.h"

extern "C" int shim_split_scales(const float* w, const float* b, float* row, float* col, float* out, float* bias) {
  static const int NK[4][2] = {{32, 256}, {64, 512}, {64, 576}, {512, 3136}};
  std::vector<float> W[4], B[4];
  for (int l = 0; l < 4; ++l) {
    W[l].assign(w, w + NK[l][0] * NK[l][1]);
    B[l].assign(b, b + NK[l][0]);
    w += W[l].size();
    b += B[l].size();
  }
  bcts::SplitScales sp;
  if (!bcts::split_scales(W, B, &sp)) return 0;
  for (int l = 0; l < 4; ++l) {
    row = std::copy(sp.row[l].begin(), sp.row[l].end(), row);
    col = std::copy(sp.col[l].begin(), sp.col[l].end(), col);
    out = std::copy(sp.out[l].begin(), sp.out[l].end(), out);
    bias = std::copy(sp.bias[l].begin(), sp.bias[l].end(), bias);
  }
  return 1;
}
