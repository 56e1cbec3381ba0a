// Internal: two 3 x 3 convolutions, the second of the first one's output, in one launch (basic_block.hip).
#pragma once
#include "fupr.h"
#include "layout.h"

namespace fupr {

struct BasicBlockArgs {
  fupr_dtype dt;
  fupr_conv_shape s1, s2;
  int H, W;              // input of the first
  bool add;              // the second adds a shortcut
};

// Shapes alone: the kernel can run these operators (at any batch size that basic_block_wanted takes).
bool basic_block_applies(const BasicBlockArgs& a);
// ... and is the faster way to at N images.
bool basic_block_wanted(const BasicBlockArgs& a, int N);
const char* basic_block_name(const BasicBlockArgs& a, int N);
// `count` images of a batch of N; the two convolutions' arguments as they would run by themselves (the
// tensor between them is neither read nor written).
fupr_status launch_basic_block(const BasicBlockArgs& a, const ConvArgs& first, const ConvArgs& second, int N, int count,
                               void* stream);

}  // namespace fupr
