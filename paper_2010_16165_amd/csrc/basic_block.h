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
  bool alone;            // nothing runs before or behind the block
};

// Shapes alone: the kernel can run these operators (at any batch size that basic_block_plan takes).
bool basic_block_applies(const BasicBlockArgs& a);
// The plan for a batch of N images, a number of this kernel's own; -1: the operators run apart.
int basic_block_plan(const BasicBlockArgs& a, int N);
// ... for `count` images of a batch that runs `plan`, which give that batch's bits.
int basic_block_plan_part(const BasicBlockArgs& a, int plan, int count);
const char* basic_block_name(int plan);
// The two convolutions' arguments as they would run by themselves (the tensor between them is neither read
// nor written).
fupr_status launch_basic_block(const BasicBlockArgs& a, const ConvArgs& first, const ConvArgs& second, int plan,
                               int count, void* stream);

}  // namespace fupr
