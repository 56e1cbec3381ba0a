// Internal: a 3 x 3 convolution, a 1 x 1 convolution of its output and optionally a 1 x 1 convolution
// of that one's output in one launch (bottleneck.hip).
#pragma once
#include "fupr.h"

namespace fupr {

struct BottleneckArgs {
  fupr_dtype dt;
  fupr_conv_shape s1, s2, s3;    // s3 only if third
  bool third;
  bool add;                      // s2 adds a tensor of its output's shape
  bool pair;                     // s2 and s3 apart from s1 may run as a pair (conv1x1.hip)
  bool two;                      // s2 reads two tensors, the 3 x 3's output and x2 at stride2
  int H, W, xcs;                 // input of the 3 x 3 convolution
  int H2, W2, x2cs, stride2;
  // of a call, not looked at by the rules
  const void *x, *x2, *res, *packed1, *packed2, *packed3;
  void *y, *h;
  int ycs, hcs;                  // (the added tensor's channel stride is the output's)
  int relu1, relu2, relu3;
};

// Shapes alone: the kernel can run these operators (at any batch size that bottleneck_plan takes).
bool bottleneck_applies(const BottleneckArgs& a);
// The plan for a batch of N images, a number of this kernel's own; -1: the operators run apart.
int bottleneck_plan(const BottleneckArgs& a, int N);
// ... for `count` images of a batch that runs `plan`, which give that batch's bits.
int bottleneck_plan_part(const BottleneckArgs& a, int plan, int count);
const char* bottleneck_name(int plan);
fupr_status launch_bottleneck(const BottleneckArgs& a, int plan, int count, void* stream);

}  // namespace fupr
