// Rules of a dispatch that are a matter of sizes alone: plain host code, so that the measured points behind them can be
// tested without a device.
#pragma once

namespace rules {

// Least samples in the largest class of a launch for the step loop that cuts classes into slices (sliced_kernels.hip).  A
// single class of more than four blocks is cut as soon as one workgroup's registers do not hold it: above 2560 samples with
// more than eight blocks, above 3072 with more than four (5120 fit, but too few registers are left).  One class, one
// workgroup / slices, in ms: eight blocks 3072 samples 12.5 / 17.5, 3073 20.0 / 17.8, five blocks 3072 11.5 / 16.8, 3073
// 18.1 / 16.9, twelve blocks 2561 18.2 / 17.2, sixteen 19.0 / 17.2.
constexpr int sliced_from(int classes, int K)
{
    if (classes > 1) return 5121;
    return K > 8 ? 2561 : K > 4 ? 3073 : 5121;
}

} // namespace rules
