// The training kernels' entry points by compile-time variant, for the host code that launches them.  Each family
// is a source file of its own, so that they compile side by side.  A null pointer means there is no such variant.
#pragma once

#define BBO_HIDDEN __attribute__((visibility("hidden")))

BBO_HIDDEN const void* tiled_kernel();
BBO_HIDDEN const void* small_kernel(int kt, int co);   // 16-wide k tiles of the input layer, output slots
BBO_HIDDEN const void* mid_kernel(int kt);             // 16-wide k tiles of the input layer
BBO_HIDDEN const void* linear_kernel(int co, int ki);  // padded outputs, rows of W per lane
