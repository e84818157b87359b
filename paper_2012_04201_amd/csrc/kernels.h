// The training kernels' entry points by compile-time variant, for the host code that launches them.  Each family
// is a source file of its own, so that they compile side by side.  A null pointer means there is no such variant.
#pragma once

#define BBO_HIDDEN __attribute__((visibility("hidden")))

BBO_HIDDEN const void* tiled_kernel(bool team);  // a team of workgroups per model
// unit tiles per wave, waves, output slots; one function per number of 16-wide k tiles of the input layer
BBO_HIDDEN const void* small_kernel1(int nt, int waves, int co);
BBO_HIDDEN const void* small_kernel2(int nt, int waves, int co);
BBO_HIDDEN const void* small_kernel3(int nt, int waves, int co);
BBO_HIDDEN const void* small_kernel4(int nt, int waves, int co);
BBO_HIDDEN const void* full_kernel(int kt, int nt, int co, int waves);  // k tiles of the input layer, unit tiles, outputs, waves
BBO_HIDDEN const void* mid_kernel(int kt, int nt, int waves, bool split);  // k tiles of the input layer, unit tiles per wave, waves, products
BBO_HIDDEN const void* deep_kernel2(int kt, int waves);         // k tiles of the input layer, waves; two hidden layers
BBO_HIDDEN const void* deep_kernel3(int kt, int waves);         // three
BBO_HIDDEN const void* linear_lds_kernel(int dd, int co, bool far);  // padded inputs and bias, outputs, columns in global memory
BBO_HIDDEN const void* linear_kernel(int co, int ki);          // padded outputs, rows of W per lane
