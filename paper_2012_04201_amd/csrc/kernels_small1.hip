#include "small_variants.h"

const void* small_kernel1(int nt, int waves, int co) { return small_by_cut<1>(nt, waves, co); }
