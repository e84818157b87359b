#include "small_variants.h"

const void* small_kernel2(int nt, int waves, int co) { return small_by_cut<2>(nt, waves, co); }
