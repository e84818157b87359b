#include "small_variants.h"

const void* small_kernel3(int nt, int waves, int co) { return small_by_cut<3>(nt, waves, co); }
