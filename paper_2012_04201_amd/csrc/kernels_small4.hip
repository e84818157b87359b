#include "small_variants.h"

const void* small_kernel4(int nt, int waves, int co) { return small_by_cut<4>(nt, waves, co); }
