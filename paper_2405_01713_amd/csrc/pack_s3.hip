// 3 species, several cells per wave.
#include "bdf_packed.h"

BDFX_DEFINE_PACKED(3)
