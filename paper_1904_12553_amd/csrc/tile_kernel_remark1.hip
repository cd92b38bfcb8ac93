// tile_kernel_remark1.hip -- the tile kernel instantiated for the force
// distribution of Remark 1 (Sec. 3.1) (see tile_kernel.hip), compiled as its own
// translation unit.
#define NPL_GS 2
#include "tile_kernel.hip"
