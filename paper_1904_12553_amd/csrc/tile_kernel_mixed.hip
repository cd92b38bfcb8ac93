// tile_kernel_mixed.hip -- the tile kernel instantiated for the isotropic
// mixed gradient scheme of eq:N40 (see tile_kernel.hip), compiled as its own
// translation unit.
#define NPL_GS 1
#include "tile_kernel.hip"
