/* Stands in for the HIP runtime's launch functions, so that the launches of a call can be looked at without a GPU: the pointers of the
 * call are never followed. */
#include <stddef.h>
typedef struct { unsigned x, y, z; } grid_t;
typedef struct { unsigned grid[3], threads, lds; } launch_t;
launch_t launches[64];
int n_launches;
static char device_memory[1];

static int record(grid_t grid, grid_t block, size_t lds) {
  if (n_launches < 64) launches[n_launches++] = (launch_t){{grid.x, grid.y, grid.z}, block.x, (unsigned)lds};
  return 0;
}
/* what <<< >>> hands to the kernel's host function (the runtime's own fails without a GPU) */
static grid_t pushed_grid, pushed_block;
static size_t pushed_lds;
int __hipPushCallConfiguration(grid_t grid, grid_t block, size_t lds, void* stream) { return pushed_grid = grid, pushed_block = block, pushed_lds = lds, 0; }
int __hipPopCallConfiguration(grid_t* grid, grid_t* block, size_t* lds, void** stream) {
  return *grid = pushed_grid, *block = pushed_block, *lds = pushed_lds, *stream = NULL, 0;
}
int hipLaunchKernel(const void* f, grid_t grid, grid_t block, void** args, size_t lds, void* stream) { return record(grid, block, lds); }
int hipExtLaunchKernel(const void* f, grid_t grid, grid_t block, void** args, size_t lds, void* stream, void* start, void* stop, int flags) {
  return record(grid, block, lds);
}
int hipFuncSetAttribute(const void* f, int attribute, int value) { return 0; }
int hipGetDevice(int* device) { return *device = 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { return *p = (void*)(((size_t)device_memory + 255) / 256 * 256), 0; }
