/* Stands in for the HIP runtime under the library's host code, on a machine without a GPU: every kernel launch is noted by
 * name and grid and nothing runs.  It answers for a device of 256 compute units. */
#include <stddef.h>
#include <stdio.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_;
static struct { const void* host; const char* name; } table[1024];
static int entries;
static char notes[1 << 20];
static size_t used;
static struct { dim3_ grid, block; size_t lds; void* stream; } pushed;

void** __hipRegisterFatBinary(const void* data) { static void* module; (void)data; return &module; }
void __hipUnregisterFatBinary(void** module) { (void)module; }
void __hipRegisterVar(void** module, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {
  (void)module; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void** module, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid,
                           void* block, void* grid, int* wsize) {
  (void)module; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
  if (entries < 1024) { table[entries].host = host; table[entries].name = name; ++entries; }
}
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t lds, void* stream) {
  pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_* grid, dim3_* block, size_t* lds, void** stream) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* host, dim3_ grid, dim3_ block, void** args, size_t lds, void* stream) {
  (void)args; (void)stream;
  const char* name = "?";
  for (int i = 0; i < entries; ++i) if (table[i].host == host) name = table[i].name;
  used += (size_t)snprintf(notes + used, sizeof notes - used, "%s %u %u %u %u %zu\n", name, grid.x, grid.y, grid.z, block.x, lds);
  return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int* value, int attribute, int device) { (void)attribute; (void)device; *value = 256; return 0; }
int hipFuncSetAttribute(const void* host, int attribute, int value) { (void)host; (void)attribute; (void)value; return 0; }
int hipGetSymbolAddress(void** address, const void* symbol) { *address = (void*)symbol; return 0; }

/* the launches since the last call, one a line: name, grid x y z, block x, LDS bytes */
const char* recorder_take(void) {
  static char out[1 << 20];
  memcpy(out, notes, used);
  out[used] = 0;
  used = 0;
  return out;
}
