/* Records kernel launches instead of making them: loaded before the library
 * under test, its definitions of the HIP runtime's launch calls are the ones
 * that the library binds to. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { const char *name; dim3 grid, block; size_t lds; } Launch;

static struct { const void *host; const char *name; } kernels[4096];
static int nkernels;
static Launch launches[256];
static int nlaunches;
static struct { dim3 grid, block; size_t lds; void *stream; } call;

void __hipRegisterFunction(void **mod, const void *host, char *dev, const char *name,
                           unsigned limit, void *tid, void *bid, dim3 *bdim, dim3 *gdim, int *ws) {
  typedef void (*fn)(void **, const void *, char *, const char *, unsigned, void *, void *, dim3 *,
                     dim3 *, int *);
  fn next = (fn)dlsym(RTLD_NEXT, "__hipRegisterFunction");
  if (nkernels < 4096) {
    kernels[nkernels].host = host;
    kernels[nkernels++].name = name;
  }
  if (next) next(mod, host, dev, name, limit, tid, bid, bdim, gdim, ws);
}

int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
  call.grid = grid;
  call.block = block;
  call.lds = lds;
  call.stream = stream;
  return 0;
}

int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
  *grid = call.grid;
  *block = call.block;
  *lds = call.lds;
  *stream = call.stream;
  return 0;
}

int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  (void)args;
  (void)stream;
  const char *name = "?";
  for (int i = 0; i < nkernels; i++)
    if (kernels[i].host == f) name = kernels[i].name;
  if (nlaunches < 256) {
    Launch l = {name, grid, block, lds};
    launches[nlaunches++] = l;
  }
  return 0;
}

int hipGetLastError(void) { return 0; }

int shim_launches(void) { return nlaunches; }
void shim_reset(void) { nlaunches = 0; }
const char *shim_name(int i) { return launches[i].name; }
uint32_t shim_grid(int i) { return launches[i].grid.x; }
uint32_t shim_block(int i) { return launches[i].block.x; }
uint64_t shim_lds(int i) { return launches[i].lds; }
