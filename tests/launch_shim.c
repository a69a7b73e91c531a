/* Stands in for the HIP runtime's launch calls on a machine without a GPU:
 * loaded with RTLD_GLOBAL before libpfresample, its definitions are the ones
 * the library binds to.  Every launch is recorded (kernel name, thread, grid,
 * block, stream) instead of run, after a short sleep that lets other threads
 * in between. */
#include <pthread.h>
#include <stdio.h>
#include <string.h>
#include <time.h>

typedef struct {
  unsigned x, y, z;
} dim3_t;

enum { MAX_KERNELS = 4096, MAX_LAUNCHES = 1 << 16 };

static struct {
  const void* stub;
  char name[512];
} kernels[MAX_KERNELS];
static int n_kernels;

static struct {
  int kernel;
  unsigned long thread;
  unsigned grid, block;
  void* stream;
} launches[MAX_LAUNCHES];
static int n_launches;
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static long sleep_ns;
static __thread int last_error;

static __thread struct {
  dim3_t grid, block;
  size_t shared;
  void* stream;
} config;

void** __hipRegisterFatBinary(const void* data) {
  static void* handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void** handle) { (void)handle; }
void __hipRegisterVar(void** m, void* var, char* host, char* name, int ext, size_t size, int constant,
                      int global) {
  (void)m, (void)var, (void)host, (void)name, (void)ext, (void)size, (void)constant, (void)global;
}
void __hipRegisterFunction(void** m, const void* stub, char* device, const char* name, unsigned limit,
                           void* tid, void* bid, void* bd, void* gd, int* wsize) {
  (void)m, (void)device, (void)limit, (void)tid, (void)bid, (void)bd, (void)gd, (void)wsize;
  if (n_kernels < MAX_KERNELS) {
    kernels[n_kernels].stub = stub;
    strncpy(kernels[n_kernels].name, name, sizeof(kernels[0].name) - 1);
    ++n_kernels;
  }
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void* stream) {
  config.grid = grid;
  config.block = block;
  config.shared = shared;
  config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shared, void** stream) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* stub, dim3_t grid, dim3_t block, void** args, size_t shared,
                    void* stream) {
  (void)args, (void)shared;
  pthread_mutex_lock(&mu);
  if (n_launches < MAX_LAUNCHES) {
    int k = 0;
    while (k < n_kernels && kernels[k].stub != stub) ++k;
    launches[n_launches].kernel = k;
    launches[n_launches].thread = (unsigned long)pthread_self();
    launches[n_launches].grid = grid.x;
    launches[n_launches].block = block.x;
    launches[n_launches].stream = stream;
    ++n_launches;
  }
  pthread_mutex_unlock(&mu);
  if (sleep_ns > 0) {
    struct timespec t = {0, sleep_ns};
    nanosleep(&t, NULL);
  }
  /* the runtime's own limit on a launch: fewer than 2^32 threads */
  if ((unsigned long long)grid.x * block.x >= (1ull << 32))
    last_error = 9; /* hipErrorInvalidConfiguration */
  return last_error;
}
int hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipGetDevice(int* device) {
  *device = 0;
  return 0;
}

void shim_sleep(long ns) { sleep_ns = ns; }
void shim_clear(void) { n_launches = 0; }
int shim_count(void) { return n_launches; }
/* "thread grid block stream name" of launch i */
int shim_launch(int i, char* out, int size) {
  if (i < 0 || i >= n_launches) return 0;
  return snprintf(out, (size_t)size, "%lu %u %u %zu %s", launches[i].thread, launches[i].grid,
                  launches[i].block, (size_t)launches[i].stream,
                  launches[i].kernel < n_kernels ? kernels[launches[i].kernel].name : "?");
}
