// Stands in for the HIP runtime's entry points that libhac calls, so that a test without a GPU sees what the library would launch and can let
// calls fail: no kernel runs, "device" memory is whatever the test passes.  Loaded with LD_PRELOAD; kernels are registered with the real
// runtime, which needs no device for that.
#include <cstdint>
#include <cstdlib>
#include <cstring>

struct dim3_t { uint32_t x, y, z; };
typedef int err_t;

namespace {
struct Event { char what; uint32_t grid; uint64_t lds; uint8_t arg[16]; };   // 'L' a launch, 'S' a wait for a stream, 'M' a copy
Event events[256];
int count, launches, wanted_launch = -1, wanted_arg, wanted_bytes, last_error, wait_error;
dim3_t pushed_grid, pushed_block; size_t pushed_lds; void* pushed_stream;
Event* add(char what)
{
    static Event spare;
    Event* e = count < 256 ? &events[count++] : &spare;
    std::memset(e, 0, sizeof *e);
    e->what = what;
    return e;
}
}

extern "C" {
// ---- for the test ----
void stub_reset() { count = launches = last_error = wait_error = 0; wanted_launch = -1; }
void stub_copy_arg(int launch, int arg, int bytes) { wanted_launch = launch; wanted_arg = arg; wanted_bytes = bytes; }   // of one launch
void stub_fail(int get_last_error, int synchronize) { last_error = get_last_error; wait_error = synchronize; }
int stub_count() { return count; }
int stub_event(int i, uint32_t* grid, uint64_t* lds, uint64_t* arg)
{
    *grid = events[i].grid; *lds = events[i].lds;
    std::memcpy(arg, events[i].arg, 8);
    return events[i].what;
}

// ---- the runtime ----
err_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* s) { pushed_grid = g; pushed_block = b; pushed_lds = lds; pushed_stream = s; return 0; }
err_t __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** s) { *g = pushed_grid; *b = pushed_block; *lds = pushed_lds; *s = pushed_stream; return 0; }
err_t hipLaunchKernel(const void*, dim3_t grid, dim3_t, void** args, size_t lds, void*)
{
    Event* e = add('L');
    e->grid = grid.x; e->lds = lds;
    if (launches++ == wanted_launch) std::memcpy(e->arg, args[wanted_arg], (size_t)wanted_bytes);
    return 0;
}
err_t hipGetLastError() { return last_error; }
err_t hipStreamSynchronize(void*) { add('S'); return wait_error; }
err_t hipMemcpyAsync(void*, const void*, size_t, int, void*) { add('M'); return 0; }
err_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return *p ? 0 : 2; }
err_t hipFuncSetAttribute(const void*, int, int) { return 0; }
err_t hipGetDevice(int* d) { *d = 0; return 0; }
err_t hipGetSymbolAddress(void** p, const void*) { static uint8_t room[65536]; *p = room; return 0; }
}
