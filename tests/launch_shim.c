/* Stands in for the runtime calls by which libfastgraph_hip.so launches kernels: nothing is launched, launches are counted and
 * their kernels named, and one of them can be made to fail.  Preloaded by tests that look at chains of launches; needs no GPU. */
#include <string.h>

static int made, fail_at, last;
static const void* launched[256];
static struct { const void* f; const char* name; } known[8192];
static int n_known;

void shim_reset(int fail) { made = 0; fail_at = fail; last = 0; }
int shim_made(void) { return made; }
const char* shim_name(int i)
{
    for (int j = 0; j < n_known; ++j)
        if (known[j].f == launched[i & 255]) return known[j].name;
    return "";
}

void __hipRegisterFunction(void** module, const void* f, char* device_function, const char* name, unsigned limit, void* a, void* b, void* c, void* d, int* e)
{
    (void)module; (void)device_function; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (n_known < 8192) { known[n_known].f = f; known[n_known++].name = strdup(name); }
}

int hipLaunchKernel(const void* f, unsigned long long grid_xy, unsigned grid_z, unsigned long long block_xy, unsigned block_z, void** args,
                    unsigned long lds, void* stream)
{
    (void)grid_xy; (void)grid_z; (void)block_xy; (void)block_z; (void)args; (void)lds; (void)stream;
    launched[made & 255] = f;
    if (++made != fail_at) return 0;
    return last = 2;                                     /* hipErrorOutOfMemory */
}
/* grid and block travel from the launch statement to its stub; what arrives is not looked at */
int __hipPushCallConfiguration(unsigned long long grid_xy, unsigned grid_z, unsigned long long block_xy, unsigned block_z, unsigned long lds, void* stream)
{
    (void)grid_xy; (void)grid_z; (void)block_xy; (void)block_z; (void)lds; (void)stream;
    return 0;
}
int __hipPopCallConfiguration(void* grid, void* block, unsigned long* lds, void** stream)
{
    (void)grid; (void)block;
    *lds = 0;
    *stream = 0;
    return 0;
}
int hipGetLastError(void) { const int e = last; last = 0; return e; }
int hipFuncSetAttribute(const void* f, int what, int value) { (void)f; (void)what; (void)value; return 0; }
