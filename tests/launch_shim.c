/* Stands in for the runtime calls by which libfastgraph_hip.so launches kernels: nothing is launched, launches are counted, and
 * one of them can be made to fail.  Preloaded by test_launch_errors.py; needs no GPU. */
static int made, fail_at, last;

void shim_reset(int fail) { made = 0; fail_at = fail; last = 0; }
int shim_made(void) { return made; }

int hipLaunchKernel(const void* f, unsigned long long grid_xy, unsigned grid_z, unsigned long long block_xy, unsigned block_z, void** args,
                    unsigned long lds, void* stream)
{
    (void)f; (void)grid_xy; (void)grid_z; (void)block_xy; (void)block_z; (void)args; (void)lds; (void)stream;
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
