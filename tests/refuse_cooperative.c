/* Refuses every cooperative launch, as a device that cannot hold the grid
 * does, and leaves the rest of the HIP runtime as it is.  Loaded with
 * RTLD_GLOBAL ahead of libschulze.so. */
#include <hip/hip_runtime_api.h>

static int refused;
int refused_launches(void) { return refused; }
hipError_t hipLaunchCooperativeKernel(const void *fn, dim3 grid, dim3 block, void **args, unsigned int lds,
                                      hipStream_t stream) {
    (void)fn, (void)grid, (void)block, (void)args, (void)lds, (void)stream;
    ++refused;
    return hipErrorCooperativeLaunchTooLarge;
}
