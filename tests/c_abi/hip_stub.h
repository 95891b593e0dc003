/*
 * Stands in for the HIP runtime's launch, error and copy calls in a program that
 * is linked against libagft and needs no GPU: nothing runs, the kernels that
 * the library asks for are counted and told apart by their addresses, and any
 * launch can be made to fail.  Test infrastructure only.
 */
#ifndef AGFT_TEST_HIP_STUB_H
#define AGFT_TEST_HIP_STUB_H

#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <hip/hip_runtime_api.h>

#include "agft.h"
#include "agft_sim.h"

static const void *ran[16];   /* kernels launched since the last start() */
static unsigned ran_block[16], ran_grid[16];   /* and their shapes: threads per workgroup, workgroups */
static int n_ran, fail_at;    /* fail_at: the launch that fails, from 1 (0: none) */
static hipError_t last_error;
static unsigned char header[256];   /* the state header that the library set up */

/* (the compiler's launch syntax hands the launch's shape over through these) */
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream)
{
    cfg_grid = grid, cfg_block = block, cfg_lds = lds, cfg_stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream)
{
    *grid = cfg_grid, *block = cfg_block, *lds = cfg_lds, *stream = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream)
{
    (void)lds, (void)stream;
    if (fail_at && --fail_at == 0) return last_error = hipErrorLaunchFailure;
    if (n_ran < 16) ran[n_ran] = f, ran_block[n_ran] = block.x, ran_grid[n_ran] = grid.x;
    ++n_ran;
    const unsigned char *a = args[0];
    for (int i = 0; f && i < 128; i += 4)   /* the set-up's arguments hold the header */
        if (memcmp(a + i, "AGFT", 4) == 0) memcpy(header, a + i, sizeof(header));
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t stream)
{
    (void)src, (void)kind, (void)stream;
    memcpy(dst, header, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t stream)
{
    (void)stream;
    return hipSuccess;
}

static void start(int fail)
{
    n_ran = 0;
    fail_at = fail;
}

#endif
