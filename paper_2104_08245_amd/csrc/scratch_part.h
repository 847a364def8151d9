// The workspace arrays of nolsm_sign_batch_noalloc, one in a source file of its
// own each: the runtime loads the device code of a file when something of it
// is first used, and for an array that takes 25 ms and its memory. So a program
// pays for as many as it has streams that call.
//
// Every GPU holds its own copy of an array, at its own address, from its load
// until the process ends. In host code the name is a stand-in, not a device
// address: kernels get the address that scratch_symbol_* returns for the
// current device.
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/nolsm.h"

hipError_t scratch_symbol_0(void **p);
hipError_t scratch_symbol_1(void **p);
hipError_t scratch_symbol_2(void **p);
static_assert(NOLSM_NOALLOC_CALLS == 3, "a file and a look-up for each");

#define SCRATCH_PART(i)                                                     \
    static __device__ __align__(256) char scratch[NOLSM_NOALLOC_WS_BYTES];  \
    hipError_t scratch_symbol_##i(void **p) { return hipGetSymbolAddress(p, HIP_SYMBOL(scratch)); }
