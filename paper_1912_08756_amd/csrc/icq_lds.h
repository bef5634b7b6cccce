// Opt-in for more dynamic LDS than the default (host side, no device code).
#pragma once
#include <hip/hip_runtime_api.h>

// hipFuncSetAttribute(fn, MaxDynamicSharedMemorySize, bytes) unless as many bytes are allowed already on the current device;
// thread-safe.  no_static_lds: also refuse (hipErrorInvalidValue) a kernel whose code object holds static LDS.
hipError_t icq_allow_lds(const void *fn, int bytes, bool no_static_lds = false);
