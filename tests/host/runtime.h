// A stand-in for the HIP runtime and the kernel launchers, so that plans, batches
// and sources can be made and called without a device.  "Device" memory is host
// memory that is counted against a budget; the launchers record what the checks
// look at and do nothing.
#pragma once

#include <atomic>
#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime.h>

#include "slos_ext.h"
#include "slos_internal.h"

struct FakeRuntime {
    size_t used = 0, peak = 0, budget = ~size_t(0);  // bytes of device memory
    bool no_threads = false;                         // pthread_create fails
    std::atomic<long> news{-1};                      // allocations until one fails, once (< 0: none does)
    SelectParams select{};                           // of the last slos_launch_select
    int selects = 0;
    size_t copied = 0;                               // bytes of the last asynchronous copy
};
extern FakeRuntime fake;
