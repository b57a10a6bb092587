// A stand-in for the HIP runtime that the built library is linked with in the CPU tests of its
// memory handling and dispatch (test infrastructure).  Device memory is address space only, with
// a capacity that a test sets; launches and copies do nothing but are recorded; any call can be
// made to fail.  The executable's definitions take the place of the runtime's.
#pragma once

#ifndef __HIP_PLATFORM_AMD__
#define __HIP_PLATFORM_AMD__
#endif
#include <hip/hip_runtime_api.h>

#include <map>
#include <set>
#include <string>
#include <vector>

namespace fake {

struct Launch {
    std::string kernel;  // mangled name
    unsigned grid, block;
};

struct Device {
    size_t capacity = (size_t)288 << 30, used = 0, peak = 0;
    std::map<char*, size_t> live;      // device allocations
    std::vector<size_t> freed;         // sizes in the order they were freed
    std::set<hipStream_t> streams;     // created and not destroyed
    std::set<hipEvent_t> events;
    std::set<hipStream_t> pending;     // streams with work that nobody has waited for
    std::vector<Launch> launches;
    int fail_at = -1, calls = 0;       // call number that fails, calls so far
    bool failed = false;
    char* next = (char*)((size_t)1 << 40);
};
Device& device();

// Whether the present call is the one to fail
bool fails();

}  // namespace fake
