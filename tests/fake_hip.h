// A stand-in for the HIP runtime, for running the library's host code on the CPU
// under the address sanitizer (tests/host_paths_driver.cpp).
//
// Device memory is host memory.  Kernels do nothing, but for those that the host
// waits for: they post the sizes that the driver asks for.  Every launch is
// checked: its pointers must be live allocations, its stream and grid valid, and
// the moments that an M2L kernel reads must have been computed into that memory.
#pragma once

#include <set>
#include <string>

struct FakeHip {
    std::string what;              // what the driver is doing, for messages
    std::set<const void*> user;    // pointers that the caller owns
    // sizes that the build and the walk report
    long leaves = 0, levels = 1, far = 0, near = 0;
    unsigned long long rows = 0;   // partial sums of the near field
    bool nonfinite = false;        // the positions hold a value that is not finite
    long pass_entries = 3000;      // the walk's largest frontier
    int overflow = 0;              // unsynchronised walks still to run out of room
    bool wait_ran_out = false;     // a walk pass sets the device error word
    // memory: allocations so far; the fail_at-th and the next one fail (0: none)
    long mallocs = 0, fail_at = 0;
    size_t bytes = 0;              // device bytes allocated
    size_t limit = 0;              // the device's size (0: no limit)
    // what was launched
    long launches = 0, list_launches = 0, near_launches = 0;
    long sized_passes = 0, emit_launches = 0, pass_launches = 0;  // walk passes by kind
    std::set<void*> busy;          // streams with work nobody has waited for
};
extern FakeHip fake;
bool fake_all_gone();              // no allocation, stream or event is left
