// What the stand-ins of fake_runtime.cpp record and inject.
#pragma once
#include <cstddef>
#include <string>
#include <vector>

namespace fake {
struct Launch {
    std::string name;     // launcher
    int tc = 0;           // axis 1: columns per block
};
extern std::vector<Launch> launches;      // since the last clear
extern double clock_ms;                   // what event timings read; advanced by cost()
extern double (*cost)(const Launch&);     // milliseconds a launch takes (null: none)
extern size_t pending;                    // asynchronous copies not waited for yet
extern size_t fail_copy_bytes;            // the asynchronous copy of this size fails (0: none)
extern std::string fail_launch;           // the launcher of this name fails
void reset();
}  // namespace fake
