// What a test can set and see of the CPU device in device_double.cpp.
#pragma once

#include <hip/hip_runtime_api.h>

#include <functional>
#include <map>
#include <string>
#include <vector>

namespace dbl {
struct Step {
  float tf;
  int n;
};
extern int fail_in;                       // launches until one fails (-1: none does)
extern std::map<std::string, int> count;  // launches of each kind
extern int source_device;                 // device of memory that is asked for (-1: host, -2: unknown)
extern hipStream_t side;                  // launches on this stream (not null) wait in
extern std::vector<std::function<void()>> waiting;  // `waiting` for the test to run them
extern std::vector<Step> steps;           // time factors in the order of the steps
// microseconds of a launch of the given kind and shape, as events see it (none: 0)
extern std::function<float(const std::string&, int)> cost;
}  // namespace dbl
