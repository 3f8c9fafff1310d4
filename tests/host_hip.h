// A stand-in for the HIP runtime, for tests of the library's host side without
// a GPU: device memory is addresses only, kernels do not run.  It keeps what
// the tests ask about: which memory was cleared, which kernels were launched
// with which grids, how often the host waited, allocated and captured; and it
// refuses allocations when told to.
#pragma once

#include <hip/hip_runtime.h>

#include <functional>
#include <map>
#include <string>
#include <vector>

struct Launch {
  std::string kernel;  // its mangled name
  unsigned grid, block;
  void** args;  // valid during the observer's call only
  bool is(const char* part) const { return kernel.find(part) != std::string::npos; }
  template <typename T>
  T arg(int k) const {
    return *static_cast<T*>(args[k]);
  }
};

struct FakeHip {
  // set by a test
  long fail_at = -1;             // the allocation (counted from 0) that is refused
  size_t most = ~(size_t)0;      // allocations above this many bytes are refused
  std::function<void(const Launch&)> on_launch;
  // kept for it
  long allocations = 0, refused = 0, waits = 0, captures = 0, replays = 0;
  std::map<std::string, long> launches;
  std::vector<std::string> too_large;  // launches of 2^32 threads or more
  long launched(const char* part) const {
    long n = 0;
    for (const auto& l : launches)
      if (l.first.find(part) != std::string::npos) n += l.second;
    return n;
  }
  // whether [p, p + bytes) lies in one live allocation and has been cleared
  // since it was allocated
  bool cleared(const void* p, size_t bytes) const;
  size_t live() const;  // allocations
};
extern FakeHip fake;
