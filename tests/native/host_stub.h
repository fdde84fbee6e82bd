// Test doubles behind the library's host orchestration (host_stub.cpp): a HIP
// runtime whose device memory is the heap and whose work runs when it is
// queued, and CPU forms of the kernel launchers, which read and write exactly
// the extents that the kernels may. What a test can set or ask:
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace stub {

// device blocks held now, and whether p is the start of one
size_t live_blocks();
bool live(const void *p);
// device bytes held now
size_t live_bytes();
// every hipMalloc of exactly `bytes` fails from now on (0: none)
void fail_mallocs(size_t bytes);
// hipMalloc fails where more than `bytes` would be held (0: never)
void set_capacity(size_t bytes);
// every hipMemcpyAsync of exactly `bytes` fails from now on (0: none)
void fail_copies(size_t bytes);

// a caller's capture of stream st: launches are kept instead of run; replay()
// runs what the last capture kept
void begin_capture(hipStream_t st);
void end_capture(hipStream_t st);
void replay();

// errors the doubles found (reads of data whose fill the reading stream does
// not follow, values out of their range): printed as they occur
int errors();

}  // namespace stub
