// OncePerDevice without a device: what runs, and what is remembered.  Built and run by tests/test_bound.py.
#include <cstdio>

#include "per_device.h"

int main() {
  asl::OncePerDevice once;
  int calls[66] = {};
  auto run = [&](int device, int result) { return once(device, 0, [&] { ++calls[device]; return result; }); };
  const bool ok = run(0, 7) == 7 && calls[0] == 1                    // a failure is returned ...
                  && run(0, 0) == 0 && calls[0] == 2                 // ... and not remembered
                  && run(0, 7) == 0 && calls[0] == 2                 // done on device 0
                  && run(1, 0) == 0 && calls[1] == 1                 // the next device has its own
                  && run(63, 0) == 0 && run(63, 7) == 0 && calls[63] == 1
                  && run(65, 0) == 0 && run(65, 7) == 7 && calls[65] == 2;    // not remembered
  puts(ok ? "ok" : "wrong");
  return ok ? 0 : 1;
}
