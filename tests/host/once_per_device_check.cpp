// Set-up once per device: every device gets it, a failure is tried again,
// threads that race run it at most once each.
#include "once_per_device.h"

#include <stdio.h>

#include <thread>
#include <vector>

#define CHECK(c)                                     \
  do {                                               \
    if (!(c)) {                                      \
      printf("line %d: %s\n", __LINE__, #c);         \
      return 1;                                      \
    }                                                \
  } while (0)

int main() {
  enum Err { OK = 0, BAD = 7 };
  int calls = 0;
  Err next = BAD;
  upir::OncePerDevice once;
  auto set = [&] {
    ++calls;
    return next;
  };
  CHECK(once.run(0, set) == BAD && calls == 1);
  CHECK(once.run(0, set) == BAD && calls == 2);  // not kept
  next = OK;
  CHECK(once.run(0, set) == OK && calls == 3);
  next = BAD;
  CHECK(once.run(0, set) == OK && calls == 3);   // done on device 0
  CHECK(once.run(1, set) == BAD && calls == 4);  // not on device 1
  next = OK;
  CHECK(once.run(1, set) == OK && once.run(63, set) == OK && calls == 6);
  CHECK(once.run(64, set) == OK && once.run(64, set) == OK && calls == 8);  // past the mask: every time
  CHECK(once.run(0, set) == OK && once.run(1, set) == OK && once.run(63, set) == OK && calls == 8);
  upir::OncePerDevice shared;
  std::atomic<int> ran{0};
  std::vector<std::thread> ts;
  for (int i = 0; i < 8; ++i)
    ts.emplace_back([&] {
      for (int k = 0; k < 1000; ++k) shared.run(k % 4, [&] { return ran.fetch_add(1) < 0 ? BAD : OK; });
    });
  for (auto &t : ts) t.join();
  CHECK(ran >= 4 && ran <= 32);
  puts("ok");
  return 0;
}
