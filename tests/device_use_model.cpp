// Exercises csrc/device_use.h; prints "ok" when every check holds.
#include <cstdio>
#include <cstdlib>

#include "device_use.h"

namespace rpca {
DeviceUse& device_use(int dev) {
  static DeviceUse u[64];
  return u[dev];
}
}  // namespace rpca

using namespace rpca;

#define CHECK(x)                                  \
  do {                                            \
    if (!(x)) {                                   \
      std::printf("line %d: %s\n", __LINE__, #x); \
      std::exit(1);                               \
    }                                             \
  } while (0)

constexpr int kCus = 256;

int main() {
  for (int i = 0; i < 3; ++i) CHECK(SingleCall(0, 256, kCus).whole());  // alone
  {  // large: not beside any other call, of either kind
    OtherCall o(0);
    CHECK(!SingleCall(0, 256, kCus).whole());
    CHECK(!SingleCall(0, 65, kCus).whole());
    CHECK(SingleCall(0, 64, kCus).whole());  // small: beside it
  }
  {
    SingleCall first(0, 256, kCus), second(0, 256, kCus);
    CHECK(first.whole() && !second.whole());
    SingleCall third(0, 100, kCus);
    CHECK(!third.whole());
  }
  {  // nor while only launched ones are left
    SingleCall* first = new SingleCall(0, 256, kCus);
    SingleCall second(0, 256, kCus);
    delete first;
    CHECK(!SingleCall(0, 256, kCus).whole());
  }
  CHECK(SingleCall(0, 256, kCus).whole());
  {  // small ones: together at most half of the CUs
    SingleCall a(1, 64, kCus), b(1, 64, kCus), c(1, 1, kCus);
    CHECK(a.whole() && b.whole() && !c.whole());
  }
  {
    SingleCall a(1, 64, kCus), b(1, 32, kCus), c(1, 32, kCus);
    CHECK(a.whole() && b.whole() && c.whole());
    CHECK(!SingleCall(1, 256, kCus).whole());
  }
  // given up: 1, 2, 4, ... 64, 64 not tried; after one that ended well, 1 again
  for (int round = 0; round < 2; ++round) {
    for (int want = 1, k = 0; k < 9; ++k, want = want < 64 ? 2 * want : 64) {
      {
        SingleCall c(2, 16, kCus);
        CHECK(c.whole());
        c.gave_up();
      }
      for (int i = 0; i < want; ++i) CHECK(!SingleCall(2, 16, kCus).whole());
    }
    CHECK(SingleCall(2, 16, kCus).whole());
  }
  OtherCall none(-1), far(64);  // devices out of the table
  std::printf("ok\n");
  return 0;
}
