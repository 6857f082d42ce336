// Which single solves may run whole, in one launch (resident_impl.h), beside the
// process's other calls on the device.  Plain C++, so that a test on the CPU can
// run it.
//
// A whole solve's workgroups hold their CUs until it ends (18 ms for 500
// iterations of 512 x 512 x 20, on every CU): launches of other streams that come
// meanwhile wait for all of it, and one by one if such solves follow each other.
//   * One that takes more than a quarter of the CUs runs whole only while no other
//     call is under way.  Otherwise it goes by launches, which share the device (a
//     server's requests of 48 iterations beside 512 x 512 x 20 solves: 167 ms each
//     beside whole ones, 16 beside launches; of two threads with such solves of 60
//     iterations one kept the device for itself and the other took 156 ms a call,
//     by launches both take 5).
//   * Smaller ones run whole beside anything while together they take at most half
//     of the CUs (a server beside 64 x 64 x 10 solves of 25 iterations: 10.4 and
//     0.6 ms; by launches 11.9 and 2.8).
//   * After one that had to be given up (its CUs held by other streams or
//     processes) the next 1, 2, 4, ... 64 are not tried.
#pragma once

#include <algorithm>
#include <mutex>

namespace rpca {

class DeviceUse {
 public:
  // A single solve of `grid` workgroups on a device of `cus` CUs: whether it runs
  // whole.  Followed by end_single with the same grid.
  bool begin_single(int grid, int cus) {
    std::lock_guard<std::mutex> lk(mu_);
    const bool small = 4 * grid <= cus;
    bool whole = small ? 2 * (held_ + grid) <= cus : calls_ == 0;
    ++calls_;
    if (whole && skip_ > 0) {
      --skip_;
      whole = false;
    }
    if (whole) held_ += grid;
    return whole;
  }
  void end_single(int grid, bool whole, bool gave_up) {
    std::lock_guard<std::mutex> lk(mu_);
    --calls_;
    if (!whole) return;
    held_ -= grid;
    next_skip_ = gave_up ? std::min(64, std::max(1, 2 * next_skip_)) : 0;
    if (gave_up) skip_ = next_skip_;
  }
  // Any other call.
  void begin() {
    std::lock_guard<std::mutex> lk(mu_);
    ++calls_;
  }
  void end() {
    std::lock_guard<std::mutex> lk(mu_);
    --calls_;
  }

 private:
  std::mutex mu_;
  int calls_ = 0;                  // under way, of every kind
  int held_ = 0;                   // CUs that whole solves take
  int skip_ = 0, next_skip_ = 0;   // after whole solves that were given up
};

// Of device `dev` (0 to 63).
DeviceUse& device_use(int dev);

class OtherCall {
 public:
  explicit OtherCall(int dev) : u_(dev >= 0 && dev < 64 ? &device_use(dev) : nullptr) {
    if (u_) u_->begin();
  }
  ~OtherCall() {
    if (u_) u_->end();
  }
  OtherCall(const OtherCall&) = delete;
  OtherCall& operator=(const OtherCall&) = delete;

 private:
  DeviceUse* u_;
};

class SingleCall {
 public:
  SingleCall(int dev, int grid, int cus)
      : u_(&device_use(dev)), grid_(grid), whole_(u_->begin_single(grid, cus)) {}
  ~SingleCall() { u_->end_single(grid_, whole_, gave_up_); }
  SingleCall(const SingleCall&) = delete;
  SingleCall& operator=(const SingleCall&) = delete;
  bool whole() const { return whole_; }
  void gave_up() { gave_up_ = true; }

 private:
  DeviceUse* u_;
  int grid_;
  bool whole_, gave_up_ = false;
};

}  // namespace rpca
