// ov_gate.hpp -- the order of the resident launches of one device.
//
// Two resident launches that share the chip wait for each other's workgroups, so the launches
// of different contexts, each on its own stream, follow one another: a context waits for the
// work enqueued by the one that launched last.  Wait and launch are one step under the gate:
// a context that came between them would wait for a stream that does not hold the launch yet.
// No HIP here (the CPU tests run it with contexts of their own).
#pragma once

#include <mutex>

namespace ov {

template <class Ctx>
class ResGate {
 public:
  // enqueue() of context c's resident work, after wait(other) when another one launched last.
  template <class Wait, class Enqueue>
  auto pass(Ctx* c, Wait&& wait, Enqueue&& enqueue) {
    std::lock_guard<std::mutex> lock(mu_);
    if (last_ && last_ != c) wait(last_);
    last_ = c;
    return enqueue();
  }
  // f() while no other context passes (nobody's stream gets an event).
  template <class F>
  auto alone(F&& f) {
    std::lock_guard<std::mutex> lock(mu_);
    return f();
  }
  // c and its stream go away.
  void forget(const Ctx* c) {
    std::lock_guard<std::mutex> lock(mu_);
    if (last_ == c) last_ = nullptr;
  }

 private:
  std::mutex mu_;
  Ctx* last_ = nullptr;
};

}  // namespace ov
