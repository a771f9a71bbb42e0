// CPU check of the gate that orders resident launches (ov_gate.hpp): contexts on threads of
// their own pass it many times.  A context's stream is a counter of what it has enqueued; an
// event holds the counter's value when it was recorded.  A launch is in order if the event its
// context waited for holds everything the previous launcher had enqueued, its launch included
// (enqueued a little after the gate was passed, as a real one is), and no event may be recorded
// while the stream's own context captures.  Prints "res_gate ok".
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>

#include "ov_gate.hpp"

struct Ctx {
  std::atomic<int> enqueued{0};   // work on the stream
  std::atomic<int> launched{0};   // its value after the last resident launch
  std::atomic<bool> capturing{false};
};

static ov::ResGate<Ctx> gate;
static std::atomic<Ctx*> last{nullptr};  // the context that launched last
static std::atomic<int> fails{0};

static void work(Ctx* c, int rounds, int id) {
  for (int n = 0; n < rounds; ++n) {
    if (n % 7 == id) {  // a capture without resident launches
      gate.alone([&]() {
        c->capturing = true;
        std::this_thread::yield();
        c->capturing = false;
      });
      continue;
    }
    Ctx* waited = nullptr;
    int event = 0;
    gate.pass(
        c,
        [&](Ctx* other) {
          if (other->capturing) ++fails;
          waited = other;
          event = other->enqueued;
        },
        [&]() {
          std::this_thread::yield();
          Ctx* before = last;
          if (before && before != c && (waited != before || event < before->launched)) ++fails;
          std::this_thread::yield();
          c->launched = ++c->enqueued;
          last = c;
        });
    ++c->enqueued;  // other work behind it
  }
}

int main() {
  std::vector<Ctx> ctx(4);
  std::vector<std::thread> t;
  for (int k = 0; k < 4; ++k) t.emplace_back(work, &ctx[k], 5000, k);
  for (auto& x : t) x.join();
  // a context that goes away is not waited for
  Ctx gone, next;
  bool waited = false;
  auto wait = [&](Ctx*) { waited = true; };
  gate.pass(&gone, wait, []() {});
  waited = false;
  gate.forget(&gone);
  gate.pass(&next, wait, []() {});
  if (waited) ++fails;
  gate.pass(&next, wait, []() {});  // nor does a context wait for itself
  if (waited) ++fails;
  gate.pass(&gone, wait, []() {});
  if (!waited) ++fails;
  if (fails) {
    std::printf("%d launches out of order\n", fails.load());
    return 1;
  }
  std::puts("res_gate ok");
  return 0;
}
