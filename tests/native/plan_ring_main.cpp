// Host-only driver for the ring of plan buffers (plan_ring.h): runs the case named by the
// argument and exits with 0 if the ring did what it has to.  "The device" is this program: a
// call reports by storing its number in its slot.
#include <atomic>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <thread>

#include "plan_ring.h"

using namespace cronus;
using namespace std::chrono;

static uint32_t header[kSlots][64];
static PlanRing ring;
static std::timed_mutex mu;
static int stream_a, stream_b;

static int index_of(const Slot* s) { return s ? (int)(s - ring.slots) : -1; }
static void enqueue(Slot* s, const void* stream, Slot::State state = Slot::kPending) {
  if (!s->host) s->host = header[index_of(s)];
  ++s->call;
  s->stream = stream;
  s->state = state;
}
static void report(int i) { *static_cast<volatile uint32_t*>(ring.slots[i].host) = ring.slots[i].call; }
#define CHECK(c) \
  if (!(c)) return std::printf("line %d: %s\n", __LINE__, #c), 1


// slots go round in order, and one that has not reported is not handed out
static int order() {
  for (int i = 0; i < 3 * kSlots; ++i) {
    Slot* s = ring.take();
    CHECK(index_of(s) == i % kSlots);
    enqueue(s, &stream_a);
    if (i >= kSlots / 2) report((i - kSlots / 2) % kSlots);
  }
  for (int i = 0; i < kSlots / 2; ++i) enqueue(ring.take(), &stream_a);
  CHECK(ring.take() == nullptr);
  report(5);  // out of turn (a call of another stream)
  CHECK(index_of(ring.take()) == 5);
  return 0;
}

// while one thread waits for a slot, the lock is free for others; the slot is had when its call reports
static int lock_is_free() {
  for (int i = 0; i < kSlots; ++i) enqueue(ring.take(), &stream_a);
  Slot* got = nullptr;
  std::atomic<bool> asked{false};
  std::thread waiter([&] {
    std::unique_lock<std::timed_mutex> lock(mu);
    got = wait_for_slot(ring, lock, &stream_b, milliseconds(5), [&] { asked = true; return StreamIs::kBusy; });
  });
  for (int n = 0; n < 20 || (!asked && n < 4000); ++n) {
    std::this_thread::sleep_for(milliseconds(2));
    CHECK(mu.try_lock_for(milliseconds(500)));
    mu.unlock();
  }
  report(3);
  waiter.join();
  CHECK(index_of(got) == 3 && asked);
  return 0;
}

// a stream whose work is over: its calls that have not reported are given up, others' are kept
static int ended_calls() {
  for (int i = 0; i < kSlots; ++i) enqueue(ring.take(), i < 6 ? (const void*)&stream_a : &stream_b);
  std::unique_lock<std::timed_mutex> lock(mu);
  int n = 0;
  Slot* s = wait_for_slot(ring, lock, &stream_a, milliseconds(2), [&] {
    if (++n == 2) report(6);
    return n == 1 ? StreamIs::kDone : StreamIs::kBusy;
  });
  CHECK(index_of(s) == 6 && lock.owns_lock());
  for (int i = 0; i < 6; ++i) CHECK(ring.slots[i].state == Slot::kLost);
  CHECK(ring.slots[7].state == Slot::kPending);
  return 0;
}

// a failed stream: the call fails, without waiting again the next time
static int failed_stream() {
  for (int i = 0; i < kSlots; ++i) enqueue(ring.take(), &stream_a);
  std::unique_lock<std::timed_mutex> lock(mu);
  CHECK(wait_for_slot(ring, lock, &stream_a, milliseconds(2), [] { return StreamIs::kFailed; }) == nullptr);
  CHECK(lock.owns_lock());
  bool asked = false;
  CHECK(wait_for_slot(ring, lock, &stream_a, milliseconds(2), [&] { asked = true; return StreamIs::kBusy; }) == nullptr);
  CHECK(!asked);
  return 0;
}

int main(int argc, char** argv) {
  const struct { const char* name; int (*run)(); } cases[] = {
      {"order", order}, {"lock_is_free", lock_is_free}, {"ended_calls", ended_calls}, {"failed_stream", failed_stream}};
  for (const auto& c : cases)
    if (argc > 1 && !std::strcmp(argv[1], c.name)) return c.run();
  return 2;
}
