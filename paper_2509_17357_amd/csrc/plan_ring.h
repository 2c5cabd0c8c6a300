// The ring of plan buffers of a device: which buffer the next call may write (no HIP here).
#pragma once

#include <atomic>
#include <chrono>
#include <cstddef>
#include <cstdint>
#include <thread>

namespace cronus {

// The work list is written into pinned, device-mapped host memory and the kernels read it
// from there (each work-group one 64-byte item): no copy sits between the caller's previous
// work on the stream and the attention kernel (a stream-ordered copy of these few KB took
// about 25 us of otherwise idle stream time on MI355X).  A slot is reused only after the
// kernels of the call that used it are done with it: the main kernel's last work-group stores
// the call's number in front of the plan image.  (An event recorded behind the kernels cost
// the host 1.5 us a call and the stream 5 us before its next kernel.)
struct Slot {
  void* host = nullptr;
  void* dev = nullptr;   // the same memory as the device sees it
  size_t cap = 0;
  uint32_t call = 0;     // number of the last call that used the slot
  const void* stream = nullptr;  // where that call was enqueued; compared, never used
  enum State { kFree, kPending, kLost } state = kFree;  // kLost: nothing tells when its kernels are done
  bool reported() const { return *static_cast<const volatile uint32_t*>(host) == call; }
};
constexpr int kSlots = 8;

struct PlanRing {
  Slot slots[kSlots];
  int next = 0;

  // A slot that no kernel reads any more, the one after the last taken if that is free; nullptr: none yet.
  Slot* take() {
    for (int i = 0; i < kSlots; ++i) {
      Slot* s = &slots[(next + i) % kSlots];
      if (s->state == Slot::kLost || (s->state == Slot::kPending && !s->reported())) continue;
      std::atomic_thread_fence(std::memory_order_acquire);
      s->state = Slot::kFree;
      next = (next + i + 1) % kSlots;
      return s;
    }
    return nullptr;
  }
  bool usable() const {
    for (const Slot& s : slots)
      if (s.state != Slot::kLost) return true;
    return false;
  }
  // The work on `stream` is over, or failed: its calls that have not reported never will.
  // before: the calls that the slots held before the stream was asked.
  void give_up(const void* stream, const uint32_t (&before)[kSlots]) {
    for (int i = 0; i < kSlots; ++i) {
      Slot& s = slots[i];
      if (s.state == Slot::kPending && s.stream == stream && s.call == before[i] && !s.reported()) s.state = Slot::kLost;
    }
  }
};

enum class StreamIs { kBusy, kDone, kFailed };

// take(), waiting while every slot is in use (a host that runs eight calls ahead of the GPU).
// `lock` guards the ring and is held on entry and exit, but not while waiting: calls of other
// threads, streams and devices go on.  After each `patience` of waiting, ask() tells about the
// calling stream, so that calls that a device error ended are not waited for for ever; it has
// to be harmless to whatever else the process does (a device-wide synchronisation is not: it
// is refused, and breaks the capture, while another stream is captured).
template <class Lock, class Ask>
Slot* wait_for_slot(PlanRing& ring, Lock& lock, const void* stream, std::chrono::milliseconds patience, Ask ask) {
  auto asked = std::chrono::steady_clock::now();
  for (int spin = 0;; spin += spin < 4096) {
    if (Slot* s = ring.take()) return s;
    if (!ring.usable()) return nullptr;
    uint32_t before[kSlots];
    for (int i = 0; i < kSlots; ++i) before[i] = ring.slots[i].call;
    lock.unlock();
    StreamIs is = StreamIs::kBusy;
    if (spin < 4096) {
      __builtin_ia32_pause();
    } else {
      std::this_thread::sleep_for(std::chrono::microseconds(2));
      if (std::chrono::steady_clock::now() - asked > patience) {
        is = ask();
        asked = std::chrono::steady_clock::now();
      }
    }
    lock.lock();
    if (is != StreamIs::kBusy) ring.give_up(stream, before);
    if (is == StreamIs::kFailed) return nullptr;
  }
}

}  // namespace cronus
