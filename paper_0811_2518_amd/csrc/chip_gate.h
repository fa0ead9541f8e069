// Who may launch kernels whose workgroups wait for each other (the resident
// solves, the batched teams) on a device, in plain C++.
//
// All workgroups of such a launch have to be on the chip at once.  Two launches
// of one process that do not fit together can each get a part of it when the one
// before them ends; then both wait until the time limits of their roll calls
// have passed and take the slower path.  A solve blocks its thread until it is
// done, so the threads can be let in in turn instead.
//
// A launch enters when everything that is inside fits on the chip: it then fits
// beside them or is the only one that does not, and waits in its hardware queue
// for the others to end, so the chip does not idle between two solves.  In the
// second case it also waits until the others have been issued, so as not to take
// their places.  A call of several kernels that each want the whole chip asks for
// more than there is: it enters when nothing is inside and keeps others out.
// Threads enter in the order of their calls.  Where several threads use the gate,
// a thread waits for the earlier work of its stream before it enters, not inside.
// Other processes and other kernels
// are not seen here; for these the roll calls have their limits.
//
// Solves per thread in turn on streams of their own, ms a solve without / with
// the gate: FP32 + refinement on G(n, 4n) with n = 130003 from 3 and 4 threads
// 0.43 / 0.35 and 0.46 / 0.35, the 64^3 grid from 3 threads 1.04 / 0.72, 192 uneven
// systems from 2 threads 7.9 / 7.8, from 3 20.4 / 8.1, colour-serial from 2 threads
// 20.5 / 9.7.  From one thread it costs nothing measurable.
#pragma once

#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <mutex>
#include <thread>

namespace gabp {

class ChipGate {
 public:
  // Waits for a turn; false when none came within `patience` (the caller's stream
  // may itself be waiting for work of a thread that stands here).
  bool enter(int64_t need, int64_t room, std::chrono::milliseconds patience) {
    std::unique_lock<std::mutex> lk(m_);
    note_thread();
    Waiter me;
    Waiter** at = &line_;
    while (*at) at = &(*at)->next;
    *at = &me;
    const bool in = cv_.wait_for(lk, patience, [&] {
      if (line_ != &me) return false;
      return need > room ? used_ == 0 : used_ + need <= room || (used_ <= room && unissued_ == 0);
    });
    for (at = &line_; *at != &me; at = &(*at)->next) {
    }
    *at = me.next;
    if (in) {
      used_ += need;
      ++unissued_;
    }
    cv_.notify_all();
    return in;
  }
  // Whether more than one thread has come here, this one included.
  bool shared() {
    std::lock_guard<std::mutex> lk(m_);
    note_thread();
    return shared_;
  }
  void issued() {
    std::lock_guard<std::mutex> lk(m_);
    --unissued_;
    cv_.notify_all();
  }
  void leave(int64_t need) {
    std::lock_guard<std::mutex> lk(m_);
    used_ -= need;
    cv_.notify_all();
  }

 private:
  struct Waiter {  // on the waiting thread's stack
    Waiter* next = nullptr;
  };
  void note_thread() {
    const std::thread::id me = std::this_thread::get_id();
    if (first_ == std::thread::id()) first_ = me;
    else if (first_ != me) shared_ = true;
  }
  std::mutex m_;
  std::condition_variable cv_;
  Waiter* line_ = nullptr;
  int64_t used_ = 0;
  int unissued_ = 0;
  std::thread::id first_;
  bool shared_ = false;
};

// A place inside, given back when the solve ends, however it ends.
class ChipPlace {
 public:
  ChipPlace(ChipGate& g, int64_t need, int64_t room, std::chrono::milliseconds patience)
      : g_(g), need_(need), in_(g.enter(need, room, patience)) {}
  ~ChipPlace() {
    issued();
    if (in_) g_.leave(need_);
  }
  ChipPlace(const ChipPlace&) = delete;
  ChipPlace& operator=(const ChipPlace&) = delete;
  bool in() const { return in_; }
  void issued() {
    if (in_ && !issued_) g_.issued();
    issued_ = true;
  }

 private:
  ChipGate& g_;
  const int64_t need_;
  const bool in_;
  bool issued_ = false;
};

}  // namespace gabp
