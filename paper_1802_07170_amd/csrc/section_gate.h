// Keeps apart, across the streams of a process, the sections of a pass whose workgroups wait for one another.  No device code and
// no HIP: Rt says how a stream waits for an event, so that the rules can be checked with a host compiler.
#pragma once
#include <mutex>

namespace cmt {

// One gate per device.  A section on the stream of one client waits, on the device, for the end of the section before it if that was
// another client's; a client's own sections follow each other on its stream.  Clients (handles) are told apart by themselves
// and not by their streams: hipStreamPerThread is one value for a stream per thread, and a new stream may get the value of
// a destroyed one.  The mutex is held while a section is enqueued.
template <typename Rt>
class SectionGate {
 public:
  struct Client { typename Rt::Event end{}; };         // the event is the caller's
  void enter(Client& c, typename Rt::Stream st) {
    mu_.lock();
    if (last_ && last_ != &c) Rt::wait(st, last_->end);
  }
  void leave(Client& c, typename Rt::Stream st) {
    if (Rt::record(c.end, st)) last_ = &c;
    mu_.unlock();
  }
  // before the client and its event go: its last section has ended by then, so nobody has to wait for it any more
  void remove(Client& c) {
    Rt::finish(c.end);
    std::lock_guard<std::mutex> lock(mu_);
    if (last_ == &c) last_ = nullptr;
  }

 private:
  std::mutex mu_;
  Client* last_ = nullptr;                             // whose section was enqueued last
};

}  // namespace cmt
