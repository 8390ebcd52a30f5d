// Keeps apart, across the streams of a process, the sections of a pass whose workgroups wait for one another.  No device code and
// no HIP: Rt says how a stream waits for an event, so that the rules can be checked with a host compiler.
#pragma once
#include <condition_variable>
#include <mutex>
#include <vector>

namespace cmt {

// One gate per device.  Two kinds of sections: those that may need every CU (a loop of more workgroups than a recurrence's group
// has: `alone`), and those that get on beside others of their kind (recur_plan.h).  On the device, one that runs alone waits for the
// end of every section before it, and any section for the end of the last one that ran alone; sections that may share the chip
// do not wait for one another.  A client's own sections follow each other on its stream anyway.
// Clients (handles) are told apart by themselves and not by their streams: hipStreamPerThread is one value for a stream per
// thread, and a new stream may get the value of a destroyed one.
// On the host, a section that runs alone is enqueued while no other one is; the others at any time between those.
template <typename Rt>
class SectionGate {
 public:
  struct Client {
    typename Rt::Event shared{}, alone{};              // the ends of its last sections of either kind; the events are the caller's
    bool pending = false;                              // its last shared section is one that the next one alone has to wait for
    typename Rt::Stream stream{};                      // where its sections go, as far as the value tells
  };
  void add(Client& c, typename Rt::Stream st) {
    std::lock_guard<std::mutex> lock(mu_);
    c.stream = st;
    clients_.push_back(&c);
  }
  // Whether there are others that short sections leave more room: some on another stream.  (Several streams of one value are
  // taken for one here: their sections are then longer than they need be, no more.)
  bool crowded(const Client& c) {
    std::lock_guard<std::mutex> lock(mu_);
    for (const Client* p : clients_)
      if (p->stream != c.stream) return true;
    return false;
  }
  void enter(Client& c, typename Rt::Stream st, bool alone) {
    std::unique_lock<std::mutex> lock(mu_);
    if (alone) {
      ++queued_;
      free_.wait(lock, [&] { return !alone_ && sharing_ == 0; });
      --queued_;
      alone_ = true;
      for (Client* p : pending_)
        if (p != &c) Rt::wait(st, p->shared);
    } else {
      free_.wait(lock, [&] { return !alone_ && queued_ == 0; });
      ++sharing_;
    }
    if (last_ && last_ != &c) Rt::wait(st, last_->alone);
  }
  void leave(Client& c, typename Rt::Stream st, bool alone) {
    std::lock_guard<std::mutex> lock(mu_);
    if (alone) {
      if (Rt::record(c.alone, st)) {                   // whoever waits for this one has waited for those before it
        last_ = &c;
        for (Client* p : pending_) p->pending = false;
        pending_.clear();
      }
      alone_ = false;
    } else {
      if (Rt::record(c.shared, st) && !c.pending) { c.pending = true; pending_.push_back(&c); }
      --sharing_;
    }
    free_.notify_all();
  }
  // before the client and its events go: its sections have ended by then, so nobody has to wait for them any more
  void remove(Client& c) {
    Rt::finish(c.shared);
    Rt::finish(c.alone);
    std::unique_lock<std::mutex> lock(mu_);
    free_.wait(lock, [&] { return !alone_; });
    if (last_ == &c) last_ = nullptr;
    for (std::vector<Client*>* v : {&clients_, &pending_})
      for (size_t i = 0; i < v->size(); ++i)
        if ((*v)[i] == &c) { (*v)[i] = v->back(); v->pop_back(); break; }
  }

 private:
  std::mutex mu_;
  std::condition_variable free_;
  std::vector<Client*> clients_;
  int queued_ = 0, sharing_ = 0;                       // sections being enqueued on the host: waiting to run alone, sharing,
  bool alone_ = false;                                 // alone
  Client* last_ = nullptr;                             // whose section ran alone last
  std::vector<Client*> pending_;                       // those with a shared section since
};

}  // namespace cmt
