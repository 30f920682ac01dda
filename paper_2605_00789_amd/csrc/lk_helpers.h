// Helper streams of the library (host side).  Some calls run independent halves side by side: they fork from the
// caller's stream onto helper streams and rejoin it before they return.  The helpers are host-side handles, kept per
// device in small pools, created on first need outside stream capture at default priority and never destroyed.
//
// Why pools: while a caller's stream is being captured into a graph, a helper stream that forked from it belongs to
// that capture until the caller ends it -- long after the call has returned.  Another caller (eager, or capturing
// a graph of its own) must not touch that helper meanwhile, or the capture is invalidated.  So a call takes a set
// whose streams are idle, or already part of the caller's own capture; if every set is held by other captures and
// no new one can be made (pool full, or the caller itself is capturing), the call gets none and enqueues everything
// on the caller's stream in order.
#pragma once
#include <hip/hip_runtime.h>
#include <mutex>

namespace lk {

constexpr int HELPER_SETS_PER_DEVICE = 4;
constexpr int HELPER_MAX_DEVICES = 64;

// TAG: a pool of its own (a call that holds a set of one pool may call into another that takes a set of a second one)
template <int N_STREAMS, int N_EVENTS, int TAG = 0>
struct HelperSet {
  hipStream_t stream[N_STREAMS] = {};
  hipEvent_t event[N_EVENTS] = {};
  bool ready = false;
  std::mutex in_use;   // one caller at a time enqueues its fork ... join sequence on a set
};

// Returns a usable set for a call on `main` with `guard` holding its in_use mutex, or nullptr (then: no helpers).
template <int N_STREAMS, int N_EVENTS, int TAG = 0>
HelperSet<N_STREAMS, N_EVENTS, TAG> *acquire_helpers(hipStream_t main, std::unique_lock<std::mutex> &guard) {
  using Set = HelperSet<N_STREAMS, N_EVENTS, TAG>;
  static Set pool[HELPER_MAX_DEVICES][HELPER_SETS_PER_DEVICE];
  static std::mutex mu[HELPER_MAX_DEVICES];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= HELPER_MAX_DEVICES) return nullptr;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  unsigned long long cid = 0;
  if (hipStreamGetCaptureInfo(main, &cs, &cid) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
  const bool capturing = cs != hipStreamCaptureStatusNone;
  std::lock_guard<std::mutex> lock(mu[dev]);
  for (int k = 0; k < HELPER_SETS_PER_DEVICE; ++k) {
    Set &h = pool[dev][k];
    if (!h.ready) {
      if (capturing) continue;   // never create objects while the caller is capturing
      bool ok = true;
      int ns = 0, ne = 0;
      for (; ok && ns < N_STREAMS; ++ns) ok = hipStreamCreateWithFlags(&h.stream[ns], hipStreamNonBlocking) == hipSuccess;
      for (; ok && ne < N_EVENTS; ++ne) ok = hipEventCreateWithFlags(&h.event[ne], hipEventDisableTiming) == hipSuccess;
      if (!ok) {   // give back what was made; the slot stays empty and is tried again by a later call
        (void)hipGetLastError();
        for (int i = 0; i < N_STREAMS; ++i) if (h.stream[i]) { (void)hipStreamDestroy(h.stream[i]); h.stream[i] = nullptr; }
        for (int i = 0; i < N_EVENTS; ++i) if (h.event[i]) { (void)hipEventDestroy(h.event[i]); h.event[i] = nullptr; }
        (void)hipGetLastError();
        return nullptr;
      }
      h.ready = true;
    }
    // idle, or already part of this caller's capture?
    std::unique_lock<std::mutex> g(h.in_use, std::try_to_lock);
    if (!g.owns_lock()) {
      // another host thread is enqueueing on it right now: wait for it only if it is the last resort
      if (k + 1 < HELPER_SETS_PER_DEVICE) continue;
      g.lock();
    }
    bool usable = true;
    for (int i = 0; usable && i < N_STREAMS; ++i) {
      hipStreamCaptureStatus hs = hipStreamCaptureStatusNone;
      unsigned long long hid = 0;
      if (hipStreamGetCaptureInfo(h.stream[i], &hs, &hid) != hipSuccess) { (void)hipGetLastError(); usable = false; break; }
      if (hs != hipStreamCaptureStatusNone && !(capturing && hid == cid)) usable = false;
    }
    if (!usable) continue;
    guard = std::move(g);
    return &h;
  }
  return nullptr;
}

// A small block of pinned host memory that a kernel of one call writes to while the host of that call waits: per device a
// pool of MAILBOXES_PER_DEVICE, each allocated on first need and kept for the life of the process (8 KB).  A call holds
// one for itself; with none free (more calls at once than there are) or none to be had the caller copies instead.
constexpr int MAILBOXES_PER_DEVICE = 4;
constexpr int MAILBOX_WORDS = 1024;
struct Mailbox {
  unsigned long long *words = nullptr;
  unsigned tag = 0;      // the last tag handed out; words start as zero, no tag is zero
  std::mutex in_use;
  unsigned next_tag() { return tag = tag + 1 ? tag + 1 : 1; }
};
inline Mailbox *acquire_mailbox(int n_words, std::unique_lock<std::mutex> &guard) {
  static Mailbox pool[HELPER_MAX_DEVICES][MAILBOXES_PER_DEVICE];
  int dev = 0;
  if (n_words > MAILBOX_WORDS || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= HELPER_MAX_DEVICES) return nullptr;
  for (int k = 0; k < MAILBOXES_PER_DEVICE; ++k) {
    Mailbox &m = pool[dev][k];
    std::unique_lock<std::mutex> g(m.in_use, std::try_to_lock);
    if (!g.owns_lock()) continue;
    if (!m.words) {
      void *p = nullptr;
      if (hipHostMalloc(&p, sizeof(unsigned long long) * MAILBOX_WORDS, hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess || !p) {
        (void)hipGetLastError();
        return nullptr;
      }
      m.words = static_cast<unsigned long long *>(p);
      for (int i = 0; i < MAILBOX_WORDS; ++i) m.words[i] = 0;
    }
    guard = std::move(g);
    return &m;
  }
  return nullptr;
}

}  // namespace lk
