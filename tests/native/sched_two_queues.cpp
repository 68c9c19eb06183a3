// CPU test driver of the serving scheduler against an executor whose steps run
// on two queues, one per slot, and may finish in either order, and whose results
// leave on a queue of their own beside the uploads, as the library's do.  Shares
// the queue, the frames and the checks of sched_fake.cpp.
#define main sched_fake_main
#include "sched_fake.cpp"
#undef main

class TwoQueueExec : public ks::Exec {
 public:
  TwoQueueExec(size_t budget, unsigned seed) : owner_(budget / 256, nullptr), rng_(seed) {}
  ~TwoQueueExec() override {
    up_.drain();
    drain();
    down_.drain();
  }
  int slow_us[ks::Scheduler::kSlots] = {0, 0};   // extra time of a slot's steps
  int64_t fail_step_at = -1;                     // the first slow step from here on reports a device error
  int slow_down_us = 0;                          // extra time of a download
  std::atomic<int64_t> steps{0};
  std::atomic<int> newer_first{0};               // steps that ended before an older one
  std::atomic<int> newer_at_fault{0};            // ... that had ended when the failing one did

  bool upload(ks::Frame* f) override {
    FakeFrame* ff = FakeExec::ff_of(f);
    ++ff->pending;
    const size_t off = f->off, bytes = ks::Arena::round(f->bytes);
    up_.push([this, ff, off, bytes]() {
      std::lock_guard<std::mutex> lk(mu_);
      for (size_t g = off / 256; g < (off + bytes) / 256; ++g) {
        FakeFrame* prev = owner_[g];
        CHECK(prev == nullptr || prev == ff || prev->pending.load() == 0, "granule %zu overwritten under frame %llu", g,
              (unsigned long long)prev->id);
        owner_[g] = ff;
      }
      ff->up = true;
      --ff->pending;
    });
    return true;
  }
  Poll upload_state(ks::Frame* f) override { return FakeExec::ff_of(f)->up ? kReady : kNotReady; }

  bool launch(int slot, const std::vector<ks::Slice>& slices) override {
    const int64_t idx = steps++;
    CHECK(done_[slot], "slot %d launched while its step runs", slot);
    done_[slot] = false;
    fault_[slot] = false;
    const bool fault = fail_step_at >= 0 && idx >= fail_step_at && slow_us[slot] > 0;
    if (fault) fail_step_at = -1;
    struct Work {
      FakeFrame* ff;
      size_t off, bytes;
      int64_t first, end;
    };
    std::vector<Work> work;
    for (const ks::Slice& s : slices) {
      ++FakeExec::ff_of(s.f)->pending;
      work.push_back({FakeExec::ff_of(s.f), s.f->off, ks::Arena::round(s.f->bytes), s.first, s.end});
    }
    const int us = slow_us[slot] + int(rng_() % 200);   // (calls come from the worker alone)
    seq_[slot] = idx;
    comp_[slot].push([this, work, slot, us, fault]() {
      std::this_thread::sleep_for(std::chrono::microseconds(us));
      std::lock_guard<std::mutex> lk(mu_);
      for (const Work& w : work) {
        for (size_t g = w.off / 256; g < (w.off + w.bytes) / 256; ++g)
          CHECK(owner_[g] == w.ff, "slice of frame %llu on memory of another", (unsigned long long)w.ff->id);
        for (int64_t p = w.first; p < w.end; ++p) ++w.ff->count[p];
        --w.ff->pending;
      }
      const int other = 1 - slot;
      if (!done_[other] && seq_[other] < seq_[slot]) ++newer_first;
      if (fault && done_[other] && seq_[other] > seq_[slot]) ++newer_at_fault;
      fault_[slot] = fault;
      done_[slot] = true;
    });
    return true;
  }
  Poll step_state(int slot) override { return !done_[slot] ? kNotReady : fault_[slot] ? kError : kReady; }

  bool download(ks::Frame* f) override {
    FakeFrame* ff = FakeExec::ff_of(f);
    for (size_t p = 0; p < ff->count.size(); ++p)
      CHECK(ff->count[p] == 1, "frame %llu downloaded with position %zu computed %d times", (unsigned long long)ff->id, p,
            ff->count[p]);
    ++ff->pending;
    const int us = slow_down_us;
    const size_t off = f->off, bytes = ks::Arena::round(f->bytes);
    down_.push([this, ff, us, off, bytes]() {
      std::this_thread::sleep_for(std::chrono::microseconds(us));
      std::lock_guard<std::mutex> lk(mu_);
      for (size_t g = off / 256; g < (off + bytes) / 256; ++g)
        CHECK(owner_[g] == ff, "results of frame %llu overwritten", (unsigned long long)ff->id);
      ff->downloaded = true;
      ff->down = true;
      --ff->pending;
    });
    return true;
  }
  Poll download_state(ks::Frame* f) override { return FakeExec::ff_of(f)->down ? kReady : kNotReady; }

  void drain() override {
    for (Queue& q : comp_) q.drain();
  }
  void forget(ks::Frame* f) override { f->exec = nullptr; }
  std::string error() override { return "injected device error"; }

 private:
  std::mutex mu_;
  std::vector<FakeFrame*> owner_;
  std::mt19937 rng_;
  std::atomic<int64_t> seq_[ks::Scheduler::kSlots] = {{-1}, {-1}};
  std::atomic<bool> done_[ks::Scheduler::kSlots] = {{true}, {true}};
  std::atomic<bool> fault_[ks::Scheduler::kSlots] = {{false}, {false}};
  Queue up_, down_, comp_[ks::Scheduler::kSlots];
};

// Frames of several steps each: one slot's steps are slow, so that the other's
// end first while both hold slices of the same frame.
void scenario(const char* name, int slow0, int slow1, int64_t fail_at, int slow_down) {
  const size_t budget = size_t(4) << 20;
  TwoQueueExec ex(budget, 7);
  ex.slow_us[0] = slow0;
  ex.slow_us[1] = slow1;
  ex.fail_step_at = fail_at;
  ex.slow_down_us = slow_down;
  ks::Scheduler s(config(budget, 3, 16384), &ex);
  s.start();
  Run r;
  std::mt19937 rng(5);
  for (int i = 0; i < 24; ++i) {
    FakeFrame* ff = new FakeFrame();
    ff->id = uint64_t(i);
    ks::Frame* f = new ks::Frame();
    f->npos = 16 * int64_t(2048 + rng() % 4096);   // two to six steps
    f->pixels = f->npos;
    f->bytes = budget / 4 + rng() % (budget / 4);   // two or three frames fit: ranges are reused at once
    f->exec = ff;
    ff->count.assign(size_t(f->npos), 0);
    uint64_t t = 0;
    std::string err;
    CHECK(s.submit(f, &t, &err) == STAP_OK, "submit failed: %s", err.c_str());
    r.frames.push_back(ff);
    r.tickets.push_back(t);
  }
  int failed = 0;
  for (uint64_t t : r.tickets) {
    double lat = 0;
    std::string err;
    r.status.push_back(s.wait(t, -1, &lat, &err));
    failed += r.status.back() != STAP_OK;
  }
  check_complete(r, name, fail_at < 0);
  if (slow0 != slow1) CHECK(ex.newer_first.load() > 0, "%s: no step ended before an older one", name);
  if (fail_at >= 0) {
    CHECK(failed >= 1 && failed <= 3, "%s: %d frames failed", name, failed);
    CHECK(ex.newer_at_fault.load() == 1, "%s: the newer step had not ended", name);
  }
  s.stop();
  CHECK(s.arena_free() == budget, "%s: arena not free after the run", name);
  free_run(r);
  std::printf("ok %s\n", name);
}

void scenario_poll_wait() {
  CHECK(ks::poll_wait_us(true, true, 0.0) == 10 && ks::poll_wait_us(true, true, 320e-6) == 10, "a short step");
  CHECK(ks::poll_wait_us(true, true, 968e-6) == 30, "1/32 of the time since the last change");
  CHECK(ks::poll_wait_us(true, true, 0.1) == 50 && ks::poll_wait_us(true, true, 1e9) == 50, "a long step");
  CHECK(ks::poll_wait_us(true, false, 0.1) == 200, "a long upload");
  CHECK(ks::poll_wait_us(false, false, 0.0) == 200, "nothing to do");
  std::printf("ok poll_wait\n");
}

int main() {
  scenario_poll_wait();
  scenario("newer_step_first", 3000, 0, -1, 0);
  scenario("newer_step_first_other_slot", 0, 3000, -1, 0);
  scenario("older_step_fails", 0, 20000, 4, 0);
  scenario("older_step_fails_other_slot", 20000, 0, 4, 0);
  scenario("slow_downloads", 0, 0, -1, 4000);
  std::printf("all scenarios passed\n");
  return 0;
}
