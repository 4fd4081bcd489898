// Timing records of kernel launches.
#pragma once
#include <map>
#include <string>
#include <vector>

#include "common.h"

// HIP-event brackets around kernel launches on sampled calls (ROLLOUT_RT_KERNEL_TIMING),
// accumulated per kernel name.
struct KernelTimer {
  bool enabled = false, active = false;
  unsigned stride = 1, calls = 0;
  struct Rec {
    const char* name;
    double bytes, flops;
    hipEvent_t a, b;
  };
  struct Acc {
    uint64_t launches = 0;
    double ms = 0, bytes = 0, flops = 0;
  };
  std::vector<hipEvent_t> pool;
  size_t used = 0;
  std::vector<Rec> pending;
  std::map<std::string, Acc> acc;

  void start_call() { active = enabled && (calls++ % (stride ? stride : 1)) == 0; }
  // A bracket with nothing inside, recorded under the name "(empty bracket)" in mid-stream of a
  // timed call: what two event records cost by themselves, for the reader of the figures
  // to subtract.
  void empty_bracket(hipStream_t s) {
    begin("(empty bracket)", 0, 0, s);
    end(s);
  }
  hipEvent_t get() {
    if (used == pool.size()) {
      hipEvent_t e;
      HIP_TRY(hipEventCreate(&e));
      pool.push_back(e);
    }
    return pool[used++];
  }
  void begin(const char* name, double bytes, double flops, hipStream_t s) {
    if (!active) return;
    Rec r{name, bytes, flops, get(), get()};
    HIP_TRY(hipEventRecord(r.a, s));
    pending.push_back(r);
  }
  void end(hipStream_t s) {
    if (active) HIP_TRY(hipEventRecord(pending.back().b, s));
  }
  void collect() {  // after the stream has been synchronised
    for (Rec& r : pending) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
        Acc& a = acc[r.name];
        a.launches += 1;
        a.ms += ms;
        a.bytes += r.bytes;
        a.flops += r.flops;
      }
    }
    pending.clear();
    used = 0;
    active = false;
  }
  ~KernelTimer() {
    for (hipEvent_t e : pool) (void)hipEventDestroy(e);
  }
};
