// Host build of the search's four lanes of a query (the text the search kernel
// includes, query_quad.inc, with the helpers of query_lane.h, learned.h, stree.h
// and curve.h), for running under the address and undefined-behaviour sanitizers.
// A C++ compiler other than the HIP one reads __device__ and __forceinline__ as
// plain inline functions, so the device logic runs here as host code.
//
// The four lanes are four threads.  A lane exchange waits until every lane that
// still works on the query has reached it; a lane that has left gives zero, as a
// lane permutation and a ballot do on the GPU.  What the text relies on ends the
// run if it does not hold: all four lanes take part in every exchange, in the same
// one, and their four places are 0..3 in some order.
//
// Reads one binary job from argv[1], writes every place's index ranges to argv[2].
// Job layout (little-endian, 8-byte words unless noted):
//   n, m, curve, refine, search, refine_min, ball, with_epochs, oldest, epoch,
//   keys[n], q[2m] (f64), delta[m] (f64), with_epochs: qepoch[m] u32,
//   search 1 (learned): xb[4097] u32, rt[65537] u32, lp[4097] (u32 x2),
//     npieces, fk[npieces], pr[npieces] (f64 slope, i32 elo, i32 ehi),
//     ps[npieces + 1] u32, dt[2^20 + 1] u32.
// Output: for each query and each of its 4 places, (b0, e0, b1, e1) u64, and then
// whether it was rejected (u32 per query).
#include <hip/hip_runtime.h>

#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

// Device builtins that the included headers name (unused by the lane code).
static inline float __fmaf_rn(float a, float b, float c) { return std::fma(a, b, c); }
static inline unsigned int __lane_id() { return 0; }

#include "query_lane.h"

using namespace sfc;

static void fail(const char* what, uint64_t j) {
  std::fprintf(stderr, "query %llu: %s\n", (unsigned long long)j, what);
  std::fflush(stderr);
  std::_Exit(4);   // (the other lanes' threads may be waiting)
}

// The lanes of one query: alive until they leave it.
class Quad {
 public:
  void start(uint64_t j) {
    std::unique_lock<std::mutex> g(mu_);
    // The next query begins once every lane has left this one.
    wait_for(g, [&] {
      j_ = j;
      alive_ = 15;
    });
  }
  // Every working lane's word for exchange `kind`; zero for a lane that has left.
  void exchange(int r, int kind, uint64_t v, uint64_t (&all)[4]) {
    std::unique_lock<std::mutex> g(mu_);
    in_[r] = v;
    kind_[r] = kind;
    here_ |= 1u << r;
    const uint64_t gen = gen_;
    if (here_ == alive_) publish();
    cv_.wait(g, [&] { return gen_ != gen; });
    std::memcpy(all, out_, sizeof(all));
  }
  void leave(int r) {
    std::unique_lock<std::mutex> g(mu_);
    alive_ &= ~(1u << r);
    if (here_ != 0 && here_ == alive_) publish();
  }

 private:
  template <typename F>
  void wait_for(std::unique_lock<std::mutex>& g, F set_up) {
    const uint64_t round = round_;
    if (++arrived_ == 4) {
      arrived_ = 0;
      set_up();
      ++round_;
      cv_.notify_all();
    }
    cv_.wait(g, [&] { return round_ != round; });
  }
  void publish() {
    if (here_ != 15) fail("an exchange without all four lanes", j_);
    for (int r = 0; r < 4; ++r) {
      if (kind_[r] != kind_[0]) fail("lanes in different exchanges", j_);
      out_[r] = in_[r];
    }
    here_ = 0;
    ++gen_;
    cv_.notify_all();
  }
  std::mutex mu_;
  std::condition_variable cv_;
  uint32_t alive_ = 0, here_ = 0, arrived_ = 0;
  uint64_t j_ = 0, gen_ = 0, round_ = 0;
  uint64_t in_[4] = {}, out_[4] = {};
  int kind_[4] = {};
};

struct Slots {
  uint64_t b0, e0, b1, e1;
};
static const Slots kUnset = {~0ull, ~0ull, ~0ull, ~0ull};

static Quad g_quad;
static thread_local int t_lane;

template <int X>
uint64_t across(uint64_t v) {
  uint64_t all[4];
  g_quad.exchange(t_lane, X, v, all);
  return all[t_lane ^ X];
}
static uint32_t quad_ballot(bool p) {
  uint64_t all[4];
  g_quad.exchange(t_lane, 0, p ? 1 : 0, all);
  return (uint32_t)(all[0] | all[1] << 1 | all[2] << 2 | all[3] << 3);
}

struct Job {
  const uint16_t* lut;
  const double2* q;
  const double* delta;
  uint64_t m;
  const uint64_t* keys;
  uint64_t n;
  LearnedView lv;
  StreeView sv;
  uint32_t refine_min;
  bool ball;
  RecordPlan record;
  Slots* out;
  uint32_t* rejected;   // per query and lane
};

template <int CURVE, bool REFINE, int SEARCH>
void one_lane(const Job& J, uint64_t j, int r) {
  const uint16_t* lut = J.lut;
  const double2* q = J.q;
  const double* delta = J.delta;
  const uint64_t m = J.m, *keys = J.keys, base = 0, nn = J.n;
  const LearnedView& lv = J.lv;
  const StreeView& sv = J.sv;
  const uint32_t refine_min = J.refine_min;
  const bool ball = J.ball;
  const RecordPlan& record = J.record;
  uint64_t sidx = 4 * j + r;
  uint64_t b0 = 0, e0 = 0, b1 = 0, e1 = 0;
  bool bad = false;
  uint32_t fb = 0, ends = 0;
#include "query_quad.inc"
  (void)fb;
  (void)ends;
  (void)refine_min;
  (void)ball;
  if (sidx < 4 * j || sidx > 4 * j + 3) fail("a place out of range", j);
  J.rejected[4 * j + r] = bad;
  J.out[sidx] = Slots{b0, e0, b1, e1};
}

template <int CURVE, bool REFINE, int SEARCH>
void run_all(const Job& J) {
  std::vector<std::thread> lanes;
  for (int r = 0; r < 4; ++r)
    lanes.emplace_back([&J, r] {
      t_lane = r;
      for (uint64_t j = 0; j < J.m; ++j) {
        g_quad.start(j);
        one_lane<CURVE, REFINE, SEARCH>(J, j, r);
        g_quad.leave(r);
      }
    });
  for (auto& t : lanes) t.join();
}

template <int CURVE, bool REFINE>
void dispatch_search(int search, const Job& J) {
  if (search == 0) run_all<CURVE, REFINE, 0>(J);
  else if (search == 1) run_all<CURVE, REFINE, 1>(J);
  else run_all<CURVE, REFINE, 2>(J);
}

template <typename T>
std::vector<T> take(FILE* f, uint64_t count) {
  std::vector<T> v(count);
  if (count && std::fread(v.data(), sizeof(T), count, f) != count) {
    std::fprintf(stderr, "short job file\n");
    std::exit(2);
  }
  return v;
}

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  FILE* f = std::fopen(argv[1], "rb");
  if (!f) return 2;
  const std::vector<uint64_t> hdr = take<uint64_t>(f, 10);
  const uint64_t n = hdr[0], m = hdr[1];
  const int curve = (int)hdr[2], refine = (int)hdr[3], search = (int)hdr[4];
  const bool with_epochs = hdr[7] != 0;
  // Exactly sized arrays, so that the sanitizer sees any access past them.
  const std::vector<uint64_t> keys = take<uint64_t>(f, n);
  const std::vector<double> qv = take<double>(f, 2 * m);
  const std::vector<double> delta = take<double>(f, m);
  const std::vector<uint32_t> qepoch = take<uint32_t>(f, with_epochs ? m : 0);
  std::vector<double2> q(m);
  for (uint64_t j = 0; j < m; ++j) q[j] = double2{qv[2 * j], qv[2 * j + 1]};
  Job J{};
  J.lut = kHilbertLutConst.v;
  J.q = q.data();
  J.delta = delta.data();
  J.m = m;
  J.keys = keys.data();
  J.n = n;
  J.refine_min = (uint32_t)hdr[5];
  J.ball = hdr[6] != 0;
  if (with_epochs) J.record.qepoch = qepoch.data();
  J.record.oldest = (uint32_t)hdr[8];
  J.record.epoch = (uint32_t)hdr[9];
  std::vector<uint32_t> xb, rt;
  std::vector<uint2> lp;
  std::vector<uint64_t> fk;
  std::vector<PieceRec> pr;
  std::vector<uint32_t> ps, dt;
  if (search == 1) {
    xb = take<uint32_t>(f, kLeaves + 1);
    rt = take<uint32_t>(f, kRouteSlots + 1);
    lp = take<uint2>(f, kLeaves + 1);
    const uint64_t np = take<uint64_t>(f, 1)[0];
    fk = take<uint64_t>(f, np);
    pr = take<PieceRec>(f, np);
    ps = take<uint32_t>(f, np + 1);
    dt = take<uint32_t>(f, kDirectSlots + 1);
    J.lv = LearnedView{xb.data(), rt.data(), lp.data(), fk.data(), pr.data(), ps.data(), dt.data()};
  }
  std::fclose(f);
  // The static search tree: layer k+1 holds the first key of every 16-entry block
  // of layer k, up to a layer of at most 16 entries (each its own array).
  std::vector<std::vector<uint64_t>> layers;
  J.sv.layer[0] = keys.data();
  J.sv.size[0] = n;
  J.sv.top = 0;
  if (search == 2) {
    const std::vector<uint64_t>* below = &keys;
    layers.reserve(kStreeMaxLayers);
    while (below->size() > (size_t)kStreeFan) {
      std::vector<uint64_t> up((below->size() + kStreeFan - 1) / kStreeFan);
      for (size_t b = 0; b < up.size(); ++b) up[b] = (*below)[b * kStreeFan];
      layers.push_back(std::move(up));
      below = &layers.back();
      ++J.sv.top;
      J.sv.layer[J.sv.top] = below->data();
      J.sv.size[J.sv.top] = below->size();
    }
  }
  std::vector<Slots> out(4 * m, kUnset);
  std::vector<uint32_t> lane_rejected(4 * m), rejected(m);
  J.out = out.data();
  J.rejected = lane_rejected.data();
  if (curve == 0 && refine) dispatch_search<0, true>(search, J);
  else if (curve == 0) dispatch_search<0, false>(search, J);
  else if (refine) dispatch_search<1, true>(search, J);
  else dispatch_search<1, false>(search, J);
  for (uint64_t j = 0; j < m; ++j) {
    rejected[j] = lane_rejected[4 * j];
    for (int r = 0; r < 4; ++r) {
      if (std::memcmp(&out[4 * j + r], &kUnset, sizeof(Slots)) == 0) fail("a place not written", j);
      if (lane_rejected[4 * j + r] != rejected[j]) fail("rejected by some of its lanes", j);
    }
  }
  FILE* o = std::fopen(argv[2], "wb");
  if (!o) return 2;
  std::fwrite(out.data(), sizeof(Slots), out.size(), o);
  std::fwrite(rejected.data(), 4, rejected.size(), o);
  std::fclose(o);
  return 0;
}
