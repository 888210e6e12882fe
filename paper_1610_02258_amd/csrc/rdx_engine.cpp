// rdx_engine.cpp -- device arena, run state, the runtime main loop of
// Algorithm 1 as planned sequences of window launches, HIP-graph replay and
// online tuning of the launch shape.
#include "rdx_engine.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace rdx {

namespace {

constexpr size_t kGranule = 256;
inline size_t align_up(size_t x) { return (x + kGranule - 1) & ~(kGranule - 1); }

#define RDX_HIP(call)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess)                                                               \
      return set_error(RDX_EHIP, std::string(#call) + ": " + hipGetErrorString(e_));    \
  } while (0)

template <typename T>
hipError_t dev_alloc(T** p, size_t count) {
  return hipMalloc(reinterpret_cast<void**>(p), sizeof(T) * (count ? count : 1));
}

// The batch step index lives in an int32 on the device; it is brought back
// near zero (keeping its parity, which selects the claim counters) before it
// could pass this.
constexpr int64_t kStepRebase = int64_t(1) << 30;

}  // namespace

// ------------------------------------------------------------------ arena ----
DeviceArena::~DeviceArena() {
  if (base_) (void)hipFree(base_);
}

hipError_t DeviceArena::reserve(size_t bytes) {
  bytes = align_up(bytes ? bytes : kGranule);
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&base_), bytes);
  if (e != hipSuccess) {
    base_ = nullptr;
    return e;
  }
  cap_ = bytes;
  free_.clear();
  used_.clear();
  free_[0] = bytes;
  used_bytes_ = 0;
  return hipSuccess;
}

size_t DeviceArena::alloc(size_t bytes) {
  bytes = align_up(bytes ? bytes : kGranule);
  for (auto it = free_.begin(); it != free_.end(); ++it) {
    if (it->second < bytes) continue;
    const size_t off = it->first, rest = it->second - bytes;
    free_.erase(it);
    if (rest) free_[off + bytes] = rest;
    used_[off] = bytes;
    used_bytes_ += bytes;
    return off;
  }
  return SIZE_MAX;
}

void DeviceArena::release(size_t off) {
  auto u = used_.find(off);
  if (u == used_.end()) return;
  size_t start = off, size = u->second;
  used_bytes_ -= size;
  used_.erase(u);
  auto next = free_.lower_bound(start);
  if (next != free_.end() && next->first == start + size) {
    size += next->second;
    next = free_.erase(next);
  }
  if (next != free_.begin()) {
    auto prev = std::prev(next);
    if (prev->first + prev->second == start) {
      start = prev->first;
      size += prev->second;
      free_.erase(prev);
    }
  }
  free_[start] = size;
}

size_t DeviceArena::largest_free() const {
  size_t m = 0;
  for (const auto& f : free_) m = std::max(m, f.second);
  return m;
}

// ------------------------------------------------------------------ model ----
void listing_pairs(const DevModel& m, int32_t pairs[32], int32_t* n_pairs, int32_t pair_of[32]) {
  int n = 0;
  for (int r = 0; r < 32; ++r) pair_of[r] = -1;
  for (int r = 0; r < m.R; ++r) {
    const int info = m.info[r];
    if ((info & 0xff) != 2) continue;
    const int a = (info >> 8) & 0xff, b = (info >> 16) & 0xff;
    const int key = a | (b << 8) | ((a == b ? 1 : 0) << 16);
    int p = 0;
    while (p < n && pairs[p] != key) ++p;
    if (p == n) pairs[n++] = key;
    pair_of[r] = p;
  }
  for (int p = n; p < 32; ++p) pairs[p] = 0;
  *n_pairs = n;
}

void listing_coefficients(const DevModel& m, const double* k, double* out) {
  int32_t pairs[32], pair_of[32], n_pairs = 0;
  listing_pairs(m, pairs, &n_pairs, pair_of);
  for (int j = 0; j < kLStride; ++j) out[j] = 0.0;
  for (int r = 0; r < m.R; ++r) {
    const int info = m.info[r];
    const int order = info & 0xff, a = (info >> 8) & 0xff, b = (info >> 16) & 0xff;
    if (order == 0) out[0] += k[r];
    else if (order == 1) out[1 + a] += k[r];
    else out[17 + pair_of[r]] += a == b ? 0.5 * k[r] : k[r];
  }
}

// Device image of a run's rate table: [kMaxRegions][32] constants, then
// [kMaxRegions][kLStride] listing coefficients, zero-padded.
static std::vector<double> rate_image(const DevModel& m, const HostInstance& I) {
  std::vector<double> kc((size_t)kMaxRegions * (32 + kLStride), 0.0);
  for (int reg = 0; reg < I.n_regions; ++reg) {
    for (int q = 0; q < I.R; ++q) kc[(size_t)reg * 32 + q] = I.kcst[(size_t)reg * I.R + q];
    listing_coefficients(m, &I.kcst[(size_t)reg * I.R], &kc[(size_t)kMaxRegions * 32 + (size_t)reg * kLStride]);
  }
  return kc;
}

DevModel make_dev_model(const HostInstance& I) {
  DevModel m;
  std::memset(&m, 0, sizeof m);
  m.S = I.S;
  m.R = I.R;
  const int S = I.S, R = I.R;
  for (int r = 0; r < R; ++r) {
    int order = 0, r0 = -1, r1 = -1;
    for (int s = 0; s < S; ++s) {
      const int nu = I.lhs[(size_t)r * S + s];
      order += nu;
      for (int c = 0; c < nu; ++c) {
        if (r0 < 0) r0 = s;
        else r1 = s;
      }
      m.delta[r][s] = (int8_t)(I.rhs[(size_t)r * S + s] - nu);
    }
    const int b0 = r0 < 0 ? 0xff : r0;
    const int b1 = (order == 2 && r1 >= 0) ? r1 : 0xff;
    m.info[r] = order | (b0 << 8) | (b1 << 16);
  }
  return m;
}

// ----------------------------------------------------------------- engine ----
size_t Engine::run_bytes(const HostInstance& I) {
  const size_t T = (size_t)I.T, S = (size_t)I.S;
  size_t b = 2 * align_up(4 * S * T) + align_up(16 * T) + align_up(32 * T) + align_up(8 * T);
  if (I.n_regions > 1) b += align_up(T);
  b += align_up(sizeof(double) * kMaxRegions * (32 + kLStride));  // rate constants, listing coefficients
  b += align_up(sizeof(unsigned long long) * kTallyWords * kTallySlots + sizeof(int32_t));  // tallies, error flag
  return b;
}

void Engine::fence(hipStream_t stream) {
  for (auto& f : fences_)
    if (f.first == stream) {
      (void)hipEventRecord(f.second, stream);
      return;
    }
  hipEvent_t ev = nullptr;
  if (fences_.size() >= 16 || hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
    (void)hipStreamSynchronize(stream);  // too many streams: wait for this one now
    return;
  }
  (void)hipEventRecord(ev, stream);
  fences_.emplace_back(stream, ev);
}

void Engine::drain() {
  for (auto& f : fences_) {
    (void)hipEventSynchronize(f.second);
    (void)hipEventDestroy(f.second);
  }
  fences_.clear();
}

namespace {
// Marks `stream` in the engine's fences when the enclosing method returns,
// whatever it enqueued before an early error return.
struct FenceOnExit {
  Engine* e;
  hipStream_t s;
  ~FenceOnExit() { e->fence(s); }
};
}  // namespace

Engine::~Engine() {
  drain();
  if (staged_) (void)hipEventSynchronize(staged_);
  graphs_.clear([](hipGraphExec_t g) { (void)hipGraphExecDestroy(g); });
  if (capture_stream_) (void)hipStreamDestroy(capture_stream_);
  if (own_) (void)hipStreamDestroy(own_);
  for (hipEvent_t e : marks_) (void)hipEventDestroy(e);
  if (staged_) (void)hipEventDestroy(staged_);
  if (reset_staged_) {
    (void)hipEventSynchronize(reset_staged_);
    (void)hipEventDestroy(reset_staged_);
  }
  if (h_reset_) (void)hipHostFree(h_reset_);
  (void)hipFree(d_reset_);
  for (hipEvent_t e : tune_ev_)
    if (e) (void)hipEventDestroy(e);
  (void)hipFree(model_);
  (void)hipFree(d_runs_);
  (void)hipFree(d_tile_map_);
  (void)hipFree(d_n_tiles_);
  (void)hipFree(d_step_);
  (void)hipFree(tile_ctr_);
  if (h_runs_) (void)hipHostFree(h_runs_);
  if (h_tile_map_) (void)hipHostFree(h_tile_map_);
  if (h_n_tiles_) (void)hipHostFree(h_n_tiles_);
}

void Engine::wait_idle(hipStream_t stream) {
  fence(stream);
  for (auto& f : fences_) (void)hipEventSynchronize(f.second);
}

rdx_status Engine::init(const HostInstance& proto, size_t arena_bytes, int max_runs, int64_t max_tets) {
  if (max_runs < 1 || max_tets < 1 || max_tets > (int64_t)INT32_MAX)
    return set_error(RDX_EINVAL, "engine capacity out of range");
  S_ = proto.S;
  R_ = proto.R;
  model_host_ = make_dev_model(proto);
  max_runs_ = max_runs;
  max_tets_ = max_tets;
  max_tiles_ = (max_tets + 63) / 64 + max_runs;
  if (max_tiles_ > (int64_t)INT32_MAX) return set_error(RDX_EINVAL, "too many tiles");
  if (64 * max_tiles_ > (int64_t)INT32_MAX) return set_error(RDX_EINVAL, "too many tets");
  bool ok = dev_alloc(&model_, 1) == hipSuccess && dev_alloc(&d_runs_, (size_t)max_runs) == hipSuccess &&
            dev_alloc(&d_tile_map_, (size_t)max_tiles_) == hipSuccess &&
            dev_alloc(&d_n_tiles_, 1) == hipSuccess && dev_alloc(&d_step_, 2) == hipSuccess &&
            dev_alloc(&tile_ctr_, (size_t)2 * 8 * kClaimSubs * kCtrStride) == hipSuccess;
  if (ok && arena_bytes) ok = arena_.reserve(arena_bytes) == hipSuccess;
  if (ok) ok = hipHostMalloc(reinterpret_cast<void**>(&h_runs_), sizeof(RunDesc) * (size_t)max_runs) == hipSuccess;
  if (ok) ok = hipHostMalloc(reinterpret_cast<void**>(&h_tile_map_), sizeof(int2) * (size_t)max_tiles_) == hipSuccess;
  if (ok) ok = hipHostMalloc(reinterpret_cast<void**>(&h_n_tiles_), sizeof(int32_t)) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    return set_error(RDX_ENOMEM, "device allocation failed");
  }
  RDX_HIP(hipEventCreateWithFlags(&staged_, hipEventDisableTiming));
  RDX_HIP(hipEventCreate(&tune_ev_[0]));
  RDX_HIP(hipEventCreate(&tune_ev_[1]));
  RDX_HIP(hipStreamCreateWithFlags(&own_, hipStreamNonBlocking));
  RDX_HIP(hipMemcpyAsync(model_, &model_host_, sizeof model_host_, hipMemcpyHostToDevice, own_));
  RDX_HIP(hipMemsetAsync(d_n_tiles_, 0, sizeof(int32_t), own_));
  RDX_HIP(hipMemsetAsync(d_step_, 0, 2 * sizeof(int32_t), own_));
  RDX_HIP(hipMemsetAsync(tile_ctr_, 0, sizeof(int32_t) * 2 * 8 * kClaimSubs * kCtrStride, own_));
  RDX_HIP(hipStreamSynchronize(own_));
  return RDX_OK;
}

bool Engine::compatible(const HostInstance& I) const {
  if (I.S != S_ || I.R != R_) return false;
  const DevModel m = make_dev_model(I);
  return std::memcmp(m.info, model_host_.info, sizeof m.info) == 0 &&
         std::memcmp(m.delta, model_host_.delta, sizeof m.delta) == 0;
}

rdx_status Engine::add_run(Run* r, hipStream_t stream) {
  FenceOnExit fence_on_exit{this, stream};
  const HostInstance& I = r->host;
  if (!compatible(I)) return set_error(RDX_EINVAL, "run does not share the engine's species/reaction structure");
  if (resident_runs_ >= max_runs_ || resident_tets_ + I.T > max_tets_)
    return set_error(RDX_EBUDGET, "engine capacity reached");
  const size_t need = run_bytes(I);
  const size_t off = arena_.alloc(need);
  if (off == SIZE_MAX) return set_error(RDX_EBUDGET, "device arena cannot hold the run now");
  const size_t T = (size_t)I.T, S = (size_t)I.S;
  char* p = arena_.base() + off;
  auto carve = [&p](size_t bytes) {
    char* q = p;
    p += align_up(bytes);
    return q;
  };
  r->arena_off = off;
  r->cnt[0] = reinterpret_cast<int32_t*>(carve(4 * S * T));
  r->cnt[1] = reinterpret_cast<int32_t*>(carve(4 * S * T));
  r->nbr = reinterpret_cast<int32_t*>(carve(16 * T));
  r->geo = reinterpret_cast<double*>(carve(32 * T));
  r->nav = reinterpret_cast<double*>(carve(8 * T));
  r->region = I.n_regions > 1 ? reinterpret_cast<uint8_t*>(carve(T)) : nullptr;
  r->kcst = reinterpret_cast<double*>(carve(sizeof(double) * kMaxRegions * (32 + kLStride)));
  r->lcoef = r->kcst + kMaxRegions * 32;
  const size_t misc_bytes = sizeof(unsigned long long) * kTallyWords * kTallySlots + sizeof(int32_t);
  char* misc = carve(misc_bytes);
  r->tally = reinterpret_cast<unsigned long long*>(misc);
  r->err = reinterpret_cast<int32_t*>(misc + sizeof(unsigned long long) * kTallyWords * kTallySlots);

  // host images of the interleaved couplings and the padded rate table; the
  // copies are synchronous so the images can go when this returns
  std::vector<double> geo(4 * T);
  for (size_t i = 0; i < T; ++i) {
    geo[4 * i + 0] = I.G[i];
    // a share that couplings without a finite sum leave indefinite is below no
    // draw: as a share of 0, everything goes to the last face
    for (size_t k = 0; k < 3; ++k) geo[4 * i + 1 + k] = I.cum[4 * i + k] > 0.0 ? I.cum[4 * i + k] : 0.0;
  }
  const std::vector<double> kc = rate_image(model_host_, I);
  hipError_t e = hipMemcpyAsync(r->nbr, I.nbr.data(), 16 * T, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipMemcpyAsync(r->geo, geo.data(), 32 * T, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipMemcpyAsync(r->nav, I.nav.data(), 8 * T, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess && r->region) e = hipMemcpyAsync(r->region, I.region.data(), T, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipMemcpyAsync(r->kcst, kc.data(), sizeof(double) * kc.size(), hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipMemsetAsync(r->cnt[0], 0, 4 * S * T, stream);
  if (e == hipSuccess) e = hipMemsetAsync(r->cnt[1], 0, 4 * S * T, stream);
  if (e == hipSuccess) e = hipMemsetAsync(misc, 0, misc_bytes, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    arena_.release(off);
    r->arena_off = SIZE_MAX;
    return set_error(RDX_EHIP, std::string("run upload: ") + hipGetErrorString(e));
  }
  r->t = 0.0;
  r->window = r->windows_run = r->voxel_steps = 0;
  resident_runs_ += 1;
  resident_tets_ += I.T;
  return RDX_OK;
}

void Engine::remove_run(Run* r, hipStream_t stream) {
  if (r->arena_off == SIZE_MAX) return;
  // the run's memory may only be reused once no launch can still touch it
  (void)hipStreamSynchronize(stream);
  arena_.release(r->arena_off);
  r->arena_off = SIZE_MAX;
  resident_runs_ -= 1;
  resident_tets_ -= r->host.T;
  tile_runs_.clear();  // the device tile map may name the run
}

rdx_status Engine::reset_run(Run* r, hipStream_t stream) {
  FenceOnExit fence_on_exit{this, stream};
  const size_t n = (size_t)r->host.S * (size_t)r->host.T;
  RDX_HIP(hipMemsetAsync(r->cnt[(r->window + 1) & 1], 0, sizeof(int32_t) * n, stream));
  RDX_HIP(hipMemsetAsync(r->tally, 0, sizeof(unsigned long long) * kTallyWords * kTallySlots, stream));
  RDX_HIP(hipMemsetAsync(r->err, 0, sizeof(int32_t), stream));
  return RDX_OK;
}

rdx_status Engine::reset_runs_device(Run* const* runs, size_t n, const int32_t* const* src, hipStream_t stream) {
  FenceOnExit fence_on_exit{this, stream};
  size_t n_chunks = 0;
  for (size_t j = 0; j < n; ++j) {
    const int64_t e = (int64_t)runs[j]->host.S * runs[j]->host.T;
    n_chunks += (size_t)std::max<int64_t>(1, (e + kResetChunk - 1) / kResetChunk);
  }
  if (n_chunks > (size_t)INT32_MAX) return set_error(RDX_EINVAL, "reset too large");
  if (!reset_staged_) RDX_HIP(hipEventCreateWithFlags(&reset_staged_, hipEventDisableTiming));
  RDX_HIP(hipEventSynchronize(reset_staged_));  // the pinned table may still be in flight
  if (n_chunks > reset_cap_) {
    if (h_reset_) RDX_HIP(hipHostFree(h_reset_));
    if (d_reset_) RDX_HIP(hipFree(d_reset_));
    h_reset_ = nullptr;
    d_reset_ = nullptr;
    reset_cap_ = 0;
    RDX_HIP(hipHostMalloc(reinterpret_cast<void**>(&h_reset_), sizeof(ResetChunk) * n_chunks));
    RDX_HIP(hipMalloc(reinterpret_cast<void**>(&d_reset_), sizeof(ResetChunk) * n_chunks));
    reset_cap_ = n_chunks;
  }
  size_t c = 0;
  for (size_t j = 0; j < n; ++j) {
    Run* r = runs[j];
    if (r->arena_off == SIZE_MAX) return set_error(RDX_ESTATE, "run is not resident");
    r->t = 0.0;
    r->window = r->windows_run = r->voxel_steps = 0;
    const int64_t e = (int64_t)r->host.S * r->host.T;
    for (int64_t b = 0; b == 0 || b < e; b += kResetChunk) {
      ResetChunk& ch = h_reset_[c++];
      ch.src = src[j];
      ch.dst = r->cnt[0];
      ch.other = r->cnt[1];
      ch.tally = r->tally;
      ch.err = r->err;
      ch.begin = b;
      ch.end = std::min<int64_t>(b + kResetChunk, e);
    }
  }
  RDX_HIP(hipMemcpyAsync(d_reset_, h_reset_, sizeof(ResetChunk) * c, hipMemcpyHostToDevice, stream));
  RDX_HIP(hipEventRecord(reset_staged_, stream));
  const hipError_t e = launch_reset_chunks(d_reset_, (int64_t)c, stream);
  if (e != hipSuccess) return set_error(RDX_EHIP, std::string("reset launch: ") + hipGetErrorString(e));
  return RDX_OK;
}

rdx_status Engine::upload_counts(Run* r, const int32_t* counts, bool device, hipStream_t stream) {
  FenceOnExit fence_on_exit{this, stream};
  const size_t n = (size_t)r->host.S * (size_t)r->host.T;
  RDX_HIP(hipMemcpyAsync(r->cnt[r->window & 1], counts, sizeof(int32_t) * n,
                         device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, stream));
  if (!device) RDX_HIP(hipStreamSynchronize(stream));
  return RDX_OK;
}

rdx_status Engine::set_rates(Run* r, const double* kcst, hipStream_t stream) {
  FenceOnExit fence_on_exit{this, stream};
  const size_t n = (size_t)r->host.n_regions * (size_t)r->host.R;
  for (size_t i = 0; i < n; ++i)
    if (!(kcst[i] >= 0.0) || !std::isfinite(kcst[i]))
      return set_error(RDX_EINVAL, "rate constants must be finite and >= 0");
  std::vector<double> old(kcst, kcst + n);
  r->host.kcst.swap(old);
  const std::vector<double> kc = rate_image(model_host_, r->host);
  // stream-ordered: windows already enqueued keep the old constants; the
  // captured window graphs read the table through its pointer and need no
  // re-capture
  hipError_t e = hipMemcpyAsync(r->kcst, kc.data(), sizeof(double) * kc.size(), hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    r->host.kcst.swap(old);  // the host copy keeps describing the device table
    return set_error(RDX_EHIP, std::string("rate table upload: ") + hipGetErrorString(e));
  }
  return RDX_OK;
}

rdx_status Engine::region_counts(const Run* r, unsigned long long* scratch, unsigned long long* out,
                                 hipStream_t stream, bool mark) {
  RDX_HIP(launch_region_counts(r->cnt[r->window & 1], r->region, r->host.T, r->host.S, r->host.n_regions,
                               scratch, out, stream));
  if (mark) fence(stream);
  return RDX_OK;
}

rdx_status Engine::download_counts(const Run* r, int32_t* out, bool device, hipStream_t stream) {
  FenceOnExit fence_on_exit{this, stream};
  const size_t n = (size_t)r->host.S * (size_t)r->host.T;
  RDX_HIP(hipMemcpyAsync(out, r->cnt[r->window & 1], sizeof(int32_t) * n,
                         device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, stream));
  if (!device) RDX_HIP(hipStreamSynchronize(stream));
  return RDX_OK;
}

rdx_status Engine::plan_until(Run* r, double t_end, int64_t max_windows) {
  if (!std::isfinite(t_end)) return set_error(RDX_EINVAL, "t_end must be finite");
  const double tau = r->host.tau;
  double t = r->t;
  // the window index is a 32-bit field of the RNG counter: reject a horizon
  // that needs more windows than are left before counting them one by one
  const int64_t left = (int64_t)0xffffffffLL - r->window;
  const int64_t cap = max_windows < 0 ? left : std::min(max_windows, left + 1);
  if (t < t_end && (max_windows < 0 || max_windows > left)) {
    const double est = (t_end - t) / tau;  // windows to t_end, to within roundings
    if (!(est <= (double)left * (1.0 + 1e-9) + 2.0))
      return set_error(RDX_EINVAL, "window index exceeds the 32-bit RNG counter field");
  }
  int64_t steps = 0, full = 0;
  double tau_last = tau;
  while (t < t_end && steps <= cap && (max_windows < 0 || steps < max_windows)) {
    if (t + tau > t_end) {  // the last window is cut at t_end
      tau_last = t_end - t;
      t = t_end;
      steps += 1;
      break;
    }
    if (!(t + tau > t))  // tau below the resolution of t: the loop would not advance
      return set_error(RDX_EINVAL, "tau is below the floating-point resolution of t");
    t = t + tau;
    steps += 1;
    full += 1;
  }
  if (r->window + steps > (int64_t)0xffffffffLL)
    return set_error(RDX_EINVAL, "window index exceeds the 32-bit RNG counter field");
  r->plan_steps = steps;
  r->plan_full = full;
  r->plan_tau_last = tau_last;
  r->plan_t_after = t;
  return RDX_OK;
}

rdx_status Engine::plan_steps(Run* r, int64_t n) {
  if (n < 0) return set_error(RDX_EINVAL, "n_windows < 0");
  if (r->window + n > (int64_t)0xffffffffLL)
    return set_error(RDX_EINVAL, "window index exceeds the 32-bit RNG counter field");
  double t = r->t;
  for (int64_t k = 0; k < n; ++k) t = t + r->host.tau;
  r->plan_steps = n;
  r->plan_full = n;
  r->plan_tau_last = r->host.tau;
  r->plan_t_after = t;
  return RDX_OK;
}

namespace {
// Tiles of the busiest SIMD when `grid` blocks walk n_tiles in static ranges.
// An XCD has an eighth of both; its block j takes the tiles j, j + blocks, ...
// and lands, in order, on SIMD j mod 128 of its 32 compute units.
int64_t busiest_simd(int64_t n_tiles, int grid) {
  constexpr int64_t kSimds = 128;
  const int64_t tiles = (n_tiles + 7) / 8, blocks = std::max(1, grid / 8);
  int64_t load = 0;
  for (int64_t j = 0; j < blocks && j < tiles; j += kSimds) load += (tiles - j + blocks - 1) / blocks;
  return load;
}

// Grid of static ranges: the fewest rounds of tiles that `resident` blocks
// need, in the fewest blocks (a multiple of the 8 XCDs) for that many rounds;
// more blocks than that where the busiest SIMD then has fewer tiles, the
// fewest that do best.  7,500 tiles of 15 species at 3,072 resident blocks:
// 2,504 blocks make three rounds, and 9 tiles for a SIMD with three of them;
// at 2,752 the third has two rounds to go, 8 tiles: 331 and 270 us a window with
// 20 molecules a species and tet, 77 and 71 with one.  At 8 species (4,096
// resident) 4,578 tiles, 6 or 5 a SIMD, 130 and 109 us, 34 and 32; 15,000 tiles,
// 16 or 15, 303 and 272.
int rounds_grid(int64_t n_tiles, int resident) {
  resident = std::max(8, resident);
  if (n_tiles < 1) return 1;
  const int64_t rounds = (n_tiles + resident - 1) / resident;
  int g = (int)((n_tiles + rounds - 1) / rounds);
  if (g >= 8) g = (g + 7) & ~7;
  if (g > resident) g = resident & ~7;
  if (rounds > 1) {
    int64_t least = busiest_simd(n_tiles, g);
    for (int more = g + 8; more <= resident; more += 8) {
      const int64_t load = busiest_simd(n_tiles, more);
      if (load < least) {
        least = load;
        g = more;
      }
    }
  }
  return g > 0 ? g : 1;
}
}  // namespace

// Tile count rounded up to a coarse bucket (at most 1/8 above it): grids of
// engines whose set of runs changes between sequences (servers, batches
// whose runs finish at different times) then repeat, and so do the captured
// graphs keyed by them.  The kernels read the exact count from the device
// and leave surplus blocks idle.
static int64_t bucket_tiles(int64_t n) {
  if (n <= 64) return n;
  int lg = 0;
  while ((int64_t(1) << (lg + 1)) <= n) ++lg;
  const int64_t g = int64_t(1) << (lg - 3);
  return (n + g - 1) / g * g;
}

// Tets of a tile and grid for n_tiles entries of the tile map.
//
// Tiles of fewer than 64 tets where 64 would leave the device idle: a wave
// then has fewer items and listed tets to go through, at the price of idle
// lanes in its per-tet passes.  Static ranges: 32 or 16 tets while the tiles
// take at most half of the resident blocks (beyond it waves share a SIMD, and
// a second round costs more than the shorter tile saves).  Per window with
// tiles of 64 / 32 / 16 / 8 tets: 2,310 tets 13.9 / 12.8 / 11.8 / 11.8 us,
// 60,000 tets (half of the blocks at 32) 26.8 / 22.9 / 24.0 / 36.3 us,
// 480,000 tets at ten times the density 74 / 89 / 123 / 185 us.  Claimed
// tiles differ in cost, and shorter ones are shared out better: up to 5/4 of
// the resident blocks.  Calcium branch, events crowded in a part of it, 64 / 32
// / 16 tets: 60,000 tets (0.61 and 1.22 times the blocks at 32 and 16) 427 / 258
// / 197 us, 112,000 (1.14, 2.27) 250 / 171 / 179, 160,000 (1.62) 195 / 172 / 200,
// 249,000 (2.53) 151 / 154 / 207.  Beyond the line the crowded loads still gain
// a little and the even ones lose: 150,000 tets of 16 species (1.53), 20
// molecules of each in a tet 124 / 120 us, nearly empty 18.8 / 23.9; 243,000 of 8
// species (1.85) 85 / 97.
//
// Without reactions a tile needs more items than half a wave's lanes: one
// species takes 64 tets, two take 32 (60,000 tets, 20 molecules each: one
// species 15.4 / 16.9 / 22.1 us at 64 / 32 / 16, two 20.8 / 18.1 / 22.2, three
// 25.3 / 22.9 / 23.4; with events a shorter tile has fewer listed tets, and one
// species with two events a tet takes 60.3 / 41.1 / 37.3).
void Engine::cover(int64_t n_tiles_exact, const ExecShape& sh, StepArgs* a) const {
  const int resident = std::max(8, grid_resident(S_, R_) / std::max(1, sh.fast_grid_div));
  const int64_t tiles64 = max_runs_ > 1 ? bucket_tiles(n_tiles_exact) : n_tiles_exact;
  const bool claim = sh.tile_claim != 0;
  const int64_t most = claim ? (int64_t)resident * 5 / 4 : resident / 2;
  a->tile_shift = 6;
  while (a->tile_shift > 4 && (tiles64 << (7 - a->tile_shift)) <= most &&
         (R_ > 0 || (S_ << (a->tile_shift - 1)) > 32))
    --a->tile_shift;
  const int64_t n_tiles = tiles64 << (6 - a->tile_shift);
  a->tile_claim = sh.tile_claim;
  // claimed tiles: every block the device holds, whatever the number of tiles
  if (claim) a->grid = (int)std::max<int64_t>(1, std::min<int64_t>((n_tiles + 7) & ~int64_t(7), resident & ~7));
  else a->grid = rounds_grid(n_tiles, resident);
}

rdx_status Engine::upload_tables(const std::vector<Run*>& active, int64_t k0, hipStream_t stream,
                                 int64_t* n_tiles_out) {
  // the pinned images may still be in flight from the previous sequence
  RDX_HIP(hipEventSynchronize(staged_));
  const size_t n = active.size();
  for (size_t j = 0; j < n; ++j) {
    const Run* r = active[j];
    const HostInstance& I = r->host;
    RunDesc& d = h_runs_[j];
    std::memset(&d, 0, sizeof d);
    d.cnt[0] = r->cnt[0];
    d.cnt[1] = r->cnt[1];
    d.nbr = r->nbr;
    d.geo = r->geo;
    d.nav = r->nav;
    d.region = r->region;
    d.kcst = r->kcst;
    d.lcoef = r->lcoef;
    d.tally = r->tally;
    d.err = r->err;
    d.T = I.T;
    d.n_steps = (int32_t)(k0 + r->plan_steps);
    d.n_full = (int32_t)(k0 + r->plan_full);
    d.window0 = (uint32_t)((uint64_t)r->window - (uint64_t)k0);
    d.key0 = (uint32_t)(r->seed & 0xffffffffu);
    d.key1 = (uint32_t)(r->seed >> 32);
    d.tau = I.tau;
    d.tau_last = r->plan_tau_last;
    for (int s = 0; s < I.S; ++s) {
      d.D[s] = I.D[s];
      if (I.D[s] > 0.0) d.dmask |= 1u << s;
    }
  }
  RDX_HIP(hipMemcpyAsync(d_runs_, h_runs_, sizeof(RunDesc) * n, hipMemcpyHostToDevice, stream));
  // tile map: rebuilt only when the set of runs changes
  bool same = tile_runs_.size() == n;
  for (size_t j = 0; same && j < n; ++j) same = tile_runs_[j] == active[j] && tile_run_T_[j] == active[j]->host.T;
  int64_t n_tiles = 0;
  for (const Run* r : active) n_tiles += (r->host.T + 63) / 64;
  if (n_tiles > max_tiles_) return set_error(RDX_EINVAL, "tile map capacity exceeded");
  if (!same) {
    int64_t t = 0;
    for (size_t j = 0; j < n; ++j)
      for (int32_t first = 0; first < active[j]->host.T; first += 64) h_tile_map_[t++] = make_int2((int)j, first);
    RDX_HIP(hipMemcpyAsync(d_tile_map_, h_tile_map_, sizeof(int2) * (size_t)n_tiles, hipMemcpyHostToDevice, stream));
    tile_runs_.assign(active.begin(), active.end());
    tile_run_T_.resize(n);
    for (size_t j = 0; j < n; ++j) tile_run_T_[j] = active[j]->host.T;
  }
  *h_n_tiles_ = (int32_t)n_tiles;
  RDX_HIP(hipMemcpyAsync(d_n_tiles_, h_n_tiles_, sizeof(int32_t), hipMemcpyHostToDevice, stream));
  *n_tiles_out = n_tiles;
  RDX_HIP(hipEventRecord(staged_, stream));
  return RDX_OK;
}

rdx_status Engine::launch_plain(const StepArgs& a0, int64_t step0, int64_t K, hipStream_t stream) {
  StepArgs a = a0;
  for (int64_t k = 0; k < K; ++k) {
    a.step = (int32_t)(step0 + k);
    a.parity = a.step & 1;
    hipEvent_t* marks = nullptr;
    if (timing_) {
      while (marks_.size() < marks_used_ + 2) {
        hipEvent_t ev;
        RDX_HIP(hipEventCreate(&ev));
        marks_.push_back(ev);
      }
      marks = marks_.data() + marks_used_;
      marks_used_ += 2;
    }
    hipError_t e = launch_window(a, stream, marks);
    if (e != hipSuccess) return set_error(RDX_EHIP, std::string("window launch: ") + hipGetErrorString(e));
    k_now_ = step0 + k + 1;
    if (rec_on_ && (k + 1) % rec_.every == 0) {
      // the counts after this window sit in buffer (window + k + 1) & 1 (the
      // run's window index advances when the sequence ends); the next window
      // clears that buffer only after this reduction in stream order
      const Run* r = rec_.run;
      const int64_t slot = (int64_t)r->host.n_regions * r->host.S;
      unsigned long long* out = rec_.ring + (rec_.records % rec_.slots) * slot;
      e = launch_region_counts(r->cnt[(r->window + k + 1) & 1], r->region, r->host.T, r->host.S,
                               r->host.n_regions, rec_.scratch, out, stream);
      if (e != hipSuccess) return set_error(RDX_EHIP, std::string("record launch: ") + hipGetErrorString(e));
      rec_.records += 1;
    }
  }
  return RDX_OK;
}

rdx_status Engine::launch_graphs(const StepArgs& a0, int64_t step0, int64_t reps, bool replay, hipStream_t stream) {
  const int W = shape_.graph_windows;
  const int parity = (int)(step0 & 1);
  const int n = (W & 1) != 0 && reps > 1 ? 2 : 1;  // graphs of an odd length alternate
  GraphCache<hipGraphExec_t>::Key keys[2];
  for (int j = 0; j < n; ++j)
    // everything of the arguments that can change between sequences is in the
    // key (pointers and tables are fixed for the engine's life)
    keys[j] = {W, ((long long)a0.grid << 6) | ((long long)a0.tile_shift << 3) | ((long long)(a0.tile_claim ? 1 : 0) << 2) |
                      ((long long)(parity ^ j) << 1) | (long long)a0.single_run};
  // W windows, captured once on a private stream; each reads its step index
  // from the word that the window before it wrote
  auto capture = [&](int j, hipGraphExec_t* exec) -> int {
    if (!capture_stream_) RDX_HIP(hipStreamCreateWithFlags(&capture_stream_, hipStreamNonBlocking));
    StepArgs a = a0;
    a.step = -1;
    RDX_HIP(hipStreamBeginCapture(capture_stream_, hipStreamCaptureModeThreadLocal));
    hipError_t e = hipSuccess;
    for (int k = 0; k < W && e == hipSuccess; ++k) {
      a.parity = (parity + j + k) & 1;
      e = launch_window(a, capture_stream_, nullptr);
    }
    hipGraph_t graph = nullptr;
    hipError_t e2 = hipStreamEndCapture(capture_stream_, &graph);
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess) e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
    if (graph) (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return set_error(RDX_EHIP, std::string("graph capture: ") + hipGetErrorString(e));
    return RDX_OK;
  };
  hipGraphExec_t execs[2] = {nullptr, nullptr};
  const int st = graphs_.take(keys, n, execs, capture, [&] { wait_idle(stream); },
                              [](hipGraphExec_t g) { (void)hipGraphExecDestroy(g); });
  if (st != RDX_OK) return (rdx_status)st;
  for (int64_t r = 0; replay && r < reps; ++r) {
    RDX_HIP(hipGraphLaunch(execs[n == 2 ? r & 1 : 0], stream));
    k_now_ = step0 + (r + 1) * W;
  }
  return RDX_OK;
}

void Engine::set_autotune(bool on) {
  tuning_ = on;
  candidates_.clear();
  cand_ms_.clear();
  cand_next_ = 0;
  if (!on) return;
  // the first entry is a warm-up of the default shape and is not scored;
  // then every shape three times, in three passes, each scored by its best
  // pass, so that a drift of the per-window cost over the tuning windows (a
  // simulation relaxing from its initial counts) biases the choice less
  // (with two passes the batched ensemble settled on a shape 3.7% slower)
  const ExecShape shapes[] = {ExecShape{1, 1, 4}, ExecShape{2, 1, 4},       ExecShape{1, 8, 4},      ExecShape{2, 8, 4},
                              ExecShape{4, 8, 4}, ExecShape{1, 1, 4, 1, 1}, ExecShape{1, 8, 4, 1, 1}};
  candidates_.push_back(shapes[0]);
  for (int pass = 0; pass < 3; ++pass)
    for (const ExecShape& c : shapes) candidates_.push_back(c);
}

rdx_status Engine::sequence(const std::vector<Run*>& runs, hipStream_t stream) {
  FenceOnExit fence_on_exit{this, stream};
  std::vector<Run*> active;
  int64_t K = 0;
  for (Run* r : runs)
    if (r->plan_steps > 0) {
      if (r->arena_off == SIZE_MAX) return set_error(RDX_ESTATE, "run is not resident");
      active.push_back(r);
      K = std::max(K, r->plan_steps);
    }
  if (active.empty()) return RDX_OK;
  if ((int)active.size() > max_runs_) return set_error(RDX_EINVAL, "too many runs in one sequence");

  int64_t k0 = k_now_;
  if (k0 + K >= kStepRebase) {
    if (K >= kStepRebase) return set_error(RDX_EINVAL, "sequence too long");
    k0 = k_now_ & 1;  // keep the parity of the claim counters
    RDX_HIP(launch_set_step(d_step_, (int32_t)k0, stream));
    k_now_ = k0;
  }
  int64_t n_tiles = 0;
  rdx_status st = upload_tables(active, k0, stream, &n_tiles);
  if (st != RDX_OK) return st;

  StepArgs a;
  std::memset(&a, 0, sizeof a);
  a.runs = d_runs_;
  a.tile_map = d_tile_map_;
  a.n_tiles = d_n_tiles_;
  a.step_words = d_step_;
  a.S = S_;
  a.R = R_;
  a.model = model_;
  {
    int32_t pair_of[32];
    listing_pairs(model_host_, a.pairs, &a.n_pairs, pair_of);
  }
  a.single_run = active.size() == 1 ? 1 : 0;
  a.tile_ctr = tile_ctr_;

  // n windows from step `at` of the sequence at launch shape `sh`
  auto run_chunk = [&](const ExecShape& sh, int64_t at, int64_t n) -> rdx_status {
    cover(n_tiles, sh, &a);
    const ExecShape keep = shape_;
    shape_ = sh;
    rdx_status r = RDX_OK;
    int64_t in_graphs = 0;
    if (!timing_ && sh.graph_windows > 1 && n >= sh.graph_windows) {
      in_graphs = n / sh.graph_windows * sh.graph_windows;
      r = launch_graphs(a, k0 + at, n / sh.graph_windows, true, stream);
    }
    if (r == RDX_OK) r = launch_plain(a, k0 + at + in_graphs, n - in_graphs, stream);
    shape_ = keep;
    return r;
  };

  int64_t done = 0;
  if (rec_on_) {  // records between windows: plain launches at the current shape
    cover(n_tiles, shape_, &a);
    st = launch_plain(a, k0, K, stream);
    if (st != RDX_OK) return st;
    done = K;
  }
  while (tuning_ && !timing_ && done < K && cand_next_ < candidates_.size()) {
    const ExecShape c = candidates_[cand_next_];
    const int64_t n = std::min<int64_t>(K - done, std::max(8, 2 * c.graph_windows));
    if (c.graph_windows > 1 && n >= c.graph_windows) {  // capture outside the timed span
      cover(n_tiles, c, &a);
      const ExecShape keep = shape_;
      shape_ = c;
      st = launch_graphs(a, k0 + done, n / c.graph_windows, false, stream);
      shape_ = keep;
      if (st != RDX_OK) return st;
    }
    RDX_HIP(hipEventRecord(tune_ev_[0], stream));
    st = run_chunk(c, done, n);
    if (st != RDX_OK) return st;
    RDX_HIP(hipEventRecord(tune_ev_[1], stream));
    RDX_HIP(hipEventSynchronize(tune_ev_[1]));
    float ms = 0.f;
    RDX_HIP(hipEventElapsedTime(&ms, tune_ev_[0], tune_ev_[1]));
    if (cand_next_ > 0) {
      const double per = (double)ms / (double)n;
      auto f = cand_ms_.find(c);
      cand_ms_[c] = f == cand_ms_.end() ? per : std::min(f->second, per);
    }
    done += n;
    cand_next_ += 1;
    if (cand_next_ == candidates_.size()) {
      ExecShape best = candidates_[0];
      double best_ms = 1e300;
      for (const auto& kv : cand_ms_)
        if (kv.second < best_ms) {
          best_ms = kv.second;
          best = kv.first;
        }
      shape_ = best;
      tuning_ = false;
    }
  }
  if (done < K) {
    st = run_chunk(shape_, done, K - done);
    if (st != RDX_OK) return st;
  }

  for (Run* r : active) {
    r->t = r->plan_t_after;
    r->window += r->plan_steps;
    r->windows_run += r->plan_steps;
    r->voxel_steps += r->plan_steps * (int64_t)r->host.T;
    r->plan_steps = r->plan_full = 0;
  }
  return RDX_OK;
}

rdx_status Engine::kernel_times(rdx_kernel_times* out, bool reset) {
  for (size_t k = 0; k + 2 <= marks_used_; k += 2) {
    RDX_HIP(hipEventSynchronize(marks_[k + 1]));
    float ms = 0.f;
    RDX_HIP(hipEventElapsedTime(&ms, marks_[k], marks_[k + 1]));
    main_ms_ += ms;
    timed_windows_ += 1;
  }
  marks_used_ = 0;
  out->windows = timed_windows_;
  out->detect_ms = 0.0;  // the listing is part of the window kernel
  out->main_ms = main_ms_;
  if (reset) {
    timed_windows_ = 0;
    main_ms_ = 0.0;
  }
  return RDX_OK;
}

rdx_status Engine::run_error(const Run* r) const {
  // on the engine's own stream: a copy on the legacy default stream is refused
  // while any other thread holds a blocking stream in graph capture
  int32_t flags = 0;
  RDX_HIP(hipMemcpyAsync(&flags, r->err, sizeof flags, hipMemcpyDeviceToHost, own_));
  RDX_HIP(hipStreamSynchronize(own_));
  if (flags & kErrOverflow) return set_error(RDX_EOVERFLOW, "a molecule count passed 2^30");
  if (flags & kErrEvents) return set_error(RDX_EEVENTS, "more than 2^22 SSA events in one tet window");
  return RDX_OK;
}

rdx_status Engine::read_run_async(const Run* r, Readout* out, hipStream_t stream) const {
  RDX_HIP(hipMemcpyAsync(&out->err, r->err, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
  RDX_HIP(hipMemcpyAsync(out->slots, r->tally, sizeof out->slots, hipMemcpyDeviceToHost, stream));
  return RDX_OK;
}

rdx_status Engine::decode_readout(const Readout& in, unsigned long long tal[3]) {
  tal[0] = tal[1] = tal[2] = 0;
  for (int j = 0; j < kTallySlots; ++j)
    for (int q = 0; q < 3; ++q) tal[q] += in.slots[kTallyWords * j + q];
  if (in.err & kErrOverflow) return set_error(RDX_EOVERFLOW, "a molecule count passed 2^30");
  if (in.err & kErrEvents) return set_error(RDX_EEVENTS, "more than 2^22 SSA events in one tet window");
  return RDX_OK;
}

rdx_status Engine::run_tally(const Run* r, unsigned long long tal[3]) const {
  unsigned long long slots[kTallyWords * kTallySlots];
  RDX_HIP(hipMemcpyAsync(slots, r->tally, sizeof slots, hipMemcpyDeviceToHost, own_));
  RDX_HIP(hipStreamSynchronize(own_));
  tal[0] = tal[1] = tal[2] = 0;
  for (int j = 0; j < kTallySlots; ++j)
    for (int q = 0; q < 3; ++q) tal[q] += slots[kTallyWords * j + q];
  return RDX_OK;
}

}  // namespace rdx
