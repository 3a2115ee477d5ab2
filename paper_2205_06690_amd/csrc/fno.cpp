// Fourier-operator screening surrogate: parameters, buffers, forward,
// backward and Adam behind the bse_fno_* C-ABI.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <random>
#include <string>
#include <system_error>
#include <thread>
#include <vector>

#include "../../include/bse.h"
#include "fno_kernels.h"

using namespace bse;

namespace {

thread_local std::string f_err;
struct FFail {
  bse_status st;
};
void ffail(bse_status st, const std::string& m) {
  f_err = m;
  throw FFail{st};
}
void fchk(hipError_t e, const char* what) {
  if (e != hipSuccess) {
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation)
      ffail(BSE_ERR_OOM, std::string(what) + ": " + hipGetErrorString(e));
    ffail(BSE_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
  }
}
#define FCK(x) fchk((x), #x)

struct Buf {
  void* p = nullptr;
  size_t bytes = 0;
  void alloc(size_t n) {
    if (p && n <= bytes) return;
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
    if (n == 0) return;
    FCK(hipMalloc(&p, n));
    bytes = n;
  }
  ~Buf() {
    if (p) (void)hipFree(p);
  }
  float* f() const { return reinterpret_cast<float*>(p); }
  float2* c() const { return reinterpret_cast<float2*>(p); }
  double* d() const { return reinterpret_cast<double*>(p); }
};

// Copies regions of a device array to pageable host memory while later kernels
// still compute other regions: a stream of its own brings chunks into pinned
// slots, a few threads move them on.  A plain pageable copy of the 67 MB
// gradient of the 64^3 network took 6.5 ms after the last kernel (10 GB/s, one
// thread touching new pages); the chunks overlap the backward pass and leave
// 0.9 ms (8 samples, loss and gradient: 10.1 -> 4.3 ms).  Threads live for one copy, the slots (12 MB) as long as the object.
class HostCopy {
 public:
  static constexpr size_t CHUNK = 1 << 20, MIN_BYTES = 4 << 20;
  static constexpr int SLOTS = 12, THREADS = 8;
  struct Region {
    size_t off, len;     // bytes
    hipEvent_t ready;    // its last kernel
  };

  ~HostCopy() {
    for (auto& e : arrived_)
      if (e) (void)hipEventDestroy(e);
    for (auto& e : ready_) (void)hipEventDestroy(e);
    if (st_) (void)hipStreamDestroy(st_);
    if (pin_) (void)hipHostFree(pin_);
  }

  // on the object's device, whichever is current: events for that many regions;
  // false where the pinned memory is not to be had (the caller then copies as
  // before)
  bool prepare(int device, int regions) {
    struct Device {
      int was = -1;
      ~Device() {
        if (was >= 0) (void)hipSetDevice(was);
      }
    } dev;
    int cur = 0;
    FCK(hipGetDevice(&cur));
    if (cur != device) {
      FCK(hipSetDevice(device));
      dev.was = cur;
    }
    if (!pin_ && hipHostMalloc(reinterpret_cast<void**>(&pin_), CHUNK * SLOTS, hipHostMallocDefault) != hipSuccess) {
      pin_ = nullptr;
      (void)hipGetLastError();
      return false;
    }
    if (!st_) FCK(hipStreamCreateWithFlags(&st_, hipStreamNonBlocking));
    for (auto& e : arrived_)
      if (!e) FCK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    while ((int)ready_.size() < regions) {
      hipEvent_t e;
      FCK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
      ready_.push_back(e);
    }
    return true;
  }
  hipEvent_t ready(int k) const { return ready_[k]; }

  // every region is in dst on return
  void copy(const std::vector<Region>& regions, const char* src, char* dst) {
    struct Chunk {
      size_t off, len;
      hipEvent_t after;   // nullable: the region's first chunk
    };
    std::vector<Chunk> chunks;
    for (const Region& r : regions)
      for (size_t o = 0; o < r.len; o += CHUNK)
        chunks.push_back({r.off + o, std::min(CHUNK, r.len - o), o ? nullptr : r.ready});
    const int nc = (int)chunks.size();
    // chunk c sits in slot c mod SLOTS; chunks are handed over in order, any
    // thread takes the next one
    std::mutex mu;
    std::condition_variable work, freed;
    int handed = 0, taken = 0;
    bool stop = false;
    std::vector<char> moved(nc, 0);
    auto worker = [&]() {
      std::unique_lock<std::mutex> lk(mu);
      for (;;) {
        work.wait(lk, [&]() { return stop || taken < handed; });
        if (taken >= handed) return;
        const int c = taken++;
        lk.unlock();
        std::memcpy(dst + chunks[c].off, pin_ + (size_t)(c % SLOTS) * CHUNK, chunks[c].len);
        lk.lock();
        moved[c] = 1;
        freed.notify_one();
      }
    };
    struct Joiner {   // also on the way out of an error
      std::mutex& mu;
      std::condition_variable& work;
      bool& stop;
      std::vector<std::thread> t;
      ~Joiner() {
        {
          std::lock_guard<std::mutex> lk(mu);
          stop = true;
        }
        work.notify_all();
        for (auto& x : t) x.join();
      }
    } pool{mu, work, stop, {}};
    struct Drain {    // no copy into the slots outlives the call
      hipStream_t st;
      ~Drain() { (void)hipStreamSynchronize(st); }
    } drain{st_};
    pool.t.reserve(THREADS);
    try {
      for (int i = 0; i < std::min(THREADS, nc); ++i) pool.t.emplace_back(worker);
    } catch (const std::system_error&) {   // no more threads: with those there are, or alone
    }
    int issued = 0;
    for (int c = 0; c < nc; ++c) {
      // keep the slots full; wait for a slot only when nothing is in flight
      while (issued < nc) {
        if (issued >= SLOTS) {
          std::unique_lock<std::mutex> lk(mu);
          if (!moved[issued - SLOTS]) {
            if (issued > c) break;
            freed.wait(lk, [&]() { return moved[issued - SLOTS] != 0; });
          }
        }
        const Chunk& k = chunks[issued];
        const int slot = issued % SLOTS;
        if (k.after) FCK(hipStreamWaitEvent(st_, k.after, 0));
        FCK(hipMemcpyAsync(pin_ + (size_t)slot * CHUNK, src + k.off, k.len, hipMemcpyDeviceToHost, st_));
        FCK(hipEventRecord(arrived_[slot], st_));
        ++issued;
      }
      FCK(hipEventSynchronize(arrived_[c % SLOTS]));
      if (pool.t.empty()) {
        std::memcpy(dst + chunks[c].off, pin_ + (size_t)(c % SLOTS) * CHUNK, chunks[c].len);
        moved[c] = 1;
        continue;
      }
      {
        std::lock_guard<std::mutex> lk(mu);
        handed = c + 1;
      }
      work.notify_one();
    }
    std::unique_lock<std::mutex> lk(mu);
    freed.wait(lk, [&]() { return std::count(moved.begin(), moved.end(), 1) == nc; });
  }

 private:
  char* pin_ = nullptr;
  hipStream_t st_ = nullptr;
  hipEvent_t arrived_[SLOTS] = {};
  std::vector<hipEvent_t> ready_;
};

}  // namespace

struct bse_fno {
  bse_fno_config cfg{};
  size_t ng = 0;
  int K = 0;
  hipStream_t stream = nullptr;
  // parameter layout (floats)
  size_t off_P = 0, off_p = 0, off_Q = 0, off_q0 = 0, n_params = 0;
  std::vector<size_t> off_R, off_W, off_b;
  Buf master, compute, grad, adam_m, adam_v, tw;
  int step = 0;
  int cap = 0;
  int mix_path = 0;   // per-mode channel mix: 0 matrix cores, 1 vector FMA
  std::vector<Buf> h, z, V;
  Buf gh_a, gh_b, work, U, GU, GV, part, gy, y, loss_part, tn;
  Buf gidx;   // sample indices of bse_fno_gather
  HostCopy out;   // the gradient on its way to the host
};

namespace {

void layout(bse_fno* f) {
  const int W = f->cfg.width, ci = f->cfg.cin, L = f->cfg.layers;
  size_t o = 0;
  f->off_P = o; o += (size_t)W * ci;
  f->off_p = o; o += W;
  f->off_Q = o; o += W;
  f->off_q0 = o; o += 1;
  f->off_R.resize(L);
  f->off_W.resize(L);
  f->off_b.resize(L);
  for (int l = 0; l < L; ++l) {
    f->off_R[l] = o; o += (size_t)f->K * W * W * 2;
    f->off_W[l] = o; o += (size_t)W * W;
    f->off_b[l] = o; o += W;
  }
  f->n_params = o;
}

void ensure(bse_fno* f, int B) {
  if (B <= f->cap) return;
  const int W = f->cfg.width, L = f->cfg.layers;
  const size_t act = sizeof(float) * (size_t)B * W * f->ng;
  f->h.resize(L + 1);
  f->z.resize(L);
  f->V.resize(L);
  for (auto& b : f->h) b.alloc(act);
  for (auto& b : f->z) b.alloc(act);
  for (auto& b : f->V) b.alloc(sizeof(float2) * (size_t)B * W * f->K);
  f->gh_a.alloc(act);
  f->gh_b.alloc(act);
  f->work.alloc(sizeof(float2) * (size_t)B * W * f->cfg.n * 2 * f->cfg.modes * f->cfg.modes);
  f->U.alloc(sizeof(float2) * (size_t)B * W * f->K);
  f->GU.alloc(sizeof(float2) * (size_t)B * W * f->K);
  f->GV.alloc(sizeof(float2) * (size_t)B * W * f->K);
  const int ci = f->cfg.cin;
  f->part.alloc(sizeof(double) * std::max(fno_outer_part_len(W, W, B, f->ng), fno_outer_part_len(W, ci, B, f->ng)));
  f->gy.alloc(sizeof(float) * (size_t)B * f->ng);
  f->y.alloc(sizeof(float) * (size_t)B * f->ng);
  f->loss_part.alloc(sizeof(double) * 2 * (size_t)B * fno_loss_blocks(f->ng));
  f->tn.alloc(sizeof(double) * B);
  f->cap = B;
}

const float* prm(const bse_fno* f, size_t off) { return f->compute.f() + off; }

// y [B][ng] from x [B][cin][ng]; keep: the pre-activations the backward pass
// reads are stored (the layers' inputs and spectra always are)
void forward(bse_fno* f, int B, const float* x, float* y, bool keep) {
  const int W = f->cfg.width, L = f->cfg.layers, m = f->cfg.modes, n = f->cfg.n;
  hipStream_t st = f->stream;
  FCK(fno_pointwise(x, f->cfg.cin, prm(f, f->off_P), prm(f, f->off_p), W, B, f->ng, f->h[0].f(), st));
  for (int l = 0; l < L; ++l) {
    const bool last = l == L - 1;
    FCK(fno_fft_fwd(n, f->h[l].f(), B * W, f->tw.c(), m, 0, f->work.c(), f->V[l].c(), st));
    FCK(fno_spec_mix(f->V[l].c(), reinterpret_cast<const float2*>(prm(f, f->off_R[l])), B, W, f->K,
                     f->U.c(), f->mix_path, st));
    FCK(fno_x_inv(n, f->U.c(), B * W, f->tw.c(), m, 1, f->work.c(), st));
    const FnoLayerArgs a{f->h[l].f(), prm(f, f->off_W[l]), 0, prm(f, f->off_b[l]), W, B, m, f->work.c(), f->tw.c(),
                         last ? 0 : 1, keep && !last ? f->z[l].f() : nullptr, nullptr, f->h[l + 1].f()};
    FCK(fno_layer(n, a, st));
  }
  FCK(fno_pointwise(f->h[L].f(), W, prm(f, f->off_Q), prm(f, f->off_q0), 1, B, f->ng, y, st));
}

// loss and gradient (into f->grad); mark: events of f->out record when layer l
// (event l) and the rest (event L) of the gradient are computed
double loss_grad(bse_fno* f, int B, const float* x, const float* t, bool mark = false) {
  const int W = f->cfg.width, L = f->cfg.layers, m = f->cfg.modes, n = f->cfg.n, ci = f->cfg.cin;
  hipStream_t st = f->stream;
  forward(f, B, x, f->y.f(), true);
  const int nbb = fno_loss_blocks(f->ng);
  FCK(fno_loss_partial(f->y.f(), t, B, f->ng, f->loss_part.d(), st));
  std::vector<double> lp(2 * (size_t)B * nbb);
  FCK(hipMemcpyAsync(lp.data(), f->loss_part.p, sizeof(double) * lp.size(), hipMemcpyDeviceToHost, st));
  FCK(hipStreamSynchronize(st));
  std::vector<double> tn(B, 0.0), sq(B, 0.0);
  for (int b = 0; b < B; ++b)
    for (int k = 0; k < nbb; ++k) {
      sq[b] += lp[2 * ((size_t)b * nbb + k)];
      tn[b] += lp[2 * ((size_t)b * nbb + k) + 1];
    }
  double loss = 0;
  for (int b = 0; b < B; ++b) {
    if (!(tn[b] > 0)) ffail(BSE_ERR_ARG, "target with zero norm");
    loss += sq[b] / tn[b];
  }
  loss /= B;
  FCK(hipMemcpyAsync(f->tn.p, tn.data(), sizeof(double) * B, hipMemcpyHostToDevice, st));
  FCK(fno_loss_grad(f->y.f(), t, f->tn.d(), B, f->ng, f->gy.f(), st));
  float* g = f->grad.f();
  FCK(fno_outer(f->gy.f(), 1, f->h[L].f(), W, B, f->ng, f->part.d(), g + f->off_Q, g + f->off_q0, st));
  float* gh = f->gh_a.f();
  float* gn = f->gh_b.f();
  FCK(fno_proj_bwd(f->gy.f(), prm(f, f->off_Q), W, B, f->ng, gh, st));
  for (int l = L - 1; l >= 0; --l) {
    FCK(fno_outer(gh, W, f->h[l].f(), W, B, f->ng, f->part.d(), g + f->off_W[l], g + f->off_b[l], st));
    FCK(fno_fft_fwd(n, gh, B * W, f->tw.c(), m, 1, f->work.c(), f->GU.c(), st));
    FCK(fno_spec_mix_bwd(f->V[l].c(), f->GU.c(), reinterpret_cast<const float2*>(prm(f, f->off_R[l])),
                         B, W, f->K, f->GV.c(), reinterpret_cast<float2*>(g + f->off_R[l]), f->mix_path,
                         st));
    if (mark) FCK(hipEventRecord(f->out.ready(l), st));
    FCK(fno_x_inv(n, f->GV.c(), B * W, f->tw.c(), m, 0, f->work.c(), st));
    // to the layer below, through its gelu
    const FnoLayerArgs a{gh, prm(f, f->off_W[l]), 1, nullptr, W, B, m, f->work.c(), f->tw.c(),
                         0, nullptr, l > 0 ? f->z[l - 1].f() : nullptr, gn};
    FCK(fno_layer(n, a, st));
    std::swap(gh, gn);
  }
  FCK(fno_outer(gh, W, x, ci, B, f->ng, f->part.d(), g + f->off_P, g + f->off_p, st));
  if (mark) FCK(hipEventRecord(f->out.ready(L), st));
  return loss;
}

void check_batch(bse_fno* f, int B) {
  if (!f) ffail(BSE_ERR_ARG, "null surrogate");
  if (B < 1 || B > f->cfg.max_batch) ffail(BSE_ERR_ARG, "batch size outside 1..max_batch");
  ensure(f, B);
}

#define FAPI_BEGIN try {
#define FAPI_END                    \
  }                                 \
  catch (const FFail& e) {          \
    return e.st;                    \
  }                                 \
  catch (const std::exception& e) { \
    f_err = e.what();               \
    return BSE_ERR_DEVICE;          \
  }                                 \
  return BSE_OK;

}  // namespace

extern "C" {

const char* bse_fno_last_error(void) { return f_err.c_str(); }

bse_status bse_fno_create(const bse_fno_config* cfg, bse_fno** out) {
  FAPI_BEGIN
  if (!cfg || !out) ffail(BSE_ERR_ARG, "null argument");
  *out = nullptr;
  const bse_fno_config& c = *cfg;
  if (!fno_grid_supported(c.n)) ffail(BSE_ERR_ARG, "unsupported grid (16, 32 or 64)");
  if (c.cin < 1 || c.cin > 64 || c.width < 1 || c.width > 64 || c.layers < 1 || c.modes < 1 ||
      2 * c.modes > c.n || c.max_batch < 1)
    ffail(BSE_ERR_ARG, "bad surrogate configuration");
  FCK(hipSetDevice(c.device));
  auto* f = new bse_fno();
  try {
    f->cfg = c;
    f->ng = (size_t)c.n * c.n * c.n;
    f->K = (2 * c.modes) * (2 * c.modes) * c.modes;
    layout(f);
    f->master.alloc(sizeof(float) * f->n_params);
    f->compute.alloc(sizeof(float) * f->n_params);
    f->grad.alloc(sizeof(float) * f->n_params);
    f->adam_m.alloc(sizeof(float) * f->n_params);
    f->adam_v.alloc(sizeof(float) * f->n_params);
    // initial parameters: uniform ranges of the usual operator-network init
    std::vector<float> p(f->n_params, 0.f);
    std::mt19937_64 rng(c.seed);
    std::uniform_real_distribution<double> U(-1.0, 1.0), U01(0.0, 1.0);
    const int W = c.width;
    for (size_t i = 0; i < (size_t)W * c.cin; ++i) p[f->off_P + i] = (float)(U(rng) / std::sqrt((double)c.cin));
    for (int i = 0; i < W; ++i) p[f->off_Q + i] = (float)(U(rng) / std::sqrt((double)W));
    for (int l = 0; l < c.layers; ++l) {
      const double sc = 1.0 / ((double)W * W);
      for (size_t i = 0; i < (size_t)f->K * W * W * 2; ++i) p[f->off_R[l] + i] = (float)(sc * U01(rng));
      for (size_t i = 0; i < (size_t)W * W; ++i) p[f->off_W[l] + i] = (float)(U(rng) / std::sqrt((double)W));
    }
    FCK(hipMemcpy(f->master.p, p.data(), sizeof(float) * f->n_params, hipMemcpyHostToDevice));
    FCK(fno_round_copy(f->master.f(), f->compute.f(), f->n_params, c.bf16_weights, nullptr));
    FCK(hipMemset(f->adam_m.p, 0, sizeof(float) * f->n_params));
    FCK(hipMemset(f->adam_v.p, 0, sizeof(float) * f->n_params));
    std::vector<float2> tw(c.n);
    for (int q = 0; q < c.n; ++q) {
      const double a = -2.0 * M_PI * q / c.n;
      tw[q] = make_float2((float)std::cos(a), (float)std::sin(a));
    }
    f->tw.alloc(sizeof(float2) * c.n);
    FCK(hipMemcpy(f->tw.p, tw.data(), sizeof(float2) * c.n, hipMemcpyHostToDevice));
    FCK(hipDeviceSynchronize());
  } catch (...) {
    delete f;
    throw;
  }
  *out = f;
  FAPI_END
}

int64_t bse_fno_num_params(const bse_fno* f) { return f ? (int64_t)f->n_params : -1; }
int32_t bse_fno_max_batch(const bse_fno* f) { return f ? f->cfg.max_batch : 0; }

bse_status bse_fno_set_params(bse_fno* f, const float* host) {
  FAPI_BEGIN
  if (!f || !host) ffail(BSE_ERR_ARG, "null argument");
  FCK(hipMemcpy(f->master.p, host, sizeof(float) * f->n_params, hipMemcpyHostToDevice));
  FCK(fno_round_copy(f->master.f(), f->compute.f(), f->n_params, f->cfg.bf16_weights, f->stream));
  FCK(hipMemsetAsync(f->adam_m.p, 0, sizeof(float) * f->n_params, f->stream));
  FCK(hipMemsetAsync(f->adam_v.p, 0, sizeof(float) * f->n_params, f->stream));
  FCK(hipStreamSynchronize(f->stream));
  f->step = 0;
  FAPI_END
}

bse_status bse_fno_get_params(bse_fno* f, float* host, int32_t which) {
  FAPI_BEGIN
  if (!f || !host || (which != 0 && which != 1)) ffail(BSE_ERR_ARG, "bad argument");
  FCK(hipStreamSynchronize(f->stream));
  FCK(hipMemcpy(host, which ? f->compute.p : f->master.p, sizeof(float) * f->n_params,
                hipMemcpyDeviceToHost));
  FAPI_END
}

bse_status bse_fno_set_stream(bse_fno* f, void* st) {
  FAPI_BEGIN
  if (!f) ffail(BSE_ERR_ARG, "null surrogate");
  f->stream = reinterpret_cast<hipStream_t>(st);
  FAPI_END
}

bse_status bse_fno_set_mix_path(bse_fno* f, int32_t path) {
  FAPI_BEGIN
  if (!f) ffail(BSE_ERR_ARG, "null surrogate");
  if (path != 0 && path != 1) ffail(BSE_ERR_ARG, "bse_fno_set_mix_path: path 0 or 1");
  f->mix_path = path;
  FAPI_END
}

bse_status bse_fno_forward(bse_fno* f, int32_t B, const void* x_dev, void* y_dev) {
  FAPI_BEGIN
  check_batch(f, B);
  if (!x_dev || !y_dev) ffail(BSE_ERR_ARG, "null buffer");
  forward(f, B, reinterpret_cast<const float*>(x_dev), reinterpret_cast<float*>(y_dev), false);
  FCK(hipStreamSynchronize(f->stream));
  FAPI_END
}

bse_status bse_fno_loss_grad(bse_fno* f, int32_t B, const void* x_dev, const void* t_dev,
                             double* loss, float* grad_host) {
  FAPI_BEGIN
  check_batch(f, B);
  if (!x_dev || !t_dev || !loss) ffail(BSE_ERR_ARG, "null buffer");
  const int L = f->cfg.layers;
  const bool staged = grad_host && sizeof(float) * f->n_params >= HostCopy::MIN_BYTES && f->out.prepare(f->cfg.device, L + 1);
  *loss = loss_grad(f, B, reinterpret_cast<const float*>(x_dev), reinterpret_cast<const float*>(t_dev), staged);
  if (staged) {
    // the layers in the order of the backward pass, then the rest
    std::vector<HostCopy::Region> regions;
    for (int l = L - 1; l >= 0; --l) {
      const size_t end = l + 1 < L ? f->off_R[l + 1] : f->n_params;
      regions.push_back({sizeof(float) * f->off_R[l], sizeof(float) * (end - f->off_R[l]), f->out.ready(l)});
    }
    regions.push_back({0, sizeof(float) * f->off_R[0], f->out.ready(L)});
    f->out.copy(regions, reinterpret_cast<const char*>(f->grad.p), reinterpret_cast<char*>(grad_host));
  } else if (grad_host)
    FCK(hipMemcpyAsync(grad_host, f->grad.p, sizeof(float) * f->n_params, hipMemcpyDeviceToHost,
                       f->stream));
  FCK(hipStreamSynchronize(f->stream));
  FAPI_END
}

bse_status bse_fno_train_step(bse_fno* f, int32_t B, const void* x_dev, const void* t_dev, double lr,
                              double* loss) {
  FAPI_BEGIN
  check_batch(f, B);
  if (!x_dev || !t_dev || !loss || !(lr > 0)) ffail(BSE_ERR_ARG, "bad argument");
  *loss = loss_grad(f, B, reinterpret_cast<const float*>(x_dev), reinterpret_cast<const float*>(t_dev));
  f->step += 1;
  FCK(fno_adam(f->master.f(), f->compute.f(), f->grad.f(), f->adam_m.f(), f->adam_v.f(), f->n_params,
               (float)lr, 0.9f, 0.999f, 1e-8f, f->step, f->cfg.bf16_weights, f->stream));
  FCK(hipStreamSynchronize(f->stream));
  FAPI_END
}

void bse_fno_destroy(bse_fno* f) {
  if (!f) return;
  (void)hipSetDevice(f->cfg.device);
  delete f;
}

bse_status bse_fno_gather(bse_fno* f, int32_t B, const int32_t* idx, int32_t n_src, const void* x_src,
                          const void* t_src, const int32_t* perm, int32_t flip_mask, void* x_dst, void* t_dst) {
  FAPI_BEGIN
  check_batch(f, B);
  if (!idx || !perm || !x_src || !t_src || !x_dst || !t_dst) ffail(BSE_ERR_ARG, "null argument");
  for (int b = 0; b < B; ++b)
    if (idx[b] < 0 || idx[b] >= n_src) ffail(BSE_ERR_ARG, "sample index outside 0..n_src-1");
  bool seen[3] = {false, false, false};
  for (int k = 0; k < 3; ++k) {
    if (perm[k] < 0 || perm[k] > 2 || seen[perm[k]]) ffail(BSE_ERR_ARG, "perm is not a permutation of 0, 1, 2");
    seen[perm[k]] = true;
  }
  if (flip_mask < 0 || flip_mask > 7) ffail(BSE_ERR_ARG, "flip_mask outside 0..7");
  const int pm[3] = {perm[0], perm[1], perm[2]};
  f->gidx.alloc(sizeof(int) * (size_t)f->cfg.max_batch);
  FCK(hipMemcpyAsync(f->gidx.p, idx, sizeof(int) * B, hipMemcpyHostToDevice, f->stream));
  const int n = f->cfg.n;
  FCK(fno_gather_sym(reinterpret_cast<const float*>(x_src), reinterpret_cast<const int*>(f->gidx.p), B,
                     f->cfg.cin, n, pm, flip_mask, reinterpret_cast<float*>(x_dst), f->stream));
  FCK(fno_gather_sym(reinterpret_cast<const float*>(t_src), reinterpret_cast<const int*>(f->gidx.p), B, 1, n,
                     pm, flip_mask, reinterpret_cast<float*>(t_dst), f->stream));
  FCK(hipStreamSynchronize(f->stream));
  FAPI_END
}

}  // extern "C"
