// sweep_dual_hbm.hip -- sweeps with the phases in device memory, two colour classes
// per pass.
//
// For graphs whose replicas do not fit in LDS.  A pass per class reads and writes
// every row once per class.  Here, as in sweep_dual.hip, a wave's entry is an edge
// (u, v) of class c + 1 with the class c partners of u and v: it reads the four
// rows, applies class c to u and to v (their own side only), then class c + 1 to the
// pair, and writes u and v to the other phase buffer.  Two classes then cost one
// write of the phases, one read from device memory and one more from the caches
// (the partners' rows are some neighbouring wave's own).  The twist, without bias
// fields, is applied in the last round, from a table of the replicas' reference
// angles.
//
// A wave takes 64 VEC replicas of one entry; waves of neighbouring entries run in
// neighbouring workgroups of one XCD.  The replicas go through all sweeps of a call
// in groups whose two buffers stay in the last-level cache (kGroupBytes).
//
// 50 sweeps of 1024 replicas, a pass per class -> this: 300 x 300 torus, FP32 26.4 ->
// 11.7 ms (12.8 without the groups), FIX16 11.7 -> 9.4; 3-regular graph of 60000, whose
// partners lie anywhere, 11.7 -> 10.7.  It is bound by the caches and device memory:
// two reads and a write of every row per pass at some 9 TB/s.
//
// A pass moves every row, also where few have an edge; rounds of small classes run
// class by class in place instead (round_pays), the last one on sweeps without a twist
// only: a twist of its own moves every row too.
#include <hip/hip_runtime.h>

#include <string>

#include "device_common.hpp"
#include "hbm_vec.hpp"
#include "internal.hpp"

namespace cosm {
namespace {

// Two buffers of a group of replicas, out of the 256 MB cache.
constexpr size_t kGroupBytes = (size_t)192 << 20;
// The second buffer is taken up to this size of the first.
constexpr size_t kAltBytesMax = (size_t)16 << 30;
// Smaller graphs forced into device memory take a pass per class: the baseline that the
// LDS forms are compared with.
constexpr int32_t kVerticesMin = 40001;

struct Entry {
  int32_t u, v, pu, pv;
  float J, Ju, Jv;
  int32_t flips;
};

// A value as its storage holds it (a store and a load).
template <int ST>
__device__ __forceinline__ float stored(float x) {
  if constexpr (ST == COSM_STORE_FP32) return x;
  else return Fmt<ST>::dec(Fmt<ST>::enc(x));
}

// Class c on one endpoint: x as the u (or, flipped, the v) of its edge to y.
template <int ST, bool LAZY>
__device__ __forceinline__ float end_update(float x, float y, float aJ, bool flip) {
  float a = flip ? y : x, b = flip ? x : y;
  pair_update<ST, LAZY>(a, b, aJ);
  return stored<ST>(flip ? b : a);
}

template <int ST, int VEC, bool LAZY>
__global__ void __launch_bounds__(256) k_dual_hbm(const void *src, void *dst, const Entry *entries,
                                                  int32_t count, int32_t R, int32_t rbeg,
                                                  int32_t rend, float alpha, const float *theta,
                                                  float twist, float win2) {
  using F = Fmt<ST>;
  const int32_t wave = xcd_block(blockIdx.x, gridDim.x) * 4 + (int32_t)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int32_t k = __builtin_amdgcn_readfirstlane(wave % count);
  const int32_t r = rbeg + (wave / count * 64 + lane) * VEC;
  if (r >= rend) return;
  const Entry e = entries[k];  // uniform: scalar loads
  const bool fu = e.flips & 1, fv = e.flips & 2;
  float xu[VEC], xv[VEC], yu[VEC], yv[VEC];
  load_vec<ST, VEC>(src, (size_t)e.u * R + r, xu);
  if (e.pu >= 0) load_vec<ST, VEC>(src, (size_t)e.pu * R + r, yu);
  if (e.v >= 0) load_vec<ST, VEC>(src, (size_t)e.v * R + r, xv);
  if (e.pv >= 0) load_vec<ST, VEC>(src, (size_t)e.pv * R + r, yv);
  if (e.pu >= 0) {
    const float aJ = alpha * e.Ju;
#pragma unroll
    for (int q = 0; q < VEC; q++) xu[q] = end_update<ST, LAZY>(xu[q], yu[q], aJ, fu);
  }
  if (e.v >= 0) {
    if (e.pv >= 0) {
      const float aJ = alpha * e.Jv;
#pragma unroll
      for (int q = 0; q < VEC; q++) xv[q] = end_update<ST, LAZY>(xv[q], yv[q], aJ, fv);
    }
    const float aJ = alpha * e.J;
    if (aJ != 0.0f) {
#pragma unroll
      for (int q = 0; q < VEC; q++) {
        pair_update<ST, LAZY>(xu[q], xv[q], aJ);
        xu[q] = stored<ST>(xu[q]);
        xv[q] = stored<ST>(xv[q]);
      }
    }
  }
  if (theta != nullptr) {
#pragma unroll
    for (int q = 0; q < VEC; q++) {
      const float c = theta[r + q];
      auto turn = [&](float x) {
        if constexpr (LAZY) {
          const float y = F::wrap(x);
          return in_windows(y, c, win2) ? y + twist : y;
        } else {
          return in_windows(x, c, win2) ? F::wrap(x + twist) : x;
        }
      };
      xu[q] = turn(xu[q]);
      if (e.v >= 0) xv[q] = turn(xv[q]);
    }
  }
  store_vec<ST, VEC>(dst, (size_t)e.u * R + r, xu);
  if (e.v >= 0) store_vec<ST, VEC>(dst, (size_t)e.v * R + r, xv);
}

// c = 2 theta - w of the twist after sweep t, for replicas [rbeg, rend).
__global__ void __launch_bounds__(256) k_theta(float *theta, int32_t rbeg, int32_t rend, uint32_t t,
                                               uint32_t rid0, uint32_t k0, uint32_t k1, float win,
                                               uint32_t tshift, float tscale) {
  const int32_t r = rbeg + (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (r >= rend) return;
  const uint32_t w = philox_first_word(0u, t, rid0 + (uint32_t)r, kTagDwt, k0, k1);
  theta[r] = 2.0f * ((float)(w >> tshift) * tscale) - win;
}

int checked(const char *what) {
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess)
    return set_error(COSM_EDEVICE, std::string(what) + ": " + hipGetErrorString(err));
  return COSM_OK;
}

// Whether classes of a and b edges are worth a pass: it reads and writes n rows, and
// reads the 2a partners' (from the caches); one class after the other reads and
// writes 2(a + b).  Few replicas are bound by their launches, of which a pass saves one.
// Two such rounds on 60000 vertices, random partners, classes -> passes in us a sweep.
// 1024 replicas, at a + 2b = 0.6 n: FP32 134 -> 191, FIX16 76 -> 95; 0.9 n: 191 -> 205,
// 103 -> 107; 1.05 n: 219 -> 211, 117 -> 112; 1.5 n: 303 -> 230, 159 -> 131.  32 replicas,
// 0.6 n: 26 -> 20, 27 -> 27; 0.9 n: 33 -> 23, 35 -> 32.
constexpr int32_t kFewReplicas = 64;
bool round_pays(int32_t n, int32_t R, int64_t a, int64_t b) {
  return (R <= kFewReplicas ? 2 : 1) * (a + 2 * b) > n;
}

template <int ST, int VEC>
int pass(cosm_state *s, int32_t q, const Entry *entries, int32_t rbeg, int32_t rend, float alpha,
         const float *theta, float twist) {
  const int32_t count = s->dual_count[(size_t)q];
  const int64_t waves = (int64_t)count * ((rend - rbeg + 64 * VEC - 1) / (64 * VEC));
  const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
  if (lazy16(*s))
    hipLaunchKernelGGL((k_dual_hbm<ST, VEC, lazy_storage(ST) && ST != COSM_STORE_FP32>), grid, block,
                       0, s->stream, s->d.phases, s->d.phases_alt, entries, count, s->R, rbeg, rend,
                       alpha, theta, twist, s->sched.window2);
  else
    hipLaunchKernelGGL((k_dual_hbm<ST, VEC, false>), grid, block, 0, s->stream, s->d.phases,
                       s->d.phases_alt, entries, count, s->R, rbeg, rend, alpha, theta, twist,
                       s->sched.window2);
  return checked("k_dual_hbm");
}

// Passes in sweeps t + 1 .. t + n (those of the last round on twist sweeps among them).
int64_t passes_in(const cosm_state &s, int64_t t, int64_t n) {
  int64_t each = 0;
  for (uint8_t p : s.dual_pays) each += p;
  const int64_t period = s.sched.dwt_period;
  const int64_t twists = period > 0 && !s.has_h ? (t + n) / period - t / period : 0;
  return each * n + (s.dual_pays.back() ? 0 : twists);
}

template <int ST>
int sweeps(cosm_state *s, int64_t n_sweeps) {
  const Schedule &sc = s->sched;
  const int32_t rounds = (int32_t)s->dual_count.size();
  // replicas per group: whole waves of the widest accesses
  const size_t row = (size_t)2 * s->n * (4 / Fmt<ST>::kPerWord);
  int64_t group = (int64_t)(kGroupBytes / row) / 256 * 256;
  group = std::max<int64_t>(256, group);
  // A call leaves the phases in the buffer it found them in: one that is captured into a
  // graph keeps its buffers, whatever calls run between the graph's replays.  An odd
  // number of passes becomes even by one round that runs class by class.
  const bool odd = passes_in(*s, s->t, n_sweeps) % 2 != 0;
  struct Buffers {
    DeviceBuffers &d;
    void *const first = d.phases, *const second = d.phases_alt;
    ~Buffers() {  // (on an error between two passes too)
      d.phases = first;
      d.phases_alt = second;
    }
  } const buffers{s->d};
  for (int32_t rbeg = 0; rbeg < s->R;) {
    int32_t rend = (int32_t)std::min<int64_t>(s->R, rbeg + group);
    if (s->R - rend < group / 2) rend = s->R;  // no small last group
    const int vec = hbm_vec(s->R, rbeg, rend - rbeg);
    bool drop = odd;  // a pass to leave out
    for (int64_t t = s->t + 1; t <= s->t + n_sweeps; t++) {
      const float alpha = host_alpha(sc, t), twist = host_twist(sc, t);
      const bool twist_now = sc.dwt_period > 0 && t % sc.dwt_period == 0;
      bool twisted = false;
      const Entry *entries = static_cast<const Entry *>(s->d.dual_entries);
      for (int32_t q = 0; q < rounds; q++) {
        const Entry *const here = entries;
        entries += s->dual_count[(size_t)q];
        const bool fused = twist_now && !s->has_h && q == rounds - 1;
        if (!(s->dual_pays[(size_t)q] || fused) || drop) {
          if (s->dual_pays[(size_t)q] || fused) drop = false;
          for (int32_t c = 2 * q; c < std::min(s->C, 2 * q + 2); c++)
            if (int rc = launch_class_hbm(s, c, alpha, rbeg, rend - rbeg)) return rc;
          continue;
        }
        if (fused) {
          hipLaunchKernelGGL(k_theta, dim3((unsigned)((rend - rbeg + 255) / 256)), dim3(256), 0,
                             s->stream, s->d.dual_theta, rbeg, rend, (uint32_t)t,
                             (uint32_t)s->rid0, (uint32_t)(s->seed & 0xffffffffu),
                             (uint32_t)(s->seed >> 32), sc.window, (uint32_t)sc.tshift, sc.tscale);
          if (int rc = checked("k_theta")) return rc;
        }
        const float *theta = fused ? s->d.dual_theta : nullptr;
        const int rc = vec == 4   ? pass<ST, 4>(s, q, here, rbeg, rend, alpha, theta, twist)
                       : vec == 2 ? pass<ST, 2>(s, q, here, rbeg, rend, alpha, theta, twist)
                                  : pass<ST, 1>(s, q, here, rbeg, rend, alpha, theta, twist);
        if (rc) return rc;
        twisted = fused;
        std::swap(s->d.phases, s->d.phases_alt);
      }
      if (s->has_h)
        if (int rc = launch_field_hbm(s, alpha, rbeg, rend - rbeg)) return rc;
      if (twist_now && !twisted)
        if (int rc = launch_dwt_hbm(s, t, rbeg, rend - rbeg)) return rc;
    }
    rbeg = rend;
  }
  return COSM_OK;
}

}  // namespace

bool dual_hbm_form(int32_t n, int64_t m, int32_t C, int32_t R, const cosm_params &p) {
  const int32_t pw = p.storage == COSM_STORE_FP32 || p.storage == COSM_STORE_FIX32 ? 1 : 2;
  if (n < kVerticesMin || dual_hbm_entry_bytes(n, m, C, R) == 0 || p.update != COSM_UPDATE_SCS ||
      (size_t)n * (size_t)R * (size_t)(4 / pw) > kAltBytesMax)
    return false;
  if (p.residency != COSM_RES_AUTO) return p.residency == COSM_RES_HBM;
  // (one word per row fits up to some 40370 vertices: those run in LDS)
  return n > 65535 || lds_sweep_bytes(n, std::max(1, p.replicas_per_wg / pw), C) >
                          (size_t)lds_capacity_bytes();
}

size_t dual_hbm_entry_bytes(int32_t n, int64_t m, int32_t C, int32_t R) {
  // two classes that pay have at least (n + 1) / 2 edges, or half of that for few
  // replicas (round_pays; b <= n / 2); with them the last round, for the twist.  A round
  // has an entry for two vertices, and one for an odd one.
  const int64_t pay = std::min<int64_t>(C / 2, (R <= kFewReplicas ? 4 : 2) * m / ((int64_t)n + 1));
  if (pay == 0) return 0;
  return (size_t)std::min<int64_t>((C + 1) / 2, pay + 1) * ((size_t)n / 2 + 1) * sizeof(Entry);
}

size_t dual_hbm_choose(cosm_state *s) {
  std::vector<uint8_t> pays((size_t)(s->C + 1) / 2, 0);
  size_t rounds = 0;
  for (int32_t q = 0; 2 * q + 1 < s->C; q++) {
    pays[(size_t)q] = round_pays(s->n, s->R, s->class_sizes[(size_t)2 * q], s->class_sizes[(size_t)2 * q + 1]);
    rounds += pays[(size_t)q];
  }
  if (rounds == 0) return 0;
  if (!pays.back() && s->sched.dwt_period > 0 && !s->has_h) rounds++;  // (the twist's)
  s->dual_pays = pays;
  return rounds * ((size_t)s->n / 2 + 1) * sizeof(Entry);
}

int upload_dual_hbm(cosm_state *s) {
  std::vector<uint8_t> wanted(s->dual_pays);
  if (s->sched.dwt_period > 0 && !s->has_h) wanted.back() = 1;
  std::vector<Entry> all;
  for (const auto &round : dual_entries(*s, &wanted)) {
    s->dual_count.push_back((int32_t)round.size());
    for (const DualEntry &e : round)
      all.push_back(Entry{e.u, e.v, e.pu, e.pv, (float)e.J, (float)e.Ju, (float)e.Jv,
                          e.fu | e.fv << 1});
  }
  COSM_HIP_CHECK(hipMemcpyAsync(s->d.dual_entries, all.data(), all.size() * sizeof(Entry),
                                hipMemcpyHostToDevice, s->stream));
  COSM_HIP_CHECK(hipStreamSynchronize(s->stream));  // all goes out of scope
  return COSM_OK;
}

int launch_sweeps_dual_hbm(cosm_state *s, int64_t n_sweeps) {
  switch (s->p.storage) {
    case COSM_STORE_FP32: return sweeps<COSM_STORE_FP32>(s, n_sweeps);
    case COSM_STORE_FP16: return sweeps<COSM_STORE_FP16>(s, n_sweeps);
    case COSM_STORE_FP16_PK: return sweeps<COSM_STORE_FP16_PK>(s, n_sweeps);
    case COSM_STORE_BF16: return sweeps<COSM_STORE_BF16>(s, n_sweeps);
    case COSM_STORE_FIX16: return sweeps<COSM_STORE_FIX16>(s, n_sweeps);
    case COSM_STORE_FIX32: return sweeps<COSM_STORE_FIX32>(s, n_sweeps);
  }
  return set_error(COSM_EINVAL, "unknown storage format");
}

}  // namespace cosm
