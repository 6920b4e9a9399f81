// sweep_full.hip -- the full-gradient update of Eq. (8) with the phases resident
// in LDS for all sweeps of a call.
//
// k_full_gradient (kernels.hip) reads and writes every phase in device memory
// once per sweep and its neighbours besides, one launch per sweep and another per
// twist.  Here a workgroup owns RW = W kPerWord whole replicas as LDS rows, as in
// k_sweep_lds: a sweep reads one copy of the rows and writes the other, with one
// barrier, and the twist is applied to the values just computed.
//
// Rows are the vertices in order of falling degree, so that the 64 rows of a wave
// have nearly the same number of neighbours.  Word [a][row] of the schedule is
// the a-th neighbour of a vertex in its incidence order: row | first << 16 |
// J << 17 (first: the vertex is the edge's u; J = 0 past the vertex's own
// degree).  The words stream from L2, four ahead; one serves all RW replicas.
//
// Device memory -> LDS, 200 sweeps of 2048 replicas: 3-regular graph of 2000
// vertices 4.35 -> 0.68 ms, Erdos-Renyi graph of 10000 (FP32) 28.3 -> 7.2 ms.  It
// waits for the gathers: random rows share LDS banks.
#include <hip/hip_runtime.h>

#include <string>

#include "device_common.hpp"
#include "internal.hpp"
#include "lds_args.hpp"

namespace cosm {
namespace {

constexpr int kAhead = 4;  // neighbour words in flight

// One neighbour's contribution to the vertex's change, in k_full_gradient's
// operations and order.  RD (the grid schedule under f32_round_down, every value
// exact): the sign of the step from the parity of floor(2(x_u - x_v)).
template <int RW, bool RD>
__device__ __forceinline__ void neighbour(const float (&xi)[RW], const float (&xj)[RW],
                                          float (&acc)[RW], uint32_t word, float alpha, float pm) {
  const bool first = (word >> 16) & 1u;
  const float aJ = alpha * (float)((int32_t)word >> 17);
#pragma unroll
  for (int k = 0; k < RW; k++) {
    if constexpr (RD) {
      const float p = __builtin_fmaf(xi[k] - xj[k], first ? 2.0f : -2.0f, pm);
      acc[k] -= __uint_as_float((__float_as_uint(p) << 31) +
                                __float_as_uint(first ? aJ : -aJ));
    } else {
      const float f = fract1(first ? xi[k] - xj[k] : xj[k] - xi[k]);
      const float s = (f < 0.5f) ? aJ : -aJ;
      acc[k] += first ? -s : s;
    }
  }
}

// The twist of a row.  FIX32: on the decoded value, as in the device-memory form
// (k_dwt_hbm), since phases set from outside may lie off the grid, where FP32 rounds them
// and the integer twist of TwistOps would not.
template <int ST, int W>
struct RowTwist : TwistOps<ST, W> {};
template <int W>
struct RowTwist<COSM_STORE_FIX32, W> {
  float c[W], t[W], win2;
  __device__ __forceinline__ void set(const float (&cth)[W], const float (&tws)[W], float w2) {
#pragma unroll
    for (int k = 0; k < W; k++) {
      c[k] = cth[k];
      t[k] = tws[k];
    }
    win2 = w2;
  }
  __device__ __forceinline__ void apply(uint32_t (&w)[W]) const {
    using F = Fmt<COSM_STORE_FIX32>;
    float x[W];
    F::template unpack<W>(w, x);
#pragma unroll
    for (int k = 0; k < W; k++)
      if (in_windows(x[k], c[k], win2)) w[k] = F::enc(F::wrap(x[k] + t[k]));
  }
};

template <int ST, int W, bool RD>
__global__ void __launch_bounds__(1024) k_full_lds(const LdsArgs a) {
  static_assert(!RD || ST == COSM_STORE_FP32, "the parity step is an FP32 grid form");
  extern __shared__ uint32_t lds[];
  using F = Fmt<ST>;
  constexpr int RW = W * F::kPerWord;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int32_t n = a.n_rows;
  const int32_t r0 = xcd_block(blockIdx.x, gridDim.x) * RW;
  const int32_t nvalid = min(RW, a.R - r0);
  const uint32_t copy_words = (uint32_t)(n + kDummyRows) * W;
  uint32_t *rows[2] = {lds, lds + copy_words};

  lds_rows_in<ST, W>(lds, a, r0, nvalid, nth);
  float *theta_buf = reinterpret_cast<float *>(lds + 2 * copy_words);
  float *dir_buf = theta_buf + kThetaFloats;
  // neighbours of the longest vertex of each group of 64 rows
  int32_t *deg = reinterpret_cast<int32_t *>(dir_buf + kThetaFloats);
  const int32_t groups = (n + 63) >> 6;
  for (int g = tid; g < groups; g += nth) deg[g] = a.reg_vertex[g];
  const gptr<uint32_t> words = as_global(a.dual);
  __syncthreads();

  const SweepSchedule sc = a.sch;
  const uint32_t nsw = (uint32_t)a.nsw;
  uint32_t t = (uint32_t)a.t0;
  uint32_t tw = 0;
  ScheduleChunk chunk;
  float pm = 0.0f;
  if constexpr (RD) pm = f32_round_down();
  int src = 0;
  for (uint32_t it = 0; it < nsw; it++) {
    t++;
    if ((it & 63u) == 0u) chunk.fill(sc, t);
    float alpha, twist;
    chunk.get(it & 63u, alpha, twist);
    const bool twist_now = chunk.twist_at(it & 63u);
    RowTwist<ST, W> op;
    if (twist_now) {
      const int q = (int)(tw % (uint32_t)kThetaChunk);
      tw++;
      if (q == 0) {
        theta_fill(theta_buf, a.h_slot != nullptr ? dir_buf : nullptr, kThetaChunk, RW, t,
                   sc.period, a.rid0 + (uint32_t)r0, a.k0, a.k1, sc.win, sc.tshift, sc.tscale);
        __syncthreads();
      }
      float cth[RW], tws[RW];
#pragma unroll
      for (int k = 0; k < RW; k++) {
        cth[k] = theta_buf[q * RW + k];
        tws[k] = a.h_slot != nullptr ? dir_buf[q * RW + k] * twist : twist;
      }
      op.set(cth, tws, sc.win2);
    }
    const uint32_t *from = rows[src];
    uint32_t *to = rows[src ^ 1];
    // the first kAhead neighbour words of row i
    uint32_t next[kAhead];
    int32_t next_deg = 0;
    auto fetch = [&](int32_t i) {
      if (i >= n) return;
      next_deg = deg[i >> 6];
#pragma unroll
      for (int q = 0; q < kAhead; q++)
        if (q < next_deg) next[q] = words[(size_t)q * n + i];
    };
    fetch(tid);
    for (int32_t i = tid; i < n; i += nth) {
      uint32_t w[kAhead];
#pragma unroll
      for (int q = 0; q < kAhead; q++) w[q] = next[q];
      const int32_t d = __builtin_amdgcn_readfirstlane(next_deg);
      uint32_t own[W];
      lds_load<W>(from, i, own);
      float xi[RW], acc[RW];
      F::template unpack<W>(own, xi);
#pragma unroll
      for (int k = 0; k < RW; k++) acc[k] = 0.0f;
      // up to kAhead neighbours: all rows read, then their contributions in order
      auto few = [&](int cnt) {
        uint32_t r[kAhead][W];
#pragma unroll
        for (int q = 0; q < kAhead; q++)
          if (q < cnt) lds_load<W>(from, (int)(w[q] & 0xffffu), r[q]);
#pragma unroll
        for (int q = 0; q < kAhead; q++)
          if (q < cnt) {
            float xj[RW];
            F::template unpack<W>(r[q], xj);
            neighbour<RW, RD>(xi, xj, acc, w[q], alpha, pm);
          }
      };
      fetch(i + nth);
      few(d);
      for (int32_t b = kAhead; b < d; b += kAhead) {
#pragma unroll
        for (int q = 0; q < kAhead; q++)
          if (b + q < d) w[q] = words[(size_t)(b + q) * n + i];
        few(d - b);
      }
      if (a.h_slot != nullptr) {  // the virtual spin at phase 0 (bias field)
        const int32_t hv = a.h_slot[i];
        if (hv != 0) {
          const float ah = alpha * (float)hv;
#pragma unroll
          for (int k = 0; k < RW; k++) acc[k] += fract1(F::to_turn(xi[k])) < 0.5f ? -ah : ah;
        }
      }
#pragma unroll
      for (int k = 0; k < RW; k++) xi[k] = F::wrap(xi[k] + acc[k]);
      F::template pack<W>(xi, own);
      if (twist_now) op.apply(own);
      lds_store<W>(to, i, own);
    }
    src ^= 1;
    __syncthreads();
  }
  if constexpr (RD) f32_round_nearest();
  lds_rows_out<ST, W, false>(rows[src], a, r0, nvalid, nth);
}

template <int ST, int W, bool RD>
int launch_k(cosm_state *s, const LdsArgs &a) {
  const size_t lds = s->shape.lds_bytes;
  (void)hipFuncSetAttribute((const void *)k_full_lds<ST, W, RD>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_full_lds<ST, W, RD>), dim3(s->shape.blocks), dim3(s->shape.threads), lds,
                     s->stream, a);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess)
    return set_error(COSM_EDEVICE, std::string("k_full_lds: ") + hipGetErrorString(err));
  return COSM_OK;
}

template <int ST, int W>
int launch_w(cosm_state *s, const LdsArgs &a) {
  // the parity step where every value of a sweep is exact: the sum of a vertex's
  // steps and its phase stay below two turns
  if constexpr (ST == COSM_STORE_FP32) {
    if (grid_drift_below_turn(*s)) return launch_k<ST, W, true>(s, a);
  }
  return launch_k<ST, W, false>(s, a);
}

template <int ST>
int launch_st(cosm_state *s, const LdsArgs &a) {
  switch (s->shape.rw / Fmt<ST>::kPerWord) {
    case 4: return launch_w<ST, 4>(s, a);
    case 2: return launch_w<ST, 2>(s, a);
    case 1: return launch_w<ST, 1>(s, a);
  }
  return set_error(COSM_EINVAL, "unsupported replicas per workgroup");
}

size_t full_lds_bytes(int32_t n, int W) {
  return (size_t)2 * (n + kDummyRows) * W * 4 + (size_t)2 * kThetaFloats * 4 +
         (size_t)((n + 63) / 64) * 4;
}

// With few replicas most CUs are idle in LDS, and a sweep takes its one workgroup as
// long as it has vertices and neighbours to visit; in device memory all CUs share them,
// and a sweep waits for launches, its longest vertex and, on twist sweeps, the twist's
// strips.  Both in us a sweep, fitted on 3-regular and Erdos-Renyi graphs of 4000 - 19000
// vertices, 1 - 128 replicas, within some 15 %.  LDS | device memory, period 6: FP32,
// 12000 vertices, 1 replica 7.4 | 5.2, 4 replicas 7.5 | 8.6; 19000 vertices, 16 replicas
// 12.0 | 10.6, 64 12.1 | 16.8; FIX16, 19000, 32 replicas 17.7 | 13.9, 128 17.8 | 21.3.
bool device_memory_faster(const cosm_state &s, int32_t dmax, bool wide) {
  const double lds = (wide ? 0.155e-3 : 0.224e-3) * ((double)s.n + 2.0 * (double)s.m);
  const double twist = s.R == 1 ? (wide ? 12 : 14) : s.R == 2 ? (wide ? 20 : 22) : (wide ? 32 : 41);
  const double hbm = 2.2 + 0.35 * dmax + 7.5e-6 * (double)s.n * (double)s.R +
                     (s.sched.dwt_period > 0 ? twist / s.sched.dwt_period : 0.0);
  return hbm < lds;
}

}  // namespace

// The rows of the LDS form, or COSM_ERANGE where it does not apply: two copies of
// at least one word per vertex, |J| below 2^14, at most kFullDegreeMax neighbours,
// replicas enough (device_memory_faster).
// Of the row widths that give every CU a workgroup the widest: a neighbour word and
// its decoding serve all replicas of a row (2000 vertices, 2048 replicas: 1, 2 and
// 4 words 1.82, 1.14 and 0.68 ms per 200 sweeps).
int full_shape(const cosm_state &s, int32_t cus, LdsSchedule *out, KernelShape *shape) {
  const int32_t n = s.n;
  const int32_t pw = s.p.storage == COSM_STORE_FP32 || s.p.storage == COSM_STORE_FIX32 ? 1 : 2;
  int W = 0;
  for (int w : {4, 2, 1}) {
    if (full_lds_bytes(n, w) > (size_t)lds_capacity_bytes()) continue;
    W = w;
    if ((s.R + w * pw - 1) / (w * pw) >= cus) break;
  }
  if (W == 0 || n + kDummyRows > 65535)
    return set_error(COSM_ERANGE, "full gradient: two copies of a replica do not fit in LDS");
  for (int32_t J : s.h_J)
    if (J >= 16384 || J < -16384)
      return set_error(COSM_ERANGE, "full gradient: the LDS form needs |J| < 2^14");
  std::vector<int32_t> degree((size_t)n, 0);
  for (int64_t k = 0; k < s.m; k++) {
    degree[(size_t)s.h_eu[(size_t)k]]++;
    degree[(size_t)s.h_ev[(size_t)k]]++;
  }
  LdsSchedule L;
  L.n_rows = n;
  L.slot_vertex.resize((size_t)n);
  for (int32_t v = 0; v < n; v++) L.slot_vertex[(size_t)v] = v;
  std::stable_sort(L.slot_vertex.begin(), L.slot_vertex.end(),
                   [&](int32_t x, int32_t y) { return degree[(size_t)x] > degree[(size_t)y]; });
  const int32_t dmax = degree[(size_t)L.slot_vertex[0]];
  if (dmax > kFullDegreeMax)
    return set_error(COSM_ERANGE, "full gradient: the LDS form takes 32 neighbours");
  if (device_memory_faster(s, dmax, pw == 1))
    return set_error(COSM_ERANGE, "full gradient: few replicas of a large graph");
  std::vector<int32_t> row((size_t)n);
  for (int32_t r = 0; r < n; r++) row[(size_t)L.slot_vertex[(size_t)r]] = r;
  // a padding word: the vertex itself with J = 0
  L.dual_words.resize((size_t)dmax * n);
  for (int32_t q = 0; q < dmax; q++)
    for (int32_t r = 0; r < n; r++) L.dual_words[(size_t)q * n + r] = (uint32_t)r;
  std::vector<int32_t> fill((size_t)n, 0);
  for (int64_t k = 0; k < s.m; k++) {
    const int32_t u = s.h_eu[(size_t)k], v = s.h_ev[(size_t)k];
    const uint32_t J = (uint32_t)s.h_J[(size_t)k] << 17;
    const int32_t ru = row[(size_t)u], rv = row[(size_t)v];
    L.dual_words[(size_t)fill[(size_t)u]++ * n + ru] = (uint32_t)rv | 1u << 16 | J;
    L.dual_words[(size_t)fill[(size_t)v]++ * n + rv] = (uint32_t)ru | J;
  }
  for (int32_t g = 0; g * 64 < n; g++)
    L.K.push_back(degree[(size_t)L.slot_vertex[(size_t)g * 64]]);
  L.full = true;
  L.fuse = true;
  // One vertex per thread as far as two workgroups of 768 fit a CU, all threads
  // once the rows fill its LDS.  2000 vertices, 2048 replicas, 200 sweeps: 512
  // threads 764, 768 681, 1024 797 us; 400 vertices: 256 301, 512 240, 768 244;
  // 10000 vertices: 768 7.86, 1024 7.23 ms.
  L.nth = n <= 768 ? (n + 63) / 64 * 64 : n <= 3072 ? 768 : 1024;
  shape->residency = COSM_RES_LDS;
  shape->rw = W * pw;
  shape->blocks = (s.R + shape->rw - 1) / shape->rw;
  shape->threads = L.nth;
  shape->lds_bytes = (int32_t)full_lds_bytes(n, W);
  *out = std::move(L);
  return COSM_OK;
}

int launch_sweeps_full(cosm_state *s, const LdsArgs &a) {
  switch (s->p.storage) {
    case COSM_STORE_FP32: return launch_st<COSM_STORE_FP32>(s, a);
    case COSM_STORE_FP16: return launch_st<COSM_STORE_FP16>(s, a);
    case COSM_STORE_FP16_PK: return launch_st<COSM_STORE_FP16_PK>(s, a);
    case COSM_STORE_BF16: return launch_st<COSM_STORE_BF16>(s, a);
    case COSM_STORE_FIX16: return launch_st<COSM_STORE_FIX16>(s, a);
    case COSM_STORE_FIX32: return launch_st<COSM_STORE_FIX32>(s, a);
  }
  return set_error(COSM_EINVAL, "unknown storage format");
}

}  // namespace cosm
