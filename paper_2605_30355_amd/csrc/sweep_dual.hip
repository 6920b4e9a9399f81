// sweep_dual.hip -- the LDS-resident sweep for small graphs: two colour classes
// per barrier interval.
//
// With up to a thousand edges per class and few workgroups per CU a sweep is a
// chain of latencies: per class a write, a barrier and a read (170 - 210 cycles
// measured, of which the arithmetic between them adds 50), and nothing to hide
// it behind.  Here a lane's entry is an edge (u, v) of class c + 1 together
// with the class c partners of u and v: it reads the four rows, applies class c
// to u and to v (only their own side: each class c edge is computed twice, once
// at either endpoint), then class c + 1 to the pair, and writes u and v.  So two
// classes cost one latency and half again the arithmetic.
//
// A round's entries cover every vertex exactly once (those without an edge in
// class c + 1 are paired with each other, J = 0), and a round reads one of two
// copies of the rows and writes the other, so one barrier ends it.  The twist
// runs inside the last round, on the rows just computed.
//
// Measured, ns per sweep, one replica per workgroup, against k_sweep_lds: 12 x 12
// torus, 1 replica 398 -> 294; 20 x 20 torus, 64 replicas 466 -> 340.  At 2000
// vertices (16 waves a round) the extra arithmetic and the rows' bank conflicts
// cost more than the barriers: 0.67 us against 0.67 with 256 replicas, and worse
// with more.
#include <hip/hip_runtime.h>

#include <string>

#include "device_common.hpp"
#include "internal.hpp"
#include "lds_args.hpp"

namespace cosm {
namespace {

// When phases are wrapped (FP32 on the grid schedule, as in wrap_at_twists: exact
// while every phase stays in (-1, 2) and the difference that either end takes of an
// edge of the first class below two turns).
enum Wrap {
  kWrapUpdates = 0,  // after every update (and always by the fixed-point formats)
  kWrapSweeps = 1,   // in the last round of a sweep (dual_wrap_at_sweeps)
  kWrapTwists = 2    // at the twists (either_end_at_twists)
};

// Class c on one endpoint: row r moves as the endpoint of its edge to row w
// (left as it is).  FP32: aJ carries the sign of the role, two is +2 where r is
// the edge's u and -2 where it is v (the difference exact, either_end_at_twists);
// the fixed-point formats take the role as flip.  The pair update's r bit for bit
// (update_reg_words).
template <int ST, int W, bool WRAP>
__device__ __forceinline__ void update_end(uint32_t (&r)[W], const uint32_t (&w)[W], float aJ,
                                           uint32_t role, float pm) {
  if constexpr (ST == COSM_STORE_FP32) {
#pragma unroll
    for (int k = 0; k < W; k++) {
      const float xr = __uint_as_float(r[k]), xw = __uint_as_float(w[k]);
      const float p = __builtin_fmaf(xr - xw, __uint_as_float(role), pm);
      const float x = xr - __uint_as_float((__float_as_uint(p) << 31) + __float_as_uint(aJ));
      r[k] = __float_as_uint(WRAP ? fract1(x) : x);
    }
  } else {
    uint32_t other[W];
#pragma unroll
    for (int k = 0; k < W; k++) other[k] = w[k];
    update_reg_words<ST, W>(r, other, aJ, role);
  }
}

template <int ST, int W, int ROUNDS, int WRAP>
__global__ void __launch_bounds__(kDualVerticesMax) k_sweep_dual(const LdsArgs a) {
  extern __shared__ uint32_t lds[];
  using F = Fmt<ST>;
  constexpr bool RD = ST == COSM_STORE_FP32;  // FP32 runs on the grid schedule
  static_assert(RD || WRAP == kWrapUpdates, "the lazy wraps are FP32 grid forms");
  constexpr int RW = W * F::kPerWord;
  constexpr uint32_t ROWB = 4 * W;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int32_t r0 = xcd_block(blockIdx.x, gridDim.x) * RW;
  const int32_t nvalid = min(RW, a.R - r0);
  // two copies of the rows; dynamic LDS starts at address 0 (no static LDS), so
  // a row's byte offset is its address
  const uint32_t copy = (uint32_t)(a.n_rows + kDummyRows) * ROWB;
  uint32_t *lds1 = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(lds) + copy);

  lds_rows_in<ST, W>(lds, a, r0, nvalid, nth);
  for (int s = tid; s < kDummyRows; s += nth) {
    const uint32_t z[W] = {};
    lds_store<W>(lds1, a.n_rows + s, z);
  }
  float *theta_buf = reinterpret_cast<float *>(reinterpret_cast<char *>(lds1) + copy);

  // the entries of every round: kDualWords words per thread (rows of u and v,
  // rows of their partners, J of the pair, of u's edge and of v's, the flips).
  // An even round reads copy 0 and writes copy 1, an odd one the reverse; with
  // an odd number of rounds the copies swap roles from sweep to sweep (swap).
  uint32_t au[ROUNDS], av[ROUNDS], pu[ROUNDS], pv[ROUNDS], du[ROUNDS], dv[ROUNDS];
  uint32_t fu[ROUNDS], fv[ROUNDS];
  float jp[ROUNDS], ju[ROUNDS], jv[ROUNDS];
#pragma unroll
  for (int q = 0; q < ROUNDS; q++) {
    uint32_t w[kDualWords];
#pragma unroll
    for (int k = 0; k < kDualWords; k++)
      w[k] = a.dual[((size_t)q * kDualWords + k) * nth + tid];
    const uint32_t src = q % 2 ? copy : 0u, dst = q % 2 ? 0u : copy;
    au[q] = (w[0] & 0xffffu) * ROWB + src;
    av[q] = (w[0] >> 16) * ROWB + src;
    pu[q] = (w[1] & 0xffffu) * ROWB + src;
    pv[q] = (w[1] >> 16) * ROWB + src;
    du[q] = (w[0] & 0xffffu) * ROWB + dst;
    dv[q] = (w[0] >> 16) * ROWB + dst;
    jp[q] = __uint_as_float(w[2]);
    ju[q] = __uint_as_float(w[3]);
    jv[q] = __uint_as_float(w[4]);
    fu[q] = w[5] & 1u;
    fv[q] = (w[5] >> 1) & 1u;
    if constexpr (RD) {
      ju[q] = fu[q] ? -ju[q] : ju[q];
      jv[q] = fv[q] ? -jv[q] : jv[q];
      fu[q] = 0x40000000u | fu[q] << 31;  // +-2
      fv[q] = 0x40000000u | fv[q] << 31;
    }
  }
  __syncthreads();

  const SweepSchedule sc = a.sch;
  const uint32_t nsw = (uint32_t)a.nsw;
  uint32_t t = (uint32_t)a.t0;  // sweeps done
  uint32_t tw = 0;
  uint32_t flipped = 0;  // odd ROUNDS: 1 when the phases are in copy 1
  ScheduleChunk chunk;
  float pm = 0.0f;
  if constexpr (RD) pm = f32_round_down();
  // the sweep whose step is in lane i of the chunk
  auto sweep = [&](uint32_t i, auto twc) {
    constexpr bool TW = decltype(twc)::value;
    float alpha, twist;
    chunk.get(i, alpha, twist);
    const float alpha_s = alpha * F::kStepScale;
    TwistOps<ST, W> op;
    if constexpr (TW) {
      const int q = (int)(tw % (uint32_t)kThetaChunk);
      tw++;
      if (q == 0) {
        theta_fill(theta_buf, nullptr, kThetaChunk, RW, t + 1, sc.period, a.rid0 + (uint32_t)r0,
                   a.k0, a.k1, sc.win, sc.tshift, sc.tscale);
        __syncthreads();
      }
      float cth[RW], tws[RW];
#pragma unroll
      for (int k = 0; k < RW; k++) {
        cth[k] = theta_buf[q * RW + k];
        tws[k] = twist;
      }
      op.set(cth, tws, sc.win2);
    }
    // (the swapped copies: a source in copy 0 moves up, one in copy 1 down)
    const uint32_t up = ROUNDS % 2 && flipped ? copy : 0u;
    unroll<ROUNDS>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      constexpr bool last = q == ROUNDS - 1;
      constexpr bool wrap_now = WRAP == kWrapUpdates;
      const uint32_t s_off = q % 2 ? 0u - up : up, d_off = 0u - s_off;
      uint32_t wu[W], wv[W], xu[W], xv[W];
      row_load<W>(au[q] + s_off, wu);
      row_load<W>(pu[q] + s_off, xu);
      row_load<W>(av[q] + s_off, wv);
      row_load<W>(pv[q] + s_off, xv);
      update_end<ST, W, wrap_now>(wu, xu, alpha_s * ju[q], fu[q], pm);
      update_end<ST, W, wrap_now>(wv, xv, alpha_s * jv[q], fv[q], pm);
      update_words<ST, W, !wrap_now && lazy_storage(ST), RD>(wu, wv, alpha_s * jp[q], pm);
      if constexpr (last && TW) {
        twist_row<ST, W, WRAP != kWrapUpdates>(op, wu);
        twist_row<ST, W, WRAP != kWrapUpdates>(op, wv);
      } else if constexpr (last && WRAP == kWrapSweeps) {
#pragma unroll
        for (int k = 0; k < W; k++) {
          wu[k] = __float_as_uint(fract1(__uint_as_float(wu[k])));
          wv[k] = __float_as_uint(fract1(__uint_as_float(wv[k])));
        }
      }
      row_store<W>(du[q] + d_off, wu);
      row_store<W>(dv[q] + d_off, wv);
      __syncthreads();
    });
    t++;
    if constexpr (ROUNDS % 2 != 0) flipped ^= 1u;
  };
  // runs of sweeps without a twist, then one with it; a lone wave per SIMD pays
  // every taken branch (some 30 cycles) in full, so neither tests per sweep
  // which it is
  uint32_t pos = 64;
  for (uint32_t left = nsw; left > 0;) {
    if (pos == 64) {
      chunk.fill(sc, t + 1);
      pos = 0;
    }
    const uint32_t here = min(left, 64u - pos);
    const uint64_t tws = chunk.twists >> pos;
    const uint32_t plain = min(here, tws ? (uint32_t)__builtin_ctzll(tws) : 64u);
    for (uint32_t i = 0; i < plain; i++) sweep(pos + i, BoolC<false>{});
    pos += plain;
    left -= plain;
    if (plain < here) {
      sweep(pos, BoolC<true>{});
      pos++;
      left--;
    }
  }
  if constexpr (RD) f32_round_nearest();
  lds_rows_out<ST, W, WRAP != kWrapUpdates>(flipped ? lds1 : lds, a, r0, nvalid, nth);
}

template <int ST, int W, int ROUNDS, int WRAP>
int launch_k(cosm_state *s, const LdsArgs &a) {
  const size_t lds = s->shape.lds_bytes;
  (void)hipFuncSetAttribute((const void *)k_sweep_dual<ST, W, ROUNDS, WRAP>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_sweep_dual<ST, W, ROUNDS, WRAP>), dim3(s->shape.blocks),
                     dim3(s->shape.threads), lds, s->stream, a);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess)
    return set_error(COSM_EDEVICE, std::string("k_sweep_dual: ") + hipGetErrorString(err));
  return COSM_OK;
}

template <int ST, int W, int WRAP>
int launch_r(cosm_state *s, const LdsArgs &a) {
  switch ((s->C + 1) / 2) {
    case 2: return launch_k<ST, W, 2, WRAP>(s, a);
    case 3: return launch_k<ST, W, 3, WRAP>(s, a);
    case 4: return launch_k<ST, W, 4, WRAP>(s, a);
    case 5: return launch_k<ST, W, 5, WRAP>(s, a);
  }
  return set_error(COSM_EINVAL, "two-class form: 3 to 10 classes");
}

template <int W>
int launch_w(cosm_state *s, const LdsArgs &a) {
  switch (s->p.storage) {
    case COSM_STORE_FP32:
      if (either_end_at_twists(*s, true)) return launch_r<COSM_STORE_FP32, W, kWrapTwists>(s, a);
      if (dual_wrap_at_sweeps(*s)) return launch_r<COSM_STORE_FP32, W, kWrapSweeps>(s, a);
      return launch_r<COSM_STORE_FP32, W, kWrapUpdates>(s, a);
    case COSM_STORE_FIX32: return launch_r<COSM_STORE_FIX32, W, kWrapUpdates>(s, a);
    case COSM_STORE_FIX16: return launch_r<COSM_STORE_FIX16, W, kWrapUpdates>(s, a);
  }
  return set_error(COSM_EINVAL, "two-class form: unsupported storage");
}

}  // namespace

size_t dual_lds_bytes(int32_t n_rows, int W) {
  return (size_t)2 * (n_rows + kDummyRows) * W * 4 + (size_t)kThetaFloats * 4;
}

bool dual_form_supported(const cosm_state &s, int32_t W) {
  const int32_t st = s.p.storage;
  if (st == COSM_STORE_FP32 ? !exact_grid_fp32(s)
                            : st != COSM_STORE_FIX32 && st != COSM_STORE_FIX16)
    return false;
  return !s.has_h && s.p.update == COSM_UPDATE_SCS && s.C >= 3 && s.C <= 10 && s.n <= kDualVerticesMax &&
         (W == 1 || W == 2) && dual_lds_bytes(s.n, W) <= (size_t)lds_capacity_bytes();
}

bool dual_form_default(const cosm_state &s, int32_t W, int32_t blocks, int32_t cus) {
  return blocks <= cus && s.p.lds_form <= COSM_LDS_FORM_PAIR && dual_form_supported(s, W);
}

// The entries of every round.  Round q holds classes 2q and 2q + 1 (an odd last
// class alone), entries in order of their first vertex, so that on lattices
// neighbouring lanes or waves read neighbouring rows.
std::vector<std::vector<DualEntry>> dual_entries(const cosm_state &s,
                                                 const std::vector<uint8_t> *wanted) {
  const int32_t n = s.n, C = s.C, rounds = (C + 1) / 2;
  // edge of each vertex in a class
  std::vector<int32_t> e0((size_t)n), e1((size_t)n);
  std::vector<std::vector<int32_t>> by_class((size_t)C);
  for (int64_t k = 0; k < s.m; k++)
    by_class[(size_t)s.h_colour[(size_t)k]].push_back((int32_t)k);
  auto edges_of = [&](int32_t c, std::vector<int32_t> &at) {
    std::fill(at.begin(), at.end(), -1);
    if (c >= C) return;
    for (int32_t k : by_class[(size_t)c]) {
      at[(size_t)s.h_eu[(size_t)k]] = k;
      at[(size_t)s.h_ev[(size_t)k]] = k;
    }
  };
  std::vector<std::vector<DualEntry>> out((size_t)rounds);
  std::vector<uint8_t> done((size_t)n);
  for (int32_t q = 0; q < rounds; q++) {
    if (wanted != nullptr && !(*wanted)[(size_t)q]) continue;
    out[(size_t)q].reserve((size_t)n / 2 + 1);
    edges_of(2 * q, e0);
    edges_of(2 * q + 1, e1);
    std::fill(done.begin(), done.end(), 0);
    // an endpoint's edge in class 2q: the partner, J and whether it is the v there
    auto end = [&](int32_t x, int32_t *partner, int32_t *J, int32_t *flip) {
      const int32_t k = x >= 0 ? e0[(size_t)x] : -1;
      *partner = -1;
      *J = 0;
      *flip = 0;
      if (k < 0) return;
      *flip = s.h_ev[(size_t)k] == x ? 1 : 0;
      *partner = *flip ? s.h_eu[(size_t)k] : s.h_ev[(size_t)k];
      *J = s.h_J[(size_t)k];
    };
    auto push = [&](int32_t u, int32_t v, int32_t J) {
      DualEntry e{};
      e.u = u;
      e.v = v;
      e.J = J;
      end(u, &e.pu, &e.Ju, &e.fu);
      end(v, &e.pv, &e.Jv, &e.fv);
      out[(size_t)q].push_back(e);
    };
    int32_t lone = -1;  // a vertex without an edge in class 2q + 1, waiting for another
    for (int32_t x = 0; x < n; x++) {
      if (done[(size_t)x]) continue;
      const int32_t k = e1[(size_t)x];
      if (k >= 0) {
        const int32_t u = s.h_eu[(size_t)k], v = s.h_ev[(size_t)k];
        done[(size_t)u] = done[(size_t)v] = 1;
        push(u, v, s.h_J[(size_t)k]);
      } else if (lone < 0) {
        lone = x;
      } else {
        push(lone, x, 0);
        lone = -1;
      }
    }
    if (lone >= 0) push(lone, -1, 0);
  }
  return out;
}

int dual_schedule_for(const cosm_state &s, int32_t W, LdsSchedule *out) {
  if (!dual_form_supported(s, W))
    return set_error(COSM_ERANGE, "the two-class form does not apply");
  const int32_t n = s.n, rounds = (s.C + 1) / 2;
  LdsSchedule L;
  L.G = W == 1 ? 32 : 64 / W;
  L.n_rows = n;
  L.slot_vertex.resize((size_t)n);
  for (int32_t v = 0; v < n; v++) L.slot_vertex[(size_t)v] = v;
  const std::vector<std::vector<DualEntry>> lists = dual_entries(s);
  size_t most = 0;
  for (const auto &l : lists) most = std::max(most, l.size());
  L.nth = (int32_t)std::max<size_t>(64, (most + 63) / 64 * 64);
  const int32_t nth = L.nth;
  L.dual_words.assign((size_t)rounds * kDualWords * nth, 0u);
  for (int32_t q = 0; q < rounds; q++)
    for (int32_t t = 0; t < nth; t++) {
      const auto &l = lists[(size_t)q];
      DualEntry e{-1, -1, -1, -1, 0, 0, 0, 0, 0};
      if ((size_t)t < l.size()) e = l[(size_t)t];
      // (lanes and endpoints without an edge take dummy rows)
      const uint32_t du = (uint32_t)(n + (t & 31)), dv = du + 32u;
      auto row = [](int32_t x, uint32_t dummy) { return x >= 0 ? (uint32_t)x : dummy; };
      auto word = [](int32_t J) { return __builtin_bit_cast(uint32_t, (float)J); };
      const uint32_t w[kDualWords] = {row(e.u, du) | row(e.v, dv) << 16,
                                      row(e.pu, du) | row(e.pv, dv) << 16,
                                      word(e.J), word(e.Ju), word(e.Jv),
                                      (uint32_t)(e.fu | e.fv << 1)};
      for (int k = 0; k < kDualWords; k++)
        L.dual_words[((size_t)q * kDualWords + k) * nth + t] = w[k];
    }
  L.dual = true;
  L.fuse = true;
  *out = std::move(L);
  return COSM_OK;
}

int launch_sweeps_dual(cosm_state *s, const LdsArgs &a, int W) {
  if (W == 2) return launch_w<2>(s, a);
  if (W == 1) return launch_w<1>(s, a);
  return set_error(COSM_EINVAL, "two-class form: one or two words per row");
}

}  // namespace cosm
