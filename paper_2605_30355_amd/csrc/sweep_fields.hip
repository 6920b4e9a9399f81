// sweep_fields.hip -- the LDS-resident sweep with bias fields, for lane schedules
// held in registers.
//
// The field sub-sweep and the twist are each a visit to every row after the last
// class; as passes of their own they cost a read and a write of all rows and a
// barrier each.  Here they run inside the last class's sub-sweep: a row is final
// for the class once its edge there is updated, so the same lane applies the
// field, on twist sweeps the twist, and writes the row once; the rows that no edge
// of the last class touches are dealt to the lanes and visited in the same
// interval.  Since every row is visited at the end of every sweep, FP32 phases on
// the grid are wrapped there only, where a sweep's drift stays below a turn.
//
#include <hip/hip_runtime.h>

#include <string>

#include "device_common.hpp"
#include "internal.hpp"
#include "lds_args.hpp"

namespace cosm {
namespace {

constexpr int kFieldInnerMax = 12, kFieldLastMax = 4;

// The end of a sweep on one row: the field h (0: none) and, with TW, the twist,
// on the row's stored (rounded) words as passes of their own would take them.
// SWEEP_WRAP: the row comes unwrapped and is wrapped here.
template <int ST, int W, bool TW, bool SWEEP_WRAP, bool LAZY, bool RD>
__device__ __forceinline__ void end_row(uint32_t (&w)[W], float ah, const TwistOps<ST, W> &op,
                                        float pm) {
  using F = Fmt<ST>;
  constexpr int RW = W * F::kPerWord;
  if constexpr (RD) {
    // s = +1 iff x lies in [0, 1/2): floor(2x) even, also for x not wrapped
#pragma unroll
    for (int k = 0; k < W; k++) {
      const float x = __uint_as_float(w[k]);
      w[k] = __float_as_uint(fract1(x - step_by_parity(x, ah, pm)));
    }
  } else if (ah != 0.0f) {
    float v[RW];
    F::template unpack<W>(w, v);
#pragma unroll
    for (int k = 0; k < RW; k++) field_update<ST, LAZY>(v[k], ah);
    F::template pack<W>(v, w);
  }
  if constexpr (TW) twist_row<ST, W, LAZY || SWEEP_WRAP>(op, w);
}

// EI: the most slots before the last class, EL: the most in it.  EXACT: one slot
// per class, EI + 1 of them.
template <int ST, int W, int EI, int EL, bool EXACT, bool SWEEP_WRAP, bool LAZY, bool RD>
__global__ void __launch_bounds__(1024) k_sweep_fields(const LdsArgs a) {
  static_assert(!SWEEP_WRAP || RD, "the wrap at sweep ends is the FP32 grid form's");
  static_assert(!RD || ST == COSM_STORE_FP32, "the parity step is an FP32 grid form");
  extern __shared__ uint32_t lds[];
  using F = Fmt<ST>;
  constexpr int RW = W * F::kPerWord;
  constexpr uint32_t ROWB = 4 * W;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int32_t r0 = xcd_block(blockIdx.x, gridDim.x) * RW;
  const int32_t nvalid = min(RW, a.R - r0);

  lds_rows_in<ST, W>(lds, a, r0, nvalid, nth);
  float *theta_buf = reinterpret_cast<float *>(lds + (size_t)(a.n_rows + kDummyRows) * W);
  float *dir_buf = theta_buf + kThetaFloats;

  // the lane schedule; the last class's slots also hold their rows' fields
  const int inner = EXACT ? EI : a.last_slot0, last = EXACT ? EL : a.total_slots - inner;
  const uint32_t du = (uint32_t)(a.n_rows + (tid & 31)) * ROWB;
  const uint32_t dv = (uint32_t)(a.n_rows + 32 + (tid & 31)) * ROWB;
  auto slot = [&](int j, bool in, uint32_t &u, uint32_t &v, float &J) {
    EdgeDesc d{kEmptySlot, 0.0f};
    if (in) d = a.desc[(size_t)j * nth + tid];
    const bool empty = d.slots == kEmptySlot;
    u = empty ? du : (d.slots & 0xffffu) * ROWB;
    v = empty ? dv : (d.slots >> 16) * ROWB;
    J = empty ? 0.0f : d.J;
  };
  uint32_t ua[EI], va[EI], ul[EL], vl[EL];
  float jr[EI], jl[EL], hu[EL], hv[EL];
#pragma unroll
  for (int j = 0; j < EI; j++) slot(j, EXACT || j < inner, ua[j], va[j], jr[j]);
  auto field = [&](uint32_t at) {  // (0 on the dummy rows)
    return at < (uint32_t)a.n_rows * ROWB ? (float)a.h_slot[at / ROWB] : 0.0f;
  };
#pragma unroll
  for (int k = 0; k < EL; k++) {
    slot(inner + k, EXACT || k < last, ul[k], vl[k], jl[k]);
    hu[k] = field(ul[k]);
    hv[k] = field(vl[k]);
  }
  // the rows outside the last class
  uint32_t fr[kFuseRowsMax];
  float fh[kFuseRowsMax];
#pragma unroll
  for (int q = 0; q < kFuseRowsMax; q++) {
    fr[q] = kEmptySlot;
    fh[q] = 0.0f;
    if (q < a.fuse_k) {
      const uint32_t sl = a.desc[(size_t)(a.total_slots + kStreamRepeat + q) * nth + tid].slots;
      if (sl != kEmptySlot) {
        fr[q] = sl * ROWB;
        fh[q] = (float)a.h_slot[sl];
      }
    }
  }
  __syncthreads();

  const SweepSchedule sc = a.sch;
  const uint32_t nsw = (uint32_t)a.nsw;
  uint32_t t = (uint32_t)a.t0;
  uint32_t tw = 0;
  ScheduleChunk chunk;
  float pm = 0.0f;
  if constexpr (RD) pm = f32_round_down();
  for (uint32_t it = 0; it < nsw; it++) {
    t++;
    if ((it & 63u) == 0u) chunk.fill(sc, t);
    float alpha, twist;
    chunk.get(it & 63u, alpha, twist);
    const float alpha_s = alpha * F::kStepScale;
    TwistOps<ST, W> op;
    const bool twist_now = chunk.twist_at(it & 63u);
    if (twist_now) {
      const int q = (int)(tw % (uint32_t)kThetaChunk);
      tw++;
      if (q == 0) {
        theta_fill(theta_buf, dir_buf, kThetaChunk, RW, t, sc.period, a.rid0 + (uint32_t)r0, a.k0,
                   a.k1, sc.win, sc.tshift, sc.tscale);
        __syncthreads();
      }
      float cth[RW], tws[RW];
#pragma unroll
      for (int k = 0; k < RW; k++) {
        cth[k] = theta_buf[q * RW + k];
        tws[k] = dir_buf[q * RW + k] * twist;
      }
      op.set(cth, tws, sc.win2);
    }
    // the last class and the rows it leaves out
    auto sweep_end = [&](auto twc) {
      constexpr bool TW = decltype(twc)::value;
#pragma unroll
      for (int k = 0; k < EL; k++) {
        if (!EXACT && k >= last) continue;
        uint32_t wu[W], wv[W];
        lds_load_at<W>(lds, ul[k], wu);
        lds_load_at<W>(lds, vl[k], wv);
        update_words<ST, W, LAZY || SWEEP_WRAP, RD>(wu, wv, alpha_s * jl[k], pm);
        end_row<ST, W, TW, SWEEP_WRAP, LAZY, RD>(wu, alpha * hu[k], op, pm);
        end_row<ST, W, TW, SWEEP_WRAP, LAZY, RD>(wv, alpha * hv[k], op, pm);
        lds_store_at<W>(lds, ul[k], wu);
        lds_store_at<W>(lds, vl[k], wv);
      }
#pragma unroll
      for (int q = 0; q < kFuseRowsMax; q++)
        if (q < a.fuse_k && fr[q] != kEmptySlot) {
          uint32_t w[W];
          lds_load_at<W>(lds, fr[q], w);
          end_row<ST, W, TW, SWEEP_WRAP, LAZY, RD>(w, alpha * fh[q], op, pm);
          lds_store_at<W>(lds, fr[q], w);
        }
    };
#pragma unroll
    for (int j = 0; j < EI; j++) {
      if (!EXACT && j >= inner) continue;
      edge_rows<ST, W, LAZY || SWEEP_WRAP, RD>(lds, ua[j], va[j], alpha_s * jr[j], pm);
      if (EXACT || ((a.bar_mask >> j) & 1u)) __syncthreads();
    }
    if (twist_now) sweep_end(BoolC<true>{});
    else sweep_end(BoolC<false>{});
    __syncthreads();
  }
  if constexpr (RD) f32_round_nearest();
  lds_rows_out<ST, W, LAZY || SWEEP_WRAP>(lds, a, r0, nvalid, nth);
}

template <int ST, int W, int EI, int EL, bool EXACT, bool SWEEP_WRAP, bool LAZY, bool RD>
int launch_k(cosm_state *s, const LdsArgs &a) {
  const size_t lds = s->shape.lds_bytes;
  (void)hipFuncSetAttribute((const void *)k_sweep_fields<ST, W, EI, EL, EXACT, SWEEP_WRAP, LAZY, RD>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_sweep_fields<ST, W, EI, EL, EXACT, SWEEP_WRAP, LAZY, RD>),
                     dim3(s->shape.blocks), dim3(s->shape.threads), lds, s->stream, a);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess)
    return set_error(COSM_EDEVICE, std::string("k_sweep_fields: ") + hipGetErrorString(err));
  return COSM_OK;
}

template <int ST, int W, int EI, int EL, bool EXACT>
int launch_v(cosm_state *s, const LdsArgs &a) {
  if constexpr (ST == COSM_STORE_FP16 || ST == COSM_STORE_BF16 || ST == COSM_STORE_FP16_PK) {
    if (lazy16(*s)) return launch_k<ST, W, EI, EL, EXACT, false, true, false>(s, a);
  }
  if constexpr (ST == COSM_STORE_FP32) {
    if (wrap_at_sweeps(*s)) return launch_k<ST, W, EI, EL, EXACT, true, false, true>(s, a);
    if (exact_grid_fp32(*s)) return launch_k<ST, W, EI, EL, EXACT, false, false, true>(s, a);
  }
  return launch_k<ST, W, EI, EL, EXACT, false, false, false>(s, a);
}

template <int ST, int W>
int launch_w(cosm_state *s, const LdsArgs &a) {
  const int inner = a.last_slot0, last = a.total_slots - inner;
  if (inner == 3 && a.C == 4 && a.bar_mask == 15u) return launch_v<ST, W, 3, 1, true>(s, a);
  if (inner <= 6 && last <= 2) return launch_v<ST, W, 6, 2, false>(s, a);
  return launch_v<ST, W, kFieldInnerMax, kFieldLastMax, false>(s, a);
}

template <int ST>
int launch_st(cosm_state *s, const LdsArgs &a, int W) {
  if (W == 4) return launch_w<ST, 4>(s, a);
  if (W == 2) return launch_w<ST, 2>(s, a);
  if (W == 1) return launch_w<ST, 1>(s, a);
  return set_error(COSM_EINVAL, "unsupported replicas per workgroup");
}

}  // namespace

// Fields and twist inside the last class: schedules in registers whose rows
// outside the last class are at most kFuseRowsMax per thread (more of them, dealt
// one at a time, lengthen the interval by more than a pass costs), and a last class
// that is not empty.
// 3-regular graph, N = 2000, 1024 replicas, whole trials of 2000 sweeps: with passes
// 3.76 ms, fused and wrapped at the sweep ends 2.56 ms.
bool fields_fused(const cosm_state &s) {
  const LdsSchedule &L = s.lds;
  if (!s.has_h || !L.fuse || L.full || L.reg_k > 0 || (int32_t)L.K.size() != s.C || s.C < 1)
    return false;
  const int32_t last = L.K.back();
  return last > 0 && last <= kFieldLastMax && L.total_slots - last <= kFieldInnerMax;
}

int launch_sweeps_fields(cosm_state *s, const LdsArgs &la, int W) {
  LdsArgs a = la;
  a.last_slot0 = a.total_slots - s->lds.K.back();
  switch (s->p.storage) {
    case COSM_STORE_FP32: return launch_st<COSM_STORE_FP32>(s, a, W);
    case COSM_STORE_FP16: return launch_st<COSM_STORE_FP16>(s, a, W);
    case COSM_STORE_FP16_PK: return launch_st<COSM_STORE_FP16_PK>(s, a, W);
    case COSM_STORE_BF16: return launch_st<COSM_STORE_BF16>(s, a, W);
    case COSM_STORE_FIX16: return launch_st<COSM_STORE_FIX16>(s, a, W);
    case COSM_STORE_FIX32: return launch_st<COSM_STORE_FIX32>(s, a, W);
  }
  return set_error(COSM_EINVAL, "unknown storage format");
}

}  // namespace cosm
