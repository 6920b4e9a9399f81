// lds_args.hpp -- the arguments of the LDS-resident sweep kernels of
// kernels.hip (the pair form) and sweep_reg.hip (the register-owner form),
// and the launcher of the latter.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.hpp"
#include "internal.hpp"

namespace cosm {

struct LdsArgs {
  void *phases;
  const EdgeDesc *desc;       // [total_slots * nth] lane schedule
  const int32_t *Kc;          // [C] slots per thread of each class
  const int32_t *slot_vertex; // [n_rows]
  const int32_t *h_slot;      // [n_rows] bias field per slot, or null (no fields)
  int32_t R, n_rows, C, total_slots;
  int64_t t0, nsw;
  SweepSchedule sch;
  uint32_t k0, k1, rid0;
  uint32_t bar_mask;          // register-resident schedule: barrier after slot j
  // fused form: the twist runs inside the last class's sub-sweep, with fuse_k
  // rows per thread (after the repeated slots in desc) that no edge of that
  // class touches
  int32_t fuse_k;
  // register-owner form: [K][nth] register vertices, and whether the slot of
  // edges between two LDS rows is in use
  const int32_t *reg_vertex;
  int32_t reg_free;
  const uint32_t *dual;       // two-class and full-gradient forms: their entries
  int32_t last_slot0;         // fused fields: the last class's first slot
};

namespace {

// HBM [n][R] -> the LDS rows of the workgroup's replicas, dummy rows zero.
template <int ST, int W>
__device__ __forceinline__ void lds_rows_in(uint32_t *lds, const LdsArgs &a, int32_t r0,
                                            int32_t nvalid, int nth) {
  using F = Fmt<ST>;
  constexpr int RW = W * F::kPerWord;
  for (int s = threadIdx.x; s < a.n_rows; s += nth) {
    const size_t base = (size_t)a.slot_vertex[s] * a.R + r0;
    float v[RW];
#pragma unroll
    for (int k = 0; k < RW; k++) v[k] = (k < nvalid) ? F::load_elem(a.phases, base + k) : 0.0f;
    uint32_t w[W];
    F::template pack<W>(v, w);
    lds_store<W>(lds, s, w);
  }
  for (int s = threadIdx.x; s < kDummyRows; s += nth) {
    const uint32_t z[W] = {};
    lds_store<W>(lds, a.n_rows + s, z);
  }
}

// LDS rows -> HBM.  16-bit float phases wrapped at the twists only go back as
// they are (|y| < 1, within the drift bound): wrapping them here would change
// how later steps round them, and with it the trajectory whenever a trial is
// split over several calls.  FP32 wraps exactly.
template <int ST, int W, bool LAZY>
__device__ __forceinline__ void lds_rows_out(uint32_t *lds, const LdsArgs &a, int32_t r0,
                                             int32_t nvalid, int nth) {
  using F = Fmt<ST>;
  constexpr int RW = W * F::kPerWord;
  for (int s = threadIdx.x; s < a.n_rows; s += nth) {
    const size_t base = (size_t)a.slot_vertex[s] * a.R + r0;
    uint32_t w[W];
    lds_load<W>(lds, s, w);
    float v[RW];
    F::template unpack<W>(w, v);
#pragma unroll
    for (int k = 0; k < RW; k++)
      if (k < nvalid)
        F::store_elem(a.phases, base + k, LAZY && ST == COSM_STORE_FP32 ? F::wrap(v[k]) : v[k]);
  }
}

// Compile-time loop indices and flags for the unrolled class loops.
template <int V>
struct IntC {
  static constexpr int value = V;
};
template <bool V>
struct BoolC {
  static constexpr bool value = V;
};
// fn(IntC<0>), ..., fn(IntC<N - 1>)
template <int N, int I = 0, typename Fn>
__device__ __forceinline__ void unroll(Fn &&fn) {
  if constexpr (I < N) {
    fn(IntC<I>{});
    unroll<N, I + 1>(fn);
  }
}

}  // namespace

// The two-class form's sweeps (sweep_dual.hip).
int launch_sweeps_dual(cosm_state *s, const LdsArgs &a, int W);

// The full-gradient sweeps in LDS (sweep_full.hip).
int launch_sweeps_full(cosm_state *s, const LdsArgs &a);

// The sweeps with fields and twist inside the last class (sweep_fields.hip), for
// states that fields_fused accepts.
int launch_sweeps_fields(cosm_state *s, const LdsArgs &a, int W);

// The register-owner form's sweeps for the state's storage and W words per
// row (sweep_reg.hip); COSM_EINVAL for a storage, register count or class
// count that has no kernel.
int launch_sweeps_reg(cosm_state *s, const LdsArgs &a, int W);

}  // namespace cosm
