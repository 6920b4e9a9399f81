// readout_group.hpp -- the bisector readout of Q replicas by one workgroup.
//
// readout_block (device_common.hpp) reads a replica's phases at stride R, its edges
// twice and scans its bisectors in one thread.  Here a workgroup takes Q consecutive
// replicas (one access per vertex row), a vertex's code is one byte per replica (the
// bisector at which its spin flips, at most 127 of them, and its first side), so that
// one word serves an edge's end in all of them and the edges are read once per Q; the
// cut follows from the energy, cut = -(sum J + H) / 2; the scan over the bisectors is
// a wave's; and spins go out four vertices at a time.
// 141 x 141 torus, 4096 replicas 1297 -> 384 us; 5-regular N = 20000, 2048 693 -> 158;
// 300 x 300 torus, 1024 (one replica per workgroup) 2099 -> 997; 12 x 12, 1 8.7 -> 4.0.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.hpp"
#include "hbm_vec.hpp"

namespace cosm {
namespace {

// LDS of readout_group: per replica 16 partial sums and the results, B + 1 bins, the
// bisector angles, then the codes (16-byte aligned).
inline size_t readout_group_lds(int32_t n, int32_t B, int Q) {
  const size_t head = ((size_t)Q * (18 + B + 1) * 8 + (size_t)B * 4 + 15) / 16 * 16;
  return head + ((size_t)n + 3) / 4 * 4 * Q + 16;
}

// SMALL: the sum of |J| is below 2^30, so energies and bins fit 32 bits.
template <int ST, int Q, bool SMALL>
__device__ void readout_group(const ReadoutArgs &a, int32_t r0, int64_t *sm64) {
  using F = Fmt<ST>;
  typedef typename std::conditional<SMALL, int32_t, int64_t>::type sum_t;
  typedef typename std::conditional<SMALL, uint32_t, unsigned long long>::type bin_t;
  typedef typename std::conditional<Q == 4, uint32_t,
                                    typename std::conditional<Q == 2, uint16_t, uint8_t>::type>::type
      code_t;
  const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, wv = tid >> 6;
  const int nw = nth >> 6;
  const int B = a.B;
  int64_t *red = sm64;               // [Q][16]
  int64_t *best_p = sm64 + Q * 16;   // [Q]
  bin_t *bins = reinterpret_cast<bin_t *>(sm64 + Q * 18);  // [Q][B + 1]
  float *beta = reinterpret_cast<float *>(sm64 + Q * (18 + B + 1));
  const size_t head = ((size_t)Q * (18 + B + 1) * 8 + (size_t)B * 4 + 15) / 16 * 16;
  code_t *code = reinterpret_cast<code_t *>(reinterpret_cast<char *>(sm64) + head);  // [n]

  for (int p = tid; p < Q * (B + 1); p += nth) bins[p] = 0;
  for (int p = tid; p < B; p += nth) {
    if (a.grid)  // (p << 23 stays below 2^31: at most 127 bisectors)
      beta[p] = (float)((((uint32_t)p << 23) + (uint32_t)B) / (2u * (uint32_t)B)) * kQ23;
    else
      beta[p] = (float)p / (float)(2 * B);
  }
  __syncthreads();
  const int nvalid = min(Q, a.R - r0);
  const bool wide = a.R % Q == 0;  // r0 is a multiple of Q
  const float per_turn = (float)(2 * B);
  for (int i = tid; i < a.n; i += nth) {
    float x[Q];
    const size_t at = (size_t)i * a.R + r0;
    if (wide) {
      load_vec<ST, Q>(a.phases, at, x);
    } else {
#pragma unroll
      for (int q = 0; q < Q; q++) x[q] = q < nvalid ? F::load_elem(a.phases, at + q) : 0.0f;
    }
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < Q; q++) {
      const float t = F::to_turn(x[q]);
      const bool neg = !(t < 0.5f);
      const float y = neg ? t - 0.5f : t;
      // the last bisector at or below y: y 2B is within one of its index
      int lo = min((int)(y * per_turn), B - 1);
      if (beta[lo] > y) lo--;
      else if (lo + 1 < B && beta[lo + 1] <= y) lo++;
      c |= ((uint32_t)(lo + 1) | (neg ? 0x80u : 0u)) << (8 * q);
    }
    code[i] = (code_t)c;
  }
  __syncthreads();
  sum_t h0[Q];
#pragma unroll
  for (int q = 0; q < Q; q++) h0[q] = 0;
  for (int64_t k = tid; k < a.m; k += nth) {
    const uint32_t cu = code[a.eu[k]], cv = code[a.ev[k]];
    const sum_t J = a.J[k];
    const uint32_t d = cu ^ cv;
#pragma unroll
    for (int q = 0; q < Q; q++) h0[q] += (d >> (8 * q)) & 0x80u ? J : -J;
    if (d & 0x7f7f7f7fu) {
#pragma unroll
      for (int q = 0; q < Q; q++) {
        const int qu = (cu >> (8 * q)) & 0x7f, qv = (cv >> (8 * q)) & 0x7f;
        if (qu == qv) continue;
        const int lo = min(qu, qv), hi = max(qu, qv);
        const sum_t e2 = 2 * ((d >> (8 * q)) & 0x80u ? J : -J);
        if (lo < B) atomicAdd(&bins[q * (B + 1) + lo], (bin_t)(-e2));
        if (hi < B) atomicAdd(&bins[q * (B + 1) + hi], (bin_t)e2);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < Q; q++) {
    const int64_t w = wave_sum((int64_t)h0[q]);
    if (lane == 0) red[q * 16 + wv] = w;
  }
  __syncthreads();
  // replica q: the energies of the bisectors by a wave's prefix sums, the lowest,
  // then the lowest index
  for (int q = wv; q < Q; q += nw) {
    int64_t run = wave_sum(lane < nw ? red[q * 16 + lane] : 0);
    int64_t best = INT64_MAX;
    int bp = 0;
    for (int p0 = 0; p0 < B; p0 += 64) {
      const int p = p0 + lane;
      int64_t v = p > 0 && p < B ? (int64_t)(sum_t)bins[q * (B + 1) + p] : 0;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int64_t o = __shfl_up(v, off, 64);
        if (lane >= off) v += o;
      }
      const int64_t H = run + v;
      if (p < B && H < best) {
        best = H;
        bp = p;
      }
      run += __shfl(v, 63, 64);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const int64_t o = __shfl_xor(best, off, 64);
      const int op = __shfl_xor(bp, off, 64);
      if (o < best || (o == best && op < bp)) {
        best = o;
        bp = op;
      }
    }
    if (lane == 0) {
      best_p[q] = bp;
      if (q < nvalid) {
        a.H[r0 + q] = best;
        a.cut[r0 + q] = -(a.sumJ + best) / 2;
        a.best_p[r0 + q] = bp;
      }
    }
  }
  __syncthreads();
  int bp[Q];
#pragma unroll
  for (int q = 0; q < Q; q++) bp[q] = (int)best_p[q];
  // spin bytes: +1 or -1 (0xff)
  auto spin = [&](uint32_t byte, int p) -> uint32_t {
    const bool plus = ((byte & 0x80u) == 0) == (p < (int)(byte & 0x7fu));
    return plus ? 0x01u : 0xffu;
  };
  const uint8_t *bytes = reinterpret_cast<const uint8_t *>(code);
  for (int i = 4 * tid; i < a.n; i += 4 * nth) {
    if (i + 4 <= a.n) {
      uint32_t w[Q];
#pragma unroll
      for (int k = 0; k < Q; k++) w[k] = reinterpret_cast<const uint32_t *>(code)[(i / 4) * Q + k];
#pragma unroll
      for (int q = 0; q < Q; q++) {
        if (q >= nvalid) continue;
        uint32_t s = 0;
#pragma unroll
        for (int v = 0; v < 4; v++) {
          const int b = v * Q + q;
          s |= spin((w[b / 4] >> (8 * (b % 4))) & 0xffu, bp[q]) << (8 * v);
        }
        __builtin_memcpy(a.spins + (size_t)(r0 + q) * a.n + i, &s, 4);
      }
    } else {
      for (int v = i; v < a.n; v++)
        for (int q = 0; q < nvalid; q++) {
          // (the index into bp stays a constant)
          int p = bp[0];
#pragma unroll
          for (int z = 1; z < Q; z++) p = q == z ? bp[z] : p;
          a.spins[(size_t)(r0 + q) * a.n + v] = (int8_t)spin(bytes[(size_t)v * Q + q], p);
        }
    }
  }
}

}  // namespace
}  // namespace cosm
