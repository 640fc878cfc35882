// How a merge block reads its partition's staged entries: the runs the
// binning pass left in every tile, concatenated per wave and taken in
// batches.  Shared by the RGB and the SH merge passes.
#pragma once

#include "psf_device.h"
#include "psf_internal.h"

namespace psf {

// Blocks are dispatched to the 8 XCDs round-robin; give each XCD a
// contiguous range of partitions so the offset rows they share stay in one
// L2.
__device__ __forceinline__ uint32_t xcd_partition(uint32_t b, uint32_t P) {
  if (P < 8 || (P & 7u)) return b;
  return (b & 7u) * (P >> 3) + (b >> 3);
}

constexpr uint32_t kRunsPerLane = 4;  // consecutive tile runs each lane keeps in registers

// Largest lane l with excl[l] <= e, where excl is a non-decreasing per-lane
// value (all lanes of the wave must call this).
__device__ __forceinline__ uint32_t wave_upper_bound(uint32_t excl, uint32_t e) {
  uint32_t a = 0;
#pragma unroll
  for (uint32_t step = 32; step > 0; step >>= 1) {
    const uint32_t v = (uint32_t)__shfl((int)excl, (int)(a + step));
    if (a + step < 64 && v <= e) a += step;
  }
  return a;
}

// A chunk: the runs of up to 64 * kRunsPerLane consecutive tiles of the
// wave's slice, lane l holding kRunsPerLane of them; pk[j] packs the start
// of the lane's run j among the lane's entries (< 3 tiles) with the run's
// offset in its tile (< 2^16); excl is the lane's first entry in the
// chunk, total the chunk's entries.
struct RunChunk {
  uint32_t pk[kRunsPerLane];
  uint32_t excl, total;
  uint32_t cbase;
};

// Each wave of a merge block owns a contiguous slice [w_lo, w_hi) of the
// tiles and takes its partition's runs there 64 * kRunsPerLane at a time.
template <uint32_t kWaves>
struct RunReader {
  const PartView& pv;
  uint32_t p, P, lane, w_lo, w_hi;
  const uint32_t *row_lo, *row_hi;

  __device__ __forceinline__ RunReader(const PartView& v, uint32_t part, uint32_t nparts, uint32_t ntiles)
      : pv(v), p(part), P(nparts), lane(__lane_id()) {
    // (in a transposed table a multiple of 4 tiles, so that a lane's runs are
    // one 16-byte load; read in place, any number: the few tiles of a small
    // launch go to as many waves)
    uint32_t per_wave = (ntiles + kWaves - 1) / kWaves;
    if (pv.runs_t) per_wave = (per_wave + 3u) & ~3u;
    w_lo = (threadIdx.x >> 6) * per_wave;
    w_hi = (w_lo + per_wave < ntiles) ? w_lo + per_wave : ntiles;
    const uint32_t stride = (pv.max_tiles + 3u) & ~3u;
    row_lo = pv.runs_t + (uint64_t)p * stride;
    row_hi = row_lo + stride;
  }

  __device__ __forceinline__ RunChunk chunk_of(uint32_t c0) const {
    const uint32_t t = c0 + lane * kRunsPerLane;  // (a multiple of 4 in a transposed table)
    uint32_t r_lo[kRunsPerLane], r_hi[kRunsPerLane];
    if (pv.runs_t) {
      // transposed table: two 16-byte loads (t + 3 < stride: inside the row)
      uint4 lo = make_uint4(0, 0, 0, 0), hi = make_uint4(0, 0, 0, 0);
      if (t < w_hi) {
        lo = *reinterpret_cast<const uint4*>(row_lo + t);
        hi = *reinterpret_cast<const uint4*>(row_hi + t);
      }
      const uint32_t l4[4] = {lo.x, lo.y, lo.z, lo.w}, h4[4] = {hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (uint32_t j = 0; j < kRunsPerLane; ++j) {
        const bool in = t + j < w_hi;
        r_lo[j] = in ? l4[j] : 0u;
        r_hi[j] = in ? h4[j] : 0u;
      }
    } else {
      // the bin pass's table: one column, read in place (the lines are
      // shared by the neighbouring partitions an XCD runs at the same time)
#pragma unroll
      for (uint32_t j = 0; j < kRunsPerLane; ++j) {
        r_lo[j] = 0;
        r_hi[j] = 0;
        if (t + j < w_hi) {
          const uint32_t* offs = pv.runs + (uint64_t)(t + j) * (P + 1) + p;
          r_lo[j] = offs[0];
          r_hi[j] = offs[1];
        }
      }
    }
    RunChunk ch;
    uint32_t lt = 0;
#pragma unroll
    for (uint32_t j = 0; j < kRunsPerLane; ++j) {
      ch.pk[j] = (lt << 16) | r_lo[j];
      lt += r_hi[j] - r_lo[j];
    }
    uint32_t inc = lt;
#pragma unroll
    for (uint32_t off = 1; off < 64; off <<= 1) {
      const uint32_t v = (uint32_t)__shfl_up((int)inc, off);
      if (lane >= off) inc += v;
    }
    ch.excl = inc - lt;
    ch.total = (uint32_t)__shfl((int)inc, 63);
    ch.cbase = c0 * pv.tile;  // (staging holds fewer than 2^32 entries)
    return ch;
  }

  // The batch at entry e0 of a chunk: at[q] is the staging index of the
  // lane's q-th entry, ev[q] whether it exists (absent entries point at a
  // tile's first entry, so that every load stays branch-free and in
  // bounds).  A batch takes the next 64 * kBatch entries of the chunk's
  // concatenated runs.
  template <uint32_t kBatch>
  __device__ __forceinline__ void batch_of(const RunChunk& ch, uint32_t e0, uint32_t* at, bool* ev) const {
#pragma unroll
    for (uint32_t q = 0; q < kBatch; ++q) {
      const uint32_t e = e0 + q * 64 + lane;
      const uint32_t a = wave_upper_bound(ch.excl, e);
      const uint32_t r = e - (uint32_t)__shfl((int)ch.excl, (int)a);
      // the last of lane a's runs that starts at or before r holds it
      uint32_t js = 0, ps = (uint32_t)__shfl((int)ch.pk[0], (int)a);
#pragma unroll
      for (uint32_t j = 1; j < kRunsPerLane; ++j) {
        const uint32_t v = (uint32_t)__shfl((int)ch.pk[j], (int)a);
        if ((v >> 16) <= r) {
          js = j;
          ps = v;
        }
      }
      ev[q] = e < ch.total;
      at[q] = ch.cbase +
              (ev[q] ? (a * kRunsPerLane + js) * pv.tile + (ps & 0xffffu) + (r - (ps >> 16)) : 0u);
    }
  }

  // Calls body(at, ev) for every batch of kBatch entries a lane, in order;
  // first is the slice's first chunk, e0 the entry of it to start at.
  template <uint32_t kBatch, class F>
  __device__ __forceinline__ void for_each_batch(const RunChunk& first, uint32_t e0, F&& body) const {
    for (uint32_t c0 = w_lo; c0 < w_hi; c0 += 64 * kRunsPerLane, e0 = 0) {
      const RunChunk ch = c0 == w_lo ? first : chunk_of(c0);
      for (; e0 < ch.total; e0 += 64 * kBatch) {
        bool ev[kBatch];
        uint32_t at[kBatch];
        batch_of<kBatch>(ch, e0, at, ev);
        body(at, ev);
      }
    }
  }
};

}  // namespace psf
