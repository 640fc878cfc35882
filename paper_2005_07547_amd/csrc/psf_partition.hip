// Partitioned insertion for gfx950.
//
// Global atomics on MI355X sustain only ~2e10 operations/s, far below what
// HBM streaming allows, so the fast insert path avoids them.  The table is
// split into partitions of 2^part_log2 consecutive slots (the partition of a
// key is the top bits of its hash, its probe sequence stays inside the
// partition).  Insertion then runs in two passes:
//
//   bin   -- one block per tile of records computes the keys, merges
//            records of one cell in neighbouring lanes into one entry,
//            counts entries per partition in LDS, sorts the tile by
//            partition in LDS and writes it out coalesced (keys, then
//            16-byte values {r, g, b, n}) to a staging area, plus the tile's
//            exclusive per-partition offsets (and, for the fused query, each
//            record's entry position in the tile);
//   (transpose -- for large launches, the offset table turned so that a
//            partition's offsets are one row);
//   merge -- one block per partition loads the partition's keys into LDS,
//            gathers the keys of that partition's entries from every tile,
//            finds or claims each one's slot, lists the touched slots, and
//            accumulates count (u32) and sums (binary64; also the weights
//            of a weighted table and the squared luminances of one that
//            keeps the variance) of the touched cells with LDS atomics
//            (a dense launch: of every slot, as the entries are read), then
//            writes them back:
//            either adding into the global accumulators (plain insert) or,
//            when the whole frame is in this launch, applying the temporal
//            blend (Eq. 10-11) directly so the accumulators never touch HBM;
//            when the frame's queries are its records, it then writes each
//            staged entry's new cell value over the entry (16-bit states'
//            over its key);
//   unstage -- one block per tile returns those values in record order.
//
// A partition is owned by exactly one block in the merge pass, so the
// write-back uses plain loads and stores.
#include "psf_device.h"
#include "psf_internal.h"
#include "psf_runs.h"

namespace psf {

constexpr uint32_t kMaxPartLog2 = 12;

bool bin_per_ok(uint32_t per) { return per == 8 || per == 12 || per == 16; }

// LDS staging bytes per record of a binning tile: 16 (every tile's values
// in one float4 pass) where two blocks per CU still fit, else 12 (a tile
// with more than 3/4 of its records as entries stages its values in two
// halves).
__host__ __device__ constexpr size_t bin_lds_per_record(uint32_t tile) { return tile <= 4096 ? 16 : 12; }
uint32_t bin_tile(uint32_t per) { return 512 * per; }

// Records per tile of a launch of n records at the default binning width.
// Tiles of 4096 records fill the 256 CUs from a million records on; a smaller
// launch takes tiles of 2048 or 1024 (up to kSmallTiles of them, two a CU),
// while a tile is still twice the partitions whose counters each tile scans
// and writes.  8,192 records: bin 14.9 -> 7.2, merge 12.9 -> 10.7, answers 5.1
// -> 4.0 us; 250,749: 21.4 -> 10.7, 16.7 -> 17.0, 8.1 -> 4.8; 921,600 of the SH
// payload (tiles of 2048): bin 32.4 -> 25.1.
uint32_t launch_tile(uint64_t n, uint32_t nparts) {
  for (uint32_t tile = 1024; tile < 4096; tile *= 2)
    if (n <= (uint64_t)kSmallTiles * tile && 2 * nparts <= tile) return tile;
  return 4096;
}

uint32_t small_tiles(uint64_t cap, uint32_t nparts) {
  uint64_t most = 0;
  for (uint32_t tile = 1024; tile < 4096; tile *= 2) {
    if (2 * nparts > tile) continue;
    const uint64_t n = cap < (uint64_t)kSmallTiles * tile ? cap : (uint64_t)kSmallTiles * tile;
    if ((n + tile - 1) / tile > most) most = (n + tile - 1) / tile;
  }
  return (uint32_t)most;
}

// Exclusive prefix sum of cnt[0..m) in LDS, in place; returns the total.
// Called by all kThreads threads of the block.
template <int kThreads>
__device__ uint32_t block_exclusive_scan(uint32_t* cnt, uint32_t m, uint32_t* s_wave) {
  const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
  const uint32_t chunk = (m + kThreads - 1) / kThreads;
  const uint32_t lo = tid * chunk;
  uint32_t local = 0;
  for (uint32_t c = 0; c < chunk; ++c)
    if (lo + c < m) local += cnt[lo + c];
  // inclusive scan across the wave
  uint32_t inc = local;
  for (uint32_t off = 1; off < 64; off <<= 1) {
    const uint32_t v = __shfl_up(inc, off);
    if (lane >= off) inc += v;
  }
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  if (tid == 0) {
    uint32_t run = 0;
    for (int w = 0; w < kThreads / 64; ++w) {
      const uint32_t v = s_wave[w];
      s_wave[w] = run;
      run += v;
    }
    s_wave[kThreads / 64] = run;
  }
  __syncthreads();
  uint32_t run = s_wave[wave] + inc - local;
  for (uint32_t c = 0; c < chunk; ++c) {
    if (lo + c < m) {
      const uint32_t v = cnt[lo + c];
      cnt[lo + c] = run;
      run += v;
    }
  }
  const uint32_t total = s_wave[kThreads / 64];
  __syncthreads();
  return total;
}

// ------------------------------------------------------------------ bin
// Dynamic LDS holds first the partition histogram (P + 1 words), then, once
// every entry knows its place, the tile's staging buffers: keys, then the
// entries' values {r, g, b, n} (as float4 when they fit, else in two
// halves), so that every global write of the partition-sorted tile is
// coalesced.  It is declared 16-byte aligned for that: it starts behind the
// static arrays, 68 or 584 bytes of them, and the 8- and 16-byte accesses
// there are undefined below their alignment (and slower: a frame of 3,686,400
// weighted records took 210 us from offset 68 and takes 198 from 80).
//
// Pre-merge: unless the records carry weights, the records of one wave that
// fall in the same cell as the lane before them (neighbouring pixels of a
// scanline usually share a cell at the first bounce) leave a single staged
// entry: the first lane of each such run carries the run's record count and
// value sums (a segmented sum over lanes, in a fixed order), and the other
// records of the run only point at it for the fused query.
//
// kX: what the records carry beyond the common fields, kXFootprint (their
// level rule) and kXWeight (MIS weights: every sample is its own entry with
// value w (r, g, b) and n = w; a weight is read only after the sort, which
// also counts the samples it rejects); separate instantiations keep the
// extra loads and their registers out of the common case.  kXNormal: a table
// with the SH payload, whose sums need every sample's normal: each sample is
// its own entry and its normal, read again after the sort, is staged beside
// the value.
constexpr uint32_t kXFootprint = 1, kXWeight = 2, kXNormal = 4;

__device__ __forceinline__ unsigned long long shfl_up_u64(unsigned long long v, uint32_t d) {
  const uint32_t lo = (uint32_t)__shfl_up((int)(uint32_t)v, d);
  const uint32_t hi = (uint32_t)__shfl_up((int)(uint32_t)(v >> 32), d);
  return ((unsigned long long)hi << 32) | lo;
}

// Records carried by the entry of a run head in lane `lane` (1 + the
// continuation lanes that follow it); cont has bit l set where lane l
// continues lane l - 1's run.
__device__ __forceinline__ uint32_t run_records(unsigned long long cont, uint32_t lane) {
  const unsigned long long after = lane == 63 ? 0ull : cont >> (lane + 1);
  return 1u + (uint32_t)__builtin_ctzll(~after);
}

// Lane of the head of `lane`'s run (the last lane at or before it that does
// not continue its predecessor).
__device__ __forceinline__ uint32_t run_head(unsigned long long cont, uint32_t lane) {
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  return 63u - (uint32_t)__builtin_clzll(~cont & upto);
}

// Threads and records per thread of the binning pass: a tile of 4096 records
// takes 1024 threads with 4 records each (6144: 768 with 8, or 512 with 12
// where records carry more; 8192: 1024 with 8).  The pass waits on one dependent
// step after another (record loads, LDS ranks, scan, staging), so twice the
// wavefronts with half the records each hide more of it: 70.6 -> 62.0 us for
// 3,686,400 records (900 tiles) against 512 threads with 8 (58.5 since), 174 ->
// 163 us for 1688 tiles of 6144 (155 since).  Compiled for the wavefronts per SIMD of two blocks a CU
// (one of 8192 records, by its LDS; twelve weighted records a thread spill at
// 128 registers and run one block a CU at 137).
constexpr int bin_waves(uint32_t threads, uint32_t per, bool weights) {
  return threads * per > 6144 ? 4 : per > 8 && weights ? 3 : (int)threads / 128;
}
template <uint32_t kThreads, uint32_t kPer, uint32_t kX>
__device__ __forceinline__ void bin_body(const RecPtrs& rec, uint64_t n, const KeyParams& kp,
                                         const TableView& tv, const PartView& pv, uint32_t tile) {
  constexpr bool kFp = (kX & kXFootprint) != 0, kW = (kX & kXWeight) != 0, kN = (kX & kXNormal) != 0;
  extern __shared__ __align__(16) uint32_t s_dyn_bin[];
  __shared__ uint32_t s_wave[kThreads / 64 + 1];
  __shared__ unsigned long long s_cont[kThreads / 64][kPer];  // per wave and record row: run continuations
  const uint32_t P = 1u << (tv.log2_slots - tv.part_log2);
  uint32_t* s_hist = s_dyn_bin;
  unsigned long long* s_k = reinterpret_cast<unsigned long long*>(s_dyn_bin);
  const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
  const uint64_t t0 = (uint64_t)tile * (kThreads * kPer);
  // records merge into runs only with integer counters and no weights; a
  // table that keeps the variance also sums each run's squared luminances
  // (in registers, in tiles of up to 4096 records; in larger ones its records
  // stay entries of their own)
  const bool var = tv.var != nullptr;
  constexpr bool kQRuns = kThreads * kPer <= 4096;
  const bool premerge = !kW && !kN && (kQRuns || !var);
  for (uint32_t p = tid; p <= P; p += kThreads) s_hist[p] = 0;
  __syncthreads();

  uint64_t key[kPer];
  // partition << 16 | rank, then the entry's position in the sorted tile
  // (for a merged record: its run head's); ~0 if the record has no entry
  uint32_t pos[kPer];
  float rgb[kPer][3];
  float qs[kQRuns ? kPer : 1];  // squared luminance (variance tables), summed over runs like rgb
  uint32_t n_skip = 0, n_ovf = 0;
  // flags riding in the top bits of a position (partition << 13 | rank, the
  // partition < 2^15 and the rank < 2^13, before the scan; the position in
  // the tile < 2^13 after it): merged into the previous lane's entry;
  // with weights, staged for lookup only and counted as a coordinate overflow
  constexpr uint32_t kPosTail = 1u << 29, kPosLookupOnly = 1u << 31, kPosOverflow = 1u << 30;
  constexpr uint32_t kPosBits = kPosTail - 1;
  const bool hr = rec.rough != nullptr;
  // Every load is unconditional (indices past the end are clamped, absent
  // arrays alias the positions) so that a batch of records is a single
  // memory round trip; validity is applied afterwards.  The records are read
  // once: non-temporal loads keep them from evicting what the merge pass
  // reads next from the caches (the staged entries, the key mirror, the
  // slots).  The tile's first element of each array is a scalar address and
  // a record's offset from it one 32-bit register for every array.
  const uint32_t m = n - t0 < kThreads * kPer ? (uint32_t)(n - t0) : kThreads * kPer;  // the tile's records
  const float* const p_px = rec.px + t0;
  const float* const p_py = rec.py + t0;
  const float* const p_pz = rec.pz + t0;
  const float* const p_nx = rec.nx + t0;
  const float* const p_ny = rec.ny + t0;
  const float* const p_nz = rec.nz + t0;
  const float* const p_ox = (hr ? rec.ox : rec.px) + t0;
  const float* const p_oy = (hr ? rec.oy : rec.px) + t0;
  const float* const p_oz = (hr ? rec.oz : rec.px) + t0;
  const float* const p_ro = (hr ? rec.rough : rec.px) + t0;
  const float* const p_r = rec.r + t0;
  const float* const p_g = rec.g + t0;
  const float* const p_b = rec.b + t0;
  const float* const p_fp = (kFp ? rec.footprint : rec.px) + t0;
  constexpr uint32_t kLoad = kPer < 2 ? 1 : 2;  // records per load round trip
#pragma unroll
  for (uint32_t j0 = 0; j0 < kPer; j0 += kLoad) {
    float f[kLoad][13];
    float fp[kLoad];
#pragma unroll
    for (uint32_t q = 0; q < kLoad; ++q) {
      const uint32_t il = (j0 + q) * kThreads + tid;
      const uint32_t ic = il < m ? il : m - 1;
      f[q][0] = ld_once_at(p_px, ic);
      f[q][1] = ld_once_at(p_py, ic);
      f[q][2] = ld_once_at(p_pz, ic);
      f[q][3] = ld_once_at(p_nx, ic);
      f[q][4] = ld_once_at(p_ny, ic);
      f[q][5] = ld_once_at(p_nz, ic);
      f[q][6] = ld_once_at(p_ox, ic);
      f[q][7] = ld_once_at(p_oy, ic);
      f[q][8] = ld_once_at(p_oz, ic);
      f[q][9] = ld_once_at(p_r, ic);
      f[q][10] = ld_once_at(p_g, ic);
      f[q][11] = ld_once_at(p_b, ic);
      f[q][12] = ld_once_at(p_ro, ic);
      fp[q] = kFp ? ld_once_at(p_fp, ic) : 0.0f;
    }
    // Every loaded value is used here, so the batch's loads all issue
    // before the first wait: left alone, the compiler sinks some of them
    // behind the key function's finiteness tests, each such group a
    // dependent round trip of its own.
#pragma unroll
    for (uint32_t q = 0; q < kLoad; ++q) {
#pragma unroll
      for (uint32_t k = 0; k < 13; ++k) asm volatile("" : : "v"(f[q][k]));
      if (kFp) asm volatile("" : : "v"(fp[q]));
    }
#pragma unroll
    for (uint32_t q = 0; q < kLoad; ++q) {
      const uint32_t j = j0 + q;
      const bool in = j * kThreads + tid < m;
      bool ovf = false;
      uint64_t k = 0;
      const bool kv = in && cell_key(kp, f[q][0], f[q][1], f[q][2], f[q][3], f[q][4], f[q][5], f[q][6],
                                        f[q][7], f[q][8], hr, f[q][12], kFp, fp[q], k, ovf);
      const bool sv = finite3(f[q][9], f[q][10], f[q][11]);
      key[j] = (kv && sv) ? k : k | kLookupOnlyBit;
      rgb[j][0] = f[q][9];
      rgb[j][1] = f[q][10];
      rgb[j][2] = f[q][11];
      if (in && !(kv && sv)) ++n_skip;
      n_ovf += (kv && sv && ovf) ? 1u : 0u;
      // a record whose sample is rejected but whose key is valid is still a
      // query vertex: with the fused query it is staged for lookup only
      const bool entry = kv && (sv || pv.perm);
      pos[j] = entry ? ((kv && sv) ? 0u : kPosLookupOnly) | ((ovf && sv) ? kPosOverflow : 0u) : ~0u;
    }
    // (the next batch's loads stay behind this one's keys: hoisted, they
    // spill)
    __builtin_amdgcn_sched_barrier(0);
  }
  // entries per partition (ranks), after merging runs of one cell in
  // neighbouring lanes: only a run's head gets an entry
#pragma unroll
  for (uint32_t j = 0; j < kPer; ++j) {
    const bool smp = pos[j] != ~0u && !(pos[j] & kPosLookupOnly);
    bool tail = false;
    if (kQRuns) {
      qs[kQRuns ? j : 0] = 0.0f;
      if (var) {
        const float y = luma32(rgb[j][0], rgb[j][1], rgb[j][2]);
        qs[kQRuns ? j : 0] = y * y;
      }
    }
    if (premerge) {
      // a sample whose key equals the previous lane's (also a sample)
      // continues that lane's run
      const unsigned long long kprev = shfl_up_u64(key[j], 1);
      const bool sprev = __shfl_up((int)smp, 1) != 0;
      tail = lane > 0 && smp && sprev && key[j] == kprev;
      const unsigned long long cont = __ballot(tail);
      if (lane == 0) s_cont[wave][j] = cont;
      if (cont) {
        // segmented suffix sums: after the step of offset d a lane holds
        // the sum over itself and the next 2d - 1 lanes of its run, so each
        // head ends with its run's total (fixed order: reproducible)
        unsigned long long live = cont;  // lanes ending runs of >= 2d
        for (uint32_t d = 1; live; d <<= 1) {
          const float vr = __shfl_down(rgb[j][0], d);
          const float vg = __shfl_down(rgb[j][1], d);
          const float vb = __shfl_down(rgb[j][2], d);
          const float vq = (kQRuns && var) ? __shfl_down(qs[kQRuns ? j : 0], d) : 0.0f;
          const bool same = lane + d < 64 &&
                            ((cont >> (lane + 1)) & ((1ull << d) - 1ull)) == ((1ull << d) - 1ull);
          if (same) {
            rgb[j][0] += vr;
            rgb[j][1] += vg;
            rgb[j][2] += vb;
            if (kQRuns) qs[kQRuns ? j : 0] += vq;
          }
          live &= live >> d;
        }
      }
    }
    if (pos[j] == ~0u) continue;
    if (tail) {
      pos[j] = kPosTail;
      continue;
    }
    const uint32_t p = partition_of(fmix64(key[j] & ~kLookupOnlyBit), tv.log2_slots, tv.part_log2);
    const uint32_t rank = atomicAdd(&s_hist[p], 1u);
    pos[j] |= (p << 13) | rank;
  }
  // rare-event counters: one atomic per wave when non-zero (with weights,
  // after the staging pass has judged them)
  auto count_events = [&]() {
    for (int off = 32; off > 0; off >>= 1) {
      n_skip += __shfl_xor(n_skip, off);
      n_ovf += __shfl_xor(n_ovf, off);
    }
    if (__lane_id() == 0) {
      if (n_skip) atomicAdd(stat_lane(tv.stats->skipped, tile), (unsigned long long)n_skip);
      if (n_ovf) atomicAdd(stat_lane(tv.stats->coord_overflow, tile), (unsigned long long)n_ovf);
    }
  };
  if (!kW) count_events();
  __syncthreads();
  const uint32_t count = block_exclusive_scan<kThreads>(s_hist, P + 1, s_wave);

  uint32_t* offs = pv.runs + (uint64_t)tile * (P + 1);
  for (uint32_t p = tid; p <= P; p += kThreads) offs[p] = s_hist[p];
#pragma unroll
  for (uint32_t j = 0; j < kPer; ++j) {
    if (pos[j] != ~0u && !(pos[j] & kPosTail)) {
      const uint32_t q = pos[j] & ((1u << 29) - 1u);
      pos[j] = (s_hist[q >> 13] + (q & 0x1fffu)) | (pos[j] & ~((1u << 29) - 1u));
    }
    if (premerge && pv.perm) {
      // a merged record is answered from its run head's entry
      const unsigned long long cont = s_cont[wave][j];
      if (cont) {
        const uint32_t hp = (uint32_t)__shfl((int)pos[j], (int)run_head(cont, lane));
        if (pos[j] == kPosTail) pos[j] = (hp & kPosBits) | kPosTail;
      }
    }
  }
  if (pv.perm) {
    uint16_t* const perm = pv.perm + t0;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      const uint32_t i = j * kThreads + tid;
      if (i < m) perm[i] = pos[j] != ~0u ? (uint16_t)(pos[j] & kPosBits) : kNoPos;
    }
  }
  __syncthreads();  // the histogram is dead from here on; its LDS becomes staging

  auto own_entry = [&](uint32_t j) { return pos[j] != ~0u && !(pos[j] & kPosTail); };
  // n of each entry: the records it carries (with weights: the record's
  // weight); 0 marks an entry staged for lookup only
  auto entry_n = [&](uint32_t j) {
    uint32_t c = 1;
    if (premerge) {
      const unsigned long long cont = s_cont[wave][j];
      if (cont) c = run_records(cont, lane);
    }
    return (pos[j] & kPosLookupOnly) ? 0u : c;
  };
  if (var) {
    // each entry's squared-luminance sum, at its staged position (a record
    // of its own: its value's)
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      if (!own_entry(j)) continue;
      float q;
      if (kQRuns) {
        q = qs[kQRuns ? j : 0];
      } else {
        const float y = luma32(rgb[j][0], rgb[j][1], rgb[j][2]);
        q = y * y;
      }
      pv.stage_q[t0 + (pos[j] & kPosBits)] = q;
    }
  }
  if (kN) {
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      if (!own_entry(j)) continue;
      const uint64_t i = t0 + (uint64_t)j * kThreads + tid;
      pv.stage_n[t0 + (pos[j] & kPosBits)] = make_float4(rec.nx[i], rec.ny[i], rec.nz[i], 0.0f);
    }
  }
  float wn[kW ? kPer : 1];
  if (kW) {
    // The weights are first read here.  A sample whose weight is not finite
    // and > 0 is rejected: counted as skipped (not as a coordinate
    // overflow) and staged for lookup only, so the merge pass only looks it
    // up (with the fused query) or ignores it; an accepted one is staged as
    // w (r, g, b) with n = w.
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      wn[j] = 0.0f;
      if (!own_entry(j)) continue;
      const float w = rec.weight[t0 + (uint64_t)j * kThreads + tid];
      if (key[j] & kLookupOnlyBit) continue;
      if (__builtin_isfinite(w) && w > 0.0f) {
        if (!kN) {  // (the SH sums weight the sample themselves, in binary64)
          rgb[j][0] *= w;
          rgb[j][1] *= w;
          rgb[j][2] *= w;
        }
        wn[j] = w;
      } else {
        key[j] |= kLookupOnlyBit;
        ++n_skip;
        n_ovf -= (pos[j] & kPosOverflow) ? 1u : 0u;
      }
    }
    count_events();
  }
#pragma unroll
  for (uint32_t j = 0; j < kPer; ++j)
    if (own_entry(j)) s_k[pos[j] & kPosBits] = key[j];
  __syncthreads();
  for (uint32_t i = tid; i < count; i += kThreads) pv.stage_key[t0 + i] = s_k[i];
  __syncthreads();
  // the entries' values {r, g, b, n}: as float4 when they fit in the LDS,
  // else in two halves, (r, g) then (b, n)
  auto entry_w = [&](uint32_t j) { return kW ? wn[kW ? j : 0] : (float)entry_n(j); };
  const size_t lds_bytes = (size_t)kThreads * kPer * bin_lds_per_record(kThreads * kPer);  // the launch's dynamic LDS
  if ((size_t)count * 16 <= lds_bytes) {
    float4* s_v = reinterpret_cast<float4*>(s_dyn_bin);
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j)
      if (own_entry(j)) s_v[pos[j] & kPosBits] = make_float4(rgb[j][0], rgb[j][1], rgb[j][2], entry_w(j));
    __syncthreads();
    for (uint32_t i = tid; i < count; i += kThreads) pv.stage_v[t0 + i] = s_v[i];
  } else {
    float2* s_v = reinterpret_cast<float2*>(s_dyn_bin);
    float2* dst = reinterpret_cast<float2*>(pv.stage_v + t0);
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j)
      if (own_entry(j)) s_v[pos[j] & kPosBits] = make_float2(rgb[j][0], rgb[j][1]);
    __syncthreads();
    for (uint32_t i = tid; i < count; i += kThreads) dst[2 * i] = s_v[i];
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j)
      if (own_entry(j)) s_v[pos[j] & kPosBits] = make_float2(rgb[j][2], entry_w(j));
    __syncthreads();
    for (uint32_t i = tid; i < count; i += kThreads) dst[2 * i + 1] = s_v[i];
  }
}

template <uint32_t kThreads, uint32_t kPer, uint32_t kX>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(bin_waves(kThreads, kPer, kX & kXWeight))))
k_bin(RecPtrs rec, uint64_t n, KeyParams kp, TableView tv, PartView pv) {
  bin_body<kThreads, kPer, kX>(rec, n, kp, tv, pv, blockIdx.x);
}

// ------------------------------------------------------------------ run table transpose
// The merge block of partition p needs the offsets of p and p + 1 in every
// tile: a column of the bin pass's [tile][P + 1] table.  A 64 x 64 LDS
// transpose turns the columns into rows, so the merge reads them coalesced.
constexpr uint32_t kTransposeDim = 64, kTransposeThreads = 256;

__device__ __forceinline__ void transpose_body(const PartView& pv, uint32_t P, uint32_t ntiles, uint32_t bx,
                                               uint32_t by) {
  __shared__ uint32_t s_t[kTransposeDim][kTransposeDim + 1];
  const uint32_t tid = threadIdx.x, c = tid % kTransposeDim, r0 = tid / kTransposeDim;
  constexpr uint32_t kRowsPerPass = kTransposeThreads / kTransposeDim;
  const uint32_t t0 = bx * kTransposeDim, p0 = by * kTransposeDim;
  const uint32_t stride = (pv.max_tiles + 3u) & ~3u;
  for (uint32_t r = r0; r < kTransposeDim; r += kRowsPerPass) {
    const uint32_t t = t0 + r, p = p0 + c;
    if (t < ntiles && p <= P) s_t[r][c] = pv.runs[(uint64_t)t * (P + 1) + p];
  }
  __syncthreads();
  for (uint32_t r = r0; r < kTransposeDim; r += kRowsPerPass) {
    const uint32_t p = p0 + r, t = t0 + c;
    if (t < ntiles && p <= P) pv.runs_t[(uint64_t)p * stride + t] = s_t[c][r];
  }
}

__global__ void __launch_bounds__(kTransposeThreads) k_transpose_runs(PartView pv, uint32_t P, uint32_t ntiles) {
  transpose_body(pv, P, ntiles, blockIdx.x, blockIdx.y);
}

// ------------------------------------------------------------------ merge
// LDS of a merge block: the partition's keys and, per slot, its place in the
// list of touched slots (16-bit; 10 bytes a slot), then sums for `cells`
// touched cells (30 bytes each: three binary64 sums, a count and the slot's
// number; 38 with a further sum per cell).  A frame touches about one slot in
// eight, so sums for 5/16 of the slots (1/4 with the further sum) do in one
// round, in half the LDS that sums for every slot would take: a CU holds 24
// wavefronts (two blocks of 4096 slots, four of 2048, eight of 1024) instead
// of 16, in separate blocks that are not all in the same phase.  3,686,400
// records into 2^22 slots: 98 -> 82 us (75 since); 10,368,000 into 2^24: 336 ->
// 278 us (266 with the answers of its 16-bit state staged in half the bytes).
// (32 wavefronts need 64 registers and spill 37 more: 176 us.)  A partition
// with more touched cells takes further rounds over its entries, each of them
// as long as the first; dense_launch tells the launches that would.
__host__ __device__ constexpr uint32_t merge_cells(uint32_t slots, bool extra) {
  return extra ? slots / 4 : slots / 16 * 5;
}
// Dense launches (many records a slot) keep sums for every slot instead: an
// entry is then added as soon as its slot is found, its key and value read
// once, and no partition needs a second round (38 bytes a slot, 46 with the
// further sum; 16 wavefronts a CU).
__host__ __device__ constexpr size_t merge_lds_bytes(uint32_t slots, bool extra, bool dense) {
  if (dense) return (size_t)slots * (8 + 24 + 4 + 2 + (extra ? 8 : 0));
  return (size_t)slots * (8 + 2) + (size_t)merge_cells(slots, extra) * (24 + 4 + 2 + (extra ? 8 : 0));
}

// Entries per lane of a wave's first batch, held in registers to the end, and
// of the batches after it, which each step reads again.
constexpr uint32_t kEntryBatch = 4, kLaterBatch = 2;

// What became of an entry's key: a slot number (with the probes it took, at
// most 15, from kProbesShift on), a key that found no slot, or an entry
// staged for lookup only.
constexpr uint32_t kProbesShift = 16, kSlotBits = 0xffffu;
constexpr uint32_t kDropped = 0xffffffffu, kLookupLater = 0xfffffffeu, kAbsent = 0xfffffffdu;

// One partition: blk is the block's index among the partition blocks of this
// table (the XCD-aware order maps it to a partition).  With results (fused
// mode only), every staged entry of the partition is overwritten with the
// value its cell holds after the blend (kDroppedBits in place of red, or
// kDropped16, when its key found no slot).
template <bool kFused, int kThreads, bool kVar, bool kDense>
__device__ __forceinline__ void merge_body(const TableView& tv, const PartView& pv, uint32_t ntiles,
                                           const BlendParams& bp, uint32_t blk, bool results) {
  // key[B] | sum[3][N] (binary64: LDS f64 atomics are both faster than f32
  // ones on gfx950 and exact enough to make the sum order immaterial), then,
  // in a table that keeps the luminance variance or has weighted counters,
  // sumx[N]: the squared luminances (staged per entry), or the weights
  // (binary64 like the value sums, rounded once to binary32 at the
  // write-back, so the counters do not depend on the order of the atomics;
  // cnt is then unused; every entry is one record) | cnt[N] | place of a
  // slot in the list of touched slots[B] (16-bit) | the round's part of that
  // list[N] (16-bit).  After the blend the sums hold the cells' new values.
  // (kDense: N = B, the sums are indexed by slot, a slot with a count is
  // touched, in a weighted table too, and there are no places, only the list.)
  extern __shared__ unsigned long long s_dyn[];
  __shared__ uint32_t s_dropped, s_nlist, s_sat;
  __shared__ uint32_t s_hist[16];
  const uint32_t tid = threadIdx.x, lane = __lane_id();
  constexpr uint32_t kWaves = kThreads / 64;
  const uint32_t P = 1u << (tv.log2_slots - tv.part_log2);
  const uint32_t B = 1u << tv.part_log2;
  const uint32_t p = xcd_partition(blk, P);
  const uint64_t base = (uint64_t)p << tv.part_log2;
  const bool stats = (tv.flags & 1u) != 0;
  const bool wtd = weighted(tv);
  const uint32_t N = kDense ? B : merge_cells(B, kVar || wtd);
  unsigned long long* s_key = s_dyn;
  double* s_sum0 = reinterpret_cast<double*>(s_key + B);
  double* s_sum1 = s_sum0 + N;
  double* s_sum2 = s_sum1 + N;
  double* s_sumx = s_sum2 + N;  // only with tv.var or wtd
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_sumx + ((kVar || wtd) ? N : 0u));
  uint16_t* s_idx = reinterpret_cast<uint16_t*>(s_cnt + N);  // not kDense
  uint16_t* s_list = kDense ? s_idx : s_idx + B;
  constexpr uint32_t kNone = 0xffffu;
  if (!kFused) results = false;

  // keys first, then the first runs, then the keys of the wave's first batch
  // of entries: all in flight together, before the key table is built
  const RunReader<kWaves> rr(pv, p, P, ntiles);
  constexpr uint32_t kKeysPerThread = kDense ? 4 : 6;  // (the launch has at least B / 4 or B / 6 threads)
  unsigned long long kk[kKeysPerThread];
#pragma unroll
  for (uint32_t j = 0; j < kKeysPerThread; ++j) {
    const uint32_t s = tid + j * kThreads;
    kk[j] = s < B ? tv.keys[base + s] : kEmpty;
  }
  RunChunk ch0{};
  uint32_t at0[kEntryBatch], code0[kEntryBatch];
  unsigned long long ek0[kEntryBatch];
  bool ev0[kEntryBatch];
  float4 v0[kEntryBatch];
  float q0[kEntryBatch];  // variance tables: the entries' squared-luminance sums
  auto load_values = [&]() {
#pragma unroll
    for (uint32_t q = 0; q < kEntryBatch; ++q) {
      v0[q] = pv.stage_v[at0[q]];
      q0[q] = kVar ? pv.stage_q[at0[q]] : 0.0f;
    }
  };
#pragma unroll
  for (uint32_t q = 0; q < kEntryBatch; ++q) ev0[q] = false;
  const bool any = rr.w_lo < rr.w_hi;  // the wave has tiles (wave-uniform)
  if (any) {
    ch0 = rr.chunk_of(rr.w_lo);
    rr.template batch_of<kEntryBatch>(ch0, 0, at0, ev0);
#pragma unroll
    for (uint32_t q = 0; q < kEntryBatch; ++q) ek0[q] = pv.stage_key[at0[q]];
    if (kDense) load_values();
  }
  auto clear_sums = [&]() {
    for (uint32_t c = tid; c < N; c += kThreads) {
      s_sum0[c] = s_sum1[c] = s_sum2[c] = 0.0;
      if (kVar || wtd) s_sumx[c] = 0.0;
      s_cnt[c] = 0;
    }
  };
  clear_sums();
#pragma unroll
  for (uint32_t j = 0; j < kKeysPerThread; ++j) {
    const uint32_t s = tid + j * kThreads;
    if (s < B) {
      s_key[s] = kk[j];
      if (!kDense) s_idx[s] = (uint16_t)kNone;
    }
  }
  if (tid == 0) s_dropped = s_nlist = s_sat = 0;
  if (tid < 16) s_hist[tid] = 0;
  __syncthreads();

  // Finds the slot of a sample's key, or claims one, and marks it touched.
  auto claim = [&](unsigned long long key) {
    const uint32_t start = (uint32_t)fmix64(key) & (B - 1);
    for (uint32_t i = 0; i < tv.max_probe; ++i) {
      const uint32_t s = (start + i) & (B - 1);
      unsigned long long cur = s_key[s];
      if (cur == kEmpty) cur = atomicCAS(&s_key[s], kEmpty, key);
      if (cur == kEmpty || cur == key) {
        if (!kDense) s_idx[s] = 0;
        return s | ((i < 15 ? i : 15u) << kProbesShift);
      }
    }
    return kDropped;
  };
  // The same once every key has its slot (also of a lookup-only entry).
  auto find = [&](unsigned long long key) {
    const uint32_t start = (uint32_t)fmix64(key) & (B - 1);
    for (uint32_t i = 0; i < tv.max_probe; ++i) {
      const uint32_t s = (start + i) & (B - 1);
      const unsigned long long cur = s_key[s];
      if (cur == key) return s | ((i < 15 ? i : 15u) << kProbesShift);
      if (cur == kEmpty) break;
    }
    return kDropped;
  };
#pragma unroll
  for (uint32_t q = 0; q < kEntryBatch; ++q)
    code0[q] = !ev0[q] ? kAbsent : (ek0[q] & kLookupOnlyBit) ? kLookupLater : claim(ek0[q]);

  // Adds an entry to its cell's sums if the cell is in the round from c0 on.
  auto add = [&](uint32_t code, const float4& v, float qv, uint32_t c0) {
    const uint32_t recs = pv.weights ? 1u : (uint32_t)v.w;  // records behind the entry
    if (code == kDropped) {
      if (c0 == 0) atomicAdd(&s_dropped, recs);
      return;
    }
    const uint32_t c = kDense ? code & kSlotBits : (uint32_t)s_idx[code & kSlotBits] - c0;
    if (c >= N) return;
    if (stats) atomicAdd(&s_hist[code >> kProbesShift], recs);
    if (wtd) {
      atomicAdd(&s_sumx[c], (double)v.w);
      if (kDense) s_cnt[c] = 1u;
    } else {
      atomicAdd(&s_cnt[c], (uint32_t)v.w);
    }
    atomicAdd(&s_sum0[c], (double)v.x);
    atomicAdd(&s_sum1[c], (double)v.y);
    atomicAdd(&s_sum2[c], (double)v.z);
    if (kVar) atomicAdd(&s_sumx[c], (double)qv);
  };
  // What the table holds of a touched slot before this launch.
  struct Old {
    Slot slot;
    Acc acc;    // not fused
    float v;    // fused: the variance
    double q;   // not fused: the pending squared-luminance sum
  };
  auto load_old = [&](uint64_t g) {
    Old o;
    o.slot = tv.slots[g];
    if (!kFused) o.acc = tv.acc[g];
    if (kVar) {
      if (kFused)
        o.v = tv.var[g];
      else
        o.q = tv.acc_q[g];
    }
    return o;
  };
  uint32_t n_sat = 0;  // cells of this thread whose 16-bit store was clamped
  // Writes touched cell c of the round back (slot s of the partition).
  auto write_back = [&](uint32_t c, uint32_t s, const Old& old) {
    const uint64_t g = base + s;
    // the frame's counter word (a weighted table's weight sum rounds once)
    const uint32_t cn = wtd ? __float_as_uint((float)s_sumx[c]) : s_cnt[c];
    const unsigned long long k = s_key[s];
    if (kFused) {
      const float alpha = blend_alpha(bp, cn, old.slot.c_old, wtd);
      float L[3];
      load_blend_state(old.slot, bp.dtype, L[0], L[1], L[2]);
      // the new sample mean, rounded once from binary64
      const double cd = wtd ? (double)__uint_as_float(cn) : (double)cn;
      const float means[3] = {(float)(s_sum0[c] / cd), (float)(s_sum1[c] / cd), (float)(s_sum2[c] / cd)};
      float out[3];
      for (int ch = 0; ch < 3; ++ch) {
        const float m = means[ch];
        out[ch] = alpha == 1.0f ? m : (1.0f - alpha) * L[ch] + alpha * m;
      }
      if (kVar) {
        double m, s2;
        frame_moments(s_sum0[c], s_sum1[c], s_sum2[c], s_sumx[c], cd, m, s2);
        tv.var[g] = blend_variance(old.v, alpha, luma32(L[0], L[1], L[2]), m, s2);
      }
      uint32_t enc[4], pad;
      bool sat = false;
      encode_state(bp.dtype, out[0], out[1], out[2], enc, pad, sat);
      n_sat += sat ? 1u : 0u;
      Slot nw;
      nw.key = k;
      nw.c_old = counter_add(old.slot.c_old, cn, wtd);
      nw.pad = pad;
      nw.L[0] = enc[0];
      nw.L[1] = enc[1];
      nw.L[2] = enc[2];
      nw.L[3] = enc[3];
      tv.slots[g] = nw;
      if (old.slot.key != k) tv.keys[g] = k;
      if (results) {
        // what a lookup of the cell returns from now on
        if (bp.dtype == 0) {
          s_sum0[c] = out[0];
          s_sum1[c] = out[1];
          s_sum2[c] = out[2];
        } else {
          reinterpret_cast<unsigned long long*>(s_sum0)[c] = ((unsigned long long)enc[1] << 32) | enc[0];
        }
      }
    } else {
      Acc a = old.acc;
      a.n = counter_add(a.n, cn, wtd);
      a.s[0] += (float)s_sum0[c];
      a.s[1] += (float)s_sum1[c];
      a.s[2] += (float)s_sum2[c];
      tv.acc[g] = a;
      if (kVar) tv.acc_q[g] = old.q + s_sumx[c];
      if (old.slot.key != k) {
        tv.slots[g].key = k;
        tv.keys[g] = k;
      }
    }
  };
  // Stages the answer of the entry at `at`, the value a lookup of its cell
  // returns: binary32 values over the entry's values, 16-bit ones over its
  // key.  From the round's sums if in_lds (a partition of one round), else
  // from the table.
  auto answer = [&](uint32_t at, uint32_t code, bool in_lds) {
    if (code == kLookupLater) code = find(pv.stage_key[at] & ~kLookupOnlyBit);
    const uint32_t s = code & kSlotBits;
    const uint32_t i = code == kDropped || !in_lds ? kNone : !kDense ? (uint32_t)s_idx[s] : s_cnt[s] ? s : kNone;
    Slot sl;
    sl.c_old = 0;
    // (with in_lds, only a lookup-only entry whose cell this launch did not
    // touch)
    if (code != kDropped && i == kNone) sl = tv.slots[base + s];
    if (bp.dtype == 0) {
      float v[3] = {__uint_as_float(kDroppedBits), 0.0f, 0.0f};
      if (i != kNone) {
        v[0] = (float)s_sum0[i];
        v[1] = (float)s_sum1[i];
        v[2] = (float)s_sum2[i];
      } else if (sl.c_old > 0) {
        load_state(sl, 0, v[0], v[1], v[2]);
      }
      pv.stage_v[at] = make_float4(v[0], v[1], v[2], 0.0f);
    } else {
      unsigned long long w = kDropped16;
      if (i != kNone)
        w = reinterpret_cast<const unsigned long long*>(s_sum0)[i];
      else if (sl.c_old > 0)
        w = ((unsigned long long)sl.L[1] << 32) | sl.L[0];
      pv.stage_key[at] = w;
    }
  };
  // Counters of the partition, once every thread is done with it.
  auto finish = [&](uint32_t n_touched) {
    if (kFused && n_sat) atomicAdd(&s_sat, n_sat);
    __syncthreads();
    if (tid == 0) {
      if (s_dropped) atomicAdd(&tv.stats->dropped, (unsigned long long)s_dropped);
      if (kFused) {
        if (s_sat) atomicAdd(&tv.stats->saturated, (unsigned long long)s_sat);
        BlockTouch* bt = &tv.touch[blk];
        bt->last = n_touched;
        bt->total += n_touched;
      }
    }
    if (stats && tid < 16 && s_hist[tid])
      atomicAdd(&tv.stats->probe_hist[tid], (unsigned long long)s_hist[tid]);
  };
  if constexpr (kDense) {
    // one sweep: every entry is added as it is read; the places of a wave's
    // second batch are kept beside those of its first for the answers
    uint32_t at1[kEntryBatch], code1[kEntryBatch];
#pragma unroll
    for (uint32_t q = 0; q < kEntryBatch; ++q) {
      if (code0[q] != kAbsent && code0[q] != kLookupLater) add(code0[q], v0[q], q0[q], 0);
      code1[q] = kAbsent;
    }
    uint32_t nb = 0;
    rr.template for_each_batch<kEntryBatch>(ch0, 64 * kEntryBatch, [&](const uint32_t* at, const bool* ev) {
      unsigned long long ek[kEntryBatch];
      float4 v[kEntryBatch];
      float qv[kEntryBatch];
#pragma unroll
      for (uint32_t q = 0; q < kEntryBatch; ++q) {
        ek[q] = pv.stage_key[at[q]];
        v[q] = pv.stage_v[at[q]];
        qv[q] = kVar ? pv.stage_q[at[q]] : 0.0f;
      }
#pragma unroll
      for (uint32_t q = 0; q < kEntryBatch; ++q) {
        const uint32_t code = !ev[q] ? kAbsent : (ek[q] & kLookupOnlyBit) ? kLookupLater : claim(ek[q]);
        if (code != kAbsent && code != kLookupLater) add(code, v[q], qv[q], 0);
        if (nb == 0) {
          at1[q] = at[q];
          code1[q] = code;
        }
      }
      ++nb;
    });
    __syncthreads();
    for (uint32_t s0 = 0; s0 < B; s0 += kThreads) {
      const uint32_t s = s0 + tid;
      const bool hit = s < B && s_cnt[s] != 0u;
      const unsigned long long m = __ballot(hit);
      uint32_t at = 0;
      if (lane == 0 && m) at = atomicAdd(&s_nlist, (uint32_t)__popcll(m));
      at = (uint32_t)__shfl((int)at, 0);
      if (hit)
        s_list[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
            (uint16_t)s;
    }
    __syncthreads();
    // two cells a thread at a time, their old slots in one round trip
    const uint32_t n_touched = s_nlist;
    for (uint32_t i = tid; i < n_touched; i += 2 * kThreads) {
      const bool two = i + kThreads < n_touched;
      const uint32_t sa = s_list[i], sb = s_list[two ? i + kThreads : i];
      const Old oa = load_old(base + sa), ob = load_old(base + sb);
      write_back(sa, sa, oa);
      if (two) write_back(sb, sb, ob);
    }
    if (results) {
      __syncthreads();
#pragma unroll
      for (uint32_t q = 0; q < kEntryBatch; ++q) {
        if (code0[q] != kAbsent) answer(at0[q], code0[q], true);
        if (code1[q] != kAbsent) answer(at1[q], code1[q], true);
      }
      nb = 0;
      rr.template for_each_batch<kEntryBatch>(ch0, 64 * kEntryBatch, [&](const uint32_t* at, const bool* ev) {
        if (nb++ == 0) return;
        unsigned long long ek[kEntryBatch];
#pragma unroll
        for (uint32_t q = 0; q < kEntryBatch; ++q) ek[q] = pv.stage_key[at[q]];
#pragma unroll
        for (uint32_t q = 0; q < kEntryBatch; ++q)
          if (ev[q]) answer(at[q], find(ek[q] & ~kLookupOnlyBit), true);
      });
    }
    finish(n_touched);
    return;
  }
  // the first batch's values arrive while the touched slots are listed
  if (any) load_values();
  rr.template for_each_batch<kLaterBatch>(ch0, 64 * kEntryBatch, [&](const uint32_t* at, const bool* ev) {
    unsigned long long ek[kLaterBatch];
#pragma unroll
    for (uint32_t q = 0; q < kLaterBatch; ++q) ek[q] = pv.stage_key[at[q]];
#pragma unroll
    for (uint32_t q = 0; q < kLaterBatch; ++q)
      if (ev[q] && !(ek[q] & kLookupOnlyBit)) claim(ek[q]);
  });
  __syncthreads();

  // List the touched slots (about one in eight, scattered), so that the sums
  // are kept for them alone and the write-back runs on full waves.
  for (uint32_t s0 = 0; s0 < B; s0 += kThreads) {
    const uint32_t s = s0 + tid;
    const bool hit = s < B && s_idx[s] != kNone;
    const unsigned long long m = __ballot(hit);
    uint32_t at = 0;
    if (lane == 0 && m) at = atomicAdd(&s_nlist, (uint32_t)__popcll(m));
    at = (uint32_t)__shfl((int)at, 0);
    if (hit) {
      at += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      s_idx[s] = (uint16_t)at;
      if (at < N) s_list[at] = (uint16_t)s;
    }
  }
  __syncthreads();
  const uint32_t n_touched = s_nlist;
  auto add_batch = [&](const uint32_t* at, const bool* ev, uint32_t c0) {
    unsigned long long ek[kLaterBatch];
    float4 v[kLaterBatch];
    float qv[kLaterBatch];
#pragma unroll
    for (uint32_t q = 0; q < kLaterBatch; ++q) {
      ek[q] = pv.stage_key[at[q]];
      v[q] = pv.stage_v[at[q]];
      qv[q] = kVar ? pv.stage_q[at[q]] : 0.0f;
    }
#pragma unroll
    for (uint32_t q = 0; q < kLaterBatch; ++q)
      if (ev[q] && !(ek[q] & kLookupOnlyBit)) add(find(ek[q]), v[q], qv[q], c0);
  };
  auto answer_batch = [&](const uint32_t* at, const bool* ev, bool in_lds) {
    unsigned long long ek[kLaterBatch];
#pragma unroll
    for (uint32_t q = 0; q < kLaterBatch; ++q) ek[q] = pv.stage_key[at[q]];
#pragma unroll
    for (uint32_t q = 0; q < kLaterBatch; ++q)
      if (ev[q]) answer(at[q], find(ek[q] & ~kLookupOnlyBit), in_lds);
  };

  // The first round (the only one unless the partition is dense), with the
  // first batch in registers and the thread's first cell's old slot on its
  // way while the entries are summed.
  const uint32_t cells0 = n_touched < N ? n_touched : N;
  const uint32_t sl0 = tid < cells0 ? (uint32_t)s_list[tid] : 0u;
  const Old old0 = load_old(base + sl0);
#pragma unroll
  for (uint32_t q = 0; q < kEntryBatch; ++q)
    if (code0[q] != kAbsent && code0[q] != kLookupLater) add(code0[q], v0[q], q0[q], 0);
  rr.template for_each_batch<kLaterBatch>(ch0, 64 * kEntryBatch,
                                          [&](const uint32_t* at, const bool* ev) { add_batch(at, ev, 0); });
  __syncthreads();
  if (tid < cells0) write_back(tid, sl0, old0);
  for (uint32_t c = tid + kThreads; c < cells0; c += kThreads) write_back(c, s_list[c], load_old(base + s_list[c]));
  if (results && n_touched <= N) {
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kEntryBatch; ++q)
      if (code0[q] != kAbsent) answer(at0[q], code0[q], true);
    rr.template for_each_batch<kLaterBatch>(ch0, 64 * kEntryBatch,
                                            [&](const uint32_t* at, const bool* ev) { answer_batch(at, ev, true); });
  }
  // Further rounds read the entries again; they are answered at the end, from
  // the cells as written back.
  for (uint32_t c0 = N; c0 < n_touched; c0 += N) {
    __syncthreads();
    clear_sums();
    for (uint32_t s = tid; s < B; s += kThreads) {
      const uint32_t i = (uint32_t)s_idx[s] - c0;
      if (s_idx[s] != kNone && i < N) s_list[i] = (uint16_t)s;
    }
    __syncthreads();
    rr.template for_each_batch<kLaterBatch>(ch0, 0,
                                            [&](const uint32_t* at, const bool* ev) { add_batch(at, ev, c0); });
    __syncthreads();
    const uint32_t cells = n_touched - c0 < N ? n_touched - c0 : N;
    for (uint32_t c = tid; c < cells; c += kThreads) write_back(c, s_list[c], load_old(base + s_list[c]));
  }
  if (results && n_touched > N) {
    __syncthreads();
    rr.template for_each_batch<kLaterBatch>(ch0, 0,
                                            [&](const uint32_t* at, const bool* ev) { answer_batch(at, ev, false); });
  }

  finish(n_touched);
}

// Threads of a merge block (768 for 4096 slots): the LDS of merge_lds_bytes
// leaves room for 24 such wavefronts on a CU, at 80 registers (a table that
// keeps the variance holds one more value an entry, and 96 registers leave 20:
// one block of 768 threads, three of 384).
static uint32_t merge_threads(uint32_t part_log2) { return part_log2 >= 12 ? 768u : part_log2 == 11 ? 384u : 192u; }

// The same for a launch of P partitions that does not fill 256 CUs: twice or
// four times the threads, as far as they fit (256 partitions of 2048 slots with
// the variance: 20.3 us with 384 threads, 16.7 with 768).
static uint32_t merge_threads(uint32_t part_log2, uint32_t P) {
  uint32_t t = merge_threads(part_log2);
  while (t < 768 && (uint64_t)P * t * 2 <= 256ull * 24 * 64) t *= 2;
  return t;
}

// Threads of a dense launch's block: 1024 where its LDS leaves no room for a
// second block on a CU (160 KB), else 512: 16 wavefronts a CU either way.
static uint32_t merge_threads_dense(size_t lds) { return lds > 80 * 1024 ? 1024u : 512u; }

constexpr int merge_waves(bool var, bool dense) { return dense ? 4 : var ? 5 : 6; }

template <bool kFused, int kThreads, bool kVar, bool kDense>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(merge_waves(kVar, kDense))))
k_merge(TableView tv, PartView pv, uint32_t ntiles, BlendParams bp, int32_t results) {
  merge_body<kFused, kThreads, kVar, kDense>(tv, pv, ntiles, bp, blockIdx.x, results != 0);
}

// ------------------------------------------------------------------ unstage
// The fused query: tile t's records take the values the merge pass left in
// the tile's staged entries (their positions in pv.perm).  The tile's staged
// values are read into LDS with 16-byte loads, then every thread answers
// four consecutive records at a time (8-byte perm loads, 16-byte stores when
// the output rows are 16-byte aligned; non-temporal, since no kernel of the
// iteration reads the answers again).
constexpr uint32_t kUnstageThreads = 1024;
static uint32_t unstage_threads(uint32_t tile) { return tile <= 4096 ? tile / 4 : tile == 6144 ? 768 : 1024; }

__device__ __forceinline__ void unstage_one(const float* s_res, uint32_t count, uint32_t pos, float& r,
                                            float& g, float& b, uint8_t& f) {
  r = g = b = 0.0f;
  f = 0;
  if (pos == kNoPos || pos >= count) return;
  const float x = s_res[3 * pos];
  if (__float_as_uint(x) == kDroppedBits) return;
  r = x;
  g = s_res[3 * pos + 1];
  b = s_res[3 * pos + 2];
  f = 1;
}

__device__ __forceinline__ void unstage_body(const PartView& pv, uint32_t P, uint64_t n, uint32_t t,
                                             float* out, uint8_t* found) {
  extern __shared__ float s_res[];  // tile * 3
  const uint32_t tid = threadIdx.x, nt = blockDim.x;
  const uint64_t t0 = (uint64_t)t * pv.tile;
  const uint32_t count = pv.runs[(uint64_t)t * (P + 1) + P];
  // the answers (r, g, b of each entry) packed into LDS
  if (pv.state_dtype == 0) {
    const float4* src = pv.stage_v + t0;
    for (uint32_t i = tid; i < count; i += nt) {
      const float4 v = src[i];
      s_res[3 * i] = v.x;
      s_res[3 * i + 1] = v.y;
      s_res[3 * i + 2] = v.z;
    }
  } else {
    const unsigned long long* src = pv.stage_key + t0;
    for (uint32_t i = tid; i < count; i += nt) {
      const unsigned long long w = src[i];
      float r, g, b;
      decode16((uint32_t)w, (uint32_t)(w >> 32), pv.state_dtype, r, g, b);
      s_res[3 * i] = w == kDropped16 ? __uint_as_float(kDroppedBits) : r;
      s_res[3 * i + 1] = g;
      s_res[3 * i + 2] = b;
    }
  }
  __syncthreads();
  const uint64_t end = t0 + pv.tile < n ? t0 + pv.tile : n;
  const bool vec = (n & 3u) == 0 && ((uintptr_t)out & 15u) == 0 && ((uintptr_t)found & 3u) == 0;
  for (uint64_t i = t0 + 4ull * tid; i < end; i += 4ull * nt) {
    float r[4], g[4], b[4];
    uint8_t f[4];
    if (i + 4 <= end) {
      // i is a multiple of 4 and perm is 256-byte aligned
      const ushort4 pp = *reinterpret_cast<const ushort4*>(pv.perm + i);
      unstage_one(s_res, count, pp.x, r[0], g[0], b[0], f[0]);
      unstage_one(s_res, count, pp.y, r[1], g[1], b[1], f[1]);
      unstage_one(s_res, count, pp.z, r[2], g[2], b[2], f[2]);
      unstage_one(s_res, count, pp.w, r[3], g[3], b[3], f[3]);
    } else {
      for (int k = 0; k < 4; ++k) {
        const uint32_t pos = i + k < end ? pv.perm[i + k] : kNoPos;
        unstage_one(s_res, count, pos, r[k], g[k], b[k], f[k]);
      }
    }
    if (vec && i + 4 <= end) {
      typedef float v4f __attribute__((ext_vector_type(4)));
      __builtin_nontemporal_store(v4f{r[0], r[1], r[2], r[3]}, reinterpret_cast<v4f*>(out + i));
      __builtin_nontemporal_store(v4f{g[0], g[1], g[2], g[3]}, reinterpret_cast<v4f*>(out + n + i));
      __builtin_nontemporal_store(v4f{b[0], b[1], b[2], b[3]}, reinterpret_cast<v4f*>(out + 2 * n + i));
      if (found) *reinterpret_cast<uchar4*>(found + i) = make_uchar4(f[0], f[1], f[2], f[3]);
    } else {
      for (int k = 0; k < 4; ++k) {
        if (i + k >= end) break;
        out[i + k] = r[k];
        out[n + i + k] = g[k];
        out[2 * n + i + k] = b[k];
        if (found) found[i + k] = f[k];
      }
    }
  }
}

__global__ void __launch_bounds__(kUnstageThreads) k_unstage(PartView pv, uint32_t P, uint64_t n, float* out,
                                                             uint8_t* found) {
  unstage_body(pv, P, n, blockIdx.x, out, found);
}

// ------------------------------------------------------------------ launchers
static size_t bin_lds(uint32_t P, uint32_t tile) {
  const size_t hist = (size_t)(P + 1) * 4, stage = (size_t)tile * bin_lds_per_record(tile);
  return hist > stage ? hist : stage;
}

static size_t merge_lds(const TableView& tv, const PartView& pv) {
  return merge_lds_bytes(1u << tv.part_log2, tv.var || weighted(tv), pv.dense != 0);
}

// Where a frame of n records is dense: beyond 5/4 records a slot.  At the usual
// eight records a touched cell a partition needs its second round from 5/2
// records a slot on (2 with the further sum), but crowded partitions need it
// sooner, and a wave's entries past its first batch are read three times
// before that.  us a frame in rounds, and in one sweep: 2^22 slots in
// partitions of 2^12, n / slots = 1: 154 and 173; 1.5: 253 and 257; 2: 388 and
// 353; 3: 701 and 567.  2^20 in partitions of 2^11: 51.4 and 51.6; 70.4 and
// 70.4; 109 and 87; 220 and 157; with the variance, 2^10: 64.7 and 61.7; 109
// and 87; 169 and 105; 297 and 153.  16 records a slot in few cells (1,048,576
// weighted records, 2^16 slots): 344 and 256.
bool dense_records(uint64_t n, uint64_t slots) { return n > slots + slots / 4; }

// (2^12 slots with the further sum take 184 KB, more than a CU has: such a
// table's launches are never that dense, by its default width.)
constexpr size_t kMostLds = 156 * 1024;

bool dense_fits(const TableView& tv) {
  return merge_lds_bytes(1u << tv.part_log2, tv.var || weighted(tv), true) <= kMostLds;
}

bool dense_launch(uint64_t n, const TableView& tv) {
  return dense_records(n, 1ull << tv.log2_slots) && dense_fits(tv);
}

// In a batch, whose other sessions' blocks fill the CUs meanwhile, rounds in
// partitions of 2^12 slots hold out to 5/2 records a slot: sixteen sessions of
// 0.75 to 4 with 1 to 4 samples a pixel 4.99 ms, from 5/4 on 5.05, in rounds for
// all 4.96; eight of 1 to 2 with one sample a pixel 413 us, 401 and 412; eight of
// 2 to 4 592 us, 592 and 1165.
bool dense_session(uint64_t n, const TableView& tv) {
  const uint64_t slots = 1ull << tv.log2_slots;
  return dense_launch(n, tv) && (tv.part_log2 < 12 || n > slots * 2 + slots / 2);
}

static bool tile_ok(uint32_t tile) {
  return tile == 1024 || tile == 2048 || (tile % 512 == 0 && bin_per_ok(tile / 512));
}

bool partition_ok(const TableView& tv, const PartView& pv, uint64_t n) {
  return n <= pv.capacity && tv.part_log2 <= kMaxPartLog2 && tile_ok(pv.tile) &&
         (n + pv.tile - 1) / pv.tile <= pv.max_tiles && (1u << (tv.log2_slots - tv.part_log2)) <= kTouchEntries;
}

template <uint32_t kThreads, uint32_t kPer, uint32_t kX>
static hipError_t launch_bin_t(const RecPtrs& rec, uint64_t n, const KeyParams& kp, const TableView& tv,
                               const PartView& pv, size_t shm, uint32_t ntiles, hipStream_t s) {
  static LdsLimit lim;  // one per instantiation
  hipError_t e = lds_limit(reinterpret_cast<const void*>(&k_bin<kThreads, kPer, kX>), shm, &lim);
  if (e != hipSuccess) return e;
  k_bin<kThreads, kPer, kX><<<ntiles, kThreads, shm, s>>>(rec, n, kp, tv, pv);
  return hipGetLastError();
}

template <uint32_t kAlso, uint32_t kThreads, uint32_t kPer, uint32_t kThreadsX = kThreads, uint32_t kPerX = kPer>
static hipError_t launch_bin_x(uint32_t x, const RecPtrs& rec, uint64_t n, const KeyParams& kp,
                               const TableView& tv, const PartView& pv, size_t shm, uint32_t ntiles,
                               hipStream_t s) {
  switch (x) {
    case 0: return launch_bin_t<kThreads, kPer, kAlso>(rec, n, kp, tv, pv, shm, ntiles, s);
    case kXFootprint: return launch_bin_t<kThreadsX, kPerX, kAlso | kXFootprint>(rec, n, kp, tv, pv, shm, ntiles, s);
    case kXWeight: return launch_bin_t<kThreadsX, kPerX, kAlso | kXWeight>(rec, n, kp, tv, pv, shm, ntiles, s);
    default: return launch_bin_t<kThreadsX, kPerX, kAlso | kXFootprint | kXWeight>(rec, n, kp, tv, pv, shm, ntiles, s);
  }
}

// What a launch's records carry (kX bits); weights need the staging array.
static uint32_t record_extras(const RecPtrs& rec) {
  return (rec.footprint ? kXFootprint : 0u) | (rec.weight ? kXWeight : 0u);
}

hipError_t launch_bin(const RecPtrs& rec, uint64_t n, const KeyParams& kp, const TableView& tv,
                      const PartView& pv, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (!partition_ok(tv, pv, n)) return hipErrorInvalidValue;
  const uint32_t P = 1u << (tv.log2_slots - tv.part_log2);
  const uint32_t ntiles = (uint32_t)((n + pv.tile - 1) / pv.tile);
  const size_t shm = bin_lds(P, pv.tile);
  const uint32_t x = record_extras(rec);
  if ((x & kXWeight) && !weighted(tv)) return hipErrorInvalidValue;
  if (tv.sh) {
    if (!pv.stage_n || pv.perm) return hipErrorInvalidValue;
    switch (pv.tile) {
      case 1024: return launch_bin_x<kXNormal, 1024, 1>(x, rec, n, kp, tv, pv, shm, ntiles, s);
      case 2048: return launch_bin_x<kXNormal, 1024, 2>(x, rec, n, kp, tv, pv, shm, ntiles, s);
      case 4096: return launch_bin_x<kXNormal, 1024, 4>(x, rec, n, kp, tv, pv, shm, ntiles, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (pv.tile) {
    case 1024: return launch_bin_x<0, 1024, 1>(x, rec, n, kp, tv, pv, shm, ntiles, s);
    case 2048: return launch_bin_x<0, 1024, 2>(x, rec, n, kp, tv, pv, shm, ntiles, s);
    case 4096: return launch_bin_x<0, 1024, 4>(x, rec, n, kp, tv, pv, shm, ntiles, s);
    case 6144: return launch_bin_x<0, 768, 8, 512, 12>(x, rec, n, kp, tv, pv, shm, ntiles, s);
    default: return launch_bin_x<0, 1024, 8>(x, rec, n, kp, tv, pv, shm, ntiles, s);
  }
}

template <bool kFused, int kThreads, bool kVar, bool kDense>
static hipError_t launch_merge_t(const TableView& tv, const PartView& pv, uint32_t ntiles, const BlendParams& bp,
                                 int32_t results, hipStream_t s) {
  static LdsLimit lim;  // one per instantiation
  const size_t shm = merge_lds(tv, pv);
  hipError_t e = lds_limit(reinterpret_cast<const void*>(&k_merge<kFused, kThreads, kVar, kDense>), shm, &lim);
  if (e != hipSuccess) return e;
  k_merge<kFused, kThreads, kVar, kDense><<<1u << (tv.log2_slots - tv.part_log2), kThreads, shm, s>>>(tv, pv, ntiles, bp, results);
  return hipGetLastError();
}

template <bool kFused, bool kVar>
static hipError_t launch_merge_f(const TableView& tv, const PartView& pv, uint32_t ntiles, const BlendParams& bp,
                                 int32_t results, hipStream_t s) {
  if (pv.dense) {
    return merge_threads_dense(merge_lds(tv, pv)) == 1024
               ? launch_merge_t<kFused, 1024, kVar, true>(tv, pv, ntiles, bp, results, s)
               : launch_merge_t<kFused, 512, kVar, true>(tv, pv, ntiles, bp, results, s);
  }
  switch (merge_threads(tv.part_log2, 1u << (tv.log2_slots - tv.part_log2))) {
    case 768: return launch_merge_t<kFused, 768, kVar, false>(tv, pv, ntiles, bp, results, s);
    case 384: return launch_merge_t<kFused, 384, kVar, false>(tv, pv, ntiles, bp, results, s);
    default: return launch_merge_t<kFused, 192, kVar, false>(tv, pv, ntiles, bp, results, s);
  }
}

hipError_t launch_merge(uint64_t n, const TableView& tv, const PartView& pv, const BlendParams* fuse,
                        bool results, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (!partition_ok(tv, pv, n)) return hipErrorInvalidValue;
  const uint32_t ntiles = (uint32_t)((n + pv.tile - 1) / pv.tile);
  // staged lookup-only entries exist exactly when the bin pass wrote perm
  if (results != (pv.perm != nullptr) || (results && !fuse)) return hipErrorInvalidValue;
  const int32_t res = results ? 1 : 0;
  if (tv.var)
    return fuse ? launch_merge_f<true, true>(tv, pv, ntiles, *fuse, res, s)
                : launch_merge_f<false, true>(tv, pv, ntiles, BlendParams{}, 0, s);
  return fuse ? launch_merge_f<true, false>(tv, pv, ntiles, *fuse, res, s)
              : launch_merge_f<false, false>(tv, pv, ntiles, BlendParams{}, 0, s);
}

static size_t unstage_lds(uint32_t tile) { return (size_t)tile * 12; }

uint32_t transpose_blocks(uint32_t ntiles, uint32_t P) {
  return ((ntiles + kTransposeDim - 1) / kTransposeDim) * ((P + 1 + kTransposeDim - 1) / kTransposeDim);
}

bool transpose_pays(uint32_t ntiles, uint32_t P) { return (uint64_t)ntiles * (P + 1) >= kTransposeMinWords; }

hipError_t launch_transpose_runs(const TableView& tv, const PartView& pv, uint32_t ntiles, hipStream_t s) {
  if (ntiles == 0 || !pv.runs_t) return hipSuccess;
  if (ntiles > pv.max_tiles) return hipErrorInvalidValue;
  const uint32_t P = 1u << (tv.log2_slots - tv.part_log2);
  const dim3 grid((ntiles + kTransposeDim - 1) / kTransposeDim, (P + 1 + kTransposeDim - 1) / kTransposeDim);
  k_transpose_runs<<<grid, kTransposeThreads, 0, s>>>(pv, P, ntiles);
  return hipGetLastError();
}

hipError_t launch_unstage(uint64_t n, const TableView& tv, const PartView& pv, float* out,
                          uint8_t* found, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (!partition_ok(tv, pv, n) || !pv.perm) return hipErrorInvalidValue;
  const uint32_t P = 1u << (tv.log2_slots - tv.part_log2);
  const uint32_t ntiles = (uint32_t)((n + pv.tile - 1) / pv.tile);
  const size_t shm = unstage_lds(pv.tile);
  static LdsLimit lim;
  hipError_t e = lds_limit(reinterpret_cast<const void*>(&k_unstage), shm, &lim);
  if (e != hipSuccess) return e;
  k_unstage<<<ntiles, unstage_threads(pv.tile), shm, s>>>(pv, P, n, out, found);
  return hipGetLastError();
}


// ------------------------------------------------------------------ batched sessions
// One launch per pass covers every session: a block finds its session by
// its index among the sessions' block ranges and runs the single-table body
// with the session's views, copied out of the descriptor first (read in
// place, the descriptor is global memory the body's stores might alias, so
// its fields would be loaded again after every store: the batched merge ran
// 15 % slower than the single-table one that way).  begins[0..k) holds each session's first block
// of the pass (non-decreasing, begins[0] = 0); the block's session is the
// last one starting at or before it: one coalesced load and a ballot per 64
// sessions (a scan through the descriptors would cost a dependent load per
// session).  Called by whole waves; the result is wave-uniform.
__device__ __forceinline__ uint32_t find_session(const uint32_t* begins, uint32_t k, uint32_t b) {
  uint32_t count = 0;
  for (uint32_t c = 0; c < k; c += 64) {
    const uint32_t i = c + __lane_id();
    count += (uint32_t)__popcll(__ballot(i < k && begins[i] <= b));
  }
  return count - 1;
}

__global__ void __launch_bounds__(kTransposeThreads) k_transpose_batch(const BatchSession* ss, const uint32_t* bg,
                                                                       uint32_t k) {
  const BatchSession& S = ss[find_session(bg, k, blockIdx.x)];
  const uint32_t local = blockIdx.x - S.trans_begin;
  const PartView pv = S.pv;
  if (local >= S.ntrans || !pv.runs_t) return;
  const uint32_t P = 1u << (S.tv.log2_slots - S.tv.part_log2);
  const uint32_t ntiles = S.ntiles;
  const uint32_t gx = (ntiles + kTransposeDim - 1) / kTransposeDim;
  transpose_body(pv, P, ntiles, local % gx, local / gx);
}

// kX: the union of the sessions' record extras; each session runs the body
// of its own.
template <uint32_t kThreads, uint32_t kPer, uint32_t kW, uint32_t kFpAllowed>
__device__ __forceinline__ void bin_session(const BatchSession& S, uint32_t local) {
  const RecPtrs rec = S.rec;
  const KeyParams kp = S.kp;
  const TableView tv = S.tv;
  const PartView pv = S.pv;
  const uint64_t n = S.n;
  if (kFpAllowed && rec.footprint)
    bin_body<kThreads, kPer, kW | kXFootprint>(rec, n, kp, tv, pv, local);
  else
    bin_body<kThreads, kPer, kW>(rec, n, kp, tv, pv, local);
}

template <uint32_t kThreads, uint32_t kPer, uint32_t kX>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(bin_waves(kThreads, kPer, kX & kXWeight))))
k_bin_batch(const BatchSession* ss, const uint32_t* bg, uint32_t k) {
  const BatchSession& S = ss[find_session(bg, k, blockIdx.x)];
  const uint32_t local = blockIdx.x - S.tile_begin;
  if (local >= S.ntiles) return;
  if constexpr ((kX & kXWeight) != 0) {
    if (S.rec.weight) {
      bin_session<kThreads, kPer, kXWeight, kX & kXFootprint>(S, local);
      return;
    }
  }
  bin_session<kThreads, kPer, 0, kX & kXFootprint>(S, local);
}

// As many threads per block as the widest session's partitions take; kVar: a
// session keeps the luminance variance; kDense: the sessions of many records
// a slot, which a launch of their own takes (the others' blocks end at once).
template <int kThreads, bool kVar, bool kDense>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(merge_waves(kVar, kDense))))
k_merge_batch(const BatchSession* ss, const uint32_t* bg, uint32_t k) {
  const BatchSession& S = ss[find_session(bg, k, blockIdx.x)];
  const uint32_t local = blockIdx.x - S.part_begin;
  if (local >= S.nparts || (S.pv.dense != 0) != kDense) return;
  const TableView tv = S.tv;
  const PartView pv = S.pv;
  const BlendParams bp = S.bp;
  if constexpr (kVar) {
    if (tv.var) {
      merge_body<true, kThreads, true, kDense>(tv, pv, S.ntiles, bp, local, S.fused_query != 0);
      return;
    }
  }
  merge_body<true, kThreads, false, kDense>(tv, pv, S.ntiles, bp, local, S.fused_query != 0);
}

// A session whose queries are its records takes one unstage block per tile;
// any other session one lookup block per kQueryBlock queries.
__global__ void __launch_bounds__(kQueryBlock) k_query_batch(const BatchSession* ss, const uint32_t* bg,
                                                              uint32_t k) {
  const BatchSession& S = ss[find_session(bg, k, blockIdx.x)];
  const uint32_t local = blockIdx.x - S.qblk_begin;
  float* out = S.out;
  uint8_t* found = S.found;
  if (S.fused_query) {
    const PartView pv = S.pv;
    if (local < S.ntiles)
      unstage_body(pv, 1u << (S.tv.log2_slots - S.tv.part_log2), S.n, local, out, found);
    return;
  }
  const uint64_t nq = S.nq;
  const uint64_t start = (uint64_t)local * kQueryBlock;
  if (start >= nq) return;
  const uint32_t last = nq - start < kQueryBlock ? (uint32_t)(nq - start) - 1 : kQueryBlock - 1;
  const TableView tv = S.tv;
  const KeyParams kp = S.kp;
  const QryPtrs q = S.q;
  const uint32_t ti = threadIdx.x < last ? threadIdx.x : last;
  Vertex v = load_vertex(q, start, ti);
  load_vertex_direction(q, kp.rough_thr, start, ti, v);
  loaded(v);
  float rgb[3];
  const uint8_t hit = lookup_key(tv, S.bp.dtype, vertex_key(kp, q, v), rgb);
  if (threadIdx.x > last) return;
  const uint64_t i = start + threadIdx.x;
  out[i] = rgb[0];
  out[nq + i] = rgb[1];
  out[2 * nq + i] = rgb[2];
  if (found) found[i] = hit;
}

template <uint32_t kThreads, uint32_t kPer, uint32_t kX>
static hipError_t launch_bin_batch_t(const BatchSession* d_ss, const uint32_t* bg, uint32_t k, uint32_t tiles,
                                     size_t lds, hipStream_t s) {
  static LdsLimit lim;  // one per instantiation
  hipError_t e = lds_limit(reinterpret_cast<const void*>(&k_bin_batch<kThreads, kPer, kX>), lds, &lim);
  if (e != hipSuccess) return e;
  k_bin_batch<kThreads, kPer, kX><<<tiles, kThreads, lds, s>>>(d_ss, bg, k);
  return hipGetLastError();
}

template <uint32_t kThreads, uint32_t kPer, uint32_t kThreadsW = kThreads, uint32_t kPerW = kPer>
static hipError_t launch_bin_batch_x(uint32_t x, const BatchSession* d_ss, const uint32_t* bg, uint32_t k,
                                     uint32_t tiles, size_t lds, hipStream_t s) {
  switch (x) {
    case 0: return launch_bin_batch_t<kThreads, kPer, 0>(d_ss, bg, k, tiles, lds, s);
    case kXFootprint: return launch_bin_batch_t<kThreads, kPer, kXFootprint>(d_ss, bg, k, tiles, lds, s);
    case kXWeight: return launch_bin_batch_t<kThreadsW, kPerW, kXWeight>(d_ss, bg, k, tiles, lds, s);
    default: return launch_bin_batch_t<kThreadsW, kPerW, kXFootprint | kXWeight>(d_ss, bg, k, tiles, lds, s);
  }
}

template <int kThreads, bool kVar, bool kDense>
static hipError_t launch_merge_batch_v(const BatchSession* d_ss, const uint32_t* bg, uint32_t k, uint32_t parts,
                                       size_t lds, hipStream_t s) {
  static LdsLimit lim;  // one per instantiation
  hipError_t e = lds_limit(reinterpret_cast<const void*>(&k_merge_batch<kThreads, kVar, kDense>), lds, &lim);
  if (e != hipSuccess) return e;
  k_merge_batch<kThreads, kVar, kDense><<<parts, kThreads, lds, s>>>(d_ss, bg, k);
  return hipGetLastError();
}

template <int kThreads, bool kDense>
static hipError_t launch_merge_batch_t(bool var, const BatchSession* d_ss, const uint32_t* bg, uint32_t k,
                                       uint32_t parts, size_t lds, hipStream_t s) {
  return var ? launch_merge_batch_v<kThreads, true, kDense>(d_ss, bg, k, parts, lds, s)
             : launch_merge_batch_v<kThreads, false, kDense>(d_ss, bg, k, parts, lds, s);
}

hipError_t launch_batch(const BatchSession* d_ss, const uint32_t* d_begins, const uint32_t* h_begins,
                        uint32_t stride, const BatchSession* h_ss, uint32_t k, hipStream_t s) {
  if (k == 0) return hipSuccess;
  if (k > stride) return hipErrorInvalidValue;
  uint32_t tiles = 0, parts = 0, qblks = 0, trans = 0;
  size_t lds_b = 0, lds_q = 0;
  uint32_t x = 0;  // what any session's records carry
  struct {
    bool any, var;
    uint32_t part_log2;  // the widest partitions
    size_t lds;
  } merge[2] = {};  // of the ordinary and of the dense sessions
  for (uint32_t i = 0; i < k; ++i) {
    const BatchSession& S = h_ss[i];
    if (h_begins[i] != S.tile_begin || h_begins[stride + i] != S.part_begin ||
        h_begins[2 * stride + i] != S.qblk_begin || h_begins[3 * stride + i] != S.trans_begin)
      return hipErrorInvalidValue;
    if (S.n == 0 || !partition_ok(S.tv, S.pv, S.n) || S.pv.tile != h_ss[0].pv.tile ||
        S.tile_begin != tiles || S.part_begin != parts || S.qblk_begin != qblks || (S.part_begin & 7u) ||
        S.trans_begin != trans ||
        S.ntrans != (S.pv.runs_t ? transpose_blocks(S.ntiles, 1u << (S.tv.log2_slots - S.tv.part_log2)) : 0u))
      return hipErrorInvalidValue;
    const uint32_t P = 1u << (S.tv.log2_slots - S.tv.part_log2);
    const size_t lb = bin_lds(P, S.pv.tile), lm = merge_lds(S.tv, S.pv);
    lds_b = lb > lds_b ? lb : lds_b;
    auto& mg = merge[S.pv.dense ? 1 : 0];
    mg.any = true;
    mg.lds = lm > mg.lds ? lm : mg.lds;
    mg.part_log2 = S.tv.part_log2 > mg.part_log2 ? S.tv.part_log2 : mg.part_log2;
    mg.var = mg.var || S.tv.var;
    if ((S.fused_query != 0) != (S.pv.perm != nullptr)) return hipErrorInvalidValue;
    if (S.fused_query) {
      if (S.nq != S.n || S.nqblk != S.ntiles) return hipErrorInvalidValue;
      lds_q = unstage_lds(S.pv.tile);
    }
    const uint32_t xs = record_extras(S.rec);
    if ((xs & kXWeight) && !weighted(S.tv)) return hipErrorInvalidValue;
    x |= xs;
    tiles += S.ntiles;
    parts += (S.nparts + 7u) & ~7u;
    qblks += S.nqblk;
    trans += S.ntrans;
  }
  static LdsLimit lim_q;
  const uint32_t* bg_tile = d_begins;
  const uint32_t* bg_part = d_begins + stride;
  const uint32_t* bg_qblk = d_begins + 2 * stride;
  const uint32_t* bg_trans = d_begins + 3 * stride;
  hipError_t e;
  switch (h_ss[0].pv.tile) {
    case 1024: e = launch_bin_batch_x<1024, 1>(x, d_ss, bg_tile, k, tiles, lds_b, s); break;
    case 2048: e = launch_bin_batch_x<1024, 2>(x, d_ss, bg_tile, k, tiles, lds_b, s); break;
    case 4096: e = launch_bin_batch_x<1024, 4>(x, d_ss, bg_tile, k, tiles, lds_b, s); break;
    case 6144: e = launch_bin_batch_x<512, 12>(x, d_ss, bg_tile, k, tiles, lds_b, s); break;
    default: e = launch_bin_batch_x<1024, 8>(x, d_ss, bg_tile, k, tiles, lds_b, s); break;
  }
  if (e != hipSuccess) return e;
  e = lds_limit(reinterpret_cast<const void*>(&k_query_batch), lds_q, &lim_q);
  if (e != hipSuccess) return e;
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (trans) k_transpose_batch<<<trans, kTransposeThreads, 0, s>>>(d_ss, bg_trans, k);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (merge[0].any) {
    const auto& mg = merge[0];
    switch (merge_threads(mg.part_log2)) {
      case 768: e = launch_merge_batch_t<768, false>(mg.var, d_ss, bg_part, k, parts, mg.lds, s); break;
      case 384: e = launch_merge_batch_t<384, false>(mg.var, d_ss, bg_part, k, parts, mg.lds, s); break;
      default: e = launch_merge_batch_t<192, false>(mg.var, d_ss, bg_part, k, parts, mg.lds, s); break;
    }
    if (e != hipSuccess) return e;
  }
  if (merge[1].any) {
    const auto& mg = merge[1];
    e = merge_threads_dense(mg.lds) == 1024
            ? launch_merge_batch_t<1024, true>(mg.var, d_ss, bg_part, k, parts, mg.lds, s)
            : launch_merge_batch_t<512, true>(mg.var, d_ss, bg_part, k, parts, mg.lds, s);
    if (e != hipSuccess) return e;
  }
  if (qblks) k_query_batch<<<qblks, kQueryBlock, lds_q, s>>>(d_ss, bg_qblk, k);
  return hipGetLastError();
}

}  // namespace psf
