// Device-side definitions shared by the PSTF kernels: the cell key, the slot
// hash, the table layout and the 16-bit state encodings.
//
// Everything here runs on gfx950 only.  The translation units that include
// this header are compiled with -ffp-contract=off and correctly rounded FP32
// division, so the floating point that decides a key is plain IEEE binary32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace psf {

constexpr uint64_t kEmpty = ~0ull;  // valid keys never set bit 63

// Parameters of the key function (spatio-directional hashing, Sec. 2.6 of the
// paper; the quantisation itself is this library's specification).
struct KeyParams {
  float cx, cy, cz;
  float kappa;
  int32_t e_min;
  int32_t max_level;
  int32_t nb_log2;
  int32_t db_log2;
  float rough_thr;
};

// One table slot, 32 bytes: everything a lookup needs sits in one sector.
struct alignas(32) Slot {
  unsigned long long key;  // kEmpty when free
  uint32_t c_old;          // cumulative counter (Sec. 2.4, c_h^old): a sample
                           // count, or in a weighted table the binary32 bits
                           // of a weight sum (0 bits = 0 either way)
  uint32_t pad;
  uint32_t L[4];           // approximant: 3 x f32, or 3 x 16-bit packed in L[0..1]
};

// Per-slot accumulator of the current frame (Eq. 5-6 numerator / counter;
// n holds binary32 bits of the weight sum in a weighted table).
struct alignas(16) Acc {
  uint32_t n;
  float s[3];
};

// Device-resident event counters (one atomic per wave or block when
// non-zero).  Rejected samples are not always rare (a field that leaves a
// sampling technique out rejects every sample of it), so the skip and
// overflow counts are spread over kStatLanes counters a cache line apart,
// picked by block index, and summed when the statistics are read: atomics
// on one address serialise.
constexpr uint32_t kStatLanes = 32;
struct alignas(256) DevStats {
  unsigned long long dropped;
  unsigned long long saturated;
  unsigned long long probe_hist[16];
  unsigned long long pad[14];
  unsigned long long skipped[kStatLanes][8];         // [lane][0] used
  unsigned long long coord_overflow[kStatLanes][8];  // [lane][0] used
};

__device__ __forceinline__ unsigned long long* stat_lane(unsigned long long (*c)[8], uint32_t block) {
  return &c[block % kStatLanes][0];
}

// Per-block count of blended cells, written by the block that owns the entry
// (no shared counters on the hot path).
struct alignas(16) BlockTouch {
  uint32_t last;
  uint32_t pad;
  unsigned long long total;
};
constexpr uint32_t kTouchEntries = 1u << 14;

// Two-band SH payload (Sec. 2.6): a cell's state, the four luminance
// coefficients and the chroma pair (24 bytes, padded to 32), and its frame
// sums in binary64: weight, Gram matrix of the basis over the sample
// normals (upper triangle), basis-weighted luminance, chroma sums.
struct alignas(16) ShState {
  float c[4];
  float co, cg;
  float pad[2];
};
struct alignas(16) ShAcc {
  double n;
  double g[10];
  double r[4];
  double co, cg;
  double pad;
};

// View of one table handed to kernels by value.
struct TableView {
  Slot* slots;
  unsigned long long* keys;  // mirror of slots[].key, read by the partitioned merge
  Acc* acc;
  ShState* sh;               // SH payload only (else null)
  ShAcc* sh_acc;
  DevStats* stats;
  BlockTouch* touch;         // kTouchEntries
  float* var;                // luminance variance per slot (PSF_FLAG_TRACK_VARIANCE, else null)
  double* acc_q;             // the frame's sum of squared luminances per slot (idem)
  uint32_t log2_slots;
  uint32_t part_log2;        // slots per partition = 2^part_log2 (<= log2_slots)
  uint32_t max_probe;
  uint32_t flags;            // public PSF_FLAG_* bits | kTvWeighted
};

// TableView::flags bit of a table with MIS-weighted (binary32) counters.
constexpr uint32_t kTvWeighted = 1u << 16;

__host__ __device__ __forceinline__ bool weighted(const TableView& tv) { return (tv.flags & kTvWeighted) != 0; }

// A counter word as a number: a count, or a weight sum's binary32 bits.
__device__ __forceinline__ float counter_value(uint32_t c, bool wtd) {
  return wtd ? __uint_as_float(c) : (float)c;
}

// c_old + n as a counter word.  In a weighted table both are binary32 weight
// sums and this addition rounds once; the frame's sum n is itself rounded
// once from binary64 by the partitioned merge, but accumulated with binary32
// atomics (in no fixed order) by the direct insert.
__device__ __forceinline__ uint32_t counter_add(uint32_t c, uint32_t n, bool wtd) {
  return wtd ? __float_as_uint(__uint_as_float(c) + __uint_as_float(n)) : c + n;
}

// Per-cell luminance variance (tables created with PSF_FLAG_TRACK_VARIANCE).
// A sample's luminance is Y of YCoCg, (r + 2 g + b) / 4, in binary64.
__device__ __forceinline__ double luma64(double r, double g, double b) { return ((r + 2.0 * g) + b) * 0.25; }

// The frame's luminance mean m and population variance s2 from its sums
// (channel sums s0..s2, squared-luminance sum q, n samples) in binary64.
__device__ __forceinline__ void frame_moments(double s0, double s1, double s2, double q, double n, double& m,
                                              double& var) {
  m = luma64(s0, s1, s2) / n;
  var = q / n - m * m;
  if (var < 0.0) var = 0.0;
}

// One blend of the variance (binary32): the two-component mixture of the
// cells' samples so far (weight 1 - alpha, variance V around mu, the
// luminance of the state the blend continues from) and the frame's (weight
// alpha, mean m, variance s2).
__device__ __forceinline__ float blend_variance(float V, float alpha, float mu, double m, double s2) {
  const float sf = (float)s2;
  if (alpha == 1.0f) return sf;
  const float d = (float)m - mu;
  return (1.0f - alpha) * V + alpha * (sf + (1.0f - alpha) * (d * d));
}

__device__ __forceinline__ float luma32(float r, float g, float b) { return ((r + 2.0f * g) + b) * 0.25f; }

struct BlendParams {
  int32_t mode;     // 0 Eq. 11, 1 constant alpha, 2 linear
  float alpha;
  float inv_t_max;
  int32_t dtype;    // 0 f32, 1 f16, 2 bf16
};

// ------------------------------------------------------------------ hashing
// 64-bit finaliser of MurmurHash3 (A. Appleby, public domain).
__device__ __forceinline__ uint64_t fmix64(uint64_t h) {
  h ^= h >> 33;
  h *= 0xff51afd7ed558ccdull;
  h ^= h >> 33;
  h *= 0xc4ceb9fe1a85ec53ull;
  h ^= h >> 33;
  return h;
}

// Probe sequence of a key: partition = top hash bits, start = low hash bits,
// linear probing wraps inside the partition.
struct ProbeSeq {
  uint64_t base;
  uint32_t start;
  uint32_t mask;
  __device__ __forceinline__ uint64_t at(uint32_t i) const { return base + ((start + i) & mask); }
};

__device__ __forceinline__ uint32_t partition_of(uint64_t h, uint32_t log2_slots, uint32_t part_log2) {
  uint32_t pbits = log2_slots - part_log2;
  return pbits == 0 ? 0u : (uint32_t)(h >> (64 - pbits));
}

__device__ __forceinline__ ProbeSeq probe_seq(uint64_t key, uint32_t log2_slots, uint32_t part_log2) {
  uint64_t h = fmix64(key);
  ProbeSeq p;
  p.mask = (1u << part_log2) - 1u;
  p.base = (uint64_t)partition_of(h, log2_slots, part_log2) << part_log2;
  p.start = (uint32_t)h & p.mask;
  return p;
}

// ------------------------------------------------------------------ key
#pragma clang fp contract(off)

__device__ __forceinline__ bool finite3(float a, float b, float c) {
  return (int)__builtin_isfinite(a) & (int)__builtin_isfinite(b) & (int)__builtin_isfinite(c);
}

// Level: floor(log2(kappa * d^2) / 2) clamped, read off the binary32 exponent.
__device__ __forceinline__ int32_t cell_level(const KeyParams& kp, float px, float py, float pz) {
  const float dx = px - kp.cx, dy = py - kp.cy, dz = pz - kp.cz;
  const float d2 = (dx * dx + dy * dy) + dz * dz;
  const float q = d2 * kp.kappa;
  const int32_t biased = (int32_t)((__float_as_uint(q) >> 23) & 0xffu);
  const int32_t e = biased ? biased - 127 : -127;
  const int32_t lvl = e >> 1;  // arithmetic shift: floor(e / 2)
  const int32_t most = kp.kappa == 0.0f ? 0 : kp.max_level;
  return lvl < 0 ? 0 : (lvl > most ? most : lvl);
}

// Level from a path footprint (the world-space width a path covers at the
// vertex, the quantity the paper selects levels by in Sec. 2.3): the largest
// l with 2^(e_min + l) <= footprint, clamped to [0, max_level], read off the
// binary32 exponent (subnormals count as 2^-127).
__device__ __forceinline__ int32_t footprint_level(const KeyParams& kp, float fp) {
  const int32_t biased = (int32_t)((__float_as_uint(fp) >> 23) & 0xffu);
  const int32_t e = biased ? biased - 127 : -127;
  const int32_t lvl = e - kp.e_min;
  return lvl < 0 ? 0 : (lvl > kp.max_level ? kp.max_level : lvl);
}

// floor(p * 2^-shift) modulo 2^16; f receives the floor itself.
__device__ __forceinline__ uint32_t grid16(float p, int32_t shift, float& f) {
  f = floorf(ldexpf(p, -shift));
  return (uint32_t)(int32_t)fminf(fmaxf(f, -2147483648.0f), 2147483520.0f) & 0xffffu;
}

// Octahedral map of a direction onto a B x B grid (B = 2^b): index iu*B + iw,
// where with l1 = (|x| + |y|) + |z|, u = x / l1 and w = y / l1 (correctly
// rounded; 0 if l1 is 0), folded over for z < 0, iu = min(floor((u / 2 + 1 / 2)
// B), B - 1) and likewise iw.
//
// Both quotients share one reciprocal: after a Newton step on it, each takes
// two remainder corrections, the last from a remainder that is exact, so it
// is the correctly rounded quotient wherever nothing underflows.  That holds
// for l1 in [2^-60, 2^60] and numerators above 2^-100; below those u is so
// small that it rounds away against 1 or 1 / 2.  A wave with a lane outside
// that range of l1 (scaled first, by a power of two) takes one more branch.
// The fold's sign is that of the rounded u, which is +0 or -0 (counted as
// positive) where |x| <= l1 2^-150.
__device__ __forceinline__ uint32_t octa_bin(float x, float y, float z, int32_t b) {
  const float l1 = (fabsf(x) + fabsf(y)) + fabsf(z);
  float xs = x, ys = y, ls = l1;
  if (__ballot(!(l1 >= 0x1p-60f && l1 <= 0x1p60f))) {
    int32_t e = 0;
    (void)frexpf(l1, &e);
    xs = ldexpf(x, -e);
    ys = ldexpf(y, -e);
    ls = ldexpf(l1, -e);
    if (!(l1 > 0.0f && l1 <= 3.402823466e38f)) {  // all zero, or the sum overflowed
      xs = ys = 0.0f;
      ls = 1.0f;
    }
  }
  const float r0 = __builtin_amdgcn_rcpf(ls);
  const float rc = __builtin_fmaf(__builtin_fmaf(-ls, r0, 1.0f), r0, r0);
  auto quotient = [&](float n) {
    float q = n * rc;
    q = __builtin_fmaf(__builtin_fmaf(-ls, q, n), rc, q);
    return __builtin_fmaf(__builtin_fmaf(-ls, q, n), rc, q);
  };
  const float u = quotient(xs), w = quotient(ys);
  const float tiny = -(l1 * 0x1p-50f);
  const float fu = copysignf(1.0f - fabsf(w), x * 0x1p100f >= tiny ? 1.0f : -1.0f);
  const float fw = copysignf(1.0f - fabsf(u), y * 0x1p100f >= tiny ? 1.0f : -1.0f);
  const bool fold = z < 0.0f;
  // (u / 2 + 1 / 2) B = u B / 2 + B / 2, rounded once either way; in [0, B]
  const float h = 0.5f * (float)(1 << b);
  const uint32_t top = (1u << b) - 1u;
  const uint32_t iu = (uint32_t)__builtin_fmaf(fold ? fu : u, h, h);
  const uint32_t iw = (uint32_t)__builtin_fmaf(fold ? fw : w, h, h);
  return ((iu < top ? iu : top) << b) + (iw < top ? iw : top);
}

// The parts of a cell key.  None decides anything by branches on the lane's
// values: a key is computed for every lane, rejected ones too, and rejected
// at the end.  (With early exits and four divisions it took 212 vector
// instructions in 15 exec-mask regions, and its scalar masks spilled in the
// binning pass.)

// Level of a vertex, from its footprint (has_fp; it must be finite and > 0)
// or the camera distance.
__device__ __forceinline__ int32_t key_level(const KeyParams& kp, float px, float py, float pz, bool has_fp, float fp,
                                             int& ok) {
  if (!has_fp) return cell_level(kp, px, py, pz);
  ok &= (int)__builtin_isfinite(fp) & (int)(fp > 0.0f);
  return footprint_level(kp, fp);
}

// High word: the normal's bin, and at glossy vertices (has_rough and rough
// below the threshold) the flag and the direction's bin.  has_rough is false
// when the caller supplied no roughness array (every vertex diffuse); the
// direction is used only for glossy vertices.
__device__ __forceinline__ uint32_t key_normal(const KeyParams& kp, float nx, float ny, float nz) {
  return octa_bin(nx, ny, nz, kp.nb_log2) << 16;
}
__device__ __forceinline__ uint32_t key_direction(const KeyParams& kp, float ox, float oy, float oz, bool has_rough,
                                                  float rough, int& ok) {
  if (!has_rough) return 0u;
  const bool glossy = rough < kp.rough_thr;
  ok &= (int)__builtin_isfinite(rough) & ((int)!glossy | (int)finite3(ox, oy, oz));
  uint32_t hi = 0u;
  if (__ballot(glossy)) hi = glossy ? (1u << 26) | (octa_bin(ox, oy, oz, kp.db_log2) << 20) : 0u;
  return hi;
}

// The whole key from the high word's bins and the position at a level.
__device__ __forceinline__ uint64_t key_at(const KeyParams& kp, float px, float py, float pz, int32_t lvl, uint32_t hi,
                                           bool& ovf) {
  const int32_t shift = kp.e_min + lvl;
  float fx, fy, fz;
  const uint32_t ix = grid16(px, shift, fx), iy = grid16(py, shift, fy), iz = grid16(pz, shift, fz);
  // a coordinate outside [-2^15, 2^15): an integer f with |f + 1/2| > 2^15 - 1/2
  ovf = fmaxf(fmaxf(fabsf(fx + 0.5f), fabsf(fy + 0.5f)), fabsf(fz + 0.5f)) > 32767.5f;
  hi |= ((uint32_t)lvl << 27) | iz;
  return ((uint64_t)hi << 32) | (iy << 16) | ix;
}

// Cell key of one vertex.  Returns false for rejected (non-finite) input.
__device__ __forceinline__ bool cell_key(const KeyParams& kp, float px, float py, float pz, float nx,
                                         float ny, float nz, float ox, float oy, float oz,
                                         bool has_rough, float rough, bool has_fp, float fp,
                                         uint64_t& key, bool& ovf) {
  int ok = (int)finite3(px, py, pz) & (int)finite3(nx, ny, nz);
  const int32_t lvl = key_level(kp, px, py, pz, has_fp, fp, ok);
  const uint32_t hi = key_normal(kp, nx, ny, nz) | key_direction(kp, ox, oy, oz, has_rough, rough, ok);
  key = key_at(kp, px, py, pz, lvl, hi, ovf);
  return ok != 0;
}

// ------------------------------------------------------------------ state encodings
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f, bool& sat) {
  (void)sat;
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

__device__ __forceinline__ float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

__device__ __forceinline__ uint32_t f32_to_f16_rne(float f, bool& sat) {
  if (fabsf(f) > 65504.0f) {
    sat = true;
    f = f > 0.0f ? 65504.0f : -65504.0f;
  }
  _Float16 h = (_Float16)f;  // v_cvt_f16_f32, round to nearest even
  return (uint32_t)__builtin_bit_cast(uint16_t, h);
}

__device__ __forceinline__ float f16_to_f32(uint32_t h) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

// State formats: 0 binary32; 1 binary16 and 2 bfloat16, each re-rounded by
// every blend; 3 and 4 the same 16-bit values plus each channel's binary32
// rounding residual (value - stored 16-bit value, exact) kept in the slot's
// otherwise unused words, so that the blend continues from the unrounded
// binary32 state and a lookup sees a single rounding.
__device__ __forceinline__ bool state_is_f16(int32_t dtype) { return dtype == 1 || dtype == 3; }
__device__ __forceinline__ bool state_has_residual(int32_t dtype) { return dtype >= 3; }

// The three 16-bit values of a slot's first two state words.
__device__ __forceinline__ void decode16(uint32_t w0, uint32_t w1, int32_t dtype, float& r, float& g, float& b) {
  if (state_is_f16(dtype)) {
    r = f16_to_f32(w0 & 0xffffu);
    g = f16_to_f32(w0 >> 16);
    b = f16_to_f32(w1 & 0xffffu);
  } else {
    r = bf16_to_f32(w0 & 0xffffu);
    g = bf16_to_f32(w0 >> 16);
    b = bf16_to_f32(w1 & 0xffffu);
  }
}

// The approximant a lookup returns.
__device__ __forceinline__ void load_state(const Slot& s, int32_t dtype, float& r, float& g, float& b) {
  // (words first: selected by address, a slot held in registers would go
  // through scratch memory)
  const uint32_t w0 = s.L[0], w1 = s.L[1], w2 = s.L[2];
  decode16(w0, w1, dtype, r, g, b);
  if (dtype == 0) {
    r = __uint_as_float(w0);
    g = __uint_as_float(w1);
    b = __uint_as_float(w2);
  }
}

// The state the blend continues from: the lookup value, plus the carried
// residual in formats 3 and 4.
__device__ __forceinline__ void load_blend_state(const Slot& s, int32_t dtype, float& r, float& g, float& b) {
  load_state(s, dtype, r, g, b);
  if (state_has_residual(dtype)) {
    r = r + __uint_as_float(s.L[2]);
    g = g + __uint_as_float(s.L[3]);
    b = b + __uint_as_float(s.pad);
  }
}

// Encode a blended value: out[0..3] become Slot::L, *pad Slot::pad.
__device__ __forceinline__ void encode_state(int32_t dtype, float r, float g, float b, uint32_t out[4],
                                             uint32_t& pad, bool& sat) {
  pad = 0u;
  if (dtype == 0) {
    out[0] = __float_as_uint(r);
    out[1] = __float_as_uint(g);
    out[2] = __float_as_uint(b);
    out[3] = 0u;
    return;
  }
  const bool f16 = state_is_f16(dtype);
  const uint32_t hr = f16 ? f32_to_f16_rne(r, sat) : f32_to_bf16_rne(r, sat);
  const uint32_t hg = f16 ? f32_to_f16_rne(g, sat) : f32_to_bf16_rne(g, sat);
  const uint32_t hb = f16 ? f32_to_f16_rne(b, sat) : f32_to_bf16_rne(b, sat);
  out[0] = hr | (hg << 16);
  out[1] = hb;
  out[2] = 0u;
  out[3] = 0u;
  if (state_has_residual(dtype)) {
    // value - stored value: exact in binary32 (the two are within one
    // 16-bit ulp of each other), except past F16 saturation, where the
    // difference itself rounds
    const float sr = f16 ? f16_to_f32(hr) : bf16_to_f32(hr);
    const float sg = f16 ? f16_to_f32(hg) : bf16_to_f32(hg);
    const float sb = f16 ? f16_to_f32(hb) : bf16_to_f32(hb);
    out[2] = __float_as_uint(r - sr);
    out[3] = __float_as_uint(g - sg);
    pad = __float_as_uint(b - sb);
  }
}

// Lookup of one key (kEmpty = rejected record): the approximant if the cell
// exists and has been blended (c_old > 0), else zeros.  Returns the hit flag.
__device__ __forceinline__ uint8_t lookup_key(const TableView& tv, int32_t dtype, uint64_t key,
                                              float rgb[3]) {
  rgb[0] = rgb[1] = rgb[2] = 0.0f;
  if (key == kEmpty) return 0;
  const ProbeSeq ps = probe_seq(key, tv.log2_slots, tv.part_log2);
  for (uint32_t j = 0; j < tv.max_probe; ++j) {
    const Slot sl = tv.slots[ps.at(j)];
    if (sl.key == key) {
      if (sl.c_old == 0) return 0;
      load_state(sl, dtype, rgb[0], rgb[1], rgb[2]);
      return 1;
    }
    if (sl.key == kEmpty) return 0;
  }
  return 0;
}

// The same lookup split in two, so that the first probes of several
// lookups can be in flight together: lookup_first issues the load of the
// key's first slot (any key, also kEmpty: the slot is then ignored),
// lookup_finish resolves it and probes further only if needed.
struct PendingLookup {
  uint64_t key;
  ProbeSeq ps;
  Slot first;
};

__device__ __forceinline__ PendingLookup lookup_first(const TableView& tv, uint64_t key) {
  PendingLookup l;
  l.key = key;
  l.ps = probe_seq(key, tv.log2_slots, tv.part_log2);
  l.first = tv.slots[l.ps.at(0)];
  return l;
}

__device__ __forceinline__ uint8_t lookup_finish(const TableView& tv, int32_t dtype, const PendingLookup& l,
                                                 float rgb[3]) {
  rgb[0] = rgb[1] = rgb[2] = 0.0f;
  if (l.key == kEmpty) return 0;
  Slot sl = l.first;
  for (uint32_t j = 0;;) {
    if (sl.key == l.key) {
      if (sl.c_old == 0) return 0;
      load_state(sl, dtype, rgb[0], rgb[1], rgb[2]);
      return 1;
    }
    if (sl.key == kEmpty || ++j >= tv.max_probe) return 0;
    sl = tv.slots[l.ps.at(j)];
  }
}

// A value a pass reads once, and one it writes that no kernel of the pass
// reads: non-temporal, so streaming them does not evict from the caches the
// table the pass gathers from.
__device__ __forceinline__ float ld_once(const float* p) { return __builtin_nontemporal_load(p); }
// (p wave-uniform, i < 2^30: a scalar address and a 32-bit offset)
__device__ __forceinline__ float ld_once_at(const float* p, uint32_t i) {
  return __builtin_nontemporal_load(reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + (i << 2)));
}
__device__ __forceinline__ void st_once(float* p, float v) { __builtin_nontemporal_store(v, p); }

// One vertex of a structure-of-arrays query set: element i of the arrays
// from a wave-uniform start on (arrays the caller left out read as 0).  The
// loads that every vertex needs are all issued before the first wait: under
// the key's conditions they would be one dependent round trip after another.
// The roughness comes first, and the direction, 12 of 40 bytes, only where it
// makes the vertex glossy, while the others are on their way (3,686,400
// lookups at diffuse vertices 81.0 -> 73.6 us, with a quarter glossy 79.3 and
// 80.1).
struct Vertex {
  float p[3], n[3], o[3], rough, fp;
};

// The direction (x, y, z) of a vertex of roughness rough, in a table of
// threshold thr (+inf: keyed on the direction everywhere); +z, whose bin costs
// a wave nothing beyond the others', where it is not glossy.
__device__ __forceinline__ void load_direction(const float* x, const float* y, const float* z, uint64_t start,
                                               uint32_t i, float rough, float thr, float o[3]) {
  o[0] = o[1] = 0.0f;
  o[2] = 1.0f;
  if (thr > 3.402823466e38f || rough < thr) {  // (the first test is wave-uniform)
    o[0] = ld_once_at(x + start, i);
    o[1] = ld_once_at(y + start, i);
    o[2] = ld_once_at(z + start, i);
  }
}

// All but the direction, which load_vertex_direction adds once everything
// else that the caller loads is on its way.
template <class Q>
__device__ __forceinline__ Vertex load_vertex(const Q& q, uint64_t start, uint32_t i) {
  const bool hr = q.rough != nullptr, hf = q.footprint != nullptr;
  Vertex v;
  v.o[0] = v.o[1] = v.o[2] = v.rough = v.fp = 0.0f;
  if (hr) v.rough = ld_once_at(q.rough + start, i);
  v.p[0] = ld_once_at(q.px + start, i);
  v.p[1] = ld_once_at(q.py + start, i);
  v.p[2] = ld_once_at(q.pz + start, i);
  v.n[0] = ld_once_at(q.nx + start, i);
  v.n[1] = ld_once_at(q.ny + start, i);
  v.n[2] = ld_once_at(q.nz + start, i);
  if (hf) v.fp = ld_once_at(q.footprint + start, i);
  return v;
}
template <class Q>
__device__ __forceinline__ void load_vertex_direction(const Q& q, float thr, uint64_t start, uint32_t i, Vertex& v) {
  if (q.rough) load_direction(q.ox, q.oy, q.oz, start, i, v.rough, thr, v.o);
}

// (an empty statement that uses the values, so their loads issue before it)
__device__ __forceinline__ void loaded(const Vertex& v) {
  asm volatile("" : : "v"(v.p[0]), "v"(v.p[1]), "v"(v.p[2]), "v"(v.n[0]), "v"(v.n[1]), "v"(v.n[2]));
  asm volatile("" : : "v"(v.o[0]), "v"(v.o[1]), "v"(v.o[2]), "v"(v.rough), "v"(v.fp));
}

// Key of a loaded vertex (kEmpty if rejected).
template <class Q>
__device__ __forceinline__ uint64_t vertex_key(const KeyParams& kp, const Q& q, const Vertex& v) {
  uint64_t key;
  bool ovf;
  const bool ok = cell_key(kp, v.p[0], v.p[1], v.p[2], v.n[0], v.n[1], v.n[2], v.o[0], v.o[1], v.o[2],
                           q.rough != nullptr, v.rough, q.footprint != nullptr, v.fp, key, ovf);
  return ok ? key : kEmpty;
}

// Block order of the lookup passes.  Blocks are dispatched to the 8 XCDs
// round-robin; each XCD takes 64 consecutive blocks of every 512, so that
// the cells neighbouring scanlines share are fetched into one L2 (the last,
// incomplete group keeps the launch order).  With the loads in one round
// trip: lookup of 2,073,600 first vertices with fallback levels 46.0 -> 36.8
// us, estimates at 3,686,400 vertices 188 -> 159 us, 2,073,600 lookups at
// scattered vertices 51.6 -> 49.8 us (those wait on the misses of their
// slots).
__device__ __forceinline__ uint32_t xcd_order(uint32_t b, uint32_t blocks) {
  const uint32_t g = b & ~511u, r = b & 511u;
  return g + 512 <= blocks ? g + (r & 7u) * 64 + (r >> 3) : b;
}

// Eq. 10-11 for one cell, FP32, on counter words (counts, or weight sums
// in a weighted table).  n > 0.
__device__ __forceinline__ float blend_alpha(const BlendParams& bp, uint32_t n, uint32_t c_old, bool wtd) {
  if (bp.mode == 1) return c_old == 0 ? 1.0f : bp.alpha;
  const float nf = counter_value(n, wtd);
  const float ratio = nf / (counter_value(c_old, wtd) + nf);
  if (bp.mode == 2) return ratio;
  return fmaxf(sqrtf(ratio), bp.inv_t_max);
}

}  // namespace psf
