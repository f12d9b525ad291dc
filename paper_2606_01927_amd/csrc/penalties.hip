// penalties.hip -- albireo_apply_penalties: the penalty step alone (the feature list of sec. 8.1), its
// result written out as fp32 logits.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <utility>

#include "albireo.h"
#include "penalties.h"

namespace {

#include "common.h"

constexpr int PEN_NT = 256;
constexpr int PEN_G = 8;                           // groups of four elements per thread
constexpr int PEN_TILE = PEN_NT * PEN_G * 4;       // elements per workgroup (32 KB of LDS words)
constexpr int PEN_IDS = 8;                         // history ids in flight per thread

struct PenArgs {
  const unsigned char* logits;
  int64_t V, ld;
  DevParams prm;
  // the prompt history (repetition only) and the per-sequence penalty state, beside the output history
  const int64_t* prompt_offsets;
  const int32_t* prompt_ids;
  int64_t prompt_len;
  const int32_t* st_ids;
  const uint32_t* st_counts;
  const int32_t* st_len;
  int32_t st_cap;
  float* out;
};

struct alignas(16) F4 {
  float v[4];
};

// Four consecutive logits from an address aligned to the element only (one 8- or 16-byte load: gfx950
// takes unaligned vector loads; a row whose length is odd leaves most rows unaligned).
template <class DT>
__device__ __forceinline__ F4 load4(const unsigned char* p) {
  F4 r;
  if constexpr (DT::ES == 2) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2), aligned(2)));
    const u2 d = *reinterpret_cast<const u2*>(p);
    r.v[0] = __uint_as_float(d.x << 16);
    r.v[1] = __uint_as_float(d.x & 0xffff0000u);
    r.v[2] = __uint_as_float(d.y << 16);
    r.v[3] = __uint_as_float(d.y & 0xffff0000u);
  } else {
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    const f4 d = *reinterpret_cast<const f4*>(p);
    r.v[0] = d.x;
    r.v[1] = d.y;
    r.v[2] = d.z;
    r.v[3] = d.w;
  }
  return r;
}

// f(id, index) for the ids [lo, hi) of an array, PEN_IDS loads per thread in flight before any is used
// (unconditional: an index past the range reloads the first of the group)
template <class F>
__device__ __forceinline__ void for_ids(const int32_t* ids, int64_t lo, int64_t hi, F&& f) {
  for (int64_t h0 = lo + threadIdx.x; h0 < hi; h0 += (int64_t)PEN_IDS * PEN_NT) {
    int32_t v[PEN_IDS];
#pragma unroll
    for (int q = 0; q < PEN_IDS; ++q) {
      const int64_t h = h0 + (int64_t)q * PEN_NT;
      v[q] = ids[h < hi ? h : h0];
    }
#pragma unroll
    for (int q = 0; q < PEN_IDS; ++q) {
      const int64_t h = h0 + (int64_t)q * PEN_NT;
      if (h < hi) f(v[q], h);
    }
  }
}

// One tile of one row per workgroup.  Tiles start at the row's first output element on a 16-byte
// boundary (tile 0 also takes the up to three elements before it), so every store but the row's ends is
// a 16-byte one whatever V is; the loads of those elements are as wide, unaligned where the row is.
// Every id of the row's output history, prompt history or penalty state that falls in the tile is
// folded into a 32-bit LDS word per element (bits 0-30 the output count, bit 31 the prompt mark: the
// penalty state's encoding), exact for any history length; the words are read back four at a time
// beside the elements.  Each element is read and written by the same thread, so the output may alias
// an fp32 input.
//
// Bound: HBM (the input once, the fp32 output once).  The tile's elements are requested before its
// history is scanned, so the scan runs under them; 32 KB of LDS leaves five workgroups per CU.
// 64 rows of 152064 bf16 logits, 2048 ids each: 54.9 us with 2- and 4-byte accesses and a tile of 64 KB,
// 14.5 us now (4.1 TB/s; a large copy reaches 4.8).
template <class DT>
__global__ __launch_bounds__(PEN_NT) void k_penalties(PenArgs a) {
  __shared__ __align__(16) uint32_t cvs[PEN_TILE + 4];  // word i + 4: element t0 + i
  const int t = threadIdx.x;
  const int64_t row = blockIdx.y;
  const unsigned char* rowp = a.logits + row * a.ld * DT::ES;
  float* orow = a.out + row * a.V;
  int head = (int)(((16u - (uint32_t)(reinterpret_cast<uintptr_t>(orow) & 15u)) & 15u) / 4u);
  if (head > a.V) head = (int)a.V;
  const int64_t t0 = head + (int64_t)blockIdx.x * PEN_TILE;  // the tile: [t0, t1), and the head in tile 0
  const int64_t t1 = min(a.V, t0 + PEN_TILE);
  const int ng = t1 > t0 ? (int)((t1 - t0) / 4) : 0;         // whole groups; the rest one by one
  const int rest = t1 > t0 ? (int)(t1 - t0) - 4 * ng : 0;
  const bool first = blockIdx.x == 0;

  F4 x[PEN_G] = {};
  if (ng > 0) {  // every load in flight at once (a group past the last reloads the last)
    static_for<PEN_G>([&](auto J) {
      constexpr int j = decltype(J)::value;
      x[j] = load4<DT>(rowp + (t0 + 4 * (int64_t)min(j * PEN_NT + t, ng - 1)) * DT::ES);
    });
  }
  // the elements outside the groups: threads 0-2 the head (tile 0), 4-6 the rest of the last tile
  int64_t xi = -1;
  if (first && t < head) xi = t;
  else if (t >= 4 && t - 4 < rest) xi = t0 + 4 * (int64_t)ng + (t - 4);
  const float xe = xi >= 0 ? DT::load1(rowp, xi) : 0.0f;

  const DevParams& q = a.prm;
  float rep = sload(q.rep ? q.rep + row : &kParamDefaults[3]);
  float freq = sload(q.freq ? q.freq + row : &kParamDefaults[4]);
  float pres = sload(q.pres ? q.pres + row : &kParamDefaults[5]);
  if (!(rep > 0.0f) || isinf(rep)) rep = 1.0f;
  if (!isfinite(freq)) freq = 0.0f;
  if (!isfinite(pres)) pres = 0.0f;
  int64_t lo = 0, hi = 0, plo = 0, phi = 0;
  if (q.hist_offsets) {
    lo = sload(q.hist_offsets + row);
    hi = sload(q.hist_offsets + row + 1);
    if (lo < 0 || hi < lo || hi > q.hist_len) lo = hi = 0;
  }
  if (a.prompt_offsets) {
    plo = sload(a.prompt_offsets + row);
    phi = sload(a.prompt_offsets + row + 1);
    if (plo < 0 || phi < plo || phi > a.prompt_len) plo = phi = 0;
  }
  int sn = 0;
  if (a.st_len) {
    sn = sload(a.st_len + row);
    sn = sn < 0 ? 0 : (sn > a.st_cap ? a.st_cap : sn);
  }
  const bool pen = hi > lo || phi > plo || sn > 0;
  const int64_t base = t0 - 4;  // element of LDS word 0
  if (pen) {
    uint4* c4 = reinterpret_cast<uint4*>(cvs);
    for (int i = t; i < PEN_TILE / 4 + 1; i += PEN_NT) c4[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const int64_t e0 = first ? 0 : t0;
    for_ids(q.hist_ids, lo, hi, [&](int32_t id, int64_t) __attribute__((always_inline)) {
      if (id >= e0 && id < t1) atomicAdd(&cvs[id - base], 1u);
    });
    for_ids(a.prompt_ids, plo, phi, [&](int32_t id, int64_t) __attribute__((always_inline)) {
      if (id >= e0 && id < t1) atomicOr(&cvs[id - base], 0x80000000u);
    });
    const int32_t* si = a.st_ids + row * a.st_cap;
    const uint32_t* sc = a.st_counts + row * a.st_cap;
    for_ids(si, 0, sn, [&](int32_t id, int64_t e) __attribute__((always_inline)) {
      if (id >= e0 && id < t1) cvs[id - base] = sc[e];  // distinct ids
    });
    __syncthreads();
  }
  static_for<PEN_G>([&](auto J) {
    constexpr int j = decltype(J)::value;
    const int g = j * PEN_NT + t;
    if (g < ng) {
      if (pen) {
        const uint4 c = reinterpret_cast<const uint4*>(cvs)[g + 1];
        if (c.x | c.y | c.z | c.w) {
          if (c.x) x[j].v[0] = penalise_cv(x[j].v[0], c.x, rep, freq, pres);
          if (c.y) x[j].v[1] = penalise_cv(x[j].v[1], c.y, rep, freq, pres);
          if (c.z) x[j].v[2] = penalise_cv(x[j].v[2], c.z, rep, freq, pres);
          if (c.w) x[j].v[3] = penalise_cv(x[j].v[3], c.w, rep, freq, pres);
        }
      }
      *reinterpret_cast<F4*>(orow + t0 + 4 * (int64_t)g) = x[j];
    }
  });
  if (xi >= 0) {
    float v = xe;
    if (pen) {
      const uint32_t c = cvs[xi - base];
      if (c) v = penalise_cv(v, c, rep, freq, pres);
    }
    orow[xi] = v;
  }
}

}  // namespace

namespace albireo_penalties {

albireo_status_t launch(const void* logits, albireo_dtype_t dtype, int64_t B, int64_t V, int64_t ld,
                        const albireo_params_t* p, float* out, hipStream_t stream) {
  PenArgs a;
  memset(&a, 0, sizeof a);
  a.logits = static_cast<const unsigned char*>(logits);
  a.V = V;
  a.ld = ld;
  a.out = out;
  if (p) {
    a.prm.rep = p->repetition_penalty;
    a.prm.freq = p->frequency_penalty;
    a.prm.pres = p->presence_penalty;
    a.prm.hist_offsets = p->hist_offsets;
    a.prm.hist_ids = p->hist_ids;
    a.prm.hist_len = p->hist_len;
    a.prompt_offsets = p->prompt_offsets;
    a.prompt_ids = p->prompt_ids;
    a.prompt_len = p->prompt_len;
    if (p->state) {
      a.st_ids = p->state->ids;
      a.st_counts = p->state->counts;
      a.st_len = p->state->len;
      a.st_cap = p->state->cap;
    }
  }
  const dim3 grid((unsigned)((V + PEN_TILE - 1) / PEN_TILE), (unsigned)B);
  if (dtype == ALBIREO_BF16) hipLaunchKernelGGL(k_penalties<BF16T>, grid, dim3(PEN_NT), 0, stream, a);
  else hipLaunchKernelGGL(k_penalties<F32T>, grid, dim3(PEN_NT), 0, stream, a);
  return hipGetLastError() == hipSuccess ? ALBIREO_OK : ALBIREO_E_LAUNCH;
}

}  // namespace albireo_penalties
