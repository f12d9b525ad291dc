// filter.hip -- the filtered distribution of fp32 logits (albireo_topk_topp): temperature, {top-k, min-p},
// top-p over their kept set, and the renormalised probabilities written out.
//
// A row is cut into chunks of at most CSLOTS 16-byte slots; four launches on the caller's stream:
//   k_filter_hist  (per chunk): the chunk's maximum, and a histogram of the values over their distance below
//     it -- counts where the kept set is bounded by top-k or min-p, fixed-point weights where top-p alone
//     decides it;
//   k_filter_stage (per chunk): merges the row's histograms to the bucket that holds the cut, stages that
//     bucket's values (or, where two filters combine, every value down to it) and sums the weights above;
//   k_filter_solve (per row): the exact cut among the staged values, the kept count, minimum and mass;
//   k_filter_write (per chunk): the probabilities; it also zeroes the chunk's workspace.
// Buckets are floor(32 z), absolute, so that chunks with different maxima share them: chunk histograms are
// merged by shifting, with no pass for the row maximum first.
//
// Bound: HBM for the first read and the written probabilities (the second and third read come from the
// caches); what is left is the four launches' ramps.  Splitting each row over its chunks is what the
// one-launch kernels cannot do without waiting for each other.  64 rows of 128256 logits, top-k and top-p
// mixed: 419-429 us in one cooperative launch of two workgroups per row, 52 us here (13 us the
// histograms, 17 the staging, 11 the cuts, 12 the writing).  Rows whose staging overflows are selected over
// memory by the third launch's one workgroup per row: 64 x 128256 flat rows with top-k 9000 and top-p 385 us (837 in
// the cooperative kernel), min-p 0.001 and top-p 240 (565), one value throughout 559 (677).
#include <hip/hip_runtime.h>

#include <float.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>
#include <utility>

#include "albireo.h"
#include "filter.h"

namespace {

#include "common.h"

constexpr int CT = 512;           // threads of a chunk workgroup: with 256, 64 rows of 7 chunks put 7 waves on a CU
constexpr int NWV = CT / 64;
constexpr int CSLOTS = 4864;      // the streaming route's chunks, so that its workspace has room for these
constexpr int CJ = (CSLOTS + CT - 1) / CT;  // slots per thread, all requested before any is used
constexpr int NB = 1024;          // histogram buckets
constexpr float BSCALE = 32.0f;   // buckets per unit of z
constexpr int LC = 1024;          // values staged per chunk
constexpr int CAP = 4096;         // values staged per row
constexpr int MAXPC = 64;         // chunks per row (one per lane)
constexpr int ST = 512;           // threads of a row's solving workgroup
constexpr int REC = 8;            // 64-bit words per chunk record
constexpr float MAX_M = 1e36f;    // above, 32 z may overflow: selected over memory
constexpr double FIX44 = 17592186044416.0;

// What decides a row's cut (record word 5 of chunk 0, with the bucket above it).
enum Kind : int { K_NONE = 0, K_COUNT = 1, K_MASS = 2, K_ALL = 3, K_SLOW = 4 };

struct FArgs {
  const float* logits;
  int64_t B, V, ld;
  const float* temperature;
  const int32_t* top_k;
  const float* top_p;
  const float* min_p;
  float* out_probs;
  float* out_threshold;
  int32_t* out_kept;
  float* out_log_norm;
  uint32_t* out_flags;
  int32_t P;
  int64_t chunk_slots;
  uint64_t* rec;    // [B * P * REC]
  uint32_t* lists;  // [B * P * LC] staged order keys
  uint64_t* hist;   // [B * P * NB]
};

struct Row {
  const float* x;
  int V, slots;  // 16-byte slots; the up to three values behind them belong to the last chunk
  bool greedy, kon, minp_on, topp_on, top_group;
  float r, p, minp;
  int k;
  uint32_t flags;
};
// which histogram the row's first pass takes
enum Hist : int { H_NONE = 0, H_COUNT = 1, H_MASS = 2 };

__device__ __forceinline__ void row_setup(const FArgs& a, int64_t row, Row& R) {
  R.x = a.logits + row * a.ld;
  R.V = (int)a.V;
  R.slots = R.V / 4;
  float T = sload(a.temperature ? a.temperature + row : &kParamDefaults[0]);
  float p = sload(a.top_p ? a.top_p + row : &kParamDefaults[1]);
  float mp = sload(a.min_p ? a.min_p + row : &kParamDefaults[2]);
  R.k = sload(a.top_k ? a.top_k + row : &kZeroI32[0]);
  uint32_t flags = 0;
  if (!isfinite(T)) { flags |= FLAG_BAD_PARAM; T = 1.0f; }
  if (isnan(p)) { flags |= FLAG_BAD_PARAM; p = 1.0f; }
  if (isnan(mp)) { flags |= FLAG_BAD_PARAM; mp = 0.0f; }
  R.greedy = T < 1e-5f;
  if (R.greedy) flags |= FLAG_GREEDY;
  R.r = R.greedy ? 1.0f : (float)(1.0 / (double)T);
  R.kon = !R.greedy && R.k > 0 && (int64_t)R.k < a.V;
  R.minp_on = !R.greedy && mp > 0.0f;
  R.minp = mp > 1.0f ? 1.0f : mp;
  R.topp_on = !R.greedy && p < 1.0f;
  R.top_group = R.topp_on && !(p > 0.0f);  // p <= 0 keeps the values equal to the maximum
  R.p = p;
  R.flags = flags;
}
__device__ __forceinline__ Hist hist_of(const Row& R) {
  if (R.greedy || R.top_group) return H_NONE;
  if (R.kon || (R.minp_on && R.topp_on)) return H_COUNT;
  return R.topp_on ? H_MASS : H_NONE;
}

// 16 bytes at any 4-byte boundary (rows start where the caller's stride puts them)
struct __attribute__((packed, aligned(4))) F4 {
  float v[4];
};

// The chunk's slots [s0, s1), slot j * CT + t of the chunk to thread t, and the row's last V % 4 values, one
// to a thread of the last chunk; unused places are -inf.  tail: this thread's tail position or -1.
struct ChunkAt {
  int s0, ns, tail;
};
__device__ __forceinline__ ChunkAt chunk_at(const FArgs& a, const Row& R, int c) {
  ChunkAt q;
  const int64_t s0 = min((int64_t)c * a.chunk_slots, (int64_t)R.slots);
  q.s0 = (int)s0;
  q.ns = (int)(min(s0 + a.chunk_slots, (int64_t)R.slots) - s0);
  q.tail = -1;
  if (c == a.P - 1 && (int)threadIdx.x < R.V - R.slots * 4) q.tail = R.slots * 4 + (int)threadIdx.x;
  return q;
}
__device__ __forceinline__ void load_slots(const Row& R, const ChunkAt& q, F4 (&d)[CJ]) {
#pragma unroll
  for (int j = 0; j < CJ; ++j)
    if (q.ns > 0) d[j] = *reinterpret_cast<const F4*>(R.x + ((int64_t)q.s0 + min(j * CT + (int)threadIdx.x, q.ns - 1)) * 4);
}
// the loaded values as processed logits, places past the chunk -inf
__device__ __forceinline__ void process_slots(const Row& R, const ChunkAt& q, F4 (&d)[CJ]) {
#pragma unroll
  for (int j = 0; j < CJ; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      d[j].v[e] = j * CT + (int)threadIdx.x < q.ns ? canon(d[j].v[e], R.r) : -INFINITY;
}

__device__ __forceinline__ float qfloor(float z) { return floorf(z * BSCALE); }
// bucket of z below the bucket number qtop of a maximum; the last one takes everything further down
__device__ __forceinline__ int bucket(float qtop, float z) { return (int)fminf(qtop - qfloor(z), (float)(NB - 1)); }

// Weight of z <= m against the maximum m in units of 2^-32, rounded down: from the difference, so that it
// holds at any magnitude of m.  At z == m the conversion saturates, one unit short of 2^32 (in 64 bits
// 64 x 128256 rows with top-p alone took 45.9 us against 45.6).
__device__ __forceinline__ uint32_t fix_weight(float z, float m) {
  const float w = __builtin_amdgcn_exp2f(__fmul_rn(__fsub_rn(z, m), L2E)) * 4294967296.0f;
  uint32_t u;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(u) : "v"(w));
  return u;
}
// The smallest z in the buckets up to b below qtop: bucket(z) <= b is 32 z >= qtop - b exactly, but past 2^24
// that difference is no float, so it is taken in double and rounded up.  (Bucket numbers near the maximum
// differ exactly at any magnitude; further away any rounding stays past the last bucket.)
__device__ __forceinline__ float bucket_edge(float qtop, int b) {
  const double x = ((double)qtop - (double)b) / (double)BSCALE;
  const float f = (float)x;
  return (double)f < x ? key2f(f2key(f) + 1u) : f;
}

// ----------------------------------------------------------------------------------------------
// Pass 1.  Record: word 0 = maximum | (NaN seen) << 32, word 1 = lowest position of the maximum (greedy).
// ----------------------------------------------------------------------------------------------
__global__ __launch_bounds__(CT, 4) void k_filter_hist(FArgs a) {
  __shared__ uint64_t h[NB];
  __shared__ float wmx[NWV], wlow[NWV];
  __shared__ int wbad[NWV], wpos[NWV];
  const int t = threadIdx.x;
  const int64_t L = blockIdx.x, row = L / a.P;
  const int c = (int)(L - row * a.P);
  Row R;
  row_setup(a, row, R);
  const ChunkAt q = chunk_at(a, R, c);
  F4 d[CJ];
  load_slots(R, q, d);
  const float zt = q.tail >= 0 ? canon(R.x[q.tail], R.r) : -INFINITY;
  for (int b = t; b < NB; b += CT) h[b] = 0;
  process_slots(R, q, d);
  float mx = zt;
  bool bad = zt != zt;
#pragma unroll
  for (int j = 0; j < CJ; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      mx = fmaxf(mx, d[j].v[e]);
      bad = bad || d[j].v[e] != d[j].v[e];
    }
  const float wm = wave_max(mx);
  const uint64_t anybad = __ballot(bad);
  if (lane_id() == 0) {
    wmx[wave_id()] = wm;
    wbad[wave_id()] = anybad != 0;
  }
  __syncthreads();
  float cm = wmx[0];
#pragma unroll
  for (int w = 1; w < NWV; ++w) cm = fmaxf(cm, wmx[w]);
  if (R.greedy) {
    int pos = INT32_MAX;
#pragma unroll
    for (int j = 0; j < CJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (d[j].v[e] == cm) pos = min(pos, (q.s0 + j * CT + t) * 4 + e);
    if (q.tail >= 0 && zt == cm) pos = min(pos, q.tail);
    pos = wave_min_i(pos);
    if (lane_id() == 0) wpos[wave_id()] = pos;
  }
  const Hist ht = hist_of(R);
  const bool finite = cm > -INFINITY && cm < INFINITY;
  if (ht != H_NONE && finite) {
    const float qtop = qfloor(cm);
    // Values below low move no cut: those under a bound of the chunk's k-th largest value (at most the row's),
    // those more than log min-p below the chunk's maximum, and those whose weight is 0 in units of 2^-32.
    // The LDS adds bound this pass (64 rows of 128256: 20 us with all of them), and these are most of them.
    float low = -FLT_MAX;
    if (ht == H_MASS) {
      low = cm - 22.5f;  // e^-22.5 < 2^-32
    } else if (R.kon) {
      // each wave holds at least rk values at or above its rk-th largest thread maximum, all waves k of them
      const int rk = (R.k + NWV - 1) / NWV;
      if (rk <= 64) {
        float v = mx, at = -INFINITY;
        for (int i = 0; i < rk; ++i) {
          at = wave_max(v);
          const uint64_t hit = __ballot(v == at);
          if (hit != 0 && lane_id() == (int)__builtin_ctzll(hit)) v = -INFINITY;
        }
        if (lane_id() == 0) wlow[wave_id()] = at;
        __syncthreads();
        float lo = wlow[0];
#pragma unroll
        for (int w = 1; w < NWV; ++w) lo = fminf(lo, wlow[w]);
        low = fmaxf(low, lo);
      }
    } else {
      low = fmaxf(low, __fadd_rn(cm, (float)log((double)R.minp)) - 1.0f / BSCALE);
    }
    auto add = [&](float z) __attribute__((always_inline)) {
      if (z >= low) {
        const uint32_t u = ht == H_MASS ? fix_weight(z, cm) : 1u;
        atomicAdd((unsigned long long*)&h[bucket(qtop, z)], (unsigned long long)u);
      }
    };
    if (anybad == 0) {  // a NaN has no bucket; its row's outputs do not come from the histogram
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        if (j * CT < q.ns) {  // uniform
#pragma unroll
          for (int e = 0; e < 4; ++e) add(d[j].v[e]);
        }
      }
      if (q.tail >= 0) add(zt);
    }
  }
  __syncthreads();
  if (ht != H_NONE)
    for (int b = t; b < NB; b += CT) a.hist[L * NB + b] = h[b];
  if (t == 0) {
    int nan = 0, pos = INT32_MAX;
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      nan |= wbad[w];
      if (R.greedy) pos = min(pos, wpos[w]);
    }
    a.rec[L * REC + 0] = ((uint64_t)(uint32_t)nan << 32) | __float_as_uint(cm);
    a.rec[L * REC + 1] = R.greedy ? (uint64_t)(uint32_t)pos : 0ull;
  }
}

// The row's maximum and state from its chunk records (uniform; the same in every workgroup of the row)
struct RowMax {
  float m, tau_m;
  bool empty, bad;
};
__device__ __forceinline__ RowMax row_max(const FArgs& a, const Row& R, int64_t row) {
  RowMax x{-INFINITY, -INFINITY, false, false};
  // lane i of every wave takes chunk i (at most 64)
  const uint64_t w = a.rec[(row * a.P + min(lane_id(), a.P - 1)) * REC];
  x.m = wave_max(__uint_as_float((uint32_t)w));
  const uint32_t nan = wave_or((uint32_t)(w >> 32));
  x.empty = !(x.m > -INFINITY);
  x.bad = nan != 0 || x.m == INFINITY;
  if (R.minp_on) x.tau_m = __fadd_rn(x.m, (float)log((double)R.minp));
  if (R.top_group) x.tau_m = x.m;
  return x;
}

__device__ __forceinline__ uint64_t wave_incl_scan_u64(uint64_t v) {
  v += dpp_mov64<DPP_ROW_SHR + 1>(v);
  v += dpp_mov64<DPP_ROW_SHR + 2>(v);
  v += dpp_mov64<DPP_ROW_SHR + 4>(v);
  v += dpp_mov64<DPP_ROW_SHR + 8>(v);
  v += dpp_mov64<DPP_ROW_BCAST15, 0xa>(v);
  v += dpp_mov64<DPP_ROW_BCAST31, 0xc>(v);
  return v;
}
__device__ __forceinline__ double wave_scan_f64(double v) {
  auto add = [](double a, uint64_t b) { return a + __longlong_as_double((long long)b); };
  v = add(v, dpp_mov64<DPP_ROW_SHR + 1>((uint64_t)__double_as_longlong(v)));
  v = add(v, dpp_mov64<DPP_ROW_SHR + 2>((uint64_t)__double_as_longlong(v)));
  v = add(v, dpp_mov64<DPP_ROW_SHR + 4>((uint64_t)__double_as_longlong(v)));
  v = add(v, dpp_mov64<DPP_ROW_SHR + 8>((uint64_t)__double_as_longlong(v)));
  v = add(v, dpp_mov64<DPP_ROW_BCAST15, 0xa>((uint64_t)__double_as_longlong(v)));
  v = add(v, dpp_mov64<DPP_ROW_BCAST31, 0xc>((uint64_t)__double_as_longlong(v)));
  return v;
}

// ----------------------------------------------------------------------------------------------
// Pass 2.  Record: word 2 = values staged, word 3 = weight of the values kept whatever the cut in the
// bucket, word 4 = their number << 32 | order key of their minimum (0 without any); chunk 0 also word 5 =
// kind | bucket << 8, word 6 = what lies above the bucket, word 7 = the row's total.
// ----------------------------------------------------------------------------------------------
struct Cross {
  int b;           // crossing bucket, NB when the target is never reached
  uint64_t above;  // sum of the buckets above it
  uint64_t upto;   // and with it
};

__global__ __launch_bounds__(CT, 4) void k_filter_stage(FArgs a) {
  constexpr int BPT = NB / CT;
  __shared__ double wsum[NWV];
  __shared__ uint64_t wtot[NWV];
  __shared__ Cross cx;
  __shared__ int n_list;
  __shared__ int wcnt[NWV];
  __shared__ uint32_t wmin[NWV];
  __shared__ double cscale[MAXPC];
  __shared__ int coff[MAXPC];
  const int t = threadIdx.x;
  const int64_t L = blockIdx.x, row = L / a.P;
  const int c = (int)(L - row * a.P);
  Row R;
  row_setup(a, row, R);
  const ChunkAt q = chunk_at(a, R, c);
  F4 d[CJ];
  load_slots(R, q, d);  // in flight while the histograms are merged
  const float xt = q.tail >= 0 ? R.x[q.tail] : 0.0f;
  const RowMax X = row_max(a, R, row);
  if (R.greedy || X.empty || X.bad) return;  // uniform; nothing to select
  const float m = X.m, qtop = qfloor(m);
  const Hist ht = hist_of(R);
  if (t == 0) {
    n_list = 0;
    cx.b = NB;
    cx.above = cx.upto = 0;
  }
  Kind kind = K_NONE;
  int bb = NB;
  uint64_t above = 0, total = 0;
  if (ht != H_NONE && fabsf(m) <= MAX_M) {
    for (int i = t; i < a.P; i += CT) {
      const float cm = __uint_as_float((uint32_t)a.rec[(row * a.P + i) * REC]);
      // a chunk whose maximum is far below, or which has no finite value, falls into the last bucket whole
      coff[i] = (int)fminf(qtop - qfloor(cm), (float)NB);
      // the chunk's weights are against its own maximum: their factor in double, so that the merge adds
      // nothing to the weights' own rounding but one unit of 2^-32 per bucket (a chunk without a finite
      // value has empty buckets: exp2 of -inf is 0)
      cscale[i] = ht == H_MASS ? exp2(((double)cm - (double)m) * (double)L2E) : 1.0;
    }
    __syncthreads();
    // row bucket b of a chunk whose maximum lies off buckets below the row's: its bucket b - off; the last
    // bucket takes all of the chunk's from there on
    // (all sums are integers, so that the threads agree on the cumulative to the last unit)
    uint64_t hv[BPT], sum = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) hv[i] = 0;
    uint64_t rest = 0;  // this thread's share of the last row bucket
    constexpr int U = 4;  // chunks whose buckets are in flight together
    for (int i0 = 0; i0 < a.P; i0 += U) {
      uint64_t v[U][BPT], own[U][BPT];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = min(i0 + u, a.P - 1), off = coff[i];
        const uint64_t* hc = a.hist + (row * a.P + i) * NB;
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
          v[u][k] = hc[max(t * BPT + k - off, 0)];
          own[u][k] = hc[t * BPT + k];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = min(i0 + u, a.P - 1), off = coff[i];
        const double sc = cscale[i];
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
          const int b = t * BPT + k;
          if (i0 + u < a.P && b >= off && b < NB - 1) hv[k] += (uint64_t)(sc * (double)v[u][k]);
          // source buckets that fall into the row's last one
          if (i0 + u < a.P && b + off >= NB - 1) rest += (uint64_t)(sc * (double)own[u][k]);
        }
      }
    }
    rest = wave_sum_u64(rest);
    if (lane_id() == 63) wtot[wave_id()] = rest;
    __syncthreads();
    uint64_t last = 0;  // the row's last bucket
#pragma unroll
    for (int w = 0; w < NWV; ++w) last += wtot[w];
    if (t == CT - 1) hv[BPT - 1] = last;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BPT; ++k) sum += hv[k];
    const uint64_t incl = wave_incl_scan_u64(sum);
    if (lane_id() == 63) wtot[wave_id()] = incl;
    __syncthreads();
    uint64_t ex = incl - sum;
    for (int w = 0; w < wave_id(); ++w) ex += wtot[w];
#pragma unroll
    for (int w = 0; w < NWV; ++w) total += wtot[w];
    const uint64_t body = total - last;
    // the bucket where the cumulative reaches the target, or the one of the min-p cut
    const bool by_cut = ht == H_COUNT && !R.kon;
    const double target = R.kon ? (double)R.k : (double)R.p * (double)total;
    const int cutb = by_cut ? bucket(qtop, X.tau_m) : -1;
    uint64_t cum = ex;
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
      const int b = t * BPT + k;
      const uint64_t nx = cum + hv[k];
      const bool hit = by_cut ? b == cutb : (hv[k] > 0 && (double)cum < target && (double)nx >= target);
      if (hit) {
        cx.b = b;
        cx.above = cum;
        cx.upto = nx;
      }
      cum = nx;
    }
    __syncthreads();
    bb = cx.b;
    above = cx.above;
    if (ht == H_MASS) {
      kind = bb < NB ? K_MASS : K_SLOW;
    } else if (!R.topp_on) {
      kind = bb < NB ? K_COUNT : K_NONE;  // fewer than k finite values: top-k keeps them all
    } else {
      // Every value down to the crossing bucket, or to the last bucket but one: what lies in the last is 32
      // below the maximum, weighs less than 2^-46 and cannot move a top-p cut (which lies where the weights do),
      // nor is it kept, as top-p < 1 keeps no more than it needs.  So a row with fewer than k finite values
      // (a mask), where nothing crosses, or with its k-th value that far down needs no selection over memory:
      // 64 x 128256, top-k 40 and top-p 0.9, 20 ids unmasked: 219 us over memory, 46 us staged; values of scale
      // 3e5: 345 us and 45 us.
      const uint64_t n_all = bb < NB - 1 ? cx.upto : body;
      bb = min(bb, NB - 2);
      kind = n_all <= (uint64_t)CAP ? K_ALL : K_SLOW;
    }
  } else if (ht != H_NONE) {
    kind = K_SLOW;
  }
  if (c == 0 && t == 0) {
    a.rec[L * REC + 5] = (uint64_t)kind | ((uint64_t)bb << 8);
    a.rec[L * REC + 6] = above;
    a.rec[L * REC + 7] = total;
  }
  if (kind == K_SLOW) return;  // uniform: selected over the whole row by the next launch
  __syncthreads();             // n_list is cleared
  process_slots(R, q, d);
  const float lo = X.tau_m;
  double acc = 0.0;
  int cnt = 0;
  float zmin = INFINITY;
  uint32_t* list = a.lists + L * LC;
  // sure: z >= zs, kept whatever the cut in the bucket; staged: zl <= z < zs0, the bucket's values (K_ALL: all
  // from the bucket up)
  float zs0 = -FLT_MAX, zl = INFINITY;  // K_NONE stages nothing
  if (kind != K_NONE) {
    zs0 = kind == K_ALL ? INFINITY : bucket_edge(qtop, bb - 1);
    zl = bb < NB - 1 ? bucket_edge(qtop, bb) : -FLT_MAX;
  }
  const float zs = fmaxf(zs0, lo);
  auto classify = [&](float z, bool& sure, bool& st) __attribute__((always_inline)) {
    sure = z >= zs;
    st = z >= zl && z < zs0;
  };
  uint64_t sb = 0;  // bit 4 j + e: value e of slot j is staged; the last bit the tail's
  static_assert(4 * CJ < 63, "a thread's values do not fit the staging mask");
#pragma unroll
  for (int j = 0; j < CJ; ++j) {
    uint32_t any = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float z = d[j].v[e];
      bool sure, st;
      classify(z, sure, st);
      any |= (sure ? 1u : 0u) << e;
      zmin = sure ? fminf(zmin, z) : zmin;
      sb |= (uint64_t)(st ? 1u : 0u) << (4 * j + e);
    }
    if (__ballot(any != 0)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc += (double)((any >> e) & 1u ? __expf(d[j].v[e] - m) : 0.0f);
      cnt += __popc(any);
    }
  }
  const float zt = canon(xt, R.r);
  if (q.tail >= 0) {
    bool sure, st;
    classify(zt, sure, st);
    if (sure) {
      acc += (double)__expf(zt - m);
      ++cnt;
      zmin = fminf(zmin, zt);
    }
    sb |= (uint64_t)(st ? 1u : 0u) << 63;
  }
  if (__ballot(sb != 0)) {
    // one claim of list places per wave (a claim per value was a chain of LDS round trips)
    const int own = __popcll(sb), incl = wave_incl_scan_i(own);
    int i = 0;
    if (lane_id() == 0) i = atomicAdd(&n_list, lane_i32(incl, 63));
    i = __builtin_amdgcn_readfirstlane(i) + incl - own;
    auto stage = [&](float z, int bit) __attribute__((always_inline)) {
      if ((sb >> bit) & 1u) {
        if (i < LC) list[i] = f2key(z);
        ++i;
      }
    };
#pragma unroll
    for (int j = 0; j < CJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) stage(d[j].v[e], 4 * j + e);
    stage(zt, 63);
  }
  acc = wave_scan_f64(acc);
  cnt = wave_sum_i(cnt);
  zmin = wave_min(zmin);
  if (lane_id() == 63) {
    wsum[wave_id()] = acc;
    wcnt[wave_id()] = cnt;
    wmin[wave_id()] = f2key(zmin);
  }
  __syncthreads();
  if (t == 0) {
    uint32_t k0 = 0xffffffffu;
    int n0 = 0;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      k0 = min(k0, wmin[w]);
      n0 += wcnt[w];
      sum += wsum[w];
    }
    a.rec[L * REC + 2] = (uint64_t)(uint32_t)n_list;
    a.rec[L * REC + 3] = (uint64_t)__double_as_longlong(sum);
    a.rec[L * REC + 4] = ((uint64_t)(uint32_t)n0 << 32) | (n0 > 0 ? k0 : 0u);
  }
}

// ----------------------------------------------------------------------------------------------
// Pass 3: selections among the staged values, or over the row in memory.
// ----------------------------------------------------------------------------------------------
struct SolveLds {
  uint32_t keys[CAP];
  uint32_t wt[ST];
  uint64_t h[256];
  uint64_t red[ST / 64];
  int32_t off[MAXPC + 1];
  int32_t hit;
  uint64_t before;
};
__device__ __forceinline__ uint64_t sum_u64(uint64_t v, SolveLds& s) {
  v = wave_sum_u64(v);
  __syncthreads();
  if (lane_id() == 0) s.red[wave_id()] = v;
  __syncthreads();
  uint64_t r = 0;
#pragma unroll
  for (int w = 0; w < ST / 64; ++w) r += s.red[w];
  return r;
}
__device__ __forceinline__ double sum_f64(double v, SolveLds& s) {
  v = wave_scan_f64(v);
  __syncthreads();
  if (lane_id() == 63) s.red[wave_id()] = (uint64_t)__double_as_longlong(v);
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int w = 0; w < ST / 64; ++w) r += __longlong_as_double((long long)s.red[w]);
  return r;
}

struct StagedSrc {  // f(z) for every staged value
  const uint32_t* keys;
  int n;
  template <class F>
  __device__ __forceinline__ void operator()(F&& f) const {
    for (int i = threadIdx.x; i < n; i += ST) f(key2f(keys[i]));
  }
};
struct RowSrc {  // f(z) for every value of the row
  const Row& R;
  template <class F>
  __device__ __forceinline__ void operator()(F&& f) const {
    constexpr int U = 4;
    for (int s0 = 0; s0 < R.slots; s0 += ST * U) {
      F4 d[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        d[u] = *reinterpret_cast<const F4*>(R.x + (int64_t)min(s0 + u * ST + (int)threadIdx.x, R.slots - 1) * 4);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s0 + u * ST + (int)threadIdx.x < R.slots) {
#pragma unroll
          for (int e = 0; e < 4; ++e) f(canon(d[u].v[e], R.r));
        }
    }
    const int i = R.slots * 4 + (int)threadIdx.x;
    if (i < R.V) f(canon(R.x[i], R.r));
  }
};

// select_key for n <= ST staged values: thread i compares value i with every other (waves without a value
// sit the loop out); two barriers where the byte rounds take twelve.  COUNT: every value weighs 1 and the
// sums are 32-bit.
template <bool COUNT, class W>
__device__ __forceinline__ uint32_t select_few(SolveLds& s, int n, float lo, double target, double above, W&& weight) {
  const int t = threadIdx.x;
  const uint32_t mine = t < n ? s.keys[t] : 0u;
  const float z = key2f(mine);
  const bool in = t < n && z > -INFINITY && z >= lo;
  __syncthreads();
  if constexpr (!COUNT) s.wt[t] = in ? (uint32_t)weight(z) : 0u;
  if (t == 0) s.hit = 0;
  __syncthreads();
  if (wave_id() * 64 < n) {
    using Sum = std::conditional_t<COUNT, uint32_t, uint64_t>;
    Sum gt = 0, ge = 0;
    const uint32_t klo = COUNT ? f2key(lo) : 0u;  // (weights below lo are 0)
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      const uint32_t k = s.keys[i];
      uint32_t w;
      if constexpr (COUNT) w = k >= klo ? 1u : 0u;
      else w = s.wt[i];
      gt += k > mine ? w : 0u;
      ge += k >= mine ? w : 0u;
    }
    if (in && ge > gt && above + (double)gt < target && above + (double)ge >= target) s.hit = (int32_t)mine;
  }
  __syncthreads();
  return (uint32_t)s.hit;
}

// The order key of the first group, in descending order, at which the cumulative of weight(z) over the
// finite values z >= lo, starting from `above`, reaches target; 0 when it never does.  Byte by byte.
template <class Src, class W>
__device__ __forceinline__ uint32_t select_key(const Src& src, SolveLds& s, float lo, double target, double above,
                                               W&& weight) {
  uint32_t prefix = 0, pmask = 0;
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int b = threadIdx.x; b < 256; b += ST) s.h[b] = 0;
    if (threadIdx.x == 0) s.hit = -1;
    __syncthreads();
    src([&](float z) __attribute__((always_inline)) {
      if (z > -INFINITY && z >= lo) {
        const uint32_t k = f2key(z);
        if ((k & pmask) == prefix) {
          const uint64_t w = weight(z);
          if (w) atomicAdd((unsigned long long*)&s.h[(k >> shift) & 255u], (unsigned long long)w);
        }
      }
    });
    __syncthreads();
    if (threadIdx.x < 64) {
      const int l = threadIdx.x;  // buckets 255 - 4 l .. 252 - 4 l, descending
      uint64_t b4[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        b4[q] = s.h[255 - 4 * l - q];
        sum += b4[q];
      }
      const uint64_t incl = wave_incl_scan_u64(sum);
      const uint64_t hit = __ballot(sum > 0 && above + (double)incl >= target);
      if (hit && l == (int)__builtin_ctzll(hit)) {
        uint64_t cum = incl - sum;
        int at = -1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (at < 0 && b4[q] > 0 && above + (double)(cum + b4[q]) >= target) at = q;
          if (at < 0) cum += b4[q];
        }
        s.hit = 255 - 4 * l - at;
        s.before = cum;
      }
    }
    __syncthreads();
    const int b = s.hit;
    if (b < 0) return 0u;  // uniform
    above += (double)s.before;
    prefix |= (uint32_t)b << shift;
    pmask |= 255u << shift;
    __syncthreads();
  }
  return prefix;
}

__global__ __launch_bounds__(ST, 2) void k_filter_solve(FArgs a) {
  __shared__ SolveLds s;
  const int t = threadIdx.x;
  const int64_t row = blockIdx.x;
  uint64_t* rec = a.rec + row * a.P * REC;
  Row R;
  row_setup(a, row, R);
  const RowMax X = row_max(a, R, row);
  const bool skip = X.empty || X.bad;
  const float m = X.m;
  uint32_t flags = R.flags | (X.empty ? FLAG_EMPTY : 0u) | (X.bad ? FLAG_BAD_INPUT : 0u);
  float tau = INFINITY, zmin = -INFINITY;
  int kept = 0, id = -1;
  double zs = 0.0;
  if (skip) {
    // no finite value, or a NaN or +inf among them
  } else if (R.greedy) {
    id = INT32_MAX;
    for (int c = 0; c < a.P; ++c)
      if (__uint_as_float((uint32_t)rec[c * REC]) == m) id = min(id, (int)(uint32_t)rec[c * REC + 1]);
    tau = zmin = m;
    kept = 1;
    zs = 1.0;
  } else {
    const uint64_t w5 = rec[5];
    Kind kind = (Kind)(w5 & 255u);
    const double above = (double)rec[6], total = (double)rec[7];
    int n = 0;
    uint32_t kmin = 0xffffffffu;
    if (kind != K_SLOW) {
      // lane c of every wave holds chunk c's record
      const int l = lane_id(), lc = min(l, a.P - 1);
      const uint64_t w2 = rec[lc * REC + 2], w3 = rec[lc * REC + 3], w4 = rec[lc * REC + 4];
      const int nc = l < a.P ? (int)(uint32_t)w2 : 0;
      const int incl = wave_incl_scan_i(nc);
      if (t < 64) s.off[t] = incl - nc;
      if (t == 63) s.off[64] = incl;
      n = lane_i32(incl, 63);
      const bool fit = __ballot(nc > LC) == 0;
      kept = wave_sum_i(l < a.P ? (int)(w4 >> 32) : 0);
      kmin = wave_min_u32(l < a.P && (w4 >> 32) ? (uint32_t)w4 : 0xffffffffu);
      for (int c = 0; c < a.P; ++c) zs += __longlong_as_double((long long)lane_u64(w3, c));
      if (!fit || n > CAP) kind = K_SLOW;
      __syncthreads();
    }
    tau = X.tau_m;
    struct One {
      __device__ __forceinline__ uint64_t operator()(float) const { return 1ull; }
    };
    const One one{};
    auto mass = [&](float z) __attribute__((always_inline)) -> uint64_t { return fix_weight(z, m); };
    // both filters over a source that holds every value they can keep
    auto select_all = [&](const auto& src, auto&& sel) __attribute__((always_inline)) {
      if (R.kon) {
        const uint32_t kk = sel(-INFINITY, (double)R.k, 0.0, one);
        if (kk) tau = fmaxf(tau, key2f(kk));
      }
      if (R.topp_on) {
        uint64_t own = 0;
        src([&](float z) __attribute__((always_inline)) {
          if (z > -INFINITY && z >= tau) own += mass(z);
        });
        const uint64_t tot = sum_u64(own, s);
        const uint32_t kk = sel(tau, (double)R.p * (double)tot, 0.0, mass);
        if (kk) tau = fmaxf(tau, key2f(kk));
      }
    };
    double add = 0.0;
    int more = 0;
    uint32_t km = 0xffffffffu;
    auto tally = [&](float z) __attribute__((always_inline)) {
      if (z > -INFINITY && z >= tau) {
        ++more;
        km = min(km, f2key(z));
      }
    };
    if (kind == K_SLOW) {
      const RowSrc src{R};
      select_all(src, [&](float lo, double target, double ab, auto&& w) __attribute__((always_inline)) {
        return select_key(src, s, lo, target, ab, w);
      });
      zs = 0.0;
      kept = 0;
      kmin = 0xffffffffu;
      src([&](float z) __attribute__((always_inline)) {
        if (z > -INFINITY && z >= tau) add += (double)__expf(z - m);
        tally(z);
      });
      add = sum_f64(add, s);
    } else if (kind != K_NONE) {
      for (int c = wave_id(); c < a.P; c += ST / 64) {  // a chunk per wave: their loads overlap
        const int nc = s.off[c + 1] - s.off[c];
        const uint32_t* src = a.lists + (row * a.P + c) * LC;
        for (int i = lane_id(); i < nc; i += 64) s.keys[s.off[c] + i] = src[i];
      }
      __syncthreads();
      const StagedSrc src{s.keys, n};
      auto sel = [&](float lo, double target, double ab, auto&& w) __attribute__((always_inline)) {
        constexpr bool COUNT = std::is_same_v<std::decay_t<decltype(w)>, One>;
        return n <= ST ? select_few<COUNT>(s, n, lo, target, ab, w) : select_key(src, s, lo, target, ab, w);
      };
      if (kind == K_ALL) {
        select_all(src, sel);
      } else if (kind == K_COUNT) {
        const uint32_t kk = sel(-INFINITY, (double)R.k - above, 0.0, one);
        if (kk) tau = fmaxf(tau, key2f(kk));
      } else {
        // the chunks' weights are in units of 2^-32 against the row's maximum, like these
        uint32_t kk = sel(-INFINITY, (double)R.p * total, above, mass);
        if (kk) {
          tau = fmaxf(tau, key2f(kk));
        } else {  // rounding left the cumulative below the target: the whole bucket is kept
          src([&](float z) __attribute__((always_inline)) { km = min(km, f2key(z)); });
          km = wave_min_u32(km);
          __syncthreads();
          if (lane_id() == 0) s.red[wave_id()] = km;
          __syncthreads();
#pragma unroll
          for (int w = 0; w < ST / 64; ++w) km = min(km, (uint32_t)s.red[w]);
          if (n > 0) tau = fmaxf(tau, key2f(km));
          km = 0xffffffffu;
        }
      }
      // the staged values' order is arbitrary: their kept weight is an integer sum
      uint64_t fx = 0;
      src([&](float z) __attribute__((always_inline)) {
        if (z >= tau) fx += (uint64_t)((double)__expf(z - m) * FIX44);
        tally(z);
      });
      add = (double)sum_u64(fx, s) / FIX44;
    }
    if (kind != K_NONE) {
      kept += (int)sum_u64((uint64_t)more, s);
      km = wave_min_u32(km);
      __syncthreads();
      if (lane_id() == 0) s.red[wave_id()] = km;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < ST / 64; ++w) kmin = min(kmin, (uint32_t)s.red[w]);
    }
    zs += add;
    zmin = key2f(kmin);
  }
  __syncthreads();  // every thread has read the records
  if (t == 0) {
    if (a.out_flags) a.out_flags[row] = flags;
    if (a.out_threshold) a.out_threshold[row] = skip ? -INFINITY : zmin;
    if (a.out_kept) a.out_kept[row] = kept;
    if (a.out_log_norm) a.out_log_norm[row] = skip ? -INFINITY : (float)((double)m + log(zs));
  }
  // for the writing pass, in every chunk's record: the cut, the maximum, 1 / mass, the greedy id
  const float inv = zs > 0.0 ? (float)(1.0 / zs) : 0.0f;
  if (t < a.P) {
    rec[t * REC + 0] = ((uint64_t)__float_as_uint(m) << 32) | __float_as_uint(tau);
    rec[t * REC + 1] = ((uint64_t)(uint32_t)id << 32) | __float_as_uint(inv);
  }
}

// ----------------------------------------------------------------------------------------------
// Pass 4: the probabilities; the chunk's workspace is left zero.
// ----------------------------------------------------------------------------------------------
__global__ __launch_bounds__(CT, 4) void k_filter_write(FArgs a) {
  const int t = threadIdx.x;
  const int64_t L = blockIdx.x, row = L / a.P;
  const int c = (int)(L - row * a.P);
  Row R;
  row_setup(a, row, R);
  const ChunkAt q = chunk_at(a, R, c);
  const int ns = q.ns;
  F4 d[CJ];
  if (a.out_probs) load_slots(R, q, d);
  uint64_t* rec = a.rec + L * REC;
  const uint64_t w0 = rec[0], w1 = rec[1];
  const float tau = __uint_as_float((uint32_t)w0), m = __uint_as_float((uint32_t)(w0 >> 32));
  const float inv = __uint_as_float((uint32_t)w1);
  const int id = (int)(uint32_t)(w1 >> 32);
  const bool greedy = R.greedy;
  // a skipped row has tau = +inf and no id, so that nothing passes (a +inf value neither: inv is 0 and m
  // may be +inf, so its product is not formed)
  auto prob = [&](float x, int pos) __attribute__((always_inline)) -> float {
    const float z = canon(x, R.r);
    const float w = __expf(z - m) * inv;
    if (greedy) return pos == id ? 1.0f : 0.0f;
    return z > -INFINITY && z >= tau && inv > 0.0f ? w : 0.0f;
  };
  if (a.out_probs) {
    float* o = a.out_probs + row * a.V;
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      const int l = j * CT + t;
      if (l < ns) {
        const int pos = (q.s0 + l) * 4;
        F4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w.v[e] = prob(d[j].v[e], pos + e);
        *reinterpret_cast<F4*>(o + pos) = w;
      }
    }
    if (q.tail >= 0) o[q.tail] = prob(R.x[q.tail], q.tail);
  }
  uint4* hz = reinterpret_cast<uint4*>(a.hist + L * NB);
  uint4* lz = reinterpret_cast<uint4*>(a.lists + L * LC);
  const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
  if (hist_of(R) != H_NONE) {
    for (int i = t; i < NB / 2; i += CT) hz[i] = zero;
    for (int i = t; i < LC / 4; i += CT) lz[i] = zero;
  }
  __syncthreads();  // every thread has read the record
  if (t < REC) rec[t] = 0;
}

// ----------------------------------------------------------------------------------------------
// Host side
// ----------------------------------------------------------------------------------------------
struct Geo {
  int P;
  int64_t chunk_slots, lists, hist, total;
};
bool geometry(int64_t B, int64_t V, Geo& g) {
  const int64_t body = V / 4;
  int64_t P = (body + CSLOTS - 1) / CSLOTS;
  if (P < 1) P = 1;
  if (P > MAXPC || B <= 0 || B * P >= ((int64_t)1 << 31)) return false;
  g.P = (int)P;
  g.chunk_slots = (body + P - 1) / P;
  g.lists = align256(B * P * (int64_t)REC * 8);
  g.hist = align256(g.lists + B * P * (int64_t)LC * 4);
  g.total = align256(g.hist + B * P * (int64_t)NB * 8);
  return true;
}

}  // namespace

namespace albireo_filter {

size_t workspace_bytes(int64_t B, int64_t V) {
  Geo g;
  return geometry(B, V, g) ? (size_t)g.total : 0;
}

albireo_status_t launch(const float* logits, int64_t B, int64_t V, int64_t ld, const albireo_params_t* p,
                        float* out_probs, float* out_threshold, int32_t* out_kept, float* out_log_norm,
                        uint32_t* out_flags, unsigned char* ws, hipStream_t stream) {
  Geo g;
  if (!geometry(B, V, g)) return ALBIREO_E_UNSUPPORTED;
  FArgs a;
  memset(&a, 0, sizeof a);
  a.logits = logits;
  a.B = B;
  a.V = V;
  a.ld = ld;
  if (p) {
    a.temperature = p->temperature;
    a.top_k = p->top_k;
    a.top_p = p->top_p;
    a.min_p = p->min_p;
  }
  a.out_probs = out_probs;
  a.out_threshold = out_threshold;
  a.out_kept = out_kept;
  a.out_log_norm = out_log_norm;
  a.out_flags = out_flags;
  a.P = g.P;
  a.chunk_slots = g.chunk_slots;
  a.rec = reinterpret_cast<uint64_t*>(ws);
  a.lists = reinterpret_cast<uint32_t*>(ws + g.lists);
  a.hist = reinterpret_cast<uint64_t*>(ws + g.hist);
  const dim3 chunks((unsigned)(B * g.P)), rows((unsigned)B);
  void* args[] = {&a};
  hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(&k_filter_hist), chunks, dim3(CT), args, 0, stream);
  if (e == hipSuccess)
    e = hipLaunchKernel(reinterpret_cast<const void*>(&k_filter_stage), chunks, dim3(CT), args, 0, stream);
  if (e == hipSuccess)
    e = hipLaunchKernel(reinterpret_cast<const void*>(&k_filter_solve), rows, dim3(ST), args, 0, stream);
  if (e == hipSuccess)
    e = hipLaunchKernel(reinterpret_cast<const void*>(&k_filter_write), chunks, dim3(CT), args, 0, stream);
  return e == hipSuccess ? ALBIREO_OK : ALBIREO_E_LAUNCH;
}

}  // namespace albireo_filter
