// Logits pass without a histogram: every logit's exponential is evaluated in fp64 as it is read, in one
// pass over the segment.  The path of fp32 rows (whose values are too many to be counted).
//
// What bounds it where the CUs have several rows each: instruction issue.  Fourteen vector instructions a logit for the exponential and the sums, twelve of them
// fp64, 23 in all by the counter (maxima, tests for NaN, the bound, the rows' tails).  2048 rows of 65536 take 130 to 137 us, 4.0 TB/s; their 48.0 k instructions a SIMD
// are, at four cycles each, 74 % of its busy cycles.  (The distance from the maximum and its cut-off by two instructions, see scaled_distance: 0.9 % longer; no
// table but a polynomial of degree 11, four instructions more: 21 % longer.)  Fewer rows wait for the start and the tail, and for CUs that have one row more than others:
// layers of 250, 320 and 510 rows of 32000 on 256 CUs take 18.0, 22.6 and 24.3 us.  The two-pass form that it replaces read
// the segment twice (the maximum first) and spent about fifty instructions in the library's exp.
//
// Sums.  Each wavefront keeps Z = sum e^(x-a) and S = sum (x-a) e^(x-a) against its own largest logit so far, a
// (uniform over the wave; re-referenced when a tile raises it, which happens a few times a segment), so
// every term of S has one sign and nothing overflows.  No barrier is needed for any of it.
//
// Exponential.  e^t = 2^(k/256) e^r with k = rint(256 t / ln 2), |r| <= ln 2 / 512 (Cody and Waite's reduction, Tang's
// table): 2^(j/256) for j = 0..255 from a 2 KB LDS table (of 32 entries the random reads of a wave would never conflict, but the
// polynomial needs a degree more, and it is issue that binds), e^r from a polynomial of degree 4 whose upper three coefficients interpolate
// (e^r - 1 - r) / r^2 at Chebyshev nodes (9.5e-18 relative); the exponent k div 256 is added to the table entry's
// upper word, from which the entry's own share has been taken off beforehand, as table-driven exponentials commonly do.  In all e^t is
// good to about 3.0e-16 + 3.8e-17 |t| relative (20000 points against 50 digits): the rounding of the table entry and of the product, and the one-constant
// reduction's.  t <= 0 here, so the last matters only as |t| e^t, at most e^-1.
//
// Top K without reading anything twice: the K-th largest of the maxima of 64 lane columns (128 for large K) is
// a lower bound of the K-th largest logit from the first tile on; the few finite logits that reach it are appended
// to a list in LDS as they stream past, and the list is ranked exactly at the end.  The bound is raised from
// the maxima so far at tiles 2, 4, 8, ...: stale maxima only make it lower, so no barrier is needed there.
// Lists that end up long (massive ties, large K), that overflowed (sorted rows, logits that only follow behind a masked
// stretch) or that are short of K (nearly everything masked) are put right by settle_list.
#pragma once
#include "k_logits.h"

namespace c2t {

constexpr int EXP_TAB_BITS = 8, EXP_TAB = 1 << EXP_TAB_BITS;
constexpr int DIRECT_CHUNKS = 4;               // chunks a lane reads per tile: 64 bytes, two tiles in flight

// 2^(j/256) with j << 12 taken off its upper word: adding k << 12 for any k = 256 q + j then gives 2^(k/256)
__device__ __forceinline__ double exp_tab_entry(int j) {
  const uint64_t u = (uint64_t)__double_as_longlong(exp2((double)j / EXP_TAB));
  return __longlong_as_double((long long)(u - ((uint64_t)j << (52 - EXP_TAB_BITS))));
}
__device__ __forceinline__ float max3_raw(float a, float b, float c) {     // without the canonicalising copies fmaxf adds per operand
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
constexpr double EXP_SHIFT = 6755399441055744.0;             // 1.5 * 2^52: the sum's low word is the rounded integer
constexpr double EXP_PER_STEP = 0x1.71547652b82fep+8, EXP_STEP = 0x1.62e42fefa39efp-9;      // 256 / ln 2, ln 2 / 256
constexpr double EXP_C4 = 0x1.5555565bb9890p-5, EXP_C3 = 0x1.555556deeba30p-3, EXP_C2 = 0.5;    // of e^r = 1 + r + C2 r^2 + C3 r^3 + C4 r^4
// e^t for t <= 0 (clamped at -700: 1e-304, nothing beside the largest term, which is 1)
__device__ __forceinline__ double exp_nonpositive(double t, const double* tab) {
  const double kf = __builtin_fma(t, EXP_PER_STEP, EXP_SHIFT);
  const int k = __double2loint(kf);
  const double r = __builtin_fma(kf - EXP_SHIFT, -EXP_STEP, t);
  const double e = tab[k & (EXP_TAB - 1)];
  double p = __builtin_fma(EXP_C4, r, EXP_C3);
  p = __builtin_fma(p, r, EXP_C2);
  p = __builtin_fma(p, r, 1.0);
  p = __builtin_fma(p, r, 1.0);
  typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
  uint2v w = __builtin_bit_cast(uint2v, e);
  w.y += (uint32_t)k << (20 - EXP_TAB_BITS);
  return __builtin_bit_cast(double, w) * p;
}

// The same for the logits of a tile, from v = (a - x) / 512 in [0, 1]: one fused multiply-add forms v and its clamp modifier cuts it off (e^-512 is nothing beside the
// largest term, which is 1), where a subtraction and a maximum were two instructions of sixteen.  The scale being a power of two, v and the
// reduced argument are those of t = x - a, rounded alike.
constexpr double TILE_SCALE = 512.0;
__device__ __forceinline__ double scaled_distance(float x, double a_scaled) {      // a_scaled = a / 512
  double v;
  asm("v_fma_f64 %0, %1, %2, %3 clamp" : "=v"(v) : "v"((double)x), "s"(-1.0 / TILE_SCALE), "v"(a_scaled));
  return v;
}
__device__ __forceinline__ double exp_of_distance(double v, const double* tab) {
  const double kf = __builtin_fma(v, -EXP_PER_STEP * TILE_SCALE, EXP_SHIFT);
  const int k = __double2loint(kf);
  const double r = __builtin_fma(kf - EXP_SHIFT, -EXP_STEP / TILE_SCALE, -v);      // a 512th of the reduced argument
  const double e = tab[k & (EXP_TAB - 1)];
  constexpr double S1 = TILE_SCALE, S2 = S1 * S1, S3 = S2 * S1, S4 = S3 * S1;
  double p = __builtin_fma(EXP_C4 * S4, r, EXP_C3 * S3);
  p = __builtin_fma(p, r, EXP_C2 * S2);
  p = __builtin_fma(p, r, S1);
  p = __builtin_fma(p, r, 1.0);
  typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
  uint2v w = __builtin_bit_cast(uint2v, e);
  w.y += (uint32_t)k << (20 - EXP_TAB_BITS);
  return __builtin_bit_cast(double, w) * p;
}

template <int NT>
struct DirectShared {
  static constexpr int NW = NT / WAVE;
  double exp_tab[EXP_TAB];
  double wave_z[NW], wave_s[NW];
  float wave_a[NW];
  float col_max[NW][WAVE];                      // running maximum of every lane
  int32_t scan_tmp[1][NW];
  int32_t n_list, bad, n_reach;
};

// K-th largest of the maxima of NV * 64 columns (a column: every 64 NV-th lane of the workgroup), to the bits above LOW_BIT: a lower
// bound of the K-th largest logit seen
template <int NT, int NV, int LOW_BIT>
__device__ __forceinline__ float bound_of_columns(const DirectShared<NT>& sh, int K) {
  float m[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) m[v] = -INFINITY;
#pragma unroll
  for (int w = 0; w < NT / WAVE; ++w)
    m[w % NV] = fmaxf(m[w % NV], __hip_atomic_load(&sh.col_max[w][threadIdx.x & (WAVE - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
  uint32_t key[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) key[v] = sortable_key(m[v]);
  const uint32_t t = wave_kth_largest<NV, LOW_BIT>(key, K);
  return t < 0x007FFFFFu ? -INFINITY : key_to_float(t);      // (below -inf's key once the low bits are cleared)
}
// Of randomly placed logits 64 (H(64) - H(64 - K)) reach the bound from 64 columns: 45 for K = 32, but 89 for K = 48 and 304 for
// K = 64, which have to be listed, cut and ranked; from 128 columns 60 and 89, for twice the ballots.  Layers of 256 rows
// of 32000, with 64 / 128 columns: K = 48 28.4 / 26.7 us, K = 64 88 / 30 us.
constexpr int COLUMNS64_MAX_K = 32;
template <int NT>
__device__ __forceinline__ float column_bound(const DirectShared<NT>& sh, int K) {
  if (__builtin_expect(K > COLUMNS64_MAX_K, 0)) return bound_of_columns<NT, 2, 16>(sh, K);
  return bound_of_columns<NT, 1, 16>(sh, K);
}

template <int NT>
struct DirectState {                            // of one wavefront
  float a, lane_max, tau;                       // a: reference of the sums, the wave's largest logit so far (uniform)
  double Z, S;                                  // S: sum of v e^(x - a), v = (a - x) / 512
  bool bad;
};

// A segment's chunks (uniform): the bounds check returns zeros past the last one without reading
__device__ __forceinline__ __amdgpu_buffer_rsrc_t segment_buffer(const uint4* rowp, const Segment& sg) {
  const uint64_t base = (uint64_t)(rowp + sg.c0);
  const uint64_t base_u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base) |
                          ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)) << 32);
  return __builtin_amdgcn_make_buffer_rsrc((void*)base_u, 0, sg.ncell * 16, 0x00020000);
}

// Logits of a tile that the segment does not have read as -inf: chunks past its end, the padding of the row's last chunk.
template <int NT>
__device__ __forceinline__ void blank_tile(uint4 (&q)[DIRECT_CHUNKS], const Segment& sg, int first) {
#pragma unroll
  for (int c = 0; c < DIRECT_CHUNKS; ++c) {
    const int g = first + c * NT + (int)threadIdx.x;
    const int nv = g >= sg.ncell ? 0 : sg.c0 + g == sg.tail_chunk ? sg.tail_valid : LogitTraits<0>::EPC;
    uint32_t w[4] = {q[c].x, q[c].y, q[c].z, q[c].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) if (j >= nv) w[j] = 0xff800000u;       // -inf
    q[c] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// One tile: sums, and the logits that reach the bound.  t: the tile's number.
template <int NT>
__device__ __forceinline__ void direct_tile(uint4 (&q)[DIRECT_CHUNKS], int t, const Segment& sg, int V, int K,
                                            DirectState<NT>& s, DirectShared<NT>& sh, const SelectLds& sel) {
  typedef LogitTraits<0> T;
  const int tid = threadIdx.x;
  float cm[DIRECT_CHUNKS];
#pragma unroll
  for (int c = 0; c < DIRECT_CHUNKS; ++c) {
    float x[T::EPC];
    T::unpack(q[c], x);
    cm[c] = max3_raw(x[0], x[1], x[2]);
#pragma unroll
    for (int j = 3; j < T::EPC; j += 2) cm[c] = max3_raw(cm[c], x[j], x[j + 1 < T::EPC ? j + 1 : j]);
  }
  const float tm = max3_raw(max3_raw(cm[0], cm[1], cm[2]), cm[3], cm[3]);
  s.lane_max = max3_raw(s.lane_max, tm, tm);
  __hip_atomic_store(&sh.col_max[tid >> 6][tid & (WAVE - 1)], s.lane_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  const float wm = wave_max(tm);
  if (wm > s.a) {                                            // uniform
    if (s.a > -INFINITY) {
      const double d = fmax((double)s.a - (double)wm, -700.0), f = exp_nonpositive(d, sh.exp_tab);
      s.S = (s.S - d / TILE_SCALE * s.Z) * f; s.Z *= f;
    }
    s.a = wm;
  }
  const double ad = (double)s.a / TILE_SCALE;
  const bool masked = !(s.a > -INFINITY);                    // (uniform) no logit yet that adds anything
#pragma unroll
  for (int c = 0; c < DIRECT_CHUNKS; ++c) {
    asm volatile("" : "+v"(q[c].x), "+v"(q[c].y), "+v"(q[c].z), "+v"(q[c].w));     // (conversions of later chunks are not hoisted: they would spill; of a copy: a move a logit)
    float x[T::EPC];
    T::unpack(q[c], x);
#pragma unroll
    for (int j = 0; j < T::EPC; ++j) {
      if (j & 1) s.bad |= __builtin_isunordered(x[j - 1], x[j]);           // (+inf shows in the maximum)
      const double v = scaled_distance(x[j], ad);
      const double e = exp_of_distance(v, sh.exp_tab);
      s.Z += e; s.S = __builtin_fma(v, e, s.S);
      if (j % 4 == 3) asm volatile("" : "+v"(s.Z), "+v"(s.S));   // four exponentials at a time cover their latency; more would spill
    }
  }
  if (masked) s.Z = s.S = 0.0;                               // (what has been added is not a number's)
  if (t == 0) __syncthreads();                               // the first tile's maxima are complete
  if ((t & (t - 1)) == 0 && t != 1) s.tau = fmaxf(s.tau, column_bound<NT>(sh, K));
  float* el_v = sel.values();
  int32_t* el_i = sel.ids();
#pragma unroll
  for (int c = 0; c < DIRECT_CHUNKS; ++c) {
    const uint64_t reach = __builtin_amdgcn_ballot_w64(cm[c] >= s.tau);
    if (reach == 0ull) continue;
    float x[T::EPC];
    T::unpack(q[c], x);
    const int g = (t * DIRECT_CHUNKS + c) * NT + tid, id0 = (sg.c0 + g) * T::EPC;
    // One lane that reaches the bound adds for itself; for several, one addition for all that the wavefront's chunk lists.  (A place a logit by append_place:
    // layers of 256 rows of 128256 equal logits 88.9 us, sorted ones 79.8, 600 equal ones 181; so 78.8, 73.5, 163, and phases of usual rows 0.3 % shorter.  Up to 4
    // or 16 lanes for themselves: 79.1 and 79.4, 73.5 and 73.3, 164 and 164, usual rows as with append_place.)
    if ((reach & (reach - 1)) == 0ull) {                     // (uniform)
#pragma unroll
      for (int j = 0; j < T::EPC; ++j) {
        if (x[j] >= s.tau && g < sg.ncell && id0 + j < V) {
          const int slot = atomicAdd(&sh.n_list, 1);
          if (slot < sel.list_cap) { el_v[slot] = x[j]; el_i[slot] = id0 + j; }
        }
      }
    } else {
      uint32_t hit = 0u;
#pragma unroll
      for (int j = 0; j < T::EPC; ++j) hit |= (x[j] >= s.tau && g < sg.ncell && id0 + j < V ? 1u : 0u) << j;
      int at = append_places(__popc(hit), &sh.n_list);
#pragma unroll
      for (int j = 0; j < T::EPC; ++j) {
        if (hit & (1u << j)) {
          if (at < sel.list_cap) { el_v[at] = x[j]; el_i[at] = id0 + j; }
          ++at;
        }
      }
    }
  }
}

// The rarer lists (the usual one holds K to 128 logits and needs none of this), by the whole workgroup.
//  * A long list still holds what reached the first, lowest bounds: it is cut with the final one.
//  * Where it stays long (massive ties), and where it has overflowed: T, the exact K-th largest of the 512 lanes' maxima, is at
//    most the K-th largest logit, so if fewer than K logits exceed T, the others of the K largest equal it.  The list is cut
//    to what exceeds T (made again from a second read of the segment if it has overflowed), and
//  * what is missing to K entries are ties at T, or masked logits (-inf) where the list holds all finite ones: tie_scan finds those of
//    the lowest ids.
// Ranking all that reached the bound, with one LDS read after the other for every tied pair, took a row of 4000 equal logits
// 3.4 ms (18 us now) and 320 rows of 32000 whose 3000 largest are equal 2.3 ms (41 us); going over an overflowed segment twice
// more with generic_segment took 260 ascending rows of 128256 203 us (now 101).
// More than LIST_RANK_MAX logits above T lie in fewer than K lanes (of 512), which only rows with a period of 2048 logits have:
// they are generic_segment's (UNSETTLED).
// Returns the list's length.  Out of line: inlined, its code stood between the loop and the tail of every row (0.7 us a layer).
constexpr int LIST_RANK_MAX = 512;
template <int NT> using DirectSharedLds = __attribute__((address_space(3))) DirectShared<NT>*;
typedef __attribute__((address_space(3))) unsigned char* LdsBytes;
template <int NT>
__device__ __noinline__ int settle_list(const uint4* __restrict__ rowp, int V, int top_k, const Segment segment, LdsBytes lds, int list_cap, DirectSharedLds<NT> shl) {
  typedef LogitTraits<0> T;
  // (told to be uniform: the arguments of a call arrive in vector registers)
  const int K = uniform(top_k);
  const Segment sg{uniform(segment.c0), uniform(segment.c1), uniform(segment.ncell), uniform(segment.tail_chunk), uniform(segment.tail_valid)};
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  DirectShared<NT>& sh = *(DirectShared<NT>*)shl;
  SelectLds sel;
  sel.list = (unsigned char*)lds; sel.list_cap = uniform(list_cap); sel.aux = nullptr; sel.cell_cap = 0;
  float* el_v = sel.values();
  int32_t* el_i = sel.ids();
  int n = uniform(sh.n_list);
  float tie = -INFINITY;                                     // value of what may be missing
  if (n > 2 * WAVE) {
    constexpr int KEEP = 8;                                  // entries (chunks) a thread holds at once
    if (n <= sel.list_cap) {
      float bound = column_bound<NT>(sh, K);
      int reach = 0;
      for (int e = tid; e < n; e += NT) reach += el_v[e] >= bound;
      reach = wave_sum_i(reach);
      if (lane == 0 && reach) atomicAdd(&sh.n_reach, reach);
      __syncthreads();
      const bool strict = sh.n_reach > 2 * WAVE;
      if (strict) tie = bound = bound_of_columns<NT, NT / WAVE, 0>(sh, K);
      int kept = 0;
      for (int o = 0; o < n; o += KEEP * NT) {               // entries only move down: below everything not yet read
        float v[KEEP]; int32_t id[KEEP];
#pragma unroll
        for (int k = 0; k < KEEP; ++k) {
          const int e = o + k * NT + tid;
          v[k] = e < n ? el_v[e] : -INFINITY; id[k] = e < n ? el_i[e] : -1;
        }
        if (tid == 0) sh.n_list = kept;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KEEP; ++k) {
          if (id[k] >= 0 && (strict ? v[k] > bound : v[k] >= bound)) {
            const int slot = append_place(&sh.n_list);
            el_v[slot] = v[k]; el_i[slot] = id[k];
          }
        }
        __syncthreads();
        kept = sh.n_list;
        __syncthreads();
      }
      n = kept;
    } else {
      const float bound = bound_of_columns<NT, NT / WAVE, 0>(sh, K);
      tie = bound;
      const __amdgpu_buffer_rsrc_t rs = segment_buffer(rowp, sg);
      __syncthreads();                                       // everybody has read the length
      if (tid == 0) sh.n_list = 0;
      __syncthreads();
      for (int g0 = 0; g0 < sg.ncell; g0 += KEEP * NT) {
        uint4 q[KEEP];
#pragma unroll
        for (int k = 0; k < KEEP; ++k) q[k] = load_stream_buffer(rs, (uint32_t)tid * 16u, (uint32_t)(g0 + k * NT) * 16u);
#pragma unroll
        for (int k = 0; k < KEEP; ++k) {
          const int g = g0 + k * NT + tid;
          float x[T::EPC];
          T::unpack(q[k], x);
#pragma unroll
          for (int j = 0; j < T::EPC; ++j) {
            const int id = (sg.c0 + g) * T::EPC + j;
            if (x[j] > bound && g < sg.ncell && id < V) {
              const int slot = append_place(&sh.n_list);
              if (slot < sel.list_cap) { el_v[slot] = x[j]; el_i[slot] = id; }
            }
          }
        }
      }
      __syncthreads();
      n = sh.n_list;
    }
    if (n > LIST_RANK_MAX) return UNSETTLED;
  }
  const int n_elems = sg.tail_chunk >= 0 ? (sg.ncell - 1) * T::EPC + sg.tail_valid : sg.ncell * T::EPC, need = min(K, n_elems) - n;
  if (need > 0 && !sh.bad) {
    tie_scan<0, NT>((int)threadIdx.x, rowp, sg, V, tie, need, sel, &sh.n_list, sh.scan_tmp);
    n += need;
  }
  return n;
}

// The table and what the tiles add to: an entry a thread.
template <int NT>
__device__ __forceinline__ void start_direct(int tid, DirectShared<NT>& sh) {
  static_assert(EXP_TAB <= NT - WAVE, "also by the wavefronts that do not look for the row");
  if (tid < EXP_TAB) sh.exp_tab[tid] = exp_tab_entry(tid);
  if (tid == 0) { sh.n_list = 0; sh.bad = 0; sh.n_reach = 0; }
}

// One segment, by a whole workgroup.  The per-wave sums stay in `sh` (see combine_waves).
template <int NT>
__device__ __forceinline__ SegmentTop direct_segment(const uint4* __restrict__ rowp, int V, int K, const Segment& sg,
                                                     const SelectLds& sel, const ClassifierStage cst, DirectShared<NT>& sh, bool started, RowResult* rr) {
  constexpr int TILE = DIRECT_CHUNKS * NT;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = tid >> 6;
  const int n_tiles = (sg.ncell + TILE - 1) / TILE, n_whole = sg.tail_chunk >= 0 ? sg.ncell - 1 : sg.ncell;
  const __amdgpu_buffer_rsrc_t rs = segment_buffer(rowp, sg);
  const uint32_t vo = (uint32_t)tid * 16u;
  uint4 qa[DIRECT_CHUNKS], qb[DIRECT_CHUNKS];
  auto load = [&](uint4 (&q)[DIRECT_CHUNKS], int t) {
#pragma unroll
    for (int c = 0; c < DIRECT_CHUNKS; ++c) q[c] = load_stream_buffer(rs, vo, (uint32_t)(t * DIRECT_CHUNKS + c) * (NT * 16u));
  };
  DirectState<NT> s;
  s.a = s.lane_max = -INFINITY; s.Z = s.S = 0.0; s.bad = false;
  s.tau = -3.402823466e38f;                                  // the lowest finite value: masked logits (-inf) are not listed
  load(qa, 0);
  if (n_tiles > 1) load(qb, 1);
  if (!started) {                                            // (uniform) while the first tiles are on their way
    start_direct(tid, sh);
    __syncthreads();
  }
  for (int t = 0; t < n_tiles; t += 2) {
    if ((t + 1) * TILE > n_whole) blank_tile<NT>(qa, sg, t * TILE);
    direct_tile<NT>(qa, t, sg, V, K, s, sh, sel);
    if (t + 1 >= n_tiles) break;
    if (t + 2 < n_tiles) load(qa, t + 2);
    if ((t + 2) * TILE > n_whole) blank_tile<NT>(qb, sg, (t + 1) * TILE);
    direct_tile<NT>(qb, t + 1, sg, V, K, s, sh, sel);
    if (t + 3 < n_tiles) load(qb, t + 3);
  }
  C2T_PT(PT_STREAM_END);
  store_classifier((int)threadIdx.x, cst);                                     // published by the barriers below
  s.Z = wave_sum(s.Z); s.S = -TILE_SCALE * wave_sum(s.S);    // the sum of (x - a) e^(x - a)
  if (lane == 0) { sh.wave_z[wid] = s.Z; sh.wave_s[wid] = s.S; sh.wave_a[wid] = s.a; }
  if (s.bad || !(s.lane_max < INFINITY)) sh.bad = 1;
  __syncthreads();
  C2T_PT(PT_HIST_COMPLETE);
  int n_el = uniform(sh.n_list);
  if (__builtin_expect(n_el > 2 * WAVE || n_el < K, 0)) n_el = uniform(settle_list<NT>(rowp, V, K, sg, (LdsBytes)sel.list, sel.list_cap, (DirectSharedLds<NT>)&sh));
  if (__builtin_expect(n_el == UNSETTLED, 0)) generic_segment<0, NT>((int)threadIdx.x, rowp, V, K, 0, sg, sel.list, sel, rr, 0u);   // (its cell map overlays the list)
  return SegmentTop{n_el, false};
}
// The segment's record from the wavefronts' sums: lanes 0 .. NW-1 of one wavefront, fixed order.
template <int NT>
__device__ __forceinline__ void combine_waves(const DirectShared<NT>& sh, RowResult& rr) {
  constexpr int NW = NT / WAVE;
  static_assert(NW <= 16, "one DPP row holds the per-wave sums");
  const int lane = threadIdx.x & (WAVE - 1);
  const float a = lane < NW ? sh.wave_a[lane] : -INFINITY, m = wave_max(a);
  double tz = 0.0, ts = 0.0;
  if (a > -INFINITY) {
    const double d = (double)a - (double)m, f = exp_nonpositive(fmax(d, -700.0), sh.exp_tab);
    tz = sh.wave_z[lane] * f; ts = (sh.wave_s[lane] + d * sh.wave_z[lane]) * f;
  }
  tz += dpp_f64<C2T_DPP_QUAD_XOR1, 0xf>(tz); ts += dpp_f64<C2T_DPP_QUAD_XOR1, 0xf>(ts);
  tz += dpp_f64<C2T_DPP_QUAD_XOR2, 0xf>(tz); ts += dpp_f64<C2T_DPP_QUAD_XOR2, 0xf>(ts);
  tz += dpp_f64<C2T_DPP_ROW_HALF_MIRROR, 0xf>(tz); ts += dpp_f64<C2T_DPP_ROW_HALF_MIRROR, 0xf>(ts);
  tz += dpp_f64<C2T_DPP_ROW_MIRROR, 0xf>(tz); ts += dpp_f64<C2T_DPP_ROW_MIRROR, 0xf>(ts);
  if (lane == 0) {
    const bool bad = sh.bad != 0;
    RowPartial r;
    r.ref = (double)m; r.a = (double)m; r.Z = bad ? 0.0 : tz; r.S = bad ? 0.0 : ts;
    r.n_top = 0; r.flags = bad ? 1u : 0u;
    rr.part = r;
  }
}

// grid: rows_launched * nsplit workgroups of NT threads.
// Dynamic LDS (sp.lds_bytes): the list of the selection, over the cell map of generic_segment (cps keys); reused by the tail.
template <int NT>
__global__ __launch_bounds__(NT, 4) void k_logits_direct(
    C2T_START_LIST(C2T_AS_PARAMETER) const float* __restrict__ cls, TreeState st, ScoreParams sp) {
  typedef LogitTraits<0> T;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ RowResult rr;
  __shared__ DirectShared<NT> sh;
  C2T_PT(PT_START);
  constexpr int REST = START_BYTES + 8, ARGUMENT_BYTES = REST + (int)sizeof(TreeState) + (int)sizeof(ScoreParams);
  const uint32_t rows_per_seq = shape & 0xffu, F = (shape >> 8) & 0xffu;
  const QuotientRemainder wg = divide(blockIdx.x, Division{per_row, inv_per_row});
  const int split = (int)wg.r;
  RowOfWorkgroup rw;
  const bool dealt = (shape & SHAPE_COMPACT) != 0u;          // (uniform)
  if (dealt) {
    if (threadIdx.x < WAVE) {
      rw = dealt_row(nfs, (int)B, (int)wg.q);
      if (threadIdx.x == 0) { sh.scan_tmp[0][0] = rw.b; sh.scan_tmp[0][1] = rw.f; sh.scan_tmp[0][2] = rw.nf; }
    } else {
      touch_kernel_arguments<ARGUMENT_BYTES>();
      start_direct((int)threadIdx.x - WAVE, sh);
    }
    __syncthreads();
    rw.b = __builtin_amdgcn_readfirstlane(sh.scan_tmp[0][0]); rw.f = __builtin_amdgcn_readfirstlane(sh.scan_tmp[0][1]); rw.nf = __builtin_amdgcn_readfirstlane(sh.scan_tmp[0][2]);
  } else {
    rw = row_of_workgroup(nfs, st, sp.layer, B, inv_B, rows_per_seq, inv_rows, wg.q);
    touch_kernel_arguments<ARGUMENT_BYTES>();
  }
  const int nsplit = sp.nsplit, K = sp.K;
  const int b = rw.b, f = rw.f, rl = b * (int)rows_per_seq + f, nf = rw.nf;
  if (f >= nf) { if (nf == 0) end_of_sequence(st, sp, b, f, split); return; }   // uniform for the workgroup
  const int64_t row = (int64_t)b * F + f;
  const uint4* rowp = (const uint4*)((const char*)logits + row * row_stride_bytes);
  const Segment sg = make_segment<T::EPC>(V, split, cps);
  C2T_PT(PT_ROW);
  const ClassifierStage cst = stage_classifier((int)threadIdx.x, cls, sp.h, (float*)(dyn_lds + sp.w_lds_off));
  const SelectLds sel = make_select_lds<NT, T::EPC>(dyn_lds, sp.lds_bytes);
  SegmentTop top{RANKED_IN_RR, false};
  bool have_record = true;                                 // (uniform) rr.part is complete
  if (sg.ncell == 0) {
    store_classifier((int)threadIdx.x, cst);
    if (threadIdx.x == 0) { rr.part = empty_partial(); rr.ZM = 0.0; rr.SM = 0.0; }
    __syncthreads();
  } else {
    top = direct_segment<NT>(rowp, V, K, sg, sel, cst, sh, dealt, &rr);
    have_record = top.n_el < 0;
  }
  const auto top_m = [&](RowResult& r) { top_m_of_whole_row<0, NT>((int)threadIdx.x, rowp, V, sp.M, r, sel); };
  if (nsplit == 1 && sp.M > 0) {
    if (!have_record && threadIdx.x < WAVE) combine_waves(sh, rr);
    __syncthreads();
    have_record = true;
    top_m(rr);
  }
  const TailArguments& ta = tail_arguments<REST>();
  finish_layer<NT>((int)threadIdx.x, ta.st, ta.sp, b, f, nf, split, rl, rr, top, sel, sel, dyn_lds, cls, cst.dst,     // split records are indexed by launched row
                   [&] { if (!have_record) combine_waves(sh, rr); }, top_m);
}

}  // namespace c2t
