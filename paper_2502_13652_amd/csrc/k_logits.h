// Logits pass: one read of a logits row (or of one split of it) gives the softmax
// normaliser, the entropy sums (Eq. 2, first line) and the K largest logits with their
// token ids (Sec. 4.2.2, TopK purpose 1).
//
// Layout: a row is a sequence of 16-byte chunks (8 bf16 or 4 fp32 logits).  Workgroup
// (row, split) owns a contiguous range of chunks; lane t reads chunks t, t+NT, t+2NT, ...
// of that range, so every load instruction of the workgroup covers NT*16 contiguous bytes.
//
// Why the sums are exact.  Which children survive the two prunings is decided by comparing
// classifier logits that are often only an ulp apart (siblings with tiny joint probability
// share H and d), so the features must round to the same fp32 values as an fp64 evaluation
// of the definition: fp32 exponentials are not enough.  These paths deliver fp64-grade sums:
//  * bf16 rows (the fast path): a bf16 logit has at most 65536 values, and all logits of
//    practical rows lie in 32 binades, |x| in [2^-25, 2^7).  The streaming loop only COUNTS
//    values: one LDS atomic per element into an 8192-bin histogram (sign, 5 exponent bits,
//    7 mantissa bits; two 16-bit counters per LDS word, overflow detected through the total).
//    Afterwards Z = sum_v n_v e^v and S = sum_v n_v (v-m) e^v are formed in fp64 from small
//    tables of exponentials: exact counts, <= 8192 fp64 terms, independent of the order in which
//    the elements were read.  Logits below the window (zeros included) are counted apart:
//    e^x = 1 + x to fp64 accuracy for |x| < 2^-25.  So are masked logits, -inf or a finite
//    x <= -2^10 (the masked tokens of constrained decoding): they add exactly nothing to either
//    sum and rank after every window value.
//  * bf16 rows holding a logit >= 2^7 or in (-2^10, -2^7], +inf or a NaN, a value held by more than
//    65535 logits, or below-window or masked logits that could rank among the K largest: two passes over the segment with
//    fp64 exponentials per element (generic_segment).
//  * fp32 rows: one pass with an fp64 exponential per element (k_direct.h).
//
// Top-K without data-dependent work in the streaming loop: the loop records the maximum of each
// cell of four chunks as a "cell key" in an LDS map.  On the histogram path a cell is four neighbouring chunks (64 bytes); on the
// two-pass path it is the four chunks a lane reads in four consecutive sweeps of the workgroup (chunks i, i+NT, i+2NT, i+3NT of the segment).
// Afterwards a bound tau <= K-th largest logit is known (from the maxima of columns of lanes, or exactly, from the histogram),
// only cells whose key reaches tau can hold a top-K element, and
// those few cells are re-read and their elements ranked exactly by (logit desc, id asc).
#pragma once
#include "k_common.h"
#include "k_tree.h"

namespace c2t {

#ifndef C2T_TAU_LOW_BIT
#define C2T_TAU_LOW_BIT 16
#endif

template <int DT> struct LogitTraits;
template <> struct LogitTraits<1> {     // bf16
  static constexpr int EPC = 8;         // elements per 16-byte chunk
  typedef uint16_t key_t;
  static __device__ __forceinline__ void unpack(const uint4& q, float (&x)[8]) {
    x[0] = bf16_lo(q.x); x[1] = bf16_hi(q.x); x[2] = bf16_lo(q.y); x[3] = bf16_hi(q.y);
    x[4] = bf16_lo(q.z); x[5] = bf16_hi(q.z); x[6] = bf16_lo(q.w); x[7] = bf16_hi(q.w);
  }
  static __device__ __forceinline__ key_t to_key(float cm) { return (key_t)(__float_as_uint(cm) >> 16); }
  static __device__ __forceinline__ float from_key(key_t k) { return __uint_as_float((uint32_t)k << 16); }
};
template <> struct LogitTraits<0> {     // fp32
  static constexpr int EPC = 4;
  typedef float key_t;
  static __device__ __forceinline__ void unpack(const uint4& q, float (&x)[4]) {
    x[0] = __uint_as_float(q.x); x[1] = __uint_as_float(q.y);
    x[2] = __uint_as_float(q.z); x[3] = __uint_as_float(q.w);
  }
  static __device__ __forceinline__ key_t to_key(float cm) { return cm; }
  static __device__ __forceinline__ float from_key(key_t k) { return k; }
};

// A logits chunk is read once per layer, but for the cells that hold one of the row's largest.  STREAMED: a non-temporal load keeps the
// stream from evicting what the workgroups reuse (the e^v table, the classifier) from the L2.  Launches of at most one workgroup a CU
// whose rows fit the L2s, and shared rows, read with the usual policy: the cells are still there when they are read again (phases: one sequence of 128256
// 123.5 -> 121.1 us, four of 20011 with 64 rows each 261.7 -> 258.2; 256 rows of 128256 a layer, 64 MB, 177.3 -> 178.9: those are STREAMED).
typedef uint32_t c2t_uint4v __attribute__((ext_vector_type(4)));
// 16 bytes at descriptor base + lane offset + scalar offset; zeros past the descriptor's size
template <bool STREAMED = true>
__device__ __forceinline__ uint4 load_stream_buffer(__amdgpu_buffer_rsrc_t rs, uint32_t lane_off, uint32_t scalar_off) {
  const c2t_uint4v v = __builtin_amdgcn_raw_buffer_load_b128(rs, lane_off, scalar_off, STREAMED ? 2 : 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 load_stream(const uint4* p) {
  const c2t_uint4v v = __builtin_nontemporal_load((const c2t_uint4v*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Range of chunks a (row, split) workgroup owns.
struct Segment {
  int c0, c1;        // chunks [c0, c1)
  int ncell;         // c1 - c0
  int tail_chunk;    // index of the row's last, partially valid chunk if it lies in [c0,c1), else -1
  int tail_valid;    // its number of valid elements
};
template <int EPC>
__device__ __forceinline__ Segment make_segment(int V, int split, int cps) {
  Segment s;
  const int n_chunks = (V + EPC - 1) / EPC;
  s.c0 = min(split * cps, n_chunks);
  s.c1 = min(s.c0 + cps, n_chunks);
  s.ncell = s.c1 - s.c0;
  s.tail_valid = V - (n_chunks - 1) * EPC;
  s.tail_chunk = (s.c1 == n_chunks && s.tail_valid != EPC && s.ncell > 0) ? n_chunks - 1 : -1;
  return s;
}

// Cells of a segment of n chunks, CPC chunks each: sweep s of the workgroup reads chunks [s*NT, (s+1)*NT);
// cell (s/4)*NT + t holds the chunks that lane t reads in sweeps 4*(s/4) .. 4*(s/4)+3.
template <int NT>
__host__ __device__ inline int cells_in_segment(int n) {
  const int full = n / (4 * NT), rem = n - full * 4 * NT;
  return full * NT + (rem < NT ? rem : NT);
}
// chunk j (0 <= j < CPC) of a cell, as an index into the segment; may lie past its end
template <int NT>
__device__ __forceinline__ int chunk_of_cell(int cell, int j) {
  const int grp = cell / NT, t = cell - grp * NT;
  return grp * 4 * NT + j * NT + t;
}

// Cells of the histogram path: four neighbouring chunks, 64 bytes of one or two lines, so that one which holds a large logit is read again at
// the price of its lines (a cell of four chunks of one lane, four sweeps apart, costs four: with K = 32
// 4096 rows of 152064 took 255 us a layer, with K = 1 193).  Cell g * NT + t of a segment: chunks (4 g + t mod 4) * NT + t - t mod 4 and the next three; a group g of four sweeps has NT cells.
template <int NT>
__host__ __device__ inline int quad_cells_in_segment(int n) { return (n + 4 * NT - 1) / (4 * NT) * NT; }
template <int NT>
__device__ __forceinline__ int chunk_of_quad_cell(int cell, int j) {
  const int grp = cell / NT, t = cell - grp * NT;
  return (grp * 4 + (t & 3)) * NT + (t & ~3) + j;
}

// ---------------------------------------------------------------------------------------
// Selection, shared by both paths.
// ---------------------------------------------------------------------------------------

// Cells whose key reaches tau (exceeds it, if strict) are pushed to cell_list, in any order.
// Returns how many there are; if that is more than cell_cap the list is incomplete.  Ends with a barrier behind the read of the count, which callers
// set to 0 again: a wavefront that read it late took none of the cells, or the other side of a branch with barriers in it.
template <int DT, int NT>
__device__ __forceinline__ int list_cells(int tid, const typename LogitTraits<DT>::key_t* map, int ncells, float tau, bool strict,
                                          int cell_cap, int32_t* cell_list, int32_t* sh_n) {
  typedef LogitTraits<DT> T;
  if (tid == 0) *sh_n = 0;
  __syncthreads();
#pragma unroll 1
  for (int c = tid; c < ncells; c += NT) {
    const float kv = T::from_key(map[c]);
    if (strict ? kv > tau : kv >= tau) {
      const int slot = append_place(sh_n);
      if (slot < cell_cap) cell_list[slot] = c;
    }
  }
  __syncthreads();
  const int n = *sh_n;
  __syncthreads();
  return n;
}

// Re-read the listed cells (CPC chunks each, one chunk per thread) and append their elements that
// reach tau (exceed it, if strict) to the element list, which may overlay the cell map: the caller has
// put a barrier after the last read of the map and after setting *sh_cnt = 0.  Ends with a barrier.
// QUAD: the cells of the histogram path.
template <int DT, int NT, bool QUAD>
__device__ __forceinline__ void collect_cells(int tid, const uint4* __restrict__ rowp, int c0, int c1, int V, float tau, bool strict,
                                              const int32_t* cell_list, int n_cells, const SelectLds& sel, int32_t* sh_cnt) {
  typedef LogitTraits<DT> T;
  float* el_v = sel.values();
  int32_t* el_i = sel.ids();
  int my_chunk = -1;
  uint4 q = make_uint4(0, 0, 0, 0);
  if (tid < n_cells * CPC) {                                 // n_cells <= cell_cap <= NT / CPC
    const int ch = c0 + (QUAD ? chunk_of_quad_cell<NT>(cell_list[tid / CPC], tid % CPC) : chunk_of_cell<NT>(cell_list[tid / CPC], tid % CPC));
    if (ch < c1) { my_chunk = ch; q = rowp[ch]; }
  }
  if ((tid & ~(WAVE - 1)) < n_cells * CPC) {                 // wavefronts with a cell
    float x[T::EPC];
    T::unpack(q, x);
    uint32_t hit = 0u;
#pragma unroll
    for (int j = 0; j < T::EPC; ++j) hit |= (my_chunk >= 0 && my_chunk * T::EPC + j < V && (strict ? x[j] > tau : x[j] >= tau) ? 1u : 0u) << j;
    int slot = append_places(__popc(hit), sh_cnt);
#pragma unroll
    for (int j = 0; j < T::EPC; ++j) {
      if ((hit >> j) & 1u) {
        if (slot < sel.list_cap) { el_v[slot] = x[j]; el_i[slot] = my_chunk * T::EPC + j; }
        ++slot;
      }
    }
  }
  __syncthreads();
}

// Massive ties: append the `need` lowest-id elements equal to tau, found by sweeping the segment in
// id order (one chunk per thread and sweep, prefix counts across the workgroup) until enough are seen.
template <int DT, int NT>
__device__ __forceinline__ void tie_scan(int tid, const uint4* __restrict__ rowp, const Segment& sg, int V, float tau, int need,
                                         const SelectLds& sel, int32_t* sh_cnt, int32_t (*scan_tmp)[NT / WAVE]) {
  typedef LogitTraits<DT> T;
  constexpr int NW = NT / WAVE;
  const int lane = tid & (WAVE - 1), wid = tid >> 6;
  float* el_v = sel.values();
  int32_t* el_i = sel.ids();
  int found = 0;                                             // uniform
#pragma unroll 1
  for (int base = sg.c0; base < sg.c1 && found < need; base += NT) {
    const int g = base + tid;
    uint32_t hit = 0;
    if (g < sg.c1) {
      float x[T::EPC];
      T::unpack(rowp[g], x);
#pragma unroll
      for (int j = 0; j < T::EPC; ++j) hit |= (g * T::EPC + j < V && x[j] == tau ? 1u : 0u) << j;
    }
    const int cnt = __popc(hit);
    const int incl = wave_scan_incl(cnt);
    if (lane == WAVE - 1) scan_tmp[0][wid] = incl;
    __syncthreads();
    int before = found + incl - cnt, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { if (w < wid) before += scan_tmp[0][w]; total += scan_tmp[0][w]; }
    while (hit && before < need) {
      const int j = __ffs(hit) - 1; hit &= hit - 1;
      const int slot = append_place(sh_cnt);
      if (slot < sel.list_cap) { el_v[slot] = tau; el_i[slot] = g * T::EPC + j; }
      ++before;
    }
    found += total;
    __syncthreads();
  }
}

// Sum of Z and S over the workgroup in a fixed order (wave butterflies, then waves ascending).
// Only thread 0 needs the totals: it leaves them in out[0..1] (LDS), so no lane keeps the
// per-wave partials alive in registers.
template <int NT>
__device__ __forceinline__ void block_sum2(int tid, double Z, double S, double (*red)[NT / WAVE], double* out) {
  constexpr int NW = NT / WAVE;
  Z = wave_sum(Z); S = wave_sum(S);
  if ((tid & (WAVE - 1)) == 0) { red[0][tid >> 6] = Z; red[1][tid >> 6] = S; }
  __syncthreads();
  if (tid == 0) {
    double tz = 0.0, ts = 0.0;
#pragma unroll 1
    for (int w = 0; w < NW; ++w) { tz += red[0][w]; ts += red[1][w]; }
    out[0] = tz; out[1] = ts;
  }
}
template <int NT>
__device__ __forceinline__ float block_max(int tid, float v, float* red /*[NT/WAVE]*/) {
  constexpr int NW = NT / WAVE;
  v = wave_max(v);
  __syncthreads();
  if ((tid & (WAVE - 1)) == 0) red[tid >> 6] = v;
  __syncthreads();
  float t = red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) t = fmaxf(t, red[w]);
  return t;
}

// ---------------------------------------------------------------------------------------
// Generic path: two passes over the segment, fp64 exponentials.  Any dtype, any values.
// ---------------------------------------------------------------------------------------
// Sums of e^(x-m) and (x-m) e^(x-m) over the M largest logits of the segment (ties at the M-th
// value: any of the equal logits, they contribute the same).  The M-th largest value is found
// exactly by a radix select over the order-preserving 32-bit keys, 8 bits per pass over the segment
// (an LDS histogram of the digit among the elements that match the prefix so far); one more pass
// sums the terms above it.  out[0..1] in LDS, valid after the caller's next barrier.
template <int DT, int NT>
__device__ __forceinline__ void top_m_sums(int tid, const uint4* __restrict__ rowp, const Segment& sg, int M, float m,
                                           double (*red)[NT / WAVE], double* out, uint32_t* dig /*[256]*/) {
  typedef LogitTraits<DT> T;
  __shared__ int32_t sh_digit, sh_above, sh_total;
  const int lane = tid & (WAVE - 1);
  uint32_t prefix = 0, care = 0;
  int remaining = M;
  bool take_all = false;
#pragma unroll 1
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int i = tid; i < 256; i += NT) dig[i] = 0u;
    __syncthreads();
    for (int g = sg.c0 + tid; g < sg.c1; g += NT) {
      float x[T::EPC];
      T::unpack(rowp[g], x);
      const int nv = (g == sg.tail_chunk) ? sg.tail_valid : T::EPC;
#pragma unroll
      for (int j = 0; j < T::EPC; ++j) {
        const uint32_t key = sortable_key(x[j]);
        if (j < nv && (key & care) == prefix) atomicAdd(&dig[(key >> shift) & 255u], 1u);
      }
    }
    __syncthreads();
    if (tid < WAVE) {                                        // wave 0: lane l owns digits 255-4l .. 252-4l
      uint32_t c[4]; int tot = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) { c[j] = dig[255 - (4 * lane + j)]; tot += (int)c[j]; }
      const int incl = wave_scan_incl(tot);
      int run = incl - tot;                                  // elements with larger digits
      if (run < remaining && incl >= remaining) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (run < remaining && run + (int)c[j] >= remaining) { sh_digit = 255 - (4 * lane + j); sh_above = run; }
          run += (int)c[j];
        }
      }
      if (lane == WAVE - 1) sh_total = incl;
    }
    __syncthreads();
    if (sh_total < remaining) { take_all = true; break; }   // fewer matching elements than wanted: only in the first pass
    remaining -= sh_above;
    prefix |= (uint32_t)sh_digit << shift; care |= 255u << shift;
    __syncthreads();
  }
  // prefix = key of the M-th largest logit; `remaining` (>= 1) of the logits equal to it are taken
  double Z = 0.0, S = 0.0;
  const double md = (double)m;
  for (int g = sg.c0 + tid; g < sg.c1; g += NT) {
    float x[T::EPC];
    T::unpack(rowp[g], x);
    const int nv = (g == sg.tail_chunk) ? sg.tail_valid : T::EPC;
#pragma unroll
    for (int j = 0; j < T::EPC; ++j) {
      if (j < nv && x[j] > -INFINITY && (take_all || sortable_key(x[j]) > prefix)) {
        const double t = (double)x[j] - md, e = exp(t);
        Z += e;
        if (e > 0.0) S += t * e;
      }
    }
  }
  if (!take_all && tid == 0) {
    const float xt = key_to_float(prefix);
    if (xt > -INFINITY) { const double t = (double)xt - md, e = exp(t); Z += remaining * e; if (e > 0.0) S += remaining * (t * e); }
  }
  block_sum2<NT>(tid, Z, S, red, out);
}

// The sums over the M largest logits of a whole row, by one workgroup in five passes: every fp32 row with M > 0 (its one pass does
// not find them), and rows that were split (they cannot be told from the splits' own sums), by the workgroup that merged the
// row.  Sums relative to the row maximum.
template <int DT, int NT>
__device__ __forceinline__ void top_m_of_whole_row(int tid, const uint4* __restrict__ rowp, int V, int M, RowResult& rr, const SelectLds& sel) {
  if (M <= 0) return;
  __shared__ double red_t[2][NT / WAVE], sum_t[2];
  const bool usable = !(rr.part.flags & 1u) && rr.part.Z > 0.0 && rr.part.ref > -INFINITY && rr.part.ref < INFINITY;
  if (usable) {
    constexpr int EPC = LogitTraits<DT>::EPC;
    const Segment whole = make_segment<EPC>(V, 0, (V + EPC - 1) / EPC);
    top_m_sums<DT, NT>(tid, rowp, whole, M, (float)rr.part.ref, red_t, sum_t, (uint32_t*)sel.aux);
  }
  __syncthreads();
  if (tid == 0) { rr.ZM = usable ? sum_t[0] : 0.0; rr.SM = usable ? sum_t[1] : 0.0; }
  __syncthreads();
}

// map_lds: one key per cell.
template <int DT, int NT>
__device__ __noinline__ void generic_segment(int tid, const uint4* __restrict__ rowp, int V, int K, int top_m, const Segment sg,
                                unsigned char* map_lds, const SelectLds sel, RowResult* rr, uint32_t info_flags) {
  typedef LogitTraits<DT> T;
  typedef typename T::key_t key_t;
  constexpr int NW = NT / WAVE;
  static_assert(CPC == 4, "a cell is four sweeps of a lane");
  key_t* map = (key_t*)map_lds;
  const int ncells = cells_in_segment<NT>(sg.ncell);
  __shared__ double red_d[2][NW], sum_d[2], sum_m[2];
  __shared__ float red_f[NW];
  uint32_t* const lane_keys = (uint32_t*)sel.aux;           // [NT]
  int32_t* const cell_list = (int32_t*)(lane_keys + NT);    // [SEL_CELL_CAP]; before the cells are listed: the digits of top_m_sums
  static_assert(NT * 4 + SEL_CELL_CAP * 4 == SEL_AUX_BYTES && SEL_CELL_CAP == 256, "they fill the place");
  __shared__ int32_t scan_tmp[2][NW];
  __shared__ uint32_t sh_tau;
  __shared__ int32_t sh_cnt, sh_bad;
  const int lane = tid & (WAVE - 1), wid = tid >> 6;
  if (tid == 0) sh_bad = 0;
  __syncthreads();

  // pass 1: cell keys, lane maxima, NaN / +inf
  float M = -INFINITY;
  bool bad = false, any = false;
  float cell_max = -INFINITY;
  int sweep = 0;
  for (int g = sg.c0 + tid; g < sg.c1; g += NT, ++sweep) {
    const uint4 q = rowp[g];
    float x[T::EPC];
    T::unpack(q, x);
    const int nv = (g == sg.tail_chunk) ? sg.tail_valid : T::EPC;
    float cm = -INFINITY;
#pragma unroll
    for (int j = 0; j < T::EPC; ++j) {
      if (j < nv) { bad |= !(x[j] < INFINITY); cm = fmaxf(cm, x[j]); }
    }
    M = fmaxf(M, cm);
    cell_max = fmaxf(cell_max, cm);
    if ((sweep & 3) == 3 || g + NT >= sg.c1) { map[(sweep >> 2) * NT + tid] = T::to_key(cell_max); cell_max = -INFINITY; }
    any = true;
  }
  lane_keys[tid] = any ? sortable_key(M) : 0u;
  if (bad) sh_bad = 1;
  const float m = block_max<NT>(tid, M, red_f);          // barriers inside also publish map, lane_keys, sh_bad
  const bool seg_bad = sh_bad != 0;
  C2T_PT(PT_STREAM_END);                            // (the marks of the histogram path, at the corresponding steps)

  // pass 2: Z = sum e^(x-m), S = sum (x-m) e^(x-m)
  double Z = 0.0, S = 0.0;
  if (!seg_bad && m > -INFINITY) {
    const double md = (double)m;
    for (int g = sg.c0 + tid; g < sg.c1; g += NT) {
      const uint4 q = rowp[g];
      float x[T::EPC];
      T::unpack(q, x);
      const int nv = (g == sg.tail_chunk) ? sg.tail_valid : T::EPC;
#pragma unroll
      for (int j = 0; j < T::EPC; ++j) {
        if (j < nv && x[j] > -INFINITY) {
          const double t = (double)x[j] - md;
          const double e = exp(t);
          Z += e;
          if (e > 0.0) S += t * e;
        }
      }
    }
  }
  block_sum2<NT>(tid, Z, S, red_d, sum_d);
  C2T_PT(PT_SUMS);
  if (top_m > 0) {
    __syncthreads();
    if (!seg_bad && m > -INFINITY) top_m_sums<DT, NT>(tid, rowp, sg, top_m, m, red_d, sum_m, (uint32_t*)cell_list);
    else if (tid == 0) { sum_m[0] = 0.0; sum_m[1] = 0.0; }
    __syncthreads();
  }

  // tau = K-th largest of the lane maxima, to its upper 16 bits (half the select's steps, each a
  // ballot per key; a few more elements pass): a lower bound of the K-th largest logit
  if (wid == 0) {
    uint32_t keys[NW];
#pragma unroll
    for (int v = 0; v < NW; ++v) keys[v] = lane_keys[v * WAVE + lane];
    uint32_t t = wave_kth_largest<NW, C2T_TAU_LOW_BIT>(keys, K);
    // -inf's key with its low bits cleared is no number's key; every key that reaches it is at least -inf's
    const uint32_t key_neg_inf = 0x007FFFFFu;             // = sortable_key(-INFINITY)
    if (t != 0u && t < key_neg_inf) t = key_neg_inf;
    if (lane == 0) sh_tau = t;
  }
  __syncthreads();
  uint32_t tau_key = sh_tau;
  float tau = tau_key ? key_to_float(tau_key) : -INFINITY;
  bool ties = false;
  int n_cells = list_cells<DT, NT>(tid, map, ncells, tau, false, sel.cell_cap, cell_list, &sh_cnt);
  if (n_cells > sel.cell_cap) {
    // Too many cells reach the bound (maxima clustered in few lanes): take the exact K-th
    // largest cell key by radix select over the whole map; fewer than K cells exceed it.
    const int cpl = (ncells + NT - 1) / NT;
    const int s0 = min(tid * cpl, ncells), s1 = min(s0 + cpl, ncells);
    uint32_t prefix = 0, care = 0;
    int k = K;
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t want = prefix | (1u << bit), cmask = care | (1u << bit);
      int cnt = 0;
      for (int s = s0; s < s1; ++s) cnt += (sortable_key(T::from_key(map[s])) & cmask) == want;
      cnt = wave_sum_i(cnt);
      if (lane == 0) scan_tmp[0][wid] = cnt;
      __syncthreads();
      int tot = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) tot += scan_tmp[0][w];
      __syncthreads();
      if (tot >= k) prefix = want; else k -= tot;
      care = cmask;
    }
    tau = prefix ? key_to_float(prefix) : -INFINITY;
    n_cells = list_cells<DT, NT>(tid, map, ncells, tau, false, sel.cell_cap, cell_list, &sh_cnt);
    if (n_cells > sel.cell_cap) {                            // massive ties at tau: the cells above it, then a tie scan
      n_cells = list_cells<DT, NT>(tid, map, ncells, tau, true, sel.cell_cap, cell_list, &sh_cnt);
      ties = true;
    }
  }
  if (tid == 0) sh_cnt = 0;
  __syncthreads();
  C2T_PT(PT_CELLS_LISTED);
  collect_cells<DT, NT, false>(tid, rowp, sg.c0, sg.c1, V, tau, ties, cell_list, n_cells, sel, &sh_cnt);
  if (ties) tie_scan<DT, NT>(tid, rowp, sg, V, tau, K, sel, &sh_cnt, scan_tmp);
  C2T_PT(PT_CELLS_READ);
  const int n_el = min(sh_cnt, sel.list_cap), n_top = min(n_el, K);
  rank_list<NT>(tid, K, sel, n_el, rr->topv, rr->topi);
  if (tid == 0) {
    RowPartial r;
    r.ref = (double)m; r.a = (double)m; r.Z = sum_d[0]; r.S = sum_d[1]; r.n_top = seg_bad ? 0 : n_top; r.flags = (seg_bad ? 1u : 0u) | info_flags;
    rr->part = r;
    if (top_m > 0) { rr->ZM = sum_m[0]; rr->SM = sum_m[1]; }
  }
  __syncthreads();                                           // rr is complete
}

// Workgroups of a sequence whose frontier is empty have nothing to read; the first of them
// records the empty next frontier (Algorithm 1's loop guard) in place of the scoring step.
__device__ __forceinline__ void end_of_sequence(const TreeState& st, const ScoreParams& sp, int b, int f, int split) {
  if (f == 0 && split == 0 && threadIdx.x == 0) { st.nf[(sp.layer + 1) & 1][b] = 0; st.n_cand[b] = 0; }
}

// Which frontier slot of which sequence a workgroup (index w among the launched rows) takes.
// A launch that fits the chip in one round (at most four workgroups per CU) is placed statically:
// workgroup w runs on CU w mod n_cus (HW_ID read-outs), so a CU hosts w, w + n_cus, w + 2 n_cus, ...
// Full layers run fastest in slot-major order (consecutive workgroups = the same slot of
// consecutive sequences: 2 % faster at B = 64 and B = 256 than sequence-major).  In a thinned-out
// layer the frontiers are of very different lengths (many sequences have used their budget up,
// others are still full), and a fixed order leaves some CUs with four live rows and others with
// none: the layer then takes as long as a full one.  Such launches (SHAPE_COMPACT) deal the rows instead: the workgroup takes the w-th
// LIVE row in slot-major order, which follows from the frontier sizes alone (no atomics): the live
// rows are dealt round the CUs, at most one more on one CU than on another.  Workgroups past the
// live rows take the sequences without a frontier (one each, for the loop guard) or exit.
struct RowOfWorkgroup { int b, f, nf; };
// position of the n-th set bit of m (n < popcount(m)); uniform over the wave
__device__ __forceinline__ int nth_set_bit(uint64_t m, int n) {
  const int lane = lane_id();
  const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  const uint64_t hit = __builtin_amdgcn_ballot_w64(((m >> lane) & 1ull) != 0ull && below == n);
  return (int)__builtin_ctzll(hit);
}
// Dealt by the first wavefront for its workgroup, while the others clear its counts: lane f forms the set of sequences that have a row in slot f, from
// ballots over the bits of the frontier sizes; the slot follows from a prefix sum of their numbers.  About a hundred instructions whatever the
// shape.  (Every wavefront for itself, a scalar loop over the slots with a search in each: the last of 1024 workgroups started 4.8 us after the first,
// and a layer of 64 sequences that have ended, 1024 workgroups, took 7.1 us.)
constexpr int COMPACT_MAX_B = 256;            // frontier sizes held by one wave: four per lane
__device__ __forceinline__ RowOfWorkgroup dealt_row(const int32_t* __restrict__ nfs, int B, int w) {
  constexpr int NB = COMPACT_MAX_B / WAVE;
  static_assert(SP_MAX_F == WAVE, "a lane a slot, six bits a slot");
  const int lane = lane_id();
  int nfv[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    nfv[k] = -1;
    if (k * WAVE < B) { const int i = lane + k * WAVE, n = nfs[min(i, B - 1)]; nfv[k] = i < B ? n : -1; }
  }
  uint64_t in_slot[NB];                                    // lane f: the sequences whose frontier is longer than f
  int rows = 0;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    in_slot[k] = 0ull;
    if (k * WAVE < B) {
      const int last = nfv[k] - 1;                         // its last slot; negative: none
      uint64_t at_least = ~0ull;                           // the last slot's bits so far are at least f's
#pragma unroll
      for (int bit = 0; bit < 6; ++bit) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(((last >> bit) & 1) != 0);
        at_least = ((lane >> bit) & 1) ? at_least & m : at_least | m;
      }
      in_slot[k] = at_least & __builtin_amdgcn_ballot_w64(last >= 0);
      rows += __builtin_popcountll(in_slot[k]);
    }
  }
  const int incl = wave_scan_incl(rows);
  const uint64_t here = __builtin_amdgcn_ballot_w64(w < incl);
  const bool has_row = here != 0ull;                        // (uniform, as all that follows) else a sequence without a frontier, if there are so many
  const int f = has_row ? (int)__builtin_ctzll(here) : WAVE - 1;
  int d = w - (__builtin_amdgcn_readlane(incl, f) - (has_row ? __builtin_amdgcn_readlane(rows, f) : 0));
  RowOfWorkgroup r{0, 1, 1};                               // nothing left for this workgroup
  bool found = false;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    if (k * WAVE < B && !found) {
      const uint64_t m = has_row ? (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)in_slot[k], f) |
                                   (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(in_slot[k] >> 32), f) << 32
                                 : __builtin_amdgcn_ballot_w64(nfv[k] == 0);
      const int c = __builtin_popcountll(m);
      if (d < c) {
        const int bl = nth_set_bit(m, d);
        r.b = k * WAVE + bl; r.f = has_row ? f : 0; r.nf = __builtin_amdgcn_readlane(nfv[k], bl);
        found = true;
      }
      d -= c;
    }
  }
  return r;
}
// Rows in a fixed order.  What bounds the start of a layer is a chain of round trips ahead of the first logit: with the start's arguments in registers, the frontier size
// requested at once and the first logits before the counts are cleared, phases of one sequence are 1.05 to 1.08 times as fast.  Each part by itself, phases of the build without it over
// those of the build with it: the arguments in registers 1.041 (one sequence of 32000, bf16), 1.016 (fp32), 1.025 (128256), others 1.003 to 1.008; divisions by multiplication
// 1.000 to 1.011; the first logits ahead of the clearing 1.016 (16 masked sequences), others 1.001 to 1.006, but 0.995 (256 of 152064, whose builds differ by as much in the place of their code);
// the dealing by one wavefront 1.009 (64 of 128256), 1.003 to 1.006 (32).
__device__ __forceinline__ RowOfWorkgroup row_of_workgroup(const int32_t* __restrict__ nfs, const TreeState& st, int layer, uint32_t B, uint32_t inv_B, uint32_t rows_per_seq,
                                                           uint32_t inv_rows, uint32_t w) {
  const QuotientRemainder by_seq = divide(w, Division{rows_per_seq, inv_rows});
  RowOfWorkgroup r{(int)by_seq.q, (int)by_seq.r, 0};
  if (B == 1u || rows_per_seq == 1u) { r.nf = nfs[r.b]; return r; }                      // both orders are the same
  const QuotientRemainder by_slot = divide(w, Division{B, inv_B});
  int nf_seq = nfs[by_seq.q], nf_slot = nfs[by_slot.r], live = st.layer_rows[layer];     // all loads issued before the choice: no dependent round trip
  asm volatile("" : "+s"(nf_seq), "+s"(nf_slot));                       // (nor one load from a chosen address)
  const bool slot_major = 4u * (uint32_t)__builtin_amdgcn_readfirstlane(live) >= 3u * B * rows_per_seq;
  if (slot_major) { r.b = (int)by_slot.r; r.f = (int)by_slot.q; }
  r.nf = slot_major ? nf_slot : nf_seq;
  return r;
}

// ---------------------------------------------------------------------------------------
// bf16 fast path: value histogram.
// ---------------------------------------------------------------------------------------
constexpr int HP_BINS = 8192;                 // sign(1) | exponent mod 32 (5) | mantissa (7)
constexpr int HP_WORDS = HP_BINS / 2;         // LDS words: low half counts +|v|, high half counts -|v|
constexpr uint32_t HP_MAG_LO = 102u << 7;     // |x| >= 2^-25
constexpr uint32_t HP_MAG_SPAN = 32u << 7;    // 32 binades: |x| < 2^7
constexpr uint32_t HP_LOWEST = 0x8000u | (HP_MAG_LO + HP_MAG_SPAN - 1);  // the window's lowest value, which also stands in for masked logits
constexpr uint32_t HP_NONE2 = 0xFC00FC00u;    // identity of the packed maximum (fp16's -inf twice): a lane without a chunk

// value-ordered rank r in [0, 8192): larger r = larger value.  r -> bf16 code.
__device__ __forceinline__ uint32_t hp_code_of_rank(int r) {
  const uint32_t s = r < 4096 ? 1u : 0u;
  const uint32_t magidx = s ? (uint32_t)(4095 - r) : (uint32_t)(r - 4096);
  return (s << 15) | (HP_MAG_LO + magidx);
}
__device__ __forceinline__ float hp_value_of_mag(uint32_t magidx, bool negative) {
  return __uint_as_float(((HP_MAG_LO + magidx) << 16) | (negative ? 0x80000000u : 0u));
}

// e^v for the window's values, factored so that the table stays in cache and a lane holds few
// factors: v = s 2^E (1 + f/128), f = 16 fh + fl, and e^v = A[s][e][fh] * prod over the set bits k
// of fl of C[s][e][k], with A = exp(s 2^E (1 + fh/8)) and C = exp(s 2^E 2^k / 128) (every argument
// exact), e = exponent index inside the window (0..31).  Layout: A+ [256] | A- [256] | C+ [32][4] |
// C- [32][4] doubles (6 KB; a table of all 8192 values is 64 KB and was re-fetched from memory by
// nearly every workgroup).  At most five correctly rounded factors and four products: within
// 1e-15 of e^v.  Filled once per context.
constexpr int HP_TAB_A = 256, HP_TAB_C = 128, HP_TAB_DOUBLES = 2 * HP_TAB_A + 2 * HP_TAB_C;
__global__ void k_init_exp_table(double* __restrict__ tab) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= HP_TAB_DOUBLES) return;
  const bool is_c = i >= 2 * HP_TAB_A;
  const int k = is_c ? i - 2 * HP_TAB_A : i, half = is_c ? HP_TAB_C : HP_TAB_A;
  const bool neg = k >= half;
  const int kk = neg ? k - half : k;
  const int e = is_c ? kk >> 2 : kk >> 3, sub = is_c ? kk & 3 : kk & 7;
  const double p2 = ldexp(1.0, (int)(HP_MAG_LO >> 7) + e - 127);                 // 2^E
  const double arg = is_c ? p2 * (double)(1 << sub) / 128.0 : p2 * (1.0 + (double)sub / 8.0);
  tab[i] = exp(neg ? -arg : arg);
}
// The lane that owns magnitude indices 8t .. 8t+7 (one exponent, fh and bit 3 of fl fixed): the
// factors of e^(+|v_j|) and e^(-|v_j|).  Ten loads, twenty registers; the sixteen products are
// formed where they are used, one bin pair at a time.
struct ExpFactors { double ap, an, cp[4], cn[4]; };
__device__ __forceinline__ ExpFactors load_exp_factors(const double* __restrict__ tab, int tid) {
  const int mag0 = 8 * tid, e = mag0 >> 7, f0 = mag0 & 127;
  ExpFactors f;
  f.ap = tab[e * 8 + (f0 >> 4)]; f.an = tab[HP_TAB_A + e * 8 + (f0 >> 4)];
  const double2* cp = (const double2*)(tab + 2 * HP_TAB_A + e * 4);
  const double2* cn = (const double2*)(tab + 2 * HP_TAB_A + HP_TAB_C + e * 4);
  const double2 p0 = cp[0], p1 = cp[1], n0 = cn[0], n1 = cn[1];
  f.cp[0] = p0.x; f.cp[1] = p0.y; f.cp[2] = p1.x; f.cp[3] = p1.y;
  f.cn[0] = n0.x; f.cn[1] = n0.y; f.cn[2] = n1.x; f.cn[3] = n1.y;
  return f;
}

typedef _Float16 c2t_half2 __attribute__((ext_vector_type(2)));
typedef unsigned short c2t_ushort2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max_f16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(c2t_half2, a), __builtin_bit_cast(c2t_half2, b)));
}
// The same instruction without the canonicalising copies the builtin adds in front of it (an
// instruction per operand): for the streaming loop, whose patterns are never signalling NaNs that matter.
__device__ __forceinline__ uint32_t pk_max_f16_raw(uint32_t a, uint32_t b) {
  uint32_t d;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ uint32_t pk_max3_f16_raw(uint32_t a, uint32_t b, uint32_t c) {     // (a NaN pattern, of a logit far outside the window, wins)
  uint32_t d;
  asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
// per 16-bit half: a * b + c (mod 2^16)
__device__ __forceinline__ uint32_t pk_mad_u16(uint32_t a, uint32_t b_sgpr, uint32_t c) {
  uint32_t d;
  asm("v_pk_mad_u16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "s"(b_sgpr), "v"(c));
  return d;
}
// (lower, upper 16 bits of a) * 2 + base, one instruction: the LDS address of a histogram word from twice its index.
// UNIFORM: base is the same for every lane
template <bool UNIFORM>
__device__ __forceinline__ uint32_t twice_lower(uint32_t a, uint32_t base) {
  uint32_t d;
  if (UNIFORM) asm("v_mad_u32_u16 %0, %1, 2, %2" : "=v"(d) : "v"(a), "s"(base));
  else asm("v_mad_u32_u16 %0, %1, 2, %2" : "=v"(d) : "v"(a), "v"(base));
  return d;
}
template <bool UNIFORM>
__device__ __forceinline__ uint32_t twice_upper(uint32_t a, uint32_t base) {
  uint32_t d;
  if (UNIFORM) asm("v_mad_u32_u16 %0, %1, 2, %2 op_sel:[1,0,0,0]" : "=v"(d) : "v"(a), "s"(base));
  else asm("v_mad_u32_u16 %0, %1, 2, %2 op_sel:[1,0,0,0]" : "=v"(d) : "v"(a), "v"(base));
  return d;
}
// the histogram increment of a positive value, 1, or of a negative one, 65536, from its sign (0 or 1) in the lower or upper half
__device__ __forceinline__ uint32_t increment_lower(uint32_t signs, uint32_t c65535_sgpr) {
  uint32_t d;
  asm("v_mad_u32_u16 %0, %1, %2, 1" : "=v"(d) : "v"(signs), "s"(c65535_sgpr));
  return d;
}
__device__ __forceinline__ uint32_t increment_upper(uint32_t signs, uint32_t c65535_sgpr) {
  uint32_t d;
  asm("v_mad_u32_u16 %0, %1, %2, 1 op_sel:[1,0,0,0]" : "=v"(d) : "v"(signs), "s"(c65535_sgpr));
  return d;
}
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(c2t_ushort2, a), __builtin_bit_cast(c2t_ushort2, b)));
}
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(c2t_ushort2, a), __builtin_bit_cast(c2t_ushort2, b)));
}

__device__ __forceinline__ uint32_t pk_sub_sat_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(c2t_ushort2, a), __builtin_bit_cast(c2t_ushort2, b)));
}
__device__ __forceinline__ uint32_t pk_shr_u16(uint32_t a, int n) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(c2t_ushort2, a) >> (unsigned short)n);
}
__device__ __forceinline__ uint32_t pk_sub_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(c2t_ushort2, a) - __builtin_bit_cast(c2t_ushort2, b));
}

// What the rows' rare logits add up to, per workgroup, in LDS: the streaming loop carries none of
// it in registers (four registers through the loop, and a copy of them per chunk, before).
struct OutsideAcc {
  double s_tiny;                    // sum of the logits with |x| < 2^-25 (zeros included): e^x = 1 + x to fp64 accuracy
  int32_t n_tiny;                   // their number
  int32_t n_masked;                 // masked logits (see hp_masked: probability 0, ranked last)
  uint32_t mag_max;                 // largest |code| seen outside the fast path: NaN, inf and |x| >= 2^7 show here
  uint32_t masked_by_lane[WAVE];    // masked logits again, counted where the rest of their chunk is in the window: lane l of every
                                    // wavefront adds to word l, in the half a negative value's count goes to (folded into n_masked)
};
typedef __attribute__((address_space(3))) OutsideAcc* OutsideAccLds;
typedef __attribute__((address_space(3))) uint32_t* LdsWords;
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p; }
__device__ __forceinline__ void lds_add(uint32_t address, uint32_t v) {
  __hip_atomic_fetch_add((LdsWords)(uintptr_t)address, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Of two packed bf16 codes w, d = 2 |code| - 2 LO (mod 2^16), with the sign shifted out by the doubling: the value lies in the
// window iff d < 2 SPAN = 8192, i.e. iff bits 13..15 of d are clear; then d is twice the index of its histogram word.
constexpr uint32_t HP_OUTSIDE2 = 0xE000E000u;
static_assert(2 * HP_MAG_SPAN == 8192 && HP_WORDS == 4096, "window test and index");
__device__ __forceinline__ uint32_t twice_index(uint32_t w) {
  return pk_mad_u16(w, 0x00020002u, ((0x10000u - 2u * HP_MAG_LO) & 0xffffu) * 0x00010001u);
}

// Chunks that hold a logit outside the window, and a row's partial last chunk (n_valid < 8).  Out
// of line: typical rows never get here, and inlined at each of the streaming loop's sites this
// code costs the whole kernel registers.  If everything outside the window is masked (see
// hp_masked), those logits are counted apart and the rest of the chunk is counted as in
// hist_chunk; otherwise one element at a time.
// Returns the maximum of the valid elements as a packed pattern; where all of them are masked, a
// value below every finite logit of the window path (a cell key only has to be an upper bound).
// Masked logits: -inf and every finite x <= -2^10 (the large negative constants used in place of
// -inf).  The row's largest logit is a window value, m > -2^7, so x - m < -896 and e^(x - m) is
// exactly 0 in fp64 (which underflows to 0 below -745.2): such a logit adds nothing to Z or S, and
// it ranks after every window value.  NaN codes (above 0xff80) are not in the range.
__device__ __forceinline__ bool hp_masked(uint32_t code16) { return code16 - 0xc480u <= 0xff80u - 0xc480u; }
__device__ __noinline__ uint32_t hist_chunk_outside(uint4 q, int n_valid, uint32_t hist, OutsideAcc* acc_generic) {     // hist: LDS address
  const OutsideAccLds acc = (OutsideAccLds)acc_generic;
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  if (n_valid == 8) {
    // codes from 0xC300 on are clamped to the window's lowest value; what must not be, codes in (-2^10, -2^7] and negative
    // NaN, shows in the packed extremes
    uint32_t w2[4], d[4], dm = 0u, hi = 0u, lo = 0xffffffffu;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      hi = pk_max_u16(hi, w[j]);
      lo = pk_min_u16(lo, pk_sub_u16(w[j], 0xC300C300u));
      w2[j] = pk_min_u16(w[j], HP_LOWEST * 0x00010001u);
      d[j] = twice_index(w2[j]);
      dm |= d[j];
    }
    if (((dm & HP_OUTSIDE2) | pk_sub_sat_u16(hi, 0xFF80FF80u) | pk_sub_sat_u16(0x01800180u, lo)) == 0u) {
      // Every lane issues all eight atomics, as for a chunk inside the window; a masked logit's goes to the
      // lane's own word of masked_by_lane instead of the histogram (one address select per logit: no
      // branches, no ballots, and the 64 words lie in 64 different places, so masked logits pile up nowhere).
      // The stand-in value is negative, so the count lands in the word's upper half.
      const uint32_t own = lds_address(&acc_generic->masked_by_lane[lane_id()]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t sg = pk_shr_u16(w2[j], 15);
        lds_add(w[j] >= 0xC4800000u ? own : twice_upper<false>(d[j], hist), increment_upper(sg, 0xffffu));
        lds_add((uint16_t)w[j] >= (uint16_t)0xC480u ? own : twice_lower<false>(d[j], hist), increment_lower(sg, 0xffffu));
      }
      return pk_max_f16(pk_max_f16(w2[0], w2[1]), pk_max_f16(w2[2], w2[3]));
    }
  }
  float cm = -INFINITY;
  uint32_t mag_max = 0u;
  int n_tiny = 0, n_masked = 0;
  double s_tiny = 0.0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float x = (j & 1) ? bf16_hi(w[j >> 1]) : bf16_lo(w[j >> 1]);
    const uint32_t code = __float_as_uint(x) >> 16, mag = code & 0x7fffu;
    if (j < n_valid) {
      if (hp_masked(code)) n_masked += 1;
      else {
        mag_max = max(mag_max, mag);
        cm = fmaxf(cm, x);
        if (mag < HP_MAG_LO) { n_tiny += 1; s_tiny += (double)x; }
        else lds_add(hist + 4u * ((mag - HP_MAG_LO) & (HP_WORDS - 1)), (code & 0x8000u) ? 0x10000u : 1u);   // (above the window: counted anywhere, the row leaves this path)
      }
    }
  }
  if (n_masked) __hip_atomic_fetch_add(&acc->n_masked, n_masked, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if (n_tiny) {
    __hip_atomic_fetch_add(&acc->n_tiny, n_tiny, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_add(&acc->s_tiny, s_tiny, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  if (mag_max >= HP_MAG_LO + HP_MAG_SPAN) __hip_atomic_fetch_max(&acc->mag_max, mag_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  const uint32_t c16 = cm == -INFINITY ? (HP_NONE2 & 0xffffu) : __float_as_uint(cm) >> 16;
  return c16 | (c16 << 16);
}

// Counts the values of a whole chunk into the histogram at LDS address `hist`; returns the chunk maximum as a packed pattern (both
// halves <= max, one of them equal to it).  32 vector instructions beside the eight additions: the address and the increment of a
// value take one each (v_mad_u32_u16 picks its half, scales and adds the lane's base), the window test three a chunk beyond the indices.
template <bool ONE_COPY>
__device__ __forceinline__ uint32_t hist_chunk(const uint4& q, uint32_t hist, OutsideAcc* acc) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  const uint32_t d[4] = {twice_index(w[0]), twice_index(w[1]), twice_index(w[2]), twice_index(w[3])};
  uint32_t pat;
  // rare: a logit outside the window.  The whole wave then takes the out-of-line routine (it counts
  // in-window chunks as well): cheaper than running both paths one after the other.
  if (__builtin_amdgcn_ballot_w64(((d[0] | d[1] | d[2] | d[3]) & HP_OUTSIDE2) != 0u) != 0ull) {   // (a hint that this is rare made the loop 10 % slower)
    pat = hist_chunk_outside(q, 8, hist, acc);
  } else {
    // inside the window bf16 bit patterns order exactly like fp16 bit patterns
    pat = pk_max_f16_raw(pk_max_f16_raw(w[0], w[1]), pk_max_f16_raw(w[2], w[3]));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // +1 into the low half for a positive value, into the high half for a negative one
      const uint32_t sg = pk_shr_u16(w[j], 15);
      lds_add(twice_upper<ONE_COPY>(d[j], hist), increment_upper(sg, 0xffffu));
      lds_add(twice_lower<ONE_COPY>(d[j], hist), increment_lower(sg, 0xffffu));
    }
  }
  return pat;
}

// The same for a row that masks part of its vocabulary, where nearly every chunk holds masked logits: those are clamped to
// the window's lowest value (which the maximum then never takes) and counted in the lane's own word of masked_by_lane
// instead of the histogram, with an address select per logit but no call and nothing kept per chunk.  What the clamp must
// not swallow, codes in (-2^10, -2^7] and negative NaN, shows in `seen` (packed maximum of the codes, packed minimum of
// codes - 0xC300), which the caller looks at once per row.
struct CodesSeen { uint32_t hi, lo; };
__device__ __forceinline__ uint32_t hist_chunk_masked(const uint4& q, uint32_t hist, uint32_t own, OutsideAcc* acc, CodesSeen& seen) {
  constexpr uint32_t FIRST_MASKED = 0xC480u;       // see hp_masked
  const uint32_t raw[4] = {q.x, q.y, q.z, q.w};
  uint32_t w[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    seen.hi = pk_max_u16(seen.hi, raw[j]);
    seen.lo = pk_min_u16(seen.lo, pk_sub_u16(raw[j], 0xC300C300u));
    w[j] = pk_min_u16(raw[j], HP_LOWEST * 0x00010001u);
  }
  const uint32_t d[4] = {twice_index(w[0]), twice_index(w[1]), twice_index(w[2]), twice_index(w[3])};
  uint32_t pat;
  if (__builtin_amdgcn_ballot_w64(((d[0] | d[1] | d[2] | d[3]) & HP_OUTSIDE2) != 0u) != 0ull) {
    pat = hist_chunk_outside(q, 8, hist, acc);
  } else {
    pat = pk_max_f16_raw(pk_max_f16_raw(w[0], w[1]), pk_max_f16_raw(w[2], w[3]));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t sg = pk_shr_u16(w[j], 15);
      lds_add(raw[j] >= (FIRST_MASKED << 16) ? own : twice_upper<false>(d[j], hist), increment_upper(sg, 0xffffu));
      lds_add((uint16_t)raw[j] >= (uint16_t)FIRST_MASKED ? own : twice_lower<false>(d[j], hist), increment_lower(sg, 0xffffu));
    }
  }
  return pat;
}

// ---- a lower bound of the K-th largest logit (K <= COLUMNS_MAX_K): the K-th largest of the maxima of 64 columns of lanes (K <= 16), or the 32nd; sorted in
// rows of 16 lanes (bitonic, a lane permutation and a v_med3 a stage).  A tenth of a microsecond, where a search by ballots takes half of one: its
// rounds are chains of scalar instructions.  Lane l's column holds the chunks l, l + 64, .. of 8 logits, so that neighbouring ids
// lie in different columns: of randomly placed logits 18 reach the bound for K = 16 and 44 for K = 32, where the ids are ordered by frequency 20 and 48
// (95 at most in 300 rows), and of a stretch of 512 ids that are likely ones all 64 columns hold some.  (Columns of whole cells put 512 ids into 16 of
// them: the bound fell to what lies around them, and layers of 256 rows of 128256 whose likely ids are neighbours, 400 to 4000, took 26 to 37 us with K = 32,
// 23 so; by frequency 31.6 and 24.1, with K = 16 23.8 and 21.8.  The smallest of the four rows' ceil(K / 4)-th, two lane permutations shorter: 400 neighbours,
// which are 50 lanes, 27.0 with K = 16, 22.0 so.)  Fewer neighbours than that, 100 to 256, may all reach the bound: 100 of them 24.8 (4 sequences of 20011 with
// K = 32 16.2, 12.7 without them).
// The exact K-th largest logit of the counts (kth_of_counts) takes a microsecond more a row:
// four sequences of 20011 with 64 x 32 candidates took 237.3 us a phase with it, 230.4 so, 256 of 152064 with 32 x 32 1820 and 1803, a layer of three rows
// of 8279 with K = 31 12.5 and 11.7.
constexpr int COLUMNS_MAX_K = 32;
// 16-bit keys that order like the values of the patterns
__device__ __forceinline__ uint32_t key_of_pattern(uint32_t c) { return (c & 0x8000u) ? c ^ 0xffffu : c | 0x8000u; }
// column: packed pattern, the maximum of the lane's column over the whole row; uniform result: a value that K logits at least reach, or the window's
// lowest where fewer columns hold a logit of the window.
__device__ __forceinline__ float bound_of_patterns(uint32_t column, int K) {
  const uint32_t own = max(key_of_pattern(column & 0xffffu), key_of_pattern(column >> 16));
  uint32_t key;                                                         // (K is uniform)
  if (K > 16) key = largest_32nd(own);
  else if (K > 1) key = nth_largest16(own, K);
  else key = wave_reduce_u32(own, 0u, [](uint32_t x, uint32_t y) { return max(x, y); });
  key = max(key, key_of_pattern(HP_LOWEST));
  return __uint_as_float(((key & 0x8000u) ? key & 0x7fffu : key ^ 0xffffu) << 16);
}

// The keys of a group's cells: of the maxima p[k] of the chunks that the lane has read in sweep k of the group, lane t of a quad gets the
// largest of the quad's p[t].  Two exchanges between neighbours, each lane giving away half of what it holds.
__device__ __forceinline__ uint32_t quad_exchange_1(uint32_t even, uint32_t odd, bool is_odd) {
  return pk_max_f16_raw(is_odd ? odd : even, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, is_odd ? even : odd));
}
__device__ __forceinline__ uint32_t quad_exchange_2(uint32_t lower, uint32_t upper, bool is_upper) {
  return pk_max_f16_raw(is_upper ? upper : lower, dpp_u32<C2T_DPP_QUAD_XOR2, 0xf>(0u, is_upper ? lower : upper));
}

// The streaming loop: `whole` chunks of the segment that rs covers and, with tail_valid > 0, a partial one behind them; q: the lane's first
// DEPTH chunks, on their way; keys: LDS, the cells' keys, the lane's first.  MASKED: see hist_chunk_masked.  ONE_COPY: of the histogram,
// with four workgroups a CU.  STREAMED: see load_stream_buffer.
typedef __attribute__((address_space(3))) uint16_t* LdsHalves;
struct StreamInput { __amdgpu_buffer_rsrc_t rs; int whole, tail_valid; uint32_t vo, hist; LdsHalves keys; OutsideAcc* acc; };
template <int NT, int DEPTH, bool MASKED, bool ONE_COPY, bool STREAMED>
__device__ __forceinline__ uint32_t hist_stream(const StreamInput& in, uint4 (&q)[DEPTH]) {
  static_assert(DEPTH % 4 == 0 && CPC == 4, "whole cells");
  const uint32_t own = MASKED ? lds_address(&in.acc->masked_by_lane[lane_id()]) : 0u;
  const int whole = in.whole, tail = in.tail_valid > 0 ? whole : -1, n = whole / (DEPTH * NT);
  CodesSeen seen{0u, 0xffffffffu};
  uint32_t M2 = HP_NONE2, so = 0u;
  LdsHalves mp = in.keys;
  const auto count = [&](const uint4& c) {
    if (MASKED) return hist_chunk_masked(c, in.hist, own, in.acc, seen);
    return hist_chunk<ONE_COPY>(c, in.hist, in.acc);
  };
  const bool odd = (lane_id() & 1) != 0, upper = (lane_id() & 2) != 0;
  for (int it = n; it > 0; --it, so += (uint32_t)DEPTH * NT * 16u, mp += (DEPTH / 4) * NT) {
#pragma unroll
    for (int c = 0; c < DEPTH; c += 4) {
      uint32_t half[2];
#pragma unroll
      for (int k = 0; k < 4; k += 2) {
        const uint32_t pe = count(q[c + k]);
        q[c + k] = load_stream_buffer<STREAMED>(in.rs, in.vo, so + (uint32_t)(DEPTH + c + k) * (NT * 16u));
        const uint32_t po = count(q[c + k + 1]);
        q[c + k + 1] = load_stream_buffer<STREAMED>(in.rs, in.vo, so + (uint32_t)(DEPTH + c + k + 1) * (NT * 16u));
        M2 = pk_max3_f16_raw(M2, pe, po);
        half[k / 2] = quad_exchange_1(pe, po, odd);
      }
      const uint32_t key = quad_exchange_2(half[0], half[1], upper);
      mp[c / 4 * NT] = (uint16_t)pk_max_f16_raw(key, key >> 16);
    }
  }
  __builtin_amdgcn_s_setprio(0);
  // the last, partial group: up to DEPTH chunks of this lane, the row's partial last chunk among them
  uint32_t vo = in.vo;
  asm volatile("" : "+v"(vo));                                          // (not a copy that has been spilled over the loop)
  const int g0 = n * (DEPTH * NT), g = g0 + (int)(vo >> 4), end = whole + (tail >= 0 ? 1 : 0);
#pragma unroll
  for (int c = 0; c < DEPTH; c += 4) {
    if (g0 + c * NT >= end) break;                                      // (uniform)
    uint32_t half[2];
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
      uint32_t p[2] = {HP_NONE2, HP_NONE2};
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (g + (c + k + i) * NT < whole) p[i] = count(q[c + k + i]);
        else if (g + (c + k + i) * NT == tail) p[i] = hist_chunk_outside(q[c + k + i], in.tail_valid, in.hist, in.acc);
      }
      M2 = pk_max3_f16_raw(M2, p[0], p[1]);
      half[k / 2] = quad_exchange_1(p[0], p[1], odd);
    }
    const uint32_t key = quad_exchange_2(half[0], half[1], upper);
    mp[c / 4 * NT] = (uint16_t)pk_max_f16(key, key >> 16);
  }
  if (MASKED && (pk_sub_sat_u16(seen.hi, 0xFF80FF80u) | pk_sub_sat_u16(0x01800180u, seen.lo)))             // neither in the window nor masked: two-pass path
    __hip_atomic_fetch_max(&((OutsideAccLds)in.acc)->mag_max, 0x7fffu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return M2;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_buffer(uint64_t base, int bytes) {      // (the builtin of readfirstlane returns int: no sign extension)
  const uint64_t base_u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base) |
                          ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)) << 32);
  return __builtin_amdgcn_make_buffer_rsrc((void*)base_u, 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// The loop of a row that masks part of its vocabulary, from its first chunk on again: in line, with the eight chunks in flight of the usual loop the build has too few registers.
// A layer of 256 rows of 128256 logits, alone on their CUs, with 30 % masked: 41 us when every chunk took hist_chunk_outside, 30; a phase of 16 sequences, 16 rows each,
// 167.0 us with this loop out of line, where it fetched its uniform arguments from vector registers, 162.3 so.
template <int NT, bool STREAMED>
__device__ __forceinline__ uint32_t hist_stream_masked(const StreamInput& in) {
  constexpr int DEPTH = 4;
  uint4 q[DEPTH];
#pragma unroll
  for (int k = 0; k < DEPTH; ++k) q[k] = load_stream_buffer<STREAMED>(in.rs, in.vo, (uint32_t)k * (NT * 16u));
  return hist_stream<NT, DEPTH, true, false, STREAMED>(in, q);
}

// 16 bytes a lane from global memory straight into LDS, to `address` (uniform over the wavefront) + 16 lane: no registers while it is on its way.
__device__ __forceinline__ void lds_chunk_load(const uint4* p, uint32_t address) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p, (__attribute__((address_space(3))) void*)(uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)address), 16, 0, 0);
}

// A thread's share of the classifier's parameters on its way from global memory to LDS.
struct ClassifierStage { float4 q; float* dst; bool mine; };
__device__ __forceinline__ ClassifierStage stage_classifier(int tid, const float* __restrict__ cls, int h, float* dst) {
  ClassifierStage c;
  c.dst = dst;
  c.mine = dst != nullptr && tid * 4 < 5 * h + 1;     // the array is padded to a multiple of four floats
  c.q = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c.mine) c.q = ((const float4*)cls)[tid];
  return c;
}
__device__ __forceinline__ void store_classifier(int tid, const ClassifierStage& c) {
  if (c.mine) ((float4*)c.dst)[tid] = c.q;
}

constexpr int HANDED_OVER = -2, RANKED_IN_RR = -1, UNSETTLED = RANKED_IN_RR;     // SegmentTop::n_el

// What a workgroup's wavefronts leave each other in LDS on the histogram path.
template <int NT>
struct HistShared {
  static constexpr int NW = NT / WAVE;
  double red_d[2][NW];              // the wavefronts' Z and S
  double red_m_d[2][NW];            // ... over the M largest logits (TOPM)
  uint32_t red_m[NW];               // their largest patterns
  int32_t total[NW], scan_p[NW], scan_n[NW];
  OutsideAcc out;
  double e_minus_m;                 // e^-m (without TOPM)
  float m;                          // largest logit of the row
  int32_t n_cells, n_el, tot_p;
  int32_t kth[3];                   // KthOfCounts: rank, n_gt, n_ge
  int32_t cells[SEL_CELL_CAP];      // cells that hold a logit above the bound
};
constexpr int HIST_LIST = 256;                  // logits the element list holds
template <int NT>
__host__ __device__ constexpr size_t hist_lds_bytes(int repl) {   // histogram copies | columns, then (a barrier later) the element list; the cell map behind
  static_assert(NT * 4 <= HIST_LIST * 8, "the columns fit the list's place");
  return (size_t)HP_WORDS * 4 * repl + HIST_LIST * 8;
}
__device__ __forceinline__ SelectLds hist_list(unsigned char* at) {
  SelectLds s;
  s.list = at; s.aux = nullptr; s.list_cap = HIST_LIST; s.cell_cap = 0;
  return s;
}

// The exact K-th largest logit of a histogram, by the whole workgroup: the value-ordered rank of its bin (see hp_code_of_rank; -1: fewer
// than K logits lie in the window), how many logits exceed it and how many reach it.  Out of line: it is looked for where K > COLUMNS_MAX_K, and in rows that
// settle_hist is asked about.
struct KthOfCounts { int rank, n_gt, n_ge; };
// As a bound: where fewer than K logits lie in the window, its lowest value, which all of them reach and cells without a chunk do not
__device__ __forceinline__ float bound_of_counts(const KthOfCounts& k) { return __uint_as_float(hp_code_of_rank(max(k.rank, 0)) << 16); }
template <int NT> using HistSharedLds = __attribute__((address_space(3))) HistShared<NT>*;
template <int NT>
__device__ __noinline__ KthOfCounts kth_of_counts(int tid, LdsWords hist, int top_k, HistSharedLds<NT> hs) {
  const int K = __builtin_amdgcn_readfirstlane(top_k);
  constexpr int NW = NT / WAVE, WPL = HP_WORDS / NT;
  __shared__ int32_t scan[2][NW];
  __attribute__((address_space(3))) int32_t* const found = hs->kth;
  const int lane = tid & (WAVE - 1), wid = tid >> 6, w0 = WPL * tid;
  int lane_pos = 0, lane_neg = 0;
  for (int j = 0; j < WPL; ++j) { lane_pos += (int)(hist[w0 + j] & 0xffffu); lane_neg += (int)(hist[w0 + j] >> 16); }
  const int incl_p = wave_scan_incl(lane_pos), incl_n = wave_scan_incl(lane_neg);
  if (lane == WAVE - 1) { scan[0][wid] = incl_p; scan[1][wid] = incl_n; }
  if (tid == 0) { found[0] = -1; found[1] = found[2] = 0; }
  __syncthreads();
  int before_p = 0, before_n = 0, tot_p = 0;
  for (int w = 0; w < NW; ++w) { if (w < wid) { before_p += scan[0][w]; before_n += scan[1][w]; } tot_p += scan[0][w]; }
  // descending: positive values from the highest lane down, then negative ones from lane 0 up
  const int above_p = tot_p - (before_p + incl_p), above_n = tot_p + before_n + incl_n - lane_neg;
  if (above_p < K && above_p + lane_pos >= K) {              // at most one lane
    int run = above_p;
    for (int j = WPL - 1; j >= 0; --j) {
      const int n = (int)(hist[w0 + j] & 0xffffu);
      if (run < K && run + n >= K) { found[0] = HP_WORDS + w0 + j; found[1] = run; found[2] = run + n; }
      run += n;
    }
  }
  if (above_n < K && above_n + lane_neg >= K) {
    int run = above_n;
    for (int j = 0; j < WPL; ++j) {
      const int n = (int)(hist[w0 + j] >> 16);
      if (run < K && run + n >= K) { found[0] = HP_WORDS - 1 - (w0 + j); found[1] = run; found[2] = run + n; }
      run += n;
    }
  }
  __syncthreads();
  return KthOfCounts{found[0], found[1], found[2]};
}

// The rows whose list of the largest logits did not come out, or that need a closer look: with the exact K-th largest logit tau
// from the counts,
//  * rows with logits below the window take the two-pass path unless tau is a positive value of it, those with fewer than K logits in the
//    window and masked ones besides do so too (they could be among the top K, which the histogram cannot rank): UNSETTLED;
//  * a list that is incomplete (too many cells or logits reach the bound) or short of K is made again from the cells that reach tau: those listed, if
//    all were, else from the map, which is still in place then.  Where too many logits equal tau, only what exceeds it is listed (fewer than K
//    logits), and the ties of the lowest ids are added (tie_scan).
// Reading the whole segment a second time for what exceeds tau took longer than the first time: layers of 256 rows of 128256 with K = 32, 400 to 4000
// neighbouring logits of each far above the others, 69 us (26 to 37 from the cells); of nine values 69 (53).
// Returns the list's length.  Out of line: see settle_list.
template <int NT>
__device__ __noinline__ int settle_hist(int tid, const uint4* __restrict__ rowp, int V, int top_k, const Segment segment, LdsWords hist, uint32_t list_address,
                                        LdsHalves cell_map, int cells_max, HistSharedLds<NT> shl) {
  typedef LogitTraits<1> T;
  __shared__ int32_t scan_tmp[1][NT / WAVE];
  // (told to be uniform: the arguments of a call arrive in vector registers)
  HistShared<NT>& hs = *(HistShared<NT>*)shl;
  const int K = uniform(top_k), cell_cap = uniform(cells_max);
  const Segment sg{uniform(segment.c0), uniform(segment.c1), uniform(segment.ncell), uniform(segment.tail_chunk), uniform(segment.tail_valid)};
  const SelectLds list = hist_list((unsigned char*)(__attribute__((address_space(3))) unsigned char*)(uintptr_t)(uint32_t)uniform((int)list_address));
  const int n_elems = sg.tail_chunk >= 0 ? (sg.ncell - 1) * T::EPC + sg.tail_valid : sg.ncell * T::EPC, want = min(K, n_elems);
  int n_cells = uniform(hs.n_cells);
  const int n_el = uniform(hs.n_el);
  KthOfCounts kth{hs.kth[0], hs.kth[1], hs.kth[2]};
  if (K <= COLUMNS_MAX_K) kth = kth_of_counts<NT>(tid, hist, K, shl);
  __syncthreads();                                             // everybody has read the lengths
  if ((uniform(hs.out.n_tiny) > 0 && kth.rank < HP_WORDS) || (uniform(hs.out.n_masked) > 0 && kth.rank < 0)) return UNSETTLED;
  if (n_cells <= cell_cap && n_el >= want && n_el <= HIST_LIST) return n_el;
  const float tau = bound_of_counts(kth);
  // Only what exceeds tau: then fewer than K cells do, else no more than n_ge reach it, but for cells of masked logits, whose keys are the lowest value
  const bool strict = kth.n_ge > (n_cells > cell_cap ? cell_cap : HIST_LIST) || kth.rank == 0;
  if (strict && kth.n_gt == 0) n_cells = 0;
  else if (n_cells > cell_cap)
    n_cells = min(list_cells<1, NT>(tid, (const uint16_t*)cell_map, quad_cells_in_segment<NT>(sg.ncell), tau, strict, cell_cap, hs.cells, &hs.n_cells), cell_cap);
  if (tid == 0) hs.n_el = 0;
  __syncthreads();
  if (n_cells > 0) collect_cells<1, NT, true>(tid, rowp, sg.c0, sg.c1, V, tau, strict, hs.cells, n_cells, list, &hs.n_el);
  const int n = hs.n_el, need = want - n;                      // (need > 0 only where it is strict)
  if (need > 0) tie_scan<1, NT>(tid, rowp, sg, V, tau, need, list, &hs.n_el, scan_tmp);
  return need > 0 ? want : n;
}

// The record of a row (or split) from its wavefronts' sums: lanes 0 .. NW-1 of one wavefront, fixed order.  To rr, and in lane 0 returned.
template <int NT, bool TOPM>
__device__ __forceinline__ RowPartial combine_hist(const HistShared<NT>& hs, int M, RowResult& rr) {
  constexpr int NW = NT / WAVE;
  static_assert(NW <= 16, "one DPP row holds the per-wave sums");
  const int lane = lane_id(), n_tiny = hs.out.n_tiny;
  const double md = (double)hs.m;
  const auto sum = [&](const double (&red)[2][NW], bool with_tiny, double& z, double& s) {
    double tz = lane < NW ? red[0][lane] : 0.0, ts = lane < NW ? red[1][lane] : 0.0;
    tz += dpp_f64<C2T_DPP_QUAD_XOR1, 0xf>(tz); ts += dpp_f64<C2T_DPP_QUAD_XOR1, 0xf>(ts);
    tz += dpp_f64<C2T_DPP_QUAD_XOR2, 0xf>(tz); ts += dpp_f64<C2T_DPP_QUAD_XOR2, 0xf>(ts);
    tz += dpp_f64<C2T_DPP_ROW_HALF_MIRROR, 0xf>(tz); ts += dpp_f64<C2T_DPP_ROW_HALF_MIRROR, 0xf>(ts);
    if (NW > 8) { tz += dpp_f64<C2T_DPP_ROW_MIRROR, 0xf>(tz); ts += dpp_f64<C2T_DPP_ROW_MIRROR, 0xf>(ts); }
    if (with_tiny && n_tiny) {                          // e^x = 1 + x, x e^x = x for |x| < 2^-25
      const double zt = (double)n_tiny + hs.out.s_tiny;
      tz += zt; ts += hs.out.s_tiny - md * zt;
    }
    z = tz; s = ts;
  };
  double Z, S, ZM = 0.0, SM = 0.0;
  sum(hs.red_d, true, Z, S);
  if (TOPM) sum(hs.red_m_d, hs.tot_p < M, ZM, SM);       // (where the tiny ones are among the M largest, all of them are)
  RowPartial r; r.ref = md; r.a = 0.0; r.Z = Z; r.S = S; r.n_top = 0; r.flags = 0u;
  if (lane == 0) {
    rr.part = r;
    if (TOPM) { rr.ZM = ZM; rr.SM = SM; }
  }
  return r;
}

// A row shared by sp.coop workgroups (launches that leave most of the chip idle: a single sequence,
// a root layer).  One workgroup counts a 256 KB row at the rate of its CU's LDS atomics, 9 us; n
// workgroups on n CUs count a segment each, and their histograms, being sums, merge exactly.  Each
// hands over through memory what the epilogue needs of its segment: the 4096 count words (copies
// already folded), the keys of its cells (segments are whole groups of four sweeps, so the row's
// map is the segments' maps laid end to end), its columns' maxima and the few numbers of OutsideAcc.  The stores are
// device-coherent and complete before the workgroup takes the row's ticket; the workgroup that takes
// the last one adds the n histograms up in its own LDS, loads the row's map, and goes on as if it
// had counted the whole row.  The sums and the selection therefore come
// out exactly as for an unshared row (the sum of the logits below the window is added up per
// segment first: a different rounding order for a term of relative size 1e-16).
// Every slot is written once and read once per launch: nothing has to be cleared between launches.
// Returns true in the workgroup that goes on.  map: the segment's keys in LDS, with room for the row's; column, m2: the lane's column maximum
// and the largest pattern, of the segment, then of the row.
constexpr int COOP_BATCH = 4;                   // other segments whose counts a lane has in flight at once (eight registers each)
template <int NT>
__device__ __forceinline__ bool share_row(int tid, const ScoreParams& sp, int split, int64_t row_launched, int32_t* row_ticket,
                                          const Segment& sg, uint32_t* __restrict__ hist, uint32_t w0, uint16_t* map,
                                          OutsideAcc* sh_out, uint32_t& column, uint32_t& m2) {
  constexpr int NW = NT / WAVE;
  constexpr uint32_t SLOT_BYTES = HP_WORDS * 4, COHERENT = 16;          // cache policy sc1: served at the device's coherence point
  const int lane = tid & (WAVE - 1), wid = tid >> 6;
  const int n = sp.coop;
  const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc((void*)(sp.coop_hist + row_launched * n * HP_WORDS), 0,
                                                                      n * (int)SLOT_BYTES, 0x00020000);
  const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc((void*)(sp.coop_map + row_launched * sp.coop_map_stride), 0,
                                                                      sp.coop_map_stride * 2, 0x00020000);
  CoopAcc* const acc = sp.coop_acc + row_launched * n;
  uint32_t* const columns = (uint32_t*)(sp.coop_map + (int64_t)COOP_MAX_ROWS * sp.coop_map_stride) + row_launched * n * WAVE;
  {
    const uint4 t0 = *(const uint4*)(hist + w0), t1 = *(const uint4*)(hist + w0 + 4);
    const c2t_uint4v u0 = {t0.x, t0.y, t0.z, t0.w}, u1 = {t1.x, t1.y, t1.z, t1.w};
    __builtin_amdgcn_raw_buffer_store_b128(u0, rh, w0 * 4u, (uint32_t)split * SLOT_BYTES, COHERENT);
    __builtin_amdgcn_raw_buffer_store_b128(u1, rh, w0 * 4u + 16u, (uint32_t)split * SLOT_BYTES, COHERENT);
    const int ncells = quad_cells_in_segment<NT>(sg.ncell);
    const uint32_t first_key_byte = (uint32_t)sg.c0 / CPC * 2u;        // sg.c0 is a multiple of CPC * NT chunks
    for (int i = tid * 8; i < ncells; i += NT * 8) {                    // (a store that reaches past the row's keys is dropped by the bounds check)
      const uint4 k = *(const uint4*)(map + i);
      const c2t_uint4v kv = {k.x, k.y, k.z, k.w};
      __builtin_amdgcn_raw_buffer_store_b128(kv, rm, (uint32_t)i * 2u, first_key_byte, COHERENT);
    }
    if (wid == NW - 1) {
      st_dev(columns + split * WAVE + lane, column);
      if (lane == 0) {                                                  // the lane that has just folded masked_by_lane into n_masked
        CoopAcc* a = acc + split;
        st_dev(&a->s_tiny, sh_out->s_tiny);
        st_dev(&a->n_tiny, sh_out->n_tiny); st_dev(&a->n_masked, sh_out->n_masked);
        st_dev(&a->mag_max, sh_out->mag_max); st_dev(&a->max_pattern, m2);
      }
    }
  }
  wait_vector_memory();                                                 // this wave's stores have reached the coherence point
  __syncthreads();                                                      // ... and every wave's; the reads of LDS above are done
  if (!last_arrival(tid, row_ticket, n)) return false;

  // Every load of the first round trip is issued before anything waits: the segments' numbers
  // (one segment per lane), their columns, the row's keys (two loads a thread cover the largest map) and the
  // first COOP_BATCH segments' counts.
  const bool have = lane < n;
  const CoopAcc* a = acc + min(lane, n - 1);
  const uint32_t mp = ld_dev(&a->max_pattern);
  double st = 0.0; int nt = 0, nm = 0; uint32_t mm = 0u;
  if (wid == 0) { st = ld_dev(&a->s_tiny); nt = ld_dev(&a->n_tiny); nm = ld_dev(&a->n_masked); mm = ld_dev(&a->mag_max); }
  uint32_t col[COOP_BATCH];
#pragma unroll
  for (int j = 0; j < COOP_BATCH; ++j) col[j] = ld_dev(columns + min(j, n - 1) * WAVE + lane);
  const int k0 = tid * 8, k1 = k0 + NT * 8;
  const c2t_uint4v kv0 = __builtin_amdgcn_raw_buffer_load_b128(rm, (uint32_t)k0 * 2u, 0u, COHERENT);   // zeros past the row's keys
  const c2t_uint4v kv1 = __builtin_amdgcn_raw_buffer_load_b128(rm, (uint32_t)k1 * 2u, 0u, COHERENT);
  // The other n - 1 segments' counts, from the next segment on round the row; its own are still in LDS.
  uint4 c0 = *(const uint4*)(hist + w0), c1 = *(const uint4*)(hist + w0 + 4);
  for (int j0 = 0; j0 < n - 1; j0 += COOP_BATCH) {
    c2t_uint4v v[2 * COOP_BATCH];
#pragma unroll
    for (int j = 0; j < COOP_BATCH; ++j) {
      int sl = split + 1 + j0 + j;
      sl = sl >= n ? sl - n : sl;
      const uint32_t so = (j0 + j < n - 1) ? (uint32_t)sl * SLOT_BYTES : (uint32_t)n * SLOT_BYTES;   // past the last slot: zeros from the bounds check, no traffic
      v[2 * j] = __builtin_amdgcn_raw_buffer_load_b128(rh, w0 * 4u, so, COHERENT);
      v[2 * j + 1] = __builtin_amdgcn_raw_buffer_load_b128(rh, w0 * 4u + 16u, so, COHERENT);
    }
#pragma unroll
    for (int j = 0; j < COOP_BATCH; ++j) {                              // a carry out of a 16-bit half shows in the total, like a counter overflow
      c0.x += v[2 * j].x; c0.y += v[2 * j].y; c0.z += v[2 * j].z; c0.w += v[2 * j].w;
      c1.x += v[2 * j + 1].x; c1.y += v[2 * j + 1].y; c1.z += v[2 * j + 1].z; c1.w += v[2 * j + 1].w;
    }
  }
  *(uint4*)(hist + w0) = c0; *(uint4*)(hist + w0 + 4) = c1;             // only this lane reads these words before the next barrier
  if (k0 < sp.coop_map_stride) *(uint4*)(map + k0) = make_uint4(kv0.x, kv0.y, kv0.z, kv0.w);
  if (k1 < sp.coop_map_stride) *(uint4*)(map + k1) = make_uint4(kv1.x, kv1.y, kv1.z, kv1.w);
  for (int i = k1 + NT * 8; i < sp.coop_map_stride; i += NT * 8) {      // (longer maps than the launch code allows today)
    const c2t_uint4v kv = __builtin_amdgcn_raw_buffer_load_b128(rm, (uint32_t)i * 2u, 0u, COHERENT);
    *(uint4*)(map + i) = make_uint4(kv.x, kv.y, kv.z, kv.w);
  }
#pragma unroll
  for (int j = 0; j < COOP_BATCH; ++j) column = pk_max_f16_raw(column, col[j]);
  for (int j = COOP_BATCH; j < n; ++j) column = pk_max_f16_raw(column, ld_dev(columns + j * WAVE + lane));
  m2 = wave_reduce_u32(have ? mp : HP_NONE2, HP_NONE2, [](uint32_t x, uint32_t y) { return pk_max_f16(x, y); });
  if (wid == 0) {                                                       // fixed order of the sums
    const double st_all = wave_sum(have ? st : 0.0);
    const int nt_all = wave_sum_i(have ? nt : 0), nm_all = wave_sum_i(have ? nm : 0);
    const uint32_t mm_all = wave_reduce_u32(have ? mm : 0u, 0u, [](uint32_t x, uint32_t y) { return max(x, y); });
    if (lane == 0) { sh_out->s_tiny = st_all; sh_out->n_tiny = nt_all; sh_out->n_masked = nm_all; sh_out->mag_max = mm_all; }
  }
  return true;                                                          // the caller's next barrier publishes map and sh_out
}

// The histogram copies and what else the streaming loop adds to, by THREADS threads.
template <int THREADS, int REPL, int NT>
__device__ __forceinline__ void clear_counts(int tid, uint32_t* __restrict__ hist, HistShared<NT>& hs) {
#pragma unroll
  for (int j = 0; j < HP_WORDS * REPL / 4; j += THREADS)
    if (HP_WORDS * REPL / 4 % THREADS == 0 || tid + j < HP_WORDS * REPL / 4) *(uint4*)(hist + 4 * (tid + j)) = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) { hs.n_cells = 0; hs.n_el = 0; hs.out.s_tiny = 0.0; hs.out.n_tiny = 0; hs.out.n_masked = 0; hs.out.mag_max = 0u; }
  if (tid < WAVE) hs.out.masked_by_lane[tid] = 0u;
}

// One (row, split) segment on the histogram path, run by a whole workgroup of NT threads.
// hist: HP_WORDS words a copy, then the columns and, in their place, the element list, and the map, one 2-byte key per cell, padded to 16 bytes
// (hist_lds_bytes); sel: see SelectLds.
// TOPM: built with the entropy over the M largest logits (a separate instantiation, so that the
// default kernel carries none of its registers).
// COOP: built with the hand-over of a shared row (see share_row); returns HANDED_OVER in the workgroups
// that have handed their segment over and are done.
template <int NT, bool TOPM, int WPS, int REPL, bool COOP, bool STREAMED>
__device__ __forceinline__ SegmentTop hist_segment(const uint4* __restrict__ rowp, int V, int K, int M, const Segment& sg_own,
                                             const double* __restrict__ tab_e, uint32_t* __restrict__ hist, const SelectLds& list, uint16_t* map,
                                             const SelectLds& sel, RowResult* rr, HistShared<NT>& hs,
                                             const ClassifierStage cst, const TreeState& st, const ScoreParams& sp, int split,
                                             int64_t row_launched, int b, int64_t slot, bool cleared, int& tid) {
  constexpr int NW = NT / WAVE;
  constexpr int WPL = HP_WORDS / NT;                   // words per lane in the epilogue (8 at 512 threads)
  static_assert(NW <= 16 && WPL % 4 == 0, "one DPP row holds the per-wave partials; a lane reads whole 16-byte runs");
  const int lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  Segment sg = sg_own;                                   // what the workgroup streams; the whole row once a shared row's counts are merged

  // ---------------- streaming loop: count values, record cell maxima ----------------
  uint32_t vo_after;
  uint32_t M2;                                         // packed running maximum of the bf16 patterns (compared as fp16 patterns)
  {
    // DEPTH chunks per lane in flight: a workgroup that streams while its neighbours on the CU are
    // in their epilogues still covers the HBM latency.  Unrolled by DEPTH so that each buffer is
    // refilled right after it has been counted, without register copies.  Eight in the build with
    // 80 registers, which has room for them (measured: no faster than four, also for a workgroup
    // that is alone on its CU: the CU's counting rate bounds it, not the latency of its loads).
    constexpr int DEPTH = WPS == 6 ? 8 : 4;
    // The chunks are read through a buffer descriptor over exactly their bytes: a lane whose
    // chunk lies past the last one gets zeros from the bounds check instead of needing a
    // compare and a select per load, and the address is the lane's fixed offset plus a scalar one:
    // no vector instruction per load (eight before, a seventh of the loop).
    const uint64_t base = (uint64_t)(rowp + sg.c0);      // the same for every lane: told to the compiler
    StreamInput in;
    in.whole = __builtin_amdgcn_readfirstlane(max((sg.tail_chunk >= 0 ? sg.c1 - 1 : sg.c1) - sg.c0, 0));   // a partial last chunk is counted apart
    in.tail_valid = __builtin_amdgcn_readfirstlane(sg.tail_chunk >= 0 ? sg.tail_valid : 0);
    in.rs = uniform_buffer(base, sg.ncell * 16);
    in.vo = (uint32_t)tid * 16u; in.keys = (LdsHalves)(map + tid); in.acc = &hs.out;
    // REPL copies of the histogram, a lane counting into copy (lane mod REPL): neighbouring lanes that
    // hold the same value (common: few hundred values carry most of a row) then add to different
    // words, which the LDS does not have to serialise.  The copies are folded after the loop.
    static_assert(REPL == 1 || REPL == 2 || REPL == 4 || REPL == 8, "a lane picks its copy with a mask");
    in.hist = lds_address(hist) + (REPL > 1 ? (uint32_t)(tid & (REPL - 1)) * (HP_WORDS * 4u) : 0u);
    uint4 q[DEPTH];
#pragma unroll
    for (int k = 0; k < DEPTH; ++k) q[k] = load_stream_buffer<STREAMED>(in.rs, in.vo, (uint32_t)k * (NT * 16u));
    if (!cleared) {                                      // (uniform) while they are on their way
      clear_counts<NT, REPL>(tid, hist, hs);
      __syncthreads();
    }
    // Streaming waves issue ahead of the waves of co-resident workgroups that are in their
    // (latency-bound) epilogue or tail: the memory pipeline stays fed.  Measured: 3 % per full layer.
    __builtin_amdgcn_s_setprio(3);
    // A row that masks part of its vocabulary shows it in the wavefront's first chunks (of 512 logits each): where half of them hold
    // a masked logit, most chunks do.  Fewer, a few masked tokens or a masked stretch, are counted chunk by chunk, out of line.  256
    // rows of 128256 by the usual loop / by the masked one: no logit masked 21.4 us / -, one 21.4 / 26.8, the first 4096 22.1 / 30.2,
    // 1 % 40.0 / 30.3, 30 % - / 30.2.  (With fewer chunks looked at, some wavefront of some row decides wrongly, and the launch waits
    // for it.)  Decided once, ahead of the loop: a test inside it costs the rows that mask nothing 4 to 6 %.
    int masks = 0;
    // Not with four workgroups per CU, where the decision alone costs rows that mask nothing 1 % and the call gains nothing; nor
    // for shared rows, whose segments are a group or two: root layer of 64 rows 26.7 us without it, 29.0 with it.
    if (WPS != 8 && !COOP && in.whole >= DEPTH * NT) {     // (shorter rows do not wait for all their loads here)
      int n = 0;
#pragma unroll
      for (int k = 0; k < DEPTH; ++k) {
        const uint32_t hi = pk_max_u16(pk_max_u16(q[k].x, q[k].y), pk_max_u16(q[k].z, q[k].w));
        n += __builtin_amdgcn_ballot_w64(pk_sub_sat_u16(hi, 0xC47FC47Fu) != 0u) != 0ull ? 1 : 0;
      }
      masks = __builtin_amdgcn_readfirstlane(2 * n >= DEPTH ? 1 : 0);      // (a scalar branch: as a lane mask both sides' registers would be live at once)
    }
    vo_after = in.vo;
    if (masks != 0) M2 = hist_stream_masked<NT, STREAMED>(in);
    else M2 = hist_stream<NT, DEPTH, false, REPL == 1, STREAMED>(in, q);
    C2T_PT(PT_STREAM_END);
    store_classifier(tid, cst);                                 // published by the barriers below
  }
  // The thread index should not be kept in a register through the loop on top of the lane's
  // buffer offset: a spill that crosses the loop is reloaded behind all the logits in flight on the
  // CU (microseconds, for every wave).  It is formed again here, for everything that follows, from the offset.
  asm volatile("" : "+v"(vo_after));
  tid = (int)(vo_after >> 4);

  // The lane owns the magnitude indices WPL*tid .. WPL*tid + WPL-1, with both signs.  The table
  // loads for their e^v are issued now so that their latency hides behind the barrier.
  static_assert(WPL == 8, "a lane's magnitudes share one exponent, one upper fraction and bit 3 of the lower");
  const bool shared_row = COOP && sp.coop > 1;          // (uniform) then the factors are loaded behind the hand-over: they would
  ExpFactors ef;                                        // only take registers from it
  if (!shared_row) ef = load_exp_factors(tab_e, tid);
  uint32_t* const columns = (uint32_t*)list.list;       // (read before the next barrier; the list's entries come after it)
  columns[tid] = M2;                                    // the lane's maximum
  {
    const uint32_t m2 = wave_reduce_u32(M2, HP_NONE2, [](uint32_t x, uint32_t y) { return pk_max_f16(x, y); });
    if (lane == 0) hs.red_m[wid] = m2;
  }
  __syncthreads();                                     // histogram, map, columns and wave results complete
  C2T_PT(PT_HIST_COMPLETE);
  if (wid == NW - 1) {                                  // masked logits counted by lane: folded into the one count (read after the next barrier)
    const int nm = wave_sum_i((int)(hs.out.masked_by_lane[lane] >> 16));
    if (lane == 0 && nm) hs.out.n_masked += nm;         // every other addition to it happened before the barrier above
  }
  uint32_t m2 = HP_NONE2;
#pragma unroll
  for (int w = 0; w < NW; ++w) m2 = pk_max_f16(m2, hs.red_m[w]);
  const uint32_t w0 = (uint32_t)(WPL * tid);            // the lane's words
  if (REPL > 1) {                                       // fold the copies into the first: only this lane touches these words
#pragma unroll
    for (int j = 0; j < WPL; j += 4) {
      uint4 t = *(const uint4*)(hist + w0 + j);
#pragma unroll
      for (int r = 1; r < REPL; ++r) {
        const uint4 u = *(const uint4*)(hist + r * HP_WORDS + w0 + j);
        t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;  // a carry out of a 16-bit half shows in the total, like a counter overflow
      }
      *(uint4*)(hist + w0 + j) = t;
    }
  }
  // ---------------- cells that can hold one of the K largest ----------------
  // All cells whose key reaches a lower bound of the K-th largest logit (for K > COLUMNS_MAX_K: that logit itself) are listed, and their chunks
  // requested, one a thread; the sums below take as long as the answer.
  uint32_t column = HP_NONE2;
#pragma unroll
  for (int w = 0; w < NW; ++w) column = pk_max_f16_raw(column, columns[w * WAVE + lane]);
  if (shared_row) {
    if (!share_row<NT>(tid, sp, split, row_launched, st.row_tickets + slot, sg, hist, w0, map, &hs.out, column, m2)) return SegmentTop{HANDED_OVER, false};
    sg = make_segment<8>(V, 0, (V + 7) / 8);             // the epilogue below is the whole row's
    ef = load_exp_factors(tab_e, tid);
    __syncthreads();                                     // the row's map
  }
  if (!TOPM && wid == NW - 1 && sp.nsplit == 1) request_parent(st, b, slot, *rr);
  float tau;
  if (__builtin_expect(K > COLUMNS_MAX_K, 0)) {
    tau = bound_of_counts(kth_of_counts<NT>(tid, (LdsWords)hist, K, (HistSharedLds<NT>)&hs));
  } else {
    tau = bound_of_patterns(column, K);
  }
  const int ncells = quad_cells_in_segment<NT>(sg.ncell);
  // Four workgroups a CU: a place for each of a lane's cells as it is found (append_place; all of a wavefront's at once was 0.6 % slower than an addition each).
  // A workgroup alone on its CU, which would wait out every round trip, takes the places of a wavefront's cells by one addition (1.3 % of a phase).
  if (WPS == 8) {
#pragma unroll 1
    for (int c8 = tid * 8; c8 < ncells; c8 += NT * 8) {  // eight keys per read (the map is padded to 16 bytes)
      const uint4 kq = *(const uint4*)(map + c8);
      const uint32_t kw[4] = {kq.x, kq.y, kq.z, kq.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float kv = (j & 1) ? bf16_hi(kw[j >> 1]) : bf16_lo(kw[j >> 1]);
        if (c8 + j < ncells && kv >= tau) {
          const int at = append_place(&hs.n_cells);
          if (at < sel.cell_cap) hs.cells[at] = c8 + j;
        }
      }
    }
  } else {
#pragma unroll 1
    for (int w8 = wid * (WAVE * 8); w8 < ncells; w8 += NT * 8) {
      const int c8 = w8 + lane * 8;
      uint32_t hit = 0u;
      if (c8 < ncells) {
        const uint4 kq = *(const uint4*)(map + c8);
        const uint32_t kw[4] = {kq.x, kq.y, kq.z, kq.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float kv = (j & 1) ? bf16_hi(kw[j >> 1]) : bf16_lo(kw[j >> 1]);
          hit |= (c8 + j < ncells && kv >= tau ? 1u : 0u) << j;
        }
      }
      int at = append_places(__popc(hit), &hs.n_cells);
      while (hit) {
        const int j = __ffs(hit) - 1; hit &= hit - 1;
        if (at < sel.cell_cap) hs.cells[at] = c8 + j;
        ++at;
      }
    }
  }
  __syncthreads();
  C2T_PT(PT_CELLS_LISTED);
  const int n_cells = uniform(hs.n_cells);
  const bool listed = n_cells <= sel.cell_cap;           // (uniform) else settle_hist makes the list
  int my_chunk = -1;
  uint4 cell_q = make_uint4(0u, 0u, 0u, 0u);
  if (listed && tid < n_cells * CPC) {                   // n_cells <= cell_cap <= NT / CPC
    const int ch = sg.c0 + chunk_of_quad_cell<NT>(hs.cells[tid / CPC], tid % CPC);
    if (ch < sg.c1) {
      my_chunk = ch;
      if (WPS == 8) lds_chunk_load(rowp + ch, lds_address(map) + (uint32_t)wid * (WAVE * 16u));   // the map has been read: its place takes a chunk a thread
      else cell_q = rowp[ch];
    }
  }
  const float m = fmaxf(bf16_lo(m2), bf16_hi(m2));      // largest logit; exact whenever the row stays on this path

  // ---------------- Z = sum n_v e^v and S = sum n_v (v - m) e^v ----------------
  // Every term of S has the same sign and nothing cancels: rows whose entropy is tiny keep their relative accuracy.
  double Z = 0.0, S = 0.0, Zp = 0.0, Sp = 0.0;
  int lane_pos = 0, lane_neg = 0;
  const double md = (double)m;
  {
    // low half: count of +|v_j|, high half: count of -|v_j|
    uint32_t cw[WPL];
#pragma unroll
    for (int j = 0; j < WPL; j += 4) {
      const uint4 t = *(const uint4*)(hist + w0 + j);
      cw[j] = t.x; cw[j + 1] = t.y; cw[j + 2] = t.z; cw[j + 3] = t.w;
    }
#pragma unroll
    for (int j = 0; j < WPL; ++j) { lane_pos += (int)(cw[j] & 0xffffu); lane_neg += (int)(cw[j] >> 16); }
    // typical rows leave the lanes (and whole waves) of the small magnitudes empty: they skip the fp64 work
    if (lane_pos | lane_neg) {
#pragma unroll
    for (int j = 0; j < WPL; ++j)                       // 64-register build: the halves are unpacked again below rather than
      if (WPS == 8) asm volatile("" : "+v"(cw[j]));     // kept from above in sixteen registers (which spilled the thread index)
    const bool b3 = ((WPL * tid) & 8) != 0;
    const double e0p = b3 ? ef.ap * ef.cp[3] : ef.ap, e0n = b3 ? ef.an * ef.cn[3] : ef.an;
#pragma unroll
    for (int j = 0; j < WPL; ++j) {
      const double vp = (double)hp_value_of_mag(WPL * tid + j, false);
      double ep = e0p, en = e0n;                                   // e^(+|v_j|), e^(-|v_j|)
      if (j & 4) { ep *= ef.cp[2]; en *= ef.cn[2]; }
      if (j & 2) { ep *= ef.cp[1]; en *= ef.cn[1]; }
      if (j & 1) { ep *= ef.cp[0]; en *= ef.cn[0]; }
      const double tp = (double)(cw[j] & 0xffffu) * ep;            // n * e^v (0 for an empty bin)
      const double tn = (double)(cw[j] >> 16) * en;
      if (TOPM) {                                                  // the positive values' share kept apart
        Zp += tp; Sp += (vp - md) * tp;
        Z += tn; S += (-vp - md) * tn;
      } else {
        Z += tp; S += (vp - md) * tp;
        Z += tn; S += (-vp - md) * tn;
      }
      __builtin_amdgcn_sched_barrier(0);                           // one bin pair at a time: keeps live registers low
    }
    }
  }
  // TOPM: the lane's sums over its positive and over its negative values
  const double Zpos = Zp, Spos = Sp, Zneg = Z, Sneg = S;
  if (TOPM) { Z += Zp; S += Sp; }
  // (uniform) wavefronts without a count, six of eight in typical rows, have nothing to add up: they go on to the listed logits
  const bool counts = TOPM || __builtin_amdgcn_ballot_w64((lane_pos | lane_neg) != 0) != 0ull;
  if (counts) { Z = wave_sum(Z); S = wave_sum(S); }
  int incl_p = 0, incl_n = 0;
  if (TOPM) {
    incl_p = wave_scan_incl(lane_pos); incl_n = wave_scan_incl(lane_neg);
    if (lane == WAVE - 1) { hs.scan_p[wid] = incl_p; hs.scan_n[wid] = incl_n; }
  }
  const int total = counts ? wave_sum_i(lane_pos + lane_neg) : 0;
  C2T_PT(PT_SUMS);
  // e^-m for the entropy, which would have to wait for it: by a wavefront of magnitudes below 2^-17, which has hardly a count ever, while the cells are on their way
  if (!TOPM && wid == 1) {
    const double e = exp(-md);
    if (lane == 0) hs.e_minus_m = e;
  }
  // ---------------- their logits that reach the bound ----------------
  {
    if (WPS == 8) { wait_vector_memory(); cell_q = *(const uint4*)((unsigned char*)map + tid * 16); }
    float* el_v = list.values();
    int32_t* el_i = list.ids();
    if (wid * WAVE < n_cells * CPC) {                    // wavefronts with a cell
      float x[8];
      LogitTraits<1>::unpack(cell_q, x);
      uint32_t hit = 0u;
#pragma unroll
      for (int j = 0; j < 8; ++j) hit |= (x[j] >= tau ? 1u : 0u) << j;
      if (my_chunk < 0) hit = 0u;
      else if (my_chunk * 8 + 8 > V) hit &= (1u << (V - my_chunk * 8)) - 1u;
      int at = 0;
      if (WPS != 8) at = append_places(__popc(hit), &hs.n_el);
      // One pass a logit that reaches the bound, of which few chunks hold a second one: a branch for each of the eight places was a
      // hundred instructions of a wavefront that issues one every four cycles (2.3 % of a phase of one sequence).
      while (hit) {
        const int j = __ffs(hit) - 1; hit &= hit - 1;
        const uint32_t w = (j & 4) ? ((j & 2) ? cell_q.w : cell_q.z) : (j & 2) ? cell_q.y : cell_q.x;
        if (WPS == 8) at = append_place(&hs.n_el);
        if (at < HIST_LIST) { el_v[at] = (j & 1) ? bf16_hi(w) : bf16_lo(w); el_i[at] = my_chunk * 8 + j; }
        ++at;
      }
    }
  }
  if (lane == 0) { hs.red_d[0][wid] = Z; hs.red_d[1][wid] = S; hs.total[wid] = total; }
  if (tid == 0) hs.m = m;
  __syncthreads();                                       // sums and list complete
  C2T_PT(PT_CELLS_READ);

  // The last wavefront forms the entropy at once, ahead of the look at the row's rarer cases and while the others rank the list (a row that leaves
  // this path has its record made again).  Its logarithm and division are 0.6 us, which the ranking hides then.  With the parent's values and e^-m requested and formed here it was 0.8 us and a
  // round trip behind the ranking.  Phases without each over those with it: the values requested ahead (request_parent) 1.025 (one sequence of 32000), 1.020 (128256), 1.017 (1024
  // chains), 1.016 (32 reranked), 1.003 (64 of 128256); e^-m by another wavefront 1.003 to 1.007; the entropy ahead of the rarer cases 1.007 (one of 32000), 0.999 to 1.003 (others).
  if (!TOPM && wid == NW - 1 && sp.nsplit == 1) {
    const RowPartial r = combine_hist<NT, false>(hs, 0, *rr);
    row_entropy(0, r.ref, hs.e_minus_m, r.Z, r.S, r.flags, *rr);
  }
  int counted = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) counted += hs.total[w];
  const int n_tiny = uniform(hs.out.n_tiny), n_ninf = hs.out.n_masked;
  const int n_elems = (sg.tail_chunk >= 0 ? (sg.ncell - 1) * 8 + sg.tail_valid : sg.ncell * 8);
  int n_el = listed ? uniform(hs.n_el) : HIST_LIST + 1;
  // Leave this path (uniformly) if a logit that is not masked lies above the window (|x| >= 2^7, +inf, NaN), or if a
  // 16-bit counter overflowed (the total is then off by a multiple of 65535 or 65536).
  bool leave = uniform(hs.out.mag_max >= HP_MAG_LO + HP_MAG_SPAN || counted + n_tiny + n_ninf != n_elems ? 1 : 0) != 0;
  int before_p = 0, before_n = 0, tot_p = 0;            // TOPM: counts in lower lanes / in the whole segment
  if (TOPM) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wid) { before_p += hs.scan_p[w]; before_n += hs.scan_n[w]; }
      tot_p += hs.scan_p[w];
    }
    tot_p = uniform(tot_p);
    // ... or if some but not all of the logits below the window are among the M largest (which ones cannot be told from the histogram)
    leave = leave || (n_tiny > 0 && tot_p < M && M < tot_p + n_tiny);
  }
  if (TOPM && !leave) {                                  // (uniform; ahead of the calls below: little is live across them)
    // Eq. 2, second line: Z and S restricted to the M largest logits.  A lane's values, from the
    // top: its positive magnitudes descending, then its negative ones ascending; `above` of them
    // lie in other lanes.
    double zm = 0.0, sm = 0.0;
    // (logits below the window, |x| < 2^-25, rank between the positive and the negative window values)
    const int above_p = tot_p - (before_p + incl_p), above_n = tot_p + n_tiny + before_n + incl_n - lane_neg;
    // A lane whose positive (negative) values all rank within the first M contributes the sums it
    // already has.  The bins of the one lane that holds the M-th largest logit are told apart by WPL lanes of its wavefront, one
    // exponential each at the same time instead of WPL one after the other (by that lane alone, out of line, 32 sequences of 128256 with M = 1000
    // took 207.5 us a phase, 194.8 so).  They are computed rather than fetched from the tables again: a load issued at this point waits behind all the logits in flight
    // on the CU, several microseconds that the whole workgroup would spend at its next barrier.
    const bool part_p = lane_pos > 0 && above_p < M && above_p + lane_pos > M;
    const bool part_n = lane_neg > 0 && above_n < M && above_n + lane_neg > M;
    if (lane_pos > 0 && above_p + lane_pos <= M) { zm += Zpos; sm += Spos; }
    if (lane_neg > 0 && above_n + lane_neg <= M) { zm += Zneg; sm += Sneg; }
    const uint64_t boundary = __builtin_amdgcn_ballot_w64(part_p || part_n);
    if (boundary != 0ull) {                              // (uniform) one lane of the workgroup at most
      const int owner = (int)__builtin_ctzll(boundary);
      const bool positive = __builtin_amdgcn_readlane(part_p ? 1 : 0, owner) != 0;
      const int above = __builtin_amdgcn_readlane(part_p ? above_p : above_n, owner);
      const int mag = WPL * (wid * WAVE + owner) + (positive ? WPL - 1 - lane : lane);       // lane 0: the largest of its values
      int n = 0;
      if (lane < WPL) n = (int)(positive ? hist[mag] & 0xffffu : hist[mag] >> 16);
      const int take = min(n, M - (above + wave_scan_incl(n) - n));
      if (take > 0) {
        const double v = (double)hp_value_of_mag((uint32_t)mag, !positive), t = (double)take * exp(v);
        zm += t; sm += (v - md) * t;
      }
    }
    zm = wave_sum(zm); sm = wave_sum(sm);
    if (lane == 0) { hs.red_m_d[0][wid] = zm; hs.red_m_d[1][wid] = sm; }
    if (tid == 0) hs.tot_p = tot_p;
    __syncthreads();
  }
  // (A bound among the window's positive values is reached by K logits, so that the K-th largest is one of them too: logits below the window change
  // nothing then.  Asked about each row with such a logit, settle_hist took a layer of three rows of 8279 from 11.8 us to 13.6, one of 128256 from 15.9 to 17.4.)
  if (__builtin_expect(!leave && ((n_tiny > 0 && !(tau >= hp_value_of_mag(0u, false))) || n_el > HIST_LIST || n_el < min(K, n_elems)), 0)) {
    n_el = uniform(settle_hist<NT>(tid, rowp, V, K, sg, (LdsWords)hist, lds_address(list.list), (LdsHalves)map, sel.cell_cap, (HistSharedLds<NT>)&hs));
    leave = n_el == UNSETTLED;
    __syncthreads();                                     // the list is complete
  }
  if (__builtin_expect(leave, 0)) {
    __syncthreads();
    generic_segment<1, NT>(tid, rowp, V, K, M, sg, (unsigned char*)hist, sel, rr, 2u);
    return SegmentTop{RANKED_IN_RR, false};
  }
  return SegmentTop{n_el, !TOPM && sp.nsplit == 1};
}

// grid: rows_launched * nsplit workgroups of NT threads.
// Dynamic LDS (sp.lds_bytes): see hist_lds_bytes; generic_segment and the tail reuse all of it.
// WPS: waves per SIMD the kernel is built for.  8 = four workgroups per CU on 64 registers a lane;
// 6 = three workgroups per CU on 80 registers, which needs no spills.
template <int NT, bool TOPM, int WPS, int REPL, bool COOP, bool STREAMED>
__global__ __launch_bounds__(NT, WPS) void k_logits_hist(
    C2T_START_LIST(C2T_AS_PARAMETER) const double* __restrict__ tab_e, const float* __restrict__ cls, TreeState st, ScoreParams sp) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ RowResult rr;
  __shared__ HistShared<NT> hs;
  C2T_PT(PT_START);
  constexpr int REST = START_BYTES + 16;
  const uint32_t rows_per_seq = shape & 0xffu, F = (shape >> 8) & 0xffu;
  const QuotientRemainder wg = divide(blockIdx.x, Division{per_row, inv_per_row});     // per_row workgroups a row: splits of it, or those that share it
  const int split = (int)wg.r;
  const bool dealt = WPS == 8 && (shape & SHAPE_COMPACT) != 0u;                          // (uniform)
  RowOfWorkgroup rw;
  constexpr int ARGUMENT_BYTES = REST + (int)sizeof(TreeState) + (int)sizeof(ScoreParams);
  if (dealt) {
    if (threadIdx.x < WAVE) {
      rw = dealt_row(nfs, (int)B, (int)wg.q);
      if (threadIdx.x == 0) { hs.kth[0] = rw.b; hs.kth[1] = rw.f; hs.kth[2] = rw.nf; }
    } else {
      touch_kernel_arguments<ARGUMENT_BYTES>();
      clear_counts<NT - WAVE, REPL>((int)threadIdx.x - WAVE, (uint32_t*)dyn_lds, hs);
    }
    __syncthreads();
    rw.b = __builtin_amdgcn_readfirstlane(hs.kth[0]); rw.f = __builtin_amdgcn_readfirstlane(hs.kth[1]); rw.nf = __builtin_amdgcn_readfirstlane(hs.kth[2]);
  } else {
    rw = row_of_workgroup(nfs, st, sp.layer, B, inv_B, rows_per_seq, inv_rows, wg.q);
    touch_kernel_arguments<ARGUMENT_BYTES>();
  }
  const int K = sp.K, b = rw.b, f = rw.f, rl = b * (int)rows_per_seq + f, nf = rw.nf;
  if (f >= nf) { if (nf == 0) end_of_sequence(st, sp, b, f, split); return; }   // uniform for the workgroup
  const int64_t row = (int64_t)b * F + f;
  const uint4* rowp = (const uint4*)((const char*)logits + row * row_stride_bytes);
  const Segment sg = make_segment<8>(V, split, cps);
  C2T_PT(PT_ROW);
  // The classifier's parameters (5h+1 <= 1281 floats) are copied to LDS for the scoring step: the
  // loads are issued now, four floats a thread, and stored behind the streaming loop.
  const ClassifierStage cst = stage_classifier(threadIdx.x, cls, sp.h, TOPM ? nullptr : (float*)(dyn_lds + sp.w_lds_off));
  const SelectLds sel = make_select_lds<NT, 8>(dyn_lds, sp.lds_bytes), list = hist_list(dyn_lds + HP_WORDS * 4 * REPL);
  SegmentTop top{RANKED_IN_RR, false};
  int tid = threadIdx.x;
  if (sg.ncell == 0) {                                     // (loaded again here: the copy above must not stay in registers for this)
    store_classifier(tid, stage_classifier(tid, cls, sp.h, cst.dst));
    if (tid == 0) { rr.part = empty_partial(); rr.ZM = 0.0; rr.SM = 0.0; }
    __syncthreads();
  } else {
    top = hist_segment<NT, TOPM, WPS, REPL, COOP, STREAMED>(rowp, V, K, TOPM ? sp.M : 0, sg, tab_e, (uint32_t*)dyn_lds, list,
                                                  (uint16_t*)(dyn_lds + hist_lds_bytes<NT>(REPL)), sel, &rr, hs, cst, st, sp, split, rl, b, row, dealt, tid);
    if (COOP && top.n_el == HANDED_OVER) { C2T_PT_FLUSH(); return; }   // a shared row's segment, handed over
  }
  const TailArguments& ta = tail_arguments<REST>();
  finish_layer<NT>(tid, ta.st, ta.sp, b, f, nf, split, rl, rr, top, list, sel, dyn_lds, cls, cst.dst,
                   [&] { if (top.n_el >= 0) combine_hist<NT, TOPM>(hs, sp.M, rr); },
                   [&](RowResult& r) { if (TOPM) top_m_of_whole_row<1, NT>(tid, rowp, V, sp.M, r, sel); });
}

// Plain streaming read: the practical HBM ceiling.
__global__ __launch_bounds__(1024) void k_stream_read(const uint4* __restrict__ p, size_t n16, uint32_t* out) {
  uint32_t acc = 0;
  size_t i = (size_t)blockIdx.x * 1024 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 1024;
  for (; i + 3 * stride < n16; i += 4 * stride) {
    const uint4 a = p[i], b = p[i + stride], c = p[i + 2 * stride], d = p[i + 3 * stride];
    acc += a.x ^ a.y ^ a.z ^ a.w; acc += b.x ^ b.y ^ b.z ^ b.w;
    acc += c.x ^ c.y ^ c.z ^ c.w; acc += d.x ^ d.y ^ d.z ^ d.w;
  }
  for (; i < n16; i += stride) { const uint4 a = p[i]; acc += a.x ^ a.y ^ a.z ^ a.w; }
  acc = (uint32_t)wave_sum_i((int)acc);
  if ((threadIdx.x & 63) == 0 && acc == 0x9e3779b9u) atomicAdd(out, acc);   // keeps the loads alive
}

// The same read with the layer kernel's access pattern and nothing else: one workgroup of 512
// threads per row, lane t reads chunks t, t+512, ... of its row, four in flight, non-temporal.  What
// the memory system delivers to that pattern is the ceiling the logits pass can be held against.
__global__ __launch_bounds__(512, 8) void k_stream_read_rows(const char* __restrict__ p, int64_t row_stride_bytes, int chunks_per_row, uint32_t* out) {
  const uint4* row = (const uint4*)(p + (int64_t)blockIdx.x * row_stride_bytes);
  uint32_t acc = 0;
  int g = threadIdx.x;
  for (; g + 3 * 512 < chunks_per_row; g += 4 * 512) {
    const uint4 a = load_stream(row + g), b = load_stream(row + g + 512), c = load_stream(row + g + 1024), d = load_stream(row + g + 1536);
    acc += a.x ^ a.y ^ a.z ^ a.w; acc += b.x ^ b.y ^ b.z ^ b.w;
    acc += c.x ^ c.y ^ c.z ^ c.w; acc += d.x ^ d.y ^ d.z ^ d.w;
  }
  for (; g < chunks_per_row; g += 512) { const uint4 a = load_stream(row + g); acc += a.x ^ a.y ^ a.z ^ a.w; }
  acc = (uint32_t)wave_sum_i((int)acc);
  if ((threadIdx.x & 63) == 0 && acc == 0x9e3779b9u) atomicAdd(out, acc);   // keeps the loads alive
}

}  // namespace c2t
