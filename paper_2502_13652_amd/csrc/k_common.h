// Shared device helpers for the C2T kernels (gfx950, 64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace c2t {

constexpr int WAVE = 64;

// Optional build (-DC2T_PHASE_TIMES): thread 0 of every workgroup of the layer kernel notes the time
// (100 MHz wall clock) at which it passes each phase boundary, PT_START ahead of everything, PT_ROW when it knows its row; c2t_phase_times_read copies the notes
// out.  In the normal build the marks expand to nothing.
constexpr int PT_WORKGROUPS = 8192, PT_SLOTS = 16;
enum PhaseMark { PT_START = 0, PT_STREAM_END, PT_HIST_COMPLETE, PT_SUMS, PT_ROW, PT_CELLS_LISTED, PT_CELLS_READ, PT_RANKED,
                 PT_PUBLISHED, PT_TICKET, PT_PRUNED, PT_PRUNE_LOADED, PT_PRUNE_FIRST, PT_PRUNE_PRESELECTED, PT_PRUNE_RANKED, PT_MERGED };
#ifdef C2T_PHASE_TIMES
__device__ unsigned long long c2t_phase_times[PT_WORKGROUPS * PT_SLOTS];
// The marks go to LDS (a store to memory would be waited for at the next hand-over) and out at the workgroup's end.
__device__ __forceinline__ unsigned long long* phase_marks() { __shared__ unsigned long long t[PT_SLOTS]; return t; }
__device__ __forceinline__ void phase_start() {
  const unsigned long long now = wall_clock64();
  for (int i = 0; i < PT_SLOTS; ++i) phase_marks()[i] = i == 0 ? now : 0ull;
}
__device__ __forceinline__ void phase_flush() {
  if (threadIdx.x == 0 && blockIdx.x < PT_WORKGROUPS) for (int i = 0; i < PT_SLOTS; ++i) c2t_phase_times[blockIdx.x * PT_SLOTS + i] = phase_marks()[i];
}
#define C2T_PT(i) do { if (threadIdx.x == 0) { if ((i) == 0) c2t::phase_start(); else c2t::phase_marks()[i] = wall_clock64(); } } while (0)
#define C2T_PT_FLUSH() c2t::phase_flush()
#else
#define C2T_PT(i) do { } while (0)
#define C2T_PT_FLUSH() do { } while (0)
#endif

// Per (row, split) result of the logits pass: Z = sum_j e^(x_j - a), S = sum_j (x_j - ref) e^(x_j - a),
// both fp64, where ref is the segment's largest logit and the exponent offset a is ref (two-pass
// path) or 0 (histogram path, whose table holds e^v itself).
struct __attribute__((aligned(16))) RowPartial {
  double ref;     // largest logit of the segment (exact); -inf for an empty or all -inf segment
  double a;       // offset of the sums
  double Z;
  double S;
  int32_t n_top;  // entries of the segment's top list that are valid (<= K)
  uint32_t flags; // bit 0: NaN or +inf seen; bit 1 (informational): a bf16 segment took the two-pass path
};

// the record of an empty segment
__device__ __forceinline__ RowPartial empty_partial() {
  RowPartial r;
  r.ref = -INFINITY; r.a = 0.0; r.Z = 0.0; r.S = 0.0; r.n_top = 0; r.flags = 0u;
  return r;
}

// Device-coherent accesses for data one workgroup writes and another reads inside the same kernel:
// they go to the coherence point, so neither side needs cache-wide write-backs or invalidations.
__device__ __forceinline__ void st_dev(uint32_t* p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_dev(int32_t* p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_dev(float* p, float v) { st_dev((uint32_t*)p, __float_as_uint(v)); }
__device__ __forceinline__ void st_dev(double* p, double v) {
  __hip_atomic_store((unsigned long long*)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t ld_dev(const int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t ld_dev(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float ld_dev(const float* p) { return __uint_as_float(ld_dev((const uint32_t*)p)); }
__device__ __forceinline__ double ld_dev(const double* p) {
  return __longlong_as_double((long long)__hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void st_dev(RowPartial* p, const RowPartial& r) {
  st_dev(&p->ref, r.ref); st_dev(&p->a, r.a); st_dev(&p->Z, r.Z); st_dev(&p->S, r.S);
  st_dev(&p->n_top, r.n_top); st_dev(&p->flags, r.flags);
}
__device__ __forceinline__ RowPartial ld_dev(const RowPartial* p) {
  RowPartial r;
  r.ref = ld_dev(&p->ref); r.a = ld_dev(&p->a); r.Z = ld_dev(&p->Z); r.S = ld_dev(&p->S);
  r.n_top = ld_dev(&p->n_top); r.flags = ld_dev(&p->flags);
  return r;
}
// every vector memory operation this wave has issued is complete
__device__ __forceinline__ void wait_vector_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Requests every 64-byte line of the kernel's arguments at once.  The compiler loads an argument where it is used,
// and a first touch of a line costs 320 cycles (0.14 us) each time, one after the other through the latency-bound tail
// of a layer; a line that is in the scalar cache costs 44.
template <int BYTES>
__device__ __forceinline__ void touch_kernel_arguments() {
  const __attribute__((address_space(4))) char* p = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  static_assert(BYTES > 448 && BYTES <= 512, "eight lines");
  uint32_t a, b, c, d, e, f, g, h;
  asm volatile("s_load_dword %0, %8, 0\n s_load_dword %1, %8, 64\n s_load_dword %2, %8, 128\n s_load_dword %3, %8, 192\n"
               "s_load_dword %4, %8, 256\n s_load_dword %5, %8, 320\n s_load_dword %6, %8, 384\n s_load_dword %7, %8, 448\n s_waitcnt lgkmcnt(0)"
               : "=&s"(a), "=&s"(b), "=&s"(c), "=&s"(d), "=&s"(e), "=&s"(f), "=&s"(g), "=&s"(h) : "s"(p));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// a value that is the same in every lane, as the compiler cannot know of one that comes from LDS: what is decided by it is then branched on, not masked
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// monotone map float -> uint32 (total order of the reals; -0 and +0 map to the same key)
__device__ __forceinline__ uint32_t sortable_key(float x) {
  uint32_t u = __float_as_uint(x + 0.0f);   // -0 + 0 = +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k) {
  uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __uint_as_float(u);
}

__device__ __forceinline__ int lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// ---- wavefront reductions and scan on DPP (data-parallel primitives: lane permutations inside
// the VALU, no LDS round trip).  Rows are groups of 16 lanes.  The combination order is fixed, so
// floating-point results are reproducible.
#define C2T_DPP_QUAD_XOR1 0xB1      /* quad_perm [1,0,3,2] */
#define C2T_DPP_QUAD_XOR2 0x4E      /* quad_perm [2,3,0,1] */
#define C2T_DPP_ROW_HALF_MIRROR 0x141
#define C2T_DPP_ROW_MIRROR 0x140
#define C2T_DPP_ROW_BCAST15 0x142
#define C2T_DPP_ROW_BCAST31 0x143
#define C2T_DPP_ROW_SHR(n) (0x110 | (n))
#define C2T_DPP_QUAD_XOR3 0x1B      /* quad_perm [3,2,1,0] */
#define C2T_DPP_ROW_SHL(n) (0x100 | (n))
#define C2T_DPP_ROW_ROR(n) (0x120 | (n))

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t identity, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v) {      // identity 0.0
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = dpp_u32<CTRL, ROW_MASK>(0u, (uint32_t)u), hi = dpp_u32<CTRL, ROW_MASK>(0u, (uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t readlane63_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }

// every lane of a row gets the row's result; then lane 63 gets the wave's (read it with readlane63)
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t v, uint32_t ident, Op op) {
  v = op(v, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(ident, v));
  v = op(v, dpp_u32<C2T_DPP_QUAD_XOR2, 0xf>(ident, v));
  v = op(v, dpp_u32<C2T_DPP_ROW_HALF_MIRROR, 0xf>(ident, v));
  v = op(v, dpp_u32<C2T_DPP_ROW_MIRROR, 0xf>(ident, v));
  v = op(v, dpp_u32<C2T_DPP_ROW_BCAST15, 0xa>(ident, v));
  v = op(v, dpp_u32<C2T_DPP_ROW_BCAST31, 0xc>(ident, v));
  return readlane63_u32(v);
}
__device__ __forceinline__ float wave_max(float v) {
  return __uint_as_float(wave_reduce_u32(__float_as_uint(v), __float_as_uint(-INFINITY),
                                         [](uint32_t a, uint32_t b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); }));
}
__device__ __forceinline__ int wave_sum_i(int v) {
  return (int)wave_reduce_u32((uint32_t)v, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ double wave_sum(double v) {
  v = v + dpp_f64<C2T_DPP_QUAD_XOR1, 0xf>(v);
  v = v + dpp_f64<C2T_DPP_QUAD_XOR2, 0xf>(v);
  v = v + dpp_f64<C2T_DPP_ROW_HALF_MIRROR, 0xf>(v);
  v = v + dpp_f64<C2T_DPP_ROW_MIRROR, 0xf>(v);
  v = v + dpp_f64<C2T_DPP_ROW_BCAST15, 0xa>(v);
  v = v + dpp_f64<C2T_DPP_ROW_BCAST31, 0xc>(v);
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = readlane63_u32((uint32_t)u), hi = readlane63_u32((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// inclusive prefix sum across the wave (Hillis-Steele inside each row, then row carries)
__device__ __forceinline__ int wave_scan_incl(int v) {
  uint32_t u = (uint32_t)v;
  u += dpp_u32<C2T_DPP_ROW_SHR(1), 0xf>(0u, u);
  u += dpp_u32<C2T_DPP_ROW_SHR(2), 0xf>(0u, u);
  u += dpp_u32<C2T_DPP_ROW_SHR(4), 0xf>(0u, u);
  u += dpp_u32<C2T_DPP_ROW_SHR(8), 0xf>(0u, u);
  u += dpp_u32<C2T_DPP_ROW_BCAST15, 0xa>(0u, u);
  u += dpp_u32<C2T_DPP_ROW_BCAST31, 0xc>(0u, u);
  return (int)u;
}

// ---- sorting in rows of 16 lanes: a lane permutation and a v_med3 a stage, no scalar instruction on the way ----
__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ uint32_t xor4_of_row(uint32_t x) {
  const uint32_t up = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, C2T_DPP_ROW_SHL(4), 0xf, 0x5, false);      // quads 0 and 2: from the lanes above
  return (uint32_t)__builtin_amdgcn_update_dpp((int)up, (int)x, C2T_DPP_ROW_SHR(4), 0xf, 0xa, false);                   // quads 1 and 3: from the lanes below
}
// of a pair of lanes that differ in bit b the one with the bit clear takes the maximum: the median with the largest number, the other with the smallest
__device__ __forceinline__ uint32_t takes_max(int bit) { return (uint32_t)(((lane_id() >> bit) & 1) - 1); }
// every row of 16 lanes descending
__device__ __forceinline__ uint32_t sort_rows_of_16(uint32_t v) {
  const uint32_t c0 = takes_max(0), c1 = takes_max(1), c2 = takes_max(2), c3 = takes_max(3);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, v), c0);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR3, 0xf>(0u, v), c1);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, v), c0);
  v = med3_u32(v, dpp_u32<C2T_DPP_ROW_HALF_MIRROR, 0xf>(0u, v), c2);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR2, 0xf>(0u, v), c1);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, v), c0);
  v = med3_u32(v, dpp_u32<C2T_DPP_ROW_MIRROR, 0xf>(0u, v), c3);
  v = med3_u32(v, xor4_of_row(v), c2);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR2, 0xf>(0u, v), c1);
  return med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, v), c0);
}
// The 32nd largest of the wavefront's 64 values; uniform.  Two falling runs, one of them reversed: the lane-wise maxima are the larger half, the minima the
// smaller, each of them rising and then falling or the other way round.  So the rows are merged to two falling runs of 32, and the
// smallest of the larger half of these is the answer.
__device__ __forceinline__ uint32_t largest_32nd(uint32_t v) {
  const uint32_t c0 = takes_max(0), c1 = takes_max(1), c2 = takes_max(2), c3 = takes_max(3), c4 = takes_max(4);
  v = sort_rows_of_16(v);
  const auto rows = __builtin_amdgcn_permlane16_swap(v, v, false, false);        // the even rows, twice each; the odd rows
  v = med3_u32((uint32_t)rows[0], dpp_u32<C2T_DPP_ROW_MIRROR, 0xf>(0u, (uint32_t)rows[1]), c4);
  v = med3_u32(v, dpp_u32<C2T_DPP_ROW_ROR(8), 0xf>(0u, v), c3);
  v = med3_u32(v, xor4_of_row(v), c2);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR2, 0xf>(0u, v), c1);
  v = med3_u32(v, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, v), c0);
  const auto runs = __builtin_amdgcn_permlane32_swap(v, v, false, false);        // the lower run, twice; the upper run
  const auto upper = __builtin_amdgcn_permlane16_swap((uint32_t)runs[1], (uint32_t)runs[1], false, false);       // its first row; its second row
  const uint32_t reversed = dpp_u32<C2T_DPP_ROW_MIRROR, 0xf>(0u, c4 ? (uint32_t)upper[1] : (uint32_t)upper[0]);
  return wave_reduce_u32(max((uint32_t)runs[0], reversed), 0xffffffffu, [](uint32_t x, uint32_t y) { return min(x, y); });
}
// The n-th largest (1 <= n <= 16) of them; uniform.  As above, the larger halves only: two rows' 16 largest, and the 16 largest of these.
__device__ __forceinline__ uint32_t nth_largest16(uint32_t v, int n) {
  const uint32_t c0 = takes_max(0), c1 = takes_max(1), c2 = takes_max(2), c3 = takes_max(3);
  const auto larger_half = [&](uint32_t x, uint32_t y) {     // of two falling rows, falling
    uint32_t t = max(x, dpp_u32<C2T_DPP_ROW_MIRROR, 0xf>(0u, y));
    t = med3_u32(t, dpp_u32<C2T_DPP_ROW_ROR(8), 0xf>(0u, t), c3);
    t = med3_u32(t, xor4_of_row(t), c2);
    t = med3_u32(t, dpp_u32<C2T_DPP_QUAD_XOR2, 0xf>(0u, t), c1);
    return med3_u32(t, dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, t), c0);
  };
  v = sort_rows_of_16(v);
  const auto rows = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = larger_half((uint32_t)rows[0], (uint32_t)rows[1]);
  const auto halves = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = larger_half((uint32_t)halves[0], (uint32_t)halves[1]);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, n - 1);
}

// Places for a wavefront's entries in a list that several wavefronts append to: `n` entries of this lane go to the returned
// place and the ones behind it.  One LDS addition a wavefront; an addition per entry has every one of them wait out its
// round trip (200 cycles).  Every lane of the wave calls it; a wave without entries returns at once.
__device__ __forceinline__ int append_places(int n, int32_t* counter) {
  if (__builtin_amdgcn_ballot_w64(n != 0) == 0ull) return 0;  // (uniform) most wavefronts have none
  const int incl = wave_scan_incl(n);
  int base = 0;
  if (lane_id() == WAVE - 1) base = atomicAdd(counter, incl);
  return __builtin_amdgcn_readlane(base, WAVE - 1) + incl - n;
}

// The place of one entry of each lane that is here, in a list that others append to as well.  Few lanes add for themselves; many at once, which the LDS would serve
// one after the other, by one addition and their count.  An append by n lanes, in cycles: one addition each 216 to 244 up to sixteen lanes, 260 with 24, 340 with 64 where one wavefront
// appends, 285 with sixteen, 413 with 24, 1056 with 64 where eight do; one for all 336.  So the line may lie anywhere up to some sixteen lanes: with 16 in place of 4
// layers of equal, sorted and few-valued rows, and the phases of usual ones, were the same within 1 %.
constexpr int APPEND_FEW = 4;
__device__ __forceinline__ int append_place(int32_t* counter) {
  const uint64_t here = __builtin_amdgcn_ballot_w64(true);
  const int n = __builtin_popcountll(here);
  if (n <= APPEND_FEW) return atomicAdd(counter, 1);         // (uniform)
  const int before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(here >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)here, 0u));
  int base = 0;
  if (before == 0) base = atomicAdd(counter, n);
  return __builtin_amdgcn_readfirstlane(base) + before;
}

// K-th largest (k >= 1) of the keys held by one wave, NV keys per lane (invalid keys = 0,
// the smallest key).  Radix select from the most significant bit with wave ballots; the
// result is wave-uniform.  If fewer than k keys are valid the result is 0.
// LOW_BIT > 0: the select stops above that bit and the result has its low bits clear: the largest
// such key that at least k keys reach (a lower bound of the k-th largest, for a fraction of the steps).
template <int NV, int LOW_BIT = 0>
__device__ __forceinline__ uint32_t wave_kth_largest(const uint32_t (&key)[NV], int k) {
  uint32_t prefix = 0, care = 0;
  for (int bit = 31; bit >= LOW_BIT; --bit) {
    const uint32_t want = prefix | (1u << bit);
    const uint32_t cmask = care | (1u << bit);
    int cnt = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) cnt += __popcll(__ballot((key[v] & cmask) == want));
    if (cnt >= k) prefix = want; else k -= cnt;
    care = cmask;
  }
  return prefix;
}

}  // namespace c2t
