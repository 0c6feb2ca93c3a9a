// Everything after a row's sums and top-K: the tail that the logits kernels run in place
// (merge of split rows, features + classifier (Eq. 1-3) per row, the two prunings of Sec. 4.2 with
// the node budget and the tree append per sequence, handed from workgroup to workgroup by tickets),
// and the small kernels: reset, emission of the tree mask, position ids and parent links, and the
// EAGLE-2-style reranked emission (Sec. 2.2).
#pragma once
#include <type_traits>

#include "k_common.h"

namespace c2t {

struct TreeState {            // device pointers into the workspace
  float* cls;                 // W1[3h] b1[h] w2[h] b2
  int32_t* n_nodes;           // [B]
  int32_t* nf[2];             // [B] frontier sizes, ping-pong: layer l reads nf[l&1], writes nf[(l+1)&1]
  int32_t* tickets;           // [B] rows of the current layer that have been scored
  int32_t* row_tickets;       // [B][F] splits of the row that have delivered their record
  uint32_t* row_info;         // [B][F] bit 0: row unusable (NaN, +inf, no finite logit); bit 1: two-pass path taken
  uint32_t* status;           // [B]
  int32_t* n_cand;            // [B]
  int32_t* layer_rows;        // [D+1]
  int32_t* fr_tok;            // [B][F]
  int32_t* fr_pslot;          // [B][F]
  int32_t* fr_node;           // [B][F]
  float* fr_P;                // [B][F]
  int32_t* fr_hidx;           // [B][F] history index of the frontier node, -1 = root (rerank contexts only)
  float* fr_s;                // [B][F] smallest classifier logit on its path, +inf for the root
  // history of every scored candidate, [B][D][F*K] (rerank contexts only, else null)
  int32_t* h_tok; int32_t* h_par; float* h_P; float* h_H; float* h_z; float* h_s;
  int32_t* h_ncand;           // [B][D] candidates scored in each layer
  int32_t* h_pos;             // [B][D*F*K] scratch of the reranking
  int32_t* t_tok;             // [B][N]
  int32_t* t_parent;
  int32_t* t_depth;
  float* t_P;
  float* t_H;
  float* t_z;
  int32_t* c_tok;             // [B][F*K]
  float* c_p;
  float* c_P;
  float* c_H;
  float* c_z;
  int32_t* c_kept;
};

__global__ void k_reset(TreeState s, int B, int F, int D) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (s.h_tok) {
    if (i < B) { s.fr_hidx[(int64_t)i * F] = -1; s.fr_s[(int64_t)i * F] = INFINITY; }
    for (int j = i; j < B * D; j += gridDim.x * blockDim.x) s.h_ncand[j] = 0;
  }
  if (i < B) {
    s.n_nodes[i] = 0; s.nf[0][i] = 1; s.nf[1][i] = 0; s.tickets[i] = 0; s.status[i] = 0; s.n_cand[i] = 0;
    s.fr_tok[(int64_t)i * F] = -1; s.fr_pslot[(int64_t)i * F] = 0;
    s.fr_node[(int64_t)i * F] = -1; s.fr_P[(int64_t)i * F] = 1.0f;
  }
  if (i <= D) s.layer_rows[i] = (i == 0) ? B : 0;
  for (int j = i; j < B * F; j += gridDim.x * blockDim.x) s.row_tickets[j] = 0;
}

// A slice of the classifier's parameters on its way to the workspace as a kernel argument.
struct ClsChunk { static constexpr int N = 240; float v[N]; };
__global__ void k_set_classifier(float* __restrict__ cls, int off, int n, ClsChunk c) {
  if ((int)threadIdx.x < n) cls[off + threadIdx.x] = c.v[threadIdx.x];
}

// Eq. 3 in fp32: fixed chain of fused multiply-adds, hidden units in ascending order.
// `w` in global memory: every lane reads the same addresses, so the loads are scalar; but each
// group of hidden units then waits for its own loads (measured: 1.2-1.4 us for 32 hidden units).
__device__ __forceinline__ float mlp_logit(const float* __restrict__ w, int h, float P, float H, float d) {
  const float* W1 = w; const float* b1 = w + 3 * h; const float* w2 = w + 4 * h;
  float z = w[5 * h];
#pragma unroll 4
  for (int j = 0; j < h; ++j) {
    float a = __fmaf_rn(W1[3 * j + 0], P, b1[j]);
    a = __fmaf_rn(W1[3 * j + 1], H, a);
    a = __fmaf_rn(W1[3 * j + 2], d, a);
    a = a > 0.0f ? a : 0.0f;
    z = __fmaf_rn(w2[j], a, z);
  }
  return z;
}
// The same chain with the parameters staged in LDS (broadcast reads, many in flight).
typedef __attribute__((address_space(3))) const float* LdsFloats;
__device__ __forceinline__ float mlp_logit_lds(LdsFloats w, int h, float P, float H, float d) {
  LdsFloats W1 = w; LdsFloats b1 = w + 3 * h; LdsFloats w2 = w + 4 * h;
  float z = w[5 * h];
  if ((h & 3) == 0) {                                        // every array starts on 16 bytes: five wide reads per four units
    typedef float float4v __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const float4v* LdsFloat4s;
#pragma unroll 2
    for (int j = 0; j < h; j += 4) {
      const float4v wa = *(LdsFloat4s)(W1 + 3 * j), wb = *(LdsFloat4s)(W1 + 3 * j + 4), wc = *(LdsFloat4s)(W1 + 3 * j + 8);
      const float4v bb = *(LdsFloat4s)(b1 + j), vv = *(LdsFloat4s)(w2 + j);
      float a0 = __fmaf_rn(wa.x, P, bb.x); a0 = __fmaf_rn(wa.y, H, a0); a0 = __fmaf_rn(wa.z, d, a0); a0 = a0 > 0.0f ? a0 : 0.0f;
      float a1 = __fmaf_rn(wa.w, P, bb.y); a1 = __fmaf_rn(wb.x, H, a1); a1 = __fmaf_rn(wb.y, d, a1); a1 = a1 > 0.0f ? a1 : 0.0f;
      float a2 = __fmaf_rn(wb.z, P, bb.z); a2 = __fmaf_rn(wb.w, H, a2); a2 = __fmaf_rn(wc.x, d, a2); a2 = a2 > 0.0f ? a2 : 0.0f;
      float a3 = __fmaf_rn(wc.y, P, bb.w); a3 = __fmaf_rn(wc.z, H, a3); a3 = __fmaf_rn(wc.w, d, a3); a3 = a3 > 0.0f ? a3 : 0.0f;
      z = __fmaf_rn(vv.x, a0, z); z = __fmaf_rn(vv.y, a1, z); z = __fmaf_rn(vv.z, a2, z); z = __fmaf_rn(vv.w, a3, z);
    }
    return z;
  }
#pragma unroll 4
  for (int j = 0; j < h; ++j) {
    float a = __fmaf_rn(W1[3 * j + 0], P, b1[j]);
    a = __fmaf_rn(W1[3 * j + 1], H, a);
    a = __fmaf_rn(W1[3 * j + 2], d, a);
    a = a > 0.0f ? a : 0.0f;
    z = __fmaf_rn(w2[j], a, z);
  }
  return z;
}

// The same by four neighbouring lanes a candidate (h a multiple of four, at most 16 candidates): each forms every fourth activation, and the
// chain takes them from the four in turn, by lane permutation; all four run it.  Eight vector instructions for four units instead of twenty, in the
// one wavefront that everything waits for: phases with 32 units, one sequence of 128256 115.5 -> 113.5 us, 64 sequences 264.0 -> 262.1.
template <int LANE>
__device__ __forceinline__ float of_quad(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), LANE * 0x55, 0xf, 0xf, true));
}
__device__ __forceinline__ float mlp_logit_quads(LdsFloats w, int h, float P, float H, float d) {
  typedef float float4v __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) const float4v* LdsFloat4s;
  const int q = lane_id() & 3;
  LdsFloats W1 = w + 3 * q; LdsFloats b1 = w + 3 * h + q; LdsFloats w2 = w + 4 * h;
  float z = w[5 * h];
  const auto fours = [&](int j, auto groups) {               // the reads of all groups ahead of the first use
    constexpr int G = decltype(groups)::value;
    float x[G], y[G], t[G], a[G]; float4v v[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int u = j + 4 * g;
      x[g] = W1[3 * u]; y[g] = W1[3 * u + 1]; t[g] = W1[3 * u + 2]; a[g] = b1[u]; v[g] = *(LdsFloat4s)(w2 + u);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      a[g] = __fmaf_rn(x[g], P, a[g]); a[g] = __fmaf_rn(y[g], H, a[g]); a[g] = __fmaf_rn(t[g], d, a[g]);
      a[g] = a[g] > 0.0f ? a[g] : 0.0f;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      z = __fmaf_rn(v[g].x, of_quad<0>(a[g]), z); z = __fmaf_rn(v[g].y, of_quad<1>(a[g]), z);
      z = __fmaf_rn(v[g].z, of_quad<2>(a[g]), z); z = __fmaf_rn(v[g].w, of_quad<3>(a[g]), z);
    }
  };
  int j = 0;
  for (; j + 16 <= h; j += 16) fours(j, std::integral_constant<int, 4>());
  if (j + 8 <= h) { fours(j, std::integral_constant<int, 2>()); j += 8; }
  if (j < h) fours(j, std::integral_constant<int, 1>());
  return z;
}

// The same for wide classifiers, by a whole workgroup of NT threads: a lane per candidate would wait for five wide LDS
// reads per four units, 256 units one after the other (6.5 us); here every thread forms hidden activations of
// one candidate, NT / K units (or groups of four) at a time, and only the chain z = fma(w2_j, a_j, z) is left to the candidate's lane.
// Same operations in the same order.  P: LDS, the candidates' joint probabilities; act: scratch of act_bytes;
// entry behind a barrier that publishes P.  Returns z in lanes tid < K.
// What bounds it: the chain, a fused multiply-add a unit, as long as its operands are there.  Where the arrays start on 16 bytes
// (h a multiple of four), a candidate's activations lie side by side and are read four at a time, as the weights are, two reads ahead
// of their use (256 units and 32 candidates 3.4 us; 5.1 with a word at a time, waited for every eight units: a phase of four sequences of 20011
// with 64 rows 258.2 -> 238.6 us).
template <int NT>
__device__ __forceinline__ float mlp_logit_spread(int tid, LdsFloats w, int h, const float* P, float H, float d, int K, uint32_t k_inverse,
                                                  float* act, int act_bytes) {
  LdsFloats W1 = w; LdsFloats b1 = w + 3 * h; LdsFloats w2 = w + 4 * h;
  const int step = NT / K, first = (int)(((uint32_t)tid * k_inverse) >> 20), cand = tid - first * K;      // first = tid / K
  const float Pc = P[cand];
  float z = w[5 * h];
  if ((h & 3) == 0) {
    typedef float float4v __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const float4v* LdsFloat4s;
    const int fours = h >> 2, block = min(fours, act_bytes / (16 * K) - 1), stride = 4 * block + 4;       // (four words more: lanes on different banks)
    for (int g0 = 0; g0 < fours; g0 += block) {
      const int n = min(block, fours - g0);
      if (first < step) {
        for (int g = first; g < n; g += step) {
          const int j = 4 * (g0 + g);
          const float4v wa = *(LdsFloat4s)(W1 + 3 * j), wb = *(LdsFloat4s)(W1 + 3 * j + 4), wc = *(LdsFloat4s)(W1 + 3 * j + 8), bb = *(LdsFloat4s)(b1 + j);
          float4v a;
          a.x = __fmaf_rn(wa.x, Pc, bb.x); a.x = __fmaf_rn(wa.y, H, a.x); a.x = __fmaf_rn(wa.z, d, a.x); a.x = a.x > 0.0f ? a.x : 0.0f;
          a.y = __fmaf_rn(wa.w, Pc, bb.y); a.y = __fmaf_rn(wb.x, H, a.y); a.y = __fmaf_rn(wb.y, d, a.y); a.y = a.y > 0.0f ? a.y : 0.0f;
          a.z = __fmaf_rn(wb.z, Pc, bb.z); a.z = __fmaf_rn(wb.w, H, a.z); a.z = __fmaf_rn(wc.x, d, a.z); a.z = a.z > 0.0f ? a.z : 0.0f;
          a.w = __fmaf_rn(wc.y, Pc, bb.w); a.w = __fmaf_rn(wc.z, H, a.w); a.w = __fmaf_rn(wc.w, d, a.w); a.w = a.w > 0.0f ? a.w : 0.0f;
          *(float4v*)(act + cand * stride + 4 * g) = a;
        }
      }
      __syncthreads();
      if (tid < K) {
        const float4v* const av = (const float4v*)(act + tid * stride);
        const LdsFloat4s wv = (LdsFloat4s)(w2 + 4 * g0);
        float4v a[2], v[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) { const int g = min(k, n - 1); a[k] = av[g]; v[k] = wv[g]; }
        const auto four = [&](int k) {
          z = __fmaf_rn(v[k].x, a[k].x, z); z = __fmaf_rn(v[k].y, a[k].y, z); z = __fmaf_rn(v[k].z, a[k].z, z); z = __fmaf_rn(v[k].w, a[k].w, z);
        };
        for (int g = 0; g + 1 < n; g += 2) {
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            four(k);
            const int next = min(g + 2 + k, n - 1);
            a[k] = av[next]; v[k] = wv[next];
          }
        }
        if (n & 1) four(0);
      }
      __syncthreads();
    }
    return z;
  }
  const int block = min(h, act_bytes / (4 * K));             // units whose activations fit the scratch
  for (int j0 = 0; j0 < h; j0 += block) {
    const int n = min(block, h - j0);
    if (first < step) {
      for (int u = first; u < n; u += step) {
        const int j = j0 + u;
        float a = __fmaf_rn(W1[3 * j + 0], Pc, b1[j]);
        a = __fmaf_rn(W1[3 * j + 1], H, a);
        a = __fmaf_rn(W1[3 * j + 2], d, a);
        act[u * K + cand] = a > 0.0f ? a : 0.0f;
      }
    }
    __syncthreads();
    if (tid < K) {
#pragma unroll 8
      for (int u = 0; u < n; ++u) z = __fmaf_rn(w2[j0 + u], act[u * K + tid], z);
    }
    __syncthreads();
  }
  return z;
}

constexpr int SP_MAX_F = 64;
constexpr int C2T_MAX_BUDGET_DEV = 1024;                  // n_out limit of the reranking
constexpr int C2T_MAX_CANDIDATES_DEV = 2048;              // F*K limit of the per-sequence step

// What a workgroup that shares a row hands over besides its counts, its cell keys and its columns' maxima.
constexpr int COOP_MAX_WORKGROUPS = 256;                  // workgroups of such a launch: one per CU at most
constexpr int COOP_MAX_ROWS = COOP_MAX_WORKGROUPS / 2;
struct __attribute__((aligned(32))) CoopAcc {
  double s_tiny; int32_t n_tiny, n_masked; uint32_t mag_max, max_pattern;   // see OutsideAcc; max_pattern: packed maximum of the segment's bf16 patterns
};

struct ScoreParams {
  RowPartial* part; float* part_topv; int32_t* part_topi;    // [launched row][split] records and their top-K lists
  int nsplit, F, K, N, h, layer, D;
  int M;                                                     // 0: entropy over the whole row; M > 0: over the M largest logits
  int lds_bytes;                                             // dynamic LDS of the launch
  int w_lds_off;                                             // byte offset of the classifier's copy in dynamic LDS
  uint32_t k_inverse;                                        // ceil(2^20 / K): (i * k_inverse) >> 20 is i / K for i < 2048, K <= 64
  int spread_min;                                            // hidden units from which on the whole workgroup evaluates the classifier
  float z_beta;
  // Shared rows of the histogram path (coop > 1, then nsplit == 1): `coop` workgroups count one row's
  // segments and hand their counts over through memory; the last to arrive runs the row's epilogue.
  int coop;
  int coop_map_stride;                                       // keys per row in coop_map (a multiple of 8)
  uint32_t* coop_hist;                                       // [launched row][coop][HP_WORDS] counts of a segment
  uint16_t* coop_map;                                        // [launched row][coop_map_stride] cell keys of the whole row; behind all COOP_MAX_ROWS of
                                                             // them [launched row][coop][WAVE] uint32: the segments' columns
  CoopAcc* coop_acc;                                         // [launched row][coop]
};

// What a workgroup needs to find its row and to request its first logits: the layer kernels' first arguments, which the compiler has the dispatcher
// put into scalar registers ahead of the wavefront's first instruction (kernel argument preload; the build's flags say how many of them).  Loaded, they cost a first touch of the arguments, a dependent one and two divisions of some twenty instructions before the frontier size was even requested.
struct Division { uint32_t n, inverse; };                    // inverse: ceil(2^32 / n), 0 for n = 1
struct QuotientRemainder { uint32_t q, r; };
__device__ __forceinline__ QuotientRemainder divide(uint32_t x, const Division& d) {
  uint32_t q = d.inverse ? __umulhi(x, d.inverse) : x;       // at most one too many
  uint32_t r = x - q * d.n;
  if ((int32_t)r < 0) { q -= 1; r += d.n; }                  // (divisors and what is divided stay below 2^31)
  return QuotientRemainder{q, r};
}
// shape: rows launched per sequence, F << 8, 1 << 16: workgroup w takes the w-th live row (see dealt_row)
constexpr uint32_t SHAPE_COMPACT = 1u << 16;
#define C2T_START_LIST(X) X(const void* __restrict__, logits) X(const int32_t* __restrict__, nfs) X(int64_t, row_stride_bytes) X(int, V) X(int, cps) X(uint32_t, B) \
                          X(uint32_t, shape) X(uint32_t, per_row) X(uint32_t, inv_per_row) X(uint32_t, inv_rows) X(uint32_t, inv_B)
#define C2T_AS_PARAMETER(type, name) type name,
#define C2T_AS_TYPE(type, name) type,
#define C2T_AS_MEMBER(type, name) type name;
#define C2T_AS_ONE(type, name) + 1
struct StartArguments { C2T_START_LIST(C2T_AS_MEMBER) };
constexpr int START_BYTES = sizeof(StartArguments), START_ARGUMENTS = 0 C2T_START_LIST(C2T_AS_ONE);
static_assert(START_BYTES <= 14 * 4, "fourteen registers take preloaded arguments");
static_assert(START_BYTES % 8 == 0, "the pointers that follow lie right behind them");
#ifdef C2T_KERNARG_PRELOAD
static_assert(C2T_KERNARG_PRELOAD == START_ARGUMENTS, "the build's flags preload as many arguments as there are");
#endif

// The last two arguments of the layer kernels, at byte OFFSET of the argument segment, read again for the tail: the compiler loads what it
// can reach early and keeps it in scalar registers through the streaming loop, or, there being too few, in lanes of vector registers.
struct TailArguments { TreeState st; ScoreParams sp; };
template <int OFFSET>
__device__ __forceinline__ const TailArguments& tail_arguments() {
  static_assert(OFFSET % 8 == 0 && sizeof(TreeState) % 8 == 0, "both lie where the kernel's argument list has them");
  typedef const __attribute__((address_space(4))) char* Arguments;
  Arguments p = (Arguments)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const TailArguments*)(const __attribute__((address_space(4))) TailArguments*)(p + OFFSET);
}

// What one workgroup of the logits pass leaves in LDS for its (row, split): the record, the segment's
// top-K list (value desc, id asc) where it has been ranked, and what scoring the row needs besides.
struct RowResult {
  RowPartial part;
  double ZM, SM;      // the sums of Z and S restricted to the M largest logits (Eq. 2, second line); M > 0 only
  double Zr;          // sum of e^(x - R) over the row, R = part.ref
  float H;            // entropy of the row
  uint32_t bad;       // no candidate comes from this row
  struct { float P; int32_t node, n_nodes, hidx; float s; } parent;   // of the row's frontier node, and nodes of the sequence's tree before this layer; hidx, s: rerank contexts only
  float topv[64];
  int32_t topi[64];
};

// sum over groups of 2^tshift neighbouring lanes (tshift <= 4, uniform), in each of them
__device__ __forceinline__ int sum_of_lanes(int tshift, int v) {
  if (tshift >= 1) v += (int)dpp_u32<C2T_DPP_QUAD_XOR1, 0xf>(0u, (uint32_t)v);
  if (tshift >= 2) v += (int)dpp_u32<C2T_DPP_QUAD_XOR2, 0xf>(0u, (uint32_t)v);
  if (tshift >= 3) v += (int)dpp_u32<C2T_DPP_ROW_HALF_MIRROR, 0xf>(0u, (uint32_t)v);
  if (tshift >= 4) v += (int)dpp_u32<C2T_DPP_ROW_MIRROR, 0xf>(0u, (uint32_t)v);
  return v;
}

// LDS of the selection of a segment's (or a row's) K largest logits: the element list ((value, id), 8 bytes an
// entry; the histogram path's own lies behind its counts, generic_segment's, the fp32 path's and that of merged rows at the start of
// the dynamic LDS) and the number of cells a launch may list: min(SEL_CELL_CAP, NT / CPC, list entries / elements per cell), which the
// host keeps >= 2K - 1.
constexpr int CPC = 4;                         // chunks per cell of the cell map: four neighbouring ones (histogram path), or four sweeps of a lane (generic_segment)
constexpr int SEL_CELL_CAP = 256;              // size of the candidate-cell list
constexpr int SEL_AUX_BYTES = 2048 + SEL_CELL_CAP * 4;   // behind the list: the lanes' maxima and the cells of generic_segment
struct SelectLds {
  unsigned char* list;
  unsigned char* aux;
  int list_cap;       // entries
  int cell_cap;
  __device__ __forceinline__ float* values() const { return (float*)list; }
  __device__ __forceinline__ int32_t* ids() const { return (int32_t*)(list + (size_t)list_cap * 4); }
};
template <int NT, int EPC>
__device__ __forceinline__ SelectLds make_select_lds(unsigned char* base, int bytes) {
  SelectLds s;
  s.list = base; s.list_cap = (bytes - SEL_AUX_BYTES) / 8 & ~3; s.aux = base + bytes - SEL_AUX_BYTES;     // (values and ids on 16 bytes)
  s.cell_cap = min(min(SEL_CELL_CAP, NT / CPC), s.list_cap / (CPC * EPC));
  return s;
}

// ---- ranking of the element list by (logit desc, id asc), exactly; the best K go to topv, topi.  By every wavefront but the last, which
// forms the row's entropy meanwhile: T lanes per element (four at least), each compares it with four entries per LDS read, of every
// T-th group of four; the partial ranks are summed over the T lanes.  Equal logits are told apart by id where a count shows them, four a read as
// well (one at a time, a layer of four rows of 20011 whose list holds 160 equal logits took 21.8 us, 17.8 so).  T is a constant in each of the three forms, and of the
// usual list (28 entries at most) every loop is one step: with T from the length, here and in the sequence step (32 listed at most there), phases of one sequence of 32000 took 1.015 times
// as long, of 128256 1.014, of 32 sequences reranked 1.020, of 64 of 128256 1.007.
template <int NT>
__device__ __forceinline__ void rank_list(int tid, int K, const SelectLds& sel, int n_el, float* topv, int32_t* topi) {
  constexpr int nt = NT - WAVE;
  const float* el_v = sel.values(); const int32_t* el_i = sel.ids();
  if (tid >= nt) return;                                     // a whole wavefront
  const auto rank = [&](auto shift) {
    constexpr int tshift = decltype(shift)::value, T = 1 << tshift;
    constexpr bool SHORT = tshift == 4;                        // the usual list: all loops are one step
    const int sub = tid & (T - 1);
#pragma unroll 1
    for (int e0 = 0; e0 < n_el; e0 += nt >> tshift) {
      const int e = e0 + (tid >> tshift);
      const bool mine = e < n_el;
      int rank = 0, id = 0; float v = 0.f;                     // rank: greater ones; equal ones (itself among them) in the upper half
      if (mine) {
        v = el_v[e]; id = el_i[e];
#pragma unroll 2
        for (int o = sub * 4; o < n_el; o += T * 4) {          // (values past the last, three at most, are read and not counted)
          const float4 q = *(const float4*)(el_v + o);
          const int past = max(o + 4 - n_el, 0);               // of the group's four
          const uint32_t gt = (q.x > v ? 1u : 0u) | (q.y > v ? 2u : 0u) | (q.z > v ? 4u : 0u) | (q.w > v ? 8u : 0u);
          const uint32_t eq = (q.x == v ? 1u : 0u) | (q.y == v ? 2u : 0u) | (q.z == v ? 4u : 0u) | (q.w == v ? 8u : 0u), in = 15u >> past;
          rank += __popc(gt & in) + (__popc(eq & in) << 16);
          if (SHORT) break;
        }
      }
      rank = sum_of_lanes(tshift, rank);
      const bool tied = mine && (rank >> 16) > 1 && (rank & 0xffff) < K;   // (the same in the element's T lanes)
      rank &= 0xffff;
      if (__builtin_amdgcn_ballot_w64(tied) != 0ull) {         // (uniform)
        int ahead = 0;
        if (tied) {
#pragma unroll 2
          for (int o = sub * 4; o < n_el; o += T * 4) {
            const float4 q = *(const float4*)(el_v + o);
            const int4 i = *(const int4*)(el_i + o);
            const uint32_t hit = (q.x == v && i.x < id ? 1u : 0u) | (q.y == v && i.y < id ? 2u : 0u) | (q.z == v && i.z < id ? 4u : 0u) | (q.w == v && i.w < id ? 8u : 0u);
            ahead += __popc(hit & (15u >> max(o + 4 - n_el, 0)));
          }
        }
        rank += sum_of_lanes(tshift, ahead);
      }
      if (mine && sub == 0 && rank < K) { topv[rank] = v; topi[rank] = id; }
      if (SHORT) break;
    }
  };
  if (n_el <= nt >> 4) rank(std::integral_constant<int, 4>());
  else if (n_el <= nt >> 3) rank(std::integral_constant<int, 3>());
  else rank(std::integral_constant<int, 2>());
}

// What the row's frontier node hands down, from global memory to rr.
// Straight to LDS, without registers meanwhile: requested by the last wavefront of an unsplit row on the histogram path ahead of the cells, and waited for behind the
// entropy.  (Requested where the entropy is formed, its round trip was the row's critical path.)
__device__ __forceinline__ void request_parent(const TreeState& s, int b, int64_t slot, RowResult& rr) {
  const int lane = lane_id();
  const void* from = s.fr_P + slot;
  if (lane == 1) from = s.fr_node + slot;
  if (lane == 2) from = s.n_nodes + b;
  if (lane == 3) from = s.fr_hidx + slot;
  if (lane == 4) from = s.fr_s + slot;
  if (lane < (s.h_tok ? 5 : 3))
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from, (__attribute__((address_space(3))) void*)&rr.parent, 4, 0, 0);
}
// The same where nothing is there to hide it, beside the entropy.
struct ParentStage { float P, s; int32_t hidx, node, n_nodes; };
__device__ __forceinline__ ParentStage load_parent(const TreeState& s, int b, int64_t slot) {
  ParentStage p{s.fr_P[slot], INFINITY, -1, s.fr_node[slot], s.n_nodes[b]};
  if (s.h_tok) { p.hidx = s.fr_hidx[slot]; p.s = s.fr_s[slot]; }
  return p;
}
__device__ __forceinline__ void store_parent(const ParentStage& p, RowResult& rr) {
  if (lane_id() == 0) { rr.parent.P = p.P; rr.parent.s = p.s; rr.parent.hidx = p.hidx; rr.parent.node = p.node; rr.parent.n_nodes = p.n_nodes; }
}

// ---- row level: entropy (Eq. 2) from the row's sums; by one wavefront.
// Re-references the sums from the offset a to the row maximum R: p_j = e^(x_j - R) / Zr, H = -sum p ln p = ln Zr - Sr / Zr.
// M: 0, or the number of logits that the sums ZM, SM in rr are restricted to; sc: e^(a - R)
__device__ __forceinline__ void row_entropy(int M, double R, double sc, double Z, double S, uint32_t flags, RowResult& rr) {
  const bool bad = (flags & 1u) != 0 || !(Z > 0.0) || !(R > -INFINITY) || !(R < INFINITY);
  const double Zr = Z * sc, Sr = S * sc;
  // Eq. 2, second line: -sum over the M most probable tokens of p ln p, p from the full softmax:
  // (ln Zr * ZMr - SMr) / Zr with the sums restricted to those tokens
  const float H = bad ? 0.f : M > 0 ? (float)((log(Zr) * (rr.ZM * sc) - rr.SM * sc) / Zr) : (float)(log(Zr) - Sr / Zr);
  if (lane_id() == 0) { rr.Zr = Zr; rr.H = H; rr.bad = bad ? 1u : 0u; }
}

__device__ __forceinline__ void row_entropy(int M, const RowPartial& r, RowResult& rr) {
  row_entropy(M, r.ref, r.a == r.ref ? 1.0 : exp(r.a - r.ref), r.Z, r.S, r.flags, rr);
}

struct Candidate { float z, P, H; int32_t tok; uint32_t info; };   // candidate t of a lone row, in lane t of the first wavefront; info: the row's flags

// ---- row level: generation and joint probability (Eq. 1) and classifier logit (Eq. 3) of the row's n candidates, from
// the complete row result in `rr`; one lane of the first wavefront per candidate, or four where there are so many (a wavefront issues the classifier's
// chain once for all of them).
// `w`: the classifier parameters in global memory, read-only for the whole kernel: every lane
// reads the same addresses, so the loads are scalar and touch neither LDS nor the vector memory path.
template <int NT>
__device__ __forceinline__ Candidate score_row(int tid, const TreeState& s, const ScoreParams& sp, int b, int f, bool lone, RowResult& rr, int n,
                                          const float* __restrict__ w, const float* w_lds, unsigned char* lds) {
  const int K = sp.K, FK = sp.F * K;
  const float H = rr.H;
  const bool spread = w_lds && sp.h >= sp.spread_min;        // (uniform)
  const bool quads = !spread && w_lds && K <= WAVE / 4 && (sp.h & 3) == 0;       // (uniform) four lanes a candidate
  const int cand = quads ? tid >> 2 : tid;
  float z = -INFINITY, p32 = 0.f, P32 = 0.f; int tok = -1;
  const bool mine = !rr.bad && cand < n;                     // n <= K
  if (mine) {
    tok = rr.topi[cand];
    p32 = (float)(exp((double)rr.topv[cand] - rr.part.ref) / rr.Zr);
    P32 = rr.parent.P * p32;
  }
  if (spread) {
    if (tid < K) rr.topv[tid] = P32;                         // each lane overwrites the logit it has just read
    __syncthreads();
    z = mlp_logit_spread<NT>(tid, (LdsFloats)w_lds, sp.h, rr.topv, H, (float)sp.layer, K, sp.k_inverse, (float*)lds, sp.lds_bytes);
    if (!mine) z = -INFINITY;
  }
  const uint32_t info = (uniform((int)rr.bad) ? 1u : 0u) | (rr.part.flags & 2u);
  if (tid >= (quads ? WAVE : K)) return Candidate{-INFINITY, 0.f, 0.f, -1, 0u};
  if (mine && !spread) {
    z = quads ? mlp_logit_quads((LdsFloats)w_lds, sp.h, P32, H, (float)sp.layer)
        : w_lds ? mlp_logit_lds((LdsFloats)w_lds, sp.h, P32, H, (float)sp.layer) : mlp_logit(w, sp.h, P32, H, (float)sp.layer);
  }
  const int64_t row = (int64_t)b * FK + (int64_t)f * K;     // uniform; the lane's offset stays 32 bits wide
  if (!quads || ((tid & 3) == 0 && cand < K)) {
    st_dev(s.c_tok + row + cand, tok); st_dev(s.c_p + row + cand, p32); st_dev(s.c_P + row + cand, P32);
    st_dev(s.c_H + row + cand, H); st_dev(s.c_z + row + cand, z);
    if (tid == 0) st_dev(s.row_info + (int64_t)b * sp.F + f, info);
    if (s.h_tok) {                                           // keep the candidate for the reranking
      const int64_t h = ((int64_t)b * sp.D + sp.layer) * FK + (int64_t)f * K;
      s.h_tok[h + cand] = tok; s.h_par[h + cand] = rr.parent.hidx;
      s.h_P[h + cand] = P32; s.h_H[h + cand] = H; s.h_z[h + cand] = z;
      s.h_s[h + cand] = fminf(rr.parent.s, z);
    }
  }
  if (quads && lone) {                                       // (uniform) for the caller a lane a candidate again
    const int from = tid * 16;
    z = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)__float_as_uint(z)));
    P32 = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)__float_as_uint(P32)));
    tok = __builtin_amdgcn_ds_bpermute(from, tok);
    if (tid >= K) return Candidate{-INFINITY, 0.f, 0.f, -1, 0u};
  }
  return Candidate{z, P32, H, tok, info};
}

// ---- row level, splits > 1, by the workgroup that delivered the row's last split.
// Everything the merge reads is requested before anything is waited for: one memory round trip.  One wavefront
// combines the split records in fp64; the others stage the lists in the element list, where an unused
// slot of a split's list lies below every entry in the order (value desc, id asc), -inf entries included.
constexpr int32_t NO_ID = 0x7fffffff;
struct RowSums { double R, Z, S; uint32_t flags; int n_valid; };       // uniform over the wavefront
__device__ __forceinline__ RowSums merge_records(const RowPartial* rp, int nsplit) {
  const int lane = lane_id();
  RowSums m; m.n_valid = 0;
  float Rf = -INFINITY; uint32_t fl = 0; double Z = 0.0, S = 0.0;       // ref holds a logit: exact as a float
  if (nsplit <= WAVE) {
    RowPartial pq = empty_partial();
    if (lane < nsplit) pq = ld_dev(rp + lane);
    Rf = wave_max(lane < nsplit ? (float)pq.ref : -INFINITY);
    fl = wave_reduce_u32(pq.flags, 0u, [](uint32_t x, uint32_t y) { return x | y; });
    m.n_valid = wave_sum_i(pq.n_top);
    const double R = (double)Rf;
    if (pq.Z > 0.0 && pq.ref > -INFINITY) {
      const double da = pq.a - R, dl = pq.ref - R;           // re-reference to the row maximum R; dl <= 0
      const double sc = da == 0.0 ? 1.0 : exp(da);
      Z = pq.Z * sc; S = (pq.S + dl * pq.Z) * sc;
    }
  } else {
    int nv = 0;
    for (int q = lane; q < nsplit; q += WAVE) { Rf = fmaxf(Rf, (float)ld_dev(&rp[q].ref)); fl |= ld_dev(&rp[q].flags); nv += ld_dev(&rp[q].n_top); }
    Rf = wave_max(Rf);
    fl = wave_reduce_u32(fl, 0u, [](uint32_t x, uint32_t y) { return x | y; });
    m.n_valid = wave_sum_i(nv);
    const double R = (double)Rf;
    for (int q = lane; q < nsplit; q += WAVE) {
      const RowPartial pq = ld_dev(rp + q);
      if (pq.Z > 0.0 && pq.ref > -INFINITY) {
        const double da = pq.a - R, dl = pq.ref - R;
        const double sc = da == 0.0 ? 1.0 : exp(da);
        Z += pq.Z * sc; S += (pq.S + dl * pq.Z) * sc;
      }
    }
  }
  m.R = (double)Rf; m.flags = fl; m.Z = wave_sum(Z); m.S = wave_sum(S);
  return m;
}
__device__ __forceinline__ void stage_lists(int tid, const ScoreParams& sp, int64_t row_launched, const SelectLds& sel) {
  const int nsplit = sp.nsplit, K = sp.K, per_row = nsplit * K, nt = blockDim.x;
  const RowPartial* rp = sp.part + row_launched * nsplit;
  const float* tv = sp.part_topv + row_launched * per_row;
  const int32_t* ti = sp.part_topi + row_launched * per_row;
  for (int ent = tid; ent < per_row; ent += nt) {
    const int n_top = ld_dev(&rp[ent / K].n_top);
    const float v = ld_dev(tv + ent); const int32_t id = ld_dev(ti + ent);
    const bool ok = ent % K < n_top;
    sel.values()[ent] = ok ? v : -INFINITY;
    sel.ids()[ent] = ok ? id : NO_ID;
  }
}
// Lists that exceed the element list (very many splits): ranked from global memory, the best K to rr.topv, rr.topi.
__device__ __forceinline__ void rank_lists_from_memory(int tid, const ScoreParams& sp, int64_t row_launched, RowResult& rr) {
  const int nsplit = sp.nsplit, K = sp.K, per_row = nsplit * K, nt = blockDim.x;
  const RowPartial* rp = sp.part + row_launched * nsplit;
  const float* tv = sp.part_topv + row_launched * per_row;
  const int32_t* ti = sp.part_topi + row_launched * per_row;
  for (int ent = tid; ent < per_row; ent += nt) {
    const int q = ent / K, e = ent % K;
    if (e >= ld_dev(&rp[q].n_top)) continue;
    const float v = ld_dev(tv + ent); const int vi = ld_dev(ti + ent);
    int ahead = 0;
    for (int q2 = 0; q2 < nsplit; ++q2) {
      const int n2 = ld_dev(&rp[q2].n_top);
      for (int e2 = 0; e2 < n2; ++e2) {
        const float v2 = ld_dev(tv + q2 * K + e2);
        ahead += (v2 > v) || (v2 == v && ld_dev(ti + q2 * K + e2) < vi);
      }
    }
    if (ahead < K) { rr.topv[ahead] = v; rr.topi[ahead] = vi; }
  }
}

// ---- sequence level: both prunings of Sec. 4.2 with the node budget, tree append, next frontier.
// Run by one whole workgroup once every row of the sequence has been scored.
//
// What bounds it: latency; a handful of dependent steps on at most 2048 candidates.  Everything the step reads is requested
// at once.  Only the n_keep best survivors of the first pruning matter: of 64 (or 128) groups of candidates, one
// per lane, the n_keep-th largest group maximum is a lower bound of the n_keep-th largest z, found by every wavefront from sorted rows of
// 16 (n_keep <= 16; from ballots, rounds of scalar instructions, 32 sequences of 10 x 10 candidates with every one a survivor took 113.7 us a phase, 111.0
// so, 16 of 16 x 16 173.2 and 172.4) or from ballots; what reaches it (two dozen candidates where 16 are kept) is listed in LDS and ranked exactly.  The
// ranking gives each listed candidate to T = 2^tshift lanes, which split the list between them, two keys per LDS read.
// Lists that stay long, layers of equal z above all, are first cut by a radix select on the whole keys; so are, without a
// bound, more than 64 survivors of more than 512 candidates (several a thread), whose bound is slower to find and lets more
// pass.  Layers with bound / radix select: 32 sequences of 32 x 32 candidates 32.1 / 30.6 us, of 32 x 64 44.5 / 42.8, 4 sequences of
// 64 x 32 21.0 / 19.1.  Up to 512, one a thread, the bound is the faster: for one sequence of 16 x 16 1.4 us against 1.9 (first pruning
// and preselection).
#ifndef C2T_PRUNE_RANK_MAX
#define C2T_PRUNE_RANK_MAX 128
#endif
#ifndef C2T_PRUNE_DIRECT_MAX
#define C2T_PRUNE_DIRECT_MAX 64
#endif
#ifndef C2T_PRUNE_UNDECIDED_MAX
#define C2T_PRUNE_UNDECIDED_MAX 64
#endif
constexpr int PRUNE_HIST_WORDS = 2048;        // 4096 bins, two 16-bit counters per word
constexpr int PRUNE_DIRECT_MAX = C2T_PRUNE_DIRECT_MAX;         // up to so many survivors are ranked without looking for a bound (100 of them: 1.6 us, with it 1.1)
constexpr int PRUNE_RANK_MAX = C2T_PRUNE_RANK_MAX;             // lists that are longer with it are cut by the radix select
constexpr int PRUNE_UNDECIDED_MAX = C2T_PRUNE_UNDECIDED_MAX; // the select stops once at most so many survivors share the selected digits

__host__ __device__ inline size_t prune_list_bytes(int FK) { return ((size_t)3 * ((FK + 31) & ~31) + PRUNE_HIST_WORDS) * 4; }

// A threshold that at least n of the NV * 64 maxima reach (0 if fewer than n are not 0), as high as it takes for at most
// `enough` of them to reach it, or their n-th largest.  Two bits a step from the top, ballots, uniform result.
template <int NV>
__device__ __forceinline__ uint32_t bound_from_maxima(const uint32_t (&m)[NV], int n, int enough) {
  // the upper bits that all maxima share need no round, nor does anything where they are all equal
  const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)m[0]);
  uint32_t differ = 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) differ |= m[v] ^ first;
  differ = wave_reduce_u32(differ, 0u, [](uint32_t x, uint32_t y) { return x | y; });
  if (differ == 0u) return first;
  const int top = (31 - __builtin_clz(differ)) & ~1;
  uint32_t prefix = top == 30 ? 0u : first & ~((4u << top) - 1u);
  for (int shift = top; shift >= 0; shift -= 2) {
    int cnt[3] = {0, 0, 0};                                  // how many reach prefix + 1, 2, 3 steps
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int v = 0; v < NV; ++v) cnt[q] += __popcll(__ballot(m[v] >= (prefix | ((uint32_t)(q + 1) << shift))));
    const int q = (cnt[0] >= n) + (cnt[1] >= n) + (cnt[2] >= n);
    prefix |= (uint32_t)q << shift;
    if (q && (q == 3 ? cnt[2] : q == 2 ? cnt[1] : cnt[0]) <= enough) break;
  }
  return prefix;
}

template <int NT>
struct PruneShared {
  int32_t n_list, n_red, flags_or, sel_bin, sel_above, sel_count;
  int32_t scan_w[NT / WAVE], surv_w[NT / WAVE];
  int32_t old_node[SP_MAX_F];
  float old_s[SP_MAX_F];
  uint32_t kept[C2T_MAX_CANDIDATES_DEV / 32];              // bit i: candidate i is appended to the tree
};

// Dynamic LDS of prune_sequence: its lists, then PruneShared (2 KB of static LDS would cost launches with K = 64, whose element
// list takes 32 KB, the fourth workgroup of a CU: 1024 rows of 32000 44 us instead of 33; another 1 KB of it launches with more than
// 1900 candidates: 2048 rows of 32000 with 64 x 31 candidates 42 us instead of 37).
template <int NT>
__host__ __device__ inline size_t score_lds_bytes(int FK) {
  static_assert(sizeof(PruneShared<NT>) <= 1024, "with 64 x 32 candidates it decides over the fourth workgroup of a CU");
  return prune_list_bytes(FK) + sizeof(PruneShared<NT>);
}

// PER: candidates per thread; F * K <= PER * NT.
template <int NT, int PER>
__device__ __forceinline__ void prune_sequence(int tid, const TreeState& s, const ScoreParams& sp, int b, int nf, unsigned char* lds, PruneShared<NT>& ps) {
  constexpr int NW = NT / WAVE;
  constexpr bool BY_DIGITS = PER > 1;                        // long lists are cut by the radix select at once
  const int F = sp.F, K = sp.K, N = sp.N, layer = sp.layer;
  const float z_beta = sp.z_beta;
  const int FK = F * K, FKp = (FK + 31) & ~31;
  // survivors: one 64-bit key each, (order-preserving key of z) << 32 | ~token, so that a greater key comes first in
  // the order (z desc, token asc); and the candidate index, which breaks the remaining ties.  Equal z is common, not
  // rare: deep in a tree P is too small to move the classifier's fp32 sum, and the K children of a row, which
  // share H and d, all get the same z.
  uint64_t* skey = (uint64_t*)lds;
  int32_t* sidx = (int32_t*)(skey + FKp);
  uint32_t* hist = (uint32_t*)(sidx + FKp);
  // in the histogram's place, which comes later, if at all: the lanes' maxima, and P and H of the first entries, as listed
  uint32_t* lane_max = hist;                                 // [NW][WAVE]
  float* list_P = (float*)(hist + NW * WAVE); float* list_H = list_P + PRUNE_RANK_MAX;
  static_assert(NW * WAVE + 2 * PRUNE_RANK_MAX <= PRUNE_HIST_WORDS, "they fit there");

  const int lane = tid & (WAVE - 1), wid = tid >> 6;
  const int64_t cb = (int64_t)b * FK, fb = (int64_t)b * F;   // uniform bases: the lanes' offsets stay 32 bits wide
  // the candidates of all F*K slots are requested up front: one memory round trip
  float my_z[PER], my_P[PER], my_H[PER]; int32_t my_tok[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = tid + k * NT;
    my_z[k] = my_P[k] = my_H[k] = 0.f; my_tok[k] = -1;
    if (i < FK) {
      my_z[k] = ld_dev(s.c_z + cb + i); my_tok[k] = ld_dev(s.c_tok + cb + i);
      if (!BY_DIGITS) { my_P[k] = ld_dev(s.c_P + cb + i); my_H[k] = ld_dev(s.c_H + cb + i); }
    }
  }
  uint32_t info = 0u;
  if (tid < F) info = ld_dev(s.row_info + fb + tid);
  const int nn = s.n_nodes[b];
  if (tid < nf) {                                            // the old frontier is read here, for good: the new one is stored over it below
    ps.old_node[tid] = s.fr_node[fb + tid];
    ps.old_s[tid] = s.h_tok ? s.fr_s[fb + tid] : INFINITY;
  }
  if (tid < (FK + 31) / 32) ps.kept[tid] = 0u;
  if (tid == 0) { ps.n_list = 0; ps.n_red = 0; ps.flags_or = 0; ps.sel_bin = 0; }

  // ---- first pruning: z > logit(beta) ----
  const int ncand = nf * K;
  uint32_t zk[PER]; int cnt = 0;                             // key of z, 0: not a survivor
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = tid + k * NT;
    zk[k] = (i < ncand && my_tok[k] >= 0 && my_z[k] > z_beta) ? sortable_key(my_z[k]) : 0u;
    cnt += __popcll(__ballot(zk[k] != 0u));
  }
  C2T_PT(PT_PRUNE_LOADED);
  // Groups for the bound below: a lane's candidate with those of other lanes in the other wavefronts.  Rows list their
  // children from the most probable down, and where K divides 64 a lane holds the same rank of every row: maxima by lane alone
  // would be maxima by rank, and half of them, all low ranks, a bound that most candidates reach.
  static_assert(NW <= 16, "lanes 0-3, 16-19, 32-35, 48-51 of the wavefronts");
  if (BY_DIGITS) { for (int i = tid; i < PRUNE_HIST_WORDS; i += NT) hist[i] = 0u; }
  else lane_max[wid * WAVE + (lane ^ ((wid & 3) | ((wid >> 2) << 4)))] = zk[0];
  if (lane == 0) ps.surv_w[wid] = cnt;
  __syncthreads();
  if (tid < nf && info) atomicOr(&ps.flags_or, (int)info);
  C2T_PT(PT_PRUNE_FIRST);

  // ---- second pruning + budget: rank survivors by (z desc, token asc, slot asc) ----
  int n_surv = 0;
#pragma unroll
  for (int v = 0; v < NW; ++v) n_surv += ps.surv_w[v];
  n_surv = uniform(n_surv);
  const int n_keep = max(0, min(min(F, N - uniform(nn)), n_surv));
  uint32_t bound = 1u;                                       // every survivor
  const bool to_digits = BY_DIGITS && n_surv > PRUNE_DIRECT_MAX;
  if (!BY_DIGITS && n_keep > 0 && n_surv > PRUNE_DIRECT_MAX) {
    uint32_t m[2] = {0u, 0u};
#pragma unroll
    for (int v = 0; v < NW; ++v) m[v & 1] = max(m[v & 1], lane_max[v * WAVE + lane]);
    if (n_keep <= 16) bound = nth_largest16(max(m[0], m[1]), n_keep);
    else if (n_keep <= 32) { const uint32_t m1[1] = {max(m[0], m[1])}; bound = bound_from_maxima<1>(m1, n_keep, n_keep + 24); }
    else bound = bound_from_maxima<2>(m, n_keep, n_keep + 24);
    bound = max(bound, 1u);
  }
  if (n_keep > 0) {
    uint64_t hit[PER]; int tot = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) { hit[k] = __ballot(zk[k] >= bound); tot += __popcll(hit[k]); }
    int at = 0;
    if (bound == 1u) {                                       // every survivor: the places follow from the wavefronts' counts
#pragma unroll
      for (int v = 0; v < NW; ++v) at += v < wid ? ps.surv_w[v] : 0;
      if (tid == 0) ps.n_list = n_surv;
    } else if (tot) {                                        // one addition a wave gives the places
      if (lane == 0) at = atomicAdd(&ps.n_list, tot);
      at = __builtin_amdgcn_readfirstlane(at);
    }
    if (tot) {
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        if (zk[k] >= bound) {
          const int u = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hit[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hit[k], 0u));
          skey[u] = ((uint64_t)zk[k] << 32) | (uint32_t)~my_tok[k]; sidx[u] = tid + k * NT;
          if (!BY_DIGITS && u < PRUNE_RANK_MAX) { list_P[u] = my_P[k]; list_H[u] = my_H[k]; }
          if (to_digits) { const uint32_t bin = zk[k] >> 20; atomicAdd(&hist[bin >> 1], (bin & 1u) ? 0x10000u : 1u); }
        }
        at += __popcll(hit[k]);
      }
    }
  }
  __syncthreads();
  // Counts are told to be uniform: the loop that finds the entries' lanes (tshift) is scalar then.  Masked, with more than 256 entries no lane ran it, and
  // the build for four workgroups a CU, as compiled, copied the thread index behind it before the lanes were switched on again: nothing was kept.
  int ns = __builtin_amdgcn_readfirstlane(ps.n_list);
  const bool listed_order = !BY_DIGITS && ns <= PRUNE_RANK_MAX;       // list_P, list_H hold the entries' P and H
  if (n_keep > 0 && (BY_DIGITS ? to_digits : !listed_order)) {
    // Radix select on the 64-bit keys, twelve bits a level, from the top: the histogram of the level's digit over
    // the survivors that are still undecided (those whose higher digits equal the digits selected so far; at the
    // first level all of them) gives the digit at which the running count from
    // the top reaches what is still needed; survivors below it are dropped.  Layers of equal z go on into the
    // token bits instead of ranking hundreds of tied survivors against each other.
    if (!BY_DIGITS) {
      for (int i = tid; i < PRUNE_HIST_WORDS; i += NT) hist[i] = 0u;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int u = tid + k * NT;
        if (u < ns) { const uint32_t bin = (uint32_t)(skey[u] >> 52); atomicAdd(&hist[bin >> 1], (bin & 1u) ? 0x10000u : 1u); }
      }
      __syncthreads();
    }
    int need = n_keep, shift = 52;                           // (uniform) still to be taken from the undecided; the level's digit is key >> shift
    uint64_t prefix = 0ull;                                  // the digits selected so far: the undecided have key >> (shift + 12) == prefix
    for (;;) {
      // thread t owns words 2047-4t .. 2047-4t-3 (bins descending)
      constexpr int WPT = PRUNE_HIST_WORDS / NT;
      uint32_t w[WPT]; int c = 0;
#pragma unroll
      for (int j = 0; j < WPT; ++j) { w[j] = hist[PRUNE_HIST_WORDS - 1 - (tid * WPT + j)]; c += (int)(w[j] & 0xffffu) + (int)(w[j] >> 16); }
      const int incl = wave_scan_incl(c);
      if (lane == WAVE - 1) ps.scan_w[wid] = incl;
      __syncthreads();
      int above = incl - c;
#pragma unroll
      for (int v = 0; v < NW; ++v) if (v < wid) above += ps.scan_w[v];
      if (above < need && above + c >= need) {               // exactly one thread
        int run = above;
#pragma unroll
        for (int j = 0; j < WPT; ++j) {
          const int word = PRUNE_HIST_WORDS - 1 - (tid * WPT + j);
          const int hi = (int)(w[j] >> 16), lo = (int)(w[j] & 0xffffu);
          if (run < need && run + hi >= need) { ps.sel_bin = 2 * word + 1; ps.sel_above = run; ps.sel_count = hi; }
          run += hi;
          if (run < need && run + lo >= need) { ps.sel_bin = 2 * word; ps.sel_above = run; ps.sel_count = lo; }
          run += lo;
        }
      }
      if (tid == 0) ps.n_red = 0;
      __syncthreads();
      // cut the list down, in place: read, barrier, write
      const uint64_t cut = (prefix << 12) | (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(ps.sel_bin);
      const int undecided = __builtin_amdgcn_readfirstlane(ps.sel_count);
      need -= __builtin_amdgcn_readfirstlane(ps.sel_above);
      uint64_t rk[PER]; int32_t ri[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int u = tid + k * NT;
        rk[k] = 0ull; ri[k] = -1;
        if (u < ns) { rk[k] = skey[u]; ri[k] = sidx[u]; }
      }
      __syncthreads();
      // one addition a wavefront (a place a survivor by append_place: phases of four sequences, 2048 candidates of equal confidence a layer, 176.6 us, 173.7 so)
      int n_mine = 0;
#pragma unroll
      for (int k = 0; k < PER; ++k) n_mine += ri[k] >= 0 && (rk[k] >> shift) >= cut ? 1 : 0;
      int to = append_places(n_mine, &ps.n_red);
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        if (ri[k] >= 0 && (rk[k] >> shift) >= cut) { skey[to] = rk[k]; sidx[to] = ri[k]; ++to; }
      }
      for (int i = tid; i < PRUNE_HIST_WORDS; i += NT) hist[i] = 0u;   // for the next level, if there is one
      __syncthreads();
      ns = __builtin_amdgcn_readfirstlane(ps.n_red);
      if (undecided <= PRUNE_UNDECIDED_MAX || shift < 12) break;      // (uniform) few enough to rank; or the last whole digit done
      prefix = cut; shift -= 12;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int u = tid + k * NT;
        if (u < ns) {
          const uint64_t key = skey[u];
          if ((key >> (shift + 12)) == prefix) {
            const uint32_t digit = (uint32_t)(key >> shift) & 0xfffu;
            atomicAdd(&hist[digit >> 1], (digit & 1u) ? 0x10000u : 1u);
          }
        }
      }
      __syncthreads();
    }
  }
  C2T_PT(PT_PRUNE_PRESELECTED);
  if (n_keep > 0) {
    // tshift: see rank_list
    const auto rank_listed = [&](auto shift) {
      constexpr bool SHORT = !std::is_same<decltype(shift), int>::value;
      const int tshift = shift, T = 1 << tshift, sub = tid & (T - 1), ustride = NT >> tshift;
#pragma unroll 1
      for (int u0 = 0; u0 < ns; u0 += ustride) {               // uniform trip count: every lane meets in the DPP sums
        const int u = u0 + (tid >> tshift);
        const bool mine = u < ns;
        const uint64_t key = mine ? skey[u] : 0ull;
        const int i = mine ? sidx[u] : 0;
        const float z = key_to_float((uint32_t)(key >> 32));
        const int tok = (int)~(uint32_t)key;
        float P = 0.f, H = 0.f;
        if (mine && sub == 0) {
          if (listed_order) { P = list_P[u]; H = list_H[u]; }
          else { P = ld_dev(s.c_P + cb + i); H = ld_dev(s.c_H + cb + i); }
        }
        // rank = survivors with a greater key, and those with the same key (the same token under two parents, with
        // the same z: looked for only where a count shows them) and a lower candidate index; the survivor's T
        // lanes take two keys a step each.  (Ties by one lane alone: 7.5 us for 100 survivors of equal z whose rows share tokens.)
        int rank = 0;                                          // lower half: greater keys, upper half: equal ones (itself among them)
        if (mine) {
#pragma unroll 2
          for (int v = sub * 2; v < ns; v += T * 2) {
            const uint4 q = *(const uint4*)(skey + v);
            const uint64_t k0 = ((uint64_t)q.y << 32) | q.x, k1 = v + 1 < ns ? ((uint64_t)q.w << 32) | q.z : 0ull;
            rank += (k0 > key ? 1 : 0) + (k1 > key ? 1 : 0) + (k0 == key ? 0x10000 : 0) + (k1 == key ? 0x10000 : 0);
            if (SHORT) break;                                  // (T lanes of two keys are all there are)
          }
        }
        rank = sum_of_lanes(tshift, rank);
        const bool tied = mine && (rank >> 16) > 1;            // (the same in the entry's T lanes)
        rank &= 0xffff;
        if (__builtin_amdgcn_ballot_w64(tied) != 0ull) {       // (uniform)
          int ahead = 0;
          if (tied) {
#pragma unroll 4
            for (int v = sub; v < ns; v += T) ahead += (int)(skey[v] == key && sidx[v] < i);
          }
          rank += sum_of_lanes(tshift, ahead);
        }
        if (mine && sub == 0 && rank < n_keep) {
          const int f = (int)(((uint32_t)i * sp.k_inverse) >> 20);         // i / K
          const int64_t tb = (int64_t)b * N + nn;
          atomicOr(&ps.kept[i >> 5], 1u << (i & 31));
          s.t_tok[tb + rank] = tok; s.t_parent[tb + rank] = ps.old_node[f]; s.t_depth[tb + rank] = layer;
          s.t_P[tb + rank] = P; s.t_H[tb + rank] = H; s.t_z[tb + rank] = z;
          s.fr_tok[fb + rank] = tok; s.fr_pslot[fb + rank] = f; s.fr_node[fb + rank] = nn + rank; s.fr_P[fb + rank] = P;
          if (s.h_tok) { s.fr_hidx[fb + rank] = layer * FK + i; s.fr_s[fb + rank] = fminf(ps.old_s[f], z); }
        }
        if (SHORT) break;
      }
    };
    static_assert((NT >> 4) <= 2 << 4, "a short list is one step of two keys a lane");
    if (ns <= NT >> 4) {
      rank_listed(std::integral_constant<int, 4>());
    } else {
      int tshift = 0;
      while (tshift < 3 && (ns << (tshift + 1)) <= NT) ++tshift;
      rank_listed(tshift);
    }
  }
  __syncthreads();                                           // ps.kept is complete
  C2T_PT(PT_PRUNE_RANKED);
#pragma unroll
  for (int k = 0; k < PER; ++k) {                            // (slots of unused rows are unspecified)
    const int i = tid + k * NT;
    if (i < FK) s.c_kept[cb + i] = (int32_t)((ps.kept[i >> 5] >> (i & 31)) & 1u);
  }
  if (tid == 0) {
    if (s.h_tok) s.h_ncand[(int64_t)b * sp.D + layer] = ncand;
    s.n_nodes[b] = nn + n_keep;
    s.nf[(layer + 1) & 1][b] = n_keep;
    s.n_cand[b] = ncand;
    if (ps.flags_or) s.status[b] |= (uint32_t)ps.flags_or;
    if (n_keep) atomicAdd(&s.layer_rows[layer + 1], n_keep);
  }
}

// The same for a sequence with one frontier node (root layers, chains), whose at most 64 candidates the first wavefront of
// this workgroup has just scored, one a lane: ranked in that wavefront's registers, no barrier, nothing of them read back
// from memory.  What bounds it: issue in one wavefront, four instructions a
// candidate for the ranking.  1024 chains: 1.0 us where prune_sequence takes 3.0; root layers of one sequence with K = 32
// 14.1 -> 12.4 us, K = 64 (all survive) 16.1 -> 14.4.  (A walk over the survivors' ballot with three compares a
// survivor: 1.5 us slower at K = 64.)
template <int NT>
__device__ __forceinline__ void prune_lone_row(int tid, const TreeState& s, const ScoreParams& sp, int b, const RowResult& rr, const Candidate& c) {
  const int F = sp.F, K = sp.K, FK = F * K, layer = sp.layer;
  const int64_t cb = (int64_t)b * FK, fb = (int64_t)b * F;
  for (int i = tid < WAVE ? tid + NT : tid; i < FK; i += NT) s.c_kept[cb + i] = 0;
  if (tid >= WAVE) return;
  const bool surv = tid < K && c.tok >= 0 && c.z > sp.z_beta;
  // order (z desc, token asc), a row's tokens being distinct; 0: not a survivor
  const uint32_t zk = surv ? sortable_key(c.z) : 0u, tk = surv ? (uint32_t)~c.tok : 0u;
  const uint64_t key = ((uint64_t)zk << 32) | tk;
  const uint64_t survivors = __ballot(surv);
  const int nn = uniform(rr.parent.n_nodes), n_keep = max(0, min(min(F, sp.N - nn), __popcll(survivors)));
  int rank = 0;
  if (n_keep > 0) {
    for (int j0 = 0; j0 < K; j0 += 4) {                      // K <= 64: lanes K .. 63 hold 0
#pragma unroll
      for (int j = j0; j < j0 + 4; ++j) {
        const uint32_t zj = (uint32_t)__builtin_amdgcn_readlane((int)zk, j), tj = (uint32_t)__builtin_amdgcn_readlane((int)tk, j);
        rank += (((uint64_t)zj << 32) | tj) > key ? 1 : 0;
      }
    }
  }
  const bool kept = surv && rank < n_keep;
  if (kept) {
    const int64_t tb = (int64_t)b * sp.N + nn;
    s.t_tok[tb + rank] = c.tok; s.t_parent[tb + rank] = rr.parent.node; s.t_depth[tb + rank] = layer;
    s.t_P[tb + rank] = c.P; s.t_H[tb + rank] = c.H; s.t_z[tb + rank] = c.z;
    s.fr_tok[fb + rank] = c.tok; s.fr_pslot[fb + rank] = 0; s.fr_node[fb + rank] = nn + rank; s.fr_P[fb + rank] = c.P;
    if (s.h_tok) { s.fr_hidx[fb + rank] = layer * FK + tid; s.fr_s[fb + rank] = fminf(rr.parent.s, c.z); }
  }
  if (tid < FK) s.c_kept[cb + tid] = kept ? 1 : 0;
  if (tid == 0) {
    if (s.h_tok) s.h_ncand[(int64_t)b * sp.D + layer] = K;
    s.n_nodes[b] = nn + n_keep;
    s.nf[(layer + 1) & 1][b] = n_keep;
    s.n_cand[b] = K;
    if (c.info) s.status[b] |= c.info;
    if (n_keep) atomicAdd(&s.layer_rows[layer + 1], n_keep);
  }
}

// Thread 0 takes a ticket once its wave's device-coherent stores are complete: true for the
// workgroup that took the last of `expected` (it resets the counter for the next layer).  Every
// store the ticket publishes is issued by wave 0 (at most 64 candidates or list entries, lanes
// 0..63), whose own wait covers them; the other waves only meet at the barrier.
__device__ __forceinline__ bool last_arrival(int tid, int32_t* ticket, int expected) {
  __shared__ int32_t sh_last;
  if (tid < WAVE) {
    wait_vector_memory();
    if (tid == 0) {
      sh_last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == expected - 1;
      if (sh_last) st_dev(ticket, 0);
    }
  }
  __syncthreads();
  return uniform(sh_last) != 0;
}

// How a workgroup leaves its segment's largest logits: n_el elements in its element list, not ranked yet, or (n_el < 0)
// ranked in rr.topv, rr.topi with rr.part.n_top of them.  recorded: the last wavefront has completed rr.part, and the entropy of an unsplit row
struct SegmentTop { int n_el; bool recorded; };

// Tail of the logits pass for the workgroup that owned (sequence b, frontier slot f, split).  The workgroup
// that completes a row scores the row's candidates; the workgroup that completes a sequence's last row prunes
// and appends.  Both overlap with the other workgroups' streaming, so the whole layer is one launch.
// On entry a barrier lies behind the last write to the list and to rr, except that `record()`, called by the last
// wavefront while the others rank the list, completes rr.part (sums, flags; its lane 0 writes).
// list: the segment's element list; sel: the one that merged rows are ranked in.
// after_merge(rr): called by the whole workgroup that has merged a split row, before the row is scored
// (the entropy over the M largest logits of a split row is computed there, over the whole row).
template <int NT, typename Record, typename AfterMerge>
__device__ __forceinline__ void finish_layer(int tid, const TreeState& s, const ScoreParams& sp, int b, int f, int nf, int split,
                                             int64_t row_launched, RowResult& rr, SegmentTop top, const SelectLds& list, const SelectLds& sel, unsigned char* lds,
                                             const float* __restrict__ cls, const float* cls_lds, Record record, AfterMerge after_merge) {
  constexpr int NW = NT / WAVE;
  const int K = sp.K;
  const bool last_wave = (tid >> 6) == NW - 1;
  const int64_t slot = (int64_t)b * sp.F + f;
  if (last_wave) {
    if (top.recorded) {
      wait_vector_memory();                                  // request_parent
    } else {
      record();
      if (sp.nsplit == 1) {
        const ParentStage p = load_parent(s, b, slot);
        row_entropy(sp.M, rr.part, rr);
        store_parent(p, rr);
      }
    }
  }
  if (top.n_el >= 0) rank_list<NT>(tid, K, list, top.n_el, rr.topv, rr.topi);
  __syncthreads();                                           // rr is complete
  int n = top.n_el >= 0 ? min(top.n_el, K) : uniform(rr.part.n_top);
  C2T_PT(PT_RANKED);
  if (sp.nsplit > 1) {
    const int nsplit = sp.nsplit, per_row = nsplit * K;
    const int64_t po = row_launched * nsplit + split;
    if (rr.part.flags & 1u) n = 0;
    if (tid < n) { st_dev(sp.part_topv + po * K + tid, rr.topv[tid]); st_dev(sp.part_topi + po * K + tid, rr.topi[tid]); }
    if (tid == 0) { RowPartial r = rr.part; r.n_top = n; st_dev(sp.part + po, r); }
    if (!last_arrival(tid, s.row_tickets + slot, nsplit)) { C2T_PT_FLUSH(); return; }
    const bool staged = per_row <= sel.list_cap;             // the lists fit the element list
    const RowPartial* rp = sp.part + row_launched * nsplit;
    RowSums m;
    if (last_wave) m = merge_records(rp, nsplit);
    if (staged) stage_lists(tid, sp, row_launched, sel); else rank_lists_from_memory(tid, sp, row_launched, rr);
    __syncthreads();
    if (last_wave) {
      if (lane_id() == 0) {
        RowPartial r; r.ref = m.R; r.a = m.R; r.Z = m.Z; r.S = m.S; r.flags = m.flags; r.n_top = min(m.n_valid, K);
        rr.part = r;
      }
      const ParentStage p = load_parent(s, b, slot);
      if (sp.M <= 0) row_entropy(0, m.R, 1.0, m.Z, m.S, m.flags, rr);
      store_parent(p, rr);
    }
    if (staged) rank_list<NT>(tid, K, sel, per_row, rr.topv, rr.topi);
    __syncthreads();
    if (sp.M > 0) {
      after_merge(rr);
      if (last_wave) row_entropy(sp.M, rr.part, rr);
      __syncthreads();
    }
    n = rr.part.n_top;
    C2T_PT(PT_MERGED);
  }
  const Candidate c = score_row<NT>(tid, s, sp, b, f, nf == 1, rr, n, cls, cls_lds, lds);
  C2T_PT(PT_PUBLISHED);
  if (nf == 1) {                                             // (uniform) the only row: nothing is handed over
    C2T_PT(PT_TICKET);
    prune_lone_row<NT>(tid, s, sp, b, rr, c);
    C2T_PT(PT_PRUNED);
    C2T_PT_FLUSH();
    return;
  }
  if (!last_arrival(tid, s.tickets + b, nf)) { C2T_PT_FLUSH(); return; }   // nf: the sequence's frontier size, known since the workgroup started
  C2T_PT(PT_TICKET);
  // one candidate a thread wherever that is enough: an eighth of the instructions of the general form
  PruneShared<NT>& ps = *(PruneShared<NT>*)(lds + prune_list_bytes(sp.F * K));
  if (sp.F * K <= NT) prune_sequence<NT, 1>(tid, s, sp, b, nf, lds, ps);
  else prune_sequence<NT, C2T_MAX_CANDIDATES_DEV / NT>(tid, s, sp, b, nf, lds, ps);
  C2T_PT(PT_PRUNED);
  C2T_PT_FLUSH();
}

struct TreeOut {
  int32_t* tokens; int32_t* parent; int32_t* position; float* conf; float* joint_prob; float* entropy;
  int32_t* n_nodes; uint8_t* mask; uint32_t* status;
};

// ---- emission: rows [r0, r1) of a sequence's N x N ancestor mask (byte j of row i: j is i or an ancestor of i), by a
// workgroup of NT threads.  What bounds it: the walks (a few dependent steps a node) and N*N bytes written; so the
// parents are read once into LDS, a thread walks one row there and sets its bits in an LDS bit array laid out like the
// bytes, and the bytes are written once, sixteen a store, from the bits (before: the mask was cleared first, every
// step of a walk was a load from memory, and one workgroup did a whole sequence: four sequences of 1024 nodes took 40.5 us a call,
// 6.2 now, five of them the launch).
constexpr int MASK_SLICE = 16384;              // bytes of the mask a workgroup writes at most (one row at least)
constexpr int MASK_BIT_WORDS = MASK_SLICE / 32 + 1;
__host__ __device__ inline int mask_rows_per_slice(int N) { return N >= MASK_SLICE ? 1 : MASK_SLICE / N; }
__device__ __forceinline__ uint32_t spread_bits(uint32_t b) { return (b * 0x00204081u) & 0x01010101u; }    // bit t of b (0..3) to byte t
// parent: LDS, [N]; bits: LDS, MASK_BIT_WORDS; n: nodes of the tree.  A barrier lies behind the writes to parent.
template <int NT>
__device__ __forceinline__ void write_mask_rows(uint8_t* __restrict__ mask, int N, int n, int r0, int r1, const int32_t* parent, uint32_t* bits) {
  const int tid = threadIdx.x, total = (r1 - r0) * N;        // <= MASK_SLICE
  for (int i = tid; i < (total >> 5) + 1; i += NT) bits[i] = 0u;
  __syncthreads();
  for (int i = r0 + tid; i < min(r1, n); i += NT) {
    const int base = (i - r0) * N;
    for (int j = i; j >= 0; j = parent[j]) atomicOr(&bits[(base + j) >> 5], 1u << ((base + j) & 31));     // parents have smaller indices: the walk ends at -1
  }
  __syncthreads();
  uint8_t* out = mask + (int64_t)r0 * N;
  const int head = min(total, (int)((0u - (uint32_t)(uintptr_t)out) & 15u)), chunks = (total - head) >> 4, tail = head + chunks * 16;
  auto bit = [&](int e) { return (uint8_t)((bits[e >> 5] >> (e & 31)) & 1u); };
  if (tid < head) out[tid] = bit(tid);
  for (int c = tid; c < chunks; c += NT) {
    const int e = head + c * 16, sh = e & 31;
    uint32_t w = bits[e >> 5] >> sh;
    if (sh > 16) w |= bits[(e >> 5) + 1] << (32 - sh);
    *(uint4*)(out + e) = make_uint4(spread_bits(w & 15u), spread_bits((w >> 4) & 15u), spread_bits((w >> 8) & 15u), spread_bits((w >> 12) & 15u));
  }
  if (tail + tid < total) out[tail + tid] = bit(tail + tid);   // fewer than sixteen
}

// Copy the node arrays, confidence = sigmoid(z), ancestor mask.  grid: (sequences, slices of the mask's rows).
constexpr int FIN_NT = 256;
__global__ __launch_bounds__(FIN_NT) void k_finalize(TreeState s, TreeOut o, int N) {
  __shared__ int32_t parent[C2T_MAX_BUDGET_DEV];
  __shared__ uint32_t bits[MASK_BIT_WORDS];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int per_slice = mask_rows_per_slice(N), r0 = blockIdx.y * per_slice, r1 = min(r0 + per_slice, N);
  const int64_t tb = (int64_t)b * N;
  const int n = s.n_nodes[b];
  for (int i = tid; i < r1; i += FIN_NT) parent[i] = s.t_parent[tb + i];      // (of nodes past the n-th: not used)
  for (int i = r0 + tid; i < r1; i += FIN_NT) {
    const bool node = i < n;
    const float z = s.t_z[tb + i], P = s.t_P[tb + i], H = s.t_H[tb + i];
    const int tok = s.t_tok[tb + i], par = s.t_parent[tb + i], depth = s.t_depth[tb + i];
    o.tokens[tb + i] = node ? tok : -1; o.parent[tb + i] = node ? par : -1; o.position[tb + i] = node ? depth + 1 : 0;
    o.conf[tb + i] = node ? 1.0f / (1.0f + expf(-z)) : 0.f;
    o.joint_prob[tb + i] = node ? P : 0.f; o.entropy[tb + i] = node ? H : 0.f;
  }
  if (blockIdx.y == 0 && tid == 0) { o.n_nodes[b] = n; o.status[b] = s.status[b]; }
  __syncthreads();
  write_mask_rows<FIN_NT>(o.mask + tb * N, N, n, r0, r1, parent, bits);
}


// EAGLE-2-style reranking (Sec. 2.2), one workgroup of RR_NT threads per sequence: the n_out best of
// every candidate scored in this draft phase under the order (s desc, history index asc), s = the
// smallest classifier logit on the candidate's path (history index = layer * F*K + slot * K + rank
// in the row, so index order is depth, then scoring order).  Parents precede children because s never increases
// along a path.
//
// What bounds it: latency, one workgroup per sequence; so the history is read once (its order-preserving keys go to LDS
// where they fit, 8192 of them; longer histories are read again at each pass).  Up to RR_BOUND_MAX nodes out, a lower
// bound of the n-th best key comes from 256 group maxima (bound_from_maxima), what reaches it is listed, ranked exactly
// on unique 64-bit keys (key, ~index) and cut to n.  More nodes, or more than RR_LIST_MAX candidates above the bound (ties, which
// are usual: a child's smallest logit is often its parent's): an exact radix select of the n-th best key (12 + 12 + 8 bits, an
// LDS histogram per pass), ties in index order.  32 sequences of 1536 candidates with many ties, 60 out: 46.5 us when up to
// 1024 candidates above the bound were ranked, 17.0 now; 16384 candidates, 60 out: 95 us when each thread went through its own
// stretch of the history for the histograms as well, 75 now.
// One phase of 32 sequences with 600 candidates each, 60 out: 16.0 us for this kernel before, when every pass
// read the history from memory again and divided for it.
constexpr int RR_NT = 1024, RR_LDS_KEYS = 8192, RR_BOUND_MAX = 160, RR_LIST_MAX = 256;
constexpr int RR_MASK_ROWS_MAX = 256;          // up to so many nodes out the reranking writes the mask itself; k_mask_of_parents for more
__global__ __launch_bounds__(RR_NT) void k_finalize_rerank(TreeState s, TreeOut o, int n_out, int D, int FK, uint32_t fk_inverse) {
  constexpr int NW = RR_NT / WAVE;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (WAVE - 1), wid = tid >> 6;
  const int total = D * FK;
  const int64_t hb = (int64_t)b * total, ob = (int64_t)b * n_out;
  const int32_t* ncand = s.h_ncand + (int64_t)b * D;
  __shared__ uint32_t keys[RR_LDS_KEYS];                    // then: rank of every selected history index
  __shared__ union { uint32_t dig[4096]; uint32_t lane_max[RR_NT]; uint32_t bits[MASK_BIT_WORDS]; } u;
  __shared__ __align__(16) uint64_t sel[C2T_MAX_BUDGET_DEV];
  __shared__ int32_t sel_par[C2T_MAX_BUDGET_DEV];
  __shared__ int32_t scan_w[NW], scan_e[NW];
  __shared__ int32_t sh_digit, sh_above, n_list;
  const bool in_lds = total <= RR_LDS_KEYS;
  auto layer_of = [&](int i) { return FK > 1 ? (int)__umulhi((uint32_t)i, fk_inverse) : i; };       // i / FK
  auto load_key = [&](int i) -> uint32_t {                   // 0: not a candidate
    const int l = layer_of(i);
    const int tok = s.h_tok[hb + i]; const float v = s.h_s[hb + i];
    return i - l * FK < ncand[l] && tok >= 0 ? sortable_key(v) : 0u;
  };
  auto key_at = [&](int i) { return in_lds ? keys[i] : load_key(i); };

  if (tid == 0) n_list = 0;
  uint32_t mx = 0u; int cnt = 0;
  for (int i = tid; i < total; i += RR_NT) {
    const uint32_t k = load_key(i);
    if (in_lds) keys[i] = k;
    mx = max(mx, k); cnt += k != 0u;
  }
  u.lane_max[wid * WAVE + (lane ^ (wid >> 2))] = mx;         // (groups of different ranks: see prune_sequence)
  cnt = wave_sum_i(cnt);
  if (lane == 0) scan_w[wid] = cnt;
  __syncthreads();
  int n_all = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) n_all += scan_w[w];
  const int n = min(n_out, n_all);
  bool listed = false;
  int m = 0;                                                 // entries of sel, a superset of the selection
  if (n > 0 && (n == n_all || n <= RR_BOUND_MAX)) {
    uint32_t bound = 1u;
    if (n < n_all) {
      uint32_t g[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int w = 0; w < NW; ++w) g[w & 3] = max(g[w & 3], u.lane_max[w * WAVE + lane]);
      bound = max(bound_from_maxima<4>(g, n, n + 32), 1u);
    }
    for (int i0 = 0; i0 < total; i0 += RR_NT) {
      const int i = i0 + tid;
      const uint32_t k = i < total ? key_at(i) : 0u;
      const uint64_t hit = __ballot(k >= bound);
      if (!hit) continue;
      int at = 0;
      if (lane == 0) at = atomicAdd(&n_list, __popcll(hit));
      at = __builtin_amdgcn_readfirstlane(at) + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hit >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hit, 0u));
      if (k >= bound && at < C2T_MAX_BUDGET_DEV) sel[at] = ((uint64_t)k << 32) | (uint32_t)~i;
    }
    __syncthreads();
    m = n_list;
    listed = m <= (n < n_all ? RR_LIST_MAX : C2T_MAX_BUDGET_DEV);
  }
  if (n > 0 && !listed) {
    // a thread owns a contiguous range of history indices, so that index order = thread order
    const int per = (total + RR_NT - 1) / RR_NT, i0 = min(tid * per, total), i1 = min(i0 + per, total);
    uint32_t prefix = 0, care = 0;
    int remaining = n;
    const int shifts[3] = {20, 8, 0}, widths[3] = {12, 12, 8};
#pragma unroll 1
    for (int ps = 0; ps < 3; ++ps) {
      const int shift = shifts[ps]; const uint32_t dmask = (1u << widths[ps]) - 1u;
      __syncthreads();
      for (int i = tid; i < 4096; i += RR_NT) u.dig[i] = 0u;
      __syncthreads();
      for (int i = tid; i < total; i += RR_NT) {
        const uint32_t key = key_at(i);
        if (key && (key & care) == prefix) atomicAdd(&u.dig[(key >> shift) & dmask], 1u);
      }
      __syncthreads();
      {                                                      // thread t owns digits 4095-4t .. 4092-4t
        uint32_t c[4]; int tot = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { c[j] = u.dig[4095 - (4 * tid + j)]; tot += (int)c[j]; }
        const int incl = wave_scan_incl(tot);
        if (lane == WAVE - 1) scan_w[wid] = incl;
        __syncthreads();
        int run = incl - tot;
#pragma unroll
        for (int w = 0; w < NW; ++w) if (w < wid) run += scan_w[w];
        if (run < remaining && run + tot >= remaining) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (run < remaining && run + (int)c[j] >= remaining) { sh_digit = 4095 - (4 * tid + j); sh_above = run; }
            run += (int)c[j];
          }
        }
        __syncthreads();
      }
      remaining -= sh_above;
      prefix |= (uint32_t)sh_digit << shift; care |= dmask << shift;
    }
    // take: keys above the n-th best key, and the first `remaining` equal to it in index order
    int my_gt = 0, my_eq = 0;
    for (int i = i0; i < i1; ++i) {
      const uint32_t key = key_at(i);
      my_gt += key > prefix; my_eq += key == prefix;         // (prefix > 0: the key of a candidate)
    }
    const int ig = wave_scan_incl(my_gt), ie = wave_scan_incl(my_eq);
    __syncthreads();
    if (lane == WAVE - 1) { scan_w[wid] = ig; scan_e[wid] = ie; }
    __syncthreads();
    int sg = ig - my_gt, se = ie - my_eq, tot_gt = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { if (w < wid) { sg += scan_w[w]; se += scan_e[w]; } tot_gt += scan_w[w]; }
    // slots: the keys above first (any order), then the ties in index order
    for (int i = i0; i < i1; ++i) {
      const uint32_t key = key_at(i);
      int slot = -1;
      if (key > prefix) slot = sg++;
      else if (key == prefix) { if (se < remaining) slot = tot_gt + se; ++se; }
      if (slot >= 0 && slot < n) sel[slot] = ((uint64_t)key << 32) | (uint32_t)~i;
    }
    m = n;
    __syncthreads();
  }
  int32_t* const rank_lds = (int32_t*)keys;                  // the keys are not read any more: a barrier lies behind their last use
  int32_t* const rank_mem = s.h_pos + hb;                    // histories that do not fit: the scratch of the caller
  // rank the list by (s desc, index asc), T lanes per entry, and emit its best n
  {
    int tshift = 0;
    while (tshift < 4 && (m << (tshift + 1)) <= RR_NT) ++tshift;
    const int T = 1 << tshift, e = tid >> tshift, sub = tid & (T - 1);
    const bool mine = e < m;
    const uint64_t key = mine ? sel[e] : 0ull;
    const int id = (int)~(uint32_t)key;
    // what the entry emits is requested ahead of the ranking
    const bool lead = mine && sub == 0;
    int tok = -1, pid = -1; float hz = 0.f, hP = 0.f, hH = 0.f;
    if (lead) { tok = s.h_tok[hb + id]; pid = s.h_par[hb + id]; hz = s.h_z[hb + id]; hP = s.h_P[hb + id]; hH = s.h_H[hb + id]; }
    int rank = 0;
    if (mine) {
#pragma unroll 2
      for (int v = sub * 2; v < m; v += T * 2) {
        const uint4 q = *(const uint4*)(sel + v);
        const uint64_t k0 = ((uint64_t)q.y << 32) | q.x, k1 = v + 1 < m ? ((uint64_t)q.w << 32) | q.z : 0ull;
        rank += (k0 > key ? 1 : 0) + (k1 > key ? 1 : 0);
      }
    }
    rank = sum_of_lanes(tshift, rank);
    if (lead && rank < n) {
      if (in_lds) rank_lds[id] = rank; else rank_mem[id] = rank;
      sel_par[rank] = pid;
      o.tokens[ob + rank] = tok; o.position[ob + rank] = layer_of(id) + 1;
      o.conf[ob + rank] = 1.0f / (1.0f + expf(-hz)); o.joint_prob[ob + rank] = hP; o.entropy[ob + rank] = hH;
    }
  }
  for (int e = n + tid; e < n_out; e += RR_NT) {
    o.tokens[ob + e] = -1; o.parent[ob + e] = -1; o.position[ob + e] = 0; o.conf[ob + e] = 0.f; o.joint_prob[ob + e] = 0.f; o.entropy[ob + e] = 0.f;
  }
  if (tid == 0) { o.n_nodes[b] = n; o.status[b] = s.status[b]; }
  if (!in_lds) __threadfence_block();
  __syncthreads();                                           // the rank of every selected candidate is written
  if (tid < n) {                                             // n <= 1024 = RR_NT
    const int pid = sel_par[tid], prank = pid < 0 ? -1 : in_lds ? rank_lds[pid] : rank_mem[pid];
    sel_par[tid] = prank;
    o.parent[ob + tid] = prank;
  }
  if (n_out > RR_MASK_ROWS_MAX) return;
  __syncthreads();
  const int per_slice = mask_rows_per_slice(n_out);
  for (int r0 = 0; r0 < n_out; r0 += per_slice) {
    write_mask_rows<RR_NT>(o.mask + ob * n_out, n_out, n, r0, min(r0 + per_slice, n_out), sel_par, u.bits);
    __syncthreads();
  }
}

// The mask of trees whose parents have been emitted, for more nodes than one workgroup should write.  grid: (sequences, slices).
__global__ __launch_bounds__(FIN_NT) void k_mask_of_parents(TreeOut o, int N) {
  __shared__ int32_t parent[C2T_MAX_BUDGET_DEV];
  __shared__ uint32_t bits[MASK_BIT_WORDS];
  const int b = blockIdx.x, per_slice = mask_rows_per_slice(N), r0 = blockIdx.y * per_slice, r1 = min(r0 + per_slice, N);
  const int64_t ob = (int64_t)b * N;
  const int n = o.n_nodes[b];
  for (int i = threadIdx.x; i < r1; i += FIN_NT) parent[i] = o.parent[ob + i];
  __syncthreads();
  write_mask_rows<FIN_NT>(o.mask + ob * N, N, n, r0, r1, parent, bits);
}

}  // namespace c2t
