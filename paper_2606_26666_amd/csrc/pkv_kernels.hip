// HIP kernels for paged grouped-query decode attention on CDNA4 (gfx950).
//
//   plan_kernel     compact workqueue of non-empty (row, KV head, split) tasks (Sec. 3.4)
//   split_kernel    online-softmax partial state per task (Sec. 3.2-3.3), optionally
//                   followed by the last-arriver merge (Sec. 3.4); also the rectangular
//                   (B, Hkv, S) grid with neutral empty splits (Sec. 3.3)
//   merge_kernel    exact segmented merge of split states (Sec. 3.3)
//
//   stream_kernel   the same tasks in launches with several per compute unit: a workgroup's
//                   tasks run as one stream of pages (pairs of KV heads)
//
// Work mapping. One workgroup owns one task: one KV head g of one row and a token
// range [t0, t1). Its W = 8 wavefronts (two per SIMD, one workgroup per compute unit)
// take the range's 16-token pages round-robin, two pages in flight per wave: lane
// (r, c) = (lane/16, lane%16) loads 16 bytes, dims 8c..8c+7, of tokens 4i+r, so every load
// covers four whole 256-byte head rows. For G = Hq / Hkv = 4 and 8, Q.K^T and P.V run on the
// matrix cores, K and V passing through LDS into the operand layouts (MatrixState); for G = 1
// and 2 on the vector ALU, from the registers the loads fill (VectorState). A task ends with
// an LDS combine of the W wave states in a fixed order. The one-launch route can give a
// workgroup KV heads g and g + 1 of one split instead (NH = 2, one page in flight per head;
// G <= 4), which balances the per-head read rates across workgroups.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "pkv_internal.h"

namespace pkv {
namespace {

constexpr int D = kHeadDim;
constexpr int P = kPageSize;

// threadIdx.x, recomputed from here on: what depends on it is not kept in registers across
// the loop around the call.
__device__ __forceinline__ int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

// Sum over the 16 lanes of a DPP row; every lane of the row receives the same value.
__device__ __forceinline__ float row_sum16(float x) {
  x += dpp<0xB1>(x);   // quad_perm [1,0,3,2]
  x += dpp<0x4E>(x);   // quad_perm [2,3,0,1]
  x += dpp<0x141>(x);  // row_half_mirror
  x += dpp<0x140>(x);  // row_mirror
  return x;
}

// N = 16: the odd 16-lane rows of a change places with the even rows of b; N = 32: the upper half of
// a with the lower half of b.
template <int N>
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
  const auto r = N == 16 ? __builtin_amdgcn_permlane16_swap(x, y, false, false) : __builtin_amdgcn_permlane32_swap(x, y, false, false);
  a = __builtin_bit_cast(float, (unsigned)r[0]);
  b = __builtin_bit_cast(float, (unsigned)r[1]);
}

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }


// Raw buffer descriptor over `bytes` bytes at `base` (word 3 as for gfx9 raw buffers);
// loads past `bytes` return zeros instead of touching memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t page_rsrc(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, 0x00020000);
}

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));

// Dot product of eight fp16 pairs in fp32.
__device__ __forceinline__ float dot8(v4u a, v4u b) {
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    s = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2v, (unsigned)a[i]), __builtin_bit_cast(h2v, (unsigned)b[i]), s, false);
  return s;
}

// Cache policy of the K and V page loads: non-temporal (the nt bit of the buffer
// instruction's cache-policy operand). A step reads every KV byte once; with the
// streaming hint the paged K/V pattern reads 7-9% faster on MI355X than with the default
// policy (read-only probe of the decode's pages: B8 two-head tasks 75.8 -> 69.2 us, B1
// 27.1 -> 25.5 us), while sc0 alone changes nothing.
constexpr int kKvPolicy = 2;

__device__ __forceinline__ uint16_t f32_to_f16_bits(float x) {
  return __builtin_bit_cast(uint16_t, static_cast<_Float16>(x));
}

constexpr float kNegInf = -__builtin_inff();

// ---------------------------------------------------------------------------------
// Partial-state slots (one per task): fp32 acc[G][D], then (m, l) of each of the G heads
// side by side (one 8-byte load fetches both), padded to a multiple of 16 bytes. m is in
// log2 units: scores are scaled by sm_scale*log2(e) and exponentiated with exp2. l < 0
// marks a split that met an invalid page.
template <int G> constexpr int slot_floats() { return G * D + ((2 * G + 3) / 4) * 4; }

// Split s of a row with `tiles` tiles cut into ns splits starts at tile
// floor(s * tiles / ns). With tiles = q * ns + r this is s * q + floor(s * r / ns), and
// s * r < 2^32 for ns <= kMaxSplits, so no 64-bit division is needed.
__device__ __forceinline__ int split_bound(int s, int tiles, int ns) {
  const unsigned q = (unsigned)tiles / (unsigned)ns, r = (unsigned)tiles % (unsigned)ns;
  return (int)((unsigned)s * q + ((unsigned)s * r) / (unsigned)ns);
}

// Slots are accessed through one raw buffer descriptor over the whole slot array. When
// another workgroup merges them inside the same kernel they use agent-scope (sc1)
// accesses, which on gfx950 are coherent across the per-XCD L2 caches, so a completed
// store is visible on every XCD without a full L2 write-back.
constexpr int kSc1 = 16;  // cache-policy operand of a buffer access: sc1

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t slots_rsrc(const DecodeArgs& a, int slot_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(a.partials, (short)0, a.max_tasks * slot_bytes, 0x00020000);
}

template <bool COHERENT>
__device__ __forceinline__ float ld_state(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, COHERENT ? kSc1 : 0));
}
template <bool COHERENT>
__device__ __forceinline__ v2f ld_state2(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, COHERENT ? kSc1 : 0));
}
template <bool COHERENT>
__device__ __forceinline__ v4f ld_state4(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, COHERENT ? kSc1 : 0));
}
template <bool COHERENT>
__device__ __forceinline__ void st_state(__amdgpu_buffer_rsrc_t r, int off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, COHERENT ? kSc1 : 0);
}
template <bool COHERENT>
__device__ __forceinline__ void st_state4(__amdgpu_buffer_rsrc_t r, int off, v4f v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, off, 0, COHERENT ? kSc1 : 0);
}

// ---------------------------------------------------------------------------------
// Merge of split states (Sec. 3.3): M = max m_s, L = sum 2^(m_s-M) l_s,
// A = sum 2^(m_s-M) a_s, O = A / L. The sums follow one fixed tree: runs of kMergeRun
// consecutive splits, each summed in split order from zero, and the run sums added in
// order, so the result depends neither on the thread count nor on the route. merge_group
// does this for a workgroup; merge_columns (several merges side by side, in the stream) and
// finish_task's direct output (one split) go through the same operations in the same order,
// which the tests compare bit by bit. A (row, KV head) with a marked split (l < 0) is zeroed.
//
// Up to 64 splits (eight runs) the column path below reads only existing states. Beyond
// that, the general path: a first pass over blocks of kMergeBlock states for the
// maximum, then per block an item is one run of one float4 column of the output; each
// thread takes at most kMergeItems items per round, so it keeps at most kMergeItems *
// kMergeRun float4 loads in flight (64 registers). A state that does not exist is read
// at an offset past the end of the slot buffer, which a buffer load returns as zero
// without touching memory, and gets weight 0.
constexpr int kMergeBlock = 64;  // split states whose m and l are staged in LDS at a time
constexpr int kMergeRun = 8;     // splits per run
constexpr int kRunsPerBlock = kMergeBlock / kMergeRun;
constexpr int kMergeItems = 2;   // (run, column) items per thread per round
constexpr int kMaxMergeWaves = 16;
constexpr int kOutOfRange = (int)0x80000000u;  // buffer offset past any slot buffer

constexpr int kColRuns = 8;      // the column path merges up to kColRuns runs (64 splits)

template <int G, int NH, int NT>
constexpr int merge_lds_floats() {
  constexpr int GH = NH * G;
  constexpr int general = 2 * kMergeBlock * GH + kRunsPerBlock * GH * D + kRunsPerBlock * GH +
                          2 * kMaxMergeWaves * GH + 3 * GH;
  constexpr int column = (NT / 64) * 256 + kColRuns * GH * D + kColRuns * GH;
  return general > column ? general : column;
}

// The nsplit states at slots slot0 + s*stride (s < nsplit) of one (row, KV head) into
// out_grp[G][D] (fp16). All NT threads of the workgroup take part. NH = 2 merges KV
// heads g and g + 1 of the row together (their slots are adjacent: slot0 + s*stride + 1
// is head g + 1's) into out_grp[2G][D]; every output element goes through the same
// operations, in the same order, as in a one-head merge.
template <int G, int NT, bool COHERENT, int NH = 1>
__device__ __forceinline__ void merge_group(__amdgpu_buffer_rsrc_t pr, int slot0, int stride, int nsplit,
                                            uint16_t* __restrict__ out_grp, float* lds) {
  constexpr int GH = NH * G;                           // query heads merged
  static_assert(NT % 64 == 0 && NT / 64 <= kMaxMergeWaves && 64 % GH == 0, "merge shape");
  constexpr int SB = slot_floats<G>() * 4;             // slot bytes
  constexpr int E4H = G * D / 4;                       // float4 columns per KV head
  constexpr int E4 = NH * E4H;                         // float4 columns of the output
  constexpr int EPT = (GH * D + NT - 1) / NT;          // output elements per thread
  constexpr int KPT = (kMergeBlock * GH + NT - 1) / NT;  // (split, head) states per thread
  float* lw = lds;                                     // [block][GH] weights 2^(m-M)
  float* ll = lw + kMergeBlock * GH;                   // [block][GH] l
  float* part = ll + kMergeBlock * GH;                 // [run][GH*D] run sums of acc
  float* partL = part + kRunsPerBlock * GH * D;        // [run][GH] run sums of l
  float* redM = partL + kRunsPerBlock * GH;            // [wave][GH]
  float* redB = redM + kMaxMergeWaves * GH;            // [wave][GH]
  float* sM = redB + kMaxMergeWaves * GH;              // [GH] max
  float* sBad = sM + GH;                               // [GH]
  float* sL = sBad + GH;                               // [GH] running L
  const int tid = fresh_tid();
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int myh = tid % GH;  // the head of every (split, head) state this thread loads
  const int my_hh = myh / G, my_h = myh % G;
  auto soff = [&](int s, int hh) { return (slot0 + s * stride + hh) * SB; };

  // At most eight runs (64 splits): column path. Column thread c (< GH * D / 4) owns the
  // four output elements 4c .. 4c + 3, so lanes 0-31 of a wave hold one query head's D
  // columns and lanes 32-63 the next head's (GH = 1: one head per half-wave). The NT
  // threads form NG groups of column threads; group i sums runs i, i + NG, i + 2 NG, ...,
  // each in split order from zero, reading its columns from every existing state of
  // those runs (one 16-byte load per state, none for states that do not exist: 1 KiB
  // per wave instruction). A round gives each group RR runs, four where one group covers
  // every column or two groups cover one KV head (32 float4 loads in flight per thread),
  // else two: with four groups, or two for one KV head, one round covers all eight runs;
  // otherwise a round covers four (32 splits), and a merge of more splits takes a second
  // round whose loads refill each run's registers as soon as they are consumed (two
  // groups for a KV-head pair keep 16 loads per thread, within the pair kernel's
  // registers). Lane j of a half loads (m, l) of
  // splits j and j + 32 of its half's head; the maximum and the marker are reduced over
  // the half, and the weights pass through LDS, which every lane of the half reads at
  // the same address. The run sums meet in LDS and group 0 adds them in run order, from
  // zero. The operations and their order are those of the general path below (entries
  // past nsplit in the last run add 0 * 0), so every path rounds alike.
  if (nsplit <= kColRuns * kMergeRun) {
    constexpr int kColThreads = GH * D / 4;
    constexpr int NG = NT / kColThreads >= 4 ? 4 : NT / kColThreads;
    constexpr int RR = NG == 1 || (NG == 2 && NH == 1) ? 4 : 2;  // runs per group and round
    constexpr int NRD = kColRuns / (NG * RR);       // rounds
    constexpr int kWaves = (NG * kColThreads + 63) / 64;
    float* rsum = lds + kWaves * 256;               // [run][GH * D] run sums of acc
    float* rsumL = rsum + kColRuns * GH * D;        // [run][GH] run sums of l
    static_assert(D == 128 && NT % kColThreads == 0 && (NG == 1 || NG == 2 || NG == 4), "column merge shape");
    static_assert(NRD * NG * RR == kColRuns, "column merge rounds");
    static_assert(kWaves * 256 + kColRuns * GH * D + kColRuns * GH <= merge_lds_floats<G, NH, NT>(),
                  "column merge LDS");
    const int gi = tid / kColThreads;              // group
    const int c = tid - gi * kColThreads;          // column thread
    const int h = c / (D / 4);                     // query head within the GH merged
    const int nrun = (nsplit + kMergeRun - 1) / kMergeRun;
    const bool wide = nsplit > 4 * kMergeRun;      // runs 4-7 exist
    float M = kNegInf, bd = 0.0f;
    if (gi < NG) {
      const int hb = lane >> 5, js = lane & 31;
      const int hh = h / G;                        // KV head within the NH merged
      const int ecol = (h % G) * D + (c % (D / 4)) * 4;  // first element in that KV head's acc
      const int ml_at = (G * D + 2 * (h % G)) * 4;
      const bool ok0 = js < nsplit, ok1 = wide && js + 32 < nsplit;
      const v2f ml0 = ld_state2<COHERENT>(pr, ok0 ? soff(js, hh) + ml_at : kOutOfRange);
      v2f ml1 = {0.0f, 0.0f};
      if (wide) ml1 = ld_state2<COHERENT>(pr, ok1 ? soff(js + 32, hh) + ml_at : kOutOfRange);
      // vq[k * kMergeRun + u]: split u of this group's run in slot k of the current round.
      // A slot is refilled with the next round's run as soon as it has been consumed, so
      // the rounds' loads overlap.
      v4f vq[RR * kMergeRun];
      auto issue = [&](int rd, int k) {  // run gi + NG * (rd * RR + k) into slot k
        if (NG * (rd * RR + k) >= 4 && !wide) return;  // a run >= 4: none exists
#pragma unroll
        for (int u = 0; u < kMergeRun; ++u) {
          const int sidx = (gi + NG * (rd * RR + k)) * kMergeRun + u;
          vq[k * kMergeRun + u] =
              sidx < nsplit ? ld_state4<COHERENT>(pr, soff(sidx, hh) + ecol * 4) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
      };
#pragma unroll
      for (int k = 0; k < RR; ++k) issue(0, k);
      M = fmaxf(ok0 ? ml0.x : kNegInf, ok1 ? ml1.x : kNegInf);
      bd = (ok0 && ml0.y < 0.0f) || (ok1 && ml1.y < 0.0f) ? 1.0f : 0.0f;
      M = fmaxf(M, dpp<0xB1>(M));   // quad_perm [1,0,3,2]
      M = fmaxf(M, dpp<0x4E>(M));   // quad_perm [2,3,0,1]
      M = fmaxf(M, dpp<0x141>(M));  // row_half_mirror
      M = fmaxf(M, dpp<0x140>(M));  // row_mirror: every lane of a row holds the row's maximum
      bd = fmaxf(bd, dpp<0xB1>(bd));
      bd = fmaxf(bd, dpp<0x4E>(bd));
      bd = fmaxf(bd, dpp<0x141>(bd));
      bd = fmaxf(bd, dpp<0x140>(bd));
      auto lane_f = [](float x, int l) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
      };
      const float M0 = fmaxf(lane_f(M, 0), lane_f(M, 16)), M1 = fmaxf(lane_f(M, 32), lane_f(M, 48));
      const float B0 = fmaxf(lane_f(bd, 0), lane_f(bd, 16)), B1 = fmaxf(lane_f(bd, 32), lane_f(bd, 48));
      M = hb ? M1 : M0;
      bd = hb ? B1 : B0;
      const float Mref = (M == kNegInf) ? 0.0f : M;
      v2f* wl = reinterpret_cast<v2f*>(lds) + wave * 128;  // (weight, l) of split j of half hb at hb * 64 + j
      wl[hb * 64 + js] = v2f{ok0 ? ex2(ml0.x - Mref) : 0.0f, ok0 ? ml0.y : 0.0f};
      if (wide) wl[hb * 64 + 32 + js] = v2f{ok1 ? ex2(ml1.x - Mref) : 0.0f, ok1 ? ml1.y : 0.0f};
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int rd = 0; rd < NRD; ++rd) {
#pragma unroll
        for (int k = 0; k < RR; ++k) {
          const int r = gi + NG * (rd * RR + k);
          if (r < nrun) {
            v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
            float lacc = 0.0f;
#pragma unroll
            for (int u = 0; u < kMergeRun; ++u) {
              const v2f wlv = wl[hb * 64 + r * kMergeRun + u];  // zero weight and l past nsplit
              const v4f x = vq[k * kMergeRun + u];
              acc.x = __builtin_fmaf(wlv.x, x.x, acc.x);
              acc.y = __builtin_fmaf(wlv.x, x.y, acc.y);
              acc.z = __builtin_fmaf(wlv.x, x.z, acc.z);
              acc.w = __builtin_fmaf(wlv.x, x.w, acc.w);
              lacc = __builtin_fmaf(wlv.x, wlv.y, lacc);
            }
            *reinterpret_cast<v4f*>(rsum + r * GH * D + 4 * c) = acc;
            if (c % (D / 4) == 0) rsumL[r * GH + h] = lacc;
          }
          if (rd + 1 < NRD) issue(rd + 1, k);  // refill the slot just consumed
        }
      }
    }
    __syncthreads();
    if (gi == 0) {  // M and bd of this thread's head are this thread's own
      v4f o = {0.0f, 0.0f, 0.0f, 0.0f};
      float L = 0.0f;
      // Run sums added in run order, from zero, four runs' LDS reads at a time; a run
      // past nrun adds +0, which leaves the sums bitwise unchanged (a sum started at +0
      // is never -0).
      for (int r0 = 0; r0 < nrun; r0 += 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int r = r0 + k;
          const v4f v = *reinterpret_cast<const v4f*>(rsum + r * GH * D + 4 * c);
          const float lr = rsumL[r * GH + h];
          o += r < nrun ? v : v4f{0.0f, 0.0f, 0.0f, 0.0f};
          L += r < nrun ? lr : 0.0f;
        }
      }
      const bool zero = M == kNegInf || bd != 0.0f;
      const float iL = 1.0f / L;  // one division per head, then products
      const unsigned lo = f32_to_f16_bits(zero ? 0.0f : o.x * iL) | ((unsigned)f32_to_f16_bits(zero ? 0.0f : o.y * iL) << 16);
      const unsigned hi = f32_to_f16_bits(zero ? 0.0f : o.z * iL) | ((unsigned)f32_to_f16_bits(zero ? 0.0f : o.w * iL) << 16);
      *reinterpret_cast<uint2*>(out_grp + 4 * c) = make_uint2(lo, hi);
    }
    return;
  }

  float mv[KPT], lv[KPT];
  auto load_ml = [&](int s0, int cnt) {
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      const int e = tid + k * NT;
      const bool ok = e < cnt * GH;
      const int off = ok ? soff(s0 + e / GH, my_hh) + (G * D + 2 * my_h) * 4 : kOutOfRange;
      const v2f ml = ld_state2<COHERENT>(pr, off);  // (m, l); zeros when absent
      lv[k] = ml.y;
      mv[k] = ok ? ml.x : kNegInf;
    }
  };
  // max and marker over this thread's states, then over lanes of the same head, then
  // over waves; folded into sM / sBad (exact: max does not depend on the order)
  auto reduce_max = [&]() {
    float mx = kNegInf, bd = 0.0f;
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      mx = fmaxf(mx, mv[k]);
      bd = fmaxf(bd, lv[k] < 0.0f ? 1.0f : 0.0f);
    }
#pragma unroll
    for (int sh = GH; sh < 64; sh <<= 1) {
      mx = fmaxf(mx, __shfl_xor(mx, sh));
      bd = fmaxf(bd, __shfl_xor(bd, sh));
    }
    if (lane < GH) {
      redM[wave * GH + lane] = mx;
      redB[wave * GH + lane] = bd;
    }
    __syncthreads();
    if (tid < GH) {
      float m2 = sM[tid], b2 = sBad[tid];
      for (int w = 0; w < NT / 64; ++w) {
        m2 = fmaxf(m2, redM[w * GH + tid]);
        b2 = fmaxf(b2, redB[w * GH + tid]);
      }
      sM[tid] = m2;
      sBad[tid] = b2;
    }
    __syncthreads();
  };

  if (tid < GH) {
    sM[tid] = kNegInf;
    sBad[tid] = 0.0f;
    sL[tid] = 0.0f;
  }
  for (int s0 = 0; s0 < nsplit; s0 += kMergeBlock) {  // pass 1: maximum over every block
    load_ml(s0, min(kMergeBlock, nsplit - s0));
    reduce_max();
  }
  float A[EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) A[q] = 0.0f;
  v4f v[kMergeItems][kMergeRun];
  for (int s0 = 0; s0 < nsplit; s0 += kMergeBlock) {
    const int cnt = min(kMergeBlock, nsplit - s0);
    const int nrun = (cnt + kMergeRun - 1) / kMergeRun;
    const int nitems = E4 * nrun;
    // item it: run it / E4 of the block, float4 column it % E4 (head it % E4 / E4H)
    auto issue = [&](int j, int it) {  // it >= nitems: every load is out of range (zeros)
      const int e4 = it % E4;
      const int hh = e4 / E4H;
      const int sb = (it / E4) * kMergeRun;
      const int n = it < nitems ? min(kMergeRun, cnt - sb) : 0;
#pragma unroll
      for (int u = 0; u < kMergeRun; ++u)
        v[j][u] = ld_state4<COHERENT>(pr, u < n ? soff(s0 + sb + u, hh) + (e4 - hh * E4H) * 16 : kOutOfRange);
    };
    auto finish = [&](int j, int it) {
      const int e4 = it % E4;  // = hh * E4H + column within KV head hh
      const int run = it / E4;
      const int sb = run * kMergeRun;
      const int h = (e4 * 4) / D;  // query head within the GH merged
      v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
      float lacc = 0.0f;
      // entries past the block's states have weight 0 and zero data: adding 0 * 0 to a
      // sum that starts at +0 leaves it unchanged, so no per-split branch is needed
#pragma unroll
      for (int u = 0; u < kMergeRun; ++u) {
        const float w = lw[(sb + u) * GH + h];
        acc.x = __builtin_fmaf(w, v[j][u].x, acc.x);
        acc.y = __builtin_fmaf(w, v[j][u].y, acc.y);
        acc.z = __builtin_fmaf(w, v[j][u].z, acc.z);
        acc.w = __builtin_fmaf(w, v[j][u].w, acc.w);
        lacc = __builtin_fmaf(w, ll[(sb + u) * GH + h], lacc);
      }
      *reinterpret_cast<v4f*>(part + run * GH * D + e4 * 4) = acc;
      if ((e4 * 4) % D == 0) partL[run * GH + h] = lacc;
    };
    __syncthreads();  // the previous block's LDS is consumed
#pragma unroll
    for (int j = 0; j < kMergeItems; ++j) issue(j, tid + j * NT);  // in flight during the weights
    load_ml(s0, cnt);
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
      const int e = tid + k * NT;
      if (e < kMergeBlock * GH) {
        const float M = sM[myh];
        const bool ok = e < cnt * GH;
        lw[e] = ok ? ex2(mv[k] - (M == kNegInf ? 0.0f : M)) : 0.0f;
        ll[e] = ok ? lv[k] : 0.0f;
      }
    }
    __syncthreads();
    for (int it0 = 0; it0 < nitems; it0 += kMergeItems * NT) {
      if (it0 > 0) {
#pragma unroll
        for (int j = 0; j < kMergeItems; ++j) issue(j, it0 + tid + j * NT);
      }
#pragma unroll
      for (int j = 0; j < kMergeItems; ++j)
        if (it0 + tid + j * NT < nitems) finish(j, it0 + tid + j * NT);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      const int e = tid + q * NT;
      if (e < GH * D)
        for (int run = 0; run < nrun; ++run) A[q] += part[run * GH * D + e];
    }
    if (tid < GH)
      for (int run = 0; run < nrun; ++run) sL[tid] += partL[run * GH + tid];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int e = tid + q * NT;
    if (e >= GH * D) break;
    const int h = e / D;
    const float o = (sM[h] == kNegInf || sBad[h] != 0.0f) ? 0.0f : A[q] * (1.0f / sL[h]);
    out_grp[e] = f32_to_f16_bits(o);
  }
}

// The column path for a team of GH * D / 4 threads (one KV head; thread c of the team owns
// output elements 4c .. 4c + 3) that merges nsplit <= 64 states by itself: the runs one after
// another, so a workgroup can merge several (row, KV head)s side by side, one per team.
// `ns_max`: the largest nsplit among the wave's teams (G = 1 has two in a wave). wl: 128
// (weight, l) pairs of LDS per wave. The operations and their order are merge_group's.
template <int G, bool COHERENT>
__device__ __forceinline__ void merge_columns(__amdgpu_buffer_rsrc_t pr, int slot0, int stride, int nsplit, int ns_max,
                                              int c, uint16_t* __restrict__ out_grp, v2f* wl) {
  constexpr int SB = slot_floats<G>() * 4;
  const int lane = fresh_tid() & 63;
  const int hb = lane >> 5, js = lane & 31;
  const int h = c / (D / 4);  // query head
  const int col_at = slot0 * SB + c * 16;
  const int ml_at = slot0 * SB + (G * D + 2 * h) * 4;
  const int step = stride * SB;
  const bool ok0 = js < nsplit, ok1 = js + 32 < nsplit;
  const v2f ml0 = ld_state2<COHERENT>(pr, ok0 ? ml_at + js * step : kOutOfRange);
  const v2f ml1 = ld_state2<COHERENT>(pr, ok1 ? ml_at + (js + 32) * step : kOutOfRange);
  v4f v[kMergeRun];
  auto issue = [&](int r) {
    const int at = col_at + r * kMergeRun * step;
#pragma unroll
    for (int u = 0; u < kMergeRun; ++u)
      v[u] = ld_state4<COHERENT>(pr, r * kMergeRun + u < nsplit ? at + u * step : kOutOfRange);
  };
  issue(0);
  float M = fmaxf(ok0 ? ml0.x : kNegInf, ok1 ? ml1.x : kNegInf);
  float bd = (ok0 && ml0.y < 0.0f) || (ok1 && ml1.y < 0.0f) ? 1.0f : 0.0f;
#pragma unroll
  for (int sh = 1; sh < 32; sh <<= 1) {  // over the half-wave
    M = fmaxf(M, __shfl_xor(M, sh));
    bd = fmaxf(bd, __shfl_xor(bd, sh));
  }
  const float Mref = (M == kNegInf) ? 0.0f : M;
  wl[hb * 64 + js] = v2f{ok0 ? ex2(ml0.x - Mref) : 0.0f, ok0 ? ml0.y : 0.0f};
  wl[hb * 64 + 32 + js] = v2f{ok1 ? ex2(ml1.x - Mref) : 0.0f, ok1 ? ml1.y : 0.0f};
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  v4f o = {0.0f, 0.0f, 0.0f, 0.0f};
  float L = 0.0f;
  const int nrun = (ns_max + kMergeRun - 1) / kMergeRun;
#pragma clang loop unroll(disable)
  for (int r = 0; r < nrun; ++r) {
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    float lacc = 0.0f;
#pragma unroll
    for (int u = 0; u < kMergeRun; ++u) {
      const v2f wlv = wl[hb * 64 + r * kMergeRun + u];  // zero weight and l past nsplit
      acc.x = __builtin_fmaf(wlv.x, v[u].x, acc.x);
      acc.y = __builtin_fmaf(wlv.x, v[u].y, acc.y);
      acc.z = __builtin_fmaf(wlv.x, v[u].z, acc.z);
      acc.w = __builtin_fmaf(wlv.x, v[u].w, acc.w);
      lacc = __builtin_fmaf(wlv.x, wlv.y, lacc);
    }
    if (r + 1 < nrun) issue(r + 1);
    o += acc;  // a run past the team's nsplit adds +0
    L += lacc;
  }
  if (nsplit > 0) {
    const bool zero = M == kNegInf || bd != 0.0f;
    const float iL = 1.0f / L;
    const unsigned lo = f32_to_f16_bits(zero ? 0.0f : o.x * iL) | ((unsigned)f32_to_f16_bits(zero ? 0.0f : o.y * iL) << 16);
    const unsigned hi = f32_to_f16_bits(zero ? 0.0f : o.z * iL) | ((unsigned)f32_to_f16_bits(zero ? 0.0f : o.w * iL) << 16);
    *reinterpret_cast<uint2*>(out_grp + 4 * c) = make_uint2(lo, hi);
  }
}

// ---------------------------------------------------------------------------------
// One task: KV head g of `row`, tokens [t0, t1), partial state into `slot`.
// The task's partial state from the W wave states staged in LDS (m, l, acc per wave
// and head, page-error flag per wave): a fixed-order combine, stored to slot `slot`.
// NH = 2: the states of KV heads g and g + 1 (tasks `slot` and `slot` + 1), side by side
// in LDS, each combined exactly as a one-head task's.
// Layout of the wave states in LDS: (m, l) pairs [NH][W][G] (l = -1: the wave met an invalid
// page), then acc [NH][W][G][kHeadPitch]. The pitch of a head's D columns puts the matrix
// body's stores of several heads at once on distinct banks (at D floats the heads of one store
// share their banks: 256 short rows at G = 8 169.5 instead of 154.3 us, 256 one-tile rows 33.5
// instead of 28.8, long tasks alike).
// `direct`: the task is its row's only split, so its state is the merged state: the output
// goes there at once (the arithmetic of a one-split merge: weight 1, sums started at +0) and
// no state is stored. Threads tid, tid + NT, ... take the columns. `heads`: how many of the NH.
constexpr int kHeadPitch = D + 4;

template <int G, int W, int NH = 1>
constexpr int lds_floats() {
  return NH * W * G * (2 + kHeadPitch);
}
template <int G, int W, int NH = 1>
__device__ __forceinline__ v2f* state_ml(float* lds) { return reinterpret_cast<v2f*>(lds); }
template <int G, int W, int NH = 1>
__device__ __forceinline__ float* state_acc(float* lds) { return lds + 2 * NH * W * G; }

template <int G, int W, bool COHERENT, int NH = 1>
__device__ __forceinline__ void finish_task(const DecodeArgs& a, int slot, float* lds, uint16_t* direct, int tid,
                                            int heads = NH) {
  constexpr int SB = slot_floats<G>() * 4;
  constexpr int E4H = G * D / 4;  // float4 columns per head
  const __amdgpu_buffer_rsrc_t pr = slots_rsrc(a, SB);
  for (int e4g = tid; e4g < heads * E4H; e4g += W * 64) {
    const int hh = e4g / E4H;
    const int e4 = e4g - hh * E4H;
    const int h = (e4 * 4) / D;
    const v2f* ml = state_ml<G, W, NH>(lds) + hh * W * G + h;
    const float* hacc = state_acc<G, W, NH>(lds) + (hh * W * G + h) * kHeadPitch + (e4 * 4) % D;
    const int so = (slot + hh) * SB;
    v2f s[W];
#pragma unroll
    for (int w = 0; w < W; ++w) s[w] = ml[w * G];
    float M = kNegInf;
    bool any_bad = false;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      M = fmaxf(M, s[w].x);
      any_bad |= s[w].y < 0.0f;
    }
    const float Mref = (M == kNegInf) ? 0.0f : M;
    float L = 0.0f;
    v4f A = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float cf = ex2(s[w].x - Mref);
      const v4f x = *reinterpret_cast<const v4f*>(hacc + w * G * kHeadPitch);
      L = __builtin_fmaf(cf, s[w].y, L);
      A.x = __builtin_fmaf(cf, x.x, A.x);
      A.y = __builtin_fmaf(cf, x.y, A.y);
      A.z = __builtin_fmaf(cf, x.z, A.z);
      A.w = __builtin_fmaf(cf, x.w, A.w);
    }
    if (any_bad && e4 == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_PAGE_ID);
    if (direct) {
      const bool zero = M == kNegInf || any_bad;
      const float iL = 1.0f / L;
      A += v4f{0.0f, 0.0f, 0.0f, 0.0f};
      const unsigned lo = f32_to_f16_bits(zero ? 0.0f : A.x * iL) | ((unsigned)f32_to_f16_bits(zero ? 0.0f : A.y * iL) << 16);
      const unsigned hi = f32_to_f16_bits(zero ? 0.0f : A.z * iL) | ((unsigned)f32_to_f16_bits(zero ? 0.0f : A.w * iL) << 16);
      *reinterpret_cast<uint2*>(direct + 4 * e4g) = make_uint2(lo, hi);
      continue;
    }
    st_state4<COHERENT>(pr, so + e4 * 16, A);
    if ((e4 * 4) % D == 0) {
      st_state<COHERENT>(pr, so + (G * D + 2 * h) * 4, M);
      st_state<COHERENT>(pr, so + (G * D + 2 * h + 1) * 4, any_bad ? -1.0f : L);
    }
  }
}

// ---------------------------------------------------------------------------------
// The task body on the matrix cores (G = 4 and 8): the path is 4 flop per byte at G = 4, far
// below their rate, but the vector form spends its issue slots on dot products and FMAs (G = 4 on
// the vector ALU: 32 K tokens 28.0 against 25.5 us, 64 chat rows 110 against 94, buckets 117
// against 100).
//
// Per 16-token page of the task's KV head, one wave computes
//   S[16 tokens x 16] = K_page[16 x 128] . Q^T[128 x 16]       (4 x mfma 16x16x32 f16)
// with the G query heads in columns 0..G-1 (the others zero), and
//   O^T[128 x 16] += V_page^T[128 x 16 tokens] . P^T[16 tokens x 16]   (16 x mfma 16x16x16 f16:
//                                                                      P as hi + lo halves)
// Lane (grp, col) = (lane / 16, lane % 16):
//   K operand   token col, dims [32 c + 8 grp, +8): K is read as V is, four 1 KiB loads
//               of four whole 256-byte head rows each (lane: token 4 i + grp, dims
//               [8 col, +8)), staged token-major in LDS and read back in this layout
//               (on MI355X, whole-row reads stream 2-4% faster than 64-byte pieces)
//   Q operand   head col, dims [32 c + 8 grp, +8) (zero for col >= G), loaded once
//   scores      tokens 4 grp + r (r = 0..3) of head col, which is also the P operand
//   V operand   dims 16 db + col, tokens 4 grp + r: V is staged token-major in LDS and
//               read back transposed with ds_read_b64_tr_b16 (within 16 lanes, lane i
//               receives element i % 4 of the rows that lanes 4 j + i / 4 address)
// The staged rows are padded (K to 272 bytes, V to 288) so that the lanes of one LDS
// pass address distinct banks.
//   output      dims 16 db + 4 grp + r of head col
// Every value a lane holds belongs to head col, so the online-softmax max (shared by the
// four groups of a head, per page) and the rescale are per lane.
typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4v lds_s4v;

// Per wave, one K and one V page of one head staged in LDS: 16 rows of 256 bytes each,
// padded (pitches in 16-byte units). One allocation per kernel, whatever the callers.
constexpr int kKPitch = D / 8 + 1, kVPitch = D / 8 + 2;
constexpr int kStageUnits = P * (kKPitch + kVPitch);
template <int W>
__device__ __forceinline__ v4u* kv_stage() {
  __shared__ v4u stage[W * kStageUnits];
  return stage;
}

// One page's arithmetic for one KV head, which both task bodies below share. A wave's staging
// area holds K as [16][kKPitch] and V as [16][kVPitch] 16-byte units. Every place a lane
// touches is one of four LDS addresses plus a constant offset; they and the two other
// per-lane constants are formed once and kept as opaque registers (left to itself the
// compiler keeps their parts, adds them up again on every page and spills some).
typedef __attribute__((address_space(3))) v4u lds_v4u;

template <typename T>
__device__ __forceinline__ T opaque(T x) {
  asm volatile("" : "+v"(x));
  return x;
}

//
// The weights p = 2^(x - m) enter the product scaled by kWeightScale (a power of two, so every
// value carries it exactly; a wave's l takes it on with its state, and the final division
// takes it out). P is multiplied as fp16 hi + lo parts, and fp16 ends at 2^-24: scaled, a
// weight keeps 22 bits down to 2^-17 of the largest and below that an absolute error of 2^-39
// (unscaled: 2^-3 and 2^-25, where the many small weights of a long row add up to a visible part
// of the sum). A V that is infinite gives a NaN where the lo part is 0 or negative.
constexpr float kWeightScale = 16384.0f;

struct PageMath {
  int kw, kr, vw, vr;  // LDS addresses of this lane's K row piece, K operand, V row piece, V operand
  int other;           // byte lane index of lane ^ 32

  __device__ __forceinline__ void init(v4u* st) {
    const int lane = threadIdx.x & 63, grp = lane >> 4, col = lane & 15;
    const int base = (int)(__UINTPTR_TYPE__)(lds_v4u*)st;
    const int vbase = base + P * kKPitch * 16;
    kw = opaque(base + (grp * kKPitch + col) * 16);
    kr = opaque(base + (col * kKPitch + grp) * 16);
    vw = opaque(vbase + (grp * kVPitch + col) * 16);
    vr = opaque(vbase + (4 * grp + (col >> 2)) * (kVPitch * 16) + (col & 3) * 8);
    other = opaque((lane ^ 32) << 2);
  }
  // K token-major into LDS.
  __device__ __forceinline__ void stage_k(const v4u (&r)[4]) const {
    lds_v4u* at = (lds_v4u*)(unsigned)kw;
#pragma unroll
    for (int i = 0; i < 4; ++i) at[4 * i * kKPitch] = r[i];
  }
  // V token-major; rows past t1 are zeroed (their p is 0, but 0 * NaN is not).
  __device__ __forceinline__ void stage_v(v4u (&r)[4], int tok0, int t1) const {
    if (tok0 + P > t1) {
      const int tok = tok0 + ((fresh_tid() & 63) >> 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned keep = tok + 4 * i < t1 ? ~0u : 0u;
        r[i] &= v4u{keep, keep, keep, keep};
      }
    }
    lds_v4u* at = (lds_v4u*)(unsigned)vw;
#pragma unroll
    for (int i = 0; i < 4; ++i) at[4 * i * kVPitch] = r[i];
  }
  // Scores of tokens 4 grp + r of head col.
  __device__ __forceinline__ v4f scores(const v4u (&qh)[4]) const {
    const lds_v4u* at = (const lds_v4u*)(unsigned)kr;
    v4f sc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 4; ++c)
      sc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8v, (v4u)at[4 * c]), __builtin_bit_cast(h8v, qh[c]),
                                                  sc, 0, 0, 0);
    return sc;
  }
  // Over the four lanes of a head: lane xor 16, then xor 32.
  template <typename Op>
  __device__ __forceinline__ float over_groups(float x, Op op) const {
    x = op(x, __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x), 0x401F)));
    return op(x, __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(other, __builtin_bit_cast(int, x))));
  }
  // The page's scores and staged V into (m, l, acc).
  __device__ __forceinline__ void accumulate(v4f sc, float scale_log2, int tok0, int t1, float& m, float& l,
                                             v4f (&acc)[D / 16]) const {
    float x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = sc[r] * scale_log2;
    if (tok0 + P > t1) {  // the row's last, partial page
      const int tok = tok0 + 4 * ((fresh_tid() & 63) >> 4);
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = tok + r < t1 ? x[r] : kNegInf;
    }
    float mp = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    // m is the same in a head's four lanes, so the page's maximum is formed, and the state
    // rescaled, only when a score exceeds it in some lane.
    if (__builtin_amdgcn_ballot_w64(mp > m)) {
      mp = over_groups(mp, [](float u, float v) { return fmaxf(u, v); });
      if (mp > m) {
        const float alpha = ex2(m - mp);
        l *= alpha;
#pragma unroll
        for (int db = 0; db < D / 16; ++db) acc[db] *= alpha;
        m = mp;
      }
    }
    // P enters the product as fp16 hi + lo parts: p - hi is exact in fp32, and its fp16 rounding
    // leaves 2^-22 of the weight or 2^-39 of the largest
    const float mref = (m == kNegInf) ? 0.0f : m;
    h4v ph, pl;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float p = ex2(x[r] - mref);
      l += p;
      const float ps = p * kWeightScale;
      ph[r] = (_Float16)ps;
      pl[r] = (_Float16)__builtin_fmaf((float)ph[r], -1.0f, ps);
    }
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      const h4v va_ = __builtin_bit_cast(h4v, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v*)(unsigned)(vr + db * 32)));
      acc[db] = __builtin_amdgcn_mfma_f32_16x16x16f16(va_, ph, acc[db], 0, 0, 0);
      acc[db] = __builtin_amdgcn_mfma_f32_16x16x16f16(va_, pl, acc[db], 0, 0, 0);
    }
  }
};

// A wave's softmax state of one KV head in the task it is in, with the arithmetic of a page: scores
// from the page's K and the queries `q` (kQ registers of four words, as load_q leaves them), then
// accumulate(). dump() leaves the state in LDS.
template <int G>
struct MatrixState {
  typedef v4f Scores;
  static constexpr int kQ = 4;
  static constexpr int kStage = kStageUnits;  // 16-byte units of LDS per wave for staged pages
  float m, l;
  v4f acc[D / 16];

  __device__ __forceinline__ void reset() {
    m = kNegInf;
    l = 0.0f;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) acc[db] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  }
  // Lane (grp, col): head col, dims [32 c + 8 grp, +8); columns G..15 read past the descriptor
  // (zeros), so the loads carry no branch. `at`: bytes of this head's queries in it.
  static __device__ __forceinline__ void load_q(v4u (&q)[kQ], __amdgpu_buffer_rsrc_t r, int at, int tid) {
    const int grp = (tid & 63) >> 4, col = tid & 15;
    const int qoff = col < G ? at + (col * D + 8 * grp) * 2 : kOutOfRange;
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = __builtin_amdgcn_raw_buffer_load_b128(r, qoff, c * 64, 0);
  }
  __device__ __forceinline__ void dump(const PageMath& pm, float* acc_at, v2f* ml_at, bool bad, int tid) {
    const int grp = (tid & 63) >> 4, col = tid & 15;
    const float lw = pm.over_groups(l, [](float u, float v) { return u + v; }) * kWeightScale;
    if (col < G) {
#pragma unroll
      for (int db = 0; db < D / 16; ++db) *reinterpret_cast<v4f*>(acc_at + col * kHeadPitch + 16 * db + 4 * grp) = acc[db];
      if (grp == 0) ml_at[col] = v2f{m, bad ? -1.0f : lw};
    }
  }
};

// On the vector ALU: lane (r, c) = (lane / 16, lane % 16) holds dims 8c .. 8c + 7 of tokens 4 i + r
// as loaded. Partial dot products (v_dot2) meet over the 16 lanes of a row; each row keeps a
// softmax state of its own (m, l, its lanes' 8 columns of acc), and the four rows meet in dump().
// Weights stay in fp32 from the exponential to the sum, and a weight times an infinite V is
// infinite, neither of which the matrix form's fp16 halves can give. As fast in the routes' kernels:
// four rows at G = 1 128.6 (matrix) and 127.9 us, eight rows at G = 2 105.8 and 105.2; with one
// head per workgroup and no LDS for pages, rectangular slots of rows of 1500 tokens (Hkv = 32,
// 8 rows) 43.7 and 28.8; slowest against it at G = 2: 2% to 4% for rows of 16-32 K tokens one by
// one (78 and 80 us), up to 7% for grids of 16384 short slots (147 and 158).
template <int G>
struct VectorState {
  struct Scores {
    float x[G][4];
  };
  static constexpr int kQ = G;
  static constexpr int kStage = 64;  // no page is staged: room for the merge's 128 (weight, l) pairs
  float m[G], l[G], acc[G][8];

  __device__ __forceinline__ void reset() {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m[h] = kNegInf;
      l[h] = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[h][k] = 0.0f;
    }
  }
  static __device__ __forceinline__ void load_q(v4u (&q)[kQ], __amdgpu_buffer_rsrc_t r, int at, int tid) {
#pragma unroll
    for (int h = 0; h < G; ++h) q[h] = __builtin_amdgcn_raw_buffer_load_b128(r, at + (tid & 15) * 16, h * D * 2, 0);
  }
  __device__ __forceinline__ Scores scores(const v4u (&q)[kQ], const v4u (&kr)[4], float scale_log2) const {
    Scores s;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int h = 0; h < G; ++h) s.x[h][i] = row_sum16(dot8(q[h], kr[i])) * scale_log2;
    return s;
  }
  __device__ __forceinline__ void accumulate(Scores& s, v4u (&vr)[4], int tok0, int t1) {
    if (tok0 + P > t1) {  // the row's last, partial page: this lane row's token in load i is tok + 4i
      const int tok = tok0 + ((fresh_tid() & 63) >> 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool valid = tok + 4 * i < t1;
#pragma unroll
        for (int h = 0; h < G; ++h) s.x[h][i] = valid ? s.x[h][i] : kNegInf;
        const unsigned keep = valid ? ~0u : 0u;  // p is 0 there, but 0 * NaN is not
        vr[i] &= v4u{keep, keep, keep, keep};
      }
    }
    float mt[G];
    bool grow = false;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      mt[h] = fmaxf(fmaxf(s.x[h][0], s.x[h][1]), fmaxf(s.x[h][2], s.x[h][3]));
      grow |= mt[h] > m[h];
    }
    if (__builtin_amdgcn_ballot_w64(grow)) {  // rescale only when some running max grows
#pragma unroll
      for (int h = 0; h < G; ++h) {
        if (mt[h] > m[h]) {
          const float alpha = ex2(m[h] - mt[h]);
          l[h] *= alpha;
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[h][k] *= alpha;
          m[h] = mt[h];
        }
      }
    }
    float vf[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const h8v v = __builtin_bit_cast(h8v, vr[i]);
#pragma unroll
      for (int k = 0; k < 8; ++k) vf[i][k] = (float)v[k];
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float mref = (m[h] == kNegInf) ? 0.0f : m[h];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = ex2(s.x[h][i] - mref);
        l[h] += p;
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[h][k] = __builtin_fmaf(p, vf[i][k], acc[h][k]);
      }
    }
  }
  // The four rows' states meet: rows 0 and 1 and rows 2 and 3, then the two pairs. An exchange of
  // two columns leaves one of them with each partner, so the second step has half the columns and
  // a lane ends with two: every column goes through the operations of a full exchange of rows
  // (2 G (8 + 2) ds_bpermute per head; G = 2, 256 rows of 64-160 tokens: 200 us against 157).
  __device__ __forceinline__ void dump(const PageMath&, float* acc_at, v2f* ml_at, bool bad, int tid) {
    const int lane = tid & 63;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      auto meet = [&](auto swap, auto& from, auto& to) __attribute__((always_inline)) {
        constexpr int n = sizeof(to) / sizeof(float);
        // (the second copies opaque: two results of a swap of one value with itself have been
        // seen folded into one)
        float m0 = m[h], m1 = opaque(m0), l0 = l[h], l1 = opaque(l0);
        swap(m0, m1);
        swap(l0, l1);
        const float M = fmaxf(m0, m1);
        const float Mref = (M == kNegInf) ? 0.0f : M;
        const float ca = ex2(m0 - Mref);
        const float cb = ex2(m1 - Mref);
        l[h] = __builtin_fmaf(cb, l1, ca * l0);
        m[h] = M;
#pragma unroll
        for (int k = 0; k < n; ++k) {
          float x = from[k], y = from[k + n];
          swap(x, y);
          to[k] = __builtin_fmaf(cb, y, ca * x);
        }
      };
      float half[4], quarter[2];
      meet([](float& a, float& b) { swap_rows<16>(a, b); }, acc[h], half);
      meet([](float& a, float& b) { swap_rows<32>(a, b); }, half, quarter);
      const int at = (lane & 15) * 8 + ((lane >> 4) & 1) * 4 + (lane >> 5) * 2;
      *reinterpret_cast<v2f*>(acc_at + h * kHeadPitch + at) = v2f{quarter[0], quarter[1]};
    }
    if (lane == 0) {  // as single floats: from a pair, the compiler loads m[h] and its neighbour as one and spills both
      float* to = reinterpret_cast<float*>(ml_at);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        to[2 * h] = m[h];
        to[2 * h + 1] = bad ? -1.0f : l[h];
      }
    }
  }
};

template <int G>
constexpr bool on_matrix_cores() { return G >= 4; }
template <bool MATRIX, int G>
struct StateSel {
  typedef VectorState<G> type;
};
template <int G>
struct StateSel<true, G> {
  typedef MatrixState<G> type;
};
template <int G>
using State = typename StateSel<on_matrix_cores<G>(), G>::type;

// The staged pages of W waves; null where none are staged.
template <int G, int W>
__device__ __forceinline__ v4u* task_stage() {
  if constexpr (on_matrix_cores<G>()) return kv_stage<W>();
  else return nullptr;
}

// A task body runs in three phases, so that the one-launch route can issue a task's
// first loads before its plan is known (split_kernel):
//   begin(row, g, t0, t1)  loads Q and the wave's first 64 page ids
//   prime()                issues the loads of the wave's first two pages (waits for the ids)
//   run(plan, lds, stage)  the page loop (pages staged at `stage`), then the wave states in
//                          `lds` (finish_task and the fused route combine them into the
//                          task's partial state)
// covers(row, g, t0, t1) tells whether a begun task read exactly what task (row, g, t0,
// t1) reads in those phases: the same row, head and first token and the same page
// count. t1 itself only masks tokens of the last page, which run() applies.
// NH = 2 runs KV heads g and g + 1 of
// the same (row, split) together: each wave reads both heads of a page (adjacent
// 256-byte slices of every token), one page ahead per head, and keeps one softmax state
// per head. Each head's state goes through exactly the operations the one-head body
// applies to it, in the same order, so its result is bitwise that of the one-head body.
template <int G, int W, int NH = 1>
struct Task {
  static_assert(G <= 16, "heads fit the 16 MFMA columns");
  static_assert(NH == 1 || NH == 2, "one or two KV heads per task body");
  int row = 0, g = 0, t0 = 0, pg_end = 0, first = 0, npw = 0, ids = 0;  // npw = 0: no task begun
  bool bad = false;
  v4u q[NH][State<G>::kQ];
  // NH = 1: pages j (ka, va) and j + 1 (kb, vb); NH = 2: page j of head g (ka, va) and of
  // head g + 1 (kb, vb)
  v4u ka[4], va[4], kb[4], vb[4];

  __device__ __forceinline__ void begin(const DecodeArgs& a, int row_, int g_, int t0_, int t1_) {
    row = row_;
    g = g_;
    t0 = t0_;
    pg_end = uniform((t1_ + P - 1) / P);
    const int lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6);
    first = uniform(t0 / P + wave);
    npw = uniform(first < pg_end ? (pg_end - first + W - 1) / W : 0);
    bad = false;
    // Q of the NH * G query heads through one buffer descriptor, with no branch, so that the
    // page-id load below need not wait for it
    const __amdgpu_buffer_rsrc_t q_rsrc = page_rsrc(a.q + ((size_t)row * a.Hq + (size_t)g * G) * D, NH * G * D * 2);
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) State<G>::load_q(q[hh], q_rsrc, hh * G * D * 2, threadIdx.x);
    ids = lane < npw ? a.block_table[(size_t)row * a.max_pages_per_row + first + lane * W] : 0;
  }

  __device__ __forceinline__ bool covers(int row_, int g_, int t0_, int t1_) const {
    return row_ == row && g_ == g && t0_ == t0 && (t1_ + P - 1) / P == pg_end;
  }

  __device__ __forceinline__ void issue(const DecodeArgs& a, v4u (&kr)[4], v4u (&vr)[4], int j, bool live,
                                        int hh = 0) {
    issue_page(a, kr, vr, __builtin_amdgcn_readlane(ids, j), live, hh);
  }
  __device__ __forceinline__ void issue_page(const DecodeArgs& a, v4u (&kr)[4], v4u (&vr)[4], int phys, bool live,
                                             int hh = 0) {
    const int lane = threadIdx.x & 63;
    const int grp = lane >> 4;
    const int col = lane & 15;
    const size_t tok_stride = (size_t)a.Hkv * D;  // halves between consecutive tokens
    const size_t page_stride = (size_t)P * tok_stride;
    const int tok_b = (int)(tok_stride * 2);
    const int kv_off = grp * tok_b + (g + hh) * D * 2 + col * 16;  // + 4 i tok_b (K and V alike)
    const bool ok = phys >= 0 && phys < a.num_pages;
    bad |= live && !ok;
    const int page_bytes = uniform(live ? (int)(page_stride * 2) : 0);
    phys = uniform(live && ok ? phys : 0);
    const __amdgpu_buffer_rsrc_t kr_rsrc = page_rsrc(a.k + (size_t)phys * page_stride, page_bytes);
    const __amdgpu_buffer_rsrc_t vr_rsrc = page_rsrc(a.v + (size_t)phys * page_stride, page_bytes);
#pragma unroll
    for (int i = 0; i < 4; ++i) kr[i] = __builtin_amdgcn_raw_buffer_load_b128(kr_rsrc, kv_off, i * 4 * tok_b, kKvPolicy);
#pragma unroll
    for (int i = 0; i < 4; ++i) vr[i] = __builtin_amdgcn_raw_buffer_load_b128(vr_rsrc, kv_off, i * 4 * tok_b, kKvPolicy);
  }

  // Both issues are unconditional (pages past the wave's count are not live), so every
  // path out of prime() has waited for the id load and issued the same loads, and the
  // page loop's wait counts stay exact.
  __device__ __forceinline__ void prime(const DecodeArgs& a) {
    if constexpr (NH == 1) {
      issue(a, ka, va, 0, npw > 0);
      issue(a, kb, vb, 1, npw > 1);
    } else {
      issue(a, ka, va, 0, npw > 0, 0);
      issue(a, kb, vb, 0, npw > 0, 1);
    }
  }

  template <typename PlanView>
  __device__ __forceinline__ void run(const DecodeArgs& a, PlanView& plan, float* lds, v4u* stage) {
    v2f* lds_ml = state_ml<G, W, NH>(lds);
    float* lds_acc = state_acc<G, W, NH>(lds);
    const int lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6);
    State<G> st[NH];
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) st[hh].reset();
    PageMath pm;
    if constexpr (on_matrix_cores<G>()) pm.init(stage + wave * kStageUnits);

    // One page of head hh into its state, whose parts are arguments of their own: reached through
    // the closure alone, the compiler keeps a second copy of acc across the loop (20 registers).
    auto consume = [&](v4u (&kr)[4], v4u (&vr)[4], int k, int hh, auto& m, auto& l, auto& acc) __attribute__((always_inline)) {
      const int pg = first + k * W;
      const int t1 = pg == pg_end - 1 ? plan.last_t1() : pg_end * P;  // pages before the last are whole
      if constexpr (on_matrix_cores<G>()) {
        pm.stage_k(kr);
        const v4f sc = pm.scores(q[hh]);
        pm.stage_v(vr, pg * P, t1);
        pm.accumulate(sc, a.scale_log2, pg * P, t1, m, l, acc);
      } else {
        auto sc = st[hh].scores(q[hh], kr, a.scale_log2);
        st[hh].accumulate(sc, vr, pg * P, t1);
      }
    };

    bool dropped = false;
    for (int k0 = 0; k0 < npw && !dropped; k0 += 64) {
      const int n = min(64, npw - k0);
      if constexpr (NH == 1) {
        if (k0 > 0) {  // begin() and prime() did this for the first id block
          ids = (k0 + lane < npw) ? a.block_table[(size_t)row * a.max_pages_per_row + first + (k0 + lane) * W] : 0;
          issue(a, ka, va, 0, true);
          issue(a, kb, vb, 1, n > 1);
        }
        // pages j (ka) and j + 1 (kb) are in flight at the top of each iteration
        int j = 0;
        for (; j + 2 < n; j += 2) {
          if ((dropped = plan.dropped())) break;
          consume(ka, va, k0 + j, 0, st[0].m, st[0].l, st[0].acc);
          issue(a, ka, va, j + 2, true);
          consume(kb, vb, k0 + j + 1, 0, st[0].m, st[0].l, st[0].acc);
          issue(a, kb, vb, (j + 3) & 63, j + 3 < n);
        }
        if (dropped) break;
        consume(ka, va, k0 + j, 0, st[0].m, st[0].l, st[0].acc);
        if (j + 1 < n) consume(kb, vb, k0 + j + 1, 0, st[0].m, st[0].l, st[0].acc);
      } else {
        if (k0 > 0) {
          ids = (k0 + lane < npw) ? a.block_table[(size_t)row * a.max_pages_per_row + first + (k0 + lane) * W] : 0;
          issue(a, ka, va, 0, true, 0);
          issue(a, kb, vb, 0, true, 1);
        }
        // page j of both heads is in flight at the top of each iteration
        int j = 0;
        for (; j + 1 < n; ++j) {
          if ((dropped = plan.dropped())) break;
          consume(ka, va, k0 + j, 0, st[0].m, st[0].l, st[0].acc);
          issue(a, ka, va, j + 1, true, 0);
          consume(kb, vb, k0 + j, NH - 1, st[NH - 1].m, st[NH - 1].l, st[NH - 1].acc);
          issue(a, kb, vb, j + 1, true, 1);
        }
        if (dropped) break;
        consume(ka, va, k0 + j, 0, st[0].m, st[0].l, st[0].acc);
        consume(kb, vb, k0 + j, NH - 1, st[NH - 1].m, st[NH - 1].l, st[NH - 1].acc);
      }
    }

#pragma unroll
    for (int hh = 0; hh < NH; ++hh)
      st[hh].dump(pm, lds_acc + (hh * W + wave) * G * kHeadPitch, lds_ml + (hh * W + wave) * G, bad, threadIdx.x);
    __syncthreads();
  }
};

// What a task body's run() needs from the plan. KnownTask: the task is the plan's.
struct KnownTask {
  int t1;
  __device__ __forceinline__ int last_t1() const { return t1; }
  __device__ __forceinline__ bool dropped() const { return false; }
};

template <int G, int W, bool COHERENT, int NH = 1>
__device__ __forceinline__ void run_split_task(const DecodeArgs& a, int row, int g, int t0, int t1, int slot,
                                               float* lds) {
  Task<G, W, NH> body;
  body.begin(a, row, g, t0, t1);
  body.prime(a);
  KnownTask known{t1};
  body.run(a, known, lds, task_stage<G, W>());
  finish_task<G, W, COHERENT, NH>(a, slot, lds, nullptr, threadIdx.x);
}

template <int G>
__device__ __forceinline__ void write_neutral(const DecodeArgs& a, int slot) {
  constexpr int SF = slot_floats<G>();
  const __amdgpu_buffer_rsrc_t pr = slots_rsrc(a, SF * 4);
  for (int e = threadIdx.x; e < SF; e += blockDim.x)
    st_state<false>(pr, (slot * SF + e) * 4, (e >= G * D && e < G * D + 2 * G && (e - G * D) % 2 == 0) ? kNegInf : 0.0f);
}

template <int G>
__device__ __forceinline__ void zero_row(const DecodeArgs& a, int row) {
  uint32_t* o = reinterpret_cast<uint32_t*>(a.out + (size_t)row * a.Hq * D);
  for (int e = threadIdx.x; e < a.Hq * D / 2; e += blockDim.x) o[e] = 0u;
}

// ---------------------------------------------------------------------------------
// Planner (Sec. 3.4), run by one workgroup. Lengths are validated; each row gets
// nsplit_i splits (policy 0: min(S, tiles_i) with S from the active batch size;
// policy 1: min(split_max, ceil(tiles_i / Q)) with the smallest tile quota Q whose task
// count fits target_tasks); split_offsets is their exclusive scan, and task
// k = (split_offsets[i] + s) * Hkv + g covers the balanced tile range
// [floor(s*tiles/nsplit), floor((s+1)*tiles/nsplit)) of row i.
constexpr int kPlanThreads = 256;

// inclusive prefix sum over the 64 lanes of a wave
// Wave-wide scans on DPP: row shifts build prefixes inside each 16-lane row, the row
// broadcasts 15 and 31 carry them across rows. Lanes without a source read 0, the
// identity of the sums and of the max over non-negative values used here. The whole
// wave must be active.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int dpp_i32(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}

template <typename Op>
__device__ __forceinline__ int wave_scan_i32(int x, Op op) {
  x = op(x, dpp_i32<0x111>(x));  // row_shr:1
  x = op(x, dpp_i32<0x112>(x));  // row_shr:2
  x = op(x, dpp_i32<0x114>(x));  // row_shr:4
  x = op(x, dpp_i32<0x118>(x));  // row_shr:8
  x = op(x, dpp_i32<0x142, 0xA>(x));  // row_bcast:15 into rows 1 and 3
  x = op(x, dpp_i32<0x143, 0xC>(x));  // row_bcast:31 into rows 2 and 3
  return x;
}

__device__ __forceinline__ int wave_incl_scan(int x) {
  return wave_scan_i32(x, [](int u, int v) { return u + v; });
}

__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_incl_scan(x), 63); }

__device__ __forceinline__ int wave_max(int x) {  // x >= 0
  return __builtin_amdgcn_readlane(wave_scan_i32(x, [](int u, int v) { return u > v ? u : v; }), 63);
}

template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ long long dpp_i64(long long x) {
  const int lo = dpp_i32<CTRL, ROWS>((int)x);
  const int hi = dpp_i32<CTRL, ROWS>((int)(x >> 32));
  return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ long long wave_sum64(long long x) {
  x += dpp_i64<0x111>(x);
  x += dpp_i64<0x112>(x);
  x += dpp_i64<0x114>(x);
  x += dpp_i64<0x118>(x);
  x += dpp_i64<0x142, 0xA>(x);
  x += dpp_i64<0x143, 0xC>(x);
  const unsigned lo = __builtin_amdgcn_readlane((int)x, 63);
  const unsigned hi = __builtin_amdgcn_readlane((int)(x >> 32), 63);
  return (long long)(((unsigned long long)hi << 32) | lo);
}

// Plan outputs read in the same kernel by other workgroups go out with agent-scope
// stores (see the partial-state slots) and are read back with agent-scope loads.
template <bool COHERENT>
__device__ __forceinline__ void st_i32(int* p, int v) {
  if (COHERENT) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
template <bool COHERENT>
__device__ __forceinline__ int ld_i32(const int* p) {
  if (COHERENT) return __hip_atomic_load(const_cast<int*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}

struct PlanLds {
  int* len;        // [B]
  int* off;        // [B + 1]
  int* wave;       // [NT / 64]
  long long* w64;  // [2 * NT / 64]
  int* wmax;       // [NT / 64]
  int* cum = nullptr;  // [B + 1] row weights' prefix sums (plan_range_begin), when wanted
};

constexpr int kCandidateRows = 16;  // batches up to this size test several quotas per step

// Steps 1-3 for a batch of at most 64 rows and no block-table check: lane i of wave 0
// holds row i, every batch quantity is a wave reduction and split_offsets a wave scan,
// so the workgroup meets a single barrier. Same results as the general path below.
// `n` is seq_lens[lane] (0 for lanes >= B), loaded by the caller.
__device__ __forceinline__ bool wave_plan(const PlanArgs& a) { return a.B <= 64 && !a.block_table; }

// seq_lens[lane] (0 for lanes >= B). Issued ahead of the wave's other loads, so that the
// planner waits for nothing else. (Scalar loads, 16 lengths at a time, took a round trip per
// group: 4.6 us for 60 rows, against 1.4.)
__device__ __forceinline__ int wave_plan_len(const PlanArgs& a) {
  const int lane = threadIdx.x & 63;
  return lane < a.B ? a.seq_lens[lane] : 0;
}

__device__ __forceinline__ void plan_compute_wave(const PlanArgs& a, const PlanLds& L, bool report, int n) {
  const int lane = threadIdx.x & 63;
  const int B = a.B;
  const int T = a.tile_tokens;
  const int cap = a.max_pages_per_row * a.page_size;
  if (n < 0 || n > cap) {
    if (report) atomicOr(a.err, (unsigned)PKV_DEVERR_SEQ_LEN);
    n = 0;
  }
  const int tiles = n > 0 ? (n - 1) / T + 1 : 0;
  const int active = __popcll(__ballot(tiles > 0));
  int nsplit;
  if (a.policy == 0) {
    // 32-bit: denom <= B * Hkv and target + denom - 1 < 2^32
    const unsigned denom = (unsigned)(active > 0 ? active : 1) * (unsigned)a.Hkv;
    const int s0 = (int)(((unsigned)a.target_tasks + denom - 1u) / denom);
    const int S = s0 < a.split_min ? a.split_min : (s0 > a.split_max ? a.split_max : s0);
    nsplit = min(tiles, S);
  } else {
    // the quota search of the general path; same result, found in fewer steps
    const int per_head = a.target_tasks / a.Hkv;
    const int max_tiles = wave_max(tiles);
    int hi = max(1, max_tiles);
    if (per_head > active) {
      const unsigned room = (unsigned)(per_head - active);
      if (max_tiles < (1 << 25)) {  // the total fits in 31 bits
        const unsigned total = (unsigned)wave_sum(tiles);
        if ((unsigned long long)total < (unsigned long long)hi * room) hi = max(1u, (total + room - 1u) / room);
      } else {
        const long long total = wave_sum64(tiles);
        if (total < (long long)hi * room) hi = (int)max(1LL, (total + room - 1) / (long long)room);
      }
    }
    auto nsplit_of = [&](int t, int q) { return t > 0 ? min(a.split_max, (t - 1) / q + 1) : 0; };
    int lo = 1;
    if (B <= kCandidateRows) {
      // R = B rounded up to a power of two; lane (c, i) = (lane / R, lane % R) counts row
      // i's splits at the c-th of 64 / R candidate quotas lo + (c + 1) * step - 1, DPP
      // row shifts sum each aligned group of R lanes into its last lane, and the first
      // candidate that fits narrows [lo, hi] to one step (the count only falls as the
      // quota grows). Rows live in lanes 0..15.
      const int R = B <= 1 ? 1 : (B <= 2 ? 2 : (B <= 4 ? 4 : (B <= 8 ? 8 : 16)));
      const int shift = R == 1 ? 0 : (R == 2 ? 1 : (R == 4 ? 2 : (R == 8 ? 3 : 4)));
      const int ncand = 64 >> shift;
      const int ti = __shfl(tiles, lane & (R - 1));
      const int c = lane >> shift;
      while (lo < hi) {
        const int step = (hi - lo + ncand) / ncand;
        const int q = min(hi, lo + (c + 1) * step - 1);
        int f = ti > 0 ? min(a.split_max, (ti - 1) / q + 1) : 0;
        if (R > 1) f += dpp_i32<0x111>(f);  // row_shr:1
        if (R > 2) f += dpp_i32<0x112>(f);  // row_shr:2
        if (R > 4) f += dpp_i32<0x114>(f);  // row_shr:4
        if (R > 8) f += dpp_i32<0x118>(f);  // row_shr:8
        const unsigned long long fit = __ballot((lane & (R - 1)) == R - 1 && f <= per_head);
        if (fit == 0) {  // nothing up to hi fits: one split per row
          lo = hi;
          break;
        }
        const int j = (__ffsll((unsigned long long)fit) - 1) >> shift;
        const int qj = min(hi, lo + (j + 1) * step - 1);
        if (j > 0) lo = min(hi, lo + j * step - 1) + 1;
        hi = qj;
      }
    } else {
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (wave_sum(nsplit_of(tiles, mid)) <= per_head) hi = mid; else lo = mid + 1;
      }
    }
    nsplit = nsplit_of(tiles, lo);
  }
  const int incl = wave_incl_scan(nsplit);
  if (lane < B) {
    L.len[lane] = n;
    L.off[lane + 1] = incl;
  }
  if (lane == 0) L.off[0] = 0;
  if (L.cum) {
    const int wincl = wave_incl_scan(nsplit + tiles);
    if (lane < B) L.cum[lane + 1] = wincl;
    if (lane == 0) L.cum[0] = 0;
  }
}

// Steps 1-3: validated lengths in L.len, split_offsets in L.off; returns the task count
// (every thread). `report` selects the workgroup that raises device error bits.
// Task count of a plan formed by plan_compute_wave (after the workgroup barrier).
__device__ __forceinline__ int plan_wave_tasks(const PlanArgs& a, const PlanLds& L, bool report) {
  long long nt = (long long)L.off[a.B] * a.Hkv;
  if (nt > a.max_tasks) {  // excluded by host validation; never write past the buffer
    if (report && threadIdx.x == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_SEQ_LEN);
    nt = 0;
  }
  return (int)nt;
}

// n_first: seq_lens[threadIdx.x], when the caller has loaded it (has_first; the general path).
template <int NT>
__device__ __forceinline__ int plan_compute(const PlanArgs& a, const PlanLds& L, bool report, bool has_first = false,
                                            int n_first = 0) {
  if (wave_plan(a)) {
    if (threadIdx.x < 64) plan_compute_wave(a, L, report, wave_plan_len(a));
    __syncthreads();
    return plan_wave_tasks(a, L, report);
  }
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int B = a.B;
  const int cap = a.max_pages_per_row * a.page_size;
  const int T = a.tile_tokens;
  // 1. validated lengths; each thread owns the contiguous rows [r0, r0 + per)
  const int per = (B + NT - 1) / NT;
  const int r0 = tid * per;
  for (int i = r0; i < r0 + per && i < B; ++i) {
    int n = has_first && per == 1 ? n_first : a.seq_lens[i];
    if (n < 0 || n > cap) {
      if (report) atomicOr(a.err, (unsigned)PKV_DEVERR_SEQ_LEN);
      n = 0;
    }
    L.len[i] = n;
  }
  if (a.block_table) {  // optional: drop rows whose used block-table entries are out of range
    __syncthreads();
    const long long total = (long long)B * a.max_pages_per_row;
    for (long long k = tid; k < total; k += NT) {
      const int i = (int)(k / a.max_pages_per_row);
      const int jp = (int)(k % a.max_pages_per_row);
      if (jp < (L.len[i] + a.page_size - 1) / a.page_size) {
        const int phys = a.block_table[k];
        if (phys < 0 || phys >= a.num_pages) {
          if (report) atomicOr(a.err, (unsigned)PKV_DEVERR_PAGE_ID);
          L.len[i] = 0;  // benign race: every writer stores 0
        }
      }
    }
    __syncthreads();
  }
  int act = 0;
  long long tsum = 0;
  int tmax = 0;
  for (int i = r0; i < r0 + per && i < B; ++i) {
    const int tiles = (L.len[i] + T - 1) / T;
    act += tiles > 0;
    tsum += tiles;
    tmax = max(tmax, tiles);
  }
  // 2. batch-level quantities: active rows, total and largest tile count
  act = wave_sum(act);
  tsum = wave_sum64(tsum);
  tmax = wave_max(tmax);
  if (lane == 0) {
    L.wave[wave] = act;
    L.w64[wave] = tsum;
    L.wmax[wave] = tmax;
  }
  __syncthreads();
  int active = 0;
  long long total_tiles = 0;
  int max_tiles = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    active += L.wave[w];
    total_tiles += L.w64[w];
    max_tiles = max(max_tiles, L.wmax[w]);
  }
  // policy 0: one split count S from the active batch size (Sec. 3.5);
  // policy 1: a tile quota Q per split from the batch's total work
  int S = 0, Q = 1;
  if (a.policy == 0) {
    const long long denom = (long long)(active > 0 ? active : 1) * a.Hkv;
    const long long s0 = (a.target_tasks + denom - 1) / denom;
    S = (int)(s0 < a.split_min ? a.split_min : (s0 > a.split_max ? a.split_max : s0));
  } else {
    // smallest Q in [1, max_tiles] with Hkv * sum_i min(split_max, ceil(tiles_i / Q))
    // <= target_tasks (the count only falls as Q grows), else max_tiles. Bisection;
    // the upper end starts at ceil(total / (target/Hkv - active)) when that bounds it.
    // Counts fit in 32 bits: B * split_max * Hkv is bounded by the task buffer's size.
    const int per_head = a.target_tasks / a.Hkv;
    int hi = max(1, max_tiles);
    if (per_head > active)
      hi = (int)min((long long)hi, max(1LL, (total_tiles + per_head - active - 1) / (per_head - active)));
    int lo = 1;
    auto nsplit_at = [&](int t, int q) { return t > 0 ? min(a.split_max, (t + q - 1) / q) : 0; };
    __syncthreads();  // every wave has read the batch sums in L.w64
    if (B <= 64) {  // one row per lane of wave 0: search without barriers
      if (wave == 0) {
        const int t = lane < B ? (L.len[lane] + T - 1) / T : 0;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (wave_sum(nsplit_at(t, mid)) <= per_head) hi = mid; else lo = mid + 1;
        }
        if (lane == 0) L.wave[0] = lo;
      }
      __syncthreads();
      Q = L.wave[0];
    } else {
      int buf = 0;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        int c = 0;
        for (int i = r0; i < r0 + per && i < B; ++i) c += nsplit_at((L.len[i] + T - 1) / T, mid);
        c = wave_sum(c);
        int* red = reinterpret_cast<int*>(L.w64) + buf * NW;  // two buffers: one barrier per round
        if (lane == 0) red[wave] = c;
        __syncthreads();
        int tot = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) tot += red[w];
        if (tot <= per_head) hi = mid; else lo = mid + 1;
        buf ^= 1;
      }
      Q = lo;
    }
  }
  auto row_nsplit = [&](int n) -> int {
    const int tiles = (n + T - 1) / T;
    if (a.policy == 0) return min(tiles, S);
    return min(a.split_max, (tiles + Q - 1) / Q);
  };
  // 3. exclusive scan of nsplit over rows -> split_offsets
  int local = 0;
  for (int i = r0; i < r0 + per && i < B; ++i) local += row_nsplit(L.len[i]);
  const int incl = wave_incl_scan(local);
  __syncthreads();  // every wave has read L.wave
  if (lane == 63) L.wave[wave] = incl;
  __syncthreads();
  int run = incl - local;
  for (int w = 0; w < wave; ++w) run += L.wave[w];
  for (int i = r0; i < r0 + per && i < B; ++i) {
    L.off[i] = run;
    run += row_nsplit(L.len[i]);
  }
  if (tid == NT - 1) L.off[B] = run;
  if (L.cum) {
    int lw = 0;
    for (int i = r0; i < r0 + per && i < B; ++i) lw += (L.len[i] + T - 1) / T + row_nsplit(L.len[i]);
    const int wincl = wave_incl_scan(lw);
    __syncthreads();  // every wave has read L.wave
    if (lane == 63) L.wave[wave] = wincl;
    __syncthreads();
    int at = wincl - lw;
    for (int w = 0; w < wave; ++w) at += L.wave[w];
    for (int i = r0; i < r0 + per && i < B; ++i) {
      L.cum[i] = at;
      at += (L.len[i] + T - 1) / T + row_nsplit(L.len[i]);
    }
    if (tid == NT - 1) L.cum[B] = at;
  }
  __syncthreads();
  long long ntasks = (long long)L.off[B] * a.Hkv;
  if (ntasks > a.max_tasks) {  // excluded by host validation; never write past the buffer
    if (report && tid == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_SEQ_LEN);
    ntasks = 0;
  }
  return (int)ntasks;
}

// Step 4: task k = (split_offsets[i] + s) * Hkv + g covers the balanced tile range s of
// row i: [floor(s*tiles/nsplit), floor((s+1)*tiles/nsplit)) tiles.
struct TaskRec {
  int row, g, split, t0, t1;
};

__device__ __forceinline__ int plan_row(const PlanLds& L, int B, int sr) {  // largest i with off[i] <= sr
  int lo = 0, hi = B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (L.off[mid] <= sr) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ TaskRec plan_task(const PlanArgs& a, const PlanLds& L, int k) {
  const int sr = (unsigned)k / (unsigned)a.Hkv;
  const int lo = plan_row(L, a.B, sr);
  const int T = a.tile_tokens;
  const int sp = sr - L.off[lo];
  const int n = L.len[lo];
  const int tiles = (n + T - 1) / T;
  const int ns = L.off[lo + 1] - L.off[lo];
  const int b0 = split_bound(sp, tiles, ns);
  const int b1 = split_bound(sp + 1, tiles, ns);
  return TaskRec{lo, k - sr * a.Hkv, sp, b0 * T, min(b1 * T, n)};
}

// Units `from` .. count (per_split units a split: tasks, or pairs of them) cut into `parts`
// contiguous ranges of about the same weight: the first unit of range w. A row's weight, its
// tiles plus one per split, is spread evenly over its units, and a bound is a whole number of
// units, so that neighbours agree on their common bound.
__device__ __forceinline__ int plan_range_begin(const PlanArgs& a, const PlanLds& L, int per_split, int w, int parts,
                                                int from, int count) {
  if (w <= 0) return from;
  if (w >= parts) return count;
  auto row_of = [&](const int* v, int x) {  // largest i with v[i] <= x
    int lo = 0, hi = a.B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (v[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
  };
  const float ps = (float)per_split;
  const int r0 = row_of(L.off, from / per_split);  // the weight in front of task `from`
  const int n0 = L.off[r0 + 1] - L.off[r0];
  const float w0 = (float)L.cum[r0] + (float)(L.cum[r0 + 1] - L.cum[r0]) * ((float)(from - L.off[r0] * per_split) / (ps * (float)max(n0, 1)));
  const float x = w0 + ((float)L.cum[a.B] - w0) * ((float)w / (float)parts);
  const int r = row_of(L.cum, (int)x);
  const int cnt = (L.off[r + 1] - L.off[r]) * per_split, wr = max(1, L.cum[r + 1] - L.cum[r]);
  const int k = (int)((x - (float)L.cum[r]) / (float)wr * (float)cnt + 0.5f);
  return min(count, max(from, L.off[r] * per_split + min(max(k, 0), cnt)));
}

// The one-launch route's speculative run of the hinted task (row hr, KV head hg, first
// token h0, h_pages pages) while wave 0 plans. Once the plan is in LDS (flag `ready`),
// the verdict is the plan's t1 for this workgroup's first task (index `task`) if that
// task is the hinted one (same row, KV head, first token and page count), else -1: the
// run is dropped. Each wave forms it once, at the first check after the plan is in LDS
// (in the page loop, overlapped with its loads). dropped() looks without waiting;
// last_t1() waits for the plan and returns the verdict.
struct SpecTask {
  const PlanArgs& pa;
  PlanLds PL;
  const int* ready;
  int task, hr, hg, h0, h_pages;
  int verdict = -2;  // -2: plan not seen yet
  __device__ __forceinline__ void judge() {
    verdict = -1;
    if (task < plan_wave_tasks(pa, PL, false)) {
      const TaskRec r = plan_task(pa, PL, task);
      if (r.row == hr && r.g == hg && r.t0 == h0 && (r.t1 + P - 1) / P == h_pages) verdict = r.t1;
    }
  }
  __device__ __forceinline__ bool dropped() {
    if (verdict == -2 && __hip_atomic_load(ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != 0) judge();
    return verdict == -1;
  }
  __device__ __forceinline__ int last_t1() {
    if (verdict == -2) {
      while (__hip_atomic_load(ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0) __builtin_amdgcn_s_sleep(1);
      judge();
    }
    return verdict;
  }
};

template <int NT>
__device__ __forceinline__ void plan_write_offsets(const PlanArgs& a, const PlanLds& L, int ntasks) {
  for (int i = threadIdx.x; i <= a.B; i += NT) a.split_offsets[i] = L.off[i];
  if (threadIdx.x == 0) *a.num_tasks = ntasks;
}

// The planner's outputs: split_offsets, num_tasks, the task list and zeroed completion
// counters.
template <int NT, bool COHERENT>
__device__ __forceinline__ void plan_write(const PlanArgs& a, const PlanLds& L, int ntasks, bool zero_counters) {
  const int tid = threadIdx.x;
  for (int i = tid; i <= a.B; i += NT) st_i32<COHERENT>(a.split_offsets + i, L.off[i]);
  if (tid == 0) st_i32<COHERENT>(a.num_tasks, ntasks);
  for (int k = tid; k < ntasks; k += NT) {
    const TaskRec r = plan_task(a, L, k);
    int* t = reinterpret_cast<int*>(a.tasks + k);
    st_i32<COHERENT>(t + 0, r.row);
    st_i32<COHERENT>(t + 1, r.g);
    st_i32<COHERENT>(t + 2, r.split);
    st_i32<COHERENT>(t + 3, r.t0);
    st_i32<COHERENT>(t + 4, r.t1);
  }
  if (zero_counters)
    for (int k = tid; k < a.B * a.Hkv; k += NT) st_i32<COHERENT>(a.counters + k, 0);
}

template <int NT, bool COHERENT>
__device__ __forceinline__ void plan_body(const PlanArgs& a, const PlanLds& L) {
  const int ntasks = plan_compute<NT>(a, L, true);
  plan_write<NT, COHERENT>(a, L, ntasks, true);
}

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(PlanArgs a) {
  __shared__ int s_len[kMaxPlanBatch];
  __shared__ int s_off[kMaxPlanBatch + 1];
  __shared__ int s_wave[kPlanThreads / 64];
  __shared__ long long s_w64[2 * kPlanThreads / 64];
  __shared__ int s_wmax[kPlanThreads / 64];
  plan_body<kPlanThreads, false>(a, PlanLds{s_len, s_off, s_wave, s_w64, s_wmax});
}

// Workqueue split kernel. FUSED: the last split of each (row, KV head) to finish merges
// all of that pair's splits in split order (Sec. 3.4, atomic completion counter).
// PLAN: the planner runs inside the launch (see below).
// NH = 2 (with PLAN and FUSED): a workgroup runs tasks 2p and 2p + 1 together, which the
// plan's order makes KV heads g and g + 1 (g even) of one (row, split); one completion
// counter per (row, head pair) counts them as one, and its last arriver merges both
// heads. Spreading every workgroup's reads over two heads' slices of each token
// balances the workgroups: on MI355X one workgroup streaming a single head's slices
// runs up to ~20% slower or faster than another, depending on the slices' offset.

template <int G, int W, bool FUSED, bool PLAN, int NH = 1>
__global__ __launch_bounds__(W * 64) void split_kernel(DecodeArgs a) {
  static_assert(NH == 1 || (NH == 2 && FUSED && PLAN), "head pairs run on the one-launch route");
  __shared__ float lds[lds_floats<G, W, NH>()];
  __shared__ float lds_merge[FUSED ? merge_lds_floats<G, NH, W * 64>() : 1];
  __shared__ int lds_last;
  __shared__ int p_len[PLAN ? kMaxFusedPlanBatch : 1];
  __shared__ int p_off[PLAN ? kMaxFusedPlanBatch + 1 : 1];
  __shared__ int p_wave[W];
  __shared__ long long p_w64[2 * W];
  __shared__ int p_wmax[W];
  // PLAN: every workgroup runs the planner's arithmetic on seq_lens and takes its tasks
  // from the result; workgroup 0 also writes the task list. The completion counters are
  // zero at launch (pkv_workspace_init sets them, every completed launch restores them).
  const PlanLds PL{p_len, p_off, p_wave, p_w64, p_wmax};
  // Bring the argument block's pointer lines and the grid size into the scalar cache at
  // the start, so later scalar loads of them do not wait on memory (after the planner,
  // and at the end of the last task).
  asm volatile("" ::"s"(a.q), "s"(a.partials), "s"(gridDim.x));
  Task<G, W, NH> body;
  bool begun = false;  // the workgroup's body holds a task begun before the plan
  int plan_ntasks = 0;
  __shared__ int plan_ready;  // wave planner: set once wave 0 has put the plan in LDS
  bool spec_kept = false;     // the speculative run was this workgroup's first task
  int hr = 0, hg = 0, h0 = 0, h1 = 0;  // the hinted task (h1: the plan's t1 once kept)
  // The speculative run is for one-head workgroups: with KV-head pairs its extra live
  // state pushes the kernel past 256 registers per lane (spills in the page loop), so a
  // pair's hinted task is only begun and primed.
  constexpr bool kSpecRun = NH == 1;
  if (PLAN) {
    if (wave_plan(a.plan)) {
      // Speculative start. Between decode steps a plan rarely changes (lengths grow by a
      // token), so while wave 0 runs the planner, each wave begins, primes and runs the
      // task listed at this workgroup's index (NH = 2: the pair's first task, at twice
      // the index) in the task list left by the previous launch (the task it ran then):
      // a hint, read with agent-scope loads because workgroup 0 rewrites the list during
      // the launch. A record is used only if it names a task inside the batch's bounds
      // (the buffer may hold anything on the first call). Every page of the hinted task
      // but its last is read and accumulated without the plan: their tokens do not depend
      // on it. The wave that holds the last page waits there for the plan, which gives the
      // row's token count for its masking, and the run's result is kept only if the plan
      // gives this workgroup a task with the same row, KV head, first token and page
      // count; otherwise the task is run again from the start. Results never depend on
      // the hint. Wave 0's lengths go out first, one load for all rows (scalar loads in
      // groups took 4.6 us until the last had arrived, this 1.4), then the hint's.
      if (threadIdx.x == 0) plan_ready = 0;
      __syncthreads();
      const int n_raw = threadIdx.x < 64 ? wave_plan_len(a.plan) : 0;
      const bool has_hint = NH * (int)blockIdx.x < a.max_tasks;
      int hv[4] = {-1, -1, -1, -1};
      if (has_hint) {
        const int* tp = reinterpret_cast<const int*>(a.tasks + NH * (int)blockIdx.x);
        hv[0] = ld_i32<true>(tp + 0);
        hv[1] = ld_i32<true>(tp + 1);
        hv[2] = ld_i32<true>(tp + 3);
        hv[3] = ld_i32<true>(tp + 4);
      }
      hr = uniform(hv[0]), hg = uniform(hv[1]), h0 = uniform(hv[2]), h1 = uniform(hv[3]);
      if (has_hint && hr >= 0 && hr < a.B && hg >= 0 && hg % NH == 0 && hg + NH <= a.Hkv && h0 >= 0 && h1 > h0 &&
          h1 <= a.max_pages_per_row * P) {
        body.begin(a, hr, hg, h0, h1);
        begun = true;
      }
      if (threadIdx.x < 64) {
        plan_compute_wave(a.plan, PL, blockIdx.x == 0, n_raw);
        __hip_atomic_store(&plan_ready, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      body.prime(a);  // nothing to issue when no task was begun (npw = 0)
      if (begun && kSpecRun) {
        SpecTask spec{a.plan, PL, &plan_ready, NH * (int)blockIdx.x, hr, hg, h0, (h1 + P - 1) / P};
        body.run(a, spec, lds, task_stage<G, W>());
        // The run ended with a workgroup barrier: wave 0's plan is visible to every wave.
        // Every wave's verdict is the same; most waves formed it in the page loop, so a
        // kept run finishes with the hint's record and the plan's t1, no lookup.
        const int t1 = spec.last_t1();
        spec_kept = t1 >= 0;
        if (spec_kept) h1 = t1;
      } else {
        __syncthreads();
      }
      plan_ntasks = plan_wave_tasks(a.plan, PL, blockIdx.x == 0);
    } else {
      plan_ntasks = plan_compute<W * 64>(a.plan, PL, blockIdx.x == 0);
    }
    if (blockIdx.x == 0) plan_write<W * 64, true>(a.plan, PL, plan_ntasks, false);
  }
  // The first task record is fetched together with the task count (the grid never
  // exceeds max_tasks, so the record lies inside the task buffer even when unused).
  int rec[4];
  auto fetch = [&](int t) {
    if (PLAN) {
      const TaskRec r = plan_task(a.plan, PL, t);
      rec[0] = r.row;
      rec[1] = r.g;
      rec[2] = r.t0;
      rec[3] = r.t1;
    } else {
      const int* tp = reinterpret_cast<const int*>(a.tasks + t);
      rec[0] = tp[0];
      rec[1] = tp[1];
      rec[2] = tp[3];
      rec[3] = tp[4];
    }
  };
  if (spec_kept) {  // the plan's record of this workgroup's first task is the hint's
    rec[0] = hr;
    rec[1] = hg;
    rec[2] = h0;
    rec[3] = h1;
  } else if (!PLAN || NH * (int)blockIdx.x < plan_ntasks) {
    fetch(NH * (int)blockIdx.x);  // PLAN: only real tasks
  }
  int ntasks = PLAN ? plan_ntasks : uniform(*a.num_tasks);
  if (ntasks > a.max_tasks) ntasks = a.max_tasks;
  // The end of task t (KV heads g .. g + NH - 1 of `row`): its partial state from the
  // wave states in LDS; on the fused route, the completion count and the last
  // arriver's merge.
  auto finish = [&](int t, int row, int g) __attribute__((always_inline)) {
    if (!FUSED) {
      finish_task<G, W, false, NH>(a, t, lds, nullptr, threadIdx.x);
    } else {
      const int off = uniform(PLAN ? PL.off[row] : a.split_offsets[row]);
      int nsplit = uniform(PLAN ? PL.off[row + 1] : a.split_offsets[row + 1]) - off;
      if (off >= 0 && nsplit == 1 && (long long)(off + 1) * a.Hkv <= a.max_tasks) {  // the row's only split
        finish_task<G, W, true, NH>(a, t, lds, a.out + ((size_t)row * a.Hq + (size_t)g * G) * D, threadIdx.x);
        __syncthreads();
        return;
      }
      finish_task<G, W, true, NH>(a, t, lds, nullptr, threadIdx.x);
      if (off < 0 || nsplit < 1 || (long long)(off + nsplit) * a.Hkv > a.max_tasks) {
        if (threadIdx.x == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_TASK);
        nsplit = 0;  // never reached by the counter: no merge from inconsistent offsets
      }
      // Completion count (Sec. 3.4). The partial state went out with agent-scope
      // stores; each wave waits until they are acknowledged, then one thread counts.
      // The last arriver invalidates its caches before the merge reads (agent-scope
      // loads) the other splits' states.
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (threadIdx.x == 0) {
        const int prev = __hip_atomic_fetch_add(&a.counters[row * a.Hkv + g], 1, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
        lds_last = (prev == nsplit - 1);
        if (lds_last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
      __syncthreads();
      if (lds_last) {
        merge_group<G, W * 64, true, NH>(slots_rsrc(a, slot_floats<G>() * 4), off * a.Hkv + g, a.Hkv, nsplit,
                                         a.out + ((size_t)row * a.Hq + (size_t)g * G) * D, lds_merge);
        if (threadIdx.x == 0) a.counters[row * a.Hkv + g] = 0;
      }
    }
    __syncthreads();
  };
  // Task t (record in rec) on body `bd`, which holds a begun task when `keep`: the loads
  // it began are used if they cover task t, else the task is begun again.
  auto task = [&](Task<G, W, NH>& bd, int t, bool keep) __attribute__((always_inline)) {
    const int row = uniform(rec[0]), g = uniform(rec[1]);
    const int t0 = uniform(rec[2]), t1 = uniform(rec[3]);
    if (row < 0 || row >= a.B || g < 0 || g % NH != 0 || g + NH > a.Hkv || t0 < 0 || t1 <= t0 ||
        t1 > a.max_pages_per_row * P) {  // not a task of a valid plan: flag and skip
      if (threadIdx.x == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_TASK);
      return;
    }
    if (!(keep && bd.covers(row, g, t0, t1))) {
      bd.begin(a, row, g, t0, t1);
      bd.prime(a);
    }
    KnownTask known{t1};
    bd.run(a, known, lds, task_stage<G, W>());
    finish(t, row, g);
  };
  // The first task is the only one a speculative start can have begun (and run); later
  // tasks run on a body of their own, so the first body's registers are free after its
  // task. NH = 2: the plan's task count is Hkv times its split count, and Hkv is even.
  int t = NH * (int)blockIdx.x;
  if (t + NH <= ntasks) {
    if (spec_kept)
      finish(t, hr, hg);  // the speculative run was this task
    else
      task(body, t, begun && !kSpecRun);  // a begun task that has not run keeps its loads if they cover t
  }
  for (t += NH * gridDim.x; t + NH <= ntasks; t += NH * gridDim.x) {
    fetch(t);
    Task<G, W, NH> next;
    task(next, t, false);
  }
  if (FUSED) {  // rows without tasks: their output is zero
    for (int i = blockIdx.x; i < a.B; i += gridDim.x) {
      const bool empty = PLAN ? PL.off[i + 1] == PL.off[i] : a.split_offsets[i + 1] == a.split_offsets[i];
      if (empty) zero_row<G>(a, i);
    }
  }
}

// ---------------------------------------------------------------------------------
// Streaming route: launches with more tasks than workgroups.
//
// A task run by itself pays a chain of dependent memory round trips around its page reads
// (page ids, first pages, state store and its acknowledgement, completion counter, merge):
// about 8 us in which its compute unit reads little. Here a workgroup (one per compute unit,
// eight waves) runs its tasks as one stream of pages instead. A unit of the stream is a pair
// of tasks, KV heads g and g + 1 of one split (adjacent 256-byte slices of every token, which
// read faster than one head's). A wave keeps one page of each head in flight: it waits for
// one, stages it in LDS, at once issues the loads of its next page of that head, and computes
// from LDS (on the vector ALU the next K is issued after the scores, the next V after the
// sums). The page after a unit's last is the next unit's first, so the reads go on while a
// unit is combined, stored, counted and merged, and what a unit leaves behind rides on the
// waits of the ones after it: its state stores have been acknowledged when the second next
// unit's first page is there, its completion counter is bumped in that unit's epilogue, and
// the count is looked at two units later.
// Every task goes through exactly the operations of the one-task kernels in their order
// (eight waves taking its pages round-robin, the same combine and merge), so results are
// bitwise the same.
//
// Whether `tasks` tasks run as a stream of KV-head pairs, `slots` (one per compute unit)
// at a time, rather than on the one-task kernels. The stream goes through ceil(tasks / 2 slots)
// rounds of units of two tasks each, the one-task kernels through ceil(tasks / slots) rounds
// with a gap after each; an odd number of rounds leaves the stream half a round behind.
// - One head per workgroup as the alternative: two rounds are one of units (the layers of 16
//   rows 258 -> 253 us; at G = 8, whose units combine twice the states, 57 -> 59), three are
//   two (608 tasks: 106 against 119), and from four on the gaps decide (1024 tasks 149 -> 145,
//   62 -> 59 for short rows; G = 8: 51 -> 48 at 1024 tasks, 250 -> 155 at 8192).
// - KV-head pairs as the alternative (`paired`: the one-launch route at G < 8): they have the
//   same rounds and a shorter start, and win while rounds are few (1888 tasks 95.5 against
//   96.5, 1024 tasks 276 against 278); from eight tasks per slot on the gaps decide (3200
//   tasks 104 -> 101 and 59 -> 45 for short rows, 8192 tasks 175 -> 135).
template <typename T>
__host__ __device__ __forceinline__ bool stream_pays(int G, T tasks, int slots, bool paired) {
  if (paired) return tasks >= 8 * (T)slots;
  return tasks > 3 * (T)slots || (G < 8 && tasks > (T)slots && tasks <= 2 * (T)slots);  // rounds >= 4, or 2
}

constexpr int kStreamRecs = 32;  // unit records a workgroup holds in LDS

struct StreamRec {
  int row, g, t0, t1, off, ns;  // row < 0: not a task of a valid plan (skipped)
};

// A wave's pages of one unit: first + k * W for k < npw.
struct StreamSlice {
  int row, g, first, npw, pg_end, t1;
};
// In scalar registers (the compiler does not see by itself that a wave's slices are uniform).
__device__ __forceinline__ StreamSlice scalar(const StreamSlice& s) {
  return StreamSlice{uniform(s.row), uniform(s.g), uniform(s.first), uniform(s.npw), uniform(s.pg_end), uniform(s.t1)};
}

// One head of a wave: its queries, the page in flight and the state.
template <int G>
struct StreamHead : State<G> {
  static constexpr int kQ = State<G>::kQ;
  v4u q[kQ], kr[4], vr[4];

  // Forgets the loaded values: they are not kept in registers up to here.
  __device__ __forceinline__ void drop() {
#pragma unroll
    for (int i = 0; i < kQ; ++i) asm volatile("" : "=v"(q[i]));
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "=v"(kr[i]), "=v"(vr[i]));
  }
  // The G query heads of KV head g.
  __device__ __forceinline__ void queries(const DecodeArgs& a, int row, int g) {
    State<G>::load_q(q, page_rsrc(a.q + ((size_t)row * a.Hq + (size_t)g * G) * D, G * D * 2), 0, fresh_tid());
  }
  // Loads of page `phys` of KV head g; unless live through an empty descriptor (zeros, no
  // memory access), so that every path issues the same loads and the wait counts stay exact.
  // An id outside the pool sets *bad (LDS); page 0 is read in its place.
  template <bool K = true, bool V = true>
  __device__ __forceinline__ void issue(const DecodeArgs& a, int kv_off, int g, int phys, bool live, int* bad) {
    const int tok_b = a.Hkv * D * 2;  // bytes between consecutive tokens
    if (live && (unsigned)phys >= (unsigned)a.num_pages) *bad = 1;
    phys = (unsigned)phys < (unsigned)a.num_pages ? phys : 0;
    const int page_b = P * tok_b;
    const size_t at = (size_t)(unsigned)phys * (unsigned)page_b;
    const int bytes = live ? page_b : 0;
    const __amdgpu_buffer_rsrc_t kr_rsrc = page_rsrc(reinterpret_cast<const char*>(a.k) + at, bytes);
    const __amdgpu_buffer_rsrc_t vr_rsrc = page_rsrc(reinterpret_cast<const char*>(a.v) + at, bytes);
#pragma unroll
    for (int i = 0; K && i < 4; ++i)
      kr[i] = __builtin_amdgcn_raw_buffer_load_b128(kr_rsrc, kv_off, g * D * 2 + i * 4 * tok_b, kKvPolicy);
#pragma unroll
    for (int i = 0; V && i < 4; ++i)
      vr[i] = __builtin_amdgcn_raw_buffer_load_b128(vr_rsrc, kv_off, g * D * 2 + i * 4 * tok_b, kKvPolicy);
  }
};

// Workgroup barrier that orders LDS accesses and leaves global loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Waits until at most N of this wave's global loads and stores are outstanding.
template <int N>
__device__ __forceinline__ void vm_wait() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// LDS of a stream's workgroup that its staged pages, the plan's row weights and the merges share.
template <int G, int W>
constexpr int stream_stage_units() {
  constexpr int pages = W * State<G>::kStage, merge = (merge_lds_floats<G, 1, W * 64>() + 3) / 4;
  constexpr int rows = (kMaxFusedPlanBatch + 1 + 3) / 4;
  return pages > merge ? (pages > rows ? pages : rows) : (merge > rows ? merge : rows);
}

// One task of a list behind pkv_plan by itself, as split_kernel runs it: two pages in flight per
// wave, then the state, the count and, for the last of its row and KV head, the merge.
template <int G, int W, bool FUSED>
__device__ __forceinline__ void lone_task(const DecodeArgs& a, int t, const TaskRec& r, float* state, v4u* stage, int* last) {
  if (r.row < 0 || r.row >= a.B || r.g < 0 || r.g >= a.Hkv || r.t0 < 0 || r.t1 <= r.t0 ||
      r.t1 > a.max_pages_per_row * P) {  // not a task of a valid plan: flag and skip
    if (threadIdx.x == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_TASK);
    return;
  }
  Task<G, W> body;
  body.begin(a, r.row, r.g, r.t0, r.t1);
  body.prime(a);
  KnownTask known{r.t1};
  body.run(a, known, state, stage);
  if (!FUSED) {
    finish_task<G, W, false>(a, t, state, nullptr, fresh_tid());
  } else {
    const int off = uniform(a.split_offsets[r.row]);
    int ns = uniform(a.split_offsets[r.row + 1]) - off;
    const bool fits = off >= 0 && ns >= 1 && (long long)(off + ns) * a.Hkv <= a.max_tasks;
    uint16_t* out = a.out + ((size_t)r.row * a.Hq + (size_t)r.g * G) * D;
    finish_task<G, W, true>(a, t, state, fits && ns == 1 ? out : nullptr, fresh_tid());
    if (!fits || ns > 1) {
      if (!fits) {
        if (threadIdx.x == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_TASK);
        ns = 0;  // never reached by the counter: no merge from inconsistent offsets
      }
      vm_wait<0>();  // this wave's stores are acknowledged
      __syncthreads();
      if (threadIdx.x == 0) {
        const int prev = __hip_atomic_fetch_add(&a.counters[r.row * a.Hkv + r.g], 1, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
        *last = prev == ns - 1;
        if (*last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
      __syncthreads();
      if (*last) {
        merge_group<G, W * 64, true>(slots_rsrc(a, slot_floats<G>() * 4), off * a.Hkv + r.g, a.Hkv, ns, out,
                                     reinterpret_cast<float*>(stage));
        if (threadIdx.x == 0) a.counters[r.row * a.Hkv + r.g] = 0;
      }
    }
  }
  __syncthreads();
}

template <int G, int W, bool FUSED, bool PLAN>
__global__ __launch_bounds__(W * 64) void stream_kernel(DecodeArgs a) {
  constexpr int NH = 2;
  constexpr int kStage = State<G>::kStage;            // per wave
  constexpr int kStageAll = stream_stage_units<G, W>();
  __shared__ v4u stage[kStageAll];                   // staged pages; the plan's row weights; merge scratch
  __shared__ float s_state[lds_floats<G, W, NH>()];  // the unit's wave states
  __shared__ int s_bad[5 * W];                       // page-error flags: unit i's at (i % 4) * W, the hint's last
  __shared__ int s_rec[kStreamRecs * 8];
  __shared__ int s_list[kStreamRecs + 1];            // records whose (row, head pair) this workgroup merges; count
  __shared__ int s_apart;                            // the stream left units out that are not pairs
  __shared__ int s_last;                             // one task by itself: whether it was the last of its states
  __shared__ int p_len[PLAN ? kMaxFusedPlanBatch : 1];
  __shared__ int p_off[PLAN ? kMaxFusedPlanBatch + 1 : 1];
  __shared__ int p_wave[W];
  __shared__ long long p_w64[2 * W];
  __shared__ int p_wmax[W];
  const PlanLds PL{p_len, p_off, p_wave, p_w64, p_wmax, reinterpret_cast<int*>(stage)};
  auto zero_rows = [&]() {
    if (FUSED) {  // rows without tasks: their output is zero
      for (int i = blockIdx.x; i < a.B; i += gridDim.x) {
        const bool empty = PLAN ? p_off[i + 1] == p_off[i] : a.split_offsets[i + 1] == a.split_offsets[i];
        if (empty) zero_row<G>(a, i);
      }
    }
  };
  // The host chose this kernel by the tasks it expects of the batch. Where the list is shorter
  // (empty or short rows) and its tasks are better run one by one, they are: the stream's units
  // would leave half of the compute units without work (64 rows, 58 of them empty, one plan and
  // two layers: G = 8 77 -> 54 us, G = 1 70 -> 52). Ahead of all else: after the stream's set-up
  // it shares that one's values and costs every launch 0.5 us.
  int ntasks = 0;
  const int grid = gridDim.x;
  if (!PLAN) {
    ntasks = uniform(*a.num_tasks);
    if (ntasks > a.max_tasks) ntasks = a.max_tasks;
  }
  if (!PLAN && __builtin_expect(!stream_pays(G, ntasks, a.S, false), 0)) {
    for (int t = blockIdx.x; t < ntasks; t += grid) {
      const int* tp = reinterpret_cast<const int*>(a.tasks + t);
      lone_task<G, W, FUSED>(a, t, TaskRec{uniform(tp[0]), uniform(tp[1]), uniform(tp[2]), uniform(tp[3]), uniform(tp[4])},
                             s_state, stage, &s_last);
    }
    zero_rows();
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  v4u* st = stage + wave * kStage;
  PageMath pm;
  if constexpr (on_matrix_cores<G>()) pm.init(st);
  const int kv_off = opaque((lane >> 4) * (a.Hkv * D * 2) + (lane & 15) * 16);  // this lane's piece of a page's head

  auto slice = [&](int row, int g, int t0, int t1) {
    StreamSlice s;
    s.row = row;
    s.g = g;
    s.t1 = t1;
    s.pg_end = (t1 + P - 1) / P;
    s.first = t0 / P + wave;
    s.npw = s.first < s.pg_end ? (s.pg_end - s.first + W - 1) / W : 0;
    return s;
  };
  // Ids of pages k0 .. k0 + 63 of the slice, one per lane (none is read past its pages).
  auto load_ids = [&](const StreamSlice& s, int k0) {
    const int tid = fresh_tid() & 63;
    const __amdgpu_buffer_rsrc_t r = page_rsrc(a.block_table + (size_t)s.row * a.max_pages_per_row + s.first + k0 * W,
                                               s.npw > k0 ? (s.pg_end - s.first - k0 * W) * 4 : 0);
    return (int)__builtin_amdgcn_raw_buffer_load_b32(r, tid * (W * 4), 0, 0);
  };
  StreamHead<G> h[NH];
  StreamSlice cur, nxt{0, 0, 0, 0, 0, 0}, nn;
  int ids = 0, ids_nxt = 0, ids_nn = 0;
  auto start = [&](const StreamSlice& s, int id, int* bad, int heads) {  // first pages of a unit
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) h[hh].issue(a, kv_off, s.g + hh, id, s.npw > 0 && hh < heads, bad);
  };
  bool primed = false;  // h and ids_nxt hold the hinted first unit's start
  int ht0 = 0;
  if (lane < 5) s_bad[lane * W + wave] = 0;  // each wave its own: it sets them before any barrier

  // This workgroup's units: blockIdx.x, then tb + i * ts for 0 < i < n. Unit u is tasks
  // 2u and 2u + 1.
  int tb, ts, n;
  if (PLAN) {
    // While the plan is formed, the waves start the unit listed at this workgroup's index by
    // the previous launch (split_kernel's speculative start): its first pages are kept if the
    // plan gives this workgroup the same ones. The lengths are loaded ahead of them.
    const bool by_wave = wave_plan(a.plan);
    int n_raw = 0;
    if (!by_wave)
      n_raw = (int)threadIdx.x < a.B ? a.seq_lens[threadIdx.x] : 0;
    else if (threadIdx.x < 64)
      n_raw = wave_plan_len(a.plan);
    const bool has_hint = NH * (int)blockIdx.x < a.max_tasks;
    int hv[4] = {-1, -1, -1, -1};
    if (has_hint) {
      const int* tp = reinterpret_cast<const int*>(a.tasks + NH * (int)blockIdx.x);
      hv[0] = ld_i32<true>(tp + 0);
      hv[1] = ld_i32<true>(tp + 1);
      hv[2] = ld_i32<true>(tp + 3);
      hv[3] = ld_i32<true>(tp + 4);
    }
    const int hr = uniform(hv[0]), hg = uniform(hv[1]), h1 = uniform(hv[3]);
    ht0 = uniform(hv[2]);
    primed = has_hint && hr >= 0 && hr < a.B && hg >= 0 && hg % NH == 0 && hg + NH <= a.Hkv && ht0 >= 0 && h1 > ht0 &&
             h1 <= a.max_pages_per_row * P;
    if (primed) {
      nxt = slice(hr, hg, ht0, h1);
      ids_nxt = load_ids(nxt, 0);
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) h[hh].queries(a, nxt.row, nxt.g + hh);
    }
    if (by_wave && threadIdx.x < 64) plan_compute_wave(a.plan, PL, blockIdx.x == 0, n_raw);
    if (primed) start(nxt, __builtin_amdgcn_readlane(ids_nxt, 0), s_bad + 4 * W + wave, NH);
    if (by_wave) {
      lds_barrier();
      ntasks = plan_wave_tasks(a.plan, PL, blockIdx.x == 0);
    } else {
      ntasks = plan_compute<W * 64>(a.plan, PL, blockIdx.x == 0, true, n_raw);
    }
    const int nunits = uniform(ntasks) / NH;
    if (blockIdx.x == 0) plan_write_offsets<W * 64>(a.plan, PL, nunits * NH);
    if (nunits <= 3 * grid) {  // few rounds: every workgroup takes the same number of units, one more or less
      tb = blockIdx.x;
      ts = grid;
      n = tb < nunits ? (nunits - 1 - tb) / ts + 1 : 0;
    } else {
      // Contiguous ranges of about the same weight; lanes 0 and 1 find where this workgroup's
      // and the next one's begin.
      const int b = plan_range_begin(a.plan, PL, a.Hkv / NH, blockIdx.x + (lane & 1), grid, grid, nunits);
      tb = __builtin_amdgcn_readlane(b, 0) - 1;
      ts = 1;
      n = __builtin_amdgcn_readlane(b, 1) - tb;
    }
  } else {
    const int nunits = (ntasks + NH - 1) / NH;  // an odd last task is a unit by itself
    tb = blockIdx.x;
    ts = grid;
    n = tb < nunits ? (nunits - 1 - tb) / ts + 1 : 0;
  }
  // Unit i's place in the task list, in units. Ranges go through a row head pair by head pair
  // (all splits of one, then of the next), so that the merges they end in are spread over the
  // range; a row that the first units reach into keeps the list's order (split by split).
  auto unit_of = [&](int i) {
    int u = i == 0 ? (int)blockIdx.x : tb + i * ts;
    if (PLAN && ts == 1 && i > 0) {
      const int per = a.Hkv / NH;
      const int row = plan_row(PL, a.B, u / per);
      const int at = p_off[row] * per, ns = p_off[row + 1] - p_off[row];
      if (at >= grid) u = at + (u - at) % ns * per + (u - at) / ns;
    }
    return u;
  };

  // One stream per kStreamRecs units. A list behind pkv_plan need not be a plan's: units whose two
  // tasks are not KV heads g and g + 1 (g even) of one split are left out of their stream and
  // follow it in two more, of their first and of their second tasks, one head at a time.
  int apart = 0;  // 0: pairs, 1 and 2: tasks 2u and 2u + 1 of the other units
  for (int c0 = 0; c0 < n;) {
    const int nc = min(kStreamRecs, n - c0);
    const int heads = PLAN || apart == 0 ? NH : 1;
    if (!PLAN && threadIdx.x == 0 && apart == 0) s_apart = 0;
    if (wave == 0 && lane < nc) {  // their records
      const int t = NH * unit_of(c0 + lane) + (!PLAN && apart == 2);
      StreamRec r;
      int split = 0;
      if (PLAN) {
        const TaskRec k = plan_task(a.plan, PL, t);
        r = StreamRec{k.row, k.g, k.t0, k.t1, p_off[k.row], p_off[k.row + 1] - p_off[k.row]};
        split = k.split;
      } else {
        const int first = t / NH * NH;
        const bool two = first + 1 < ntasks;
        const int* tp = reinterpret_cast<const int*>(a.tasks + first);
        const int* tq = tp + (two ? 5 : 0);
        StreamRec q{tq[0], tq[1], tq[3], tq[4], 0, 0};  // both tasks at once: one round trip
        r = StreamRec{tp[0], tp[1], tp[3], tp[4], 0, 0};
        const bool pair = two & (q.row == r.row) & (q.g == r.g + 1) & (r.g % NH == 0) & (q.t0 == r.t0) & (q.t1 == r.t1);
        if (!pair && apart == 0) s_apart = 1;
        if (t > first) r = q;
        const bool mine = apart == 0 ? pair : !pair && t < ntasks;
        if (!mine) r.row = -1;
        if (mine && (r.row < 0 || r.row >= a.B || r.g < 0 || r.g + heads > a.Hkv || r.t0 < 0 || r.t1 <= r.t0 ||
                     r.t1 > a.max_pages_per_row * P)) {  // not a task of this batch: flag and skip
          atomicOr(a.err, (unsigned)PKV_DEVERR_TASK);
          r.row = -1;
        }
        if (r.row < 0) {
        } else if (FUSED) {
          r.off = a.split_offsets[r.row];
          r.ns = a.split_offsets[r.row + 1] - r.off;
          if (r.off < 0 || r.ns < 1 || (long long)(r.off + r.ns) * a.Hkv > a.max_tasks) {
            atomicOr(a.err, (unsigned)PKV_DEVERR_TASK);
            r.ns = 0;  // never reached by the counter: no merge from inconsistent offsets
          }
        }
      }
      int* s = s_rec + lane * 8;
      s[0] = r.row;
      s[1] = r.g;
      s[2] = r.t0;
      s[3] = r.t1;
      s[4] = r.off;
      s[5] = r.ns;
      s[6] = t;
      s[7] = split;
    }
    if (threadIdx.x == 0) s_list[kStreamRecs] = 0;
    lds_barrier();
    const bool left_out = !PLAN && uniform(s_apart) != 0;

    auto slice_of = [&](int i) {  // an empty slice past the stream's end and for a skipped unit
      const int* r = s_rec + min(i, nc - 1) * 8;
      const int row = uniform(r[0]), g = uniform(r[1]), t0 = uniform(r[2]), t1 = uniform(r[3]);
      StreamSlice s = slice(row, g, t0, t1);
      if (i >= nc || row < 0) s = StreamSlice{0, 0, 0, 0, 0, 0};
      return s;
    };
    // Thread 0's bookkeeping of stored states (-1: none): s1, s2 are the last two units'; ta
    // and tb_ were counted in the last odd and the last even unit's epilogue, na and nb the
    // counts read.
    int s1 = -1, s2 = -1, ta = -1, tb_ = -1, na = 0, nb = 0;
    // KV heads g and g + 1 (g even) have one count, in which (behind pkv_plan) each head's task is one.
    constexpr int kTasks = PLAN ? 1 : NH;
    const int counted = PLAN ? 1 : heads;
    auto count = [&](int i) {
      return __hip_atomic_fetch_add(&a.counters[s_rec[i * 8] * a.Hkv + s_rec[i * 8 + 1] / NH * NH], counted, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
    };
    auto list = [&](int i, int seen) {  // the count says that it was its row's last state
      if (i >= 0 && seen == kTasks * s_rec[i * 8 + 5] - counted) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // before any wave reads the states
        const int at = s_list[kStreamRecs];  // other waves may be reading: the entry, then the count
        __hip_atomic_store(s_list + at, i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(s_list + kStreamRecs, at + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    };
    // Merges of listed records. A team of kTeam threads (one column each) takes every
    // kTeams-th head; the waves of a team need not run together. done: entries this wave has
    // seen.
    constexpr int kTeam = G * D / 4, kTeams = W * 64 / kTeam;
    const __amdgpu_buffer_rsrc_t pr = slots_rsrc(a, slot_floats<G>() * 4);
    int done = 0;
    auto merges = [&]() __attribute__((always_inline)) {
      const int nl = uniform(__hip_atomic_load(s_list + kStreamRecs, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
      if (done >= NH * nl) return;
      const int mt = fresh_tid();
      const int team = mt / kTeam, c = mt % kTeam;
      for (; done < NH * nl; ++done) {
        const int* r = s_rec + s_list[done / NH] * 8;
        const int row = uniform(r[0]), g = uniform(r[1]) / NH * NH + done % NH, off = uniform(r[4]), ns = uniform(r[5]);
        const bool mine = done % kTeams == team && ns <= kColRuns * kMergeRun;
        if (__builtin_amdgcn_ballot_w64(mine) == 0) continue;
        merge_columns<G, true>(pr, off * a.Hkv + g, a.Hkv, mine ? ns : 0, ns, c,
                               a.out + ((size_t)row * a.Hq + (size_t)g * G) * D, reinterpret_cast<v2f*>(st));
        if (mine && c == 0 && g % NH == 0) a.counters[row * a.Hkv + g] = 0;
      }
    };

    {
      const StreamSlice s0 = slice_of(0);
      const bool keep = c0 == 0 && primed && s0.row == nxt.row && s0.g == nxt.g && uniform(s_rec[2]) == ht0 &&
                        s0.pg_end == nxt.pg_end;
      nxt = s0;
      nn = slice_of(1);
      if (!keep) {
        ids_nxt = load_ids(nxt, 0);
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) h[hh].queries(a, nxt.row, nxt.g + min(hh, heads - 1));
      } else if (lane == 0) {
        s_bad[wave] = s_bad[4 * W + wave];
      }
      ids_nn = load_ids(nn, 0);
      if (!keep) start(nxt, __builtin_amdgcn_readlane(ids_nxt, 0), s_bad + wave, heads);
      vm_wait<0>();  // on every path, or the compiler would drain the stream at each unit for ids_nn
    }
    for (int i = 0; i < nc; ++i) {
      // The first head's first page, and with it all that was issued before it: the unit's
      // queries, the next one's ids, and the state stores of the unit before the last. (What
      // may be outstanding after it: the other head's page.) A wave without pages of this
      // unit has none in flight.
      if (nxt.npw > 0) vm_wait<8>(); else vm_wait<0>();
      cur = scalar(nxt);
      ids = opaque(ids_nxt);  // copied here, behind the wait, and not at the loop's end
      nxt = scalar(nn);
      ids_nxt = opaque(ids_nn);
      if (FUSED && threadIdx.x == 0) {
        if (i & 1) list(ta, na); else list(tb_, nb);
      }
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) h[hh].reset();
      int* bad = s_bad + (i % 4) * W + wave;
      int* bad_nxt = s_bad + ((i + 1) % 4) * W + wave;
      s_bad[((i + 2) % 4) * W + wave] = 0;  // unit i - 2 has been combined
      int k = 0;
#pragma clang loop unroll(disable)
      do {  // a wave without pages of this unit goes through once, for the next one's first
        const bool live = k < cur.npw;
        const int pg = cur.first + k * W;
        const int t1 = pg == cur.pg_end - 1 ? cur.t1 : cur.pg_end * P;  // pages before the last are whole
        ++k;
        const bool more = k < cur.npw;
        if (more && (k & 63) == 0) {  // the next block of ids, waited for here: rare
          ids = load_ids(cur, k);
          vm_wait<0>();
        }
        if (!more) {
          nn = slice_of(i + 2);
          ids_nn = load_ids(nn, 0);
        }
        const int own = __builtin_amdgcn_readlane(ids, k & 63), other = __builtin_amdgcn_readlane(ids_nxt, 0);
        const int phys = more ? own : other;
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) {
          // The next page's loads go out as soon as the registers are free: all of them once K and V
          // are staged, or K's after the scores and V's after the sums.
          constexpr bool kStaged = on_matrix_cores<G>();
          typename State<G>::Scores sc{};
          if (live) {
            if constexpr (kStaged) {
              pm.stage_k(h[hh].kr);
              sc = pm.scores(h[hh].q);
              pm.stage_v(h[hh].vr, pg * P, t1);
            } else {
              sc = h[hh].scores(h[hh].q, h[hh].kr, a.scale_log2);
            }
          }
          if (!more) h[hh].queries(a, nxt.row, nxt.g + min(hh, heads - 1));
          const int g = (more ? cur.g : nxt.g) + hh;
          const bool next_live = (more || nxt.npw > 0) && hh < heads;
          h[hh].template issue<true, kStaged>(a, kv_off, g, phys, next_live, more ? bad : bad_nxt);
          if constexpr (kStaged) {
            if (live) pm.accumulate(sc, a.scale_log2, pg * P, t1, h[hh].m, h[hh].l, h[hh].acc);
          } else {
            if (live) h[hh].accumulate(sc, h[hh].vr, pg * P, t1);
          }
          if (!kStaged) h[hh].template issue<false, true>(a, kv_off, g, phys, next_live, more ? bad : bad_nxt);
        }
      } while (k < cur.npw);
      lds_barrier();  // the unit before this one has been combined
#pragma unroll
      for (int hh = 0; hh < NH; ++hh)
        h[hh].dump(pm, state_acc<G, W, NH>(s_state) + (hh * W + wave) * G * kHeadPitch,
                   state_ml<G, W, NH>(s_state) + (hh * W + wave) * G, *bad != 0, fresh_tid());
      lds_barrier();
      const int* r = s_rec + i * 8;
      const int row = uniform(r[0]), g = uniform(r[1]), ns = uniform(r[5]);
      if (FUSED && threadIdx.x == 0) {
        // Every wave has waited for its stores of the unit before the last: count it.
        if (i & 1) {
          ta = s2;
          if (s2 >= 0) na = count(s2);
        } else {
          tb_ = s2;
          if (s2 >= 0) nb = count(s2);
        }
        s2 = s1;
        s1 = row >= 0 && ns != 1 ? i : -1;  // a row's only split stores no state
      }
      // G < 8 leaves half of the threads without a column: the halves take turns.
      constexpr int kCols = NH * G * D / 4;
      const int ct = fresh_tid() - (kCols <= W * 32 && (i & 1) ? W * 32 : 0);
      if (row >= 0 && ct >= 0)
        finish_task<G, W, FUSED, NH>(a, uniform(r[6]), s_state,
                                     FUSED && ns == 1 ? a.out + ((size_t)row * a.Hq + (size_t)g * G) * D : nullptr, ct,
                                     heads);
      if (FUSED) merges();
    }
    if (PLAN && wave == W - 1 && lane < nc) {  // the units' tasks in the task list (off the stream's way)
      const int* r = s_rec + lane * 8;
      int* o = reinterpret_cast<int*>(a.plan.tasks + r[6]);
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) {
        o[5 * hh] = r[0];
        o[5 * hh + 1] = r[1] + hh;
        o[5 * hh + 2] = r[7];
        o[5 * hh + 3] = r[2];
        o[5 * hh + 4] = r[3];
      }
    }
    if (FUSED) {  // the last counts, then the merges that are left
      vm_wait<0>();
      lds_barrier();
      if (threadIdx.x == 0) {
        list(ta, na);
        list(tb_, nb);
        if (s2 >= 0) list(s2, count(s2));
        if (s1 >= 0) list(s1, count(s1));
      }
      lds_barrier();
      const int nl = uniform(s_list[kStreamRecs]);
      // Several left: side by side. One or two: by the whole workgroup, one round of loads each.
      constexpr int kHeads = merge_lds_floats<G, NH, W * 64>() <= kStageAll * 4 ? NH : 1;  // per merge_group
      const int from = nl - uniform(done) / NH > 2 ? nl : uniform(done) / NH;
      if (from == nl) merges();
      for (int j = 0; j < nl; ++j) {
        const int* r = s_rec + s_list[j] * 8;
        const int row = uniform(r[0]), g = uniform(r[1]) / NH * NH, off = uniform(r[4]), ns = uniform(r[5]);
        if (j < from && ns <= kColRuns * kMergeRun) continue;
        for (int hh = 0; hh < NH; hh += kHeads) {
          lds_barrier();
          merge_group<G, W * 64, true, kHeads>(pr, off * a.Hkv + g + hh, a.Hkv, ns,
                                               a.out + ((size_t)row * a.Hq + (size_t)(g + hh) * G) * D,
                                               reinterpret_cast<float*>(stage));
        }
        if (threadIdx.x == 0) a.counters[row * a.Hkv + g] = 0;
      }
      lds_barrier();
    } else {
      lds_barrier();  // every wave has read its last unit's record: the next stream's may be written
    }
    for (int hh = 0; hh < NH; ++hh) h[hh].drop();
    if (left_out && apart < 2) {
      ++apart;
    } else {
      apart = 0;
      c0 += kStreamRecs;
    }
  }
  zero_rows();
}

// Rectangular grid: slot (j*S + s)*Hkv + g is split s of KV head g of launch row j, which is
// row_ids[j] when the launch names its rows (a length bucket; Q and out are then read and
// written by index), else row j.
struct RectTask {
  int row, tiles, ns, t0, t1;  // ns: the row's splits; split s of a row is empty for s >= ns
};
__device__ __forceinline__ RectTask rect_task(const DecodeArgs& a, int split_slot, bool report) {
  const int s = split_slot % a.S, j = split_slot / a.S;
  RectTask r{a.n_rows > 0 ? a.row_ids[j] : j, 0, 0, 0, 0};
  int n = uniform(a.seq_lens[r.row]);
  if (n < 0 || n > a.max_pages_per_row * P) {
    if (threadIdx.x == 0 && s == 0 && report) atomicOr(a.err, (unsigned)PKV_DEVERR_SEQ_LEN);
    n = 0;
  }
  const int T = a.tile_tokens;
  r.tiles = (n + T - 1) / T;
  r.ns = r.tiles < a.S ? r.tiles : a.S;
  if (s < r.ns) {
    r.t0 = uniform(split_bound(s, r.tiles, r.ns) * T);
    r.t1 = uniform(min(split_bound(s + 1, r.tiles, r.ns) * T, n));
  }
  return r;
}

// NH adjacent slots (KV heads of one split) per workgroup, in slot order. Empty splits write
// the neutral state and end without Q or KV traffic (Sec. 3.3).
template <int G, int W, int NH>
__global__ __launch_bounds__(W * 64) void rect_kernel(DecodeArgs a) {
  __shared__ float lds[lds_floats<G, W, NH>()];
  const int slot = NH * (int)blockIdx.x;
  const int g = slot % a.Hkv;
  const RectTask r = rect_task(a, slot / a.Hkv, g == 0);
  if (r.t1 <= r.t0) {
    for (int hh = 0; hh < NH; ++hh) write_neutral<G>(a, slot + hh);
    return;
  }
  run_split_task<G, W, false, NH>(a, r.row, g, r.t0, r.t1, slot, lds);
}

// The same for grids of many small slots (rect_dense): NH adjacent slots (KV heads of one
// split) per workgroup, one after another, the next head's first page in flight while one is
// combined. The hardware deals the workgroups out, so what else a slot spends outside its page
// reads is hidden only by other workgroups on the compute unit: a wave keeps one page in
// flight (as in the stream above), which with the wave states laid over the staged pages holds
// a workgroup to 128 registers and 72 KB of LDS, two of them per compute unit (on the vector ALU
// to 80 registers: three).
template <int G, int W, int NH>
__global__ __launch_bounds__(W * 64, on_matrix_cores<G>() ? 4 : 6) void rect_dense_kernel(DecodeArgs a) {
  constexpr int kPages = on_matrix_cores<G>() ? W * kStageUnits : 0, kStates = (lds_floats<G, W>() + 3) / 4;
  __shared__ v4u stage[kPages > kStates ? kPages : kStates];
  __shared__ int s_bad[NH * W];
  float* state = reinterpret_cast<float*>(stage);
  const int slot = NH * (int)blockIdx.x;
  const int g = slot % a.Hkv;
  const RectTask r = rect_task(a, slot / a.Hkv, g == 0);
  if (r.t1 <= r.t0) {
    for (int hh = 0; hh < NH; ++hh) write_neutral<G>(a, slot + hh);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  PageMath pm;
  if constexpr (on_matrix_cores<G>()) pm.init(stage + wave * kStageUnits);
  const int kv_off = opaque((lane >> 4) * (a.Hkv * D * 2) + (lane & 15) * 16);
  const int pg_end = (r.t1 + P - 1) / P, first = r.t0 / P + wave;
  const int npw = first < pg_end ? (pg_end - first + W - 1) / W : 0;
  const int32_t* idrow = a.block_table + (size_t)r.row * a.max_pages_per_row + first;
  auto load_ids = [&](int k0) { return lane < npw - k0 ? idrow[(size_t)(k0 + lane) * W] : 0; };
  if (lane < NH) s_bad[lane * W + wave] = 0;
  StreamHead<G> h;
  const int first_ids = load_ids(0);
  h.issue(a, kv_off, g, __builtin_amdgcn_readlane(first_ids, 0), npw > 0, s_bad + wave);
  h.queries(a, r.row, g);
#pragma clang loop unroll(disable)
  for (int hh = 0; hh < NH; ++hh) {
    h.reset();
    int ids = first_ids;
#pragma clang loop unroll(disable)
    for (int k = 0; k < npw; ++k) {
      const int pg = first + k * W;
      const int end = pg == pg_end - 1 ? r.t1 : pg_end * P;  // pages before the last are whole
      const bool more = k + 1 < npw;
      auto next = [&](auto k_too, auto v_too) __attribute__((always_inline)) {
        const int phys = __builtin_amdgcn_readlane(ids, (k + 1) & 63), phys0 = __builtin_amdgcn_readlane(first_ids, 0);
        h.template issue<decltype(k_too)::value, decltype(v_too)::value>(
            a, kv_off, more ? g + hh : g + hh + 1, more ? phys : phys0, more || hh + 1 < NH,
            s_bad + (more || hh + 1 == NH ? hh : hh + 1) * W + wave);
      };
      if constexpr (on_matrix_cores<G>()) {
        pm.stage_k(h.kr);
        pm.stage_v(h.vr, pg * P, end);
        if (more && ((k + 1) & 63) == 0) ids = load_ids(k + 1);
        next(std::true_type{}, std::true_type{});
        pm.accumulate(pm.scores(h.q), a.scale_log2, pg * P, end, h.m, h.l, h.acc);
      } else {
        if (more && ((k + 1) & 63) == 0) ids = load_ids(k + 1);
        auto sc = h.scores(h.q, h.kr, a.scale_log2);
        next(std::true_type{}, std::false_type{});
        h.accumulate(sc, h.vr, pg * P, end);
        next(std::false_type{}, std::true_type{});
      }
    }
    if (hh + 1 < NH) h.queries(a, r.row, g + hh + 1);
    lds_barrier();  // every wave is done with its staged page
    h.dump(pm, state_acc<G, W>(state) + wave * G * kHeadPitch, state_ml<G, W>(state) + wave * G,
           s_bad[hh * W + wave] != 0, fresh_tid());
    lds_barrier();
    finish_task<G, W, false>(a, slot + hh, state, nullptr, fresh_tid());
    lds_barrier();
  }
}

// Segmented merge: one workgroup per (row, KV head), the same merge_group code as the
// fused route. RECT: slots (row*S + s)*Hkv + g for s < S; else the planner's
// split_offsets.
constexpr int kMergeThreads = 256;

template <int G, bool RECT>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(DecodeArgs a) {
  __shared__ float lds[merge_lds_floats<G, 1, kMergeThreads>()];
  const int j = blockIdx.x / a.Hkv;  // the launch's row index
  const int g = blockIdx.x % a.Hkv;
  const int row = (RECT && a.n_rows > 0) ? a.row_ids[j] : j;
  int slot0, nsplit;
  if (RECT) {
    slot0 = j * a.S * a.Hkv + g;
    nsplit = a.S;
  } else {
    const int off = a.split_offsets[row];
    slot0 = off * a.Hkv + g;
    nsplit = a.split_offsets[row + 1] - off;
    if (off < 0 || nsplit < 0 || (long long)(off + nsplit) * a.Hkv > a.max_tasks) {
      // offsets that do not belong to a plan of this capacity: never read past the slots
      if (threadIdx.x == 0 && g == 0) atomicOr(a.err, (unsigned)PKV_DEVERR_TASK);
      nsplit = 0;
    }
  }
  merge_group<G, kMergeThreads, false>(slots_rsrc(a, slot_floats<G>() * 4), uniform(slot0), a.Hkv, uniform(nsplit),
                                a.out + ((size_t)row * a.Hq + (size_t)g * G) * D, lds);
}

__global__ void zero_kernel(uint32_t* p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// Workspace set-up: header and counters zeroed, then the counter count and its check
// word recorded in header words 1 and 2 (read back by pkv_check_device_status).
__global__ void ws_init_kernel(uint32_t* p, size_t n, uint32_t counters) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = i == kWsCountWord ? counters : (i == kWsCheckWord ? counters ^ kWsCheckKey : 0u);
}

__global__ __launch_bounds__(256) void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// NT: non-temporal loads, the cache policy of the decode kernel's K/V page loads.
template <bool NT>
__global__ __launch_bounds__(256) void read_kernel(const v4u* __restrict__ src, size_t n, unsigned* sink) {
  unsigned x = 0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const v4u v = NT ? __builtin_nontemporal_load(src + i) : src[i];
    x += v.x ^ (v.y * 3u) ^ (v.z * 5u) ^ (v.w * 7u);
  }
  if (x == 0x9E3779B9u) *sink = x;  // keeps the loads; practically never taken
}

// Read-only probe of the decode kernel's KV access pattern: for every task of a task
// list (records as the planner writes them), the waves of a workgroup read the K and V
// bytes of the task's NH KV heads over its pages as the decode body does (wave w takes
// pages w, w + W, ... of the task, page ids fetched 64 at a time, per page and head four
// 16-byte buffer loads of K and four of V, each covering four whole 256-byte rows; two
// (page, head) units in flight per wave: two pages of one head, or one page of each of
// two heads), with the decode's grid (one workgroup per compute unit, held by the LDS
// reservation) and, as long as tasks are dealt in strides (the one-task kernels, and streams
// of up to three rounds), its task-to-workgroup mapping. Nothing else: no queries, no arithmetic
// beyond folding the bytes into a sink word, no state, no merge. Its time is the read
// time of the decode's pages in the decode's pattern.
constexpr int kPageReadHoldWords = 24 * 1024;  // 96 KiB of LDS: one workgroup per compute unit

template <int W, int NH>
__global__ __launch_bounds__(W * 64) void page_read_kernel(PageReadArgs a) {
  __shared__ unsigned hold[kPageReadHoldWords];
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  const int grp = lane >> 4, col = lane & 15;
  const size_t tok_stride = (size_t)a.Hkv * D;  // halves between consecutive tokens
  const size_t page_stride = (size_t)P * tok_stride;
  const int tok_b = (int)(tok_stride * 2);
  const int page_bytes = (int)(page_stride * 2);
  int ntasks = uniform(*a.num_tasks);
  if (ntasks > a.max_tasks) ntasks = a.max_tasks;
  unsigned x = 0;
  for (int t = NH * blockIdx.x; t + NH <= ntasks; t += NH * gridDim.x) {
    const int* tp = reinterpret_cast<const int*>(a.tasks + t);
    const int row = uniform(tp[0]), g = uniform(tp[1]), t0 = uniform(tp[3]), t1 = uniform(tp[4]);
    if (row < 0 || row >= a.B || g < 0 || g % NH != 0 || g + NH > a.Hkv || t0 < 0 || t1 <= t0 ||
        t1 > a.max_pages_per_row * P)
      continue;  // not a task of a valid plan: read nothing
    const int first = t0 / P + wave;
    const int pg_end = (t1 + P - 1) / P;
    const int npw = first < pg_end ? (pg_end - first + W - 1) / W : 0;
    const int nunits = npw * NH;  // unit u: page u / NH of the wave, head g + u % NH
    const int* idrow = a.block_table + (size_t)row * a.max_pages_per_row + first;
    auto fetch_ids = [&](int base) {  // ids of the wave's pages base .. base + 63
      return lane < npw - base ? idrow[(size_t)(base + lane) * W] : 0;
    };
    int ids = fetch_ids(0);
    auto issue = [&](v4u (&kr)[4], v4u (&vr)[4], int u) {  // u >= nunits: empty descriptors
      const int j = u / NH, hh = u - (u / NH) * NH;
      int phys = __builtin_amdgcn_readlane(ids, j & 63);
      const bool ok = u < nunits && phys >= 0 && phys < a.num_pages;
      phys = uniform(ok ? phys : 0);
      const int bytes = uniform(ok ? page_bytes : 0);
      const __amdgpu_buffer_rsrc_t kr_rsrc = page_rsrc(a.k + (size_t)phys * page_stride, bytes);
      const __amdgpu_buffer_rsrc_t vr_rsrc = page_rsrc(a.v + (size_t)phys * page_stride, bytes);
      const int kv_off = grp * tok_b + (g + hh) * D * 2 + col * 16;
#pragma unroll
      for (int i = 0; i < 4; ++i) kr[i] = __builtin_amdgcn_raw_buffer_load_b128(kr_rsrc, kv_off, i * 4 * tok_b, kKvPolicy);
#pragma unroll
      for (int i = 0; i < 4; ++i) vr[i] = __builtin_amdgcn_raw_buffer_load_b128(vr_rsrc, kv_off, i * 4 * tok_b, kKvPolicy);
    };
    auto fold = [&](const v4u (&kr)[4], const v4u (&vr)[4]) {
#pragma unroll
      for (int c = 0; c < 4; ++c) x += (kr[c].x ^ kr[c].y ^ kr[c].z ^ kr[c].w) + (vr[c].x ^ vr[c].y ^ vr[c].z ^ vr[c].w);
    };
    v4u ka[4], va[4], kb[4], vb[4];
    issue(ka, va, 0);
    issue(kb, vb, 1);
    for (int u = 0; u < nunits; u += 2) {
      fold(ka, va);
      // unit u + 2 is the first head of a page; a new block of 64 ids starts there
      if (u + 2 < nunits && ((u + 2) / NH) % 64 == 0) ids = fetch_ids((u + 2) / NH);
      issue(ka, va, u + 2);
      fold(kb, vb);
      issue(kb, vb, u + 3);
    }
  }
  hold[threadIdx.x] = x;
  __syncthreads();
  if (hold[(threadIdx.x + 1) % (W * 64)] == 0x9E3779B9u) *a.sink = x;  // keeps the loads; practically never taken
}

// Compute units of the device (of the first one that asks).
int compute_units() {
  static const int n = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 256;
    return cus;
  }();
  return n;
}

// Workgroups of `kernel` resident on the current device at once (occupancy x CUs),
// at least one per CU. The split kernels loop over tasks with the grid as stride, so
// their grid is the task bound capped at this count (taken once per kernel, on the
// first device that launches it).
int resident_blocks(const void* kernel, int threads) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  return per_cu * compute_units();
}

// Kernels go out through hipExtLaunchKernelGGL: with events it stamps `start` when the
// first kernel of the call begins and `stop` when the last one ends (kernel execution
// time, as a profiler reports it); without events it is a plain launch.
template <typename K>
hipError_t launch(K kernel, int grid, int threads, hipStream_t s, hipEvent_t start, hipEvent_t stop,
                  const DecodeArgs& a) {
  hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, s, start, stop, 0, a);
  return hipGetLastError();
}

// Whether a launch goes to the stream kernel, by the tasks the host expects.
bool streams(int G, int Hkv, int max_tasks, int64_t tasks, int slots, bool paired) {
  return Hkv % 2 == 0 && max_tasks >= 2 && stream_pays(G, tasks, slots, paired);
}

template <int G, int W, bool FUSED, bool PLAN>
int stream_slots() {
  static const int r = resident_blocks((const void*)stream_kernel<G, W, FUSED, PLAN>, W * 64);
  return r;
}

DecodeArgs with_slots(DecodeArgs a, int slots) {
  a.S = slots;
  return a;
}

template <int G, int W>
hipError_t launch_decode_g(const DecodeArgs& a, int mode, int grid, hipStream_t s, hipEvent_t start,
                           hipEvent_t stop) {
  if (mode == 2) {
    const int rows = a.n_rows > 0 ? a.n_rows : a.B;
    const int slots = rows * a.Hkv * a.S;
    const int64_t tiles = ((int64_t)a.max_pages * P + a.tile_tokens - 1) / a.tile_tokens;
    const int64_t slot_pages = (tiles + a.S - 1) / a.S * (a.tile_tokens / P);
    const bool even = a.Hkv % 2 == 0;
    const int cus = compute_units();  // (256 in the figures below)
    bool pairs, dense;  // two heads per workgroup; the dense kernel
    if constexpr (on_matrix_cores<G>()) {
      // A slot of at most two pages per wave is a chain of round trips more than a read. Beyond one
      // slot per compute unit a workgroup then runs the chains of two KV heads as one (16 splits of
      // rows of 2048 tokens: 512 slots 14.4 -> 12.5 us, 640 18.8 -> 18.3, 1408 33.9 -> 28.2; of 4096
      // tokens 19.9 -> 17.5, 25.9 -> 25.9, 47.7 -> 41.3). Longer slots are balanced better one by
      // one (four rows of 17-32 K tokens twice: 108 against 102), and from 1536 slots on the dense
      // kernel is the faster (rows of 1024 tokens: 1536 slots 21.4 against 22.7, 8192 76 against 94).
      // Many slots are small ones (each row has S of them): from six per compute unit on, two
      // workgroups a unit with one page in flight per wave beat one with two (13 rows of up to
      // 8250 tokens, 1664 slots: 46 against 48 us; 21 rows of up to 39 K, 1344 slots: 146 against
      // 139), and from twelve rounds of them on two slots per workgroup beat one (60 rows of up
      // to 4096 tokens, 7680 slots: 103 against 112 us; 2560 slots: 86 against 82).
      dense = slots >= 6 * cus;
      pairs = even && (dense ? slots >= 24 * cus : G <= 4 && slots > cus && slot_pages <= 2 * W);
    } else if (G == 1) {
      // Without staged pages two one-head workgroups fit a compute unit. Pairs pay as soon as one
      // round of those does not hold the slots (Hkv = 32, 1024 slots of rows of 1500 tokens 11.4 ->
      // 9.9 us, 32 rows 122.6 -> 93.7; 512 slots of 24 K tokens 17.0 against 21.4). An odd head
      // left over: short slots dense from six per compute unit on (Hkv = 3, 64 rows of 1500
      // tokens 28.6 -> 24.8 us, 24 K tokens 115 against 122).
      pairs = even && slots > 2 * cus;
      dense = !even && slots >= 6 * cus && slot_pages <= 2 * W;
    } else {
      // G = 2: one by one, dense (three workgroups a unit) from six slots per compute unit on
      // (Hkv = 16: 2048 slots of rows of 1500 tokens 23.8 -> 22.4 us, 16384 of 400 tokens 83 -> 78;
      // pairs of heads in the dense kernel 83 and 141 against 79 and 138, rows of 64 tokens 52
      // against 44), with an odd head short slots only (Hkv = 3, 32 rows of 24 K tokens 124 against 118).
      pairs = false;
      dense = slots >= 6 * cus && (even || slot_pages <= 2 * W);
    }
    hipError_t e;
    if (dense && pairs) e = launch(rect_dense_kernel<G, W, on_matrix_cores<G>() ? 2 : 1>, slots / 2, W * 64, s, start, nullptr, a);
    else if (dense) e = launch(rect_dense_kernel<G, W, 1>, slots, W * 64, s, start, nullptr, a);
    else if (pairs) e = launch(rect_kernel<G, W, G == 1 || G == 4 ? 2 : 1>, slots / 2, W * 64, s, start, nullptr, a);
    else e = launch(rect_kernel<G, W, 1>, slots, W * 64, s, start, nullptr, a);
    if (e != hipSuccess) return e;
    return launch(merge_kernel<G, true>, rows * a.Hkv, kMergeThreads, s, nullptr, stop, a);
  }
  if (mode == 3) {
    // The stream's row weights (tiles plus splits) are summed in 32 bits.
    const int64_t weight = (int64_t)a.B * ((int64_t)a.max_pages_per_row * P / a.plan.tile_tokens + 1 + a.plan.split_max);
    const int r = stream_slots<G, W, true, true>();
    if (weight <= INT32_MAX && streams(G, a.Hkv, grid, a.plan.target_tasks, r, G < 8))
      return launch(stream_kernel<G, W, true, true>, grid / 2 < r ? grid / 2 : r, W * 64, s, start, stop, a);
    // KV-head pairs when the task target gives every resident workgroup two tasks (at G = 8
    // the pair merge needs two rounds of loads and the pairs ran 11% slower on the B8 traces)
    if constexpr (G <= 4) {
      static const int resident2 = resident_blocks((const void*)split_kernel<G, W, true, true, 2>, W * 64);
      if (a.Hkv % 2 == 0 && a.plan.target_tasks >= 2 * resident2) {
        const int pairs = grid / 2;
        return launch(split_kernel<G, W, true, true, 2>, pairs < resident2 ? pairs : resident2, W * 64, s, start,
                      stop, a);
      }
    }
    static const int resident = resident_blocks((const void*)split_kernel<G, W, true, true>, W * 64);
    return launch(split_kernel<G, W, true, true>, grid < resident ? grid : resident, W * 64, s, start, stop, a);
  }
  // A task list made elsewhere: its length is on the device only. The default target's
  // four splits per row and KV head stand for it, and the stream kernel looks at the list's
  // own length again.
  const int64_t expected = (int64_t)4 * a.B * a.Hkv;
  if (mode == 1) {
    const int r = stream_slots<G, W, true, false>();
    if (streams(G, a.Hkv, grid, expected, r, false))
      return launch(stream_kernel<G, W, true, false>, grid < r ? grid : r, W * 64, s, start, stop, with_slots(a, r));
    static const int resident = resident_blocks((const void*)split_kernel<G, W, true, false>, W * 64);
    return launch(split_kernel<G, W, true, false>, grid < resident ? grid : resident, W * 64, s, start, stop, a);
  }
  hipError_t e;
  const int r = stream_slots<G, W, false, false>();
  if (streams(G, a.Hkv, grid, expected, r, false)) {
    e = launch(stream_kernel<G, W, false, false>, grid < r ? grid : r, W * 64, s, start, nullptr, with_slots(a, r));
  } else {
    static const int resident = resident_blocks((const void*)split_kernel<G, W, false, false>, W * 64);
    e = launch(split_kernel<G, W, false, false>, grid < resident ? grid : resident, W * 64, s, start, nullptr, a);
  }
  if (e != hipSuccess) return e;
  return launch(merge_kernel<G, false>, a.B * a.Hkv, kMergeThreads, s, nullptr, stop, a);
}

}  // namespace

// Waves per workgroup. Eight (two per SIMD) stream a paged KV pattern ~1-2% faster per
// step than four here, and the kernels are written to fit two waves per SIMD (at most
// 256 registers per lane: the merge keeps at most 16 float4 loads in flight per thread).
constexpr int kWaves = 8;

hipError_t launch_decode(const DecodeArgs& a, int G, int mode, int grid, hipStream_t s, hipEvent_t start,
                         hipEvent_t stop) {
  switch (G) {
    case 1: return launch_decode_g<1, kWaves>(a, mode, grid, s, start, stop);
    case 2: return launch_decode_g<2, kWaves>(a, mode, grid, s, start, stop);
    case 4: return launch_decode_g<4, kWaves>(a, mode, grid, s, start, stop);
    case 8: return launch_decode_g<8, kWaves>(a, mode, grid, s, start, stop);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_plan(const PlanArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 4;
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t*)p, n);
  return hipGetLastError();
}

hipError_t launch_ws_init(void* ws, size_t bytes, uint32_t counters, hipStream_t s) {
  const size_t n = bytes / 4;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(ws_init_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t*)ws, n, counters);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Library-held scratch for pkv_plan_decode_noalloc: completion counters, then partial-
// state slots. Each device holds its own copy; host code reaches it only through the
// device address returned by hipGetSymbolAddress, taken once per device.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(hipStream_t s, char** base) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if ((e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    // counters start at zero; every completed call leaves them at zero
    if ((e = launch_zero(ptr, kScratchCounterBytes, s)) != hipSuccess) return e;
    g_scratch_ptr[dev] = ptr;
  }
  *base = static_cast<char*>(g_scratch_ptr[dev]);
  return hipSuccess;
}

// One 16-byte load per lane per trip with up to 4096 workgroups (16 per compute unit):
// of the read shapes measured on MI355X (1, 2, 4, 8 or 16 loads in flight per lane,
// 512 to 8192 workgroups) this streams fastest, 6.2-6.4 TB/s with the default cache
// policy and 6.3-6.7 TB/s with non-temporal loads.
hipError_t launch_read(const void* src, size_t bytes, unsigned* sink, hipStream_t s, hipEvent_t start,
                       hipEvent_t stop, bool non_temporal) {
  const size_t n = bytes / 16;
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (non_temporal)
    hipExtLaunchKernelGGL(read_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, start, stop, 0,
                          (const v4u*)src, n, sink);
  else
    hipExtLaunchKernelGGL(read_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s, start, stop, 0,
                          (const v4u*)src, n, sink);
  return hipGetLastError();
}

// The decode kernel's grid: the task bound (in NH-task units) capped at one workgroup
// per compute unit.
hipError_t launch_page_read(const PageReadArgs& a, int heads_per_workgroup, hipStream_t s, hipEvent_t start,
                            hipEvent_t stop) {
  auto go = [&](auto kernel, int nh) {
    static_assert(kWaves * 64 <= kPageReadHoldWords, "hold covers the workgroup");
    const int resident = resident_blocks((const void*)kernel, kWaves * 64);
    const int units = a.max_tasks / nh > 0 ? a.max_tasks / nh : 1;
    const int grid = units < resident ? units : resident;
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(kWaves * 64), 0, s, start, stop, 0, a);
    return hipGetLastError();
  };
  if (heads_per_workgroup == 2) return go(page_read_kernel<kWaves, 2>, 2);
  return go(page_read_kernel<kWaves, 1>, 1);
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 16;
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, n);
  return hipGetLastError();
}

}  // namespace pkv
