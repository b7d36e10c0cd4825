// Speculative segmented sum CSR SpMV for gfx950 (MI355X), y = A x.
//
// Stage 1 (Section 3.2, the appendix algorithm's first-stage function): one
// 64-lane wavefront per thread-bunch of S tiles, each tile W*64 nonzeros
// (Section 3.1).  Per bunch:
//   * the bunch's first row r0 = rightmost row with row_ptr[r] <= b0, by a
//     wave-parallel 64-ary search (each round narrows the range 64x with one
//     load per lane and a ballot), or read from the plan when the plan ran
//     that search once for all calls (bound rows);
//   * one pass over the bunch's rows in 64-row chunks builds the segment
//     descriptor of all S tiles as a bit mask in LDS (head at row_ptr[r] - b0
//     for each non-empty row), finds every tile's start row (the rightmost
//     match of each tile boundary, counted by ballots) and detects the dirty
//     tiles (an empty row among rows start..stop-1 of the tile);
//   * per tile: coalesced vector loads of col/val in a grouped order (lane
//     j loads G consecutive entries of each row of 64*G; 16 bytes of values
//     per load), gathers of x in the same order, the products moved through
//     LDS to lane j's entries [jW, jW+W), an exclusive scan of head counts giving each
//     partial sum its compact rank q, one pass over the lane's products that
//     stores every segment closed inside the lane, a 64-lane segmented scan
//     of the lanes' open segments (DPP) that completes the segments crossing
//     lanes, and the store of partial q to y[start + q].
//     The bunch's first segment goes to the synchronizer instead; a tile that
//     ends inside row `stop` hands its last partial to the next tile through
//     the transmitter.  Dirty tiles are recorded, as <start, stop, tile>, in
//     the bunch's own speculator slots, with a per-bunch dirty mask.
// sss_csr_spmv_execute and batches run the fused kernel (sss_fused), which
// does both stages' work in one launch; the split kernels below it serve
// sss_csr_spmv_stage1 / stage2 and debug plans, which record the paper's
// intermediate state.
// Stage 2 (Section 3.2, checking prediction; the paper runs it on a CPU core)
// is one device kernel with three independent parts: the synchronizer carries
// (one thread per run of bunches sharing a first row; the wavefront for long
// runs), the re-arrangement of each dirty tile's partial sums to its non-empty
// rows (one wavefront per thread-bunch), and zeroing the leading empty rows no
// tile covers.
//
// Differences from the paper's listing, on purpose:
//  * a dirty tile that ends inside row `stop` also passes its last partial on
//    through the transmitter and writes it at y[stop] (its true row), where
//    the listing clears the transmitter and leaves that partial to the
//    re-arrangement.  The result is the same sum; the gain is that the
//    re-arrangement then only touches rows strictly inside dirty tiles, so all
//    three parts of stage 2 are disjoint and run concurrently in one launch,
//    with no ordering between them.
//  * the speculator is packed per thread-bunch (S slots each, plus a dirty
//    mask) instead of through one global atomic counter.  On a multi-die GPU a
//    device-wide counter needs either a cross-die atomic per dirty tile and a
//    grid-wide "last block" handshake to reset it between calls, or an extra
//    launch; per-bunch slots need neither, and stage 2's wavefront for a bunch
//    finds that bunch's dirty tiles directly.
//
// Precision: F32/BF16 multiply in float; every sum is in double: the segments',
// the partials, the transmitter, the synchronizer and the stage-2 carry sums are double.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <climits>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <vector>

#include "sss_internal.h"

namespace {

constexpr int kWave = 64;
constexpr int kMaxB = 4;  // wavefronts per workgroup
constexpr int kShortRun = 16;  // stage-2 carry runs up to this many bunches: one thread

thread_local hipError_t g_last_hip = hipSuccess;

#define SSS_HIP(call)                         \
  do {                                        \
    hipError_t e_ = (call);                   \
    if (e_ != hipSuccess) {                   \
      g_last_hip = e_;                        \
      return SSS_ERR_HIP;                     \
    }                                         \
  } while (0)

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

#ifndef SSS_NT_LOADS
#define SSS_NT_LOADS 0
#endif
#ifndef SSS_NT_STORES
#define SSS_NT_STORES 0
#endif

// streaming loads of the matrix arrays (plain loads stream faster than
// non-temporal ones on gfx950 for this pattern)
template <typename T>
__device__ __forceinline__ T stream_load(const T *p) {
  if constexpr (SSS_NT_LOADS) return __builtin_nontemporal_load(p);
  else return *p;
}
template <typename T>
__device__ __forceinline__ void y_store(T v, T *p) {
  if constexpr (SSS_NT_STORES) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// ---------------------------------------------------------------- value types

template <int DT> struct VT;
template <> struct VT<SSS_F64> { using val_t = double;   using x_t = double; using y_t = double; using prod_t = double; };
template <> struct VT<SSS_F32> { using val_t = float;    using x_t = float;  using y_t = float;  using prod_t = float; };
template <> struct VT<SSS_BF16>{ using val_t = uint16_t; using x_t = float;  using y_t = float;  using prod_t = float; };

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) {
  return __uint_as_float(bits16 << 16);
}

// The segment sums of every type are doubles.  F32 and BF16 round each product
// to float once and add the products in double: a float pair kept by TwoSum
// has at most the same accuracy, takes seven float additions per entry where
// this takes a conversion and one double addition (which issues at the same
// rate), and eleven per scan step where this takes one.  It had made those
// types issue 2.4 times FP64's vector instructions on the same tiles (FEM band
// 778K x 50, W = 8, S = 2: 1,595 per wavefront against 661 on the 27-point
// stencil).
struct AccD {
  double s;
  __device__ __forceinline__ void zero() { s = 0.0; }
  __device__ __forceinline__ void add(double v) { s += v; }
  // this := earlier (+) this
  __device__ __forceinline__ void prepend(const AccD &earlier) { s = earlier.s + s; }
  __device__ __forceinline__ double value() const { return s; }
};

// ---------------------------------------------------------------- loads

__device__ __forceinline__ double scalar_val(const double *v, int k) { return v[k]; }
__device__ __forceinline__ float scalar_val(const float *v, int k) { return v[k]; }
__device__ __forceinline__ float scalar_val(const uint16_t *v, int k) { return bf16_to_f32(v[k]); }

// Integer minimum (HIP's min for 64-bit integers goes through double).
__device__ __forceinline__ int64_t imin64(int64_t a, int64_t b) { return a < b ? a : b; }

// ---------------------------------------------------------------- search

// Largest r in [0, m] with rp[r] <= b (rp non-decreasing, rp[0] <= b).
// Wave-parallel 64-ary search: each round the 64 lanes probe 64 evenly spaced
// points of (lo, hi]; the predicate rp[p] <= b holds for a prefix of lanes, so
// its ballot's popcount picks the sub-interval.
template <typename T, typename I>
__device__ __forceinline__ I wave_rightmost(const T *__restrict__ rp, I m, T b, int lane) {
  I lo = 0, hi = m;
  while (hi - lo >= kWave) {
    const int64_t span = (int64_t)(hi - lo);
    const I p = lo + (I)(((int64_t)(lane + 1) * span) / kWave);
    const uint64_t bal = __ballot(rp[p] <= b);
    const int c = __popcll(bal);
    const I newlo = c > 0 ? lo + (I)(((int64_t)c * span) / kWave) : lo;
    const I newhi = c < kWave ? lo + (I)(((int64_t)(c + 1) * span) / kWave) - 1 : hi;
    lo = newlo;
    hi = newhi;
  }
  const I p = lo + lane;
  const bool pred = (p <= hi) && (rp[p <= hi ? p : hi] <= b);
  return lo + __popcll(__ballot(pred)) - 1;
}

// ---------------------------------------------------------------- wave scans

// 64-lane scans with DPP: Hillis-Steele shifts by 1, 2, 4, 8 inside each
// 16-lane row, then row broadcasts of lane 15 (into rows 1 and 3) and lane 31
// (into rows 2 and 3).  Lanes whose source is out of range read 0, the
// identity of both scans below.
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143, kWaveShr1 = 0x138, kWaveShl1 = 0x130;

// lane l reads lane l + 1; the last lane keeps `last`
__device__ __forceinline__ int wave_next(int v, int last) {
  return __builtin_amdgcn_update_dpp(last, v, kWaveShl1, 0xf, 0xf, false);
}
// lane l reads lane l - 1; lane 0 keeps `first`
__device__ __forceinline__ int wave_prev(int v, int first) {
  return __builtin_amdgcn_update_dpp(first, v, kWaveShr1, 0xf, 0xf, false);
}
// this wavefront's index in its workgroup, in a scalar register (what hangs
// on it -- the bunch, its bounds and addresses -- then stays scalar too)
__device__ __forceinline__ int wave_in_block() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)); }
// how many of the lanes before this one are in `mask` (the same in every lane)
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
// v of lane `l`, for a lane index the same in every lane
__device__ __forceinline__ int lane_value(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

// *p for an address the same in every lane, of data no kernel of the launch
// writes (plan arrays written before it): read through the scalar unit into
// scalar registers instead of once per lane into vector registers
template <typename T>
__device__ __forceinline__ T uniform_load(const T *p) {
  static_assert(sizeof(T) % 4 == 0, "whole 32-bit words");
  typedef const __attribute__((address_space(4))) uint32_t cword;
  uint32_t w[sizeof(T) / 4];
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = ((cword *)p)[i];
  T v;
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, true);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp_i<CTRL, ROWS>((int)(unsigned long long)b);
  const int hi = dpp_i<CTRL, ROWS>((int)((unsigned long long)b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ AccD dpp_acc(const AccD &v) { AccD r; r.s = dpp_d<CTRL, ROWS>(v.s); return r; }

// one step of the segmented scan: (v, f) := (v_src, f_src) (+) (v, f), where
// (a, fa) (+) (b, fb) = (fb ? b : a + b, fa | fb)
template <int CTRL, int ROWS, class A>
__device__ __forceinline__ void seg_step(A &v, int &f) {
  const A up = dpp_acc<CTRL, ROWS>(v);
  const int fu = dpp_i<CTRL, ROWS>(f);
  if (!f) v.prepend(up);
  f |= fu;
}

// inclusive segmented scan over the wave of (v, head flag)
template <class A>
__device__ __forceinline__ void wave_seg_scan(A &v, int &f) {
  seg_step<kRowShr1, 0xf>(v, f);
  seg_step<kRowShr2, 0xf>(v, f);
  seg_step<kRowShr4, 0xf>(v, f);
  seg_step<kRowShr8, 0xf>(v, f);
  seg_step<kRowBcast15, 0xa>(v, f);
  seg_step<kRowBcast31, 0xc>(v, f);
}

// inclusive integer scan over the wave
__device__ __forceinline__ int wave_iscan(int x) {
  x += dpp_i<kRowShr1, 0xf>(x);
  x += dpp_i<kRowShr2, 0xf>(x);
  x += dpp_i<kRowShr4, 0xf>(x);
  x += dpp_i<kRowShr8, 0xf>(x);
  x += dpp_i<kRowBcast15, 0xa>(x);
  x += dpp_i<kRowBcast31, 0xc>(x);
  return x;
}

// the last lane's value, in scalar registers
__device__ __forceinline__ double last_lane(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, kWave - 1);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), kWave - 1);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// sum over the 64 lanes in a fixed tree (pairs 1 apart, 2 apart, ... 32
// apart); every lane returns the total
__device__ __forceinline__ double wave_sum_tree(double v) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) v += __shfl_xor(v, d, kWave);
  return v;
}

// Where lanes of a wavefront hand LDS words to each other, or a word changes its
// type (products of prod_t, then partials in double, in the same words).  One
// wavefront owns the words and its LDS operations run in order, so nothing
// waits; the fence keeps the compiler from moving accesses of different lanes
// or types, which it may take for independent, past each other.
__device__ __forceinline__ void lds_handover() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- stage 1

// What a bunch leaves for stage 2.  One record, stored by one instruction:
// four arrays cost a bunch four partly written cache lines, which on a 160^3
// 27-point stencil took 3 us of 266.
struct BunchState {
  double sync_val;
  double tail_val;      // its last partial, when the bunch ends inside a row that is not its first row and
                        // continues into the next bunch
  int32_t sync_idx;
  uint32_t dirty_mask;  // bit t: tile t is dirty
};
static_assert(sizeof(BunchState) == 24, "six words");

// One matrix as the kernels see it: the caller's arrays, sizes, and the
// plan's auxiliary arrays for this matrix (already offset to it).
struct MatCtx {
  const int32_t *row_ptr;
  const int32_t *col;
  const void *val;
  const void *x;
  void *y;
  int32_t m;
  int32_t nnz;
  int32_t S;
  int32_t W;
  int64_t n_bunches;
  int64_t n_tiles;
  BunchState *state;     // per bunch
  int4 *speculator;      // per bunch, S slots: <start, stop, tile, 0> of its dirty tiles, packed
  const int32_t *bunch_row;  // per bunch: its first row, found at plan time (NULL: search); the top
                             // bit is set on the bunches listed in dirty_list
  const int32_t *dirty_list; // bound plans: the bunches whose tiles the plan found dirty (NULL: every
                             // bunch gets a stage-2 wavefront)
  int64_t n_fix;             // stage-2 re-arrangement wavefronts: entries of dirty_list, else n_bunches
  int32_t *stale;            // bound plans: set (and never cleared) when stage 1 finds a dirty tile in a
                             // bunch outside dirty_list (row_ptr rewritten in place since plan time)
  int32_t carries;       // fused kernel: a sss_carries launch follows and completes the rows that cross
  int32_t keep_state;    // fused kernel: every bunch stores its state
  int32_t *arrivals;     // bound plans, per bunch: see finish_row (zero between launches)
  const int4 *slots;     // bound plans (and calls that made them), per wavefront slot: <bunch (-1: none), its first row (top bit: listed in
                         // dirty_list), slot_need, 0>; NULL: slot = bunch
  int64_t n_slots;
  int64_t n_shares;      // fused kernel, single matrices: its wavefronts, which share the leading rows
  int32_t *dbg_start;    // debug plans only
  int32_t *dbg_dirty;
  uint32_t *dbg_heads;
};

// LDS words per wavefront: S tiles of descriptor bits, the dirty-tile bits
// (padded to 2 words), then W*T double slots for one tile's compact partials.
__host__ __device__ constexpr int stage1_lds_words(int W, int S) { return S * (W * kWave / 32) + 2 + 2 * W * kWave; }

// Grouped order of a tile's entries: the tile is W/G rows of 64*G entries,
// and lane j holds G consecutive entries of every row, so entry (r, g) of
// lane j (array index r*G + g) is tile offset r*64*G + j*G + g.  G entries
// of the value type make 16 bytes (G = W when that is fewer), so every load
// instruction of the wavefront reads one contiguous 1-KiB stretch of val,
// and the x gathers of one instruction fall on 64*G consecutive nonzeros.
template <int DT> constexpr int group_of() { return DT == SSS_F64 ? 2 : (DT == SSS_F32 ? 4 : 8); }
template <int DT, int W> constexpr int group_w() { return group_of<DT>() < W ? group_of<DT>() : W; }

template <int G>
__device__ __forceinline__ void load_cols_g(const int32_t *__restrict__ p, int *c) {
  if constexpr (G == 2) {
    const v2u v = stream_load(reinterpret_cast<const v2u *>(p));
    c[0] = (int)v.x; c[1] = (int)v.y;
  } else {
#pragma unroll
    for (int i = 0; i < G / 4; ++i) {
      const v4i v = stream_load(reinterpret_cast<const v4i *>(p) + i);
      c[4 * i] = v.x; c[4 * i + 1] = v.y; c[4 * i + 2] = v.z; c[4 * i + 3] = v.w;
    }
  }
}

template <int G>
__device__ __forceinline__ void load_vals_g(const double *__restrict__ p, double *a) {
  static_assert(G % 2 == 0, "double groups are pairs");
#pragma unroll
  for (int i = 0; i < G / 2; ++i) {
    const v2d v = stream_load(reinterpret_cast<const v2d *>(p) + i);
    a[2 * i] = v.x; a[2 * i + 1] = v.y;
  }
}
template <int G>
__device__ __forceinline__ void load_vals_g(const float *__restrict__ p, float *a) {
  static_assert(G % 4 == 0, "float groups are quadruples");
#pragma unroll
  for (int i = 0; i < G / 4; ++i) {
    const v4f v = stream_load(reinterpret_cast<const v4f *>(p) + i);
    a[4 * i] = v.x; a[4 * i + 1] = v.y; a[4 * i + 2] = v.z; a[4 * i + 3] = v.w;
  }
}
template <int G>
__device__ __forceinline__ void load_vals_g(const uint16_t *__restrict__ p, float *a) {
  if constexpr (G == 8) {
    const v4u v = stream_load(reinterpret_cast<const v4u *>(p));
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) { a[2 * j] = bf16_to_f32(w[j] & 0xffffu); a[2 * j + 1] = bf16_to_f32(w[j] >> 16); }
  } else {
    static_assert(G == 4, "bfloat16 groups are 4 or 8");
    const v2u v = stream_load(reinterpret_cast<const v2u *>(p));
    a[0] = bf16_to_f32(v.x & 0xffffu); a[1] = bf16_to_f32(v.x >> 16);
    a[2] = bf16_to_f32(v.y & 0xffffu); a[3] = bf16_to_f32(v.y >> 16);
  }
}

// col/val of one tile in the grouped order; entries past nnz read as column 0
// with value 0.
template <int DT, int W, typename val_t, typename prod_t>
__device__ __forceinline__ void load_tile_g(const int32_t *__restrict__ col, const val_t *__restrict__ val, int b,
                                            int nnz, int lane, int (&c)[W], prod_t (&av)[W]) {
  constexpr int G = group_w<DT, W>();
  constexpr int R = W / G;
  if (b + W * kWave <= nnz) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int k0 = b + r * kWave * G + lane * G;
      load_cols_g<G>(col + k0, &c[r * G]);
      load_vals_g<G>(val + k0, &av[r * G]);
    }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int k = b + r * kWave * G + lane * G + g;
        const bool in = k < nnz;
        c[r * G + g] = in ? col[k] : 0;
        av[r * G + g] = in ? (prod_t)scalar_val(val, k) : (prod_t)0;
      }
  }
}

// The products leave the grouped order through LDS: each lane writes its G
// products of every row as 16-byte chunks, then reads back the W products
// of tile offsets lane*W .. lane*W+W-1 (the order the segmented sum walks).
// 16-byte chunk c is stored at chunk c ^ ((c >> 4) & (K - 1)), K = the chunks
// one lane reads: the 16 lanes of a read then touch 16 different chunk
// columns of a 256-byte LDS row, as do the lanes of a write.
template <typename P, int W>
__device__ __forceinline__ int tr_chunk(int c) {
  constexpr int K = (W * (int)sizeof(P)) / 16 > 0 ? (W * (int)sizeof(P)) / 16 : 1;
  return c ^ ((c >> 4) & (K - 1));
}

template <int DT, int W, typename P>
__device__ __forceinline__ void products_out(const P (&av)[W], const P (&xv)[W], P *buf, int lane, P (&pr)[W]) {
  constexpr int G = group_w<DT, W>();
  constexpr int R = W / G;
  constexpr int CH = 16 / (int)sizeof(P);  // products per 16-byte chunk
  static_assert(W % CH == 0, "a lane's products fill whole chunks");
  if constexpr (G == W) {
    // one row per tile: the grouped order is the lane order already
#pragma unroll
    for (int i = 0; i < W; ++i) pr[i] = av[i] * xv[i];
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < G / CH; ++t) {
        const int c = (r * kWave * G + lane * G) / CH + t;
        P *dst = buf + tr_chunk<P, W>(c) * CH;
#pragma unroll
        for (int e = 0; e < CH; ++e) dst[e] = av[r * G + t * CH + e] * xv[r * G + t * CH + e];
      }
  }
}

template <int W, typename P>
__device__ __forceinline__ void products_read(const P *buf, int lane, P (&pr)[W]) {
  constexpr int CH = 16 / (int)sizeof(P);
  lds_handover();
#pragma unroll
  for (int k = 0; k < W / CH; ++k) {
    const P *src = buf + tr_chunk<P, W>((lane * W) / CH + k) * CH;
#pragma unroll
    for (int e = 0; e < CH; ++e) pr[k * CH + e] = src[e];
  }
  lds_handover();  // the same words take the partials next
}

template <int DT, int W, typename P>
__device__ __forceinline__ void products_in(const P *buf, int lane, P (&pr)[W]) {
  if constexpr (group_w<DT, W>() != W) products_read<W>(buf, lane, pr);
}

template <int DT, int W, bool DEBUG>
__device__ __forceinline__ void stage1_bunch(const MatCtx &a, const int64_t tb, uint32_t *lds_wave, const int lane,
                                             const int32_t brow) {
  using val_t = typename VT<DT>::val_t;
  using x_t = typename VT<DT>::x_t;
  using y_t = typename VT<DT>::y_t;
  using prod_t = typename VT<DT>::prod_t;
  constexpr int WT = W * kWave;
  constexpr int WPT = WT / 32;  // descriptor words per tile
  constexpr uint32_t LOW = (W >= 32) ? 0xffffffffu : ((1u << W) - 1u);

  const int32_t *__restrict__ rp = a.row_ptr;
  const int32_t *__restrict__ col = a.col;
  const val_t *__restrict__ val = static_cast<const val_t *>(a.val);
  const x_t *__restrict__ x = static_cast<const x_t *>(a.x);
  y_t *__restrict__ y = static_cast<y_t *>(a.y);
  const int m = a.m, nnz = a.nnz, S = a.S;
  uint32_t *mask = lds_wave;
  uint32_t *dflag = mask + S * WPT;
  double *part = reinterpret_cast<double *>(mask + S * WPT + 2);

  const int64_t SWT = (int64_t)S * WT;
  const int b0 = (int)(tb * SWT);  // < nnz
  const int bS = (int)imin64(tb * SWT + SWT, nnz);

  // ---- tile 0's col/val do not depend on the row structure: issue first
  int cc[W];
  prod_t av[W];
  load_tile_g<DT, W>(col, val, b0, nnz, lane, cc, av);

  // ---- tile boundary search (rightmost match) for the bunch's first row,
  // unless the plan found it once for all calls; such a row is checked in the
  // row pass below
  // brow: -1 = search for the first row; else the first row found at plan
  // time, top bit set when the plan listed this bunch as dirty (decoded
  // here, after tile 0's loads are issued, so nothing waits for it earlier)
  const bool known = brow != -1;
  const bool listed = brow < 0;
  int r0 = known ? (brow & 0x7fffffff) : wave_rightmost(rp, m, b0, lane);
  bool verify = known;

  // ---- x gathers of tile 0: they need only the columns, so they go out
  // before the row pass and travel with its loads
  prod_t xv[W];
#pragma unroll
  for (int i = 0; i < W; ++i) xv[i] = (prod_t)x[cc[i]];

  // ---- descriptor, tile start rows, dirty tiles: one pass over the rows
  for (int i = lane; i < S * WPT; i += kWave) mask[i] = 0u;
  if (lane == 0) *dflag = 0u;
  lds_handover();

  const int my_b = (int)imin64(tb * SWT + (int64_t)min(lane, S) * WT, nnz);
  int my_count = 0;  // lane t <= S: rows r >= r0 with rp[r] <= b_t
  int my_rp = 0;     // lane t <= S: rp of the last such row (the tile's start row)
  for (int rbase = __builtin_amdgcn_readfirstlane(r0);; rbase += kWave) {
    const int r = rbase + lane;
    const int p = (r <= m) ? rp[r] : INT_MAX;
    // q = rp[r + 1]: the next lane's p, and one uniform load for the last lane
    const int q = wave_next(p, (rbase + kWave - 1 < m) ? rp[rbase + kWave] : INT_MAX);
    if (verify) {
      // a row found at plan time is the rightmost match of b0 exactly when
      // rp[r0] <= b0 < rp[r0 + 1]; if row_ptr no longer says so, search
      // (the pass has accumulated nothing yet)
      verify = false;
      const int p0 = lane_value(p, 0), q0 = lane_value(q, 0);
      if (!(p0 <= b0 && b0 < q0)) {
        r0 = __builtin_amdgcn_readfirstlane(wave_rightmost(rp, m, b0, lane));
        rbase = r0 - kWave;
        continue;
      }
    }
    if (r < m && q > p && p >= b0 && p < bS) {
      const int off = p - b0;
      atomicOr(&mask[off >> 5], 1u << (off & 31));
    }
    // an empty row at position p lies in rows start..stop-1 of the tile t
    // with b_t < p <= b_{t+1}
    if (r < m && q == p && p > b0 && p <= bS) atomicOr(dflag, 1u << ((p - b0 - 1) / WT));
    for (int t = 0; t <= S; ++t) {
      // rows with rp <= b_t are a prefix of the chunk; the last of them
      // (so far) is the start row of tile t
      const int bt = lane_value(my_b, t);
      const int c = __popcll(__ballot(p <= bt));
      const int p_last_in = lane_value(p, c > 0 ? c - 1 : 0);
      if (lane == t) {
        my_count += c;
        if (c > 0) my_rp = p_last_in;
      }
    }
    const int p_last = lane_value(p, kWave - 1);
    if (!(p_last <= bS && rbase + (kWave - 1) < m)) break;
  }
  lds_handover();
  const uint32_t dirty_bits = *dflag;
  const int my_start = (lane <= S) ? r0 + my_count - 1 : 0;

  double transmitter = 0.0;
  double sync_v = 0.0;
  for (int t = 0; t < S; ++t) {
    const int64_t b64 = tb * SWT + (int64_t)t * WT;
    if (b64 >= nnz) break;
    const int b = (int)b64;
    const int e = (int)imin64(b64 + WT, nnz);
    const int start = lane_value(my_start, t);
    const int stop = lane_value(my_start, t + 1);
    const int rp_stop = lane_value(my_rp, t + 1);
    const bool ends_mid = (stop < m) && (rp_stop < e);
    const bool dirty = (dirty_bits >> t) & 1u;
    const int64_t tile = tb * S + t;
    const bool has_next = (t + 1 < S) && (b64 + WT < nnz);

    // ---- prefetch the next tile's col/val; products of this tile
    int cn[W];
    prod_t an[W];
    if (has_next) load_tile_g<DT, W>(col, val, b + WT, nnz, lane, cn, an);
    // ---- this lane's W descriptor bits; the tile's first bit is forced
    uint32_t hb = (mask[t * WPT + ((lane * W) >> 5)] >> ((lane * W) & 31)) & LOW;
    const bool bit0 = __builtin_amdgcn_readlane((int)hb, 0) & 1;
    if (lane == 0) hb |= 1u;
    const double tx = bit0 ? 0.0 : transmitter;  // carry into a tile that starts mid-row
    if (DEBUG) {
      for (int w = lane; w < WPT; w += kWave) {
        uint32_t word = mask[t * WPT + w];
        if (w == 0) word |= 1u;
        a.dbg_heads[tile * WPT + w] = word;
      }
      if (lane == 0) {
        a.dbg_start[tile] = start;
        a.dbg_dirty[tile] = dirty ? 1 : 0;
      }
    }

    // ---- exclusive scan of head counts: the compact index of every partial
    // (integers only, so it does not wait for the products)
    const int c_heads = __popc(hb);
    const int incl = wave_iscan(c_heads);
    const int cnt = __builtin_amdgcn_readlane(incl, kWave - 1);
    const int rank0 = incl - c_heads;  // segments closed before this lane's first head

    // ---- one pass over the lane's products.  `pre` = the entries before the
    // lane's first head (they continue a segment opened in an earlier lane);
    // every later head closes a segment that lies wholly in this lane, whose
    // partial goes to its LDS slot at once; `run` = the entries after the
    // last head (a segment still open at the lane's end).
    // ---- the lane's W products, from the grouped order of the loads to the
    // order of its entries lane*W .. lane*W+W-1, through `part` (no partial
    // is staged there yet); the next tile's x gathers go out in between
    prod_t pr[W];
    products_out<DT, W>(av, xv, reinterpret_cast<prod_t *>(part), lane, pr);
    if (has_next) {
#pragma unroll
      for (int i = 0; i < W; ++i) { xv[i] = (prod_t)x[cn[i]]; av[i] = an[i]; }
    }
    products_in<DT, W>(reinterpret_cast<const prod_t *>(part), lane, pr);
    // one running sum per lane: before the lane's first head it is the part
    // of a segment opened in an earlier lane (pre); every later head closes
    // the segment summed so far, whose partial goes to its LDS slot at once.
    // At the first head the running sum is staged at that segment's slot
    // too (q - 1 = rank0 - 1, or 0 for the tile's first entry); the segment's
    // full sum overwrites it after the wave scan.  The transmitter is added
    // to the tile's first partial where that partial is read.
    AccD acc, pre;
    acc.zero();
    pre.zero();
    bool seen = false;
    int q = rank0;  // slot of the segment that the lane's next head closes, plus one
#pragma unroll
    for (int i = 0; i < W; ++i) {
      if ((hb >> i) & 1u) {
        part[q > 0 ? q - 1 : 0] = acc.value();
        if (!seen) pre = acc;
        seen = true;
        ++q;
        acc.zero();
      }
      acc.add(pr[i]);
    }
    if (!seen) pre = acc;
    // ---- wave segmented scan of the open segments (the lane's running
    // sum: its run after the last head, or all of it); carry into each lane
    AccD inc = acc;
    int f = seen ? 1 : 0;
    wave_seg_scan(inc, f);
    const AccD carry = dpp_acc<kWaveShr1, 0xf>(inc);

    // ---- the segment closed by this lane's first head: carry + pre; the
    // segment open at the tile's end (last lane): its run, or carry + pre
    // when the last lane holds no head
    if (seen && rank0 > 0) {
      AccD c = pre;
      c.prepend(carry);
      part[rank0 - 1] = c.value();
    }
    if (lane == kWave - 1) {
      AccD c = pre;
      c.prepend(carry);
      part[cnt - 1] = seen ? acc.value() : c.value();
    }
    lds_handover();

    // ---- coalesced store of the compact partials to y[start + q] (the
    // first with the transmitter added).  Two partials stay in double
    // instead: the bunch's first segment goes to the synchronizer, and the
    // last partial of a tile that ends inside row `stop` is not stored -- it
    // travels on in the transmitter to the next tile of the bunch, which
    // stores the row's sum, or, after the bunch's last tile, to the bunch's
    // tail, which stage 2 adds to the row's carries before the row's only
    // rounding to y's type.
    for (int q = lane; q < cnt; q += kWave) {
      const bool last = (q == cnt - 1);
      const int idx = start + q;
      if (!(q == 0 && start == r0) && !(last && ends_mid) && (unsigned)idx < (unsigned)m) {
        double v = part[q];
        if (q == 0) v += tx;
        y_store((y_t)v, &y[idx]);
      }
    }
    const double p0 = part[0] + tx;
    const double plast = cnt == 1 ? p0 : part[cnt - 1];
    if (start == r0) sync_v = p0;
    transmitter = ends_mid ? plast : 0.0;
    if (!has_next && ends_mid && !(cnt == 1 && start == r0) && lane == 0) a.state[tb].tail_val = plast;
    lds_handover();

    // ---- dirty tile: label it for the re-arrangement, in this bunch's own
    // speculator slots (no global counter)
    if (dirty && lane == 0) {
      const int slot = __popc(dirty_bits & ((1u << t) - 1u));
      a.speculator[tb * S + slot] = make_int4(start, stop, (int)tile, 0);
    }
  }
  if (lane == 0) {
    a.state[tb].sync_idx = r0;
    a.state[tb].sync_val = sync_v;
    a.state[tb].dirty_mask = dirty_bits;
    // a bound plan re-arranges only the bunches it listed; a dirty tile
    // anywhere else sends stage 2 to its fallback for every later call
    if (dirty_bits && !listed && a.stale) *a.stale = 1;
  }
}


template <int DT, int W, bool DEBUG>
__global__ __launch_bounds__(256) void sss_stage1(MatCtx a) {
  extern __shared__ uint32_t lds_words[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  int64_t tb = (int64_t)blockIdx.x * (blockDim.x / kWave) + wid;
  if (a.slots) {
    if (tb >= a.n_slots) return;
    tb = __builtin_amdgcn_readfirstlane(a.slots[tb].x);
    if (tb < 0) return;
  } else if (tb >= a.n_bunches) {
    return;
  }
  const int32_t brow = a.bunch_row ? a.bunch_row[tb] : -1;
  stage1_bunch<DT, W, DEBUG>(a, tb, lds_words + wid * stage1_lds_words(W, a.S), lane, brow);
}

// ---------------------------------------------------------------- fused kernel

// Execute's kernel: stage 1 and, for its own bunch, the work of stage 2, so
// that y needs no second launch.
//  * A dirty tile stores its partials straight to its non-empty rows and
//    zeroes the empty ones, from row_ptr and the partials in LDS, instead of
//    storing them side by side for a re-arrangement to read back.
//  * Where no row that crosses into a bunch began more than kBack nonzeros
//    before it (no long crossing row, a plan finds: MatCtx::carries = 0), the
//    bunch in which a row ends loads and sums those itself (back_sum), and the
//    bunch before drops its tail: no second launch, and no bunch waits for
//    another.  Else sss_carries completes the rows that cross, adding the
//    synchronizer entries in double as stage 2 does (see back_limit).  A long
//    crossing row of a row_ptr rewritten in place since the plan saw none is
//    added up by the last of its bunches to finish (finish_row).
//  * The leading empty rows are shared out over the bunches.
//
// What bounds it is the latency of the loads a wavefront waits for one after
// the other, so every load goes out as early as its address is known: the
// first two tiles' columns and values, the row pointers and the entries
// before the bunch at once, tile 0's gathers behind them; in the tile loop
// the gathers of tile t + 1 (whose columns came in while tile t - 1 was
// summed) and the columns and values of tile t + 2 go out before tile t is
// summed.  The loads are buffer loads whose range ends with the bunch: past
// it they return 0 without touching memory, so nothing in the loop branches
// on what is left (a branch around a load makes the compiler wait for every
// load in flight where the paths meet), and one 32-bit offset replaces a
// 64-bit address per load.
//
// Per product, the two launches before / this kernel (and sss_carries where
// needed): 160^3 27-point stencil FP64 276 / 262 us (1.39 GB: 5.0 / 5.3
// TB/s), 1414^2 5-point stencil FP64 39.9 / 31.9 us (160 MB: 4.0 / 5.0 TB/s),
// FEM band 778K x 50 FP32 74.2 / 61.7 us (320 MB: 4.3 / 5.2 TB/s), 1M-row
// power law FP64 182.9 / 171 us and BF16 117.8 / 111 us (both in column
// order), 30K-row web-like FP32 12.3 / 5.8 to 7.3 us over boxes (5.8 us of that is
// the host's call; it was 9.3).  The double sums gave the band 2.5 of its 12 us.
constexpr int kBack = kWave;

// Row [rs, re) against the bunch [b0, b0 + SWT) that holds some of it: is it
// a long crossing row (left to sss_carries)?  back: how many entries before the
// bunch it may begin.
__device__ __forceinline__ bool long_crossing(int64_t rs, int64_t re, int64_t b0, int64_t SWT, int back) {
  return re > b0 + SWT ? true : rs < b0 - back;
}
// Where the plan (or an unbound call) makes the carry launch anyway, it takes
// every row that crosses: reading the entries before each bunch again would
// only cost.  With / without that, us per product at W = 4, S = 1: 100K rows of 70
// bound 41.7 / 38.4, searched 52.1 / 47.2 (two stages 39.4, 48.2); 50K Poisson
// rows of 60 FP32, the selector's plan, 18.1 / 16.9; 256 uneven matrices 707 / 702.
__device__ __forceinline__ int back_limit(bool carries) { return carries ? 0 : kBack; }

// How the loads go out.
//  kCached: plain loads.
//  kStreamed: the columns and values as non-temporal loads, which leave L2 to
//    x.  Faster where the matrix comes from memory anyway, slower where much
//    of it would still be cached at the next product (see form_of).
//  kWide: streamed, and x is 4 GB or more, past a buffer load's 32-bit offset.
enum Form { kCached, kStreamed, kWide };

// What a plan tells a bunch of its first row, rp[r0] <= b0 < rp[r0 + 1]: its
// entries before the bunch that the bunch sums itself (7 bits), and above them how many entries of row_ptr after
// rp[r0] the bunch needs, up to the first that is past its end (kSpanMax: that
// many or more, which the bunch finds itself).
constexpr int kSpanMax = 1 << 22;
// r_next: the next bunch's first row, m after the last bunch.
__device__ __forceinline__ int slot_need(const int32_t *__restrict__ rp, int32_t m, int64_t SWT, int64_t tb, int32_t r,
                                         int32_t r_next, bool carries) {
  const int64_t b0 = tb * SWT;
  const int back =
      r < m && !long_crossing(rp[r], rp[r + 1], b0, SWT, back_limit(carries)) ? (int)(b0 - rp[r]) : 0;
  return back | (int)imin64((int64_t)(r_next < m ? r_next + 1 : m) - r, kSpanMax) << 8;
}

// Buffer loads: the descriptor's range is in bytes, checked per 32-bit word
// against the vector offset.  The instruction's scalar offset is not part of
// that check, so it stays 0: what moves along an array moves the descriptor.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kRsrcWord3 = 0x00020000;  // raw buffer, 32-bit data format
__device__ __forceinline__ rsrc_t make_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, kRsrcWord3);
}
template <typename T, bool NT = false>
__device__ __forceinline__ T buffer_load(rsrc_t r, int voffset) {
  constexpr int kAux = NT ? 2 : 0;
  static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "one load");
  T v;
  if constexpr (sizeof(T) == 2) {
    const auto w = __builtin_amdgcn_raw_buffer_load_b16(r, voffset, 0, kAux);
    __builtin_memcpy(&v, &w, 2);
  } else if constexpr (sizeof(T) == 4) {
    const auto w = __builtin_amdgcn_raw_buffer_load_b32(r, voffset, 0, kAux);
    __builtin_memcpy(&v, &w, 4);
  } else if constexpr (sizeof(T) == 8) {
    const auto w = __builtin_amdgcn_raw_buffer_load_b64(r, voffset, 0, kAux);
    __builtin_memcpy(&v, &w, 8);
  } else {
    const auto w = __builtin_amdgcn_raw_buffer_load_b128(r, voffset, 0, kAux);
    __builtin_memcpy(&v, &w, 16);
  }
  return v;
}

// The fused kernel's grouped order (see group_of): G entries of a lane are
// consecutive.  Two for FP64 and four for FP32 are 16 bytes of values; BF16
// takes four as well, 8 bytes: its gathers then fall on half as many
// consecutive nonzeros as with eight, which on a 160^3 27-point stencil is
// worth 20 of 186 us (1M-row power law 111.0 / 106.2, FEM band 57.0 / 53.3;
// 5-point stencils 0.5% slower).  One or two for the others measured 4 to 12%
// slower on stencils and batches (more registers for the same bytes).
template <int DT> constexpr int fused_group() { return DT == SSS_F64 ? 2 : 4; }

template <int N, bool NT>
__device__ __forceinline__ void load_words(rsrc_t r, int voffset, uint32_t *w) {
  if constexpr (N == 1) {
    w[0] = buffer_load<uint32_t, NT>(r, voffset);
  } else if constexpr (N == 2) {
    const v2u v = buffer_load<v2u, NT>(r, voffset);
    w[0] = v.x; w[1] = v.y;
  } else {
    static_assert(N % 4 == 0, "1, 2 or quadruples of words");
#pragma unroll
    for (int i = 0; i < N; i += 4) {
      const v4u v = buffer_load<v4u, NT>(r, voffset + 4 * i);
      w[i] = v.x; w[i + 1] = v.y; w[i + 2] = v.z; w[i + 3] = v.w;
    }
  }
}

// One tile's columns and stored values, as loaded.
template <int DT, int W>
struct Tile {
  static constexpr int G = fused_group<DT>(), R = W / G;
  static constexpr int VB = (int)sizeof(typename VT<DT>::val_t);
  static constexpr int VW = G * VB / 4;  // words of values per row
  uint32_t c[W], v[R * VW];

  // rc, rv: descriptors that begin with the tile
  template <bool NT>
  __device__ __forceinline__ void load(rsrc_t rc, rsrc_t rv, int lane) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      load_words<G, NT>(rc, lane * G * 4 + r * kWave * G * 4, &c[r * G]);
      load_words<VW, NT>(rv, lane * G * VB + r * kWave * G * VB, &v[r * VW]);
    }
  }
  __device__ __forceinline__ uint32_t column(int i) const { return c[i]; }
  __device__ __forceinline__ typename VT<DT>::prod_t value(int i) const {
    if constexpr (DT == SSS_F64)
      return __longlong_as_double((long long)((uint64_t)v[2 * i] | ((uint64_t)v[2 * i + 1] << 32)));
    else if constexpr (DT == SSS_F32)
      return __uint_as_float(v[i]);
    else
      return __uint_as_float(i % 2 ? v[i / 2] & 0xffff0000u : v[i / 2] << 16);
  }
  // where in the tile a lane's entry i is
  __device__ __forceinline__ static int offset(int i, int lane) { return (i / G) * kWave * G + lane * G + i % G; }

  // the products into LDS, in the layout that products_read reads, or into
  // pr where the loads' order is the lane order
  template <typename P>
  __device__ __forceinline__ static void store(const P (&av)[W], const P (&bv)[W], P *buf, int lane, P (&pr)[W]) {
    if constexpr (G == W) {
#pragma unroll
      for (int i = 0; i < W; ++i) pr[i] = av[i] * bv[i];
    } else {
      constexpr int CH = 16 / (int)sizeof(P);
      static_assert(CH == G, "a lane's consecutive entries are one chunk");
#pragma unroll
      for (int i = 0; i < W; i += G) {
        P *dst = buf + tr_chunk<P, W>(offset(i, lane) / CH) * CH;
#pragma unroll
        for (int g = 0; g < G; ++g) dst[g] = av[i + g] * bv[i + g];
      }
    }
  }
};

// The sum of row entries rs .. b0-1, the part of a row before the bunch that
// begins at b0; lane l holds the product of entry b0 - kBack + l.  Up to
// kBack of them are summed as the bunch before sums its tail (its last lanes,
// W entries each, then the wave scan), so y is the same bit for bit wherever
// the row's parts are added.
template <int DT, int W, typename prod_t>
__device__ __forceinline__ double back_sum(prod_t product, int rs, int b0, double *lds, int lane) {
  prod_t *buf = reinterpret_cast<prod_t *>(lds);
  buf[lane] = product;
  lds_handover();
  constexpr int kFirst = kWave - kBack / W;  // the first lane whose entries are among the last kBack
  AccD acc;
  acc.zero();
  if (lane >= kFirst) {
#pragma unroll
    for (int i = 0; i < W; ++i) acc.add(buf[(lane - kFirst) * W + i]);
  }
  lds_handover();
  const int head = kFirst + (rs - (b0 - kBack)) / W;
  AccD inc = acc;
  int f = lane == head ? 1 : 0;
  wave_seg_scan(inc, f);
  const AccD carry = dpp_acc<kWaveShr1, 0xf>(inc);
  AccD c = acc;
  if (head != kWave - 1) c.prepend(carry);
  return last_lane(c.value());
}

// What the tiles of a bunch share.  DOT (square FP64 matrices): beside y, the
// sum of x[r] y[r] over the rows that the bunch writes.
template <int DT, int W, bool DOT>
struct Bunch {
  using y_t = typename VT<DT>::y_t;
  using prod_t = typename VT<DT>::prod_t;
  const int32_t *__restrict__ rp;
  y_t *__restrict__ y;
  int4 *speculator;      // this bunch's slots, or NULL
  uint32_t *mask;        // LDS: descriptor bits
  double *part;          // LDS: products, then partials, of one tile
  int m, lane, r0, first_tile;
  uint32_t dirty_bits;
  int my_start, my_rp;   // lane t: tile t's start row and its row_ptr
  uint64_t filled_rows;  // lane c: which of the rows r0 + 64 c + 0 .. 63 hold entries
  double transmitter, sync_v;
  const double *x;  // DOT only, as the next three
  double x_row;     // x of row start + lane of the tile
  double dot;

  // x of the tile's rows, loaded ahead of the next tile's gathers so that the
  // store loop need not wait for those
  __device__ __forceinline__ void load_rows(int t) {
    if constexpr (DOT) x_row = x[min(lane_value(my_start, t) + lane, m - 1)];
  }

  // The segmented sum of tile t, entries b .. e-1 of the matrix, whose
  // products lie in `part` (in `pr` where the loads' order is the lane order);
  // as in stage1_bunch.
  __device__ __forceinline__ double sum_tile(int t, int e, prod_t (&pr)[W]) {
    constexpr int WT = W * kWave;
    constexpr int WPT = WT / 32;
    constexpr uint32_t LOW = (W >= 32) ? 0xffffffffu : ((1u << W) - 1u);
    const int start = lane_value(my_start, t);
    const int stop = lane_value(my_start, t + 1);
    const bool ends_mid = (stop < m) && (lane_value(my_rp, t + 1) < e);
    const bool dirty = (dirty_bits >> t) & 1u;

    uint32_t hb = (mask[t * WPT + ((lane * W) >> 5)] >> ((lane * W) & 31)) & LOW;
    const bool bit0 = __builtin_amdgcn_readlane((int)hb, 0) & 1;
    if (lane == 0) hb |= 1u;
    const double tx = bit0 ? 0.0 : transmitter;

    const int c_heads = __popc(hb);
    const int incl = wave_iscan(c_heads);
    const int cnt = __builtin_amdgcn_readlane(incl, kWave - 1);
    const int rank0 = incl - c_heads;

    if constexpr (fused_group<DT>() != W) products_read<W>(reinterpret_cast<const prod_t *>(part), lane, pr);
    AccD acc, pre;
    acc.zero();
    pre.zero();
    bool seen = false;
    int q = rank0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      if ((hb >> i) & 1u) {
        part[q > 0 ? q - 1 : 0] = acc.value();
        if (!seen) pre = acc;
        seen = true;
        ++q;
        acc.zero();
      }
      acc.add(pr[i]);
    }
    if (!seen) pre = acc;
    AccD inc = acc;
    int f = seen ? 1 : 0;
    wave_seg_scan(inc, f);
    const AccD carry = dpp_acc<kWaveShr1, 0xf>(inc);
    if (seen && rank0 > 0) {
      AccD c = pre;
      c.prepend(carry);
      part[rank0 - 1] = c.value();
    }
    if (lane == kWave - 1) {
      AccD c = pre;
      c.prepend(carry);
      part[cnt - 1] = seen ? acc.value() : c.value();
    }
    lds_handover();

    if (dirty) {
      // rows start + 1 .. stop - 1: the k-th non-empty one takes partial k
      // (k >= 1), the empty ones 0.  Which are empty the row pass has kept for
      // its first 64 chunks (row_ptr read again here would make the tile wait
      // for every load in flight).
      if (lane == 0 && start != r0 && !(cnt == 1 && ends_mid)) {
        y_store((y_t)(part[0] + tx), &y[start]);
        if constexpr (DOT) dot += x_row * (part[0] + tx);
      }
      // (a loop of its own past those, with the next chunk's entries read ahead,
      // is 12% faster there and costs every kernel 0.3 us: 60K Poisson rows 7.3
      // for 6.9 us)
      int k = 1;
      for (int c = (start + 1 - r0) / kWave; r0 + c * kWave < stop; ++c) {
        const int r = r0 + c * kWave + lane;
        const bool in = r > start && r < stop;
        uint64_t filled;
        if (c < kWave) {
          filled = ((uint64_t)(uint32_t)lane_value((int)(filled_rows >> 32), c) << 32) |
                   (uint32_t)lane_value((int)(uint32_t)filled_rows, c);
          filled &= __ballot(in);
        } else {
          filled = __ballot(in && rp[r] != rp[r + 1]);
        }
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(filled);
        const double v = part[min(k + lanes_below(filled), WT - 1)];
        if (in) y_store(mine ? (y_t)v : (y_t)0, &y[r]);
        if constexpr (DOT)
          if (mine) dot += x[r] * v;
        k += __popcll(filled);
      }
      if (lane == 0 && speculator)
        speculator[__popc(dirty_bits & ((1u << t) - 1u))] = make_int4(start, stop, first_tile + t, 0);
    } else {
      for (int q = lane; q < cnt; q += kWave) {
        const bool last = (q == cnt - 1);
        const int idx = start + q;
        if (!(q == 0 && start == r0) && !(last && ends_mid) && (unsigned)idx < (unsigned)m) {
          double v = part[q];
          if (q == 0) v += tx;
          y_store((y_t)v, &y[idx]);
          if constexpr (DOT) dot += (q < kWave ? x_row : x[idx]) * v;
        }
      }
    }
    const double p0 = part[0] + tx;
    const double plast = cnt == 1 ? p0 : part[cnt - 1];
    if (start == r0) sync_v = p0;
    transmitter = ends_mid ? plast : 0.0;
    lds_handover();
    // the tail, where this is the bunch's last tile: what its last row holds
    // of it, unless that row is the bunch's first (then the synchronizer's)
    return ends_mid && !(cnt == 1 && start == r0) ? plast : 0.0;
  }
};

// The rows before the first non-empty one are empty and in no tile: zero those
// of this wavefront's share of y, where rp[1] = 0.  (A row_ptr read per 64 rows
// made the wavefront wait for each: 4M such rows before 1,000 rows of 5
// entries, on two bunches, took 9.9 ms a product; the stores alone 0.96 ms, and
// shared out over more wavefronts than bunches, see kLeadingRows, 20 us.)
template <typename YT>
__device__ __forceinline__ void zero_leading(const int32_t *__restrict__ rp, YT *__restrict__ y, int m, int64_t share,
                                             int64_t shares, int lane) {
  const int64_t lo = (int64_t)m * share / shares, hi = (int64_t)m * (share + 1) / shares;
  if (lo >= hi || rp[lo + 1] != 0) return;
  const int64_t end = rp[hi] == 0 ? hi : (int64_t)wave_rightmost(rp, m, 0, lane);
  // 16 bytes a lane: what bounds a wavefront here is how many stores it may have
  // in flight
  constexpr int N = 16 / (int)sizeof(YT);
  typedef YT many __attribute__((ext_vector_type(N), aligned(sizeof(YT))));
  for (int64_t r = lo + lane * N; r < end; r += kWave * N) {
    if (r + N <= end) {
      *reinterpret_cast<many *>(y + r) = (many)(YT)0;
    } else {
      for (int64_t i = r; i < end; ++i) y[i] = (YT)0;
    }
  }
}

// The sum of entries first .. end - 1, all of one row, by one wavefront.
template <int DT>
__device__ __forceinline__ double row_part(const MatCtx &a, int first, int end, int lane) {
  constexpr int U = 4;
  const auto *val = static_cast<const typename VT<DT>::val_t *>(a.val);
  const auto *x = static_cast<const typename VT<DT>::x_t *>(a.x);
  double sum = 0.0;
  for (int k = first + lane; k - lane < end; k += U * kWave) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = min(k + u * kWave, end - 1);
      v[u] = (double)scalar_val(val, at) * (double)x[a.col[at]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u * kWave < end) sum += v[u];
  }
  return last_lane(wave_sum_tree(sum));
}

// A long crossing row [rs, re) in a launch that no sss_carries follows.  Each
// bunch that begins in it stores its part of the row (the first of them with
// what lies before it, at most a bunch's worth) and counts itself in; the last
// to do so adds the parts, in their order whoever is last, and writes y[row].
// No bunch waits.  Called by a whole wavefront after its state is stored.
template <typename YT>
__device__ __forceinline__ void finish_row(const MatCtx &a, int row, int64_t rs, int64_t re, int64_t SWT, int lane) {
  const int64_t head = (rs + SWT - 1) / SWT, end = (re + SWT - 1) / SWT;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  int before = 0;
  if (lane == 0) before = __hip_atomic_fetch_add(&a.arrivals[head], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (__builtin_amdgcn_readfirstlane(before) != (int)(end - head) - 1) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  double sum = 0.0;
  for (int64_t k = head + lane; k < end; k += kWave) sum += a.state[k].sync_val;
  sum = wave_sum_tree(sum);
  if (lane == 0) {
    static_cast<YT *>(a.y)[row] = (YT)sum;
    a.arrivals[head] = 0;
  }
}

// tb, the bunch; brow, its first row at plan time or -1; need, its slot_need
// (0 without a plan); share of shares, its part of the leading rows: the same
// in every lane.  Returns the lane's part of the bunch's dot product (DOT).
template <int DT, int W, Form FORM, bool DOT = false>
__device__ __forceinline__ double fused_bunch(const MatCtx &a, const int tb, const int brow, const int need,
                                              const int64_t share, const int64_t shares, uint32_t *lds_wave,
                                              const int lane) {
  using val_t = typename VT<DT>::val_t;
  using x_t = typename VT<DT>::x_t;
  using y_t = typename VT<DT>::y_t;
  using prod_t = typename VT<DT>::prod_t;
  constexpr int WT = W * kWave;
  constexpr int WPT = WT / 32;
  const int S = a.S, m = a.m;
  const int SWT = S * WT;
  const int b0 = tb * SWT;  // < nnz
  const int left = min(a.nnz - b0, SWT);
  const int bS = b0 + left;
  const int tiles = (left + WT - 1) / WT;
  const bool known = brow != -1;
  const int back_n = need & 0xff;
  uint32_t *mask = lds_wave;
  uint32_t *dflag = mask + S * WPT;

  // ---- the loads that need nothing
  const rsrc_t rx = make_rsrc(a.x, 0xffffffffu);
  auto gather = [&](uint32_t c) {
    if constexpr (FORM == kWide) return static_cast<const x_t *>(a.x)[c];
    else return buffer_load<x_t>(rx, (int)(c * (uint32_t)sizeof(x_t)));
  };
  constexpr bool NT = FORM != kCached;
  Tile<DT, W> cur, next;
  // tile t of the bunch; nothing of a tile past the bunch's end (rest = 0)
  auto load_tile = [&](Tile<DT, W> &tile, int t) {
    const uint32_t rest = (uint32_t)max(left - t * WT, 0);
    tile.template load<NT>(make_rsrc(a.col + (b0 + t * WT), rest * 4u),
                           make_rsrc(static_cast<const val_t *>(a.val) + (b0 + t * WT),
                                     value_range(rest, sizeof(val_t))),
                           lane);
  };
  load_tile(cur, 0);
  const int back_off = lane - (kBack - back_n);  // lanes below 0: outside
  const uint32_t back_c =
      buffer_load<uint32_t>(make_rsrc(a.col + (b0 - back_n), (uint32_t)back_n * 4u), back_off * 4);
  const val_t back_v = buffer_load<val_t>(
      make_rsrc(static_cast<const val_t *>(a.val) + (b0 - back_n), (uint32_t)back_n * sizeof(val_t)),
      back_off * (int)sizeof(val_t));
  // A bunch without a row from the plan searches for it here, ahead of the
  // gathers: loads return in order, so behind them every round of the search
  // would wait for tile 0's gathers first.  Unbound products, us behind /
  // ahead, W = 4, S = 1: power law 70K rows FP64 18.2 / 17.0, FP32 17.3 / 15.7,
  // Poisson 60K rows 11.5 / 10.9, 500^2 5-point stencil 13.5 / 12.9.
  int r0 = brow & 0x7fffffff;
  if (!known) r0 = __builtin_amdgcn_readfirstlane(wave_rightmost(a.row_ptr, m, b0, lane));
  const int span = known ? need >> 8 : m - r0;
  const bool ahead = !known || span < kSpanMax;
  const rsrc_t rr = make_rsrc(a.row_ptr + r0, ahead ? (uint32_t)(min(span, 2 * kWave - 1) + 1) * 4u : 0u);
  const int rows0 = buffer_load<int>(rr, lane * 4);
  const int rows1 = buffer_load<int>(rr, lane * 4 + kWave * 4);
  const int past_span = a.row_ptr[ahead ? imin64((int64_t)r0 + span, m) : 0];
  const int second_row = a.row_ptr[1];
  if (S > 1) load_tile(next, 1);

  // ---- the gathers of tile 0
  x_t xv[W];
#pragma unroll
  for (int i = 0; i < W; ++i) xv[i] = gather(cur.column(i));
  const x_t back_x = gather(back_c);  // (column 0 in the lanes that hold none)

  // ---- descriptor, tile start rows, dirty tiles: one pass over the rows
  for (int i = lane; i < S * WPT; i += kWave) mask[i] = 0u;
  if (lane == 0) *dflag = 0u;
  lds_handover();

  const int32_t *__restrict__ rp = a.row_ptr;
  const int my_b = b0 + min(min(lane, S) * WT, left);
  int my_count = 0, my_rp = 0;  // lane t <= S: as in stage1_bunch
  int first_rs = 0, first_re = 0;
  uint64_t filled_rows = 0;
  // the plan's rows hold where rp[r0] <= b0 < rp[r0 + 1] and the entry after
  // the span is past bS (or the last): row_ptr ascends, so every row between
  // is the bunch's.  Else (a longer span, or row_ptr rewritten in place since)
  // the bunch searches for its first row and reads on from there.  A row just
  // searched for holds, with every row to the last as its span.
  const bool loaded = ahead && lane_value(rows0, 0) <= b0 && b0 < lane_value(rows0, 1) &&
                      ((int64_t)r0 + span >= m || past_span > bS);
  if (__builtin_expect(!loaded, 0)) {
    if (!known || !(rp[r0] <= b0 && b0 < rp[r0 + 1]))
      r0 = __builtin_amdgcn_readfirstlane(wave_rightmost(rp, m, b0, lane));
  }
  const int last = loaded ? (int)imin64((int64_t)r0 + span, m) : m;  // the last entry to read
  // entries rbase .. rbase + 63, INT_MAX past the last
  auto entries = [&](int rbase) {
    const int n = min(last - rbase + 1, kWave);
    const int v = buffer_load<int>(make_rsrc(rp + rbase, n > 0 ? (uint32_t)n * 4u : 0u), lane * 4);
    return lane < n ? v : INT_MAX;
  };
  // one chunk of 64 rows: p = rp[r], after = the entry past the chunk (a value
  // past bS beyond the last entry, or beyond the span); true when more follow
  auto row_chunk = [&](int rbase, int p, int after) {
    const int r = rbase + lane;
    const int q = wave_next(p, after);  // rp[r + 1]
    if (rbase == r0) {
      first_rs = lane_value(p, 0);
      first_re = lane_value(q, 0);
    }
    if (r < m && q > p && p >= b0 && p < bS) {
      const int off = p - b0;
      atomicOr(&mask[off >> 5], 1u << (off & 31));
    }
    // (of empty rows in a run, which all begin at p, the chunk's first marks the
    // tile: the wavefront takes its lanes of one address one after another)
    if (r < m && q == p && wave_prev(p, -1) != p && p > b0 && p <= bS) atomicOr(dflag, 1u << ((p - b0 - 1) / WT));
    const uint64_t filled = __ballot(q != p);
    if (lane == (rbase - r0) / kWave) filled_rows = filled;
    const int p_first = lane_value(p, 0), p_last = lane_value(p, kWave - 1);
    // empty rows only: every tile boundary counts all of them or none (100K Poisson
    // rows and 100K empty ones behind them: 1,456 -> 929 us; two stages 1,431)
    if (__builtin_expect(p_first == p_last, 0)) {
      if (p_first <= my_b) {
        my_count += kWave;
        my_rp = p_first;
      }
    } else {
      for (int t = 0; t <= S; ++t) {
        const int c = __popcll(__ballot(p <= lane_value(my_b, t)));
        const int p_last_in = lane_value(p, c > 0 ? c - 1 : 0);
        if (lane == t) {
          my_count += c;
          if (c > 0) my_rp = p_last_in;
        }
      }
    }
    return p_last <= bS && rbase + (kWave - 1) < m;
  };
  // the two chunks that are there hold the bunch (apart from the loop below,
  // whose loads would make this wait for tile 0's gathers)
  if (loaded && (span < 2 * kWave || lane_value(rows1, kWave - 1) > bS)) {
    for (int chunk = 0; chunk < 2; ++chunk) {
      const int p = chunk * kWave + lane <= span ? (chunk == 0 ? rows0 : rows1) : INT_MAX;
      const int after = chunk == 0 && span >= kWave ? lane_value(rows1, 0) : INT_MAX;
      if (!row_chunk(r0 + chunk * kWave, p, after)) break;
    }
  } else {
    // two chunks ahead: a chunk needs the first entry of the next
    int p = loaded ? rows0 : entries(r0), next_p = loaded ? rows1 : entries(r0 + kWave);
    for (int rbase = r0;; rbase += kWave) {
      const int p2 = entries(rbase + 2 * kWave);
      if (!row_chunk(rbase, p, lane_value(next_p, 0))) break;
      p = next_p;
      next_p = p2;
    }
  }
  lds_handover();

  Bunch<DT, W, DOT> u;
  u.rp = rp;
  u.y = static_cast<y_t *>(a.y);
  u.speculator = a.speculator ? a.speculator + (int64_t)tb * S : nullptr;
  u.mask = mask;
  u.part = reinterpret_cast<double *>(mask + S * WPT + 2);
  u.m = m;
  u.lane = lane;
  u.r0 = r0;
  u.first_tile = tb * S;
  u.dirty_bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)*dflag);
  u.my_start = lane <= S ? r0 + my_count - 1 : 0;
  u.my_rp = my_rp;
  u.filled_rows = filled_rows;
  u.transmitter = 0.0;
  u.sync_v = 0.0;
  if constexpr (DOT) u.x = static_cast<const double *>(a.x);
  u.dot = 0.0;

  // ---- does this bunch write y[r0]: it does when the row ends here and is
  // no long crossing row; the row's entries before the bunch are summed here
  const bool is_long = r0 < m && long_crossing(first_rs, first_re, b0, SWT, back_limit(a.carries));
  const bool own_first = r0 < m && !is_long;
  double before = 0.0;
  if (own_first && first_rs < b0) {
    const val_t *__restrict__ val = static_cast<const val_t *>(a.val);
    const x_t *__restrict__ x = static_cast<const x_t *>(a.x);
    prod_t product = back_off >= 0 ? (prod_t)scalar_val(&back_v, 0) * (prod_t)back_x : (prod_t)0;
    if (b0 - first_rs != back_n) {  // not found at plan time, or row_ptr rewritten since
      const int k = b0 - kBack + lane;
      product = k >= first_rs ? (prod_t)scalar_val(val, k) * (prod_t)x[a.col[k]] : (prod_t)0;
    }
    before = back_sum<DT, W>(product, first_rs, b0, u.part, lane);
  }

  // ---- the tiles
  prod_t pr[W];
  auto products = [&](auto last_tile) {
    prod_t av[W], bv[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
      av[i] = cur.value(i);
      bv[i] = (prod_t)xv[i];
    }
    const int rest = left - (tiles - 1) * WT;
    if (decltype(last_tile)::value && rest < WT) {  // the matrix's last tile: entries past its end add 0
#pragma unroll
      for (int i = 0; i < W; ++i)
        if (Tile<DT, W>::offset(i, lane) >= rest) av[i] = bv[i] = (prod_t)0;
      if constexpr (DT == SSS_BF16) {
        if (left & 1) {  // (the value that its load's range leaves out)
          const prod_t odd = scalar_val(static_cast<const val_t *>(a.val), bS - 1);
#pragma unroll
          for (int i = 0; i < W; ++i)
            if (Tile<DT, W>::offset(i, lane) == rest - 1) av[i] = odd;
        }
      }
    }
    Tile<DT, W>::store(av, bv, reinterpret_cast<prod_t *>(u.part), lane, pr);
  };
  double tail = 0.0;
  for (int t = 0; t + 1 < tiles; ++t) {
    products(std::false_type{});
    u.load_rows(t);
    cur = next;
#pragma unroll
    for (int i = 0; i < W; ++i) xv[i] = gather(cur.column(i));
    if (t + 2 < tiles) load_tile(next, t + 2);
    (void)u.sum_tile(t, b0 + (t + 1) * WT, pr);
  }
  products(std::true_type{});
  u.load_rows(tiles - 1);
  tail = u.sum_tile(tiles - 1, bS, pr);

  if (own_first && lane == 0) {
    y_store((y_t)(before + u.sync_v), &u.y[r0]);
    if constexpr (DOT) u.dot += u.x[r0] * (before + u.sync_v);
  }
  if (__builtin_expect(second_row == 0, 0)) zero_leading(rp, u.y, m, share, shares, lane);
  const bool shared = is_long && !a.carries && a.arrivals;  // a row that the plan did not know
  if (__builtin_expect(shared, 0)) {
    if (first_rs < b0 && first_rs > b0 - SWT) u.sync_v += row_part<DT>(a, first_rs, b0, lane);
    if constexpr (DOT)
      if (lane == 0) u.dot += u.x[r0] * u.sync_v;
  }
  if (a.keep_state || shared) {  // (a batch that needs no carries keeps none)
    const uint64_t sv = (uint64_t)__double_as_longlong(u.sync_v), tv = (uint64_t)__double_as_longlong(tail);
    const uint32_t words[6] = {(uint32_t)sv, (uint32_t)(sv >> 32), (uint32_t)tv, (uint32_t)(tv >> 32), (uint32_t)r0,
                               u.dirty_bits};
    uint32_t w = words[0];
#pragma unroll
    for (int i = 1; i < 6; ++i) w = lane == i ? words[i] : w;
    if (lane < 6) reinterpret_cast<uint32_t *>(a.state + tb)[lane] = w;
  }
  if (__builtin_expect(shared, 0)) finish_row<y_t>(a, r0, first_rs, first_re, SWT, lane);
  return u.dot;
}

template <int DT, int W, Form FORM>
__global__ __launch_bounds__(256) void sss_fused(MatCtx a) {
  extern __shared__ uint32_t lds_words[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = wave_in_block();
  const int64_t g = (int64_t)blockIdx.x * (blockDim.x / kWave) + wid;
  int4 slot = make_int4((int)g, -1, 0, 0);
  if (g >= (a.slots ? a.n_slots : a.n_bunches)) slot.x = -1;
  else if (a.slots) slot = uniform_load(a.slots + g);
  // (the paths that few products take are marked: in line they cost the others'
  // instruction fetch, a 4,096-row Poisson matrix 13.5 / 13.25 us)
  if (__builtin_expect(slot.x < 0, 0)) {  // no bunch
    using y_t = typename VT<DT>::y_t;
    if (a.row_ptr[1] == 0) zero_leading(a.row_ptr, static_cast<y_t *>(a.y), a.m, g, a.n_shares, lane);
    return;
  }
  fused_bunch<DT, W, FORM>(a, slot.x, slot.y, slot.z, g, a.n_shares, lds_words + wid * stage1_lds_words(W, a.S), lane);
}

// The same with the partial sums of x . y, one per workgroup, for bound FP64
// plans without long crossing rows (those are completed by another launch).
// An iterative method that needs the product and its dot product with x (CG's
// p . A p) saves a launch and a pass over both vectors.
template <int W, Form FORM>
__global__ __launch_bounds__(256) void sss_fused_dot(MatCtx a, double *__restrict__ dots) {
  extern __shared__ uint32_t lds_words[];
  __shared__ double sums[kMaxB];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = wave_in_block();
  const int64_t g = (int64_t)blockIdx.x * (blockDim.x / kWave) + wid;
  double dot = 0.0;
  if (g < a.n_slots) {
    const int4 slot = uniform_load(a.slots + g);
    if (slot.x >= 0)
      dot = fused_bunch<SSS_F64, W, FORM, true>(a, slot.x, slot.y, slot.z, slot.x, a.n_bunches,
                                                lds_words + wid * stage1_lds_words(W, a.S), lane);
  }
  dot = wave_sum_tree(dot);
  if (lane == 0) sums[wid] = dot;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < (int)(blockDim.x / kWave); ++i) dot += sums[i];
    dots[blockIdx.x] = dot;
  }
}

// gfx950 (one partition) hands consecutive workgroups to its 8 XCDs in turn,
// workgroup b to XCD b mod 8, and every XCD has its own L2.
constexpr int kXcds = 8;

constexpr int kOrderBins = 256;  // column order: places in a row; bin kOrderBins holds the short rows
constexpr int kOrderShare = 16;

// Plan time: the first row of every thread-bunch, the rightmost match of its
// first nonzero (Section 3.2's tile boundary search), one thread per bunch.
__device__ __forceinline__ int32_t rightmost_row(const int32_t *__restrict__ rp, int32_t m, int64_t b) {
  int32_t lo = 0, hi = m;  // rp[0] = 0 <= b
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo + 1) / 2;
    if ((int64_t)rp[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// *any_long is set when some bunch's first row is a long crossing row.
__global__ void sss_bunch_rows(const int32_t *__restrict__ rp, int32_t m, int64_t SWT, int64_t n_bunches,
                               int32_t *__restrict__ out, int32_t *__restrict__ any_long) {
  for (int64_t tb = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; tb < n_bunches;
       tb += (int64_t)gridDim.x * blockDim.x) {
    const int32_t r = rightmost_row(rp, m, tb * SWT);
    out[tb] = r;
    if (r < m && long_crossing(rp[r], rp[r + 1], tb * SWT, SWT, kBack)) *any_long = 1;
  }
}

// Plan time: mark every bunch with a dirty tile by OR-ing `bit` into
// words[bunch].  A tile is dirty exactly when an empty row r with
// row_ptr[r] = p > 0 lies in it (tile (p - 1) / WT, Section 3.2's dirty
// condition), so its bunch is (p - 1) / SWT.
__global__ void sss_mark_dirty_bunches(const int32_t *__restrict__ rp, int32_t m, int64_t SWT,
                                       uint32_t *__restrict__ words, uint32_t bit) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)gridDim.x * blockDim.x) {
    const int32_t p = rp[r];
    if (p > 0 && p == rp[r + 1]) atomicOr(words + (p - 1) / SWT, bit);
  }
}

// The place in its row, as a bin of the column order (below), of nonzero `at`
// of row [p, q); kOrderBins where the row is short.
__device__ __forceinline__ uint32_t order_bin(int64_t at, int64_t p, int64_t q, int64_t SWT) {
  return q - p >= SWT && at >= p ? (uint32_t)imin64((at - p) * kOrderBins / (q - p), kOrderBins - 1)
                                 : (uint32_t)kOrderBins;
}

// The same for one call of a plan that binds no rows, with the bunches' keys
// for the column order: one thread per row writes the first row of the bunches
// that begin in it and the keys of those whose middle lies in it (a wavefront
// writes those of a row with many), one pass over row_ptr instead of a search
// per bunch.  Clears the two lists of hist.
constexpr int kFewBunches = 4;

__global__ __launch_bounds__(256) void sss_call_rows(const int32_t *__restrict__ rp, int32_t m, int32_t nnz,
                                                     int32_t SWT, uint32_t n_bunches, int32_t *__restrict__ rows,
                                                     uint32_t *__restrict__ keys, uint32_t *__restrict__ hist) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t u = (uint32_t)SWT, half = u / 2;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < 2 * (kOrderBins + 1); i += blockDim.x) hist[i] = 0u;
    // (a last bunch that ends before its middle)
    if (threadIdx.x == 0 && (n_bunches - 1) * u + half >= (uint32_t)nnz) keys[n_bunches - 1] = kOrderBins;
  }
  for (int64_t r0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; r0 < m;
       r0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = r0 + lane;
    const uint32_t p = r < m ? (uint32_t)rp[r] : 0u, q = r < m ? (uint32_t)rp[r + 1] : 0u;
    // bunches k0 .. k1-1 begin in [p, q); m0 .. m1-1 have their middle there
    // (the minima hold in every valid matrix)
    const uint32_t k0 = (p + u - 1u) / u, m0 = (max(p, half) - half + u - 1u) / u;
    const uint32_t k1 = q > p ? min((q + u - 1u) / u, n_bunches) : k0;
    const uint32_t m1 = q > p ? min((max(q, half) - half + u - 1u) / u, n_bunches) : m0;
    const bool many = k1 > k0 + kFewBunches;
    if (!many) {
      for (uint32_t k = k0; k < k1; ++k) rows[k] = (int32_t)r;
      for (uint32_t k = m0; k < m1; ++k) keys[k] = order_bin((int64_t)k * u + half, p, q, SWT);
    }
    uint64_t todo = __ballot(many);
    while (todo) {
      const int l = __ffsll((unsigned long long)todo) - 1;
      todo &= todo - 1;
      const uint32_t pl = (uint32_t)lane_value((int)p, l), ql = (uint32_t)lane_value((int)q, l);
      const uint32_t end = (uint32_t)lane_value((int)k1, l), mend = (uint32_t)lane_value((int)m1, l);
      for (uint32_t k = (uint32_t)lane_value((int)k0, l) + lane; k < end; k += kWave) rows[k] = (int32_t)(r0 + l);
      for (uint32_t k = (uint32_t)lane_value((int)m0, l) + lane; k < mend; k += kWave)
        keys[k] = order_bin((int64_t)k * u + half, pl, ql, SWT);
    }
  }
}

// Stage 1's column order.  A bunch inside a long row reads a narrow slice of
// the columns (a row's columns ascend), so such bunches are sorted by their
// place in their row and dealt to the XCDs in eight equal runs: each XCD's L2
// then holds one moving slice of x instead of all of it.  The bunches of
// short rows read all over x and follow in their own order, dealt in turn.
// What bounds these gathers is how long a miss of L1 takes, and a hit in L2
// takes less than half of a miss: 1M-row power law in FP64 (8 MB of x, W = 4,
// S = 4) 221 -> 183 us per product, 4M-row Zipf 1.8 in FP32 (16 MB, W = 16,
// S = 2) 1,103 -> 812 us, both with the same y bit for bit.
//
// A bunch counts as inside a long row when the row of its middle nonzero has
// at least SWT of them.  SWT / 2 and SWT / 4 measured 2% faster on the first
// matrix (179 us) and 2 to 5% slower on the second (848 us), whose bunches
// are twice as long; 2 SWT and 4 SWT 2 to 10% slower on both.
//
// FIND: find the keys, else they are there (the lists of one call).
template <bool FIND>
__global__ __launch_bounds__(256) void sss_order_keys(const int32_t *__restrict__ rp, int32_t m, int32_t nnz,
                                                      int64_t SWT, int64_t n_bunches,
                                                      const int32_t *__restrict__ bunch_row,
                                                      uint32_t *__restrict__ keys, uint32_t *__restrict__ hist) {
  __shared__ uint32_t count[kOrderBins + 1];
  for (int i = threadIdx.x; i <= kOrderBins; i += blockDim.x) count[i] = 0u;
  __syncthreads();
  const int64_t tb = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tb < n_bunches) {
    uint32_t key;
    if constexpr (FIND) {
      const int32_t mid = (int32_t)imin64(tb * SWT + SWT / 2, (int64_t)nnz - 1);
      // the row of nonzero mid, between the first rows of this bunch and the next
      int32_t lo = bunch_row[tb] & 0x7fffffff;
      int32_t hi = tb + 1 < n_bunches ? bunch_row[tb + 1] & 0x7fffffff : m;
      while (lo < hi) {
        const int32_t c = lo + (hi - lo + 1) / 2;
        if (rp[c] <= mid) lo = c;
        else hi = c - 1;
      }
      key = order_bin(mid, rp[lo], lo < m ? rp[lo + 1] : nnz, SWT);
      keys[tb] = key;
    } else {
      key = min(keys[tb], (uint32_t)kOrderBins);
    }
    atomicAdd(&count[key], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i <= kOrderBins; i += blockDim.x)
    if (count[i]) atomicAdd(&hist[i], count[i]);
}

// The slot of the t-th wavefront of XCD k: workgroup b of B wavefronts runs
// on XCD b mod kXcds.
__device__ __forceinline__ int64_t xcd_slot(int64_t k, int64_t t, int B) { return (k + kXcds * (t / B)) * B + t % B; }

// A slot's entry for bunch tb (bunch_row: first rows, with the top bit).
__device__ __forceinline__ int4 slot_entry(const int32_t *__restrict__ rp, int32_t m, int64_t SWT, int64_t tb,
                                           int64_t n_bunches, const int32_t *__restrict__ bunch_row, bool carries) {
  const int32_t row = bunch_row[tb];
  const int32_t next = tb + 1 < n_bunches ? bunch_row[tb + 1] & 0x7fffffff : m;
  return make_int4((int)tb, row, slot_need(rp, m, SWT, tb, row & 0x7fffffff, next, carries), 0);
}

// Slots in bunch order.
__global__ __launch_bounds__(256) void sss_slots(const int32_t *__restrict__ rp, int32_t m, int64_t SWT,
                                                 int64_t n_bunches, const int32_t *__restrict__ bunch_row,
                                                 bool carries, int4 *__restrict__ slots) {
  const int64_t tb = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tb < n_bunches) slots[tb] = slot_entry(rp, m, SWT, tb, n_bunches, bunch_row, carries);
}

// Slots in column order; in bunch order where fewer than one bunch in
// kOrderShare is long.  hist: the bunches per bin; cursor: zeros.  Within a bin the order is that
// of the atomics, which decides only when a bunch runs.
__global__ __launch_bounds__(256) void sss_order_scatter(const int32_t *__restrict__ rp, int32_t m, int64_t SWT,
                                                         int64_t n_bunches, const int32_t *__restrict__ bunch_row,
                                                         const uint32_t *__restrict__ keys, int64_t n_slots, int B,
                                                         const uint32_t *__restrict__ hist,
                                                         uint32_t *__restrict__ cursor, bool carries,
                                                         int4 *__restrict__ slots) {
  __shared__ uint32_t first[kOrderBins], count[kOrderBins + 1], base[kOrderBins + 1];
  const int t = threadIdx.x;
  static_assert(kOrderBins == 256, "one bin per thread");
  first[t] = hist[t];
  count[t] = 0u;
  if (t == 0) count[kOrderBins] = 0u;
  __syncthreads();
  for (int d = 1; d < kOrderBins; d <<= 1) {  // inclusive scan of the long bins
    const uint32_t v = t >= d ? first[t - d] : 0u;
    __syncthreads();
    first[t] += v;
    __syncthreads();
  }
  const int64_t n_long = first[kOrderBins - 1];
  const int64_t tb = (int64_t)blockIdx.x * blockDim.x + t;
  if (n_long * kOrderShare < n_bunches) {
    if (tb < n_slots)
      slots[tb] = tb < n_bunches ? slot_entry(rp, m, SWT, tb, n_bunches, bunch_row, carries) : make_int4(-1, 0, 0, 0);
    return;
  }
  uint32_t key = 0, mine = 0;
  if (tb < n_bunches) {
    key = min(keys[tb], (uint32_t)kOrderBins);
    mine = atomicAdd(&count[key], 1u);
  }
  __syncthreads();
  for (int i = t; i <= kOrderBins; i += blockDim.x) base[i] = count[i] ? atomicAdd(&cursor[i], count[i]) : 0u;
  __syncthreads();
  const int64_t each = n_long / kXcds, more = n_long % kXcds;  // the first `more` XCDs take one long bunch more
  if (tb < n_bunches) {
    int64_t i = (int64_t)base[key] + mine;
    int64_t slot;
    if (key < (uint32_t)kOrderBins) {
      i += key > 0 ? first[key - 1] : 0u;
      const int64_t head = more * (each + 1);
      const int64_t k = i < head ? i / (each + 1) : more + (i - head) / each;
      slot = xcd_slot(k, i < head ? i % (each + 1) : (i - head) % each, B);
    } else {
      i += n_long;
      slot = xcd_slot(i % kXcds, i / kXcds, B);
    }
    slots[slot] = slot_entry(rp, m, SWT, tb, n_bunches, bunch_row, carries);
  } else if (tb < n_slots) {
    slots[xcd_slot(tb % kXcds, tb / kXcds, B)] = make_int4(-1, 0, 0, 0);
  }
}

// Plan time, batches: for global bunch g its matrix (the rightmost i with
// bunch_base[i] <= g), its first row and its index within the matrix;
// *any_long as in sss_bunch_rows.
__global__ void sss_batch_bunch_info(const MatCtx *__restrict__ mats, const int64_t *__restrict__ bunch_base,
                                     int32_t count, int64_t total, int4 *__restrict__ out,
                                     int32_t *__restrict__ any_long) {
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    int32_t lo = 0, hi = count;
    while (lo < hi) {
      const int32_t mid = lo + (hi - lo + 1) / 2;
      if (bunch_base[mid] <= g) lo = mid;
      else hi = mid - 1;
    }
    const MatCtx &a = mats[lo];
    const int64_t tb = g - bunch_base[lo], SWT = (int64_t)a.S * a.W * kWave;
    const int32_t r = rightmost_row(a.row_ptr, a.m, tb * SWT);
    if (r < a.m && long_crossing(a.row_ptr[r], a.row_ptr[r + 1], tb * SWT, SWT, kBack)) *any_long = 1;
    const int32_t next = tb + 1 < a.n_bunches ? rightmost_row(a.row_ptr, a.m, (tb + 1) * SWT) : a.m;
    out[g] = make_int4(lo, r, (int)tb, slot_need(a.row_ptr, a.m, SWT, tb, r, next, false));
  }
}

// Measurement aid, not part of the method: the memory floor of stage 1's
// access pattern.  Same tiling, same grouped col/val loads and the same
// one-tile-ahead prefetch as stage 1, with no row pass, no segmentation and no
// partial stores: each lane sums its products (GATHER) or its values plus
// columns (stream only) and writes one value, so the loads cannot be dropped.
template <int DT, int W, bool GATHER>
__device__ __forceinline__ double floor_bunch(const MatCtx &a, const int64_t tb, const int lane) {
  using val_t = typename VT<DT>::val_t;
  using x_t = typename VT<DT>::x_t;
  using prod_t = typename VT<DT>::prod_t;
  constexpr int WT = W * kWave;
  const int32_t *__restrict__ col = a.col;
  const val_t *__restrict__ val = static_cast<const val_t *>(a.val);
  const x_t *__restrict__ x = static_cast<const x_t *>(a.x);
  const int nnz = a.nnz, S = a.S;
  const int64_t SWT = (int64_t)S * WT;
  int cc[W];
  prod_t av[W], xv[W];
  load_tile_g<DT, W>(col, val, (int)(tb * SWT), nnz, lane, cc, av);
#pragma unroll
  for (int i = 0; i < W; ++i) xv[i] = GATHER ? (prod_t)x[cc[i]] : (prod_t)cc[i];
  double acc = 0.0;
  for (int t = 0; t < S; ++t) {
    const int64_t b64 = tb * SWT + (int64_t)t * WT;
    if (b64 >= nnz) break;
    const bool has_next = (t + 1 < S) && (b64 + WT < nnz);
    int cn[W];
    prod_t an[W];
    if (has_next) load_tile_g<DT, W>(col, val, (int)b64 + WT, nnz, lane, cn, an);
#pragma unroll
    for (int i = 0; i < W; ++i) acc += GATHER ? (double)(av[i] * xv[i]) : (double)(av[i] + xv[i]);
    if (has_next) {
#pragma unroll
      for (int i = 0; i < W; ++i) { xv[i] = GATHER ? (prod_t)x[cn[i]] : (prod_t)cn[i]; av[i] = an[i]; }
    }
  }
  return acc;
}

template <int DT, int W, bool GATHER>
__global__ __launch_bounds__(256) void sss_floor(MatCtx a, typename VT<DT>::y_t *__restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t tb = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (tb >= a.n_bunches) return;
  out[tb * kWave + lane] = (typename VT<DT>::y_t)floor_bunch<DT, W, GATHER>(a, tb, lane);
}

// Many matrices in one launch per stage: the thread-bunches of all matrices
// form one nnz-balanced index space (bunch_base = prefix of the per-matrix
// bunch counts).  Stage 1 reads each bunch's matrix, first row and index
// within the matrix from the plan (found at plan time by the same
// rightmost-match search the method uses for rows); stage 2 runs that search
// over bunch_base itself.
struct BatchArgs {
  const MatCtx *mats;
  const int64_t *bunch_base;  // [count+1]
  const int64_t *chunk_base;  // [count+1] prefix of ceil(n_bunches / 64)
  int32_t count;
  int32_t S_max;
  int64_t total_bunches;
  int64_t total_chunks;
  int64_t total_waves;        // second-launch work items: the carry chunks (0 without long crossing
                              // rows), then one per matrix where some matrix has no nonzero
  int32_t carries;            // MatCtx::carries of every matrix of the batch
  const int4 *bunch_info;     // per global bunch: <matrix, first row, bunch within the matrix, slot_need>
  // stage 1's XCD windows: the workgroups b with b mod n_windows = k take the
  // global bunches window[k] .. window[k+1]-1, in order.  n_windows is kXcds
  // (one contiguous window per XCD, holding an equal share of the nonzeros)
  // or 1 for grids of at most kXcds workgroups.
  int32_t n_windows;
  int64_t window[kXcds + 1];
};

// A global bunch's plan entry and its matrix's context, read once per
// wavefront through the scalar unit into scalar registers (g < 2^31: the grid
// is limited to that many wavefronts).
__device__ __forceinline__ void batch_entry(const BatchArgs &b, int64_t g, int4 &bi, MatCtx &a) {
  bi = uniform_load(b.bunch_info + g);
  a = uniform_load(b.mats + bi.x);
  a.carries = a.keep_state = b.carries;
  if (b.carries) bi.w &= ~0xff;  // (found before the plan knew: no entries before the bunch)
}


// The global bunch of wavefront `wid` of this workgroup in a launch of one
// wavefront per bunch over the XCD windows, or -1 past its window's end.
__device__ __forceinline__ int64_t window_bunch(const BatchArgs &b, int wid) {
  const int G = b.n_windows;
  const int k = (int)(blockIdx.x % G);
  const int64_t g = b.window[k] + (int64_t)(blockIdx.x / G) * (blockDim.x / kWave) + wid;
  return g < b.window[k + 1] ? g : -1;
}

// The types' default W runs three wavefronts on a SIMD, for which the registers
// would allow four (FP64) or nearly do (FP32): the x of fewer matrices is in
// flight.  256 uneven matrices FP64 716 / 707 us with four / three, FP32 529 / 520.
struct WavesPerSimd { int least, most; };
template <int DT, int W> constexpr WavesPerSimd batch_waves() {
  return (DT == SSS_F64 && W == 8) || (DT == SSS_F32 && W == 16) ? WavesPerSimd{3, 3} : WavesPerSimd{1, 8};
}

template <int DT, int W, Form FORM>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(batch_waves<DT, W>().least, batch_waves<DT, W>().most)))
void sss_fused_batch(BatchArgs b) {
  extern __shared__ uint32_t lds_words[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = wave_in_block();
  uint32_t *lds_wave = lds_words + wid * stage1_lds_words(W, b.S_max);
  // One wavefront per thread-bunch, XCD-aware: workgroup blockIdx.x, which
  // runs on XCD blockIdx.x mod kXcds, takes the (blockIdx.x / kXcds)-th
  // workgroup's worth of bunches of that XCD's window, a contiguous run of
  // the global bunch space holding an eighth of the nonzeros (bunches of
  // matrices with a larger S hold more).  Each XCD then works through its
  // own run of matrices in order, and its L2 holds the x of the few matrices
  // in its window instead of those of every matrix in flight on the chip.
  // (Any placement of workgroups gives the same result; the placement only
  // decides the speed.)
  const int64_t g = window_bunch(b, wid);
  if (g < 0) return;
  int4 bi;
  MatCtx a;
  batch_entry(b, g, bi, a);
  fused_bunch<DT, W, FORM>(a, bi.z, bi.y, bi.w, bi.z, a.n_bunches, lds_wave, lane);
}

// The same work as a persistent grid (batch_persistent plans): as many
// workgroups as stay resident, a multiple of kXcds; the workgroups with
// blockIdx.x mod kXcds = k stride over window k, one bunch per wavefront per
// step.
template <int DT, int W, Form FORM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))  // (at W = 16 else one)
void sss_fused_batch_persistent(BatchArgs b) {
  extern __shared__ uint32_t lds_words[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = wave_in_block();
  uint32_t *lds_wave = lds_words + wid * stage1_lds_words(W, b.S_max);
  const int G = b.n_windows;
  const int k = (int)(blockIdx.x % G);
  const int wpb = blockDim.x / kWave;
  const int64_t stride = (int64_t)((gridDim.x - k + G - 1) / G) * wpb;  // waves of the workgroups b mod G = k
  const int64_t hi = b.window[k + 1];
  for (int64_t g = b.window[k] + (int64_t)(blockIdx.x / G) * wpb + wid; g < hi; g += stride) {
    int4 bi;
    MatCtx a;
    batch_entry(b, g, bi, a);
    fused_bunch<DT, W, FORM>(a, bi.z, bi.y, bi.w, bi.z, a.n_bunches, lds_wave, lane);
  }
}

// Measurement aid for the batched stage 1: its launch (one wavefront per
// bunch, the same XCD-contiguous mapping and the same per-bunch lookup) with
// floor_bunch in place of the method's work; out has 64 entries per global
// bunch.
template <int DT, int W, bool GATHER>
__global__ __launch_bounds__(256) void sss_floor_batch(BatchArgs b, typename VT<DT>::y_t *__restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = wave_in_block();
  const int64_t g = window_bunch(b, wid);
  if (g < 0) return;
  int4 bi;
  MatCtx a;
  batch_entry(b, g, bi, a);
  out[g * kWave + lane] = (typename VT<DT>::y_t)floor_bunch<DT, W, GATHER>(a, bi.z, lane);
}

// ---------------------------------------------------------------- stage 2

// the carry kernels' workgroup, and a wavefront's staging in doubles: the
// values and (half as wide) the row indices of its chunk and kShortRun more
constexpr int kCarryThreads = 128;
constexpr int kCarryLds = (kWave + kShortRun) * 3 / 2;

// (1) re-arrange the dirty tiles of thread-bunch tb: a dirty tile's partials
// 1.. sit at y[start+1..]; the k-th non-empty row strictly between start and
// stop receives partial k, the empty rows there receive 0.  Only rows strictly
// inside the tile are touched.  The partials are gathered into LDS first.
template <typename YT>
__device__ __forceinline__ void fixup_dirty(const MatCtx &a, const int64_t tb, YT *slots, const int lane) {
  const int32_t *__restrict__ rp = a.row_ptr;
  YT *y = static_cast<YT *>(a.y);
  const int WT = a.W * kWave;
  const uint32_t dm = a.state[tb].dirty_mask;
  const int n_dirty = __popc(dm);
  if (n_dirty == 0) return;
  // all of the bunch's speculator entries in one load: lane e holds entry e
  // (loading the slots beside the mask saves a round on bunches with dirty
  // tiles but costs more on clean ones)
  int2 ent_lane = make_int2(0, 0);
  if (lane < n_dirty) {
    const int4 s = a.speculator[tb * a.S + lane];
    ent_lane = make_int2(s.x, s.y);
  }
  for (int ent = 0; ent < n_dirty; ++ent) {
    const int start = lane_value(ent_lane.x, ent);
    const int stop = lane_value(ent_lane.y, ent);
    const int n_slots = min(stop - start - 1, WT - 1);
    // the first chunk's row bounds and the partials do not depend on each
    // other: issue both before waiting
    int r = start + 1 + lane;
    bool in = r < stop;
    int p0 = in ? rp[r] : 0, p1 = in ? rp[r + 1] : 0;
    for (int i = lane; i < n_slots; i += kWave) slots[i] = y[start + 1 + i];
    // one wavefront owns `slots` and its LDS operations execute in order:
    // only the compiler must keep the order (no wait for memory); every load
    // of y above has returned before its value reached LDS, so the stores
    // below cannot overtake them, and other tiles touch other rows
    lds_handover();
    int base = 0;
    for (int rb = start + 1; rb < stop; rb += kWave) {
      if (rb != start + 1) {
        r = rb + lane;
        in = r < stop;
        p0 = in ? rp[r] : 0;
        p1 = in ? rp[r + 1] : 0;
      }
      const bool ne = in && (p0 != p1);
      const uint64_t bal = __ballot(ne);
      const int before = __popcll(bal & ((1ull << lane) - 1ull));
      if (in) y[r] = ne ? slots[min(base + before, max(n_slots - 1, 0))] : (YT)0;
      base += __popcll(bal);
    }
    lds_handover();
  }
}

// (2) synchronizer carries for thread-bunches chunk0 .. chunk0+63 (one lane
// each): for each run of bunches whose first row is the same row r, sum their
// first-segment sums in double and write y[r] once.  Unless row r begins
// exactly where the run's first bunch begins, the part of r computed before
// the run is the tail of the bunch before the run (double), added first; y[r]
// is rounded to its type only here.  Runs of up to kShortRun bunches are
// summed by the run's first lane in bunch order, from this chunk's entries
// and the kShortRun after it staged in the wavefront's LDS (`lds`: at least
// (64 + kShortRun) * 12 bytes; register arrays for that look-ahead would cap
// the kernel's occupancy); longer runs (rows longer than kShortRun bunches)
// by the whole wavefront: coalesced loads, per-lane partial sums, then a
// fixed-shape tree over the lanes, so the rounding does not depend on timing.
// CROSSING_ONLY: only rows that began before their bunch or end behind it, the
// others are complete.
template <typename YT, bool CROSSING_ONLY>
__device__ __forceinline__ void fixup_carries(const MatCtx &a, const int64_t chunk0, const int lane, void *lds) {
  const int32_t *__restrict__ rp = a.row_ptr;
  YT *y = static_cast<YT *>(a.y);
  const int64_t SWT = (int64_t)a.S * a.W * kWave;
  const int64_t nb = a.n_bunches;
  const int64_t tb = chunk0 + lane;
  const bool valid = tb < nb;
  // one round of loads: this chunk's entries, the kShortRun entries after it
  // (lanes 0..kShortRun-1) and the one before it.  Entries past the last
  // bunch read as index -1, value 0.
  const int idx = valid ? a.state[tb].sync_idx : -1;
  const double own_v = valid ? a.state[tb].sync_val : 0.0;
  const int64_t tt = chunk0 + kWave + lane;
  const bool tail_in = lane < kShortRun && tt < nb;
  const int tail_i = tail_in ? a.state[tt].sync_idx : -1;
  const double tail_v = tail_in ? a.state[tt].sync_val : 0.0;
  const int before_chunk = chunk0 > 0 ? a.state[chunk0 - 1].sync_idx : -1;
  double *s_val = static_cast<double *>(lds);
  int *s_idx = reinterpret_cast<int *>(s_val + kWave + kShortRun);
  s_idx[lane] = idx;
  s_val[lane] = own_v;
  if (lane < kShortRun) {
    s_idx[kWave + lane] = tail_i;
    s_val[kWave + lane] = tail_v;
  }
  // one wavefront owns `lds` and its LDS operations run in order
  lds_handover();
  const int prev = wave_prev(idx, before_chunk);
  const bool head = valid && (tb == 0 || prev != idx);
  const bool is_long = head && (tb + kShortRun < nb) && (s_idx[lane + kShortRun] == idx);
  if (head && !is_long) {
    const int rs = rp[idx];
    // (the row of a run of more than one bunch ends behind its first)
    if (!CROSSING_ONLY || long_crossing(rs, rp[idx + 1], tb * SWT, SWT, back_limit(true))) {
      // sync_idx is non-decreasing (entries past the end read -1): the run is
      // the prefix of the next kShortRun entries equal to idx
      double sum = 0.0;
      for (int j = 0; j < kShortRun; ++j) {
        if (s_idx[lane + j] != idx) break;
        sum += s_val[lane + j];
      }
      const bool fresh = (int64_t)rs == tb * SWT;
      y[idx] = (YT)(fresh ? sum : a.state[tb - 1].tail_val + sum);
    }
  }
  uint64_t longs = __ballot(is_long);
  while (longs) {
    const int l = __ffsll((unsigned long long)longs) - 1;
    longs &= longs - 1;
    const int64_t t0 = __shfl(tb, l, kWave);
    const int ridx = __shfl(idx, l, kWave);
    double acc = 0.0;
    // (kRound chunks of loads in flight: one after another, a row of 3M entries
    // over 2,930 bunches took 52.1 us a product, with them 41.5)
    constexpr int kRound = 4;
    for (int64_t off = 0;; off += kRound * kWave) {
      int at[kRound];
      double v[kRound];
#pragma unroll
      for (int u = 0; u < kRound; ++u) {
        const int64_t j = t0 + off + u * kWave + lane;
        const BunchState &st = a.state[imin64(j, nb - 1)];
        at[u] = j < nb ? st.sync_idx : -1;
        v[u] = st.sync_val;
      }
#pragma unroll
      for (int u = 0; u < kRound; ++u)
        if (at[u] == ridx) acc += v[u];
      if (__ballot(at[kRound - 1] == ridx) != ~0ull) break;
    }
    const double total = wave_sum_tree(acc);
    if (lane == l) {
      const bool fresh = (int64_t)rp[ridx] == t0 * SWT;
      y[ridx] = (YT)(fresh ? total : a.state[t0 - 1].tail_val + total);
    }
  }
  // the staged entries are read before the wavefront's next use of `lds`
  lds_handover();
}

// (2b) a bound plan whose row_ptr was rewritten in place: the dirty bunches
// of chunk0 .. chunk0+63 that its list lacks, one after another (the listed
// ones have their own wavefronts).
template <typename YT>
__device__ __forceinline__ void fixup_unlisted(const MatCtx &a, const int64_t chunk0, YT *slots, const int lane) {
  // listed: the top bit of bunch_row
  const int64_t tb = chunk0 + lane;
  const bool todo = tb < a.n_bunches && a.state[tb].dirty_mask != 0 && a.bunch_row[tb] >= 0;
  uint64_t todo_bits = __ballot(todo);
  while (todo_bits) {
    const int l = __ffsll((unsigned long long)todo_bits) - 1;
    todo_bits &= todo_bits - 1;
    fixup_dirty<YT>(a, chunk0 + l, slots, lane);
  }
}

// (3) rows before the first tile's start row are empty and covered by no
// tile (all rows when nnz = 0): zero them, threads first..first+stride..
template <typename YT>
__device__ __forceinline__ void fixup_leading(const MatCtx &a, const int64_t first, const int64_t stride) {
  YT *y = static_cast<YT *>(a.y);
  const int64_t r_first = a.n_bunches > 0 ? a.state[0].sync_idx : a.m;
  for (int64_t r = first; r < r_first; r += stride) y[r] = (YT)0;
}

// Stage 2 of one matrix: the first ceil(n_bunches / 64) wavefronts settle the
// carries of 64 bunches each, the next n_bunches wavefronts re-arrange one
// bunch's dirty tiles each (separate wavefronts, so the two chains of
// dependent loads run side by side; a wavefront per bunch measured faster
// than a resident grid striding over the bunches, even where most bunches
// are clean); all threads share the leading rows.  The three parts write
// disjoint rows.
template <typename YT>
__global__ __launch_bounds__(1024) void sss_fixup(MatCtx a) {
  extern __shared__ unsigned char lds_raw[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  YT *slots = reinterpret_cast<YT *>(lds_raw) + (size_t)wid * a.W * kWave;
  const int64_t wave = (int64_t)blockIdx.x * (blockDim.x / kWave) + wid;
  const int64_t n_chunks = (a.n_bunches + kWave - 1) / kWave;
  if (wave < n_chunks) {
    fixup_carries<YT, false>(a, wave * kWave, lane, slots);
    if (a.dirty_list && *a.stale) fixup_unlisted<YT>(a, wave * kWave, slots, lane);
  } else if (wave < n_chunks + a.n_fix) {
    fixup_dirty<YT>(a, a.dirty_list ? (int64_t)a.dirty_list[wave - n_chunks] : wave - n_chunks, slots, lane);
  }
  fixup_leading<YT>(a, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

// After the fused kernel, where some row is a long crossing row: the carries of
// the rows that cross, one wavefront per 64 bunches.  What it costs is a launch that depends on the
// one before it (4 to 5 us behind a running kernel) and one chain of loads,
// so a plan that knows it has no such row leaves it out.
template <typename YT>
__global__ __launch_bounds__(kCarryThreads) void sss_carries(MatCtx a) {
  __shared__ double lds[kCarryThreads / kWave][kCarryLds];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const int64_t chunk0 = ((int64_t)blockIdx.x * (kCarryThreads / kWave) + wid) * kWave;
  if (chunk0 < a.n_bunches) fixup_carries<YT, true>(a, chunk0, lane, lds[wid]);
}

// The same for a batch, persistent: work items 0..total_chunks-1 settle one
// carry chunk (64 bunches of one matrix) each (none when no matrix has a long
// crossing row), the last count zero the y of the matrices without a nonzero.
template <typename YT>
__global__ __launch_bounds__(kCarryThreads) void sss_carries_batch(BatchArgs b) {
  __shared__ double lds[kCarryThreads / kWave][kCarryLds];
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const int64_t n_waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  for (int64_t w = (int64_t)blockIdx.x * (blockDim.x / kWave) + wid; w < b.total_waves; w += n_waves) {
    if (w < b.total_chunks) {
      const int i = __builtin_amdgcn_readfirstlane((int)wave_rightmost(b.chunk_base, (int64_t)b.count, w, lane));
      const MatCtx a = uniform_load(b.mats + i);
      fixup_carries<YT, true>(a, (w - uniform_load(b.chunk_base + i)) * kWave, lane, lds[wid]);
    } else {
      const MatCtx a = uniform_load(b.mats + __builtin_amdgcn_readfirstlane((int)(w - b.total_chunks)));
      if (a.n_bunches == 0) fixup_leading<YT>(a, lane, kWave);
    }
  }
}

template <typename YT>
__global__ void sss_fill_zero(YT *y, int64_t m) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (YT)0;
}

__global__ void sss_validate_kernel(const int32_t *rp, const int32_t *col, int64_t m, int64_t n, int64_t nnz,
                                    int *bad) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  if (tid == 0 && (rp[0] != 0 || (int64_t)rp[m] != nnz)) atomicOr(bad, 1);
  for (int64_t i = tid; i < m; i += nt)
    if (rp[i] > rp[i + 1]) atomicOr(bad, 2);
  for (int64_t k = tid; k < nnz; k += nt)
    if (col[k] < 0 || (int64_t)col[k] >= n) atomicOr(bad, 4);
}

// ---------------------------------------------------------------- host side

int default_W(int dt) { return dt == SSS_F64 ? 8 : 16; }
int default_S(int dt) { return dt == SSS_F64 ? 5 : 2; }
constexpr int kDefaultB = 2;
// threads per stage-2 workgroup: 64 and 128 measured ~0.8 us faster than
// 256 on the 1M-row matrix (fewer waves wait on the slowest in a workgroup)
#ifndef SSS_FIXUP_THREADS
#define SSS_FIXUP_THREADS 128
#endif
constexpr int kFixupThreads = SSS_FIXUP_THREADS;
constexpr size_t kFixupLdsBytes = 64 * 1024;  // LDS of one fixup workgroup
// a stage-2 wavefront's LDS (W * 64 y values, W >= 4, y at least 4 bytes)
// also holds the carry pass's staged entries
static_assert(4 * kWave * 4 >= (kWave + kShortRun) * (sizeof(double) + sizeof(int)), "carry staging fits");
constexpr int kMaxS = 16;

bool dtype_ok(int dt) { return dt == SSS_F64 || dt == SSS_F32 || dt == SSS_BF16; }
size_t y_size(int dt) { return dt == SSS_F64 ? 8 : 4; }

int fixup_waves_per_block(int W, int dt) {
  return (int)std::max<size_t>(1, std::min<size_t>(kFixupThreads / kWave,
                                                    kFixupLdsBytes / ((size_t)W * kWave * y_size(dt))));
}

using Stage1Fn = void (*)(MatCtx);
using BatchFn = void (*)(BatchArgs);

template <int DT, int W>
Stage1Fn pick_stage1(bool debug) { return debug ? sss_stage1<DT, W, true> : sss_stage1<DT, W, false>; }

template <int DT, int W>
Stage1Fn pick_fused(Form form) {
  return form == kCached ? sss_fused<DT, W, kCached>
                         : (form == kStreamed ? sss_fused<DT, W, kStreamed> : sss_fused<DT, W, kWide>);
}

using DotFn = void (*)(MatCtx, double *);
template <int W>
DotFn pick_dot(Form form) { return form == kCached ? sss_fused_dot<W, kCached> : sss_fused_dot<W, kStreamed>; }

template <int DT, int W, Form FORM>
BatchFn pick_batch_form(bool persistent) {
  return persistent ? sss_fused_batch_persistent<DT, W, FORM> : sss_fused_batch<DT, W, FORM>;
}

template <int DT, int W>
BatchFn pick_batch(Form form, bool persistent) {
  return form == kCached ? pick_batch_form<DT, W, kCached>(persistent)
                         : (form == kStreamed ? pick_batch_form<DT, W, kStreamed>(persistent)
                                              : pick_batch_form<DT, W, kWide>(persistent));
}

// the instance of a value type and W: PICK<DT, W>(args)
#define SSS_PICK_W(PICK, DT, W, ...) \
  (W == 4 ? PICK<DT, 4>(__VA_ARGS__) : (W == 8 ? PICK<DT, 8>(__VA_ARGS__) : (W == 16 ? PICK<DT, 16>(__VA_ARGS__) : nullptr)))
#define SSS_PICK(PICK, dt, W, ...)                                            \
  ((dt) == SSS_F64 ? SSS_PICK_W(PICK, SSS_F64, W, __VA_ARGS__)                \
                   : ((dt) == SSS_F32 ? SSS_PICK_W(PICK, SSS_F32, W, __VA_ARGS__) \
                                      : SSS_PICK_W(PICK, SSS_BF16, W, __VA_ARGS__)))

}  // namespace

struct sss_plan_s {
  int device = 0;
  int64_t m = 0, n = 0, nnz = 0;
  int dt = SSS_F64;
  int W = 8, S = 5, B = 2;
  int debug = 0;
  int bind_rows = 0;
  const int32_t *bound_row_ptr = nullptr;  // bind_rows plans: the row_ptr they were made for
  int64_t n_tiles = 0, n_bunches = 0;
  void *aux = nullptr;
  bool owns_aux = false;  // false: caller-provided workspace, or the static scratch
  BunchState *state = nullptr;
  int4 *speculator = nullptr;
  int32_t *bunch_row = nullptr;  // plans made with bind_rows only
  int32_t *dirty_list = nullptr; // bind_rows plans: the bunches with a dirty tile, found at plan time
  int64_t n_listed = 0;
  int32_t *stale = nullptr;      // bind_rows plans: see MatCtx::stale; the word after it: any long crossing row
  int32_t *arrivals = nullptr;   // bind_rows plans: see MatCtx::arrivals
  int32_t carries = 1;           // 0: no long crossing row at plan time (see sss_fused), so no second launch
  int4 *slots = nullptr;         // bind_rows plans: see MatCtx::slots
  uint32_t *order_hist = nullptr;
  double *dots = nullptr;        // bind_rows FP64 plans: see sss_fused_dot
  bool ordered = false;          // bind_rows plans: slots are in column order
  bool call_order = false;       // plans without bind_rows: every call makes bunch_row and slots, see orders_calls
  int64_t n_slots = 0;
  int32_t *dbg_start = nullptr;
  int32_t *dbg_dirty = nullptr;
  uint32_t *dbg_heads = nullptr;
  // batch plans only
  bool batch = false;
  bool batch_persistent = false;
  Form batch_form = kCached;
  BatchArgs bargs{};
  std::vector<int> mat_S;  // each matrix's tiles per thread-bunch
  int blocks1 = 0, blocks2 = 0;
  hipStream_t capture_stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t graph_exec = nullptr;
};

namespace {

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Byte offsets of a plan's auxiliary arrays in one device buffer (Section
// 3.3 sizes them: one synchronizer entry per thread-bunch, one speculator
// entry per tile), every array 256-byte aligned.
struct AuxLayout {
  int64_t n_tiles = 0, n_bunches = 0;
  size_t state = 0, spec = 0, brow = 0, dlist = 0, stale = 0, slots = 0, ohist = 0, dots = 0, arrivals = 0,
         dstart = 0, ddirty = 0, dheads = 0;
  size_t total = 0;
};

AuxLayout aux_layout(int64_t nnz, int W, int S, bool bind, bool debug, bool call_order) {
  AuxLayout L;
  const int WT = W * kWave;
  L.n_tiles = nnz > 0 ? (nnz + WT - 1) / WT : 0;
  const int64_t SWT = (int64_t)S * WT;
  L.n_bunches = nnz > 0 ? (nnz + SWT - 1) / SWT : 0;
  const size_t nt = (size_t)L.n_tiles, nb = (size_t)L.n_bunches;
  size_t off = 0;
  // (the size of two 4-byte and two 8-byte arrays, which the largest nnz of
  // sss_csr_spmv_noalloc is stated for)
  L.state = off; off += 2 * align256(sizeof(int32_t) * (nb + 1)) + 2 * align256(sizeof(double) * (nb + 1));
  L.spec = off; off = align256(off + sizeof(int4) * (nb * (size_t)S + 1));
  if (bind || call_order) {
    L.brow = off; off += sizeof(int32_t) * nb;
    L.stale = off; off = align256(off + sizeof(int32_t) * 2);  // (behind the rows: the plan copies both at once)
    L.dlist = off; off = align256(off + sizeof(int32_t) * (nb + 1));
  }
  if (bind || call_order) {
    L.slots = off; off = align256(off + sizeof(int4) * (nb + kXcds * kMaxB));
    L.ohist = off; off = align256(off + sizeof(uint32_t) * 2 * (kOrderBins + 1));
  }
  if (bind) {
    L.dots = off; off = align256(off + sizeof(double) * (nb + kXcds * kMaxB));
    L.arrivals = off; off = align256(off + sizeof(int32_t) * (nb + 1));
  }
  if (debug) {
    L.dstart = off; off = align256(off + sizeof(int32_t) * (nt + 1));
    L.ddirty = off; off = align256(off + sizeof(int32_t) * (nt + 1));
    L.dheads = off; off = align256(off + sizeof(uint32_t) * (nt + 1) * (size_t)(WT / 32));
  }
  L.total = off;
  return L;
}

// Point the plan's arrays into `base` (a buffer of at least L.total bytes).
void plan_bind_aux(sss_plan p, const AuxLayout &L, void *base_v) {
  char *base = static_cast<char *>(base_v);
  p->n_tiles = L.n_tiles;
  p->n_bunches = L.n_bunches;
  p->aux = base_v;
  p->state = reinterpret_cast<BunchState *>(base + L.state);
  p->speculator = reinterpret_cast<int4 *>(base + L.spec);
  p->arrivals = p->bind_rows ? reinterpret_cast<int32_t *>(base + L.arrivals) : nullptr;
  p->dots = p->bind_rows ? reinterpret_cast<double *>(base + L.dots) : nullptr;
  p->bunch_row = p->bind_rows || p->call_order ? reinterpret_cast<int32_t *>(base + L.brow) : nullptr;
  p->dirty_list = p->bind_rows ? reinterpret_cast<int32_t *>(base + L.dlist) : nullptr;
  p->stale = p->bind_rows ? reinterpret_cast<int32_t *>(base + L.stale) : nullptr;
  p->carries = L.n_bunches > 1 ? 1 : 0;
  const bool slots = p->bind_rows || p->call_order;
  p->slots = slots ? reinterpret_cast<int4 *>(base + L.slots) : nullptr;
  p->order_hist = slots ? reinterpret_cast<uint32_t *>(base + L.ohist) : nullptr;
  p->dbg_start = p->debug ? reinterpret_cast<int32_t *>(base + L.dstart) : nullptr;
  p->dbg_dirty = p->debug ? reinterpret_cast<int32_t *>(base + L.ddirty) : nullptr;
  p->dbg_heads = p->debug ? reinterpret_cast<uint32_t *>(base + L.dheads) : nullptr;
}

// The plan's auxiliary buffer: the caller's workspace when given (nothing is
// allocated), else one hipMalloc owned by the plan.  Cleared on `stream`
// (stream-ordered; the caller of plan_create synchronises that stream).
int plan_alloc(sss_plan p, void *workspace, size_t workspace_bytes, hipStream_t stream) {
  const AuxLayout L = aux_layout(p->nnz, p->W, p->S, p->bind_rows != 0, p->debug != 0, p->call_order);
  void *base = workspace;
  if (workspace) {
    if (workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return SSS_ERR_INVALID_VALUE;
  } else {
    SSS_HIP(hipMalloc(&base, L.total));
    p->owns_aux = true;
  }
  plan_bind_aux(p, L, base);
  SSS_HIP(hipMemsetAsync(base, 0, L.total, stream));
  return SSS_OK;
}

bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

int check_call(sss_plan p, const int32_t *row_ptr, const int32_t *col, const void *val, const void *x, void *y) {
  if (p->m == 0) return SSS_OK;
  if (!row_ptr || !y) return SSS_ERR_INVALID_VALUE;
  if (p->nnz > 0) {
    if (!col || !val || !x) return SSS_ERR_INVALID_VALUE;
    if (misaligned(col) || misaligned(val)) return SSS_ERR_INVALID_VALUE;
  }
  // a plan whose rows were bound at plan time serves the row_ptr it was made
  // for (stage 1 also checks every bound row against row_ptr's contents and
  // searches again where one no longer holds, so y stays right even if that
  // array was rewritten in place)
  if (p->bind_rows && row_ptr != p->bound_row_ptr) return SSS_ERR_PLAN_MISMATCH;
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev != p->device) return SSS_ERR_PLAN_MISMATCH;
  return SSS_OK;
}

// The form of a matrix (or a whole batch; n_max, its largest x).
// Streamed from 300 MB of matrix and vectors on: less of it stays in the 256 MB
// last-level cache from one product to the next, and non-temporal loads would
// give that up.  us per product cached / streamed, one matrix again and again:
// 120 MB power law 62.2 / 72.0, 163 MB 27-point stencil 33.3 / 36.8, 248 MB FEM
// band 41.0 / 45.4, 285 MB FEM band 46.6 / 51.7, 322 MB FEM band 60.6 / 61.0,
// FP32 320 MB 63.5 / 61.8, 455 MB 27-point stencil 89.1 / 85.3.
// Where x has outgrown what an XCD's 4 MiB of L2 keep beside the streamed
// matrix, keeping the matrix out of it is worth more, and the line is 100 MB.
// The time streamed over cached, in the mean of random rows, power law, dense
// rows and a band (W = 8, S = 2), one matrix again and again | three in turn:
//   x, MB     80 MB           100 MB          140 MB          260 MB
//   FP64 4.0  1.007 | 1.044   1.043 | 0.981   1.060 | 0.935   1.097 | 0.929
//        5.0  0.996 | 1.025   1.013 | 0.993   1.032 | 0.941   1.052 | 0.941
//        5.6  0.954 | 0.990   0.989 | 0.978   0.995 | 0.931   1.005 | 0.923
//   FP32 4.4  1.022 | 1.050   1.031 | 0.990   1.052 | 0.943   1.084 | 0.943
//        5.6  0.967 | 0.997   0.982 | 0.969   0.997 | 0.935   1.022 | 0.933
// so the two uses cross between 5.0 and 5.6 MB of x.  At 80 MB a product alone
// would gain already, but a CG step, whose vectors pass the cache between
// products, loses 1.2% (1024^2 Laplacian, 84 MB) and nothing at 97 MB.  The
// mean hides a spread: from 140 to 300 MB, multiplied again and again, rows that
// read all over x gain 3 to 9% and a band, whose gathers hit, loses up to 16%;
// in turn all gain 4 to 9%.
constexpr int64_t kStreamBytes = 300000000, kStreamX = 5500000, kStreamBytesX = 100000000;
Form form_of(int64_t m, int64_t n, int64_t nnz, int dt, int64_t n_max) {
  if (n_max * (int64_t)y_size(dt) > 0xfffffff0ll) return kWide;
  const int64_t value = dt == SSS_F64 ? 8 : (dt == SSS_F32 ? 4 : 2);
  const int64_t from = n_max * (int64_t)y_size(dt) >= kStreamX ? kStreamBytesX : kStreamBytes;
  return nnz * (4 + value) + 4 * m + (m + n) * (int64_t)y_size(dt) >= from ? kStreamed : kCached;
}

// The kernels' view of a single-matrix plan and the caller's arrays.
MatCtx plan_ctx(sss_plan p, const int32_t *row_ptr, const int32_t *col, const void *val, const void *x, void *y) {
  MatCtx a{};
  a.row_ptr = row_ptr; a.col = col; a.val = val; a.x = x; a.y = y;
  a.m = (int32_t)p->m; a.nnz = (int32_t)p->nnz; a.S = p->S; a.W = p->W;
  a.n_bunches = p->n_bunches; a.n_tiles = p->n_tiles;
  a.state = p->state; a.speculator = p->speculator;
  a.bunch_row = p->bind_rows ? p->bunch_row : nullptr;
  a.dirty_list = p->dirty_list;
  a.n_fix = p->dirty_list ? p->n_listed : p->n_bunches;
  a.stale = p->stale;
  a.carries = p->carries; a.keep_state = 1; a.arrivals = p->arrivals;
  a.slots = p->bind_rows ? p->slots : nullptr;
  a.n_slots = p->n_slots;
  a.dbg_start = p->dbg_start; a.dbg_dirty = p->dbg_dirty; a.dbg_heads = p->dbg_heads;
  return a;
}

// Stage 1's column order (see sss_order_keys) can gain where x is larger than
// what stays in an XCD's 4 MB L2 beside the streamed matrix (power law, Zipf
// and dense rows: 2.16 MB of x 1% slower to 1% faster, 2.8 MB 1 to 3%, 3.2 MB
// 2 to 4%, 4 MB 6 to 9%, 8 MB 9 to 22% faster).
constexpr int64_t kOrderMinX = int64_t(5) << 19;
constexpr int64_t kOrderMinBunches = 2048;

// Whether the calls of a plan without bind_rows make the slots in column order
// themselves, three short launches before the fused kernel.  us per product
// without / with: 4M-row Zipf 1.8 FP32 (80M nonzeros) 1,095 / 818, 2M-row
// power law FP64 (40M) 569 / 465, 1M rows of it (20M) 213 / 189; where no row
// is long they only cost, 8 us beside a short kernel: 5-point stencils 42 /
// 51 (10M) and 97 / 107 (24M), 27-point stencils 59 / 65 (19M) and 128 / 130
// (46M), a FEM band 125 / 126 (50M).
constexpr int64_t kCallOrderNnz = 32000000;
bool orders_calls(int64_t nnz, int64_t n, int dt) {
  return nnz >= kCallOrderNnz && n * (int64_t)y_size(dt) >= kOrderMinX;
}

int64_t slots_of(sss_plan p) {
  const int64_t group = (int64_t)kXcds * p->B;
  return (p->n_bunches + group - 1) / group * group;
}

int launch_call_order(sss_plan p, const int32_t *row_ptr, MatCtx &a, hipStream_t s) {
  const int64_t nb = p->n_bunches, n_slots = slots_of(p);
  const int32_t m = (int32_t)p->m, SWT = p->S * p->W * kWave;
  const unsigned row_blocks = (unsigned)std::min<int64_t>((p->m + 255) / 256, 8192);
  uint32_t *keys = reinterpret_cast<uint32_t *>(p->speculator), *hist = p->order_hist;
  hipLaunchKernelGGL(sss_call_rows, dim3(row_blocks), dim3(256), 0, s, row_ptr, m,
                     (int32_t)p->nnz, SWT, (uint32_t)nb, p->bunch_row, keys, hist);
  SSS_HIP(hipGetLastError());
  hipLaunchKernelGGL(sss_order_keys<false>, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, row_ptr, m,
                     (int32_t)p->nnz, (int64_t)SWT, nb, p->bunch_row, keys, hist);
  SSS_HIP(hipGetLastError());
  hipLaunchKernelGGL(sss_order_scatter, dim3((unsigned)((n_slots + 255) / 256)), dim3(256), 0, s, row_ptr, m,
                     (int64_t)SWT, nb, p->bunch_row, keys, n_slots, p->B, hist, hist + kOrderBins + 1, p->carries != 0, p->slots);
  SSS_HIP(hipGetLastError());
  a.slots = p->slots;
  a.n_slots = n_slots;
  return SSS_OK;
}

// Rows per wavefront from which on the fused kernel gets wavefronts without a
// bunch, which only take their share of the leading rows (see zero_leading).
// Matrices with 0.6 entries per row and more (SWT = 2,560) have enough bunches.
constexpr int64_t kLeadingRows = 4096;

// Stage 1 alone (`split`), or the fused kernel.  (nnz = 0: y is zeroed here.)
int launch_stage1(sss_plan p, const int32_t *row_ptr, const int32_t *col, const void *val, const void *x, void *y,
                  bool split, hipStream_t stream) {
  if (p->m == 0) return SSS_OK;
  if (p->nnz == 0) {
    const int blocks = (int)std::min<int64_t>((p->m + 255) / 256, 4096);
    if (p->dt == SSS_F64)
      hipLaunchKernelGGL(sss_fill_zero<double>, dim3(blocks), dim3(256), 0, stream, (double *)y, p->m);
    else
      hipLaunchKernelGGL(sss_fill_zero<float>, dim3(blocks), dim3(256), 0, stream, (float *)y, p->m);
    SSS_HIP(hipGetLastError());
    return SSS_OK;
  }
  Stage1Fn k1 = split ? SSS_PICK(pick_stage1, p->dt, p->W, p->debug != 0)
                      : SSS_PICK(pick_fused, p->dt, p->W, form_of(p->m, p->n, p->nnz, p->dt, p->n));
  if (!k1) return SSS_ERR_UNSUPPORTED;
  MatCtx a1 = plan_ctx(p, row_ptr, col, val, x, y);
  if (!split && p->call_order) {
    const int rc = launch_call_order(p, row_ptr, a1, stream);
    if (rc != SSS_OK) return rc;
  }
  int64_t waves1 = a1.slots ? a1.n_slots : p->n_bunches;
  if (!split) waves1 = std::max(waves1, p->m / kLeadingRows);
  const int64_t blocks1 = (waves1 + p->B - 1) / p->B;
  a1.n_shares = blocks1 * p->B;
  const size_t lds1 = (size_t)p->B * stage1_lds_words(p->W, p->S) * sizeof(uint32_t);
  hipLaunchKernelGGL(k1, dim3((unsigned)blocks1), dim3(p->B * kWave), lds1, stream, a1);
  SSS_HIP(hipGetLastError());
  return SSS_OK;
}

// Stage 2: checking prediction (synchronizer carries, dirty-tile
// re-arrangement, leading empty rows).
int launch_stage2(sss_plan p, const int32_t *row_ptr, void *y, hipStream_t stream) {
  if (p->m == 0 || p->nnz == 0) return SSS_OK;
  const int WT = p->W * kWave;
  const MatCtx a2 = plan_ctx(p, row_ptr, nullptr, nullptr, nullptr, y);
  // one wavefront per 64 bunches (their carry runs), then one per thread-bunch
  // that can hold dirty tiles: every bunch, or a bound plan's listed ones
  const int wpb = fixup_waves_per_block(p->W, p->dt);
  const int64_t waves2 = (p->n_bunches + kWave - 1) / kWave + a2.n_fix;
  const int64_t blocks2 = std::max<int64_t>(1, (waves2 + wpb - 1) / wpb);
  const size_t lds2 = (size_t)wpb * WT * y_size(p->dt);
  if (p->dt == SSS_F64)
    hipLaunchKernelGGL(sss_fixup<double>, dim3((unsigned)blocks2), dim3(wpb * kWave), lds2, stream, a2);
  else
    hipLaunchKernelGGL(sss_fixup<float>, dim3((unsigned)blocks2), dim3(wpb * kWave), lds2, stream, a2);
  SSS_HIP(hipGetLastError());
  return SSS_OK;
}

int launch(sss_plan p, const int32_t *row_ptr, const int32_t *col, const void *val, const void *x, void *y,
           hipStream_t stream) {
  int rc = check_call(p, row_ptr, col, val, x, y);
  if (rc != SSS_OK || p->m == 0) return rc;
  // a debug plan records the two stages as the paper has them
  rc = launch_stage1(p, row_ptr, col, val, x, y, p->debug != 0, stream);
  if (rc != SSS_OK || p->nnz == 0) return rc;
  if (p->debug) return launch_stage2(p, row_ptr, y, stream);
  if (!p->carries) return SSS_OK;
  const MatCtx a = plan_ctx(p, row_ptr, nullptr, nullptr, nullptr, y);
  const int64_t per_block = (int64_t)(kCarryThreads / kWave) * kWave;
  const unsigned blocks = (unsigned)((p->n_bunches + per_block - 1) / per_block);
  if (p->dt == SSS_F64)
    hipLaunchKernelGGL(sss_carries<double>, dim3(blocks), dim3(kCarryThreads), 0, stream, a);
  else
    hipLaunchKernelGGL(sss_carries<float>, dim3(blocks), dim3(kCarryThreads), 0, stream, a);
  SSS_HIP(hipGetLastError());
  return SSS_OK;
}

// Every workgroup of the reader adds up all the sums of sss_fused_dot, which
// from some number on costs more than the launch saved.  50 CG steps on
// Laplacians, us with a pass of its own / with the sums: 64^2 (80 sums) 775 /
// 625, 256^2 786 / 664, 512^2 (2,560) 972 / 927, 700^2 1,383 / 1,319, 1024^2
// (5,117) 1,955 / 1,996, 900^2 (3,950) 1,681 / 1,704, (7,900) 1,672 / 1,858.
constexpr int64_t kMaxDots = 3072;

// A batch plan: the fused launch (one wavefront per thread-bunch of every
// matrix, or the persistent form), then the carries where the plan needs them.
int launch_batch(sss_plan p, hipStream_t stream) {
  if (p->bargs.total_bunches > 0) {
    BatchFn k1 = SSS_PICK(pick_batch, p->dt, p->W, p->batch_form, p->batch_persistent);
    if (!k1) return SSS_ERR_UNSUPPORTED;
    const size_t lds1 = (size_t)p->B * stage1_lds_words(p->W, p->bargs.S_max) * sizeof(uint32_t);
    hipLaunchKernelGGL(k1, dim3((unsigned)p->blocks1), dim3(p->B * kWave), lds1, stream, p->bargs);
    SSS_HIP(hipGetLastError());
  }
  if (p->bargs.total_waves == 0) return SSS_OK;
  if (p->dt == SSS_F64)
    hipLaunchKernelGGL(sss_carries_batch<double>, dim3((unsigned)p->blocks2), dim3(kCarryThreads), 0, stream, p->bargs);
  else
    hipLaunchKernelGGL(sss_carries_batch<float>, dim3((unsigned)p->blocks2), dim3(kCarryThreads), 0, stream, p->bargs);
  SSS_HIP(hipGetLastError());
  return SSS_OK;
}

// The tile schedule of the one-call forms, which keep no plan of the
// caller's.  The paper's S = 5 leaves a GPU of 256 CUs idle on all but large
// matrices; each line is where the next schedule's geometric mean over 5- and
// 27-point stencils, a FEM band, Poisson, web-like, power-law, Zipf and
// dense-row matrices takes over (three matrices in turn, time of the schedule
// below the line over the one above it): W = 4, S = 1 over W = 8, S = 1 0.975 at
// 500K nonzeros, 0.978 at 600K, 1.011 at 700K, 1.017 at 1M; over S = 2 0.975 at
// 1.4M, 0.988 at 2M, 1.020 at 2.8M, 1.057 at 4M; S = 2 over S = 5 0.991 at 5.6M,
// 1.005 at 8M, 0.980 at 11M, 1.027 at 16M.
void one_call_params(int64_t nnz, int *W, int *S) {
  *W = nnz < 650000 ? 4 : 8;
  *S = nnz < 2300000 ? 1 : (nnz < 8000000 ? 2 : 5);
}

std::mutex g_cache_mu;
std::map<std::tuple<int, void *, int64_t, int64_t, int64_t>, sss_plan> g_cache;

// sss_validate_csr's result word: one per device, in the code object (no
// allocation per call); calls are serialised by a mutex, each waits for its
// stream before it returns
__device__ int validate_flag;
constexpr int kMaxDevices = 64;
std::mutex g_validate_mu;
int *g_validate_ptr[kMaxDevices] = {};

// sss_csr_spmv_noalloc's plan arrays (what a double-precision plan of its
// schedule holds): a static array in the code
// object, one per device, held until the process ends.  Host code never uses
// its name as an address: the device address comes from hipGetSymbolAddress,
// once per device.  Every call on a device shares it; stage 1 writes every
// entry stage 2 reads, so nothing needs clearing between calls.
constexpr size_t kScratchBytes = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

template <int DT, int W>
int launch_floor(sss_plan p, const MatCtx &a, void *out, int gather, hipStream_t stream) {
  using y_t = typename VT<DT>::y_t;
  const int64_t blocks = (p->n_bunches + p->B - 1) / p->B;
  if (gather)
    hipLaunchKernelGGL((sss_floor<DT, W, true>), dim3((unsigned)blocks), dim3(p->B * kWave), 0, stream, a,
                       static_cast<y_t *>(out));
  else
    hipLaunchKernelGGL((sss_floor<DT, W, false>), dim3((unsigned)blocks), dim3(p->B * kWave), 0, stream, a,
                       static_cast<y_t *>(out));
  SSS_HIP(hipGetLastError());
  return SSS_OK;
}

template <int DT, int W>
int launch_floor_batch(sss_plan p, void *out, int gather, hipStream_t stream) {
  using y_t = typename VT<DT>::y_t;
  if (gather)
    hipLaunchKernelGGL((sss_floor_batch<DT, W, true>), dim3((unsigned)p->blocks1), dim3(p->B * kWave), 0, stream,
                       p->bargs, static_cast<y_t *>(out));
  else
    hipLaunchKernelGGL((sss_floor_batch<DT, W, false>), dim3((unsigned)p->blocks1), dim3(p->B * kWave), 0, stream,
                       p->bargs, static_cast<y_t *>(out));
  SSS_HIP(hipGetLastError());
  return SSS_OK;
}

template <int DT>
int launch_floor_batch_w(sss_plan p, void *out, int gather, hipStream_t stream) {
  switch (p->W) {
    case 4: return launch_floor_batch<DT, 4>(p, out, gather, stream);
    case 8: return launch_floor_batch<DT, 8>(p, out, gather, stream);
    case 16: return launch_floor_batch<DT, 16>(p, out, gather, stream);
    default: return SSS_ERR_UNSUPPORTED;
  }
}

template <int DT>
int launch_floor_w(sss_plan p, const MatCtx &a, void *out, int gather, hipStream_t stream) {
  switch (p->W) {
    case 4: return launch_floor<DT, 4>(p, a, out, gather, stream);
    case 8: return launch_floor<DT, 8>(p, a, out, gather, stream);
    case 16: return launch_floor<DT, 16>(p, a, out, gather, stream);
    default: return SSS_ERR_UNSUPPORTED;
  }
}

// Stage 2 on a host core, as the paper runs it (Section 3.2, Section 3.4): the
// same three parts as the device kernel, on host arrays, one thread.
template <typename YT>
void stage2_host(sss_plan p, const int32_t *rp, YT *y, const BunchState *st, const int4 *spec) {
  const int64_t nb = p->n_bunches;
  const int64_t WT = (int64_t)p->W * kWave, SWT = (int64_t)p->S * WT;
  // leading empty rows
  const int64_t r_first = nb > 0 ? st[0].sync_idx : p->m;
  for (int64_t r = 0; r < r_first; ++r) y[r] = (YT)0;
  // dirty tiles: partial k >= 1 to the k-th non-empty row strictly inside
  std::vector<YT> slots((size_t)WT);
  for (int64_t tb = 0; tb < nb; ++tb) {
    const int n_dirty = __builtin_popcount(st[tb].dirty_mask);
    for (int e = 0; e < n_dirty; ++e) {
      const int4 s = spec[tb * p->S + e];
      const int start = s.x, stop = s.y;
      const int64_t n_slots = std::min<int64_t>((int64_t)stop - start - 1, WT - 1);
      for (int64_t i = 0; i < n_slots; ++i) slots[(size_t)i] = y[start + 1 + i];
      int64_t k = 0;
      for (int64_t r = start + 1; r < stop; ++r) {
        if (rp[r] != rp[r + 1]) y[r] = slots[(size_t)std::min<int64_t>(k++, std::max<int64_t>(n_slots - 1, 0))];
        else y[r] = (YT)0;
      }
    }
  }
  // carries: runs of bunches that begin in the same row, summed in bunch
  // order after the tail of the bunch before the run (unless the row begins
  // with the run)
  for (int64_t tb = 0; tb < nb;) {
    const int idx = st[tb].sync_idx;
    int64_t e = tb;
    double sum = 0.0;
    while (e < nb && st[e].sync_idx == idx) sum += st[e++].sync_val;
    const bool fresh = (int64_t)rp[idx] == tb * SWT;
    y[idx] = (YT)(fresh ? sum : st[tb - 1].tail_val + sum);
    tb = e;
  }
}

}  // namespace

extern "C" {

int sss_csr_spmv_plan_workspace_size(int64_t m, int64_t n, int64_t nnz, sss_dtype dt, const sss_plan_opts *opts,
                                     size_t *bytes) {
  if (!bytes) return SSS_ERR_INVALID_VALUE;
  *bytes = 0;
  if (m < 0 || n < 0 || nnz < 0 || m > SSS_MAX_INDEX || n > SSS_MAX_INDEX || nnz > SSS_MAX_INDEX)
    return SSS_ERR_INVALID_VALUE;
  if (!dtype_ok(dt)) return SSS_ERR_UNSUPPORTED;
  sss_plan_opts o{};
  o.mode = SSS_MODE_FIXED;
  if (opts) o = *opts;
  if (o.mode != SSS_MODE_FIXED && o.mode != SSS_MODE_SELECTOR) return SSS_ERR_UNSUPPORTED;
  const bool bind = o.bind_rows && m > 0 && nnz > 0, dbg = o.debug != 0;
  const bool order = !bind && !dbg && orders_calls(nnz, n, dt);
  size_t need = 0;
  if (o.mode == SSS_MODE_FIXED) {
    const int W = o.W ? o.W : default_W(dt), S = o.S ? o.S : default_S(dt);
    if (!(W == 4 || W == 8 || W == 16)) return SSS_ERR_UNSUPPORTED;
    if (S < 1 || S > kMaxS) return SSS_ERR_INVALID_VALUE;
    need = aux_layout(nnz, W, S, bind, dbg, order).total;
  } else {
    // the selector's choice is not known yet: the largest of the grid's
    // classes and the type's defaults
    need = aux_layout(nnz, default_W(dt), default_S(dt), bind, dbg, order).total;
    for (int c = 0; c < SSS_N_CLASSES; ++c) {
      int W = 0, S = 0;
      (void)sss_class_params(c, &W, &S);
      need = std::max(need, aux_layout(nnz, W, S, bind, dbg, order).total);
    }
  }
  *bytes = need;
  return SSS_OK;
}

namespace {

// Bound plans: stage 1's slots, in column order where that can gain and
// enough bunches lie in long rows.  The order is made on the device; the host
// reads back only how many bunches are short.  The speculator's space holds
// the keys (stage 1 writes every entry that stage 2 reads).
int plan_slots(sss_plan p, const int32_t *row_ptr, int64_t SWT, hipStream_t s) {
  const int64_t nb = p->n_bunches, x_bytes = p->n * (int64_t)y_size(p->dt);
  const unsigned blocks = (unsigned)((nb + 255) / 256);
  const int32_t m = (int32_t)p->m;
  if (x_bytes >= kOrderMinX && nb >= kOrderMinBunches) {
    const int64_t n_slots = slots_of(p);
    uint32_t *keys = reinterpret_cast<uint32_t *>(p->speculator), *hist = p->order_hist;
    hipLaunchKernelGGL(sss_order_keys<true>, dim3(blocks), dim3(256), 0, s, row_ptr, m, (int32_t)p->nnz, SWT, nb,
                       p->bunch_row, keys, hist);
    SSS_HIP(hipGetLastError());
    uint32_t n_short = 0;
    SSS_HIP(hipMemcpyAsync(&n_short, hist + kOrderBins, sizeof(n_short), hipMemcpyDeviceToHost, s));
    SSS_HIP(hipStreamSynchronize(s));
    if ((nb - (int64_t)n_short) * kOrderShare >= nb) {
      hipLaunchKernelGGL(sss_order_scatter, dim3((unsigned)((n_slots + 255) / 256)), dim3(256), 0, s, row_ptr, m, SWT,
                         nb, p->bunch_row, keys, n_slots, p->B, hist, hist + kOrderBins + 1, p->carries != 0, p->slots);
      SSS_HIP(hipGetLastError());
      p->n_slots = n_slots;
      p->ordered = true;
      return SSS_OK;
    }
  }
  hipLaunchKernelGGL(sss_slots, dim3(blocks), dim3(256), 0, s, row_ptr, m, SWT, nb, p->bunch_row, p->carries != 0,
                     p->slots);
  SSS_HIP(hipGetLastError());
  p->n_slots = nb;
  return SSS_OK;
}

// Bound plans: mark every bunch with a dirty tile on the device, then list
// them on the host (bunch order) and copy the list to the plan; reads back
// whether any row is a long crossing row; synchronises `s`.
int plan_list_dirty(sss_plan p, const int32_t *row_ptr, int64_t SWT, hipStream_t s) {
  const size_t nb = (size_t)p->n_bunches;
  const unsigned blocks = (unsigned)std::min<int64_t>((p->m + 255) / 256, 4096);
  hipLaunchKernelGGL(sss_mark_dirty_bunches, dim3(blocks), dim3(256), 0, s, row_ptr, (int32_t)p->m, SWT,
                     reinterpret_cast<uint32_t *>(p->bunch_row), 0x80000000u);
  SSS_HIP(hipGetLastError());
  std::vector<int32_t> br(nb + 2);  // the first rows and, behind them, the stale words
  SSS_HIP(hipMemcpyAsync(br.data(), p->bunch_row, br.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  SSS_HIP(hipStreamSynchronize(s));
  p->carries = br[nb + 1];
  std::vector<int32_t> list;
  for (size_t tb = 0; tb < nb; ++tb)
    if (br[tb] < 0) list.push_back((int32_t)tb);
  p->n_listed = (int64_t)list.size();
  if (!list.empty()) {
    SSS_HIP(hipMemcpyAsync(p->dirty_list, list.data(), list.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    SSS_HIP(hipStreamSynchronize(s));
  }
  return SSS_OK;
}

}  // namespace

int sss_csr_spmv_plan_create(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr, sss_dtype dt,
                             const sss_plan_opts *opts, void *stream, sss_plan *out) {
  if (!out) return SSS_ERR_INVALID_VALUE;
  *out = nullptr;
  if (m < 0 || n < 0 || nnz < 0 || m > SSS_MAX_INDEX || n > SSS_MAX_INDEX || nnz > SSS_MAX_INDEX)
    return SSS_ERR_INVALID_VALUE;
  if (!dtype_ok(dt)) return SSS_ERR_UNSUPPORTED;
  sss_plan_opts o{};
  o.mode = SSS_MODE_FIXED;
  if (opts) o = *opts;
  if (o.mode != SSS_MODE_FIXED && o.mode != SSS_MODE_SELECTOR) return SSS_ERR_UNSUPPORTED;
  int W = o.W ? o.W : default_W(dt);
  int S = o.S ? o.S : default_S(dt);
  const int B = o.B ? o.B : kDefaultB;
  if (o.mode == SSS_MODE_SELECTOR && m > 0 && nnz > 0) {
    if (!row_ptr) return SSS_ERR_INVALID_VALUE;
    if (sss_selector_loaded()) {
      float f[SSS_N_FEATURES];
      int cls = 0;
      int rc = sss_csr_features(m, n, nnz, row_ptr, dt, stream, f);
      if (rc == SSS_OK) rc = sss_selector_predict(f, &cls);
      if (rc == SSS_OK) rc = sss_class_params(cls, &W, &S);
      if (rc != SSS_OK) return rc;
    } else {
      W = default_W(dt);
      S = default_S(dt);
    }
  }
  if (!(W == 4 || W == 8 || W == 16)) return SSS_ERR_UNSUPPORTED;
  if (S < 1 || S > kMaxS || B < 1 || B > kMaxB) return SSS_ERR_INVALID_VALUE;
  if (o.bind_rows && m > 0 && nnz > 0 && !row_ptr) return SSS_ERR_INVALID_VALUE;
  if (!o.workspace && o.workspace_bytes) return SSS_ERR_INVALID_VALUE;
  sss_plan p = new sss_plan_s();
  p->m = m; p->n = n; p->nnz = nnz; p->dt = dt; p->W = W; p->S = S; p->B = B; p->debug = o.debug ? 1 : 0;
  p->bind_rows = (o.bind_rows && m > 0 && nnz > 0) ? 1 : 0;
  p->bound_row_ptr = p->bind_rows ? row_ptr : nullptr;
  p->call_order = !p->bind_rows && !p->debug && orders_calls(nnz, n, dt);
  hipStream_t s = static_cast<hipStream_t>(stream);
  int rc = SSS_OK;
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) { g_last_hip = e; rc = SSS_ERR_HIP; }
  if (rc == SSS_OK) rc = plan_alloc(p, o.workspace, o.workspace_bytes, s);
  if (rc == SSS_OK && p->bind_rows) {
    // each thread-bunch's first row, once for every later call
    const int64_t SWT = (int64_t)p->S * p->W * kWave;
    const unsigned blocks = (unsigned)std::min<int64_t>((p->n_bunches + 255) / 256, 65535);
    hipLaunchKernelGGL(sss_bunch_rows, dim3(blocks), dim3(256), 0, s, row_ptr, (int32_t)m, SWT, p->n_bunches,
                       p->bunch_row, p->stale + 1);
    e = hipGetLastError();
    if (e != hipSuccess) { g_last_hip = e; rc = SSS_ERR_HIP; }
    // the bunches with a dirty tile (marked in bunch_row's top bit), listed
    // in order so that stage 2 gives only them a wavefront
    if (rc == SSS_OK) rc = plan_list_dirty(p, row_ptr, SWT, s);
    if (rc == SSS_OK) rc = plan_slots(p, row_ptr, SWT, s);
  }
  if (rc == SSS_OK) {
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) { g_last_hip = e; rc = SSS_ERR_HIP; }
  }
  if (rc != SSS_OK) {
    if (p->owns_aux && p->aux) (void)hipFree(p->aux);
    delete p;
    return rc;
  }
  *out = p;
  return SSS_OK;
}

int sss_plan_dirty_list(sss_plan p, int32_t *host_out, int64_t cap, int64_t *n) {
  if (!p || !n || p->batch || cap < 0 || (cap > 0 && !host_out)) return SSS_ERR_INVALID_VALUE;
  if (!p->bind_rows && p->n_bunches > 0) return SSS_ERR_INVALID_VALUE;  // (no bunches: nothing to list)
  *n = p->n_listed;
  const int64_t k = std::min(cap, p->n_listed);
  if (k > 0) SSS_HIP(hipMemcpy(host_out, p->dirty_list, (size_t)k * sizeof(int32_t), hipMemcpyDeviceToHost));
  return SSS_OK;
}

int sss_execute_dot(sss_plan p, const int32_t *row_ptr, const int32_t *col, const double *val, const double *x,
                    double *y, void *stream, const double **dots, int *n_dots) {
  *n_dots = 0;
  if (!p || p->batch) return SSS_ERR_INVALID_VALUE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const Form form = form_of(p->m, p->n, p->nnz, p->dt, p->n);
  const int64_t blocks = (p->n_slots + p->B - 1) / p->B;
  // (in column order, the bunches of a workgroup, and so the bits of its sum,
  // depend on the atomics that made the order: another plan of the same matrix
  // would not repeat them)
  if (!p->bind_rows || p->dt != SSS_F64 || p->m != p->n || p->carries || p->debug || p->ordered || form == kWide ||
      blocks > kMaxDots)
    return launch(p, row_ptr, col, val, x, y, s);
  const int rc = check_call(p, row_ptr, col, val, x, y);
  if (rc != SSS_OK) return rc;
  const DotFn k = p->W == 4 ? pick_dot<4>(form) : (p->W == 8 ? pick_dot<8>(form) : pick_dot<16>(form));
  const size_t lds = (size_t)p->B * stage1_lds_words(p->W, p->S) * sizeof(uint32_t);
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(p->B * kWave), lds, s, plan_ctx(p, row_ptr, col, val, x, y),
                     p->dots);
  SSS_HIP(hipGetLastError());
  *dots = p->dots;
  *n_dots = (int)blocks;
  return SSS_OK;
}

int sss_csr_spmv_execute(sss_plan p, const int32_t *row_ptr, const int32_t *col, const void *val, const void *x,
                         void *y, void *stream) {
  if (!p || p->batch) return SSS_ERR_INVALID_VALUE;
  return launch(p, row_ptr, col, val, x, y, static_cast<hipStream_t>(stream));
}

int sss_csr_spmv_stage1(sss_plan p, const int32_t *row_ptr, const int32_t *col, const void *val, const void *x,
                        void *y, void *stream) {
  if (!p || p->batch) return SSS_ERR_INVALID_VALUE;
  const int rc = check_call(p, row_ptr, col, val, x, y);
  if (rc != SSS_OK || p->m == 0) return rc;
  return launch_stage1(p, row_ptr, col, val, x, y, true, static_cast<hipStream_t>(stream));
}

int sss_floor_probe(sss_plan p, const int32_t *col, const void *val, const void *x, void *out, int gather,
                    void *stream) {
  if (!p || p->batch) return SSS_ERR_INVALID_VALUE;
  if (p->m == 0 || p->nnz == 0) return SSS_OK;
  if (!col || !val || !out || (gather && !x)) return SSS_ERR_INVALID_VALUE;
  if (misaligned(col) || misaligned(val)) return SSS_ERR_INVALID_VALUE;
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev != p->device) return SSS_ERR_PLAN_MISMATCH;
  MatCtx a{};
  a.col = col; a.val = val; a.x = x;
  a.m = (int32_t)p->m; a.nnz = (int32_t)p->nnz; a.S = p->S; a.W = p->W;
  a.n_bunches = p->n_bunches; a.n_tiles = p->n_tiles;
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (p->dt) {
    case SSS_F64: return launch_floor_w<SSS_F64>(p, a, out, gather, s);
    case SSS_F32: return launch_floor_w<SSS_F32>(p, a, out, gather, s);
    case SSS_BF16: return launch_floor_w<SSS_BF16>(p, a, out, gather, s);
    default: return SSS_ERR_UNSUPPORTED;
  }
}

int sss_csr_spmv_stage2(sss_plan p, const int32_t *row_ptr, void *y, void *stream) {
  if (!p || p->batch) return SSS_ERR_INVALID_VALUE;
  if (p->m == 0) return SSS_OK;
  if (!row_ptr || !y) return SSS_ERR_INVALID_VALUE;
  if (p->bind_rows && row_ptr != p->bound_row_ptr) return SSS_ERR_PLAN_MISMATCH;
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev != p->device) return SSS_ERR_PLAN_MISMATCH;
  return launch_stage2(p, row_ptr, y, static_cast<hipStream_t>(stream));
}

int sss_csr_spmv(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col, const double *val,
                 const double *x, double *y, void *stream) {
  if (m < 0 || n < 0 || nnz < 0) return SSS_ERR_INVALID_VALUE;
  if (m == 0) return SSS_OK;
  int dev = 0;
  SSS_HIP(hipGetDevice(&dev));
  sss_plan p = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto key = std::make_tuple(dev, stream, m, n, nnz);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
      p = it->second;
    } else {
      sss_plan_opts o{};
      o.mode = SSS_MODE_FIXED;
      one_call_params(nnz, &o.W, &o.S);
      const int rc = sss_csr_spmv_plan_create(m, n, nnz, row_ptr, SSS_F64, &o, stream, &p);
      if (rc != SSS_OK) return rc;
      g_cache[key] = p;
    }
  }
  return launch(p, row_ptr, col, val, x, y, static_cast<hipStream_t>(stream));
}

int sss_csr_spmv_noalloc(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col,
                         const double *val, const double *x, double *y, void *stream) {
  if (m < 0 || n < 0 || nnz < 0 || m > SSS_MAX_INDEX || n > SSS_MAX_INDEX || nnz > SSS_MAX_INDEX)
    return SSS_ERR_INVALID_VALUE;
  if (m == 0) return SSS_OK;
  int W = 0, S = 0;
  one_call_params(nnz, &W, &S);
  // column order where the scratch holds its lists too
  bool order = orders_calls(nnz, n, SSS_F64);
  AuxLayout L = aux_layout(nnz, W, S, false, false, order);
  if (order && L.total > kScratchBytes) {
    order = false;
    L = aux_layout(nnz, W, S, false, false, order);
  }
  if (L.total > kScratchBytes) return SSS_ERR_TOO_LARGE;
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return SSS_ERR_UNSUPPORTED;
  void *base = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
      void *ptr = nullptr;
      SSS_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
      g_scratch_ptr[dev] = ptr;
    }
    base = g_scratch_ptr[dev];
  }
  sss_plan_s p;
  p.device = dev;
  p.m = m; p.n = n; p.nnz = nnz; p.dt = SSS_F64;
  p.W = W; p.S = S; p.B = kDefaultB; p.call_order = order;
  plan_bind_aux(&p, L, base);
  return launch(&p, row_ptr, col, val, x, y, static_cast<hipStream_t>(stream));
}

int sss_csr_spmv_cache_clear(void) {
  std::lock_guard<std::mutex> lk(g_cache_mu);
  if (g_cache.empty()) return SSS_OK;
  int rc = SSS_OK, cur = -1;
  const hipError_t eg = hipGetDevice(&cur);
  for (auto &kv : g_cache) {
    // each plan is destroyed with its own device current
    hipError_t e = hipSetDevice(kv.second->device);
    int r = e == hipSuccess ? sss_plan_destroy(kv.second) : SSS_ERR_HIP;
    if (e != hipSuccess) g_last_hip = e;
    if (rc == SSS_OK) rc = r;
  }
  g_cache.clear();
  if (eg == hipSuccess && cur >= 0) (void)hipSetDevice(cur);
  return rc;
}

int sss_csr_spmv_stage2_host(sss_plan p, const int32_t *row_ptr, void *y) {
  if (!p || p->batch) return SSS_ERR_INVALID_VALUE;
  if (p->m == 0 || p->nnz == 0) return SSS_OK;
  if (!row_ptr || !y) return SSS_ERR_INVALID_VALUE;
  const size_t nb = (size_t)p->n_bunches;
  std::vector<BunchState> st(nb);
  std::vector<int4> spec(nb * (size_t)p->S);
  SSS_HIP(hipDeviceSynchronize());
  SSS_HIP(hipMemcpy(st.data(), p->state, nb * sizeof(BunchState), hipMemcpyDeviceToHost));
  SSS_HIP(hipMemcpy(spec.data(), p->speculator, spec.size() * sizeof(int4), hipMemcpyDeviceToHost));
  if (p->dt == SSS_F64)
    stage2_host(p, row_ptr, static_cast<double *>(y), st.data(), spec.data());
  else
    stage2_host(p, row_ptr, static_cast<float *>(y), st.data(), spec.data());
  return SSS_OK;
}

int sss_plan_destroy(sss_plan p) {
  if (!p) return SSS_OK;
  int rc = SSS_OK;
  // hipFree waits for the device's outstanding work before it frees (so a
  // replay of the plan's graph has ended before the graph goes); a
  // caller-provided workspace stays with the caller
  // every resource is released even when an earlier release fails; the
  // first failure is the one reported
  hipError_t first = hipSuccess;
  auto release = [&first](hipError_t e) { if (first == hipSuccess) first = e; };
  if (p->owns_aux && p->aux) release(hipFree(p->aux));
  if (p->graph_exec) release(hipGraphExecDestroy(p->graph_exec));
  if (p->graph) release(hipGraphDestroy(p->graph));
  if (p->capture_stream) release(hipStreamDestroy(p->capture_stream));
  if (first != hipSuccess) { g_last_hip = first; rc = SSS_ERR_HIP; }
  delete p;
  return rc;
}

int sss_batch_plan_create(int count, const sss_csr_desc *mats, sss_dtype dt, const sss_plan_opts *opts,
                          void *stream, sss_plan *out) {
  if (!out || count < 0 || (count > 0 && !mats)) return SSS_ERR_INVALID_VALUE;
  *out = nullptr;
  if (!dtype_ok(dt)) return SSS_ERR_UNSUPPORTED;
  sss_plan_opts o{};
  o.mode = SSS_MODE_FIXED;
  if (opts) o = *opts;
  if (o.mode != SSS_MODE_FIXED && o.mode != SSS_MODE_SELECTOR) return SSS_ERR_UNSUPPORTED;
  int W = o.W ? o.W : default_W(dt);
  const int S = o.S ? o.S : default_S(dt);
  const int B = o.B ? o.B : kDefaultB;
  if (!(W == 4 || W == 8 || W == 16)) return SSS_ERR_UNSUPPORTED;
  if (S < 1 || S > kMaxS || B < 1 || B > kMaxB || o.debug) return SSS_ERR_INVALID_VALUE;
  // SELECTOR mode: every matrix's S from its class scores, W shared
  std::vector<int> sel_S;
  if (o.mode == SSS_MODE_SELECTOR && count > 0 && sss_selector_loaded()) {
    for (int i = 0; i < count; ++i)
      if (mats[i].m < 0 || mats[i].n < 0 || mats[i].nnz < 0 || mats[i].m > SSS_MAX_INDEX ||
          mats[i].n > SSS_MAX_INDEX || mats[i].nnz > SSS_MAX_INDEX || (mats[i].m > 0 && !mats[i].row_ptr))
        return SSS_ERR_INVALID_VALUE;
    std::vector<float> scores((size_t)count * SSS_N_CLASSES, 0.f);
    double w_votes[17] = {};
    // a matrix is scored with its own row-structure features but the size
    // features of the whole launch: the batch's bunches share one grid, so
    // how well a tile schedule fills the device depends on the total work,
    // not on the one matrix
    double tot_m = 0, tot_n = 0, tot_nnz = 0;
    for (int i = 0; i < count; ++i) { tot_m += (double)mats[i].m; tot_n += (double)mats[i].n; tot_nnz += (double)mats[i].nnz; }
    for (int i = 0; i < count; ++i) {
      const sss_csr_desc &d = mats[i];
      if (d.m == 0 || d.nnz == 0) continue;
      float f[SSS_N_FEATURES];
      int rc = sss_csr_features(d.m, d.n, d.nnz, d.row_ptr, dt, stream, f);
      f[0] = (float)std::log2(tot_m + 1.0);
      f[1] = (float)std::log2(tot_n + 1.0);
      f[2] = (float)std::log2(tot_nnz + 1.0);
      if (rc == SSS_OK) rc = sss_selector_scores(f, &scores[(size_t)i * SSS_N_CLASSES]);
      if (rc != SSS_OK) return rc;
      const float *z = &scores[(size_t)i * SSS_N_CLASSES];
      const int best = (int)(std::max_element(z, z + SSS_N_CLASSES) - z);
      int Wc = 0, Sc = 0;
      (void)sss_class_params(best, &Wc, &Sc);
      w_votes[Wc] += (double)d.nnz;
    }
    if (!o.W) W = w_votes[4] > w_votes[8] && w_votes[4] > w_votes[16] ? 4 : (w_votes[16] > w_votes[8] ? 16 : 8);
    sel_S.assign((size_t)count, S);
    for (int i = 0; i < count; ++i) {
      if (mats[i].m == 0 || mats[i].nnz == 0) continue;
      const float *z = &scores[(size_t)i * SSS_N_CLASSES];
      float best = -INFINITY;
      for (int c = 0; c < SSS_N_CLASSES; ++c) {
        int Wc = 0, Sc = 0;
        (void)sss_class_params(c, &Wc, &Sc);
        if (Wc == W && z[c] > best) { best = z[c]; sel_S[(size_t)i] = Sc; }
      }
    }
  }
  const int WT = W * kWave;
  std::vector<MatCtx> ctx((size_t)count);
  std::vector<int64_t> bb((size_t)count + 1, 0), cb((size_t)count + 1, 0);
  int s_max = 1;
  int64_t n_max = 0;
  bool any_zero = false;  // a matrix with rows and no nonzero
  int64_t tot_m = 0, tot_n = 0, tot_nnz = 0, tot_tiles = 0;
  for (int i = 0; i < count; ++i) {
    const sss_csr_desc &d = mats[i];
    if (d.m < 0 || d.n < 0 || d.nnz < 0 || d.m > SSS_MAX_INDEX || d.n > SSS_MAX_INDEX || d.nnz > SSS_MAX_INDEX)
      return SSS_ERR_INVALID_VALUE;
    if (d.m > 0 && (!d.row_ptr || !d.y)) return SSS_ERR_INVALID_VALUE;
    if (d.nnz > 0 && (!d.col || !d.val || !d.x || misaligned(d.col) || misaligned(d.val))) return SSS_ERR_INVALID_VALUE;
    const int Si = !sel_S.empty() ? sel_S[(size_t)i] : (d.S ? d.S : S);
    if (Si < 1 || Si > kMaxS) return SSS_ERR_INVALID_VALUE;
    s_max = std::max(s_max, Si);
    const int64_t nb = (d.m > 0 && d.nnz > 0) ? (d.nnz + (int64_t)Si * WT - 1) / ((int64_t)Si * WT) : 0;
    MatCtx &c = ctx[(size_t)i];
    c.row_ptr = d.row_ptr; c.col = d.col; c.val = d.val; c.x = d.x; c.y = d.y;
    c.m = (int32_t)d.m; c.nnz = (int32_t)d.nnz; c.S = Si; c.W = W; c.n_bunches = nb;
    c.n_tiles = d.nnz > 0 ? (d.nnz + WT - 1) / WT : 0;
    c.dbg_start = nullptr; c.dbg_dirty = nullptr; c.dbg_heads = nullptr;
    bb[(size_t)i + 1] = bb[(size_t)i] + nb;
    cb[(size_t)i + 1] = cb[(size_t)i] + (nb + kWave - 1) / kWave;
    n_max = std::max(n_max, d.n);
    any_zero = any_zero || (d.m > 0 && nb == 0);
    tot_m += d.m; tot_n += d.n; tot_nnz += d.nnz; tot_tiles += c.n_tiles;
  }
  const int64_t nb_all = bb[(size_t)count];
  // one wavefront per bunch in one grid: more bunches than this is beyond
  // any batch that fits in memory
  if (nb_all > INT32_MAX) return SSS_ERR_INVALID_VALUE;
  size_t off = 0;
  const size_t o_mats = off; off = align256(off + sizeof(MatCtx) * (size_t)std::max(count, 1));
  const size_t o_bb = off; off = align256(off + sizeof(int64_t) * ((size_t)count + 1));
  const size_t o_cb = off; off = align256(off + sizeof(int64_t) * ((size_t)count + 1));
  const size_t o_bs = off; off = align256(off + sizeof(BunchState) * (size_t)(nb_all + 1));
  const size_t o_bi = off; off = align256(off + sizeof(int4) * (size_t)(nb_all + 1));
  const size_t o_ar = off; off = align256(off + sizeof(int32_t) * (size_t)(nb_all + 1));
  const size_t o_al = off; off = align256(off + sizeof(int32_t));

  sss_plan p = new sss_plan_s();
  p->batch = true; p->dt = dt; p->W = W; p->S = S; p->B = B; p->batch_persistent = o.batch_persistent != 0;
  p->batch_form = form_of(tot_m, tot_n, tot_nnz, dt, n_max);
  p->mat_S.resize((size_t)count);
  for (int i = 0; i < count; ++i) p->mat_S[(size_t)i] = ctx[(size_t)i].S;
  p->m = tot_m; p->n = tot_n; p->nnz = tot_nnz; p->n_tiles = tot_tiles; p->n_bunches = nb_all;
  auto fail = [&](hipError_t e) {
    g_last_hip = e;
    if (p->aux) (void)hipFree(p->aux);
    delete p;
    return SSS_ERR_HIP;
  };
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) return fail(e);
  e = hipMalloc(&p->aux, off);
  if (e != hipSuccess) { p->aux = nullptr; return fail(e); }
  p->owns_aux = true;
  e = hipMemsetAsync(p->aux, 0, off, s);
  if (e != hipSuccess) return fail(e);
  char *base = static_cast<char *>(p->aux);
  for (int i = 0; i < count; ++i) {
    MatCtx &c = ctx[(size_t)i];
    c.state = reinterpret_cast<BunchState *>(base + o_bs) + bb[(size_t)i];
    c.arrivals = reinterpret_cast<int32_t *>(base + o_ar) + bb[(size_t)i];
  }
  // host arrays stay alive until the stream synchronisation below
  if (count > 0)
    e = hipMemcpyAsync(base + o_mats, ctx.data(), sizeof(MatCtx) * (size_t)count, hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(base + o_bb, bb.data(), sizeof(int64_t) * ((size_t)count + 1), hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(base + o_cb, cb.data(), sizeof(int64_t) * ((size_t)count + 1), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return fail(e);
  BatchArgs &ba = p->bargs;
  ba.mats = reinterpret_cast<const MatCtx *>(base + o_mats);
  ba.bunch_base = reinterpret_cast<const int64_t *>(base + o_bb);
  ba.chunk_base = reinterpret_cast<const int64_t *>(base + o_cb);
  ba.count = count;
  ba.S_max = s_max;
  ba.total_bunches = nb_all;
  // every global bunch's matrix, first row and index within the matrix, once
  // for all calls (the descriptors, and so the row pointers, are bound to the plan)
  int4 *binfo = reinterpret_cast<int4 *>(base + o_bi);
  ba.bunch_info = binfo;
  if (nb_all > 0) {
    const unsigned blocks = (unsigned)std::min<int64_t>((nb_all + 255) / 256, 65535);
    hipLaunchKernelGGL(sss_batch_bunch_info, dim3(blocks), dim3(256), 0, s, ba.mats, ba.bunch_base, count, nb_all,
                       binfo, reinterpret_cast<int32_t *>(base + o_al));
    e = hipGetLastError();
    if (e != hipSuccess) return fail(e);
  }
  e = hipMemcpyAsync(&ba.carries, base + o_al, sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return fail(e);
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(e);
  ba.total_chunks = ba.carries ? cb[(size_t)count] : 0;
  ba.total_waves = ba.total_chunks + (any_zero ? count : 0);
  // the carries' persistent grid: as many workgroups as stay resident on the device
  int cus = 0;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device);
  if (e != hipSuccess) return fail(e);
  int per_cu2 = 0;
  const void *k2 = dt == SSS_F64 ? reinterpret_cast<const void *>(sss_carries_batch<double>)
                                 : reinterpret_cast<const void *>(sss_carries_batch<float>);
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu2, k2, kCarryThreads, 0);
  if (e != hipSuccess) return fail(e);
  // stage 1: B bunches per workgroup, the count rounded up to a multiple of
  // kXcds so that every XCD gets an equal contiguous run (the extra
  // wavefronts find no bunch and exit); persistent: as many workgroups as
  // stay resident, a multiple of kXcds
  int64_t wgs1 = std::max<int64_t>(1, (nb_all + B - 1) / B);
  if (p->batch_persistent) {
    int per_cu1 = 0;
    const size_t lds1 = (size_t)B * stage1_lds_words(W, s_max) * sizeof(uint32_t);
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu1, reinterpret_cast<const void *>(SSS_PICK(pick_batch, dt, W, p->batch_form, true)), B * kWave, lds1);
    if (e != hipSuccess) return fail(e);
    wgs1 = std::min<int64_t>(wgs1, (int64_t)cus * std::max(per_cu1, 1));
    if (wgs1 > kXcds) wgs1 -= wgs1 % kXcds;
  }
  // the XCD windows: one per XCD when the grid has more than kXcds
  // workgroups, each a contiguous run of global bunches that holds an equal
  // share of the nonzeros (a bunch holds S W 64 of its matrix's, the last
  // one of a matrix fewer), so that matrices with a larger S do not load
  // their XCD more; else a single window
  ba.n_windows = wgs1 > kXcds ? kXcds : 1;
  for (int k = 0; k <= kXcds; ++k) ba.window[k] = nb_all;
  ba.window[0] = 0;
  if (ba.n_windows == kXcds) {
    int k = 1;
    int64_t before = 0;  // nonzeros of the matrices before matrix i
    for (int i = 0; i < count && k < kXcds; ++i) {
      const MatCtx &c = ctx[(size_t)i];
      const int64_t swt = (int64_t)c.S * WT;
      while (k < kXcds && c.n_bunches > 0 && before + c.nnz >= tot_nnz * k / kXcds) {
        const int64_t j = std::min<int64_t>(c.n_bunches, (tot_nnz * k / kXcds - before + swt / 2) / swt);
        ba.window[k] = std::max(ba.window[k - 1], bb[(size_t)i] + j);
        ++k;
      }
      before += c.nnz;
    }
    int64_t per = 0;  // workgroups per XCD: enough for its largest window
    for (int w = 0; w < kXcds; ++w) per = std::max(per, (ba.window[w + 1] - ba.window[w] + B - 1) / B);
    if (!p->batch_persistent) wgs1 = kXcds * std::max<int64_t>(per, 1);
  }
  if (wgs1 > INT32_MAX) {  // more bunches than a grid holds: beyond any batch that fits in memory
    (void)hipFree(p->aux);
    delete p;
    return SSS_ERR_INVALID_VALUE;
  }
  p->blocks1 = (int)wgs1;
  const int64_t wpb2 = kCarryThreads / kWave;
  p->blocks2 = (int)std::max<int64_t>(
      1, std::min<int64_t>((ba.total_waves + wpb2 - 1) / wpb2, (int64_t)cus * std::max(per_cu2, 1)));
  *out = p;
  return SSS_OK;
}

int sss_batch_execute(sss_plan p, void *stream) {
  if (!p || !p->batch) return SSS_ERR_INVALID_VALUE;
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev != p->device) return SSS_ERR_PLAN_MISMATCH;
  return launch_batch(p, static_cast<hipStream_t>(stream));
}

int sss_batch_graph_launch(sss_plan p, void *stream) {
  if (!p || !p->batch) return SSS_ERR_INVALID_VALUE;
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev != p->device) return SSS_ERR_PLAN_MISMATCH;
  if (!p->graph_exec) {
    if (!p->capture_stream) SSS_HIP(hipStreamCreateWithFlags(&p->capture_stream, hipStreamNonBlocking));
    SSS_HIP(hipStreamBeginCapture(p->capture_stream, hipStreamCaptureModeThreadLocal));
    const int rc = launch_batch(p, p->capture_stream);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(p->capture_stream, &g);
    if (rc != SSS_OK) {
      if (g) (void)hipGraphDestroy(g);
      return rc;
    }
    if (e != hipSuccess) { g_last_hip = e; return SSS_ERR_HIP; }
    const hipError_t ei = hipGraphInstantiate(&p->graph_exec, g, nullptr, nullptr, 0);
    if (ei != hipSuccess) {
      // nothing is kept: the next call captures again
      (void)hipGraphDestroy(g);
      p->graph_exec = nullptr;
      g_last_hip = ei;
      return SSS_ERR_HIP;
    }
    p->graph = g;
  }
  SSS_HIP(hipGraphLaunch(p->graph_exec, static_cast<hipStream_t>(stream)));
  return SSS_OK;
}

int sss_batch_floor_probe(sss_plan p, void *out, int gather, void *stream) {
  if (!p || !p->batch) return SSS_ERR_INVALID_VALUE;
  if (p->batch_persistent) return SSS_ERR_UNSUPPORTED;  // the probe mirrors the default launch
  if (p->bargs.total_bunches == 0) return SSS_OK;
  if (!out) return SSS_ERR_INVALID_VALUE;
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev != p->device) return SSS_ERR_PLAN_MISMATCH;
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (p->dt) {
    case SSS_F64: return launch_floor_batch_w<SSS_F64>(p, out, gather, s);
    case SSS_F32: return launch_floor_batch_w<SSS_F32>(p, out, gather, s);
    case SSS_BF16: return launch_floor_batch_w<SSS_BF16>(p, out, gather, s);
    default: return SSS_ERR_UNSUPPORTED;
  }
}

int sss_batch_plan_schedule(sss_plan p, int count, int *W, int *S) {
  if (!p || !p->batch || count != (int)p->mat_S.size()) return SSS_ERR_INVALID_VALUE;
  if (W) *W = p->W;
  if (S) std::copy(p->mat_S.begin(), p->mat_S.end(), S);
  return SSS_OK;
}

int sss_plan_info(sss_plan p, int *W, int *S, int *B, int64_t *n_tiles, int64_t *n_bunches) {
  if (!p) return SSS_ERR_INVALID_VALUE;
  if (W) *W = p->W;
  if (S) *S = p->S;
  if (B) *B = p->B;
  if (n_tiles) *n_tiles = p->n_tiles;
  if (n_bunches) *n_bunches = p->n_bunches;
  return SSS_OK;
}

int sss_plan_shape(sss_plan p, int64_t *m, int64_t *n, int64_t *nnz, sss_dtype *dt) {
  if (!p || p->batch) return SSS_ERR_INVALID_VALUE;
  if (m) *m = p->m;
  if (n) *n = p->n;
  if (nnz) *nnz = p->nnz;
  if (dt) *dt = static_cast<sss_dtype>(p->dt);
  return SSS_OK;
}

int sss_validate_csr(int64_t m, int64_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col, void *stream) {
  if (m < 0 || n < 0 || nnz < 0) return SSS_ERR_INVALID_VALUE;
  if (!row_ptr || (nnz > 0 && !col)) return SSS_ERR_INVALID_VALUE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  int dev = -1;
  SSS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return SSS_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lk(g_validate_mu);
  if (!g_validate_ptr[dev]) {
    void *ptr = nullptr;
    SSS_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(validate_flag)));
    g_validate_ptr[dev] = static_cast<int *>(ptr);
  }
  int *d_bad = g_validate_ptr[dev];
  int rc = SSS_OK;
  hipError_t e = hipMemsetAsync(d_bad, 0, sizeof(int), s);
  if (e == hipSuccess) {
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((std::max(m, nnz) + 255) / 256, 4096));
    hipLaunchKernelGGL(sss_validate_kernel, dim3(blocks), dim3(256), 0, s, row_ptr, col, m, n, nnz, d_bad);
    e = hipGetLastError();
  }
  int bad = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&bad, d_bad, sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) { g_last_hip = e; rc = SSS_ERR_HIP; }
  if (rc == SSS_OK && bad) rc = SSS_ERR_INVALID_CSR;
  return rc;
}

int sss_plan_debug_size(sss_plan p, size_t *bytes) {
  if (!p || !bytes) return SSS_ERR_INVALID_VALUE;
  const size_t wpt = (size_t)p->W * kWave / 32;
  *bytes = 4 * sizeof(int64_t) + (size_t)p->n_tiles * (2 * sizeof(int32_t) + wpt * sizeof(uint32_t)) +
           (size_t)p->n_tiles * 4 * sizeof(int32_t) + (size_t)p->n_bunches * (sizeof(int32_t) + 2 * sizeof(double));
  return SSS_OK;
}

int sss_plan_debug_dump(sss_plan p, void *host_buf, size_t bytes) {
  if (p && p->batch) return SSS_ERR_INVALID_VALUE;
  size_t need = 0;
  int rc = sss_plan_debug_size(p, &need);
  if (rc != SSS_OK) return rc;
  if (!host_buf || bytes < need) return SSS_ERR_INVALID_VALUE;
  SSS_HIP(hipDeviceSynchronize());
  std::memset(host_buf, 0, need);
  const int64_t nt = p->n_tiles, nb = p->n_bunches;
  const int64_t wpt = (int64_t)p->W * kWave / 32;
  // the per-bunch speculator segments, packed into one list in bunch order
  std::vector<BunchState> st((size_t)nb);
  std::vector<int4> spec((size_t)(nb * p->S));
  if (nb > 0) {
    SSS_HIP(hipMemcpy(st.data(), p->state, nb * sizeof(BunchState), hipMemcpyDeviceToHost));
    SSS_HIP(hipMemcpy(spec.data(), p->speculator, nb * p->S * sizeof(int4), hipMemcpyDeviceToHost));
  }
  std::vector<int4> packed;
  for (int64_t b = 0; b < nb; ++b)
    for (int i = 0; i < __builtin_popcount(st[(size_t)b].dirty_mask); ++i) packed.push_back(spec[(size_t)(b * p->S + i)]);
  int64_t *hdr = static_cast<int64_t *>(host_buf);
  hdr[0] = nt; hdr[1] = nb; hdr[2] = (int64_t)packed.size(); hdr[3] = wpt;
  char *cur = reinterpret_cast<char *>(hdr + 4);
  if (p->debug && nt > 0) {
    SSS_HIP(hipMemcpy(cur, p->dbg_start, nt * sizeof(int32_t), hipMemcpyDeviceToHost));
    SSS_HIP(hipMemcpy(cur + nt * sizeof(int32_t), p->dbg_dirty, nt * sizeof(int32_t), hipMemcpyDeviceToHost));
    SSS_HIP(hipMemcpy(cur + 2 * nt * sizeof(int32_t), p->dbg_heads, nt * wpt * sizeof(uint32_t),
                      hipMemcpyDeviceToHost));
  }
  cur += nt * (2 * sizeof(int32_t) + wpt * sizeof(uint32_t));
  if (!packed.empty()) std::memcpy(cur, packed.data(), packed.size() * sizeof(int4));
  cur += nt * 4 * sizeof(int32_t);
  for (int64_t b = 0; b < nb; ++b) {
    std::memcpy(cur + b * sizeof(int32_t), &st[(size_t)b].sync_idx, sizeof(int32_t));
    std::memcpy(cur + nb * sizeof(int32_t) + b * sizeof(double), &st[(size_t)b].sync_val, sizeof(double));
    std::memcpy(cur + nb * (sizeof(int32_t) + sizeof(double)) + b * sizeof(double), &st[(size_t)b].tail_val,
                sizeof(double));
  }
  return SSS_OK;
}

const char *sss_status_string(int status) {
  switch (status) {
    case SSS_OK: return "ok";
    case SSS_ERR_INVALID_VALUE: return "invalid value";
    case SSS_ERR_UNSUPPORTED: return "unsupported dtype or parameters";
    case SSS_ERR_PLAN_MISMATCH: return "plan does not match the call";
    case SSS_ERR_HIP: return "HIP runtime error";
    case SSS_ERR_INVALID_CSR: return "malformed CSR matrix";
    case SSS_ERR_TOO_LARGE: return "matrix too large for the static scratch of sss_csr_spmv_noalloc";
    default: return "unknown status";
  }
}

const char *sss_last_hip_error(void) { return hipGetErrorString(g_last_hip); }

const char *sss_version(void) { return "sss-spmv 0.1 gfx950"; }

}  // extern "C"
