// Grouped fp32 GEMMs on the CDNA4 matrix cores.
//
// Two kernel families cover every expert contraction of the training step:
//
//  * gemm_rows: C[r, :] = op(A)[r, :] x B_g for the rows r of group g.
//    A is a slot buffer [M, K] (row r = one routed edge token, grouped by
//    expert), B_g the expert weight, stored [K, N] ("NN") or [N, K] ("NT").
//    The A loader may transform elements on their way into LDS (SiLU of
//    stored pre-activations, ...) and the epilogue functor decides what is
//    written (plain store, gate scaling, the SiLU'/SiLU'' products of the
//    double backward, per-row partial sums).
//
//  * gemm_wgrad: G_g[p, q] = sum_{r in group g} A[r, p] B[r, q], the weight
//    gradients, whose contraction runs over the tokens of an expert.  The
//    rows of each group are cut into chunks; a group's only chunk writes the
//    gradient itself, else each chunk writes a partial P x Q block and a second
//    kernel adds the chunks of a group in order, so the result does not depend
//    on scheduling.
//
// Work decomposition: a workgroup of 256 threads (4 waves as 2 x 2) owns a
// 128 x 128 output tile; each wave owns 64 x 64 = 2 x 2 MFMA blocks of
// 32 x 32.  Two ways to multiply, chosen per launch:
//
//  * Split products (v_mfma_f32_32x32x16_f16).  An fp32 operand value, scaled
//    by a power of two per row of A and per column of B, is the sum of two
//    fp16 numbers, x s = h + 2^-11 l, to 2^-23 of itself: h and l hold 11 significant bits each and l
//    its sign, 23 of the 24 bits (a quarter of all values lose the last one).  C = sum h h' +
//    2^-11 sum (h l' + l h') takes three 16-bit matrix products in place of one fp32 product at a
//    sixteenth of their rate; what is left out, 2^-22 l l', is up to 2^-22 of a product (root mean square
//    2^-24.6).  The two sums have accumulators of their own (the matrix unit truncates small addends when
//    it aligns them to a large accumulator, a bias that grows with the length of the contraction when both
//    share one).  Each product is thus good to about 2^-21 where fp32 is to 2^-24, and a sum of many is nearer to
//    the 64-bit result than on the fp32 instructions, because there are fewer and smaller roundings as it adds up:
//    relative error (2-norm) at K = 128 / 512 / 2048: 1.1 / 1.7 / 3.0e-7, fp32 instructions 2.0 / 4.1 / 8.1e-7.
//    The scale comes from the largest magnitude of the row's (column's) first 32 k and bounds the range:
//    row products take values from 2^-21 to 2^7 times that magnitude with all these bits, weight gradients from
//    2^-13 to 2^15 (scale_field).  A larger value (or one after 32 zeros) overflows to infinity, and the
//    tile is taken again on the fp32 instructions, as is any tile with infinities or NaN.  A smaller
//    value loses bits; where that can matter (LowCount) the tile is taken again as well.
//    Two workgroups per CU (about 250 registers); a stage's registers are loaded a whole
//    stage before they are converted, and the conversion runs in eight parts between the matrix
//    instructions, so that vector and matrix units work at once.  Left for the end of a stage, on
//    loads issued at its beginning, the conversion made the stage a serial chain: K = 512, N = 2048
//    208 TFLOP/s (NN) and 242 (NT), weight gradient 178, against 266, 281 and 248.
//    Measured against the fp32 instructions, 500 000 rows over 64 groups: K = 512,
//    N = 2048 126 -> 242 TFLOP/s (NN), 128 -> 258 (NT); K = 2048, N = 512 130 -> 292
//    and 130 -> 299; weight gradient 512 x 2048 115 -> 223; 340 000 rows over 8 groups,
//    128 x 512: 108 -> 171, 113 -> 167 and 107 -> 160 (0.87 GB in 260-278 us).
//    Three bf16 terms and six products, which need no
//    scale, reach 131-190 and 121-140 TFLOP/s (with the unspread conversion): the six products
//    bring the clock down to 1.7 GHz.
//
//  * fp32 instructions (v_mfma_f32_32x32x2_f32), for callers that keep their
//    results bit for bit and for tiles that the split cannot take.  K advances in
//    stages of 16 through double-buffered LDS; operands stored as they are used go from
//    global memory straight into LDS (global_load_lds_dwordx4), transformed ones through
//    registers.  Inside a stage the k index of MFMA step j for lane half hf is
//    8g + 4hf + j (g = 0, 1), so an operand stored k-contiguous is read from LDS with one
//    16-byte load per lane per 8 k, and an operand stored m-contiguous with 4-byte loads
//    whose 32-lane halves read consecutive words.
//
// Epilogue: the accumulators are staged through LDS, 64 rows at a time, and
// then visited row-major as float4, so every epilogue read and write of
// global memory is a coalesced 512-byte row segment; a thread issues the
// epilogue reads of four pieces before it uses any of them.
#pragma once

#include <type_traits>

#include "common.h"

namespace janus {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int GBM = 128;            // tile rows
constexpr int GBN = 128;            // tile cols
constexpr int GBK = 16;             // k per LDS stage
constexpr int LD_MK = GBK;          // row stride of an [m][k] LDS tile (floats; float4 columns swizzled)
constexpr int LD_KM = GBM + 8;      // row stride of a [k][m] LDS tile (floats)
constexpr int LD_C = GBN + 8;       // row stride of the staged output (floats)
constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int B_BUF = cmax(GBN * LD_MK, GBK * LD_KM);             // one B stage, [n][k] or [k][n]
constexpr int SMEM_MAIN = cmax(2 * GBM * LD_MK + 2 * B_BUF,       // gemm_rows
                               4 * GBK * LD_KM);                   // gemm_wgrad
constexpr int SMEM_EPI = 64 * LD_C;
constexpr int SMEM_FP32 = cmax(SMEM_MAIN, SMEM_EPI);
// One operand stage of the split products: two fp16 planes of 128 rows x 32 k, each plane
// four k-octets of [row][8 fp16].  The octets lie 64 bytes apart (mod 256), so that the 8-byte
// stores of 32 lanes (4 rows x 8 k-quads) touch 64 distinct banks.
constexpr int SBK = 32;                       // k per stage (row products: K is a multiple)
constexpr int SP_OCT = GBM * 16 + 64;         // bytes of one octet
constexpr int SP_PLANE = 4 * SP_OCT;
constexpr int SP_OPER = 2 * SP_PLANE;
constexpr int SP_STAGE = 2 * SP_OPER;
constexpr int SMEM_BODY = cmax(2 * SP_STAGE / 4, SMEM_FP32);   // floats
// + exponents, low counts and largest values of the rows and columns, flags
constexpr int SMEM_FLOATS = SMEM_BODY + 3 * (GBM + GBN) + 64;

// How a row product multiplies: fp32 instructions, split products, or split products on tiles of 64
// rows (a wave owns 32 x 64).
enum { kModeFp32 = 0, kModeSplit = 1, kModeHalfRows = 2 };

struct RowsTile {   // one 128-row tile of a group
  int group;
  int r0;           // first row (global)
  int r1;           // one past the last row of the group
  int pad;
};

// Where a row product finds its tiles: a table, or (tiles null) the row offsets of at most 64
// groups, from which every wave works out its tile: 0.3 us per workgroup in place of a launch.
struct RowsTable {
  const RowsTile* tiles;
  const int* n_tiles;
  const int* off;
  int groups;
  __device__ __forceinline__ bool find(int t, RowsTile& out) const {
    if (tiles) {
      if (t >= *n_tiles) return false;
      out = tiles[t];
      return true;
    }
    const int l = threadIdx.x & 63;
    const int a = off[l < groups ? l : groups], b = off[l < groups ? l + 1 : groups];
    const int c = (b - a + GBM - 1) / GBM;
    int inc = c;   // tiles of groups 0..l
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(inc, o, 64);
      if (l >= o) inc += v;
    }
    const unsigned long long m = __ballot(inc > t);
    if (!m) return false;
    const int g = __builtin_ctzll(m);
    out.group = g;
    out.r0 = __builtin_amdgcn_readlane(a, g) + (t - __builtin_amdgcn_readlane(inc - c, g)) * GBM;
    out.r1 = __builtin_amdgcn_readlane(b, g);
    out.pad = 0;
    return true;
  }
};

__device__ __forceinline__ float4 f4zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float2 ld2(const float* p) { return *reinterpret_cast<const float2*>(p); }
__device__ __forceinline__ void st4(float* p, float4 v) { *reinterpret_cast<float4*>(p) = v; }
typedef float f32x4v __attribute__((ext_vector_type(4)));
// Streaming accesses of the epilogues (each element is read or written once per launch).
__device__ __forceinline__ float4 ld4nt(const float* p) {
  const f32x4v v = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4nt(float* p, float4 v) {
  const f32x4v x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<f32x4v*>(p));
}

// XCD-aware block order.  Workgroups are handed to the 8 XCDs round-robin
// by linear id, and each XCD has its own L2.  Block b runs on XCD b % 8 as
// that XCD's (b / 8)-th block, so the ntile output tiles that share one row
// range (or one weight-gradient chunk) are given to consecutive blocks of
// one XCD: row range r = (slot / ntile) * 8 + xcd, tile = slot % ntile.
// The grid is rows8(nrange) * ntile blocks; ids past the last range exit.
__device__ __forceinline__ void xcd_map(int b, int ntile, int& range, int& tile) {
  const int xcd = b & 7, slot = b >> 3;
  tile = slot % ntile;
  range = (slot / ntile) * 8 + xcd;
}
inline unsigned xcd_grid(long long nrange, int ntile) { return (unsigned)(((nrange + 7) / 8) * 8 * ntile); }

// ---------------------------------------------------------------- loaders
// load(r, k) fetches what element (r, k..k+3) needs from global memory;
// apply(raw, k) turns it into the 4 operand values (only for valid rows).

struct LoadPlain {
  const float* p;
  long long ld;
  using Raw = float4;
  __device__ __forceinline__ Raw load(long long r, int k) const { return ld4(p + r * ld + k); }
  __device__ __forceinline__ float4 apply(const Raw& v, int) const { return v; }
  static constexpr bool kRowFactor = false;
  static constexpr bool kZeroToZero = true;   // apply2 of zeros is zero (SplitKM's rows past the end)
  __device__ __forceinline__ const float* base() const { return p; }
  __device__ __forceinline__ float2 apply2(float2 v, float, int) const { return v; }
};

struct LoadSilu {   // SiLU of stored pre-activations
  const float* p;
  long long ld;
  using Raw = float4;
  __device__ __forceinline__ const float* base() const { return p; }
  __device__ __forceinline__ Raw load(long long r, int k) const { return ld4(p + r * ld + k); }
  __device__ __forceinline__ float4 apply(const Raw& v, int) const {
    return make_float4(silu(v.x), silu(v.y), silu(v.z), silu(v.w));
  }
};

struct LoadSiluRowScale {   // s[r] * SiLU(p[r, k])
  const float* p;
  const float* s;
  long long ld;
  struct Raw {
    float4 v;
    float s;
  };
  __device__ __forceinline__ Raw load(long long r, int k) const { return Raw{ld4(p + r * ld + k), s[r]}; }
  __device__ __forceinline__ float4 apply(const Raw& x, int) const {
    return make_float4(x.s * silu(x.v.x), x.s * silu(x.v.y), x.s * silu(x.v.z), x.s * silu(x.v.w));
  }
  static constexpr bool kRowFactor = true;   // apply2's second argument: s[r]
  static constexpr bool kZeroToZero = true;
  __device__ __forceinline__ const float* base() const { return p; }
  __device__ __forceinline__ float2 apply2(float2 v, float f, int) const {
    return make_float2(f * silu(v.x), f * silu(v.y));
  }
};

struct LoadSiluD1Scaled {   // SiLU'(z[r, k]) * w[k]
  const float* z;
  const float* w;
  long long ld;
  using Raw = float4;
  __device__ __forceinline__ Raw load(long long r, int k) const { return ld4(z + r * ld + k); }
  __device__ __forceinline__ float4 apply(const Raw& v, int k) const {
    const float4 ww = ld4(w + k);
    return make_float4(silu_d1(v.x) * ww.x, silu_d1(v.y) * ww.y, silu_d1(v.z) * ww.z, silu_d1(v.w) * ww.w);
  }
  static constexpr bool kRowFactor = false;
  static constexpr bool kZeroToZero = false;   // SiLU'(0) = 1/2
  __device__ __forceinline__ const float* base() const { return z; }
  __device__ __forceinline__ float2 apply2(float2 v, float, int k) const {
    return make_float2(silu_d1(v.x) * w[k], silu_d1(v.y) * w[k + 1]);
  }
};

// ---------------------------------------------------------------- epilogues
// An epilogue works on output row r, columns c..c+3 (c % 4 == 0) in two
// steps so that all of a thread's global reads are in flight together:
// load(r, c) fetches what the piece needs, store(r, c, v, raw) writes the
// results and returns the piece's contribution to the row sum (kRowSum).

struct NoRaw {};

struct EpiStore {
  float* c;
  long long ld;
  static constexpr bool kRowSum = false;
  using Raw = NoRaw;
  __device__ __forceinline__ Raw load(long long, int) const { return Raw{}; }
  __device__ __forceinline__ float store(long long r, int col, float4 v, const Raw&) const {
    st4nt(c + r * ld + col, v);
    return 0.f;
  }
};

// Same store for the dense readout products (a distinct type keeps their
// kernels apart from the expert ones in profiles).
struct EpiDense : EpiStore {};

struct EpiRowScale {   // c = s[r] * v
  float* c;
  const float* s;
  long long ld;
  static constexpr bool kRowSum = false;
  using Raw = float;
  __device__ __forceinline__ Raw load(long long r, int) const { return s[r]; }
  __device__ __forceinline__ float store(long long r, int col, float4 v, const Raw& a) const {
    st4nt(c + r * ld + col, make_float4(a * v.x, a * v.y, a * v.z, a * v.w));
    return 0.f;
  }
};

// C = A B + R (residual R may be null): the attention output added to the atom features.
struct EpiAdd {
  float* c;
  const float* r;
  long long ld;
  static constexpr bool kRowSum = false;
  using Raw = float4;
  __device__ __forceinline__ Raw load(long long row, int col) const {
    return r ? ld4nt(r + row * ld + col) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __device__ __forceinline__ float store(long long row, int col, float4 v, const Raw& x) const {
    st4nt(c + row * ld + col, make_float4(v.x + x.x, v.y + x.y, v.z + x.z, v.w + x.w));
    return 0.f;
  }
};

// Force backward, after Sbar = Ybar W2^T: keep Sbar and Abar = SiLU'(A) Sbar.
struct EpiP2 {
  const float* A;
  float* Sb;
  float* Ab;
  long long ld;
  static constexpr bool kRowSum = false;
  using Raw = float4;
  __device__ __forceinline__ Raw load(long long r, int c) const { return ld4nt(A + r * ld + c); }
  __device__ __forceinline__ float store(long long r, int c, float4 v, const Raw& a) const {
    const long long i = r * ld + c;
    st4nt(Sb + i, v);
    st4nt(Ab + i, make_float4(silu_d1(a.x) * v.x, silu_d1(a.y) * v.y, silu_d1(a.z) * v.z, silu_d1(a.w) * v.w));
    return 0.f;
  }
};

struct Float4x2 {
  float4 a, b;
};

// Double backward, after Abt = Xbt W1:
//   Sbt = SiLU'(A) Abt        (overwrites Abar, which the weight gradient has consumed)
//   C   = SiLU''(A) Sbar Abt  (overwrites Sbar; consumed by the final backward)
struct EpiP3 {
  const float* A;
  float* Sb;
  float* Ab;
  long long ld;
  static constexpr bool kRowSum = false;
  using Raw = Float4x2;
  __device__ __forceinline__ static void d12(float a, float& d1, float& d2) {
    const float s = sig(a);
    d1 = s + a * s * (1.f - s);
    d2 = s * (1.f - s) * (2.f + a * (1.f - 2.f * s));
  }
  __device__ __forceinline__ Raw load(long long r, int c) const {
    const long long i = r * ld + c;
    return Raw{ld4nt(A + i), ld4nt(Sb + i)};
  }
  __device__ __forceinline__ float store(long long r, int c, float4 v, const Raw& x) const {
    const long long i = r * ld + c;
    const float4 a = x.a, sb = x.b;
    float4 o1, o2;
    float d1, d2;
    d12(a.x, d1, d2); o1.x = d1 * v.x; o2.x = d2 * sb.x * v.x;
    d12(a.y, d1, d2); o1.y = d1 * v.y; o2.y = d2 * sb.y * v.y;
    d12(a.z, d1, d2); o1.z = d1 * v.z; o2.z = d2 * sb.z * v.z;
    d12(a.w, d1, d2); o1.w = d1 * v.w; o2.w = d2 * sb.w * v.w;
    st4nt(Ab + i, o1);
    st4nt(Sb + i, o2);
    return 0.f;
  }
};

// Final backward, after St = mt W2^T (ungated adjoint of the message):
//   At = g SiLU'(A) St + C  (overwrites C); returns St . SiLU(A) for the gate adjoint.
// KeepS: also g SiLU(A) over A (its last use), the operand of dW2, whose weight gradient else
// evaluates SiLU and gate once per 128 output columns as it loads.
template <bool KeepS>
struct EpiP4 {
  std::conditional_t<KeepS, float, const float>* A;
  float* Sb;
  const float* gate;
  long long ld;
  static constexpr bool kRowSum = true;
  struct Raw {
    float4 a, c;
    float g;
  };
  __device__ __forceinline__ static float one(float a, float v, float c, float g, float& sum, float& gs) {
    const float s = sig(a);
    sum += v * a * s;
    gs = g * (a * s);
    return g * (s + a * s * (1.f - s)) * v + c;
  }
  __device__ __forceinline__ Raw load(long long r, int c) const {
    const long long i = r * ld + c;
    return Raw{ld4nt(A + i), ld4nt(Sb + i), gate[r]};
  }
  __device__ __forceinline__ float store(long long r, int c, float4 v, const Raw& x) const {
    float sum = 0.f;
    float4 o, gs;
    o.x = one(x.a.x, v.x, x.c.x, x.g, sum, gs.x);
    o.y = one(x.a.y, v.y, x.c.y, x.g, sum, gs.y);
    o.z = one(x.a.z, v.z, x.c.z, x.g, sum, gs.z);
    o.w = one(x.a.w, v.w, x.c.w, x.g, sum, gs.w);
    st4nt(Sb + r * ld + c, o);
    if constexpr (KeepS) st4nt(A + r * ld + c, gs);
    return sum;
  }
};

// ------------------------------------------------------------ LDS staging
// [m][k] tiles hold the 4 float4 columns of row m in the order
// kq ^ ((m / 4) % 4): a 16-lane group then touches 64 distinct banks both
// when it stores 4 rows x 4 columns and when it reads one column of 16 rows.
static_assert(GBK == 16, "the [m][k] swizzle assumes 4 float4 columns per row");
__device__ __forceinline__ int mk_off(int m, int kq) { return m * LD_MK + 4 * (kq ^ ((m >> 2) & 3)); }

// The loads are unconditional: rows (and columns) past the end of the range
// read the last valid one and are replaced by zeros when stored to LDS.  A
// conditional load would put a branch around every load, and at the join
// the compiler waits for all earlier loads, which serialises them.  Ranges
// are never empty (tiles and chunks are built only over rows that exist;
// widths are multiples of 4).

// [m][k] tile from a k-contiguous operand: thread q loads row q/4, k-quad q%4.
template <class L>
struct StageMK {
  typename L::Raw raw[2];
  bool ok[2];
  __device__ __forceinline__ void load(const L& ld, int r0, int r1, int k0, int tid) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = tid + 256 * i;
      const long long r = (long long)r0 + (q >> 2);
      ok[i] = r < r1;
      raw[i] = ld.load(ok[i] ? r : (long long)r1 - 1, k0 + 4 * (q & 3));
    }
  }
  __device__ __forceinline__ void store(const L& ld, float* s, int k0, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = tid + 256 * i;
      st4(s + mk_off(q >> 2, q & 3), ok[i] ? ld.apply(raw[i], k0 + 4 * (q & 3)) : f4zero());
    }
  }
};

// [k][m] tile from an m-contiguous operand: thread q loads k-row q/32, m-quad q%32.
template <class L>
struct StageKM {
  typename L::Raw raw[2];
  bool ok[2];
  __device__ __forceinline__ void load(const L& ld, long long rk, long long rk_end, int m0, int m_end, int tid) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = tid + 256 * i;
      const long long r = rk + (q >> 5);
      const int m = m0 + 4 * (q & 31);
      ok[i] = r < rk_end && m < m_end;
      raw[i] = ld.load(r < rk_end ? r : rk_end - 1, m < m_end ? m : m_end - 4);
    }
  }
  __device__ __forceinline__ void store(const L& ld, float* s, int m0, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = tid + 256 * i;
      st4(s + (q >> 5) * LD_KM + 4 * (q & 31), ok[i] ? ld.apply(raw[i], m0 + 4 * (q & 31)) : f4zero());
    }
  }
  // the same into the unpadded swizzled layout of direct_km
  __device__ __forceinline__ void store_sw(const L& ld, float* s, int m0, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = tid + 256 * i, k = q >> 5;
      st4(s + k * GBM + ((4 * (q & 31)) ^ (((k >> 2) & 1) << 5)),
          ok[i] ? ld.apply(raw[i], m0 + 4 * (q & 31)) : f4zero());
    }
  }
};

// Direct global-to-LDS loads of one [m][k] stage of a plain operand (128 rows x 16 k):
// lane l of wave w writes the 16 bytes at LDS float (i*256 + w*64 + l)*4, which is row
// m = i*64 + w*16 + l/4, column slot l%4 of the swizzled layout, so it loads k-quad
// (l%4) ^ ((m/4)%4) of row m.  Rows past r1 load row r1 - 1 (their products are never stored).
template <class L>
struct IsPlainLoad : std::false_type {};
template <>
struct IsPlainLoad<LoadPlain> : std::true_type {};
typedef __attribute__((address_space(3))) void* lds_ptr;
__device__ __forceinline__ void direct_mk(const float* __restrict__ p, long long ld, int r0, int r1, int k0,
                                          float* s, int tid) {
  const int l = tid & 63, w = tid >> 6;
  const int kq = (l & 3) ^ ((l >> 4) & 3);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const long long r = (long long)r0 + i * 64 + w * 16 + (l >> 2);
    const float* src = p + (r < r1 ? r : (long long)r1 - 1) * ld + k0 + 4 * kq;
    __builtin_amdgcn_global_load_lds(src, (lds_ptr)(s + (i * 256 + w * 64) * 4), 16, 0, 0);
  }
}
// Direct loads of one [k][m] stage (16 k-rows x 128 columns of an m-contiguous plain
// operand) into an unpadded layout whose rows k with (k / 4) odd hold their two 32-column
// halves of each 64 swapped (column c at c ^ 32): the two half-waves of an MFMA operand
// read, rows 4 apart, then fall on different banks.  Lane l of wave w writes LDS float
// (i*256 + w*64 + l)*4: row k = i*8 + w*2 + l/32, position 4 (l % 32).  Columns past
// m_end load column m_end - 4 (their products are never stored).
__device__ __forceinline__ void direct_km(const float* __restrict__ p, long long ld, long long rk, int m0, int m_end,
                                          float* s, int tid) {
  const int l = tid & 63, w = tid >> 6;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = i * 8 + w * 2 + (l >> 5);
    const int m = m0 + ((4 * (l & 31)) ^ (((k >> 2) & 1) << 5));
    const float* src = p + (rk + k) * ld + (m < m_end ? m : m_end - 4);
    __builtin_amdgcn_global_load_lds(src, (lds_ptr)(s + (i * 256 + w * 64) * 4), 16, 0, 0);
  }
}
__device__ __forceinline__ void wait_direct() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int BI>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[BI][2]) {
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
}

// One LDS stage of MFMAs.  AMK / BMK: operand tile stored [m][k] (else [k][m]).
template <bool AMK, bool BMK, bool SW = false>
__device__ __forceinline__ void mfma_stage(const float* a_s, const float* b_s, int wm, int wn, int lr, int hf,
                                           f32x16 (&acc)[2][2]) {
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    float af[2][4], bf[2][4];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) {
      const int m = wm * 64 + bi * 32 + lr;
      if (AMK) {
        const float4 v = ld4(a_s + mk_off(m, 2 * g + hf));
        af[bi][0] = v.x; af[bi][1] = v.y; af[bi][2] = v.z; af[bi][3] = v.w;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          af[bi][j] = SW ? a_s[(8 * g + 4 * hf + j) * GBM + (m ^ (hf << 5))] : a_s[(8 * g + 4 * hf + j) * LD_KM + m];
      }
    }
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const int n = wn * 64 + bj * 32 + lr;
      if (BMK) {
        const float4 v = ld4(b_s + mk_off(n, 2 * g + hf));
        bf[bj][0] = v.x; bf[bj][1] = v.y; bf[bj][2] = v.z; bf[bj][3] = v.w;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          bf[bj][j] = SW ? b_s[(8 * g + 4 * hf + j) * GBN + (n ^ (hf << 5))] : b_s[(8 * g + 4 * hf + j) * LD_KM + n];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
          acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[bi][j], bf[bj][j], acc[bi][bj], 0, 0, 0);
  }
}

// ---------------------------------------------------------- split products
// Split of a scaled value: x s = h + 2^-11 l with h, l in fp16, each rounded to nearest.  h holds 11
// significant bits; what is left has 12 and its sign, of which l holds 11.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// What LowCount adds up.  top: the largest |x|; low: sum of the low weights, in 2048ths.
__device__ __forceinline__ void count_pair(float a, float b, unsigned h, float& top, unsigned& low) {
  top = fmaxf(fmaxf(top, fabsf(a)), fabsf(b));
  // fp16 numbers up to 2^-13 (0x0800) are proportional to their bits
  const u16x2 u = __builtin_elementwise_min(__builtin_bit_cast(u16x2, h & 0x7fff7fffu), (u16x2){0x800, 0x800});
  low = __builtin_amdgcn_sad_u16(__builtin_bit_cast(unsigned, u), 0x08000800u, low);
}
template <bool Count>
__device__ __forceinline__ void split_pair(float a, float b, float s, unsigned& h, unsigned& l, float& top,
                                           unsigned& low) {
  a *= s;
  b *= s;
  const f16x2 hv = __builtin_convertvector((f32x2v){a, b}, f16x2);
  const float ra = 2048.f * (a - (float)hv.x), rb = 2048.f * (b - (float)hv.y);
  h = __builtin_bit_cast(unsigned, hv);
  l = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2v){ra, rb}, f16x2));
  if constexpr (Count) count_pair(a, b, h, top, low);
}
// h alone, counted.
__device__ __forceinline__ unsigned split_high(float a, float b, float s, float& top, unsigned& low) {
  a *= s;
  b *= s;
  const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2v){a, b}, f16x2));
  count_pair(a, b, h, top, low);
  return h;
}
// Power-of-two scale that brings a value of magnitude m to [2^target, 2^(target + 1)), as its exponent field.  The
// lower the target, the more growth fits (up to 2^(16 - target)) and the higher the floor below which bits are
// lost (2^-(36 + target) of m).
// Weight gradients, target 0: short bonds make some rows far larger than the first 32 of a chunk, and a tile
// that overflows costs a second, fp32 pass.  Step of 32 mixed structures with target 2^6 370 ms, 2^2 334, 1 325, 2^-3
// 323; small batch 14.1, 13.4, 13.4 and 13.3 ms.
// Row products contract over features, which differ less: fewer than one tile in 10^4 of the training steps
// measured below outgrows target 2^8, and it makes 2^16, the largest magnitude that fp16 holds, a bound of
// every value that is close enough for one comparison per tile (LowCount).  With target 1 the largest value of the
// tile has to be kept instead: product of 150 001 rows, K = 512, N = 2048 1359 us against 1272.
constexpr int kRowsTarget = 8;
__device__ __forceinline__ int scale_field(float m, int target) {
  const int f = 254 + target - (int)(__float_as_uint(m) >> 23);
  return f < 1 ? 1 : f > 254 ? 254 : f;
}

// Buffer loads of the staged operands: 32-bit offsets from the tile's (uniform) base, zero past `bytes`.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const float* p, long long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)bytes, 0x00027000);
}

// What the split may lose at the low end, and whether that matters.  A scaled value x is off by at most
// 2^-23 |x| + w(x) 2^-36, w = max(0, 1 - 2^13 |x|): half a unit of the smallest l.  The product l l' that
// is left out adds at most as much again.  With low(i) the sum of w over row i (column j) and top(i) its
// largest |x|, entry (i, j) is off by less than 2^-35 (low(i) top(j) + low(j) top(i)) beyond what full
// splits leave.  That is harmless up to 2^-21 sum |a b|, the size of eight roundings; a tile where it may
// be more is taken on the fp32 instructions.  Lower bounds of sum |a b| are sums of h h' of the magnitudes
// over some of the k, one after the other:
//  * the last one or two stages, whose planes are in LDS anyway.  Row products compare the tile's smallest
//    entry with low <= K and top <= 2^16.  In weight gradients magnitudes differ much more along the
//    contraction: they count low and top of every column as they convert, and compare entry by entry.
//  * four stages spread over K, weight gradients 16 also.
//  * all stages, entry by entry.
// In a step of 32 mixed structures at d = 512 the first clears 99.95 % of the row products' tiles (the rest have rows
// of zeros) and 52 % of the weight gradients', four stages 42 %, 16 stages 4.0 %, all 1.1 %; 0.1 % lose too much, and
// 0.3 % have overflowed.  In the small batch the first clears all and 93 %.  What it costs: that product
// 1294 -> 1321 us, weight gradient 330 011 x 128 x 512 262 -> 278 (half of it the counting), step of 32 mixed structures 330 -> 346 ms,
// small batch 13.2 -> 13.7.  Counting in row products as well: 1262 -> 1358 us.
struct LowCount {   // low and top of the tile's rows [0, 128) and columns [128, 256), in LDS
  unsigned* low;   // in 2048ths while they are added up; share() makes them floats, low / 2^14
  float* top;
  __device__ __forceinline__ explicit LowCount(float* smem)
      : low(reinterpret_cast<unsigned*>(smem + SMEM_BODY + GBM + GBN)), top(smem + SMEM_BODY + 2 * (GBM + GBN)) {}
  __device__ __forceinline__ void add(int p, unsigned l, float t) const {   // t >= 0: ordered like its bits
    atomicAdd(low + p, l);
    atomicMax(reinterpret_cast<unsigned*>(top + p), __float_as_uint(t));
  }
  // 2^-35 / 2^-21 of the counts; a row of zeros loses nothing
  __device__ __forceinline__ void share(int p) const {
    low[p] = __float_as_uint(top[p] > 0.f ? 1.f / 2048.f / 16384.f * (float)low[p] : 0.f);
  }
  __device__ __forceinline__ const float* shares() const { return reinterpret_cast<const float*>(low); }
};
// Whether every entry of m (this wave's sums of magnitudes) reaches its bound.
template <int BI>
__device__ __forceinline__ bool covered(const LowCount& c, int wm, int wn, int lr, int hf, const f32x16 (&m)[BI][2]) {
  float miss = 0.f, lc[2], tc[2];
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    const int p = GBM + wn * 64 + bj * 32 + lr;
    tc[bj] = c.top[p];
    lc[bj] = c.shares()[p];
  }
#pragma unroll
  for (int bi = 0; bi < BI; ++bi)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      const int p = wm * 32 * BI + bi * 32 + 8 * v4 + 4 * hf;
      const float4 l4 = ld4(c.shares() + p), t4 = ld4(c.top + p);
      const float l[4] = {l4.x, l4.y, l4.z, l4.w};
      const float t[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
          miss = fmaxf(miss, fmaf(l[v], tc[bj], fmaf(lc[bj], t[v], -m[bi][bj][4 * v4 + v])));
    }
  return !__any(miss > 0.f);
}
// The smallest entry of the wave's m, in lane 63.
template <int BI>
__device__ __forceinline__ float smallest(const f32x16 (&m)[BI][2]) {
  float x = m[0][0][0];
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) x = fminf(x, m[i][j][v]);
  auto step = [&](auto ctrl, auto rows) {
    const int y = __float_as_int(x);
    x = fminf(x, __int_as_float(__builtin_amdgcn_update_dpp(y, y, decltype(ctrl)::value, decltype(rows)::value, 0xf, false)));
  };
  using std::integral_constant;
  const integral_constant<int, 0xf> all;
  step(integral_constant<int, 0x111>(), all);   // row_shr 1, 2, 4, 8
  step(integral_constant<int, 0x112>(), all);
  step(integral_constant<int, 0x114>(), all);
  step(integral_constant<int, 0x118>(), all);
  step(integral_constant<int, 0x142>(), integral_constant<int, 0xa>());   // row_bcast 15, 31
  step(integral_constant<int, 0x143>(), integral_constant<int, 0xc>());
  return x;
}

// One operand's stage registers.  load() issues the global loads of stage k; values() gives the
// operand values of the stage loaded last; publish() and scales() choose the scales from the first stage's
// values (a barrier lies between them) and store the exponents that undo them, ex[position]; store()
// writes the planes.  With Count low and top of every column are counted on the way (LowCount).
// store_high() writes the plane of h alone and counts; publish_counts() adds the counts up.
//
// Operand stored k-contiguous: thread q takes k-quad q % 8 of rows q / 8 + 32 i, so that eight
// lanes read one row's 128 bytes.  Rows past the end read the last one (their products are never stored).
// R: loads per thread, 32 R rows.
template <class L, int R = 4>
struct SplitMK {
  static constexpr int kPieces = R;
  static constexpr bool kPaired = false;   // position of row m in the tile: m
  static constexpr bool kCount = false;
  using Values = float4[R];
  const L& ld;
  __amdgpu_buffer_rsrc_t rs;
  int vo[R];
  float4 raw[R];
  float s[R];
  __device__ __forceinline__ SplitMK(const L& l, int r0, int r1, int, int, int tid) : ld(l) {
    const int n = r1 - r0 < 32 * R ? r1 - r0 : 32 * R;
    rs = buffer_of(l.base() + (long long)r0 * l.ld, 4LL * n * l.ld);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int r = (tid >> 3) + 32 * i;
      vo[i] = 4 * ((r < n ? r : n - 1) * (int)l.ld + 4 * (tid & 7));
    }
  }
  __device__ __forceinline__ void load(int k) {
#pragma unroll
    for (int i = 0; i < R; ++i)
      raw[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo[i], 4 * k, 0));
  }
  __device__ __forceinline__ void values(int k, int tid, Values& x) const {
#pragma unroll
    for (int i = 0; i < R; ++i) x[i] = ld.apply(raw[i], k + 4 * (tid & 7));
  }
  __device__ __forceinline__ static void publish(const Values&, float*, int) {}
  __device__ __forceinline__ void scales(const Values& x, const float*, int* ex, int tid) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      float m = fmaxf(fmaxf(fabsf(x[i].x), fabsf(x[i].y)), fmaxf(fabsf(x[i].z), fabsf(x[i].w)));
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
      const int f = scale_field(m, kRowsTarget);
      s[i] = __uint_as_float((unsigned)f << 23);
      if ((tid & 7) == 0) ex[(tid >> 3) + 32 * i] = 127 - f;
    }
  }
  // a quarter of the stage: values, planes, and the loads of the stage that follows
  __device__ __forceinline__ void store(int i, float4 x, char* d, int tid) const {
    const int kq = tid & 7;
    d += (kq >> 1) * SP_OCT + ((tid >> 3) + 32 * i) * 16 + (kq & 1) * 8;
    unsigned h[2], l[2], low;
    float top;
    split_pair<false>(x.x, x.y, s[i], h[0], l[0], top, low);
    split_pair<false>(x.z, x.w, s[i], h[1], l[1], top, low);
    *reinterpret_cast<uint2*>(d) = make_uint2(h[0], h[1]);
    *reinterpret_cast<uint2*>(d + SP_PLANE) = make_uint2(l[0], l[1]);
  }
  __device__ __forceinline__ void piece(int i, int k, int next, char* d, int tid) {
    store(i, ld.apply(raw[i], k + 4 * (tid & 7)), d, tid);
    raw[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo[i], 4 * next, 0));
  }
  __device__ __forceinline__ void store_all(const Values& x, char* d, int tid) const {
#pragma unroll
    for (int i = 0; i < R; ++i) store(i, x[i], d, tid);
  }
  struct Counts {
    unsigned low[R] = {};
    float top[R] = {};
  };
  __device__ __forceinline__ void store_high(const Values& x, int, Counts& c, char* d, int tid) const {
    const int kq = tid & 7;
    d += (kq >> 1) * SP_OCT + (tid >> 3) * 16 + (kq & 1) * 8;
#pragma unroll
    for (int i = 0; i < R; ++i)
      *reinterpret_cast<uint2*>(d + 32 * 16 * i) = make_uint2(split_high(x[i].x, x[i].y, s[i], c.top[i], c.low[i]),
                                                              split_high(x[i].z, x[i].w, s[i], c.top[i], c.low[i]));
  }
  __device__ __forceinline__ static void publish_counts(const Counts& c, const LowCount& to, int p0, int tid) {
#pragma unroll
    for (int i = 0; i < R; ++i) to.add(p0 + (tid >> 3) + 32 * i, c.low[i], c.top[i]);
  }
};

// Operand stored row-contiguous ([k][m]): wave w takes the eight k-rows of octet w and lane q its
// columns 2 q and 2 q + 1, so that a load reads a whole 512-byte row of the tile.  Even columns of a
// 64-column half go to its first 32 positions, odd ones to the last (each lane's store is then next
// to its neighbour's).  k-rows past the end are zeros; columns past m_end read the last pair.
// Count: low and top of every column are kept.
template <class L, bool Count = false>
struct SplitKM {
  static constexpr bool kPaired = true;
  static constexpr bool kCount = Count;
  static constexpr int kPieces = 4;
  using Values = float2[8];
  const L& ld;
  __amdgpu_buffer_rsrc_t rs;
  int vo, mc, kb, ke;
  unsigned h[4], l[4];
  float2 raw[8];
  float s[2], top[2] = {0.f, 0.f};
  unsigned low[2] = {0, 0};
  __device__ __forceinline__ static int pos(int lane, int j) { return ((lane & 32) << 1) | (j << 5) | (lane & 31); }
  __device__ __forceinline__ static int octet(int tid) { return __builtin_amdgcn_readfirstlane(tid >> 6); }
  __device__ __forceinline__ SplitKM(const L& l, int m0, int m_end, int kb_, int ke_, int tid)
      : ld(l), kb(kb_), ke(ke_) {
    rs = buffer_of(l.base() + (long long)kb_ * l.ld, 4LL * (ke_ - kb_) * l.ld);
    const int m = m0 + 2 * (tid & 63);
    mc = m < m_end ? m : m_end - 2;
    vo = 4 * (8 * octet(tid) * (int)l.ld + mc);
  }
  __device__ __forceinline__ void load_rows(int k, int i0, int n) {
    const int row = 4 * (int)ld.ld, at = vo + (k - kb) * row;
#pragma unroll
    for (int i = i0; i < i0 + n; ++i)
      raw[i] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, at + i * row, 0, 0));
  }
  __device__ __forceinline__ void load(int k) { load_rows(k, 0, 8); }
  __device__ __forceinline__ float2 value(int i, int k, int tid) const {
    const int r = k + 8 * octet(tid) + i;
    float f = 1.f;
    if constexpr (L::kRowFactor) f = ld.s[r < ke ? r : ke - 1];
    const float2 v = ld.apply2(raw[i], f, mc);
    // a padded row must not take part in the choice of a column's scale: loaded as zeros, it stays zero
    return L::kZeroToZero || r < ke ? v : make_float2(0.f, 0.f);
  }
  __device__ __forceinline__ void values(int k, int tid, Values& x) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = value(i, k, tid);
  }
  __device__ __forceinline__ static void publish(const Values& x, float* mx, int tid) {
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      a = fmaxf(a, fabsf(x[i].x));
      b = fmaxf(b, fabsf(x[i].y));
    }
    reinterpret_cast<float2*>(mx)[tid] = make_float2(a, b);
  }
  __device__ __forceinline__ void scales(const Values&, const float* mx, int* ex, int tid) {
    const int lane = tid & 63;
    float m[2] = {0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float2 v = reinterpret_cast<const float2*>(mx)[w * 64 + lane];
      m[0] = fmaxf(m[0], v.x);
      m[1] = fmaxf(m[1], v.y);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int f = scale_field(m[j], Count ? 0 : kRowsTarget);
      s[j] = __uint_as_float((unsigned)f << 23);
      if (tid < 64) ex[pos(lane, j)] = 127 - f;
    }
  }
  __device__ __forceinline__ void put(int j, char* d, int tid) const {
    d += octet(tid) * SP_OCT + pos(tid & 63, j) * 16;
    *reinterpret_cast<uint4*>(d) = make_uint4(h[0], h[1], h[2], h[3]);
    *reinterpret_cast<uint4*>(d + SP_PLANE) = make_uint4(l[0], l[1], l[2], l[3]);
  }
  // a quarter of the stage: one column of each pair, four k; and the loads of the stage that follows
  __device__ __forceinline__ void piece(int n, int k, int next, char* d, int tid) {
    const int j = n >> 1, i0 = 4 * (n & 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float2 u = value(i0 + 2 * i, k, tid), v = value(i0 + 2 * i + 1, k, tid);
      split_pair<Count>(j ? u.y : u.x, j ? v.y : v.x, s[j], h[i0 / 2 + i], l[i0 / 2 + i], top[j], low[j]);
    }
    if (n & 1) put(j, d, tid);
    if (j) load_rows(next, i0, 4);
  }
  __device__ __forceinline__ void store_all(const Values& x, char* d, int tid) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 u = x[2 * i], v = x[2 * i + 1];
        split_pair<Count>(j ? u.y : u.x, j ? v.y : v.x, s[j], h[i], l[i], top[j], low[j]);
      }
      put(j, d, tid);
    }
  }
  struct Counts {
    unsigned low[2] = {};
    float top[2] = {};
  };
  __device__ __forceinline__ unsigned past(int k, int tid) const {   // 2048ths that a stage's zeros past the end count
    const int n = k + 8 * octet(tid) + 8 - ke;
    return 2048 * (n < 0 ? 0 : n < 8 ? n : 8);
  }
  // what the loop has counted
  __device__ __forceinline__ Counts counts(int last, int tid) const {
    Counts c;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      c.low[j] = low[j] - past(last, tid);
      c.top[j] = top[j];
    }
    return c;
  }
  __device__ __forceinline__ void store_high(const Values& x, int k, Counts& c, char* d, int tid) const {
    d += octet(tid) * SP_OCT;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      unsigned u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 a = x[2 * i], b = x[2 * i + 1];
        u[i] = split_high(j ? a.y : a.x, j ? b.y : b.x, s[j], c.top[j], c.low[j]);
      }
      c.low[j] -= past(k, tid);
      *reinterpret_cast<uint4*>(d + pos(tid & 63, j) * 16) = make_uint4(u[0], u[1], u[2], u[3]);
    }
  }
  __device__ __forceinline__ static void publish_counts(const Counts& c, const LowCount& to, int p0, int tid) {
#pragma unroll
    for (int j = 0; j < 2; ++j) to.add(p0 + pos(tid & 63, j), c.low[j], c.top[j]);
  }
};

// One stage of split products: per 32 x 32 block and 16 k, hi += h h' and lo += h l' + l h'.  Between
// the 12 BI matrix instructions piece(0..NP - 1) run at equal distances: the conversion of the next
// stage in parts, spread so that the vector units work while the matrix unit does.
template <int BI, int NP, class F>
__device__ __forceinline__ void split_stage(const char* st, int wm, int wn, int lr, int hf, f32x16 (&hi)[BI][2],
                                            f32x16 (&lo)[BI][2], const F& piece) {
  constexpr int kEvery = 12 * BI / NP;
  f16x8 a[BI][2], b[2][2];
#pragma unroll
  for (int q = 0; q < 12 * BI; ++q) {
    const int g = q / (6 * BI), t = q / (2 * BI) % 3, bi = q / 2 % BI, bj = q % 2;
    if (q % (6 * BI) == 0) {
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const char* o = st + p * SP_PLANE + (2 * g + hf) * SP_OCT;
#pragma unroll
        for (int c = 0; c < BI; ++c)
          a[c][p] = *reinterpret_cast<const f16x8*>(o + (wm * 32 * BI + c * 32 + lr) * 16);
#pragma unroll
        for (int c = 0; c < 2; ++c)
          b[c][p] = *reinterpret_cast<const f16x8*>(o + SP_OPER + (wn * 64 + c * 32 + lr) * 16);
      }
    }
    if (t == 0)
      hi[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[bi][0], b[bj][0], hi[bi][bj], 0, 0, 0);
    else
      lo[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[bi][t == 2], b[bj][t == 1], lo[bi][bj], 0, 0, 0);
    if (q % kEvery == kEvery - 1) piece(q / kEvery);
  }
}

// One stage of sum h h' of the operands' magnitudes.
template <int BI>
__device__ __forceinline__ void magnitude_stage(const char* st, int wm, int wn, int lr, int hf, f32x16 (&m)[BI][2]) {
  auto octet = [&](const char* o, int row) {
    uint4 x = *reinterpret_cast<const uint4*>(o + row * 16);
    x.x &= 0x7fff7fffu;
    x.y &= 0x7fff7fffu;
    x.z &= 0x7fff7fffu;
    x.w &= 0x7fff7fffu;
    return __builtin_bit_cast(f16x8, x);
  };
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const char* o = st + (2 * g + hf) * SP_OCT;
    f16x8 a[BI], b[2];
#pragma unroll
    for (int c = 0; c < BI; ++c) a[c] = octet(o, wm * 32 * BI + c * 32 + lr);
#pragma unroll
    for (int c = 0; c < 2; ++c) b[c] = octet(o + SP_OPER, wn * 64 + c * 32 + lr);
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) m[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], b[j], m[i][j], 0, 0, 0);
  }
}

// Whether a tile has lost nothing that matters, where its last stages do not show it.  m holds their magnitudes;
// kCount: the tile's counts are complete; else every entry of m from `most` on is enough.  The registers hold
// the operands' first stage.
template <int BI, class SA, class SB>
__device__ __forceinline__ bool enough(float* smem, SA& sa, SB& sb, float most, int kb, int ke, int wm, int wn, int lr,
                                       int hf, int tid, f32x16 (&m)[BI][2]) {
  constexpr bool kCount = SA::kCount && SB::kCount;
  char* st = reinterpret_cast<char*>(smem);
  float* flag = smem + SMEM_BODY + 3 * (GBM + GBN);
  const LowCount count(smem);
  auto all = [&](int f, bool ok) {
    if ((tid & 63) == 63) flag[f + (tid >> 6)] = ok ? 0.f : 1.f;
    __syncthreads();
    return flag[f] + flag[f + 1] + flag[f + 2] + flag[f + 3] == 0.f;
  };
  // The order of the stages: of 6 or more first a sample (every n / 4-th; with kCount, of 18 or more, then
  // every n / 16-th between them; none of the last two), then all from the beginning.
  const int n = (ke - kb + SBK - 1) / SBK, sample = n < 6 ? 0 : kCount && n >= 18 ? 16 : 4;
  auto at = [&](int q) {
    if (q >= sample) return q - sample;
    return (n - 2) * (q < 4 ? 4 * q : q - 3 + (q - 4) / 3) / 16;
  };
  for (int q = 0, f = 4, i = 0;; ++q) {
    if (q == sample || (q == 0 && !kCount)) zero_acc(m);
    const bool last = q == sample + n - 1;
    {   // the stage's loads have been issued; issue the next one's
      typename SA::Values xa;
      typename SB::Values xb;
      typename SA::Counts ca;
      typename SB::Counts cb;
      sa.values(kb + i * SBK, tid, xa);
      sa.store_high(xa, kb + i * SBK, ca, st, tid);
      sb.values(kb + i * SBK, tid, xb);
      sb.store_high(xb, kb + i * SBK, cb, st + SP_OPER, tid);
      if (!kCount && q >= sample) {
        SA::publish_counts(ca, count, 0, tid);
        SB::publish_counts(cb, count, GBM, tid);
      }
      i = last ? 0 : at(q + 1);
      sa.load(kb + i * SBK);
      sb.load(kb + i * SBK);
    }
    __syncthreads();
    magnitude_stage<BI>(st, wm, wn, lr, hf, m);
    __syncthreads();
    if constexpr (kCount) {
      if (last || (q == 3 && sample) || (q == 15 && sample == 16)) {
        if (all(f, covered<BI>(count, wm, wn, lr, hf, m))) return true;
        if (last) return false;
        f += 4;
      }
    } else {
      if (last) break;
      if (sample && q == 3 && all(4, smallest<BI>(m) >= most)) return true;
    }
  }
  count.share(tid);
  __syncthreads();
  return all(8, covered<BI>(count, wm, wn, lr, hf, m));
}

// The K loop of the split products over [kb, ke).  A and B: loader, first and last row (column)
// of the tile's operand.  On return hi holds h h' + 2^-11 (h l' + l h') of the scaled operands and
// smem the exponents that undo the scales; false if a value is not finite or the split may have lost too much.
template <class SA, class SB, int BI, class LA, class LB>
__device__ __forceinline__ bool split_loop(float* smem, const LA& al, int a0, int a1, const LB& bl, int b0, int b1,
                                           int kb, int ke, int wm, int wn, int lr, int hf, int tid,
                                           f32x16 (&hi)[BI][2]) {
  char* lds = reinterpret_cast<char*>(smem);
  int* ex = reinterpret_cast<int*>(smem + SMEM_BODY);   // [128] rows, [128] columns
  float* flag = smem + SMEM_BODY + 3 * (GBM + GBN);   // [4] each, one of a wave
  const LowCount count(smem);
  count.low[tid] = 0;
  count.top[tid] = 0.f;
  f32x16 lo[BI][2];
  constexpr bool kCount = SA::kCount && SB::kCount;
  zero_acc(hi);
  zero_acc(lo);
  SA sa(al, a0, a1, kb, ke, tid);
  SB sb(bl, b0, b1, kb, ke, tid);
  sa.load(kb);
  sb.load(kb);
  {
    typename SA::Values xa;
    typename SB::Values xb;
    sa.values(kb, tid, xa);
    sb.values(kb, tid, xb);
    float* mx = smem + SP_STAGE / 4;   // the second stage buffer, not in use yet
    sa.publish(xa, mx, tid);
    sb.publish(xb, mx + 512, tid);
    if constexpr (SA::kPaired || SB::kPaired) __syncthreads();
    sa.scales(xa, mx, ex, tid);
    sb.scales(xb, mx + 512, ex + GBM, tid);
    sa.store_all(xa, lds, tid);
    sb.store_all(xb, lds + SP_OPER, tid);
  }
  // The registers run one stage ahead of the planes: while stage k is multiplied, stage k + 1 (whose
  // loads were issued a whole stage earlier) is converted and the loads of stage k + 2 are issued.
  const int last = kb + (ke - kb - 1) / SBK * SBK;
  int k1 = kb + SBK < last ? kb + SBK : last;
  sa.load(k1);
  sb.load(k1);
  auto publish_counts = [&]() {   // every value has been split
    if constexpr (kCount) {
      SA::publish_counts(sa.counts(last, tid), count, 0, tid);
      SB::publish_counts(sb.counts(last, tid), count, GBM, tid);
    }
  };
  if (kCount && kb == last) {
    __syncthreads();   // the counts are zero
    publish_counts();
  }
  __syncthreads();
  int cur = 0;
  for (int k = kb; k < last; k += SBK) {
    char* d = lds + (cur ^ 1) * SP_STAGE;
    const int next = k1 < last ? k1 + SBK : kb;   // the first stage again for enough()
    split_stage<BI, SA::kPieces + SB::kPieces>(lds + cur * SP_STAGE, wm, wn, lr, hf, hi, lo, [&](int n) {
      if (n < SA::kPieces) sa.piece(n, k1, next, d, tid); else sb.piece(n - SA::kPieces, k1, next, d + SP_OPER, tid);
      __builtin_amdgcn_sched_barrier(0);   // keeps the parts where they are
    });
    if (k1 == last) publish_counts();
    k1 = next;
    __syncthreads();
    cur ^= 1;
  }
  if constexpr (kCount) count.share(tid);
  split_stage<BI, 1>(lds + cur * SP_STAGE, wm, wn, lr, hf, hi, lo, [](int) {});
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        hi[i][j][v] = fmaf(lo[i][j][v], 1.f / 2048.f, hi[i][j][v]);
        z = fmaf(hi[i][j][v], 0.f, z);   // not a number once a value is infinite or not a number
      }
  auto put = [&](int f, float x) {
    if ((tid & 63) == 63) flag[f + (tid >> 6)] = x;
  };
  put(0, __any(z != z) ? 1.f : 0.f);
  // the magnitudes of the last stage, and of the one before it, whose planes are still there
  zero_acc(lo);
  magnitude_stage<BI>(lds + cur * SP_STAGE, wm, wn, lr, hf, lo);
  if (last >= kb + (kCount ? 7 : 31) * SBK) magnitude_stage<BI>(lds + (cur ^ 1) * SP_STAGE, wm, wn, lr, hf, lo);
  if constexpr (!kCount) put(4, smallest<BI>(lo));
  __syncthreads();
  if (flag[0] + flag[1] + flag[2] + flag[3] != 0.f) return false;
  const float most = 8.f * (float)(ke - kb);   // K (2^16 + 2^16) 2^-35 / 2^-21
  if constexpr (kCount) {
    put(4, covered<BI>(count, wm, wn, lr, hf, lo) ? 0.f : 1.f);
    __syncthreads();
    if (flag[4] + flag[5] + flag[6] + flag[7] == 0.f) return true;
  } else {
    if (fminf(fminf(flag[4], flag[5]), fminf(flag[6], flag[7])) >= most) return true;
  }
  __syncthreads();   // the flags are written again
  return enough<BI>(smem, sa, sb, most, kb, ke, wm, wn, lr, hf, tid, lo);
}

// Undo the scales: acc[bi][bj][v] is row 32 bi + 8 (v / 4) + 4 hf + v % 4, column 32 bj + lr of the wave.
template <int BI>
__device__ __forceinline__ void unscale(const float* smem, int wm, int wn, int lr, int hf, f32x16 (&acc)[BI][2]) {
  const int* ex = reinterpret_cast<const int*>(smem + SMEM_BODY);
#pragma unroll
  for (int bi = 0; bi < BI; ++bi)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      const int4 er = *reinterpret_cast<const int4*>(ex + wm * 32 * BI + bi * 32 + 8 * v4 + 4 * hf);
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const int ec = ex[128 + wn * 64 + bj * 32 + lr];
        acc[bi][bj][4 * v4] = ldexpf(acc[bi][bj][4 * v4], er.x + ec);
        acc[bi][bj][4 * v4 + 1] = ldexpf(acc[bi][bj][4 * v4 + 1], er.y + ec);
        acc[bi][bj][4 * v4 + 2] = ldexpf(acc[bi][bj][4 * v4 + 2], er.z + ec);
        acc[bi][bj][4 * v4 + 3] = ldexpf(acc[bi][bj][4 * v4 + 3], er.w + ec);
      }
    }
}

// ---------------------------------------------------------------- gemm_rows

// The K loop on the fp32 matrix instructions.
template <bool NT, class ALoad>
__device__ __forceinline__ void rows_fp32(float* smem, const ALoad& al, const float* __restrict__ Bg, int K, int N,
                                          int r0, int r1, int n0, int wm, int wn, int lr, int hf, int tid,
                                          f32x16 (&acc)[2][2]) {
  // double buffers: A at smem + b * GBM * LD_MK, B after both A buffers
  auto sA = [&](int b) { return smem + b * (GBM * LD_MK); };
  auto sB = [&](int b) { return smem + 2 * GBM * LD_MK + b * B_BUF; };
  StageMK<ALoad> sa;
  constexpr bool DA = IsPlainLoad<ALoad>::value;
  auto load_a = [&](int k, float* dst) {
    if constexpr (DA) direct_mk(reinterpret_cast<const LoadPlain&>(al).p, reinterpret_cast<const LoadPlain&>(al).ld,
                                r0, r1, k, dst, tid);
    else sa.load(al, r0, r1, k, tid);
  };
  auto load_b = [&](int k, float* dst) {
    if (NT) direct_mk(Bg, K, n0, N, k, dst, tid); else direct_km(Bg, N, k, n0, N, dst, tid);
  };
  zero_acc(acc);
  load_a(0, sA(0));
  load_b(0, sB(0));
  if constexpr (!DA) sa.store(al, sA(0), 0, tid);
  wait_direct();
  __syncthreads();

  const int nk = K / GBK;
  int cur = 0;
  for (int kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    const int k1 = (kt + 1) * GBK;
    if (more) {
      load_a(k1, sA(cur ^ 1));
      load_b(k1, sB(cur ^ 1));
    }
    // the stage's matrix instructions issue at raised wave priority, ahead of the
    // staging and epilogue work of the other workgroups on the SIMD (0.2-1 % faster)
    __builtin_amdgcn_s_setprio(1);
    mfma_stage<true, NT, true>(sA(cur), sB(cur), wm, wn, lr, hf, acc);
    __builtin_amdgcn_s_setprio(0);
    if (more) {
      if constexpr (!DA) sa.store(al, sA(cur ^ 1), k1, tid);
    }
    wait_direct();
    __syncthreads();
    cur ^= 1;
  }
}

// The same on split products, for a tile of 64 BI rows; false (and acc undefined) if a value is
// infinite or not a number.
template <bool NT, int BI, class ALoad>
__device__ __forceinline__ bool rows_split(float* smem, const ALoad& al, const float* __restrict__ Bg, int K, int N,
                                           int r0, int r1, int n0, int wm, int wn, int lr, int hf, int tid,
                                           f32x16 (&acc)[BI][2]) {
  const LoadPlain bl{Bg, NT ? K : N};
  using SA = SplitMK<ALoad, 2 * BI>;
  using SB = std::conditional_t<NT, SplitMK<LoadPlain>, SplitKM<LoadPlain>>;
  if (!split_loop<SA, SB, BI>(smem, al, r0, r1, bl, n0, N, 0, K, wm, wn, lr, hf, tid, acc)) return false;
  unscale<BI>(smem, wm, wn, lr, hf, acc);
  return true;
}

// One output tile of gemm_rows for (XCD-mapped) block number vb; smem holds
// SMEM_FLOATS floats of LDS.
template <bool NT, class ALoad, class Epi, int Mode>
__device__ __forceinline__ void gemm_rows_block(int vb, float* smem, const ALoad& al, const float* __restrict__ B,
                                                int K, int N, const RowsTable& table, const Epi& epi,
                                                float* __restrict__ rowsum_out) {
  constexpr int BI = Mode == kModeHalfRows ? 1 : 2;
  const int ncol = (N + GBN - 1) / GBN;
  int t, ctile;
  xcd_map(vb, BI == 1 ? 2 * ncol : ncol, t, ctile);
  RowsTile tile;
  if (!table.find(t, tile)) return;
  int r0 = tile.r0, r1 = tile.r1;
  if (BI == 1) {   // the upper or lower 64 rows of the tile
    r0 += 64 * (ctile & 1);
    ctile >>= 1;
    if (r0 >= r1) return;
    r1 = r1 < r0 + 64 ? r1 : r0 + 64;
  }
  const int n0 = ctile * GBN;
  const float* Bg = B + (long long)tile.group * K * N;

  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63;
  const int wm = w >> 1, wn = w & 1;
  const int lr = l & 31, hf = l >> 5;

  f32x16 acc[2][2];
  bool paired = false;   // columns of the two blocks: 2 lr and 2 lr + 1 (else lr and 32 + lr)
  bool wide = true;      // a wave holds 64 rows (else 32, in acc[0])
  if constexpr (Mode == kModeFp32) {
    rows_fp32<NT>(smem, al, Bg, K, N, r0, r1, n0, wm, wn, lr, hf, tid, acc);
  } else {
    bool done;
    if constexpr (BI == 1) {
      f32x16 a1[1][2];
      done = rows_split<NT, 1>(smem, al, Bg, K, N, r0, r1, n0, wm, wn, lr, hf, tid, a1);
      acc[0][0] = a1[0][0];
      acc[0][1] = a1[0][1];
      wide = !done;
    } else {
      done = rows_split<NT, 2>(smem, al, Bg, K, N, r0, r1, n0, wm, wn, lr, hf, tid, acc);
    }
    if (!done) rows_fp32<NT>(smem, al, Bg, K, N, r0, r1, n0, wm, wn, lr, hf, tid, acc);
    paired = done && !NT;
  }

  // Epilogue in two halves of 64 rows: the waves of row half `half` stage
  // their accumulators (lane l of block (bi, bj) holds column lr and rows
  // 8 (v / 4) + 4 hf + v % 4), then every thread visits 8 float4 pieces in
  // two batches: first the batch's global reads, then arithmetic and stores.
  float* sC = smem;
#pragma unroll
  for (int half = 0; half < BI; ++half) {
    auto stage = [&](int bi, int row) {
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          sC[(row + 8 * (v >> 2) + 4 * hf + (v & 3)) * LD_C + wn * 64 + (paired ? 2 * lr + bj : bj * 32 + lr)] =
              acc[bi][bj][v];
    };
    if (BI == 1 && !wide) {
      stage(0, 32 * wm);
    } else if (wm == half) {
      stage(0, 0);
      stage(1, 32);
    }
    // 4 pieces per batch; loads past the range read the last valid row.
    const int c4 = tid & 31;
    const int col = n0 + 4 * c4;
    const int colc = col < N ? col : N - 4;
#pragma unroll
    for (int i0 = 0; i0 < 8; i0 += 4) {
      typename Epi::Raw raw[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const long long row = (long long)r0 + half * 64 + (tid >> 5) + 8 * (i0 + j);
        raw[j] = epi.load(row < r1 ? row : (long long)r1 - 1, colc);
      }
      if (i0 == 0) __syncthreads();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int rl = (tid >> 5) + 8 * (i0 + j);
        const long long row = (long long)r0 + half * 64 + rl;
        float part = 0.f;
        if (row < r1 && col < N) part = epi.store(row, col, ld4(sC + rl * LD_C + 4 * c4), raw[j]);
        if (Epi::kRowSum) {
#pragma unroll
          for (int o = 16; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
          if (c4 == 0 && row < r1) rowsum_out[row * ncol + ctile] = part;
        }
      }
    }
    __syncthreads();
  }
}

template <bool NT, class ALoad, class Epi, int Mode>
__global__ __launch_bounds__(256, 2) void gemm_rows_kernel(
    ALoad al, const float* __restrict__ B, int K, int N, RowsTable table, Epi epi, float* __restrict__ rowsum_out) {
  __shared__ __attribute__((aligned(16)))
  float smem[Mode == kModeFp32 ? SMEM_FP32 : SMEM_FLOATS];
  gemm_rows_block<NT, ALoad, Epi, Mode>(blockIdx.x, smem, al, B, K, N, table, epi, rowsum_out);
}

// --------------------------------------------------------------- gemm_wgrad
// Both operands are row-major over the contraction index r: A [M, P], B [M, Q].

struct WChunk {
  int group;
  int r0;
  int r1;
  int alone;        // 1: the group's only chunk
};

// The contraction on the fp32 matrix instructions.
template <class ALoad, class BLoad>
__device__ __forceinline__ void wgrad_fp32(float* smem, const ALoad& al, const BLoad& bl, int P, int Q,
                                           const WChunk& ch, int p0, int q0, int wm, int wn, int lr, int hf, int tid,
                                           f32x16 (&acc)[2][2]) {
  auto sA = [&](int b) { return smem + b * (GBK * LD_KM); };
  auto sB = [&](int b) { return smem + (2 + b) * (GBK * LD_KM); };
  zero_acc(acc);
  StageKM<ALoad> sa;
  StageKM<BLoad> sb;
  // Both operands in the unpadded swizzled [k][m] layout.  A plain operand loads its whole
  // 16-row stages straight into LDS, and the chunk's last partial stage through registers
  // (its rows past the chunk become zeros); a transformed operand always goes through
  // registers.
  constexpr bool DA = IsPlainLoad<ALoad>::value, DB = IsPlainLoad<BLoad>::value;
  auto stage_load = [&](long long rk, int buf) {
    const bool full = rk + GBK <= ch.r1;
    if constexpr (DA) {
      if (full) direct_km(al.p, al.ld, rk, p0, P, sA(buf), tid); else sa.load(al, rk, ch.r1, p0, P, tid);
    } else {
      sa.load(al, rk, ch.r1, p0, P, tid);
    }
    if constexpr (DB) {
      if (full) direct_km(bl.p, bl.ld, rk, q0, Q, sB(buf), tid); else sb.load(bl, rk, ch.r1, q0, Q, tid);
    } else {
      sb.load(bl, rk, ch.r1, q0, Q, tid);
    }
  };
  auto stage_store = [&](long long rk, int buf) {
    const bool full = rk + GBK <= ch.r1;
    if (!DA || !full) sa.store_sw(al, sA(buf), p0, tid);
    if (!DB || !full) sb.store_sw(bl, sB(buf), q0, tid);
  };
  stage_load(ch.r0, 0);
  stage_store(ch.r0, 0);
  wait_direct();
  __syncthreads();

  const int nk = (ch.r1 - ch.r0 + GBK - 1) / GBK;
  int cur = 0;
  for (int kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    const long long rk = (long long)ch.r0 + (kt + 1) * GBK;
    if (more) stage_load(rk, cur ^ 1);
    __builtin_amdgcn_s_setprio(1);
    mfma_stage<false, false, true>(sA(cur), sB(cur), wm, wn, lr, hf, acc);
    __builtin_amdgcn_s_setprio(0);
    if (more) stage_store(rk, cur ^ 1);
    wait_direct();
    __syncthreads();
    cur ^= 1;
  }
}

// The same on split products; false (and acc undefined) if a value is infinite or not a number.
template <class ALoad, class BLoad>
__device__ __forceinline__ bool wgrad_split(float* smem, const ALoad& al, const BLoad& bl, int P, int Q,
                                            const WChunk& ch, int p0, int q0, int wm, int wn, int lr, int hf, int tid,
                                            f32x16 (&acc)[2][2]) {
  if (!split_loop<SplitKM<ALoad, true>, SplitKM<BLoad, true>, 2>(smem, al, p0, P, bl, q0, Q, ch.r0, ch.r1, wm, wn, lr, hf, tid, acc))
    return false;
  unscale<2>(smem, wm, wn, lr, hf, acc);
  return true;
}

// One partial tile of gemm_wgrad for (XCD-mapped) block number vb.
template <class ALoad, class BLoad, bool Split>
__device__ __forceinline__ void gemm_wgrad_block(int vb, float* smem, const ALoad& al, const BLoad& bl, int P, int Q,
                                                 const WChunk* __restrict__ chunks,
                                                 const int* __restrict__ n_chunks, float* __restrict__ partial,
                                                 float* __restrict__ G, int accumulate) {
  const int ntq = (Q + GBN - 1) / GBN;
  int c, pq;
  xcd_map(vb, ((P + GBM - 1) / GBM) * ntq, c, pq);
  if (c >= *n_chunks) return;
  const WChunk ch = chunks[c];
  const int p0 = (pq / ntq) * GBM;
  const int q0 = (pq % ntq) * GBN;

  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63;
  const int wm = w >> 1, wn = w & 1;
  const int lr = l & 31, hf = l >> 5;

  f32x16 acc[2][2];
  bool paired = false;   // rows and columns of the two blocks: 2 i and 2 i + 1 (else i and 32 + i)
  if constexpr (Split) {
    paired = wgrad_split(smem, al, bl, P, Q, ch, p0, q0, wm, wn, lr, hf, tid, acc);
    if (!paired) wgrad_fp32(smem, al, bl, P, Q, ch, p0, q0, wm, wn, lr, hf, tid, acc);
  } else {
    wgrad_fp32(smem, al, bl, P, Q, ch, p0, q0, wm, wn, lr, hf, tid, acc);
  }

  // the only chunk of a group writes (adds to) its gradient, one of several writes a partial block
  auto put = [&](float* out, auto add) {
    constexpr bool Add = decltype(add)::value;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = 8 * (v >> 2) + 4 * hf + (v & 3);
        const int pr = p0 + wm * 64 + (paired ? 2 * i + bi : bi * 32 + i);
        if (paired) {
          const int qc = q0 + wn * 64 + 2 * lr;
          if (pr < P && qc < Q) {
            float2* o = reinterpret_cast<float2*>(out + (long long)pr * Q + qc);
            float2 x = make_float2(acc[bi][0][v], acc[bi][1][v]);
            if (Add) x = make_float2(o->x + x.x, o->y + x.y);
            *o = x;
          }
        } else {
#pragma unroll
          for (int bj = 0; bj < 2; ++bj) {
            const int qc = q0 + wn * 64 + bj * 32 + lr;
            float* o = out + (long long)pr * Q + qc;
            if (pr < P && qc < Q) *o = Add ? *o + acc[bi][bj][v] : acc[bi][bj][v];
          }
        }
      }
  };
  if (!ch.alone)
    put(partial + (long long)c * P * Q, std::false_type{});
  else if (accumulate)
    put(G + (long long)ch.group * P * Q, std::true_type{});
  else
    put(G + (long long)ch.group * P * Q, std::false_type{});
}

template <class ALoad, class BLoad, bool Split>
__global__ __launch_bounds__(256, 2) void gemm_wgrad_kernel(ALoad al, BLoad bl, int P, int Q,
                                                            const WChunk* __restrict__ chunks,
                                                            const int* __restrict__ n_chunks,
                                                            float* __restrict__ partial, float* __restrict__ G,
                                                            int accumulate) {
  __shared__ __attribute__((aligned(16))) float smem[Split ? SMEM_FLOATS : SMEM_FP32];
  gemm_wgrad_block<ALoad, BLoad, Split>(blockIdx.x, smem, al, bl, P, Q, chunks, n_chunks, partial, G,
                                        accumulate);
}

// ---------------------------------------------------------- skinny wgrad
// G[p, q] = sum_r s[r] A[r, p] B[r, q] for a short P (P <= 32, a multiple of 4;
// Q = 64, 128, 256 or 512: the radial-filter gradient, P = basis size, Q = d).
// A 128-row MFMA tile would be mostly padding there, so the vector units do it,
// straight from global memory.  A workgroup owns one chunk of rows and the whole
// P x Q output.  Lane l of a wave owns CW = min(4, Q / 64) consecutive columns of
// a 64 CW-wide column slice; the NS = Q / (64 CW) slices and RG = 4 / NS row
// groups split the four waves, wave (g, slice) accumulating all P output rows of
// its columns over the chunk rows g, g + RG, g + 2 RG, ...  A row's P values of A
// and its scale are the same for the whole wave, so they come through scalar loads
// and the vector registers hold only B and the accumulators; each step takes U
// rows and issues all their loads before using any.  Per row, b' = s[r] B[r, :]
// (B[r, :] if s is null) and acc[p] += A[r, p] b'.  The row groups are summed
// through LDS (P Q floats of dynamic LDS) in group order, and the workgroup writes
// one partial per chunk, reduced like gemm_wgrad's.
inline int skinny_cw(int Q) { return Q >= 256 ? 4 : Q / 64; }
inline int skinny_rows(int Q) {   // rows of one step of the workgroup (U = 4 rows per row group)
  return 4 * (4 / (Q / (64 * skinny_cw(Q))));
}

template <int PM, int CW>
__global__ __launch_bounds__(256) void wgrad_skinny_kernel(const float* __restrict__ A, const float* __restrict__ s,
                                                           const float* __restrict__ B, int P, int Q,
                                                           const WChunk* __restrict__ chunks,
                                                           const int* __restrict__ n_chunks,
                                                           float* __restrict__ partial) {
  constexpr int U = 8;
  extern __shared__ __attribute__((aligned(16))) float sk_lds[];
  const int c = blockIdx.x;
  if (c >= *n_chunks) return;
  const WChunk ch = chunks[c];
  const int NS = Q / (64 * CW), RG = 4 / NS;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, la = lane % P;
  const int g = w / NS, col = (w - g * NS) * 64 * CW + lane * CW;
  float acc[PM][CW];
#pragma unroll
  for (int p = 0; p < PM; ++p)
#pragma unroll
    for (int k = 0; k < CW; ++k) acc[p][k] = 0.f;
  auto load_b = [&](long long r, float* v) {
    const float* q = B + r * Q + col;
    if constexpr (CW == 4) {
      const float4 x = ld4(q);
      v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else if constexpr (CW == 2) {
      const float2 x = *reinterpret_cast<const float2*>(q);
      v[0] = x.x; v[1] = x.y;
    } else {
      v[0] = *q;
    }
  };
  // lane l holds A[r, l mod P]; row p's value is read from lane p (lanes p >= P
  // hold a repeated column: those accumulator rows are never stored)
  auto sweep = [&](auto scaled) {
    constexpr bool SC = decltype(scaled)::value;
    auto row = [&](float av, float sc, const float* b) {
      float x[CW];
#pragma unroll
      for (int k = 0; k < CW; ++k) x[k] = SC ? sc * b[k] : b[k];
      const int ai = __float_as_int(av);
#pragma unroll
      for (int p = 0; p < PM; ++p) {
        const float ap = __int_as_float(__builtin_amdgcn_readlane(ai, p));
#pragma unroll
        for (int k = 0; k < CW; ++k) acc[p][k] += ap * x[k];
      }
    };
    long long r = (long long)ch.r0 + g;
    for (; r + (long long)(U - 1) * RG < ch.r1; r += (long long)U * RG) {
      float b[U][CW], av[U], sc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long long ru = r + (long long)u * RG;
        load_b(ru, b[u]);
        av[u] = A[ru * P + la];
        sc[u] = SC ? s[ru] : 1.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) row(av[u], sc[u], b[u]);
    }
    for (; r < ch.r1; r += RG) {
      float b[CW];
      load_b(r, b);
      row(A[r * P + la], SC ? s[r] : 1.f, b);
    }
  };
  if (s)
    sweep(std::true_type{});
  else
    sweep(std::false_type{});
  float* red = sk_lds;   // [P][Q]
  for (int gg = 0; gg < RG; ++gg) {
    if (g == gg) {
#pragma unroll
      for (int p = 0; p < PM; ++p) {
        if (p < P) {
#pragma unroll
          for (int k = 0; k < CW; ++k) {
            float v = acc[p][k];
            if (gg) v += red[p * Q + col + k];
            red[p * Q + col + k] = v;
          }
        }
      }
    }
    __syncthreads();
  }
  float4* out = reinterpret_cast<float4*>(partial + (long long)c * P * Q);
  const float4* red4 = reinterpret_cast<const float4*>(red);
  for (int i = threadIdx.x; i < P * Q / 4; i += 256) out[i] = red4[i];
}

}  // namespace janus
