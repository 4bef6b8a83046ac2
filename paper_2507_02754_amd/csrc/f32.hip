// Trilinear attention in float32 arithmetic on the gfx950 matrix cores: float32
// data of any head_dim, and the bf16 shapes the bf16 kernels do not take
// (head_dim 16 / 32, w2 > 64), whose operands are widened to float32 on load.
// Modulated queries, logits, probabilities and every partial sum are float32.
//
// Rows as in the bf16 kernels: r = (i, k) with q~_r = scale log2(e) q_i o k'_k,
// S^T = K q~^T, U^T += V^T P^T, on v_mfma_f32_32x32x2_f32 (4096 FLOPs in 64
// cycles, 1/16 of the bf16 rate). That rate decides the design: a 32 x 32 block
// of one product keeps a SIMD's matrix core busy for 32 D cycles while it reads
// 128 D bytes, so the operands go from L1 / L2 straight into registers, one
// chunk of 16 products ahead, with no LDS tiles and no barriers in the loops;
// the exponentials are under 3% of a block's time. What counts is that every
// SIMD has rows to work on, and that few of them are padding:
//   * a wavefront's 32 rows are 32 / W queries with W k-rows each, W = 8, 16 or
//     32 (w2 rounded up; more than 32 k-rows take several row groups);
//   * where a head has few queries the wavefronts of a workgroup split the key
//     blocks (query side) or the row blocks (key side) of the same outputs and
//     add their float32 sums in a fixed order.
//
// Measured, forward + backward: float32, B=1 H=4 N=2000 D=64 w1=256 w2=16, 16.8 ms
// on the plain kernels (one thread per pair, operands read per pair), 0.51 ms
// here; bf16, N=1024 D=128 w1=w2=128, 44.8 ms and 2.55 ms (1.55 ms on bf16 parts,
// below). The matrix cores are busy 60% of the time at these sizes. Vector
// instructions are what costs the rest: they add to the products' time even with
// two wavefronts per SIMD (6.9 per product: 0.54 ms; masks and operand checks on
// the edge blocks only: 0.51 ms), while loads issued further ahead of their use
// changed nothing.
//
// Operand layout (lane = 32 h + c). A row operand (rows along the lanes): lane
// (h, c) holds row c, columns 8 t + 4 h .. + 3 of float4 t; product 4 t + e
// contracts columns 8 t + e and 8 t + 4 + e. A transposed operand (columns d
// along the lanes, rows x along the contraction): product v contracts rows
// acc_row(v, 0) and acc_row(v, 1), the order in which an accumulator holds its
// rows, so probabilities go from accumulator to operand registers as they are;
// for accumulator tile dt lane (h, c) reads column 32 dt + c of that row.
//
// Every block's products start from zero and are added to the running sums
// afterwards: sums over thousands of rows then round once per 32 of them. The
// float32 products of a logit run in two chains of D / 2 columns added at the
// end: the rounding of one chain of D is the largest error of every output (D =
// 64: 2.0e-7 of O, the products' operands 0.3e-7; two chains 1.3e-7). The second
// chain takes the registers of dP (or of the products with V), free at that point.
//
// Masked pairs: their probabilities are set to 0. A row of V (or K, dO, ...)
// that only some of the pairs of a block may see is then multiplied by 0 for
// the others, which is not 0 if it holds infinities or NaN: such blocks add
// their products term by term with the masked ones left out (masked_tile).
#include "f32_offsets.h"
#include "mfma_common.h"

#include <algorithm>

namespace sa {
namespace {

constexpr int kFWaves = 4;
constexpr int kFThreads = 64 * kFWaves;
constexpr int kScratch = 32 * 33;  // floats of one wavefront's masked_tile scratch

// log2(e) and ln 2 minus their float32 values
constexpr float kLog2eLo = static_cast<float>(1.4426950408889634074 - static_cast<double>(kLog2e));
constexpr float kLn2Lo = static_cast<float>(0.69314718055994530942 - static_cast<double>(kLn2));
// 2^(x - lse log2 e) with lse log2 e as hi + lo: the normaliser's product is not
// rounded before the difference (it is several times larger than the differences
// that matter). x has the scale in its q~, rounded as in the forward: its errors
// then largely cancel against those in lse. An infinite lse has no low part (its
// remainder is NaN): +inf gives probabilities of 0, a query left out.
struct Norm {
  float hi, lo;
  __device__ __forceinline__ explicit Norm(float lse) : hi(lse * kLog2e) {
    const float r = __builtin_fmaf(lse, kLog2eLo, __builtin_fmaf(lse, kLog2e, -hi));
    lo = fabsf(hi) < __builtin_inff() ? r : 0.f;
  }
};
__device__ __forceinline__ float prob(float x, const Norm& n) { return fast_exp2((x - n.hi) - n.lo); }

__device__ __forceinline__ f32x16_t mfma_f32(float a, float b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Four consecutive elements, as loaded, and in float32.
template <typename T>
struct Raw4;
template <>
struct Raw4<float> {
  u32x4_t a;
  __device__ __forceinline__ float at(int e) const { return __uint_as_float(a[e]); }
};
template <>
struct Raw4<uint16_t> {
  u32x2_t a;
  __device__ __forceinline__ float at(int e) const { return (e & 1) ? bf16_hi(a[e >> 1]) : bf16_lo(a[e >> 1]); }
};
template <typename T>
__device__ __forceinline__ Raw4<T> ld4(const T* p) {
  return *reinterpret_cast<const Raw4<T>*>(p);
}
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(uint16_t x) { return bf16_to_f32(x); }

// Rows n0 .. N - 1 of one head (row stride `rsb` bytes) as a buffer: loads take
// a 32-bit byte offset from row n0 and rows past the sequence, or before n0
// (negative offsets), load as zeros. A head may span more than 2^31 bytes: the
// buffer starts at the block's own row and reaches as far as offsets do
// (f32_offsets.h: shapes whose blocks span more do not come here).
constexpr int kFar = static_cast<int>(f32_offsets::kReach);  // an offset past every buffer's end
template <typename T, int D>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_from(const T* head, int n0, int N, size_t rsb) {
  const size_t left = n0 < N ? static_cast<size_t>(N - 1 - n0) * rsb + D * sizeof(T) : 0;
  return make_rsrc(reinterpret_cast<const char*>(head) + static_cast<size_t>(n0) * rsb,
                   static_cast<unsigned>(left < kFar ? left : kFar));
}
template <typename T>
__device__ __forceinline__ Raw4<T> ldb4(__amdgpu_buffer_rsrc_t r, int off) {
  if constexpr (sizeof(T) == 4)
    return Raw4<T>{ldbuf128(r, off)};
  else
    return Raw4<T>{ldbuf64(r, off)};
}
template <typename T>
__device__ __forceinline__ T ldb1(__amdgpu_buffer_rsrc_t r, int off) {
  if constexpr (sizeof(T) == 4)
    return __uint_as_float(ldbuf32(r, off));
  else
    return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
}

__device__ __forceinline__ void st1(float* p, float x) { *p = x; }
__device__ __forceinline__ void st1(uint16_t* p, float x) { *p = f32_to_bf16(x); }

// Geometry of one head_dim.
template <int D>
struct Geo {
  static constexpr int NF = D / 8;                // float4 of a row operand per lane
  static constexpr int RC = NF < 4 ? NF : 4;      // of them in a chunk (16 products)
  static constexpr int NRC = NF / RC;             // chunks of a row-operand product
  static constexpr int NDT = D < 32 ? 1 : D / 32; // accumulator tiles over d
  static constexpr int NV = D < 32 ? 8 : 16;      // accumulator registers that hold a column
};

template <typename T, int D>
struct RowChunk {
  Raw4<T> x[Geo<D>::RC];
};
// Columns of the accumulator tiles: row m of tile dt is column 32 dt + m, or for
// bf16 data of several tiles NDT m + dt, so that one load of a row (8 bytes a
// lane at head_dim 128) serves every tile of a transposed operand: a quarter of
// the load instructions, 1.62 -> 1.55 ms at B=1 H=4 N=1024 w1=w2=128.
template <typename T, int D>
constexpr bool kWide = sizeof(T) == 2 && D >= 64;
template <typename T, int D>
struct Wide {
  using W = T;  // what a lane loads of a row
};
template <>
struct Wide<uint16_t, 64> {
  using W = unsigned;
};
template <>
struct Wide<uint16_t, 128> {
  using W = u32x2_t;
};
template <typename T, int D>
__device__ __forceinline__ typename Wide<T, D>::W ldw(__amdgpu_buffer_rsrc_t r, int off) {
  if constexpr (!kWide<T, D>)
    return ldb1<T>(r, off);
  else if constexpr (D == 64)
    return ldbuf32(r, off);
  else
    return ldbuf64(r, off);
}
template <typename T, int D>
__device__ __forceinline__ unsigned word(const typename Wide<T, D>::W& w, int dt) {
  if constexpr (D == 128)
    return w[dt >> 1];
  else
    return w;
}
// Element of tile dt, in float32.
template <typename T, int D>
__device__ __forceinline__ float elem(const typename Wide<T, D>::W& w, int dt) {
  if constexpr (kWide<T, D>)
    return (dt & 1) ? bf16_hi(word<T, D>(w, dt)) : bf16_lo(word<T, D>(w, dt));
  else
    return to_f32(w);
}
// Column of row m of tile dt, and 32 dt + m of column d.
template <typename T, int D>
__device__ __forceinline__ int column(int dt, int m) {
  return kWide<T, D> ? Geo<D>::NDT * m + dt : 32 * dt + m;
}
template <typename T, int D>
__device__ __forceinline__ int place(int d) {
  return kWide<T, D> ? 32 * (d % Geo<D>::NDT) + d / Geo<D>::NDT : d;
}
// One accumulator tile's operand (kWide: every tile's): the lane's column of
// rows acc_row(v, h).
template <typename T, int D>
struct TrChunk {
  typename Wide<T, D>::W x[16];
};
// Rows d .. d + 3 of tile dt: the columns of one row of a tensor.
template <typename T, int D>
__device__ __forceinline__ void ldcols(__amdgpu_buffer_rsrc_t b, int off, int dt, int d, float* z) {
  if constexpr (kWide<T, D>) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      z[e] = to_f32(ldb1<T>(b, off + column<T, D>(dt, d + e) * static_cast<int>(sizeof(T))));
  } else {
    const Raw4<T> r = ldb4<T>(b, off + (32 * dt + d) * static_cast<int>(sizeof(T)));
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = r.at(e);
  }
}
// A row in accumulator order: get gives rows 8 vq + 4 h .. + 3 of tile dt.
template <typename T, int D>
struct RowCols {
  using W = typename Wide<T, D>::W;
  const T* p;
  W x[kWide<T, D> ? 16 : 1];
  __device__ __forceinline__ RowCols(const T* row, int h) : p(row + 4 * h) {
    if constexpr (kWide<T, D>) {
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] = *reinterpret_cast<const W*>(row + Geo<D>::NDT * acc_row(v, h));
    }
  }
  __device__ __forceinline__ void get(int dt, int vq, float* z) const {
    if constexpr (kWide<T, D>) {
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = elem<T, D>(x[4 * vq + e], dt);
    } else {
      const Raw4<T> y = ld4(p + 32 * dt + 8 * vq);
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = y.at(e);
    }
  }
};
// Chunk ch of the lane's row at byte offset `off` (already at its half: + 4 h
// elements).
template <typename T, int D>
__device__ __forceinline__ RowChunk<T, D> load_rows(__amdgpu_buffer_rsrc_t b, int off, int ch) {
  RowChunk<T, D> r;
#pragma unroll
  for (int t = 0; t < Geo<D>::RC; ++t)
    r.x[t] = ldb4<T>(b, off + 8 * (ch * Geo<D>::RC + t) * static_cast<int>(sizeof(T)));
  return r;
}
// Tile dt of a transposed operand (kWide: every tile, with tile 0); `off` is the
// lane's offset at tile 0: 4 h rows and tr_col().
template <typename T, int D>
__device__ __forceinline__ void load_tr(TrChunk<T, D>& r, __amdgpu_buffer_rsrc_t b, int off, int rsb, int dt) {
  if (kWide<T, D> && dt > 0) return;
  asm volatile("" : "+v"(off));  // the sixteen offsets are formed here, not kept in registers
#pragma unroll
  for (int v = 0; v < 16; ++v)
    r.x[v] = ldw<T, D>(b, off + acc_row(v, 0) * rsb + 32 * dt * static_cast<int>(sizeof(T)));
}
// Byte offset of the lane's column in tile 0 (head_dim 16: the lanes past the
// row repeat it; their operand is set to 0).
template <typename T, int D>
__device__ __forceinline__ int tr_col(int c) {
  return (D < 32 ? c & (D - 1) : c) * static_cast<int>(sizeof(typename Wide<T, D>::W));
}

// bf16 operands are exact in bf16, and a float32 value is the sum of three bf16
// values (24 bits cut into 8, 8 and 8; the cuts toward zero are exact). So a
// product of bf16 data with float32 values (q~, P, dS, do~) is three bf16
// products of 16 contractions each: the same exact terms in float32 sums at
// 16 / 3 of the float32 products' rate. Infinities and NaN do not split (an
// infinity's remainder is NaN, and parts that are 0 turn an infinite operand
// into NaN): kernels whose sums come out non-finite walk their blocks again
// with float32 products. B=1 H=4 N=1024 D=128 w1=w2=128: forward and query side
// together 1.43 -> 0.92 ms, key side (do~ and q~ without scale, products of two
// bf16 values, times P and dS: two parts by three) 1.10 -> 0.77 ms; LSE against 64 bits 5.2e-8 -> 4.9e-8.
template <typename T>
constexpr bool kSplit = sizeof(T) == 2;
// (a product of two bf16 values is the sum of two parts)
template <int NP>
struct Parts8 {
  u32x4_t p[NP];
};
template <int NP = 3>
__device__ __forceinline__ Parts8<NP> split8(const float* x) {
  Parts8<NP> r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
      r.p[n][i] = __builtin_amdgcn_perm(ub, ua, 0x07060302);  // the upper halves
      a -= __uint_as_float(ua & 0xffff0000u);
      b -= __uint_as_float(ub & 0xffff0000u);
    }
  }
  return r;
}
template <int NP>
__device__ __forceinline__ f32x16_t mfma_parts(u32x4_t a, const Parts8<NP>& b, f32x16_t c) {
#pragma unroll
  for (int n = NP - 1; n >= 0; --n) c = mfma32(a, b.p[n], c);
  return c;
}
template <int NP>
__device__ __forceinline__ f32x16_t mfma_parts(const Parts8<NP>& a, u32x4_t b, f32x16_t c) {
#pragma unroll
  for (int n = NP - 1; n >= 0; --n) c = mfma32(a.p[n], b, c);
  return c;
}
// Operand of 16 contractions: float4s 2 u and 2 u + 1 of a row chunk, or rows
// 8 u .. 8 u + 7 (per lane half) of a transposed one.
template <typename T, int D>
__device__ __forceinline__ u32x4_t frag(const RowChunk<T, D>& r, int u) {
  if constexpr (kSplit<T>)
    return u32x4_t{r.x[2 * u].a[0], r.x[2 * u].a[1], r.x[2 * u + 1].a[0], r.x[2 * u + 1].a[1]};
  else
    return u32x4_t{};
}
template <typename T, int D>
__device__ __forceinline__ u32x4_t frag(const TrChunk<T, D>& r, int u, int dt) {
  u32x4_t y = {};
  if constexpr (kSplit<T>) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      y[e] = __builtin_amdgcn_perm(word<T, D>(r.x[8 * u + 2 * e + 1], dt), word<T, D>(r.x[8 * u + 2 * e], dt),
                                   kWide<T, D> && (dt & 1) ? 0x07060302 : 0x05040100);
  }
  return y;
}

// Sum / maximum over the 2^lw lanes (8, 16 or 32 of a half-wavefront) that hold
// the k-rows of one query; every lane gets it.
template <int LW, typename Op>
__device__ __forceinline__ float seg_reduce(float x, Op op) {
  x = op(x, dpp_f<0xB1>(x));
  x = op(x, dpp_f<0x4E>(x));
  x = op(x, dpp_f<0x141>(x));
  if constexpr (LW >= 4) x = op(x, dpp_f<0x140>(x));
  if constexpr (LW >= 5) {
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(p[0]), __uint_as_float(p[1]));
  }
  return x;
}
struct OpSum {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct OpMax {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
template <typename F>
__device__ __forceinline__ void with_lw(int lw, F f) {
  if (lw == 5)
    f(std::integral_constant<int, 5>{});
  else if (lw == 4)
    f(std::integral_constant<int, 4>{});
  else
    f(std::integral_constant<int, 3>{});
}

__device__ __forceinline__ bool nonfinite(float x) { return !(fabsf(x) < __builtin_inff()); }

// Whether a tile of products has an infinity or NaN: one in any operand row
// reaches every lane of it (its masked pairs multiply it by 0), so the products
// need no look at the operands. (Sums that overflow take the slow path too.)
__device__ __forceinline__ bool any_nonfinite(const f32x16_t& u) {
  float x = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) x += u[v];
  return __builtin_amdgcn_ballot_w64(nonfinite(x)) != 0;
}

// Whether any lane's `x` or accumulators do.
template <int N>
__device__ __forceinline__ bool nonfinite_sums(float x, const f32x16_t (&u)[N]) {
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int v = 0; v < 16; ++v) x += u[n][v];
  return __builtin_amdgcn_ballot_w64(nonfinite(x)) != 0;
}

// One accumulator tile of sum over the 32 contraction rows x of p[x] op[x][d],
// term by term and for the pairs with ok(x) only: the rare tile whose operand
// holds infinities or NaN in rows that are masked for some lanes. p:
// accumulator order; put through this wavefront's LDS scratch (32 x 33 floats)
// so that the loop stays rolled. row(x, d, y) gives the operand's four values
// at columns d .. d + 3 (of the tile) of row x.
template <int D, typename Ok, typename Row>
__device__ __forceinline__ f32x16_t masked_tile(const float* p, float* scratch, int c, int h, Ok ok, Row row) {
  f32x16_t u = {};
#pragma unroll
  for (int v = 0; v < 16; ++v) scratch[acc_row(v, h) * 33 + c] = p[v];
  __builtin_amdgcn_s_waitcnt(0xC07F);  // this wavefront's writes are in LDS
  __builtin_amdgcn_wave_barrier();
#pragma unroll 1
  for (int x = 0; x < 32; ++x) {
    const float px = scratch[x * 33 + c];
    const bool use = ok(x);
#pragma unroll
    for (int vq = 0; vq < Geo<D>::NV / 4; ++vq) {
      float y[4];
      row(x, 8 * vq + 4 * h, y);
#pragma unroll
      for (int e = 0; e < 4; ++e) u[4 * vq + e] += use ? px * y[e] : 0.f;
    }
  }
  __builtin_amdgcn_wave_barrier();
  return u;
}

// Work-item order: each of the 8 XCDs takes a contiguous run of `total`.
__device__ __forceinline__ long xcd_order(long total) {
  const long per = (total + 7) / 8;
  return static_cast<long>(blockIdx.x & 7) * per + (blockIdx.x >> 3);
}
unsigned xcd_grid(long total) { return static_cast<unsigned>((total + 7) / 8 * 8); }

// ---------------------------------------------------------------- forward ---
// A wavefront takes 32 >> lw consecutive queries (all their k-rows; groups of
// 32 k-rows in turn where w2 > 32) and walks their key window once per group:
// online softmax per row, then the log-sum-exp merge of a query's rows.
template <typename T, int D>
__global__ __launch_bounds__(kFThreads, D == 128 ? 1 : 2) void fwd_f32_kernel(
    Shape s, int lw, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ kp,
    const T* __restrict__ v, const T* __restrict__ vp, T* __restrict__ out, float* __restrict__ lse) {
  using Ge = Geo<D>;
  constexpr int NDT = Ge::NDT;
  __shared__ float scratch[kFWaves][kScratch];
  const int SP = 32 >> lw;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
  const int steps = (s.N + SP - 1) / SP;
  const long total = static_cast<long>(steps) * s.B * s.H;
  const long item = xcd_order((total + kFWaves - 1) / kFWaves) * kFWaves + wave;
  if (item >= total) return;
  const int bh = static_cast<int>(item / steps);
  const int i0 = static_cast<int>(item - static_cast<long>(bh) * steps) * SP;
  const int b = bh / s.H, hh = bh - b * s.H;
  const int N = s.N, w1 = s.w1, w2 = s.w2;
  const size_t rs = static_cast<size_t>(s.H) * D, rsk = static_cast<size_t>(s.Hkv) * D;
  const size_t base = (static_cast<size_t>(b) * N * s.H + hh) * D;
  const size_t basek = (static_cast<size_t>(b) * N * s.Hkv + hh / (s.H / s.Hkv)) * D;
  const float qscale = s.scale * kLog2e;
  const int i = i0 + (c >> lw);  // this lane's query
  const int lo = max(0, i - w1 + 1);
  const int jlo = max(0, i0 - w1 + 1), jhi = min(i0 + SP - 1, N - 1);  // window union
  const T* const kb = k + basek;
  const T* const vb = v + basek;
  const int rsb = static_cast<int>(rsk * sizeof(T));
  const int roff = c * rsb + 4 * h * static_cast<int>(sizeof(T)), toff = 4 * h * rsb + tr_col<T, D>(c);

  float M = -INFINITY, L = 0.f;  // merged over row groups, in log2 units
  float o[Ge::NV * NDT];
#pragma unroll
  for (int x = 0; x < Ge::NV * NDT; ++x) o[x] = 0.f;
  const int groups = lw == 5 ? (w2 + 31) / 32 : 1;
  for (int g = 0; g < groups; ++g) {
    const int t0 = (c & ((1 << lw) - 1)) + 32 * g;
    const int kk = i - t0;
    const bool rowvalid = i < N && t0 < w2 && kk >= 0;
    float m, l;
    f32x16_t acc[NDT];
    // The group's key window; `split`: float32 values as three bf16 parts.
    auto walk = [&](auto SPLIT) __attribute__((always_inline)) {
    constexpr bool split = decltype(SPLIT)::value;
    m = -INFINITY;
    l = 0.f;
    float qt[4 * Ge::NF];
    Parts8<3> qp[split ? Ge::NF / 2 : 1];
    {
      const T* qr = q + base + static_cast<size_t>(min(i, N - 1)) * rs + 4 * h;
      const T* kr = kp + basek + static_cast<size_t>(max(min(kk, N - 1), 0)) * rsk + 4 * h;
#pragma unroll
      for (int t = 0; t < Ge::NF; ++t) {
        const Raw4<T> a = ld4(qr + 8 * t), x = ld4(kr + 8 * t);
#pragma unroll
        for (int e = 0; e < 4; ++e) qt[4 * t + e] = rowvalid ? a.at(e) * qscale * (x.at(e) + s.kp_bias) : 0.f;
      }
      if constexpr (split) {
#pragma unroll
        for (int t = 0; t < Ge::NF / 2; ++t) qp[t] = split8(qt + 8 * t);
      }
    }
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) acc[dt] = f32x16_t{};
    __amdgpu_buffer_rsrc_t bk = rows_from<T, D>(kb, jlo, N, rsb);
    RowChunk<T, D> kc = load_rows<T, D>(bk, roff, 0);
    for (int jb = jlo; jb <= jhi; jb += 32) {
      const __amdgpu_buffer_rsrc_t bv = rows_from<T, D>(vb, jb, N, rsb);
      f32x16_t sc = {}, sc2 = {};
      TrChunk<T, D> vc;
#pragma unroll
      for (int ch = 0; ch < Ge::NRC; ++ch) {
        RowChunk<T, D> nx;
        if (ch + 1 < Ge::NRC)
          nx = load_rows<T, D>(bk, roff, ch + 1);
        else
          load_tr<T, D>(vc, bv, toff, rsb, 0);
        if constexpr (split) {
#pragma unroll
          for (int u = 0; u < Ge::RC / 2; ++u) sc = mfma_parts(frag<T, D>(kc, u), qp[ch * Ge::RC / 2 + u], sc);
        } else {
#pragma unroll
          for (int t = 0; t < Ge::RC; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              f32x16_t& chain = t & 1 ? sc2 : sc;
              chain = mfma_f32(kc.x[t].at(e), qt[4 * (ch * Ge::RC + t) + e], chain);
            }
        }
        kc = nx;
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (!split) sc += sc2;
      // Online softmax over this block's 32 keys (16 in each lane half).
      float p[16], mx = -INFINITY;
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) p[vv] = sc[vv];
      // Blocks with keys that not every query of the wavefront sees.
      const bool edge = jb < i0 + SP - w1 || jb + 31 > i0;
      if (edge) {
        asm volatile("" ::: "memory");  // a branch, not selects on every block
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) {
          const int j = jb + acc_row(vv, h);
          p[vv] = j >= lo && j <= i ? p[vv] : -INFINITY;
        }
      }
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) mx = fmaxf(mx, p[vv]);
      const float mn = fmaxf(m, fmaxf(mx, swap_halves(mx)));
      const float mu = mn == -INFINITY ? 0.f : mn;  // no key of the row's window so far
      const float alpha = fast_exp2(m - mu);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) {
        p[vv] = fast_exp2(p[vv] - mu);
        l += p[vv];
      }
      bk = rows_from<T, D>(kb, jb + 32, N, rsb);  // the next block's
      Parts8<3> pp[split ? 2 : 1];
      if constexpr (split) pp[0] = split8(p), pp[1] = split8(p + 8);
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const TrChunk<T, D> cur = vc;
        if (dt + 1 < NDT)
          load_tr<T, D>(vc, bv, toff, rsb, dt + 1);
        else
          kc = load_rows<T, D>(bk, roff, 0);
        f32x16_t u = {};
        if constexpr (split) {
#pragma unroll
          for (int n = 0; n < 2; ++n)
            u = mfma_parts(D >= 32 || c < D ? frag<T, D>(cur, n, dt) : u32x4_t{}, pp[n], u);
        } else {
#pragma unroll
          for (int vv = 0; vv < 16; ++vv) {
            const float y = elem<T, D>(cur.x[vv], dt);
            u = mfma_f32(D >= 32 || c < D ? y : 0.f, p[vv], u);
          }
        }
        if (!split && edge && any_nonfinite(u))
          u = masked_tile<D>(
              p, scratch[wave], c, h, [&](int x) { return jb + x >= lo && jb + x <= i; },
              [&](int x, int d, float* y) {
                ldcols<T, D>(bv, x * rsb, dt, d, y);
              });
        acc[dt] = acc[dt] * alpha + u;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    };
    walk(std::bool_constant<kSplit<T>>{});
    if constexpr (kSplit<T>) {
      if (nonfinite_sums(l, acc)) walk(std::false_type{});
    }
    // Merge this group's rows into the query's O, M, L.
    const float lsum = l + swap_halves(l);
    const RowCols<T, D> vr(vp + basek + static_cast<size_t>(max(min(kk, N - 1), 0)) * rsk, h);
    with_lw(lw, [&](auto LC) __attribute__((always_inline)) {
      constexpr int LW = decltype(LC)::value;
      const float mg = seg_reduce<LW>(rowvalid ? m : -INFINITY, OpMax());
      const float mn = fmaxf(M, mg), mu = mn == -INFINITY ? 0.f : mn;
      const float a = fast_exp2(M - mu), w = fast_exp2(m - mu);
      M = mn;
      L = L * a + seg_reduce<LW>(rowvalid ? w * lsum : 0.f, OpSum());
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
#pragma unroll
        for (int vq = 0; vq < Ge::NV / 4; ++vq) {
          float y[4];
          vr.get(dt, vq, y);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = rowvalid ? w * (y[e] + s.vp_bias) * acc[dt][4 * vq + e] : 0.f;
            float& oo = o[Ge::NV * dt + 4 * vq + e];
            oo = oo * a + seg_reduce<LW>(x, OpSum());
          }
        }
        __builtin_amdgcn_sched_barrier(0);  // no more of the v' loads in registers at once
      }
    });
  }
  if (i < N && (c & ((1 << lw) - 1)) == 0) {
    T* dst = out + base + static_cast<size_t>(i) * rs;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int vv = 0; vv < Ge::NV; ++vv) st1(dst + column<T, D>(dt, acc_row(vv, h)), o[Ge::NV * dt + vv] / L);
    // ln 2 in two parts: the product with M is not rounded before the sum
    if (h == 0) lse[static_cast<size_t>(bh) * N + i] = __builtin_fmaf(M, kLn2, __builtin_fmaf(M, kLn2Lo, logf(L)));
  }
}

// ------------------------------------------------------------- query side ---
// dQ, dK', dV' for w2 <= 128. A workgroup walks a chunk of CQ consecutive
// queries. Its four wavefronts are `groups` row groups of 32 k-rows times QS
// query slots of 32 >> lw consecutive queries: each accumulates dQ~^T = K^T dS^T
// and U~^T = V^T P^T of its rows over their key window. The sums leave the
// registers once per step: dq over the rows (lane reductions, then the groups
// in order through LDS), q_i o dQ~ and dO_i o U~ into a float32 LDS ring of
// k-rows, in QS phases of column slices so that the slots add in a fixed order.
// k-rows no later query of the chunk sees are written out; the rows before a
// chunk boundary are partial sums for the fix-up kernel. Where a head has too
// few queries for chunks of W2T to fill the chip (plan.full) the chunks are
// shorter than the k-row window, and every k-row leaves as a partial sum.
template <typename T, int D, bool BIAS>
__global__ __launch_bounds__(kFThreads, D == 128 ? 1 : 2) void bwd_query_f32_kernel(
    Shape s, F32Plan plan, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ kp,
    const T* __restrict__ v, const T* __restrict__ vp, const T* __restrict__ dout,
    const float* __restrict__ lse, const float* __restrict__ delta, T* __restrict__ dq, T* __restrict__ dkp,
    T* __restrict__ dvp, float* __restrict__ ws) {
  using Ge = Geo<D>;
  constexpr int NDT = Ge::NDT, RS = D + 4;
  // Per wavefront kScratch floats (masked_tile's, or its dq rows at the end of a
  // step), then the rings (as many rows as w2 asks for).
  extern __shared__ __attribute__((aligned(16))) float f32_lds[];
  static_assert(4 * D <= kScratch, "dq rows of a step");
  float* const dqx = f32_lds;
  float* const ring = f32_lds + kFWaves * kScratch;
  const int lw = plan.lw, SP = 32 >> lw, WT = plan.W2T;
  const int groups = plan.groups, QS = plan.qs, SQ = QS * SP;  // queries per step
  const int RB = WT + SQ;
  float* const ring_k = ring;
  float* const ring_v = ring + RB * RS;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, c = lane & 31, h = lane >> 5;
  const int g = wave % groups, slot = wave / groups;
  const bool busy = slot < QS;
  const long total = static_cast<long>(plan.nchunks) * s.B * s.H;
  const long item = xcd_order(total);
  if (item >= total) return;
  const int bh = static_cast<int>(item / plan.nchunks), chunk = static_cast<int>(item % plan.nchunks);
  const int b = bh / s.H, hh = bh - b * s.H;
  const int N = s.N, w1 = s.w1, w2 = s.w2;
  const int cs = chunk * plan.CQ, ce = min(N, cs + plan.CQ);
  const size_t rs = static_cast<size_t>(s.H) * D;
  const size_t base = (static_cast<size_t>(b) * N * s.H + hh) * D;
  const size_t stat = static_cast<size_t>(bh) * N;
  const float qscale = s.scale * kLog2e;
  const T* const kb = k + base;
  const T* const vb = v + base;
  const int rsb = static_cast<int>(rs * sizeof(T));
  const int roff = c * rsb + 4 * h * static_cast<int>(sizeof(T)), toff = 4 * h * rsb + tr_col<T, D>(c);
  float* const scratch = f32_lds + wave * kScratch;

  for (int x = tid; x < 2 * RB * RS; x += kFThreads) ring[x] = 0.f;
  __syncthreads();

  const size_t halo = static_cast<size_t>(WT - 1) * D;
  float* const hk = ws + (static_cast<size_t>(bh) * plan.nchunks + chunk) * halo;
  float* const pk = ws + (static_cast<size_t>(bh) * plan.nchunks + chunk) * static_cast<size_t>(plan.CQ + WT - 1) * D;
  auto flush_rows = [&](int klo, int khi, bool last) {  // k-rows klo .. khi
    const int n = khi - klo + 1;
    for (int x = tid; x < n * D; x += kFThreads) {
      const int kr = klo + x / D, d = x % D;
      const int row = (kr + WT) % RB;
      float* a = ring_k + row * RS + place<T, D>(d);
      float* y = ring_v + row * RS + place<T, D>(d);
      if (kr >= 0) {
        if (plan.full) {
          const size_t at = static_cast<size_t>(kr - (cs - WT + 1)) * D + d;
          pk[at] = *a;
          pk[at + plan.halo_floats] = *y;
        } else if (kr < cs) {  // head partial
          const size_t at = static_cast<size_t>(kr - (cs - WT + 1)) * D + d;
          hk[at] = *a;
          hk[at + plan.halo_floats] = *y;
        } else if (last && ce < N) {  // tail partial
          const size_t at = static_cast<size_t>(kr - (ce - WT + 1)) * D + d;
          hk[at + 2 * plan.halo_floats] = *a;
          hk[at + 3 * plan.halo_floats] = *y;
        } else {
          st1(dkp + base + static_cast<size_t>(kr) * rs + d, *a * s.scale);
          st1(dvp + base + static_cast<size_t>(kr) * rs + d, *y);
        }
      }
      *a = 0.f;
      *y = 0.f;
    }
  };

  for (int ib = cs; ib < ce; ib += SQ) {
    const int i0 = ib + slot * SP;  // first query of this wavefront
    const int i = i0 + (c >> lw);
    const int t0 = (c & ((1 << lw) - 1)) + 32 * g;
    const int kk = i - t0;
    const bool rowvalid = busy && i < ce && t0 < w2 && kk >= 0;
    const int lo = max(0, i - w1 + 1);
    const int jlo = max(0, i0 - w1 + 1), jhi = min(i0 + SP - 1, N - 1);
    const int ic = min(i, N - 1), kc_ = max(min(kk, N - 1), 0);
    f32x16_t au[NDT], aq[NDT];
    // The rows' key window; `split`: float32 values as three bf16 parts.
    auto walk = [&](auto SPLIT) __attribute__((always_inline)) {
    constexpr bool split = decltype(SPLIT)::value, FLY = D >= 64 && !split;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      au[dt] = f32x16_t{};
      aq[dt] = f32x16_t{};
    }
    if (busy && i0 < ce) {
      const Norm norm(lse[stat + ic]);
      const float dlt = delta[stat + ic];
      // q~ and do~ of the lane's row: in registers, or (FLY) formed again for
      // every block from rows that stay in L1 / L2.
      const __amdgpu_buffer_rsrc_t bq = rows_from<T, D>(q + base, i0, N, rsb), bg = rows_from<T, D>(dout + base, i0, N, rsb);
      const int k0 = max(0, i0 - WT + 1);
      const __amdgpu_buffer_rsrc_t bkp = rows_from<T, D>(kp + base, k0, N, rsb), bvp = rows_from<T, D>(vp + base, k0, N, rsb);
      const int ro = (c >> lw) * rsb + 4 * h * static_cast<int>(sizeof(T));
      const int ko = rowvalid ? (kk - k0) * rsb + 4 * h * static_cast<int>(sizeof(T)) : kFar;
      float qt[FLY || split ? 1 : 4 * Ge::NF], ot[FLY || split ? 1 : 4 * Ge::NF];
      Parts8<3> qp[split ? Ge::NF / 2 : 1];
      Parts8<BIAS ? 3 : 2> op[split ? Ge::NF / 2 : 1];
      // (a row outside the window or the sequence loads k', v' as zeros; its S
      // and dP are masked below)
      auto form = [&](const RowChunk<T, D>& a, const RowChunk<T, D>& x, bool scaled, float bias, float* y) {
#pragma unroll
        for (int t = 0; t < Ge::RC; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            y[4 * t + e] = (scaled ? a.x[t].at(e) * qscale : a.x[t].at(e)) * plus_bias<BIAS>(x.x[t].at(e), bias);
      };
      if constexpr (split) {
#pragma unroll
        for (int ch = 0; ch < Ge::NRC; ++ch) {
          float y[4 * Ge::RC];
          form(load_rows<T, D>(bq, ro, ch), load_rows<T, D>(bkp, ko, ch), true, s.kp_bias, y);
#pragma unroll
          for (int u = 0; u < Ge::RC / 2; ++u) qp[ch * Ge::RC / 2 + u] = split8(y + 8 * u);
          form(load_rows<T, D>(bg, ro, ch), load_rows<T, D>(bvp, ko, ch), false, s.vp_bias, y);
#pragma unroll
          for (int u = 0; u < Ge::RC / 2; ++u) op[ch * Ge::RC / 2 + u] = split8<BIAS ? 3 : 2>(y + 8 * u);
        }
      } else if constexpr (!FLY) {
#pragma unroll
        for (int ch = 0; ch < Ge::NRC; ++ch) {
          form(load_rows<T, D>(bq, ro, ch), load_rows<T, D>(bkp, ko, ch), true, s.kp_bias, qt + 4 * Ge::RC * ch);
          form(load_rows<T, D>(bg, ro, ch), load_rows<T, D>(bvp, ko, ch), false, s.vp_bias, ot + 4 * Ge::RC * ch);
        }
      }
      __amdgpu_buffer_rsrc_t bk = rows_from<T, D>(kb, jlo, N, rsb);
      RowChunk<T, D> rc = load_rows<T, D>(bk, roff, 0), fa, fm;
      if constexpr (FLY) {
        fa = load_rows<T, D>(bq, ro, 0);
        fm = load_rows<T, D>(bkp, ko, 0);
      }
      for (int jb = jlo; jb <= jhi; jb += 32) {
        const __amdgpu_buffer_rsrc_t bv = rows_from<T, D>(vb, jb, N, rsb);
        // S^T and dP^T
        f32x16_t sc = {}, dp = {};
        TrChunk<T, D> tc;
#pragma unroll
        for (int ph = 0; ph < 2; ++ph) {
#pragma unroll
          for (int ch = 0; ch < Ge::NRC; ++ch) {
            float y[4 * Ge::RC];
            if constexpr (FLY) {
              form(fa, fm, ph == 0, ph ? s.vp_bias : s.kp_bias, y);
            } else if constexpr (!split) {
#pragma unroll
              for (int e = 0; e < 4 * Ge::RC; ++e) y[e] = (ph ? ot : qt)[4 * Ge::RC * ch + e];
            }
            const RowChunk<T, D> cur = rc;
            const int nch = ch + 1 < Ge::NRC ? ch + 1 : 0;
            const bool second = ph == 1 || nch == 0;  // the next chunk is dP's
            if (ph == 1 && nch == 0) {
              load_tr<T, D>(tc, bv, toff, rsb, 0);
            } else {
              rc = load_rows<T, D>(second ? bv : bk, roff, nch);
              if constexpr (FLY) {
                fa = load_rows<T, D>(second ? bg : bq, ro, nch);
                fm = load_rows<T, D>(second ? bvp : bkp, ko, nch);
              }
            }
            if constexpr (split) {
              f32x16_t& acc = ph ? dp : sc;
#pragma unroll
              for (int u = 0; u < Ge::RC / 2; ++u)
                acc = ph ? mfma_parts(frag<T, D>(cur, u), op[ch * Ge::RC / 2 + u], acc)
                         : mfma_parts(frag<T, D>(cur, u), qp[ch * Ge::RC / 2 + u], acc);
            } else {
#pragma unroll
              for (int t = 0; t < Ge::RC; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  f32x16_t& acc = ph || (t & 1) ? dp : sc;  // S: its second chain
                  acc = mfma_f32(cur.x[t].at(e), y[4 * t + e], acc);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          if (!split && ph == 0) {
            sc += dp;
            dp = f32x16_t{};
          }
        }
        float p[16], ds[16];
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) {
          const int j = jb + acc_row(vv, h);
          const bool ok = rowvalid && j >= lo && j <= i;
          const float e = prob(sc[vv], norm);
          p[vv] = ok ? e : 0.f;
          ds[vv] = ok ? e * (dp[vv] - dlt) : 0.f;
        }
        // Keys that only some of the step's queries see: see masked_tile.
        const bool edge = jb < i0 + SP - w1 || jb + 31 > i0;  // keys that not every query sees
        // U~^T += V^T P^T, dQ~^T += K^T dS^T
        const __amdgpu_buffer_rsrc_t bkc = bk;  // this block's (bk moves on below)
        Parts8<3> pp[split ? 2 : 1], dsp[split ? 2 : 1];
        if constexpr (split) pp[0] = split8(p), pp[1] = split8(p + 8), dsp[0] = split8(ds), dsp[1] = split8(ds + 8);
#pragma unroll
        for (int x = 0; x < 2 * NDT; ++x) {
          const int dt = x % NDT;
          const TrChunk<T, D> cur = tc;
          if (x + 1 < 2 * NDT) {
            load_tr<T, D>(tc, x + 1 < NDT ? bv : bkc, toff, rsb, (x + 1) % NDT);
          } else {
            bk = rows_from<T, D>(kb, jb + 32, N, rsb);
            rc = load_rows<T, D>(bk, roff, 0);
            if constexpr (FLY) {
              fa = load_rows<T, D>(bq, ro, 0);
              fm = load_rows<T, D>(bkp, ko, 0);
            }
          }
          f32x16_t u = {};
          if constexpr (split) {
#pragma unroll
            for (int n = 0; n < 2; ++n)
              u = mfma_parts(D >= 32 || c < D ? frag<T, D>(cur, n, dt) : u32x4_t{}, (x < NDT ? pp : dsp)[n], u);
          } else {
#pragma unroll
            for (int vv = 0; vv < 16; ++vv) {
              const float y = elem<T, D>(cur.x[vv], dt);
              u = mfma_f32(D >= 32 || c < D ? y : 0.f, x < NDT ? p[vv] : ds[vv], u);
            }
          }
          if (!split && edge && any_nonfinite(u))
            u = masked_tile<D>(
                x < NDT ? p : ds, scratch, c, h, [&](int y) { return rowvalid && jb + y >= lo && jb + y <= i; },
                [&](int y, int d, float* z) {
                  ldcols<T, D>(x < NDT ? bv : bkc, y * rsb, dt, d, z);
                });
          if (x < NDT)
            au[dt] += u;
          else
            aq[dt] += u;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    };
    walk(std::bool_constant<kSplit<T>>{});
    if constexpr (kSplit<T>) {
      if (nonfinite_sums(0.f, au) || nonfinite_sums(0.f, aq)) walk(std::false_type{});
    }
    // ---- end of the step: dq, then the k-row contributions ----
    if (busy) {
      const RowCols<T, D> kr(kp + base + static_cast<size_t>(kc_) * rs, h);
      float* dst = dqx + wave * kScratch + (c >> lw) * D;
      with_lw(lw, [&](auto LC) __attribute__((always_inline)) {
        constexpr int LW = decltype(LC)::value;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
#pragma unroll
          for (int vq = 0; vq < Ge::NV / 4; ++vq) {
            const int d = 32 * dt + 8 * vq + 4 * h;
            float y[4];
            kr.get(dt, vq, y);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float x =
                  seg_reduce<LW>(rowvalid ? (y[e] + s.kp_bias) * aq[dt][4 * vq + e] : 0.f, OpSum());
              if ((c & ((1 << LW) - 1)) == 0) dst[d + e] = x;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    }
    // Phase ph: slot adds column tiles dt (head_dim 128), or quarters / halves of
    // them, whose number is (slot + ph) % QS.
    const int row = max(kk + WT, 0) % RB;
    const RowCols<T, D> qr(q + base + static_cast<size_t>(ic) * rs, h), gr(dout + base + static_cast<size_t>(ic) * rs, h);
    for (int ph = 0; ph < QS; ++ph) {
      const int sl = (slot + ph) & (QS - 1);
      for (int st = 0; st < SP; ++st) {  // a k-row belongs to one lane per query
        if (rowvalid && (c >> lw) == st) {
#pragma unroll
          for (int dt = 0; dt < NDT; ++dt) {
#pragma unroll
            for (int vq = 0; vq < Ge::NV / 4; ++vq) {
              if (((NDT * vq + dt) & (QS - 1)) != sl) continue;
              const int d = 32 * dt + 8 * vq + 4 * h;
              float x[4], y[4];
              qr.get(dt, vq, x);
              gr.get(dt, vq, y);
              float4* a = reinterpret_cast<float4*>(ring_k + row * RS + d);
              float4* z = reinterpret_cast<float4*>(ring_v + row * RS + d);
              float4 av = *a, zv = *z;
              av.x += x[0] * aq[dt][4 * vq], av.y += x[1] * aq[dt][4 * vq + 1];
              av.z += x[2] * aq[dt][4 * vq + 2], av.w += x[3] * aq[dt][4 * vq + 3];
              zv.x += y[0] * au[dt][4 * vq], zv.y += y[1] * au[dt][4 * vq + 1];
              zv.z += y[2] * au[dt][4 * vq + 2], zv.w += y[3] * au[dt][4 * vq + 3];
              *a = av;
              *z = zv;
            }
          }
        }
        __builtin_amdgcn_wave_barrier();
      }
      __syncthreads();
    }
    for (int x = tid; x < SQ * D; x += kFThreads) {
      const int qi = x / D, d = x % D;
      if (ib + qi < ce) {
        float sum = 0.f;
        for (int gg = 0; gg < groups; ++gg) sum += dqx[((qi / SP) * groups + gg) * kScratch + (qi % SP) * D + place<T, D>(d)];
        st1(dq + base + static_cast<size_t>(ib + qi) * rs + d, sum * s.scale);
      }
    }
    flush_rows(ib - WT + 1, min(ib + SQ, ce) - WT, false);
    __syncthreads();
  }
  flush_rows(ce - WT + 1, ce - 1, true);
}

// dk', dv' of the k-rows that left the query side as partial sums, added in the
// order of the chunks. Chunks of at least W2T queries: the W2T - 1 rows before
// each boundary, tail of chunk c - 1 plus head of chunk c. plan.full: every row,
// over the chunks whose queries see it (up to W2T of them: eight loads in flight).
template <typename T>
__global__ __launch_bounds__(256) void fixup_f32_kernel(Shape s, F32Plan plan, const float* __restrict__ ws,
                                                        T* __restrict__ dkp, T* __restrict__ dvp) {
  const long idx = static_cast<long>(blockIdx.x) * 256 + threadIdx.x;
  const int W1 = plan.W2T - 1;
  int bh, kr, d;
  float a, y;
  if (plan.full) {
    const long row = idx / s.D;
    if (row >= static_cast<long>(s.B) * s.H * s.N) return;
    d = static_cast<int>(idx % s.D);
    bh = static_cast<int>(row / s.N);
    kr = static_cast<int>(row % s.N);
    const size_t per = static_cast<size_t>(plan.CQ + W1) * s.D;
    a = y = 0.f;
#pragma unroll 8
    for (int c = kr / plan.CQ; c <= min(plan.nchunks - 1, (kr + W1) / plan.CQ); ++c) {
      const float* p = ws + (static_cast<size_t>(bh) * plan.nchunks + c) * per +
                       static_cast<size_t>(kr - (c * plan.CQ - W1)) * s.D + d;
      a += p[0];
      y += p[plan.halo_floats];
    }
  } else {
    const long per = static_cast<long>(W1) * s.D;
    const long bound = idx / per, rem = idx - bound * per;
    if (bound >= static_cast<long>(s.B) * s.H * (plan.nchunks - 1)) return;
    bh = static_cast<int>(bound / (plan.nchunks - 1));
    const int cb = static_cast<int>(bound % (plan.nchunks - 1)) + 1;  // chunk after the boundary
    kr = cb * plan.CQ - W1 + static_cast<int>(rem / s.D);
    d = static_cast<int>(rem % s.D);
    const float* head = ws + (static_cast<size_t>(bh) * plan.nchunks + cb) * per + rem;
    const float* tail = ws + (static_cast<size_t>(bh) * plan.nchunks + cb - 1) * per + rem + 2 * plan.halo_floats;
    a = tail[0] + head[0];
    y = tail[plan.halo_floats] + head[plan.halo_floats];
  }
  const size_t dst = ((static_cast<size_t>(bh / s.H) * s.N + kr) * s.H + bh % s.H) * s.D + d;
  st1(dkp + dst, a * s.scale);
  st1(dvp + dst, y);
}

// --------------------------------------------------------------- key side ---
// dK, dV. A workgroup owns 32 keys (one per lane; K and V as LDS operands) and
// its wavefronts share out the row blocks (32 >> lw queries times 2^lw k-rows)
// whose windows reach them: S = q~ K^T, dP = do~ V^T,
// dV^T += do~^T P, dK^T += q~^T dS, the row operands formed from q, k', dO, v'
// as they arrive. Their sums are added in order through LDS.
template <int D>
constexpr int key_waves() {
  return D == 128 ? 4 : 8;  // head_dim 128 takes more than 256 registers
}
template <typename T, int D, bool BIAS>
__global__ __launch_bounds__(64 * key_waves<D>(), 1) void bwd_key_f32_kernel(
    Shape s, int lw, int ks, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ kp,
    const T* __restrict__ v, const T* __restrict__ vp, const T* __restrict__ dout,
    const float* __restrict__ lse, const float* __restrict__ delta, T* __restrict__ dk, T* __restrict__ dv,
    float* __restrict__ part) {
  using Ge = Geo<D>;
  using W = typename Wide<T, D>::W;
  constexpr int NDT = Ge::NDT, RS = D + 4, KW = key_waves<D>();
  // K and V operands, then masked_tile scratch; at the end the wavefronts' sums.
  constexpr int kPer = kSplit<T> ? 2 : 1;  // float4s of an operand in 16 bytes
  constexpr int kOps = 2 * 32 * D, kScr = KW * kScratch, kSum = KW * 32 * RS;
  __shared__ __attribute__((aligned(16))) float lds[kSum > kOps + kScr ? kSum : kOps + kScr];
  const int SP = 32 >> lw;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
  const int jblocks = (s.N + 31) / 32;
  const long total = static_cast<long>(jblocks) * ks * s.B * s.H;
  const long item = xcd_order(total);
  if (item >= total) return;
  const int sp = static_cast<int>(item % ks);
  const long jb = item / ks;
  const int bh = static_cast<int>(jb / jblocks), j0 = static_cast<int>(jb % jblocks) * 32;
  const int b = bh / s.H, hh = bh - b * s.H;
  const int N = s.N, w1 = s.w1, w2 = s.w2;
  const size_t rs = static_cast<size_t>(s.H) * D;
  const size_t base = (static_cast<size_t>(b) * N * s.H + hh) * D;
  const size_t stat = static_cast<size_t>(bh) * N;
  const float qscale = s.scale * kLog2e;
  const T *const qb = q + base, *const kpb = kp + base, *const gb = dout + base, *const vpb = vp + base;
  const int j = j0 + c;
  const int rsb = static_cast<int>(rs * sizeof(T));

  // K and V rows as operands, in the order the products take them: float4 t of
  // lane (h, c) (key j0 + c, columns 8 t + 4 h .. + 3) at 64 t + lane; bf16: 2 t
  // and 2 t + 1 there (frag's order).
  u32x4_t* const opk = reinterpret_cast<u32x4_t*>(lds) + lane;
  u32x4_t* const opv = opk + 64 * Ge::NF;
  {
    const __amdgpu_buffer_rsrc_t rk = rows_from<T, D>(k + base, j0, N, rsb), rv = rows_from<T, D>(v + base, j0, N, rsb);
    const int off = c * rsb + 4 * h * static_cast<int>(sizeof(T));
    for (int t = wave; t < Ge::NF / kPer; t += KW) {
      Raw4<T> a[kPer], y[kPer];
#pragma unroll
      for (int n = 0; n < kPer; ++n) {
        a[n] = ldb4<T>(rk, off + 8 * (kPer * t + n) * static_cast<int>(sizeof(T)));
        y[n] = ldb4<T>(rv, off + 8 * (kPer * t + n) * static_cast<int>(sizeof(T)));
      }
      opk[64 * t] = __builtin_bit_cast(u32x4_t, a);
      opv[64 * t] = __builtin_bit_cast(u32x4_t, y);
    }
  }
  __syncthreads();
  // Element e of float4 t of such an operand.
  auto op_at = [&](const u32x4_t& w, int t, int e) {
    if constexpr (kSplit<T>)
      return Raw4<uint16_t>{u32x2_t{w[2 * (t & 1)], w[2 * (t & 1) + 1]}}.at(e);
    else
      return __uint_as_float(w[e]);
  };
  f32x16_t ak[NDT], av[NDT];
  // The row blocks of the key window; `split`: float32 values as bf16 parts.
  auto walk = [&](auto SPLIT) __attribute__((always_inline)) {
  constexpr bool split = decltype(SPLIT)::value;
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt) {
    ak[dt] = f32x16_t{};
    av[dt] = f32x16_t{};
  }
  const int i_end = static_cast<int>(min(static_cast<long>(N), static_cast<long>(j0) + 31 + w1));
  const int groups = lw == 5 ? (w2 + 31) / 32 : 1;
  const int nrb = (i_end - j0 + SP - 1) / SP * groups;
  for (int rb = sp * KW + wave; rb < nrb; rb += ks * KW) {
    const int g = rb % groups, i0 = j0 + rb / groups * SP;
    if (i0 + SP - 1 < 32 * g) continue;  // every k of the block is before the sequence
    // Row r of the block: query i0 + st, k-row that minus t, st = r >> lw and
    // t = r % 2^lw + 32 g. The pair exists for t < lim(st): k-rows in the w2
    // window and the sequence, queries that see the keys.
    const int tmask = (1 << lw) - 1;
    auto lim = [&](int st) { return i0 + st < i_end ? min(w2, i0 + st + 1) : 0; };
    auto tof = [&](int r) { return (r & tmask) + 32 * g; };
    // Row acc_row(4 vq + e, h): the query does not depend on the lane half, and
    // t = tq[vq] + e + 4 h.
    int tq[4], room[4];
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      tq[vq] = ((8 * vq) & tmask) + 32 * g;
      room[vq] = lim((8 * vq) >> lw) - tq[vq];
    }
    auto okr = [&](int vv) { return 4 * h < room[vv >> 2] - (vv & 3); };
    const int k0 = max(0, i0 - tmask - 32 * g);  // first k-row of the block
    const __amdgpu_buffer_rsrc_t bq = rows_from<T, D>(qb, i0, N, rsb), bg = rows_from<T, D>(gb, i0, N, rsb);
    const __amdgpu_buffer_rsrc_t bkp = rows_from<T, D>(kpb, k0, N, rsb), bvp = rows_from<T, D>(vpb, k0, N, rsb);
    const bool okc = tof(c) < lim(c >> lw);
    const int ro = (c >> lw) * rsb + 4 * h * static_cast<int>(sizeof(T));
    const int ko = okc ? (i0 + (c >> lw) - tof(c) - k0) * rsb + 4 * h * static_cast<int>(sizeof(T)) : kFar;
    f32x16_t sc = {}, dp = {};
    RowChunk<T, D> a = load_rows<T, D>(bq, ro, 0), m = load_rows<T, D>(bkp, ko, 0);
#pragma unroll
    for (int ch = 0; ch < Ge::NRC; ++ch) {
      const RowChunk<T, D> na = ch + 1 < Ge::NRC ? load_rows<T, D>(bq, ro, ch + 1) : load_rows<T, D>(bg, ro, 0);
      const RowChunk<T, D> nm = ch + 1 < Ge::NRC ? load_rows<T, D>(bkp, ko, ch + 1) : load_rows<T, D>(bvp, ko, 0);
      float x[4 * Ge::RC];
#pragma unroll
      for (int t = 0; t < Ge::RC; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x[4 * t + e] = a.x[t].at(e) * qscale * plus_bias<BIAS>(m.x[t].at(e), s.kp_bias);
      if constexpr (split) {
#pragma unroll
        for (int u = 0; u < Ge::RC / 2; ++u)
          sc = mfma_parts(split8(x + 8 * u), opk[64 * (ch * Ge::RC / 2 + u)], sc);
      } else {
#pragma unroll
        for (int t = 0; t < Ge::RC; ++t) {
          const u32x4_t w = opk[64 * ((ch * Ge::RC + t) / kPer)];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            f32x16_t& chain = t & 1 ? dp : sc;
            chain = mfma_f32(x[4 * t + e], op_at(w, t, e), chain);
          }
        }
      }
      a = na;
      m = nm;
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!split) {
      sc += dp;
      dp = f32x16_t{};
    }
    // Transposed operands: rows acc_row(v, h) of q / dO (their query's) and of
    // k' / v' (zero rows outside the sequence).
    auto load_q = [&](__amdgpu_buffer_rsrc_t bb, int dt, W* r) __attribute__((always_inline)) {
      if (kWide<T, D> && dt > 0) return;
      int off = tr_col<T, D>(c);
      asm volatile("" : "+v"(off));
#pragma unroll
      for (int vq = 0; vq < 4; ++vq)  // eight rows share a query
        r[vq] = ldw<T, D>(bb, off + ((8 * vq) >> lw) * rsb + 32 * dt * static_cast<int>(sizeof(T)));
    };
    auto load_k = [&](__amdgpu_buffer_rsrc_t bb, int dt, TrChunk<T, D>& r) __attribute__((always_inline)) {
      if (kWide<T, D> && dt > 0) return;
      int off = tr_col<T, D>(c) - 4 * h * rsb;
      asm volatile("" : "+v"(off));  // the sixteen offsets are formed here, not kept in registers
#pragma unroll
      for (int v = 0; v < 16; ++v)
        r.x[v] = ldw<T, D>(bb, off + (i0 - k0 + ((8 * (v >> 2)) >> lw) - tq[v >> 2] - (v & 3)) * rsb +
                                   32 * dt * static_cast<int>(sizeof(T)));
    };
    W ta[4];
    TrChunk<T, D> tm;
#pragma unroll
    for (int ch = 0; ch < Ge::NRC; ++ch) {
      RowChunk<T, D> na, nm;
      if (ch + 1 < Ge::NRC) {
        na = load_rows<T, D>(bg, ro, ch + 1);
        nm = load_rows<T, D>(bvp, ko, ch + 1);
      } else {
        load_q(bg, 0, ta);
        load_k(bvp, 0, tm);
      }
      float x[4 * Ge::RC];
#pragma unroll
      for (int t = 0; t < Ge::RC; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * t + e] = a.x[t].at(e) * plus_bias<BIAS>(m.x[t].at(e), s.vp_bias);
      if constexpr (split) {
#pragma unroll
        for (int u = 0; u < Ge::RC / 2; ++u)
          dp = mfma_parts(split8<BIAS ? 3 : 2>(x + 8 * u), opv[64 * (ch * Ge::RC / 2 + u)], dp);
      } else {
#pragma unroll
        for (int t = 0; t < Ge::RC; ++t) {
          const u32x4_t w = opv[64 * ((ch * Ge::RC + t) / kPer)];
#pragma unroll
          for (int e = 0; e < 4; ++e) dp = mfma_f32(x[4 * t + e], op_at(w, t, e), dp);
        }
      }
      a = na;
      m = nm;
      __builtin_amdgcn_sched_barrier(0);
    }
    float p[16], ds[16];
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      const int i = i0 + ((8 * vq) >> lw);  // eight rows share a query
      const Norm norm(lse[stat + min(i, N - 1)]);
      const float dlt = delta[stat + min(i, N - 1)];
      const bool okj = j <= i && j > i - w1 && j < N;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int vv = 4 * vq + e;
        const bool ok = okj && okr(vv);
        const float x = prob(sc[vv], norm);
        p[vv] = ok ? x : 0.f;
        ds[vv] = ok ? x * (dp[vv] - dlt) : 0.f;
      }
    }
    // Row blocks with rows that not all of the 32 keys see, or (w2 not filling
    // them, the start of the sequence) that are no pair's.
    const bool edge = i0 < j0 + 31 || i0 + SP - 1 - w1 >= j0 || j0 + 32 > N || room[0] < 8 || room[1] < 8 ||
                      room[2] < 8 || room[3] < 8;
    auto seen = [&](int r) {
      const int i = i0 + (r >> lw);
      return tof(r) < lim(r >> lw) && j <= i && j > i - w1 && j < N;
    };
    Parts8<3> pp[split ? 2 : 1], dsp[split ? 2 : 1];
    if constexpr (split) pp[0] = split8(p), pp[1] = split8(p + 8), dsp[0] = split8(ds), dsp[1] = split8(ds + 8);
    // dV^T += do~^T P, dK^T += q~^T dS (unscaled q~)
#pragma unroll
    for (int x = 0; x < 2 * NDT; ++x) {
      const int dt = x % NDT;
      const W ca[4] = {ta[0], ta[1], ta[2], ta[3]};
      const TrChunk<T, D> cm = tm;
      if (x + 1 < 2 * NDT) {
        load_q(x + 1 < NDT ? bg : bq, (x + 1) % NDT, ta);
        load_k(x + 1 < NDT ? bvp : bkp, (x + 1) % NDT, tm);
      }
      const float bias = x < NDT ? s.vp_bias : s.kp_bias;
      f32x16_t u = {};
      float y[16];
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) {
        y[vv] = elem<T, D>(ca[vv >> 2], dt) * plus_bias<BIAS>(elem<T, D>(cm.x[vv], dt), bias);
        if (D < 32) y[vv] = c < D ? y[vv] : 0.f;
      }
      if constexpr (split) {
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const auto yp = split8<BIAS ? 3 : 2>(y + 8 * n);
#pragma unroll
          for (int o = (BIAS ? 3 : 2) - 1; o >= 0; --o) u = mfma_parts(yp.p[o], (x < NDT ? pp : dsp)[n], u);
        }
      } else {
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) u = mfma_f32(y[vv], x < NDT ? p[vv] : ds[vv], u);
      }
      if (!split && edge && any_nonfinite(u))
        u = masked_tile<D>(x < NDT ? p : ds, lds + kOps + wave * kScratch, c, h, seen, [&](int r, int d, float* z) {
          float y1[4];
          ldcols<T, D>(x < NDT ? bg : bq, (r >> lw) * rsb, dt, d, z);
          ldcols<T, D>(x < NDT ? bvp : bkp, (i0 - k0 + (r >> lw) - tof(r)) * rsb, dt, d, y1);
#pragma unroll
          for (int e = 0; e < 4; ++e) z[e] *= plus_bias<BIAS>(y1[e], bias);
        });
      if (x < NDT)
        av[dt] += u;
      else
        ak[dt] += u;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  };
  walk(std::bool_constant<kSplit<T>>{});
  if constexpr (kSplit<T>) {
    if (nonfinite_sums(0.f, ak) || nonfinite_sums(0.f, av)) walk(std::false_type{});
  }
  // ---- sum of the wavefronts, dV then dK ----
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    __syncthreads();
    float* o = lds + (wave * 32 + c) * RS;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int vv = 0; vv < Ge::NV; ++vv) o[32 * dt + acc_row(vv, h)] = pass ? ak[dt][vv] : av[dt][vv];
    __syncthreads();
    T* dst = pass ? dk : dv;
    for (int x = threadIdx.x; x < 32 * D; x += (64 * KW)) {
      const int r = x / D, d = x % D;
      if (j0 + r >= N) continue;
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) sum += lds[(w * 32 + r) * RS + place<T, D>(d)];
      if (ks > 1)
        part[((static_cast<size_t>(sp) * 2 + pass) * s.B * s.H * N + stat + j0 + r) * D + d] = sum;
      else
        st1(dst + base + static_cast<size_t>(j0 + r) * rs + d, pass ? sum * s.scale : sum);
    }
  }
}

// dV, dK from the ks partial sums of each key block, in order.
template <typename T>
__global__ __launch_bounds__(256) void key_sum_f32_kernel(Shape s, int ks, const float* __restrict__ part,
                                                          T* __restrict__ dk, T* __restrict__ dv) {
  const size_t idx = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  const size_t n = static_cast<size_t>(s.B) * s.H * s.N * s.D;  // [B * H, N, D]
  if (idx >= n) return;
  float a = 0.f, y = 0.f;
  for (int p = 0; p < ks; ++p) {
    a += part[(2 * p + 1) * n + idx];
    y += part[2 * p * n + idx];
  }
  const int d = static_cast<int>(idx % s.D), j = static_cast<int>(idx / s.D % s.N);
  const size_t bh = idx / s.D / s.N;
  const size_t dst = ((bh / s.H * s.N + j) * s.H + bh % s.H) * s.D + d;
  st1(dk + dst, a * s.scale);
  st1(dv + dst, y);
}

using f32_offsets::row_bits;

// Whether the row offsets of a tensor of `heads` heads fit the kernels' buffers.
bool rows_fit(const Shape& s, int rows, int heads) {
  return f32_offsets::fits(rows, static_cast<long long>(heads) * s.D * (s.dtype == 0 ? 4 : 2));
}

template <typename T, int D>
hipError_t fwd_go(const Shape& s, const void* q, const void* k, const void* kp, const void* v, const void* vp,
                  void* out, float* lse, hipStream_t st) {
  const int lw = row_bits(s.w2), SP = 32 >> lw;
  const long total = static_cast<long>((s.N + SP - 1) / SP) * s.B * s.H;
  hipLaunchKernelGGL((fwd_f32_kernel<T, D>), dim3(xcd_grid((total + kFWaves - 1) / kFWaves)), dim3(kFThreads), 0, st,
                     s, lw, static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(kp),
                     static_cast<const T*>(v), static_cast<const T*>(vp), static_cast<T*>(out), lse);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t bwd_go(const Shape& s, BwdStage stage, const void* q_, const void* k_, const void* kp_, const void* v_,
                  const void* vp_, const void* dout_, const float* lse, const float* delta, void* g0, void* g1,
                  void* g2, float* halo, hipStream_t st) {
  const auto *q = static_cast<const T*>(q_), *k = static_cast<const T*>(k_), *kp = static_cast<const T*>(kp_);
  const auto *v = static_cast<const T*>(v_), *vp = static_cast<const T*>(vp_), *dout = static_cast<const T*>(dout_);
  const F32Plan plan = f32_bwd_plan(s);
  const bool bias = s.kp_bias != 0.f || s.vp_bias != 0.f;
  if (stage == BwdStage::Key) {
    const long total = static_cast<long>((s.N + 31) / 32) * plan.ks * s.B * s.H;
    float* part = halo + plan.key_floats;
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(xcd_grid(total)), dim3(64 * key_waves<D>()), 0, st, s, row_bits(s.w2), plan.ks, q, k,
                         kp, v, vp, dout, lse, delta, static_cast<T*>(g0), static_cast<T*>(g1), part);
    };
    bias ? go(bwd_key_f32_kernel<T, D, true>) : go(bwd_key_f32_kernel<T, D, false>);
    if (plan.ks > 1) {
      const size_t n = static_cast<size_t>(s.B) * s.H * s.N * D;
      hipLaunchKernelGGL(key_sum_f32_kernel<T>, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, s,
                         plan.ks, part, static_cast<T*>(g0), static_cast<T*>(g1));
    }
    return hipGetLastError();
  }
  const long total = static_cast<long>(plan.nchunks) * s.B * s.H;
  const size_t lds = 4 * (kFWaves * kScratch + 2 * (plan.W2T + plan.qs * (32 >> plan.lw)) * (D + 4));
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(xcd_grid(total)), dim3(kFThreads), lds, st, s, plan, q, k, kp, v, vp, dout, lse, delta,
                       static_cast<T*>(g0), static_cast<T*>(g1), static_cast<T*>(g2), halo);
  };
  bias ? go(bwd_query_f32_kernel<T, D, true>) : go(bwd_query_f32_kernel<T, D, false>);
  if (plan.nchunks > 1) {
    const long n = static_cast<long>(s.B) * s.H * D *
                   (plan.full ? s.N : static_cast<long>(plan.nchunks - 1) * (plan.W2T - 1));
    hipLaunchKernelGGL(fixup_f32_kernel<T>, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, s, plan,
                       halo, static_cast<T*>(g1), static_cast<T*>(g2));
  }
  return hipGetLastError();
}

}  // namespace

bool f32_fwd_supported(const Shape& s) {
  return s.form == 0 && rows_fit(s, f32_offsets::kBlockRows, s.Hkv);  // q is indexed in 64 bits
}
bool f32_bwd_key_supported(const Shape& s) {
  return s.form == 0 && s.Hkv == s.H && rows_fit(s, f32_offsets::kBlockRows, s.H);
}
// The query side's ring holds 128 k-rows in LDS; longer w2 take the plain kernels.
bool f32_bwd_query_supported(const Shape& s) {
  return s.form == 0 && s.w2 <= 128 && s.Hkv == s.H && rows_fit(s, f32_offsets::query_rows(s.w2), s.H);
}

F32Plan f32_bwd_plan(const Shape& s) {
  F32Plan p{};
  p.lw = row_bits(s.w2);
  p.groups = p.lw == 5 ? (s.w2 + 31) / 32 : 1;
  p.W2T = p.lw == 5 ? 32 * p.groups : 1 << p.lw;
  p.qs = p.groups < kFWaves ? kFWaves / p.groups : 1;  // 4, 2, 1, 1
  p.ks = 1;
  const long bh = static_cast<long>(s.B) * s.H;
  p.halo_off = ((bh * static_cast<size_t>(s.N) * 4) + 255) & ~size_t(255);
  p.bytes = p.halo_off;
  p.CQ = s.N;
  p.nchunks = 1;
  const size_t room = s.ws_cap > p.halo_off ? (s.ws_cap - p.halo_off) / 4 : 0;  // floats
  auto fits = [&](size_t floats) { return s.ws_cap == 0 || floats <= room; };
  if (f32_bwd_query_supported(s)) {
    auto set_chunk = [&](long c) {
      p.CQ = static_cast<int>(c);
      p.nchunks = static_cast<int>((s.N + c - 1) / c);
      p.full = p.nchunks > 1 && c < p.W2T;
      const size_t rows = p.nchunks <= 1 ? 0 : p.full ? c + p.W2T - 1 : p.W2T - 1;
      p.halo_floats = bh * static_cast<size_t>(p.nchunks) * rows * s.D;
      p.key_floats = (p.full ? 2 : 4) * p.halo_floats;
    };
    // A workgroup per CU at least: from 128 queries down to 16, below W2T at the
    // price of a partial sum for every k-row; to a single step while the
    // workgroups still fit the CUs at once (a chunk's steps run one after another:
    // 24 us each at D=128 w2=128 and one key block; N=300 H=1 w1=1 w2=100 D=128:
    // 381 us in chunks of 16, 76 in chunks of 2, 105 on the plain kernels). 512:
    // up to two workgroups share a CU; stopping at 256 costs 14 to 30% (N=3000 H=4
    // D=64 w1=256 w2=32 float32 704 us for 619, N=3000 H=8 D=128 w1=100 w2=8 568
    // for 434), going on to 1024 gains nothing (617, 444). Longer chunks where
    // there are more than 4096 (within 1% of a limit of 1024 or 16384 at 8000 to
    // 33000 chunks: it bounds the partial sums), and where the caller's workspace
    // is capped.
    long cq = 128;
    while (cq > 16 && bh * ((s.N + cq - 1) / cq) < 512) cq /= 2;
    while (cq > p.qs * (32 >> p.lw) && bh * ((s.N + cq / 2 - 1) / (cq / 2)) <= 256) cq /= 2;
    set_chunk(cq);
    while (p.CQ < s.N && (bh * p.nchunks > 4096 || !fits(p.key_floats))) set_chunk(2l * p.CQ);
    // Chunks of more than an eighth of all queries, in a workspace of little
    // more than Delta: a workgroup's walk then takes longer than one thread per
    // pair on the whole chip. One chunk per head of N=2000 D=64 w1=256 w2=16,
    // float32: 14.5 ms for 1 to 32 heads, the plain kernels 2.2, 4.3, 8.4, 16.6
    // (8 heads), 33.1 ms; N=1024 D=128 w1=w2=128, bf16: 35 ms and 5.8 .. 44 (8), 88.
    if (p.CQ > 128 && 8l * p.CQ > bh * s.N) {
      p.plain = true;
      set_chunk(s.N);
    }
  }
  // Key side: a key block's row blocks go to up to four workgroups while there
  // are too few key blocks for the CUs (the sum costs a launch: 5 us), to up to 16
  // where that leaves every wavefront a row block and the workgroups fit the CUs
  // at once (N=300 H=1 w1=1 w2=100 D=64: 56 us in four, 27 in 16, 25 on the plain
  // kernels). 192 key blocks: a limit of 128 leaves N=1024 H=4 D=128 w1=w2=128
  // whole (1310 us for 684; 119 -> 103 us at N=600 H=4 D=64 w1=256 w2=16), one of
  // 256 splits where the CUs are nearly full (N=2000 H=4 D=64: 204 us for 193).
  const size_t n = bh * static_cast<size_t>(s.N) * s.D;
  const long blocks = bh * ((s.N + 31) / 32);
  const int SP = 32 >> p.lw, kw = s.D == 128 ? key_waves<128>() : key_waves<64>();
  const long nrb = (std::min<long>(s.N, 31l + s.w1) + SP - 1) / SP * p.groups;  // row blocks of a key block
  while (f32_bwd_key_supported(s) && fits(p.key_floats + 4 * p.ks * n) &&
         (p.ks < 4 ? blocks * p.ks < 192 : p.ks < 16 && blocks * p.ks <= 128 && 2 * p.ks * kw <= nrb))
    p.ks *= 2;
  p.bytes += 4 * (p.key_floats + (p.ks > 1 ? 2 * p.ks * n : 0));
  return p;
}

#define SA_F32_D(T, FN, ...)                  \
  switch (s.D) {                              \
    case 16: return FN<T, 16>(__VA_ARGS__);   \
    case 32: return FN<T, 32>(__VA_ARGS__);   \
    case 64: return FN<T, 64>(__VA_ARGS__);   \
    case 128: return FN<T, 128>(__VA_ARGS__); \
    default: return hipErrorInvalidValue;     \
  }

hipError_t f32_fwd(const Shape& s, const void* q, const void* k, const void* kp, const void* v, const void* vp,
                   void* out, float* lse, hipStream_t st) {
  if (s.dtype == 0) {
    SA_F32_D(float, fwd_go, s, q, k, kp, v, vp, out, lse, st);
  }
  SA_F32_D(uint16_t, fwd_go, s, q, k, kp, v, vp, out, lse, st);
}

hipError_t f32_bwd_stage(const Shape& s, BwdStage stage, const void* q, const void* k, const void* kp, const void* v,
                         const void* vp, const void* dout, const float* lse, const float* delta, void* g0, void* g1,
                         void* g2, float* halo, hipStream_t st) {
  if (s.dtype == 0) {
    SA_F32_D(float, bwd_go, s, stage, q, k, kp, v, vp, dout, lse, delta, g0, g1, g2, halo, st);
  }
  SA_F32_D(uint16_t, bwd_go, s, stage, q, k, kp, v, vp, dout, lse, delta, g0, g1, g2, halo, st);
}

}  // namespace sa
