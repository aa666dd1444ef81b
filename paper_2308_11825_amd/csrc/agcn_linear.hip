// Linear transformation of a GCNConv layer, H = X W (Sec. II-A), on the
// matrix cores of gfx950, with float32 accuracy.
//
// k_linear_split (any shape) multiplies on the bf16 matrix cores: X and W are
// cut into three bf16 parts each while they are staged (x = x0 + x1 + x2, each
// part the rounded rest of the one before, 24 bits in all, so the sum is x
// itself), and eight of the nine part products are added in fp32; the one left
// out, x2 w2, is at most 2^-34 |x||w|. A product of bf16 numbers is exact in
// fp32, but v_mfma_f32_16x16x32_bf16 cuts off what falls below the last bit of
// the accumulator it adds to (single products summed in one chain: relative
// error 3.5e-8 rms, 1.5e-7 at most, where one rounding makes 2.5e-8 and 6.0e-8).
// So the products below the leading one share an accumulator of their own (at
// most 2^-7 of the sum), and x0 w0 starts from zero in every chunk of 32 k and is
// added by one fp32 add: per element fin / 32 roundings where the fp32 matrix
// instruction makes fin. 2-norm error against 64 bits, fp32 matrix instruction
// and now, 40,000 rows: one nonzero per row 2.53e-8 and 2.53e-8 (largest 6.0e-8
// and 6.0e-8), two 3.1e-8 and 2.6e-8, eight 5.3e-8 and 2.8e-8, dense fin 2
// 3.1e-8 and 2.6e-8, 33 1.07e-7 and 4.0e-8, 128 2.0e-7 and 5.5e-8, 602 4.4e-7
// and 9.2e-8. Eight bf16 products cost half of one fp32 product's matrix time.
// Infinities, NaN and values that round past bf16's range turn the parts into
// NaN, and so every element they take part in: any element that is not finite
// is computed again by the fp32 matrix instruction (sp_redo), which gives the
// infinity or NaN (or finite value) of the fp32 product.
// bf16 has fp32's exponents and ends at 2^-133, so the third part of a value below
// 2^-109 loses bits, at most 2^-134, whatever the other factor is; and the small
// products of a sum near 2^-126 lose bits there. The kernels note where a third
// part is subnormal (values below 2^-103 only), and sp_redo also computes the
// elements that such a loss could reach (sp_floor) and those below 2^-100.
// k_linear_ksplit is the same product for few rows: the k range is cut over
// the waves of a workgroup. k_linear_rw (fp32 matrix instruction, W resident
// on chip) serves fin < 32, where a chunk of 32 k is partly empty.
#include <algorithm>

#include "agcn_internal.hpp"

namespace agcn {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

// The layer's activation where H is the layer's output (act = 1: ReLU, negative
// values become 0; NaN and -0 pass through).
__device__ inline float act_v(float v, int32_t act) { return (act && v < 0.0f) ? 0.0f : v; }
__device__ inline f4 act_v(f4 v, int32_t act) {
  return act ? f4{act_v(v.x, 1), act_v(v.y, 1), act_v(v.z, 1), act_v(v.w, 1)} : v;
}
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// --- X and W as three bf16 parts each ---------------------------------------------
//
// k_linear_split: one workgroup of WAVES waves per (WAVES * RB * 16 rows of X,
// NB * 16 columns of W). k is walked in chunks of 32:
//   1. the W chunk (32 x NB * 16) is cut into parts by the whole workgroup and
//      written to LDS, one 16-byte unit per (part, column, lane group): the 8
//      values of k that a lane feeds to one instruction. Units of a column are
//      rotated by its index so that the writes of consecutive columns fall in
//      different banks; a fragment read is 1 KiB in a row;
//   2. X needs no LDS: lane (i, g) of a wave loads X[row i][k0 + 4 g .. + 3]
//      and [k0 + 16 + 4 g .. + 3] (two 16-byte loads, 64 consecutive bytes of a
//      row over the four g) and cuts them in registers. The order of k inside
//      a chunk is that of the loads, on both sides;
//   3. both chunks for the next step are loaded before the current one is
//      multiplied; two LDS buffers, one barrier per chunk.
// W^T is the left operand, so that lane (i, g) ends with H[row i][16 b + 4 g ..
// + 3] of every column block b: one 16-byte store each. 16-byte loads and
// stores need 4-byte alignment only, so every stride and offset takes this
// path; a row's last chunk is loaded by elements where it is not whole.
// A wave takes 16 rows: with 32 the two accumulators leave 3 waves per SIMD or
// fewer (1e6 x 64 -> 64 120 us against 109, 64 -> 128 128 against 95, 230,000 x
// 602 -> 64 184 against 167; with 256 columns a tile spills).
// Bound: matrix cores from fin 256 up, memory below. Measured with the fp32 matrix
// instruction and now, us: 230,000 rows 602 -> 256 797 and 500 (1.15 PFLOP/s of bf16
// products, what a library's bf16 product of 8192^3 reaches on this card is 1.16),
// 512 -> 128 280 and 231, 128 -> 128 70 and 69, 128 -> 64 41 and 44, 33 -> 17 22 and
// 19; 170,000 x 256 -> 40 63 and 44; 1e6 rows 100 -> 100 283 and 277, 64 -> 64 101
// and 119, 64 -> 16 58 and 67. (Six products in one sum, which lost bits: 395, 191,
// 56, 35, 17; 38; 235, 101, 60.)
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kSpK = 32;  // k per chunk: one v_mfma_f32_16x16x32_bf16

// The three parts of eight values; tiny: some third part is subnormal.
__device__ inline void split8(const float* v, b8* part, bool& tiny) {
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    f2 r = {v[i], v[i + 1]};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const b2 h = __builtin_convertvector(r, b2);
      part[p][i] = h.x;
      part[p][i + 1] = h.y;
      if (p < 2) {
        r.x -= (float)h.x;
        r.y -= (float)h.y;
      }
    }
    constexpr int kSubnormal = 0x90;  // of v_cmp_class: either sign
    tiny |= __builtin_amdgcn_classf(r.x, kSubnormal) | __builtin_amdgcn_classf(r.y, kSubnormal);
  }
}

// One chunk's eight part products, W parts w and X parts x: the seven small ones
// are added in `lo` from the smallest up, x0 w0 (sixteen bits each way, so the sum
// of one is exact) alone; `hi` takes it in one fp32 add per chunk.
constexpr int kSpLo = 7;
__device__ constexpr int kSpW[kSpLo] = {1, 2, 2, 0, 1, 1, 0}, kSpX[kSpLo] = {2, 1, 0, 2, 1, 0, 1};

// hi + lo += W^T chunk (LDS) * X chunk, column block by column block.
template <int NB>
__device__ inline void sp_mma(const b8* xf, const b8* __restrict__ sw, int i, int g, f4* hi,
                              f4* lo) {
  const int at = i * 4 + ((g + (i >> 1)) & 3);
  const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    b8 w[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) w[p] = sw[p * NB * 64 + b * 64 + at];
    const f4 top = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], xf[0], zero, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < kSpLo; ++q)
      lo[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[kSpW[q]], xf[kSpX[q]], lo[b], 0, 0, 0);
    hi[b] += top;
  }
}

// The lane's 8 values of a row in the chunk at k0, zero past fin.
__device__ inline void sp_load_x(const float* __restrict__ row, int k0, int g, int32_t fin,
                                 float* v) {
  if (k0 + kSpK <= fin) {  // uniform
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f4u t = *reinterpret_cast<const f4u*>(row + k0 + 16 * h + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * h + e] = t[e];
    }
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = k0 + 16 * h + 4 * g;
      if (k + 4 <= fin) {
        const f4u t = *reinterpret_cast<const f4u*>(row + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * h + e] = t[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * h + e] = k + e < fin ? row[k + e] : 0.0f;
      }
    }
  }
}

// A thread's share of a W chunk between its loads and its parts' way to LDS.
// Rows past fin and columns past fout repeat the last ones (X is zero there,
// or the columns are not stored), so no load is out of range.
template <int NB, int T>
struct WStage {
  static constexpr int N = (NB * 64 + T - 1) / T;
  float v[N][8];
  __device__ inline void load(const float* __restrict__ W, int64_t ldw, int col0, int32_t fout,
                              int k0, int32_t fin) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int idx = threadIdx.x + u * T;
      const int c = min(col0 + idx % (NB * 16), fout - 1), g = idx / (NB * 16);
      if (NB * 64 % T == 0 || idx < NB * 64) {
        const float* p = W + c;
        if (k0 + kSpK <= fin) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            v[u][e] = p[(int64_t)(k0 + 4 * g + (e & 3) + 16 * (e >> 2)) * ldw];
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            v[u][e] = p[(int64_t)min(k0 + 4 * g + (e & 3) + 16 * (e >> 2), fin - 1) * ldw];
        }
      }
    }
  }
  __device__ inline void store(b8* sw, bool& tiny) const {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int idx = threadIdx.x + u * T;
      const int c = idx % (NB * 16), g = idx / (NB * 16);
      if (NB * 64 % T == 0 || idx < NB * 64) {
        b8 part[3];
        split8(v[u], part, tiny);
#pragma unroll
        for (int p = 0; p < 3; ++p) sw[p * NB * 64 + c * 4 + ((g + (c >> 1)) & 3)] = part[p];
      }
    }
  }
};

// What a wave has met: bit r: a third part of row r was subnormal, bit 16: one of
// the W columns was. A wave leaves its word in LDS before a barrier.
constexpr uint32_t kSpTinyW = 1u << 16;
__device__ inline uint32_t sp_tiny(bool x_tiny, bool w_tiny) {
  const uint64_t r = __ballot(x_tiny);
  const uint32_t rows = (uint32_t)(r | r >> 16 | r >> 32 | r >> 48) & 0xFFFFu;
  return rows | (__ballot(w_tiny) != 0 ? kSpTinyW : 0u);
}
template <int WAVES>
__device__ inline uint32_t sp_any(const uint32_t* words) {
  uint32_t m = 0;
#pragma unroll
  for (int v = 0; v < WAVES; ++v) m |= words[v];
  return __builtin_amdgcn_readfirstlane(m);
}

// By a wave that met some: the magnitude above which an element of the lane's
// row has lost at most 2^-26 of itself. The third parts' loss is at most 2^-134
// in each value of the row or of the W columns, times the largest value that it
// multiplies, fin times. 230,000 x 602 -> 256, 498 us without such values: one tiny
// weight 531, a seventh of the weights' rows 589, a third of X's rows 757, all of X
// (every element computed again) 2014.
template <int NB>
__device__ inline float sp_floor(uint32_t tiny, const float* __restrict__ xr, int i, int g,
                                 int col0, int32_t fin, int32_t fout,
                                 const float* __restrict__ W, int64_t ldw) {
  float wm = 0.0f, xm = 0.0f;  // (fmaxf drops NaN)
  if ((tiny & 0xFFFFu) != 0) {
    const int cols = min(NB * 16, fout - col0);
    for (int c = threadIdx.x & 63; c < cols; c += 64) {
      const float* p = W + col0 + c;
#pragma unroll 8
      for (int k = 0; k < fin; ++k) wm = fmaxf(wm, fabsf(p[(int64_t)k * ldw]));
    }
  }
  if ((tiny & kSpTinyW) != 0)
#pragma unroll 2
    for (int k0 = 0; k0 < fin; k0 += kSpK) {
      float v[8];
      sp_load_x(xr, k0, g, fin, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) xm = fmaxf(xm, fabsf(v[e]));
    }
#pragma unroll
  for (int m = 32; m >= 1; m /= 2) {
    wm = fmaxf(wm, __shfl_xor(wm, m));
    if (m >= 16) xm = fmaxf(xm, __shfl_xor(xm, m));
  }
  return 0x1p-108f * (float)fin *
         ((tiny >> i & 1 ? wm : 0.0f) + ((tiny & kSpTinyW) != 0 ? xm : 0.0f));
}

// Four elements of an H row from column col on, those that lie inside it.
__device__ inline void sp_put(float* __restrict__ Hrow, int col, int32_t fout, f4 v, int32_t act) {
  if (col + 3 < fout) {
    *reinterpret_cast<f4u*>(Hrow + col) = act_v(v, act);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < fout) Hrow[col + e] = act_v(v[e], act);
  }
}

// The chunk at k0 as the fp32 matrix instruction takes it: instruction e of a
// chunk multiplies X[row i][k] by W[k][column i of block b], k = k0 + 4 g + (e & 3)
// + 16 (e >> 2), both zero past fin.
template <int GB>
__device__ inline void sp_load_fp32(const float* __restrict__ xr, const float* __restrict__ W,
                                    int64_t ldw, int col, int32_t fout, int k0, int g, int32_t fin,
                                    float* xv, float (*wv)[8]) {
  sp_load_x(xr, k0, g, fin, xv);
#pragma unroll
  for (int b = 0; b < GB; ++b) {
    const float* p = W + min(col + 16 * b, fout - 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = k0 + 4 * g + (e & 3) + 16 * (e >> 2);
      const float w = p[(int64_t)min(k, fin - 1) * ldw];
      wv[b][e] = k < fin ? w : 0.0f;
    }
  }
}

// Computes the wave's 16 rows again with the fp32 matrix instruction, GB column
// blocks at a time and only where some lane's bit of `bad` is set, and writes
// the groups of four whose bit is set. The next chunk is loaded before the
// current one is multiplied. Where every element is NaN, 230,000 x 602 -> 256
// takes 1.62 ms and the finite product 0.49 (a serial sum per element in its own
// lane: 79), 230,000 x 128 -> 128 0.18 and 0.066 (7.5), 3000 x 1000 -> 16 28 and
// 12 us (445).
template <int NB>
__device__ inline void sp_redo(uint32_t bad, const float* __restrict__ xr, int i, int g, int col0,
                               int32_t fin, int32_t fout, const float* __restrict__ W, int64_t ldw,
                               float* __restrict__ Hrow, int32_t act) {
  constexpr int GB = NB == 8 ? 2 : 1;
  static_assert(NB % GB == 0, "");
#pragma unroll 1
  for (int b0 = 0; b0 < NB; b0 += GB, bad >>= GB) {
    const uint32_t mine = bad & ((1u << GB) - 1);
    if (__ballot(mine != 0) == 0) continue;
    const int cb = col0 + 16 * b0;
    f4 acc[GB];
#pragma unroll
    for (int b = 0; b < GB; ++b) acc[b] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    float xv[8], wv[GB][8], xn[8], wn[GB][8];
    sp_load_fp32<GB>(xr, W, ldw, cb + i, fout, 0, g, fin, xv, wv);
#pragma unroll 1
    for (int k0 = 0; k0 < fin; k0 += kSpK) {
      if (k0 + kSpK < fin)
        sp_load_fp32<GB>(xr, W, ldw, cb + i, fout, k0 + kSpK, g, fin, xn, wn);
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int b = 0; b < GB; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[b][e], xv[e], acc[b], 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xv[e] = xn[e];
#pragma unroll
        for (int b = 0; b < GB; ++b) wv[b][e] = wn[b][e];
      }
    }
#pragma unroll
    for (int b = 0; b < GB; ++b)
      if (mine >> b & 1) sp_put(Hrow, cb + 16 * b + 4 * g, fout, acc[b], act);
  }
}

constexpr uint32_t kSpSmall = ((127u - 100u) << 24) - 1;  // 2 bits(2^-100) - 1

// Writes the lane's elements of H, and again (sp_redo) the groups of four that
// hold a value that is not finite (or add up to none), below `floor` or so small
// that its products were subnormal.
template <int NB>
__device__ inline void sp_store(const f4* acc, const float* __restrict__ xr, int64_t row, int i,
                                int g, int col0, int64_t n, int32_t fin, int32_t fout,
                                const float* __restrict__ W, int64_t ldw, float* __restrict__ H,
                                int64_t ldh, int32_t act, float floor) {
  float* Hrow = H + (row < n ? row : n - 1) * ldh;
  uint32_t bad = 0;
  if (row < n) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const f4 v = acc[b];
      const float m = fabsf(v.x) + fabsf(v.y) + fabsf(v.z) + fabsf(v.w);
      uint32_t lo = 0xFFFFFFFFu;  // (2 bits(|v|) - 1: zero is the largest)
#pragma unroll
      for (int e = 0; e < 4; ++e) lo = min(lo, (__float_as_uint(v[e]) << 1) - 1);
      bad |= (m < __builtin_inff() && lo >= kSpSmall ? 0u : 1u) << b;
      if (floor > 0.0f)
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= (fabsf(v[e]) < floor ? 1u : 0u) << b;
      sp_put(Hrow, col0 + 16 * b + 4 * g, fout, v, act);
    }
  }
  if (__ballot(bad != 0) != 0)
    sp_redo<NB>(bad, xr, i, g, col0, fin, fout, W, ldw, Hrow, act);
}

// (The second launch bound keeps the registers of the rare sp_redo from costing
// waves: 230,000 x 602 -> 256 566 us without it, 170,000 x 256 -> 40 47.5 with 4
// for 48 columns and 44.5 with 6. One column block at a time in sp_redo for the
// narrower tiles, for the same reason.)
template <int NB, int WAVES>
__global__ __launch_bounds__(WAVES * 64, NB <= 3 ? 6 : NB == 4 ? 5 : 4) void k_linear_split(
    int64_t n, int32_t fin, int32_t fout, int32_t n_ct, const float* __restrict__ X, int64_t ldx,
    const float* __restrict__ W, int64_t ldw, float* __restrict__ H, int64_t ldh, int32_t act) {
  constexpr int T = WAVES * 64, BM = WAVES * 16;
  __shared__ b8 sw[2][3 * NB * 64];
  __shared__ uint32_t s_tiny[WAVES];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  // The column tiles of a row tile run on one XCD (workgroups go to the XCDs in turn).
  const int64_t q = blockIdx.x >> 3;
  const int64_t rt = (q / n_ct) * 8 + (blockIdx.x & 7);
  const int ct = (int)(q % n_ct);
  const int64_t row = rt * BM + wave * 16 + i;
  const int col0 = ct * NB * 16;
  if (rt * BM >= n) return;
  const float* xr = X + (row < n ? row : n - 1) * ldx;
  f4 hi[NB], lo[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) hi[b] = lo[b] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  WStage<NB, T> ws;
  bool x_tiny = false, w_tiny = false;
  float xv[8];
  if (fin > 0) {  // (fin = 0: H = 0, X and W may be NULL)
    ws.load(W, ldw, col0, fout, 0, fin);
    sp_load_x(xr, 0, g, fin, xv);
  }
  int buf = 0;
  for (int k0 = 0; k0 < fin; k0 += kSpK, buf ^= 1) {
    ws.store(sw[buf], w_tiny);
    const bool more = k0 + kSpK < fin;
    if (more) ws.load(W, ldw, col0, fout, k0 + kSpK, fin);
    const uint32_t w_any = sp_tiny(false, w_tiny);
    if (lane == 0) s_tiny[wave] = w_any;
    __syncthreads();
    b8 xf[3];
    split8(xv, xf, x_tiny);
    if (more) sp_load_x(xr, k0 + kSpK, g, fin, xv);
    sp_mma<NB>(xf, sw[buf], i, g, hi, lo);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) hi[b] += lo[b];
  // The lane's place again: kept over the loop, it costs registers (128 columns
  // spill, and any scratch costs a short tile a quarter: 1e6 x 32 -> 32 41 -> 52 us).
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  const int i2 = t & 15, g2 = (t >> 4) & 3;
  const int64_t row2 = rt * BM + (t >> 6) * 16 + i2;
  const float* xr2 = X + (row2 < n ? row2 : n - 1) * ldx;
  float floor = 0.0f;
  const uint32_t tiny = sp_tiny(x_tiny, false) | (fin > 0 ? sp_any<WAVES>(s_tiny) : 0u);
  if (tiny != 0) floor = sp_floor<NB>(tiny, xr2, i2, g2, col0, fin, fout, W, ldw);
  sp_store<NB>(hi, xr2, row2, i2, g2, col0, n, fin, fout, W, ldw, H, ldh, act, floor);
}

// k_linear_ksplit: few rows leave k_linear_split a handful of workgroups that
// walk the chunks in series (3000 x 1000 -> 16: 26 us, a load latency per
// chunk). Here a workgroup takes 16 rows and NB * 16 columns, its waves take the
// chunks in turn (each loads and cuts its own W fragments from L2), and wave 0
// adds the waves' sums in wave order: 5.9 us. (The second launch bound as in
// k_linear_split: 16,000 x 256 -> 64 13.6 us without it, 11.3 with.)
template <int NB, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_linear_ksplit(
    int64_t n, int32_t fin, int32_t fout, const float* __restrict__ X, int64_t ldx,
    const float* __restrict__ W, int64_t ldw, float* __restrict__ H, int64_t ldh, int32_t act) {
  __shared__ f4 part[WAVES][2][NB][64];  // the waves' hi and lo sums
  __shared__ uint32_t s_tiny[WAVES];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const int64_t row0 = (int64_t)blockIdx.x * 16;
  const int col0 = (int)blockIdx.y * NB * 16;
  const float* xr = X + min(row0 + i, n - 1) * ldx;
  f4 hi[NB], lo[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) hi[b] = lo[b] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  bool x_tiny = false, w_tiny = false;
  for (int k0 = wave * kSpK; k0 < fin; k0 += WAVES * kSpK) {
    float xv[8], wv[NB][8];
    sp_load_x(xr, k0, g, fin, xv);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float* p = W + min(col0 + b * 16 + i, fout - 1);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        wv[b][e] = p[(int64_t)min(k0 + 4 * g + (e & 3) + 16 * (e >> 2), fin - 1) * ldw];
    }
    b8 xf[3];
    split8(xv, xf, x_tiny);
    const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      b8 w[3];
      split8(wv[b], w, w_tiny);
      const f4 top = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], xf[0], zero, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < kSpLo; ++q)
        lo[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[kSpW[q]], xf[kSpX[q]], lo[b], 0, 0, 0);
      hi[b] += top;
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    part[wave][0][b][lane] = hi[b];
    part[wave][1][b][lane] = lo[b];
  }
  const uint32_t mine = sp_tiny(x_tiny, w_tiny);
  if (lane == 0) s_tiny[wave] = mine;
  __syncthreads();
  if (wave != 0) return;
  constexpr int kAhead = NB == 4 ? 1 : NB == 2 ? 3 : WAVES;  // (more at once cost registers)
#pragma unroll kAhead
  for (int w = 1; w < WAVES; ++w)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      hi[b] += part[w][0][b][lane];
      lo[b] += part[w][1][b][lane];
    }
#pragma unroll
  for (int b = 0; b < NB; ++b) hi[b] += lo[b];
  int t = threadIdx.x;  // (as in k_linear_split)
  asm volatile("" : "+v"(t));
  const int i2 = t & 15, g2 = (t >> 4) & 3;
  const int64_t row2 = row0 + i2;
  const float* xr2 = X + (row2 < n ? row2 : n - 1) * ldx;
  float floor = 0.0f;
  const uint32_t tiny = sp_any<WAVES>(s_tiny);
  if (tiny != 0) floor = sp_floor<NB>(tiny, xr2, i2, g2, col0, fin, fout, W, ldw);
  sp_store<NB>(hi, xr2, row2, i2, g2, col0, n, fin, fout, W, ldw, H, ldh, act, floor);
}

// --- W resident in LDS --------------------------------------------------------
//
// k_linear_rw: for fin < 32 and fout <= 128 (wider outputs: one launch per
// 128 columns; 128-bit path, X and H each under 4 GiB), W^T stays in
// LDS for the whole kernel and every wave works alone on 16-row tiles of X, so
// the main loop has no workgroup barrier:
//   1. each workgroup (4 waves) writes W^T into LDS once: NB * 16 rows (output
//      columns) of KP floats (fin rounded up to 32), zero outside W; the
//      16-byte chunk c of row j sits at chunk c ^ (j & 7), so the 8 rows a
//      group of lanes reads for one chunk fall in 8 different bank groups;
//   2. wave v takes tiles v, v + waves, ... of 16 rows while every wave has a
//      whole round left; the next tile's X is loaded into registers while the
//      current one is multiplied. The tiles of the last, partial round are
//      cut by output columns into as many ranges (1, 2, 4 or 8) as still give
//      each range a wave of its own, so that round takes a fraction of a
//      tile's time instead of a whole one;
//   3. v_mfma_f32_16x16x4f32 with W^T as the left operand, so one instruction
//      computes (X W)^T for 16 rows and 16 output columns (lane l supplies
//      A[l % 16][l / 16] = W^T[col][k] and B[l / 16][l % 16] = X[row][k];
//      accumulator register r of lane l holds C[4 (l / 16) + r][l % 16], that
//      is H[row l % 16][4 (l / 16) + r]: four consecutive columns of one row,
//      written with one 16-byte store). The contraction order is permuted so
//      that one 16-byte load per lane feeds four instructions: in k-step s,
//      lane l loads X[row][16 s + 4 g .. + 3] (g = l / 16) and instruction t
//      takes element t, paired with W^T[col][16 s + 4 g + t] from one 16-byte
//      LDS read; the four instructions together cover k = 16 s .. 16 s + 15.
// fp32 products, bound by memory at these sizes. Against k_linear_split, whose
// only chunk is then partly empty: 230,000 rows 12 -> 128 28.9 and 30.5 us, 16 ->
// 64 16.9 and 19.9; 2.4 M rows 8 -> 8 47.6 and 72.8, 16 -> 32 109 and 126.
constexpr int kRwThreads = 256;
constexpr int kRwWaves = kRwThreads / 64;
constexpr int kRwRows = 16;

// Offset of a masked element. A raw buffer access is out of range when its
// offset is >= the resource's byte count; every resource here covers at most
// kRwOutOfRange - 16 bytes (checked by the host), so this offset is always
// out of range: the load returns 0 and the store is dropped.
constexpr uint32_t kRwOutOfRange = 0xFFFFFFF0u;

__device__ inline __amdgpu_buffer_rsrc_t rw_resource(const void* base, uint32_t bytes) {
  // Raw buffer (stride 0) of `bytes` bytes; dword3 = 32-bit data format (gfx9 family).
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           0x00020000);
}

__device__ inline int wt_index(int j, int k, int kc) {  // float index of W^T[j][k]
  return (j * kc + ((k >> 2) ^ (j & 7))) * 4 + (k & 3);
}

template <int NB>
__global__ __launch_bounds__(kRwThreads) void k_linear_rw(int64_t n, int32_t fin, int32_t fout,
                                                          const float* __restrict__ X, int64_t ldx,
                                                          const float* __restrict__ W, int64_t ldw,
                                                          float* __restrict__ H, int64_t ldh,
                                                          int32_t act) {
  constexpr int KS = 2, KP = KS * 16, KC = KP / 4, NJ = NB * 16;
  __shared__ __attribute__((aligned(16))) float swt[NJ * KP];
  // 1. W^T into LDS: W row k is read as float4 (4 output columns) and
  //    scattered into 4 rows of W^T. Consecutive lanes take consecutive k, so
  //    their LDS writes land in consecutive words of one W^T row.
  for (int idx = threadIdx.x; idx < KP * (NJ / 4); idx += kRwThreads) {
    const int j0 = (idx / KP) * 4, k = idx - (idx / KP) * KP;
    f4 w = {0.0f, 0.0f, 0.0f, 0.0f};
    if (k < fin && j0 < fout) w = *reinterpret_cast<const f4*>(W + (int64_t)k * ldw + j0);
    swt[wt_index(j0 + 0, k, KC)] = w.x;
    swt[wt_index(j0 + 1, k, KC)] = w.y;
    swt[wt_index(j0 + 2, k, KC)] = w.z;
    swt[wt_index(j0 + 3, k, KC)] = w.w;
  }
  __syncthreads();

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const int64_t n_tiles = (n + kRwRows - 1) / kRwRows;
  const int64_t n_waves = (int64_t)gridDim.x * kRwWaves;
  // X and H through buffer resources: a masked element gets an offset past
  // the 4 GiB range, so its load returns 0 and its store is dropped, with no
  // branch; the compiler then counts the memory operations in flight exactly
  // and waits only for the loads it needs.
  const __amdgpu_buffer_rsrc_t xr = rw_resource(X, (uint32_t)(n * ldx * 4));
  const __amdgpu_buffer_rsrc_t hr = rw_resource(H, (uint32_t)(n * ldh * 4));
  auto load_x = [&](int64_t tile, f4* xv) {
    const int64_t row = tile * kRwRows + i;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int k = 16 * s + 4 * g;
      const uint32_t off = (row < n && k < fin) ? (uint32_t)((row * ldx + k) * 4) : kRwOutOfRange;
      xv[s] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)off, 0, 0));
    }
  };
  // H stores of one tile: lane (i, g) holds H[row i][16 b + 4 g .. + 3] of
  // every column block b, one 16-byte store each.
  const uint32_t ldh4 = (uint32_t)(ldh * 4);
  auto store_h = [&](int64_t tile, const f4* acc) {
    const int64_t row = tile * kRwRows + i;
    const uint32_t base = (uint32_t)(row * ldh4) + (uint32_t)(16 * g);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bool ok = row < n && 16 * b + 4 * g < fout;
      const uint32_t off = ok ? base + (uint32_t)(64 * b) : kRwOutOfRange;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, act_v(acc[b], act)), hr, (int)off, 0, 0);
    }
  };
  // Full rounds: every wave takes n_tiles / n_waves tiles.
  const int64_t wid = (int64_t)blockIdx.x * kRwWaves + wave;
  const int64_t n_full = (n_tiles / n_waves) * n_waves;
  f4 xa[KS], xb[KS];
  int64_t tile = wid;
  if (tile < n_full) load_x(tile, xa);
  for (; tile < n_full; tile += n_waves) {
    if (tile + n_waves < n_full) load_x(tile + n_waves, xb);  // uniform
    f4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      f4 wv[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b)
        wv[b] = *reinterpret_cast<const f4*>(swt + wt_index(16 * b + i, 16 * s + 4 * g, KC));
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[b][t], xa[s][t], acc[b], 0, 0, 0);
    }
    store_h(tile, acc);
#pragma unroll
    for (int s = 0; s < KS; ++s) xa[s] = xb[s];
  }
  // The last, partial round: its tiles are cut into `split` column ranges of
  // NB / split blocks each, as many as keep every unit on its own wave.
  const int64_t rem = n_tiles - n_full;
  if (rem == 0) return;
  int split = 1;
  while (split < NB && rem * split * 2 <= n_waves) split *= 2;
  const int per = NB / split;
  for (int64_t u = wid; u < rem * split; u += n_waves) {
    const int64_t t2 = n_full + u / split;
    const int b0 = (int)(u % split) * per;
    load_x(t2, xa);
    const int64_t row = t2 * kRwRows + i;
    for (int bb = 0; bb < per; ++bb) {
      const int b = b0 + bb;
      f4 acc = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const f4 wv = *reinterpret_cast<const f4*>(swt + wt_index(16 * b + i, 16 * s + 4 * g, KC));
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[t], xa[s][t], acc, 0, 0, 0);
      }
      const bool ok = row < n && 16 * b + 4 * g < fout;
      const uint32_t off = ok ? (uint32_t)(row * ldh4) + (uint32_t)(16 * g) + (uint32_t)(64 * b)
                              : kRwOutOfRange;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, act_v(acc, act)), hr, (int)off, 0, 0);
    }
  }
}

// Workgroups for k_linear_rw: as many as are resident at once on the device
// (each loads W^T once and then loops over tiles), fewer when there are fewer
// tiles.
template <int NB>
int rw_grid(int64_t n) {
  static const int resident = [] {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_linear_rw<NB>, kRwThreads, 0) !=
            hipSuccess) {
      (void)hipGetLastError();
      cus = 256;
      per_cu = 1;
    }
    return std::max(1, cus) * std::max(1, per_cu);
  }();
  const int64_t tiles = (n + kRwRows - 1) / kRwRows;
  return (int)std::max<int64_t>(1, std::min<int64_t>(resident, (tiles + kRwWaves - 1) / kRwWaves));
}

template <int NB>
int launch_rw(int64_t n, int32_t fin, int32_t fout, const float* X, int64_t ldx, const float* W,
              int64_t ldw, float* H, int64_t ldh, hipStream_t st, int32_t act) {
  k_linear_rw<NB><<<rw_grid<NB>(n), kRwThreads, 0, st>>>(n, fin, fout, X, ldx, W, ldw, H,
                                                             ldh, act);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? AGCN_OK : hip_fail(e, "k_linear_rw launch");
}

template <int NB, int WAVES>
int launch_split(int64_t n, int32_t fin, int32_t fout, const float* X, int64_t ldx, const float* W,
                 int64_t ldw, float* H, int64_t ldh, hipStream_t st, int32_t act) {
  constexpr int64_t BM = WAVES * 16;
  const int64_t n_rt = ceil_div64(n, BM);
  const int32_t n_ct = (int32_t)ceil_div64(fout, NB * 16);
  // Row tiles in groups of 8, one per XCD; a last group may be partly empty.
  const int64_t max_rt = (int64_t)UINT32_MAX / (WAVES * 64) / n_ct / 8 * 8;
  if (max_rt == 0) return fail(AGCN_ERR_UNSUPPORTED, "matrix too large for one launch");
  for (int64_t r0 = 0; r0 < n_rt; r0 += max_rt) {
    const int64_t row0 = r0 * BM;
    const int64_t rows = std::min<int64_t>(max_rt * BM, n - row0);
    const int64_t blocks = ceil_div64(ceil_div64(rows, BM), 8) * 8 * n_ct;
    k_linear_split<NB, WAVES><<<dim3((unsigned)blocks), WAVES * 64, 0, st>>>(
        rows, fin, fout, n_ct, X + row0 * ldx, ldx, W, ldw, H + row0 * ldh, ldh, act);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_linear_split launch");
  }
  return AGCN_OK;
}

template <int NB, int WAVES>
int launch_ksplit(int64_t n, int32_t fin, int32_t fout, const float* X, int64_t ldx, const float* W,
                  int64_t ldw, float* H, int64_t ldh, hipStream_t st, int32_t act) {
  k_linear_ksplit<NB, WAVES>
      <<<dim3((unsigned)ceil_div64(n, 16), (unsigned)ceil_div64(fout, NB * 16)), WAVES * 64, 0,
         st>>>(n, fin, fout, X, ldx, W, ldw, H, ldh, act);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? AGCN_OK : hip_fail(e, "k_linear_ksplit launch");
}

// Workgroups that fill the chip about twice: with fewer, smaller tiles or the
// k split are the faster (below).
constexpr int64_t kFewGroups = 512;

}  // namespace

int run_linear(int64_t n, int32_t fin, int32_t fout, const float* X, int64_t ldx, const float* W,
               int64_t ldw, float* H, int64_t ldh, hipStream_t st, int32_t act) {
  if (n == 0 || fout == 0) return AGCN_OK;
  const bool vec = fin % 4 == 0 && fout % 4 == 0 && ldx % 4 == 0 && ldw % 4 == 0 &&
                   aligned16(X) && aligned16(W);
  // k_linear_rw addresses X and H with 32-bit byte offsets, and its masked
  // offset must lie past both (see kRwOutOfRange); it writes H in 16-byte
  // pieces, so H's rows must be 16-byte aligned too.
  const int64_t lim = (int64_t)kRwOutOfRange - 16;
  const bool rw_fits = n * ldx * 4 <= lim && n * ldh * 4 <= lim && ldh % 4 == 0 && aligned16(H);
  if (vec && rw_fits && fin >= 1 && fin < 32) {
    for (int32_t c0 = 0; c0 < fout; c0 += 128) {
      const int32_t w = std::min<int32_t>(128, fout - c0);
      const float* Wc = W + c0;
      float* Hc = H + c0;
      int rc;
      if (w <= 32) rc = launch_rw<2>(n, fin, w, X, ldx, Wc, ldw, Hc, ldh, st, act);
      else if (w <= 64) rc = launch_rw<4>(n, fin, w, X, ldx, Wc, ldw, Hc, ldh, st, act);
      else rc = launch_rw<8>(n, fin, w, X, ldx, Wc, ldw, Hc, ldh, st, act);
      if (rc) return rc;
    }
    return AGCN_OK;
  }
  // Few (16 rows, 64 columns) tiles and more than one chunk: the k split.
  // 3000 x 1000 -> 16 / 64 / 256 5.9 / 11.5 / 26 us against 26 / 40 / 63 in tiles,
  // 12,000 x 128 -> 64 6.6 against 7.2, 16,000 x 256 -> 64 10.6 against 12.0. Past
  // the line it repeats the W cuts too often: 12,000 x 128 -> 256 16.6 against 12.3,
  // 25,000 x 64 -> 64 9.9 against 6.7, 30,000 x 500 -> 40 38 against 23.
  if (fin > 32 && ceil_div64(n, 16) * ceil_div64(fout, 64) <= 2 * kFewGroups) {
    const bool many = fin > 256;
    if (fout <= 16)
      return many ? launch_ksplit<1, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act)
                  : launch_ksplit<1, 4>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
    if (fout <= 32)
      return many ? launch_ksplit<2, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act)
                  : launch_ksplit<2, 4>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
    return many ? launch_ksplit<4, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act)
                : launch_ksplit<4, 4>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
  }
  // 64 rows by 64 columns where 128-row tiles are few: 20,000 x 64 -> 100 7.9 us
  // against 8.6, 40,000 x 128 -> 64 12.0 against 12.8.
  if (fout > 32 && ceil_div64(n, 128) * ceil_div64(fout, 64) < kFewGroups && fin <= 256)
    return launch_split<4, 4>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
  // The narrowest tile that holds fout (a wider one multiplies padding): 170,000 x
  // 256 -> 40 40.7 us with 48 columns and 49 with 64; 128 columns past 64, X being
  // cut once for all of them (230,000 x 128 -> 128 62 against 65 with two of 64,
  // 602 -> 256 504 against 560).
  if (fout <= 16) return launch_split<1, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
  if (fout <= 32) return launch_split<2, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
  if (fout <= 48) return launch_split<3, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
  if (fout <= 64) return launch_split<4, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
  return launch_split<8, 8>(n, fin, fout, X, ldx, W, ldw, H, ldh, st, act);
}

}  // namespace agcn
