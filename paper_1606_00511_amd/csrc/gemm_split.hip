// fp32 GEMMs on the fp16 matrix cores: every operand is held as a pair of
// fp16 numbers (the weights, over short contractions, as three) and three
// (four) partial products are accumulated in fp32 by
// v_mfma_f32_16x16x32_f16.
//
// An operand value v is stored as hi + lo with hi = fp16(v 2^(14 - e)) and
// lo = fp16(v 2^(14 - e) - hi), e being the exponent of the tensor's largest
// magnitude (2^e <= max |v| < 2^(e + 1)): 22 to 24 significant bits for every
// element within 2^-16 of the largest, an absolute error of 2^-39 of the
// largest for the others.  A product keeps lo hi + hi lo + hi hi; the term
// left out is at most 2^-22 of it.  Three fp16 products cost less than one
// fp32 product: dense rates are 2.5 PFLOP/s and 0.16 PFLOP/s.
//
// Errors against 64 bits stay below those of the fp32 MFMAs
// (v_mfma_f32_16x16x4_f32 rounds its accumulator after every term).  Relative
// 2-norm error of 16 x 16 outputs over K = 64 / 288 / 1,024 / 2,048 normal
// terms, in units of 2^-24: 1.5 / 1.8 / 2.4 / 3.0 (fp32 MFMA 2.4 / 5.1 / 9.4
// / 13.4).  What it takes:
//  - A K block's products of an output block go into a temporary from 0,
//    which is then added to the accumulator: one rounding at the
//    accumulator's size per 32 terms (accumulating in place: 8.6 at 2,048).
//  - The fp16 MFMA sums 8 products at a time on a common exponent and drops
//    what lies below 24 bits; the fp32 result rounds towards minus infinity
//    where parts of unlike size meet, by 0.3 x 2^-24 on average.  That is the
//    same for every row of a batch, and a gradient, whose batch sums nearly
//    cancel, showed it (4 to 6 times the fp32 kernels' error on 300 to 1,000
//    wide tanh nets).  So odd rows of the left operand X, and odd K blocks of
//    the right one Y, are stored negated, and the temporary is added with the
//    sign that undoes it: the offset changes sign from row to row and from
//    block to block.
//  - The bits of a weight that a pair cannot hold are off for all rows alike
//    as well; over short contractions they go into a third plane.
//
// The input X has features of unrelated scales, so each of its columns
// carries an exponent of its own (absmax_columns): the columns of W_1 and V_1
// are scaled by the powers of two before their own split, and the layer's
// weight gradient by the same powers.
//
// A tensor with an infinity or a NaN cannot be split.  Its exponent slot
// then says so, and the GEMMs that read it accumulate the fp32 operands with
// v_mfma_f32_16x16x4_f32, as slow as that is.
//
// Layout: 32 consecutive k of a row are stored as 32 hi, then 32 lo (then 32
// of the third plane).  Every operand is K-contiguous; the transposed copies
// come from the same pass that splits a tensor.  Operand buffers have rows up
// to the next multiple of 256 (rows past M or N feed only outputs that are
// not stored) and zeros from K to the next multiple of 32.
#include <algorithm>

#include "epi.h"
#include "hf_internal.h"
#include "lds_dma.h"
#include "tile16.h"

namespace hfk {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int KG = 32;       // k values per group (and per K block)

// A ROWS x KG operand tile of PL planes in LDS: [row][plane][k], the 4 PL
// 16-byte chunks of a row swizzled so that 16 consecutive rows hold one chunk
// in distinct banks (rows are 128 or 192 bytes apart).
template <int ROWS, int PL, int NW>
struct TileP {
  static constexpr int CH = 4 * PL;                  // chunks per row
  static constexpr int BK = 8 * CH;                  // elements per row
  static constexpr int SIZE = ROWS * BK;
  static constexpr int INSTR = ROWS * CH / 64 / NW;  // direct loads per wave
  static_assert(ROWS * CH % (64 * NW) == 0, "tile does not split over the waves");

  // position of chunk c in its row (its own inverse)
  __device__ static __forceinline__ int at(int row, int c) {
    return PL == 2 ? c ^ ((row >> 1) & 7) : (c & ~3) | ((c & 3) ^ ((row >> 2) & 3));
  }
  // element offset, within an operand of leading dimension ld, of the chunk
  // that lane `lane` of wave `wave` fetches with its instruction j
  __device__ static __forceinline__ uint32_t src(int ld, int wave, int lane, int j) {
    const int P = (wave * INSTR + j) * 64 + lane;
    const int row = P / CH;
    return (uint32_t)row * (uint32_t)ld + 8u * (uint32_t)at(row, P % CH);
  }
  __device__ static __forceinline__ int dst(int wave, int j) {
    return (wave * INSTR + j) * 512;
  }
};

__device__ __forceinline__ f32x4 mfma(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// exponent slot of a tensor whose largest magnitude has the given bits
__device__ __forceinline__ int slot_of(uint32_t bits) {
  const int be = (int)(bits >> 23);
  return be == 255 ? SPLIT_NONFINITE : (be == 0 ? -126 : be - 127);
}

// split-K partials and weight gradients: out0 already points at the split
struct ESplitStore {
  static __device__ __forceinline__ float apply(const EpiArgs& e, int r, int c,
                                                float v0, float) {
    e.out0[(size_t)r * e.ldo + c] = v0;
    return 0.0f;
  }
};

// The same epilogues for 4 consecutive columns c .. c + 3 of a row (c, ldo
// and lda multiples of 4, every buffer 16-byte aligned): apply4 returns the
// values apply would.
__device__ __forceinline__ f32x4 ld4(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ void st4(float* p, const f32x4& v) { *(f32x4*)p = v; }
__device__ __forceinline__ f32x4 add_bias(const float* b, int c, const f32x4& v) {
  return f32x4{v[0] + b[c], v[1] + b[c + 1], v[2] + b[c + 2], v[3] + b[c + 3]};
}
template <class F>
__device__ __forceinline__ f32x4 map4(F f) {
  return f32x4{f(0), f(1), f(2), f(3)};
}
template <class Epi>
struct E4;
template <>
struct E4<EFwd> {
  static __device__ __forceinline__ f32x4 apply(const EpiArgs& e, int r, int c, const f32x4& v) {
    const f32x4 z = add_bias(e.bias, c, v);
    const f32x4 a = e.hidden ? map4([&](int k) { return act_f(e.act, z[k]); }) : z;
    st4(e.out0 + (size_t)r * e.ldo + c, a);
    return a;
  }
};
template <>
struct E4<ERFwd> {
  static __device__ __forceinline__ f32x4 apply(const EpiArgs& e, int r, int c, const f32x4& v) {
    const size_t o = (size_t)r * e.ldo + c;
    const f32x4 rz = add_bias(e.rbias, c, v);
    if (e.out1) st4(e.out1 + o, rz);
    if (!e.hidden) return rz;
    const f32x4 a = ld4(e.aux0 + (size_t)r * e.lda + c);
    const f32x4 ra = map4([&](int k) { return act_d1(e.act, a[k]) * rz[k]; });
    st4(e.out2 + o, ra);
    return ra;
  }
};
template <>
struct E4<EBwd> {
  static __device__ __forceinline__ f32x4 apply(const EpiArgs& e, int r, int c, const f32x4& v) {
    const f32x4 a = ld4(e.aux0 + (size_t)r * e.lda + c);
    const f32x4 d = map4([&](int k) { return v[k] * act_d1(e.act, a[k]); });
    st4(e.out0 + (size_t)r * e.ldo + c, d);
    return d;
  }
};
template <>
struct E4<EBwdE2> {
  static __device__ __forceinline__ f32x4 apply(const EpiArgs& e, int r, int c, const f32x4& v) {
    const size_t o = (size_t)r * e.ldo + c;
    const f32x4 a = ld4(e.aux0 + (size_t)r * e.lda + c);
    const f32x4 d = map4([&](int k) { return v[k] * act_d1(e.act, a[k]); });
    st4(e.out0 + o, d);
    st4(e.out2 + o, map4([&](int k) { return v[k] * act_d2(e.act, a[k]); }));
    return d;
  }
};
template <>
struct E4<ERBwd> {
  static __device__ __forceinline__ f32x4 apply(const EpiArgs& e, int r, int c, const f32x4& v) {
    const size_t ia = (size_t)r * e.lda + c;
    const f32x4 a = ld4(e.aux0 + ia), rz = ld4(e.aux1 + ia), e2 = ld4(e.aux2 + ia);
    const f32x4 d = map4([&](int k) { return v[k] * act_d1(e.act, a[k]) + e2[k] * rz[k]; });
    st4(e.out1 + (size_t)r * e.ldo + c, d);
    return d;
  }
};
template <>
struct E4<EGNBwd> {
  static __device__ __forceinline__ f32x4 apply(const EpiArgs& e, int r, int c, const f32x4& v) {
    const f32x4 a = ld4(e.aux0 + (size_t)r * e.lda + c);
    const f32x4 d = map4([&](int k) { return v[k] * act_d1(e.act, a[k]); });
    st4(e.out1 + (size_t)r * e.ldo + c, d);
    return d;
  }
};
template <>
struct E4<ESplitStore> {
  static __device__ __forceinline__ f32x4 apply(const EpiArgs& e, int r, int c, const f32x4& v) {
    st4(e.out0 + (size_t)r * e.ldo + c, v);
    return f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
};

// One workgroup of GM x GN waves owns a (16 WM GM) x (16 WN GN) output tile,
// each wave WM x WN blocks of 16 x 16; K advances 32 at a time through S LDS
// stages filled by direct loads.  Y feeds the MFMA's row operand, so that a
// lane holds 4 consecutive columns of one output row.
template <class Epi, int YP, int WM, int WN, int GM, int GN, int S>
__device__ __forceinline__ void sgemm_body(const GemmShapeS& s, EpiArgs e) {
  if (s.skip && *s.skip) return;
  constexpr int NW = GM * GN;
  constexpr int RM = 16 * WM * GM, RN = 16 * WN * GN;
  using TX = TileP<RM, 2, NW>;
  using TY = TileP<RN, YP, NW>;
  constexpr int STAGE = TX::SIZE + TY::SIZE;
  constexpr int LPB = TX::INSTR + TY::INSTR;   // loads per block per wave
  constexpr int LPA = (LPB + WM / 2 - 1) / (WM / 2);
  static_assert(S >= 2 && S <= 4 && (S - 2) * LPB < 64, "pipeline depth");
  __shared__ __attribute__((aligned(16))) uint16_t lds[S * STAGE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / GN, wn = wave % GN;
  const int li = lane & 15, g = lane >> 4;
  int tn, tm, tz;
  tile_of(tn, tm, tz);
  const int m0 = tm * RM;
  const int n0 = tn * RN;

  const int kbps = (s.K + KG - 1) / KG;
  const int nvb = s.nseg * kbps;
  int vb0 = 0, vb1 = nvb;
  if (s.splits > 1) {
    const int per = (nvb + s.splits - 1) / s.splits;
    vb0 = tz * per;
    vb1 = min(nvb, vb0 + per);
    e.out0 += (size_t)tz * e.split_stride;
  }
  const int nblk = vb1 > vb0 ? vb1 - vb0 : 0;

  // Exponents of the segments' products.  The segment with the smaller one
  // goes first, so that the accumulators are scaled down where the segments
  // meet and cannot overflow there.
  const int a0 = *s.ex[0], b0 = *s.ey[0];
  const int a1 = s.nseg > 1 ? *s.ex[1] : a0, b1 = s.nseg > 1 ? *s.ey[1] : b0;
  const bool finite = a0 != SPLIT_NONFINITE && b0 != SPLIT_NONFINITE &&
                      a1 != SPLIT_NONFINITE && b1 != SPLIT_NONFINITE;
  const bool swap = finite && a1 + b1 < a0 + b0;
  const int E0 = swap ? a1 + b1 : a0 + b0;
  const int E1 = swap ? a0 + b0 : a1 + b1;

  f32x4 acc[WM][WN];
#pragma unroll
  for (int a = 0; a < WM; ++a)
#pragma unroll
    for (int b = 0; b < WN; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  if (finite) {
    uint32_t offx[TX::INSTR], offy[TY::INSTR];
#pragma unroll
    for (int j = 0; j < TX::INSTR; ++j) offx[j] = TX::src(s.ldx, wave, lane, j);
#pragma unroll
    for (int j = 0; j < TY::INSTR; ++j) offy[j] = TY::src(s.ldy, wave, lane, j);
    const size_t bx = (size_t)m0 * s.ldx, by = (size_t)n0 * s.ldy;
    const uint16_t* const X0 = (swap ? s.X[1] : s.X[0]) + bx;
    const uint16_t* const X1 = (swap ? s.X[0] : s.X[1]) + bx;
    const uint16_t* const Y0 = (swap ? s.Y[1] : s.Y[0]) + by;
    const uint16_t* const Y1 = (swap ? s.Y[0] : s.Y[1]) + by;
    const uint32_t lds0 = lds_address(lds);
    struct Next { const uint16_t* x; const uint16_t* y; uint32_t base; };   // base: LDS bytes
    auto next = [&](int vb, int st) {
      const bool seg = vb >= kbps;
      const int kb = seg ? vb - kbps : vb;
      return Next{(seg ? X1 : X0) + kb * TX::BK, (seg ? Y1 : Y0) + kb * TY::BK,
                  lds0 + 2u * (uint32_t)(st * STAGE)};
    };
    auto issue1 = [&](const Next& n, int j) {
      if (j < TX::INSTR)
        dma16_at(n.x + offx[j < TX::INSTR ? j : 0], n.base + 2u * (uint32_t)TX::dst(wave, j));
      else
        dma16_at(n.y + offy[j >= TX::INSTR ? j - TX::INSTR : 0],
                 n.base + 2u * (uint32_t)(TX::SIZE + TY::dst(wave, j - TX::INSTR)));
    };
    auto issue = [&](int vb, int st) {
      const Next n = next(vb, st);
#pragma unroll
      for (int j = 0; j < LPB; ++j) issue1(n, j);
    };
    // odd rows of X and odd K blocks of Y are stored negated (see the file's
    // head)
    const float sgn = li & 1 ? -1.0f : 1.0f;
    // lane (li, g) of an operand block reads k 8 g .. 8 g + 7 of its row li:
    // chunk g of each plane.  The swizzle depends only on the row within its
    // block of 16.
    const int xoff = (wm * 16 * WM + li) * TX::BK;
    const int yoff = TX::SIZE + (wn * 16 * WN + li) * TY::BK;
    const int xc0 = TX::at(li, g) * 8, xc1 = TX::at(li, 4 + g) * 8;
    const int yc0 = TY::at(li, g) * 8, yc1 = TY::at(li, 4 + g) * 8;
    const int yc2 = YP > 2 ? TY::at(li, 8 + g) * 8 : 0;
    // Temporaries of the row blocks a (odd and even); those of the last one
    // wait, with their sign, for the next K block.
    f32x4 t[2][WN];
    float tsg = 0.0f;
#pragma unroll
    for (int b = 0; b < WN; ++b) t[(WM - 1) & 1][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // addition k of the temporaries of the row block before a
    auto add1 = [&](int a, int k, float sg) {
      const int ap = (a + WM - 1) % WM;
      acc[ap][k / 4][k % 4] = fmaf(t[ap & 1][k / 4][k % 4], sg, acc[ap][k / 4][k % 4]);
    };
    auto add_last = [&]() {
#pragma unroll
      for (int k = 0; k < 4 * WN; ++k) add1(0, k, tsg);
      tsg = 0.0f;
    };
    auto compute = [&](int st, float sg, const Next& nx) {
      const uint16_t* lx = lds + st * STAGE + xoff;
      const uint16_t* ly = lds + st * STAGE + yoff;
      f16x8 y0[WN], y1[WN], y2[WN], x0[2], x1[2];
#pragma unroll
      for (int b = 0; b < WN; ++b) y0[b] = *(const f16x8*)(ly + b * 16 * TY::BK + yc0);
      x1[0] = *(const f16x8*)(lx + xc1);
      x0[0] = *(const f16x8*)(lx + xc0);
#pragma unroll
      for (int b = 0; b < WN; ++b) y1[b] = *(const f16x8*)(ly + b * 16 * TY::BK + yc1);
      if (YP > 2) {
#pragma unroll
        for (int b = 0; b < WN; ++b) y2[b] = *(const f16x8*)(ly + b * 16 * TY::BK + yc2);
      }
#pragma unroll
      for (int a = 0; a < WM; ++a) {
        const int i = a & 1;
        // The MFMAs of the row block, y0 x1 first, each followed by its share
        // of the additions of the row block before (t[1 - i], complete by
        // then), of the fragment reads of the next row block and, over the
        // first half of the rows, of the next K block's direct loads.  The order is held: left to itself the scheduler puts
        // the additions right behind their MFMAs and waits for them.  Speech
        // net, G-N solve at 16,384 rows 37.0 -> 35.8 ms, exact product 14.6
        // -> 14.0 ms, gradient at 4,096 rows 1.73 -> 1.67 ms, bit-identical.
        const float sp = a ? sg : tsg;
        constexpr int PASSES = YP > 2 ? 4 : 3, NQ = PASSES * WN, NADD = 4 * WN;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int b = q % WN, p = q / WN;
          const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
          if (p == 0) t[i][b] = mfma(y0[b], x1[i], zero);
          else if (p == PASSES - 1) t[i][b] = mfma(y0[b], x0[i], t[i][b]);
          else t[i][b] = mfma(p == 1 ? y1[b] : y2[b], x0[i], t[i][b]);
#pragma unroll
          for (int k = NADD * q / NQ; k < NADD * (q + 1) / NQ; ++k) add1(a, k, sp);
#pragma unroll
          for (int j = a * LPA; j < min((a + 1) * LPA, LPB); ++j)
            if (q == 2 * (j - a * LPA) + 1) issue1(nx, j);
          if (q == 2 && a + 1 < WM) {
            x1[1 - i] = *(const f16x8*)(lx + (a + 1) * 16 * TX::BK + xc1);
            x0[1 - i] = *(const f16x8*)(lx + (a + 1) * 16 * TX::BK + xc0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      tsg = sg;
    };
    auto steps = [&](int it0, int it1) {
      for (int it = it0; it < it1; ++it) {
        // this wave's loads of block it have landed once at most S - 2 later
        // blocks are still pending; past the last block the loads repeat it
        wait_vm<(S - 2) * LPB>();
        stage_barrier();     // every wave's loads landed; stage it - 1 is free
        const int vb = vb0 + it, kb = vb >= kbps ? vb - kbps : vb;
        compute(it % S, kb & 1 ? -sgn : sgn, next(min(vb + S - 1, vb1 - 1), (it + S - 1) % S));
      }
    };
#pragma unroll
    for (int i = 0; i < S - 1; ++i)
      if (nblk > 0) issue(vb0 + min(i, nblk - 1), i);
    // blocks of the first segment, then, on its scale, those of the second
    const int n0blk = min(max(kbps - vb0, 0), nblk);
    steps(0, n0blk);
    if (n0blk < nblk) {
      add_last();
      if (n0blk > 0 && E0 != E1) {
        const float f = ldexpf(1.0f, max(E0 - E1, -200));
#pragma unroll
        for (int a = 0; a < WM; ++a)
#pragma unroll
          for (int b = 0; b < WN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] *= f;
      }
      steps(n0blk, nblk);
    }
    add_last();
    wait_vm<0>();          // no load may land after the workgroup has ended
  } else {
    // fp32 operands straight from memory, 4 k at a time
    for (int vb = vb0; vb < vb1; ++vb) {
      const int seg = vb >= kbps ? 1 : 0;
      const int k0 = (vb - seg * kbps) * KG;
      const float* xf = s.Xf[seg];
      const float* yf = s.Yf[seg];
      for (int kk = 0; kk < KG; kk += 4) {
        const int k = k0 + kk + g;
        float x[WM], y[WN];
#pragma unroll
        for (int a = 0; a < WM; ++a) {
          const int r = m0 + (wm * WM + a) * 16 + li;
          x[a] = (r < s.M && k < s.K) ? xf[r * s.xr + k * s.xk] : 0.0f;
        }
#pragma unroll
        for (int b = 0; b < WN; ++b) {
          const int c = n0 + (wn * WN + b) * 16 + li;
          y[b] = (c < s.N && k < s.K) ? yf[c * s.yr + k * s.yk] : 0.0f;
        }
#pragma unroll
        for (int a = 0; a < WM; ++a)
#pragma unroll
          for (int b = 0; b < WN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[b], x[a], acc[a][b], 0, 0, 0);
      }
    }
  }
  // lane (li, g), register r holds row li, column 4 g + r of a block
  const int Eacc = !finite ? 0
                   : (s.nseg > 1 && vb1 > kbps ? E1 : E0) - 2 * SPLIT_TOP;
  const bool v4 = (e.ldo & 3) == 0 && ((uintptr_t)e.out0 & 15u) == 0;
  uint32_t big = 0;
#pragma unroll
  for (int a = 0; a < WM; ++a) {
    const int row = m0 + (wm * WM + a) * 16 + li;
#pragma unroll
    for (int b = 0; b < WN; ++b) {
      const int col = n0 + (wn * WN + b) * 16 + 4 * g;
      if (row < s.M && col < s.N) {
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          v[r] = ldexpf(acc[a][b][r],
                        Eacc + (finite && s.yc && col + r < s.N ? s.yc[col + r] : 0));
        if (v4 && col + 3 < s.N) {
          const f32x4 o = E4<Epi>::apply(e, row, col, v);
#pragma unroll
          for (int r = 0; r < 4; ++r) big = max(big, __float_as_uint(o[r]) & 0x7fffffffu);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (col + r < s.N)
              big = max(big, __float_as_uint(Epi::apply(e, row, col + r, v[r], 0.0f)) &
                                 0x7fffffffu);
        }
      }
    }
    // keep the scheduler from hoisting every block's loads to the top
    __builtin_amdgcn_sched_barrier(0);
  }
  if (e.amax) {
#pragma unroll
    for (int o = 32; o; o >>= 1) big = max(big, (uint32_t)__shfl_xor((int)big, o));
    if (lane == 0) e.amax[((size_t)tm * gridDim.x + tn) * NW + wave] = big;
  }
}

}  // namespace

// Two tile shapes: 256 x 256 on eight waves (each 128 x 64), one workgroup
// per CU, and 128 x 128 on four waves (each 64 x 64) where the larger tiles
// leave CUs without one.  The smaller ones have two stages, so that two
// workgroups fit a CU, or (t128d) as many as fill one CU's LDS, for grids that
// give a CU one workgroup at most: nothing else covers its loads' latency
// there.
#define HF_SGEMM_KERNEL(NAME, EPI, YP)                                          \
  extern "C" __global__ __launch_bounds__(512, 2) void NAME##_t256(GemmShapeS s, \
                                                                   EpiArgs e) { \
    sgemm_body<EPI, YP, 8, 4, 2, 4, 2>(s, e);                                   \
  }                                                                             \
  extern "C" __global__ __launch_bounds__(256, 2) void NAME##_t128(GemmShapeS s, \
                                                                   EpiArgs e) { \
    sgemm_body<EPI, YP, 4, 4, 2, 2, 2>(s, e);                                   \
  }                                                                             \
  extern "C" __global__ __launch_bounds__(256, 2) void NAME##_t128d(GemmShapeS s, \
                                                                    EpiArgs e) { \
    sgemm_body<EPI, YP, 4, 4, 2, 2, YP == 2 ? 4 : 3>(s, e);                     \
  }
#define HF_SGEMM_ROWS(NAME, EPI)            \
  HF_SGEMM_KERNEL(NAME##2, EPI, 2)          \
  HF_SGEMM_KERNEL(NAME##3, EPI, 3)
HF_SGEMM_ROWS(hf_sgemm_fwd, EFwd)
HF_SGEMM_ROWS(hf_sgemm_rfwd, ERFwd)
HF_SGEMM_ROWS(hf_sgemm_bwd, EBwd)
HF_SGEMM_ROWS(hf_sgemm_bwd_e2, EBwdE2)
HF_SGEMM_ROWS(hf_sgemm_rbwd, ERBwd)
HF_SGEMM_ROWS(hf_sgemm_gnbwd, EGNBwd)
HF_SGEMM_ROWS(hf_sgemm_part, ESplitStore)
HF_SGEMM_KERNEL(hf_sgemm_wgrad, ESplitStore, 2)

namespace {

// Largest magnitude bits of a block's threads (256), in every thread.
__device__ __forceinline__ uint32_t block_max(uint32_t v) {
  __shared__ uint32_t w[4];
#pragma unroll
  for (int o = 32; o; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = v;
  __syncthreads();
  v = max(max(w[0], w[1]), max(w[2], w[3]));
  __syncthreads();
  return v;
}

__device__ __forceinline__ uint32_t mag(float v) { return __float_as_uint(v) & 0x7fffffffu; }

}  // namespace

// amax[b] = largest magnitude bits in block b's share of R x C values
extern "C" __global__ __launch_bounds__(256) void hf_absmax(
    const float* __restrict__ in, int R, int C, int ld, uint32_t* __restrict__ amax,
    const int* __restrict__ skip) {
  if (skip && *skip) return;
  uint32_t m = 0;
  if ((ld & 3) == 0 && ((uintptr_t)in & 15u) == 0) {
    const uint32_t cq = (uint32_t)(C + 3) / 4;
    const long long n = (long long)R * cq;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (long long)gridDim.x * 256) {
      const uint32_t r = (uint32_t)i / cq, c = 4 * ((uint32_t)i - r * cq);
      const float4 v = *(const float4*)(in + (size_t)r * ld + c);
      m = max(m, mag(v.x));
      if ((int)c + 1 < C) m = max(m, mag(v.y));
      if ((int)c + 2 < C) m = max(m, mag(v.z));
      if ((int)c + 3 < C) m = max(m, mag(v.w));
    }
  } else {
    const long long n = (long long)R * C;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (long long)gridDim.x * 256) {
      const int r = (int)(i / C);
      m = max(m, mag(in[(size_t)r * ld + (i - (long long)r * C)]));
    }
  }
  m = block_max(m);
  if (threadIdx.x == 0) amax[blockIdx.x] = m;
}

// The same over the weight blocks of a parameter-layout vector (grid y = the
// block), the columns of a block with exponents cexp scaled by them.
extern "C" __global__ __launch_bounds__(256) void hf_absmax_weights(
    SplitJobs js, const int* __restrict__ skip) {
  if (skip && *skip) return;
  const SplitJob& j = js.j[blockIdx.y];
  const long long n = (long long)j.R * j.C;
  uint32_t m = 0;
  const long long stride = (long long)gridDim.x * 256;
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (j.cexp) {
    for (; i < n; i += stride) m = max(m, mag(ldexpf(j.in[i], j.cexp[(uint32_t)i % (uint32_t)j.C])));
  } else {
    for (; i + 3 * stride < n; i += 4 * stride) {
      const float a = j.in[i], b = j.in[i + stride];
      const float c = j.in[i + 2 * stride], d = j.in[i + 3 * stride];
      m = max(max(m, max(mag(a), mag(b))), max(mag(c), mag(d)));
    }
    for (; i < n; i += stride) m = max(m, mag(j.in[i]));
  }
  m = block_max(m);
  if (threadIdx.x == 0) j.amax[blockIdx.x] = m;
}

// Per-column largest magnitudes of R x C values: part[b * C + c] over row
// chunk b (grid y), 64 columns per block.  *slot = 0: the exponent slot of the
// tensor, which its split turns into SPLIT_NONFINITE where need be.
extern "C" __global__ __launch_bounds__(256) void hf_absmax_columns(
    const float* __restrict__ in, int R, int C, int ld, uint32_t* __restrict__ part,
    int* __restrict__ slot) {
  __shared__ uint32_t w[4][64];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *slot = 0;
  const int c = blockIdx.x * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
  const int per = (R + (int)gridDim.y - 1) / (int)gridDim.y;
  const int r0 = blockIdx.y * per, r1 = min(R, r0 + per);
  uint32_t m = 0;
  if (c < C) {
#pragma unroll 4
    for (int r = r0 + q; r < r1; r += 4) m = max(m, mag(in[(size_t)r * ld + c]));
  }
  w[q][threadIdx.x & 63] = m;
  __syncthreads();
  if (q == 0 && c < C)
    part[(size_t)blockIdx.y * C + c] =
        max(max(w[0][threadIdx.x], w[1][threadIdx.x]), max(w[2][threadIdx.x], w[3][threadIdx.x]));
}

// fp32 -> fp16 pairs in 64 x 64 tiles, row-major and / or transposed (through
// LDS), and the column sums of the tensor (the bias part of a weight
// gradient).  Grid x is (column tile, row chunk): a block takes the row tiles
// chunk, chunk + chunks, ...  The tensor's exponent comes from its largest
// magnitudes (every block reduces the partials once; block 0 stores the
// slot).  Bound by HBM.
namespace {
template <int PL>
__device__ __forceinline__ void split_body(const SplitJobs& js, const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ uint32_t t[64][65];
  __shared__ uint16_t t2[PL > 2 ? 64 : 1][66];
  __shared__ double bs[4][64];
  const SplitJob& j = js.j[blockIdx.y];
  const int C32 = (j.C + 31) & ~31, R32 = (j.R + 31) & ~31;
  const int tc = (C32 + 63) / 64, tr = (R32 + 63) / 64;
  if ((int)blockIdx.x >= tc * j.chunks) return;
  const int c0 = blockIdx.x % tc * 64, chunk = blockIdx.x / tc;
  int e = 0;
  __shared__ int ces[64];              // the input's column exponents
  if (j.cpart) {
    __shared__ uint32_t cm[4][64];
    const int cc = threadIdx.x & 63, q = threadIdx.x >> 6;
    uint32_t m = 0;
    if (c0 + cc < j.C)
#pragma unroll 4
      for (int b = q; b < j.namax; b += 4) m = max(m, j.cpart[(size_t)b * j.C + c0 + cc]);
    cm[q][cc] = m;
    __syncthreads();
    m = max(max(cm[0][cc], cm[1][cc]), max(cm[2][cc], cm[3][cc]));
    const int ec = slot_of(m);
    if (q == 0) {
      // (a feature that is 0 throughout gets the smallest exponent, -126, so
      // that its weights, whatever their size, do not set their tensor's)
      ces[cc] = ec == SPLIT_NONFINITE ? 0 : ec;
      if (chunk == 0 && c0 + cc < j.C) j.cexp[c0 + cc] = ces[cc];
    }
    // (the reduction's barriers also publish ces)
    if (block_max(ec == SPLIT_NONFINITE)) {
      e = SPLIT_NONFINITE;
      if (threadIdx.x == 0) *j.slot = e;
    }
  } else {
    uint32_t m = 0;
    for (int i = threadIdx.x; i < j.namax; i += 256) m = max(m, j.amax[i]);
    e = slot_of(block_max(m));
    if (blockIdx.x == 0 && threadIdx.x == 0) *j.slot = e;
  }
  const bool ok = e != SPLIT_NONFINITE;
  if (!ok && !j.bias) return;
  const int up = ok ? SPLIT_TOP - e : 0;
  const bool v4 = (j.ldi & 3) == 0 && ((uintptr_t)j.in & 15u) == 0;
  const int cl = (threadIdx.x & 15) * 4, rl = threadIdx.x >> 4;
  const int c = c0 + cl;
  int ce[4] = {up, up, up, up};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (j.cpart) ce[k] -= ces[cl + k];
    else if (j.cexp && c + k < j.C) ce[k] += j.cexp[c + k];
  }
  // negated: the odd rows of a left operand (every row-major pair; the
  // transposed pairs of a delta, whose column sums are wanted), the odd K
  // groups of a right one (the weights; the other transposed pairs)
  const uint32_t nrow = (PL == 2 ? rl & 1 : (c >> 5) & 1) ? 0x80008000u : 0u;
  const bool left_tr = PL == 2 && j.bias;
  const uint32_t ntr = left_tr ? 0x80008000u : 0u;
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  for (int rt = chunk; rt < tr; rt += j.chunks) {
    const int r0 = rt * 64;
    float v[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + rl + 16 * i;
      const float* p = j.in + (size_t)r * j.ldi + c;
      if (v4 && r < j.R && c + 3 < j.C) {
        const float4 q = *(const float4*)p;
        v[i][0] = q.x; v[i][1] = q.y; v[i][2] = q.z; v[i][3] = q.w;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[i][k] = (r < j.R && c + k < j.C) ? p[k] : 0.0f;
      }
    }
    if (j.bias) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        sum[k] += ((double)v[0][k] + (double)v[1][k]) + ((double)v[2][k] + (double)v[3][k]);
    }
    if (!ok) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + rl + 16 * i;
      f16x4 hi, lo, l2;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x = ldexpf(v[i][k], ce[k]);
        hi[k] = (_Float16)x;
        const float y = x - (float)hi[k];
        lo[k] = (_Float16)y;
        l2[k] = (_Float16)(y - (float)lo[k]);
      }
      const u32x2 hb = __builtin_bit_cast(u32x2, hi), lb = __builtin_bit_cast(u32x2, lo);
      if (j.row && r < j.R && c < C32) {
        uint16_t* d = j.row + (size_t)r * j.ldr + (c >> 5) * (KG * (PL > 2 ? j.prow : 2)) + (c & 31);
        *(u32x2*)d = hb ^ nrow;
        *(u32x2*)(d + 32) = lb ^ nrow;
        if (PL > 2 && j.prow > 2) *(u32x2*)(d + 64) = __builtin_bit_cast(u32x2, l2) ^ nrow;
      }
      if (j.tr) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          t[rl + 16 * i][cl + 2 * k] = (hb[k] & 0xffffu) | (lb[k] << 16);
          t[rl + 16 * i][cl + 2 * k + 1] = ((hb[k] >> 16) | (lb[k] & 0xffff0000u)) ^ ntr;
        }
        if (PL > 2) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            t2[rl + 16 * i][cl + k] = __builtin_bit_cast(uint16_t, (_Float16)l2[k]);
        }
      }
    }
    if (j.tr) {
      __syncthreads();
      const int cc = threadIdx.x >> 2, q = threadIdx.x & 3;
      const int r = r0 + 16 * q;               // 16 rows of column c0 + cc
      if (c0 + cc < j.C && r < R32) {
        const uint32_t ng = !left_tr && ((r >> 5) & 1) ? 0x80008000u : 0u;
        uint32_t w[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) w[i] = t[16 * q + i][cc] ^ ng;
        u32x4 hb[2], lb[2];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          hb[i >> 2][i & 3] = (w[2 * i] & 0xffffu) | (w[2 * i + 1] << 16);
          lb[i >> 2][i & 3] = (w[2 * i] >> 16) | (w[2 * i + 1] & 0xffff0000u);
        }
        uint16_t* d = j.tr + (size_t)(c0 + cc) * j.ldt + (r >> 5) * (KG * (PL > 2 ? j.ptr : 2)) +
                      (r & 31);
        *(u32x4*)d = hb[0];
        *(u32x4*)(d + 8) = hb[1];
        *(u32x4*)(d + 32) = lb[0];
        *(u32x4*)(d + 40) = lb[1];
        if (PL > 2 && j.ptr > 2) {
          u32x4 b2[2];
#pragma unroll
          for (int i = 0; i < 8; ++i)
            b2[i >> 2][i & 3] = (uint32_t)t2[16 * q + 2 * i][cc] |
                                ((uint32_t)t2[16 * q + 2 * i + 1][cc] << 16);
          *(u32x4*)(d + 64) = b2[0] ^ ng;
          *(u32x4*)(d + 72) = b2[1] ^ ng;
        }
      }
      __syncthreads();
    }
  }
  if (j.bias) {
    // over the 4 row groups of a wave, then over the waves
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      sum[k] += __shfl_xor(sum[k], 16);
      sum[k] += __shfl_xor(sum[k], 32);
      if ((threadIdx.x & 63) < 16) bs[threadIdx.x >> 6][cl + k] = sum[k];
    }
    __syncthreads();
    if (threadIdx.x < 64 && c0 + (int)threadIdx.x < j.C)
      j.bias[(size_t)chunk * j.C + c0 + threadIdx.x] =
          (bs[0][threadIdx.x] + bs[1][threadIdx.x]) + (bs[2][threadIdx.x] + bs[3][threadIdx.x]);
  }
}

}  // namespace
extern "C" __global__ __launch_bounds__(256) void hf_split2(SplitJobs js,
                                                            const int* __restrict__ skip) {
  split_body<2>(js, skip);
}
extern "C" __global__ __launch_bounds__(256) void hf_split3(SplitJobs js,
                                                            const int* __restrict__ skip) {
  split_body<3>(js, skip);
}

// out[m] = sum of the nparts partials part[b * M + m] (a weight gradient
// without split-K partials, whose reduce would do it)
extern "C" __global__ __launch_bounds__(256) void hf_bias_sum(
    const double* __restrict__ part, int nparts, int M, float* __restrict__ out,
    const int* __restrict__ skip) {
  if (skip && *skip) return;
  const int m = blockIdx.x * 256 + threadIdx.x;
  if (m >= M) return;
  double t = 0.0;
#pragma unroll 8
  for (int b = 0; b < nparts; ++b) t += part[(size_t)b * M + m];
  out[m] = (float)t;
}

namespace {

// Sum of the split-K partials in split order (fp64), then the GEMM's own
// epilogue; per-wave largest magnitudes for the split of the result.
template <class Epi, int SP>
__global__ __launch_bounds__(256) void hf_split_reduce_epi(EpiArgs e, const float* part, int M,
                                                           int N, const int* skip) {
  if (skip && *skip) return;
  const size_t mn = (size_t)M * N;
  uint32_t big = 0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < mn;
       i += (size_t)gridDim.x * 256) {
    float p[SP];
#pragma unroll
    for (int z = 0; z < SP; ++z) p[z] = part[z * mn + i];
    double v = 0.0;
#pragma unroll
    for (int z = 0; z < SP; ++z) v += (double)p[z];
    const int r = (int)(i / (size_t)N);
    big = max(big, mag(Epi::apply(e, r, (int)(i - (size_t)r * N), (float)v, 0.0f)));
  }
  if (e.amax) {
    big = block_max(big);
    if (threadIdx.x == 0) e.amax[blockIdx.x] = big;
  }
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

typedef void (*SKernel)(GemmShapeS, EpiArgs);
struct SKernels {
  SKernel t256, t128, t128d;
};
#define HF_SKERNELS(NAME) SKernels{NAME##_t256, NAME##_t128, NAME##_t128d}
#define HF_SROWS(NAME) \
  (s.yplanes == 3 ? HF_SKERNELS(NAME##3) : HF_SKERNELS(NAME##2))

// returns the number of largest-magnitude partials
int launch(const Launch& L, const char* name, const SKernels& k, const GemmShapeS& s,
           const EpiArgs& e, int ts, double flops, double bytes) {
  const dim3 grid(cdiv(s.N, ts), cdiv(s.M, ts), s.splits > 1 ? s.splits : 1);
  prof_begin(L, name);
  // at most one workgroup per CU: the whole LDS goes into stages (speech net's
  // G-N solve at 1,024 rows 10.72 -> 10.02 ms; with two workgroups per CU the
  // two-stage form is the one that fits)
  const bool deep = grid.x * grid.y * grid.z <= 256;
  hipExtLaunchKernelGGL(ts == 256 ? k.t256 : deep ? k.t128d : k.t128, grid, dim3(ts == 256 ? 512 : 256), 0,
                        L.stream, prof_a(L), prof_b(L), 0, s, e);
  prof_end(L, name, flops, bytes);
  return (int)(grid.x * grid.y) * (ts == 256 ? 8 : 4);
}

inline double mnk(const GemmShapeS& s) { return 2.0 * s.M * s.N * (double)s.K * s.nseg; }
inline double io(const GemmShapeS& s, int nout) {
  return 4.0 * (((double)s.M * s.K + (double)s.N * s.K) * s.nseg + (double)s.M * s.N * nout);
}

// A batch-row GEMM: one kernel with its epilogue or, where even 128 x 128
// tiles leave CUs without one, split-K partials and a reduce that applies it.
template <class Epi>
int launch_rows(const Launch& L, const char* name, const SKernels& k, const GemmShapeS& s,
                const EpiArgs& e, int nout) {
  const int ts = split_tile(s.M, s.N, 1);
  const long long tiles = (long long)cdiv(s.M, ts) * cdiv(s.N, ts);
  const int ktot = s.K * s.nseg;
  int sp = 1;
  while (sp < 8 && tiles * sp < 256 && ktot / (2 * sp) >= 128) sp *= 2;
  while (sp > 1 && (long long)sp * s.M * s.N > e.split_cap) sp /= 2;
  if (sp == 1) return launch(L, name, k, s, e, ts, mnk(s), io(s, nout));
  GemmShapeS ps = s;
  ps.splits = sp;
  EpiArgs pe = e;
  pe.out0 = e.split_buf;
  pe.ldo = s.N;
  pe.split_stride = (long long)s.M * s.N;
  pe.amax = nullptr;
  launch(L, name, HF_SROWS(hf_sgemm_part), ps, pe, ts, mnk(s), io(s, sp));
  const long long mn = (long long)s.M * s.N;
  const int nb = (int)std::min<long long>((mn + 255) / 256, 2048);
  // sp is a power of two from 2 to 8
  void (*kr)(EpiArgs, const float*, int, int, const int*) =
      sp == 2 ? hf_split_reduce_epi<Epi, 2>
              : sp == 4 ? hf_split_reduce_epi<Epi, 4> : hf_split_reduce_epi<Epi, 8>;
  prof_begin(L, "hf_splitk_epi");
  hipExtLaunchKernelGGL(kr, dim3(nb), dim3(256), 0, L.stream, prof_a(L), prof_b(L), 0, e,
                        (const float*)e.split_buf, s.M, s.N, s.skip);
  prof_end(L, "hf_splitk_epi", 0.0, 4.0 * (sp + nout) * (double)mn);
  return nb;
}

}  // namespace

// 256 x 256 tiles once they give every CU one (with the given split along
// K), 128 x 128 below.
int split_tile(int M, int N, int splits) {
  return (long long)cdiv(M, 256) * cdiv(N, 256) * splits >= 200 ? 256 : 128;
}

int sgemm_fwd(const Launch& L, const GemmShapeS& s, const EpiArgs& e) {
  return launch_rows<EFwd>(L, "hf_sgemm_fwd", HF_SROWS(hf_sgemm_fwd), s, e, 1);
}
int sgemm_rfwd(const Launch& L, const GemmShapeS& s, const EpiArgs& e) {
  return launch_rows<ERFwd>(L, "hf_sgemm_rfwd", HF_SROWS(hf_sgemm_rfwd), s, e,
                            e.hidden ? (e.out1 ? 3 : 2) : 1);
}
int sgemm_bwd(const Launch& L, const GemmShapeS& s, const EpiArgs& e) {
  if (e.out2)
    return launch_rows<EBwdE2>(L, "hf_sgemm_bwd_e2", HF_SROWS(hf_sgemm_bwd_e2), s, e, 3);
  return launch_rows<EBwd>(L, "hf_sgemm_bwd", HF_SROWS(hf_sgemm_bwd), s, e, 2);
}
int sgemm_rbwd(const Launch& L, const GemmShapeS& s, const EpiArgs& e) {
  return launch_rows<ERBwd>(L, "hf_sgemm_rbwd", HF_SROWS(hf_sgemm_rbwd), s, e, 4);
}
int sgemm_gnbwd(const Launch& L, const GemmShapeS& s, const EpiArgs& e) {
  return launch_rows<EGNBwd>(L, "hf_sgemm_gnbwd", HF_SROWS(hf_sgemm_gnbwd), s, e, 2);
}
void sgemm_wgrad(const Launch& L, const GemmShapeS& s, const EpiArgs& e) {
  launch(L, "hf_sgemm_wgrad", HF_SKERNELS(hf_sgemm_wgrad), s, e,
         split_tile(s.M, s.N, s.splits), mnk(s), io(s, s.splits));
}

int absmax(const Launch& L, const float* in, int R, int C, int ld, uint32_t* amax,
           const int* skip) {
  const long long q = (long long)R * ((C + 3) / 4);
  const int nb = (int)std::max<long long>(1, std::min<long long>((q + 1023) / 1024, 1024));
  prof_begin(L, "hf_absmax");
  hipExtLaunchKernelGGL(hf_absmax, dim3(nb), dim3(256), 0, L.stream, prof_a(L), prof_b(L), 0, in,
                        R, C, ld, amax, skip);
  prof_end(L, "hf_absmax", 0.0, 4.0 * (double)R * C);
  return nb;
}

void absmax_weights(const Launch& L, const SplitJobs& js, const int* skip) {
  double bytes = 0.0;
  for (int i = 0; i < js.n; ++i) bytes += 4.0 * (double)js.j[i].R * js.j[i].C;
  prof_begin(L, "hf_absmax");
  hipExtLaunchKernelGGL(hf_absmax_weights, dim3(SPLIT_WPARTS, js.n), dim3(256), 0, L.stream,
                        prof_a(L), prof_b(L), 0, js, skip);
  prof_end(L, "hf_absmax", 0.0, bytes);
}

int absmax_columns(const Launch& L, const float* in, int R, int C, int ld, uint32_t* part,
                   int* slot) {
  const int nb = std::max(1, std::min(SPLIT_CPARTS, R / 64));
  prof_begin(L, "hf_absmax");
  hipExtLaunchKernelGGL(hf_absmax_columns, dim3(cdiv(C, 64), nb), dim3(256), 0, L.stream,
                        prof_a(L), prof_b(L), 0, in, R, C, ld, part, slot);
  prof_end(L, "hf_absmax", 0.0, 4.0 * (double)R * C);
  return nb;
}

int split_chunks(int R, int C) {
  return std::max(1, std::min(std::min(cdiv(R, 64), SPLIT_BPARTS), 2048 / cdiv(C, 64)));
}

void bias_sum(const Launch& L, const double* part, int nparts, int M, float* out,
              const int* skip) {
  prof_begin(L, "hf_bias_sum");
  hipExtLaunchKernelGGL(hf_bias_sum, dim3(cdiv(M, 256)), dim3(256), 0, L.stream, prof_a(L),
                        prof_b(L), 0, part, nparts, M, out, skip);
  prof_end(L, "hf_bias_sum", 0.0, 8.0 * (double)nparts * M);
}

void split(const Launch& L, const SplitJobs& js, const int* skip) {
  double bytes = 0.0;
  int tiles = 1;
  for (int i = 0; i < js.n; ++i) {
    const SplitJob& j = js.j[i];
    bytes += (double)j.R * j.C * (4.0 + 2.0 * ((j.row ? j.prow : 0) + (j.tr ? j.ptr : 0)));
    tiles = std::max(tiles, j.chunks * cdiv(j.C, 64));
  }
  prof_begin(L, "hf_split");
  hipExtLaunchKernelGGL(js.weights ? hf_split3 : hf_split2, dim3(tiles, js.n), dim3(256), 0, L.stream,
                        prof_a(L), prof_b(L), 0, js, skip);
  prof_end(L, "hf_split", 0.0, bytes);
}

}  // namespace hfk
