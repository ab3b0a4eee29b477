// Coded products on operands split into BF16 planes beforehand: FP32, BF16x3
// and BF16 products that are large enough (bpx_plan::has_planes) and not faster in
// the fused form.
//
// One streaming pass packs the coded blocks (the encode: members summed in
// FP32, ascending) and B as BF16 planes, x = h + m + l with every plane
// rounded to nearest even, and one kernel multiplies the packed planes on
// v_mfma_f32_32x32x16_bf16 with FP32 accumulation:
//   BF16:   h.h
//   BF16x3: l.h + h.l + h.h          (two planes)
//   FP32:   m.m + h.m + m.h + h.l + l.h + h.h   (three planes)
// Three BF16 planes hold an FP32 value exactly (3 x 8 bits) and the products of
// planes are exact in FP32.  Left out are m.l, l.m and l.l: |m| <= 2^-8 and |l|
// <= 2^-17 of a value's power of two, so up to 2^-24 of a product, and the MFMA
// cuts its accumulator at the last place of a larger product before it adds the
// two.  A product on its own (one nonzero per row of A) so comes out within 3.0
// times 2^-24 of it, one and a half units in the last place, where the FP32
// matrix instruction is within half a unit, 1.0 times 2^-24 (in the Frobenius
// norm 3.1e-8 against 2.5e-8, 4.0e-8 for the mantissas that lose most).  In sums
// of many products the roundings of the accumulator count for more: a k step of
// 16 rounds it 6 times where the FP32 instruction rounds it for every 4 k,
// so the error against float64 is the smaller one: N(0,1), K = 8192: 1.4e-6
// against 1.6e-6; the 8192 x 8192 x 4096 coded product of the (12,8,4) code
// 5.2e-6 against 6.2e-6.  BF16 MFMAs run 16 times the FP32 rate, so six of them
// still are 2.7 times faster.
//
// Range: BF16 has FP32's exponents, and the conversions and MFMAs keep subnormal
// values (checked lane by lane against float64), but l's last bit lies 23 bits
// below x's first.  Packed times 2^16 even the last bit of a subnormal x, 2^-149,
// is a BF16 value, so no value is too small; sums are stored times 2^-32, exact
// down to subnormal results.  Upwards the scale costs range: a value whose scaled
// products could overflow a sum over K (PlaneParams::max_bits: 2^40 at K = 8192),
// infinities and NaN included, flags its pack block: the GEMM skips the 256-wide
// row or column panel, and an FP32 launch (gemm_f32.hip) computes it, which also
// keeps the results for infinities and NaN those of FP32 arithmetic.
//
// The two-dimensional form packs the distinct sums of A row blocks and of B
// column blocks once each, and a tile runs over all passes of its symbol, the
// K-concatenated product of a gray symbol being one longer loop: 8192^3,
// (12,8,2) on the 4 x 4 grid, 37 passes: 22.9 -> 10.8 ms per call.
//
// Packed layout: MFMA fragments.  For every 32 rows of the stacked coded
// rows (or columns of B) and 16 k there is 1 KiB per plane: lane l's eight
// values, row l % 32, k 8 (l / 32) .. +7.  The planes of one k chunk follow
// each other, chunks follow in k, 32-row panels come last; rows are padded to
// 256 and k to whole stages with zeros, so the GEMM has no edges except in
// its stores.  A stage is copied straight to LDS in whole KiB, and every LDS
// read is lane-linear (no bank conflicts, no swizzle).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <type_traits>

#include "kernels.hpp"
#include "planes.hpp"

namespace bpx {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned short us;

// ------------------------------------------------------------------ pack --
// Eight consecutive k of one row, split into P planes.
template <int P>
struct Granule {
  v8bf p[P];
};
template <int P>
__device__ __forceinline__ Granule<P> split8(const float (&x)[8]) {
  Granule<P> g;
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = x[e];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      g.p[p][e] = (__bf16)r[e];
      if (p + 1 < P) r[e] -= (float)g.p[p][e];
    }
  return g;
}
// FP32: scales the values and returns whether one is too large to be split.
__device__ __forceinline__ bool scale_up(float (&x)[8], unsigned max_bits) {
  unsigned hi = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const unsigned a = __builtin_bit_cast(unsigned, x[e]) & 0x7fffffffu;
    hi = a > hi ? a : hi;
    x[e] *= kPlaneUp;
  }
  return hi >= max_bits;
}

// 32 stacked coded rows x 256 k.  Bound by HBM: the members are read once
// each, 8 lanes to 256 consecutive bytes of a row, all loads of a member
// issued together, and the planes leave as whole 128-byte lines (8 rows of a
// fragment), so nothing goes through LDS.  8192 x 8192 (12,8,4): A and B
// packed in 245 us, 0.98 GB read and 0.65 GB written at 6.7 TB/s.
template <int P, bool GRID>
__device__ __forceinline__ void pack_a_block(const PlaneParams& p, int b, int tid) {
  const int rp = b / p.nka, kb = b - rp * p.nka;
  const int lane = tid & 63, wave = tid >> 6;
  const int r = wave * 8 + (lane >> 3), g8 = (lane & 7) * 8;
  const unsigned gr = (unsigned)rp * 32u + (unsigned)r;
  // the op (symbol) of the row, and the row of its blocks
  const int Mb = (int)p.Mb;
  const unsigned per = GRID ? (unsigned)p.tiles_m * 256u : (unsigned)Mb;
  const int32_t* ids = GRID ? p.op_ids : p.ids;
  const int op = (int)(gr / per), lr = (int)(gr - (unsigned)op * per);
  int deg = 0, id_off = 0;
  if (GRID ? lr < Mb : op < p.n_sym) {
    id_off = gld(GRID ? p.a_ops + 2 * op : p.syms + 4 * op);
    deg = gld(GRID ? p.a_ops + 2 * op + 1 : p.syms + 4 * op + 1);
  }
  const int K = (int)p.K, Kp = p.kc * 16;
  const int k0 = kb * 256 + g8;
  v4f s[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i][0] = s[i][1] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int m = 0; m < deg; ++m) {
    const int64_t row = (int64_t)gld(ids + id_off + m) * Mb + lr;
    if (row >= p.M) continue;
    const float* src = p.A + row * p.lda;
    v4f v[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = k0 + 64 * i + 4 * h;
        v[i][h] = v4f{0.f, 0.f, 0.f, 0.f};
        if (k < K) v[i][h] = *(const gv4f*)(src + k);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) s[i][h] += v[i][h];
  }
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = k0 + 64 * i;
    if (k < Kp) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = s[i][e >> 2][e & 3];
      if (P == 3) bad |= scale_up(x, p.max_bits);
      const Granule<P> g = split8<P>(x);
      us* dst = p.ap + (((int64_t)rp * p.kc + (k >> 4)) * P * 64 + ((k >> 3) & 1) * 32 + r) * 8;
#pragma unroll
      for (int q = 0; q < P; ++q) *(v8bf*)(dst + q * 512) = g.p[q];
    }
  }
  if (P == 3) {
    const int any = __syncthreads_or(bad ? 1 : 0);
    if (tid == 0) p.fa[b] = any ? 1u : 0u;
  }
}

// 64 k x 64 columns of B, transposed through LDS: rows of 64 floats written
// 16 bytes per lane and read 4 bytes per lane along n, both conflict-free.
template <int P, bool GRID>
__device__ __forceinline__ void pack_b_block(const PlaneParams& p, int b, int tid, float* t) {
  const int kb = b / p.cols64, nb = b - kb * p.cols64;
  const int64_t k0 = (int64_t)kb * 64, K = p.K, Nb = p.Nb;
  // the op of the columns (in the row-block form B itself)
  const int per = p.tiles_n * 4, op = GRID ? nb / per : 0;
  const int64_t n0 = (int64_t)(nb - op * per) * 64;
  const int id_off = GRID ? p.b_ops[2 * op] : 0, deg = GRID ? p.b_ops[2 * op + 1] : 1;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int f = tid + 256 * i;
    const int kr = f >> 4, nc = (f & 15) * 4;
    const int64_t k = k0 + kr, n = n0 + nc;
    v4f v = {0.f, 0.f, 0.f, 0.f};
    for (int m = 0; m < deg; ++m) {
      if (k >= K) break;
      const float* src = p.B + k * p.ldb + (GRID ? p.op_ids[id_off + m] * Nb : 0) + n;
      if (n + 3 < Nb) {
        v += *(const gv4f*)src;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < Nb) v[e] += src[e];
      }
    }
    *reinterpret_cast<v4f*>(t + kr * 64 + nc) = v;
  }
  __syncthreads();
  const int lane = tid & 63, wave = tid >> 6;
  const int kc = (int)(k0 >> 4) + wave;
  bool bad = false;
  if (kc < p.kc) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float* src = t + (wave * 16 + (lane >> 5) * 8) * 64 + h * 32 + (lane & 31);
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = src[e * 64];
      if (P == 3) bad |= scale_up(x, p.max_bits);
      const Granule<P> g = split8<P>(x);
      us* dst = p.bp + ((((int64_t)nb * 2 + h) * p.kc + kc) * P * 64 + lane) * 8;
#pragma unroll
      for (int q = 0; q < P; ++q) *(v8bf*)(dst + q * 512) = g.p[q];
    }
  }
  if (P == 3) {
    const int any = __syncthreads_or(bad ? 1 : 0);
    if (tid == 0) p.fb[nb * p.nkb + kb] = any ? 1u : 0u;
  }
}

template <int P, bool GRID>
__global__ __launch_bounds__(256) void pack_planes_kernel(PlaneParams p) {
  __shared__ __attribute__((aligned(16))) float t[64 * 64];
  const int b = blockIdx.x, blocks_b = p.cols64 * p.nkb;
  if (b < blocks_b)
    pack_b_block<P, GRID>(p, b, threadIdx.x, t);
  else
    pack_a_block<P, GRID>(p, b - blocks_b, threadIdx.x);
}

// ------------------------------------------------------------------ GEMM --
// 256 x 256 tiles of the stacked rows, 8 waves (2 x 4) of 128 x 64, each 4 x 2
// accumulators of 32 x 32, or (see launch_gemm_planes) 128 x 128 tiles, 4 waves
// (2 x 2) of 64 x 64.  Against the 16 x 16 MFMA the 32 x 32 one reads
// half the operand bytes per product, which counts twice here: LDS (6
// fragment reads per plane for 8 MFMAs per plane product) and power (at full
// MFMA load the clock falls to 1.6-1.8 GHz).
//
// Stages of 16 STEPS k are copied straight to LDS NBUF stages ahead.  A wave
// reads the next k step's fragments before it multiplies the current ones; in
// the last step of a stage it first waits for its own copies of the next
// stage and its LDS reads of this one, then for the other waves, and refills
// the buffer.  One barrier per 48 MFMAs and wave, with the copies of up to
// NBUF - 1 stages in flight across it.  FP32's planes do not fit twice in the
// registers, so there the order of the plane products lets each plane be
// read while others multiply (m first, h under m.m, l under h.m and m.h, the
// next m under the rest).
//
// Measured on 8192 x 8192 x 4096, 36 coded products (618 GFLOP): FP32 2.35
// ms, 1.58 PFLOP/s of BF16 products, MFMA busy 0.83 at 1.6 GHz (0.75 ms less
// on zero operands: power, not issue, is what is left); the FP32 MFMA
// kernels took 4.64 ms.  BF16x3 1.27 ms against 2.31 ms for the kernel that
// encodes and splits A while staging.
// The small tile reads 4/3 of the fragments per product, at two workgroups to
// a CU: FP32 and BF16x3 stay within 85 % of the MFMA rate, BF16 is bound by LDS
// (192 of 128 cycles).  1999 x 1500 x 1001: FP32 GEMM and sums 55 -> 42 us;
// 3000 x 2060 x 1530, all 12 workers' rows: BF16 GEMM 53 -> 35 us.
// k steps per stage and stages in LDS (144, 128 and 128 KiB).
template <int P>
struct Cfg;
template <>
struct Cfg<1> {
  static constexpr int STEPS = 2, NBUF = 4;
};
template <>
struct Cfg<2> {
  static constexpr int STEPS = 2, NBUF = 2;
};
template <>
struct Cfg<3> {
  static constexpr int STEPS = 1, NBUF = 3;
};

// One k step's fragments of a wave.
template <int P, int S>
struct Frags {
  v8bf a[S / 64][P], b[2][P];
};

template <int P, int S>
struct Tile {
  static constexpr int STEPS = Cfg<P>::STEPS, NBUF = Cfg<P>::NBUF;
  static constexpr int MI = S / 64, WN = S / 64;  // 32-row accumulators; waves side by side
  static constexpr int PANELS = S / 32, THREADS = 128 * WN;
  static constexpr int RPB = STEPS * P * 1024;  // bytes of one 32-row panel per stage
  static constexpr int STAGE = 2 * PANELS * RPB;  // A's panels, then B's
  static constexpr int L = 2 * STEPS * P;       // 1 KiB copies per wave per stage
  static constexpr int LDS = NBUF * STAGE;
};

// The copies of one tile's stages to LDS, in order: wave w copies panels 2w,
// 2w + 1 of a stage (the first half of the waves A's, the others B's).
template <int P, bool GRID, int S>
struct Feed {
  using T = Tile<P, S>;
  const char *ap, *bp;
  const int32_t* passes;
  int64_t rp_stride;
  int wave, pad_m, pad_n, mt, nt;
  int soff0, voff, lds0;
  int nk1, n_pass;  // stages of a pass; passes
  int pass, kp;     // the next stage
  v4i rsrc;

  __device__ __forceinline__ void set_pass() {
    int64_t panel = wave < T::WN ? mt : nt;
    if (GRID)
      panel += wave < T::WN ? (int64_t)passes[2 * pass] * pad_m
                            : (int64_t)passes[2 * pass + 1] * pad_n;
    const uint64_t src =
        reinterpret_cast<uint64_t>(wave < T::WN ? ap : bp) + (uint64_t)(panel * T::PANELS * rp_stride);
    rsrc = v4i{(int)src, (int)(src >> 32) & 0xffff, (int)(T::PANELS * rp_stride), kRsrcWord3};
#pragma unroll
    for (int c = 0; c < 4; ++c) rsrc[c] = __builtin_amdgcn_readfirstlane(rsrc[c]);
  }
  // Tile (mt, nt) of symbol si from stage kt0 on.
  __device__ __forceinline__ void open(const PlaneParams& p, char* lds, int wave_, int lane, int si,
                                       int mt_, int nt_) {
    ap = reinterpret_cast<const char*>(p.ap);
    bp = reinterpret_cast<const char*>(p.bp);
    passes = GRID ? p.passes + 2 * p.sym_passes[2 * si] : nullptr;
    n_pass = GRID ? p.sym_passes[2 * si + 1] : 1;
    rp_stride = (int64_t)p.kc * P * 1024;
    nk1 = p.kc / T::STEPS;
    wave = wave_;
    pad_m = p.pad_m;
    pad_n = p.pad_n;
    mt = mt_;
    nt = nt_;
    soff0 = wave % T::WN * 2 * (int)rp_stride;
    voff = lane * 16;
    lds0 = (int)(uintptr_t)(lds_addr)lds + 2 * wave * T::RPB;
  }
  // Starts at stage kt0 of nk and copies what fits in LDS.
  __device__ __forceinline__ void start(int kt0, int nk) {
    pass = GRID ? kt0 / nk1 : 0;
    kp = kt0 - pass * nk1;
    set_pass();
#pragma unroll
    for (int i = 0; i < T::NBUF; ++i)
      if (i < nk) copy(i * T::STAGE);
  }
  __device__ __forceinline__ void copy(int st) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      copy_panel<T::STEPS * P>(rsrc, lds0 + st + u * T::RPB, voff,
                               soff0 + u * (int)rp_stride + kp * T::RPB);
    ++kp;
    if (GRID && kp == nk1) {
      kp = 0;
      if (++pass < n_pass) set_pass();
    }
  }
};

// Multiplies the nk stages of a started feed.
template <int P, bool GRID, int S>
__device__ __forceinline__ void multiply(Feed<P, GRID, S>& feed, int nk, const char* lds, int wave,
                                         int lane, Acc<S / 64>& acc) {
  using T = Tile<P, S>;
  constexpr int MI = T::MI;
  constexpr int NBUF = T::NBUF, STAGE = T::STAGE, RPB = T::RPB, L = T::L;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const int a_base = wave / T::WN * MI * RPB + lane * 16;
  const int b_base = (T::PANELS + wave % T::WN * 2) * RPB + lane * 16;
  auto read_a = [&](Frags<P, S>& f, const char* st, int s, int q) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
      f.a[i][q] = *reinterpret_cast<const v8bf*>(st + a_base + i * RPB + (s * P + q) * 1024);
  };
  auto read_b = [&](Frags<P, S>& f, const char* st, int s, int q) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      f.b[j][q] = *reinterpret_cast<const v8bf*>(st + b_base + j * RPB + (s * P + q) * 1024);
  };
  auto mul = [&](const Frags<P, S>& f, auto pa, auto pb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            f.a[i][decltype(pa)::value], f.b[j][decltype(pb)::value], acc[i][j], 0, 0, 0);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, P >= 2 ? 1 : 0>;
  using I2 = std::integral_constant<int, P == 3 ? 2 : 0>;

  // Ends a stage: the next stage has landed everywhere, and this stage's
  // buffer may be refilled.  MORE: a further stage is copied into it; the loop
  // body that copies has no branch, so that nothing is moved from one side of
  // the barrier to the other.
  using More = std::integral_constant<bool, true>;
  using Last = std::integral_constant<bool, false>;
  auto turn = [&](auto more) __attribute__((always_inline)) {
    wait_counts<decltype(more)::value ? (NBUF - 2) * L : 0, true>();
    barrier();
  };

  // first stage
  if (nk >= NBUF)
    wait_counts<(NBUF - 1) * L, true>();
  else
    wait_counts<0, true>();
  barrier();

  int cur = 0;
  if constexpr (P == 3 && S == 128) {
    // One wave per SIMD or two, 24 MFMAs each: all of the next stage's fragments
    // are read while this stage's multiply, from a second set of registers.
    Frags<P, S> f0, f1;
    auto read = [&](Frags<P, S>& f, const char* st) __attribute__((always_inline)) {
#pragma unroll
      for (int q : {1, 0, 2}) {
        read_a(f, st, 0, q);
        read_b(f, st, 0, q);
      }
    };
    read(f0, lds);
    auto stage = [&](auto more, bool refill, const Frags<P, S>& f, Frags<P, S>& g)
                     __attribute__((always_inline)) {
      const int nxt = cur + STAGE == NBUF * STAGE ? 0 : cur + STAGE;
      const char* next = lds + nxt;  // (past the last stage: read, never used)
      turn(more);
      mul(f, I1{}, I1{});
      __builtin_amdgcn_sched_barrier(0);
      read_a(g, next, 0, 1);
      read_b(g, next, 0, 1);
      __builtin_amdgcn_sched_barrier(0);
      mul(f, I0{}, I1{});
      __builtin_amdgcn_sched_barrier(0);
      read_a(g, next, 0, 0);
      if (refill) feed.copy(cur);
      __builtin_amdgcn_sched_barrier(0);
      mul(f, I1{}, I0{});
      __builtin_amdgcn_sched_barrier(0);
      read_b(g, next, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      mul(f, I0{}, I2{});
      __builtin_amdgcn_sched_barrier(0);
      read_b(g, next, 0, 2);
      read_a(g, next, 0, 2);
      __builtin_amdgcn_sched_barrier(0);
      mul(f, I2{}, I0{});
      mul(f, I0{}, I0{});
      __builtin_amdgcn_sched_barrier(0);
      cur = nxt;
    };
    int kt = 0;
    for (; kt + 2 <= nk - NBUF; kt += 2) {
      stage(More{}, true, f0, f1);
      stage(More{}, true, f1, f0);
    }
    for (; kt < nk; kt += 2) {
      stage(Last{}, kt < nk - NBUF, f0, f1);
      if (kt + 1 < nk) stage(Last{}, false, f1, f0);
    }
  } else if constexpr (P == 3) {
    Frags<P, S> f;
    read_a(f, lds, 0, 1);
    read_b(f, lds, 0, 1);
    auto stage = [&](auto more) __attribute__((always_inline)) {
      const int nxt = cur + STAGE == NBUF * STAGE ? 0 : cur + STAGE;
      const char* here = lds + cur;
      const char* next = lds + nxt;
      read_a(f, here, 0, 0);
      read_b(f, here, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      mul(f, I1{}, I1{});
      __builtin_amdgcn_sched_barrier(0);
      read_b(f, here, 0, 2);
      read_a(f, here, 0, 2);
      __builtin_amdgcn_sched_barrier(0);
      mul(f, I0{}, I1{});
      mul(f, I1{}, I0{});
      __builtin_amdgcn_sched_barrier(0);
      turn(more);
      read_a(f, next, 0, 1);  // (past the last stage: read, never used)
      read_b(f, next, 0, 1);
      if (decltype(more)::value) feed.copy(cur);
      __builtin_amdgcn_sched_barrier(0);
      mul(f, I0{}, I2{});
      mul(f, I2{}, I0{});
      mul(f, I0{}, I0{});
      __builtin_amdgcn_sched_barrier(0);
      cur = nxt;
    };
    for (int kt = 0; kt < nk - NBUF; ++kt) stage(More{});
    for (int kt = nk - NBUF < 0 ? 0 : nk - NBUF; kt < nk; ++kt) stage(Last{});
  } else {
    static_assert(P == 3 || T::STEPS == 2, "two k steps per stage");
    Frags<P, S> f0, f1;
    auto read = [&](Frags<P, S>& f, const char* st, int s) __attribute__((always_inline)) {
#pragma unroll
      for (int q = P - 1; q >= 0; --q) {
        read_a(f, st, s, q);
        read_b(f, st, s, q);
      }
    };
    auto step = [&](const Frags<P, S>& f) __attribute__((always_inline)) {
      if constexpr (P == 2) {
        mul(f, I1{}, I0{});
        mul(f, I0{}, I1{});
      }
      mul(f, I0{}, I0{});
    };
    read(f0, lds, 0);
    auto stage = [&](auto more) __attribute__((always_inline)) {
      const int nxt = cur + STAGE == NBUF * STAGE ? 0 : cur + STAGE;
      read(f1, lds + cur, 1);
      __builtin_amdgcn_sched_barrier(0);
      step(f0);
      __builtin_amdgcn_sched_barrier(0);
      turn(more);
      read(f0, lds + nxt, 0);  // (past the last stage: read, never used)
      if (decltype(more)::value) feed.copy(cur);
      __builtin_amdgcn_sched_barrier(0);
      step(f1);
      __builtin_amdgcn_sched_barrier(0);
      cur = nxt;
    };
    for (int kt = 0; kt < nk - NBUF; ++kt) stage(More{});
    for (int kt = nk - NBUF < 0 ? 0 : nk - NBUF; kt < nk; ++kt) stage(Last{});
  }
}

template <int P, bool GRID, int S>
__global__ __launch_bounds__(2 * S, 2) void gemm_planes_kernel(PlaneParams p) {
  using T = Tile<P, S>;
  __shared__ __attribute__((aligned(1024))) char lds[T::LDS];
  __shared__ float* rows[S];  // output rows of the tile

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // The tile and its stages: all of its passes over K, or one piece of them.
  // Row blocks give each XCD one contiguous range of tiles; in the
  // two-dimensional form, whose symbols come longest first, each XCD takes its
  // share of every symbol (tile_at).
  int lin = (int)blockIdx.x, piece = -1;
  if (lin >= p.full) {
    piece = lin - p.full;
    lin = p.full + piece / p.split;
  } else if (!GRID) {
    lin = xcd_remap(lin, p.full);
  }
  int si, mt, nt;
  tile_at<GRID>(p, lin, &si, &mt, &nt);
  Feed<P, GRID, S> feed;
  feed.open(p, lds, wave, lane, si, mt, nt);
  int kt0 = 0, kt1 = feed.nk1 * feed.n_pass;
  if (piece >= 0) {
    const int s = piece % p.split, n = kt1;
    kt0 = (int)((int64_t)s * n / p.split);
    kt1 = (int)((int64_t)(s + 1) * n / p.split);
  }
  feed.start(kt0, kt1 - kt0);

  if (tid < S) rows[tid] = out_row<GRID>(p, si, (unsigned)(mt * S + tid));
  if (P == 3) {
    unsigned bad = 0;
    for (int i = 0; i < feed.n_pass; ++i) {
      // (of the 256-wide panels, which the FP32 launch computes whole)
      const int64_t pa = (GRID ? (int64_t)feed.passes[2 * i] * p.pad_m + mt : mt) / (256 / S);
      const int64_t pb = (GRID ? (int64_t)feed.passes[2 * i + 1] * p.pad_n + nt : nt) / (256 / S);
      for (int t = tid; t < 8 * p.nka; t += T::THREADS) bad |= p.fa[pa * 8 * p.nka + t];
      for (int t = tid; t < 4 * p.nkb; t += T::THREADS) bad |= p.fb[pb * 4 * p.nkb + t];
    }
    const int left = __syncthreads_or((int)bad);
    if (tid == 0) p.ft[((int64_t)si * p.tiles_m + mt) * p.tiles_n + nt] = left ? 1u : 0u;
    if (left) {
      wait_counts<0, false>();  // no copy may land in LDS that is no longer ours
      return;
    }
  }

  Acc<T::MI> acc;
  multiply<P, GRID, S>(feed, kt1 - kt0, lds, wave, lane, acc);
  if (piece >= 0) {
    store_part<T::MI, T::WN>(acc, p.part + (int64_t)piece * (S * S), wave, lane);
    return;
  }
  store_tile<T::MI, T::WN, P == 3>(acc, rows, (int64_t)nt * S, p.Nb, wave, lane);
}

// Grouped form, persistent: workgroup w multiplies tiles tiles[wstart[w]] ..
// tiles[wstart[w + 1] - 1] (GroupTile.lin = mt tiles_n + nt of the product).
// The next tile's first stages are copied, and its output rows looked up,
// before this tile is stored, so a tile costs its stores but not the latency
// of the first copies.  rows alternates: a wave that has passed a tile's first
// barrier knows that every wave has stored the tile before it.  256 products
// (256-4096, BF16x3): GEMM 4.8 -> 3.2 ms, MFMA busy 0.73 at 1.53 GHz.
template <int P>
__global__ __launch_bounds__(NT) void gemm_planes_grouped_kernel(
    const GroupDesc* __restrict__ d, const GroupTile* __restrict__ tiles,
    const int32_t* __restrict__ wstart) {
  __shared__ __attribute__((aligned(1024))) char lds[Tile<P, 256>::LDS];
  __shared__ float* rows[2][256];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int t = wstart[blockIdx.x];
  const int t1 = wstart[blockIdx.x + 1];
  if (t >= t1) return;
  Feed<P, false, 256> feed;
  int n_tile, Nb;
  auto begin = [&](int i, int buf) __attribute__((always_inline)) {
    const PlaneParams& p = d[__builtin_amdgcn_readfirstlane(tiles[i].prod)].pl;
    const int lin = __builtin_amdgcn_readfirstlane(tiles[i].lin);
    const int mt = lin / p.tiles_n, nt = lin - mt * p.tiles_n;
    feed.open(p, lds, wave, lane, 0, mt, nt);
    feed.start(0, feed.nk1);
    if (tid < 256) rows[buf][tid] = out_row<false>(p, 0, (unsigned)mt * 256u + (unsigned)tid);
    n_tile = nt * 256;
    Nb = (int)p.Nb;
    // (in registers before the loop: a scalar load in flight there would make
    // every LDS wait of the loop wait for everything)
    asm volatile("" ::"s"(n_tile), "s"(Nb));
  };
  begin(t, 0);
  for (int buf = 0; t < t1; ++t, buf ^= 1) {
    Acc<4> acc;
    multiply<P, false, 256>(feed, feed.nk1, lds, wave, lane, acc);
    const int n0 = n_tile, cols = Nb;
    if (t + 1 < t1) begin(t + 1, buf ^ 1);
    store_tile<4, 4>(acc, rows[buf], n0, cols, wave, lane);
  }
}

// Grouped pack: block b belongs to product bmap[b] and is block
// b - bstart[bmap[b]] of that product's pack grid.  Bound by HBM: 1.41 ms for
// the 256 products' 9.2 GB, 6.5 TB/s with the members that L2 still holds
// (splitting B alone took 0.69 ms).
template <int P>
__global__ __launch_bounds__(256) void pack_planes_grouped_kernel(const GroupDesc* __restrict__ d,
                                                                  const int64_t* __restrict__ bstart,
                                                                  const int32_t* __restrict__ bmap) {
  __shared__ __attribute__((aligned(16))) float t[64 * 64];
  const int prod = __builtin_amdgcn_readfirstlane(bmap[blockIdx.x]);
  const PlaneParams p = d[prod].pl;
  const int b = (int)(blockIdx.x - bstart[prod]), blocks_b = p.cols64 * p.nkb;
  if (b < blocks_b)
    pack_b_block<P, false>(p, b, threadIdx.x, t);
  else
    pack_a_block<P, false>(p, b - blocks_b, threadIdx.x);
}

// Sums the pieces of each split tile of S x S, one float4 per thread, in
// piece order (fixed, so results do not depend on scheduling).
template <bool GRID, int S, bool SCALED>
__global__ __launch_bounds__(256) void planes_reduce_kernel(PlaneParams p) {
  constexpr int BLOCKS = S * S / 1024;
  const int t = blockIdx.x / BLOCKS;
  const int e = (blockIdx.x % BLOCKS << 8) + threadIdx.x;
  const int row = e / (S / 4), col = e % (S / 4) * 4;
  int si, mt, nt;
  tile_at<GRID>(p, p.full + t, &si, &mt, &nt);
  float* out = out_row<GRID>(p, si, (unsigned)(mt * S + row));
  const int64_t n = (int64_t)nt * S + col;
  if (!out || n >= p.Nb) return;
  const float* src = p.part + (int64_t)t * p.split * (S * S) + row * S + col;
  v4f sum = *reinterpret_cast<const v4f*>(src);
  for (int k = 1; k < p.split; ++k)
    sum += *reinterpret_cast<const v4f*>(src + (int64_t)k * (S * S));
  if (SCALED) sum *= kPlaneDown;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (n + c < p.Nb) out[n + c] = sum[c];
}

}  // namespace

void planes_tiles(PlaneParams* p) {
  const int64_t rows = p->grid > 1 ? p->Mb : (int64_t)p->n_sym * p->Mb;
  p->tile = 256;
  p->tiles_m = p->pad_m = (int32_t)((rows + 255) / 256);
  p->tiles_n = p->pad_n = (int32_t)((p->Nb + 255) / 256);
  p->row_group = p->grid > 1 ? 4 : 8;
  p->nka = (p->kc + 15) / 16;
  p->nkb = (p->kc + 3) / 4;
}
static void tiles_of_128(PlaneParams* p) {
  const int64_t rows = p->grid > 1 ? p->Mb : (int64_t)p->n_sym * p->Mb;
  p->tile = 128;
  p->tiles_m = (int32_t)((rows + 127) / 128);
  p->tiles_n = (int32_t)((p->Nb + 127) / 128);
  p->pad_m *= 2;
  p->pad_n *= 2;
}

int64_t planes_group_setup(PlaneParams* p) {
  planes_tiles(p);
  return (int64_t)p->cols64 * p->nkb + (int64_t)p->rows32 * p->nka;
}

hipError_t launch_pack_planes_grouped(const GroupDesc* d, const int64_t* bstart,
                                      const int32_t* bmap, int64_t blocks, int32_t planes,
                                      hipStream_t stream) {
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(planes == 2 ? pack_planes_grouped_kernel<2> : pack_planes_grouped_kernel<1>,
                     dim3((unsigned)blocks), dim3(256), 0, stream, d, bstart, bmap);
  return hipGetLastError();
}

hipError_t launch_gemm_planes_grouped(const GroupDesc* d, const GroupTile* tiles,
                                      const int32_t* wstart, int32_t planes, int32_t grid,
                                      hipStream_t stream) {
  hipLaunchKernelGGL(planes == 2 ? gemm_planes_grouped_kernel<2> : gemm_planes_grouped_kernel<1>,
                     dim3((unsigned)grid), dim3(NT), 0, stream, d, tiles, wstart);
  return hipGetLastError();
}

hipError_t launch_pack_planes(const PlaneParams& p0, hipStream_t stream) {
  PlaneParams p = p0;
  planes_tiles(&p);
  const unsigned blocks = (unsigned)p.cols64 * (unsigned)p.nkb + (unsigned)p.rows32 * (unsigned)p.nka;
  void (*k)(PlaneParams) = p.grid > 1      ? pack_planes_kernel<3, true>
                           : p.planes == 3 ? pack_planes_kernel<3, false>
                           : p.planes == 2 ? pack_planes_kernel<2, false>
                                           : pack_planes_kernel<1, false>;
  hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, stream, p);
  return hipGetLastError();
}

// Passes the busiest of S CUs runs when every symbol's per tiles, all but the
// last skip ones, longest symbols first, each go to the CU that is free first.
static int64_t longest_queue(const int32_t* passes, int64_t n_sym, int64_t per, int64_t skip,
                             int64_t S) {
  std::map<int64_t, int64_t> cus = {{0, S}};  // passes dealt -> CUs
  int64_t left = n_sym * per - skip;
  for (int64_t i = 0; i < n_sym && left > 0; ++i)
    for (int64_t n = std::min(per, left); n > 0;) {
      const auto first = cus.begin();
      const int64_t m = std::min(n, first->second), to = first->first + passes[i];
      if (m == first->second)
        cus.erase(first);
      else
        first->second -= m;
      cus[to] += m;
      n -= m;
      left -= m;
    }
  return cus.rbegin()->first;
}

// The last round: R of the tiles, each split into q pieces of its K range
// whose sums a second kernel forms, where a model of both says that ends
// sooner: rounds of pieces at the measured time of a k chunk of one tile, 6 us
// for the second launch and 0.125 us per 256 x 256 piece written and read back
// (4 TB/s).  (Summed by the last of a tile's workgroups instead, over counters,
// the second launch is saved and 5 to 25 us lost: the pieces are then read at
// the pace of few CUs.)  R is what the products of all tiles leave over after
// whole rounds (everything if that is less than one round); in the
// two-dimensional form only one-pass tiles, which come last, can fill up a
// round, and the symbols' passes (host memory) give the time of the others:
// 4096 x 2048 x 4096, 288 large tiles of up to three passes, takes three
// passes' time on 256 CUs however the last tiles are split.
double planes_split(PlaneParams* p, const int32_t* passes, int64_t T, double us, int min_chunks,
                    int64_t S) {
  const bool grid = p->grid > 1;
  const int64_t per = grid ? T / p->n_sym : 1;
  const int64_t units = grid ? p->n_passes * per : T;
  const int64_t rest = units <= S ? units : units % S;  // of the last round
  const int64_t R = units <= S ? T : grid ? std::min(rest, p->n_single * per) : rest;
  const int64_t ru = units <= S ? units : R;
  const int64_t pieces = (int64_t)p->part_tiles * (256 / p->tile) * (256 / p->tile);
  const double piece_us = 0.125 * p->tile * p->tile / 65536.0, tile_us = (double)p->kc * us;
  const double before = tile_us * (double)(grid ? longest_queue(passes, p->n_sym, per, R, S)
                                                : (units - rest) / S);
  int64_t best_q = 1;
  double best = grid      ? tile_us * (double)longest_queue(passes, p->n_sym, per, 0, S)
                : rest > 0 ? before + tile_us
                           : before;
  for (int64_t q = 2; q <= 16 && R > 0; ++q) {
    if (R * q > pieces || p->kc / q < min_chunks) break;
    const double t = before + (double)((ru * q + S - 1) / S) * tile_us / (double)q + 6.0 +
                     piece_us * (double)(R * q);
    if (t < best) {
      best = t;
      best_q = q;
    }
  }
  p->split = (int32_t)best_q;
  p->full = (int32_t)(best_q > 1 ? T - R : T);
  return best;
}

hipError_t launch_planes_reduce(const PlaneParams& p, int64_t T, hipStream_t stream) {
  if (p.full == T) return hipSuccess;
  const bool small = p.tile == 128;
  void (*k)(PlaneParams) =
      p.grid > 1 ? (small ? planes_reduce_kernel<true, 128, true> : planes_reduce_kernel<true, 256, true>)
      : p.planes == 3
          ? (small ? planes_reduce_kernel<false, 128, true> : planes_reduce_kernel<false, 256, true>)
          : (small ? planes_reduce_kernel<false, 128, false> : planes_reduce_kernel<false, 256, false>);
  hipLaunchKernelGGL(k, dim3((unsigned)((T - p.full) * (small ? 16 : 64))), dim3(256), 0, stream, p);
  return hipGetLastError();
}

template <int S>
static hipError_t launch_gemm_tiles(const PlaneParams& p, int64_t T, hipStream_t stream) {
  const unsigned blocks = (unsigned)(p.full + (T - p.full) * p.split);
  void (*k)(PlaneParams) = p.grid > 1      ? gemm_planes_kernel<3, true, S>
                           : p.planes == 3 ? gemm_planes_kernel<3, false, S>
                           : p.planes == 2 ? gemm_planes_kernel<2, false, S>
                                           : gemm_planes_kernel<1, false, S>;
  hipLaunchKernelGGL(k, dim3(blocks), dim3(2 * S), 0, stream, p);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_planes_reduce(p, T, stream);
}

// Tiles of 256 x 256 or 128 x 128, whichever the model of planes_split expects
// to end sooner.  Times of a k chunk on a CU (per tile; two workgroups of the
// small tile share a CU at the time of two): large ones FP32 2.0, BF16x3 1.05,
// BF16 0.45 us, small ones 0.53, 0.295 and 0.123 us.  So the large tile is the
// faster one per product (8192 x 4096 x 4096: FP32 1.15 against 1.22 ms, BF16
// 284 against 313 us), the small one where large tiles leave CUs idle or have
// to be split (all of coded_gemm: 2000 x 4000 x 2000, 64 large tiles: BF16 73
// -> 59, BF16x3 121 -> 113, FP32 187 -> 181 us; 1500^3: 36 -> 26, 52 -> 46, 71
// -> 67 us).  The large tile keeps what the model puts within 7 %: it draws less
// power, which the model leaves out (Construction B, 8192 x 8192 x 4096, 3.75
// rounds of large tiles: FP32 4.52 ms, 4.76 in small ones).
static double choose_tiles(PlaneParams* p, const int32_t* passes, int64_t S, int64_t* tiles) {
  planes_tiles(p);
  const int64_t syms = p->grid > 1 ? p->n_sym : 1, lim = 0x7fffffff / 32;
  const int64_t T = (int64_t)p->tiles_m * p->tiles_n * syms;
  *tiles = T;
  if (T > lim) return 0.0;
  PlaneParams s = *p;
  tiles_of_128(&s);
  const int64_t T128 = (int64_t)s.tiles_m * s.tiles_n * syms;
  const int P = p->planes;
  const double t = planes_split(p, passes, T, P == 3 ? 2.0 : P == 2 ? 1.05 : 0.45, 8, S);
  if (T128 > lim) return t;
  const double t128 =
      planes_split(&s, passes, T128, P == 3 ? 0.53 : P == 2 ? 0.295 : 0.123, 8, S);
  if (t128 >= 0.93 * t) return t;
  *p = s;
  *tiles = T128;
  return t128;
}

int32_t planes_parts(const PlaneParams& p, int64_t T) {
  const int64_t pieces = (T - p.full) * p.split, per = (256 / p.tile) * (256 / p.tile);
  return p.split > 1 ? (int32_t)((pieces + per - 1) / per) : 0;
}

int32_t planes_part_tiles(const PlaneParams& p0, const int32_t* passes) {
  PlaneParams p = p0;
  int64_t T;
  choose_tiles(&p, passes, 256, &T);
  return planes_parts(p, T);
}

hipError_t launch_gemm_planes(PlaneParams* p, const int32_t* passes, hipStream_t stream) {
  int64_t T;
  choose_tiles(p, passes, device_cu_count(), &T);
  if (T > 0x7fffffff / 32) return hipErrorInvalidValue;
  return p->tile == 128 ? launch_gemm_tiles<128>(*p, T, stream)
                        : launch_gemm_tiles<256>(*p, T, stream);
}

// 15 us of launches (FP32, with its second product launch, 18), the GEMM's
// rounds, and the operands, planes and products at 4 TB/s.  512^3 with eight
// symbols: FP32 29 us expected, 27.7 measured, BF16x3 25 and 23.8, BF16 20 and
// 17.5; 768 x 1024 x 768: 38 and 36, 32 and 30, 25 and 23.7.
double planes_us(const PlaneParams& p0) {
  PlaneParams p = p0;
  int64_t T;
  const double gemm = choose_tiles(&p, nullptr, device_cu_count(), &T);
  const double K = (double)p.K, N = (double)p.N, rows = (double)p.n_sym * (double)p.Mb;
  const double bytes = 4.0 * K * ((double)p.M + N) + 4.0 * p.planes * K * (rows + N) +
                       12.0 * rows * N;
  return (p.planes == 3 ? 18.0 : 15.0) + gemm + bytes / 4e6;
}

}  // namespace bpx
