// Host-side objects of libbpx: codes, plans, and the device tables a plan
// uploads.  Integer work only; no HIP types appear here.
#pragma once

#include "../../include/bpx.h"

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

struct bpx_code {
  int32_t kind = 0;
  int32_t n = 0, k = 0, b = 0;
  std::vector<int32_t> col_ptr;   // n + 1
  std::vector<int32_t> sym_ptr;   // n_sym + 1
  std::vector<uint16_t> sym_data; // ids, ascending per symbol
  int32_t n_sym() const { return (int32_t)sym_ptr.size() - 1; }
  int32_t kb() const { return k * b; }
  int32_t deg(int32_t g) const { return sym_ptr[g + 1] - sym_ptr[g]; }
  int32_t max_degree() const;
};

// One step of the device peel program (see plan.cpp).
struct PeelStep {
  int32_t s;        // data block written / loaded
  int32_t src;      // Y slot of the releaser, or -1 when X_s already sits in C
  int32_t nsub;     // number of subtrahends
  int32_t sub_off;  // offset of the subtrahends' LDS slots in the slot list
  int32_t f64;      // 1: accumulate in FP64 (depth > 4), 0: FP32 Kahan
  int32_t slot;     // LDS slot that keeps X_s for later steps, or -1
  int32_t write;    // 1: write X_s to C
  int32_t brow;     // block row of s (s itself for row blocks)
  int32_t bcol;     // block column of s (0 for row blocks)
};

// Operands of a two-dimensional plan's products on split planes: the distinct
// sums of A row blocks (a_ops) and of B column blocks (b_ops) its symbols
// need, each {offset, count} into ids (ascending blocks), and per GEMM-table
// symbol its passes, {A op, B op} each: one pass for a symbol whose members
// share a block, one per member for any other.
struct PlaneOps {
  std::vector<int32_t> a_ops, b_ops, ids;  // {offset, count}
  std::vector<int32_t> sym_passes;         // {first pass, passes}
  std::vector<int32_t> passes;             // {A op, B op}
  std::vector<int32_t> counts;             // passes of each symbol
};

struct bpx_plan {
  // copy of the code (a plan outlives nothing it does not own)
  bpx_code code;
  int32_t mode = 0, prec = 0;
  int64_t M = 0, K = 0, N = 0, Mb = 0;
  // Two-dimensional form: data block s = r * grid + c is A row block r times
  // B column block c (Mb rows, Nb columns); grid = 1 is the row-block form
  // (Nb = N).
  int32_t grid = 1;
  int64_t Nb = 0;

  bool decodable = false;
  int32_t prefix_m = 0;
  int32_t depth_max = 0;
  std::vector<int32_t> computed;    // ascending g
  std::vector<int32_t> dest;        // per computed: Y slot or -1-s
  std::vector<int32_t> releaser;    // per data id
  std::vector<int32_t> depth;       // per data id
  std::vector<int32_t> sub_ptr;     // kb + 1
  std::vector<uint16_t> sub_data;
  std::vector<int32_t> unrecovered;
  int32_t n_yslots = 0;

  // device peel program
  std::vector<PeelStep> steps;
  std::vector<int32_t> step_subs;   // LDS slots of subtrahends
  int32_t n_lds_slots = 0;

  // The same program for the peel whose values all stay in LDS, one record per
  // step: {src, nsub | f64 << 8 | write << 9, eight subtrahends a byte each (the
  // steps that recover them), brow | bcol << 16, where in peel_more the other
  // subtrahends are, 0, 0}.  Empty if the program has more steps than a byte names.
  static constexpr int32_t kPeelRec = 8;
  std::vector<int32_t> peel_recs, peel_more;

  // GEMM symbol table: per computed symbol {id_off, deg, dest, 0} + ids
  std::vector<int32_t> gemm_syms;
  std::vector<int32_t> gemm_ids;

  // Fused peel program (every recovered block has a step; src is the
  // releaser's LDS Y tile) and, per GEMM-table entry, its Y tile or -1.
  std::vector<PeelStep> fused_steps;
  std::vector<int32_t> fused_subs;
  std::vector<int32_t> fused_ytile;
  int32_t n_ytiles = 0;

  PlaneOps ops;  // grid > 1

  // device copies
  void* dev_block = nullptr;
  int32_t dev_id = -1;
  const int32_t* d_gemm_syms = nullptr;
  const int32_t* d_gemm_ids = nullptr;
  const PeelStep* d_steps = nullptr;
  const int32_t* d_step_subs = nullptr;
  const PeelStep* d_fused_steps = nullptr;
  const int32_t* d_fused_subs = nullptr;
  const int32_t* d_fused_ytile = nullptr;
  const int32_t* d_peel_recs = nullptr;
  const int32_t* d_peel_more = nullptr;
  const int32_t* d_ops = nullptr;  // PlaneOps: a_ops, b_ops, ids, sym_passes, passes

  size_t y_bytes() const { return (size_t)n_yslots * (size_t)Mb * (size_t)Nb * sizeof(float); }
  // K rounded up to the BF16 kernels' 32-wide k step
  int64_t kp() const { return (K + 31) / 32 * 32; }
  static size_t align256(size_t x) { return (x + 255) / 256 * 256; }
  // Workspace: [Y slots][Bt_hi][Bt_lo] for the BF16 precisions.
  size_t bt_plane_bytes() const { return align256((size_t)N * (size_t)kp() * 2); }
  // FP8: [Y][Aq][Aq2][sA][Bq][sB] with Mb, K, N rounded up to 128.
  int64_t r128(int64_t x) const { return (x + 127) / 128 * 128; }
  bool is_fp8() const { return prec == BPX_PREC_FP8 || prec == BPX_PREC_FP8X2; }
  bool is_bf16() const { return prec == BPX_PREC_BF16 || prec == BPX_PREC_BF16X3; }
  // FP32 plans whose shape takes the 256 x 256 tiling reserve room for the
  // split-K partial tiles of its last round: at most 4 pieces per tile and
  // at most 256 partial tiles (one per CU) of 256 x 256 FP32.
  size_t part_bytes() const {
    if (grid != 1 || prec != BPX_PREC_F32 || Mb % 256 != 0 || N % 256 != 0 || K % 32 != 0 ||
        M % Mb != 0)
      return 0;
    const int64_t T = (int64_t)computed.size() * (Mb / 256) * (N / 256);
    const int64_t tiles = T * 4 < 256 ? T * 4 : 256;
    return (size_t)tiles * 256 * 256 * sizeof(float);
  }
  // Offsets in bytes of the workspace parts:
  //   F32:    [0] Y, [1] split-K partial tiles (256 x 256 tiling only)
  //   BF16*:  [0] Y, [1] Bt_hi, [2] Bt_lo (BF16x3)
  //   FP8*:   [0] Y, [1] Aq, [2] Aq2 (FP8x2), [3] sA, [4] Bq, [5] sB
  // Missing parts get the offset of the next part (size 0).  [6] = total.
  void layout(size_t off[7]) const {
    size_t b = align256(y_bytes());
    for (int i = 0; i < 7; ++i) off[i] = 0;
    if (is_bf16()) {
      off[1] = b;
      b += bt_plane_bytes();
      off[2] = b;
      if (prec == BPX_PREC_BF16X3) b += bt_plane_bytes();
      for (int i = 3; i < 7; ++i) off[i] = b;
    } else if (is_fp8()) {
      const size_t nc = computed.size();
      const size_t aq = align256(nc * (size_t)r128(Mb) * (size_t)r128(K));
      off[1] = b;
      b += aq;
      off[2] = b;
      if (prec == BPX_PREC_FP8X2) b += aq;
      off[3] = b;
      b += align256(nc * (size_t)(r128(Mb) / 128) * (size_t)(r128(K) / 128) * 4);
      off[4] = b;
      b += align256((size_t)r128(N) * (size_t)r128(K));
      off[5] = b;
      b += align256((size_t)(r128(K) / 128) * (size_t)(r128(N) / 128) * 4);
      off[6] = b;
    } else {
      off[1] = b;
      b += part_bytes();
      for (int i = 2; i < 7; ++i) off[i] = b;
    }
    off[6] = b;
  }
  // Bytes the kernels that read A and B directly need: what a call has to
  // bring at least.
  size_t base_bytes() const {
    size_t off[7];
    layout(off);
    return off[6];
  }
  // Operands packed in the order of MFMA fragments (gemm_planes.hip: BF16
  // planes; gemm_fp8.hip: codes).
  int32_t planes() const {
    switch (prec) {
      case BPX_PREC_F32: return 3;
      case BPX_PREC_BF16X3: case BPX_PREC_FP8X2: return 2;
      default: return 1;
    }
  }
  // k chunks of the packed operands, whole stages of the GEMM: 16 wide, for
  // FP8 64 wide (and K padded to 128).
  int64_t plane_kc() const {
    if (is_fp8()) return r128(K) / 64;
    return planes() == 3 ? (K + 15) / 16 : (K + 31) / 32 * 2;
  }
  static int64_t r256(int64_t x) { return (x + 255) / 256 * 256; }
  int64_t plane_rows() const {
    return grid > 1 ? (int64_t)(ops.a_ops.size() / 2) * r256(Mb)
                    : r256((int64_t)computed.size() * Mb);
  }
  int64_t plane_cols() const {
    return grid > 1 ? (int64_t)(ops.b_ops.size() / 2) * r256(Nb) : r256(N);
  }
  // Products of Mb x K and K x Nb blocks the computed symbols take.
  int64_t n_products() const {
    return grid > 1 ? (int64_t)ops.passes.size() / 2 : (int64_t)computed.size();
  }
  // ... and at most one symbol (summed without rounding to FP32 in between).
  int32_t max_passes() const {
    int32_t n = 1;
    for (int32_t c : ops.counts) n = std::max(n, c);
    return n;
  }
  const int32_t* pass_counts() const { return ops.counts.data(); }
  double n_macs() const { return (double)n_products() * (double)Mb * (double)K * (double)Nb; }
  int64_t plane_tiles() const {
    return grid > 1 ? (int64_t)computed.size() * (r256(Mb) / 256) * (r256(Nb) / 256)
                    : plane_rows() / 256 * (plane_cols() / 256);
  }
  // Whether the products run on packed operands where the workspace holds them
  // (small row-block products may still take the fused form).  us, direct and
  // packed, at the lines:
  //   BF16  from 2^24 multiply-adds, below which nearly all of either way is
  //     launches (400 x 64 x 400 on Construction B, 2^24: 14 and 13; 2048 x 300 x
  //     2048 on the (12,8,4) code: 41 and 34).
  //   FP32  packs six bytes per value, so it takes longer K to pay: (12,8,4), 1024 x
  //     K x 1024: K = 128 28 and 29, 192 35 and 32, 300 47 and 38; 321 x 3256 x 451
  //     256 and 45; past 2^31 it does for any K.
  //   Two-dimensional  from K = 128 and 2^25 where a tile's K over all its passes is
  //     more than 288 (Table I's code, two passes, 1058 x 320 x 3224 46 and 45, 1229
  //     x 320 x 1032 53 and 41; (12,8,2) 2895 x 256 x 720 84 and 83; uncoded 1035 x
  //     256 x 1568 21 and 26, 3809 x 320 x 304 25 and 26, 649 x 448 x 464 32 and 24),
  //     from 2^29 otherwise (uncoded 2191 x 128 x 1256, 2^28.4, 18 and 21; 3076 x 128
  //     x 1344, 2^29, 27 and 27; 5116 x 128 x 1744 42 and 35).
  //   FP8  past 2^31 only, since up to there a call leaves the codes and scales that
  //     layout() names in the workspace.  It costs time where blocks have under 128
  //     rows (packed rows are not padded: (12,8,4) 1024^3 FP8 38 and 36, 640 x 2048 x
  //     640 89 and 38; Mojette (24,16,8) 1024^3 65 and 29) and saves some for FP8x2
  //     in blocks of whole 128s ((6,4,2) 1024^3 34 and 40, FP8 29 and 29).
  bool has_planes() const {
    const double macs = n_macs();
    const bool enough = is_fp8()    ? false
                        : is_bf16() ? macs > 16777216.0
                        : grid > 1  ? K >= 128 && macs > (K * max_passes() > 288 ? 33554432.0
                                                                                 : 536870912.0)
                                    : macs > 16777216.0 && K > 192;
    return (enough || macs > 2147483648.0) && planes_fit();
  }
  // Bytes of 32 packed rows (columns) and one k chunk, all planes.
  int64_t a_chunk_bytes() const { return (int64_t)planes() * (is_fp8() ? 2048 : 1024); }
  int64_t b_chunk_bytes() const { return is_fp8() ? 2048 : a_chunk_bytes(); }
  // The kernels' 32-bit indices and offsets hold.
  bool planes_fit() const {
    if (K % 4 != 0) return false;
    const int64_t lim = (int64_t)1 << 31, kc = plane_kc();
    if (plane_rows() >= lim || plane_cols() >= lim || plane_tiles() >= lim / 32 ||
        (double)n_products() * (double)kc >= (double)lim || kc * a_chunk_bytes() * 8 >= lim)
      return false;
    if (is_fp8())
      return (double)kc * (double)plane_rows() < (double)lim &&
             (double)kc * (double)plane_cols() < (double)lim &&
             (double)computed.size() * (double)r128(Mb) / 128 * (double)kc < (double)lim;
    return plane_rows() / 32 * ((kc + 15) / 16) + plane_cols() / 64 * ((kc + 3) / 4) < lim;
  }
  size_t packed_bytes() const {
    return (size_t)plane_kc() * ((size_t)plane_rows() / 32 * a_chunk_bytes() +
                                 (size_t)plane_cols() / 32 * b_chunk_bytes());
  }
  // Workspace of a grouped product on split planes (no flags, no partial tiles).
  size_t group_plane_bytes() const { return align256(y_bytes()) + align256(packed_bytes()); }
  // Offsets of the plane parts, from the start of the workspace: packed A,
  // packed B, flags (FP32) or scales (FP8) of A, of B (FP32: then of up to four
  // tiles per 256 x 256); [4] the end, what a call on packed operands has to
  // bring.  Of the parts of layout() these calls use Y and, for FP32, the partial
  // tiles; BF16's planes of B give up their place (packed A and B are larger), the
  // FP8 codes keep theirs.
  void plane_layout(size_t off[5]) const {
    const size_t kc = (size_t)plane_kc();
    size_t b = is_bf16() ? align256(y_bytes()) : base_bytes(), sa = 0, sb = 0;
    if (planes() == 3) {
      sa = (size_t)(plane_rows() / 32) * ((kc + 15) / 16) * 4;
      sb = ((size_t)(plane_cols() / 64) * ((kc + 3) / 4) + 4 * (size_t)plane_tiles()) * 4;
    } else if (is_fp8()) {
      sa = kc / 2 * (size_t)plane_rows();
      sb = kc / 2 * (size_t)(plane_cols() / 128) * 4;
    }
    off[0] = b;
    b += (size_t)plane_rows() / 32 * kc * a_chunk_bytes();
    off[1] = b;
    b += (size_t)plane_cols() / 32 * kc * b_chunk_bytes();
    off[2] = b;
    b += align256(sa);
    off[3] = b;
    b += align256(sb);
    off[4] = b;
  }
  size_t plane_bytes() const {
    size_t off[5];
    plane_layout(off);
    return off[4];
  }
  // Partial tiles (256 x 256 FP32) of tiles split along K: at most 16 pieces of a
  // tile, of 8 k chunks (FP8: 4) at least.  part_want is what the split takes on
  // 256 CUs; a card run in partitions of fewer CUs splits otherwise, which gets
  // room for 256 as long as that is no more than the packed operands themselves.
  static constexpr int32_t kPartTiles = 512;
  static constexpr size_t kPartBytes = 65536 * sizeof(float);
  int32_t part_want = 0;
  int32_t plane_part_tiles() const {
    const int64_t q = std::min<int64_t>(16, plane_kc() / (is_fp8() ? 4 : 8));
    if (q < 2) return 0;
    const int64_t room = std::min<int64_t>(256, (int64_t)(packed_bytes() / kPartBytes));
    return (int32_t)std::max<int64_t>(part_want, std::min<int64_t>(plane_tiles() * q, room));
  }
  // Where a call with this much workspace keeps them, and how many: behind the
  // packed operands, or in layout()'s place for them if that holds more.
  int32_t plane_parts(size_t have, size_t* at) const {
    size_t off[7];
    layout(off);
    const size_t end = plane_bytes(), most = (size_t)plane_part_tiles();
    const size_t own = std::min(most, part_bytes() / kPartBytes);
    const size_t behind = have > end ? std::min(most, (have - end) / kPartBytes) : 0;
    *at = behind >= own ? end : off[1];
    return (int32_t)std::max(own, behind);
  }
  size_t ws_bytes() const {
    if (!has_planes()) return base_bytes();
    const size_t most = (size_t)plane_part_tiles();
    return plane_bytes() + (most > part_bytes() / kPartBytes ? most * kPartBytes : 0);
  }
};

namespace bpx {

// SplitMix64 (Steele, Lea, Flood 2014).
struct SplitMix64 {
  uint64_t state;
  explicit SplitMix64(uint64_t seed) : state(seed) {}
  uint64_t next() {
    state += 0x9E3779B97F4A7C15ull;
    uint64_t z = state;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  uint64_t below(uint64_t n) { return next() % n; }
};

// Thread-local error message.
void set_error(const std::string& msg);
const char* get_error();

// code.cpp
int build_code(const bpx_code_params& p, bpx_code* out, std::string* err);

// plan.cpp
struct PeelResult {
  std::vector<int32_t> releaser;  // -1 = unknown
  std::vector<int32_t> depth;
  int32_t n_known = 0;
  int32_t rounds = 0;
};
// Round-based peel over the given symbols (ids into code), canonical releaser.
PeelResult peel(const bpx_code& code, const std::vector<int32_t>& syms);
// grid = 1: row blocks of A; grid = m > 1: the two-dimensional form (k*b = m^2).
int make_plan(const bpx_code& code, const int32_t* arrival, int32_t n_arrival, int32_t n_lost,
              int32_t mode, int64_t M, int64_t K, int64_t N, int32_t prec, int32_t grid,
              bpx_plan* plan, std::string* err);

}  // namespace bpx

