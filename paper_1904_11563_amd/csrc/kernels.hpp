// Device kernels of libbpx: parameter blocks and host-side launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "host.hpp"

namespace bpx {

// Coded GEMM: for every computed symbol i (table entry {id_off, deg, dest, g}
// in syms[4*i..4*i+3], member ids in ids[id_off .. id_off+deg)),
//   out_i = (sum over members s of A rows [s*Mb, s*Mb+Mb)) . B
// where out_i is Y slot dest (Mb x N, ld N) or, for dest < 0, the C rows of
// block -1-dest (ld ldc, rows past M skipped).
struct GemmParams {
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  float* C;
  int64_t ldc;
  float* Y;
  int64_t M, K, N, Mb;
  const int32_t* syms;
  const int32_t* ids;
  int32_t n_sym;
  int32_t tiles_m, tiles_n;
  int32_t prec;  // bpx_prec
  int32_t group_m;  // tile order: row panels per group (1 = row-major order)
  // Remainder mode of the 256 x 256 tiling (FP32 only): when wide_rem is set,
  // tiles_m / tiles_n count 256 x 256 tiles and block b computes sub-tile
  // b % per of 256 x 256 tile wide_lin0 + b / per (per = sub-tiles per tile).
  int32_t wide_rem;
  int32_t wide_lin0;
  // Split-K mode of the 256 x 256 tiling: when wide_split = P > 0, block b
  // computes k-slice range (b % P) of tile wide_lin0 + b / P into partial
  // tile b of part (256 x 256 FP32, row-major); a reduction kernel sums the
  // P partials of each tile in piece order and writes the tile's output.
  int32_t wide_split;
  int32_t part_tiles;  // capacity of part in 256 x 256 tiles (0: no split-K)
  float* part;
  // Two-dimensional form (launch_coded_gemm_2d): data block s = r * grid + c
  // is A row block r times B column block c; Y slots are Mb x Nb.
  int32_t grid;
  int32_t pad1;
  int64_t Nb;
  // BF16 / BF16x3: B split into transposed bf16 planes (N x kp, k contiguous)
  const unsigned short* bt_hi;
  const unsigned short* bt_lo;
  int64_t kp;
  // FP32 launch that only computes the tiles the split planes leave out:
  // PlaneParams::ft, null for an ordinary launch, the edge of those tiles and
  // how many (per symbol in the two-dimensional form)
  const unsigned* left;
  int32_t left_edge, left_m, left_n;
};

// FP8 path (see gemm_fp8.hip for the workspace layout).
struct Fp8Params {
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  float* C;
  int64_t ldc;
  float* Y;
  int64_t M, K, N, Mb;
  int64_t Mbp, Kp, Np;  // Mb, K, N rounded up to 128
  const int32_t* syms;
  const int32_t* ids;
  int32_t n_sym;
  int32_t tiles_m, tiles_n;
  unsigned char* aq;
  unsigned char* aq2;  // null unless FP8x2
  float* sa;
  unsigned char* bq;
  float* sb;
  int32_t group_m;  // wide tiles: row panels per group of the tile order (0: default)
};

// Peel: see PeelStep in host.hpp.
struct PeelParams {
  const float* Y;
  float* C;
  int64_t ldc;
  int64_t M, N, Mb;
  const PeelStep* steps;
  const int32_t* subs;
  int32_t nsteps;
  int32_t nslots;
  int32_t nsubs;  // length of subs
  // bpx_plan::peel_recs, peel_more; null if the program does not fit
  const int32_t* recs;
  const int32_t* more;
  int32_t nload;  // leading steps that only fetch a block from C
  // Block layout: data block s covers C rows (s / grid) * Mb .., columns
  // (s % grid) * Nb ..; Y slots are Mb x Nb.  grid = 1, Nb = N for row
  // blocks (the vector form assumes that layout).
  int32_t grid;
  int64_t Nb;
};
// Bytes of LDS a peel workgroup holds besides its slots: the step program
// (steps, then subs), staged once per workgroup.
__host__ __device__ inline size_t peel_program_bytes(int32_t nsteps, int32_t nsubs) {
  return ((size_t)nsteps * sizeof(PeelStep) + (size_t)nsubs * 4 + 15) / 16 * 16;
}

// Standalone encode: out block i (Mb x K, ld K) = sum of member blocks of A.
struct EncodeParams {
  const float* A;
  int64_t lda;
  float* out;
  int64_t M, K, Mb;
  const int32_t* syms;
  const int32_t* ids;
  int32_t n_sym;
};

// Tile shapes compiled for the GEMM.
struct TileShape {
  int32_t bm, bn, bk;
};
int32_t gemm_tile_count();
TileShape gemm_tile_shape(int32_t t);

hipError_t launch_coded_gemm(const GemmParams& p, int32_t tile, hipStream_t stream);
// Whether a product's blocks are small enough for the two-dimensional
// kernels' 32-bit offsets.
bool gemm_2d_fits(const GemmParams& p);
// FP32 coded GEMM of the two-dimensional form (64 x 128 tiles).
// tile: the FP32 tile shape chosen for the call; the 256 x 256 shapes (4-6)
// take the wide 2-D kernel where the blocks allow it, others 64 x 128.
hipError_t launch_coded_gemm_2d(const GemmParams& p, int32_t tile, hipStream_t stream);

// ---------------------------------------------------------- split planes --
// Products whose operands are split into BF16 planes beforehand (see
// gemm_planes.hip).  FP32 operands are packed times 2^kPlaneScale, which the
// stores take back: the last bit of any FP32 value, 2^-149, is then the smallest
// BF16 value, so three planes hold everything down to zero.  A magnitude from
// PlaneParams::max_bits up (infinities and NaN among them) is not split: the
// FP32 kernels compute the tiles it belongs to.
constexpr int kPlaneScale = 16;
constexpr float kPlaneUp = 1 << kPlaneScale, kPlaneDown = 1.f / (kPlaneUp * kPlaneUp);
// The bits of the largest power of two whose scaled products cannot overflow a
// sum of n of them: 2^40 for n = 8192, 2^47 for one.
inline unsigned plane_max_bits(double n) {
  int lg = 0;
  while (lg < 100 && (double)(1ull << std::min(lg, 62)) < n) ++lg;
  return (unsigned)(127 + (126 - lg) / 2 - kPlaneScale) << 23;
}
struct PlaneParams {
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  float* C;
  int64_t ldc;
  float* Y;
  int64_t M, K, N, Mb;
  const int32_t* syms;
  const int32_t* ids;
  int32_t n_sym;
  int32_t planes;      // 1: BF16, 2: BF16x3, 3: FP32 (FP8: codes of A, 1 or 2)
  unsigned short* ap;  // packed planes of the stacked coded rows
  unsigned short* bp;  // packed planes of B's columns
  unsigned* fa;        // planes == 3: per pack block, 1 if it holds a value
  unsigned* fb;        //   that is not split
  float* part;         // partial 256 x 256 tiles of the last round
  int32_t part_tiles;  // how many part holds
  int32_t kc;          // 16-wide k chunks of the packed operands (FP8: 64-wide)
  int32_t rows32, cols64;  // 32-row panels of ap, 64-column pack blocks of bp
  // Two-dimensional form (grid > 1): ap and bp hold the distinct sums of A row
  // blocks and of B column blocks the symbols need, op by op, every op padded
  // to 256 rows or columns; see PlaneOps in host.hpp for the tables.
  int32_t grid;
  int64_t Nb;
  const int32_t* a_ops;   // {id offset, degree} per op
  const int32_t* b_ops;
  const int32_t* op_ids;
  const int32_t* sym_passes;  // {first pass, passes} per symbol
  const int32_t* passes;      // {A op, B op} per pass
  int32_t n_passes, n_single;  // passes of all symbols; symbols with one
  // FP8 (launch_pack_fp8, launch_gemm_fp8_packed): E8M0 scale bytes per 128-wide
  // k chunk, of every stacked row and of every 128 columns (four equal bytes)
  unsigned char* ea;
  unsigned* eb;
  // set by the launcher
  int32_t tiles_m, tiles_n;   // per symbol in the two-dimensional form
  int32_t tile;        // edge of the GEMM's tiles, 256 or 128
  int32_t pad_m, pad_n;       // as packed, an op padded to 256 rows and columns
  int32_t row_group;   // row panels per group of the tile order
  int32_t nka, nkb;    // pack blocks along k of A (256 wide) and of B (64 wide)
  int32_t full, split; // tiles computed whole; K pieces of each of the others
  unsigned* ft;        // planes == 3: per tile, 1 if it belongs to a panel with a value
  unsigned max_bits;   //   that is not split; bits of the smallest such magnitude
};
hipError_t launch_pack_planes(const PlaneParams& p, hipStream_t stream);
// passes: in the two-dimensional form the passes of each symbol (host memory).
// Sets the tiles it chose.
hipError_t launch_gemm_planes(PlaneParams* p, const int32_t* passes, hipStream_t stream);
// Time that pack, product and peel of a row-block product are expected to take, in us.
double planes_us(const PlaneParams& p);
hipError_t launch_pack_fp8(const PlaneParams& p, hipStream_t stream);
hipError_t launch_gemm_fp8_packed(const PlaneParams& p, hipStream_t stream);
// tiles_m, tiles_n of a row-block product; how many of its T tiles run whole
// and in how many K pieces the others (full, split), given the time of one
// k chunk of a tile in us (returns the time it expects); and the kernel that
// sums the pieces.
void planes_tiles(PlaneParams* p);
double planes_split(PlaneParams* p, const int32_t* passes, int64_t T, double us, int min_chunks,
                    int64_t cus);
// Room for partial tiles (of 256 x 256) that a split takes; that a product's split
// takes on 256 CUs (host work only).
int32_t planes_parts(const PlaneParams& p, int64_t T);
int32_t planes_part_tiles(const PlaneParams& p, const int32_t* passes);
int32_t fp8_part_tiles(const PlaneParams& p);
hipError_t launch_planes_reduce(const PlaneParams& p, int64_t T, hipStream_t stream);

int32_t bf16_tile_count();
TileShape bf16_tile_shape(int32_t t);
// Tile 4 is the flat-row tiling (tiles over all symbols' stacked rows); it
// needs K a multiple of 32 and offsets within 31 bits (bf16_flat_ok).
bool bf16_tile_is_flat(int32_t t);
bool bf16_flat_ok(const GemmParams& p);
// Bt_hi[n][k] = bf16(B[k][n]), Bt_lo = bf16(B - Bt_hi) (bt_lo may be null),
// zero for k in [K, Kp).
hipError_t launch_split_b(const float* B, int64_t ldb, int64_t K, int64_t N, int64_t Kp,
                          void* bt_hi, void* bt_lo, hipStream_t stream);
hipError_t launch_coded_gemm_bf16(const GemmParams& p, int32_t tile, hipStream_t stream);
// ------------------------------------------------------------ grouped --
// Per-product descriptor of a grouped launch (device memory).
struct GroupDesc {
  GemmParams g;      // tiles_m / tiles_n set for the product's tile shape
  PlaneParams pl;    // the product on split planes (planes_group_setup), instead of g
  PeelParams pe;
  int32_t b_tn, b_tk;  // split-B grid of the product (64 x 64 tiles)
  int32_t tile;        // tile shape index
  int32_t pad;
};
// A grouped GEMM tile: product and tile index inside that product's grid.
struct GroupTile {
  int32_t prod;
  int32_t lin;
};
// Grouped split-B: block b belongs to product bmap[b] and is block
// b - bstart[bmap[b]] of that product's grid.
hipError_t launch_split_b_grouped(const GroupDesc* d, const int64_t* bstart, const int32_t* bmap,
                                  int64_t total_blocks, hipStream_t stream);
// Persistent grouped BF16 / BF16x3 GEMM over a tile list of one tile shape.
hipError_t launch_gemm_bf16_grouped(const GroupDesc* d, const GroupTile* tiles, int32_t n_tiles,
                                    int32_t tile, int32_t split, int32_t grid,
                                    hipStream_t stream);
// Groups on split planes: sets the launch fields of a product and returns its
// pack blocks; one pack launch over all products' blocks (as split-B's); and
// one persistent GEMM launch, workgroup w taking tiles[wstart[w]] ..
// tiles[wstart[w + 1] - 1].
int64_t planes_group_setup(PlaneParams* p);
hipError_t launch_pack_planes_grouped(const GroupDesc* d, const int64_t* bstart,
                                      const int32_t* bmap, int64_t blocks, int32_t planes,
                                      hipStream_t stream);
hipError_t launch_gemm_planes_grouped(const GroupDesc* d, const GroupTile* tiles,
                                      const int32_t* wstart, int32_t planes, int32_t grid,
                                      hipStream_t stream);
// Compute units of the current device (cached per device; 256 if unknown).
int device_cu_count();

// Grouped peel: block b belongs to product pmap[b] and is block
// b - pstart[pmap[b]] of that product's peel grid; workgroup w of the
// persistent grid runs blocks wstart[w] .. wstart[w + 1] - 1.  The grid is
// peel_grouped_grid(...) workgroups (as many as the CUs hold at once).
int64_t peel_grouped_grid(int64_t total_blocks, int32_t max_slots, size_t max_program);
hipError_t launch_peel_grouped(const GroupDesc* d, const int64_t* pstart, const int32_t* pmap,
                               const int64_t* wstart, int64_t grid, int32_t max_slots,
                               size_t max_program, hipStream_t stream);

// ------------------------------------------------------ fused peel --
// One launch computing every computed symbol's product for a 16 x BN output
// tile of all data blocks and peeling it in LDS (see fused.hip).  syms/ids
// as in GemmParams (GEMM-table order); ytile[i]: the LDS Y tile of computed
// symbol i, or -1 if it releases nothing; steps/subs: the fused peel
// program (src = Y tile of the releaser, every recovered block written).
struct FusedParams {
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  float* C;
  int64_t ldc;
  int64_t M, K, N, Mb;
  const int32_t* syms;
  const int32_t* ids;
  const int32_t* ytile;
  int32_t n_sym;
  int32_t n_ytiles;
  int32_t n_ids;  // length of ids
  // The plan's device tables are one block; the kernel copies the span from
  // syms to the end of ytile to LDS in one pass (word offsets from syms).
  int32_t blob_words;
  int32_t off_ids, off_steps, off_subs, off_ytile;
  const PeelStep* steps;
  const int32_t* subs;
  int32_t nsteps;
  int32_t nsubs;
  int32_t nslots;
  int32_t prec;
  // set by fused_configure
  int32_t jn;  // column tile = 16 jn
  int32_t tiles_m, tiles_n;
  int32_t kb;       // data blocks
  int32_t max_deg;  // largest degree of a computed symbol
  int32_t kg;       // k per A-stage group (32 or 64)
  int32_t stages;   // LDS buffers of a k group (3: copied straight to LDS)
  int32_t pair;     // two workgroups share a CU
  int64_t kp;  // K rounded up to the k group
};
// Picks the tile width and checks that the workgroup's LDS fits; false if
// the fused form cannot run this product (precision or LDS).
bool fused_configure(FusedParams* p);
size_t fused_lds_bytes(const FusedParams& p);
hipError_t launch_fused(const FusedParams& p, hipStream_t stream);
// Time a configured product is expected to take, in us.
double fused_us(const FusedParams& p);

hipError_t launch_quant_a(const Fp8Params& p, hipStream_t stream);
hipError_t launch_quant_b(const Fp8Params& p, hipStream_t stream);
int32_t fp8_tile_count();
hipError_t launch_coded_gemm_fp8(const Fp8Params& p, int32_t tile, hipStream_t stream);
hipError_t launch_peel(const PeelParams& p, hipStream_t stream);
hipError_t launch_encode(const EncodeParams& p, hipStream_t stream);

}  // namespace bpx
