// Device helpers of the kernels that multiply packed operands on 256 x 256
// tiles with eight waves (2 x 4) of 128 x 64, or on 128 x 128 tiles with four
// (2 x 2) of 64 x 64 (gemm_planes.hip, gemm_fp8.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace bpx {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_addr;
typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) v4f gv4f;

constexpr int NT = 512;  // threads of a 256 x 256 tile's workgroup
constexpr int kRsrcWord3 = 0x00020000;  // gfx9 raw buffer, 32-bit elements

__device__ __forceinline__ int32_t gld(const int32_t* ptr) {
  return *(const __attribute__((address_space(1))) int32_t*)ptr;
}

// Waits until at most VM vector-memory operations of this wave are in
// flight, and for all of its LDS operations if LGKM.
template <int VM, bool LGKM>
__device__ __forceinline__ void wait_counts() {
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4) | ((LGKM ? 0 : 15) << 8));
}
__device__ __forceinline__ void barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Copies COUNT consecutive KiB of a packed panel straight to LDS, 16 bytes
// per lane (the instruction offset moves both addresses).  Written as asm
// because the compiler would wait for every copy in flight before any later
// LDS read; the waits are the loop's own.
template <int COUNT>
__device__ __forceinline__ void copy_panel(v4i rsrc, int lds, int voff, int soff) {
  if constexpr (COUNT == 1)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds"
                 ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
  if constexpr (COUNT == 2)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:1024 lds"
                 ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
  if constexpr (COUNT == 3)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:2048 lds"
                 ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
  if constexpr (COUNT == 4)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen offset:3072 lds"
                 ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
  static_assert(COUNT >= 1 && COUNT <= 4, "KiB per panel and stage");
}
// 64 words straight to LDS, lane l the word at voff.
__device__ __forceinline__ void copy_words(v4i rsrc, int lds, int voff, int soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
               "buffer_load_dword %1, %2, %3 offen lds"
               ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// Consecutive workgroups go to different XCDs; each XCD gets a contiguous
// range of tiles.
__device__ __forceinline__ int xcd_remap(int lin, int total) {
  if ((total & 7) != 0) return lin;
  return (lin & 7) * (total >> 3) + (lin >> 3);
}

// Tile order: groups of row_group (8) row panels, column panel by column panel, so
// the 32 tiles an XCD runs at once share 8 row panels and 4 column panels in
// its L2.  (The BF16 planes run the same time with 4 and 16; FP8x2, whose rows
// have two planes and whose columns one, takes 2: 6.16 ms per call on the
// Mojette workload, with 4 6.25, with 8 0.14 and with 16 0.48 more than that.)
// In the two-dimensional form one symbol comes after the other, and an eighth
// of each goes to each XCD, in groups of 4 row panels (whole ranges of 32
// tiles per XCD gave some XCDs more of the long symbols: 12.2 against 10.8 ms
// for the 8192^3 workload's call).
template <bool GRID>
__device__ __forceinline__ void tile_at(const PlaneParams& p, int lin, int* si, int* mt, int* nt) {
  *si = 0;
  if (GRID) {
    const int per_sym = p.tiles_m * p.tiles_n;
    *si = lin / per_sym;
    lin -= *si * per_sym;
    if ((per_sym & 7) == 0) lin = (lin & 7) * (per_sym >> 3) + (lin >> 3);
  }
  const int per_group = p.row_group * p.tiles_n;
  const int first = lin / per_group * p.row_group;
  const int gsz = p.tiles_m - first < p.row_group ? p.tiles_m - first : p.row_group;
  const int r = lin - (first / p.row_group) * per_group;
  *mt = first + r % gsz;
  *nt = r / gsz;
}

// Where row r of the coded products goes (null: nowhere): of the stacked rows
// of all symbols, or of symbol si's product in the two-dimensional form.
template <bool GRID>
__device__ __forceinline__ float* out_row(const PlaneParams& p, int si, unsigned r) {
  if (!GRID) {
    if (r >= (unsigned)p.n_sym * (unsigned)p.Mb) return nullptr;
    si = (int)(r / (unsigned)p.Mb);
    r -= (unsigned)si * (unsigned)p.Mb;
  } else if (r >= (unsigned)p.Mb) {
    return nullptr;
  }
  const int dest = gld(p.syms + 4 * si + 2);
  if (dest >= 0) return p.Y + ((int64_t)dest * p.Mb + r) * p.Nb;
  const int s = -1 - dest, br = GRID ? s / p.grid : s;
  const int64_t row = (int64_t)br * p.Mb + r;
  return row < p.M ? p.C + row * p.ldc + (int64_t)(s - br * p.grid) * (GRID ? p.Nb : 0) : nullptr;
}

// Accumulators of a wave: MI x 2 of 32 x 32.  WN waves side by side and two
// above each other make a tile of 64 MI rows and 64 WN columns.
template <int MI>
using Acc = v16f[MI][2];

// Writes an accumulated tile to its output rows: lane l holds column l % 32,
// rows 8 (e / 4) + 4 (l / 32) + e % 4 of each 32 x 32.  SCALED: the sums of
// operands packed times kPlaneUp.
template <int MI, int WN, bool SCALED = false>
__device__ __forceinline__ void store_tile(const Acc<MI>& acc, float* const* rows, int64_t n_tile,
                                           int64_t Nb, int wave, int lane) {
  constexpr float f = SCALED ? kPlaneDown : 1.f;
  const int64_t n0 = n_tile + wave % WN * 64 + (lane & 31);
  const bool in0 = n0 < Nb, in1 = n0 + 32 < Nb;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    float* out[16];  // read together: one LDS latency per 16 rows
#pragma unroll
    for (int e = 0; e < 16; ++e)
      out[e] = rows[wave / WN * (32 * MI) + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      gfloat* o = (gfloat*)out[e] + n0;
      if (out[e] && in0) o[0] = acc[i][0][e] * f;
      if (out[e] && in1) o[32] = acc[i][1][e] * f;
    }
  }
}

// Writes an accumulated tile as one piece of a split tile (row major).
template <int MI, int WN>
__device__ __forceinline__ void store_part(const Acc<MI>& acc, float* part, int wave, int lane) {
  gfloat* out = (gfloat*)part + wave % WN * 64 + (lane & 31);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = wave / WN * (32 * MI) + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
#pragma unroll
      for (int j = 0; j < 2; ++j) out[row * (64 * WN) + 32 * j] = acc[i][j][e];
    }
}

}  // namespace
}  // namespace bpx
