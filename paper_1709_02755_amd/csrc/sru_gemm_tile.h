// Pieces the matrix product kernels share: operand access through buffer
// resources, bf16 packing, kernel arguments, tile order and the epilogue of
// the register-staged kernels.  Everything here has internal linkage.
#pragma once

#include <type_traits>

#include "sru_internal.h"

namespace sru {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  bf16x2 v;
  v[0] = (__bf16)lo;  // RNE (v_cvt_pk_bf16_f32)
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(unsigned, v);
}

// Vector loads go through a buffer resource: the hardware returns zeros for
// any offset at or beyond its byte size, so an out-of-range chunk is loaded
// from the sentinel offset kOOB instead of being masked afterwards (no select
// on the loaded data, so nothing has to wait for it).  Operands must then be
// smaller than kOOB bytes; the launcher checks this.
constexpr unsigned kOOB = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  // dword 3 = 0x00020000: 32-bit data format, the raw-buffer setting of gfx9 parts
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                           0x00020000);
}

// Resource for the bytes of an operand from `base` on (extent `bytes`),
// its range capped below kOOB so that sentinel offsets stay out of range.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel_rsrc(const void* p, long long base,
                                                             long long bytes) {
  return make_rsrc(static_cast<const unsigned char*>(p) + base,
                   (unsigned)min(bytes - base, (long long)kOOB - 1));
}

__device__ __forceinline__ u32x4 buf_load16(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}

// Element e of a 16-byte chunk as fp32.  The element is copied to a scalar
// first: a bit cast applied directly to a vector-element lvalue reads element
// 0 with this compiler.
__device__ __forceinline__ float f32_of(const u32x4& v, int e) {
  const unsigned x = v[e];
  return __builtin_bit_cast(float, x);
}

struct KernelArgs {
  const void* A;
  const void* B;
  // operand extents in bytes: the register-staged kernels address whole
  // operands through buffer resources (VEC: extents below kOOB); the direct
  // kernel bases its resources at each workgroup's panels
  long long a_bytes, b_bytes;
  float* out;               // C, or the split partials
  long long lda, ldb, ldo;
  long long split_stride;   // elements between split outputs (0 when splits == 1)
  int M, N, K;
  int k_per_split;          // multiple of BK
  int tiles_m, tiles_n, splits;
  const float* add;
  long long add_ld, add_off;
  int add_count;
  int vec_out;  // output (and addend) rows allow 16-byte accesses: see write_tile_rows
  uint16_t* outb;  // bf16 copy of the result (direct kernel, OB), out may be nullptr
  long long ldob;
};

// Epilogue shared by the kernels.  32x32 accumulator layout: element e of
// lane l is row 8*(e/4) + 4*(l/32) + e%4, column l%32 of the MFMA tile.
// ADD = number of addend tensors (0..2, see KernelArgs).  For each MFMA
// tile the addend loads are issued together (rows and columns clamped into
// range, so no branch separates them) before the stores.
template <class C, int ADD>
__device__ __forceinline__ void write_tile_add(const KernelArgs& g,
                                               const floatx16 (&acc)[C::FM][C::FN], int m0,
                                               int n0, int wm0, int wn0, int lane, int split) {
  float* out = g.out + (long long)split * g.split_stride;
  const bool full = m0 + C::BM <= g.M && n0 + C::BN <= g.N;
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
      const int n = n0 + wn0 + j * 32 + (lane & 31);
      const int mb = m0 + wm0 + i * 32 + (lane >> 5) * 4;
      float v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = acc[i][j][e];
      if constexpr (ADD > 0) {
        const int nc = min(n, g.N - 1);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int mc = min(mb + (e >> 2) * 8 + (e & 3), g.M - 1);
          const float* ar = g.add + (long long)mc * g.add_ld + nc;
          v[e] += ar[0];
          if constexpr (ADD > 1) v[e] += ar[g.add_off];
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = mb + (e >> 2) * 8 + (e & 3);
        if (full || (m < g.M && n < g.N)) out[(long long)m * g.ldo + n] = v[e];
      }
    }
}

// XCD-aware remap of the linear workgroup id: workgroups are dispatched
// round-robin over the 8 XCDs; each XCD gets a contiguous run of tiles.
struct TileIdx {
  int split, tm, tn;
};
// w: the workgroup's index among the nwg of its product.
__device__ __forceinline__ TileIdx tile_of(const KernelArgs& g, int w, int nwg) {
  const int q = nwg / 8, rmd = nwg % 8, x = w % 8;
  const int u = x * q + (x < rmd ? x : rmd) + w / 8;
  const int nt = g.tiles_m * g.tiles_n;
  TileIdx r;
  r.split = u / nt;
  const int t = u - r.split * nt;
  // tiles in groups of GM tile rows, column by column within a group: the
  // 32 tiles an XCD runs at once then span 4 A panels x 8 B panels instead
  // of 3 x 12 (gemm_u's 12 column tiles), fewer distinct panels in its L2
  // (measured: GM = 4 slightly ahead of 8, 16 behind)
  constexpr int GM = 4;
  const int gsz = GM * g.tiles_n;
  const int first = (t / gsz) * GM;
  const int rows = min(g.tiles_m - first, GM);
  const int tg = t - (t / gsz) * gsz;
  r.tm = first + tg % rows;
  r.tn = tg / rows;
  return r;
}

// Two products in one launch: workgroup p.w of the first (n1) or the second
// (n2), which comes first where second_first.
struct PairIdx {
  bool dx;
  int w;
};
__device__ __forceinline__ PairIdx pair_index(int n1, int n2, bool second_first) {
  const int b = blockIdx.x;
  const bool dx = second_first ? b >= n2 : b < n1;
  return {dx, b - (dx == second_first ? (dx ? n2 : n1) : 0)};
}

// Time in us of n1 workgroups of s1 steps and n2 of s2 together, two slots per
// CU: a1, a2 per step of one alone on its CU, `shared` (and `start` each) per
// step of each of two.  Up to 256 workgroups the longest alone; up to 512 two
// on some CU, the longer of which ends alone; beyond, all steps over the CUs
// and about a third of a long workgroup's time as the tail.
inline double pair_time(long long n1, double s1, double a1, long long n2, double s2, double a2,
                        double start, double shared) {
  const double longest = s1 > s2 ? s1 : s2, least = s1 > s2 ? s2 : s1;
  if (n1 + n2 <= 256) return s1 * a1 > s2 * a2 ? s1 * a1 : s2 * a2;
  if (n1 + n2 <= 512)
    return 2 * (start + shared * least) + (longest - least) * (s1 > s2 ? a1 : a2);
  return (n1 * (start + shared * s1) + n2 * (start + shared * s2)) / 256.0 +
         0.6 * shared * longest;
}

}  // namespace
}  // namespace sru
