// Split-bfloat16 products of the polar iteration on pre-split operands (gfx950).
//
// Most iterates and every n x n matrix of the iteration are kept as bfloat16
// parts x = hi + lo + r made once by the kernel that produced them, instead of
// as float32 that every product splits again: the same bytes (2 + 2) up to the
// padding, the same products, and operand slabs that go from memory straight into
// LDS (buffer loads with an LDS destination) without passing through registers or
// the vector ALU.  What float32 held beyond the two parts reached the products
// nowhere but in the polynomial's linear term; errors against float64 are no
// larger for it (geometric means, on float32 operands / on planes: 400 Gaussian
// matrices 96 x 96 1.70e-5 / 1.56e-5, 200 of 256 x 100 1.67e-5 / 1.2e-5, 200 of
// 130 x 100 with sigma_min 1e-5 4.47e-4 / 4.42e-4; the factored steps' products
// are another matter, see isoloco_host.cpp).
//
// Layout ("planes"): a column of length L padded to a multiple of 32 is a run
// of blocks of 32 consecutive elements, each block its 32 hi parts followed by
// its 32 lo parts (128 bytes, a line of every cache).  The padding holds zeros,
// which every product keeps at zero, so that odd sizes need no bounds checks
// inside the loops.  The n x n matrices have their columns padded to a multiple
// of 32 too, the iterates (for thin ones that would multiply the memory) only
// their n: a tile that reaches past the columns or blocks there are reads the
// last one again, and its outputs there are not stored (update) or zeroed (Gram).
//
// What bounds these products: at long K the power limit of the matrix cores
// (update of one 4096 x 4096 matrix on 256 x 256 tiles: 68% MFMA busy at a clock
// down to 1.87 GHz, 1.34 PFLOP/s of part products; torch's bf16 matrix product
// of 16384^3 reaches 1.38 on the same card), at K = 768 the bursts of output
// stores of workgroups that run in step (leaving the stores out: Gram of 48
// matrices 84 -> 64 us, update 135 -> 105 us) and the latency of each tile's first
// loads.  Against the kernels that split float32 in every product (they serve the
// plans that keep float32 operands): ragged sizes (d 612, f 1637) 2.4x, one
// d = 512 block 1.8x, 8 blocks of d = 2048 1.1x, 12 blocks of d = 768 1.03x per
// step.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "isoloco_device.h"
#include "isoloco_kernels.h"

namespace isoloco {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// A tile shape: TM x TN outputs per workgroup, WM x WN waves, ST slabs of 32 k
// values in LDS (ST - 1 of them in flight while one is multiplied).
template <int TM_, int TN_, int WM_, int WN_, int ST_>
struct TileShape {
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, ST = ST_;
  static constexpr int waves = WM * WN, threads = 64 * waves;
  static constexpr int NA = TM / WM / 32, NB = TN / WN / 32;  // 32 x 32 accumulator blocks per wave
};
// Waves of 128 x 64, 64 x 64 and 32 x 32.  Two slabs of 32 beat 4 to 5 slabs of
// 16 in the same LDS on the two large shapes (update of 48 matrices of 768 x 768
// 135 against 159 us: rows of 64 bytes halve what a line brings); the small one
// has few tiles per CU and hides its loads' latency behind two slabs in flight
// (three slabs of LDS let three workgroups share a CU: one d = 768 block, 312 to
// 624 tiles a launch, 1309 -> 1237 us a step against four slabs).
typedef TileShape<256, 256, 2, 4, 2> TileL;
typedef TileShape<128, 128, 2, 2, 2> TileM;
typedef TileShape<64, 64, 2, 2, 3> TileS;
constexpr int kSlabK = 32;

// 16 bytes per lane from memory to LDS: lane l's bytes land at lds_off + 16 l
// (lds_off is wave-uniform).  No register receives the data; the loads count
// in vmcnt like any other, and wait_slabs() below waits for them.  m0 holds
// the LDS address.  It is listed as clobbered, so that the compiler sets it again
// for any use of its own (it has none here today); m0 is a reserved register,
// of which the compiler warns.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(uint32_t lds_off, u32x4 rsrc, uint32_t voff, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// Wait until at most N of this wave's loads are outstanding and its LDS reads
// have returned, then for every wave of the workgroup.
template <int N>
__device__ __forceinline__ void wait_slabs() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ __forceinline__ u32x4 tile_rsrc(uint64_t base) {
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
  r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
  r[2] = 0xffffffffu;
  r[3] = kBufferFlags;
  return r;
}

// The next bf16 part of 4 values, which keep the remainder (exact: the parts
// are x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1))
__device__ __forceinline__ bf16x4 part_of(floatx4& x) {
  const bf16x2 a = __builtin_convertvector((floatx2){x[0], x[1]}, bf16x2);
  const bf16x2 b = __builtin_convertvector((floatx2){x[2], x[3]}, bf16x2);
  const floatx2 fa = __builtin_convertvector(a, floatx2), fb = __builtin_convertvector(b, floatx2);
  x[0] -= fa[0];
  x[1] -= fa[1];
  x[2] -= fb[0];
  x[3] -= fb[1];
  return (bf16x4){a[0], a[1], b[0], b[1]};
}

// A slab of ROWS x 32 k values of an operand whose columns run along k (128
// bytes of a row per slab): the 16-byte pieces of an LDS row are XORed with
// bits 1-3 of the row, so that a fragment read (16 rows, one piece each, per
// pass of 256 bytes) touches every bank once.
template <int ROWS, int WAVES>
struct KSlab {
  static constexpr int kBytes = ROWS * 128;
  static constexpr int kLoads = kBytes / 1024 / WAVES;
  uint32_t vo[kLoads];
  u32x4 rsrc;
  __device__ static __forceinline__ int swizzle(int row) { return (row >> 1) & 7; }
  __device__ __forceinline__ void init(const uint16_t* tile, uint32_t row_bytes, int rows_left) {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int at = q * WAVES * 64 + threadIdx.x;
      const int row = at / 8;
      vo[q] = (uint32_t)min(row, rows_left - 1) * row_bytes + 16u * ((at % 8) ^ swizzle(row));
    }
    rsrc = tile_rsrc((uint64_t)tile);
  }
  __device__ __forceinline__ void load(uint32_t lds, int slab) const {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int q = 0; q < kLoads; ++q) load_to_lds(lds + 1024u * (q * WAVES + wave), rsrc, vo[q], 128u * slab);
  }
  // 8 k values from k = kk + 8 (lane / 32) of row `row0 + lane % 32`, part p
  __device__ static __forceinline__ bf16x8 frag(const char* lds, int row0, int kk, int p) {
    const int lane = threadIdx.x & 63;
    const int piece = (p * 4 + (kk >> 3) + (lane >> 5)) ^ swizzle(lane & 31);
    return *reinterpret_cast<const bf16x8*>(lds + (row0 + (lane & 31)) * 128 + piece * 16);
  }
  // 4 k values from k = 8 grp + 4 (lane / 32) of row `row0 + lane % 32`, part p
  __device__ static __forceinline__ bf16x4 quad(const char* lds, int row0, int grp, int p) {
    const int lane = threadIdx.x & 63;
    const int piece = (p * 4 + grp) ^ swizzle(lane & 31);
    return *reinterpret_cast<const bf16x4*>(lds + (row0 + (lane & 31)) * 128 + piece * 16 + 8 * (lane >> 5));
  }
};

// 4 consecutive float32 values at byte offset `off`, of which the first `left`
// exist (zeros otherwise).  v4: one 16-byte load whatever `left` is (an offset
// past the resource's 2 GiB reads zeros), so that the count of loads in flight
// is known.
constexpr uint32_t kFloatSpan = 0x80000000u;
__device__ __forceinline__ floatx4 load_quad(__amdgpu_buffer_rsrc_t r, uint32_t off, int left, bool v4) {
  if (v4)
    return __builtin_bit_cast(
        floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(left > 0 ? off : kFloatSpan), 0, 0));
  floatx4 x;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    x[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)(e < left ? off + 4 * e : kFloatSpan), 0, 0));
  return x;
}

// The same slab from float32 columns (m values each, no padding), split on the
// way: a thread holds 4 k values of each of its rows.  A pass of 32 lanes
// stores rows r, r + 1, r + 8, r + 9, which fall on distinct banks.
template <int ROWS, int WAVES>
struct KSlabF {
  static constexpr int kLoads = ROWS * 128 / 1024 / WAVES;
  const float* base;  // the tile's first column
  int ld, cols_left, k_left;
  bool v4;
  floatx4 v[kLoads];
  __device__ static __forceinline__ int row_of(int at) {
    const int g = at >> 3;
    return (g & ~15) | (g & 1) | ((g & 2) << 2) | ((g & 12) >> 1);
  }
  __device__ __forceinline__ void init(const float* tile, int m, int cols, int k_end) {
    base = tile;
    ld = m;
    cols_left = cols;
    k_left = k_end;
    v4 = (m & 3) == 0;
  }
  __device__ __forceinline__ void load(int slab) {
    const __amdgpu_buffer_rsrc_t r = stream_rsrc(base, kFloatSpan);
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int at = q * WAVES * 64 + threadIdx.x;
      const int row = row_of(at), k = slab * kSlabK + 4 * (at & 7);
      v[q] = load_quad(r, 4u * ((uint32_t)row * ld + k), row < cols_left ? k_left - k : 0, v4);
    }
  }
  __device__ __forceinline__ void store(char* lds, float scale) const {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int at = q * WAVES * 64 + threadIdx.x;
      const int row = row_of(at), piece = at & 7;
      floatx4 x = v[q] * scale;
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<bf16x4*>(lds + row * 128 + (((p * 4 + (piece >> 1)) ^ KSlab<ROWS, WAVES>::swizzle(row)) * 16) +
                                   (piece & 1) * 8) = part_of(x);
    }
  }
};

// A slab of ROWS x 32 k values of an operand whose columns run along the rows
// (X as the left factor of the update): per k the tile's blocks of 32 rows, PB
// bytes each (128: hi and lo; 64: one part).  The fragments need k along a
// lane's registers: they are read with the transposing LDS load (16 lanes read
// 16 consecutive rows of 4 k values each and receive one row's 4 k values).
// Its 32-byte quarter-rows (4 k values x two halves of a block per 32 lanes)
// take 8 different places in 256 bytes: the 16-byte pieces of a k row are XORed
// with k mod 4 in the two bits above the half.
template <int ROWS, int WAVES, int PB>
struct RowSlab {
  static constexpr int kRow = ROWS / 32 * PB;  // bytes per k
  static constexpr int kBytes = kSlabK * kRow;
  static constexpr int kLoads = kBytes / 1024 / WAVES;
  static constexpr int kPieces = kRow / 16;
  // (a row of 8 pieces: its parity already picks one half of the 256 bytes)
  __device__ static __forceinline__ int swizzle(int kq) { return kPieces >= 16 ? kq << 2 : (kq & 2) << 1; }
  uint32_t vo[kLoads];
  uint64_t base;
  uint64_t step;
  uint32_t col_b;
  int cols;
  __device__ __forceinline__ void init(const uint16_t* tile, uint32_t col_bytes, int blocks_left, int n) {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int at = q * WAVES * 64 + threadIdx.x;  // 16-byte piece of the slab
      const int k = at / kPieces;
      const int piece = (at % kPieces) ^ swizzle(k & 3);
      const int blk = piece / (PB / 16);
      vo[q] = (uint32_t)k * col_bytes + (uint32_t)min(blk, blocks_left - 1) * PB + 16u * (piece % (PB / 16));
    }
    base = (uint64_t)tile;
    step = (uint64_t)kSlabK * col_bytes;
    col_b = col_bytes;
    cols = n;
  }
  __device__ __forceinline__ void load(uint32_t lds, int slab) const {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u32x4 r = tile_rsrc(base + step * (uint64_t)slab);
    const int left = cols - slab * kSlabK;
    if (left >= kSlabK) {
#pragma unroll
      for (int q = 0; q < kLoads; ++q) load_to_lds(lds + 1024u * (q * WAVES + wave), r, vo[q], 0);
    } else {
      // the last columns: past them the last one again (P's rows there are zero)
#pragma unroll
      for (int q = 0; q < kLoads; ++q) {
        const int k = (q * WAVES * 64 + (int)threadIdx.x) / kPieces;
        load_to_lds(lds + 1024u * (q * WAVES + wave), r, vo[q] - (uint32_t)max(k - left + 1, 0) * col_b, 0);
      }
    }
  }
  // 8 k values from k = kk + 8 (lane / 32) of row 32 blk + lane % 32, part p
  __device__ static __forceinline__ bf16x8 frag(const char* lds, int blk, int kk, int p) {
    const int lane = threadIdx.x & 63;
    const int j = lane & 15, kq = j >> 2;
    const int piece = (blk * (PB / 16) + p * 4 + ((lane >> 4) & 1) * 2 + ((j & 3) >> 1)) ^ swizzle(kq);
    const char* at = lds + (kk + 8 * (lane >> 5) + kq) * kRow + piece * 16 + (j & 1) * 8;
    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at);
    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + 4 * kRow));
    return __builtin_shufflevector(__builtin_bit_cast(bf16x4, v0), __builtin_bit_cast(bf16x4, v1), 0, 1, 2, 3, 4, 5, 6,
                                   7);
  }
};

// The same slab (and the third parts of its values in a slab of their own)
// from float32 columns, split on the way: a thread holds 4 rows of its k values.
template <int ROWS, int WAVES>
struct RowSlabF {
  static constexpr int kLoads = ROWS * 128 / 1024 / WAVES;
  static constexpr int kQuads = ROWS / 4;  // per k
  typedef RowSlab<ROWS, WAVES, 128> S2;
  typedef RowSlab<ROWS, WAVES, 64> S3;
  const float* base;  // the tile's first row in column 0
  int ld, rows_left, cols;
  bool v4;
  floatx4 v[kLoads];
  __device__ __forceinline__ void init(const float* tile, int m, int rows, int n) {
    base = tile;
    ld = m;
    rows_left = rows;
    cols = n;
    v4 = (m & 3) == 0;
  }
  __device__ __forceinline__ void load(int slab) {
    const __amdgpu_buffer_rsrc_t rs = stream_rsrc(base + (int64_t)slab * kSlabK * ld, kFloatSpan);
    const int cols_left = cols - slab * kSlabK;
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int at = q * WAVES * 64 + threadIdx.x;
      const int k = at / kQuads, r = 4 * (at % kQuads);
      v[q] = load_quad(rs, 4u * ((uint32_t)k * ld + r), k < cols_left ? rows_left - r : 0, v4);
    }
  }
  template <bool THIRD>
  __device__ __forceinline__ void store(char* lds, char* lds3, float scale) const {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int at = q * WAVES * 64 + threadIdx.x;
      const int k = at / kQuads, r4 = at % kQuads, blk = r4 >> 3, w = (r4 & 7) >> 1;
      floatx4 x = v[q] * scale;
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<bf16x4*>(lds + k * S2::kRow + ((blk * 8 + p * 4 + w) ^ S2::swizzle(k & 3)) * 16 +
                                   (r4 & 1) * 8) = part_of(x);
      if constexpr (THIRD)
        *reinterpret_cast<bf16x4*>(lds3 + k * S3::kRow + ((blk * 4 + w) ^ S3::swizzle(k & 3)) * 16 + (r4 & 1) * 8) =
            part_of(x);
    }
  }
};

__device__ __forceinline__ const uint16_t* planes(const float* p) { return reinterpret_cast<const uint16_t*>(p); }

enum { kGram = 0, kPoly = 1, kUpdate = 2 };

template <class C>
__device__ __forceinline__ floatx4 acc4(const floatx16 (&acc)[C::NA][C::NB], int a, int b, int grp) {
  return (floatx4){acc[a][b][4 * grp], acc[a][b][4 * grp + 1], acc[a][b][4 * grp + 2], acc[a][b][4 * grp + 3]};
}

// The accumulators of a wave, acc[a][b][4 grp + r] = C(i, j) with
//   i = i0 + (wm NA + a) 32 + 8 grp + 4 (lane / 32) + r,  j = j0 + (wn NB + b) 32 + lane % 32,
// stored through the wave's own LDS region so that every store instruction
// writes whole runs of consecutive bytes.

// Columns j of C as planes: column j at out + j * col_bytes.
template <class C>
__device__ __forceinline__ void store_columns(const floatx16 (&acc)[C::NA][C::NB], char* ws, char* out,
                                              int64_t col_bytes, int bi0, int nbi, int j0, int nj) {
  constexpr int P = C::NA * 128 + 16, LPC = C::NA * 8, CPI = 64 / LPC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / C::WN, wn = wave % C::WN;
#pragma unroll
  for (int b = 0; b < C::NB; ++b) {
#pragma unroll
    for (int a = 0; a < C::NA; ++a)
#pragma unroll
      for (int grp = 0; grp < 4; ++grp) {
        floatx4 x = acc4<C>(acc, a, b, grp);
        char* at = ws + (lane & 31) * P + a * 128 + (8 * grp + 4 * (lane >> 5)) * 2;
        *reinterpret_cast<bf16x4*>(at) = part_of(x);
        *reinterpret_cast<bf16x4*>(at + 64) = part_of(x);
      }
#pragma unroll
    for (int q = 0; q < 32 / CPI; ++q) {
      const int jj = q * CPI + lane / LPC, ch = lane % LPC;
      const u32x4 v = *reinterpret_cast<const u32x4*>(ws + jj * P + ch * 16);
      const int gj = j0 + (wn * C::NB + b) * 32 + jj, gb = bi0 + wm * C::NA + ch / 8;
      if (gj < nj && gb < nbi)
        *reinterpret_cast<u32x4*>(out + gj * col_bytes + gb * 128 + (ch % 8) * 16) = v;
    }
  }
}

// The third parts (x - hi - lo) of columns j, in an array of their own.
template <class C>
__device__ __forceinline__ void store_third(const floatx16 (&acc)[C::NA][C::NB], char* ws, char* out,
                                            int64_t col_bytes, int bi0, int nbi, int j0, int nj) {
  constexpr int P = C::NA * 64 + 16, LPC = C::NA * 4, CPI = 64 / LPC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / C::WN, wn = wave % C::WN;
#pragma unroll
  for (int b = 0; b < C::NB; ++b) {
#pragma unroll
    for (int a = 0; a < C::NA; ++a)
#pragma unroll
      for (int grp = 0; grp < 4; ++grp) {
        floatx4 x = acc4<C>(acc, a, b, grp);
        part_of(x);
        part_of(x);
        *reinterpret_cast<bf16x4*>(ws + (lane & 31) * P + a * 64 + (8 * grp + 4 * (lane >> 5)) * 2) = part_of(x);
      }
#pragma unroll
    for (int q = 0; q < 32 / CPI; ++q) {
      const int jj = q * CPI + lane / LPC, ch = lane % LPC;
      const u32x4 v = *reinterpret_cast<const u32x4*>(ws + jj * P + ch * 16);
      const int gj = j0 + (wn * C::NB + b) * 32 + jj, gb = bi0 + wm * C::NA + ch / 4;
      if (gj < nj && gb < nbi) *reinterpret_cast<u32x4*>(out + gj * col_bytes + gb * 64 + (ch % 4) * 16) = v;
    }
  }
}

// Columns j in float32, m rows, no padding.
template <class C>
__device__ __forceinline__ void store_float(const floatx16 (&acc)[C::NA][C::NB], char* ws, float* out, int m, int n,
                                            int i0, int j0) {
  constexpr int P = C::NA * 128 + 16, LPC = C::NA * 8, CPI = 64 / LPC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / C::WN, wn = wave % C::WN;
  const bool v4 = (m & 3) == 0;
#pragma unroll
  for (int b = 0; b < C::NB; ++b) {
#pragma unroll
    for (int a = 0; a < C::NA; ++a)
#pragma unroll
      for (int grp = 0; grp < 4; ++grp)
        *reinterpret_cast<floatx4*>(ws + (lane & 31) * P + a * 128 + (8 * grp + 4 * (lane >> 5)) * 4) =
            acc4<C>(acc, a, b, grp);
#pragma unroll
    for (int q = 0; q < 32 / CPI; ++q) {
      const int jj = q * CPI + lane / LPC, ch = lane % LPC;
      const floatx4 v = *reinterpret_cast<const floatx4*>(ws + jj * P + ch * 16);
      const int gj = j0 + (wn * C::NB + b) * 32 + jj, gi = i0 + wm * C::NA * 32 + ch * 4;
      if (gj >= n) continue;
      float* o = out + (int64_t)gj * m + gi;
      if (v4 && gi + 3 < m) {
        *reinterpret_cast<floatx4*>(o) = v;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (gi + r < m) o[r] = v[r];
      }
    }
  }
}

// Rows i of C as planes (the mirror image of a symmetric product's
// off-diagonal tile): row i at out + i * row_bytes.
template <class C>
__device__ __forceinline__ void store_rows(const floatx16 (&acc)[C::NA][C::NB], char* ws, char* out,
                                           int64_t row_bytes, int i0, int ni, int bj0, int nbj) {
  constexpr int P = C::NB * 128 + 16, LPC = C::NB * 8, CPI = 64 / LPC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / C::WN, wn = wave % C::WN;
#pragma unroll
  for (int a = 0; a < C::NA; ++a) {
#pragma unroll
    for (int b = 0; b < C::NB; ++b)
#pragma unroll
      for (int grp = 0; grp < 4; ++grp) {
        floatx4 x = acc4<C>(acc, a, b, grp);
        const bf16x4 hi = part_of(x), lo = part_of(x);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          char* at = ws + (8 * grp + 4 * (lane >> 5) + r) * P + b * 128 + (lane & 31) * 2;
          *reinterpret_cast<__bf16*>(at) = hi[r];
          *reinterpret_cast<__bf16*>(at + 64) = lo[r];
        }
      }
#pragma unroll
    for (int q = 0; q < 32 / CPI; ++q) {
      const int ii = q * CPI + lane / LPC, ch = lane % LPC;
      const u32x4 v = *reinterpret_cast<const u32x4*>(ws + ii * P + ch * 16);
      const int gi = i0 + (wm * C::NA + a) * 32 + ii, gb = bj0 + wn * C::NB + ch / 8;
      if (gi < ni && gb < nbj)
        *reinterpret_cast<u32x4*>(out + gi * row_bytes + gb * 128 + (ch % 8) * 16) = v;
    }
  }
}

// One output tile.
//   Gram:    C(i, j) = sum_k X[k][i] Y[k][j] over the task's K slice (Y = X
//            unless a second operand is given); symmetric, tiles tm <= tn
//   Poly:    P' = g (a I + b g^2 A + c g^4 A^2) as gamma (rho A + A A) + a g I;
//            symmetric
//   Update:  X'(i, j) = sum_k X[i][k] P[k][j], P symmetric (read as P[j][k])
// XF: X is float32 (the first iterates, whose third parts the bf16x5 updates
// need, and those at a phase end, where the factor itself is wanted), split on
// its way through registers; else planes, loaded straight into LDS.
template <int MODE, int NP, bool XF, class C>
__global__ void __launch_bounds__(C::threads, 2) plane_gemm_kernel(PlaneArgs g) {
  constexpr bool X5 = NP == 5;
  constexpr bool UP = MODE == kUpdate;
  static_assert(UP || C::TM == C::TN, "symmetric products: square tiles");
  static_assert(!X5 || UP, "bf16x5 serves the updates");
  static_assert(!XF || MODE != kPoly, "A is kept as planes");
  constexpr int ST = XF ? 2 : C::ST;
  typedef KSlab<C::TM, C::waves> AK;
  typedef RowSlab<C::TM, C::waves, 128> AR;
  typedef RowSlab<C::TM, C::waves, 64> AR3;
  typedef KSlab<C::TN, C::waves> BK;
  constexpr int kA = AK::kBytes, kA3 = X5 ? AR3::kBytes : 0, kB = BK::kBytes;
  constexpr int kStage = kA + kA3 + kB, kMain = ST * kStage;
  constexpr int kColWs = 32 * (C::NA * 128 + 16), kRowWs = 32 * (C::NB * 128 + 16);
  constexpr int kWs = kColWs > kRowWs ? kColWs : kRowWs;
  constexpr int kLds = kMain > C::waves * kWs ? kMain : C::waves * kWs;
  static_assert(kLds <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char lds[kLds];

  const Task task = g.tasks[blockIdx.x];
  if (task.mat < 0) return;
  if (g.only_active && !g.sc[task.mat].active) return;
  const MatInfo& mi = g.mats[task.mat];
  const int m = mi.m, n = mi.n, mp = mi.mp, np = mi.np, nb = np / 32;
  const int i0 = task.tm * C::TM, j0 = task.tn * C::TN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / C::WN, wn = wave % C::WN;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)lds;

  // operands (planes: 2 uint16 per element, at the offsets of a float buffer)
  AK ak;
  AR ar;
  AR3 ar3;
  BK bk;
  KSlabF<C::TM, C::waves> akf;
  RowSlabF<C::TM, C::waves> arf;
  KSlabF<C::TN, C::waves> bkf;
  bool same = false;  // both operands are the same panel: staged once
  float scale = 1.f;
  int nslab;
  if constexpr (MODE == kGram) {
    const bool alt = g.xa_alt && g.sc[task.mat].qbuf;
    const int kb = task.ks * mi.kchunk;
    const int ke = min(mp, kb + mi.kchunk);
    nslab = (ke - kb) / kSlabK;
    const float* x = alt ? g.xa_alt : g.xa;
    const float* y = g.xb ? g.xb : x;
    same = !g.xb && task.tm == task.tn;
    if constexpr (XF) {
      if (g.first) scale = g.sc[task.mat].inv_fro;
      akf.init(x + mi.ws_off + (int64_t)i0 * m + kb, m, n - i0, min(m, ke) - kb);
      bkf.init(y + mi.ws_off + (int64_t)j0 * m + kb, m, n - j0, min(m, ke) - kb);
    } else {
      ak.init(planes(x + mi.ws_off + (int64_t)i0 * mp + kb), 4u * mp, n - i0);
      bk.init(planes(y + mi.ws_off + (int64_t)j0 * mp + kb), 4u * mp, n - j0);
    }
  } else if constexpr (MODE == kPoly) {
    nslab = nb;
    same = task.tm == task.tn;
    ak.init(planes(g.sq + mi.sq_off + (int64_t)i0 * np), 4u * np, np - i0);
    bk.init(planes(g.sq + mi.sq_off + (int64_t)j0 * np), 4u * np, np - j0);
  } else {
    nslab = nb;
    if constexpr (XF) {
      if (g.first) scale = g.sc[task.mat].inv_fro;
      arf.init(g.xa + mi.ws_off + i0, m, m - i0, n);
    } else {
      ar.init(planes(g.xa + mi.ws_off + i0), 4u * mp, (mp - i0) / 32, n);
      if constexpr (X5)
        ar3.init(g.third + 2 * mi.ws_off + (g.step & 1 ? (int64_t)mp * n : 0) + i0, 2u * mp, (mp - i0) / 32, n);
    }
    bk.init(planes(g.sq + mi.sq_off + (int64_t)j0 * np), 4u * np, np - j0);
  }

  // the slabs that go straight to LDS
  constexpr int kLoadsA = UP ? AR::kLoads + (X5 ? AR3::kLoads : 0) : AK::kLoads;
  constexpr int kLoadsAB = kLoadsA + BK::kLoads;
  auto issue = [&](int slab, int buf) {
    const uint32_t at = lds0 + (uint32_t)buf * kStage;
    if constexpr (UP && !XF) {
      ar.load(at, slab);
      if constexpr (X5) ar3.load(at + kA, slab);
    }
    if constexpr (!UP && !XF) ak.load(at, slab);
    if constexpr (UP || !XF)
      if (UP || !same) bk.load(at + kA + kA3, slab);
  };
  // the slabs that go through registers; the count of their loads is kFetch
  // where they are 16-byte loads
  constexpr int kFetch = (UP ? 1 : 2) * (C::TM * 128 / 1024 / C::waves);
  const bool fast = (m & 3) == 0;
  auto fetch = [&](int slab) {
    if constexpr (UP) {
      arf.load(slab);
    } else {
      akf.load(slab);
      if (!same) bkf.load(slab);
    }
  };
  // (a symmetric product's slabs all go through registers: its loads need no wait)
  auto put = [&](int buf) {
    char* at = lds + buf * kStage;
    if constexpr (UP) {
      arf.template store<X5>(at, at + kA, scale);
    } else {
      akf.store(at, scale);
      if (!same) bkf.store(at + kA, scale);
    }
  };

  // A diagonal tile of a symmetric product: the waves strictly below the
  // diagonal leave their blocks to the mirror images of those strictly above.
  const bool on_diag = !UP && task.tm == task.tn;
  const bool below = on_diag && wm * C::NA >= (wn + 1) * C::NB;
  const bool mirrored = !UP && (!on_diag || (wm + 1) * C::NA <= wn * C::NB);

  if constexpr (XF) fetch(0);
#pragma unroll
  for (int s = 0; s < ST - 1; ++s)
    if (s < nslab) issue(s, s);
  if constexpr (XF) {
    put(0);
    fetch(min(1, nslab - 1));
  }

  floatx16 acc[C::NA][C::NB];
#pragma unroll
  for (int a = 0; a < C::NA; ++a)
#pragma unroll
    for (int b = 0; b < C::NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
  // (Poly) the step's polynomial with g folded in; g = 0 marks a zero or
  // non-finite Delta: P' = 0 then, and rho is kept finite
  float gamma = 1.f, diag = 0.f, rho = 0.f;
  if constexpr (MODE == kPoly) {
    const float* c = g.coef + ((int64_t)mi.sched * g.n_steps + g.step) * 3;
    const float gs = g.first ? g.sc[task.mat].gscale : 1.f;
    const float g2 = gs * gs;
    rho = gs != 0.f ? c[1] / (c[2] * gs * gs) : 0.f;
    gamma = c[2] * g2 * g2 * gs;
    diag = c[0] * gs;
  }

  // the products of 16 k values of a slab
  auto multiply = [&](const char* at, const char* bt, int kk) {
    bf16x8 av[C::NA][X5 ? 3 : 2], bv[C::NB][2];
#pragma unroll
    for (int b = 0; b < C::NB; ++b)
#pragma unroll
      for (int p = 0; p < 2; ++p) bv[b][p] = BK::frag(bt, (wn * C::NB + b) * 32, kk, p);
#pragma unroll
    for (int a = 0; a < C::NA; ++a) {
      if constexpr (UP) {
#pragma unroll
        for (int p = 0; p < 2; ++p) av[a][p] = AR::frag(at, wm * C::NA + a, kk, p);
        if constexpr (X5) av[a][2] = AR3::frag(at + kA, wm * C::NA + a, kk, 0);
      } else {
#pragma unroll
        for (int p = 0; p < 2; ++p) av[a][p] = AK::frag(at, (wm * C::NA + a) * 32, kk, p);
      }
    }
    // part products, smallest order first
#pragma unroll
    for (int a = 0; a < C::NA; ++a)
#pragma unroll
      for (int b = 0; b < C::NB; ++b) {
        floatx16 c = acc[a][b];
        if constexpr (X5) {
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][2], bv[b][0], c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][1], bv[b][1], c, 0, 0, 0);
        }
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][1], bv[b][0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][0], bv[b][1], c, 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][0], bv[b][0], c, 0, 0, 0);
      }
  };

  int buf = 0, buf_in = ST - 1;  // the buffers of slabs s and s + ST - 1
#pragma unroll 1
  for (int s = 0; s < nslab; ++s) {
    // slab s is in LDS (at most ST - 2 later slabs in flight), and every wave
    // is done with slab s - 1, whose buffer slab s + ST - 1 takes
    if constexpr (XF) {
      // (the loads of slab s + 1 into registers, issued last, stay in flight)
      if (!fast) wait_slabs<0>();
      else wait_slabs<kFetch>();
    } else {
      if (ST == 2 || nslab - 1 - s < ST - 2) wait_slabs<0>();
      else if (UP || !same) wait_slabs<(ST - 2) * kLoadsAB>();
      else wait_slabs<(ST - 2) * kLoadsA>();
    }
    if (s + ST - 1 < nslab) issue(s + ST - 1, buf_in);
    const int buf_put = buf_in;
    const char* at = lds + buf * kStage;
    const char* bt = same ? at : at + kA + kA3;
    buf_in = buf;
    buf = buf + 1 == ST ? 0 : buf + 1;
    if constexpr (XF) {
      // slab s + 1 is split and stored between the halves of this slab's
      // products, and its registers reloaded after them
      if (!below) multiply(at, bt, 0);
      if (s + 1 < nslab) put(buf_put);
      if (!below) multiply(at, bt, 16);
      fetch(min(s + 2, nslab - 1));
      continue;
    }
    if (below) continue;
    if constexpr (MODE == kPoly) {
      // the linear term rho A(i, j) = rho A(j, i), from the slab of the right
      // operand whose k values are this wave's rows i: A is read as an operand
      // only (reading the tile again before the loop: 95 us against 83 for 48
      // matrices of 768 x 768)
#pragma unroll
      for (int a = 0; a < C::NA; ++a)
        if (s * kSlabK == i0 + (wm * C::NA + a) * 32) {
#pragma unroll
          for (int b = 0; b < C::NB; ++b)
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
              const bf16x4 hi = BK::quad(bt, (wn * C::NB + b) * 32, grp, 0);
              const bf16x4 lo = BK::quad(bt, (wn * C::NB + b) * 32, grp, 1);
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[a][b][4 * grp + r] += rho * ((float)hi[r] + (float)lo[r]);
            }
        }
    }
    multiply(at, bt, 0);
    multiply(at, bt, 16);
  }
  wait_slabs<0>();  // every wave is done with the operands: LDS is free
  char* ws = lds + wave * kWs;

  if constexpr (MODE == kUpdate) {
    if (g.out_float)
      store_float<C>(acc, ws, g.out + mi.ws_off, m, n, i0, j0);
    else {
      // (X_k's third parts are in the half of the matrix's span of k's parity)
      if (g.third_out)
        store_third<C>(acc, ws,
                       reinterpret_cast<char*>(g.third_out + 2 * mi.ws_off + (g.step & 1 ? 0 : (int64_t)mp * n)),
                       2 * (int64_t)mp, i0 / 32, mp / 32, j0, n);
      store_columns<C>(acc, ws, reinterpret_cast<char*>(g.out + mi.ws_off), 4 * (int64_t)mp, i0 / 32, mp / 32, j0, n);
    }
    return;
  }

  const int T = (np + C::TM - 1) / C::TM;
  const int tile = task.tm * T - task.tm * (task.tm - 1) / 2 + (task.tn - task.tm);
  double* red = reinterpret_cast<double*>(lds);
  int* last = reinterpret_cast<int*>(lds + 128);
  if constexpr (MODE == kGram) {
    if (mi.ksplit > 1) {
      // This K slice's partial tile, in 32 x 32 blocks of the accumulators'
      // own order (16 bytes per lane, consecutive lanes consecutive), at agent
      // scope; the last of the tile's ksplit workgroups to arrive adds the
      // slices in slice order and finishes the tile.  No workgroup waits for
      // another.  (The planner keeps a matrix's slices under 2 GiB, the range
      // of the buffer offsets.)
      const int64_t nn = (int64_t)np * np;
      const __amdgpu_buffer_rsrc_t pr = stream_rsrc(g.gpart + mi.part_off, (uint32_t)(4 * mi.ksplit * nn));
#pragma unroll
      for (int a = 0; a < C::NA; ++a)
#pragma unroll
        for (int b = 0; b < C::NB; ++b) {
          const int bi = i0 / 32 + wm * C::NA + a, bj = j0 / 32 + wn * C::NB + b;
          if (bi >= nb || bj >= nb || below) continue;
          const int off = (int)(4 * (task.ks * nn + ((int64_t)bi * nb + bj) * 1024 + lane * 4));
#pragma unroll
          for (int grp = 0; grp < 4; ++grp)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc4<C>(acc, a, b, grp)), pr,
                                                   off + 1024 * grp, 0, kAgentCoherent);
        }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's slice is in place
      __syncthreads();
      if (threadIdx.x == 0) *last = arrive(g.split_cnt + mi.cnt_off + tile, mi.ksplit);
      __syncthreads();
      if (!*last) return;
#pragma unroll
      for (int a = 0; a < C::NA; ++a)
#pragma unroll
        for (int b = 0; b < C::NB; ++b) {
          const int bi = i0 / 32 + wm * C::NA + a, bj = j0 / 32 + wn * C::NB + b;
          if (bi >= nb || bj >= nb || below) continue;
#pragma unroll
          for (int grp = 0; grp < 4; ++grp) {
            floatx4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < kMaxKSplit; ++k) {
              if (k >= mi.ksplit) break;
              const int off = (int)(4 * (k * nn + ((int64_t)bi * nb + bj) * 1024 + lane * 4)) + 1024 * grp;
              const floatx4 x = __builtin_bit_cast(
                  floatx4, __builtin_amdgcn_raw_buffer_load_b128(pr, off, 0, kAgentCoherent));
              t = k == 0 ? x : t + x;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][4 * grp + r] = t[r];
          }
        }
      __syncthreads();  // *last has been read: the staging may overwrite it
    }
    if (np != n) {
      // past X's columns the operands were the last one again
#pragma unroll
      for (int a = 0; a < C::NA; ++a)
#pragma unroll
        for (int b = 0; b < C::NB; ++b) {
          const int j = j0 + (wn * C::NB + b) * 32 + (lane & 31);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = i0 + (wm * C::NA + a) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (i >= n || j >= n) acc[a][b][r] = 0.f;
          }
        }
    }
  } else {
#pragma unroll
    for (int a = 0; a < C::NA; ++a)
#pragma unroll
      for (int b = 0; b < C::NB; ++b) {
        const int j = j0 + (wn * C::NB + b) * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = i0 + (wm * C::NA + a) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          acc[a][b][r] = gamma * acc[a][b][r] + (i == j && i < n ? diag : 0.f);
        }
      }
  }
  char* out = reinterpret_cast<char*>(g.out + mi.sq_off);
  if (!below) store_columns<C>(acc, ws, out, 4 * (int64_t)np, i0 / 32, nb, j0, np);
  if (mirrored) store_rows<C>(acc, ws, out, 4 * (int64_t)np, i0, np, j0 / 32, nb);
  if constexpr (MODE == kGram) {
    if (g.norm_mode < 0) return;
    // the tile's share of ||A||_F^2 or ||A - I||_F^2; the last tile of the
    // matrix to arrive takes its decisions
    const float unit = g.norm_mode == kNormFirst ? 0.f : 1.f;
    double sq = 0.0;
#pragma unroll
    for (int a = 0; a < C::NA; ++a)
#pragma unroll
      for (int b = 0; b < C::NB; ++b) {
        const int j = j0 + (wn * C::NB + b) * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = i0 + (wm * C::NA + a) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          const double d = (double)acc[a][b][r] - (i == j ? unit : 0.f);
          if (i < n && j < n) sq += d * d;
        }
      }
    sq = below ? 0.0 : mirrored ? 2.0 * sq : sq;
    __syncthreads();  // every wave is done with its staging region
    sq = block_sum<C::waves>(sq, red);
    if (threadIdx.x == 0) {
      partial_store(g.part_norm + mi.norm_off + tile, sq);
      const int nt = T * (T + 1) / 2;
      if (arrive(g.mat_cnt + task.mat, nt)) norm_decide(mi, g.part_norm, g.sc[task.mat], g.na, nt);
    }
  }
}

template <int MODE, int NP, bool XF>
static void launch_tiles(const PlaneList& l, const PlaneArgs& g, hipStream_t st) {
  const dim3 grid(l.cnt);
  if (l.tile == kTileL)
    hipLaunchKernelGGL((plane_gemm_kernel<MODE, NP, XF, TileL>), grid, dim3(TileL::threads), 0, st, g);
  else if (l.tile == kTileM)
    hipLaunchKernelGGL((plane_gemm_kernel<MODE, NP, XF, TileM>), grid, dim3(TileM::threads), 0, st, g);
  else
    hipLaunchKernelGGL((plane_gemm_kernel<MODE, NP, XF, TileS>), grid, dim3(TileS::threads), 0, st, g);
}

hipError_t launch_plane_gemm(const PlaneList& l, int mode, int arith, PlaneArgs g, hipStream_t st) {
  if (l.cnt == 0) return hipSuccess;
  g.tasks = l.tasks;
  if (mode == kGram) {
    if (g.x_float) launch_tiles<kGram, 3, true>(l, g, st);
    else launch_tiles<kGram, 3, false>(l, g, st);
  } else if (mode == kPoly) {
    launch_tiles<kPoly, 3, false>(l, g, st);
  } else if (arith == kArithBf16x5) {
    if (g.x_float) launch_tiles<kUpdate, 5, true>(l, g, st);
    else launch_tiles<kUpdate, 5, false>(l, g, st);
  } else {
    if (g.x_float) launch_tiles<kUpdate, 3, true>(l, g, st);
    else launch_tiles<kUpdate, 3, false>(l, g, st);
  }
  return hipGetLastError();
}

}  // namespace isoloco
