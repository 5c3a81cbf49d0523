// Applies of the scan-symmetric model: s = A x and x = A^T s.
//
// Both operators have the same shape once the table is cut into band tiles (Methods,
// "Efficient reconstruction based on scanning symmetries": an absolute index over the voxel
// grid and a relative one from each scan position select the model vector):
//     out[p][16 t + m] = sum_{K-groups q of tile t} sum_{j < G} pack[q][m][j] * in[p + d_q + j]
// where p runs over scan positions, the K-group q names one lateral offset o and a run of G
// consecutive depths (forward) or time samples (adjoint), and d_q is the offset of
// (p + o, run start) in the zero-padded input (p - o for the adjoint).  The lateral halo
// of the padded input supplies the zeros outside the region of interest.
//
// GEMM view per tile: M = 16 output rows, N = scan positions (16 per MFMA), K = the tile's
// K-groups.  Kernels: FP64 MFMA (v_mfma_f64_16x16x4f64), FP32 as products of three-part BF16
// splits on the BF16 MFMA, BF16 MFMA (v_mfma_f32_16x16x32_bf16) and the block-scaled FP8 MFMA
// (v_mfma_scale_f32_16x16x128_f8f6f4, e4m3 table and operand) on gfx950.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "internal.h"

namespace aroam {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
// Register operands are clang vector types and are reinterpreted with __builtin_bit_cast, so
// no local variable has its address taken (which would place it in scratch memory).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// Stage an input vector [ny][nx][L] as zero-padded BF16 in blocks of the ring's chunks,
// [chunk][nyp][nxp][8 entries]: a row of a chunk is contiguous, so that the ring's loads use whole
// cache lines (from [nyp][nxp][L] each 128-byte line would be fetched once per chunk in it: 149 GB
// instead of 76 beyond the L2 in a 400 x 400 adjoint).  A workgroup covers 32 columns of a row
// (grid.x: rows x column blocks) and eight chunks; reads are runs of 256 bytes, writes of 512.
__global__ __launch_bounds__(256) void k_stage_bf16(const float* __restrict__ in,
                                                    u32x4* __restrict__ out, int K, int nx, int ny,
                                                    int nxp, int nyp, int L, int nch) {
  const int nb = (nxp + 31) / 32, row = blockIdx.x / nb;
  const int c = blockIdx.y * 8 + threadIdx.x % 8, col = blockIdx.x % nb * 32 + threadIdx.x / 8;
  if (c >= nch || col >= nxp) return;
  const int px = col - K, py = row - K, l0 = 8 * c;
  u32x4 w = {0, 0, 0, 0};
  if (px >= 0 && px < nx && py >= 0 && py < ny) {
    const float* p = in + ((long long)py * nx + px) * L + l0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      floatx2 f;
      f[0] = l0 + 2 * i < L ? p[2 * i] : 0.0f;
      f[1] = l0 + 2 * i + 1 < L ? p[2 * i + 1] : 0.0f;
      w[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
    }
  }
  out[((long long)c * nyp + row) * nxp + col] = w;
}

// LDS bytes of the FP8 kernel's final sums: S tiles of MH halves per wave, four waves.
constexpr size_t red_bytes(int S, int MH) { return (size_t)4 * S * MH * 64 * 16; }

// ------------------------------------------------------------------------------------------
// LDS-ring applies (FP32, FP64 and BF16).
//
// A workgroup (W waves) owns one output tile of kHalves 16-row halves and a patch of BR x BC scan
// positions.  The tile's bundles are grouped into stage units (chunk of the inner axis, kRingStep
// consecutive input row offsets) in the order chunk, row.  The LDS holds the rows a unit reads (the patch's
// columns and K more on each side, the chunk's entries) and room for kRingStep more, as a ring
// indexed by padded row: a unit loads only the rows it adds into registers while the unit before
// it computes, and one barrier makes them visible.  Four row offsets to a unit share one
// barrier and one trip to memory and pool their bundles over the waves: against one, on chunks
// of two runs, that took 10 % off the 400 x 400 FP32 forward of the time (105.4 -> 94.8 ms), 7 % off
// the 64 x 64 one (161 -> 150 us) and 6 % off the FP64 96 x 96 adjoint (1.40 -> 1.32 ms).  The rows
// come straight from the caller's vector (BF16: from k_stage_bf16); positions outside the scan and
// entries past the end of the axis are written as zeros.  The waves form P row groups
// of BR / P patch rows, and the S = W / P waves of a group take the bundles of each unit in
// turn, so that a table fragment is loaded once per row group; at the end the S partial sums of
// a position are added in wave order through the LDS.
//
// The element type's part is an operation class: how a staged vector is written to the LDS,
// what a lane holds of a table bundle and of a position, and the MFMAs that combine them.
// Lane (n = lane % 16, g = lane / 16) holds row n of K-group g of the table and K-group g's
// entries of position n.

typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex2u __attribute__((ext_vector_type(2), aligned(8)));

// Bit j: entry j of the lane's K-group (lane group g) meets a nonzero table entry in some row.
template <class T, int N>
__device__ __forceinline__ unsigned live_entries(const T (&v)[N], int g) {
  unsigned keep = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) keep |= (__ballot(v[j] != T(0)) >> (16 * g) & 0xffff) ? 1u << j : 0u;
  return keep;
}

// FP32 on the BF16 MFMA: an FP32 value is the exact sum of three BF16 values (8 bits each, rounded
// to nearest in turn) where the last of them is not below BF16's smallest normal number.  That holds
// for all FP32 numbers after a scaling by powers of two, which the outputs take back: operands by
// 2^kF32OperandExp, the table by a power chosen from its range (set_f32_scale; OpF32Far where there
// is none).  Operands beyond 2^104 become infinite; a workgroup whose sums are not finite, for this
// or any other reason, takes them again on FP32 MFMAs (ring_guarded).  Without the scaling, operands
// of 2^-120 lost 6e-5 of their value; it costs nothing that could be measured.
// A product is the six products of parts whose exponents add up to no less than 2^-16 of the leading
// one; the three left out are below 2^-24 of it (0.24 2^-24 rms).  The BF16 MFMA cuts its sum to
// FP32 less exactly than an FP32 addition rounds, so a bundle's leading products and its smaller ones
// are summed from zero (the leading product of a single entry is exact in FP32) and then added to
// the accumulator.  Six MFMAs in a row on the accumulator cut the running sum six times a bundle: the
// 400 x 400 forward took 90.0 ms at a relative error of 1.9e-6 instead of 99.6 at 4.2e-7, the
// 200 x 200 adjoint 4.10 ms at 1.2e-6 instead of 4.55 at 3.0e-7, and outputs of one to ten products
// came out 1.3 to 1.4 times as far off as sums of FP32 products (now 1.0 to 1.2 times).  Against eight
// FP32 MFMAs of K = 4, which take 256 cycles where the six take 96 (400 x 400 forward 181 ms at
// 6.8e-6, 200 x 200 adjoint 8.05 ms at 2.3e-6), the sum is rounded less often.  With two of the three
// products that are left out the 400 x 400 forward took 126 ms instead of 102, at the same error.
// Tile after tile: with the MFMAs of two tiles alternating the 200 x 200 adjoint takes 1.5 % longer.
// Splitting at the staging costs nothing visible: a staged entry feeds hundreds of MFMAs.
struct OpF32 {
  using In = float;
  using Vec = floatx4;             // 16 staged bytes
  using VecU = floatx4u;           // the same with the alignment of one entry
  using Acc = floatx4;
  static constexpr int kVec = 4;   // entries of a staged vector
  static constexpr int kCol = kRingColumnBytes;  // LDS bytes of a staged column
  static constexpr int kVecs = kRingF32.G / kVec;   // staged vectors per column
  static constexpr int kTiles = 2;                  // position tiles per phase
  static constexpr int kHalves = 1;                 // 16-row halves of an output tile
  static constexpr bool kBlocked = false;           // input staged as [chunk][row][column] before
  static constexpr int kPlane = 2 * kRingF32.G;     // LDS bytes of one part of a column
  struct A {
    u32x4 v[3];
  };
  struct X {
    u32x4 v[3];
  };
  static __device__ __forceinline__ void load_a(const void* __restrict__ pack, int b, int lane,
                                                A& f) {
    const u32x4* p = reinterpret_cast<const u32x4*>(pack) + (long long)b * 192 + lane;
#pragma unroll
    for (int i = 0; i < 3; ++i) f.v[i] = p[64 * i];
  }
  static __device__ __forceinline__ X read_x(const unsigned char* p) {
    X x;
#pragma unroll
    for (int i = 0; i < 3; ++i) x.v[i] = *reinterpret_cast<const u32x4*>(p + i * kPlane);
    return x;
  }
  static __device__ __forceinline__ void write(unsigned char* col, int v, Vec f) {
    constexpr float kScale = 1 << kF32OperandExp;
    u32x2 part[3];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      floatx2 r = {f[2 * h] * kScale, f[2 * h + 1] * kScale};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
        part[i][h] = w;
        r[0] -= __uint_as_float(w << 16);
        r[1] -= __uint_as_float(w & 0xffff0000u);
      }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
      *reinterpret_cast<u32x2*>(col + 8 * v + i * kPlane) = part[i];
  }
  // the MFMAs of a bundle's half H for NX tiles whose accumulators lie STEP apart
  template <int NX, int STEP, int H>
  static __device__ __forceinline__ void mma(const A& a, const X (&x)[NX], Acc* acc) {
    constexpr int pa[5] = {2, 0, 1, 1, 0}, px[5] = {0, 2, 1, 0, 1};  // ascending size
#pragma unroll
    for (int t = 0; t < NX; ++t) {
      const Acc high = product(a, 0, x[t], 0, Acc{0, 0, 0, 0});
      Acc low = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < 5; ++i) low = product(a, pa[i], x[t], px[i], low);
      acc[t * STEP] += high + low;
    }
  }
  static __device__ __forceinline__ Acc product(const A& a, int i, const X& x, int j, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.v[i]),
                                                   __builtin_bit_cast(bf16x8, x.v[j]), c, 0, 0, 0);
  }
  // output row (within the tile) of accumulator element i of lane group g
  static __device__ __forceinline__ int row(int i, int g) { return 4 * g + i; }

  // The guarded sweep: FP32 entries, a column's eight after one another, on FP32 MFMAs.
  static constexpr bool kScaled = true;
  struct Guard {
    float v[8];
    unsigned keep;
  };
  static __device__ __forceinline__ Guard load_guard(const void* __restrict__ pack, int b,
                                                     int lane, int exp) {
    A f;
    load_a(pack, b, lane, f);
    Guard r;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float e = 0;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const uint32_t w = f.v[i][j / 2];
        e += __uint_as_float(j % 2 ? w & 0xffff0000u : w << 16);
      }
      r.v[j] = ldexpf(e, -exp);
    }
    r.keep = live_entries(r.v, lane / 16);
    return r;
  }
  static __device__ __forceinline__ void write_guard(unsigned char* col, int v, Vec f) {
    *reinterpret_cast<Vec*>(col + 16 * v) = f;
  }
  template <int H>
  static __device__ __forceinline__ void mma_guard(const Guard& a, const unsigned char* p, Acc& acc) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float x = reinterpret_cast<const float*>(p)[j];
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[j], a.keep >> j & 1 ? x : 0.0f, acc, 0, 0, 0);
    }
  }
};

// FP32 on v_mfma_f32_16x16x4_f32, for tables whose entries are too far apart to be split after one
// scaling (set_f32_scale): entry j of the four K-groups' runs feeds a bundle's j-th MFMA.
struct OpF32Far : OpF32 {
  static constexpr bool kScaled = false;
  struct A {
    floatx4 v[2];
  };
  struct X {
    floatx4 v[2];
  };
  static __device__ __forceinline__ void load_a(const void* __restrict__ pack, int b, int lane,
                                                A& f) {
    const floatx4* p = reinterpret_cast<const floatx4*>(pack) + (long long)b * 128 + lane;
    f.v[0] = p[0];
    f.v[1] = p[64];
  }
  static __device__ __forceinline__ X read_x(const unsigned char* p) {
    X x;
    x.v[0] = *reinterpret_cast<const floatx4*>(p);
    x.v[1] = *reinterpret_cast<const floatx4*>(p + 16);
    return x;
  }
  static __device__ __forceinline__ void write(unsigned char* col, int v, Vec f) {
    write_guard(col, v, f);
  }
  template <int NX, int STEP, int H>
  static __device__ __forceinline__ void mma(const A& a, const X (&x)[NX], Acc* acc) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int t = 0; t < NX; ++t)
        acc[t * STEP] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[j / 4][j % 4], x[t].v[j / 4][j % 4],
                                                             acc[t * STEP], 0, 0, 0);
  }
  static __device__ __forceinline__ Guard load_guard(const void* __restrict__ pack, int b,
                                                     int lane, int) {
    A f;
    load_a(pack, b, lane, f);
    Guard r;
#pragma unroll
    for (int j = 0; j < 8; ++j) r.v[j] = f.v[j / 4][j % 4];
    r.keep = live_entries(r.v, lane / 16);
    return r;
  }
};

// FP64 on v_mfma_f64_16x16x4_f64: entry j of the four K-groups' runs feeds a bundle's j-th MFMA.
// The adjoint of a 96 x 96 scan (Nz 64, Nt 256, K 20) takes 1.31 ms, which is 61 TFLOP/s on what it
// issues (of 78.6; MFMA busy 0.86): what is left are the zeros of the tiles, 0.58 of it.  With
// positions read from global memory it took 3.42 ms (bound by the texture path), with one FMA per
// load 68.4 ms.
struct OpF64 {
  using In = double;
  using Vec = doublex2;
  using VecU = doublex2u;
  using Acc = doublex4;
  static constexpr int kVec = 2;
  static constexpr int kCol = kRingColumnBytes;
  static constexpr int kVecs = kRingF64.G / kVec;
  static constexpr int kTiles = 2;
  static constexpr int kHalves = 1;
  static constexpr bool kBlocked = false;
  struct A {
    doublex4 v;
  };
  struct X {
    doublex2 v[2];
  };
  static __device__ __forceinline__ void load_a(const void* __restrict__ pack, int b, int lane,
                                                A& f) {
    f.v = reinterpret_cast<const doublex4*>(pack)[(long long)b * 64 + lane];
  }
  static __device__ __forceinline__ X read_x(const unsigned char* p) {
    X x;
    x.v[0] = *reinterpret_cast<const doublex2*>(p);
    x.v[1] = *reinterpret_cast<const doublex2*>(p + 16);
    return x;
  }
  static __device__ __forceinline__ void write(unsigned char* col, int v, Vec f) {
    *reinterpret_cast<doublex2*>(col + 16 * v) = f;
  }
  template <int NX, int STEP, int H>
  static __device__ __forceinline__ void mma(const A& a, const X (&x)[NX], Acc* acc) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int t = 0; t < NX; ++t)
        acc[t * STEP] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.v[j], x[t].v[j / 2][j % 2],
                                                             acc[t * STEP], 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int i, int g) { return 4 * i + g; }

  static constexpr bool kScaled = false;
  struct Guard {
    double v[4];
    unsigned keep;
  };
  static __device__ __forceinline__ Guard load_guard(const void* __restrict__ pack, int b,
                                                     int lane, int) {
    A f;
    load_a(pack, b, lane, f);
    Guard r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r.v[j] = f.v[j];
    r.keep = live_entries(r.v, lane / 16);
    return r;
  }
  static __device__ __forceinline__ void write_guard(unsigned char* col, int v, Vec f) {
    write(col, v, f);
  }
  template <int H>
  static __device__ __forceinline__ void mma_guard(const Guard& a, const unsigned char* p, Acc& acc) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double x = reinterpret_cast<const double*>(p)[j];
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.v[j], a.keep >> j & 1 ? x : 0.0, acc, 0, 0, 0);
    }
  }
};

// BF16: output tiles of two 16-row halves that share the position fragments; a unit's bundles
// come in the order half 0 alone, half 1 alone, both, so that each run's loop issues only the
// MFMAs its bundles reach (a test per bundle cost 10 %).  Against one row offset to a unit on
// chunks of 32 entries, reading ahead within a bundle only: the 200 x 200 x 128 forward (K 20)
// takes 0.86 ms instead of 0.97, the refined 96 x 96 LSQR 39.6 instead of 41.8, the 400 x 400 adjoint
// the same 20.2.  That one is bound by what an MFMA costs besides itself: a read of the position
// fragments feeds 1.57 of them (MFMA busy 0.66), 50 registers are spilled (4 GB written an apply) and
// the table stream misses the L2 in 0.58 of its requests (80 GB an apply from beyond it; 36 before).
struct OpBF16 {
  using In = float;  // outputs; the input is read as k_stage_bf16 leaves it
  using Vec = u32x4;
  using Acc = floatx4;
  static constexpr int kVec = 8;
  static constexpr int kCol = kRing16ColumnBytes;
  static constexpr int kVecs = 1;
  static constexpr int kTiles = 2;
  static constexpr int kHalves = 2;
  static constexpr bool kBlocked = true;
  static constexpr bool kScaled = false;
  struct A {
    u32x4 v[2];
  };
  struct X {
    u32x4 v;
  };
  static __device__ __forceinline__ void load_a(const void* __restrict__ pack, int b, int lane,
                                                A& f) {
    const u32x4* p =
        reinterpret_cast<const u32x4*>(pack) + (long long)b * 128 + lane / 16 * 32 + lane % 16;
    f.v[0] = p[0];
    f.v[1] = p[16];
  }
  static __device__ __forceinline__ X read_x(const unsigned char* p) {
    return X{*reinterpret_cast<const u32x4*>(p)};
  }
  static __device__ __forceinline__ void write(unsigned char* col, int, Vec f) {
    *reinterpret_cast<u32x4*>(col) = f;
  }
  template <int NX, int STEP, int H>
  static __device__ __forceinline__ void mma(const A& a, const X (&x)[NX], Acc* acc) {
#pragma unroll
    for (int t = 0; t < NX; ++t)
      acc[t * STEP] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.v[H]),
                                                              __builtin_bit_cast(bf16x8, x[t].v),
                                                              acc[t * STEP], 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int i, int g) { return 4 * g + i; }

  struct Guard {
    A a;
    u32x4 keep[2];  // per half: all bits of the live entries
  };
  static __device__ __forceinline__ Guard load_guard(const void* __restrict__ pack, int b,
                                                     int lane, int) {
    Guard r;
    load_a(pack, b, lane, r.a);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t v[8];  // magnitudes
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = r.a.v[h][j / 2] >> 16 * (j % 2) & 0x7fff;
      const unsigned keep = live_entries(v, lane / 16);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        r.keep[h][i] = (keep >> 2 * i & 1 ? 0xffffu : 0) | (keep >> (2 * i + 1) & 1 ? 0xffff0000u : 0);
    }
    return r;
  }
  static __device__ __forceinline__ void write_guard(unsigned char* col, int v, Vec f) {
    write(col, v, f);
  }
  template <int H>
  static __device__ __forceinline__ void mma_guard(const Guard& a, const unsigned char* p, Acc& acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.a.v[H]),
                                                  __builtin_bit_cast(bf16x8, read_x(p).v & a.keep[H]),
                                                  acc, 0, 0, 0);
  }
};

struct RingArgs {
  const int4* pieces;  // (tile, unit begin, unit end, partial slot or -1)
  const int4* units;   // (row offset, chunk start, bundle begin, bundle end)
  const int2* classes; // two halves: per unit, the end of its bundles of half 0 alone and of half 1
                       // alone; the rest reach both
  const int* meta;     // per K-group: LDS byte offset of its run from the position's column
  void* partial;       // [slot][patch][position][tile rows] partial sums of cut tiles
  int n_patches;
  int out_len, nx, ny, K, L;
  int ncc;             // patch columns
  int NCOL;            // staged columns
  int row_bytes;       // LDS bytes of a staged row
  int nxp, nyp;        // blocked input: padded columns and rows of a chunk
  int exp;             // FP32: the pack holds the parts of the table times 2^exp
};

// Staged vectors in flight: the 16-byte pieces of the rows a unit adds.  off < 0: none.
template <class Op, int PF>
struct RingFetch {
  typename Op::Vec v[PF];
  int off[PF];
  unsigned zero;  // bit i: vector i lies outside the scan or past the end of the axis
};

// Address of staged vector idx of the rows from padded patch row `lo`, for the chunk at e0; the
// loads are unconditional (an invalid one reads the vector's first entries), so that the waits
// of the table fragments in flight can count them.
template <class Op, int RS, bool RAGGED>
__device__ __forceinline__ typename Op::Vec ring_load(const RingArgs& a,
                                                      const typename Op::In* __restrict__ in,
                                                      int lo, int e0, int idx, int nv, int py0,
                                                      int px0, int rowvec, int& off, bool& zero) {
  const int G = lo + idx / rowvec, rem = idx % rowvec;
  const int c = rem / Op::kVecs, v = rem % Op::kVecs;
  if constexpr (Op::kBlocked) {
    off = idx < nv ? (G % RS) * a.row_bytes + c * Op::kCol : -1;
    zero = false;
    // rows past the last padded one belong to row offsets without K-groups
    const int row = min(py0 + G, a.nyp - 1);
    return reinterpret_cast<const u32x4*>(
        in)[((long long)(e0 / Op::kVec) * a.nyp + row) * a.nxp + px0 + c];
  } else {
    const int py = py0 + G - a.K, px = px0 + c - a.K, l = e0 + v * Op::kVec;
    const bool ok = idx < nv && py >= 0 && py < a.ny && px >= 0 && px < a.nx && l < a.L;
    off = idx < nv ? (G % RS) * a.row_bytes + c * Op::kCol + (v << 8 * 3) : -1;
    zero = !ok;
    const typename Op::In* p = in + (ok ? ((long long)py * a.nx + px) * a.L + l : 0);
    typename Op::Vec r;
    if constexpr (RAGGED) {
#pragma unroll
      for (int i = 0; i < Op::kVec; ++i) {
        const bool in_axis = ok && l + i < a.L;
        const typename Op::In e = p[in_axis ? i : 0];
        r[i] = in_axis ? e : typename Op::In(0);
      }
    } else {
      r = *reinterpret_cast<const typename Op::VecU*>(p);
    }
    return r;
  }
}

// The output of a piece, or for a piece of a cut tile its partial slot: the sums over the S waves
// of a group in wave order, S tiles per phase, times 2^-shift.  Returns whether the thread's sums
// are finite.
template <class Op, int BR, int BC, int W, int P>
__device__ __forceinline__ bool ring_store(const typename Op::Acc (&acc)[Op::kHalves][BR / P * BC / 16],
                                           unsigned char* lds, const RingArgs& a, const int4& piece,
                                           typename Op::In* __restrict__ out, int tid, int py0,
                                           int px0, int shift) {
  using In = typename Op::In;
  using Acc = typename Op::Acc;
  constexpr int S = W / P, RW = BR / P, TPR = BC / 16, NT = RW * TPR;
  constexpr int MH = Op::kHalves, TM = kTile * MH;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int grp = wave / S, sw = wave % S, n = lane % 16, g = lane / 16;
  const int tile = piece.x;
  bool finite = true;
  In* slot = piece.w >= 0 ? reinterpret_cast<In*>(a.partial) +
                                ((long long)piece.w * a.n_patches + blockIdx.x) * (BR * BC * TM)
                          : nullptr;
  Acc* red = reinterpret_cast<Acc*>(lds);
#pragma unroll
  for (int p = 0; p < NT; p += S) {
    Acc v[MH];
    if constexpr (S > 1) {
      __syncthreads();  // the ring, or the phase before
#pragma unroll
      for (int k = 0; k < S; ++k)
#pragma unroll
        for (int h = 0; h < MH; ++h) red[((wave * S + k) * MH + h) * 64 + lane] = acc[h][p + k];
      __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < MH; ++h) {
      if constexpr (S > 1) {
        v[h] = red[((grp * S * S + sw) * MH + h) * 64 + lane];
#pragma unroll
        for (int s = 1; s < S; ++s) v[h] += red[(((grp * S + s) * S + sw) * MH + h) * 64 + lane];
      } else {
        v[h] = acc[h][p];
      }
    }
#pragma unroll
    for (int h = 0; h < MH; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) finite &= __builtin_isfinite(v[h][i]);
    const int t = p + sw;
    const int r = grp * RW + t / TPR, c = (t % TPR) * 16 + n;
    const int py = py0 + r, px = px0 + c;
    if (py < a.ny && px < a.nx) {
      In* dst = slot ? slot + (r * BC + c) * TM
                     : out + ((long long)py * a.nx + px) * a.out_len + TM * tile;
#pragma unroll
      for (int h = 0; h < MH; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = kTile * h + Op::row(i, g);
          if (TM * tile + row < a.out_len) {
            if constexpr (Op::kScaled) dst[row] = ldexpf(v[h][i], -shift);
            else dst[row] = v[h][i];
          }
        }
    }
  }
  return finite;
}

// The sweep over a piece's units in which a non-finite entry meets only outputs whose row tile
// has a nonzero table entry for it (elsewhere in the K-group's run, and in null K-groups, the
// others would read 0 * NaN), and in which an infinity stays one.  Taken by a workgroup whose sums
// were not finite, after it has stored them; plain loads and a barrier per unit, since that is rare.
// Nothing of it is live in the main loop (written as a second turn of a loop around both, it spilled
// 90 bytes more a lane there); the test of the sums costs up to 1 % (64 x 64 FP32 forward 148.1 ->
// 149.5 us, 200 x 200 adjoint 4.18 -> 4.21 ms, 96 x 96 FP64 1.318 -> 1.320; BF16 nothing measurable).
template <class Op, int BR, int BC, int W, int P, bool RAGGED>
__device__ __forceinline__ void ring_guarded(const void* __restrict__ pack,
                                             const typename Op::In* __restrict__ in,
                                             typename Op::In* __restrict__ out, unsigned char* lds,
                                             const RingArgs& a, const int4& piece, int tid, int py0,
                                             int px0) {
  using Acc = typename Op::Acc;
  constexpr int S = W / P, RW = BR / P, TPR = BC / 16, NT = RW * TPR;
  constexpr int UR = BR + kRingStep - 1, RS = UR + kRingStep;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int grp = wave / S, sw = wave % S, n = lane % 16, g = lane / 16;
  const int rowvec = a.NCOL * Op::kVecs;
  Acc acc[Op::kHalves][NT];
#pragma unroll
  for (int h = 0; h < Op::kHalves; ++h)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[h][t] = Acc{0, 0, 0, 0};
  for (int u = piece.y; u < piece.z; ++u) {
    const int4 U = a.units[u];
    const int lo = U.x + a.K, nv = UR * rowvec;
    __syncthreads();
    for (int i = tid; i < nv; i += 64 * W) {
      int off;
      bool zero;
      typename Op::Vec v =
          ring_load<Op, RS, RAGGED>(a, in, lo, U.y, i, nv, py0, px0, rowvec, off, zero);
      if (zero) v = typename Op::Vec{};
      Op::write_guard(lds + (off & 0xffffff), off >> 24, v);
    }
    __syncthreads();
    const int s0 = ((grp * RW + lo) % RS) * a.row_bytes;
    for (int b = U.z + sw; b < U.w; b += S) {
      const typename Op::Guard f = Op::load_guard(pack, b, lane, a.exp);
      const unsigned first = (unsigned)(a.meta[b * kLaneGroups + g] + n * Op::kCol + s0);
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        const unsigned q = first + r * a.row_bytes;
        const unsigned char* row = lds + min(q, q - RS * a.row_bytes);
#pragma unroll
        for (int t = 0; t < TPR; ++t) {
          const unsigned char* p = row + t * 16 * Op::kCol;
          Op::template mma_guard<0>(f, p, acc[0][r * TPR + t]);
          if constexpr (Op::kHalves > 1)
            Op::template mma_guard<1>(f, p, acc[Op::kHalves - 1][r * TPR + t]);
        }
      }
    }
  }
  ring_store<Op, BR, BC, W, P>(acc, lds, a, piece, out, tid, py0, px0, 0);
}

// The bundle loop is a pipeline of phases of kTiles position tiles: the fragments of a phase are
// read from the LDS while the phase before multiplies, the LDS offset of a bundle is loaded two
// bundles ahead and its table fragments between one and two.  Without the scheduling barriers the
// compiler moves each read next to its use: 400 x 400 FP32 forward 102.5 -> 104.7 ms, 200 x 200
// adjoint 4.67 -> 4.74, 40 x 40 FISTA 15.25 -> 15.94, 400 x 400 BF16 adjoint 19.9 -> 21.4.  Four rows
// are held to 168 registers, for three waves per SIMD where the LDS allows; with two, the 200 x 200
// adjoint takes 5.07 ms, the FISTA 19.3, the 64 x 64 forward 170 us instead of 156.  The FP32 forward
// issues 1.46 PFLOP/s of BF16 products (a large library product reaches 1.1), at which the chip lowers
// its clock from 2.1 to 1.7-1.9 GHz: besides the additions of the bundles' sums what is left is
// power, spent on the table stream (L2 and beyond) and on the zeros of the tiles.
template <class Op, int BR, int BC, int W, int P, bool RAGGED>
__global__ __launch_bounds__(64 * W)
    __attribute__((amdgpu_waves_per_eu(BR == 8 ? 2 : 3))) void k_apply_ring(
    const void* __restrict__ pack, const typename Op::In* __restrict__ in,
    typename Op::In* __restrict__ out, RingArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  using Acc = typename Op::Acc;
  constexpr int S = W / P;        // waves that share a row group's bundles
  constexpr int RW = BR / P;      // patch rows per group
  constexpr int TPR = BC / 16;
  constexpr int NT = RW * TPR;    // position tiles per wave
  constexpr int XT = Op::kTiles;  // tiles per phase
  constexpr int PH = NT / XT;
  constexpr int RPP = XT / TPR;   // patch rows per phase
  constexpr int ST = kRingStep;   // row offsets of a unit
  constexpr int UR = BR + ST - 1; // rows a unit reads
  constexpr int RS = UR + ST;     // rows of the ring
  constexpr int PF = Op::kBlocked ? 2 : BR == 8 ? 4 : 3;  // staged vectors in flight per thread
  constexpr int TH = 64 * W;
  constexpr int MH = Op::kHalves;
  static_assert(W % P == 0 && BR % P == 0 && NT % XT == 0 && XT % TPR == 0 && NT % S == 0, "shape");
  const int4 piece = a.pieces[blockIdx.y];
  const int py0 = (blockIdx.x / a.ncc) * BR, px0 = (blockIdx.x % a.ncc) * BC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int grp = wave / S, sw = wave % S;
  const int n = lane % 16, g = lane / 16;
  const int rowvec = a.NCOL * Op::kVecs;
  Acc acc[MH][NT];
#pragma unroll
  for (int h = 0; h < MH; ++h)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[h][t] = Acc{0, 0, 0, 0};

  struct Bundle {
    typename Op::A a;
    int mo;
  };
  RingFetch<Op, PF> f;
  // the rows unit U adds: padded patch rows [lo, U.x + K + UR) of its chunk
  auto fetch = [&](const int4& U, int lo) {
    const int nv = (U.x + a.K + UR - lo) * rowvec;
    f.zero = 0;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      bool z;
      f.v[i] = ring_load<Op, RS, RAGGED>(a, in, lo, U.y, threadIdx.x + TH * i, nv, py0, px0, rowvec,
                                         f.off[i], z);
      f.zero |= z ? 1u << i : 0u;
    }
  };
  auto put = [&](typename Op::Vec v, int off, bool zero) {
    if (off >= 0) {
      const typename Op::Vec z = {};
      Op::write(lds + (off & 0xffffff), off >> 24, zero ? z : v);
    }
  };
  auto stage = [&](const int4& U, int lo) {
#pragma unroll
    for (int i = 0; i < PF; ++i) put(f.v[i], f.off[i], (f.zero >> i) & 1);
    const int nv = (U.x + a.K + UR - lo) * rowvec;
    for (int base = TH * PF; base < nv; base += TH * 4) {
      typename Op::Vec v[4];
      int off[4];
      bool z[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        v[i] = ring_load<Op, RS, RAGGED>(a, in, lo, U.y, base + threadIdx.x + TH * i, nv, py0, px0,
                                         rowvec, off[i], z[i]);
#pragma unroll
      for (int i = 0; i < 4; ++i) put(v[i], off[i], z[i]);
    }
  };

  const int u0 = piece.y, u1 = piece.z;
  if (u0 < u1) {
    // Table fragments: two bundles of the unit (r0, r1), and on eight rows the first of the next one
    // (n0), whose loads are issued when the unit starts; on four rows its registers are spilled (200 x
    // 200 adjoint 4.63 ms without, 5.00 with it; the 400 x 400 forward on eight rows 106 and 104).
    constexpr bool kAhead = BR == 8;
    Bundle r0, r1, n0;
    auto load_mo = [&](Bundle& r, int b) { r.mo = a.meta[b * kLaneGroups + g]; };
    auto load_a = [&](Bundle& r, int b) { Op::load_a(pack, b, lane, r.a); };
    int4 U = a.units[u0];
    if constexpr (kAhead) {
      load_mo(n0, min(U.z + sw, U.w - 1));
      load_a(n0, min(U.z + sw, U.w - 1));
    }
    fetch(U, U.x + a.K);
    stage(U, U.x + a.K);
    __syncthreads();
    for (int u = u0; u < u1; ++u) {
      const int4 Un = a.units[min(u + 1, u1 - 1)];
      const int2 C = MH > 1 ? a.classes[u] : make_int2(0, 0);
      // rows the next unit finds in the ring: those of this unit, in the same chunk
      const int lo = Un.y == U.y && Un.x < U.x + UR ? U.x + a.K + UR : Un.x + a.K;
      if constexpr (kAhead) {
        r0 = n0;
      } else {
        load_mo(r0, min(U.z + sw, U.w - 1));
        load_a(r0, min(U.z + sw, U.w - 1));
      }
      load_mo(r1, min(U.z + sw + S, U.w - 1));
      load_a(r1, min(U.z + sw + S, U.w - 1));
      if constexpr (kAhead) {
        load_mo(n0, min(Un.z + sw, Un.w - 1));
        load_a(n0, min(Un.z + sw, Un.w - 1));
      }
      fetch(Un, lo);
      // LDS offset of the wave's first row at the unit's first row offset (the same for all
      // lanes); a wave whose rows have no output row or no input row inside the scan skips the
      // unit
      const int s0 = ((grp * RW + U.x + a.K) % RS) * a.row_bytes;
      const int o = py0 + grp * RW, i0 = o + U.x;
      const bool live = o < a.ny && i0 + RW + ST - 1 > 0 && i0 < a.ny;
      auto read = [&](auto ntc, int p, int mo, auto& x) {
        constexpr int NTC = decltype(ntc)::value;
        const unsigned first = (unsigned)(mo + n * Op::kCol + s0);
#pragma unroll
        for (int r = 0; r < RPP; ++r) {
          // row p RPP + r after the K-group's first, wrapped into the ring (the subtraction
          // underflows to a larger value where there is nothing to wrap)
          const unsigned q = first + (p * RPP + r) * a.row_bytes;
          const unsigned char* row = lds + min(q, q - RS * a.row_bytes);
#pragma unroll
          for (int t = 0; t < NTC; ++t) x[r * NTC + t] = Op::read_x(row + t * 16 * Op::kCol);
        }
      };
      // The wave's bundles for the tiles of the first NTC tile columns, all PH phases: the
      // position fragments of a phase are read while the phase before multiplies (the barriers
      // keep the compiler from moving the reads next to their use).
      auto all = [&](auto ntc) {
        constexpr int NTC = decltype(ntc)::value, NX = RPP * NTC;
        typename Op::X x[2][NX];
        // bundle b, of the halves in MASK
        auto body = [&](auto mask, Bundle& r, const int& mo_next, int b) {
          constexpr int MASK = decltype(mask)::value;
#pragma unroll
          for (int p = 0; p < PH; ++p) {
            read(ntc, (p + 1) % PH, p + 1 < PH ? r.mo : mo_next, x[(p + 1) % 2]);
            if (p + 2 == PH) load_mo(r, min(b + 2 * S, U.w - 1));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (MASK & 1)
              Op::template mma<NX, TPR / NTC, 0>(r.a, x[p % 2], acc[0] + p * XT);
            if constexpr (MASK & 2)
              Op::template mma<NX, TPR / NTC, 1>(r.a, x[p % 2], acc[MH - 1] + p * XT);
            __builtin_amdgcn_sched_barrier(0);
          }
          load_a(r, min(b + 2 * S, U.w - 1));
        };
        static_assert(PH % 2 == 0, "a bundle's first phase is in x[0]");
        int b = U.z + sw;
        if (b >= U.w) return;
        read(ntc, 0, r0.mo, x[0]);
        if constexpr (MH == 1) {
          std::integral_constant<int, 1> mask;
          for (; b + S < U.w; b += 2 * S) {
            body(mask, r0, r1.mo, b);
            body(mask, r1, r0.mo, b + S);
          }
          if (b < U.w) body(mask, r0, r1.mo, b);
        } else {
          // bundles of the same halves in turn; r0 holds the first of each run
          auto run = [&](auto mask, int end) {
            for (; b + S < end; b += 2 * S) {
              body(mask, r0, r1.mo, b);
              body(mask, r1, r0.mo, b + S);
            }
            if (b < end) {
              body(mask, r0, r1.mo, b);
              const Bundle t = r0;
              r0 = r1;
              r1 = t;
              b += S;
            }
          };
          run(std::integral_constant<int, 1>{}, C.x);
          run(std::integral_constant<int, 2>{}, C.y);
          run(std::integral_constant<int, 3>{}, U.w);
        }
      };
      if (!live) {
      } else if (px0 + 16 >= a.nx)  // the patch's second tile column lies outside the scan
        all(std::integral_constant<int, 1>{});
      else
        all(std::integral_constant<int, TPR>{});
      if (u + 1 < u1) {
        // the next row offsets' new rows go to the free slots while other waves still read this
        // unit
        if (!(Un.x == U.x + ST && Un.y == U.y)) __syncthreads();
        stage(Un, lo);
        __syncthreads();
        U = Un;
      }
    }
  }
  const bool finite = ring_store<Op, BR, BC, W, P>(acc, lds, a, piece, out, threadIdx.x, py0, px0,
                                                   kF32OperandExp + a.exp);
  __syncthreads();
  int* flag = reinterpret_cast<int*>(lds);
  const int mine = __any(!finite);
  if (lane == 0) flag[wave] = mine;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) any |= flag[w];
  if (any) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // nothing is kept in registers for this
    ring_guarded<Op, BR, BC, W, P, RAGGED>(pack, in, out, lds, a, piece, tid, py0, px0);
  }
}

// Output of the cut tiles: the sum of a tile's partial slots in slot order (the order of the
// tile's stage units).  Grid: (patch, tile); workgroups of tiles that were not cut return at
// once.  A thread adds four consecutive rows of a position.
template <typename T, int BR, int BC, int TM>
__global__ __launch_bounds__(256) void k_add_slots(const int2* __restrict__ tile_split,
                                                   const T* __restrict__ partial,
                                                   T* __restrict__ out, int n_patches, int ncc,
                                                   int nx, int ny, int out_len) {
  typedef T T4 __attribute__((ext_vector_type(4)));
  constexpr int PS4 = BR * BC * TM / 4;  // quads per slot and patch
  const int tile = blockIdx.y;
  const int2 sp = tile_split[tile];
  if (sp.x < 2) return;
  const int py0 = (blockIdx.x / ncc) * BR, px0 = (blockIdx.x % ncc) * BC;
  const T4* base = reinterpret_cast<const T4*>(partial) + ((long long)sp.y * n_patches + blockIdx.x) * PS4;
  const long long stride = (long long)n_patches * PS4;
  for (int e = threadIdx.x; e < PS4; e += 256) {
    const int pos = e / (TM / 4), row = TM * tile + 4 * (e % (TM / 4));
    const int py = py0 + pos / BC, px = px0 + pos % BC;
    if (py >= ny || px >= nx || row >= out_len) continue;
    T4 v = base[e];
    int j = 1;
    for (; j + 3 < sp.x; j += 4) {  // four loads in flight
      const T4 a = base[j * stride + e], b = base[(j + 1) * stride + e],
               c = base[(j + 2) * stride + e], d = base[(j + 3) * stride + e];
      v += a;
      v += b;
      v += c;
      v += d;
    }
    for (; j < sp.x; ++j) v += base[j * stride + e];
    T* o = out + ((long long)py * nx + px) * out_len + row;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (row + i < out_len) o[i] = v[i];
  }
}

// ------------------------------------------------------------------------------------------
// FP8 applies: e4m3 table and e4m3 operand on the block-scaled FP8 MFMA
// (v_mfma_scale_f32_16x16x128_f8f6f4).  The operand (image or signals) gets one power-of-two
// scale per chunk of 64 entries of its fast axis over all scan positions, so every K-group of a
// stage unit (one chunk) shares it; the table's scale per (offset, 16-depth block) is carried
// per scale block of a bundle (see the layout).

// NaN-carrying maximum (fmaxf drops a NaN).
__device__ inline float nan_maxf(float a, float b) { return (a > b || a != a) ? a : b; }

// part[c * nparts + p] = max |in| over the entries of chunk c (64 entries of the fast axis) of
// the scan positions p, p + nparts, ...  Grid (nparts, chunks); 256 threads = 4 positions x 64.
__global__ __launch_bounds__(256) void k_chunk_amax(const float* __restrict__ in, long long npos,
                                                    int L, float* __restrict__ part) {
  __shared__ float sh[256];
  const int c = blockIdx.y, nparts = gridDim.x;
  const int e = threadIdx.x % 64, r = threadIdx.x / 64;
  const int l = c * 64 + e;
  float m = 0.0f;
  if (l < L)
    for (long long i = blockIdx.x + (long long)nparts * r; i < npos; i += 4LL * nparts)
      m = nan_maxf(m, fabsf(in[i * L + l]));
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] = nan_maxf(sh[threadIdx.x], sh[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(long long)c * nparts + blockIdx.x] = sh[0];
}

// Per chunk: the smallest power of two 2^e >= amax / 448 (e = 0 for a chunk of zeros or a
// non-finite amax, whose NaN codes then reach the output), as the E8M0 byte e + 127 and 2^-e.
// 448 = 0.875 2^9, so with amax = m 2^ea (0.5 <= m < 1): e = ea - 9 if m <= 0.875, else ea - 8.
__global__ void k_chunk_scales(const float* __restrict__ part, int nparts, int nch,
                               int* __restrict__ xexp, float* __restrict__ xinv) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nch) return;
  float a = 0.0f;
  for (int p = 0; p < nparts; ++p) a = nan_maxf(a, part[(long long)c * nparts + p]);
  int e = 0;
  if (a > 0.0f && a <= 3.402823466e38f) {
    int ea;
    const float mnt = frexpf(a, &ea);
    e = mnt <= 0.875f ? ea - 9 : ea - 8;
  }
  e = max(-126, min(127, e));
  xexp[c] = e + 127;
  xinv[c] = ldexpf(1.0f, -e);
}

// Stage an FP32 input into the zero-padded e4m3 layout [nyp][nxp][Lp] (codes of x 2^-e of its
// chunk); one workgroup of 64 threads per padded column, each thread four consecutive entries
// (one chunk, since Lp and the chunk are multiples of 4) written as one 32-bit word.  vec4: the
// input rows are 16-byte aligned (L % 4 == 0 and an aligned base), so they load as float4.
__global__ __launch_bounds__(64) void k_stage_fp8(const float* __restrict__ in,
                                                  uint8_t* __restrict__ out,
                                                  const float* __restrict__ xinv, int K, int nx,
                                                  int ny, int nxp, int L, int Lp, int vec4) {
  const int col = blockIdx.x;
  const int px = col % nxp - K, py = col / nxp - K;
  uint32_t* o = reinterpret_cast<uint32_t*>(out + (long long)col * Lp);
  const bool inside = px >= 0 && px < nx && py >= 0 && py < ny;
  const float* src = in + ((long long)py * nx + px) * L;
  for (int q = threadIdx.x; q < Lp / 4; q += blockDim.x) {
    const int l0 = 4 * q;
    uint32_t w = 0;
    if (inside && l0 < L) {
      float v[4];
      if (vec4) {
        const float4 f = *reinterpret_cast<const float4*>(src + l0);
        v[0] = f.x, v[1] = f.y, v[2] = f.z, v[3] = f.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = l0 + i < L ? src[l0 + i] : 0.0f;
      }
      const float sc = xinv[l0 / 64];
#pragma unroll
      for (int i = 0; i < 4; ++i) w |= (uint32_t)f32_to_e4m3(v[i] * sc) << (8 * i);
    }
    o[q] = w;
  }
}

struct Fp8Args {
  const int4* pieces;  // (tile, unit begin, unit end, partial slot or -1)
  float* partial;      // [slot][patch][position][TM rows] partial sums of cut tiles
  int n_patches;
  const int4* units;   // (row offset, chunk start, bundle begin, bundle end)
  const int2* classes; // per unit: the end of its bundles of half 0 alone and of half 1 alone
  const u32x4* rec;    // per bundle and lane group: LDS offsets of its 4 K-groups within a row (16
                       // bits each), the E8M0 scale bytes of its block for the two halves and, from
                       // bit 16, the K-groups' row offset in the unit
  const int* xexp;     // per scale chunk of the operand: E8M0 scale byte
  int out_len, nx, ny, K, nxp, nyp, Lp;
  int ncc;             // patch columns
  int NCOL, CS;
};

constexpr int kFp8Vecs = kFp8Chunk / 16;  // staged vectors per column

// Table operand of one FP8 bundle for one lane: 32 bytes per half.
struct F8Frag {
  u32x4 v[2][2];
};

__device__ __forceinline__ void load_f8(const uint8_t* __restrict__ pack, int b, int lane,
                                        F8Frag& f) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const u32x4* p = reinterpret_cast<const u32x4*>(pack + (((long long)b * 2 + h) * 64 + lane) * 32);
    f.v[h][0] = p[0];
    f.v[h][1] = p[1];
  }
}

// One word of lane group g's record for bundle b: lane 4q + j of each quad loads word j, and
// rec8_word broadcasts word J within the quad (a lane needs only its own lane group's words).
// Vector loads, since a record that came through the scalar path would make every wait on the
// LDS reads wait for it as well (scalar loads complete out of order, so the shared counter can
// only be waited to zero); one word per lane, since the texture path bounds this loop.
__device__ __forceinline__ uint32_t load_rec8(const Fp8Args& a, int b, int g, int lane) {
  return reinterpret_cast<const uint32_t*>(a.rec)[((long long)b * kLaneGroups + g) * 4 + (lane & 3)];
}

// Word J of the lane group's record: lane 4q + J of each quad loaded it (quad_perm [J,J,J,J]).
template <int J>
__device__ __forceinline__ uint32_t rec8_word(uint32_t w) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x55 * J, 0xF, 0xF, false);
}

// LDS offsets of the lane group's four K-groups in an FP8 bundle (record words 0 and 1).
struct X8Offs {
  int o[4];
};

__device__ __forceinline__ X8Offs x8_offsets(uint32_t w) {
  const uint32_t r0 = rec8_word<0>(w), r1 = rec8_word<1>(w);
  return X8Offs{{(int)(r0 & 0xffff), (int)(r0 >> 16), (int)(r1 & 0xffff), (int)(r1 >> 16)}};
}

// Position fragments of one FP8 bundle for the TPR tiles of row r of the wave's rows: for each of
// the lane group's four K-groups, 8 bytes of the lane's position from the LDS.  The K-groups' first
// row is at `first`; rows wrap into the ring of `ring` bytes (the subtraction underflows to a larger
// value where there is nothing to wrap).  The reads are volatile: otherwise the compiler pairs the
// reads of neighbouring tiles into one instruction whose registers then have to be moved into
// each MFMA's operand order (or, with the tiles' distance as a run-time value, needs an addition
// for each read).
typedef const volatile __attribute__((address_space(3))) u32x2 LdsPair;

template <int TPR>
__device__ __forceinline__ void read_x8(const uint8_t* lds, unsigned first, unsigned row_bytes,
                                        unsigned ring, int r, const X8Offs& o, u32x4 (&x)[TPR][2]) {
  const unsigned q = first + r * row_bytes;
  const uint8_t* row = lds + min(q, q - ring);
#pragma unroll
  for (int t = 0; t < TPR; ++t) {
    u32x2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      v[k] = *((LdsPair*)(row + o.o[k]) + t * 16 * kRingColumnBytes / 8);
    x[t][0] = u32x4{v[0].x, v[0].y, v[1].x, v[1].y};
    x[t][1] = u32x4{v[2].x, v[2].y, v[3].x, v[3].y};
  }
}

// The block-scaled MFMAs of half H of one FP8 bundle for tiles [t0, t0 + NX) (t0 a constant
// after unrolling) whose fragments are x[0 .. NX): 16 rows x 128 K x 16 positions each, with
// the lane's block scale byte H of sc and the unit's operand scale xs.
template <int H, int NT, int NX>
__device__ __forceinline__ void fp8_mma_h(const F8Frag& f, int sc, int xs, int t0,
                                          const u32x4 (&x)[NX][2], floatx4 (&acc)[2][NT]) {
  const intx8 av = __builtin_bit_cast(
      intx8, u32x8{f.v[H][0].x, f.v[H][0].y, f.v[H][0].z, f.v[H][0].w, f.v[H][1].x, f.v[H][1].y,
                   f.v[H][1].z, f.v[H][1].w});
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const intx8 bv = __builtin_bit_cast(intx8, u32x8{x[i][0].x, x[i][0].y, x[i][0].z, x[i][0].w,
                                                     x[i][1].x, x[i][1].y, x[i][1].z, x[i][1].w});
    acc[H][t0 + i] =
        __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, acc[H][t0 + i], 0, 0, H, sc, 0, xs);
  }
}

constexpr int kSplit8 = 4;  // waves that share a unit's bundles

// LDS-staged FP8 kernel: the ring kernel's units of kRingStep row offsets (of chunks of 32 entries)
// and order of bundles (half 0 alone, half 1 alone, both), with bundles of 16 K-groups: per reached
// 16-row half and position tile one block-scaled MFMA of K = 128.  The waves form 4 / S row groups
// of the BR x BC patch; the S waves of a row group take every S-th bundle of each stage unit, and
// the S partial sums of a position are added in wave order through the LDS at the end.  Lane (n, g)
// reads, for each of its lane group's four K-groups, 8 bytes of position n from the LDS (the
// K-group's row, column and run) and 32 bytes of table row n per half.
//
// What bounds it is latency at two waves per SIMD (the accumulators take half the registers).  With
// one row offset to a unit (of 64 entries) a unit had four bundles or so, which four waves share
// unevenly and with a barrier each; with a test of the reached halves per bundle the compiler
// waits for all reads of a row before its MFMAs.  Units of four row offsets, runs of bundles of the
// same halves, a row's fragments read while the row before multiplies and a staging without
// registers to spill: 400 x 400 forward 12.2 -> 10.7 ms, 200 x 200 x 128 (K 20) 741 -> 599 us,
// its adjoint 786 -> 663, 256 x 256 x 64 (K 10) 280 -> 217.
template <int BR, int BC, int S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_apply_fp8s(
    const uint8_t* __restrict__ pack, const uint8_t* __restrict__ in, float* __restrict__ out,
    Fp8Args a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  uint8_t* lds = lds_raw;
  constexpr int TPR = BC / 16;
  constexpr int P = 4 / S;
  constexpr int RW = BR / P;
  constexpr int NT = RW * TPR;
  static_assert(4 % S == 0 && BR % P == 0 && NT % S == 0 && RW % 2 == 0, "split shape");
  constexpr int UR = BR + kRingStep - 1, RS = UR + kRingStep;  // rows of a unit, of the ring
  constexpr int MH = 2;
  const int4 piece = a.pieces[blockIdx.y];
  const int tile = piece.x;
  const int py0 = (blockIdx.x / a.ncc) * BR, px0 = (blockIdx.x % a.ncc) * BC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int grp = wave / S, sw = wave % S;
  const int n = lane % 16, g = lane / 16;
  const int rowvec = a.NCOL * kFp8Vecs;
  const unsigned row_bytes = a.NCOL * a.CS;
  floatx4 acc[MH][NT];
#pragma unroll
  for (int h = 0; h < MH; ++h)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[h][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  // Write the rows that unit U adds, padded patch rows [lo, U.x + K + UR), to the ring.  A wave takes
  // every fourth row, 64 vectors at a time, so that rows are uniform and a lane's offsets within
  // them fixed.  Nothing is fetched ahead: the registers that takes are spilled (400 x 400 forward
  // 11.1 ms with one vector ahead, 11.8 with three).
  const unsigned lane_lds = lane / kFp8Vecs * kRingColumnBytes + lane % kFp8Vecs * 16;
  const unsigned lane_in = lane / kFp8Vecs * a.Lp + lane % kFp8Vecs * 16;
  constexpr int kCols = 64 / kFp8Vecs;  // columns of 64 vectors
  auto stage = [&](const int4& U, int lo) {
    for (int G = lo + wave; G < U.x + a.K + UR; G += 4) {
      uint8_t* dst = lds + G % RS * row_bytes + lane_lds;
      // rows past the last padded one belong to row offsets without K-groups
      const uint8_t* row =
          in + ((long long)min(py0 + G, a.nyp - 1) * a.nxp + px0) * a.Lp + U.y;
      for (int i0 = 0; 64 * i0 < rowvec; i0 += 4) {
        u32x4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (lane + 64 * (i0 + i) < rowvec)
            v[i] = *reinterpret_cast<const u32x4*>(
                row + (lane_in + (unsigned)((i0 + i) * kCols * a.Lp)));
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (lane + 64 * (i0 + i) < rowvec)
            *reinterpret_cast<u32x4*>(dst + (i0 + i) * kCols * kRingColumnBytes) = v[i];
      }
    }
  };
  const int u0 = piece.y, u1 = piece.z;
  if (u0 < u1) {
    // Two bundles of the wave: table fragments and record words.
    struct Bundle {
      F8Frag f;
      uint32_t w;
    };
    Bundle r0, r1;
    auto load = [&](Bundle& r, int b) {
      load_f8(pack, b, lane, r.f);
      r.w = load_rec8(a, b, g, lane);
    };
    int4 U = a.units[u0];
    load(r0, min(U.z + sw, U.w - 1));
    load(r1, min(U.z + sw + S, U.w - 1));
    stage(U, U.x + a.K);
    __syncthreads();
    for (int u = u0; u < u1; ++u) {
      const int4 Un = a.units[min(u + 1, u1 - 1)];
      const int2 C = a.classes[u];
      // rows the next unit finds in the ring: those of this unit, in the same chunk
      const int lo = Un.y == U.y && Un.x < U.x + UR ? U.x + a.K + UR : Un.x + a.K;
      const int xs = a.xexp[U.y / kFp8ScaleChunk];
      const unsigned s0 = (grp * RW + U.x + a.K) % RS * row_bytes + n * kRingColumnBytes;
      const unsigned ring = RS * row_bytes;
      int b = U.z + sw;
      if (b < U.w) {
        // The fragments of a row are read while the row before multiplies (the barriers keep the
        // compiler from moving the reads next to their use).
        u32x4 x[2][TPR][2];
        X8Offs o = x8_offsets(r0.w);
        int sc = (int)rec8_word<2>(r0.w);
        unsigned first = s0 + ((unsigned)sc >> 16) * row_bytes;
        read_x8<TPR>(lds, first, row_bytes, ring, 0, o, x[0]);
        // bundle b, of the halves in MASK; `next` holds the wave's next one
        auto body = [&](auto mask, Bundle& r, const Bundle& next) {
          constexpr int MASK = decltype(mask)::value;
          int scn = 0;
#pragma unroll
          for (int p = 0; p < RW; ++p) {
            if (p + 1 == RW) {
              o = x8_offsets(next.w);
              scn = (int)rec8_word<2>(next.w);
              first = s0 + ((unsigned)scn >> 16) * row_bytes;
            }
            read_x8<TPR>(lds, first, row_bytes, ring, (p + 1) % RW, o, x[(p + 1) % 2]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (MASK & 1) fp8_mma_h<0, NT, TPR>(r.f, sc, xs, p * TPR, x[p % 2], acc);
            if constexpr (MASK & 2) fp8_mma_h<1, NT, TPR>(r.f, sc, xs, p * TPR, x[p % 2], acc);
            __builtin_amdgcn_sched_barrier(0);
          }
          sc = scn;
          b += S;
        };
        // bundles of the same halves in turn; r0 holds the first of each run
        auto run = [&](auto mask, int end) {
          while (b + S < end) {
            body(mask, r0, r1);
            load(r0, min(b + S, U.w - 1));
            body(mask, r1, r0);
            load(r1, min(b + S, U.w - 1));
          }
          if (b < end) {
            body(mask, r0, r1);
            r0 = r1;
            load(r1, min(b + S, U.w - 1));
          }
        };
        run(std::integral_constant<int, 1>{}, C.x);
        run(std::integral_constant<int, 2>{}, C.y);
        run(std::integral_constant<int, 3>{}, U.w);
      }
      if (u + 1 < u1) {
        load(r0, min(Un.z + sw, Un.w - 1));
        load(r1, min(Un.z + sw + S, Un.w - 1));
        // the next row offsets' new rows go to the free slots while other waves still read this unit
        if (!(Un.x == U.x + kRingStep && Un.y == U.y)) __syncthreads();
        stage(Un, lo);
        __syncthreads();
        U = Un;
      }
    }
  }
  constexpr int PS = BR * BC * 16 * MH;
  float* slot =
      piece.w >= 0 ? a.partial + ((long long)piece.w * a.n_patches + blockIdx.x) * PS : nullptr;
  floatx4* red = reinterpret_cast<floatx4*>(lds_raw);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < NT; p += S) {
#pragma unroll
    for (int k = 0; k < S; ++k)
#pragma unroll
      for (int h = 0; h < MH; ++h) red[((wave * S + k) * MH + h) * 64 + lane] = acc[h][p + k];
    __syncthreads();
    floatx4 v[MH];
#pragma unroll
    for (int h = 0; h < MH; ++h) {
      v[h] = red[(((grp * S) * S + sw) * MH + h) * 64 + lane];
#pragma unroll
      for (int s = 1; s < S; ++s) v[h] += red[(((grp * S + s) * S + sw) * MH + h) * 64 + lane];
    }
    const int t = p + sw;
    const int py = py0 + grp * RW + t / TPR, px = px0 + (t % TPR) * 16 + n;
    if (py < a.ny && px < a.nx) {
      const int local = (grp * RW + t / TPR) * BC + (t % TPR) * 16 + n;
      float* dst = slot ? slot : out;
      const long long off = slot ? (long long)local * (16 * MH) - 16 * MH * tile
                                 : ((long long)py * a.nx + px) * a.out_len;
#pragma unroll
      for (int h = 0; h < MH; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * MH * tile + 16 * h + 4 * g + i;
          if (row < a.out_len) dst[off + row] = v[h][i];
        }
    }
    __syncthreads();
  }
}

size_t elem_bytes(int dtype) {
  switch (dtype) {
    case AROAM_FP64: return 8;
    case AROAM_FP32: return 4;
    case AROAM_BF16: return 2;
    default: return 1;  // e4m3
  }
}

constexpr int kAmaxParts = 512;  // position slices of the FP8 operand's chunk maxima

}  // namespace

const Layout& layout_for(const Model& m, bool adjoint, int dtype) {
  if (dtype == AROAM_FP64) return adjoint ? m.r64a : m.r64f;
  if (dtype == AROAM_FP32) return adjoint ? m.r32a : m.r32f;
  if (dtype == AROAM_BF16) return adjoint ? m.r16a : m.r16f;
  return adjoint ? m.f8a : m.f8f;
}

namespace {

// The stage buffer of an apply.  FP64 and FP32: the partial slots of a layout with cut tiles,
// [slot][patch][position of the patch][tile rows]; nothing where no tile is cut.  BF16 and FP8: the
// padded input, then the partial slots (FP32), then for FP8 the operand's chunk scales: partial
// maxima [chunk][kAmaxParts] (FP32), E8M0 bytes [chunk] (int) and inverse scales [chunk] (FP32).
struct StageParts {
  size_t input = 0, partial = 0, scales = 0;
  int chunks = 0;
};

StageParts stage_parts(const Model& m, bool adjoint, int dtype) {
  const Layout& lay = layout_for(m, adjoint, dtype);
  StageParts p;
  p.input = (size_t)round_up(lay.in.elems() * elem_bytes(dtype), 256);
  p.chunks = dtype == AROAM_FP8E4M3 ? (int)ceil_div(lay.in.L, kFp8ScaleChunk) : 0;
  p.scales = (size_t)round_up((size_t)p.chunks * (kAmaxParts + 2) * 4, 256);
  if (lay.n_slots > 0)
    p.partial = (size_t)lay.n_slots * lay.n_patches * lay.TM * lay.BR * lay.BC *
                (dtype == AROAM_FP64 ? sizeof(double) : sizeof(float));
  return p;
}

}  // namespace

size_t input_bytes(const Model& m, bool adjoint, int dtype) {
  const StageParts p = stage_parts(m, adjoint, dtype);
  return p.input + p.scales;
}

size_t stage_bytes(const Model& m, bool adjoint, int dtype) {
  const StageParts p = stage_parts(m, adjoint, dtype);
  if (dtype == AROAM_FP64 || dtype == AROAM_FP32) return p.partial;
  return p.input + p.partial + p.scales;
}

namespace {

// Allow the full LDS of a CU for a kernel, once per device.
template <typename F>
int allow_full_lds(F kern, std::atomic<unsigned long long>& done) {
  int dev = 0;
  AROAM_HIP(hipGetDevice(&dev));
  const unsigned long long bit = 1ull << (dev & 63);
  if (!(done.load() & bit)) {
    AROAM_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)kLdsBytes));
    done.fetch_or(bit);
  }
  return AROAM_OK;
}

template <class Op, int BR>
int launch_ring(const Model& m, const Layout& lay, const Pack& pk, const void* in, void* partial,
                void* out, hipStream_t st) {
  constexpr int W = 4, P = 1;  // waves of a workgroup, row groups they form
  using In = typename Op::In;
  auto kern = k_apply_ring<Op, BR, kPatchCols, W, P, false>;
  bool ragged = false;
  if constexpr (!Op::kBlocked) {  // a blocked input is padded to whole vectors
    ragged = lay.in.L % Op::kVec != 0;
    if (ragged) kern = k_apply_ring<Op, BR, kPatchCols, W, P, true>;
  }
  static std::atomic<unsigned long long> attr_set[2];
  AROAM_TRY(allow_full_lds(kern, attr_set[ragged]));
  RingArgs a;
  a.pieces = lay.d_pieces;
  a.units = lay.d_units;
  a.meta = lay.d_meta;
  a.partial = partial;
  a.n_patches = lay.n_patches;
  a.out_len = lay.out_len;
  a.nx = lay.in.nx;
  a.ny = lay.in.ny;
  a.K = lay.in.K;
  a.L = lay.in.L;
  a.ncc = (int)ceil_div(lay.in.nx, kPatchCols);
  a.NCOL = lay.NCOL;
  a.row_bytes = ring_row_bytes(a.K, Op::kCol);
  a.classes = lay.d_classes;
  a.nxp = lay.in.nxp;
  a.nyp = lay.in.nyp;
  a.exp = m.f32_exp;
  AROAM_CHECK(lay.TM == kTile * Op::kHalves && lay.BR == BR && lay.BC == kPatchCols &&
                  lay.NCOL == kPatchCols + 2 * a.K && lay.CH == Op::kVec * Op::kVecs &&
                  (!Op::kBlocked || lay.in.nxp >= (int)round_up(a.nx, kPatchCols) + 2 * a.K),
              AROAM_EINVAL, "ring layout shape mismatch");
  AROAM_CHECK(lay.n_patches == ceil_div(lay.in.ny, BR) * a.ncc, AROAM_EINVAL, "patch count mismatch");
  AROAM_CHECK(lay.n_slots == 0 || partial, AROAM_EINVAL, "no partial slots for a cut layout");
  const size_t red = (size_t)W * (W / P) * Op::kHalves * 64 * sizeof(typename Op::Acc);
  const dim3 grid((unsigned)lay.n_patches, (unsigned)lay.n_pieces);
  hipLaunchKernelGGL(kern, grid, dim3(64 * W), std::max(lay.lds_bytes, red), st, (const void*)pk.d,
                     (const In*)in, (In*)out, a);
  if (lay.n_slots > 0)
    hipLaunchKernelGGL((k_add_slots<In, BR, kPatchCols, kTile * Op::kHalves>),
                       dim3((unsigned)lay.n_patches, (unsigned)lay.n_tiles), dim3(256), 0, st,
                       lay.d_tile_split, (const In*)partial, (In*)out, lay.n_patches, a.ncc, a.nx,
                       a.ny, a.out_len);
  return AROAM_OK;
}

}  // namespace

namespace {

// FP8 apply: chunk maxima and scales of the operand, the e4m3 staging, the staged FP8 kernel,
// and the slot sums of cut tiles.
int launch_fp8(const Model& m, const Layout& lay, const Pack& pk, const float* in, void* buf,
               const StageParts& sp, void* out, hipStream_t st) {
  auto kern = k_apply_fp8s<kPatchRows, kPatchCols, kSplit8>;
  static std::atomic<unsigned long long> attr_set{0};
  AROAM_TRY(allow_full_lds(kern, attr_set));
  AROAM_CHECK(lay.TM == kTileRows8 && lay.CH == kFp8Chunk && lay.CS == kRingColumnBytes &&
                  lay.NCOL == kPatchCols + 2 * lay.in.K &&
                  lay.in.nxp >= (int)round_up(lay.in.nx, kPatchCols) + 2 * lay.in.K,
              AROAM_EINVAL, "FP8 layout shape mismatch");
  const PadGeom& pg = lay.in;
  char* base = static_cast<char*>(buf);
  uint8_t* staged = reinterpret_cast<uint8_t*>(base);
  float* partial = sp.partial > 0 ? reinterpret_cast<float*>(base + sp.input) : nullptr;
  float* amax = reinterpret_cast<float*>(base + sp.input + sp.partial);
  int* xexp = reinterpret_cast<int*>(amax + (size_t)sp.chunks * kAmaxParts);
  float* xinv = reinterpret_cast<float*>(xexp + sp.chunks);
  const long long npos = (long long)pg.nx * pg.ny;
  hipLaunchKernelGGL(k_chunk_amax, dim3(kAmaxParts, (unsigned)sp.chunks), dim3(256), 0, st, in,
                     npos, pg.L, amax);
  hipLaunchKernelGGL(k_chunk_scales, dim3((unsigned)ceil_div(sp.chunks, 64)), dim3(64), 0, st,
                     (const float*)amax, kAmaxParts, sp.chunks, xexp, xinv);
  AROAM_CHECK(pg.Lp % 64 == 0, AROAM_EINVAL, "FP8 staging needs whole 64-entry chunks");
  const int vec4 = pg.L % 4 == 0 && reinterpret_cast<uintptr_t>(in) % 16 == 0;
  hipLaunchKernelGGL(k_stage_fp8, dim3((unsigned)(pg.nyp * pg.nxp)), dim3(64), 0, st, in, staged,
                     (const float*)xinv, pg.K, pg.nx, pg.ny, pg.nxp, pg.L, pg.Lp, vec4);
  Fp8Args a;
  a.pieces = lay.d_pieces;
  a.partial = partial;
  a.n_patches = lay.n_patches;
  a.units = lay.d_units;
  a.classes = lay.d_classes;
  a.rec = reinterpret_cast<const u32x4*>(lay.d_meta);
  a.xexp = xexp;
  a.out_len = lay.out_len;
  a.nx = pg.nx;
  a.ny = pg.ny;
  a.K = pg.K;
  a.nxp = pg.nxp;
  a.nyp = pg.nyp;
  a.Lp = pg.Lp;
  a.ncc = (int)ceil_div(pg.nx, kPatchCols);
  a.NCOL = lay.NCOL;
  a.CS = lay.CS;
  AROAM_CHECK(lay.n_patches == ceil_div(pg.ny, kPatchRows) * a.ncc, AROAM_EINVAL,
              "patch count mismatch");
  AROAM_CHECK(lay.n_slots == 0 || partial, AROAM_EINVAL, "no partial slots for a cut layout");
  const dim3 grid((unsigned)lay.n_patches, (unsigned)lay.n_pieces);
  hipLaunchKernelGGL(kern, grid, dim3(256), std::max(lay.lds_bytes, red_bytes(kSplit8, 2)), st,
                     (const uint8_t*)pk.d, (const uint8_t*)staged, (float*)out, a);
  if (lay.n_slots > 0)
    hipLaunchKernelGGL((k_add_slots<float, kPatchRows, kPatchCols, kTileRows8>),
                       dim3((unsigned)lay.n_patches, (unsigned)lay.n_tiles), dim3(256), 0, st,
                       lay.d_tile_split, (const float*)partial, (float*)out, lay.n_patches, a.ncc,
                       a.nx, a.ny, a.out_len);
  return AROAM_OK;
}

// The launches of one apply into the stage buffer `buf` (stage_bytes() bytes).
int launch_apply(const Model& m, bool adjoint, int dtype, const void* in, void* out, void* buf,
                 hipStream_t st) {
  const Layout& lay = layout_for(m, adjoint, dtype);
  const Pack& pk = adjoint ? m.adj_pack[dtype] : m.fwd_pack[dtype];
  if (dtype == AROAM_FP8E4M3) {
    AROAM_TRY(launch_fp8(m, lay, pk, (const float*)in, buf, stage_parts(m, adjoint, dtype), out,
                         st));
  } else if (dtype == AROAM_FP64) {
    AROAM_TRY((launch_ring<OpF64, 4>(m, lay, pk, in, buf, out, st)));
  } else if (dtype == AROAM_FP32) {
    auto launch = m.f32_far ? (lay.BR == 8 ? launch_ring<OpF32Far, 8> : launch_ring<OpF32Far, 4>)
                            : (lay.BR == 8 ? launch_ring<OpF32, 8> : launch_ring<OpF32, 4>);
    AROAM_TRY(launch(m, lay, pk, in, buf, out, st));
  } else {
    const PadGeom& pg = lay.in;
    const int nch = (int)ceil_div(pg.L, kRingBF16.G);
    hipLaunchKernelGGL(k_stage_bf16,
                       dim3((unsigned)(ceil_div(pg.nxp, 32) * pg.nyp), (unsigned)ceil_div(nch, 8)),
                       dim3(256), 0, st, (const float*)in, (u32x4*)buf, pg.K, pg.nx, pg.ny, pg.nxp,
                       pg.nyp, pg.L, nch);
    const StageParts sp = stage_parts(m, adjoint, dtype);
    void* partial = static_cast<char*>(buf) + sp.input;
    AROAM_TRY((launch_ring<OpBF16, kPatchRows>(m, lay, pk, buf, partial, out, st)));
  }
  AROAM_HIP(hipGetLastError());
  return AROAM_OK;
}

}  // namespace

int apply(const Model& m, bool adjoint, int dtype, const void* in, void* out, void* stage,
          hipStream_t st) {
  AROAM_CHECK(dtype >= AROAM_FP64 && dtype <= AROAM_FP8E4M3, AROAM_EINVAL, "bad dtype %d", dtype);
  AROAM_CHECK(in && out, AROAM_EINVAL, "NULL vector");
  AROAM_CHECK((m.dtype_mask >> dtype) & 1u, AROAM_EUNSUPPORTED,
              "model was not packed for dtype %d", dtype);
  const Layout& lay = layout_for(m, adjoint, dtype);
  AROAM_CHECK(lay.lds_bytes <= kLdsBytes, AROAM_EINVAL,
              "lateral footprint too wide for the LDS stage (%zu bytes)", lay.lds_bytes);
  if (stage) return launch_apply(m, adjoint, dtype, in, out, stage, st);
  const size_t need = stage_bytes(m, adjoint, dtype);
  if (need == 0) return launch_apply(m, adjoint, dtype, in, out, nullptr, st);
  // a stage buffer of its own from the pool, returned to the pool on every path
  void* buf = nullptr;
  AROAM_TRY(pool_alloc(&buf, need, st));
  const int rc = launch_apply(m, adjoint, dtype, in, out, buf, st);
  const hipError_t e = hipFreeAsync(buf, st);
  if (rc != AROAM_OK) return rc;
  AROAM_CHECK(e == hipSuccess, AROAM_EDEVICE, "hipFreeAsync failed: %s", hipGetErrorString(e));
  return AROAM_OK;
}

// Stage buffer of the allocation-free applies: a static device array, one copy per GPU the
// library runs on, held until the process ends.  In host code `scratch` names a host-side
// stand-in, so its device address is looked up once per device and only that address is
// passed to kernels.
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

int static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  AROAM_HIP(hipGetDevice(&dev));
  AROAM_CHECK(dev >= 0 && dev < kMaxDevices, AROAM_EDEVICE, "device %d out of range", dev);
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    AROAM_CHECK(e == hipSuccess && p, AROAM_EDEVICE,
                "hipGetSymbolAddress of the static scratch buffer failed: %s", hipGetErrorString(e));
    addr[dev] = p;
  }
  *out = addr[dev];
  return AROAM_OK;
}

}  // namespace

int apply_noalloc(const Model& m, bool adjoint, int dtype, const void* in, void* out,
                  hipStream_t st) {
  AROAM_CHECK(dtype >= AROAM_FP64 && dtype <= AROAM_FP8E4M3, AROAM_EINVAL, "bad dtype %d", dtype);
  AROAM_CHECK(in && out, AROAM_EINVAL, "NULL vector");
  AROAM_CHECK((m.dtype_mask >> dtype) & 1u, AROAM_EUNSUPPORTED,
              "model was not packed for dtype %d", dtype);
  const Layout& lay = layout_for(m, adjoint, dtype);
  AROAM_CHECK(lay.lds_bytes <= kLdsBytes, AROAM_EINVAL,
              "lateral footprint too wide for the LDS stage (%zu bytes)", lay.lds_bytes);
  // The padded input counts for FP64 and FP32 too, so that the limit is one of the scan's size; the
  // launches are planned so that the slots then fit as well.
  const size_t need =
      std::max(stage_bytes(m, adjoint, dtype), input_bytes(m, adjoint, dtype));
  AROAM_CHECK(need <= kStaticScratchBytes, AROAM_EINVAL,
              "the apply's padded input and scratch come to %zu bytes; the static buffer holds %zu",
              need, (size_t)kStaticScratchBytes);
  void* buf = nullptr;
  AROAM_TRY(static_scratch(&buf));
  return launch_apply(m, adjoint, dtype, in, out, buf, st);
}

int apply_batch(int n, const Model* const* ms, bool adjoint, int dtype, const float* const* in,
                float* const* out, hipStream_t st) {
  AROAM_CHECK(n >= 0 && (n == 0 || (ms && in && out)), AROAM_EINVAL, "bad batch arguments");
  // the batch's vectors are FP32: FP64 applies would read and write doubles
  AROAM_CHECK(dtype == AROAM_FP32 || dtype == AROAM_BF16 || dtype == AROAM_FP8E4M3, AROAM_EINVAL,
              "batched applies take FP32, BF16 or FP8 (dtype %d)", dtype);
  for (int i = 0; i < n; ++i) {
    AROAM_CHECK(ms[i], AROAM_EINVAL, "NULL model in batch");
    AROAM_TRY(apply(*ms[i], adjoint, dtype, in[i], out[i], nullptr, st));
  }
  return AROAM_OK;
}

}  // namespace aroam
