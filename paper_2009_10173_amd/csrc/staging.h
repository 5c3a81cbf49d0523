// Shape of the LDS stage of the staged applies (host-visible constants, no device types, so
// that the limits they imply can be built and tested on their own).
//
// A workgroup of a staged apply owns a patch of 4 or kPatchRows rows x kPatchCols columns of scan
// positions.  A stage unit covers kRingStep consecutive row offsets of one chunk of the inner
// axis, and the LDS holds the input rows a unit reads and the kRingStep rows the next one adds,
// as a ring.  A row holds the patch's columns plus a halo of k_half columns on each side; a column
// is one chunk, padded so that neighbouring columns spread over the LDS banks.  The lateral model
// extent k_half is therefore limited by the LDS of one compute unit.
#pragma once

namespace aroam {

constexpr int kPatchRows = 8;        // scan rows per workgroup patch
constexpr int kPatchCols = 32;       // scan columns per workgroup patch (two 16-position tiles)
constexpr long long kLdsBytes = 160 * 1024;  // LDS of one gfx950 compute unit

constexpr int kRingStep = 4;  // row offsets of a unit
// LDS bytes of a column: FP64, FP32 and FP8 (chunk of 32 bytes or three parts of 16, padding), BF16
constexpr int kRingColumnBytes = 48, kRing16ColumnBytes = 16;

// FP64, FP32, BF16: rows start at multiples of 256 bytes (all LDS banks), so that the row does not
// change a column's banks.
constexpr int ring_row_bytes(int k_half, int column_bytes = kRingColumnBytes) {
  return ((kPatchCols + 2 * k_half) * column_bytes + 255) / 256 * 256;
}
constexpr long long ring_lds_bytes(int k_half, int patch_rows, int column_bytes = kRingColumnBytes) {
  return (long long)(patch_rows + 2 * kRingStep - 1) * ring_row_bytes(k_half, column_bytes);
}

// LDS bytes of the FP8 ring of offsets -k_half .. k_half; the largest, with the FP32 ring of four
// patch rows: it limits k_half.
constexpr long long staged_lds_bytes(int k_half) {
  return (long long)(kPatchRows + 2 * kRingStep - 1) * (kPatchCols + 2 * k_half) * kRingColumnBytes;
}

// Largest k_half whose row ring fits the LDS.
constexpr int max_k_half() {
  int k = 0;
  while (staged_lds_bytes(k + 1) <= kLdsBytes) ++k;
  return k;
}

static_assert(ring_lds_bytes(max_k_half(), 4) <= kLdsBytes,
              "the ring of four patch rows fits wherever the FP8 one does");

// Patch rows of an FP32 ring launch.  Four rows leave room for three workgroups per CU while the
// LDS holds three rings; a wider footprint (K = 35 .. 40) leaves two either way, and then eight
// rows, which load the table half as often, are faster once the launch fills the chip (256 x 256
// x 128 forward: K 40 17.0 ms on four rows, 15.2 on eight; K 35 15.1 and 13.7; 150 x 210 x 100 adjoint,
// K 38 7.0 and 5.6).  At K 30 four rows hold their third workgroup (11.6 and 11.3 ms; 150 x 210 x 100
// 4.65 and 5.15).  FP64 keeps four rows: eight would need twice the accumulators' registers.
inline int ring_rows(int K, long long tiles, int nx, int ny, int cus) {
  const long long patches = (long long)((ny + 7) / 8) * ((nx + kPatchCols - 1) / kPatchCols);
  return 3 * ring_lds_bytes(K, 4) > kLdsBytes && 2 * ring_lds_bytes(K, 8) <= kLdsBytes &&
                 patches * tiles >= 4 * cus
             ? 8
             : 4;
}

}  // namespace aroam
