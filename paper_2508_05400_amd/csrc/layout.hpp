// Sizes of the SpMV data layouts, shared by the kernels (kernels.hip) and the
// host code that builds the layouts (rks_api.cpp, panels.cpp).  Plain C++: no
// HIP types, so host-only code can include it.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace rks {

constexpr int kTileRows = 64;    // rows per SpMV wave tile
constexpr int kTileNnz = 512;    // nonzeros staged per SpMV wave tile (LDS slice)
constexpr int kTileFill = kTileNnz - 2;  // nonzeros a tile may hold: paired loads start at the even
                                         // index at or below its first nonzero
constexpr int kCsrPad = 2;       // readable padding entries after col[] and val[] (paired loads)
constexpr int kSpmvWaves = 4;    // waves per SpMV workgroup
constexpr int kSpmvMaxG = 1280;  // SpMV workgroups at most (5 per CU: LDS-bound for FP64 with d <= 360)

// Sliced layout: slices of kSliceRows consecutive rows (one per lane of a
// wave), each stored k-th nonzero of every row together; at most
// kSellMaxG workgroups of kSpmvWaves waves (6 per CU; no product staging in
// LDS, only the sketch bins).
constexpr int kSliceRows = 64;
constexpr int kSellMaxG = 1536;

// Column-blocked layout (operators whose rows gather x from everywhere):
// kCb column blocks (n / kCb values of x, which fit in an XCD's L2); row
// panels of consecutive rows, one workgroup each; panel tiles of up to
// kPanelTileRows rows.  Measured on a 2M-row power-law operator: 4, 16 or 32
// blocks and 128-row tiles are slower, as are twice as many, smaller panels.
constexpr int kCb = 8;
constexpr int kPanelTileRows = 256;
constexpr int kPanelRowsMin = 64;    // rows per panel at least (small matrices)
constexpr int kPanelRowsMax = 4096;  // rows per panel at most (the row sums live in LDS)

// Work before row r of a CSR matrix for a slot that walks rows one after the
// other (k_resid_csr): its nonzeros, and kResidRowCost of them for each row
// (an empty row waits for the next row pointer, 0.26 us; 1, 2, 4 and 16 measured
// within 2% of one another on power-law rows, with and without a run of empty ones).
constexpr int kResidRowCost = 2;
constexpr int64_t resid_key(int64_t e, int64_t r) { return e + kResidRowCost * r; }

// The first row of 0 .. n whose work before it is at least key.
constexpr int64_t resid_row_at(const int* rp, int64_t n, int64_t key) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (resid_key(rp[mid], mid) < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Entry q of the batch of entries at e, e < et (past the end: e).  Unsigned: et
// may be 2^31 - 1, past which e + q must not wrap (forming what is left of the
// range in signed arithmetic instead took k_resid_csr 6% longer).
constexpr uint32_t batch_entry(uint32_t e, uint32_t q, uint32_t et) { return e + q < et ? e + q : e; }

}  // namespace rks
