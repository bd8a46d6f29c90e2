// Device-side tables shared by the kernels and the host code that builds them.
#pragma once
#include <cstdint>
#include <type_traits>

namespace scasm {

// Width of a column tile of X (and of an F output tile): 4 stripes of 16
// columns, one stripe per wavefront in the TRSM.
constexpr int kTile = 64;
constexpr int kStripe = 16;
constexpr int kMaxPanel = 64;      // GPU panel width bound the TRSM kernel is built for
constexpr int kSyrkTile = 128;     // edge of an F output tile (two X column tiles)
constexpr int kFTileElems = kSyrkTile * kSyrkTile;
// Workgroups are dispatched to the accelerator's XCDs round-robin (workgroup
// k runs on XCD k mod kNumXcd); work lists are interleaved so that the items
// of one subdomain share an XCD and its L2, as far as that keeps all XCDs busy.
constexpr int kNumXcd = 8;
// Overlapped assembly: the batch is cut into this many groups of subdomains
// (each XCD's list into consecutive parts); the SYRK of a group runs on a
// second stream while the TRSM of the next group runs.
constexpr int kOverlapGroups = 8;

struct SubDev {
    int32_t n, m, nblocks, ntiles;
    int64_t blk_off;     // first block in the global block table
    int64_t rows_off;    // first entry of this subdomain's row array
    int64_t lval_off;    // first factor value
    int64_t col_off;     // first entry of piv / pi / sign (sorted order)
    int64_t tile_off;    // first tile in the global tile table
    int64_t F_off;       // first element of F: packed lower tiles in sorted column order
    int64_t ftile_off;   // first stored F tile of this subdomain (apply partial sums)
    int64_t dual_off;    // offset of the subdomain's multipliers in dual vectors
};

// One column tile of X: sorted columns [64*tile, 64*tile + ncols) of subdomain
// `sub`.  Its slab holds rows [kstart, n) x 64 columns, row-major.
struct TileDev {
    int32_t sub, tile, kstart, ncols;
    int64_t x_off;
    int64_t visit_off;        // blocks the tile visits: visits[visit_off .. + nvisit),
    int64_t fresh_off;        // increasing; their VisitDev::fresh masks from here on
    int64_t clear_off;        // rows cleared before the sweep: clear[clear_off .. + nclear)
    int32_t nvisit, nclear;
    int32_t nchunk, pad;      // chunks of the visits (TRSM steps)
};

// One factor block a TRSM tile visits, as the kernel walks it (offsets
// relative to the subdomain's factor values and row array).
struct VisitDev {
    uint64_t on;              // bit i: row row0 + i is in the slab and on the tile's paths
    uint64_t held;            // ... and was written before this visit (pivots, earlier updates)
    int64_t linv_off;         // inverse of the diagonal block
    int64_t aoff;             // pruned rows as MFMA A tiles
    int64_t pair_aoff;        // second block of a pair: the first block's A tiles of the same rows
    int64_t rows_off;
    int32_t row0, w;
    int32_t urows;            // rows the visit's update covers
    int32_t pair_nks;         // k-slices of those A tiles
    int32_t fresh;            // masks of the update's chunks at TileDev::fresh_off + fresh: bit i =
                              // row i of the chunk was never written before
    int32_t flags;            // bits 0-1: role in a merged pair (0 alone, 1 first block: updates only
                              // the next block's rows, 2 second block: also applies the first's
                              // update); kVisitNextEarly; kVisitActShift + v: stripe v has started
    int32_t pad;
};
// the last chunk of the visit's update holds no row of the next visit's block
constexpr int kVisitNextEarly = 4;
constexpr int kVisitActShift = 4;
// Pruned row tiles per TRSM chunk: 16 KB of A tiles, two FP64 or four FP32
// row tiles of 16 k-slices.
template <class TA>
constexpr int kPruneTiles = sizeof(TA) == 8 ? 2 : 4;
// X slabs from this size on are out of the 32-bit offsets of a buffer resource
constexpr int64_t kTrsmSlabBytes = 0xFFFFFF00ll;
// Where the TRSM finds an element of a slab: the byte offset in a buffer
// resource (an unsigned one, below kTrsmSlabBytes), or in larger slabs the
// element index, which outgrows 32 bits from 2^25 rows on (rows go up to 2^27).
template <class TX, bool LARGE>
constexpr typename std::conditional<LARGE, int64_t, int32_t>::type slab_offset(int row, int col) {
    using Off = typename std::conditional<LARGE, int64_t, int32_t>::type;
    return LARGE ? (Off)row * kTile + col : (Off)((uint32_t)(row * kTile + col) * (uint32_t)sizeof(TX));
}

// SYRK work item: a 64 x 64 block of F (I >= J in units of 64-column X
// tiles), its k-range a list of 16-row steps (first rows at
// ksteps[step_off .. step_off + nsteps)) where both X tiles can hold a nonzero
// row; or a 128 x 128 tile of F (I >= J in units of kSyrkTile), each step entry
// = first row | slab bits << kStepSlabShift, bit q set when 64-column slab q
// (2I, 2I+1, 2J, 2J+1) has a nonzero row in the step.  Every other step adds
// zero products.  Also used, in units of kSyrkTile and without steps, for the
// stored F tiles of the apply.
struct SyrkItem {
    int32_t sub;
    int32_t I, J;
    int32_t nsteps;
    int64_t step_off;
};
// Blocks or tiles, per subdomain: the tiles where the products they execute
// (zero columns of a slab included) are at most this multiple of the blocks'.
// A tile reads half as much X per product, a block skips more zeros: 2.2 times
// fewer products on a 2D mesh of 129^2 nodes (m = 512), 1.04 times on a 20^3
// elasticity box.  Measured, blocks / tiles at products tiles : blocks: FP64
// 0.39 / 0.89 ms at 2.25, 7.04 / 7.24 at 1.064, 8.19 / 8.22 at 1.054, 14.1 /
// 13.5 at 1.051, 13.7 / 12.5 at 1.036; mixed 0.148 / 0.301 at 2.25, 1.39 / 1.41
// at 1.143, 2.63 / 2.64 at 1.139, 1.81 / 1.76 at 1.112, 3.00 / 2.75 at 1.064,
// 3.32 / 3.05 at 1.054.  Batches of one shape each; from one batch to the next
// the two differ by a few percent at the same ratio, and next to the line the
// choice is worth no more than that.
constexpr double kSyrkTileCost = 1.053, kSyrkTileCostMixed = 1.12;
// The mixed SYRK splits 2^kSplitScale X into bf16 values: the last bit of the
// smallest FP32 number is then that of the smallest bf16 number, and no value
// of X loses bits.  X values from 2^kSplitMaxExp on, where a partial sum could
// overflow although the sum does not (2^27 rows of 2^100), and infinities, which
// do not split, take the FP32 units: the TRSM flags the tiles that hold some.
constexpr int kSplitScale = 16, kSplitMaxExp = 50 - kSplitScale;
constexpr int kStepSlabShift = 27;
constexpr int kStepRowMask = (1 << kStepSlabShift) - 1;   // rows below 2^27 (checked at plan creation)

struct BlockDev {
    int32_t row0, w, nbelow;
    int32_t pad;
    int64_t lval_off;    // diagonal block (w x w, column-major), relative to the subdomain's lval_off
    int64_t rows_off;    // relative to the subdomain's rows_off
    int64_t aoff;        // pruned rows as MFMA A tiles, relative to the subdomain's lval_off
    int64_t linv_off;    // inverse of the diagonal block as MFMA A tiles (same base)
};

// One diagonal triangle to invert: offsets into the factor values.
struct InvItem {
    int64_t diag, linv;
    int32_t w, pad;
};

}  // namespace scasm
