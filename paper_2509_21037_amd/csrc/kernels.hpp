// Kernel launchers (host side) over the device tables of a plan.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "device.hpp"

namespace scasm {

constexpr int kNumTimed = 5;   // timed kernels: TRSM, SYRK, apply, implicit apply, overlapped assembly

struct DevTables {
    const SubDev* subs = nullptr;
    const TileDev* tiles = nullptr;
    const BlockDev* blocks = nullptr;
    const int32_t* rows = nullptr;
    const VisitDev* visits = nullptr;      // blocks visited per TRSM tile (TileDev::visit_off)
    const uint64_t* fresh = nullptr;       // rows first written by an update (TileDev::fresh_off)
    const int32_t* clear = nullptr;        // rows a TRSM tile clears (TileDev::clear_off)
    const int32_t* ksteps = nullptr;       // SYRK k-steps per item (SyrkItem::step_off)
    const double* lval = nullptr;
    const float* lval32 = nullptr;
    const int32_t* piv = nullptr;
    const int32_t* pi = nullptr;
    const int8_t* sgn = nullptr;
    const SyrkItem* syrk = nullptr;
    const int32_t* tile_order = nullptr;   // TRSM workgroup -> tile index (-1 = idle)
    double* X = nullptr;
    float* X32 = nullptr;
    double* F = nullptr;
    float* F32 = nullptr;
    const SyrkItem* ftiles = nullptr;      // stored F tiles (subdomain order): symmetric apply pass 1
    const int2* frows = nullptr;           // (subdomain, 128-row block): symmetric apply pass 2
    double* part = nullptr;                // 256 partial sums per stored F tile
    int32_t* xwide = nullptr;              // mixed: per X tile and wavefront, != 0 where some value is
                                           // beyond the bf16 split (kSplitMaxExp)
    int64_t ntiles = 0;          // TRSM workgroups (length of tile_order)
    bool trsm_merge = false;     // TRSM with the merged pairs (VisitDev::flags)
    bool trsm_large = false;     // some X slab holds kTrsmSlabBytes or more
    int64_t nsyrk = 0;           // SYRK workgroups (items with sub < 0 are idle)
    int64_t nsyrk_tile = 0;      // the first nsyrk_tile of them are 128 x 128 tiles, the rest 64 x 64 blocks
    int64_t nftiles = 0;
    int64_t nfrows = 0;
};

// Assembly kernels; FP64, or mixed precision when t.X32 is set (FP64
// diagonal solves, FP32 X / updates / SYRK and FP32 F).
//   launch_trsm: TRSM workgroups over `order[0, count)` (tile indices, -1 idle)
//   launch_syrk: SYRK workgroups over `items[0, count)` (sub < 0 idle)
//   launch_assemble: all tiles, then all SYRK items, on one stream; optional
//     events ev[2k] before and ev[2k+1] after kernel k (0 = TRSM, 1 = SYRK).
hipError_t launch_trsm(const DevTables& t, const int32_t* order, int64_t count, hipStream_t stream);
// SYRK over items[0, ntile) (128 x 128 tiles) then items[ntile, ntile + nblock)
// (64 x 64 blocks).
hipError_t launch_syrk(const DevTables& t, const SyrkItem* items, int64_t ntile, int64_t nblock,
                       hipStream_t stream);
hipError_t launch_assemble(const DevTables& t, hipStream_t stream, hipEvent_t* ev);

// Inverses of `count` diagonal triangles, in place in the factor values.
hipError_t launch_invert_diag(const InvItem* items, int64_t count, double* lval, hipStream_t stream);

// FP64 factor -> FP32 copy (mixed precision).
hipError_t launch_convert_f32(const double* a, float* b, int64_t n, hipStream_t stream);

struct PcpgArgs {
    const double* G;        // concatenated m_i x k_i column-major blocks
    const int64_t* g_off;   // [nsub] offsets into G
    const int32_t* kdim;    // [nsub] kernel dimension k_i (<= 8)
    const double* GtGinv;   // [nsub][64] (G^T G)^{-1}, k_i x k_i row-major
    const double* d;        // right-hand side (dual layout)
    double* lambda;         // solution (dual layout)
    double *r, *w, *p, *q;  // workspace (dual layout)
    double* ww;             // [nsub]
    double* hist;           // [(iters + 1) * nsub] or null
    int32_t nsub;
    int32_t iters;
    int64_t dual_total;     // multipliers of all subdomains
};

struct ImplicitLevels;
// Projected CG on every subdomain, `iters` iterations: F applied explicitly
// to the assembled subdomains, and, when lvh is given, with the factor to the
// nimpl subdomains of lvh->subs (workspace xwork at xoff).
hipError_t launch_pcpg(const DevTables& t, const PcpgArgs& a, hipStream_t stream, const ImplicitLevels* lvh,
                       const int64_t* xoff, double* xwork, int32_t nimpl);

// One factor block as the implicit sweeps walk it: offsets into the factor
// values, the row array, the work vectors and rptr.
struct ImplBlock {
    int64_t linv, aoff, rows, x, rptr;
    int32_t row0, w, nbelow, pad;
};

constexpr int kImplThreads = 1024;
constexpr int kImplParts = kImplThreads / 64;
// Implicit sweeps, the levels next to the roots that hold fewer blocks than
// this run as one launch per sweep (a chain); levels of more blocks, and those
// between them and the leaves, as one launch each.  Levels of 256 / 512 / 2048
// blocks and all in chains: 16 x 20^3 elasticity 1.43 / 1.40 / 1.32 / 1.33 ms,
// 64 x 20^3 4.18 / 4.13 / 4.03 / 4.06, 512 x 12^3 heat 0.845 / 0.844 / 0.839 /
// 0.871 (0.853 with every level a launch).
constexpr int64_t kImplChainBelow = 2048;
// Subdomains of near-chain block DAGs and fewer blocks than this on average:
// one workgroup per subdomain runs both sweeps.  One workgroup / chains: 512
// heat squares of 16^2 elements (5 blocks) 71 / 95 us, 24^2 (10) 161 / 164, 28^2
// (14) 243 / 233; 64 of 24^2 71 / 84, 28^2 100 / 107, 32^2 (18) 111 / 88; one 12^3
// heat cube (46) 304 / 286, 512 of them 1000 / 895; 16 x 20^3 elasticity in
// uniform blocks (435) 10.1 / 4.9 ms.
constexpr int64_t kImplChainBlocks = 16;
// A block of a chain is split over up to kImplSplit workgroups, as many as
// fill the chip twice.  Forward, each repeats the update sums and the diagonal
// product and takes its share of the row tiles (at least one per wavefront).
// Backward, from kImplBwdSplitRows rows on, each sums a share of the rows and
// the last one to finish adds the shares and does the diagonal product.  16 x
// 20^3 elasticity with up to 8 / 4 shares 1.43 / 1.51 ms; backward from 512 /
// 1024 rows 1.43 / 1.47.
constexpr int kImplSplit = 8;
constexpr int kImplBwdSplitRows = 512;
inline int impl_split(int64_t blocks, int tiles) {
    return (int)std::max<int64_t>(1, std::min<int64_t>({kImplSplit, 512 / blocks, tiles}));
}
// ints between the counters that waiting workgroups read over and over: with
// all subdomains' counters in one cache line the sweeps took twice as long
constexpr int64_t kImplCounterStride = 64;
// looks (of about a microsecond) at a counter before a wait gives up, and the
// value that it leaves in the counter, above every count
constexpr int32_t kImplLooks = 1 << 24;
constexpr int32_t kImplGaveUp = 1 << 30;

// One workgroup of a chain of levels run in one launch: a block (or
// share g of G of its row tiles) that starts when `need` workgroups (forward)
// or blocks (backward) of its subdomain have finished before it.
struct ImplChainItem {
    ImplBlock b;
    int32_t sub, need, g, G;
};

// Level schedule of the blocked triangular solves of the implicit apply:
// blocks grouped by level (host offsets, levels run in order); per row of a
// subdomain (rptr at rptr_off[sub], CSR) the positions in the row array where
// it is a pruned row: its entries in the update buffer ubuf, which runs
// parallel to the row array.
struct ImplicitLevels {
    const ImplBlock* fw_items = nullptr;
    const ImplBlock* bw_items = nullptr;
    const int64_t* rptr_off = nullptr;
    const int32_t* rptr = nullptr;
    const int32_t* rpos = nullptr;
    double* ubuf = nullptr;
    // y = L^{-1} x of the forward sweep (n_i doubles per subdomain at the
    // xwork offsets): kept apart from x so that several workgroups of one
    // forward block step read x while one of them writes y
    double* ywork = nullptr;
    std::vector<int64_t> fw_off, bw_off;
    // the chains of levels next to the roots (forward levels fw_chain and on,
    // backward levels before bw_chain), one launch each, their workgroups in
    // level order (shares of a block next to each other); counters: a ticket
    // per sweep, the finished workgroups / blocks of every subdomain in each,
    // the finished shares of each backward item; cleared by
    // launch_implicit_init.  cpart: 64 sums for each backward item
    const ImplChainItem* fw_chain_items = nullptr;
    const ImplChainItem* bw_chain_items = nullptr;
    int32_t* counters = nullptr;
    double* cpart = nullptr;
    int64_t nfw_chain = 0, nbw_chain = 0, nsub = 0;
    size_t fw_chain = SIZE_MAX, bw_chain = 0;
    int64_t ncounters() const { return kImplCounterStride * (2 + 2 * nsub) + nbw_chain; }
    int32_t* fw_done() const { return counters + 2 * kImplCounterStride; }
    int32_t* bw_done() const { return fw_done() + nsub * kImplCounterStride; }
    // set when a wait gave up (and never cleared by the sweeps)
    int32_t* fault = nullptr;
    int32_t looks = kImplLooks;
    // true: one workgroup per subdomain runs both sweeps block by block
    bool per_subdomain = false;
    // the subdomains covered (device list; null = all, in index order)
    const int32_t* subs = nullptr;
};

// Implicit apply q = B P^T L^{-T} L^{-1} P B^T p; xwork holds n_i doubles per
// subdomain at xoff[i]; optional events ev[0] before, ev[1] after.  It is the
// three launches below in order: x = P B^T p (init), the two blocked
// triangular sweeps on x in place (they read no caller pointer, so a captured
// graph of them stays valid for any p and q), q = B P^T x (gather).
// `count` subdomains: those of `sub_list` / lv.subs, or 0 .. count - 1 when
// the list is null.
hipError_t launch_implicit_init(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff, double* xwork,
                                const double* p, int32_t count, hipStream_t stream);
hipError_t launch_implicit_sweeps(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff, double* xwork,
                                  int32_t count, hipStream_t stream);
hipError_t launch_implicit_gather(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff,
                                  const double* xwork, double* q, int32_t count, hipStream_t stream);
hipError_t launch_apply_implicit(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff, double* xwork,
                                 const double* p, double* q, int32_t count, hipStream_t stream, hipEvent_t* ev);

// q = F p for every subdomain (FP32 F when t.F32 is set, else FP64 F), two
// passes over the packed sorted F; optional events ev[0] before, ev[1] after.
hipError_t launch_apply(const DevTables& t, const double* p, double* q, hipStream_t stream, hipEvent_t* ev);

// F of subdomain `sub` (m multipliers, assembled) as a dense FP64 matrix in
// multiplier order, column-major with leading dimension ld >= m.
hipError_t launch_expand_F(const DevTables& t, int32_t sub, int32_t m, double* out, int64_t ld, hipStream_t stream);

// Allocation-free explicit apply.  Its partial sums live in a fixed device
// array of kApplyScratchTiles stored tiles (256 doubles each: 32 MiB), one per
// GPU for the life of the process.
constexpr int64_t kApplyScratchTiles = 16384;
// largest m whose nst (nst + 1) / 2 stored tiles (nst = ceil(m / 128)) fit
constexpr int32_t kApplyMaxM = 180 * kSyrkTile;
static_assert(180 * 181 / 2 <= kApplyScratchTiles && 181 * 182 / 2 > kApplyScratchTiles, "kApplyMaxM");
constexpr int kMaxDevices = 64;
// Whole subdomains whose stored tiles [t0, t1) fit the array; their row
// blocks [r0, r1) (h_frows order).
struct ApplyChunk {
    int64_t t0, t1, r0, r1;
};
// Looks up (once per device, with `device` current) the device address of
// the array; *out receives it.  Thread-safe.
hipError_t apply_scratch_init(int device, double** out);
// q = F p chunk by chunk on `stream`, partial sums in `scratch_ptr` (from
// apply_scratch_init); no allocation.
hipError_t launch_apply_chunked(const DevTables& t, const ApplyChunk* chunks, int64_t nchunks, double* scratch_ptr,
                                const double* p, double* q, hipStream_t stream);

}  // namespace scasm
