// HIP kernels for gfx950 (CDNA4, wave64): staircase TRSM and SYRK of the
// dual Schur-complement assembly (paper, Sec. 3.2 and 3.3), FP64 and mixed
// precision.  The solution-stage kernels are in apply.hip.
//
// MFMA operand layouts used throughout (v_mfma_f64_16x16x4f64):
//   A (16 x 4):  lane l holds A[l % 16][l / 16]
//   B (4 x 16):  lane l holds B[l / 16][l % 16]
//   C/D (16x16): lane l, register r holds D[4 r + l / 16][l % 16]
// so the D registers of a 16 x 16 tile are, register r, exactly the B operand
// of k-slice r of the same tile used as a right-hand side.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace scasm {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma_f64(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

typedef float v4f __attribute__((ext_vector_type(4)));

// v_mfma_f32_16x16x4f32 takes A and B in the same lane layout as the FP64
// instruction, but its accumulator is laid out differently:
//   C/D (16x16): lane l, register r holds D[4 (l / 16) + r][l % 16].
__device__ __forceinline__ v4f mfma_f32(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// Staircase TRSM, X = L^{-1} P B^T (Sec. 3.2, factor splitting with pruning).
// One workgroup = one 64-column tile of one subdomain; wavefront v owns the
// 16-column stripe v and holds the X rows of the current factor block in
// registers (FP64 accumulator layout).  The four wavefronts walk the factor
// blocks together, from the block holding the tile's first pivot (rows above
// it are zero and stay zero: forward substitution only propagates
// downwards); a stripe whose first pivot lies further down joins at its own
// first block.  Per block b:
//   1. X[b] <- L_bb^{-1} X[b], FP64 MFMA with the inverse of the diagonal
//      block (invert_diag; its lower 16 x 4 tiles, one chunk);
//   2. the pruned rows below the block, 32 at a time (64 in mixed precision):
//      X[R_b] -= L[R_b, b] X[b] (MFMA, rows gathered and scattered).
// The factor flows through the workgroup as a stream of chunks (the inverse
// of a diagonal block, up to 20 KB, or 16 KB of pruned-row tiles), one per
// step.  The loads of the next chunk are issued at the start of a step and go
// from registers to the other half of a double buffer in LDS at its end; one
// barrier per chunk, on LDS only (X columns of a stripe are private to its
// wavefront, so no barrier waits on global memory).  Rows of the next chunk of the same block are gathered before the
// current chunk's MFMAs (the chunks of one block update disjoint rows), and
// the rows of the next block before those of the last chunk where it does
// not update them (VisitDev); a wavefront reads rows it wrote itself in
// program order.
// What bounds it is the traffic and the latency of the X rows.  Traffic: a
// row is read only if the tile wrote it before (VisitDev::held and the fresh
// masks; it counts as zero until then), so X is not cleared and a first
// update only writes.  Latency: no load or store waits for another: global
// memory operations complete in issue order, and the wait for one of them can
// leave younger ones in flight only where the compiler knows how many there
// are.  Rows that are not there (past a row list, off the paths, not written
// yet) are therefore out-of-range offsets of a buffer resource (read as zero,
// not written) instead of branches, a load is waited for in the code path
// that issued it, and no register holding a load in flight is copied (the
// last chunk of a block, which loads the next block's rows, is a step of its
// own).  Before (branches, a cleared X, and a two-chunk prefetch whose
// register rotation waited for every operation in flight at each step) / now:
// 16 x 20^3 elasticity 23.3 / 18.4 ms FP64, 17.1 / 9.6 ms mixed; 64 uneven
// elasticity boxes 4.61 / 3.36 ms; 512 x 12^3 heat 3.33 / 2.64 and 2.94 / 1.57
// ms; 128 2D triangle meshes of 129^2 nodes 1.11 / 0.86 ms (3 workgroups per
// CU without merged pairs; 0.93 with 2).
// Mixed precision: the same with FP32 X and FP32 A tiles / MFMA for step 2;
// step 1 stays FP64 (the block rows are widened, solved, rounded back).  The
// FP32 A tiles are read with their rows permuted (4a + b -> 4b + a), which
// gives the FP32 accumulator the row layout of the FP64 one.
// Merged pairs: two consecutive blocks b, b + 1 that a tile visits one after
// the other and whose rows below nest, R_b = rows(b + 1) followed by R_{b+1}
// (planner's merge_pairs: two panels of one supernode, or a child
// block with its parent's structure).  Block b then
// updates only the rows of b + 1, which stay in registers for the solve of
// b + 1; its solved rows -X[b] wait in LDS (one 64 x
// 16 slot per wavefront); block b + 1 updates R_{b+1} once with both:
// X[R] -= L[R, b] X[b] + L[R, b + 1] X[b + 1], two chunk steps per row group
// (the A tiles of b, then those of b + 1), one gather and one scatter.  The
// sums run in the same order as two separate updates (a read-modify-write in
// the X precision is exact), so X and F are bit for bit the same; the rows
// below are read and written once instead of twice.
// ---------------------------------------------------------------------------
// a chunk: the 40 lower tiles of a 64 x 64 diagonal inverse (20 KB), or 16 KB
// of pruned-row tiles
constexpr int kChunkBytes = 40 * 64 * 8;
constexpr int kRowsBytes = 64 * 4;               // row indices carried by a chunk (up to 64)
constexpr int kIdxBytes = kRowsBytes + 16;       // ... and the mask of those never written before
constexpr int kBufBytes = kChunkBytes + kIdxBytes;
constexpr int kTrsmSmem = 2 * kBufBytes;

// Barrier that waits for this wavefront's LDS traffic only: global loads in
// flight (prefetches, gathers) stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_at4 __attribute__((aligned(4)));     // in memory, on any 4-byte boundary

// Raw buffer resource over `bytes` bytes at p (wave-uniform): loads past them
// return zero, stores past them are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}

// Access to the rows of one X slab by element offset.  LARGE = false: 32-bit
// byte offsets of a buffer resource, kNone an offset past any slab.  LARGE =
// true (slabs of kTrsmSlabBytes and more, which those offsets cannot span):
// 64-bit element indices and plain accesses under a branch.
template <class TX, bool LARGE>
struct SlabRows {
    using Off = decltype(slab_offset<TX, LARGE>(0, 0));
    static constexpr Off kNone = LARGE ? -1 : -16;
    TX* p;
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ SlabRows(TX* x, int64_t elems)
        : p(x), r(buffer_of(x, LARGE ? 0u : (uint32_t)(elems * (int64_t)sizeof(TX)))) {}
    __device__ __forceinline__ static Off at(int row, int col) { return slab_offset<TX, LARGE>(row, col); }
    // or-ed to an offset: kNone where c holds
    __device__ __forceinline__ static Off none_if(bool c) { return c ? kNone : 0; }
    __device__ __forceinline__ TX load(Off off) const {
        if constexpr (LARGE) return off >= 0 ? p[off] : TX(0);
        else if constexpr (sizeof(TX) == 8) return __builtin_bit_cast(TX, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
        else return __builtin_bit_cast(TX, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    }
    __device__ __forceinline__ void store(Off off, TX v) const {
        if constexpr (LARGE) {
            if (off >= 0) p[off] = v;
        } else if constexpr (sizeof(TX) == 8) {
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), r, off, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 0);
        }
    }
};

// LDS slot of the first block's solved rows: 16 values per lane and wavefront.
template <class TX>
constexpr int kSlotBytes = 4 * 16 * 64 * (int)sizeof(TX);

// acc[u] += A row tile u x B over nks k-slices (up to 16), NT row tiles of a
// chunk at sA (this lane's values); B(t, s) = k-slice 4 t + s, zero past nks
// (the A values met there are those of the next row tile or the zeros a chunk
// ends in).  Four slices of every row tile are read ahead of the four in use.
template <bool MIXED, int NT, class TX, class VX, class FB>
__device__ __forceinline__ void mma_group(const TX* __restrict__ sA, int nks, const FB& B, VX* acc) {
    TX a[2][NT][4];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int s = 0; s < 4; ++s) a[0][u][s] = sA[(u * nks + s) * 64];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (4 * t >= nks) break;
        TX b[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) b[s] = B(t, s);
        if (t < 3) {
#pragma unroll
            for (int u = 0; u < NT; ++u)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    a[(t + 1) & 1][u][s] = sA[(u * nks + 4 * (t + 1) + s) * 64];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                if constexpr (MIXED) acc[u] = mfma_f32(a[t & 1][u][s], b[s], acc[u]);
                else acc[u] = mfma_f64(a[t & 1][u][s], b[s], acc[u]);
            }
    }
}

// The chunk stream of one tile: chunk c of visit record p.  c = 0 is the
// inverse of the diagonal block (its lower tiles), the rest groups of PT
// pruned row tiles; the second block of a pair alternates the first block's A
// tiles of a row group with its own.  The diagonal chunk carries the row
// indices (and the mask of those never written before) of the first row
// group, the (second) chunk of row group q those of group q + 1: they are
// gathered while the chunk is in use.
template <class TX, bool MERGE>
struct ChunkStream {
    static constexpr int PT = kPruneTiles<TX>;
    const VisitDev* __restrict__ V;
    const double* __restrict__ L;
    const TX* __restrict__ LA;
    const int32_t* __restrict__ R;
    const uint64_t* __restrict__ FR;
    int nv;
    int pk = 0, pc = 0;
    VisitDev p;
    __device__ __forceinline__ ChunkStream(const VisitDev* v, int n, const double* l, const TX* la, const int32_t* r,
                                           const uint64_t* fr)
        : V(v), L(l), LA(la), R(r), FR(fr), nv(n), p(v[0]) {}
    // the next chunk: `bytes` bytes at src (none past the end), its row
    // indices at ip and their mask at fp (valid addresses in any case)
    __device__ __forceinline__ void next(const char*& src, uint32_t& bytes, const int32_t*& ip, const uint64_t*& fp) {
        src = reinterpret_cast<const char*>(L);
        ip = R;
        fp = FR;
        bytes = 0;
        if (pk >= nv) return;
        const int prole = MERGE ? p.flags & 3 : 0;
        const int nks = (p.w + 3) >> 2;
        const int nrt = (p.urows + 15) >> 4;
        const int np = (nrt + PT - 1) / PT;
        if (pc == 0) {
            const int nrt_d = (p.w + 15) >> 4;
            src = reinterpret_cast<const char*>(L + p.linv_off);
            bytes = (2 * (nrt_d - 1) * nrt_d + nks) * 64 * 8;
            ip = R + p.rows_off;
            fp = FR + p.fresh;
        } else {
            const int q = prole == 2 ? (pc - 1) >> 1 : pc - 1;
            const int nt = min(PT, nrt - PT * q);
            const bool first = prole == 2 && ((pc - 1) & 1) == 0;
            const int ks = first ? p.pair_nks : nks;
            src = reinterpret_cast<const char*>(LA + (first ? p.pair_aoff : p.aoff) + (int64_t)PT * q * ks * 64);
            bytes = nt * ks * 64 * (int)sizeof(TX);
            ip = R + p.rows_off + 16 * PT * min(q + 1, np - 1);
            fp = FR + p.fresh + min(q + 1, np - 1);
        }
        if (++pc > (prole == 2 ? 2 * np : np)) {
            ++pk;
            pc = 0;
            if (pk < nv) p = V[pk];
        }
    }
};

// Launches of at most kLoaderMaxTiles tiles, one workgroup per CU: a fifth
// wavefront streams the chunks into LDS, two of them in flight in registers of
// its own, so that a step no longer lasts as long as a chunk takes to arrive.
// Larger launches hide that behind the other workgroups of the CU, and the
// fifth wavefront would cost one of them (registers).  Without / with, FP64:
// one 16 x 16 heat square (1 tile) 30.6 / 26.7 us, one 12^3 heat cube (14) 154
// / 122, 16 of them (224) 159 / 127, 32 triangle meshes of 129^2 nodes (256)
// 309 / 247; beyond, 8 uneven elasticity boxes (288) 1020 / 1031.
constexpr int64_t kLoaderMaxTiles = 256;

template <class TX, bool MERGE>
__device__ __forceinline__ void trsm_load_wave(ChunkStream<TX, MERGE> stream, int nchunk, char* __restrict__ smem) {
    constexpr int kPieces = kChunkBytes / 1024;
    const int lane = threadIdx.x & 63;
    struct Set {
        v4u c[kPieces], ci;
    };
    auto load = [&](Set& x) __attribute__((always_inline)) {
        const char* src;
        const int32_t* ip;
        const uint64_t* fp;
        uint32_t bytes;
        stream.next(src, bytes, ip, fp);
        const __amdgpu_buffer_rsrc_t rc = buffer_of(src, bytes);
#pragma unroll
        for (int e = 0; e < kPieces; ++e) x.c[e] = __builtin_amdgcn_raw_buffer_load_b128(rc, lane * 16, e * 1024, 0);
        x.ci = *reinterpret_cast<const v4u_at4*>(lane < kRowsBytes / 16 ? reinterpret_cast<const char*>(ip) + 16 * lane
                                                                    : reinterpret_cast<const char*>(fp));
    };
    auto put = [&](const Set& x, int buf) __attribute__((always_inline)) {
        char* dst = smem + buf * kBufBytes + lane * 16;
#pragma unroll
        for (int e = 0; e < kPieces; ++e) *reinterpret_cast<v4u*>(dst + e * 1024) = x.c[e];
        if (lane <= kRowsBytes / 16) *reinterpret_cast<v4u*>(dst + kChunkBytes) = x.ci;
    };
    Set s0, s1;
    load(s0);
    load(s1);
    put(s0, 0);
    load(s0);
    lds_barrier();
    int s = 0;
    for (; s + 1 < nchunk; s += 2) {
        put(s1, 1);
        load(s1);
        lds_barrier();
        put(s0, 0);
        load(s0);
        lds_barrier();
    }
    if (s < nchunk) {
        put(s1, 1);
        lds_barrier();
    }
}

template <bool MIXED, bool MERGE, bool LARGE, bool LOADER>
__device__ __forceinline__ void trsm_tile(
    const SubDev* __restrict__ subs, const TileDev* __restrict__ tiles, const int32_t* __restrict__ rows,
    const VisitDev* __restrict__ visits, const uint64_t* __restrict__ fresh, const int32_t* __restrict__ clear,
    const double* __restrict__ lval,
    const float* __restrict__ lval32, const int32_t* __restrict__ piv, const int8_t* __restrict__ sgn,
    typename std::conditional<MIXED, float, double>::type* __restrict__ X, int32_t* __restrict__ xwide, int ti,
    char* __restrict__ smem)
{
    using TX = typename std::conditional<MIXED, float, double>::type;
    using VX = typename std::conditional<MIXED, v4f, v4d>::type;
    using Rows = SlabRows<TX, LARGE>;
    constexpr int PT = kPruneTiles<TX>;          // pruned row tiles per chunk
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;
    const int j = lane & 15;
    const int la = MIXED ? 4 * (j & 3) + (j >> 2) + 16 * g : lane;   // A tile position this lane reads
    const TileDev T = tiles[ti];
    const SubDev S = subs[T.sub];
    const int kstart = T.kstart;
    TX* __restrict__ Xs = X + T.x_off;
    const Rows xr_(Xs, (int64_t)(S.n - kstart) * kTile);
    const int col = wv * kStripe + j;
    const int64_t cbase = S.col_off + (int64_t)T.tile * kTile;
    const int32_t* __restrict__ R = rows + S.rows_off;
    const double* __restrict__ L = lval + S.lval_off;
    const TX* __restrict__ LA;
    if constexpr (MIXED) LA = lval32 + S.lval_off;
    else LA = lval + S.lval_off;
    // the blocks this tile visits, increasing: those holding rows on the
    // elimination-tree paths of its pivots (all other rows of X are zero)
    const int nv = T.nvisit;
    const VisitDev* __restrict__ V = visits + T.visit_off;
    const uint64_t* __restrict__ FR = fresh + T.fresh_off;
    if constexpr (LOADER)
        if (wv == 4) {
            if (nv > 0) trsm_load_wave<TX, MERGE>(ChunkStream<TX, MERGE>(V, nv, L, LA, R, FR), T.nchunk, smem);
            return;
        }

    // right-hand side P B^T: sign at the pivot row, zero elsewhere.  Only the
    // pivot rows are set in memory, and the rows off the paths that the SYRK
    // reads (in its 16-row steps with a row on them) cleared: every other row
    // counts as zero until the sweep first writes it
    const int32_t* __restrict__ CL = clear + T.clear_off;
    for (int i = g; i < T.nclear; i += 4) Xs[(int64_t)(CL[i] - kstart) * kTile + col] = TX(0);
    __threadfence_block();
    if (g == 0 && col < T.ncols) Xs[(int64_t)(piv[cbase + col] - kstart) * kTile + col] = (TX)sgn[cbase + col];
    if (nv <= 0) return;
    __threadfence_block();

    TX* __restrict__ slot = reinterpret_cast<TX*>(smem + kTrsmSmem) + wv * 16 * 64 + lane;

    ChunkStream<TX, MERGE> stream(V, nv, L, LA, R, FR);
    v4u c0, c1, c2, c3, c4, ci;                  // the chunk after the one in LDS
    auto load_chunk = [&]() {
        const char* src;
        const int32_t* ip;
        const uint64_t* fp;
        uint32_t bytes;
        stream.next(src, bytes, ip, fp);
        const __amdgpu_buffer_rsrc_t rc = buffer_of(src, bytes);
        const int e = threadIdx.x * 16;
        c0 = __builtin_amdgcn_raw_buffer_load_b128(rc, e, 0, 0);
        c1 = __builtin_amdgcn_raw_buffer_load_b128(rc, e, 4096, 0);
        c2 = __builtin_amdgcn_raw_buffer_load_b128(rc, e, 8192, 0);
        c3 = __builtin_amdgcn_raw_buffer_load_b128(rc, e, 12288, 0);
        c4 = __builtin_amdgcn_raw_buffer_load_b128(rc, e, 16384, 0);
        ci = *reinterpret_cast<const v4u_at4*>(lane < kRowsBytes / 16 ? reinterpret_cast<const char*>(ip) + 16 * lane
                                                                   : reinterpret_cast<const char*>(fp));
    };
    auto put_chunk = [&](char* dst) {
        const int e = threadIdx.x * 16;
        *reinterpret_cast<v4u*>(dst + e) = c0;
        *reinterpret_cast<v4u*>(dst + e + 4096) = c1;
        *reinterpret_cast<v4u*>(dst + e + 8192) = c2;
        *reinterpret_cast<v4u*>(dst + e + 12288) = c3;
        *reinterpret_cast<v4u*>(dst + e + 16384) = c4;
        if (threadIdx.x <= kRowsBytes / 16) *reinterpret_cast<v4u*>(dst + kChunkBytes + e) = ci;
    };
    int buf = 0;
    auto step_begin = [&]() {
        if constexpr (!LOADER) load_chunk();
    };
    auto step_end = [&]() {
        if constexpr (!LOADER) put_chunk(smem + (buf ^ 1) * kBufBytes);
        lds_barrier();
        buf ^= 1;
    };
    if constexpr (!LOADER) {
        load_chunk();
        put_chunk(smem);
    }
    lds_barrier();

    TX xin[4][4];                                // X rows of the next block, accumulator layout
    auto load_block = [&](const VisitDev& v, uint64_t held, bool act) {
        const uint64_t onl = act ? held >> g : 0;
        const auto b0 = Rows::at(v.row0 + g - kstart, col);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                xin[t][r] = xr_.load(((onl >> (16 * t + 4 * r)) & 1) ? b0 + Rows::at(16 * t + 4 * r, 0) : Rows::kNone);
    };

    bool wide = false;                           // some value is beyond the bf16 split (mixed)
    VisitDev v = V[0];
    load_block(v, v.held, (v.flags >> (kVisitActShift + wv)) & 1);
    int pair_nks = 0;
    for (int k = 0; k < nv; ++k) {
        const VisitDev nx = V[min(k + 1, nv - 1)];
        const uint64_t nx_held = k + 1 < nv ? nx.held : 0;
        const bool nx_act = (nx.flags >> (kVisitActShift + wv)) & 1;
        const bool act = (v.flags >> (kVisitActShift + wv)) & 1;
        const int role = MERGE ? v.flags & 3 : 0;
        const bool early = (v.flags & kVisitNextEarly) != 0;
        const int urows = v.urows;
        const int nks = (v.w + 3) >> 2;
        const int nrt_d = (v.w + 15) >> 4;
        const int nrt = (urows + 15) >> 4;
        const int np = (nrt + PT - 1) / PT;
        // the first block of a pair hands the next block's rows on in
        // registers: they are read for the stripes active there
        const bool gact = role == 1 ? nx_act : act;

        VX accn[PT];                             // rows of the next pruned chunk
        typename Rows::Off offn[PT][4];                         // where they are written
        auto gather = [&](int q) {               // row indices and mask from the chunk in LDS
            const int32_t* __restrict__ sidx = reinterpret_cast<const int32_t*>(smem + buf * kBufBytes + kChunkBytes);
            const int left = urows - 16 * PT * q;
            // rows never written before are zero: not read
            uint64_t fr = *reinterpret_cast<const uint64_t*>(sidx + kRowsBytes / 4) >> g;
            typename Rows::Off offl[PT][4];
#pragma unroll
            for (int u = 0; u < PT; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) offn[u][r] = Rows::at(sidx[16 * u + 4 * r + g] - kstart, col);
            if (left < 16 * PT) {
#pragma unroll
                for (int u = 0; u < PT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) offn[u][r] |= Rows::none_if(16 * u + 4 * r + g >= left);
            }
            if (!gact) fr = ~0ull;
#pragma unroll
            for (int u = 0; u < PT; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) offl[u][r] = offn[u][r] | Rows::none_if((fr >> (16 * u + 4 * r)) & 1);
            if (!act) {                          // a stripe not started writes its zeros once
                fr = *reinterpret_cast<const uint64_t*>(sidx + kRowsBytes / 4) >> g;
#pragma unroll
                for (int u = 0; u < PT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) offn[u][r] |= Rows::none_if(!((fr >> (16 * u + 4 * r)) & 1));
            }
#pragma unroll
            for (int u = 0; u < PT; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) accn[u][r] = xr_.load(offl[u][r]);
        };

        // ---- 1. X[b] <- L_bb^{-1} X[b]
        TX xb[4][4];                             // -X[b]: B operands of step 2
        step_begin();
        if (np > 0) gather(0);
        __builtin_amdgcn_sched_barrier(0);
        {
            v4d xr[4], tmp[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) xr[t][r] = (double)xin[t][r];
            // lower tiles only: row tile u needs k-slices of row tiles t <= u
            const double* __restrict__ sA = reinterpret_cast<const double*>(smem + buf * kBufBytes) + lane;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                tmp[u] = v4d{0.0, 0.0, 0.0, 0.0};
                if (u < nrt_d) {
#pragma unroll
                    for (int t = 0; t <= u; ++t)
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            tmp[u] = mfma_f64(sA[(2 * u * (u + 1) + 4 * t + s) * 64], xr[t][s], tmp[u]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            const uint64_t onl = (act ? v.on : v.on & ~v.held) >> g;
            const auto b0 = Rows::at(v.row0 + g - kstart, col);
            float most = 0.f;                    // largest |x|
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const TX x = (TX)tmp[t][r];
                    xr_.store(((onl >> (16 * t + 4 * r)) & 1) ? b0 + Rows::at(16 * t + 4 * r, 0) : Rows::kNone, x);
                    xb[t][r] = -x;
                    if constexpr (MIXED) most = fmaxf(most, fabsf(x));
                }
            if constexpr (MIXED) wide |= __builtin_amdgcn_ballot_w64(most >= (float)(1ull << kSplitMaxExp)) != 0;
        }
        // the first block of a pair keeps its solved rows for the second
        // (zero for a wavefront that starts at the second)
        if (role == 1) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) slot[(4 * t + r) * 64] = xb[t][r];
        }
        step_end();

        // ---- 2. X[R_b] -= L[R_b, b] X[b], pruned row tiles PT q .. PT q + PT - 1
        VX acc[PT];
        auto own = [&](int t, int s) { return xb[t][s]; };
        auto kept = [&](int t, int s) { return slot[(4 * t + s) * 64]; };
        auto update = [&](int nk, const auto& B, int nt) {
            const TX* __restrict__ sA = reinterpret_cast<const TX*>(smem + buf * kBufBytes) + la;
            if (!act && role != 2) return;
            if (nt > PT / 2) mma_group<MIXED, PT>(sA, nk, B, acc);
            else mma_group<MIXED, PT / 2>(sA, nk, B, acc);
        };
        if (MERGE && role == 1) {
            // the rows of the next block: kept in registers, zero off the paths
            const uint64_t onl = nx.on >> g;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) xin[t][r] = TX(0);
#pragma unroll
            for (int q = 0; q < 4 / PT; ++q)
                if (q < np) {
                    step_begin();
#pragma unroll
                    for (int u = 0; u < PT; ++u) acc[u] = accn[u];
                    if (q + 1 < np) gather(q + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    update(nks, own, min(PT, nrt - PT * q));
#pragma unroll
                    for (int u = 0; u < PT; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            xin[PT * q + u][r] = ((onl >> (16 * (PT * q + u) + 4 * r)) & 1) ? acc[u][r] : TX(0);
                    step_end();
                }
            pair_nks = nks;
        } else if (np > 0) {
            typename Rows::Off off[PT][4];
            auto take_rows = [&]() {
#pragma unroll
                for (int u = 0; u < PT; ++u) {
                    acc[u] = accn[u];
#pragma unroll
                    for (int r = 0; r < 4; ++r) off[u][r] = offn[u][r];
                }
            };
            auto scatter = [&]() {
#pragma unroll
                for (int u = 0; u < PT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) xr_.store(off[u][r], acc[u][r]);
            };
            // the last chunk: the rows of the next block are loaded with it,
            // before its products unless it updates them
            auto last = [&]() {
                if (early) {
                    load_block(nx, nx_held, nx_act);
                    __builtin_amdgcn_sched_barrier(0);
                    update(nks, own, nrt - PT * (np - 1));
                    scatter();
                } else {
                    __builtin_amdgcn_sched_barrier(0);
                    update(nks, own, nrt - PT * (np - 1));
                    scatter();
                    load_block(nx, nx_held, nx_act);
                }
                step_end();
            };
            if (MERGE && role == 2) {
                for (int q = 0; q + 1 < np; ++q) {
                    step_begin();
                    take_rows();
                    __builtin_amdgcn_sched_barrier(0);
                    update(pair_nks, kept, PT);
                    step_end();
                    step_begin();
                    gather(q + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    update(nks, own, PT);
                    scatter();
                    step_end();
                }
                step_begin();
                take_rows();
                __builtin_amdgcn_sched_barrier(0);
                update(pair_nks, kept, nrt - PT * (np - 1));
                step_end();
                step_begin();
                last();
            } else {
                for (int q = 0; q + 1 < np; ++q) {
                    step_begin();
                    take_rows();
                    gather(q + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    update(nks, own, PT);
                    scatter();
                    step_end();
                }
                step_begin();
                take_rows();
                last();
            }
        } else {
            load_block(nx, nx_held, nx_act);
        }
        v = nx;
    }
    if constexpr (MIXED)
        if (lane == 0) xwide[4 * (int64_t)ti + wv] = wide;
}

// MERGE: with the merged pairs (the visits' roles); without, every visit is
// alone and the merged code paths compile away.  LARGE: some X slab holds
// kTrsmSlabBytes or more.  LOADER: a fifth wavefront streams the chunks
// (launches of at most kLoaderMaxTiles tiles).
template <bool MERGE, bool LARGE, bool LOADER>
__global__ __launch_bounds__(LOADER ? 320 : 256, LOADER ? 1 : MERGE || LARGE ? 2 : 3) void trsm_stair_f64(
    const SubDev* __restrict__ subs, const TileDev* __restrict__ tiles, const int32_t* __restrict__ rows,
    const VisitDev* __restrict__ visits, const uint64_t* __restrict__ fresh, const int32_t* __restrict__ clear,
    const double* __restrict__ lval,
    const int32_t* __restrict__ piv, const int8_t* __restrict__ sgn, const int32_t* __restrict__ order, double* __restrict__ X)
{
    __shared__ __align__(16) char smem[kTrsmSmem + (MERGE ? kSlotBytes<double> : 0)];
    const int ti = order[blockIdx.x];
    if (ti < 0) return;
    trsm_tile<false, MERGE, LARGE, LOADER>(subs, tiles, rows, visits, fresh, clear, lval, nullptr, piv, sgn, X, nullptr, ti, smem);
}

template <bool MERGE, bool LARGE, bool LOADER>
__global__ __launch_bounds__(LOADER ? 320 : 256, LOADER ? 1 : MERGE || LARGE ? 2 : 3) void trsm_stair_mixed(
    const SubDev* __restrict__ subs, const TileDev* __restrict__ tiles, const int32_t* __restrict__ rows,
    const VisitDev* __restrict__ visits, const uint64_t* __restrict__ fresh, const int32_t* __restrict__ clear,
    const double* __restrict__ lval,
    const float* __restrict__ lval32, const int32_t* __restrict__ piv, const int8_t* __restrict__ sgn,
    const int32_t* __restrict__ order, float* __restrict__ X, int32_t* __restrict__ xwide)
{
    __shared__ __align__(16) char smem[kTrsmSmem + (MERGE ? kSlotBytes<float> : 0)];
    const int ti = order[blockIdx.x];
    if (ti < 0) return;
    trsm_tile<true, MERGE, LARGE, LOADER>(subs, tiles, rows, visits, fresh, clear, lval, lval32, piv, sgn, X, xwide, ti, smem);
}

// ---------------------------------------------------------------------------
// Staircase SYRK, F = X^T X (Sec. 3.3, output splitting): one workgroup per
// 64 x 64 block (EDGE = 64; I >= J, in units of 64-column X tiles) or 128 x
// 128 tile (EDGE = 128; units of kSyrkTile) of the lower triangle of the
// column-sorted F, wavefront (wi, wj) its (EDGE / 2)^2 quadrant (2 x 2 or 4 x
// 4 MFMA tiles).  The k-range is the item's list of 16-row steps: those where
// both sides hold rows on the elimination-tree paths of their pivots (every
// other step adds zero products; the staircase bound, rows below the first
// pivot of tile I, is the outer limit of that set).  A tile's step entry
// marks which of its four 64-column slabs hold such rows (bits at
// kStepSlabShift); the others read as zero, as do rows above the first pivot
// of a slab.  Items with an empty list are structurally zero and are not
// launched: the plan clears F once when it is created.  The blocks execute
// fewer steps, the tiles read half as much of X per product; both sum in the
// same order, so F is the same bit for bit.  F stays in the sorted column
// order (the permutation back to the multiplier order is applied to the
// vectors of the apply and by sc_get_F), stored as the lower triangle of 128 x
// 128 tiles, tile (I, J) at I(I+1)/2 + J, each row-major, diagonal tiles
// whole: block (2T+1, 2T) also writes its transpose, the upper quadrant of
// diagonal tile T.  Columns past m are never written and stay zero.
// Bound by the FP64 matrix units.  X rows go through double-buffered LDS, 16
// per step; the loads of two further steps are in flight in two register sets
// (the loop takes two steps, so that no load in flight is copied), through
// buffer resources whose range ends at the rows that exist (no branches), and
// a step's rows are written to LDS before the last quarter of its products.
// Before (one step in flight, loads under branches, step entries loaded when
// used) / now: 16 x 20^3 elasticity 29.9 / 27.2 ms, 64 uneven elasticity boxes
// 4.32 / 3.87, 512 x 12^3 heat 2.26 / 1.99, 32 tetrahedral meshes of 21^3
// nodes 2.16 / 1.84 ms; with one step in flight 27.6, 3.97, 2.10 and 1.94.
// ---------------------------------------------------------------------------
constexpr int kSyrkKC = 16;                  // X rows per step

template <int EDGE, bool QUARTER = false>
__global__ __launch_bounds__(256, EDGE == 128 ? 2 : 4) void syrk_f64(
    const SubDev* __restrict__ subs, const TileDev* __restrict__ tiles,
    const SyrkItem* __restrict__ items, const int32_t* __restrict__ ksteps, const double* __restrict__ X,
    double* __restrict__ F)
{
    constexpr int NS = EDGE / 64;                // 64-column slabs per side
    constexpr int kSide = QUARTER ? EDGE / 2 : EDGE;      // of the part this workgroup computes
    constexpr int MT = kSide / 32;               // 16-column MFMA tiles per side of a wavefront's quadrant
    constexpr int kLd = EDGE + 4;                // LDS row stride (elements)
    __shared__ __align__(16) double lds[2][2][kSyrkKC * kLd];    // [buffer][side]
    const int nitem = QUARTER ? gridDim.x / 4 : gridDim.x;
    const SyrkItem it = items[blockIdx.x % nitem];
    if (it.sub < 0) return;
    const int part = blockIdx.x / nitem;         // QUARTER: row half 2 x, column half x & 1
    const SubDev S = subs[it.sub];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;
    const int j = lane & 15;
    const int n = S.n;
    const bool diag = it.I == it.J;              // one side: J reads I's rows
    // this wavefront's slab of each side it loads (EDGE = 64: wavefronts 0-1
    // load side I, 2-3 side J) and the half of the 16 rows; a lane loads two
    // columns of every second row
    const int half = EDGE == 128 ? wv >> 1 : wv & 1;
    const double* xs[NS];
    int ks[NS], bit[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int side = EDGE == 128 ? q : wv >> 1;
        const int t64 = (side ? it.J : it.I) * NS + (EDGE == 128 ? wv & 1 : 0);
        const bool have = t64 < S.ntiles && !(side && diag);
        const TileDev& T = tiles[S.tile_off + (have ? t64 : 0)];
        xs[q] = X + T.x_off;
        ks[q] = have ? T.kstart : INT_MAX;
        bit[q] = EDGE == 128 ? 2 * side + (wv & 1) : 0;
    }
    const int32_t* __restrict__ KS = ksteps + it.step_off;
    const int nsteps = it.nsteps;
    const int lrow = 8 * half + (lane >> 5), lcol = 2 * (lane & 31);

    // rows lrow + 2 e of a step (zeros for a step past the last)
    auto load_step = [&](v4u (&v)[NS][4], int ent, bool have) __attribute__((always_inline)) {
        const int kb = EDGE == 128 ? ent & kStepRowMask : ent;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            // rows [r0, kb + 16) of the slab, fewer at its ends, none where
            // the step entry says so (they may never have been written): the
            // others read as zero
            const int r0 = max(kb, ks[q]);
            const bool on = EDGE == 64 || ((ent >> (kStepSlabShift + bit[q])) & 1);
            const int rows = on && have ? min(kb + kSyrkKC, n) - r0 : 0;
            const __amdgpu_buffer_rsrc_t r =
                buffer_of(xs[q] + (int64_t)(rows > 0 ? r0 - ks[q] : 0) * kTile, rows > 0 ? rows * kTile * 8 : 0);
            const int skip = rows > 0 ? r0 - kb : 0;       // rows of the step above the slab
            int o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = ((lrow + 2 * e) * kTile + lcol) * 8;
            if (skip > 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    o[e] = lrow + 2 * e >= skip ? o[e] - skip * (kTile * 8) : SlabRows<double, false>::kNone;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[q][e] = __builtin_amdgcn_raw_buffer_load_b128(r, o[e], 0, 0);
        }
    };
    auto store_step = [&](const v4u (&v)[NS][4], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int side = EDGE == 128 ? q : wv >> 1;
            if (side && diag) continue;
            double* d = &lds[buf][side][lrow * kLd + (EDGE == 128 ? 64 * (wv & 1) : 0) + lcol];
#pragma unroll
            for (int e = 0; e < 4; ++e) *reinterpret_cast<v4u*>(d + 2 * e * kLd) = v[q][e];
        }
    };

    const int wi = (part >> 1) * kSide + (wv >> 1) * (kSide / 2), wj = (part & 1) * kSide + (wv & 1) * (kSide / 2);
    v4d acc[MT][MT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
    auto entry = [&](int st) { return KS[min(st, nsteps - 1)]; };
    // step st from LDS buffer `buf`; v: the rows of step st + 1, then st + 3
    auto step = [&](v4u (&v)[NS][4], int st, int buf) __attribute__((always_inline)) {
        const int ent = entry(st + 3);
        const double* pa = &lds[buf][0][g * kLd + wi + j];
        const double* pb = &lds[buf][diag ? 0 : 1][g * kLd + wj + j];
#pragma unroll
        for (int s = 0; s < kSyrkKC / 4; ++s) {
            double a[MT], b[MT];
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                a[t] = pa[4 * s * kLd + 16 * t];
                b[t] = pb[4 * s * kLd + 16 * t];
            }
            // the next step goes to LDS before the last products, so that
            // those cover the write
            if (s == kSyrkKC / 4 - 1) {
                __builtin_amdgcn_sched_barrier(0);
                store_step(v, buf ^ 1);
                load_step(v, ent, st + 3 < nsteps);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int ta = 0; ta < MT; ++ta)
#pragma unroll
                for (int tb = 0; tb < MT; ++tb) acc[ta][tb] = mfma_f64(a[ta], b[tb], acc[ta][tb]);
        }
        lds_barrier();
    };
    v4u v0[NS][4], v1[NS][4];                    // two steps in flight
    load_step(v0, entry(0), nsteps > 0);
    load_step(v1, entry(1), nsteps > 1);
    store_step(v0, 0);
    load_step(v0, entry(2), nsteps > 2);
    lds_barrier();
    int st = 0;
    for (; st + 1 < nsteps; st += 2) {
        step(v1, st, 0);
        step(v0, st + 1, 1);
    }
    if (st < nsteps) step(v1, st, 0);
    const int I2 = EDGE == 128 ? it.I : it.I >> 1, J2 = EDGE == 128 ? it.J : it.J >> 1;
    double* __restrict__ Ft = F + S.F_off + (int64_t)(I2 * (I2 + 1) / 2 + J2) * kFTileElems;
    const int r0 = (EDGE == 128 ? 0 : 64 * (it.I & 1)) + wi;
    const int c0 = (EDGE == 128 ? 0 : 64 * (it.J & 1)) + wj;
    const bool mirror = EDGE == 64 && I2 == J2 && !diag;
#pragma unroll
    for (int ta = 0; ta < MT; ++ta)
#pragma unroll
        for (int tb = 0; tb < MT; ++tb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = r0 + 16 * ta + 4 * r + g;
                const int col = c0 + 16 * tb + j;
                Ft[row * kSyrkTile + col] = acc[ta][tb][r];
                if (mirror) Ft[col * kSyrkTile + row] = acc[ta][tb][r];
            }
}

// ---------------------------------------------------------------------------
// Mixed precision (FP64 diagonal solves; FP32 X and off-diagonal updates with
// FP32 MFMA; SYRK with FP32 products formed from bf16 ones, FP32 sums).
// ---------------------------------------------------------------------------

// FP64 factor values -> FP32 copy (round to nearest even).
__global__ __launch_bounds__(256) void convert_f64_f32(const double* __restrict__ a, float* __restrict__ b,
                                                       int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) b[i] = (float)a[i];
}
// ---------------------------------------------------------------------------
// SYRK of the FP32 X, F stored FP32: as the FP64 kernels above over 64 x 64
// blocks (EDGE = 64) or 128 x 128 tiles (EDGE = 128) of F, on the bf16 matrix
// units.  An FP32 value is exactly the sum of three bf16 values (24 = 3 x 8
// significant bits, each the rounded remainder of the last), so x y is a sum
// of nine exact bf16 products; all but the last, at most 2^-34 of x y, are
// formed.  (The two before it, a middle value times a last one, are at most
// 2^-25 each, together a whole FP32 rounding: without them an entry that is
// one product was off by up to 0.95 ulp, now by 0.51, an FP32 product by 0.5;
// sums of many terms do not show it.)  Sums stay FP32:
// v_mfma_f32_32x32x16_bf16 adds the products of a whole 16-row step at once,
// where the FP32 instruction takes four of its rows, and the seven smaller
// products have their own accumulator, so that the main one is rounded once a
// step.  The bf16 units do 16 times the FP32 rate: eight products take half
// the time.  Mixed F against the FP64 F, FP32 units before / now (relative
// Frobenius; largest element error over sqrt(F_ii F_jj)): 16 x 16 heat square
// 8.2e-8 / 7.1e-8; 3.6e-7 / 2.6e-7, 12^3 heat 1.10e-7 / 1.08e-7; 1.0e-6 /
// 5.6e-7, 20^3 elasticity 4.38e-7 / 4.28e-7; 5.5e-6 / 3.7e-6, 129^2 triangles
// 1.72e-7 / 1.22e-7; 1.1e-6 / 5.2e-7 (one accumulator for the six largest
// products: 8.4e-8, 1.08e-7, 4.31e-7, 1.52e-7, and up to 1.3 times the old
// element error).
// Range: planes of 2^16 x hold every FP32 value exactly, F is scaled back at
// the end; items whose tiles hold values from 2^34 on (K of about 2^-68) run on
// the FP32 units, operands straight from memory (36 ms for 16 x 20^3 elasticity).
// Per step a thread loads 8 rows of one column (a wavefront: 8 rows of 256
// bytes), splits them and writes three 16-byte pieces, [plane][row half]
// [column], the operand layout of the instruction (lane l: column l % 32, rows
// 8 (l / 32) .. + 7): LDS reads and writes of 16 consecutive bytes a lane.
// The loads of two steps are in flight, in two register sets (the loop takes
// two steps: no copies between them).  Wavefront (wi, wj) computes the
// (EDGE / 2)^2 quadrant.  The two sides of a tile on the diagonal would be
// summed in different orders: the lower one is written to both.
// Bound by the bf16 matrix units at the clock that they leave (1.2 PFLOP/s, as
// torch's bf16 product of 8192^2 matrices): FP32 units / six products / now,
// 16 x 20^3 elasticity 15.0 / 10.1 / 12.4 ms, 512 x 12^3 heat 1.22 / 0.86 /
// 0.99, 64 uneven elasticity boxes 2.45 / 1.52 / 1.81, 128 triangle meshes of
// 129^2 nodes 0.258 / 0.132 / 0.147.
// ---------------------------------------------------------------------------
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));

// 2^kSplitScale x[0..8) as three bf16 planes, h + m + l
__device__ __forceinline__ void split_bf16(const float (&x)[8], v4u& h, v4u& m, v4u& l) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v2f r = {x[2 * i] * (float)(1 << kSplitScale), x[2 * i + 1] * (float)(1 << kSplitScale)};
        h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2bf));
        r[0] -= __builtin_bit_cast(float, h[i] << 16);
        r[1] -= __builtin_bit_cast(float, h[i] & 0xFFFF0000u);
        m[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2bf));
        r[0] -= __builtin_bit_cast(float, m[i] << 16);
        r[1] -= __builtin_bit_cast(float, m[i] & 0xFFFF0000u);
        l[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2bf));
    }
}

template <int EDGE>
__global__ __launch_bounds__(256, EDGE == 128 ? 2 : 4) void syrk_split_f32(
    const SubDev* __restrict__ subs, const TileDev* __restrict__ tiles,
    const SyrkItem* __restrict__ items, const int32_t* __restrict__ ksteps, const float* __restrict__ X,
    const int32_t* __restrict__ xwide, float* __restrict__ F)
{
    constexpr int NS = EDGE / 64;                // 64-column slabs per side, sub-tiles per wavefront and side
    constexpr int kPlane = EDGE * 2;             // 16-byte pieces of one plane of one side
    __shared__ v4u lds[2][2][3 * kPlane];        // [buffer][side]
    const SyrkItem it = items[blockIdx.x];
    if (it.sub < 0) return;
    const SubDev S = subs[it.sub];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = S.n;
    const bool diag = it.I == it.J;              // one side: J reads I's planes
    // this wavefront's slab of each side it loads (EDGE = 64: wavefronts 0-1
    // load side I, 2-3 side J) and the half of the 16 rows
    const int half = EDGE == 128 ? wv >> 1 : wv & 1;
    const float* xs[NS];
    int ks[NS], bit[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int side = EDGE == 128 ? q : wv >> 1;
        const int t64 = (side ? it.J : it.I) * NS + (EDGE == 128 ? wv & 1 : 0);
        const bool have = t64 < S.ntiles && !(side && diag);
        const TileDev& T = tiles[S.tile_off + (have ? t64 : 0)];
        xs[q] = X + T.x_off;
        ks[q] = have ? T.kstart : INT_MAX;
        bit[q] = EDGE == 128 ? 2 * side + (wv & 1) : 0;
    }
    const int32_t* __restrict__ KS = ksteps + it.step_off;
    const int nsteps = it.nsteps;

    auto load_step = [&](float (&v)[NS][8], int ent, bool have) __attribute__((always_inline)) {
        const int kb = EDGE == 128 ? ent & kStepRowMask : ent;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            // rows [r0, kb + 16) of the slab, fewer at its ends, none where
            // the step entry says so: the others read as zero
            const int r0 = max(kb, ks[q]);
            const bool on = EDGE == 64 || ((ent >> (kStepSlabShift + bit[q])) & 1);
            const int rows = on && have ? min(kb + kSyrkKC, n) - r0 : 0;
            const __amdgpu_buffer_rsrc_t r =
                buffer_of(xs[q] + (int64_t)(rows > 0 ? r0 - ks[q] : 0) * kTile, rows > 0 ? rows * kTile * 4 : 0);
            const int skip = rows > 0 ? r0 - kb : 0;       // rows of the step above the slab
            int o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = lane * 4 + (8 * half + e) * (kTile * 4);
            if (skip > 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    o[e] = 8 * half + e >= skip ? o[e] - skip * (kTile * 4) : SlabRows<float, false>::kNone;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[q][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, o[e], 0, 0));
        }
    };
    auto store_step = [&](const float (&v)[NS][8], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int side = EDGE == 128 ? q : wv >> 1;
            if (side && diag) continue;
            v4u h, m, l;
            split_bf16(v[q], h, m, l);
            v4u* d = &lds[buf][side][half * EDGE + (EDGE == 128 ? 64 * (wv & 1) : 0) + lane];
            d[0] = h;
            d[kPlane] = m;
            d[2 * kPlane] = l;
        }
    };

    v16f acc[NS][NS], low[NS][NS];               // h h products; the smaller ones
#pragma unroll
    for (int a = 0; a < NS; ++a)
#pragma unroll
        for (int b = 0; b < NS; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = low[a][b][r] = 0.f;
    const int wi = wv >> 1, wj = wv & 1;
    const int frag = (lane & 31) + (lane >> 5) * EDGE;
    auto entry = [&](int st) { return KS[min(st, nsteps - 1)]; };
    // step st from LDS buffer `buf`; `v`: the rows of step st + 1, then st + 3
    auto step = [&](float (&v)[NS][8], int st, int buf) __attribute__((always_inline)) {
        const int ent = entry(st + 3);
        const v4u* pa = &lds[buf][0][wi * (EDGE / 2) + frag];
        const v4u* pb = &lds[buf][diag ? 0 : 1][wj * (EDGE / 2) + frag];
        v8bf a[NS][3], b[NS][3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                a[q][k] = __builtin_bit_cast(v8bf, pa[k * kPlane + 32 * q]);
                b[q][k] = __builtin_bit_cast(v8bf, pb[k * kPlane + 32 * q]);
            }
        // smallest products first
        constexpr int kOrder[8][2] = {{2, 1}, {1, 2}, {2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int q = 0; q < NS; ++q)
#pragma unroll
                for (int p = 0; p < NS; ++p) {
                    v16f& c = k == 7 ? acc[q][p] : low[q][p];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q][kOrder[k][0]], b[p][kOrder[k][1]], c, 0, 0, 0);
                }
        store_step(v, buf ^ 1);
        load_step(v, ent, st + 3 < nsteps);
        lds_barrier();
    };
    bool wide = false;                           // values beyond the split, on either side
#pragma unroll
    for (int q = 0; q < 2 * NS; ++q) {
        const int t64 = (q < NS ? it.I : it.J) * NS + q % NS;
        if (t64 < S.ntiles) {
            const int4 w = reinterpret_cast<const int4*>(xwide)[S.tile_off + t64];
            wide |= (w.x | w.y | w.z | w.w) != 0;
        }
    }
    const double scale = wide ? 1.0 : 1.0 / (double)(1ull << 2 * kSplitScale);
    if (!wide) {
        float v0[NS][8], v1[NS][8];              // two steps in flight
        load_step(v0, entry(0), nsteps > 0);
        load_step(v1, entry(1), nsteps > 1);
        store_step(v0, 0);
        load_step(v0, entry(2), nsteps > 2);
        lds_barrier();
        int st = 0;
        for (; st + 1 < nsteps; st += 2) {
            step(v1, st, 0);
            step(v0, st + 1, 1);
        }
        if (st < nsteps) step(v1, st, 0);
    } else {
        // the FP32 units, operands straight from memory: two rows at a time,
        // lane l row l / 32, column l % 32 of this wavefront's slab
        const float* xo[2];
        int k0[2], on[2];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int w = side ? wj : wi;
            const int t64 = (side ? it.J : it.I) * NS + (EDGE == 128 ? w : 0);
            const TileDev& T = tiles[S.tile_off + (t64 < S.ntiles ? t64 : 0)];
            k0[side] = t64 < S.ntiles ? T.kstart : INT_MAX;
            xo[side] = X + T.x_off + (EDGE == 128 ? 0 : 32 * w) + (lane & 31);
            on[side] = EDGE == 128 ? 1 << (kStepSlabShift + 2 * side + w) : 0;
        }
        for (int st = 0; st < nsteps; ++st) {
            const int ent = KS[st];
            const int kb = EDGE == 128 ? ent & kStepRowMask : ent;
#pragma unroll
            for (int s = 0; s < kSyrkKC / 2; ++s) {
                const int row = kb + 2 * s + (lane >> 5);
                float x[2][NS];
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const bool have = row >= k0[side] && row < n && (EDGE == 64 || (ent & on[side]));
#pragma unroll
                    for (int q = 0; q < NS; ++q)
                        x[side][q] = have ? xo[side][(int64_t)(row - k0[side]) * kTile + 32 * q] : 0.f;
                }
#pragma unroll
                for (int q = 0; q < NS; ++q)
#pragma unroll
                    for (int p = 0; p < NS; ++p)
                        acc[q][p] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[0][q], x[1][p], acc[q][p], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < NS; ++a)
#pragma unroll
        for (int b = 0; b < NS; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r)         // rounded once, subnormal results too
                acc[a][b][r] = (float)(((double)acc[a][b][r] + (double)low[a][b][r]) * scale);
    // D: lane l, register r holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
    const int I2 = EDGE == 128 ? it.I : it.I >> 1, J2 = EDGE == 128 ? it.J : it.J >> 1;
    float* __restrict__ Ft = F + S.F_off + (int64_t)(I2 * (I2 + 1) / 2 + J2) * kFTileElems;
    const int r0 = (EDGE == 128 ? 0 : 64 * (it.I & 1)) + wi * (EDGE / 2);
    const int c0 = (EDGE == 128 ? 0 : 64 * (it.J & 1)) + wj * (EDGE / 2);
    const bool mirror = I2 == J2;                // a stored tile on the diagonal is kept whole
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int p = 0; p < NS; ++p)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = r0 + 32 * q + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                const int col = c0 + 32 * p + (lane & 31);
                if (mirror && row < col) continue;
                Ft[row * kSyrkTile + col] = acc[q][p][r];
                if (mirror && row > col) Ft[col * kSyrkTile + row] = acc[q][p][r];
            }
}

// ---------------------------------------------------------------------------
// Inverses of the factor blocks' diagonal triangles (lower triangular, w <=
// 64), written as the lower MFMA A tiles the TRSM and the implicit apply read.
// One workgroup per block, four lanes per column: forward substitution on the
// unit vectors, the dot products of a row split over the four lanes.  Sums in
// double-double (products and their errors by fma, error-free additions, the
// quotient corrected once), rounded to FP64 at the end: more digits than the
// 64-bit mantissas of x87, in which the host computed the inverses before (22%
// of its time on an 11^3 elasticity subdomain, 40% on 12^3 heat).  Bound by the
// latency of a row (LDS, two reductions, two divisions), three workgroups a CU
// (50 KB of LDS each); LDS is busy 27% of the time, a quarter to a third of
// that with bank conflicts of the packed triangles.  0.12 ms for the 700
// blocks of 8 uneven elasticity boxes, 0.78 for the 7616 of 16 x 20^3
// elasticity, 1.5 for the 26112 of 512 x 12^3 heat, 3.4 for the 43008 of 128
// triangle meshes of 129^2 nodes.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int tri(int i, int k) { return i * (i + 1) / 2 + k; }

__global__ __launch_bounds__(256) void invert_diag(const InvItem* __restrict__ items, double* lval) {
#pragma clang fp contract(off)
    __shared__ double sl[kMaxPanel * (kMaxPanel + 1) / 2];
    __shared__ double zh[kMaxPanel * (kMaxPanel + 1) / 2], zl[kMaxPanel * (kMaxPanel + 1) / 2];
    const InvItem it = items[blockIdx.x];
    const int w = it.w;
    for (int e = threadIdx.x; e < w * w; e += 256) {
        const int k = e / w, i = e - k * w;
        if (i >= k) sl[tri(i, k)] = lval[it.diag + e];
    }
    __syncthreads();
    const int c = threadIdx.x >> 2, part = threadIdx.x & 3;      // column; share of the dot products
    const int c0 = (threadIdx.x >> 6) * 16;                      // first column of the wavefront
    for (int i = c0; i < w; ++i) {
        double hi = 0.0, lo = 0.0;
        for (int k = c + part; k < i; k += 4) {
            const double a = sl[tri(i, k)], b = zh[tri(k, c)];
            const double p = a * b;
            const double e = __builtin_fma(a, zl[tri(k, c)], __builtin_fma(a, b, -p));
            const double s = hi - p;
            const double t = s - hi;
            lo += ((hi - (s - t)) - (p + t)) - e;
            hi = s;
        }
#pragma unroll
        for (int off = 1; off < 4; off <<= 1) {
            const double h2 = __shfl_xor(hi, off, 64), l2 = __shfl_xor(lo, off, 64);
            const double s = hi + h2;
            const double t = s - hi;
            lo = (lo + l2) + ((hi - (s - t)) + (h2 - t));
            hi = s;
        }
        if (i >= c && c < w && part == 0) {
            if (i == c) {                                        // the sums are empty
                hi = 1.0;
                lo = 0.0;
            }
            const double d = sl[tri(i, i)];
            const double s = hi + lo;
            const double t = s - hi;
            lo = (hi - (s - t)) + (lo - t);
            const double q = s / d;
            const double q2 = (__builtin_fma(-q, d, s) + lo) / d;
            const double z = q + q2;
            zh[tri(i, c)] = z;
            zl[tri(i, c)] = q2 - (z - q);
        }
        // the four lanes of a column are one wavefront: its LDS accesses stay
        // in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    __syncthreads();
    const int nks = (w + 3) >> 2, nrt = (w + 15) >> 4;
    const int ntile = 2 * (nrt - 1) * nrt + nks;
    for (int e = threadIdx.x; e < ntile * 64; e += 256) {
        const int tile = e >> 6, pos = e & 63;
        const int rt = (tile >= 4) + (tile >= 12) + (tile >= 24);
        const int row = 16 * rt + (pos & 15), col = 4 * (tile - 2 * rt * (rt + 1)) + (pos >> 4);
        lval[it.linv + e] = row < w && col <= row ? zh[tri(row, col)] : 0.0;
    }
}

hipError_t launch_invert_diag(const InvItem* items, int64_t count, double* lval, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(invert_diag, dim3((unsigned)count), dim3(256), 0, stream, items, lval);
    return hipGetLastError();
}

template <bool MERGE, bool LARGE, bool LOADER>
static void trsm_launch(const DevTables& t, const int32_t* order, int64_t count, hipStream_t stream) {
    const dim3 grid((unsigned)count), block(LOADER ? 320 : 256);
    if (t.X32)
        hipLaunchKernelGGL((trsm_stair_mixed<MERGE, LARGE, LOADER>), grid, block, 0, stream, t.subs, t.tiles, t.rows,
                           t.visits, t.fresh, t.clear, t.lval, t.lval32, t.piv, t.sgn, order, t.X32, t.xwide);
    else
        hipLaunchKernelGGL((trsm_stair_f64<MERGE, LARGE, LOADER>), grid, block, 0, stream, t.subs, t.tiles, t.rows,
                           t.visits, t.fresh, t.clear, t.lval, t.piv, t.sgn, order, t.X);
}

hipError_t launch_trsm(const DevTables& t, const int32_t* order, int64_t count, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    if (t.trsm_large) {
        if (t.trsm_merge) trsm_launch<true, true, false>(t, order, count, stream);
        else trsm_launch<false, true, false>(t, order, count, stream);
    } else if (count <= kLoaderMaxTiles) {
        if (t.trsm_merge) trsm_launch<true, false, true>(t, order, count, stream);
        else trsm_launch<false, false, true>(t, order, count, stream);
    } else {
        if (t.trsm_merge) trsm_launch<true, false, false>(t, order, count, stream);
        else trsm_launch<false, false, false>(t, order, count, stream);
    }
    return hipGetLastError();
}

// FP64 launches of at most this many 64 x 64 blocks give each to four
// workgroups, a 32 x 32 quarter each (all load both sides): a block alone on a
// CU takes as long as the CU's matrix units need for it, while others idle.
// Whole blocks / quarters: one 16 x 16 heat square (1 block) 14 / 7 us, one 129^2
// triangle mesh (36) 58 / 29, 8 (288) 65 / 49, one 12^3 heat cube (105) 30 / 20;
// triangle meshes of 17^2 nodes, one block each: 64 of them 17.0 / 10.8, 128 18.2
// / 14.0, 192 18.5 / 17.2, 256 19.1 / 20.1, 288 26.9 / 24.2, 320 26.9 / 25.7, 352
// 27.3 / 27.8, 512 29 / 42; of 9^2 nodes 128 9.7 / 8.6, 256 10.3 / 11.2; one uneven
// elasticity box (861) 92 / 157.  Around 256 very short blocks, one a CU, lose up
// to 1 us; long ones gain, which the count does not tell apart.  (Not tried for
// the mixed kernel.)
constexpr int64_t kSyrkQuarterItems = 320;

hipError_t launch_syrk(const DevTables& t, const SyrkItem* items, int64_t ntile, int64_t nblock,
                       hipStream_t stream) {
    if (ntile > 0) {
        if (t.X32)
            hipLaunchKernelGGL(syrk_split_f32<128>, dim3((unsigned)ntile), dim3(256), 0, stream, t.subs, t.tiles, items,
                               t.ksteps, t.X32, t.xwide, t.F32);
        else
            hipLaunchKernelGGL(syrk_f64<128>, dim3((unsigned)ntile), dim3(256), 0, stream, t.subs, t.tiles, items,
                               t.ksteps, t.X, t.F);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (nblock > 0) {
        if (t.X32)
            hipLaunchKernelGGL(syrk_split_f32<64>, dim3((unsigned)nblock), dim3(256), 0, stream, t.subs, t.tiles,
                               items + ntile, t.ksteps, t.X32, t.xwide, t.F32);
        else
            if (nblock <= kSyrkQuarterItems)
                hipLaunchKernelGGL((syrk_f64<64, true>), dim3((unsigned)(4 * nblock)), dim3(256), 0, stream, t.subs,
                                   t.tiles, items + ntile, t.ksteps, t.X, t.F);
            else
                hipLaunchKernelGGL(syrk_f64<64>, dim3((unsigned)nblock), dim3(256), 0, stream, t.subs, t.tiles,
                                   items + ntile, t.ksteps, t.X, t.F);
        return hipGetLastError();
    }
    return hipSuccess;
}

hipError_t launch_assemble(const DevTables& t, hipStream_t stream, hipEvent_t* ev) {
    hipError_t e = hipSuccess;
    if (ev && (e = hipEventRecord(ev[0], stream)) != hipSuccess) return e;
    if ((e = launch_trsm(t, t.tile_order, t.ntiles, stream)) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[1], stream)) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[2], stream)) != hipSuccess) return e;
    if ((e = launch_syrk(t, t.syrk, t.nsyrk_tile, t.nsyrk - t.nsyrk_tile, stream)) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[3], stream)) != hipSuccess) return e;
    return hipSuccess;
}

hipError_t launch_convert_f32(const double* a, float* b, int64_t n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(convert_f64_f32, dim3((unsigned)blocks), dim3(256), 0, stream, a, b, n);
    return hipGetLastError();
}

}  // namespace scasm
