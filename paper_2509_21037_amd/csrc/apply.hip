// HIP kernels for gfx950 (CDNA4, wave64): the solution stage on the
// assembled F (explicit apply, Sec. 2.2 eq. (12); PCPG, Sec. 2.1 eq. (7))
// and the implicit apply with the factor (Sec. 2.2 eq. (11)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <mutex>

#include "device.hpp"
#include "kernels.hpp"

namespace scasm {

// ---------------------------------------------------------------------------
// Explicit apply q = F p (Sec. 2.2, eq. (12)) on the packed sorted F, FP64
// accumulation (FP32 or FP64 F).  Each stored lower tile T = F_s[I, J] is
// read once and used twice: pass 1, one workgroup per tile, writes
// u = T p_s[J] and v = T^T p_s[I] (p_s: p in sorted column order, gathered
// through pi; diagonal tiles are stored whole, v unused); pass 2, one
// workgroup per 128-row block K of a subdomain, sums u of (K, J <= K) and v
// of (I > K, K) in a fixed order and scatters the result to q in multiplier
// order (a subdomain of one tile, m <= 128, has no pass 2: pass 1 writes q).  Deterministic; reads F once, about half of the dense m x m.
// The partial sums of stored tile k live at part[(k - part_base) * 256]: the
// plan-owned buffer holds every tile (part_base 0); the fixed scratch array of
// the allocation-free apply holds one chunk of subdomains at a time.
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void load8(const T* __restrict__ src, double (&t)[8]) {
    if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double2 d = reinterpret_cast<const double2*>(src)[e];
            t[2 * e] = d.x;
            t[2 * e + 1] = d.y;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float4 f = reinterpret_cast<const float4*>(src)[e];
            t[4 * e] = f.x;
            t[4 * e + 1] = f.y;
            t[4 * e + 2] = f.z;
            t[4 * e + 3] = f.w;
        }
    }
}

template <class T>
__global__ __launch_bounds__(256) void symv_tiles(
    const SubDev* __restrict__ subs, const SyrkItem* __restrict__ ftiles, const T* __restrict__ F,
    const int32_t* __restrict__ pi, const double* __restrict__ p, double* __restrict__ part, int64_t part_base,
    double* __restrict__ q)
{
    __shared__ double sp[2][kSyrkTile];                 // p_s of the tile's columns (J) and rows (I)
    __shared__ double su[kSyrkTile][17];                // row sums per group of 8 columns
    __shared__ double sv[kSyrkTile][17];                // column sums per group of 8 rows
    const SyrkItem it = ftiles[blockIdx.x];
    const SubDev S = subs[it.sub];
    const int tid = threadIdx.x;
    {
        const int half = tid >> 7;
        const int a = (half ? it.I : it.J) * kSyrkTile + (tid & 127);
        sp[half][tid & 127] = a < S.m ? p[S.dual_off + pi[S.col_off + a]] : 0.0;
    }
    __syncthreads();
    const int64_t tile = (int64_t)it.I * (it.I + 1) / 2 + it.J;
    const T* __restrict__ Ft = F + S.F_off + tile * kFTileElems;
    const int tr = tid >> 4;                            // rows 8 tr .. 8 tr + 7
    const int tc = tid & 15;                            // columns 8 tc .. 8 tc + 7
    double pj[8], u[8], v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        pj[c] = sp[0][8 * tc + c];
        u[c] = 0.0;
        v[c] = 0.0;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 8 * tr + i;
        const double pr = sp[1][row];
        double t[8];
        load8(Ft + row * kSyrkTile + 8 * tc, t);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            u[i] += t[c] * pj[c];
            v[c] += t[c] * pr;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        su[8 * tr + i][tc] = u[i];
        sv[8 * tc + i][tr] = v[i];
    }
    __syncthreads();
    const int k = tid & 127;
    double acc = 0.0;
    if (tid < 128) {
#pragma unroll
        for (int g = 0; g < 16; ++g) acc += su[k][g];
    } else {
#pragma unroll
        for (int g = 0; g < 16; ++g) acc += sv[k][g];
    }
    if (S.m <= kSyrkTile) {                             // the only tile: u is the result
        if (tid < S.m) q[S.dual_off + pi[S.col_off + tid]] = acc;
        return;
    }
    part[((S.ftile_off + tile - part_base) << 8) + tid] = acc;
}

// 128 rows x kRowParts threads, each a share of the row block's partial sums
// (four loads in flight), combined in LDS.  16 x 20^3 elasticity (62 tiles per
// row block): 34 us with one thread per row, now 14.7;
// 64 uneven boxes (37 tiles) 19.2 / 8.2 us.
constexpr int kRowParts = 4;

__global__ __launch_bounds__(128 * kRowParts) void symv_rows(
    const SubDev* __restrict__ subs, const int2* __restrict__ frows, const int32_t* __restrict__ pi,
    const double* __restrict__ part, int64_t part_base, double* __restrict__ q)
{
    __shared__ double sum[kRowParts][kSyrkTile];
    const int2 it = frows[blockIdx.x];                  // (subdomain, row block K)
    const SubDev S = subs[it.x];
    const int K = it.y;
    const int r = threadIdx.x & (kSyrkTile - 1);
    const int pt = threadIdx.x / kSyrkTile;
    const int nt = (S.m + kSyrkTile - 1) / kSyrkTile;
    const double* __restrict__ P = part + ((S.ftile_off - part_base) << 8);
    double y = 0.0;
#pragma unroll 4
    for (int T = pt; T < nt; T += kRowParts) {          // u of tile (K, T), or v of tile (T, K)
        const int64_t hi = max(K, T), lo = min(K, T);
        y += P[((hi * (hi + 1) / 2 + lo) << 8) + (T > K ? 128 : 0) + r];
    }
    sum[pt][r] = y;
    __syncthreads();
    if (pt) return;
#pragma unroll
    for (int k = 1; k < kRowParts; ++k) y += sum[k][r];
    const int a = K * kSyrkTile + r;
    if (a < S.m) q[S.dual_off + pi[S.col_off + a]] = y;
}

// pass 1 over stored tiles [t0, t1), pass 2 over row blocks [r0, r1): the
// tiles of whole subdomains, partial sums at part[(k - t0) * 256]
static hipError_t apply_range(const DevTables& t, const double* p, double* q, double* part, int64_t t0, int64_t t1,
                              int64_t r0, int64_t r1, hipStream_t stream) {
    if (t1 <= t0) return hipSuccess;
    if (t.F32)
        hipLaunchKernelGGL(symv_tiles<float>, dim3((unsigned)(t1 - t0)), dim3(256), 0, stream, t.subs,
                           t.ftiles + t0, (const float*)t.F32, t.pi, p, part, t0, q);
    else
        hipLaunchKernelGGL(symv_tiles<double>, dim3((unsigned)(t1 - t0)), dim3(256), 0, stream, t.subs,
                           t.ftiles + t0, (const double*)t.F, t.pi, p, part, t0, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || r1 <= r0) return e;
    hipLaunchKernelGGL(symv_rows, dim3((unsigned)(r1 - r0)), dim3(128 * kRowParts), 0, stream, t.subs, t.frows + r0, t.pi,
                       (const double*)part, t0, q);
    return hipGetLastError();
}

hipError_t launch_apply(const DevTables& t, const double* p, double* q, hipStream_t stream, hipEvent_t* ev) {
    hipError_t e = hipSuccess;
    if (ev && (e = hipEventRecord(ev[0], stream)) != hipSuccess) return e;
    if ((e = apply_range(t, p, q, t.part, 0, t.nftiles, 0, t.nfrows, stream)) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[1], stream)) != hipSuccess) return e;
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// F_i as a dense matrix (column-major, leading dimension ld, multiplier
// order, FP64): one workgroup per 64 x 64 quadrant of a stored tile, read
// row by row into LDS and written twice, as stored and (off-diagonal tiles)
// mirrored, so that consecutive lanes write increasing addresses of one
// column of the result: the 64 sorted columns of a side are taken in the
// order of their multiplier indices (ranks counted in LDS).  Bound by those
// writes, runs of a few multipliers each.  Before, the host permuted a copy
// of the tiles: 32 tetrahedral subdomains of 14^3 nodes (m = 1016) took 346
// ms with their assembly, now 1.73.
// ---------------------------------------------------------------------------
constexpr int kExpandLd = 65;

template <class T>
__global__ __launch_bounds__(256) void expand_F(const SubDev* __restrict__ subs, int sub, const T* __restrict__ F,
                                                const int32_t* __restrict__ pi, double* __restrict__ out, int64_t ld)
{
    __shared__ T st[64 * kExpandLd];
    __shared__ int dst[2][64], srt[2][64];              // rows, columns: multiplier index; sorted by it
    const SubDev S = subs[sub];
    const int64_t tile = blockIdx.x >> 2;
    int I = (int)((sqrt(8.0 * (double)tile + 1.0) - 1.0) * 0.5);
    while ((int64_t)(I + 1) * (I + 2) / 2 <= tile) ++I;
    while ((int64_t)I * (I + 1) / 2 > tile) --I;
    const int J = (int)(tile - (int64_t)I * (I + 1) / 2);
    const int qr = 64 * ((blockIdx.x >> 1) & 1), qc = 64 * (blockIdx.x & 1);
    const int a0 = I * kSyrkTile + qr, b0 = J * kSyrkTile + qc;
    const int na = min(64, S.m - a0), nb = min(64, S.m - b0);
    if (na <= 0 || nb <= 0) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const T* __restrict__ Ft = F + S.F_off + tile * kFTileElems + qr * kSyrkTile + qc;
    for (int r = wv; r < 64; r += 4) st[r * kExpandLd + lane] = Ft[r * kSyrkTile + lane];
    if (wv < 2) {
        const int n = wv ? nb : na;
        dst[wv][lane] = lane < n ? pi[S.col_off + (wv ? b0 : a0) + lane] : INT_MAX;
    }
    __syncthreads();
    if (wv < 2) {
        const int me = dst[wv][lane];
        int rank = 0;
        for (int k = 0; k < 64; ++k) rank += dst[wv][k] < me || (dst[wv][k] == me && k < lane);
        srt[wv][rank] = lane;
    }
    __syncthreads();
    const int ra = srt[0][lane], rb = srt[1][lane];
    const int64_t da = dst[0][ra], db = dst[1][rb];
    for (int k = wv; k < nb; k += 4) {
        const int b = srt[1][k];
        if (lane < na) out[dst[1][b] * ld + da] = (double)st[ra * kExpandLd + b];
    }
    if (I == J) return;                                 // stored whole
    for (int k = wv; k < na; k += 4) {
        const int a = srt[0][k];
        if (lane < nb) out[dst[0][a] * ld + db] = (double)st[a * kExpandLd + rb];
    }
}

hipError_t launch_expand_F(const DevTables& t, int32_t sub, int32_t m, double* out, int64_t ld, hipStream_t stream) {
    const int64_t nt = (m + kSyrkTile - 1) / kSyrkTile;
    const dim3 grid((unsigned)(nt * (nt + 1) / 2 * 4));
    if (t.F32)
        hipLaunchKernelGGL(expand_F<float>, grid, dim3(256), 0, stream, t.subs, sub, (const float*)t.F32, t.pi, out, ld);
    else
        hipLaunchKernelGGL(expand_F<double>, grid, dim3(256), 0, stream, t.subs, sub, (const double*)t.F, t.pi, out, ld);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Allocation-free explicit apply: the partial sums go to a fixed device array
// (one per GPU, for the life of the process) instead of the plan's buffer;
// the batch runs in chunks of whole subdomains whose stored tiles fit it, one
// chunk after the other on the caller's stream.  Every call on a GPU shares
// that GPU's array, so calls that overlap on one GPU race.  Nothing needs
// clearing: pass 1 writes every partial sum that pass 2 of its chunk reads.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[kApplyScratchTiles * 256];

namespace {
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t apply_scratch_init(int device, double** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;     // caller makes `device` current
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = (double*)ptr;
    }
    if (out) *out = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_apply_chunked(const DevTables& t, const ApplyChunk* chunks, int64_t nchunks, double* scratch_ptr,
                                const double* p, double* q, hipStream_t stream) {
    for (int64_t c = 0; c < nchunks; ++c) {
        const ApplyChunk& k = chunks[c];
        if (k.t1 - k.t0 > kApplyScratchTiles) return hipErrorInvalidValue;
        hipError_t e = apply_range(t, p, q, scratch_ptr, k.t0, k.t1, k.r0, k.r1, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Projected conjugate gradients on each subdomain's dual problem (Sec. 2.1,
// eq. (7), with e = 0 and the identity preconditioner), FP64 vectors; the
// per-subdomain scalars stay on the device.
//   lambda_0 = 0, r_0 = d, w_0 = P r_0, p_0 = w_0,  P = I - G (G^T G)^{-1} G^T
//   q = F p;  alpha = (w.w)/(p.q);  lambda += alpha p;  r -= alpha q
//   w' = P r;  beta = (w'.w')/(w.w);  p = w' + beta p
// ---------------------------------------------------------------------------
constexpr int kMaxKer = 8;

struct PcpgDev {
    const double* G;        // per subdomain m x k, column-major, at g_off
    const int64_t* g_off;
    const int32_t* kdim;
    const double* GtGinv;   // per subdomain k x k at 64 * sub
    double* r;
    double* w;
    double* pvec;
    double* q;
    double* ww;             // per subdomain w.w
    double* hist;           // (iters + 1) x nsub or null
    int32_t nsub;
};

// One workgroup of NT threads per subdomain; thread i owns the rows i, i + NT,
// ... of every vector, so only the sums need barriers.  Bound by latency (the
// vectors are a few tens of KB): three reductions per step, the kernel
// dimension's dot products in one of them.  64 uneven elasticity boxes (m up
// to 4614, k = 6): 84 us per step with 256 threads and one reduction per dot
// product, now 38.
template <int NT>
struct BlockSums {
    double part[kMaxKer][NT / 64];
};

// sums of v[0 .. k) over the workgroup, to all threads, in a fixed order
template <int NT>
__device__ __forceinline__ void block_sums(double (&v)[kMaxKer], int k, BlockSums<NT>& red) {
#pragma unroll
    for (int c = 0; c < kMaxKer; ++c) {
        if (c >= k) break;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[c] += __shfl_xor(v[c], off, 64);
    }
    __syncthreads();                             // the last sums have been read
    if ((threadIdx.x & 63) == 0)
        for (int c = 0; c < k; ++c) red.part[c][threadIdx.x >> 6] = v[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kMaxKer; ++c) {
        if (c >= k) break;
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) t += red.part[c][i];
        v[c] = t;
    }
}

// w = r - G (G^T G)^{-1} G^T r over one subdomain, gr = G^T r; returns w.w
template <int NT>
__device__ __forceinline__ double project(int m, const PcpgDev& D, int sub, double (&gr)[kMaxKer], const double* r,
                                          double* w, BlockSums<NT>& red) {
    const int k = D.kdim[sub];
    const double* __restrict__ G = D.G + D.g_off[sub];
    block_sums<NT>(gr, k, red);
    double u[kMaxKer];
#pragma unroll
    for (int a = 0; a < kMaxKer; ++a) {
        u[a] = 0.0;
        if (a < k)
#pragma unroll
            for (int c = 0; c < kMaxKer; ++c)
                if (c < k) u[a] += D.GtGinv[64 * sub + a * k + c] * gr[c];
    }
    double ww[kMaxKer];
    ww[0] = 0.0;
#pragma unroll 2
    for (int i = threadIdx.x; i < m; i += NT) {
        double v = r[i];
#pragma unroll
        for (int c = 0; c < kMaxKer; ++c)
            if (c < k) v -= G[(int64_t)c * m + i] * u[c];
        w[i] = v;
        ww[0] += v * v;
    }
    block_sums<NT>(ww, 1, red);
    return ww[0];
}

template <int NT>
__global__ __launch_bounds__(NT) void pcpg_init(const SubDev* __restrict__ subs, PcpgDev D,
                                                const double* __restrict__ d, double* __restrict__ lambda) {
    __shared__ BlockSums<NT> red;
    const int sub = blockIdx.x;
    const int m = subs[sub].m;
    const int64_t o = subs[sub].dual_off;
    const int k = D.kdim[sub];
    const double* __restrict__ G = D.G + D.g_off[sub];
    double gr[kMaxKer] = {};
    for (int i = threadIdx.x; i < m; i += NT) {
        const double v = d[o + i];
        lambda[o + i] = 0.0;
        D.r[o + i] = v;
#pragma unroll
        for (int c = 0; c < kMaxKer; ++c)
            if (c < k) gr[c] += G[(int64_t)c * m + i] * v;
    }
    const double ww = project<NT>(m, D, sub, gr, D.r + o, D.w + o, red);
    for (int i = threadIdx.x; i < m; i += NT) D.pvec[o + i] = D.w[o + i];
    if (threadIdx.x == 0) {
        D.ww[sub] = ww;
        if (D.hist) D.hist[sub] = sqrt(ww);
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void pcpg_step(const SubDev* __restrict__ subs, PcpgDev D,
                                                double* __restrict__ lambda, int iter) {
    __shared__ BlockSums<NT> red;
    const int sub = blockIdx.x;
    const int m = subs[sub].m;
    const int64_t o = subs[sub].dual_off;
    const int k = D.kdim[sub];
    const double* __restrict__ G = D.G + D.g_off[sub];
    double* r = D.r + o;
    double* w = D.w + o;
    double* pv = D.pvec + o;
    const double* q = D.q + o;
    const double ww = D.ww[sub];
    double pq[kMaxKer];
    pq[0] = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < m; i += NT) pq[0] += pv[i] * q[i];
    block_sums<NT>(pq, 1, red);
    const bool go = pq[0] > 0.0 && ww > 0.0;    // converged (or breakdown): keep the iterate
    const double alpha = go ? ww / pq[0] : 0.0;
    double gr[kMaxKer] = {};
#pragma unroll 2
    for (int i = threadIdx.x; i < m; i += NT) {
        lambda[o + i] += alpha * pv[i];
        const double v = r[i] - alpha * q[i];
        r[i] = v;
#pragma unroll
        for (int c = 0; c < kMaxKer; ++c)
            if (c < k) gr[c] += G[(int64_t)c * m + i] * v;
    }
    const double ww2 = go ? project<NT>(m, D, sub, gr, r, w, red) : ww;
    const double beta = go ? ww2 / ww : 0.0;
    if (go)
#pragma unroll 4
        for (int i = threadIdx.x; i < m; i += NT) pv[i] = w[i] + beta * pv[i];
    if (threadIdx.x == 0) {
        D.ww[sub] = ww2;
        if (D.hist) D.hist[(int64_t)(iter + 1) * D.nsub + sub] = sqrt(ww2);
    }
}

// Threads per subdomain: 1024 from this mean number of multipliers on (5 rows
// a thread at m = 4614); below, 256 threads cover them in as few rounds and
// more subdomains share a CU.
constexpr int64_t kPcpgWideFrom = 768;

hipError_t launch_pcpg(const DevTables& t, const PcpgArgs& a, hipStream_t stream, const ImplicitLevels* lvh,
                       const int64_t* xoff, double* xwork, int32_t nimpl) {
    PcpgDev D;
    D.G = a.G; D.g_off = a.g_off; D.kdim = a.kdim; D.GtGinv = a.GtGinv;
    D.r = a.r; D.w = a.w; D.pvec = a.p; D.q = a.q; D.ww = a.ww; D.hist = a.hist; D.nsub = a.nsub;
    if (a.nsub <= 0) return hipSuccess;
    const bool wide = a.dual_total >= kPcpgWideFrom * a.nsub;
    const dim3 grid((unsigned)a.nsub);
    if (wide) hipLaunchKernelGGL(pcpg_init<1024>, grid, dim3(1024), 0, stream, t.subs, D, a.d, a.lambda);
    else hipLaunchKernelGGL(pcpg_init<256>, grid, dim3(256), 0, stream, t.subs, D, a.d, a.lambda);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int it = 0; it < a.iters; ++it) {
        if ((e = launch_apply(t, a.p, a.q, stream, nullptr)) != hipSuccess) return e;
        if (lvh && (e = launch_apply_implicit(t, *lvh, xoff, xwork, a.p, a.q, nimpl, stream, nullptr)) != hipSuccess)
            return e;
        if (wide) hipLaunchKernelGGL(pcpg_step<1024>, grid, dim3(1024), 0, stream, t.subs, D, a.lambda, it);
        else hipLaunchKernelGGL(pcpg_step<256>, grid, dim3(256), 0, stream, t.subs, D, a.lambda, it);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Implicit apply (Sec. 2.2, eq. (11)): q = B P^T L^{-T} L^{-1} P B^T p with the
// factor blocks, FP64.  x (n doubles per subdomain, workspace) holds P B^T p,
// then y = L^{-1} x, then z = L^{-T} y, in place.  The blocked triangular
// solves run level by level (planner: a block's forward level is one more
// than that of every block whose pruned rows reach it; its backward level one
// more than that of every block its own pruned rows lie in), one workgroup of
// kImplThreads threads per block step, wide levels a launch each, the levels next
// to the roots a chain in one launch (implicit_fwd_chain):
//   forward, block b:   y_b = L_bb^{-1} (x_b - sum of the update entries of
//                       its rows), then u_b = L[R_b, b] y_b into the update
//                       buffer (parallel to the pruned-row lists); a row's
//                       entries are summed in a fixed order (planner lists),
//                       no atomics
//   backward, block b:  z_b = L_bb^{-T} (y_b - L[R_b, b]^T z[R_b])
// The diagonal inverses are the ones the TRSM uses.  Repeated DOFs (several
// multipliers on one DOF) are summed by one thread per run of equal pivots.
// ---------------------------------------------------------------------------
// Linv[r][k], k <= r (or within r's diagonal 16 x 16 tile), of a block's
// inverse diagonal: lower tiles only, tile (rt, ks) at 64 (2 rt (rt + 1) + ks)
__device__ __forceinline__ double linv_at(const double* __restrict__ Lv, int r, int k) {
    const int rt = r >> 4;
    return Lv[(2 * rt * (rt + 1) + (k >> 2)) * 64 + (r & 15) + 16 * (k & 3)];
}

// x = P B^T p (and the chains' counters cleared) and q = B P^T x: 1024-thread workgroups, on small batches up to
// kInitSplit per subdomain, each a share of the rows (it walks all multipliers
// and keeps those whose pivot is in its share) or of the multipliers.
// 16 x 20^3 elasticity (27783 rows, 7938 multipliers): 30 + 10 us with one per
// subdomain, now 11 + 5.
constexpr int kInitThreads = 1024;
constexpr int kInitSplit = 8;
static inline int init_split(int64_t subdomains) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(kInitSplit, 256 / subdomains));
}

__global__ __launch_bounds__(kInitThreads) void implicit_init(
    const SubDev* __restrict__ subs, const int32_t* __restrict__ piv, const int32_t* __restrict__ pi,
    const int8_t* __restrict__ sgn, const int64_t* __restrict__ xoff, const double* __restrict__ p,
    double* __restrict__ xwork, const int32_t* __restrict__ sub_list, int C, int32_t* __restrict__ counters,
    int64_t ncounters)
{
    for (int64_t i = blockIdx.x * (int64_t)kInitThreads + threadIdx.x; i < ncounters;
         i += gridDim.x * (int64_t)kInitThreads)
        counters[i] = 0;
    const int at = (int)blockIdx.x / C, c = (int)blockIdx.x % C;
    const int sub = sub_list ? sub_list[at] : at;
    const SubDev S = subs[sub];
    double* __restrict__ x = xwork + xoff[sub];
    const int32_t* __restrict__ pv = piv + S.col_off;
    const int32_t* __restrict__ pis = pi + S.col_off;
    const int8_t* __restrict__ sg = sgn + S.col_off;
    const double* __restrict__ ps = p + S.dual_off;
    const int r0 = (int)((int64_t)S.n * c / C), r1 = (int)((int64_t)S.n * (c + 1) / C);
    for (int i = r0 + threadIdx.x; i < r1; i += kInitThreads) x[i] = 0.0;
    __syncthreads();
    for (int a = threadIdx.x; a < S.m; a += kInitThreads) {
        const int row = pv[a];
        if (row < r0 || row >= r1 || (a > 0 && pv[a - 1] == row)) continue;
        double v = 0.0;
        for (int b = a; b < S.m && pv[b] == row; ++b) v += (double)sg[b] * ps[pis[b]];
        x[row] = v;
    }
}

// One block step per workgroup of kImplThreads threads (16 wavefronts): the
// blocks of a level are few (the chain of one subdomain each), so each step
// spreads its short dependent sums over many threads; partial sums meet in
// LDS in a fixed order.
// factor tiles each wavefront has in flight in the off-diagonal products (16:
// 100 registers, one workgroup per CU)
constexpr int kImplBatch = 8;

__device__ __forceinline__ double sum_parts(const double (*sp)[64], int r) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < kImplParts; ++k) v += sp[k][r];
    return v;
}

// forward step of block b: x_b <- L_bb^{-1}(x_b - updates), then its updates
// L[R_b, b] x_b into its entries of ubuf; share g of G of the row tiles.
// EARLY (where few workgroups hide it): the loads of the diagonal inverse and
// of the first factor tiles are in flight during the update sums.
// wait(): before the first read of what other blocks write; kShared: they run
// in the same launch, and what passes between them goes through memory (loads
// and stores at agent scope, past the caches of one XCD).
struct NoWait {
    static constexpr bool kShared = false;
    __device__ void operator()() const {}
};
template <bool SHARED>
__device__ __forceinline__ double get(const double* p) {
    if constexpr (SHARED) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}
template <bool SHARED>
__device__ __forceinline__ void put(double* p, double v) {
    if constexpr (SHARED) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}
template <int NB, bool EARLY, class Wait = NoWait>
__device__ __forceinline__ void implicit_fwd_block(
    const ImplBlock& b, const double* __restrict__ lval, const int32_t* __restrict__ rptr,
    const int32_t* __restrict__ rpos, const double* __restrict__ x, double* __restrict__ yo,
    double* ubuf, double (*sp)[64], double* sx, int g = 0, int G = 1, const Wait& wait = Wait())
{
    const int tid = threadIdx.x;
    const int r = tid & 63;
    const int part = tid >> 6;
    const int w = b.w;
    const int nks = (w + 3) >> 2;
    const int nrt = (b.nbelow + 15) >> 4;
    const double* __restrict__ At = lval + b.aoff + r;
    double* u = ubuf + b.rows;
    // L_bb^{-1}: k split in kImplParts ranges of 4
    const double* __restrict__ Lv = lval + b.linv;
    double li[4];
    auto load_inverse = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i) li[i] = r < w && 4 * part + i <= r ? linv_at(Lv, r, 4 * part + i) : 0.0;
    };
    int t = part + kImplParts * g;
    double a[NB];
    auto load_tile = [&](int s0) {
#pragma unroll
        for (int i = 0; i < NB; ++i) a[i] = s0 + i < nks ? At[((int64_t)t * nks + s0 + i) * 64] : 0.0;
    };
    if (EARLY) {
        load_inverse();
        if (t < nrt) load_tile(0);
    }
    // x_b minus the update entries of its rows: wavefront `part` rows 4 part
    // .. 4 part + 3, 16 lanes each, four loads a lane in flight
    {
        const int q = 4 * part + (r >> 4);
        double v = 0.0;
        int e = 0, e1 = 0, at[4] = {};
        auto load_positions = [&]() {
#pragma unroll
            for (int i = 0; i < 4; ++i) at[i] = rpos[min(e + 16 * i, e1 - 1)];
        };
        if (q < w) {
            const int32_t* __restrict__ rp = rptr + b.rptr + b.row0 + q;
            e1 = rp[1];
            e = rp[0] + (r & 15);
            if (e < e1) load_positions();
            if ((r & 15) == 0) v = x[b.x + b.row0 + q];
        }
        wait();
        double sum = 0.0;
        while (e < e1) {
            double c[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = get<Wait::kShared>(ubuf + at[i]);
            const int e0 = e;
            e += 64;
            if (e < e1) load_positions();
#pragma unroll
            for (int i = 0; i < 4; ++i) sum -= e0 + 16 * i < e1 ? c[i] : 0.0;
        }
        v = sum + v;
        v += __shfl_xor(v, 1, 64);
        v += __shfl_xor(v, 2, 64);
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 8, 64);
        if ((r & 15) == 0) sx[q] = v;
    }
    if (!EARLY) load_inverse();
    __syncthreads();
    double y = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) y += li[i] * sx[4 * part + i];
    sp[part][r] = y;
    __syncthreads();
    if (tid < 64) {
        const double yb = sum_parts(sp, tid);
        sx[tid] = tid < w ? yb : 0.0;
        if (g == 0 && tid < w) yo[b.x + b.row0 + tid] = yb;   // one writer of the G copies
    }
    __syncthreads();
    // u_b = L[R_b, b] y_b: wavefront `part` takes row tiles part, part +
    // kImplParts, ...; lane l the products L[16 t + l % 16, 4 s + l / 16]
    // y[4 s + l / 16] over the k-slices s of row tile t, each wavefront load
    // one whole 512-byte A tile, NB in flight at a time; then the four
    // lanes of a row combine (y is zero past w, the tiles' padding is zero)
    if (!EARLY && t < nrt) load_tile(0);
    while (t < nrt) {
        const int row = 16 * t + r;
        double acc = 0.0;
        for (int s0 = 0;;) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (s0 + i < nks) acc += a[i] * sx[4 * (s0 + i) + (r >> 4)];
            s0 += NB;
            if (s0 >= nks) break;
            load_tile(s0);
        }
        t += kImplParts * G;
        if (t < nrt) load_tile(0);
        acc += __shfl_xor(acc, 16, 64);
        acc += __shfl_xor(acc, 32, 64);
        if (r < 16 && row < b.nbelow) put<Wait::kShared>(u + row, acc);
    }
}

__global__ __launch_bounds__(kImplThreads) void implicit_fwd(
    const ImplBlock* __restrict__ items, const double* __restrict__ lval, const int32_t* __restrict__ rptr,
    const int32_t* __restrict__ rpos, double* __restrict__ xwork, double* __restrict__ ywork, double* ubuf)
{
    __shared__ double sp[kImplParts][64];
    __shared__ double sx[64];
    implicit_fwd_block<kImplBatch, false>(items[blockIdx.x], lval, rptr, rpos, xwork, ywork, ubuf, sp, sx);
}

// L[R_b, b]^T z[R_b] over the pruned row tiles [t0, t1): column 4 part + l / 16
// in the lanes l of wavefront `part`.  Rows in groups of kImplThreads;
// wavefront `part` takes k-slice `part` (columns 4 part .. 4 part + 3), lane l
// the products L[16 t + l % 16, 4 part + l / 16] z[16 t + l % 16] over the row
// tiles t: each wavefront load is one whole 512-byte A tile, NB in flight at
// a time (EARLY: the first ones while z is gathered).  Rows past nb read the
// tiles' zero padding against zero z entries.
template <int NB, bool EARLY, class Wait = NoWait>
__device__ __forceinline__ double implicit_bwd_sum(
    const ImplBlock& b, const int32_t* __restrict__ rows, const double* __restrict__ lval, const double* x, int t0,
    int t1, double* sz, const Wait& wait = Wait())
{
    const int32_t* __restrict__ rw = rows + b.rows;
    const int tid = threadIdx.x;
    const int r = tid & 63;
    const int part = tid >> 6;
    const int nks = (b.w + 3) >> 2;
    const int nb = min(b.nbelow, 16 * t1);
    const double* __restrict__ At = lval + b.aoff;
    double acc = 0.0;
    for (int c0 = 16 * t0; c0 < nb; c0 += kImplThreads) {
        const int nrt = part < nks ? (min(kImplThreads, nb - c0) + 15) >> 4 : 0;
        const double* __restrict__ Ts = At + ((int64_t)(c0 >> 4) * nks + part) * 64 + r;
        double a[NB];
        auto load_tiles = [&](int u0) {
#pragma unroll
            for (int i = 0; i < NB; ++i) a[i] = u0 + i < nrt ? Ts[(int64_t)(u0 + i) * nks * 64] : 0.0;
        };
        if (EARLY) load_tiles(0);
        const int row = c0 + tid < nb ? rw[c0 + tid] : -1;
        if (c0 == 16 * t0) wait();
        const double z = row >= 0 ? get<Wait::kShared>(x + b.x + row) : 0.0;               // z of the pruned rows: final
        __syncthreads();
        sz[tid] = z;
        __syncthreads();
        for (int u0 = 0; u0 < nrt; u0 += NB) {
            if (!EARLY || u0 > 0) load_tiles(u0);
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (u0 + i < nrt) acc += a[i] * sz[16 * (u0 + i) + (r & 15)];
        }
    }
    acc += __shfl_xor(acc, 1, 64);
    acc += __shfl_xor(acc, 2, 64);
    acc += __shfl_xor(acc, 4, 64);
    acc += __shfl_xor(acc, 8, 64);
    return acc;
}

// z_b = L_bb^{-T} v (v in sv): k split in kImplParts ranges of 4; li: this
// thread's values of the inverse (linv_col)
__device__ __forceinline__ void linv_col(const ImplBlock& b, const double* __restrict__ lval, double (&li)[4]) {
    const double* __restrict__ Lv = lval + b.linv;
    const int r = threadIdx.x & 63, part = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * part + i;
        li[i] = k >= r && k < b.w ? linv_at(Lv, k, r) : 0.0;
    }
}

template <bool SHARED = false>
__device__ __forceinline__ void implicit_bwd_finish(const ImplBlock& b, const double (&li)[4], double* x,
                                                    double (*sp)[64], const double* sv) {
    const int r = threadIdx.x & 63, part = threadIdx.x >> 6;
    double z = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) z += li[i] * sv[4 * part + i];
    sp[part][r] = z;
    __syncthreads();
    if ((int)threadIdx.x < b.w) put<SHARED>(x + b.x + b.row0 + threadIdx.x, sum_parts(sp, threadIdx.x));
}

// backward step of block b: z_b <- L_bb^{-T}(y_b - L[R_b, b]^T z[R_b])
template <int NB, bool EARLY>
__device__ __forceinline__ void implicit_bwd_block(
    const ImplBlock& b, const int32_t* __restrict__ rows, const double* __restrict__ lval,
    const double* __restrict__ yi, double* x, double (*sp)[64], double* sz, double* sv)
{
    const int r = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int c = 4 * part + (r >> 4);
    double li[4];
    if (EARLY) linv_col(b, lval, li);
    const double acc = implicit_bwd_sum<NB, EARLY>(b, rows, lval, x, 0, (b.nbelow + 15) >> 4, sz);
    if (!EARLY) linv_col(b, lval, li);
    if ((r & 15) == 0) sv[c] = c < b.w ? yi[b.x + b.row0 + c] - acc : 0.0;
    __syncthreads();
    implicit_bwd_finish(b, li, x, sp, sv);
}

__global__ __launch_bounds__(kImplThreads) void implicit_bwd(
    const ImplBlock* __restrict__ items, const int32_t* __restrict__ rows, const double* __restrict__ lval,
    const double* __restrict__ ywork, double* xwork)
{
    __shared__ double sp[kImplParts][64];
    __shared__ double sz[kImplThreads];
    __shared__ double sv[64];
    implicit_bwd_block<kImplBatch, false>(items[blockIdx.x], rows, lval, ywork, xwork, sp, sz, sv);
}

// A chain of levels in one launch: a workgroup waits for its own subdomain's
// earlier levels instead of for a launch.  A workgroup takes the next item of
// the list when it starts and waits only for items before its own, which
// started workgroups hold: whatever the order of dispatch, the earliest
// unfinished item waits for none, so every wait ends.  Bound by the latency of
// a level (a counter and the rows it depends on through memory, two reductions
// over the workgroup, 8.5 us): the factor tiles, the inverse and all indices
// are loaded while it waits, several levels ahead of the sweep.  A launch (or
// two) per level / chains: 16 x 20^3 elasticity 1.80 / 1.32 ms, 64 uneven
// boxes 1.03 / 0.74, 8 triangle meshes of 129^2 nodes 0.198 / 0.161.  What passes
// between workgroups is written through to memory and read from there; with
// the caches written back and invalidated instead (agent-scope fences) a level
// took 100 us.
__device__ __forceinline__ int chain_ticket(int32_t* ticket, int* sh) {
    if (threadIdx.x == 0) *sh = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*sh);
}
// Until `need` items have finished; what they wrote is visible afterwards.
// Calls that overlap on one plan (they may not) share the counters: a wait
// that they leave without an end gives up after `looks` looks at the counter
// and releases all others of its subdomain.  The gather then writes NaN for
// the subdomain, whose sums may be incomplete, and the plan's fault word is
// set.  Looks and not time: while the queue is preempted no time is up.
struct ChainWait {
    static constexpr bool kShared = true;
    int32_t* done;
    int need;
    int looks;
    int32_t* fault;
    __device__ __forceinline__ void operator()() const {
        if (threadIdx.x == 0 && need > 0) {
            int left = looks;
            while (__hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
                if (left-- > 0) {
                    __builtin_amdgcn_s_sleep(8);
                } else {
                    __hip_atomic_store(done, kImplGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
        }
        __syncthreads();
    }
};
// counts this workgroup's item, once its stores have reached memory; returns
// the count before (thread 0)
__device__ __forceinline__ int chain_done(int32_t* done) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) return __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return 0;
}

__global__ __launch_bounds__(kImplThreads, 8) void implicit_fwd_chain(
    const ImplChainItem* __restrict__ items, const double* __restrict__ lval, const int32_t* __restrict__ rptr,
    const int32_t* __restrict__ rpos, const double* __restrict__ xwork, double* __restrict__ ywork, double* ubuf,
    int32_t* ticket, int32_t* done, int n, int looks, int32_t* fault)
{
    __shared__ double sp[kImplParts][64];
    __shared__ double sx[64];
    __shared__ int sh;
    const int at = chain_ticket(ticket, &sh);
    if (at >= n) return;
    const ImplChainItem it = items[at];
    implicit_fwd_block<kImplBatch, true>(it.b, lval, rptr, rpos, xwork, ywork, ubuf, sp, sx, it.g, it.G,
                                              ChainWait{done + it.sub * kImplCounterStride, it.need, looks, fault});
    chain_done(done + it.sub * kImplCounterStride);
}

__global__ __launch_bounds__(kImplThreads, 8) void implicit_bwd_chain(
    const ImplChainItem* __restrict__ items, const int32_t* __restrict__ rows, const double* __restrict__ lval,
    const double* __restrict__ ywork, double* xwork, double* cpart, int32_t* ticket, int32_t* done, int32_t* shares,
    int n, int looks, int32_t* fault)
{
    __shared__ double sp[kImplParts][64];
    __shared__ double sz[kImplThreads];
    __shared__ double sv[64];
    __shared__ int sh;
    const int at = chain_ticket(ticket, &sh);
    if (at >= n) return;
    const ImplChainItem it = items[at];
    const ImplBlock& b = it.b;
    const int r = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int c = 4 * part + (r >> 4);
    const int nrt = (b.nbelow + 15) >> 4;
    const int per = (nrt + it.G - 1) / it.G;
    const ChainWait wait{done + it.sub * kImplCounterStride, it.need, looks, fault};
    double li[4];
    if (it.G == 1) linv_col(b, lval, li);
    const double acc = implicit_bwd_sum<kImplBatch, true>(b, rows, lval, xwork, it.g * per,
                                                               min(nrt, (it.g + 1) * per), sz, wait);
    if (it.G == 1) {
        if ((r & 15) == 0) sv[c] = c < b.w ? ywork[b.x + b.row0 + c] - acc : 0.0;
    } else {
        // the last share to finish adds them up, in their order
        if ((r & 15) == 0) put<true>(cpart + (int64_t)at * 64 + c, acc);
        const int before = chain_done(shares + at - it.g);
        if (threadIdx.x == 0) sh = before;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(sh) != it.G - 1) return;
        linv_col(b, lval, li);
        if (threadIdx.x < 64) {
            const int k = threadIdx.x;
            double v = k < b.w ? ywork[b.x + b.row0 + k] : 0.0;
            double s[kImplSplit];
#pragma unroll
            for (int g = 0; g < kImplSplit; ++g) s[g] = g < it.G ? get<true>(cpart + (int64_t)(at - it.g + g) * 64 + k) : 0.0;
#pragma unroll
            for (int g = 0; g < kImplSplit; ++g) v -= s[g];
            sv[k] = k < b.w ? v : 0.0;
        }
    }
    __syncthreads();
    implicit_bwd_finish<true>(b, li, xwork, sp, sv);
    chain_done(done + it.sub * kImplCounterStride);
}

// Both sweeps of one subdomain in one workgroup: its blocks in increasing
// order (forward) and decreasing order (backward) are dependency orders, and
// a workgroup barrier (a workgroup-scope release / acquire of the global
// writes) separates consecutive blocks; no launch per level.
__global__ __launch_bounds__(kImplThreads) void implicit_sweeps(
    const SubDev* __restrict__ subs, const BlockDev* __restrict__ blocks, const int32_t* __restrict__ rows,
    const double* __restrict__ lval, const int64_t* __restrict__ rptr_off, const int32_t* __restrict__ rptr,
    const int32_t* __restrict__ rpos, const int64_t* __restrict__ xoff, double* xwork, double* ywork, double* ubuf,
    const int32_t* __restrict__ sub_list)
{
    __shared__ double sp[kImplParts][64];
    __shared__ double sx[64];
    __shared__ double sz[kImplThreads];
    const int sub = sub_list ? sub_list[blockIdx.x] : (int)blockIdx.x;
    const SubDev S = subs[sub];
    const int64_t xo = xoff[sub], ro = rptr_off[sub];
    auto block = [&](int k) {
        const BlockDev d = blocks[S.blk_off + k];
        return ImplBlock{S.lval_off + d.linv_off, S.lval_off + d.aoff, S.rows_off + d.rows_off, xo, ro,
                         d.row0, d.w, d.nbelow, 0};
    };
    for (int k = 0; k < S.nblocks; ++k) {
        implicit_fwd_block<kImplBatch, true>(block(k), lval, rptr, rpos, xwork, ywork, ubuf, sp, sx);
        __syncthreads();
    }
    for (int k = S.nblocks - 1; k >= 0; --k) {
        implicit_bwd_block<kImplBatch, true>(block(k), rows, lval, ywork, xwork, sp, sz, sx);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kInitThreads) void implicit_gather(
    const SubDev* __restrict__ subs, const int32_t* __restrict__ piv, const int32_t* __restrict__ pi,
    const int8_t* __restrict__ sgn, const int64_t* __restrict__ xoff, const double* __restrict__ xwork,
    double* __restrict__ q, const int32_t* __restrict__ sub_list, int C, const int32_t* __restrict__ fw_done,
    const int32_t* __restrict__ bw_done)
{
    const int at = (int)blockIdx.x / C, c = (int)blockIdx.x % C;
    const int sub = sub_list ? sub_list[at] : at;
    const SubDev S = subs[sub];
    const double* __restrict__ x = xwork + xoff[sub];
    // a wait of the chains gave up (ChainWait): no value is known to be right
    const bool bad = fw_done && (fw_done[sub * kImplCounterStride] >= kImplGaveUp ||
                                 bw_done[sub * kImplCounterStride] >= kImplGaveUp);
    for (int a = c * kInitThreads + threadIdx.x; a < S.m; a += C * kInitThreads)
        q[S.dual_off + pi[S.col_off + a]] =
            bad ? __builtin_nan("") : (double)sgn[S.col_off + a] * x[piv[S.col_off + a]];
}

hipError_t launch_implicit_init(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff, double* xwork,
                                const double* p, int32_t count, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    const int C = init_split(count);
    hipLaunchKernelGGL(implicit_init, dim3((unsigned)(count * C)), dim3(kInitThreads), 0, stream, t.subs, t.piv, t.pi,
                       t.sgn, xoff, p, xwork, lv.subs, C, lv.counters, lv.counters ? lv.ncounters() : 0);
    return hipGetLastError();
}

hipError_t launch_implicit_sweeps(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff, double* xwork,
                                  int32_t count, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    // every table and workspace the sweeps dereference must be in place
    if (!xoff || !xwork || !lv.ywork || !lv.ubuf || !lv.rptr_off || !lv.rptr || !lv.rpos) return hipErrorInvalidValue;
    if ((lv.nfw_chain > 0 || lv.nbw_chain > 0) &&
        (!lv.counters || !lv.fault || (lv.nfw_chain > 0 && !lv.fw_chain_items) || (lv.nbw_chain > 0 && (!lv.bw_chain_items || !lv.cpart))))
        return hipErrorInvalidValue;
    if (!lv.per_subdomain && ((lv.fw_off.size() > 1 && !lv.fw_items) || (lv.bw_off.size() > 1 && !lv.bw_items)))
        return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    if (lv.per_subdomain) {
        hipLaunchKernelGGL(implicit_sweeps, dim3((unsigned)count), dim3(kImplThreads), 0, stream, t.subs, t.blocks,
                           t.rows, t.lval, lv.rptr_off, lv.rptr, lv.rpos, xoff, xwork, lv.ywork, lv.ubuf, lv.subs);
        return hipGetLastError();
    }
    int32_t* const fw_done = lv.fw_done();
    int32_t* const bw_done = lv.bw_done();
    for (size_t l = 0; l < lv.fw_chain && l + 1 < lv.fw_off.size(); ++l) {
        const int64_t cnt = lv.fw_off[l + 1] - lv.fw_off[l];
        if (cnt <= 0) continue;
        hipLaunchKernelGGL(implicit_fwd, dim3((unsigned)cnt), dim3(kImplThreads), 0, stream,
                           lv.fw_items + lv.fw_off[l], t.lval, lv.rptr, lv.rpos, xwork, lv.ywork, lv.ubuf);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (lv.nfw_chain > 0) {
        hipLaunchKernelGGL(implicit_fwd_chain, dim3((unsigned)lv.nfw_chain), dim3(kImplThreads), 0, stream,
                           lv.fw_chain_items, t.lval, lv.rptr, lv.rpos, xwork, lv.ywork, lv.ubuf, lv.counters, fw_done,
                           (int)lv.nfw_chain, lv.looks, lv.fault);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (lv.nbw_chain > 0) {
        hipLaunchKernelGGL(implicit_bwd_chain, dim3((unsigned)lv.nbw_chain), dim3(kImplThreads), 0, stream,
                           lv.bw_chain_items, t.rows, t.lval, lv.ywork, xwork, lv.cpart, lv.counters + kImplCounterStride,
                           bw_done, bw_done + lv.nsub * kImplCounterStride, (int)lv.nbw_chain, lv.looks, lv.fault);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (size_t l = lv.bw_chain; l + 1 < lv.bw_off.size(); ++l) {
        const int64_t cnt = lv.bw_off[l + 1] - lv.bw_off[l];
        if (cnt <= 0) continue;
        hipLaunchKernelGGL(implicit_bwd, dim3((unsigned)cnt), dim3(kImplThreads), 0, stream,
                           lv.bw_items + lv.bw_off[l], t.rows, t.lval, lv.ywork, xwork);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_implicit_gather(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff,
                                  const double* xwork, double* q, int32_t count, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    const int C = init_split(count);
    const bool chains = lv.counters && !lv.per_subdomain;
    hipLaunchKernelGGL(implicit_gather, dim3((unsigned)(count * C)), dim3(kInitThreads), 0, stream, t.subs, t.piv, t.pi,
                       t.sgn, xoff, xwork, q, lv.subs, C, chains ? lv.fw_done() : nullptr,
                       chains ? lv.bw_done() : nullptr);
    return hipGetLastError();
}

hipError_t launch_apply_implicit(const DevTables& t, const ImplicitLevels& lv, const int64_t* xoff, double* xwork,
                                 const double* p, double* q, int32_t count, hipStream_t stream, hipEvent_t* ev) {
    hipError_t e = hipSuccess;
    if (ev && (e = hipEventRecord(ev[0], stream)) != hipSuccess) return e;
    if ((e = launch_implicit_init(t, lv, xoff, xwork, p, count, stream)) != hipSuccess) return e;
    if ((e = launch_implicit_sweeps(t, lv, xoff, xwork, count, stream)) != hipSuccess) return e;
    if ((e = launch_implicit_gather(t, lv, xoff, xwork, q, count, stream)) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[1], stream)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace scasm
