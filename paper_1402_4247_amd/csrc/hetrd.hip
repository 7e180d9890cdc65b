// Blocked Householder tridiagonalisation of a batch of Hermitian matrices
// (lower storage): Section III, Procedures 1-6 of Eigen_HH, arXiv:1402.4247,
// reorganised in panels of nb columns.
//
// Per column i of a panel starting at p (j = i - p, o = i + 1), two kernels:
//   zhemv  : one chunk of the Hermitian product z = A22 u (Procedure 4) from
//       the lower triangle only, with u the column below the sub-diagonal as
//       it stands (u_o = 0, u_r = A(r, i)), plus the chunk's share of
//       q = Re(u^H z).  It needs nothing derived in this step, so the
//       workgroups only stream their tiles.  A few more workgroups form the
//       panel products W^H u and V^H u and ||u||^2 meanwhile.
//   update : every wave derives the reflector (Procedure 2, stable sign, real
//       beta), v = (1, scale * A(o+1:n, i)), and forms for its rows
//       y = tau (A22(:, o) + scale z - V (W^H v) - W (V^H v))
//       (A22 v = A22(:, o) + scale A22 u by linearity) and
//       w = y - (tau/2)(y^H v) v (Procedure 5).  y^H v needs no reduction over
//       y: with h = A22(:, o), v^H A22 v = h_o + 2 Re(scale z_o) + |scale|^2 q
//       and y^H v = conj(tau) (v^H A22 v - 2 Re((V^H v)^H (W^H v))), so
//       alpha2 = -(tau/2) y^H v = -|tau|^2 / 2 (...) is real and every
//       wave computes it, and row o of w, from the same partials.
//       Then the next column of the panel is brought up to date,
//       A(o:n, o) -= V(o:n, 0:j) conj(W(o, 0:j))^T + W(o:n, 0:j) conj(V(o, 0:j))^T.
// After the panel the trailing matrix takes the rank-2nb update
// A22 -= V W^H + W V^H (Procedure 6, on MFMA).
// Once a panel's trailing matrix is small enough, the rest of the reduction
// runs in one launch, unblocked, with the matrix in registers (hetrd_res.hip).
// Every sum is taken in a fixed order (no atomic adds to a value; a group's
// members meet through atomics), so results are bitwise reproducible run to run.
#include <type_traits>

#include "common.hpp"
#include "lanes.hpp"
#include "kernels.hpp"
#include "reflector.hpp"

namespace kgev {

// 32-bit raw buffer load (the 64- and 128-bit forms are in common.hpp)
__device__ int raw_buffer_load_i32(i4_t rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.i32");

namespace {

constexpr int ZT = 64;          // ZHEMV tile edge
constexpr int ZCH = 4;          // tiles per ZHEMV chunk: one per wave of the workgroup

// chunks of block column C in the four-tile form, and in the form a
// reduction uses (ws.zch: 4 tiles per chunk, or 1 for the one-tile form)
__device__ __host__ inline int nchunks(int NB, int C) { return (NB - C + ZCH - 1) / ZCH; }
__device__ __host__ inline int nchunks_z(int NB, int C, int zch) { return zch == 1 ? NB - C : (NB - C + 3) >> 2; }

// One halving step of the transposing reduction: lanes with the MASK bit set
// keep values HALF..2HALF-1 (moved down to 0..HALF-1), the others keep
// 0..HALF-1; each adds its partner's copy of the values it keeps.  Across
// rows (MASK 16, 32) a permlane swap of the pair (t[q], t[q + HALF]) leaves
// both addends in place; within a row the sent value is selected and moved
// by DPP.
template <int MASK, int HALF, int NV, typename R>
__device__ __attribute__((always_inline)) inline void halve_step(cx<R> (&t)[NV], bool up)
{
#pragma unroll
    for (int q = 0; q < HALF; ++q) {
        if constexpr (MASK >= 16) {
            cx<R> a = t[q], c = t[q + HALF];
            swap_across<MASK>(a.x, c.x);
            swap_across<MASK>(a.y, c.y);
            t[q] = cadd(a, c);
        } else {
            const cx<R> send = csel(up, t[q], t[q + HALF]);
            const cx<R> keep = csel(up, t[q + HALF], t[q]);
            cx<R> rcv;
            rcv.x = lane_xor<MASK>(send.x);
            rcv.y = lane_xor<MASK>(send.y);
            t[q] = cadd(keep, rcv);
        }
    }
}

// r + r(lane ^ MASK), as vector-ALU lane exchanges
template <int MASK, typename R>
__device__ __attribute__((always_inline)) inline cx<R> xor_add_v(cx<R> r)
{
    r.x = xor_sum<MASK>(r.x);
    r.y = xor_sum<MASK>(r.y);
    return r;
}

// 8 complex values per lane -> lane l holds the sum over the wave of value
// (l >> 3) & 7 (three halving steps over lane bits 5..3, then plain xor sums
// over bits 2..0).
template <typename R>
__device__ __attribute__((always_inline)) inline cx<R> transpose_sum8(cx<R> (&t)[8], int lane)
{
    halve_step<32, 4, 8, R>(t, (lane & 32) != 0);
    halve_step<16, 2, 8, R>(t, (lane & 16) != 0);
    halve_step<8, 1, 8, R>(t, (lane & 8) != 0);
    cx<R> r = t[0];
    r = xor_add_v<4, R>(r);
    r = xor_add_v<2, R>(r);
    r = xor_add_v<1, R>(r);
    return r;
}

// ---------------------------------------------------------------------------
// The panel products with column i, W^H u and V^H u (u below the sub-diagonal),
// and ||u||^2: workgroup `unit` of a problem takes DV of the 2 j vectors
// W(:, 0..j-1), V(:, p..p+j-1), one row per thread and step.
constexpr int DV = 8;
__host__ __device__ inline int dot_units(int j) { return j == 0 ? 1 : (2 * j + DV - 1) / DV; }

template <typename R>
__device__ __attribute__((always_inline)) inline void panel_dots(const HetrdWs<R>& ws, int i, int p, int unit, int64_t b)
{
    __shared__ cx<R> sd[4][DV];
    __shared__ R sn[4];
    const int n = ws.n, j = i - p;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const cx<R>* Ai = ws.A + b * ws.sA + (int64_t)i * ws.lda;
    const cx<R>* Wp = ws.W + b * ws.sW;
    const cx<R>* Vp = ws.V + b * ws.sV + (int64_t)p * n;
    const cx<R>* P[DV];
#pragma unroll
    for (int k = 0; k < DV; ++k) {
        const int idx = unit * DV + k;
        P[k] = idx < j ? Wp + (int64_t)idx * n : Vp + (int64_t)(idx < 2 * j ? idx - j : 0) * n;
    }
    cx<R> acc[DV];
#pragma unroll
    for (int k = 0; k < DV; ++k) acc[k] = czero<cx<R>>();
    R nrm = 0;
#pragma unroll 2
    for (int r = i + 2 + tid; r < n; r += 256) {
        const cx<R> u = Ai[r];
#pragma unroll
        for (int k = 0; k < DV; ++k) acc[k] = cfmac(P[k][r], u, acc[k]);
        nrm = fma(u.x, u.x, fma(u.y, u.y, nrm));
    }
    const cx<R> s = transpose_sum8<R>(acc, lane);
    nrm = dpp_wave_sum(nrm);
    if ((lane & 7) == 0) sd[w][lane >> 3] = s;
    if (lane == 0) sn[w] = nrm;
    __syncthreads();
    const int idx = unit * DV + tid;
    if (tid < DV && idx < 2 * j)
        ws.pdot[b * ws.s_pdot + (idx < j ? idx : ws.nb + idx - j)] =
            cadd(cadd(sd[0][tid], sd[1][tid]), cadd(sd[2][tid], sd[3][tid]));
    if (unit == 0 && tid == 0) {
        ws.unorm[b] = (sn[0] + sn[1]) + (sn[2] + sn[3]);
        if (j == 0) ws.d[b * n + i] = Ai[i].x;
    }
}

// ---------------------------------------------------------------------------
// One chunk of z = A22 u.  A chunk is up to four 64x64 tiles (R0..R0+3, C) of
// one block column of the lower triangle; wave w owns tile R0 + w whole: the
// direct part z_R += A_RC u_C comes out complete per row, the transposed part
// z_C += A_RC^H u_R per column.  Each group of 8 columns is multiplied, its
// products go to the wave's LDS block, the next group is requested into the
// same registers, and the column sums are taken from LDS while it is in
// flight; the four waves' column sums are added once.  Three workgroups per
// CU.  The first `units` workgroups of a problem form the panel products.
template <typename R, bool BUF>
__global__ __launch_bounds__(256, 3) void hetrd_zhemv(HetrdWs<R> ws, int i, int p, int units, int rev)
{
    __shared__ cx<R> svC[ZCH][ZT];
    __shared__ cx<R> sT[ZCH][ZT];
    __shared__ cx<R> sP[ZCH][8][ZT + 1];      // per-wave staging of one group's products
    // rev: the workgroups take the chunks in reverse order (last k-point's
    // last chunk first), so that a launch after a forward one starts on the
    // tiles its predecessor read last
    const int64_t b = rev ? (int64_t)(gridDim.y - 1 - blockIdx.y) : (int64_t)blockIdx.y;
    if ((int)blockIdx.x < units) {
        panel_dots(ws, i, p, blockIdx.x, b);
        return;
    }
    const int lid = rev ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x - units;
    const int n = ws.n;
    const int o = i + 1;
    const int m = n - o;
    const int NB = (m + ZT - 1) / ZT;

    // which (block column C, chunk ch) is ours
    int bid = lid, C = 0;
    for (; C < NB; ++C) {
        const int nc = nchunks(NB, C);
        if (bid < nc) break;
        bid -= nc;
    }
    if (C >= NB) return;
    const int ch = bid;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const cx<R>* A = ws.A + b * ws.sA;
    const cx<R>* Ai = A + (int64_t)i * ws.lda;
    const int64_t lda = ws.lda;
    const int Rb = C + ch * ZCH + w;
    const bool have_tile = Rb < NB;
    const int64_t gr = (int64_t)o + (int64_t)(have_tile ? Rb : C) * ZT + lane;
    const bool row_ok = gr < n;
    // Loads are unconditional from a clamped (in-bounds) address and the value
    // is masked afterwards, so no branch guards them.
    // Matrices under 2 GiB are read with buffer loads: one 32-bit row offset
    // per lane shared by every load of the tile, the column offset in a
    // scalar register (fewer vector registers and no 64-bit address
    // arithmetic); larger ones with plain global loads.
    const int rowc = row_ok ? (int)gr : n - 1;
    const int64_t gcb = (int64_t)o + (int64_t)C * ZT;
    const i4_t rsrc = buffer_rsrc(A, (uint32_t)(BUF ? (int64_t)sizeof(cx<R>) * lda * n : 0));
    auto load_one = [&](int g, int cc) -> cx<R> {
        const int64_t gc = gcb + g * 8 + cc;
        const int64_t gcc = gc < n ? gc : (int64_t)n - 1;
        if constexpr (BUF) {
            const int soff = (int)(gcc * lda * (int64_t)sizeof(cx<R>));
            if constexpr (sizeof(R) == 8)
                return __builtin_bit_cast(cx<R>, raw_buffer_load_v4i32(rsrc, rowc * (int)sizeof(cx<R>), soff, 0));
            else
                return __builtin_bit_cast(cx<R>, raw_buffer_load_v2i32(rsrc, rowc * (int)sizeof(cx<R>), soff, 0));
        } else {
            return A[gcc * lda + rowc];
        }
    };
    auto load_group = [&](int g, cx<R> (&a)[8]) {
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) a[cc] = load_one(g, cc);
    };
    // u first, then the first column group; each wave keeps its own copy of
    // u_C in LDS, so the waves do not wait for each other before the products
    const int64_t gcu = gcb + lane;
    const cx<R> uC = Ai[gcu < n ? gcu : (int64_t)n - 1];
    cx<R> uR = Ai[row_ok ? gr : (int64_t)n - 1];
    cx<R> a[8];
    load_group(0, a);
    svC[w][lane] = csel(gcu > o && gcu < n, uC, czero<cx<R>>());
    if (!(row_ok && gr > o)) uR = czero<cx<R>>();
    wave_sync();

    __shared__ R sq[ZCH];
    R qd = 0;
    if (have_tile) {
        const bool diag_tile = (Rb == C);
        cx<R> yd = czero<cx<R>>();
        // one group of 8 columns; NEXT: the next group's columns are requested
        // as this group's registers free up (the last group has none to fetch)
        auto group = [&](int g, auto next) {
            constexpr bool NEXT = decltype(next)::value;
            const int64_t gc0 = gcb + g * 8;
#pragma unroll
            for (int cc = 0; cc < 8; ++cc) {
                const int64_t gc = gc0 + cc;
                const bool ok = row_ok && gc < n && (!diag_tile || gr >= gc);
                const bool diag = diag_tile && (gr == gc);
                cx<R> x;
                x.x = ok ? a[cc].x : (R)0;
                x.y = (ok && !diag) ? a[cc].y : (R)0;
                yd = cfma(x, svC[w][g * 8 + cc], yd);
                // the diagonal entry is counted once (direct part only)
                sP[w][cc][lane] = csel(diag, czero<cx<R>>(), cmulc(x, uR));
                // the column's register is free: request the next group's
                // column at once, so that group streams in while this one is
                // still being multiplied out
                if constexpr (NEXT) a[cc] = load_one(g + 1, cc);
            }
            // the products are in this wave's LDS block; the column sums are
            // taken from LDS while the next group is in flight: lane l adds
            // rows 8 (l / 8) .. +7 of column l mod 8, then the eight lanes of
            // a column combine
            __builtin_amdgcn_wave_barrier();
            const int c = lane & 7, r0 = (lane >> 3) * 8;
            cx<R> cs = czero<cx<R>>();
#pragma unroll
            for (int r = 0; r < 8; ++r) cs = cadd(cs, sP[w][c][r0 + r]);
            cs = xor_add_v<8, R>(cs);
            cs = xor_add_v<16, R>(cs);
            cs = xor_add_v<32, R>(cs);
            if (lane < 8) sT[w][g * 8 + lane] = cs;
            __builtin_amdgcn_wave_barrier();
        };
#pragma unroll 1
        for (int g = 0; g < 7; ++g) group(g, std::true_type{});
        group(7, std::false_type{});
        ws.ypart[b * ws.s_ypart + ((int64_t)Rb * ws.NBmax + C) * ZT + lane] = yd;
        qd = uR.x * yd.x + uR.y * yd.y;
    } else {
        sT[w][lane] = czero<cx<R>>();
    }
    qd = dpp_wave_sum(qd);
    if (lane == 0) sq[w] = qd;
    __syncthreads();
    if (tid < ZT) {
        const cx<R> s = cadd(cadd(sT[0][tid], sT[1][tid]), cadd(sT[2][tid], sT[3][tid]));
        ws.ypartT[b * ws.s_ypartT + ((int64_t)C * ws.CHmax + ch) * ZT + tid] = s;
        R qt = svC[0][tid].x * s.x + svC[0][tid].y * s.y;
        qt = dpp_wave_sum(qt);
        if (tid == 0) ws.qpart[b * ws.s_qpart + lid] = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + qt;
    }
}

// The same product in one-tile chunks, for launches where the four-tile form
// would give fewer workgroups than three per CU (few k-points): the four
// waves share one tile, wave w taking column groups 2w and 2w + 1; their
// direct parts are added in LDS, and each column's sum comes from the one
// wave that owns it.  Same partial-sum layout with one chunk per tile.
template <typename R, bool BUF>
__global__ __launch_bounds__(256, 3) void hetrd_zhemv_tile(HetrdWs<R> ws, int i, int p, int units, int rev)
{
    __shared__ cx<R> svC[ZCH][ZT];
    __shared__ cx<R> sT[ZCH][ZT];
    __shared__ cx<R> sP[ZCH][8][ZT + 1];
    const int64_t b = rev ? (int64_t)(gridDim.y - 1 - blockIdx.y) : (int64_t)blockIdx.y;
    if ((int)blockIdx.x < units) {
        panel_dots(ws, i, p, blockIdx.x, b);
        return;
    }
    const int lid = rev ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x - units;
    const int n = ws.n;
    const int o = i + 1;
    const int m = n - o;
    const int NB = (m + ZT - 1) / ZT;
    // which tile (Rb, C) of the lower triangle is ours: tiles enumerated down
    // each block column
    int bid = lid, C = 0;
    for (; C < NB; ++C) {
        const int nc = NB - C;
        if (bid < nc) break;
        bid -= nc;
    }
    if (C >= NB) return;
    const int ch = bid;
    const int Rb = C + ch;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const cx<R>* A = ws.A + b * ws.sA;
    const cx<R>* Ai = A + (int64_t)i * ws.lda;
    const int64_t lda = ws.lda;
    const int64_t gr = (int64_t)o + (int64_t)Rb * ZT + lane;
    const bool row_ok = gr < n;
    const int rowc = row_ok ? (int)gr : n - 1;
    const int64_t gcb = (int64_t)o + (int64_t)C * ZT;
    const i4_t rsrc = buffer_rsrc(A, (uint32_t)(BUF ? (int64_t)sizeof(cx<R>) * lda * n : 0));
    auto load_one = [&](int g, int cc) -> cx<R> {
        const int64_t gc = gcb + g * 8 + cc;
        const int64_t gcc = gc < n ? gc : (int64_t)n - 1;
        if constexpr (BUF) {
            const int soff = (int)(gcc * lda * (int64_t)sizeof(cx<R>));
            if constexpr (sizeof(R) == 8)
                return __builtin_bit_cast(cx<R>, raw_buffer_load_v4i32(rsrc, rowc * (int)sizeof(cx<R>), soff, 0));
            else
                return __builtin_bit_cast(cx<R>, raw_buffer_load_v2i32(rsrc, rowc * (int)sizeof(cx<R>), soff, 0));
        } else {
            return A[gcc * lda + rowc];
        }
    };
    // u first, then the wave's first column group (the second group's columns
    // are requested as the first group's registers free up).  Each wave keeps
    // its own copy of u in LDS, so the waves do not wait for each other before
    // the products.
    const int64_t gcu = gcb + lane;
    const cx<R> uC = Ai[gcu < n ? gcu : (int64_t)n - 1];
    cx<R> uR = Ai[row_ok ? gr : (int64_t)n - 1];
    const int g0 = 2 * w;
    cx<R> a[8];
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) a[cc] = load_one(g0, cc);
    sT[w][lane] = czero<cx<R>>();      // the other waves' columns add zero
    // (every wave stores its own copy: a store in one wave only would let the
    // compiler move the load of u behind the tile's)
    svC[w][lane] = csel(gcu > o && gcu < n, uC, czero<cx<R>>());
    if (!(row_ok && gr > o)) uR = czero<cx<R>>();
    wave_sync();

    __shared__ R sq[ZCH];
    const bool diag_tile = (Rb == C);
    cx<R> yd = czero<cx<R>>();
    // WHOLE: an entry of every row and column (most tiles): no masks
    auto group = [&](int g, auto next, auto whole) {
        constexpr bool NEXT = decltype(next)::value, WHOLE = decltype(whole)::value;
        const int64_t gc0 = gcb + g * 8;
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) {
            const int64_t gc = gc0 + cc;
            const bool ok = WHOLE || (row_ok && gc < n && (!diag_tile || gr >= gc));
            const bool diag = !WHOLE && diag_tile && (gr == gc);
            cx<R> x;
            x.x = ok ? a[cc].x : (R)0;
            x.y = (ok && !diag) ? a[cc].y : (R)0;
            yd = cfma(x, svC[w][g * 8 + cc], yd);
            sP[w][cc][lane] = csel(diag, czero<cx<R>>(), cmulc(x, uR));
            if constexpr (NEXT) a[cc] = load_one(g + 1, cc);
        }
        __builtin_amdgcn_wave_barrier();
        const int c = lane & 7, r0 = (lane >> 3) * 8;
        cx<R> cs = czero<cx<R>>();
#pragma unroll
        for (int r = 0; r < 8; ++r) cs = cadd(cs, sP[w][c][r0 + r]);
        cs = xor_add_v<8, R>(cs);
        cs = xor_add_v<16, R>(cs);
        cs = xor_add_v<32, R>(cs);
        if (lane < 8) sT[w][g * 8 + lane] = cs;
        __builtin_amdgcn_wave_barrier();
    };
    if (!diag_tile && o + (Rb + 1) * ZT <= n) {
        group(g0, std::true_type{}, std::true_type{});
        group(g0 + 1, std::false_type{}, std::true_type{});
    } else {
        group(g0, std::true_type{}, std::false_type{});
        group(g0 + 1, std::false_type{}, std::false_type{});
    }
    // the four waves' shares of the tile's direct part
    sP[w][0][lane] = yd;
    R qd = uR.x * yd.x + uR.y * yd.y;
    qd = dpp_wave_sum(qd);
    if (lane == 0) sq[w] = qd;
    __syncthreads();
    if (w == 0) {
        const cx<R> ys = cadd(cadd(sP[0][0][lane], sP[1][0][lane]), cadd(sP[2][0][lane], sP[3][0][lane]));
        ws.ypart[b * ws.s_ypart + ((int64_t)Rb * ws.NBmax + C) * ZT + lane] = ys;
        const cx<R> s = cadd(cadd(sT[0][lane], sT[1][lane]), cadd(sT[2][lane], sT[3][lane]));
        ws.ypartT[b * ws.s_ypartT + ((int64_t)C * ws.CHmax + ch) * ZT + lane] = s;
        R qt = svC[0][lane].x * s.x + svC[0][lane].y * s.y;
        qt = dpp_wave_sum(qt);
        if (lane == 0) ws.qpart[b * ws.s_qpart + lid] = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + qt;
    }
}

// ---------------------------------------------------------------------------
// Partial sums read as buffer loads: an offset at or beyond the buffer's size
// returns 0, so a term that does not exist is read past the end and added as 0, and
// every batch is loaded and added whole, without selects.

// A descriptor built from workgroup-uniform values, pinned to scalar
// registers (64-bit offset arithmetic can leave it in vector registers, and a
// buffer load from those would loop over the lanes' distinct descriptors).
__device__ inline i4_t uniform_rsrc(const void* base, uint32_t bytes)
{
    i4_t r = buffer_rsrc(base, bytes);
    r.x = __builtin_amdgcn_readfirstlane(r.x);
    r.y = __builtin_amdgcn_readfirstlane(r.y);
    r.z = __builtin_amdgcn_readfirstlane(r.z);
    r.w = __builtin_amdgcn_readfirstlane(r.w);
    return r;
}

template <typename R>
__device__ inline R bload_r(i4_t rsrc, int voff)
{
    if constexpr (sizeof(R) == 8)
        return __builtin_bit_cast(R, raw_buffer_load_v2i32(rsrc, voff, 0, 0));
    else
        return __builtin_bit_cast(R, raw_buffer_load_i32(rsrc, voff, 0, 0));
}

template <typename R>
__device__ inline cx<R> bload(i4_t rsrc, int voff)
{
    if constexpr (sizeof(R) == 8)
        return __builtin_bit_cast(cx<R>, raw_buffer_load_v4i32(rsrc, voff, 0, 0));
    else
        return __builtin_bit_cast(cx<R>, raw_buffer_load_v2i32(rsrc, voff, 0, 0));
}

// z at row o (row 0 of block 0), needed by every wave: the 1 + nc terms
// (block column 0, then the chunks of block row 0) spread over the lanes of
// the wave and summed by a fixed lane tree, so every wave holds the same
// bits.  z0_first is the lane's first term, requested with the kernel's first
// batch of loads; z0_rest adds the others (lane + 64, ...).
template <typename R>
__device__ inline cx<R> z0_first(const HetrdWs<R>& ws, int64_t b, int NB, int lane)
{
    const int T = 1 + nchunks_z(NB, 0, ws.zch);
    return lane == 0 ? ws.ypart[b * ws.s_ypart] : ws.ypartT[b * ws.s_ypartT + (int64_t)(lane < T ? lane - 1 : 0) * ZT];
}
template <typename R>
__device__ inline cx<R> z0_rest(const HetrdWs<R>& ws, int64_t b, int NB, int lane, cx<R> first)
{
    const cx<R>* yq = ws.ypartT + b * ws.s_ypartT;
    const int T = 1 + nchunks_z(NB, 0, ws.zch);
    cx<R> acc = csel(lane < T, first, czero<cx<R>>());
    for (int s = lane + 64; s < T; s += 64) acc = cadd(acc, yq[(int64_t)(s - 1) * ZT]);
    return acc;
}

// Column i: reflector, v and w, then (update_next) column o brought up to
// date.  A workgroup has the 64 rows of a row block, a wave 16 of them with
// four lanes per row: lane (r, k) takes every fourth panel column and every
// fourth partial sum of z, k first, and two lane exchanges add the four.  The
// waves share nothing, so the launch has no barrier; each forms the scalars of
// the column (reflector, W^H v, V^H v, row o) from the same loads.
//
// Bound by the instructions of a wave (few problems: one wave a SIMD, 64: all of
// them): one pass over the panel columns serves the corrections and the next
// column, and the panel products come finished from the launch before.  Against
// four waves sharing 64 rows by panel columns, with the panel products of the
// next column formed here in per-block partials: one problem at m = 1500 6.6 ->
// 5.6 us, 16 at m = 780 7.2 -> 5.7 us, 64 at m = 780 17 -> 12 us (and 0.4, 0.7, 1.9 us
// more in the launch of the product, which has the panel products now).
constexpr int PC = 4;           // panel columns of V and W per lane and batch

template <typename R, int ZB>
__global__ __launch_bounds__(256, 2) void hetrd_update(HetrdWs<R> ws, int i, int p, int update_next, int nch)
{
    // per wave: W^H v, V^H v, row o of W and of V over the panel's columns
    // (zero beyond j)
    __shared__ cx<R> sc[4][4][64];
    const int64_t b = blockIdx.y;
    const int n = ws.n, o = i + 1, m = n - o;
    const int NB = (m + ZT - 1) / ZT;
    const int Rb = blockIdx.x;
    const int j = i - p;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform (scalar) wave index
    const int k = lane >> 4, row = 16 * w + (lane & 15);
    const int64_t gr = (int64_t)o + (int64_t)Rb * ZT + row;
    if ((int64_t)o + (int64_t)Rb * ZT + 16 * w >= n) return;
    const int64_t grc = gr < n ? gr : (int64_t)n - 1;     // clamped row for unconditional loads
    cx<R>* A = ws.A + b * ws.sA;
    cx<R>* V = ws.V + b * ws.sV;
    cx<R>* W = ws.W + b * ws.sW;
    const cx<R> zero = czero<cx<R>>();

    // ---- every load that depends on nothing computed here, issued whole
    // before any of it is waited for (longer lists load the rest as they go):
    // what the scalars need first
    const cx<R> alpha = A[(int64_t)o + (int64_t)i * ws.lda];
    const R hoo = A[(int64_t)o + (int64_t)o * ws.lda].x;
    const R un = ws.unorm[b];
    const int lc = lane < j ? lane : 0;
    const cx<R> wd = ws.pdot[b * ws.s_pdot + lc];
    const cx<R> vd = ws.pdot[b * ws.s_pdot + ws.nb + lc];
    const cx<R> wo_l = W[(int64_t)o + (int64_t)lc * n];
    const cx<R> vo_l = V[(int64_t)o + (int64_t)(p + lc) * n];
    const cx<R> z0f = z0_first(ws, b, NB, lane);
    constexpr int QL = 4;
    const i4_t rq = uniform_rsrc(ws.qpart + b * ws.s_qpart, (uint32_t)((int64_t)nch * (int64_t)sizeof(R)));
    R qt[QL];
#pragma unroll
    for (int u = 0; u < QL; ++u) qt[u] = bload_r<R>(rq, (lane + 64 * u) * (int)sizeof(R));
    const cx<R> ai = A[grc + (int64_t)i * ws.lda];
    cx<R> h = A[grc + (int64_t)o * ws.lda];
    if (gr == o) h.y = 0;
    // the row's z terms: block columns C = k, k + 4, ... <= Rb and the chunks
    // k, k + 4, ... < nc of block column Rb
    const int nc = nchunks_z(NB, Rb, ws.zch);
    const i4_t rp = uniform_rsrc(ws.ypart + b * ws.s_ypart + (int64_t)Rb * ws.NBmax * ZT,
                                 (uint32_t)((Rb + 1) * ZT * (int)sizeof(cx<R>)));
    const i4_t rt = uniform_rsrc(ws.ypartT + b * ws.s_ypartT + (int64_t)Rb * ws.CHmax * ZT,
                                 (uint32_t)(nc * ZT * (int)sizeof(cx<R>)));
    constexpr int ZSTEP = 4 * ZT * (int)sizeof(cx<R>);
    const int zoff = (k * ZT + row) * (int)sizeof(cx<R>);
    cx<R> zp[ZB], zq[ZB];
#pragma unroll
    for (int t = 0; t < ZB; ++t) {
        zp[t] = bload<R>(rp, zoff + t * ZSTEP);
        zq[t] = bload<R>(rt, zoff + t * ZSTEP);
    }
    // this row of the panel columns k, k + 4, ... < j (0 beyond), in batches
    const i4_t rV = uniform_rsrc(V + (int64_t)p * n, (uint32_t)((int64_t)n * j * (int64_t)sizeof(cx<R>)));
    const i4_t rW = uniform_rsrc(W, (uint32_t)((int64_t)n * j * (int64_t)sizeof(cx<R>)));
    const int pstep = 4 * n * (int)sizeof(cx<R>);
    int poff = (k * n + (int)grc) * (int)sizeof(cx<R>);
    cx<R> pv[PC], pw[PC];
    auto load_panel = [&]() {
#pragma unroll
        for (int q = 0; q < PC; ++q) {
            pv[q] = bload<R>(rV, poff);
            pw[q] = bload<R>(rW, poff);
            poff += pstep;
        }
    };
    load_panel();

    // ---- scalars of the column, the same bits in every wave: reflector, panel
    // products with v (lane = panel column), y_o, alpha2 and w_o
    cx<R> tau, scale;
    R beta;
    reflector_core(alpha, un, tau, scale, beta);
    cx<R> wvl = zero, vvl = zero, wol = zero, vol = zero;
    if (lane < j) {
        wvl = cfma(scale, wd, cconj(wo_l));
        vvl = cfma(scale, vd, cconj(vo_l));
        wol = wo_l;
        vol = vo_l;
    }
    sc[w][0][lane] = wvl;
    sc[w][1][lane] = vvl;
    sc[w][2][lane] = cconj(wol);
    sc[w][3][lane] = cconj(vol);
    R qq = 0;
    for (int c0 = lane;; c0 += 64 * QL) {
#pragma unroll
        for (int u = 0; u < QL; ++u) qq += qt[u];
        if (c0 - lane + 64 * QL >= nch) break;
#pragma unroll
        for (int u = 0; u < QL; ++u) qt[u] = bload_r<R>(rq, (c0 + 64 * (QL + u)) * (int)sizeof(R));
    }
    cx<R> z0 = z0_rest(ws, b, NB, lane, z0f);
    cx<R> co = cfma(vol, wvl, cmul(wol, vvl));
    R cross = vvl.x * wvl.x + vvl.y * wvl.y;   // Re(conj(V^H v) W^H v)
    co.x = dpp_wave_sum(co.x);
    co.y = dpp_wave_sum(co.y);
    cross = dpp_wave_sum(cross);
    z0.x = dpp_wave_sum(z0.x);
    z0.y = dpp_wave_sum(z0.y);
    qq = dpp_wave_sum(qq);
    const cx<R> sz = cmul(scale, z0);
    const R vav = hoo + (R)2 * sz.x + (scale.x * scale.x + scale.y * scale.y) * qq;
    const R a2 = (R)-0.5 * (tau.x * tau.x + tau.y * tau.y) * (vav - (R)2 * cross);
    const cx<R> wo = cadd(cmul(tau, csub(cadd(mk<R>(hoo, 0), sz), co)), mk<R>(a2, 0));
    wave_sync();

    // ---- the lane's shares of z, of the corrections V (W^H v) + W (V^H v) and
    // of the next column's
    cx<R> z = zero, acc = zero;
#pragma unroll
    for (int t = 0; t < ZB; ++t) z = cadd(z, cadd(zp[t], zq[t]));
    const int tmax = max(Rb + 1, nc);
    for (int t = 4 * ZB; t < tmax; t += 4 * ZB) {
        const int off = zoff + t * (ZSTEP / 4);
#pragma unroll
        for (int u = 0; u < ZB; ++u) {
            zp[u] = bload<R>(rp, off + u * ZSTEP);
            zq[u] = bload<R>(rt, off + u * ZSTEP);
        }
#pragma unroll
        for (int u = 0; u < ZB; ++u) z = cadd(z, cadd(zp[u], zq[u]));
    }
    z = cmul(scale, z);
#pragma unroll 1
    for (int c = k; c - k < j; c += 4 * PC) {
#pragma unroll
        for (int q = 0; q < PC; ++q) {
            const int jj = min(c + 4 * q, 63);
            z = csub(z, cmul(pv[q], sc[w][0][jj]));
            z = csub(z, cmul(pw[q], sc[w][1][jj]));
            acc = cfma(pv[q], sc[w][2][jj], acc);
            acc = cfma(pw[q], sc[w][3][jj], acc);
        }
        load_panel();
    }
    z = xor_add_v<16, R>(z);
    z = xor_add_v<32, R>(z);
    acc = xor_add_v<16, R>(acc);
    acc = xor_add_v<32, R>(acc);

    const cx<R> myv = csel(gr == o, mk<R>(1, 0), cmul(ai, scale));
    cx<R> myw = cfma(mk<R>(a2, 0), myv, cmul(tau, cadd(h, z)));
    myw = csel(gr == o, wo, myw);
    if (gr < n) {
        if (k == 0) V[gr + (int64_t)i * n] = myv;
        if (k == 1) W[gr + (int64_t)j * n] = myw;
        if (k == 2 && update_next) {
            const cx<R> a = csub(csub(csub(h, acc), cmul(myv, cconj(wo))), myw);
            if (gr == o)
                // the diagonal goes to d only: A(o, o) is read as it stood by
                // every wave of this launch and is not needed afterwards
                ws.d[b * n + o] = a.x;
            else
                A[gr + (int64_t)o * ws.lda] = a;
        }
        if (k == 3 && gr == o) {
            ws.e[b * n + i] = beta;
            ws.tau[b * n + i] = tau;
        }
    }
}

}  // namespace

namespace {
// reductions of order 1: T is the matrix
template <typename R>
__global__ __launch_bounds__(256) void hetrd_order1(HetrdWs<R> ws, int64_t nk)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b < nk) ws.d[b] = ws.A[b * ws.sA].x;
}
}  // namespace

template <typename R>
hipError_t hetrd(hipStream_t st, const HetrdWs<R>& ws0, int64_t nk)
{
    const int n = ws0.n, nb = ws0.nb;
    if (n < 1 || nk < 1) return hipSuccess;
    HetrdWs<R> ws = ws0;
    // Buffer offsets are 32-bit: a matrix (ld x n) of 2 GiB or more is read
    // with plain global loads instead.
    const bool buf = (double)sizeof(cx<R>) * (double)ws.lda * (double)n < 2147483648.0;
    const int cus = ws.groups && n > HETRD_RES_M ? stream_compute_units(st) : 0;
    const int limit = hetrd_res_order(n, nb, nk, ws.groups, cus);
    for (int p = 0; p <= n - 1; p += nb) {
        if (n - p <= limit && p < n - 1) {
            const hipError_t e = hetrd_res<R>(st, ws, p, nk, cus);
            if (e != hipSuccess) return e;
            break;
        }
        if (p == n - 1)      // (n = 1)
            hipLaunchKernelGGL(hetrd_order1<R>, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, st, ws, nk);
        const int iend = min(p + nb, n - 1);
        for (int i = p; i < iend; ++i) {
            const int o = i + 1, m = n - o;
            const int NB = (m + ZT - 1) / ZT;
            // The one-tile form when the four-tile form would launch fewer
            // workgroups than ws.slots1 (default three per CU: its chains of
            // loads are a quarter as long); the product and the update of a column agree on the
            // chunk layout of the partial sums through ws.zch and ws.CHmax
            // (the buffers hold the one-tile form's NBmax chunks per column).
            int nch4 = 0;
            for (int C = 0; C < NB; ++C) nch4 += nchunks(NB, C);
            const int64_t slots1 = ws0.slots1 > 0 ? ws0.slots1 : 3 * 256;
            ws.zch = (int64_t)nch4 * nk < slots1 ? 1 : ZCH;
            ws.CHmax = ws.zch == 1 ? ws0.NBmax : (ws0.NBmax + ZCH - 1) / ZCH;
            const int nch = ws.zch == 1 ? NB * (NB + 1) / 2 : nch4;
            // Consecutive columns traverse their tiles in opposite orders (odd
            // columns from the last k-point's last chunk back), so each launch
            // starts on the tiles its predecessor read last, which the 256 MB
            // memory-side cache still holds once the lower triangles of all
            // k-points exceed it (n = 2000 x 16: 9% faster at m = 1500..1750).
            const int rev = i & 1;
            const ProfLaunch pl = prof_launch_begin(PH_HEMV, st);
            const int units = dot_units(i - p);
            const dim3 gz((unsigned)(units + nch), (unsigned)nk);
            if (ws.zch == 1) {
                if (buf)
                    launch_timed(pl, hetrd_zhemv_tile<R, true>, gz, dim3(256), st, ws, i, p, units, rev);
                else
                    launch_timed(pl, hetrd_zhemv_tile<R, false>, gz, dim3(256), st, ws, i, p, units, rev);
            } else {
                if (buf)
                    launch_timed(pl, hetrd_zhemv<R, true>, gz, dim3(256), st, ws, i, p, units, rev);
                else
                    launch_timed(pl, hetrd_zhemv<R, false>, gz, dim3(256), st, ws, i, p, units, rev);
            }
            prof_launch_end(PH_HEMV, st, pl,
                            (double)sizeof(cx<R>) * 0.5 * (double)m * (double)(m + 1) * (double)nk, 0.0);
            const int upd = (i + 1 < p + nb) && (o <= n - 1);
            // up to 16 row blocks a wave's share of the partial sums is four
            // terms of each list at most: half the loads of the wider form
            // (64 reductions of order 1024: 50.8 ms against 51.5)
            hipLaunchKernelGGL((NB <= 16 ? hetrd_update<R, 4> : hetrd_update<R, 8>), dim3((unsigned)NB, (unsigned)nk),
                               dim3(256), 0, st, ws, i, p, upd, nch);
        }
        if (p + nb <= n - 1) {
            const int t0 = p + nb;
            const int64_t m2 = n - t0;
            hipError_t e = cher2k_lower<R>(st, m2, nb, ws.V + (int64_t)t0 + (int64_t)p * n, n, ws.sV,
                                           ws.W + t0, n, ws.sW, ws.A + (int64_t)t0 + (int64_t)t0 * ws.lda,
                                           ws.lda, ws.sA, nk);
            if (e != hipSuccess) return e;
        }
    }
    return hipGetLastError();
}

template hipError_t hetrd<double>(hipStream_t, const HetrdWs<double>&, int64_t);
template hipError_t hetrd<float>(hipStream_t, const HetrdWs<float>&, int64_t);

}  // namespace kgev
