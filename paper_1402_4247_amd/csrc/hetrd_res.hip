// The on-chip Householder reduction (Section III, Procedures 1-6 of Eigen_HH,
// arXiv:1402.4247, unblocked): one launch reduces a trailing matrix that stays
// in registers from the first column to the last.
//
// The trailing matrix (order M, full storage: both triangles) is held in 16 x
// 16 tiles laid out as FP64 (FP32) MFMA accumulators, in the registers of one
// workgroup of eight waves; wave w owns the tile rows w, w + 8, ... .
// Column c is eliminated in two workgroup barriers:
//   A  the pending rank-2 update a_rs -= v_r conj(w_s) + w_r conj(v_s) of the
//      previous column (Procedure 6).  Its inner dimension as a real product
//      is exactly four, (vr vi wr wi) . (wr wi vr vi), so one MFMA per tile
//      forms the real parts and one the imaginary parts with no padding and
//      three LDS reads per lane.  Then Procedure 4 with the column x as it
//      stands below its sub-diagonal: z_s = sum_r conj(a_rs) x_r (a Hermitian
//      matrix's column sums, which a lane accumulates over its own rows, so
//      the cross-lane part is two steps), one partial sum per wave to LDS with
//      the wave's share of q = Re(x^H z); row c + 1 to LDS.  The first wave,
//      whose rows finish first, forms the reflector (Procedure 2) meanwhile.
//   B  one thread per row: z summed over the waves, v = (1, scale x),
//      y = tau (A(:, c+1) + scale z) (A v by linearity), w = y - (tau/2)(y^H v) v
//      with y^H v from q and z_{c+1} (Procedures 3, 5), and the next column
//      x' = A(:, c+1) - v conj(w_{c+1}) - w with its partial norms.
// Bound by the FP64 arithmetic of one compute unit in A (12 multiply-adds an
// entry, about half of a column's time at order 128; FP64 MFMA and vector
// multiply-adds measured no overlap) and by the latency of B's chain.
// Order 128: 249 us, against 439 us for the previous form, which kept the lower
// triangle in LDS, moved every entry through it in both products and took
// five barriers a column.  Four threads per row in B (every wave taking part)
// measured 269 us, __syncthreads() for both barriers (which waits for the
// stores of v) with run-time tile bounds 359 us.
// Sums are taken in a fixed order: results are bitwise reproducible.
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "lanes.hpp"
#include "kernels.hpp"
#include "reflector.hpp"

namespace kgev {

namespace {

constexpr int RT_T = 512;           // threads of a workgroup
constexpr int RT_W = RT_T / WAVE;   // waves: tile row R belongs to wave R mod RT_W

template <typename R> using acc4 = typename Mfma<R>::acc_t;

// row r of an accumulator register's four (lane group lk holds row
// Mfma<R>::row(lk, r)); the inverse: lane group and register of a row
template <typename R> __device__ inline int row_lk(int row) { return sizeof(R) == 8 ? (row & 3) : (row >> 2); }
template <typename R> __device__ inline int row_r(int row) { return sizeof(R) == 8 ? (row >> 2) : (row & 3); }

// Workgroup barrier that waits for this wave's LDS operations only:
// __syncthreads() also waits for its global stores (v, d, e, tau), which
// nothing in the kernel reads back.
__device__ inline void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <typename Fn, int... K> __device__ __attribute__((always_inline)) inline void for_tiles(Fn& f, std::integer_sequence<int, K...>)
{
    (f(std::integral_constant<int, K>{}), ...);
}

// RT tile rows per wave, KC tile columns: the trailing order is at most
// min(RT * RT_W, KC) * 16.
template <typename R, int RT, int KC>
__global__ __launch_bounds__(RT_T) void hetrd_resident(HetrdWs<R> ws, int i0)
{
    using M_ = Mfma<R>;
    constexpr int NT = RT * RT_W < KC ? RT * RT_W : KC;     // tile rows and columns at most
    constexpr int MP = NT * 16;                             // padded order
    static_assert(MP <= RT_T, "one thread per row");
    constexpr int FS = MP + 16;     // stride of the four operand rows, in 16-bank steps
    __shared__ R F[4][FS];          // Re v, Im v, Re w, Im w of the pending update
    __shared__ cx<R> x[MP];         // the column below its sub-diagonal, zero above
    __shared__ cx<R> zp[RT_W][KC * 16];   // per-wave partial sums of z
    __shared__ cx<R> hrow[KC * 16];       // A(:, c+1)
    __shared__ R red[RT_W];               // partial squared norms
    __shared__ R sq[RT_W];                // partial sums of q
    __shared__ cx<R> salpha;              // x_{c+1}
    __shared__ cx<R> sref[2];             // tau, scale

    const int64_t b = blockIdx.x;
    const int n = ws.n, M = n - i0;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const cx<R>* A = ws.A + b * ws.sA + (int64_t)i0 + (int64_t)i0 * ws.lda;
    const int64_t lda = ws.lda;
    cx<R>* V = ws.V + b * ws.sV;
    const cx<R> zero = czero<cx<R>>();

    // the tiles, from the lower triangle
    acc4<R> tr[RT][KC], ti[RT][KC];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int k = 0; k < KC; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = (w + RT_W * i) * 16 + M_::row(lk, r), col = k * 16 + li;
                cx<R> a = zero;
                if (row < M && col < M) {
                    const bool low = row >= col;
                    a = A[low ? (int64_t)row + (int64_t)col * lda : (int64_t)col + (int64_t)row * lda];
                    a.y = row == col ? (R)0 : (low ? a.y : -a.y);
                }
                tr[i][k][r] = a.x;
                ti[i][k][r] = a.y;
            }
    // column 0, and no pending update
    R nrm = 0;
    for (int e = tid; e < 4 * FS; e += RT_T) (&F[0][0])[e] = (R)0;
    if (tid < MP) {
        const cx<R> a = csel(tid < M, A[tid < M ? tid : 0], zero);
        const cx<R> a2 = csel(tid >= 2, a, zero);
        x[tid] = a2;
        nrm = a2.x * a2.x + a2.y * a2.y;
        if (tid == 0) ws.d[b * n + i0] = a.x;
        if (tid == 1) salpha = a;
    }
    nrm = dpp_wave_sum(nrm);
    if (lane == 0) red[w] = nrm;
    lds_barrier();

    auto zsum = [&](int s) {
        return cadd(cadd(cadd(zp[0][s], zp[1][s]), cadd(zp[2][s], zp[3][s])),
                    cadd(cadd(zp[4][s], zp[5][s]), cadd(zp[6][s], zp[7][s])));
    };
    int c = 0;
    // the columns c with c + 1 in tile row k1 (a constant, so the tiles of the
    // finished columns drop out at compile time)
    auto columns = [&](auto k1c) __attribute__((always_inline)) {
    constexpr int k1 = decltype(k1c)::value;
#pragma unroll 1
    for (; c + 1 < M && c + 1 < (k1 + 1) * 16; ++c) {
        const int c1 = c + 1, i = i0 + c;
        // ---- A
        R opB[KC];
#pragma unroll
        for (int k = k1; k < KC; ++k) opB[k] = F[lk ^ 2][k * 16 + li];
        cx<R> za[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) za[k] = zero;
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            const int Rt = w + RT_W * q;
            if (Rt >= k1 && Rt < NT) {
                const R are = -F[lk][Rt * 16 + li], aim = -F[lk ^ 1][Rt * 16 + li];
                cx<R> xr[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) xr[r] = x[Rt * 16 + M_::row(lk, r)];
                // tile k is updated on the matrix cores while tile k - 1,
                // updated before it, is multiplied
#pragma unroll
                for (int k = k1; k <= KC; ++k) {
                    if (k < KC) {
                        tr[q][k] = M_::mma(are, opB[k], tr[q][k]);
                        ti[q][k] = M_::mma(aim, (lk & 1) ? -opB[k] : opB[k], ti[q][k]);
                    }
                    if (k > k1) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            za[k - 1] = cfmac(mk<R>(tr[q][k - 1][r], ti[q][k - 1][r]), xr[r], za[k - 1]);
                    }
                }
                if (Rt == k1) {
                    // this wave holds row c + 1: A(:, c+1) is its conjugate
                    const int rr = row_r<R>(c1 & 15);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r == rr && lk == row_lk<R>(c1 & 15)) {
#pragma unroll
                            for (int k = k1; k < KC; ++k) hrow[k * 16 + li] = mk<R>(tr[q][k][r], -ti[q][k][r]);
                        }
                }
            }
        }
        if (w == 0) {
            // Procedure 2, by the wave whose tile rows finish first
            const R sig2 = ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
            cx<R> tau, scale;
            R beta;
            reflector_core(salpha, sig2, tau, scale, beta);
            if (lane == 0) {
                sref[0] = tau;
                sref[1] = scale;
                ws.e[b * n + i] = beta;
                ws.tau[b * n + i] = tau;
            }
        }
        // over the four lane groups: halve the set of columns across lane bit
        // 5, then bit 4, so that lane group lk ends with a quarter of them
        static_assert(KC % 4 == 0, "four lane groups");
        R qs = 0;
#pragma unroll
        for (int k = 0; k < KC / 2; ++k) {
            swap_across<32>(za[k].x, za[k + KC / 2].x);
            swap_across<32>(za[k].y, za[k + KC / 2].y);
            za[k] = cadd(za[k], za[k + KC / 2]);
        }
#pragma unroll
        for (int k = 0; k < KC / 4; ++k) {
            swap_across<16>(za[k].x, za[k + KC / 4].x);
            swap_across<16>(za[k].y, za[k + KC / 4].y);
            za[k] = cadd(za[k], za[k + KC / 4]);
            const int kk = k + ((lk & 2) ? KC / 2 : 0) + ((lk & 1) ? KC / 4 : 0);
            zp[w][kk * 16 + li] = za[k];
            const cx<R> xc = x[kk * 16 + li];
            qs = fma(xc.x, za[k].x, fma(xc.y, za[k].y, qs));
        }
        qs = dpp_wave_sum(qs);
        if (lane == 0) sq[w] = qs;
        lds_barrier();
        // ---- B
        nrm = 0;
        if (w * WAVE < MP) {
            const int s = tid;
            const bool live = s >= c1 && s < M;
            const cx<R> tau = sref[0], scale = sref[1];
            const cx<R> z = zsum(s), z1 = zsum(c1);
            const R hoo = hrow[c1].x;
            cx<R> h = hrow[s];
            const cx<R> xs = x[s];
            const R qq = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + ((sq[4] + sq[5]) + (sq[6] + sq[7]));
            const cx<R> sz = cmul(scale, z1);
            const R vav = hoo + (R)2 * sz.x + (scale.x * scale.x + scale.y * scale.y) * qq;
            const R a2 = (R)-0.5 * (tau.x * tau.x + tau.y * tau.y) * vav;
            const cx<R> w1 = cadd(cmul(tau, cadd(mk<R>(hoo, 0), sz)), mk<R>(a2, 0));
            cx<R> vs = zero, wv = zero, xn = zero;
            if (live) {
                vs = csel(s == c1, mk<R>(1, 0), cmul(scale, xs));
                wv = csel(s == c1, w1, cfma(tau, cfma(scale, z, h), cscale(vs, a2)));
                V[(int64_t)(i0 + s) + (int64_t)i * n] = vs;
                // x'_s = h_s - (v_s conj(w_{c+1}) + w_s)
                xn = csub(h, cadd(cmulc(w1, vs), wv));
                if (s == c1) ws.d[b * n + i + 1] = xn.x;
                if (s == c1 + 1) salpha = xn;
                xn = csel(s >= c1 + 2, xn, zero);
                nrm = xn.x * xn.x + xn.y * xn.y;
            }
            F[0][s] = vs.x;
            F[1][s] = vs.y;
            F[2][s] = wv.x;
            F[3][s] = wv.y;
            x[s] = xn;
        }
        nrm = dpp_wave_sum(nrm);
        if (lane == 0) red[w] = nrm;
        lds_barrier();
    }
    };
    for_tiles(columns, std::make_integer_sequence<int, NT>{});
}

}  // namespace

template <typename R>
hipError_t hetrd_res(hipStream_t st, const HetrdWs<R>& ws, int i0, int64_t nk)
{
    if (ws.n - i0 <= 64)
        hipLaunchKernelGGL((hetrd_resident<R, 1, 4>), dim3((unsigned)nk), dim3(RT_T), 0, st, ws, i0);
    else
        hipLaunchKernelGGL((hetrd_resident<R, 1, 8>), dim3((unsigned)nk), dim3(RT_T), 0, st, ws, i0);
    return hipGetLastError();
}
template hipError_t hetrd_res<double>(hipStream_t, const HetrdWs<double>&, int, int64_t);
template hipError_t hetrd_res<float>(hipStream_t, const HetrdWs<float>&, int, int64_t);

}  // namespace kgev
