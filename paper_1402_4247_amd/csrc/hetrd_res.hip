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
// Sums are taken in a fixed order, here and in the groups below, also where a
// group is given up: results are bitwise reproducible.
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "lanes.hpp"
#include "kernels.hpp"
#include "reflector.hpp"

namespace kgev {

namespace {

// how long a workgroup of a group waits for the others to start, in ticks of
// the 100 MHz wall clock: 200 ms
constexpr int64_t GROUP_WAIT_TICKS = 20000000;
// how often a member looks again for the others' columns before it gives up
// (a constant: as an argument it cost 45 to 70 ns a column)
constexpr int POLLS_MAX = 1 << 21;
// set by tests: 0 gives every group up before it starts
thread_local int64_t tl_group_wait_ticks = GROUP_WAIT_TICKS;
// set by tests: a launch lacks its last member
thread_local bool tl_group_lacks_one = false;

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

// Sum of KC values per lane over the four lane groups.  Where the count halves,
// the set is halved across lane bit 5, then bit 4 (each lane group ends with
// its share); otherwise every group adds and one of them passes the sum on.
// f(k, sum) is called by the lanes that hold sum k.
template <typename R, int KC, typename Fn>
__device__ __attribute__((always_inline)) inline void sum_lane_groups(cx<R> (&v)[KC], int lk, Fn f)
{
    constexpr int K1 = KC % 2 == 0 ? KC / 2 : KC, K2 = K1 % 2 == 0 ? K1 / 2 : K1;
#pragma unroll
    for (int k = 0; k < K1; ++k) {
        if constexpr (K1 < KC) {
            swap_across<32>(v[k].x, v[k + K1].x);
            swap_across<32>(v[k].y, v[k + K1].y);
            v[k] = cadd(v[k], v[k + K1]);
        } else {
            v[k].x = xor_sum<32>(v[k].x);
            v[k].y = xor_sum<32>(v[k].y);
        }
    }
#pragma unroll
    for (int k = 0; k < K2; ++k) {
        if constexpr (K2 < K1) {
            swap_across<16>(v[k].x, v[k + K2].x);
            swap_across<16>(v[k].y, v[k + K2].y);
            v[k] = cadd(v[k], v[k + K2]);
        } else {
            v[k].x = xor_sum<16>(v[k].x);
            v[k].y = xor_sum<16>(v[k].y);
        }
    }
    const bool holds = (K1 < KC || !(lk & 2)) && (K2 < K1 || !(lk & 1));
    const int k0 = (K1 < KC && (lk & 2) ? K1 : 0) + (K2 < K1 && (lk & 1) ? K2 : 0);
    if (holds) {
#pragma unroll
        for (int k = 0; k < K2; ++k) f(k0 + k, v[k]);
    }
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
        R qs = 0;
        sum_lane_groups<R, KC>(za, lk, [&](int k, cx<R> v) {
            zp[w][k * 16 + li] = v;
            const cx<R> xc = x[k * 16 + li];
            qs = fma(xc.x, v.x, fma(xc.y, v.y, qs));
        });
        qs = dpp_wave_sum(qs);
        if (lane == 0) sq[w] = qs;
        lds_barrier();
        // ---- B
        nrm = 0;
        if (MP % WAVE == 0 ? w * WAVE < MP : tid < MP) {
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


// ---------------------------------------------------------------------------
// The same reduction by a group of G workgroups per problem, for trailing
// orders one workgroup's registers do not hold.  Member g owns the tile columns
// g, g + G, ... (KC of them at most) over all tile rows; x, v and w are kept
// by every member.  A member's column sums are complete, so one exchange per
// column joins the group: each member publishes z_s and A(s, c+1) of its
// columns, and every member reads all of them (each line once per member: with
// every wave also reading z_{c+1} and the members' shares of q, 3.0 us a column
// at order 200 instead of 2.6).
//
// The exchange is the data itself: a slot that holds SENTINEL (a NaN no
// arithmetic produces; a value with its bits is published as another NaN) has
// not been published.  Slots form a ring of three: whoever has read every
// member's column c knows that every member has read column c - 1, so an
// owner clears its slots of column c - 1 then, and publishes column c + 1 only
// after the clears have reached memory; a reader of column c + 2 (the same
// slots) has read that owner's column c + 1 first, so it cannot see column
// c - 1's values.  A member publishes as long as it has unfinished columns and
// leaves, without reading, once it has none: whoever still reads still
// publishes, so the others' knowledge covers it.
//
// The members of a group must run together.  Workgroups take their (problem,
// member) from a counter when they start, so groups fill in order and at most
// one group of a launch is partly placed; a member waits for the others to
// start for a bounded time, after which the group is given up (the last one to
// arrive and the one that gives up decide by an atomic on the same word) and
// hetrd_memory reduces that problem instead, to the same bits.  Once all have
// started, every wait ends; the poll is bounded all the same.  A group has at
// most a quarter of the compute units that its stream may use (64 of the 256 of
// a whole GPU; a partition of one or a stream with a mask has fewer), so four
// launches on different streams (the hardware queues of a process by default)
// cannot hold each other's partly placed groups.  More queues or several
// processes can; their groups are given up after the wait.
//
// Bound by the latency of a column: the exchange (a store and a load through
// the coherent level, 0.5-0.7 us between any two compute units), three
// workgroup barriers and phase B's chain: 2.3 us a column at order 200, 2.75 us
// at 512, 3.8 us at 1024 (one problem), against 11-13 us for the two launches
// of a blocked column.
constexpr uint64_t SENTINEL = 0xFFF4DEADFFF4BEEFull;   // two NaNs as well for a pair of floats
constexpr uint32_t GIVEN_UP = 0x80000000u;
constexpr int GROUP_MAX = 64;             // members of a group at most (the shapes' largest)
constexpr int GROUP_MIN = 160;            // orders up to this stay with panels and one workgroup

template <typename T> __device__ __attribute__((always_inline)) inline T load_agent(const T* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __attribute__((always_inline)) inline void store_agent(T* p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The exchange area of one problem, in the panel buffer W (which the blocked
// columns before have finished with; 64 n complex values a problem): a header
// of two 64-bit words {members started | GIVEN_UP, next ticket (problem 0
// only)}, then three slots of {z (MP complex), A(:, c+1) (MP complex)}.
template <typename R> struct Exchange {
    static constexpr int WPC = 2 * sizeof(R) / 8;      // 64-bit words per complex value
    uint64_t* base;
    int MP;
    __device__ __host__ Exchange(const HetrdWs<R>& ws, int64_t b, int M)
        : base(reinterpret_cast<uint64_t*>(ws.W + b * 64 * (int64_t)ws.n)), MP((M + 15) & ~15) {}
    __device__ uint32_t* started() const { return reinterpret_cast<uint32_t*>(base); }
    __device__ uint32_t* ticket() const { return reinterpret_cast<uint32_t*>(base + 1); }
    __device__ __host__ int slot_words() const { return 2 * WPC * MP; }
    __device__ uint64_t* slot(int q) const { return base + 2 + (int64_t)q * slot_words(); }
    // word c of value s of list l (0: z, 1: A(:, c+1)) in a slot
    __device__ int at(int l, int s, int c) const { return (l * WPC + c) * MP + s; }
};

__device__ inline uint64_t word_of(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    return u == SENTINEL ? 0x7FF8000000000000ull : u;
}
__device__ inline uint64_t word_of(float lo, float hi)
{
    const uint64_t u = (uint64_t)__float_as_uint(lo) | ((uint64_t)__float_as_uint(hi) << 32);
    return u == SENTINEL ? 0x7FC000007FC00000ull : u;
}

// values from published words
template <typename R> __device__ inline cx<R> value_of(const uint64_t* u)
{
    if constexpr (sizeof(R) == 8)
        return mk<R>(__longlong_as_double((long long)u[0]), __longlong_as_double((long long)u[1]));
    else
        return mk<R>(__uint_as_float((uint32_t)u[0]), __uint_as_float((uint32_t)(u[0] >> 32)));
}

template <typename R>
__global__ __launch_bounds__(256) void k_exchange_init(HetrdWs<R> ws, int M, uint32_t started, uint32_t started_last)
{
    const Exchange<R> ex(ws, blockIdx.y, M);
    const int words = 2 + 3 * ex.slot_words();
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q < words) ex.base[q] = q > 1 ? SENTINEL : q == 1 ? 0 : blockIdx.y + 1 < gridDim.y ? started : started_last;
}

template <typename R, int RT, int KC>
__global__ __launch_bounds__(RT_T) void hetrd_group(HetrdWs<R> ws, int i0, int G, int64_t wait_ticks)
{
    using M_ = Mfma<R>;
    using Ex = Exchange<R>;
    constexpr int MPX = RT * RT_W * 16;          // largest order
    constexpr int SP = (MPX + RT_T - 1) / RT_T;  // rows per thread
    constexpr int FS = MPX + 16;
    constexpr int WPC = Ex::WPC;
    static_assert(KC * 16 <= WAVE, "a lane of the first wave per owned column");
    __shared__ R F[4][FS];
    __shared__ cx<R> x[MPX];
    __shared__ cx<R> zp[RT_W][KC * 16];
    __shared__ cx<R> hrow[KC * 16];
    __shared__ R red[RT_W], sq[RT_W];
    __shared__ cx<R> salpha, sref[2], sz1;   // x_{c+1}; tau, scale; z_{c+1}
    __shared__ R shoo;                       // A(c+1, c+1)
    __shared__ int sgo, sdead;
    __shared__ uint32_t sticket;

    const int n = ws.n, M = n - i0;
    const int nt = (M + 15) >> 4;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const cx<R> zero = czero<cx<R>>();

    // which problem and member, and whether all members have started
    if (tid == 0) {
        sticket = __hip_atomic_fetch_add(Ex(ws, 0, M).ticket(), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sdead = 0;
        uint32_t* started = Ex(ws, (int64_t)(sticket / (uint32_t)G), M).started();
        uint32_t seen = 1u + __hip_atomic_fetch_add(started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int64_t t0 = wall_clock64();
        while (seen < (uint32_t)G) {
            if ((int64_t)wall_clock64() - t0 >= wait_ticks) {
                // gives the group up unless the last member arrives first
                uint32_t expect = seen;
                if (__hip_atomic_compare_exchange_strong(started, &expect, seen | GIVEN_UP, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    expect = seen | GIVEN_UP;
                seen = expect;
            } else {
                __builtin_amdgcn_s_sleep(8);
                seen = load_agent(started);
            }
        }
        sgo = seen == (uint32_t)G;      // a group given up has GIVEN_UP set
    }
    __syncthreads();
    if (!sgo) return;
    const int64_t b = __builtin_amdgcn_readfirstlane((int)(sticket / (uint32_t)G));
    const int g = __builtin_amdgcn_readfirstlane((int)(sticket % (uint32_t)G));
    const Ex ex(ws, b, M);
    const cx<R>* A = ws.A + b * ws.sA + (int64_t)i0 + (int64_t)i0 * ws.lda;
    const int64_t lda = ws.lda;
    cx<R>* V = ws.V + b * ws.sV;

    acc4<R> tr[RT][KC], ti[RT][KC];
#pragma unroll
    for (int q = 0; q < RT; ++q)
#pragma unroll
        for (int k = 0; k < KC; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = (w + RT_W * q) * 16 + M_::row(lk, r), col = (g + G * k) * 16 + li;
                cx<R> a = zero;
                if (row < M && col < M) {
                    const bool low = row >= col;
                    a = A[low ? (int64_t)row + (int64_t)col * lda : (int64_t)col + (int64_t)row * lda];
                    a.y = row == col ? (R)0 : (low ? a.y : -a.y);
                }
                tr[q][k][r] = a.x;
                ti[q][k][r] = a.y;
            }
    R nrm = 0;
    for (int e = tid; e < 4 * FS; e += RT_T) (&F[0][0])[e] = (R)0;
#pragma unroll
    for (int u = 0; u < SP; ++u) {
        const int s = tid + RT_T * u;
        const cx<R> a = csel(s < M, A[s < M ? s : 0], zero);
        const cx<R> a2 = csel(s >= 2, a, zero);
        if (s < MPX) x[s] = a2;
        nrm += a2.x * a2.x + a2.y * a2.y;
        if (s == 0 && g == 0) ws.d[b * n + i0] = a.x;
        if (s == 1) salpha = a;
    }
    nrm = dpp_wave_sum(nrm);
    if (lane == 0) red[w] = nrm;
    lds_barrier();

    // wave 0 publishes: lane's local column, its share of it, and the column
    constexpr int PARTS = KC == 1 ? (WPC == 2 ? 4 : 2) : KC == 2 ? 2 : 1;
    const int pcol = lane / PARTS, part = lane % PARTS;
    const int own = pcol < KC * 16 ? (g + G * (pcol >> 4)) * 16 + (pcol & 15) : M;
    const int last = g + G * ((nt - 1 - g) / G);          // this member's last tile column
    int ring = 0;                       // c mod 3
    for (int c = 0; c + 1 < M; ++c) {
        const int c1 = c + 1, i = i0 + c, k1 = c1 >> 4;
        uint64_t* const cur = ex.slot(ring);
        uint64_t* const old = ex.slot(ring == 0 ? 2 : ring - 1);     // column c - 1's, c + 2's next
        // ---- A: pending update and column sums of the live tiles (the
        // operands of the next tile row are requested ahead, whether it is
        // live or not: no wait inside the branches)
        R opB[KC];
        cx<R> za[KC];
        bool livek[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int C = g + G * k;
            opB[k] = F[lk ^ 2][(C < nt ? C : 0) * 16 + li];
            livek[k] = C >= k1 && C < nt;
            za[k] = zero;
        }
        constexpr bool AHEAD = RT * KC < 8;      // (the registers of more tiles leave no room)
        R are = AHEAD ? F[lk][w * 16 + li] : (R)0, aim = AHEAD ? F[lk ^ 1][w * 16 + li] : (R)0;
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            const int Rt = w + RT_W * q;
            if (!AHEAD) {
                are = F[lk][Rt * 16 + li];
                aim = F[lk ^ 1][Rt * 16 + li];
            }
            const R nre = -are, nim = -aim;
            if (AHEAD && q + 1 < RT) {
                are = F[lk][(Rt + RT_W) * 16 + li];
                aim = F[lk ^ 1][(Rt + RT_W) * 16 + li];
            }
            if (Rt >= k1 && Rt < nt) {
#pragma unroll
                for (int k = 0; k < KC; ++k)
                    if (livek[k]) {
                        tr[q][k] = M_::mma(nre, opB[k], tr[q][k]);
                        ti[q][k] = M_::mma(nim, (lk & 1) ? -opB[k] : opB[k], ti[q][k]);
                    }
            }
        }
        cx<R> xn4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) xn4[r] = csel(AHEAD, x[w * 16 + M_::row(lk, r)], zero);
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            const int Rt = w + RT_W * q;
            cx<R> xr[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (AHEAD) xr[r] = xn4[r];
                else xr[r] = x[Rt * 16 + M_::row(lk, r)];
                if (AHEAD && q + 1 < RT) xn4[r] = x[(Rt + RT_W) * 16 + M_::row(lk, r)];
            }
            if (Rt >= k1 && Rt < nt) {
#pragma unroll
                for (int k = 0; k < KC; ++k)
                    if (livek[k]) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) za[k] = cfmac(mk<R>(tr[q][k][r], ti[q][k][r]), xr[r], za[k]);
                    }
                if (Rt == k1) {
                    // this wave holds row c + 1: A(:, c+1) is its conjugate
                    const int rr = row_r<R>(c1 & 15);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r == rr && lk == row_lk<R>(c1 & 15)) {
#pragma unroll
                            for (int k = 0; k < KC; ++k) hrow[k * 16 + li] = mk<R>(tr[q][k][r], -ti[q][k][r]);
                        }
                }
            }
        }
        sum_lane_groups<R, KC>(za, lk, [&](int k, cx<R> v) { zp[w][k * 16 + li] = v; });
        lds_barrier();
        if (w == 0) {
            // ---- publish, after the last clears have reached memory
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            // PARTS lanes per column: each adds its share of the waves and
            // stores its share of the words (the pairwise sums are the same
            // for any PARTS)
            cx<R> v[RT_W / PARTS];
#pragma unroll
            for (int u = 0; u < RT_W / PARTS; ++u) v[u] = zp[part * (RT_W / PARTS) + u][pcol < KC * 16 ? pcol : 0];
            const cx<R> h1 = hrow[pcol < KC * 16 ? pcol : 0];
#pragma unroll
            for (int st = 1; st < RT_W / PARTS; st *= 2)
#pragma unroll
                for (int u = 0; u < RT_W / PARTS; u += 2 * st) v[u] = cadd(v[u], v[u + st]);
            cx<R> zs = v[0];
            if constexpr (PARTS >= 2) {
                zs.x = dpp_sum<PARTS>(zs.x);
                zs.y = dpp_sum<PARTS>(zs.y);
            }
            if (own >= c1 && own < M) {
                uint64_t word[2 * WPC];
                if constexpr (WPC == 2) {
                    word[0] = word_of(zs.x);
                    word[1] = word_of(zs.y);
                    word[2] = word_of(h1.x);
                    word[3] = word_of(h1.y);
                } else {
                    word[0] = word_of(zs.x, zs.y);
                    word[1] = word_of(h1.x, h1.y);
                }
#pragma unroll
                for (int e = 0; e < 2 * WPC; ++e)
                    if (e % PARTS == part) store_agent(cur + e * ex.MP + own, word[e]);
            }
        } else if (w == RT_W - 1) {
            // ---- Procedure 2 while the columns travel
            const R sig2 = ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
            cx<R> tau, scale;
            R beta;
            reflector_core(salpha, sig2, tau, scale, beta);
            if (lane == 0) {
                sref[0] = tau;
                sref[1] = scale;
                if (last == nt - 1) {
                    ws.e[b * n + i] = beta;
                    ws.tau[b * n + i] = tau;
                }
            }
        }
        // a member whose columns are finished has nothing left to do (and
        // must not read on: the others no longer wait for it)
        const int k1n = (c1 + 1) >> 4;
        if (last < k1n && last != nt - 1) return;
        // ---- read every member's columns
        cx<R> z[SP], h[SP];
        R qs = 0;
        if (w * WAVE < M) {
            uint64_t uz[SP][WPC], uh[SP][WPC];
            bool wants[SP];
#pragma unroll
            for (int u = 0; u < SP; ++u) wants[u] = tid + RT_T * u >= c1 && tid + RT_T * u < M;
            // The columns arrive 0.5 us and more after they were published; a poll
            // issued before that only loads the fabric that carries them (512
            // x 8 problems: 4.0 us a column without this wait, 2.8 with 770
            // cycles; the reflector's wave has used most of it already).
            if (w == RT_W - 1) __builtin_amdgcn_s_sleep(4);
            else __builtin_amdgcn_s_sleep(12);
            for (int polls = 0;; ++polls) {
                bool missing = false;
#pragma unroll
                for (int u = 0; u < SP; ++u) {
                    const int s = tid + RT_T * u;
                    if (wants[u]) {
                        bool none = false;
#pragma unroll
                        for (int e = 0; e < WPC; ++e) {
                            uz[u][e] = load_agent(cur + ex.at(0, s, e));
                            uh[u][e] = load_agent(cur + ex.at(1, s, e));
                        }
#pragma unroll
                        for (int e = 0; e < WPC; ++e) none |= uz[u][e] == SENTINEL || uh[u][e] == SENTINEL;
                        wants[u] = none;
                        missing |= none;
                    }
                }
                if (!__any(missing)) break;
                if (polls >= POLLS_MAX) {
                    sdead = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (int u = 0; u < SP; ++u) {
                const int s = tid + RT_T * u;
                if (s >= c1 && s < M) {
                    z[u] = value_of<R>(uz[u]);
                    h[u] = value_of<R>(uh[u]);
                    const cx<R> xs = x[s];
                    qs = fma(xs.x, z[u].x, fma(xs.y, z[u].y, qs));
                    if (s == c1) {
                        sz1 = z[u];
                        shoo = h[u].x;
                    }
                }
            }
            qs = dpp_wave_sum(qs);
        }
        if (lane == 0) sq[w] = qs;
        lds_barrier();
        // ---- B
        if (w == 0 && own < M) {
            // every member has published column c, so every member has read
            // column c - 1: clear its slots
#pragma unroll
            for (int e = 0; e < 2 * WPC; ++e)
                if (e % PARTS == part) store_agent(old + e * ex.MP + own, SENTINEL);
        }
        // v is stored by the owners of the last eight tile columns in turn
        const int Cv = nt - 1 - (c & 7) >= k1n ? nt - 1 - (c & 7) : nt - 1;
        bool stores_v = false;
#pragma unroll
        for (int k = 0; k < KC; ++k) stores_v |= g + G * k == Cv;
        const cx<R> tau = sref[0], scale = sref[1];
        const R hoo = shoo;
        const R qq = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + ((sq[4] + sq[5]) + (sq[6] + sq[7]));
        const cx<R> sz = cmul(scale, sz1);
        const R vav = hoo + (R)2 * sz.x + (scale.x * scale.x + scale.y * scale.y) * qq;
        const R a2 = (R)-0.5 * (tau.x * tau.x + tau.y * tau.y) * vav;
        const cx<R> w1 = cadd(cmul(tau, cadd(mk<R>(hoo, 0), sz)), mk<R>(a2, 0));
        nrm = 0;
#pragma unroll
        for (int u = 0; u < SP; ++u) {
            const int s = tid + RT_T * u;
            if (s < MPX) {
                cx<R> vs = zero, wv = zero, xn = zero;
                if (s >= c1 && s < M) {
                    vs = csel(s == c1, mk<R>(1, 0), cmul(scale, x[s]));
                    wv = csel(s == c1, w1, cfma(tau, cfma(scale, z[u], h[u]), cscale(vs, a2)));
                    // x'_s = h_s - (v_s conj(w_{c+1}) + w_s)
                    xn = csub(h[u], cadd(cmulc(w1, vs), wv));
                    if (stores_v) V[(int64_t)(i0 + s) + (int64_t)i * n] = vs;
                    if (s == c1 && last == nt - 1) ws.d[b * n + i + 1] = hoo - (R)2 * w1.x;
                    if (s == c1 + 1) salpha = xn;
                    xn = csel(s >= c1 + 2, xn, zero);
                    nrm += xn.x * xn.x + xn.y * xn.y;
                }
                F[0][s] = vs.x;
                F[1][s] = vs.y;
                F[2][s] = wv.x;
                F[3][s] = wv.y;
                x[s] = xn;
            }
        }
        nrm = dpp_wave_sum(nrm);
        if (lane == 0) red[w] = nrm;
        lds_barrier();
        if (sdead) {
            if (tid == 0) __hip_atomic_fetch_or(ex.started(), GIVEN_UP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        ring = ring == 2 ? 0 : ring + 1;
    }
}

// The problems whose group was given up: one workgroup each, with the same
// operations on the same values in the same order as a group's members, so
// the results have the same bits whether a group ran or not.  The trailing
// matrix (both triangles, as a group holds it) lies in the buffers of the
// tridiagonal eigensolver, which has not run yet: real parts in Fr, imaginary
// parts in Fi, tile by tile down each tile column, a tile in the order of its
// lanes.  Sixteen waves: wave w takes the tile rows w mod 8, w mod 8 + 8, ... of two
// of four tile columns at a time, whose sums are joined through LDS.  The rows of
// phase B belong to the threads of a member's workgroup (s, s + 512).
//
// Reached only when other work holds the GPU's compute units for longer than
// the members' wait.  Bound by one compute unit's traffic to memory, which the
// matrix crosses twice a column: 2.6 ms at order 200, 23 ms at 512 and 172 ms at
// 1024, after the wait.  (In place on the lower triangle, one thread per row and
// other bits than a group's: 6.4, 39 and 297 ms.)
__device__ unsigned int groups_given_up;     // for tests

template <typename R>
__global__ __launch_bounds__(2 * RT_T) void hetrd_memory(HetrdWs<R> ws, int i0, int G)
{
    using M_ = Mfma<R>;
    constexpr int MPX = HETRD_GROUP_M, SP = MPX / RT_T, FS = MPX + 16;
    constexpr int CC = 4;                    // tile columns per pass: 64 columns
    static_assert(CC * 16 == WAVE && SP == 2, "a wave's rows are a pass's columns");
    __shared__ R F[4][FS];
    __shared__ cx<R> x[MPX];
    __shared__ cx<R> zp[RT_W][CC * 16];
    __shared__ cx<R> hrow[CC * 16];
    __shared__ R red[RT_W], sq[RT_W];
    __shared__ cx<R> salpha, sref[2], sz1;
    __shared__ R shoo;

    const int64_t b = blockIdx.x;
    const int n = ws.n, M = n - i0, nt = (M + 15) >> 4;
    if (*Exchange<R>(ws, b, M).started() == (uint32_t)G) return;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wr = w & (RT_W - 1), wc = w / RT_W;
    const bool rows = w < RT_W;              // this thread has rows of phase B
    const cx<R>* A = ws.A + b * ws.sA + (int64_t)i0 + (int64_t)i0 * ws.lda;
    const int64_t lda = ws.lda;
    cx<R>* V = ws.V + b * ws.sV;
    R* Fr = ws.Fr + b * ws.sF;
    R* Fi = ws.Fi + b * ws.sF;
    const cx<R> zero = czero<cx<R>>();
    if (tid == 0) atomicAdd(&groups_given_up, 1u);

    // Register r of this lane in tile (Rt, C): its place in Fr and Fi, and
    // whether the entry exists (0 and false past the matrix).  The last tile row and
    // column hold the entries that exist only, so the M x M entries fill M x M places.
    auto place = [&](int Rt, int C, int r, bool& in) -> int {
        const int mr = min(16, M - Rt * 16), mc = min(16, M - C * 16);
        const int base = C * 16 * M + Rt * 16 * mc;
        in = true;
        if (mr == 16 && mc == 16) return base + r * WAVE + lane;
        const int row = M_::row(lk, r);
        in = row < mr && li < mc;
        return in ? base + li * mr + row : 0;
    };
    // the full matrix from the lower triangle, by the lanes that update it below
    for (int C = 0; C < nt; ++C) {
        if (((C & (CC - 1)) >> 1) != wc) continue;
        for (int Rt = wr; Rt < nt; Rt += RT_W)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = Rt * 16 + M_::row(lk, r), col = C * 16 + li;
                bool in;
                const int at = place(Rt, C, r, in);
                if (in) {
                    const bool low = row >= col;
                    const cx<R> a = A[low ? (int64_t)row + (int64_t)col * lda : (int64_t)col + (int64_t)row * lda];
                    Fr[at] = a.x;
                    Fi[at] = row == col ? (R)0 : (low ? a.y : -a.y);
                }
            }
    }
    R nrm = 0;
    for (int e = tid; e < 4 * FS; e += 2 * RT_T) (&F[0][0])[e] = (R)0;
    if (rows) {
#pragma unroll
        for (int u = 0; u < SP; ++u) {
            const int s = tid + RT_T * u;
            const cx<R> a = csel(s < M, A[s < M ? s : 0], zero);
            const cx<R> a2 = csel(s >= 2, a, zero);
            x[s] = a2;
            nrm += a2.x * a2.x + a2.y * a2.y;
            if (s == 0) ws.d[b * n + i0] = a.x;
            if (s == 1) salpha = a;
        }
        nrm = dpp_wave_sum(nrm);
        if (lane == 0) red[w] = nrm;
    }
    __syncthreads();

    for (int c = 0; c + 1 < M; ++c) {
        const int c1 = c + 1, i = i0 + c, k1 = c1 >> 4;
        cx<R> z[SP], h[SP];
#pragma unroll
        for (int u = 0; u < SP; ++u) z[u] = h[u] = zero;
        // ---- A: pending update, column sums, row c + 1
        for (int C0 = k1 & ~(CC - 1); C0 < nt; C0 += CC) {
#pragma unroll 1
            for (int C = max(C0 + 2 * wc, k1); C < min(C0 + 2 * wc + 2, nt); ++C) {
                const R opB = F[lk ^ 2][C * 16 + li];
                cx<R> za[1] = {zero};
                auto multiply = [&](int Rt, acc4<R>& tr, acc4<R>& ti) __attribute__((always_inline)) {
                    const R nre = -F[lk][Rt * 16 + li], nim = -F[lk ^ 1][Rt * 16 + li];
                    tr = M_::mma(nre, opB, tr);
                    ti = M_::mma(nim, (lk & 1) ? -opB : opB, ti);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        za[0] = cfmac(mk<R>(tr[r], ti[r]), x[Rt * 16 + M_::row(lk, r)], za[0]);
                    if (Rt == k1) {
                        // row c + 1: A(:, c+1) is its conjugate
                        const int rr = row_r<R>(c1 & 15);
                        const R hr = rr < 2 ? (rr < 1 ? tr[0] : tr[1]) : (rr < 3 ? tr[2] : tr[3]);
                        const R hi = rr < 2 ? (rr < 1 ? ti[0] : ti[1]) : (rr < 3 ? ti[2] : ti[3]);
                        if (lk == row_lk<R>(c1 & 15)) hrow[(C - C0) * 16 + li] = mk<R>(hr, -hi);
                    }
                };
                const int whole = C < (M >> 4) ? M >> 4 : 0;     // whole tiles of the column
                int Rt = k1 + ((wr - k1) & (RT_W - 1));
                // whole tiles: the next one is requested before this one is multiplied
                R* const pr = Fr + C * 16 * M + lane;
                R* const pi = Fi + C * 16 * M + lane;
                acc4<R> nr, ni;
                auto request = [&](int T) __attribute__((always_inline)) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        nr[r] = pr[T * 256 + r * WAVE];
                        ni[r] = pi[T * 256 + r * WAVE];
                    }
                };
                if (Rt < whole) request(Rt);
#pragma unroll 1
                for (; Rt < whole; Rt += RT_W) {
                    acc4<R> tr = nr, ti = ni;
                    if (Rt + RT_W < whole) request(Rt + RT_W);
                    multiply(Rt, tr, ti);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        pr[Rt * 256 + r * WAVE] = tr[r];
                        pi[Rt * 256 + r * WAVE] = ti[r];
                    }
                }
#pragma unroll 1
                for (; Rt < nt; Rt += RT_W) {
                    acc4<R> tr, ti;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        bool in;
                        const int at = place(Rt, C, r, in);
                        tr[r] = in ? Fr[at] : (R)0;
                        ti[r] = in ? Fi[at] : (R)0;
                    }
                    multiply(Rt, tr, ti);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        bool in;
                        const int at = place(Rt, C, r, in);
                        if (in) {
                            Fr[at] = tr[r];
                            Fi[at] = ti[r];
                        }
                    }
                }
                sum_lane_groups<R, 1>(za, lk, [&](int, cx<R> v) { zp[wr][(C - C0) * 16 + li] = v; });
            }
            __syncthreads();
            // the thread whose row a column's sum is takes it
            if (rows && w == ((C0 / CC) & (RT_W - 1))) {
                cx<R> v[RT_W];
#pragma unroll
                for (int q = 0; q < RT_W; ++q) v[q] = zp[q][lane];
                const cx<R> zs = cadd(cadd(cadd(v[0], v[1]), cadd(v[2], v[3])), cadd(cadd(v[4], v[5]), cadd(v[6], v[7])));
                const bool second = C0 / CC >= RT_W;
                z[0] = csel(second, z[0], zs);
                h[0] = csel(second, h[0], hrow[lane]);
                z[1] = csel(second, zs, z[1]);
                h[1] = csel(second, hrow[lane], h[1]);
            }
            __syncthreads();
        }
        // ---- Procedure 2
        if (w == RT_W - 1) {
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
        if (rows) {
            R qs = 0;
#pragma unroll
            for (int u = 0; u < SP; ++u) {
                const int s = tid + RT_T * u;
                if (s >= c1 && s < M) {
                    const cx<R> xs = x[s];
                    qs = fma(xs.x, z[u].x, fma(xs.y, z[u].y, qs));
                    if (s == c1) {
                        sz1 = z[u];
                        shoo = h[u].x;
                    }
                }
            }
            qs = dpp_wave_sum(qs);
            if (lane == 0) sq[w] = qs;
        }
        __syncthreads();
        // ---- B
        if (rows) {
            // (tau and scale come from LDS and the expressions are a member's, so
            // that products and sums are fused alike)
            const cx<R> tau = sref[0], scale = sref[1];
            const R hoo = shoo;
            const R qq = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + ((sq[4] + sq[5]) + (sq[6] + sq[7]));
            const cx<R> sz = cmul(scale, sz1);
            const R vav = hoo + (R)2 * sz.x + (scale.x * scale.x + scale.y * scale.y) * qq;
            const R a2 = (R)-0.5 * (tau.x * tau.x + tau.y * tau.y) * vav;
            const cx<R> w1 = cadd(cmul(tau, cadd(mk<R>(hoo, 0), sz)), mk<R>(a2, 0));
            nrm = 0;
#pragma unroll
            for (int u = 0; u < SP; ++u) {
                const int s = tid + RT_T * u;
                cx<R> vs = zero, wv = zero, xn = zero;
                if (s >= c1 && s < M) {
                    vs = csel(s == c1, mk<R>(1, 0), cmul(scale, x[s]));
                    wv = csel(s == c1, w1, cfma(tau, cfma(scale, z[u], h[u]), cscale(vs, a2)));
                    xn = csub(h[u], cadd(cmulc(w1, vs), wv));
                    V[(int64_t)(i0 + s) + (int64_t)i * n] = vs;
                    if (s == c1) ws.d[b * n + i + 1] = hoo - (R)2 * w1.x;
                    if (s == c1 + 1) salpha = xn;
                    xn = csel(s >= c1 + 2, xn, zero);
                    nrm += xn.x * xn.x + xn.y * xn.y;
                }
                F[0][s] = vs.x;
                F[1][s] = vs.y;
                F[2][s] = wv.x;
                F[3][s] = wv.y;
                x[s] = xn;
            }
            nrm = dpp_wave_sum(nrm);
            if (lane == 0) red[w] = nrm;
        }
        __syncthreads();
    }
}

template <typename R, int RT, int KC>
hipError_t launch_group(hipStream_t st, const HetrdWs<R>& ws, int i0, int64_t nk)
{
    const int M = ws.n - i0, nt = (M + 15) / 16;
    const int G = (nt + KC - 1) / KC;
    if (M > HETRD_GROUP_M || nt > RT * RT_W || G > GROUP_MAX) return hipErrorInvalidValue;
    const Exchange<R> ex(ws, 0, M);
    const int words = 2 + 3 * ex.slot_words();
    hipLaunchKernelGGL(k_exchange_init<R>, dim3((unsigned)((words + 255) / 256), (unsigned)nk), dim3(256), 0, st, ws, M,
                       tl_group_wait_ticks == 0 ? GIVEN_UP : 0u,
                       tl_group_wait_ticks == 0 ? GIVEN_UP : tl_group_lacks_one ? 1u : 0u);
    hipLaunchKernelGGL((hetrd_group<R, RT, KC>), dim3((unsigned)(nk * G - (tl_group_lacks_one ? 1 : 0))), dim3(RT_T), 0,
                       st, ws, i0, G, tl_group_wait_ticks);
    hipLaunchKernelGGL(hetrd_memory<R>, dim3((unsigned)nk), dim3(2 * RT_T), 0, st, ws, i0, G);
    return hipGetLastError();
}

// For each largest order: the tile rows of a wave and the widest share of a
// member (tile columns), set by the registers (RT * KC tiles of 16 each in FP64),
// and the microseconds a column takes with that share when the groups fill the
// chip (measured at 256 x 64, 384 x 32, 512 x 16, 640 x 12, 768 x 5 and 1024 x 4
// problems).
struct GroupShape {
    int M, RT, KC;
    double us;
};
constexpr GroupShape GROUP_SHAPES[] = {{256, 2, 4, 3.2}, {384, 3, 3, 3.7}, {512, 4, 2, 3.6},
                                       {640, 5, 2, 4.4}, {768, 6, 1, 3.4}, {HETRD_GROUP_M, 8, 1, 3.9}};

int group_members(int M, int KC) { return ((M + 15) / 16 + KC - 1) / KC; }

// whether groups with this share may run on cus compute units
bool group_allowed(int M, int KC, int cus) { return group_members(M, KC) <= std::min(GROUP_MAX, cus / 4); }

// How often the compute units are filled with whole groups.  Where groups take
// turns and do not divide them, the partly placed one holds some idle:
// measured 2.7 times one round for 24 problems of order 640 (12 at once).
double group_rounds(int M, int KC, int64_t nk, int cus)
{
    const int64_t G = group_members(M, KC), at_once = cus / G;
    const int64_t rounds = (nk + at_once - 1) / at_once;
    return (double)rounds + (rounds > 1 && cus % G != 0 ? 0.7 : 0.0);
}

// The shape and share for a trailing order: the narrowest share whose groups all
// run at once (more compute units per column); where not even the widest do,
// the widest, so that the groups take turns in as few rounds as possible.  The
// sums do not depend on the share.  {0, 0}: no group may run.
struct GroupChoice {
    int RT, KC;
};
GroupChoice group_choice(int M, int64_t nk, int cus)
{
    for (const GroupShape& g : GROUP_SHAPES) {
        if (M > g.M) continue;
        for (int KC = 1; KC < g.KC; ++KC) {
            if (g.RT == 2 && KC == 3) continue;      // (2, 3) is not instantiated
            if (group_allowed(M, KC, cus) && group_rounds(M, KC, nk, cus) < 1.5) return {g.RT, KC};
        }
        return group_allowed(M, g.KC, cus) ? GroupChoice{g.RT, g.KC} : GroupChoice{0, 0};
    }
    return {0, 0};
}

thread_local int tl_compute_units = 0;       // set by tests

}  // namespace

// The compute units that work on a stream may use: the device's, without those
// that a mask of the stream leaves out (the runtime's own streams, whose handles
// are small numbers, have the process's mask).
int stream_compute_units(hipStream_t st)
{
    if (tl_compute_units > 0) return tl_compute_units;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    uint32_t mask[32] = {};
    const uint32_t words = (uint32_t)std::min((cus + 31) / 32, 32);
    if (st == hipStreamLegacy || st == hipStreamPerThread) st = nullptr;
    if (hipExtStreamGetCUMask(st, words, mask) == hipSuccess) {
        int in = 0;
        for (uint32_t q = 0; q < words; ++q) in += __builtin_popcount(mask[q]);
        if (in > 0) cus = std::min(cus, in);
    } else {
        (void)hipGetLastError();
    }
    return cus;
}

// The hand-over order with the least estimated time for the whole reduction:
// blocked columns at 12 us plus 4 TB/s over the lower triangles (two launches
// and the HBM reads of a column; 16 us at m = 192, 33 us at m = 390 and 90 us at
// m = 780 with 64 problems, 11 us at m = 500 with one), then the groups' columns
// times their rounds.  512 columns: 1 problem 5.1 -> 1.75 ms, 8 problems 5.2 ->
// 2.1 ms, 64 problems (4 rounds) 11.0 -> 8.2 ms; 1024 columns of one problem
// 11.3 -> 4.9 ms.
int hetrd_res_order(int n, int nb, int64_t nk, int groups, int cus)
{
    int best = HETRD_RES_M;
    if (!groups || n <= GROUP_MIN) return best;
    double least = 0.0;
    for (int q = -1; q < (int)(sizeof(GROUP_SHAPES) / sizeof(GROUP_SHAPES[0])); ++q) {
        const int cap = q < 0 ? HETRD_RES_M : GROUP_SHAPES[q].M;
        const int p = n > cap ? (n - cap + nb - 1) / nb * nb : 0;      // the hand-over column
        const int M = n - p;
        if (q >= 0 && (M <= HETRD_RES_M || !group_allowed(M, GROUP_SHAPES[q].KC, cus))) continue;
        const double dn = n, dM = M;
        double us = 12.0 * (dn - dM) + 8.0 * (double)nk / 4.0e6 * (dn * dn * dn - dM * dM * dM) / 3.0;
        us += q < 0 ? 2.0 * dM : group_rounds(M, GROUP_SHAPES[q].KC, nk, cus) * dM * GROUP_SHAPES[q].us;
        if (q < 0 || us < least) {
            least = us;
            best = cap;
        }
    }
    return best;
}

template <typename R>
hipError_t hetrd_res(hipStream_t st, const HetrdWs<R>& ws, int i0, int64_t nk, int cus)
{
    const int M = ws.n - i0;
    if (M <= HETRD_RES_M) {
        // A column costs about the same at any order that a form holds: 4000
        // problems of order 2 took 51 us with the form for 64, 20 with that for 16,
        // of order 8 207 and 72; 4000 of order 65 2.6 ms with that for 128, 2.2 with
        // that for 80.
        const dim3 grid((unsigned)nk), block(RT_T);
        if (M <= 16)
            hipLaunchKernelGGL((hetrd_resident<R, 1, 1>), grid, block, 0, st, ws, i0);
        else if (M <= 64)
            hipLaunchKernelGGL((hetrd_resident<R, 1, 4>), grid, block, 0, st, ws, i0);
        else if (M <= 80)
            hipLaunchKernelGGL((hetrd_resident<R, 1, 5>), grid, block, 0, st, ws, i0);
        else
            hipLaunchKernelGGL((hetrd_resident<R, 1, 8>), grid, block, 0, st, ws, i0);
        return hipGetLastError();
    }
    const GroupChoice g = group_choice(M, nk, cus);
    switch (10 * g.RT + g.KC) {
    case 21: return launch_group<R, 2, 1>(st, ws, i0, nk);
    case 22: return launch_group<R, 2, 2>(st, ws, i0, nk);
    case 24: return launch_group<R, 2, 4>(st, ws, i0, nk);
    case 31: return launch_group<R, 3, 1>(st, ws, i0, nk);
    case 32: return launch_group<R, 3, 2>(st, ws, i0, nk);
    case 33: return launch_group<R, 3, 3>(st, ws, i0, nk);
    case 41: return launch_group<R, 4, 1>(st, ws, i0, nk);
    case 42: return launch_group<R, 4, 2>(st, ws, i0, nk);
    case 51: return launch_group<R, 5, 1>(st, ws, i0, nk);
    case 52: return launch_group<R, 5, 2>(st, ws, i0, nk);
    case 61: return launch_group<R, 6, 1>(st, ws, i0, nk);
    case 81: return launch_group<R, 8, 1>(st, ws, i0, nk);
    }
    return hipErrorInvalidValue;
}
template hipError_t hetrd_res<double>(hipStream_t, const HetrdWs<double>&, int, int64_t, int);
template hipError_t hetrd_res<float>(hipStream_t, const HetrdWs<float>&, int, int64_t, int);

}  // namespace kgev

// For tests, for the calling thread: the wait for a group's members to start, in
// 100 MHz ticks (0 gives every group up before it starts; negative: the
// default), and launches whose last problem lacks a member that counts as
// started, so that the others wait for its columns in vain.
extern "C" void kgev_internal_group_wait(int64_t ticks)
{
    kgev::tl_group_wait_ticks = ticks < 0 ? kgev::GROUP_WAIT_TICKS : ticks;
}
extern "C" void kgev_internal_group_lacks_one(int32_t on) { kgev::tl_group_lacks_one = on != 0; }
// the problems of the current device that hetrd_memory has reduced so far
// (waits for the device); -1 if they can't be read
extern "C" int64_t kgev_internal_groups_given_up()
{
    unsigned int count = 0;
    if (hipDeviceSynchronize() != hipSuccess) return -1;
    if (hipMemcpyFromSymbol(&count, HIP_SYMBOL(kgev::groups_given_up), sizeof(count)) != hipSuccess) return -1;
    return count;
}
// what a reduction would do on cus compute units: the hand-over order, and the
// tile rows, tile columns and members of its groups (0 where it hands over to one
// workgroup)
extern "C" void kgev_internal_hetrd_plan(int32_t n, int32_t nb, int64_t nk, int32_t cus, int32_t* out)
{
    const int order = kgev::hetrd_res_order(n, nb, nk, 1, cus);
    const int p = n > order ? (n - order + nb - 1) / nb * nb : 0;
    const kgev::GroupChoice g =
        n - p > kgev::HETRD_RES_M ? kgev::group_choice(n - p, nk, cus) : kgev::GroupChoice{0, 0};
    out[0] = n - p;
    out[1] = g.RT;
    out[2] = g.KC;
    out[3] = g.KC ? kgev::group_members(n - p, g.KC) : 0;
}
// compute units: of a stream, and for the calling thread in place of the
// device's (0: the device's)
extern "C" int32_t kgev_internal_stream_units(void* stream) { return kgev::stream_compute_units((hipStream_t)stream); }
extern "C" void kgev_internal_compute_units(int32_t cus) { kgev::tl_compute_units = cus > 0 ? cus : 0; }
