// Real symmetric tridiagonal eigensolver on the GPU: the tridiagonal step of
// Eigen_HH (Section III of arXiv:1402.4247 calls a LAPACK routine there; the
// paper does not fix which).  Divide and conquer, batched over k-points:
//
//  * Cuppen's rank-one tearing down to leaves of at most LEAF rows: at a split
//    between rows mid-1 and mid, T = diag(T1', T2') + |beta| u u^T with
//    u = e_{mid-1} + sign(beta) e_mid and the two corner diagonal entries
//    lowered by |beta|;
//  * each leaf solved by the parallel cyclic Jacobi method (Golub & Van Loan
//    §8.5), one wave per leaf;
//  * per merge: z = Q^T u / sqrt(2), rho = 2 |beta|, deflation of negligible
//    z components and of close pole pairs by Givens rotations (Dongarra &
//    Sorensen 1987);
//  * the secular equation 1 + rho sum z_i^2 / (d_i - lambda) = 0 solved for
//    each root in coordinates shifted to its nearer pole, with a two-pole
//    rational model step (Li 1993, "middle way") safeguarded by bisection;
//  * eigenvectors from the Loewner-recomputed z (Gu & Eisenstat 1994), so
//    they are numerically orthogonal whatever the root spacing;
//  * Q_new = Q V as a real product on FP64 MFMA, one launch per tree level.
// The tree over [0, n) splits segment [floor(j n / 2^t), floor((j+1) n / 2^t))
// at depth t; every segment of size >= 2 has two non-empty children.
#include <algorithm>

#include "common.hpp"
#include "lanes.hpp"
#include "kernels.hpp"

namespace kgev {

namespace {

constexpr double EPS = 2.220446049250313e-16;

__device__ __host__ inline int64_t seg_bound(int64_t j, int64_t n, int t) { return (j * n) >> t; }

struct Seg {
    int64_t s, e, mid;
};

__device__ inline Seg seg_of(int64_t j, int64_t n, int t)
{
    Seg g;
    g.s = seg_bound(j, n, t);
    g.e = seg_bound(j + 1, n, t);
    g.mid = seg_bound(2 * j + 1, n, t + 1);
    return g;
}

constexpr int LEAF = 16;   // largest leaf of the tree
// on a kept column of a merge: a deflation rotation has mixed columns of both
// halves in it; the others are zero in the rows of the half they don't belong to
constexpr int MIXED = 1 << 30;

// depth of the leaves: the smallest depth whose segments have at most LEAF rows
__host__ __device__ inline int dc_leaf_depth(int64_t n)
{
    int t = 0;
    while (((int64_t)LEAF << t) < n) ++t;
    return t;
}

// row i starts a segment at depth t (i > 0: the boundary before it is torn)
__device__ inline bool starts_segment(int64_t i, int64_t n, int t)
{
    const int64_t j = ((i << t) + n - 1) / n;      // smallest j with j n / 2^t >= i
    return seg_bound(j, n, t) == i;
}

// ---------------------------------------------------------------------------
// Scale T to max |entry| = 1 and lower the diagonal by the rank-one tears of
// the leaf boundaries (depth tl); D = the torn diagonal.
__global__ __launch_bounds__(256) void dc_init(DcWs ws, int tl)
{
    __shared__ double sh[4];
    const int64_t b = blockIdx.x;
    const int n = ws.n;
    const double* d = ws.din + b * ws.s_din;
    const double* e = ws.ein + b * ws.s_din;
    double mx = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) {
        mx = fmax(mx, fabs(d[i]));
        if (i + 1 < n) mx = fmax(mx, fabs(e[i]));
    }
    mx = dpp_wave_max(mx);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
    __syncthreads();
    double org = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    if (!(org > 0.0) || !isfinite(org)) org = (org == 0.0) ? 1.0 : org;
    if (threadIdx.x == 0) ws.onrm[b] = org;
    const double inv = 1.0 / org;
    double* D = ws.D[0] + b * ws.n;
    double* es = ws.es + b * ws.n;
    for (int i = threadIdx.x; i < n; i += 256) {
        double v = d[i] * inv;
        if (i > 0 && starts_segment(i, n, tl)) v -= fabs(e[i - 1] * inv);
        if (i + 1 < n && starts_segment(i + 1, n, tl)) v -= fabs(e[i] * inv);
        D[i] = v;
        es[i] = (i + 1 < n) ? e[i] * inv : 0.0;
    }
}

// d (double) of lane i: a wave-uniform read of a lane-distributed array
__device__ inline double rdl(double v, int i) { return lane_read(v, i); }

// ---------------------------------------------------------------------------
// Leaf eigensolver: one wave per leaf segment (at most LEAF rows) of the torn
// tridiagonal, by the parallel cyclic Jacobi method (Golub & Van Loan §8.5):
// the leaf is held as a dense symmetric LEAF x LEAF matrix in LDS (rows past
// the leaf are zero and never rotated), and each sweep takes LEAF - 1 rounds of
// LEAF / 2 disjoint rotations (round-robin pairing with the last index fixed).
// A rotation of the (p, q) plane with s / c = sign(tau) / (|tau| +
// sqrt(1 + tau^2)), tau = (a_qq - a_pp) / (2 a_pq), zeroes a_pq; each lane forms the rotation of pair lane mod 8 and applies it
// to two rows (then two columns): the columns of A and of the accumulated V
// together, then the rows of A.  An off-diagonal entry
// at most eps * max_i(|d_i| + |e_i|) is left alone (the normwise deflation
// threshold of implicit QL); a sweep that rotates nothing ends the iteration.
// Eigenvalues go to D[0] ascending, the eigenvectors (columns of V) to the
// leaf's diagonal block of Q[0], with zeros in the rows of its parent segment
// outside the leaf (the parent merge reads its whole diagonal block).
// The rounds are short dependent chains of LDS traffic, where a QL sweep is a
// chain of rotations, each with a square root and a reciprocal.
constexpr int LEAF_SWEEPS = 30;

// 1 / sqrt(x): the hardware's estimate and two Newton steps (a third of the
// latency of a square root and a division, which a round's chain is made of)
__device__ inline double rsqrt_nr(double x)
{
    double r = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const double e = fma(-x * r, r, 1.0);
        r = fma(0.5 * r, e, r);
    }
    return r;
}

__device__ inline void leaf_pair(int r, int k, int& p, int& q)
{
    // round r of the circle method on LEAF indices: index LEAF - 1 is fixed,
    // the others rotate; pair k of the round
    constexpr int M = LEAF - 1;
    if (k == 0) {
        p = r;
        q = M;
    } else {
        p = (r + k) % M;
        q = (r + M - k) % M;
    }
    if (p > q) {
        const int t = p;
        p = q;
        q = t;
    }
}

__global__ __launch_bounds__(64) void dc_leaf(DcWs ws, int tl)
{
    __shared__ double As[LEAF][LEAF + 1];
    __shared__ double Vs[LEAF][LEAF + 1];
    const int64_t b = blockIdx.y;
    const int64_t n = ws.n;
    const Seg g = seg_of(blockIdx.x, n, tl);
    const int s = (int)g.s, ns = (int)(g.e - g.s);
    if (ns < 1) return;
    const int lane = threadIdx.x;
    double* D = ws.D[0] + b * n;
    const double* es = ws.es + b * n;
    const double dr = lane < ns ? D[s + lane] : 0.0;
    const double er = lane + 1 < ns ? es[s + lane] : 0.0;
    // the deflation threshold from the leaf's norm (max over rows of |d| + |e|)
    const double norm = dpp_wave_max(fabs(dr) + fabs(er));
    // the leaf is taken at norm 0.5..1 (an exact power of two away), so that
    // the squares of entries above the threshold stay in range
    int ex = 0;
    (void)frexp(norm, &ex);
    ex = norm > 0.0 && isfinite(norm) ? max(ex, -1000) : 0;
    const double up = ldexp(1.0, -ex), down = ldexp(1.0, ex);
    const double tol = 2.220446049250313e-16 * (norm * up);
    for (int e = lane; e < LEAF * LEAF; e += 64) {
        const int i = e / LEAF, j = e % LEAF;
        double a = 0.0;
        if (i < ns && j < ns) {
            if (i == j) a = D[s + i] * up;
            else if (j == i + 1) a = es[s + i] * up;
            else if (i == j + 1) a = es[s + j] * up;
        }
        As[i][j] = a;
        Vs[i][j] = (i == j) ? 1.0 : 0.0;
    }
    wave_sync();
    bool conv = false;
    for (int sweep = 0; sweep < LEAF_SWEEPS; ++sweep) {
        bool rotated = false;
        for (int r = 0; r < LEAF - 1; ++r) {
            // every lane forms the rotation of pair k = lane mod 8, the pair
            // of both its items below, so no LDS round trip shares it
            int p, q;
            leaf_pair(r, lane % (LEAF / 2), p, q);
            const double apq = As[p][q];
            double c = 1.0, sn = 0.0;
            if (fabs(apq) > tol) {
                // |cot 2 theta| = |a| / |g|: c^2 = (1 + |a| / h) / 2 and
                // c s = sign(a) g / (2 h), h = sqrt(a^2 + g^2)
                const double a = As[q][q] - As[p][p], g = 2.0 * apq;
                const double ih = rsqrt_nr(fma(a, a, g * g));
                const double c2 = fma(0.5 * fabs(a), ih, 0.5);
                const double ic = rsqrt_nr(c2);
                c = c2 * ic;
                sn = copysign(0.5, a) * g * ih * ic;
                rotated = true;
            }
            // a round in which no pair rotates (all of the final sweep) leaves
            // A and V as they are: skip its two phases
            if (!__builtin_amdgcn_ballot_w64(sn != 0.0)) continue;
            wave_sync();
            // columns p, q of A and of V: rows i = lane / 8 and lane / 8 + 8
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = lane / (LEAF / 2) + 8 * h;
                const double aip = As[i][p], aiq = As[i][q];
                const double vip = Vs[i][p], viq = Vs[i][q];
                As[i][p] = c * aip - sn * aiq;
                As[i][q] = sn * aip + c * aiq;
                Vs[i][p] = c * vip - sn * viq;
                Vs[i][q] = sn * vip + c * viq;
            }
            wave_sync();
            // rows p, q of A: columns j = lane / 8 and lane / 8 + 8; the
            // rotated entry is set to its exact value 0
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = lane / (LEAF / 2) + 8 * h;
                const double apj = As[p][j], aqj = As[q][j];
                const bool rot = sn != 0.0;
                As[p][j] = (rot && j == q) ? 0.0 : c * apj - sn * aqj;
                As[q][j] = (rot && j == p) ? 0.0 : sn * apj + c * aqj;
            }
            wave_sync();
        }
        if (!__builtin_amdgcn_ballot_w64(rotated)) {
            conv = true;
            break;
        }
    }
    if (!conv && lane == 0 && ws.status) atomicOr(ws.status + b, ST_NOCONV);
    // ascending order: the rank of lane j's value (ties by index)
    const double lam = lane < ns ? As[lane][lane] * down : 0.0;
    int rank = 0;
    for (int k = 0; k < ns; ++k) {
        const double dk = rdl(lam, k);
        rank += (dk < lam || (dk == lam && k < lane)) ? 1 : 0;
    }
    if (lane < ns) D[s + rank] = lam;
    double* Q = ws.Q[0] + b * ws.sQ;
    const Seg pg = tl > 0 ? seg_of(blockIdx.x >> 1, n, tl - 1) : g;
    for (int j = 0; j < ns; ++j) {
        const int rj = __builtin_amdgcn_readlane(rank, j);
        if (lane < ns) Q[(int64_t)(s + lane) + (int64_t)(s + rj) * n] = Vs[lane][j];
        const int64_t r = pg.s + lane;
        if (r < pg.e && (r < g.s || r >= g.e)) Q[r + (int64_t)(s + j) * n] = 0.0;
    }
}

// ---------------------------------------------------------------------------
constexpr int DEFLATE_T = 256;

// The deflation rotations, in order, on the columns of Q: rows DEFLATE_T * block .. of the
// segment, one thread per row.  Consecutive rotations chain through their second
// column (the pending candidate), so that column is carried in a register: no
// rotation waits for the store of the one before it to come back from memory.
// Segments of more than DEFLATE_T rows are rotated in the launch of the roots, which
// don't need Q, by a workgroup per DEFLATE_T rows: one for all rows took 60 of 91 ms
// for a Toeplitz matrix of order 6000 (now 12.5 in all).  Smaller ones gain nothing
// from more workgroups: 64 rows x 1000 problems 0.51 against 0.48 ms.
__device__ inline void dc_rotate(const DcWs& ws, const Seg& g, int64_t b, int64_t n, int block, int rb, int nr)
{
    const int64_t s = g.s;
    const int r = block * DEFLATE_T + threadIdx.x;
    if (r >= (int)(g.e - g.s)) return;
    double* Qr = ws.Q[rb] + b * ws.sQ;
    const int* rota = ws.rota + b * n + s;
    const int* rotb = ws.rotb + b * n + s;
    const double* rotc = ws.rotc + b * n + s;
    const double* rots = ws.rots + b * n + s;
    const int64_t row = s + r;
    int cur = -1;            // column held in cv (not yet stored), or -1
    double cv = 0.0;
    for (int q = 0; q < nr; ++q) {
        const int ca = rota[q], cb = rotb[q];
        const double x = ca == cur ? cv : Qr[row + (s + ca) * n];
        const double y = cb == cur ? cv : Qr[row + (s + cb) * n];
        if (cur >= 0 && cur != ca && cur != cb) Qr[row + (s + cur) * n] = cv;
        Qr[row + (s + ca) * n] = rotc[q] * x + rots[q] * y;
        cur = cb;
        cv = rotc[q] * y - rots[q] * x;
    }
    if (cur >= 0) Qr[row + (s + cur) * n] = cv;
}

// ---------------------------------------------------------------------------
// Deflation for one merge (one workgroup per segment and problem).  The lists
// (sorted poles sd, components sz, columns perm, indices kidx) stay in LDS when
// the segment fits: 24 bytes a row.
//
// Which candidates go: one with a negligible z_q alone, and of two neighbouring
// others (pending p, then q) with |gap c s| <= tol, c = z_q / tau,
// s = -z_p / tau, tau^2 = z_q^2 + z_p^2 (tested without the square root and the
// divisions), the first, after a rotation that folds it into the second.
// As long as no rotation has changed the pending candidate the test of a pair
// reads that pair alone, so all pairs are tested at once, and one wave
// follows only the chains that start where a test succeeds; the lists are
// compacted by prefix counts in the order of a serial scan (the same results,
// bit for bit).  One thread scanning all candidates took 0.17 us each: 25 us
// at 128 rows, 64 us at 333, 333 us at 2000.
__global__ __launch_bounds__(DEFLATE_T) void dc_deflate(DcWs ws, int t, int rb, int lds_cap, int rotate)
{
    __shared__ double sh[8];
    __shared__ int s_cnt[2][4], s_nrot;
    extern __shared__ double dyn[];   // lds_cap doubles sd, lds_cap doubles sz, lds_cap ints perm, lds_cap ints kidx
    const int64_t b = blockIdx.y;
    const int64_t n = ws.n;
    const Seg g = seg_of(blockIdx.x, n, t);
    const int ns = (int)(g.e - g.s);
    if (ns <= 0) return;
    const int64_t s = g.s;
    const double* Dr = ws.D[rb] + b * n;
    const double* Qr = ws.Q[rb] + b * ws.sQ;
    int* kc = ws.kcnt + b * n;
    int* ndc = ws.ndcnt + b * n;
    const bool in_lds = ns <= lds_cap;
    double* sd = in_lds ? dyn : ws.sd + b * n + s;
    double* sz = in_lds ? dyn + lds_cap : ws.sz + b * n + s;
    int* perm = in_lds ? reinterpret_cast<int*>(dyn + 2 * lds_cap) : ws.perm + b * n + s;
    int* kidx = in_lds ? reinterpret_cast<int*>(dyn + 2 * lds_cap) + lds_cap : ws.orgi + b * n + s;
    int* ndx = ws.ndx + b * n + s;
    double* ndd = ws.ndd + b * n + s;
    double* ndz = ws.ndz + b * n + s;
    int* dfx = ws.dfx + b * n + s;
    double* dfd = ws.dfd + b * n + s;
    int* rota = ws.rota + b * n + s;
    int* rotb = ws.rotb + b * n + s;
    double* rotc = ws.rotc + b * n + s;
    double* rots = ws.rots + b * n + s;
    // scratch until the secular equation writes these
    int* what = ws.cmap + b * n + s;      // 4 * column that goes here | 2: one goes here | 1: kept
    double* goes = ws.lam + b * n + s;    // its value
    int* starts = ws.ndx + b * n + s;     // pairs that rotate as they stand (kidx positions)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;

    if (ns == 1) {
        if (tid == 0) {
            kc[s] = 0;
            ndc[s] = 1;
            dfx[0] = 0;
            dfd[0] = Dr[s];
            ws.rho[b * n + s] = 0.0;
        }
        return;
    }
    const int n1 = (int)(g.mid - g.s);
    const double beta = ws.es[b * n + g.mid - 1];
    const double rho = 2.0 * fabs(beta);
    const double sgn = (beta >= 0.0) ? 1.0 : -1.0;
    const double rs2 = 0.70710678118654752440;

    // stable merge of the two sorted halves: perm[pos] = local column.  The
    // poles are staged in sz for the binary searches.  perm starts as the
    // identity so it stays a valid index list even if the inputs hold NaNs
    // (then positions may collide).
    for (int c = tid; c < ns; c += 256) {
        perm[c] = c;
        sz[c] = Dr[s + c];
    }
    __syncthreads();
    for (int c = tid; c < ns; c += 256) {
        const double dc = sz[c];
        int pos;
        if (c < n1) {
            int lo = n1, hi = ns;      // count right-half entries strictly below dc
            while (lo < hi) { int md = (lo + hi) >> 1; if (sz[md] < dc) lo = md + 1; else hi = md; }
            pos = c + (lo - n1);
        } else {
            int lo = 0, hi = n1;       // count left-half entries <= dc
            while (lo < hi) { int md = (lo + hi) >> 1; if (sz[md] <= dc) lo = md + 1; else hi = md; }
            pos = (c - n1) + lo;
        }
        kidx[c] = min(max(pos, 0), ns - 1);
    }
    __syncthreads();
    double dmx = 0.0, zmx = 0.0;
    for (int c = tid; c < ns; c += 256) {
        const double dc = Dr[s + c];
        const double zc = (c < n1) ? Qr[(g.mid - 1) + (s + c) * n] * rs2 : sgn * Qr[g.mid + (s + c) * n] * rs2;
        const int pos = kidx[c];
        perm[pos] = c;
        sd[pos] = dc;
        sz[pos] = zc;
        dmx = fmax(dmx, fabs(dc));
        zmx = fmax(zmx, fabs(zc));
    }
    dmx = dpp_wave_max(dmx);
    zmx = dpp_wave_max(zmx);
    if (lane == 0) { sh[wv] = dmx; sh[4 + wv] = zmx; }
    __syncthreads();
    dmx = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    zmx = fmax(fmax(sh[4], sh[5]), fmax(sh[6], sh[7]));
    const double tol = 8.0 * EPS * fmax(dmx, zmx);

    // this thread's place in the list of all flagged ones (thread order),
    // which had `count` entries; two lists at a time
    auto place2 = [&](bool f0, bool f1, int& count0, int& count1, int& at0, int& at1) {
        const unsigned long long m0 = __builtin_amdgcn_ballot_w64(f0), m1 = __builtin_amdgcn_ballot_w64(f1);
        if (lane == 0) {
            s_cnt[0][wv] = __popcll(m0);
            s_cnt[1][wv] = __popcll(m1);
        }
        __syncthreads();
        const unsigned long long below = ((unsigned long long)1 << lane) - 1;
        at0 = count0 + __popcll(m0 & below);
        at1 = count1 + __popcll(m1 & below);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wv) {
                at0 += s_cnt[0][w];
                at1 += s_cnt[1][w];
            }
            count0 += s_cnt[0][w];
            count1 += s_cnt[1][w];
        }
        __syncthreads();
    };
    auto rotates = [&](double dp, double zp, double dq, double zq) {
        return fabs((dq - dp) * zq * zp) <= tol * (zq * zq + zp * zp);
    };
    // the candidates with z not negligible (none if the whole update is)
    const bool none = rho * zmx <= tol;
    int K1 = 0, dummy = 0, at0, at1;
    for (int q0 = 0; q0 < ns; q0 += 256) {
        const int q = q0 + tid;
        const bool keep = q < ns && !none && !(rho * fabs(sz[q < ns ? q : 0]) <= tol);
        place2(keep, false, K1, dummy, at0, at1);
        if (keep) kidx[at0] = q;
        if (q < ns) {
            what[q] = keep ? 1 : 4 * perm[q] + 2;
            if (!keep) goes[q] = sd[q];
        }
    }
    if (tid == 0) s_nrot = 0;
    __syncthreads();
    int nst = 0;
    for (int r0 = 0; r0 + 1 < K1; r0 += 256) {
        const int r = r0 + tid;
        bool f = false;
        if (r + 1 < K1) {
            const int p = kidx[r], q = kidx[r + 1];
            f = rotates(sd[p], sz[p], sd[q], sz[q]);
        }
        place2(f, false, nst, dummy, at0, at1);
        if (f) starts[at0] = r;
    }
    __syncthreads();
    if (nst > 0) {
        if (wv == 0) {
            // The chains, one after another: every lane follows them with the same
            // values, which come from a window of 64 starts and one of 64
            // candidates, read whole, so that no step waits for memory.  A chain over
            // all rows, 700 x 10 1.97 -> 1.70 ms, 2000 x 1 4.5 -> 4.1, 3000 x 4 9.5 ->
            // 8.8 against one thread that read and wrote as it went.
            int nr = 0, from = 0, c0 = -WAVE;
            int wp = 0, wc = 0;              // this lane's candidate: its place, its column
            double wd = 0.0, wz = 0.0;       // its pole and component
            auto window = [&](int r) {       // candidates r, r + 1, ... into the lanes
                c0 = r;
                wp = kidx[min(r + lane, K1 - 1)];
                wd = sd[wp];
                wz = sz[wp];
                wc = perm[wp];
            };
            int s0 = 0, sv = lane < nst ? starts[lane] : -1;
            while (s0 < nst) {
                // the next start that no chain has reached
                const unsigned long long ok = __builtin_amdgcn_ballot_w64(sv >= from);
                if (ok == 0) {
                    s0 += WAVE;
                    sv = s0 + lane < nst ? starts[s0 + lane] : -1;
                    continue;
                }
                int r = __builtin_amdgcn_readlane(sv, __builtin_ctzll(ok));
                if (r < c0 || r >= c0 + WAVE) window(r);
                int at = r - c0;
                int p = __builtin_amdgcn_readlane(wp, at), pp = __builtin_amdgcn_readlane(wc, at), gone = 0;
                double dp = rdl(wd, at), zp = rdl(wz, at);
                while (r + 1 < K1) {
                    if (r + 1 >= c0 + WAVE) window(r + 1);
                    at = r + 1 - c0;
                    const int q = __builtin_amdgcn_readlane(wp, at), cq = __builtin_amdgcn_readlane(wc, at);
                    const double dq = rdl(wd, at), zq = rdl(wz, at);
                    if (!rotates(dp, zp, dq, zq)) break;
                    const double tau = hypot(zq, zp);
                    const double c = zq / tau, sn = -zp / tau;
                    const int cp = pp & ~MIXED;
                    const bool mixed = (pp & MIXED) || (cp < n1) != (cq < n1);
                    if (lane == 0) {
                        rota[nr] = cp;
                        rotb[nr] = cq;
                        rotc[nr] = c;
                        rots[nr] = sn;
                        what[p] = gone;                  // no longer kept
                        what[q] = 4 * cp + 2 + 1;
                        if (mixed) perm[q] = cq | MIXED;
                        goes[q] = dp * c * c + dq * sn * sn;
                    }
                    ++nr;
                    zp = tau;
                    dp = dp * sn * sn + dq * c * c;
                    gone = 4 * cp + 2;
                    p = q;
                    pp = mixed ? cq | MIXED : cq;
                    ++r;
                }
                if (lane == 0) {
                    sd[p] = dp;
                    sz[p] = zp;
                }
                from = r + 1;
            }
            if (lane == 0) s_nrot = nr;
        }
        __syncthreads();
    }
    // the lists, in order of position
    int K = 0, nd = 0;
    for (int q0 = 0; q0 < ns; q0 += 256) {
        const int q = q0 + tid;
        const int f = q < ns ? what[q] : 0;
        const bool keep = (f & 1) != 0, go = (f & 2) != 0;
        place2(keep, go, K, nd, at0, at1);
        if (keep) {
            ndx[at0] = perm[q];
            ndd[at0] = sd[q];
            ndz[at0] = sz[q];
        }
        if (go) {
            dfx[at1] = f >> 2;
            dfd[at1] = goes[q];
        }
    }
    if (tid == 0) {
        kc[s] = K;
        ndc[s] = nd;
        ws.rho[b * n + s] = rho;
        if (!rotate) ws.ksplit[b * n + s] = s_nrot;     // (for dc_secular; then dc_zhat's)
    }
    if (rotate) dc_rotate(ws, g, b, n, 0, rb, s_nrot);
}

// ---------------------------------------------------------------------------
// Secular equation: SEC_LANES lanes cooperate on one root: lane `sub` sums
// the terms q = sub mod SEC_LANES and a butterfly of xor steps adds the
// partial sums.  Floating-point addition is commutative, so every lane of the
// root ends with bitwise equal sums and takes the same branches.  Sixteen
// lanes (four roots per wave) gave the top merges enough waves to hide the
// divide latency: 1.1% off the n = 2000 x 16 step against four lanes, with 32
// lanes equal and 64 slower.
//
// A workgroup's sixteen roots share the poles and z^2 in LDS (segments of up
// to SEC_CAP rows).  Small merges are bound by the slowest root's chain of
// evaluations, so each root starts from the two-pole model through the midpoint
// with its neighbours' own z^2, and the last root takes the two-pole model
// too (its poles K-2 and K-1): at most 9 evaluations on the spectra of dense and
// LCAO pencils where starting at the middle of the bracket and a one-pole
// model for the last root took up to 28.
constexpr int SEC_LANES = 16;
constexpr int SEC_T = DEFLATE_T;     // (a launch has workgroups of both kinds)
constexpr int SEC_CAP = 4000;

__device__ inline double root_sum(double v)
{
    return dpp_sum<SEC_LANES>(v);
}

struct SecularSums {
    double f, psi, dpsi, phi, dphi;
};

// f and its two parts at tau (relative to the pole dorg): psi over q <= js,
// phi over q > js
__device__ inline SecularSums secular_eval(int K, const double* dl, const double* z2, double rho, int js, double dorg,
                                           double tau, int sub)
{
    SecularSums v{0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int q = sub; q < K; q += SEC_LANES) {
        const double del = (dl[q] - dorg) - tau;
        const double r = 1.0 / del;
        const double tq = z2[q] * r;
        const bool left = q <= js;
        v.psi += left ? tq : 0.0;
        v.dpsi = left ? fma(tq, r, v.dpsi) : v.dpsi;
        v.phi += left ? 0.0 : tq;
        v.dphi = left ? v.dphi : fma(tq, r, v.dphi);
    }
    v.psi = rho * root_sum(v.psi);
    v.dpsi = rho * root_sum(v.dpsi);
    v.phi = rho * root_sum(v.phi);
    v.dphi = rho * root_sum(v.dphi);
    v.f = 1.0 + v.psi + v.phi;
    return v;
}

// the root eta of c eta^2 - B eta + C = 0 with tau + eta inside (lo, hi), as
// tau + eta; lo where there is none
__device__ inline double model_root(double c, double B, double C, double tau, double lo, double hi)
{
    const double disc = B * B - 4.0 * c * C;
    if (!(disc >= 0.0)) return lo;
    const double sq = sqrt(disc);
    const double den = B >= 0.0 ? B + sq : B - sq;
    const double x1 = tau + 2.0 * C / den, x2 = tau + den / (2.0 * c);
    if (x1 > lo && x1 < hi) return x1;
    return x2 > lo && x2 < hi ? x2 : lo;
}

// z^2 of every kept pole, in zhat (which the next step overwrites), for the
// segments that do not fit in LDS
__global__ __launch_bounds__(256) void dc_square(DcWs ws)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= ws.n) return;
    const double z = ws.ndz[blockIdx.y * (int64_t)ws.n + q];
    ws.zhat[blockIdx.y * (int64_t)ws.n + q] = z * z;
}

__global__ __launch_bounds__(SEC_T) void dc_secular(DcWs ws, int t, int cap, int rb, int row_blocks)
{
    extern __shared__ double dyn[];      // cap poles, cap z^2
    const int64_t b = blockIdx.z;
    const int64_t n = ws.n;
    const Seg g = seg_of(blockIdx.y, n, t);
    if (g.e - g.s < 2) return;
    // the first workgroups of a row rotate Q's columns, which the roots don't need
    if ((int)blockIdx.x < row_blocks) {
        dc_rotate(ws, g, b, n, blockIdx.x, rb, ws.ksplit[b * n + g.s]);
        return;
    }
    const int64_t s = g.s;
    const int K = ws.kcnt[b * n + s];
    const int block = (int)blockIdx.x - row_blocks;
    if (block * (SEC_T / SEC_LANES) >= K) return;
    const int gt = block * SEC_T + threadIdx.x;
    const int j = gt / SEC_LANES, sub = gt % SEC_LANES;
    const double* dl = ws.ndd + b * n + s;
    const double* zl = ws.ndz + b * n + s;
    const double* z2 = ws.zhat + b * n + s;
    const double rho = ws.rho[b * n + s];
    if (K <= cap) {
        for (int q = threadIdx.x; q < K; q += SEC_T) {
            const double z = zl[q];
            dyn[q] = dl[q];
            dyn[cap + q] = z * z;
        }
        dl = dyn;
        z2 = dyn + cap;
    }
    __syncthreads();
    if (j >= K) return;          // the lanes of a root leave together
    if (K == 1) {
        // one pole: lambda = d + rho z^2 exactly
        const double tau1 = rho * zl[0] * zl[0];
        if (sub == 0) {
            ws.orgi[b * n + s] = 0;
            ws.tauv[b * n + s] = tau1;
            ws.lam[b * n + s] = dl[0] + tau1;
        }
        return;
    }
    // the poles left and right of the model: j and j + 1, for the last root
    // K - 2 and K - 1
    const int js = j < K - 1 ? j : K - 2;
    const double gap = dl[js + 1] - dl[js];
    int org = j;
    double lo, hi, at;
    if (j < K - 1) {
        at = 0.5 * gap;
    } else {
        double zz = 0.0;
        for (int q = sub; q < K; q += SEC_LANES) zz += z2[q];
        hi = rho * root_sum(zz);
        at = 0.5 * hi;
    }
    SecularSums v = secular_eval(K, dl, z2, rho, js, dl[j], at, sub);
    // everything but the two poles' own terms, at the first point
    const double s1o = rho * z2[js], s2o = rho * z2[js + 1];
    const double rest = v.f - s1o / ((dl[js] - dl[j]) - at) - s2o / ((dl[js + 1] - dl[j]) - at);
    double P1, P2;               // the two poles relative to the origin
    if (j < K - 1) {
        if (v.f >= 0.0) { lo = 0.0; hi = at; P1 = 0.0; P2 = gap; }
        else { org = j + 1; lo = -at; hi = 0.0; P1 = -gap; P2 = 0.0; }
    } else {
        if (v.f >= 0.0) { lo = 0.0; hi = at; }
        else { lo = at; hi *= 1.0 + 8.0 * EPS; }
        P1 = -gap; P2 = 0.0;
    }
    const double dorg = dl[org];
    double tau = model_root(rest, rest * (P1 + P2) + s1o + s2o, rest * P1 * P2 + s1o * P2 + s2o * P1, 0.0, lo, hi);
    if (!(tau > lo && tau < hi)) tau = 0.5 * (lo + hi);
    bool conv = false;
    for (int it = 0; it < 400; ++it) {
        v = secular_eval(K, dl, z2, rho, js, dorg, tau, sub);
        if (v.f == 0.0) { conv = true; break; }
        if (v.f < 0.0) lo = tau; else hi = tau;
        if (fabs(v.f) <= 8.0 * EPS * (1.0 + fabs(v.psi) + fabs(v.phi)) * (double)(K > 8 ? 8 : K)) { conv = true; break; }
        if (hi - lo <= 4.0 * EPS * fmax(fabs(lo), fabs(hi))) { conv = true; break; }
        // two-pole rational model through (tau, f, f')
        double cand = 0.5 * (lo + hi);
        if ((it & 7) != 7) {
            const double d1 = P1 - tau, d2 = P2 - tau;
            const double s1 = v.dpsi * d1 * d1, s2 = v.dphi * d2 * d2;
            const double c = 1.0 + (v.psi - v.dpsi * d1) + (v.phi - v.dphi * d2);
            const double x = model_root(c, c * (d1 + d2) + s1 + s2, d1 * d2 * v.f, tau, lo, hi);
            if (x > lo && x < hi) cand = x;
        }
        if (cand == tau) cand = 0.5 * (lo + hi);
        tau = cand;
    }
    if (sub != 0) return;
    ws.orgi[b * n + s + j] = org;
    ws.tauv[b * n + s + j] = tau;
    ws.lam[b * n + s + j] = dorg + tau;
    if (!conv && ws.status) atomicOr(ws.status + b, ST_NOCONV);
}

// z recomputed from the roots (Loewner).
__device__ inline void dc_zhat(const DcWs& ws, const Seg& g, int64_t b, int64_t n, int block)
{
    if (g.e - g.s < 2) return;
    const int64_t s = g.s;
    const int K = ws.kcnt[b * n + s];
    // SEC_LANES lanes per index i: lane `sub` multiplies the factors
    // q = sub mod SEC_LANES, a butterfly of products combines them (bitwise
    // equal in every lane of the group)
    const int gt = block * 64 + threadIdx.x;
    const int i = gt / SEC_LANES, sub = gt % SEC_LANES;
    if (i >= K) return;          // the lanes of an index leave together
    const double* dl = ws.ndd + b * n + s;
    const double* zl = ws.ndz + b * n + s;
    const int* org = ws.orgi + b * n + s;
    const double* tv = ws.tauv + b * n + s;
    const double rho = ws.rho[b * n + s];
    const double di = dl[i];
    double p = sub == 0 ? ((dl[org[i]] - di) + tv[i]) / rho : 1.0;
    // the place of pole i when the poles whose columns live in the first half's
    // rows come first, then the mixed ones, then the second half's
    const int* ndx = ws.ndx + b * n + s;
    const int n1 = (int)(g.mid - g.s);
    auto half = [&](int c) { return c & MIXED ? 1 : c < n1 ? 0 : 2; };
    const int ci = ndx[i], hi = half(ci);
    int place = 0, first = 0, both = 0;
    for (int q = sub; q < K; q += SEC_LANES) {
        const int hq = half(ndx[q]);
        place += hq < hi || (hq == hi && q < i) ? 1 : 0;
        first += hq == 0 ? 1 : 0;
        both += hq <= 1 ? 1 : 0;
        if (q == i) continue;
        p *= ((dl[org[q]] - di) + tv[q]) / (dl[q] - di);
    }
    p = dpp_prod<SEC_LANES>(p);
    place = dpp_sum<SEC_LANES>(place);
    first = dpp_sum<SEC_LANES>(first);
    both = dpp_sum<SEC_LANES>(both);
    if (sub == 0) {
        ws.zhat[b * n + s + i] = copysign(sqrt(fmax(p, 0.0)), zl[i]);
        ws.rota[b * n + s + i] = place;
        ws.rotb[b * n + s + place] = ci & ~MIXED;
        if (i == 0) {
            ws.ksplit[b * n + s] = first;
            ws.ksplit[b * n + s + 1] = both;
        }
    }
}

// Eigenvectors of D + rho z z^T: column j = zhat / (d - lambda_j), normalised,
// its rows in the order of the poles' places.  One wave per column, the lanes
// over its rows.
__device__ inline void dc_vectors(const DcWs& ws, const Seg& g, int64_t b, int64_t n, int j)
{
    if (g.e - g.s < 2) return;
    const int64_t s = g.s;
    const int K = ws.kcnt[b * n + s];
    if (j >= K) return;
    const int lane = threadIdx.x;
    const double* dl = ws.ndd + b * n + s;
    const double* zh = ws.zhat + b * n + s;
    const int oj = ws.orgi[b * n + s + j];
    const double tj = ws.tauv[b * n + s + j];
    const double dorg = dl[oj];
    double ss = 0.0;
    for (int i = lane; i < K; i += 64) {
        const double v = zh[i] / ((dl[i] - dorg) - tj);
        ss += v * v;
    }
    ss = dpp_wave_sum(ss);
    const double inv = 1.0 / sqrt(ss);
    double* Vc = ws.Vsec + b * ws.sQ + (s + j) * n + s;
    const int* place = ws.rota + b * n + s;
    for (int i = lane; i < K; i += 64) Vc[place[i]] = zh[i] / ((dl[i] - dorg) - tj) * inv;
}

// Final ascending order of the merged eigenvalues (secular roots and deflated
// poles): each value counts the values that precede it.
__device__ inline void dc_order(const DcWs& ws, const Seg& g, int64_t b, int64_t n, int block, int wb)
{
    const int ns = (int)(g.e - g.s);
    if (ns < 1) return;
    const int64_t s = g.s;
    const int K = ws.kcnt[b * n + s];
    const int nd = ws.ndcnt[b * n + s];
    // SEC_LANES lanes per value, each counting a strided share of the others
    const int gt = block * 64 + threadIdx.x;
    const int q = gt / SEC_LANES, sub = gt % SEC_LANES;
    if (q >= K + nd) return;          // the lanes of a value leave together
    const double* lam = ws.lam + b * n + s;
    const double* dfd = ws.dfd + b * n + s;
    const double v = (q < K) ? lam[q] : dfd[q - K];
    int rank = 0;
    for (int r = sub; r < K + nd; r += SEC_LANES) {
        const double u = (r < K) ? lam[r] : dfd[r - K];
        if (u < v || (u == v && r < q)) ++rank;
    }
    rank = dpp_sum<SEC_LANES>(rank);
    if (sub != 0) return;
    rank = min(rank, ns - 1);
    ws.D[wb][b * n + s + rank] = v;
    ws.cmap[b * n + s + q] = rank;      // entries [0,K): product columns, [K,K+nd): deflated
}

// Deflated columns move unchanged (after rotation) to their place, and every
// column of the segment gets zeros in the rows of its parent segment that lie
// outside it (the parent merge reads its whole diagonal block).
__device__ inline void dc_place(const DcWs& ws, const Seg& g, int64_t b, int64_t n, int q, int t, int rb, int wb)
{
    const int ns = (int)(g.e - g.s);
    if (q >= ns) return;
    const int64_t s = g.s;
    double* Qw = ws.Q[wb] + b * ws.sQ;
    if (t > 0) {
        const Seg pg = seg_of(blockIdx.y >> 1, n, t - 1);
        double* col = Qw + (s + q) * n;
        for (int64_t r = pg.s + threadIdx.x; r < pg.e; r += 64)
            if (r < g.s || r >= g.e) col[r] = 0.0;
    }
    const int K = ws.kcnt[b * n + s];
    const int nd = ws.ndcnt[b * n + s];
    if (q >= nd) return;
    const int src = ws.dfx[b * n + s + q];
    const int dst = ws.cmap[b * n + s + K + q];
    const double* Qr = ws.Q[rb] + b * ws.sQ + (s + src) * n + s;
    double* Qd = Qw + (s + dst) * n + s;
    for (int r = threadIdx.x; r < ns; r += 64) Qd[r] = Qr[r];
}

// Two independent steps each in one launch (a launch of either costs 4.5 us at
// least, whatever the size): the first nb workgroups of a row take the first,
// the others the second.
__global__ __launch_bounds__(64) void dc_zhat_order(DcWs ws, int t, int wb, int nb)
{
    const int64_t b = blockIdx.z, n = ws.n;
    const Seg g = seg_of(blockIdx.y, n, t);
    if ((int)blockIdx.x < nb) dc_zhat(ws, g, b, n, blockIdx.x);
    else dc_order(ws, g, b, n, blockIdx.x - nb, wb);
}
__global__ __launch_bounds__(64) void dc_vectors_place(DcWs ws, int t, int rb, int wb, int nb)
{
    const int64_t b = blockIdx.z, n = ws.n;
    const Seg g = seg_of(blockIdx.y, n, t);
    if ((int)blockIdx.x < nb) dc_vectors(ws, g, b, n, blockIdx.x);
    else dc_place(ws, g, b, n, blockIdx.x - nb, t, rb, wb);
}

// Q_new(s:e, s + cmap[j]) = sum_q Q(s:e, s + col[q]) V(q, j): real product on
// FP64 MFMA with a column gather on A and a column scatter on C.  The columns
// are ordered by the half of the rows they live in and a tile has rows of one
// half, so it takes only that half's columns and the mixed ones: half the work
// (top merge of n = 2000: 343 -> 192 us, of 16 of them 4.07 -> 2.48 ms).
// Workgroups go round the dice and shader engines: problems go first in the
// grid, so that a die reads few of them (2.55 -> 2.33 ms), then column tiles, as
// each engine would get the same few row tiles otherwise.  Loads two K steps
// ahead took 118 registers and were slower (2.63 ms).
constexpr int DB = 64, DK = 16;
__global__ __launch_bounds__(256) void dc_gemm(DcWs ws, int t, int rb, int wb, int tiles, int half_tiles)
{
    __shared__ double sA[2][DK][DB + 1];
    __shared__ double sB[2][DK][DB + 1];
    const int64_t b = blockIdx.x % (unsigned)ws.nk;
    const int64_t n = ws.n;
    const Seg g = seg_of(blockIdx.y, n, t);
    const int ns = (int)(g.e - g.s);
    if (ns < 2) return;
    const int64_t s = g.s;
    const int K = ws.kcnt[b * n + s];
    const int tile = (int)(blockIdx.x / (unsigned)ws.nk), tm = tile / tiles, tn = tile % tiles;
    // row tiles of the first half, then of the second; rows i0..ie-1
    const bool second = tm >= half_tiles;
    const int n1 = (int)(g.mid - g.s), ie = second ? ns : n1;
    const int i0 = second ? n1 + (tm - half_tiles) * DB : tm * DB, j0 = tn * DB;
    if (i0 >= ie || j0 >= K) return;
    const double* Qr = ws.Q[rb] + b * ws.sQ;
    const double* Vs = ws.Vsec + b * ws.sQ;
    const int* col = ws.rotb + b * n + s;
    const int* cmap = ws.cmap + b * n + s;
    double* Qw = ws.Q[wb] + b * ws.sQ;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w & 1, wn = w >> 1;
    const int li = lane & 15, lk = lane >> 4;
    d4_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][c][r] = 0.0;

    const int kb = second ? ws.ksplit[b * n + s] : 0, ke = second ? K : ws.ksplit[b * n + s + 1];
    const int nkt = (ke - kb + DK - 1) / DK;
    // tile loads from clamped (in-bounds) indices with no branch, so the next
    // K step stays in flight during the MFMA work; the bounds mask is applied
    // when the registers are stored to LDS
    double ra[DK / 4], rbv[DK / 4];
    unsigned oka = 0, okb = 0;
    // the columns of a K step are looked up a step before its loads
    int ca[DK / 4];
    auto cload = [&](int k0) {
#pragma unroll
        for (int q = 0; q < DK / 4; ++q) {
            const int k = k0 + (tid >> 6) + 4 * q;
            ca[q] = col[k < ke ? k : 0];
        }
    };
    auto gload = [&](int k0) {
        // A tile: rows i0..i0+63 (lanes), k = k0 + kq + 4q, columns gathered through col
        const int r = tid & 63, kq = tid >> 6;
        const int ic = i0 + r < ie ? i0 + r : 0;
        oka = 0;
#pragma unroll
        for (int q = 0; q < DK / 4; ++q) {
            const int k = k0 + kq + 4 * q;
            ra[q] = Qr[(s + ic) + (s + ca[q]) * n];
            oka |= (unsigned)(i0 + r < ie && k < ke) << q;
        }
        // B tile: k = k0 + kk, cols j0 + jq + 256 / DK q
        const int kk = tid % DK, jq = tid / DK;
        const int k = k0 + kk;
        const int kc = k < ke ? k : 0;
        okb = 0;
#pragma unroll
        for (int q = 0; q < DK / 4; ++q) {
            const int jj = j0 + jq + 256 / DK * q;
            const int jc = jj < K ? jj : 0;
            rbv[q] = Vs[(s + kc) + (s + jc) * n];
            okb |= (unsigned)(jj < K && k < ke) << q;
        }
    };
    auto sstore = [&](int buf) {
        const int r = tid & 63, kq = tid >> 6;
#pragma unroll
        for (int q = 0; q < DK / 4; ++q) sA[buf][kq + 4 * q][r] = ((oka >> q) & 1u) ? ra[q] : 0.0;
        const int kk = tid % DK, jq = tid / DK;
#pragma unroll
        for (int q = 0; q < DK / 4; ++q) sB[buf][kk][jq + 256 / DK * q] = ((okb >> q) & 1u) ? rbv[q] : 0.0;
    };
    int cur = 0;
    if (nkt > 0) {
        cload(kb);
        gload(kb);
        cload(kb + DK);
        sstore(0);
    }
    __syncthreads();
    for (int kt = 0; kt < nkt; ++kt) {
        if (kt + 1 < nkt) {
            gload(kb + (kt + 1) * DK);
            cload(kb + (kt + 2) * DK);
        }
#pragma unroll
        for (int ks = 0; ks < DK; ks += 4) {
            double a0 = sA[cur][ks + lk][wm * 32 + li];
            double a1 = sA[cur][ks + lk][wm * 32 + 16 + li];
            double b0 = sB[cur][ks + lk][wn * 32 + li];
            double b1 = sB[cur][ks + lk][wn * 32 + 16 + li];
            acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
        }
        if (kt + 1 < nkt) sstore(cur ^ 1);
        __syncthreads();
        cur ^= 1;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + wm * 32 + a * 16 + Mfma<double>::row(lk, r);
                const int jj = j0 + wn * 32 + c * 16 + li;
                if (i < ie && jj < K) Qw[(s + i) + (s + cmap[jj]) * n] = acc[a][c][r];
            }
}

__global__ __launch_bounds__(256) void dc_finish(DcWs ws, int fb, double* w)
{
    const int64_t b = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= ws.n) return;
    w[b * ws.s_w + i] = ws.D[fb][b * ws.n + i] * ws.onrm[b];
}

}  // namespace

hipError_t stedc(hipStream_t st, const DcWs& ws0, double* w, double* Z, double* Qscratch, int64_t nk)
{
    DcWs ws = ws0;
    ws.nk = nk;
    const int64_t n = ws.n;
    if (n < 1 || nk < 1) return hipSuccess;
    const int L = dc_leaf_depth(n);
    // the leaves write buffer 0 and the last merge level buffer L & 1: make
    // that the caller's Z
    ws.Q[L & 1] = Z;
    ws.Q[(L & 1) ^ 1] = Qscratch;
    hipLaunchKernelGGL(dc_init, dim3((unsigned)nk), dim3(256), 0, st, ws, L);
    hipLaunchKernelGGL(dc_leaf, dim3(1u << L, (unsigned)nk), dim3(64), 0, st, ws, L);
    for (int t = L - 1; t >= 0; --t) {
        const int rb = (L - t - 1) & 1, wb = (L - t) & 1;
        const unsigned segs = 1u << t;
        const int64_t nsmax = ((n + segs - 1) / segs) + 1;
        const int cap = (int)std::min<int64_t>(nsmax, 2700);
        const size_t dyn_bytes = (size_t)cap * (2 * sizeof(double) + 2 * sizeof(int));
        hipLaunchKernelGGL(dc_deflate, dim3(segs, (unsigned)nk), dim3(DEFLATE_T), dyn_bytes, st, ws, t, rb, cap,
                           (int)(nsmax <= DEFLATE_T));
        const int scap = (int)std::min<int64_t>(nsmax, SEC_CAP);
        if (nsmax > SEC_CAP)
            hipLaunchKernelGGL(dc_square, dim3((unsigned)((n + 255) / 256), (unsigned)nk), dim3(256), 0, st, ws);
        const unsigned row_blocks = nsmax <= DEFLATE_T ? 0u : (unsigned)((nsmax + DEFLATE_T - 1) / DEFLATE_T);
        hipLaunchKernelGGL(dc_secular,
                           dim3(row_blocks + (unsigned)((nsmax * SEC_LANES + SEC_T - 1) / SEC_T), segs, (unsigned)nk),
                           dim3(SEC_T), (size_t)scap * 2 * sizeof(double), st, ws, t, scap, rb, (int)row_blocks);
        const unsigned gxs = (unsigned)((nsmax * SEC_LANES + 63) / 64);
        hipLaunchKernelGGL(dc_zhat_order, dim3(2 * gxs, segs, (unsigned)nk), dim3(64), 0, st, ws, t, wb, (int)gxs);
        hipLaunchKernelGGL(dc_vectors_place, dim3((unsigned)(2 * nsmax), segs, (unsigned)nk), dim3(64), 0, st, ws, t, rb,
                           wb, (int)nsmax);
        const int tiles = (int)((nsmax + DB - 1) / DB);
        const int half_tiles = (int)((n + 2 * segs - 1) / (2 * segs) + DB - 1) / DB;
        hipLaunchKernelGGL(dc_gemm, dim3((unsigned)(nk * (2 * half_tiles * tiles)), segs), dim3(256), 0, st, ws, t, rb, wb,
                           tiles, half_tiles);
    }
    hipLaunchKernelGGL(dc_finish, dim3((unsigned)((n + 255) / 256), (unsigned)nk), dim3(256), 0, st, ws, L & 1, w);
    return hipGetLastError();
}

}  // namespace kgev
