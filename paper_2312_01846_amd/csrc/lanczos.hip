// Truncated-Lanczos vector algebra (Sec. 2.1, Eqs. 10-11) and the small
// generalized eigenproblem T x = lambda S x, all on the device.
//
// Reductions come in two flavours:
//   fast    -- fixed-grid tree (run-to-run reproducible, not sequential order);
//   ordered -- the sum of the products strictly in ascending-rank order, which
//              reproduces a sequential CPU sum bit for bit.
#include <algorithm>
#include <vector>

#include "sfci_internal.h"

namespace {

constexpr int RB = 256;
constexpr int RGRID = 1024;

__device__ __forceinline__ double block_sum(double x, double* sh) {
    // fixed shape tree over 256 threads
    sh[threadIdx.x] = x;
    __syncthreads();
    for (int s = RB / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + s];
        __syncthreads();
    }
    double r = sh[0];
    __syncthreads();
    return r;
}

__device__ __forceinline__ double y_at(const u64* __restrict__ yr, const double* __restrict__ ya, u64 yn, u64 key) {
    // lower bound in the ascending rank list
    u64 lo = 0, hi = yn;
    while (lo < hi) {
        u64 mid = lo + ((hi - lo) >> 1);
        if (yr[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return (lo < yn && yr[lo] == key) ? ya[lo] : 0.0;
}

// partial[b] = sum over a grid-stride slice of x_amp[i] * D[x_rank[i]]
__global__ __launch_bounds__(RB) void k_dot_dense_part(const u64* __restrict__ r, const double* __restrict__ a,
                                                       const u64* __restrict__ nnz, const double* __restrict__ D,
                                                       double* __restrict__ part) {
    __shared__ double sh[RB];
    const u64 n = *nnz;
    double s = 0.0;
    for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)gridDim.x * RB) s += a[i] * D[r[i]];
    double b = block_sum(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = b;
}

__global__ __launch_bounds__(RB) void k_dot_sparse_part(const u64* __restrict__ xr, const double* __restrict__ xa,
                                                        const u64* __restrict__ xn, const u64* __restrict__ yr,
                                                        const double* __restrict__ ya, const u64* __restrict__ yn,
                                                        double* __restrict__ part) {
    __shared__ double sh[RB];
    const u64 n = *xn, m = *yn;
    double s = 0.0;
    for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)gridDim.x * RB) {
        double yv = y_at(yr, ya, m, xr[i]);
        if (yv != 0.0) s += xa[i] * yv;
    }
    double b = block_sum(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = b;
}

__global__ __launch_bounds__(RB) void k_dot_final(const double* __restrict__ part, int np, double* out1, double* out2) {
    __shared__ double sh[RB];
    double s = 0.0;
    for (int i = threadIdx.x; i < np; i += RB) s += part[i];
    double b = block_sum(s, sh);
    if (threadIdx.x == 0) {
        *out1 = b;
        if (out2) *out2 = b;
    }
}

// Ordered sums: s = ((0 + t_0) + t_1) + ... strictly in index order, t_i the
// term of entry i (x_i; a_i * D[r_i]; a_i * a_i), to the bit, but
// not one add after another.  While s stays inside one binade, s = S u with u
// its unit in the last place and 2^52 < |S| < 2^53, and adding t rounds to
// (S + rint(t / u)) u unless t / u lies exactly half way between integers (a
// tie, whose direction depends on S).  So a stretch without a tie whose every
// prefix sum of the integers rint(t / u) stays strictly inside that range is
// an integer sum, which may be taken in any order.  A workgroup takes OS_STEP
// terms at a time: every wavefront reduces its chunk of OS_CHUNK terms to the
// sum, the least and the greatest prefix, and the chunks are then applied in
// order; a chunk that leaves the binade or holds a tie is added by its
// wavefront in stretches that end at such a term, which is added by itself
// (os_events), or term by term where such terms are frequent.
// Bound by: added one by one, the latency of the chain (~17 cycles a term:
// 7.34 ms for 1e6 squares); this way the loads and reductions of one compute
// unit (0.69 ms); long sums are spread over the chip (launch_ordered).  Sums
// that wander about zero leave their binade every few dozen terms and gain
// little.
enum { OS_SUM = 0, OS_DOT = 1, OS_SUMSQ = 2 };
constexpr int OS_WAVES = 8;
constexpr int OS_BLOCK = 64 * OS_WAVES;
constexpr int OS_K = 8;                        // terms per lane
constexpr int OS_CHUNK = 64 * OS_K;            // terms per wavefront
constexpr int OS_STEP = OS_WAVES * OS_CHUNK;   // terms per step
constexpr int OS_PAD = OS_CHUNK + OS_CHUNK / 8;  // a chunk in LDS, one slot of padding per 8
constexpr int OS_EVENTS = 24;                  // singly added terms of a chunk before the rest is added one by one

__device__ __forceinline__ int os_slot(int i) { return i + (i >> 3); }

// the wavefront's minimum (of finite values or infinities), in every lane
__device__ __forceinline__ double os_min(double x) {
    x = fmin(x, wave_dpp<0x111, 0xf>(x, x));
    x = fmin(x, wave_dpp<0x112, 0xf>(x, x));
    x = fmin(x, wave_dpp<0x114, 0xf>(x, x));
    x = fmin(x, wave_dpp<0x118, 0xf>(x, x));
    x = fmin(x, wave_dpp<0x142, 0xa>(x, x));
    x = fmin(x, wave_dpp<0x143, 0xc>(x, x));
    return lane_f64(x, 63);
}

// s's biased exponent, and whether s is a normal number (then s = S 2^-sh)
__device__ __forceinline__ bool os_normal(double s, int& sh) {
    const int b = (__double2hiint(s) >> 20) & 0x7ff;
    sh = 52 + 1023 - b;
    return b >= 1 && b <= 2046;
}

// Every prefix S + [lo, hi] strictly inside S's binade (the bounds themselves
// are out: next to them the rounding unit may be another one).
__device__ __forceinline__ bool os_inside(double S, double lo, double hi) {
    constexpr double L = 4503599627370496.0, H = 9007199254740992.0;
    return S > 0.0 ? (S + lo > L && S + hi < H) : (S + hi < -L && S + lo > -H);
}

// A chunk's terms (in LDS) added to s in order by one wavefront: 64 at a time
// as an integer prefix sum up to the first one that cannot be, that one by
// itself, and on from there.
__device__ double os_events(const double* st, double s, int lane) {
    int pos = 0, ev = 0;
    while (pos < OS_CHUNK) {
        if (ev > OS_EVENTS) {
            for (; pos < OS_CHUNK && (pos & 7); ++pos) s += st[os_slot(pos)];
            for (; pos < OS_CHUNK; pos += 8) {
                const double* q = st + os_slot(pos);
                const double x0 = q[0], x1 = q[1], x2 = q[2], x3 = q[3], x4 = q[4], x5 = q[5], x6 = q[6], x7 = q[7];
                s += x0;
                s += x1;
                s += x2;
                s += x3;
                s += x4;
                s += x5;
                s += x6;
                s += x7;
            }
            break;
        }
        const int m = min(64, OS_CHUNK - pos);
        const double t = lane < m ? st[os_slot(pos + lane)] : 0.0;
        int sh;
        int first = 0;  // terms accepted together
        if (s == 0.0) {
            const u64 nz = __ballot(!(t == 0.0));
            first = nz ? __builtin_ctzll(nz) : 64;
        } else if (os_normal(s, sh)) {
            const double x = ldexp(t, sh), r = rint(x);
            const double S = ldexp(s, sh);
            const double P = wave_scan_dpp(r);
            const u64 bad = __ballot(!(fabs(x - r) < 0.5 && os_inside(S, P, P)));
            first = bad ? __builtin_ctzll(bad) : 64;
            if (first > 0) {
                const int l = first - 1;
                const double Pl = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(P), l),
                                                   __builtin_amdgcn_readlane(__double2loint(P), l));
                s = ldexp(S + Pl, -sh);
            }
        }
        if (first >= m) {
            pos += m;
        } else {
            pos += first;
            s += st[os_slot(pos)];
            ++pos;
            ++ev;
        }
    }
    return s;
}

struct OsChunk {
    double d, lo, hi;  // the sum of the integers, their least and greatest prefix
    int ok;            // 1: no tie; 2: every term is zero
    int pad;
};

// A lane's OS_K terms and, over the wavefront, its chunk's: 1 / unit = 2^sh.
__device__ __forceinline__ OsChunk os_chunk(const double (&t)[OS_K], int sh, bool normal) {
    double d = 0.0, lo = INFINITY, hi = -INFINITY;
    bool exact = true, zero = true;
#pragma unroll
    for (int k = 0; k < OS_K; ++k) {
        const double v = ldexp(t[k], sh), r = rint(v);
        exact = exact && fabs(v - r) < 0.5;
        zero = zero && t[k] == 0.0;
        d += r;
        lo = fmin(lo, d);
        hi = fmax(hi, d);
    }
    const double inc = wave_scan_dpp(d);
    const double before = inc - d;
    const double wlo = os_min(before + lo), whi = -os_min(-(before + hi));
    const bool all_exact = __ballot(!exact) == 0, all_zero = __ballot(!zero) == 0;
    return OsChunk{inc, wlo, whi, all_zero ? 2 : (all_exact && normal ? 1 : 0), 0};  // d in lane 63
}

// s and, after it, the terms term(x, y), first <= i < n, of the values
// load(i, x, y) reads, the same in every thread.
template <class Load, class Term>
__device__ __forceinline__ double os_block_sum(u64 n, const Load& load, const Term& term, u64 first = 0,
                                               double s = 0.0) {
    __shared__ double stage[OS_WAVES][OS_PAD];
    __shared__ OsChunk ch[2][OS_WAVES];
    __shared__ double s_next;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double* const st = stage[wave];
    double x[OS_K], y[OS_K];
    const u64 mine = (u64)wave * OS_CHUNK + lane;
#pragma unroll
    for (int k = 0; k < OS_K; ++k) load(first + mine + (u64)k * 64, x[k], y[k]);
    int par = 0;
    for (u64 base = first; base < n; base += OS_STEP) {
        // coalesced loads, then each lane's OS_K consecutive terms by way of LDS
#pragma unroll
        for (int k = 0; k < OS_K; ++k) st[os_slot(k * 64 + lane)] = term(x[k], y[k]);
#pragma unroll
        for (int k = 0; k < OS_K; ++k) load(base + OS_STEP + mine + (u64)k * 64, x[k], y[k]);
        wave_sync();
        double t[OS_K];
#pragma unroll
        for (int k = 0; k < OS_K; ++k) t[k] = st[lane * (OS_K + 1) + k];
        int w0 = 0;
        for (;;) {
            int sh;
            const bool normal = os_normal(s, sh);
            if (wave >= w0) {
                const OsChunk c = os_chunk(t, sh, normal);
                if (lane == 63) ch[par][wave] = c;
            }
            __syncthreads();
            double S = normal ? ldexp(s, sh) : 0.0;
            int f = w0;
            for (; f < OS_WAVES; ++f) {
                const OsChunk c = ch[par][f];
                if (c.ok == 2) continue;  // adds nothing, whatever s is
                if (c.ok == 0 || !os_inside(S, c.lo, c.hi)) break;
                S += c.d;
            }
            if (normal) s = ldexp(S, -sh);
            par ^= 1;  // (the next write to this half lies behind a barrier)
            if (f == OS_WAVES) break;
            if (wave == f) {
                const double v = os_events(st, s, lane);
                if (lane == 0) s_next = v;
            }
            __syncthreads();
            s = s_next;
            w0 = f + 1;
            if (w0 == OS_WAVES) break;
        }
    }
    return s;
}

template <int MODE>
struct OsTerms {
    const u64* r;
    const double *a, *D;
    u64 n;
    __device__ __forceinline__ void operator()(u64 i, double& x, double& y) const {
        x = 0.0;
        y = 0.0;
        if (i < n) {
            x = a[i];
            if (MODE == OS_DOT) y = D[r[i]];
        }
    }
    static __device__ __forceinline__ double term(double x, double y) {
        return MODE == OS_SUM ? x : (MODE == OS_SUMSQ ? x * x : x * y);
    }
};

template <int MODE>
__global__ __launch_bounds__(OS_BLOCK) void k_ordered(const u64* __restrict__ r, const double* __restrict__ a,
                                                      const u64* __restrict__ nnz, const double* __restrict__ D,
                                                      double* out1, double* out2) {
    const u64 n = *nnz;
    const double s = os_block_sum(n, OsTerms<MODE>{r, a, D, n}, OsTerms<MODE>::term);
    if (threadIdx.x == 0) {
        *out1 = s;
        if (out2) *out2 = s;
    }
}

// Long sums over the chip: blocks of span terms (at most OS_BLOCKS of them)
// are summed in any order, which tells the binade s will be in when a block
// begins; each block is then reduced as if s were in it, and one workgroup
// applies the blocks in order, going through the terms only of those that do
// not fit (another binade, a tie, a prefix that leaves it).  The result does
// not depend on the guess.  Bound by: the blocks gone through again, ~3 us per
// 4096 terms (1e6 squares in 0.14 ms, 0.69 by one workgroup; truncation of 4e6
// entries to 1e6 with its norm 0.91 -> 0.32 ms).
constexpr int OS_BLOCKS = 256;

struct OsBlock {
    OsChunk c;
    int sh, pad;
};

template <int MODE>
__global__ __launch_bounds__(OS_BLOCK) void k_os_guess(const u64* __restrict__ r, const double* __restrict__ a,
                                                       const u64* __restrict__ nnz, const double* __restrict__ D,
                                                       u64 span, double* __restrict__ guess) {
    __shared__ double part[OS_WAVES];
    const u64 n = *nnz, b = (u64)blockIdx.x * span, e = min(n, b + span);
    const OsTerms<MODE> load{r, a, D, n};
    double s = 0.0;
    for (u64 i = b + threadIdx.x; i < e; i += OS_BLOCK) {
        double x, y;
        load(i, x, y);
        s += OsTerms<MODE>::term(x, y);
    }
    s = wave_sum_dpp(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < OS_WAVES; ++w) s += part[w];
        guess[blockIdx.x] = s;
    }
}

template <int MODE>
__global__ __launch_bounds__(OS_BLOCK) void k_os_blocks(const u64* __restrict__ r, const double* __restrict__ a,
                                                        const u64* __restrict__ nnz, const double* __restrict__ D,
                                                        u64 span, const double* __restrict__ guess,
                                                        OsBlock* __restrict__ out) {
    __shared__ double stage[OS_WAVES][OS_PAD], part[OS_WAVES];
    __shared__ OsChunk ch[OS_WAVES];
    const u64 n = *nnz, b = (u64)blockIdx.x * span, e = min(n, b + span);
    if (b >= e) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double g = threadIdx.x < blockIdx.x ? guess[threadIdx.x] : 0.0;
    g = wave_sum_dpp(g);
    if (lane == 0) part[wave] = g;
    __syncthreads();
    double s = part[0];
    for (int w = 1; w < OS_WAVES; ++w) s += part[w];
    int sh;
    const bool normal = os_normal(s, sh);
    const OsTerms<MODE> load{r, a, D, e};
    double* const st = stage[wave];
    OsChunk all{0.0, INFINITY, -INFINITY, 2, 0};
    for (u64 base = b; base < e; base += OS_STEP) {
#pragma unroll
        for (int k = 0; k < OS_K; ++k) {
            double x, y;
            load(base + (u64)wave * OS_CHUNK + lane + (u64)k * 64, x, y);
            st[os_slot(k * 64 + lane)] = OsTerms<MODE>::term(x, y);
        }
        wave_sync();
        double t[OS_K];
#pragma unroll
        for (int k = 0; k < OS_K; ++k) t[k] = st[lane * (OS_K + 1) + k];
        const OsChunk c = os_chunk(t, sh, normal);
        __syncthreads();
        if (lane == 63) ch[wave] = c;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int w = 0; w < OS_WAVES; ++w) {
                const OsChunk q = ch[w];
                if (q.ok == 2) continue;
                all.ok = q.ok == 1 && all.ok != 0 ? 1 : 0;
                all.lo = fmin(all.lo, all.d + q.lo);
                all.hi = fmax(all.hi, all.d + q.hi);
                all.d += q.d;
            }
    }
    if (threadIdx.x == 0) out[blockIdx.x] = OsBlock{all, sh, 0};
}

template <int MODE>
__global__ __launch_bounds__(OS_BLOCK) void k_os_apply(const u64* __restrict__ r, const double* __restrict__ a,
                                                       const u64* __restrict__ nnz, const double* __restrict__ D,
                                                       u64 span, const OsBlock* __restrict__ blocks, double* out1,
                                                       double* out2) {
    __shared__ OsBlock bl[OS_BLOCKS];
    const u64 n = *nnz;
    const int nb = (int)((n + span - 1) / span);
    for (int t = threadIdx.x; t < nb; t += OS_BLOCK) bl[t] = blocks[t];
    __syncthreads();
    double s = 0.0;
    for (int b = 0; b < nb; ++b) {
        const OsBlock q = bl[b];
        if (q.c.ok == 2) continue;
        int sh;
        if (q.c.ok == 1 && os_normal(s, sh) && sh == q.sh) {
            const double S = ldexp(s, sh);
            if (os_inside(S, q.c.lo, q.c.hi)) {
                s = ldexp(S + q.c.d, -sh);
                continue;
            }
        }
        __syncthreads();  // the last call's LDS
        const u64 e = min(n, (u64)(b + 1) * span);
        s = os_block_sum(e, OsTerms<MODE>{r, a, D, e}, OsTerms<MODE>::term, (u64)b * span, s);
    }
    if (threadIdx.x == 0) {
        *out1 = s;
        if (out2) *out2 = s;
    }
}

// Sparse-sparse products x_i * y(rank_i) (0 where y has no entry), formed
// in parallel; the ordered sum below then adds them in index order.  Adding
// +0 for a missing entry changes nothing: the running sum starts at +0 and
// round-to-nearest never turns it into -0.
__global__ __launch_bounds__(RB) void k_sparse_products(const u64* __restrict__ xr, const double* __restrict__ xa,
                                                        const u64* __restrict__ xn, const u64* __restrict__ yr,
                                                        const double* __restrict__ ya, const u64* __restrict__ yn,
                                                        double* __restrict__ prod) {
    const u64 n = *xn, m = *yn;
    for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)gridDim.x * RB) {
        const double yv = y_at(yr, ya, m, xr[i]);
        prod[i] = (yv != 0.0) ? xa[i] * yv : 0.0;
    }
}

// ---- all dots of one iteration step in one launch ----
// T_lj = <w_l|y> and S_lj = <w_l|w_j> for every l <= j (blockIdx.y = 2 (l - l0)
// for T, + 1 for S): 2 (j + 1) independent reductions over at most a few MB
// each, which take a launch pair each only in launch gaps and in idle compute
// units when issued one by one.  y is dense (indexed by rank) or gathered
// per basis entry (ystride apart per l).
__device__ __forceinline__ double step_y(const StepDots& d, int l, const u64* xr, u64 i) {
    return d.ystride ? d.y[(u64)l * d.ystride + i] : d.y[xr[i]];
}

__device__ __forceinline__ void step_out(const StepDots& d, int l, int s_dot, double v) {
    double* M = s_dot ? d.S : d.T;
    M[l * d.nL + d.j] = v;
    M[d.j * d.nL + l] = v;
}

// fast: the partial sums of the tree reduction, gridDim.x per dot
__global__ __launch_bounds__(RB) void k_step_dots_part(StepDots d, double* __restrict__ part) {
    __shared__ double sh[RB];
    const int l = (int)(blockIdx.y >> 1);
    const u64* xr = d.Wr + (u64)l * d.cap;
    const double* xa = d.Wa + (u64)l * d.cap;
    const u64 n = d.nnz[l];
    double s = 0.0;
    if ((blockIdx.y & 1u) == 0) {
        for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)gridDim.x * RB) s += xa[i] * step_y(d, l, xr, i);
    } else {
        const u64* yr = d.Wr + (u64)d.j * d.cap;
        const double* ya = d.Wa + (u64)d.j * d.cap;
        const u64 m = d.nnz[d.j];
        for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)gridDim.x * RB) {
            const double yv = (l == d.j) ? ya[i] : y_at(yr, ya, m, xr[i]);
            if (yv != 0.0) s += xa[i] * yv;
        }
    }
    const double b = block_sum(s, sh);
    if (threadIdx.x == 0) part[(u64)blockIdx.y * gridDim.x + blockIdx.x] = b;
}

__global__ __launch_bounds__(RB) void k_step_dots_final(StepDots d, const double* __restrict__ part, int np) {
    __shared__ double sh[RB];
    double s = 0.0;
    for (int i = threadIdx.x; i < np; i += RB) s += part[(u64)blockIdx.x * np + i];
    const double b = block_sum(s, sh);
    if (threadIdx.x == 0) step_out(d, (int)(blockIdx.x >> 1), (int)(blockIdx.x & 1u), b);
}

// deterministic: the products of the dots of w_l, l >= l0, in entry order
// (cap apart; 0 where w_j has no entry), ...
__global__ __launch_bounds__(RB) void k_step_products(StepDots d, int l0, double* __restrict__ prod) {
    const int l = l0 + (int)(blockIdx.y >> 1);
    const u64* xr = d.Wr + (u64)l * d.cap;
    const double* xa = d.Wa + (u64)l * d.cap;
    double* out = prod + (u64)blockIdx.y * d.cap;
    const u64 n = d.nnz[l];
    const u64 i0 = (u64)blockIdx.x * RB + threadIdx.x, step = (u64)gridDim.x * RB;
    if ((blockIdx.y & 1u) == 0) {
        for (u64 i = i0; i < n; i += step) out[i] = xa[i] * step_y(d, l, xr, i);
    } else {
        const u64* yr = d.Wr + (u64)d.j * d.cap;
        const double* ya = d.Wa + (u64)d.j * d.cap;
        const u64 m = d.nnz[d.j];
        for (u64 i = i0; i < n; i += step) {
            const double yv = (l == d.j) ? ya[i] : y_at(yr, ya, m, xr[i]);
            out[i] = (yv != 0.0) ? xa[i] * yv : 0.0;
        }
    }
}

// ... and their in-order sums, a workgroup each
__global__ __launch_bounds__(OS_BLOCK) void k_step_ordered(StepDots d, int l0, const double* __restrict__ prod) {
    const int l = l0 + (int)(blockIdx.x >> 1);
    const double* a = prod + (u64)blockIdx.x * d.cap;
    const u64 n = d.nnz[l];
    const double s = os_block_sum(
        n, [&](u64 i, double& x, double& y) { x = (i < n) ? a[i] : 0.0, y = 0.0; }, [](double x, double) { return x; });
    if (threadIdx.x == 0) step_out(d, l, (int)(blockIdx.x & 1u), s);
}

// D[r_i] = D[r_i] - coef * a_i  (SUB)   or   D[r_i] = D[r_i] + coef * a_i  (ADD)
template <bool ADD>
__global__ void k_axpy_scatter(double* __restrict__ D, const u64* __restrict__ r, const double* __restrict__ a,
                               const u64* __restrict__ nnz, const double* __restrict__ coef) {
    const u64 n = *nnz;
    const double c = *coef;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) {
        double prod = c * a[i];
        u64 k = r[i];
        if (ADD) D[k] = D[k] + prod;
        else D[k] = D[k] - prod;
    }
}

__global__ void k_scatter_set(double* __restrict__ D, const u64* __restrict__ r, const double* __restrict__ a,
                              const u64* __restrict__ nnz) {
    const u64 n = *nnz;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) D[r[i]] = a[i];
}

__global__ __launch_bounds__(RB) void k_sumsq_part(const double* __restrict__ a, const u64* __restrict__ nnz,
                                                   double* __restrict__ part) {
    __shared__ double sh[RB];
    const u64 n = *nnz;
    double s = 0.0;
    for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)gridDim.x * RB) s += a[i] * a[i];
    double b = block_sum(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = b;
}

__global__ __launch_bounds__(RB) void k_sum_part(const double* __restrict__ x, const u64* __restrict__ nnz,
                                                 double* __restrict__ part) {
    __shared__ double sh[RB];
    const u64 n = *nnz;
    double s = 0.0;
    for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)gridDim.x * RB) s += x[i];
    double b = block_sum(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = b;
}

// Eq. 11: a_i = a_i / sqrt(sum of squares); untouched when the sum is 0.
__global__ void k_div_norm(double* __restrict__ a, const u64* __restrict__ nnz, const double* __restrict__ ss) {
    const u64 n = *nnz;
    const double s = *ss;
    if (!(s > 0.0)) return;
    const double nrm = sqrt(s);
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) a[i] = a[i] / nrm;
}

// ---- generalized eigenproblem, one wavefront (m <= 32) ----
#define GE_MAX 32

// Cyclic Jacobi on the m x m symmetric matrix A (row-major, stride GE_MAX),
// eigenvectors into V's columns, eigenvalues into w.  Same rotation rule,
// sweep order and stopping rule as the CPU reference.  Lane r updates row r
// of every rotation; the rows are independent, so the results are the same
// bits as a sequential sweep.
__device__ void jacobi_dev(int m, double (*A)[GE_MAX], double (*V)[GE_MAX], double* w, int* flag) {
    const int r = threadIdx.x;
    if (r < m)
        for (int q = 0; q < m; ++q) V[r][q] = (r == q) ? 1.0 : 0.0;
    wave_sync();
    for (int sweep = 0; sweep < 64; ++sweep) {
        if (r == 0) {
            double off = 0.0, dg = 0.0;
            for (int p = 0; p < m; ++p) {
                dg += A[p][p] * A[p][p];
                for (int q = p + 1; q < m; ++q) off += A[p][q] * A[p][q];
            }
            *flag = (off <= 1e-30 * dg) ? 1 : 0;
        }
        wave_sync();
        if (*flag) break;
        for (int p = 0; p < m; ++p)
            for (int q = p + 1; q < m; ++q) {
                const double apq = A[p][q];
                if (apq == 0.0) continue;
                const double app = A[p][p], aqq = A[q][q];
                const double theta = (aqq - app) / (2.0 * apq);
                double t = 1.0 / (fabs(theta) + sqrt(theta * theta + 1.0));
                if (theta < 0.0) t = -t;
                const double c = 1.0 / sqrt(t * t + 1.0);
                const double s = t * c;
                const double tau = s / (1.0 + c);
                const bool row = r < m && r != p && r != q;
                double arp = 0.0, arq = 0.0, vrp = 0.0, vrq = 0.0;
                if (row) {
                    arp = A[r][p];
                    arq = A[r][q];
                }
                if (r < m) {
                    vrp = V[r][p];
                    vrq = V[r][q];
                }
                wave_sync();  // every read of this rotation before any write
                if (r == 0) {
                    A[p][p] = app - t * apq;
                    A[q][q] = aqq + t * apq;
                    A[p][q] = 0.0;
                    A[q][p] = 0.0;
                }
                if (row) {
                    const double nrp = arp - s * (arq + tau * arp);
                    const double nrq = arq + s * (arp - tau * arq);
                    A[r][p] = nrp;
                    A[p][r] = nrp;
                    A[r][q] = nrq;
                    A[q][r] = nrq;
                }
                if (r < m) {
                    V[r][p] = vrp - s * (vrq + tau * vrp);
                    V[r][q] = vrq + s * (vrp - tau * vrq);
                }
                wave_sync();
            }
    }
    if (r < m) w[r] = A[r][r];
    wave_sync();
}

// The same decomposition for fast mode: the rotations of a sweep in rounds of
// floor(m / 2) disjoint pairs (a round robin), a lane per pair, so that a sweep
// is m - 1 dependent steps instead of m (m - 1) / 2.  What a step costs is the
// chain of divisions and square roots of a rotation (~1 000 cycles); 10 x 10:
// 320 -> 118 us for the two decompositions of a block.  Same stopping rule, and
// rotations in the same form, x - s (y + tau x) with tau = s / (1 + c): as
// c x - s y they rounded the lowest eigenvalue of 10 x 10 blocks to 1.1e-15 on
// average, this way to 1.9e-16 (one rotation after another 2.2e-16).
__device__ void jacobi_rounds(int m, double (*A)[GE_MAX], double (*V)[GE_MAX], double* w,
                              double (*st)[2], int (*pq)[2]) {
    const int lane = threadIdx.x;
    for (int e = lane; e < m * m; e += 64) V[e / m][e % m] = (e / m == e % m) ? 1.0 : 0.0;
    const int me = m + (m & 1);  // players, one idle where m is odd
    wave_sync();
    for (int sweep = 0; sweep < 64; ++sweep) {
        double off = 0.0, dg = 0.0;
        for (int e = lane; e < m * m; e += 64) {
            const int p = e / m, q = e % m;
            const double x = A[p][q] * A[p][q];
            if (p == q) dg += x;
            else if (p < q) off += x;
        }
        for (int o = 32; o >= 1; o >>= 1) {
            off += __shfl_xor(off, o);
            dg += __shfl_xor(dg, o);
        }
        if (off <= 1e-30 * dg || m < 2) break;
        for (int round = 0; round < me - 1; ++round) {
            double dp = 0.0, dq = 0.0;  // this lane's pair: its diagonal elements after the rotation
            if (lane < me / 2) {
                // player me - 1 stays, the others move on by one seat per round
                int p = lane == 0 ? me - 1 : (round + lane) % (me - 1);
                int q = lane == 0 ? round : (round + me - 1 - lane) % (me - 1);
                if (p > q) {
                    const int x = p;
                    p = q;
                    q = x;
                }
                double s = 0.0, tau = 0.0;
                if (q < m) {
                    const double apq = A[p][q];
                    dp = A[p][p];
                    dq = A[q][q];
                    if (apq != 0.0) {
                        const double theta = (dq - dp) / (2.0 * apq);
                        double t = 1.0 / (fabs(theta) + sqrt(theta * theta + 1.0));
                        if (theta < 0.0) t = -t;
                        const double c = 1.0 / sqrt(t * t + 1.0);
                        s = t * c;
                        tau = s / (1.0 + c);
                        dp = dp - t * apq;
                        dq = dq + t * apq;
                    }
                }
                pq[lane][0] = p;
                pq[lane][1] = q < m ? q : -1;
                st[lane][0] = s;
                st[lane][1] = tau;
            }
            wave_sync();
            // columns of A and V, then rows of A, by every pair's rotation
            for (int e = lane; e < (me / 2) * m; e += 64) {
                const int k = e / m, r = e % m, p = pq[k][0], q = pq[k][1];
                if (q < 0) continue;
                const double s = st[k][0], tau = st[k][1];
                const double ap = A[r][p], aq = A[r][q], vp = V[r][p], vq = V[r][q];
                A[r][p] = ap - s * (aq + tau * ap);
                A[r][q] = aq + s * (ap - tau * aq);
                V[r][p] = vp - s * (vq + tau * vp);
                V[r][q] = vq + s * (vp - tau * vq);
            }
            wave_sync();
            for (int e = lane; e < (me / 2) * m; e += 64) {
                const int k = e / m, r = e % m, p = pq[k][0], q = pq[k][1];
                if (q < 0) continue;
                const double s = st[k][0], tau = st[k][1];
                const double ap = A[p][r], aq = A[q][r];
                A[p][r] = ap - s * (aq + tau * ap);
                A[q][r] = aq + s * (ap - tau * aq);
            }
            wave_sync();
            if (lane < me / 2 && pq[lane][1] >= 0) {
                const int p = pq[lane][0], q = pq[lane][1];
                A[p][p] = dp;
                A[q][q] = dq;
                A[p][q] = 0.0;
                A[q][p] = 0.0;
            }
            wave_sync();
        }
    }
    if (lane < m) w[lane] = A[lane][lane];
    wave_sync();
}

// Canonical orthogonalisation: S = U s U^T, keep s_k > 1e-10 max s,
// X = U_k s_k^(-1/2), Jacobi on X^T T X, x = X y for the lowest eigenvalue,
// sign fixed so that the largest |x_i| (lowest i on ties) is positive.
// One wavefront; every sum keeps the reference's order.  ORDERED: the
// decompositions too (deterministic mode's bits).
template <bool ORDERED>
__device__ __forceinline__ void geneig_body(int m, const double* __restrict__ T, const double* __restrict__ S,
                                            double* lambda, double* x, double* energy_slot, const int* blk,
                                            int* status) {
    __shared__ double A[GE_MAX][GE_MAX], U[GE_MAX][GE_MAX], X[GE_MAX][GE_MAX], TX[GE_MAX][GE_MAX];
    __shared__ double sv[GE_MAX], lam[GE_MAX], xs[GE_MAX];
    __shared__ int keep[GE_MAX];
    __shared__ int s_r, s_best, s_flag;
    __shared__ double st[GE_MAX / 2][2];
    __shared__ int pq[GE_MAX / 2][2];
    auto jacobi = [&](int k, double* w) {
        if (ORDERED) jacobi_dev(k, A, U, w, &s_flag);
        else jacobi_rounds(k, A, U, w, st, pq);
    };
    const int i = threadIdx.x;
    if (i < m)
        for (int j = 0; j < m; ++j) A[i][j] = S[i * m + j];
    wave_sync();
    jacobi(m, sv);
    if (i == 0) {
        double smax = 0.0;
        for (int k = 0; k < m; ++k)
            if (sv[k] > smax) smax = sv[k];
        int r = 0;
        for (int k = 0; k < m; ++k)
            if (sv[k] > 1e-10 * smax) keep[r++] = k;
        s_r = r;
    }
    wave_sync();
    const int r = s_r;
    if (r == 0) {
        if (i == 0) *status = 1;
        return;
    }
    if (i < m)
        for (int c = 0; c < r; ++c) X[i][c] = U[i][keep[c]] / sqrt(sv[keep[c]]);
    wave_sync();
    if (i < m)
        for (int c = 0; c < r; ++c) {
            double acc = 0.0;
            for (int k = 0; k < m; ++k) acc += T[i * m + k] * X[k][c];
            TX[i][c] = acc;
        }
    wave_sync();
    if (i < r)
        for (int c = 0; c < r; ++c) {
            double acc = 0.0;
            for (int k = 0; k < m; ++k) acc += X[k][i] * TX[k][c];
            A[i][c] = acc;
        }
    wave_sync();
    if (i < r)
        for (int c = i + 1; c < r; ++c) {
            const double v = 0.5 * (A[i][c] + A[c][i]);
            A[i][c] = v;
            A[c][i] = v;
        }
    wave_sync();
    jacobi(r, lam);  // U now holds the eigenvectors y of X^T T X
    if (i == 0) {
        int best = 0;
        for (int k = 1; k < r; ++k)
            if (lam[k] < lam[best]) best = k;
        s_best = best;
    }
    wave_sync();
    const int best = s_best;
    if (i < m) {
        double acc = 0.0;
        for (int c = 0; c < r; ++c) acc += X[i][c] * U[c][best];
        xs[i] = acc;
    }
    wave_sync();
    if (i == 0) {
        int imax = 0;
        for (int k = 1; k < m; ++k)
            if (fabs(xs[k]) > fabs(xs[imax])) imax = k;
        s_flag = xs[imax] < 0.0 ? 1 : 0;
    }
    wave_sync();
    const bool neg = s_flag != 0;
    if (i < m) x[i] = neg ? -xs[i] : xs[i];
    if (i == 0) {
        *lambda = lam[best];
        if (energy_slot) energy_slot[blk ? *blk : 0] = lam[best];
        *status = 0;
    }
}

template <bool ORDERED>
__global__ __launch_bounds__(64) void k_geneig(int m, const double* __restrict__ T, const double* __restrict__ S,
                                               double* lambda, double* x, double* energy_slot, const int* blk,
                                               int* status) {
    geneig_body<ORDERED>(m, T, S, lambda, x, energy_slot, blk, status);
}

unsigned gsz(u64 cap) {
    u64 g = (cap + 255) / 256;
    if (g < 1) g = 1;
    if (g > 16384) g = 16384;
    return (unsigned)g;
}

}  // namespace

// In-order sum of up to cap terms.  From OS_LONG on over the chip: 1e6 squares
// 0.69 ms by one workgroup, 0.14 this way; 1e5 squares with a binade change or
// tie in most blocks 75 and 71 us, so that shorter sums gain nothing.
constexpr u64 OS_LONG = 65536;

template <int MODE>
static void launch_ordered(sfci_problem* P, const u64* r, const double* a, const u64* nnz, u64 cap, const double* D,
                           double* out1, double* out2) {
    if (cap < OS_LONG) {
        hipLaunchKernelGGL(k_ordered<MODE>, dim3(1), dim3(OS_BLOCK), 0, P->stream, r, a, nnz, D, out1, out2);
        return;
    }
    const u64 steps = (cap + OS_STEP - 1) / OS_STEP, per = (steps + OS_BLOCKS - 1) / OS_BLOCKS;
    const u64 span = per * OS_STEP;
    const unsigned nb = (unsigned)((cap + span - 1) / span);
    double* guess = (double*)P->ws_os.get(OS_BLOCKS * (sizeof(double) + sizeof(OsBlock)));
    OsBlock* blocks = (OsBlock*)(guess + OS_BLOCKS);
    hipLaunchKernelGGL(k_os_guess<MODE>, dim3(nb), dim3(OS_BLOCK), 0, P->stream, r, a, nnz, D, span, guess);
    hipLaunchKernelGGL(k_os_blocks<MODE>, dim3(nb), dim3(OS_BLOCK), 0, P->stream, r, a, nnz, D, span,
                       (const double*)guess, blocks);
    hipLaunchKernelGGL(k_os_apply<MODE>, dim3(1), dim3(OS_BLOCK), 0, P->stream, r, a, nnz, D, span,
                       (const OsBlock*)blocks, out1, out2);
}

void launch_dot_dense(sfci_problem* P, const u64* r, const double* a, const u64* nnz, u64 cap, const double* D,
                      double* out1, double* out2, bool ordered) {
    if (ordered) {
        launch_ordered<OS_DOT>(P, r, a, nnz, cap, D, out1, out2);
    } else {
        double* part = (double*)P->ws_red.get(RGRID * sizeof(double));
        unsigned g = std::min<unsigned>(RGRID, gsz(cap));
        hipLaunchKernelGGL(k_dot_dense_part, dim3(g), dim3(RB), 0, P->stream, r, a, nnz, D, part);
        hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(RB), 0, P->stream, part, (int)g, out1, out2);
    }
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_sum(sfci_problem* P, const double* x, const u64* nnz, u64 cap, double* out, bool ordered) {
    if (ordered) {
        launch_ordered<OS_SUM>(P, nullptr, x, nnz, cap, nullptr, out, nullptr);
    } else {
        double* part = (double*)P->ws_red.get(RGRID * sizeof(double));
        unsigned g = std::min<unsigned>(RGRID, gsz(cap));
        hipLaunchKernelGGL(k_sum_part, dim3(g), dim3(RB), 0, P->stream, x, nnz, part);
        hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(RB), 0, P->stream, part, (int)g, out, (double*)nullptr);
    }
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_sumsq(sfci_problem* P, const double* a, const u64* nnz, u64 cap, double* out, bool ordered) {
    if (ordered) {
        launch_ordered<OS_SUMSQ>(P, nullptr, a, nnz, cap, nullptr, out, nullptr);
    } else {
        double* part = (double*)P->ws_red.get(RGRID * sizeof(double));
        unsigned g = std::min<unsigned>(RGRID, gsz(cap));
        hipLaunchKernelGGL(k_sumsq_part, dim3(g), dim3(RB), 0, P->stream, a, nnz, part);
        hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(RB), 0, P->stream, part, (int)g, out, (double*)nullptr);
    }
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_dot_sparse(sfci_problem* P, const u64* xr, const double* xa, const u64* xn, u64 xcap, const u64* yr,
                       const double* ya, const u64* yn, double* out1, double* out2, bool ordered) {
    if (ordered) {
        double* prod = (double*)P->ws_prod.get(std::max<u64>(1, xcap) * sizeof(double));
        hipLaunchKernelGGL(k_sparse_products, dim3(gsz(xcap)), dim3(RB), 0, P->stream, xr, xa, xn, yr, ya, yn, prod);
        launch_ordered<OS_SUM>(P, nullptr, prod, xn, xcap, nullptr, out1, out2);
    } else {
        double* part = (double*)P->ws_red.get(RGRID * sizeof(double));
        unsigned g = std::min<unsigned>(RGRID, gsz(xcap));
        hipLaunchKernelGGL(k_dot_sparse_part, dim3(g), dim3(RB), 0, P->stream, xr, xa, xn, yr, ya, yn, part);
        hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(RB), 0, P->stream, part, (int)g, out1, out2);
    }
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_step_dots(sfci_problem* P, const StepDots& d, bool ordered) {
    const unsigned g = std::min<unsigned>(RGRID, gsz(d.cap));
    if (!ordered) {
        double* part = (double*)P->ws_red.get((size_t)2 * d.nL * RGRID * sizeof(double));
        hipLaunchKernelGGL(k_step_dots_part, dim3(g, 2 * (d.j + 1)), dim3(RB), 0, P->stream, d, part);
        hipLaunchKernelGGL(k_step_dots_final, dim3(2 * (d.j + 1)), dim3(RB), 0, P->stream, d, part, (int)g);
    } else {
        // as many w_l at a time as their products fit in 256 MiB (at least one)
        const u64 fit = (256ull << 20) / (2 * std::max<u64>(1, d.cap) * sizeof(double));
        const int group = (int)std::max<u64>(1, std::min<u64>(fit, (u64)d.nL));
        double* prod = (double*)P->ws_prod.get((size_t)2 * group * std::max<u64>(1, d.cap) * sizeof(double));
        for (int l0 = 0; l0 <= d.j; l0 += group) {
            const unsigned dots = 2u * (unsigned)std::min(group, d.j + 1 - l0);
            hipLaunchKernelGGL(k_step_products, dim3(g, dots), dim3(RB), 0, P->stream, d, l0, prod);
            hipLaunchKernelGGL(k_step_ordered, dim3(dots), dim3(OS_BLOCK), 0, P->stream, d, l0, prod);
        }
    }
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_axpy_scatter(sfci_problem* P, double* D, const u64* r, const double* a, const u64* nnz, u64 cap,
                         const double* coef, double sign) {
    if (sign > 0)
        hipLaunchKernelGGL(k_axpy_scatter<true>, dim3(gsz(cap)), dim3(256), 0, P->stream, D, r, a, nnz, coef);
    else
        hipLaunchKernelGGL(k_axpy_scatter<false>, dim3(gsz(cap)), dim3(256), 0, P->stream, D, r, a, nnz, coef);
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_scatter_set(sfci_problem* P, double* D, const u64* r, const double* a, const u64* nnz, u64 cap) {
    hipLaunchKernelGGL(k_scatter_set, dim3(gsz(cap)), dim3(256), 0, P->stream, D, r, a, nnz);
    SFCI_CHECK_HIP(hipGetLastError());
}

u64 normalise_ws_doubles() { return RGRID + 8; }

void launch_normalise(sfci_problem* P, double* a, const u64* nnz, u64 cap, bool ordered, double* part_ws) {
    double* part = part_ws ? part_ws : (double*)P->ws_red.get((RGRID + 8) * sizeof(double));
    double* ss = part + RGRID;
    if (ordered) {
        if (part_ws)  // the caller's scratch holds no more
            hipLaunchKernelGGL(k_ordered<OS_SUMSQ>, dim3(1), dim3(OS_BLOCK), 0, P->stream, (const u64*)nullptr, a, nnz,
                               (const double*)nullptr, ss, (double*)nullptr);
        else launch_ordered<OS_SUMSQ>(P, nullptr, a, nnz, cap, nullptr, ss, nullptr);
    } else {
        unsigned g = std::min<unsigned>(RGRID, gsz(cap));
        hipLaunchKernelGGL(k_sumsq_part, dim3(g), dim3(RB), 0, P->stream, a, nnz, part);
        hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(RB), 0, P->stream, part, (int)g, ss, (double*)nullptr);
    }
    hipLaunchKernelGGL(k_div_norm, dim3(gsz(cap)), dim3(256), 0, P->stream, a, nnz, ss);
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_geneig_full(sfci_problem* P, int m, const double* T, const double* S, double* lambda, double* x,
                        double* energy_slot, int* status, bool ordered, const int* blk) {
    hipLaunchKernelGGL(ordered ? k_geneig<true> : k_geneig<false>, dim3(1), dim3(64), 0, P->stream, m, T, S, lambda,
                       x, energy_slot, blk, status);
    SFCI_CHECK_HIP(hipGetLastError());
}

namespace {
__global__ void k_inc_int(int* p) {
    if (threadIdx.x == 0) *p += 1;
}
__global__ void k_screen(double* __restrict__ D, u64 n, double eps) {
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) {
        const double v = D[i];
        if (v != 0.0 && fabs(v) < eps) D[i] = 0.0;
    }
}
__global__ void k_add_u64(u64* dst, const u64* src) {
    if (threadIdx.x == 0) *dst += *src;
}
__global__ void k_scale_copy(const double* __restrict__ a, const u64* __restrict__ nnz, const double* __restrict__ ss,
                             double* __restrict__ out) {
    const u64 n = *nnz;
    const double s = *ss;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x)
        out[i] = (s > 0.0) ? a[i] / s : 0.0;
}
}  // namespace

void launch_inc_int(sfci_problem* P, int* p) {
    hipLaunchKernelGGL(k_inc_int, dim3(1), dim3(64), 0, P->stream, p);
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_screen(sfci_problem* P, double* D, u64 n, double eps) {
    hipLaunchKernelGGL(k_screen, dim3(gsz(n)), dim3(256), 0, P->stream, D, n, eps);
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_add_u64(sfci_problem* P, u64* dst, const u64* src) {
    hipLaunchKernelGGL(k_add_u64, dim3(1), dim3(64), 0, P->stream, dst, src);
    SFCI_CHECK_HIP(hipGetLastError());
}

// out = a / sum(a^2) (the cotangent of the Rayleigh quotient's numerator).
void launch_div_by_sumsq(sfci_problem* P, const double* a, const u64* nnz, u64 cap, double* out) {
    double* part = (double*)P->ws_red.get((RGRID + 8) * sizeof(double));
    double* ss = part + RGRID + 1;
    unsigned g = std::min<unsigned>(RGRID, gsz(cap));
    hipLaunchKernelGGL(k_sumsq_part, dim3(g), dim3(RB), 0, P->stream, a, nnz, part);
    hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(RB), 0, P->stream, part, (int)g, ss, (double*)nullptr);
    hipLaunchKernelGGL(k_scale_copy, dim3(gsz(cap)), dim3(256), 0, P->stream, a, nnz, ss, out);
    SFCI_CHECK_HIP(hipGetLastError());
}

// ---- batched steps: every instance of a batch in one launch (blockIdx.y or
// blockIdx.z picks the instance).  The same products and sums as the
// per-instance fast reductions above, over a fixed grid of BG partials.
namespace {

constexpr unsigned BG = 256;  // partial sums per dot

__device__ __forceinline__ void bvec(const BInst& b, int l, const u64*& r, const double*& a, u64& n) {
    r = b.Wr + (u64)l * b.cap;
    a = b.Wa + (u64)l * b.cap;
    n = b.sc[l];
}

__device__ __forceinline__ int bout_index(int kind, int j) { return kind == BOUT_W0 ? 0 : j + 1; }

// grid (BG, 2 (j + 1), n): y = 2 l, <w_l|D>; y = 2 l + 1, <w_l|w_j>
__global__ __launch_bounds__(RB) void k_bdot_part(const BInst* __restrict__ B, int j) {
    const BInst& b = B[blockIdx.z];
    __shared__ double sh[RB];
    const int l = (int)(blockIdx.y >> 1);
    const u64* xr;
    const double* xa;
    u64 nx;
    bvec(b, l, xr, xa, nx);
    double s = 0.0;
    if ((blockIdx.y & 1u) == 0) {
        for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < nx; i += (u64)BG * RB) s += xa[i] * b.D[xr[i]];
    } else {
        const u64* yr;
        const double* ya;
        u64 ny;
        bvec(b, j, yr, ya, ny);
        for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < nx; i += (u64)BG * RB) {
            const double yv = y_at(yr, ya, ny, xr[i]);
            if (yv != 0.0) s += xa[i] * yv;
        }
    }
    const double t = block_sum(s, sh);
    if (threadIdx.x == 0) b.red[(u64)blockIdx.y * BG + blockIdx.x] = t;
}

// grid (2 (j + 1), n): the BG partials of each dot into T or S (both triangles)
__global__ __launch_bounds__(RB) void k_bdot_final(const BInst* __restrict__ B, int j) {
    const BInst& b = B[blockIdx.y];
    __shared__ double sh[RB];
    double s = 0.0;
    for (unsigned i = threadIdx.x; i < BG; i += RB) s += b.red[(u64)blockIdx.x * BG + i];
    const double t = block_sum(s, sh);
    if (threadIdx.x == 0) {
        const int l = (int)(blockIdx.x >> 1);
        double* M = (blockIdx.x & 1u) ? b.S : b.T;
        M[l * b.nL + j] = t;
        M[j * b.nL + l] = t;
    }
}

// kind 0: D[r_i] = D[r_i] - T[l][j] a_i;  kind 1: D[r_i] = D[r_i] + x[l] a_i
__global__ void k_baxpy(const BInst* __restrict__ B, int l, int j, int kind) {
    const BInst& b = B[blockIdx.y];
    const u64* r;
    const double* a;
    u64 n;
    bvec(b, l, r, a, n);
    const double c = kind ? b.x[l] : b.T[l * b.nL + j];
    double* D = b.D;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) {
        const double prod = c * a[i];
        const u64 k = r[i];
        if (kind) D[k] = D[k] + prod;
        else D[k] = D[k] - prod;
    }
}

// Eq. 11 on w_{j+1} (or w_0): partial sums of squares, their sum, the division
__global__ __launch_bounds__(RB) void k_bsumsq_part(const BInst* __restrict__ B, int kind, int j) {
    const BInst& b = B[blockIdx.y];
    __shared__ double sh[RB];
    const u64* r;
    const double* a;
    u64 n;
    bvec(b, bout_index(kind, j), r, a, n);
    double s = 0.0;
    for (u64 i = (u64)blockIdx.x * RB + threadIdx.x; i < n; i += (u64)BG * RB) s += a[i] * a[i];
    const double t = block_sum(s, sh);
    if (threadIdx.x == 0) b.red[(u64)2 * b.nL * BG + blockIdx.x] = t;
}

__global__ __launch_bounds__(RB) void k_bsumsq_final(const BInst* __restrict__ B) {
    const BInst& b = B[blockIdx.y];
    __shared__ double sh[RB];
    const double* part = b.red + (u64)2 * b.nL * BG;
    double s = 0.0;
    for (unsigned i = threadIdx.x; i < BG; i += RB) s += part[i];
    const double t = block_sum(s, sh);
    if (threadIdx.x == 0) b.red[(u64)2 * b.nL * BG + BG] = t;
}

__global__ void k_bdiv(const BInst* __restrict__ B, int kind, int j) {
    const BInst& b = B[blockIdx.y];
    const double ss = b.red[(u64)2 * b.nL * BG + BG];
    if (!(ss > 0.0)) return;
    const double nrm = sqrt(ss);
    const int l = bout_index(kind, j);
    double* a = b.Wa + (u64)l * b.cap;
    const u64 n = b.sc[l];
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) a[i] = a[i] / nrm;
}

__global__ void k_bfill_zero(const BInst* __restrict__ B) {
    const BInst& b = B[blockIdx.y];
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < b.Ndet; i += (u64)gridDim.x * blockDim.x) b.D[i] = 0.0;
}

__global__ __launch_bounds__(64) void k_bgeneig(const BInst* __restrict__ B, int m) {
    const BInst& b = B[blockIdx.y];
    geneig_body<false>(m, b.T, b.S, b.lam, b.x, b.energies, b.blk, b.status);
}

__global__ void k_binc_blk(const BInst* __restrict__ B) {
    if (threadIdx.x == 0) *B[blockIdx.y].blk += 1;
}

unsigned bgrid(u64 n, u64 per, u64 cap) {
    u64 g = (n + per - 1) / per;
    return (unsigned)std::max<u64>(1, std::min<u64>(g, cap));
}

}  // namespace

u64 bstep_red_doubles(int nL) { return (u64)2 * nL * BG + BG + 8; }

void bstep_dots(hipStream_t st, const BInst* d, int n, int j, int nL) {
    (void)nL;
    hipLaunchKernelGGL(k_bdot_part, dim3(BG, 2 * (j + 1), n), dim3(RB), 0, st, d, j);
    hipLaunchKernelGGL(k_bdot_final, dim3(2 * (j + 1), n), dim3(RB), 0, st, d, j);
    SFCI_CHECK_HIP(hipGetLastError());
}

void bstep_axpy(hipStream_t st, const BInst* d, int n, int l, int j, int kind, u64 max_cap) {
    hipLaunchKernelGGL(k_baxpy, dim3(bgrid(max_cap, 256, 16384), n), dim3(256), 0, st, d, l, j, kind);
    SFCI_CHECK_HIP(hipGetLastError());
}

void bstep_normalise(hipStream_t st, const BInst* d, int n, int out_kind, int j, u64 max_cap) {
    hipLaunchKernelGGL(k_bsumsq_part, dim3(BG, n), dim3(RB), 0, st, d, out_kind, j);
    hipLaunchKernelGGL(k_bsumsq_final, dim3(1, n), dim3(RB), 0, st, d);
    hipLaunchKernelGGL(k_bdiv, dim3(bgrid(max_cap, 256, 16384), n), dim3(256), 0, st, d, out_kind, j);
    SFCI_CHECK_HIP(hipGetLastError());
}

void bstep_fill_zero(hipStream_t st, const BInst* d, int n, u64 max_ndet) {
    hipLaunchKernelGGL(k_bfill_zero, dim3(bgrid(max_ndet, 256 * 16, 65535), n), dim3(256), 0, st, d);
    SFCI_CHECK_HIP(hipGetLastError());
}

void bstep_geneig(hipStream_t st, const BInst* d, int n, int nL) {
    hipLaunchKernelGGL(k_bgeneig, dim3(1, n), dim3(64), 0, st, d, nL);
    SFCI_CHECK_HIP(hipGetLastError());
}

void bstep_inc_blk(hipStream_t st, const BInst* d, int n) {
    hipLaunchKernelGGL(k_binc_blk, dim3(1, n), dim3(64), 0, st, d);
    SFCI_CHECK_HIP(hipGetLastError());
}
