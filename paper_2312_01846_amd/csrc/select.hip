// Truncation to the M largest amplitudes (Sec. 2.1, Eqs. 10-11; the paper
// sorts the whole intermediate vector, Sec. 3).  Here: a radix select over
// the 128-bit key K = bits(|c|) ++ (N_det - 1 - rank), which orders entries by
// |c| descending and breaks exact ties by rank ascending, followed by an
// order-preserving compaction that writes the kept entries by rank.  Exactly
// min(M, nonzero) entries are kept, unless the problem's tie_band extension is
// on (then entries within a relative 2^-36 of the M-th |c| stay too, at most
// SFCI_TIE_SLACK of them).
//
// Steps (every pass a streaming read; launches end in a "last workgroup" that
// does the single-workgroup part, so that none is launched for it):
//   1. histogram of the top digit (the exponent), pick the M-th entry's;
//   2. dense sources: the entries at or above that binade go to fixed
//      segments (a segment per chunk of slots, no scan needed), the
//      accumulator is zeroed on the way;
//   3. histogram of the next 11 bits over the segments, pick;
//   4. the few entries that share those 22 bits are gathered and the M-th key
//      is found among them by counting; where they are many (ties in masses)
//      the remaining digits are picked one histogram at a time instead;
//   5. kept entries per segment, their scan; 6. the compaction.
// Sources of at most SEL_ONE entries are done by one workgroup in one launch.
// Measured (a histogram of every digit over the whole source, before -> now):
// 2.35e7 slots, M = 9e5: 450 -> 240 us; 4.33e9 slots, M = 1e6: 41 -> 20.5 ms;
// a list of 4e6, M = 1e6: 215 -> 110 us.
#include <algorithm>

#include "../../include/sfci.h"
#include "sfci_internal.h"

namespace {

typedef unsigned __int128 u128;

constexpr int DIG = 11;
constexpr int NBIN = 1 << DIG;
constexpr int CBLOCK = 256;
constexpr int CITEMS = 16;
constexpr u64 CCHUNK = (u64)CBLOCK * CITEMS;
constexpr int SEG_UNROLL = 4;  // groups of 64 entries whose loads are in flight together
constexpr int ONE_BLOCK = 1024;
constexpr int ONE_ITEMS = SEL_ONE / ONE_BLOCK;
constexpr int SEG_BLOCK = 1024;  // threads of the segment passes that end in histograms or gathers

struct Geo {
    int tb;    // total key bits = 63 + rank_bits
    int ndig;  // ceil(tb / 11)
    u64 ndet_m1;
    int rank_bits;
};

__host__ __device__ __forceinline__ Geo geo_of(int rank_bits, u64 ndet_m1) {
    Geo g;
    g.rank_bits = rank_bits;
    g.tb = 63 + rank_bits;
    g.ndig = (g.tb + DIG - 1) / DIG;
    g.ndet_m1 = ndet_m1;
    return g;
}

__device__ __forceinline__ u64 abs_bits(double c) { return (u64)__double_as_longlong(c) & 0x7FFFFFFFFFFFFFFFull; }

__device__ __forceinline__ u128 sel_key(u64 rank, double c, const Geo& g) {
    return ((u128)abs_bits(c) << g.rank_bits) | (u128)(g.ndet_m1 - rank);
}

__device__ __forceinline__ int dig_lo(const Geo& g, int L) {
    int lo = g.tb - DIG * (L + 1);
    return lo < 0 ? 0 : lo;
}

// One selection.  Candidates lie in segments: segment s holds count(s) entries
// from (s << shift) on, cnt[s] of them (dense source), or a list's own
// stretch of *n entries in all (cnt == nullptr).
struct SelJob {
    const double* D;  // dense source (rank = index) of Dn slots, nullptr: the list itself
    u64 Dn;
    const u64* r;
    const double* a;
    u32* cnt;
    const u64* n;
    u64 cap;   // slots (dense) or the list's capacity: nseg() segments
    int shift;
    u64* off;  // per segment: kept entries, then their exclusive scan
    SelState* st;
    u64 M;
    int band;
    Geo g;
    u64* out_r;
    double* out_a;
    u64* out_n;  // may be nullptr
    double* Dz;  // the accumulator to zero on the way, or nullptr
    __device__ __forceinline__ u64 nseg() const { return (cap + (1ull << shift) - 1) >> shift; }
    __device__ __forceinline__ u32 count(u64 s) const {
        if (cnt) return cnt[s];
        const u64 m = *n, b = s << shift;
        return b >= m ? 0u : (u32)min((u64)1 << shift, m - b);
    }
    __device__ __forceinline__ bool all() const { return M == UINT64_MAX; }
};

// Where a launch's jobs come from: one by value, or a batch's instances
// (blockIdx.y).
struct OneJob {
    SelJob j;
    __device__ __forceinline__ SelJob operator()(unsigned) const { return j; }
};

struct BatchJobs {
    const BInst* B;
    int kind, j, band, all, zero;
    __device__ __forceinline__ SelJob operator()(unsigned y) const {
        const BInst& b = B[y];
        SelJob s;
        s.D = b.D;
        s.Dn = b.Ndet;
        s.r = b.cr;
        s.a = b.ca;
        s.cnt = b.ccnt;
        s.n = nullptr;
        s.cap = b.Ndet;
        s.shift = SEL_DENSE_SHIFT;
        s.off = b.cnt;
        s.st = b.st;
        s.M = all ? UINT64_MAX : b.M;
        s.band = band;
        s.g = geo_of(b.rank_bits, b.ndet_m1);
        if (kind == BOUT_PSI) {
            s.out_r = b.psi_r;
            s.out_a = b.psi_a;
            s.out_n = b.psi_n;
        } else {
            const u64 l = kind == BOUT_W0 ? 0 : (u64)j + 1;
            s.out_r = b.Wr + l * b.cap;
            s.out_a = b.Wa + l * b.cap;
            s.out_n = b.sc + l;
        }
        s.Dz = zero ? b.D : nullptr;
        return s;
    }
};

// Words that one workgroup leaves for the last one of the same launch go
// through agent-scope atomics on both sides (they bypass the caches that are
// not shared): a __threadfence() per workgroup instead writes back and drops a
// whole L2 each time (0.1 us per workgroup, 0.5 ms in a launch of 5 740).
__device__ __forceinline__ u64 shared_load(const u64* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shared_store(u64* p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True in every thread of the workgroup that is the last of `total` to get
// here.  The atomics every wavefront issued before are complete by then.
__device__ __forceinline__ bool last_workgroup(unsigned* ticket, unsigned total) {
    __shared__ unsigned s_t;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) s_t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const bool last = s_t == total - 1;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    return last;
}

template <class JP>
__global__ __launch_bounds__(256) void k_sel_init(JP jp) {
    const SelJob J = jp(blockIdx.y);
    SelState* st = J.st;
    for (int t = threadIdx.x; t < NBIN; t += blockDim.x) st->hist[t] = 0;
    if (threadIdx.x == 0) {
        st->need = J.M;
        st->pre_hi = 0;
        st->pre_lo = 0;
        st->level = 0;
        st->done = (J.all() || J.M == 0) ? 1 : 0;
        st->take_all = J.all() ? 1 : 0;
        st->total = 0;
        st->count_out = 0;
        st->count_thr = 0;
        st->cmin = ~0ull;
        st->key_hi = ~0ull;  // above every key: nothing is kept
        st->key_lo = ~0ull;
        st->thr_bits = ~0ull;
        st->use_thr = 0;
        st->cand_bits = J.all() ? 1ull : ~0ull;
        st->bin = 0;
        st->small_n = 0;
        for (int k = 0; k < SEL_TICKETS; ++k) st->ticket[k] = 0;
    }
}

// A workgroup's counts of a digit, flushed to the state's histogram.
__device__ __forceinline__ void hist_flush(SelState* st, unsigned bin, u32 c) {
    if (c) atomicAdd((unsigned long long*)&st->hist[bin], (unsigned long long)c);
}

// Counts of exponents: neighbouring entries share a few of them, so the 256
// around 1 have 16 copies each side by side (16 lanes hitting one word cost
// 16 turns); the others one.
struct ExpHist {
    static constexpr int LO = 1023 - 200, WIN = 256, R = 16;
    u32* h;  // WIN * R, then NBIN
    __device__ __forceinline__ void clear() {
        for (int t = threadIdx.x; t < WIN * R + NBIN; t += blockDim.x) h[t] = 0;
    }
    __device__ __forceinline__ void add(double c) {
        const unsigned e = (unsigned)(abs_bits(c) >> 52), w = e - (unsigned)LO;
        atomicAdd(w < (unsigned)WIN ? &h[w * R + (threadIdx.x & (R - 1))] : &h[WIN * R + e], 1u);
    }
    __device__ __forceinline__ void flush(SelState* st) {
        for (int t = threadIdx.x; t < NBIN; t += blockDim.x) {
            u32 c = h[WIN * R + t];
            const unsigned w = (unsigned)t - (unsigned)LO;
            if (w < (unsigned)WIN)
                for (int k = 0; k < R; ++k) c += h[w * R + k];
            hist_flush(st, (unsigned)t, c);
        }
    }
};

// The M-th key is known: what is kept, and the tie band's threshold.
__device__ __forceinline__ void sel_decide(SelState* st, u128 K, const Geo& g) {
    st->key_hi = (u64)(K >> 64);
    st->key_lo = (u64)K;
    st->cmin = (u64)(K >> g.rank_bits);
    st->thr_bits = abs_bits(__longlong_as_double((long long)st->cmin) * (1.0 - 1.0 / 68719476736.0));
    st->done = 1;
}

// Digit of level L: the largest d >= 1 whose bins d.. hold at least `need`
// entries (else 0), a suffix scan over the histogram by one workgroup of at
// least 256 threads (the first 256 work); the histogram is cleared.  At level
// 0 also the total, and the bound of a dense source's candidates.
constexpr int PICK_T = 256;
constexpr int PICK_PER = NBIN / PICK_T;
__device__ __forceinline__ void sel_pick(SelState* st, const SelJob& J, int L) {
    __shared__ u64 wtot[PICK_T / 64];
    __shared__ int s_d;
    __shared__ u64 s_acc, s_hd;
    const Geo g = J.g;
    const int t = threadIdx.x, lane = t & 63;
    const bool on = t < PICK_T;
    u64 h[PICK_PER];
    u64 mine = 0;
    if (on)
        for (int k = 0; k < PICK_PER; ++k) {
            h[k] = shared_load(&st->hist[t * PICK_PER + k]);
            mine += h[k];
        }
    u64 suf = mine;  // suffix sum within the wavefront, then over the wavefronts
    if (on) {
        for (int off = 1; off < 64; off <<= 1) {
            const u64 y = (u64)__shfl_down((long long)suf, off);
            if (lane + off < 64) suf += y;
        }
        if (lane == 0) wtot[t >> 6] = suf;
    }
    if (t == 0) {
        s_d = 0;
        s_acc = 0;
        s_hd = 0;
    }
    __syncthreads();
    u64 total = 0;
    for (int w = 0; w < PICK_T / 64; ++w) total += wtot[w];
    const u64 need = st->need;
    if (on) {
        u64 above = suf - mine;
        for (int w = (t >> 6) + 1; w < PICK_T / 64; ++w) above += wtot[w];
        u64 incl = above;  // entries in bins > the current one
        for (int k = PICK_PER - 1; k >= 0; --k) {
            const int b = t * PICK_PER + k;
            const u64 hi = incl;
            incl += h[k];
            if ((b >= 1 && incl >= need && hi < need) || (b == 0 && hi < need)) {
                s_d = b;
                s_acc = hi;
                s_hd = h[k];
            }
        }
        for (int k = 0; k < PICK_PER; ++k) st->hist[t * PICK_PER + k] = 0;
    }
    __syncthreads();
    if (t != 0) return;
    if (L == 0) {
        st->total = total;
        if (total <= J.M) {
            st->take_all = 1;
            st->done = 1;
            st->cand_bits = 1;
            return;
        }
    }
    const int d = s_d;
    st->need = need - s_acc;
    st->bin = s_hd;
    const int width = (g.tb - DIG * L) - dig_lo(g, L);
    const u128 pre = ((((u128)st->pre_hi) << 64 | st->pre_lo) << width) | (u128)(unsigned)d;
    st->pre_hi = (u64)(pre >> 64);
    st->pre_lo = (u64)pre;
    st->level = L + 1;
    if (L == 0) {
        // every entry that can still be kept has |c| >= 2^e, e the binade of
        // the M-th |c| (with the tie band: >= 2^e (1 - 2^-36))
        const u64 lo = (u64)d << 52;
        st->cand_bits = d == 0 ? 1ull
                        : J.band ? abs_bits(__longlong_as_double((long long)lo) * (1.0 - 1.0 / 68719476736.0))
                                 : lo;
    }
    if (L == g.ndig - 1) sel_decide(st, pre, g);  // every digit fixed
}

// Step 1 on a dense source.  Bound by the read of the accumulator (188 MB per
// 20-orbital instance).
template <class JP>
__global__ __launch_bounds__(512) void k_sel_hist0_dense(JP jp) {
    __shared__ u32 hb[ExpHist::WIN * ExpHist::R + NBIN];
    const SelJob J = jp(blockIdx.y);
    if (J.st->done) return;
    ExpHist H{hb};
    H.clear();
    __syncthreads();
    const u64 n = J.Dn, step = (u64)gridDim.x * blockDim.x;
    u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 7 * step < n; i += 8 * step) {
        double c[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = J.D[i + (u64)k * step];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (c[k] != 0.0) H.add(c[k]);
    }
    for (; i < n; i += step) {
        const double c = J.D[i];
        if (c != 0.0) H.add(c);
    }
    __syncthreads();
    H.flush(J.st);
    if (last_workgroup(&J.st->ticket[0], gridDim.x)) sel_pick(J.st, J, 0);
}

// Step 2: a workgroup per chunk of slots.  Chunk order and slot order are rank
// order, so the segments are rank-ordered without a scan over the chunks.
template <class JP>
__global__ __launch_bounds__(CBLOCK) void k_sel_collect(JP jp) {
    const SelJob J = jp(blockIdx.y);
    const u64 base = (u64)blockIdx.x * CCHUNK;
    if (base >= J.Dn) return;
    __shared__ unsigned c64[64];  // entries of (item k, wavefront w) at 4 k + w, then their exclusive scan
    const u64 bound = J.st->cand_bits;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[CITEMS];
#pragma unroll
    for (int k = 0; k < CITEMS; ++k) {
        const u64 i = base + (u64)k * CBLOCK + threadIdx.x;
        v[k] = i < J.Dn ? J.D[i] : 0.0;
    }
    u64 m[CITEMS];
#pragma unroll
    for (int k = 0; k < CITEMS; ++k) {
        m[k] = __ballot(v[k] != 0.0 && abs_bits(v[k]) >= bound);
        if (lane == 0) c64[k * (CBLOCK / 64) + wave] = (unsigned)__popcll(m[k]);
        if (J.Dz && v[k] != 0.0) J.Dz[base + (u64)k * CBLOCK + threadIdx.x] = 0.0;
    }
    static_assert(CITEMS * (CBLOCK / 64) == 64, "one count per lane");
    __syncthreads();
    if (wave == 0) {
        const unsigned c = c64[lane];
        unsigned inc = c;
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned y = __shfl_up(inc, off);
            if (lane >= off) inc += y;
        }
        c64[lane] = inc - c;
        if (lane == 63) J.cnt[blockIdx.x] = inc;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CITEMS; ++k) {
        if ((m[k] >> lane) & 1u) {
            const u64 at = base + c64[k * (CBLOCK / 64) + wave] + __popcll(m[k] & ((1ull << lane) - 1ull));
            const_cast<u64*>(J.r)[at] = base + (u64)k * CBLOCK + threadIdx.x;
            const_cast<double*>(J.a)[at] = v[k];
        }
    }
}

// fn(rank, value) for every entry, wavefronts over the segments.
template <class F>
__device__ __forceinline__ void for_segments(const SelJob& J, F&& fn) {
    const u64 ns = J.nseg();
    const u64 nw = (u64)gridDim.x * (blockDim.x >> 6);
    const int lane = threadIdx.x & 63;
    for (u64 s = (u64)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); s < ns; s += nw) {
        const u32 m = J.count(s);
        const u64 b = s << J.shift;
        for (u32 i0 = 0; i0 < m; i0 += 64 * SEG_UNROLL) {
            u64 r[SEG_UNROLL];
            double c[SEG_UNROLL];
#pragma unroll
            for (int u = 0; u < SEG_UNROLL; ++u) {
                const u32 i = i0 + (u32)u * 64 + lane;
                r[u] = 0;
                c[u] = 0.0;
                if (i < m) {
                    r[u] = J.r[b + i];
                    c[u] = J.a[b + i];
                }
            }
#pragma unroll
            for (int u = 0; u < SEG_UNROLL; ++u)
                if (c[u] != 0.0) fn(r[u], c[u]);
        }
    }
}

// Step 1 on a list.
template <class JP>
__global__ __launch_bounds__(SEG_BLOCK) void k_sel_hist0(JP jp) {
    __shared__ u32 hb[ExpHist::WIN * ExpHist::R + NBIN];
    const SelJob J = jp(blockIdx.y);
    if (J.st->done) return;
    ExpHist H{hb};
    H.clear();
    __syncthreads();
    for_segments(J, [&](u64, double c) { H.add(c); });
    __syncthreads();
    H.flush(J.st);
    if (last_workgroup(&J.st->ticket[0], gridDim.x)) sel_pick(J.st, J, 0);
}

// Step 3 and the remaining digits: histogram of digit L among the entries that
// share the digits above, pick (nothing once the key is known).  Large
// workgroups: every one flushes up to 2 048 bins with global atomics.
template <class JP>
__global__ __launch_bounds__(SEG_BLOCK) void k_sel_hist(JP jp, int L) {
    __shared__ u32 hb[NBIN];
    const SelJob J = jp(blockIdx.y);
    SelState* st = J.st;
    if (st->done || L >= J.g.ndig) return;
    for (int t = threadIdx.x; t < NBIN; t += blockDim.x) hb[t] = 0;
    __syncthreads();
    const u128 pre = ((u128)st->pre_hi << 64) | st->pre_lo;
    const int lo = dig_lo(J.g, L), hi_sh = J.g.tb - DIG * L;
    for_segments(J, [&](u64 r, double c) {
        const u128 K = sel_key(r, c, J.g);
        if ((K >> hi_sh) == pre) atomicAdd(&hb[(unsigned)((K >> lo) & (u128)(NBIN - 1))], 1u);
    });
    __syncthreads();
    for (int t = threadIdx.x; t < NBIN; t += blockDim.x) hist_flush(st, (unsigned)t, hb[t]);
    if (last_workgroup(&st->ticket[L], gridDim.x)) sel_pick(st, J, L);
}

// LDS of block_kth.
struct KthLds {
    u32 hist[NBIN];
    u64 p[64], q[64];
    u64 wsum[ONE_BLOCK / 64];
    u64 need, pre, kp, kq;
    u32 bin, n;
};

// A key's two halves: the bits of |c| (63) and N_det - 1 - rank.
struct KeyPair {
    u64 p, q;
};

// The need-th largest key of a workgroup's keys (each(f) calls f(p, q) for the
// keys of the calling thread; those that do not start with the digits pre
// above level L are skipped): digit by digit, first of the magnitude (levels
// 0 to 5: 11 bits, the last 8), then of the rank, until at most 64 share them,
// then by counting.  Every thread gets it.  A workgroup of ONE_BLOCK threads.
// (64-bit halves: shifts and compares of the 128-bit key took most of the
// time.)
template <class Each>
__device__ __forceinline__ KeyPair block_kth(KthLds& S, const Each& each, u64 need0, int L, u64 pre0, int rank_bits) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    constexpr int NW = ONE_BLOCK / 64;
    constexpr int PL = 6;  // levels of the magnitude
    if (t == 0) {
        S.need = need0;
        S.pre = pre0;
        S.n = 0;
    }
    u64 pfull = 0;  // the magnitude, once every digit of it is fixed
    for (;; ++L) {
        S.hist[t] = 0;
        S.hist[t + ONE_BLOCK] = 0;
        __syncthreads();
        const u64 pre = S.pre, need = S.need;
        const bool mag = L < PL;
        if (L == PL) pfull = pre;
        // this level's digit: bits [lo, hi) of its half
        const int hi = mag ? 63 - DIG * L : rank_bits - DIG * (L - PL);
        const int lo = max(0, hi - DIG);
        const unsigned mask = (1u << (hi - lo)) - 1u;
        const u64 pq = L > PL ? pre : 0;  // digits of the rank fixed so far
        auto in_prefix = [&](u64 p, u64 q) {
            return mag ? (L == 0 || (p >> hi) == pre) : (p == pfull && (L == PL || (q >> hi) == pq));
        };
        each([&](u64 p, u64 q) {
            if (in_prefix(p, q)) atomicAdd(&S.hist[(unsigned)((mag ? p : q) >> lo) & mask], 1u);
        });
        __syncthreads();
        // two bins per thread: the entries above each, by a suffix scan
        const u32 h0 = S.hist[2 * t], h1 = S.hist[2 * t + 1];
        u32 suf = h0 + h1;
        for (int off = 1; off < 64; off <<= 1) {
            const u32 y = (u32)__shfl_down((int)suf, off);
            if (lane + off < 64) suf += y;
        }
        if (lane == 0) S.wsum[wave] = suf;
        __syncthreads();
        u64 above = suf - h0 - h1;
        for (int w = wave + 1; w < NW; ++w) above += S.wsum[w];
        auto picked = [&](unsigned b, u64 over, u32 h) {
            S.pre = ((L == PL ? 0 : pre) << (hi - lo)) | b;
            S.need = need - over;
            S.bin = h;
        };
        if (above < need && above + h1 >= need) picked(2u * t + 1, above, h1);
        else if (above + h1 < need && above + h1 + h0 >= need) picked(2u * t, above + h1, h0);
        __syncthreads();
        const u64 pre2 = S.pre;
        if (!mag && lo == 0) return KeyPair{pfull, pre2};  // every digit fixed
        if (S.bin > 64) continue;
        each([&](u64 p, u64 q) {
            if (mag ? (p >> lo) == pre2 : (p == pfull && (q >> lo) == pre2)) {
                const unsigned at = atomicAdd(&S.n, 1u);
                S.p[at] = p;
                S.q[at] = q;
            }
        });
        __syncthreads();
        const unsigned c = S.bin;
        if ((unsigned)t < c) {
            const u64 need2 = S.need;
            const u64 p = S.p[t], q = S.q[t];
            unsigned more = 0, same = 0;
            for (unsigned x = 0; x < c; ++x) {
                const u64 P = S.p[x], Q = S.q[x];
                more += (P > p || (P == p && Q > q)) ? 1u : 0u;
                same += (P == p && Q == q) ? 1u : 0u;
            }
            if (more < need2 && more + same >= need2) {  // (equal keys write the same)
                S.kp = p;
                S.kq = q;
            }
        }
        __syncthreads();
        return KeyPair{S.kp, S.kq};
    }
}

// Step 4: the entries of the picked bin, when they are few, and the M-th key
// among them.
template <class JP>
__global__ __launch_bounds__(ONE_BLOCK) void k_sel_small(JP jp) {
    __shared__ KthLds S;
    __shared__ u64 kp[SEL_SMALL], kq[SEL_SMALL];
    const SelJob J = jp(blockIdx.y);
    SelState* st = J.st;
    if (st->done || st->bin > SEL_SMALL) return;
    const u128 pre = ((u128)st->pre_hi << 64) | st->pre_lo;
    const int sh = dig_lo(J.g, st->level - 1);
    for_segments(J, [&](u64 r, double c) {
        const u128 K = sel_key(r, c, J.g);
        if ((K >> sh) == pre) {
            const unsigned at = atomicAdd(&st->small_n, 1u);
            shared_store(&st->small_p[at], abs_bits(c));
            shared_store(&st->small_q[at], J.g.ndet_m1 - r);
        }
    });
    if (!last_workgroup(&st->ticket[SEL_TICKETS - 2], gridDim.x)) return;
    const unsigned n = (unsigned)st->bin;
    for (unsigned t = threadIdx.x; t < n; t += blockDim.x) {
        kp[t] = shared_load(&st->small_p[t]);
        kq[t] = shared_load(&st->small_q[t]);
    }
    __syncthreads();
    // two digits are fixed: the top 22 bits of the magnitude
    const KeyPair K = block_kth(
        S,
        [&](auto&& f) {
            for (unsigned t = threadIdx.x; t < n; t += ONE_BLOCK) f(kp[t], kq[t]);
        },
        st->need, st->level, (u64)pre, J.g.rank_bits);
    if (threadIdx.x == 0) sel_decide(st, ((u128)K.p << J.g.rank_bits) | K.q, J.g);
}

struct SelPred {
    bool all, thr;
    u64 thr_bits;
    u128 K;
    __device__ __forceinline__ explicit SelPred(const SelState& s)
        : all(s.take_all != 0), thr(s.use_thr != 0), thr_bits(s.thr_bits), K(((u128)s.key_hi << 64) | s.key_lo) {}
    // c != 0
    __device__ __forceinline__ bool operator()(u64 r, double c, const Geo& g) const {
        return all || (thr ? abs_bits(c) >= thr_bits : sel_key(r, c, g) >= K);
    }
};

// Exclusive scan of n counts in place by one workgroup, each taken as
// (x >> sh) & mask; returns the total.
__device__ __forceinline__ u64 scan_in_place(u64* x, u64 n, int sh, u64 mask) {
    __shared__ u64 w_tot[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
    constexpr int PER = 8;
    u64 carry = 0;
    for (u64 base = 0; base < n; base += (u64)blockDim.x * PER) {
        const u64 i0 = base + (u64)threadIdx.x * PER;
        u64 v[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            v[k] = i0 + k < n ? (shared_load(&x[i0 + k]) >> sh) & mask : 0;
            sum += v[k];
        }
        u64 inc = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const u64 y = (u64)__shfl_up((long long)inc, off);
            if (lane >= off) inc += y;
        }
        if (lane == 63) w_tot[wave] = inc;
        __syncthreads();
        u64 run = carry + inc - sum, tot = 0;
        for (int w = 0; w < nw; ++w) {
            if (w < wave) run += w_tot[w];
            tot += w_tot[w];
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (i0 + k < n) x[i0 + k] = run;
            run += v[k];
        }
        carry += tot;
        __syncthreads();
    }
    return carry;
}

// Step 5: per segment the entries kept by the M-th key (low 32 bits) and by
// the tie band's threshold (high 32 bits); the last workgroup settles which
// of the two rules holds and scans.
template <class JP>
__global__ __launch_bounds__(256) void k_sel_count(JP jp) {
    const SelJob J = jp(blockIdx.y);
    SelState* st = J.st;
    const SelPred keep(*st);
    const u64 thr = st->thr_bits;
    const bool band = J.band && st->cmin != ~0ull;
    const u64 ns = J.nseg();
    const u64 nw = (u64)gridDim.x * (blockDim.x >> 6);
    const int lane = threadIdx.x & 63;
    u64 by_thr = 0;
    for (u64 s = (u64)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); s < ns; s += nw) {
        const u32 m = J.count(s);
        const u64 b = s << J.shift;
        u32 kc = 0, kt = 0;
        for (u32 i0 = 0; i0 < m; i0 += 64 * SEG_UNROLL) {
            u64 r[SEG_UNROLL];
            double c[SEG_UNROLL];
#pragma unroll
            for (int u = 0; u < SEG_UNROLL; ++u) {
                const u32 i = i0 + (u32)u * 64 + lane;
                r[u] = 0;
                c[u] = 0.0;
                if (i < m) {
                    r[u] = J.r[b + i];
                    c[u] = J.a[b + i];
                }
            }
#pragma unroll
            for (int u = 0; u < SEG_UNROLL; ++u) {
                kc += (u32)__popcll(__ballot(c[u] != 0.0 && keep(r[u], c[u], J.g)));
                if (band) kt += (u32)__popcll(__ballot(c[u] != 0.0 && abs_bits(c[u]) >= thr));
            }
        }
        if (lane == 0) shared_store(&J.off[s], ((u64)kt << 32) | kc);
        by_thr += kt;
    }
    if (band && lane == 0 && by_thr) atomicAdd((unsigned long long*)&st->count_thr, (unsigned long long)by_thr);
    if (!last_workgroup(&st->ticket[SEL_TICKETS - 1], gridDim.x)) return;
    const u64 ct = shared_load(&st->count_thr);
    const bool use_thr = band && ct <= J.M + (u64)SFCI_TIE_SLACK;
    const u64 total = scan_in_place(J.off, ns, use_thr ? 32 : 0, 0xFFFFFFFFull);
    if (threadIdx.x == 0) {
        st->use_thr = use_thr ? 1 : 0;
        st->count_out = total;
        st->count_thr = 0;
        if (J.out_n) *J.out_n = total;
    }
}

// Step 6: a wavefront per segment writes its kept entries at the segment's offset.
template <class JP>
__global__ __launch_bounds__(256) void k_sel_write(JP jp) {
    const SelJob J = jp(blockIdx.y);
    const SelPred keep(*J.st);
    const u64 ns = J.nseg();
    const u64 nw = (u64)gridDim.x * (blockDim.x >> 6);
    const int lane = threadIdx.x & 63;
    for (u64 s = (u64)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); s < ns; s += nw) {
        const u32 m = J.count(s);
        const u64 b = s << J.shift;
        u64 at = J.off[s];
        for (u32 i0 = 0; i0 < m; i0 += 64 * SEG_UNROLL) {
            u64 r[SEG_UNROLL];
            double c[SEG_UNROLL];
#pragma unroll
            for (int u = 0; u < SEG_UNROLL; ++u) {
                const u32 i = i0 + (u32)u * 64 + lane;
                r[u] = 0;
                c[u] = 0.0;
                if (i < m) {
                    r[u] = J.r[b + i];
                    c[u] = J.a[b + i];
                }
            }
#pragma unroll
            for (int u = 0; u < SEG_UNROLL; ++u) {
                const bool p = c[u] != 0.0 && keep(r[u], c[u], J.g);
                const u64 pm = __ballot(p);
                if (p) {
                    const u64 o = at + (u64)__popcll(pm & ((1ull << lane) - 1ull));
                    J.out_r[o] = r[u];
                    J.out_a[o] = c[u];
                }
                at += (u64)__popcll(pm);
            }
        }
    }
}

// Every nonzero slot of a dense source, in rank order, without a candidate
// stage (M = all; also the candidates of a space too large for segments:
// |c| >= cand_bits): counts per chunk and their scan, then the compaction.
template <class JP>
__global__ __launch_bounds__(CBLOCK) void k_dense_count(JP jp, u64 nchunk) {
    const SelJob J = jp(blockIdx.y);
    const u64 bound = J.st->cand_bits;
    __shared__ unsigned sh[CBLOCK / 64];
    for (u64 ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
        const u64 base = ch * CCHUNK;
        unsigned c = 0;
#pragma unroll
        for (int k = 0; k < CITEMS; ++k) {
            const u64 i = base + (u64)k * CBLOCK + threadIdx.x;
            const double v = i < J.Dn ? J.D[i] : 0.0;
            c += (v != 0.0 && abs_bits(v) >= bound) ? 1u : 0u;
        }
        for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
        __syncthreads();
        if (threadIdx.x == 0) {
            u64 t = 0;
            for (int w = 0; w < CBLOCK / 64; ++w) t += sh[w];
            shared_store(&J.off[ch], t);
        }
        __syncthreads();
    }
    if (!last_workgroup(&J.st->ticket[SEL_TICKETS - 1], gridDim.x)) return;
    const u64 total = scan_in_place(J.off, nchunk, 0, ~0ull);
    if (threadIdx.x == 0) {
        J.st->count_out = total;
        J.st->ticket[SEL_TICKETS - 1] = 0;
        if (J.out_n) *J.out_n = total;
    }
}

template <class JP>
__global__ __launch_bounds__(CBLOCK) void k_dense_write(JP jp) {
    const SelJob J = jp(blockIdx.y);
    const u64 base = (u64)blockIdx.x * CCHUNK;
    if (base >= J.Dn) return;
    __shared__ unsigned c64[64];
    const u64 bound = J.st->cand_bits;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[CITEMS];
#pragma unroll
    for (int k = 0; k < CITEMS; ++k) {
        const u64 i = base + (u64)k * CBLOCK + threadIdx.x;
        v[k] = i < J.Dn ? J.D[i] : 0.0;
    }
    u64 m[CITEMS];
#pragma unroll
    for (int k = 0; k < CITEMS; ++k) {
        m[k] = __ballot(v[k] != 0.0 && abs_bits(v[k]) >= bound);
        if (lane == 0) c64[k * (CBLOCK / 64) + wave] = (unsigned)__popcll(m[k]);
        if (J.Dz && v[k] != 0.0) J.Dz[base + (u64)k * CBLOCK + threadIdx.x] = 0.0;
    }
    __syncthreads();
    if (wave == 0) {
        const unsigned c = c64[lane];
        unsigned inc = c;
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned y = __shfl_up(inc, off);
            if (lane >= off) inc += y;
        }
        c64[lane] = inc - c;
    }
    __syncthreads();
    const u64 at0 = J.off[blockIdx.x];
#pragma unroll
    for (int k = 0; k < CITEMS; ++k) {
        if ((m[k] >> lane) & 1u) {
            const u64 at = at0 + c64[k * (CBLOCK / 64) + wave] + __popcll(m[k] & ((1ull << lane) - 1ull));
            J.out_r[at] = base + (u64)k * CBLOCK + threadIdx.x;
            J.out_a[at] = v[k];
        }
    }
}

// The whole selection of a source of at most SEL_ONE entries by one
// workgroup, the values in registers: one launch (20 us at 3 136 slots) where
// the steps above are 7 and the histogram per digit took 24.
struct OneLds {
    KthLds S;
    u64 wsum[ONE_BLOCK / 64];
    double dsum[ONE_BLOCK / 64];
    unsigned cpos[ONE_ITEMS * (ONE_BLOCK / 64)];
    u64 count;
};

__device__ __forceinline__ u64 one_sum(OneLds& S, u64 x) {
    for (int off = 32; off >= 1; off >>= 1) x += (u64)__shfl_xor((long long)x, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) S.wsum[threadIdx.x >> 6] = x;
    __syncthreads();
    u64 s = 0;
    for (int w = 0; w < ONE_BLOCK / 64; ++w) s += S.wsum[w];
    return s;
}

struct OneResult {
    u64 total, count, cmin;
    bool all;
};

// v[k]: the value of entry k ONE_BLOCK + threadIdx.x (0 beyond n); on return
// keep's bit k tells whether it is kept and at[k] where it goes (by entry order).
template <class Rank>
__device__ __forceinline__ OneResult one_select(OneLds& L, const double (&v)[ONE_ITEMS], int nk, const Rank& rank_of,
                                                u64 M, bool band, const Geo& g, unsigned& keep,
                                                unsigned (&at)[ONE_ITEMS]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int NW = ONE_BLOCK / 64;
    OneResult R;
    u64 nz = 0;
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) nz += v[k] != 0.0 ? 1 : 0;
    R.total = one_sum(L, nz);
    R.all = M == UINT64_MAX || R.total <= M;
    const bool none = M == 0;
    bool use_thr = false;
    KeyPair KM{~0ull, ~0ull};
    u64 thr = ~0ull;
    R.cmin = ~0ull;
    if (!R.all && !none) {
        KM = block_kth(
            L.S,
            [&](auto&& f) {
#pragma unroll
                for (int k = 0; k < ONE_ITEMS; ++k)
                    if (k < nk && v[k] != 0.0) f(abs_bits(v[k]), g.ndet_m1 - rank_of(k));
            },
            M, 0, 0, g.rank_bits);
        R.cmin = KM.p;
        thr = abs_bits(__longlong_as_double((long long)R.cmin) * (1.0 - 1.0 / 68719476736.0));
        if (band) {
            u64 c = 0;
#pragma unroll
            for (int k = 0; k < ONE_ITEMS; ++k) c += (v[k] != 0.0 && abs_bits(v[k]) >= thr) ? 1 : 0;
            use_thr = one_sum(L, c) <= M + (u64)SFCI_TIE_SLACK;
        }
    }
    u64 m[ONE_ITEMS];
    keep = 0;
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) {
        bool p = k < nk && v[k] != 0.0 && !none;
        if (p && !R.all) {
            const u64 b = abs_bits(v[k]);
            p = use_thr ? b >= thr : b > KM.p || (b == KM.p && g.ndet_m1 - rank_of(k) >= KM.q);
        }
        m[k] = __ballot(p);
        keep |= p ? 1u << k : 0u;
        if (lane == 0) L.cpos[k * NW + wave] = (unsigned)__popcll(m[k]);
    }
    __syncthreads();
    if (wave == 0) {
        unsigned carry = 0;
        for (int b = 0; b < ONE_ITEMS * NW; b += 64) {
            const unsigned c = L.cpos[b + lane];
            unsigned inc = c;
            for (int off = 1; off < 64; off <<= 1) {
                const unsigned y = __shfl_up(inc, off);
                if (lane >= off) inc += y;
            }
            L.cpos[b + lane] = carry + inc - c;
            carry += (unsigned)__shfl((int)inc, 63);
        }
        if (lane == 0) L.count = carry;
    }
    __syncthreads();
    R.count = L.count;
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k)
        at[k] = L.cpos[k * NW + wave] + (unsigned)__popcll(m[k] & ((1ull << lane) - 1ull));
    return R;
}

template <class JP>
__global__ __launch_bounds__(ONE_BLOCK) void k_sel_one(JP jp) {
    __shared__ OneLds L;
    const SelJob J = jp(blockIdx.y);
    const u64 n = J.D ? J.Dn : min(*J.n, J.cap);
    const int nk = (int)((n + ONE_BLOCK - 1) / ONE_BLOCK);
    auto rank_of = [&](int k) -> u64 {
        const u64 i = (u64)k * ONE_BLOCK + threadIdx.x;
        return J.D ? i : J.r[i];
    };
    double v[ONE_ITEMS];
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) {
        const u64 i = (u64)k * ONE_BLOCK + threadIdx.x;
        v[k] = 0.0;
        if (k < nk && i < n) v[k] = J.D ? J.D[i] : J.a[i];
        if (J.Dz && v[k] != 0.0) J.Dz[i] = 0.0;
    }
    unsigned keep, at[ONE_ITEMS];
    const OneResult R = one_select(L, v, nk, rank_of, J.M, J.band != 0, J.g, keep, at);
    u64 r[ONE_ITEMS];
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) r[k] = ((keep >> k) & 1u) ? rank_of(k) : 0;
    __syncthreads();  // the output may stand in the list's place
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) {
        if ((keep >> k) & 1u) {
            J.out_r[at[k]] = r[k];
            J.out_a[at[k]] = v[k];
        }
    }
    if (threadIdx.x == 0) {
        if (J.out_n) *J.out_n = R.count;
        J.st->total = R.total;
        J.st->take_all = R.all ? 1 : 0;
        J.st->count_out = R.count;
        J.st->cmin = R.cmin;
    }
}

// ---- one step of the iteration on a space of at most SEL_ONE determinants ----
// (smallh.hip forms y = H w_j in D.)  One workgroup, the accumulator in LDS:
// the dots T_lj, S_lj of all l (a wavefront each), Eq. 10's two subtractions,
// the truncation, Eq. 11, and w_{j+1} both as a list and as the dense vector
// the next y = H w is formed from.
struct StepLds {
    OneLds one;
    double t_jj, t_mj;
    u64 nz;
};

// w = the kept entries of u, divided by their norm: list l and the dense copy.
__device__ __forceinline__ void small_store(const SmallStep& s, StepLds& L, double (&v)[ONE_ITEMS], int nk, int l) {
    const Geo g = geo_of(s.rank_bits, s.N - 1);
    unsigned keep, at[ONE_ITEMS];
    const OneResult R = one_select(
        L.one, v, nk, [&](int k) -> u64 { return (u64)k * ONE_BLOCK + threadIdx.x; }, s.M, s.band != 0, g, keep, at);
    double ss = 0.0;
    u64 nz = 0;
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k)
        if ((keep >> k) & 1u) {
            ss += v[k] * v[k];
            nz += s.nz[(u64)k * ONE_BLOCK + threadIdx.x];
        }
    for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
    if ((threadIdx.x & 63) == 0) L.one.dsum[threadIdx.x >> 6] = ss;
    nz = one_sum(L.one, nz);  // (its barriers also publish dsum)
    ss = 0.0;
    for (int w = 0; w < ONE_BLOCK / 64; ++w) ss += L.one.dsum[w];
    const bool div = ss > 0.0;
    const double nrm = sqrt(ss);
    u64* const Wr = s.Wr + (u64)l * s.cap;
    double* const Wa = s.Wa + (u64)l * s.cap;
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) {
        const u64 i = (u64)k * ONE_BLOCK + threadIdx.x;
        if (k >= nk || i >= s.N) continue;
        const bool on = (keep >> k) & 1u;
        const double a = on ? (div ? v[k] / nrm : v[k]) : 0.0;
        s.vd[i] = a;
        if (on) {
            Wr[at[k]] = i;
            Wa[at[k]] = a;
        }
    }
    if (threadIdx.x == 0) {
        s.nnz[l] = R.count;
        s.hist[l] = R.count;
        *s.emitted += nz;
    }
}

__global__ __launch_bounds__(ONE_BLOCK) void k_small_step(SmallStep s, int j) {
    extern __shared__ double lds[];
    __shared__ StepLds L;
    double* const y = lds;          // N
    double* const w = lds + s.N;    // N when it fits (s.w_lds), else the global copy
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (u64 i = threadIdx.x; i < s.N; i += ONE_BLOCK) {
        y[i] = s.D[i];
        if (s.w_lds) w[i] = s.vd[i];
    }
    __syncthreads();
    for (int l = wave; l <= j; l += ONE_BLOCK / 64) {
        const u64* r = s.Wr + (u64)l * s.cap;
        const double* a = s.Wa + (u64)l * s.cap;
        const u64 n = s.nnz[l];
        double st = 0.0, sv = 0.0;
        constexpr int U = 8;
        for (u64 i0 = 0; i0 < n; i0 += 64 * U) {
            u64 rr[U];
            double aa[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const u64 i = i0 + (u64)u * 64 + lane;
                rr[u] = i < n ? r[i] : 0;
                aa[u] = i < n ? a[i] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + (u64)u * 64 + lane >= n) continue;
                st += aa[u] * y[rr[u]];
                sv += aa[u] * (s.w_lds ? w[rr[u]] : s.vd[rr[u]]);
            }
        }
        for (int off = 32; off >= 1; off >>= 1) {
            st += __shfl_xor(st, off);
            sv += __shfl_xor(sv, off);
        }
        if (lane == 0) {
            s.T[l * s.nL + j] = st;
            s.T[j * s.nL + l] = st;
            s.S[l * s.nL + j] = sv;
            s.S[j * s.nL + l] = sv;
            if (l == j) L.t_jj = st;
            if (l == j - 1) L.t_mj = st;
        }
    }
    if (j + 1 == s.nL) return;
    __syncthreads();
    for (int b = 0; b < 2; ++b) {
        // u = (y - T_jj w_j) - T_{j-1,j} w_{j-1}
        const int l = j - b;
        if (l < 0) break;
        const double c = b ? L.t_mj : L.t_jj;
        const u64 n = s.nnz[l];
        for (u64 i = threadIdx.x; i < n; i += ONE_BLOCK) {
            const double prod = c * s.Wa[(u64)l * s.cap + i];
            const u64 k = s.Wr[(u64)l * s.cap + i];
            y[k] = y[k] - prod;
        }
        __syncthreads();
    }
    const int nk = (int)((s.N + ONE_BLOCK - 1) / ONE_BLOCK);
    double v[ONE_ITEMS];
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) {
        const u64 i = (u64)k * ONE_BLOCK + threadIdx.x;
        v[k] = (k < nk && i < s.N) ? y[i] : 0.0;
    }
    small_store(s, L, v, nk, j + 1);
}

// Block end: Psi = sum_j x_j w_j into D (final) or, truncated and normalised, w_0.
__global__ __launch_bounds__(ONE_BLOCK) void k_small_psi(SmallStep s, const double* __restrict__ x, int final) {
    extern __shared__ double lds[];
    __shared__ StepLds L;
    for (u64 i = threadIdx.x; i < s.N; i += ONE_BLOCK) lds[i] = 0.0;
    __syncthreads();
    for (int l = 0; l < s.nL; ++l) {
        const double c = x[l];
        const u64 n = s.nnz[l];
        for (u64 i = threadIdx.x; i < n; i += ONE_BLOCK) {
            const double prod = c * s.Wa[(u64)l * s.cap + i];
            const u64 k = s.Wr[(u64)l * s.cap + i];
            lds[k] = lds[k] + prod;
        }
        __syncthreads();
    }
    const int nk = (int)((s.N + ONE_BLOCK - 1) / ONE_BLOCK);
    double v[ONE_ITEMS];
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) {
        const u64 i = (u64)k * ONE_BLOCK + threadIdx.x;
        const bool in = k < nk && i < s.N;
        v[k] = in ? lds[i] : 0.0;
        if (final && in) s.D[i] = v[k];
    }
    if (!final) small_store(s, L, v, nk, 0);
}

unsigned seg_grid(int num_cu, u64 nseg) {
    return (unsigned)std::max<u64>(1, std::min<u64>((nseg + 3) / 4, (u64)num_cu * 8));
}

unsigned hist0_grid(int num_cu, u64 n) {
    return (unsigned)std::max<u64>(1, std::min<u64>((n + 4095) / 4096, (u64)num_cu * 3));
}

// Steps 3 and 4 for candidates whose top digit is picked (from = 1), or all
// digits of a list (from = 0).
template <class JP>
void run_digits(hipStream_t st, const JP& jp, unsigned n, int num_cu, u64 nseg, int from, int max_ndig) {
    const unsigned grid = (unsigned)std::max<u64>(1, std::min<u64>((nseg + 15) / 16, (u64)num_cu));
    if (from == 0) hipLaunchKernelGGL(k_sel_hist0<JP>, dim3(grid, n), dim3(SEG_BLOCK), 0, st, jp);
    hipLaunchKernelGGL(k_sel_hist<JP>, dim3(grid, n), dim3(SEG_BLOCK), 0, st, jp, 1);
    hipLaunchKernelGGL(k_sel_small<JP>, dim3(grid, n), dim3(ONE_BLOCK), 0, st, jp);
    // the remaining digits one by one, for bins that hold more than SEL_SMALL
    // entries (their kernels return at once otherwise)
    for (int L = 2; L < max_ndig; ++L)
        hipLaunchKernelGGL(k_sel_hist<JP>, dim3(grid, n), dim3(SEG_BLOCK), 0, st, jp, L);
}

SelJob make_job(sfci_problem* P, u64 M, SelState* st) {
    SelJob J{};
    J.st = st;
    J.M = M;
    J.band = P->tie_band ? 1 : 0;
    J.g = geo_of(P->kg.rank_bits, P->kg.ndet_m1);
    return J;
}

SelJob dense_job(sfci_problem* P, const CandSrc& src, u64 M, bool zero) {
    SelJob J = make_job(P, M, (SelState*)P->ws_sel.get(sizeof(SelState)));
    J.D = src.dense;
    J.Dn = P->Ndet;
    J.cap = P->Ndet;
    J.shift = SEL_DENSE_SHIFT;
    J.Dz = zero ? (double*)src.dense : nullptr;
    return J;
}

SelJob list_job(sfci_problem* P, const CandSrc& src, u64 M, SelState* st, u64* off) {
    SelJob J = make_job(P, M, st);
    J.r = src.lrank;
    J.a = src.lval;
    J.n = src.lcount;
    J.cap = src.lcap;
    J.shift = select_shift(src.lcap);
    J.off = off;
    return J;
}

// Steps 1 to 5 on a list.
void list_prepare(sfci_problem* P, const SelJob& J) {
    const u64 ns = select_segments(J.cap);
    const unsigned grid = seg_grid(P->num_cu, ns);
    const OneJob jp{J};
    hipLaunchKernelGGL(k_sel_init<OneJob>, dim3(1), dim3(256), 0, P->stream, jp);
    if (J.M != UINT64_MAX && J.M != 0) run_digits(P->stream, jp, 1, P->num_cu, ns, 0, J.g.ndig);
    hipLaunchKernelGGL(k_sel_count<OneJob>, dim3(grid), dim3(256), 0, P->stream, jp);
    SFCI_CHECK_HIP(hipGetLastError());
}

// An output in the list's place is written by one wavefront: an entry never
// moves up, so in order nothing is overwritten before it is read.
void list_write(sfci_problem* P, const SelJob& J) {
    const bool in_place = J.out_r == J.r || J.out_a == J.a;
    hipLaunchKernelGGL(k_sel_write<OneJob>, dim3(in_place ? 1 : seg_grid(P->num_cu, select_segments(J.cap))),
                       dim3(in_place ? 64 : 256), 0, P->stream, OneJob{J});
    SFCI_CHECK_HIP(hipGetLastError());
}

// Dense source, candidates in segments: the buffers (N_det entries: a chunk's
// segment has a slot for each of its entries).
void dense_segments(sfci_problem* P, SelJob& J) {
    const u64 nch = select_chunks(P->Ndet);
    J.r = (u64*)P->ws_cand_r.get(P->Ndet * sizeof(u64));
    J.a = (double*)P->ws_cand_a.get(P->Ndet * sizeof(double));
    J.off = (u64*)P->ws_cnt.get(nch * (sizeof(u64) + sizeof(u32)));
    J.cnt = (u32*)(J.off + nch);
}

template <class JP>
void dense_seg_prepare(hipStream_t st, const JP& jp, unsigned n, int num_cu, u64 max_n, int max_ndig, bool trunc) {
    const u64 nch = select_chunks(max_n);
    const unsigned grid = seg_grid(num_cu, nch);
    hipLaunchKernelGGL(k_sel_init<JP>, dim3(1, n), dim3(256), 0, st, jp);
    if (trunc) hipLaunchKernelGGL(k_sel_hist0_dense<JP>, dim3(hist0_grid(num_cu, max_n), n), dim3(512), 0, st, jp);
    hipLaunchKernelGGL(k_sel_collect<JP>, dim3((unsigned)nch, n), dim3(CBLOCK), 0, st, jp);
    if (trunc) run_digits(st, jp, n, num_cu, nch, 1, max_ndig);
    hipLaunchKernelGGL(k_sel_count<JP>, dim3(grid, n), dim3(256), 0, st, jp);
}

// Dense source in place: every slot with |c| >= cand_bits.
template <class JP>
void dense_count(hipStream_t st, const JP& jp, unsigned n, int num_cu, u64 max_n) {
    const u64 nch = select_chunks(max_n);
    hipLaunchKernelGGL(k_dense_count<JP>, dim3((unsigned)std::min<u64>(nch, (u64)num_cu * 8), n), dim3(CBLOCK), 0,
                       st, jp, nch);
}

u64 read_u64(sfci_problem* P, const u64* d) {
    u64 h = 0;
    SFCI_CHECK_HIP(hipMemcpyAsync(&h, d, sizeof(u64), hipMemcpyDeviceToHost, P->stream));
    SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
    return h;
}

// A source one workgroup takes in one launch.
bool one_block(sfci_problem* P, const CandSrc& src) { return (src.dense ? P->Ndet : src.lcap) <= (u64)SEL_ONE; }

}  // namespace

bool select_one_step(const sfci_problem* P, u64 M) {
    return M == UINT64_MAX || M == 0 || P->Ndet <= (u64)SEL_ONE || P->Ndet * 16 <= SEL_SEG_BYTES;
}

u64 select_chunks(u64 n_upper) { return std::max<u64>(1, (n_upper + CCHUNK - 1) / CCHUNK); }
// Lists of up to 4 Mi entries in segments of 1 024 (a wavefront each: more of
// them in flight), longer ones of 4 096.
int select_shift(u64 lcap) { return lcap <= (4ull << 20) ? 10 : SEL_DENSE_SHIFT; }
u64 select_segments(u64 lcap) {
    const int sh = select_shift(lcap);
    return std::max<u64>(1, (lcap + (1ull << sh) - 1) >> sh);
}

// Two steps, for callers that must know the count before the entries are
// written.  What the second one needs is kept in P->sel_mode: 1 segments of
// the dense source, 2 a list, 3 the dense source in place.
void select_prepare(sfci_problem* P, const CandSrc& src, u64 M, u64* count_dev) {
    if (!src.dense) {
        SelJob J = list_job(P, src, M, (SelState*)P->ws_sel.get(sizeof(SelState)),
                            (u64*)P->ws_cnt.get(select_segments(src.lcap) * sizeof(u64)));
        J.out_n = count_dev;
        list_prepare(P, J);
        P->sel_mode = 2;
        return;
    }
    SelJob J = dense_job(P, src, M, false);
    J.out_n = count_dev;
    const bool trunc = M != UINT64_MAX && M != 0;
    if (trunc && P->Ndet * 16 <= SEL_SEG_BYTES) {
        // (the accumulator is zeroed when the candidates are taken: the caller zeroes it anyway)
        J.Dz = (double*)src.dense;
        dense_segments(P, J);
        dense_seg_prepare(P->stream, OneJob{J}, 1, P->num_cu, P->Ndet, J.g.ndig, true);
        P->sel_mode = 1;
    } else {
        const u64 nch = select_chunks(P->Ndet);
        J.off = (u64*)P->ws_cnt.get(nch * sizeof(u64));
        hipLaunchKernelGGL(k_sel_init<OneJob>, dim3(1), dim3(256), 0, P->stream, OneJob{J});
        if (trunc) {
            // a space too large for segments: the candidates' number decides their buffers
            hipLaunchKernelGGL(k_sel_hist0_dense<OneJob>, dim3(hist0_grid(P->num_cu, P->Ndet)), dim3(512), 0,
                               P->stream, OneJob{J});
        }
        dense_count(P->stream, OneJob{J}, 1, P->num_cu, P->Ndet);
        P->sel_mode = 3;
        if (trunc) {
            const u64 nc = read_u64(P, &J.st->count_out);
            J.out_r = (u64*)P->ws_cand_r.get(std::max<u64>(1, nc) * sizeof(u64));
            J.out_a = (double*)P->ws_cand_a.get(std::max<u64>(1, nc) * sizeof(double));
            J.Dz = (double*)src.dense;
            hipLaunchKernelGGL(k_dense_write<OneJob>, dim3((unsigned)nch), dim3(CBLOCK), 0, P->stream, OneJob{J});
            CandSrc ls{};
            ls.lrank = J.out_r;
            ls.lval = J.out_a;
            ls.lcount = &J.st->count_cand;
            ls.lcap = std::max<u64>(1, nc);
            launch_set_u64(P, &J.st->count_cand, nc);
            SelJob K = list_job(P, ls, M, J.st, (u64*)P->ws_cnt.get(select_segments(ls.lcap) * sizeof(u64)));
            K.out_n = count_dev;
            const unsigned grid = seg_grid(P->num_cu, select_segments(ls.lcap));
            run_digits(P->stream, OneJob{K}, 1, P->num_cu, select_segments(ls.lcap), 1, K.g.ndig);
            hipLaunchKernelGGL(k_sel_count<OneJob>, dim3(grid), dim3(256), 0, P->stream, OneJob{K});
            P->sel_mode = 2;
            P->sel_src = ls;
        }
    }
    SFCI_CHECK_HIP(hipGetLastError());
}

void select_write(sfci_problem* P, const CandSrc& src, u64* out_rank, double* out_amp, bool zero_dense) {
    SelState* st = (SelState*)P->ws_sel.p;
    u64* off = (u64*)P->ws_cnt.p;
    if (P->sel_mode == 3) {
        SelJob J = dense_job(P, src, UINT64_MAX, zero_dense);
        J.off = off;
        J.out_r = out_rank;
        J.out_a = out_amp;
        hipLaunchKernelGGL(k_dense_write<OneJob>, dim3((unsigned)select_chunks(P->Ndet)), dim3(CBLOCK), 0, P->stream,
                           OneJob{J});
        SFCI_CHECK_HIP(hipGetLastError());
        return;
    }
    SelJob J;
    if (P->sel_mode == 1) {
        J = dense_job(P, src, 0, false);
        dense_segments(P, J);
    } else {
        J = list_job(P, src.dense ? P->sel_src : src, 0, st, off);
    }
    J.out_r = out_rank;
    J.out_a = out_amp;
    list_write(P, J);
}

void select_prepare_ws(sfci_problem* P, const CandSrc& src, u64 M, u64* count_dev, const SelWs& ws) {
    SelJob J = list_job(P, src, M, ws.st, ws.off);
    J.out_n = count_dev;
    list_prepare(P, J);
}

void select_write_ws(sfci_problem* P, const CandSrc& src, u64* out_rank, double* out_amp, const SelWs& ws) {
    SelJob J = list_job(P, src, 0, ws.st, ws.off);
    J.out_r = out_rank;
    J.out_a = out_amp;
    list_write(P, J);
}

// One step, for outputs that hold whatever may be kept.
void select_topm(sfci_problem* P, const CandSrc& src, u64 M, u64* out_rank, double* out_amp, u64* out_count_dev,
                 bool zero_dense) {
    if (one_block(P, src)) {
        SelState* st = (SelState*)P->ws_sel.get(sizeof(SelState));
        SelJob J = src.dense ? dense_job(P, src, M, zero_dense) : list_job(P, src, M, st, nullptr);
        J.out_r = out_rank;
        J.out_a = out_amp;
        J.out_n = out_count_dev;
        hipLaunchKernelGGL(k_sel_one<OneJob>, dim3(1), dim3(ONE_BLOCK), 0, P->stream, OneJob{J});
        SFCI_CHECK_HIP(hipGetLastError());
        return;
    }
    if (!src.dense || M == UINT64_MAX || M == 0) {
        select_prepare(P, src, M, out_count_dev);
        select_write(P, src, out_rank, out_amp, zero_dense);
        return;
    }
    SelJob J = dense_job(P, src, M, zero_dense);
    dense_segments(P, J);
    J.out_r = out_rank;
    J.out_a = out_amp;
    J.out_n = out_count_dev;
    dense_seg_prepare(P->stream, OneJob{J}, 1, P->num_cu, P->Ndet, J.g.ndig, true);
    list_write(P, J);
}

void bstep_select(hipStream_t st, const BInst* d, int n, int out_kind, int j, u64 max_ndet, int num_cu, int band,
                  int max_ndig, int all, bool zero) {
    const BatchJobs jp{d, out_kind, j, band, all, zero ? 1 : 0};
    const unsigned N = (unsigned)n;
    if (max_ndet <= (u64)SEL_ONE) {
        hipLaunchKernelGGL(k_sel_one<BatchJobs>, dim3(1, N), dim3(ONE_BLOCK), 0, st, jp);
    } else {
        dense_seg_prepare(st, jp, N, num_cu, max_ndet, max_ndig, all == 0);
        hipLaunchKernelGGL(k_sel_write<BatchJobs>, dim3(seg_grid(num_cu, select_chunks(max_ndet)), N), dim3(256), 0,
                           st, jp);
    }
    SFCI_CHECK_HIP(hipGetLastError());
}

// Dynamic LDS of the small-space kernels: one array of N doubles, or two where they fit.
size_t small_step_lds(u64 N, bool two) { return (size_t)(two ? 2 : 1) * N * sizeof(double); }

void small_step_setup(sfci_problem* P) {
    for (const void* f : {(const void*)k_small_step, (const void*)k_small_psi})
        SFCI_CHECK_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(SEL_ONE * sizeof(double))));
    (void)P;
}

void launch_small_step(sfci_problem* P, const SmallStep& s, int j) {
    hipLaunchKernelGGL(k_small_step, dim3(1), dim3(ONE_BLOCK), small_step_lds(s.N, s.w_lds != 0), P->stream, s, j);
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_small_psi(sfci_problem* P, const SmallStep& s, const double* x, bool final) {
    hipLaunchKernelGGL(k_small_psi, dim3(1), dim3(ONE_BLOCK), small_step_lds(s.N, false), P->stream, s, x,
                       final ? 1 : 0);
    SFCI_CHECK_HIP(hipGetLastError());
}
