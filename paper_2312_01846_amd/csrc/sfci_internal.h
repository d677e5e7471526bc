// Internal host-side declarations of libsfci (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <utility>
#include <vector>

#include "../../include/sfci.h"
#include "sfci_device.h"

#define SFCI_CHECK_HIP(expr)                                                       \
    do {                                                                           \
        hipError_t _e = (expr);                                                    \
        if (_e != hipSuccess) throw sfci_error(-6, std::string(#expr) + ": " + hipGetErrorString(_e)); \
    } while (0)

struct sfci_error {
    int code;
    std::string msg;
    sfci_error(int c, std::string m) : code(c), msg(std::move(m)) {}
};

// Grow-only device buffer.
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    void* get(size_t need);
    void release();
};

// Counter of frees of library-owned device memory (workspaces, tables,
// problem arrays), process-wide.  A captured graph stays launchable only
// while the counter is unchanged since its capture: every buffer it points
// to is then still allocated.
u64 device_free_epoch();
void note_device_free();

// Launch buffers of the gradient passes through the target-owned tiles.
struct RowTileGradWs {
    DevBuf desc, prefix, counter, scratch;
    void release() { desc.release(); prefix.release(); counter.release(); scratch.release(); }
};

// Top-M selection (select.hip).
constexpr int SEL_ONE = 16384;             // sources of at most this many entries: one workgroup, one launch
constexpr unsigned SEL_SMALL = 2048;       // entries of the picked bin among which the M-th key is found by counting
constexpr int SEL_TICKETS = 16;            // a ticket per kernel of a selection that ends in a last workgroup
constexpr int SEL_DENSE_SHIFT = 12;        // slots per segment of a dense source (log2)
constexpr u64 SEL_SEG_BYTES = 1ull << 30;  // a single sigma's candidate segments may take this much

// Selection state (device resident): a radix select over the 128-bit key
// K = (bits(|c|) << rank_bits) | (N_det - 1 - rank), 11-bit digits from the
// top, so that larger K = larger |c|, then lower rank.
struct SelState {
    u64 need;       // entries still to take inside the current prefix
    u64 pre_hi, pre_lo;
    int level;      // digits fixed so far
    int done;       // the M-th key is known, or not needed
    int take_all;   // keep every nonzero entry
    int use_thr;    // keep every |c| >= thr (they are at most M + SFCI_TIE_SLACK)
    u64 total;      // nonzero entries of the source
    u64 count_out;  // entries kept
    u64 cmin;       // bits of the smallest |c| among the M selected
    u64 key_hi, key_lo;  // the M-th key
    u64 thr_bits;   // bits of cmin * (1 - 2^-36)
    u64 count_thr;  // entries with |c| >= that
    u64 cand_bits;  // bits of the bound on a dense source's candidates (binade of the M-th |c|, less 2^-36)
    u64 count_cand; // number of candidates where they form one list
    u64 bin;        // entries that share the current prefix
    unsigned small_n, pad;
    unsigned ticket[SEL_TICKETS];
    u64 hist[2048];
    u64 small_p[SEL_SMALL], small_q[SEL_SMALL];  // the picked bin's keys: bits of |c|, N_det - 1 - rank
};

// What a selection reads: the dense accumulator or a list.
struct CandSrc {
    const double* dense;  // if non-null: D[0..Ndet)
    const u64* lrank;     // else list
    const double* lval;
    const u64* lcount;    // device scalar
    u64 lcap;
};

struct KeyGeom {
    int rank_bits;  // bits of N_det - 1 (>= 1)
    int ndig;       // number of 11-bit digits covering 63 + rank_bits bits
    int pad_bits;   // left shift that aligns the key to ndig digits
    u64 ndet_m1;
};

// Buffers of the target-row-driven sort-path emission (rowpass.hip).
struct RowPassWs {
    DevBuf beg, end, cnt, npair, tup_pre, pair_pre, pairs, scal, tile_pre, tile_row;
    void release() {
        for (DevBuf* b : {&beg, &end, &cnt, &npair, &tup_pre, &pair_pre, &pairs, &scal, &tile_pre, &tile_row})
            b->release();
    }
};

// Buffers of the list-based iteration and sigma (listlz.hip).
struct ListWs {
    DevBuf scal, pr, pa, mark, Rr, Ra, R2r, R2a, yg, taken, psi_r, psi_a, dpass, dcnt, scal2, rowptr, fo, heavy, hr_cnt, hr_pre, hr_src,
        hr_list, hr_ctr;
    void release() {
        for (DevBuf* b : {&scal, &pr, &pa, &mark, &Rr, &Ra, &R2r, &R2a, &yg, &taken, &psi_r, &psi_a, &dpass, &dcnt,
                          &scal2, &rowptr, &fo, &heavy, &hr_cnt, &hr_pre, &hr_src, &hr_list, &hr_ctr})
            b->release();
    }
};

// A kernel's answer of up to seven words to the host, by way of coherent pinned
// memory: the host goes on launching and reads it as soon as it is there.
struct HostLine {
    static constexpr int WORDS = 8;  // the last one is the question's number, written after the others
    u64* p;
    u64 number;
#ifdef __HIPCC__
    __device__ __forceinline__ void answer() const {
        __hip_atomic_store(p + WORDS - 1, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
#endif
};
HostLine host_line(sfci_problem* P);                   // the next question (its memory on first use)
const u64* wait_line(sfci_problem* P, const HostLine& l);  // the answer

// Launch shape of the in-order kernel (inorder.hip).
struct InOrderGeom {
    u32 words, off_rows, per_wave;
    int waves, per_cu;
    size_t lds;
};

struct sfci_problem {
    int n, na, nb;
    u64 Na, Nb, Ndet;
    KeyGeom kg;
    hipStream_t stream;
    int device;
    double* d_h = nullptr;
    double* d_g = nullptr;
    u64* d_binom = nullptr;
    double* d_D = nullptr;  // dense accumulator (N_det doubles), all zero between calls
    int dense_state = 0;    // 0 untried, 1 allocated, -1 does not fit
    int num_cu = 256;
    DevBuf ws_sel, ws_cnt, ws_scan, ws_scan2, ws_scalar, ws_red;
    DevBuf ws_tup_k, ws_tup_v, ws_tup_k2, ws_tup_v2, ws_seg_v, ws_seg_f, ws_src_cnt, ws_src_off, ws_hist;
    DevBuf ws_list_r, ws_list_a, ws_prod;
    DevBuf ws_cand_r, ws_cand_a;  // top-M of a dense source: its candidates
    DevBuf sh_idx, sh_val, sh_nz, sh_vd;  // small spaces (smallh.hip): H by rows, terms per column, dense v
    int sh_state = 0;                     // 0 untried, 1 built, -1 the space is too large
    DevBuf ws_os;       // blocks of a long in-order sum
    DevBuf io_tab;      // in-order sigma: alpha strings, nonzero (ia|..) slabs
    int io_state = 0;   // 0 untried, 1 available, -1 not
    InOrderGeom io_geom{};
    unsigned* io_state_words = nullptr;  // of k_io_load, within io_tab
    bool io_ab = false, io_pairs = false;  // some (ia|jb), i != a, j != b, and some same-spin double are nonzero
    hipEvent_t ev[2] = {nullptr, nullptr};  // around a call, created on first use
    u64* line = nullptr;    // pinned words that a kernel answers in (HostLine)
    u64 line_asked = 0;
    int sel_mode = 0;             // what select_prepare left for select_write (select.hip)
    CandSrc sel_src{};
    DevBuf ws_lz[8];
    DevBuf ws_rt_rows, ws_rt_beta, ws_rt_nbr, ws_rt_desc;
    DevBuf ws_ab_rc, ws_ab_cr, ws_ab_off, ws_ab_it;  // alpha-beta item lists (rows of several tiles)
    DevBuf ws_rt_phase;  // optional per-phase timing of the tile kernel (SFCI_RT_PHASES=1)
    void* rowtile = nullptr;  // tables of the target-owned dense kernel (rowtile.hip)
    // The same space with alpha and beta exchanged (gradient second pass):
    // shares this problem's integrals, binomial table and dense array.
    sfci_problem* swapped = nullptr;
    RowTileGradWs grad_ws;
    ListWs list_ws;
    RowPassWs rowpass_ws;
    // projected roots of the excited-state iteration: H Psi_i lists and scalars
    DevBuf ws_hroot_r[SFCI_MAX_ROOTS], ws_hroot_a[SFCI_MAX_ROOTS], ws_roots_sc, ws_roots_cnt;
    bool borrowed = false;  // true for such a shadow: d_h, d_g, d_binom, d_D belong to another problem
    // Truncation extension (off = the paper's rule, exactly min(M, nonzero)
    // entries kept): also keep entries within a relative 2^-36 of the M-th
    // |c|, at most SFCI_TIE_SLACK of them.  Set from the options of each call.
    int tie_band = 0;
    // Sort-path tuples per pass assigned by a batch (0: a quarter of free memory).
    u64 tup_cap_hint = 0;
    // Excitation screen of the sigma kernels (0 = off): a double excitation's
    // term H_ki v_i with |H_ki v_i| < excite_eps is not added.  Set from the
    // options of each call.
    double excite_eps = 0.0;
};

// Entries a truncated vector can hold beyond M (the tie band's reach).
inline u64 tie_extra(const sfci_problem* P) { return P->tie_band ? (u64)SFCI_TIE_SLACK : 0; }

// ---- launchers (sigma.hip) ----
struct SigmaLaunch {
    const u64* v_rank;
    const double* v_amp;
    const u64* v_nnz;  // device scalar
    u64 cap;           // upper bound on nnz (grid sizing)
};
void launch_sigma_dense(sfci_problem* P, const SigmaLaunch& v, double* D, unsigned long long* emitted);
void launch_sigma_count(sfci_problem* P, const SigmaLaunch& v, u64 alo, u64 ahi, u64* counts);
void launch_sigma_emit(sfci_problem* P, const SigmaLaunch& v, u64 alo, u64 ahi, const u64* offs, u64 key_base,
                       u64* keys, double* vals);
void launch_rank(sfci_problem* P, const u64* a, const u64* b, u64 cnt, u64* rank, int* bad);
void launch_unrank(sfci_problem* P, const u64* rank, u64 cnt, u64* a, u64* b, int* bad);
// Backward of sigma = H v (backward.hip).  The cotangent must already be
// scattered into the zero dense array D.  Rh (n^2) and Rg (n^4) are scratch.
// bad (device, may be NULL): four flags; with one set vbar, dh and dg are left
// as they are (v must then count as empty).
void launch_backward_dense(sfci_problem* P, const SigmaLaunch& v, const double* D, double* vbar, double* dh, double* dg,
                           double* Rh, double* Rg, const int* bad = nullptr);
void launch_scatter_zero(sfci_problem* P, double* D, const u64* r, const u64* nnz, u64 cap);
struct RowTileDesc;
// The same from the row view of v and the beta-single table (backrows.hip),
// where they are available; s_rank: the ranks of the cotangent, Rg = Rh + n^2.
bool back_rows_available(sfci_problem* P, u64 nnz, u64 nnz_s);
// Asks the device whether this is the faster way for the entries (the cotangent
// already in D); true without asking when SFCI_BACK_ROWS forces it.
bool ask_back_rows(sfci_problem* P, const SigmaLaunch& v, const double* D, const u64* s_rank, const u64* s_nnz,
                   HostLine* l);
bool back_rows_answer(sfci_problem* P, const HostLine& l);
void launch_back_rows(sfci_problem* P, const SigmaLaunch& v, const RowTileDesc& d, const double* D, const u64* s_rank,
                      const u64* s_nnz, u64 s_cap, double* vbar, double* dh, double* dg, double* Rh, double* Rg,
                      const int* bad = nullptr);

// ---- target-owned dense sigma (rowtile.hip) ----
bool rowtile_available(sfci_problem* P);  // builds the per-problem tables on first use
// The packed beta singles of every beta string (sorted by target rank), or
// nullptr where the tables cannot be built (or SFCI_RP_NO_T1=1).
const u32* rowtile_T1(sfci_problem* P);
// Beta-rank tiles per target row of the tile kernel (0 where it is unavailable).
int rowtile_ntiles(sfci_problem* P);
void rowtile_release(sfci_problem* P);
// eps > 0: accumulated entries with |c| < eps are written as zero (screening, Sec. 3).
void launch_sigma_rowtile(sfci_problem* P, const SigmaLaunch& v, double* D, unsigned long long* emitted,
                          double eps = 0.0);
// Batched form: prepare each instance, put the descriptions on the device,
// then one launch drains the items of all instances.
struct RowTileDesc {
    alignas(8) unsigned char raw[384];  // kernel-side description of one instance
    u64 n_items, nbr_cap;
    u64 cap;           // entries of the input at most
    size_t lds_bytes;  // the tile
    unsigned n2;       // n^2 of the instance
    unsigned ja_doubles;  // n_alpha n^2: the identity row's alpha-part table
    int max_lds;       // LDS per workgroup on the device
};
// Launch geometry for a set of descriptions: dynamic LDS, and where the
// per-wavefront integral slabs start (slab_n2 = 0: no slabs, the kernel
// reads the integrals from global memory).
struct RowTileGeom {
    size_t lds;
    unsigned slab_off, slab_n2;
    unsigned itab_off;  // per-item element tables
    unsigned ja_off;    // the identity row's alpha-part table (0: not staged)
    bool whole = false; // every instance's rows are one tile (the one-tile kernel runs)
    int waves = 16;     // wavefronts per workgroup (8: two workgroups to a compute unit)
};
RowTileGeom rowtile_geom(const RowTileDesc* d, int n_inst);
// Launch-time work sizes of the sigma tile kernel (0 = the built-in default):
// identity-row beta singles and beta-beta doubles per work unit (entries),
// and workgroups per compute unit in the grid.
struct RowTileTune {
    unsigned b1_chunk = 0, bb_chunk = 0, per_cu = 0;
};
// ab_lists: for rows of several tiles, also list the alpha-beta doubles' items
// per (input chunk, target tile) for the sigma kernel (when they fit in memory).
// full_rows: every target row of D is written (zeros where no term lands), so
// D need not be zero before the launch.
RowTileDesc rowtile_prepare(sfci_problem* P, const SigmaLaunch& v, double* D, unsigned long long* emitted,
                            double eps = 0.0, bool ab_lists = false, bool full_rows = false);
// The input view and tables a prepared description points to.
struct RowView {
    const u64 *rowbeg, *rowend;   // per alpha row: its entries
    const u32 *v_beta, *v_rb;     // per entry: beta string, beta rank
    const u32* T1;                // beta singles per beta rank (rowtile.hip)
    const double* K4;             // same-spin double elements by orbital pairs
};
RowView rowtile_view(const RowTileDesc& d);
void rowtile_many(RowTileDesc& d);  // for a launch of several instances
// The per-problem tables (rowtile_available(P) must hold; T2 may be NULL).
struct RowTables {
    const u32* T1;
    const double* TS;
    const u32* T2r;
    const double *T2e, *K2, *K4;
};
RowTables rowtile_tables(sfci_problem* P);
// Deterministic sigma into D, every row written, without a sort (inorder.hip):
// where a target row fits in LDS, the alpha strings are at most 65 536 and nnz
// entries are worth writing N_det sums; ...
bool inorder_available(sfci_problem* P, u64 nnz);
// ... whether it is the faster way for the entries of v (else the sort path);
// called before each launch_sigma_inorder, which it prepares.  May wait for the
// device.
bool inorder_pays(sfci_problem* P, const SigmaLaunch& v, RowTileDesc* d);
void launch_sigma_inorder(sfci_problem* P, const SigmaLaunch& v, const RowTileDesc& d, double* D,
                          unsigned long long* emitted, double eps);
size_t rowtile_desc_bytes();
// Target alpha rows [lo, hi) of a prepared description only, written into
// Dp[rank - lo * N_beta] (touched tiles are overwritten, the rest is left
// as it is: Dp must be zero there).  Synchronises the stream.
void launch_sigma_rowtile_rows(sfci_problem* P, const RowTileDesc& all, u64 lo, u64 hi, double* Dp);
// What the tile kernel does with each finished tile instead of writing it to
// a dense slice (the list iteration's passes, fused): (1) y is gathered at the
// entries of w_l, l < nl, that fall in the tile (T_lj; Y[l cap + i]); (2) the
// entries of w_l, l >= mark_from, are left out of the candidates (Eq. 10 forms
// them afterwards); (3) with collect, every other entry with |y| above the
// running bound joins the candidate list (Rr, Ra at atomically taken
// positions; overflow set when Rcap is reached, Rn still counts); (4) the
// nonzero entries are counted into *distinct when it is set.  y is the
// screened value (|y| < eps written as 0).  Lives in device memory.
struct FusedOut {
    const u64* Wr;      // basis ranks, w_l at Wr + l cap (rank-sorted)
    const u64* rowptr;  // per l < nl: na_rows + 1 offsets, the first entry of w_l in each alpha row
    double* Y;          // gathered y, Y[l cap + i]
    u64 cap;
    u64 na_rows;
    int nl, mark_from;
    int collect, pad;
    const u64* bound;   // bits of |c| a candidate must exceed
    u64* Rr;
    double* Ra;
    u64* Rn;
    u64 Rcap;
    int* overflow;
    u64* distinct;      // may be NULL
};
// Sigma by target rows with an LDS hash table each (hashrows.hip): the terms
// of every target row and the lists of source rows that reach it (kept in
// list_ws), then rows[lo .. hi) (device) handed to the FusedOut at d_fo.  A
// part of a row that did not fit sets *overflow to 2 or 3: to be run again with
// a larger more.  The counts and the rows synchronise the stream.
struct HashReach {
    std::vector<u64> count;    // terms per target row
    u64 terms = 0, pairs = 0;  // of all rows; pairs of a target row and a source row
    bool placed = false;
};
// lists_follow: the lists are made next in any case, and the counts are the
// host's only after that.
void hash_rows_count(sfci_problem* P, const RowTileDesc& all, bool lists_follow, HashReach* out);
bool hash_rows_lists(sfci_problem* P, const RowTileDesc& all, HashReach* reach);  // false: too long for the device
u64 hash_rows_parts(u64 terms);  // in how many parts a row of so many terms is taken
void launch_hash_rows(sfci_problem* P, const SigmaLaunch& sl, const RowTileDesc& all, u64 lo, u64 hi, const u32* rows,
                      const FusedOut* d_fo, unsigned long long* emitted, double eps, u32 more, bool small);
u64 hash_rows_small();  // rows of at most so many terms take the small table
// Target alpha rows [lo, hi) of a prepared description, or rows[lo .. hi) of a
// device list, each finished tile handed to the FusedOut at d_fo (device)
// instead of being written.  Synchronises the stream.
void launch_sigma_rowtile_rows_fused(sfci_problem* P, const RowTileDesc& all, u64 lo, u64 hi, const FusedOut* d_fo,
                                     const u32* rows = nullptr);
unsigned rowtile_grid(int num_cu, const RowTileGeom& geom, u64 total_items, unsigned per_cu_override = 0);
unsigned rowtile_grid(int num_cu, size_t lds_bytes, u64 total_items, unsigned per_cu_override = 0);
size_t rowtile_scratch_bytes(unsigned grid, u64 nbr_cap);
// fill_counter = false: the caller has already zeroed *d_counter on the stream.
// timed: the diagnostic build with per-phase timing (descriptions carrying phase_ns).
void rowtile_run(hipStream_t stream, int num_cu, const void* d_descs, const u64* d_prefix, int n_inst,
                 unsigned* d_counter, void* scratch, u64 nbr_cap, const RowTileGeom& geom, u64 total_items,
                 bool fill_counter = true, const RowTileTune& tune = RowTileTune{}, bool timed = false);

// Integral gradients through the target-owned tiles: for each job,
// L = s^T H(h, g) v with s and v sparse (ascending unique ranks).  Raw
// gradients accumulate into Rh (n^2) and Rg (n^4), which the call zeroes
// first, and are then symmetrised into dh / dg (either may be NULL).  The
// dense array of every problem must be zero on entry; it is zero on exit.
// vt_* is scratch for the transposed v (capacity v.cap).
struct GradJob {
    sfci_problem* P;
    SigmaLaunch v;
    const u64* s_rank;
    const double* s_amp;
    const u64* s_nnz;
    u64 s_cap;
    double *Rh, *Rg, *dh, *dg;
    u64* vt_rank;
    double* vt_amp;
    u64* vt_nnz;
    // sbar is v scaled by a constant (the energy's gradient): each pair of
    // distinct connected rows is then visited once and counted twice
    bool pair_sym;
    const int* bad;  // as in launch_backward_dense
};
bool rowtile_grad_available(sfci_problem* P);
void rowtile_gradients(hipStream_t st, int n_jobs, const GradJob* jobs, RowTileGradWs& ws);
void launch_symmetrise(sfci_problem* P, const double* Rh, const double* Rg, double* dh, double* dg,
                       const int* bad = nullptr);

// ---- utilities (util.hip) ----
void launch_fill_f64(double* p, u64 n, double val, hipStream_t s);
void launch_fill_u64(u64* p, u64 n, u64 val, hipStream_t s);
// exclusive scan of n u64 counts into out (may alias); total -> *total_dev (device scalar).
void exclusive_scan_u64(sfci_problem* P, const u64* in, u64* out, u64 n, u64* total_dev);

// ---- selection (select.hip) ----
// ---- batched iteration steps: one launch serves every instance ----
// One instance of a batch, in a device array indexed by blockIdx.y: its basis
// vectors, dense accumulator, block matrices, and selection workspaces.
struct BInst {
    u64* Wr;                  // basis vector l: ranks Wr + l cap, amplitudes Wa + l cap, count sc[l]
    double* Wa;
    u64* sc;
    u64 cap;
    double* D;                // dense accumulator, N_det doubles (all zero between steps)
    u64 Ndet;
    double* T;                // n_L x n_L, T[l n_L + j]
    double* S;
    double* x;                // block end: the lowest eigenvector, its eigenvalue, energies[*blk]
    double* lam;
    double* energies;
    int* blk;
    int* status;
    double* red;              // reduction partials, bstep_red_doubles(n_L)
    SelState* st;             // selection
    u64* cr;                  // candidate segments (N_det capacity)
    double* ca;
    u64* cnt;                 // per segment (select chunks of N_det): kept entries and their scan,
    u32* ccnt;                // and candidates
    u64* psi_r;               // the final Psi of the last block
    double* psi_a;
    u64* psi_n;
    u64 M;                    // truncation (UINT64_MAX: every nonzero entry)
    u64 ndet_m1;              // key geometry of the selection
    int rank_bits;
    int nL;
};
// Where a batched selection writes: w_{j+1}, w_0 (a block end) or Psi.
enum { BOUT_NEXT = 0, BOUT_W0 = 1, BOUT_PSI = 2 };
u64 bstep_red_doubles(int nL);
// T[l][j] = T[j][l] = <w_l|D> and S[l][j] = S[j][l] = <w_l|w_j> for l <= j
void bstep_dots(hipStream_t st, const BInst* d, int n, int j, int nL);
// kind 0: D -= T[l][j] w_l;  kind 1: D += x[l] w_l
void bstep_axpy(hipStream_t st, const BInst* d, int n, int l, int j, int kind, u64 max_cap);
// Eq. 11 on the selection's output vector
void bstep_normalise(hipStream_t st, const BInst* d, int n, int out_kind, int j, u64 max_cap);
void bstep_fill_zero(hipStream_t st, const BInst* d, int n, u64 max_ndet);
void bstep_geneig(hipStream_t st, const BInst* d, int n, int nL);
void bstep_inc_blk(hipStream_t st, const BInst* d, int n);
// select_topm of every instance's dense accumulator (zeroed on the way unless
// !zero) into the out_kind vector, keeping M entries (all != 0: every nonzero entry).
void bstep_select(hipStream_t st, const BInst* d, int n, int out_kind, int j, u64 max_ndet, int num_cu, int band,
                  int max_ndig, int all, bool zero = true);

// Select the M largest (|c|, then lower rank) nonzero candidates and write them
// by ascending rank to (out_rank, out_amp); *out_count_dev receives the count.
// If zero_dense, the dense source is cleared to 0.0 in the same pass.
// M == UINT64_MAX keeps all nonzero candidates.
void select_topm(sfci_problem* P, const CandSrc& src, u64 M, u64* out_rank, double* out_amp, u64* out_count_dev,
                 bool zero_dense);
// Two-phase form: prepare (selection levels + counts; the count goes to
// *count_dev), then write.  The state lives in the problem's workspace, so no
// other selection may run in between.  Truncating a dense source (M neither 0
// nor UINT64_MAX) clears it in the first phase already.
void select_prepare(sfci_problem* P, const CandSrc& src, u64 M, u64* count_dev);
void select_write(sfci_problem* P, const CandSrc& src, u64* out_rank, double* out_amp, bool zero_dense);
// The same two phases on a candidate list with caller-given working memory
// (no allocation): the state and select_segments(lcap) offsets.
struct SelWs {
    SelState* st;
    u64* off;
};
// Whether select_topm of the dense accumulator takes no more memory than the two-phase form.
bool select_one_step(const sfci_problem* P, u64 M);
u64 select_chunks(u64 n_upper);  // of a dense source of n_upper slots
int select_shift(u64 lcap);      // log2 of a list's entries per segment
u64 select_segments(u64 lcap);
void select_prepare_ws(sfci_problem* P, const CandSrc& src, u64 M, u64* count_dev, const SelWs& ws);
void select_write_ws(sfci_problem* P, const CandSrc& src, u64* out_rank, double* out_amp, const SelWs& ws);

// ---- small spaces (smallh.hip; the step kernels in select.hip) ----
// Whether H is kept as a table (builds it on first use).
bool small_h_ready(sfci_problem* P);
// The input vector of the next launch_small_sigma: n_host entries, or *n_dev.
// check: flags[0] a rank out of range, flags[1] ranks not strictly ascending
// (the vector then counts as empty).  nnz_out, hist (may be NULL) receive the
// length; its terms are added to *emitted.
void launch_small_load(sfci_problem* P, const u64* r, const double* a, const u64* n_dev, u64 n_host, bool check,
                       u64* nnz_out, u64* hist, u64* emitted, int* flags);
// D = H v (every slot written; |y| < eps written as 0).
void launch_small_sigma(sfci_problem* P, double eps);
// The rest of an iteration step: the basis and what a step writes.
struct SmallStep {
    u64* Wr;
    double* Wa;
    u64* nnz;  // of w_l
    u64 cap;
    double* D;
    u64 N;
    double* vd;    // dense copy of the vector sigma is applied to
    const u32* nz; // terms per column of H
    double *T, *S;
    int nL, band;
    u64 M;
    u64* emitted;
    u64* hist;  // nnz of the block's vectors
    int rank_bits;
    int w_lds;  // the dense copy fits in LDS beside the accumulator
};
void small_step_setup(sfci_problem* P);
void launch_small_step(sfci_problem* P, const SmallStep& s, int j);
void launch_small_psi(sfci_problem* P, const SmallStep& s, const double* x, bool final);

// ---- sort path (sortpath.hip) ----
// sigma = H v by stable sort + in-order segmented sum; result sorted by rank,
// zeros dropped, in (out_rank, out_amp) with *out_count_dev; returns false if
// the result would exceed out_cap (then *out_count_dev = needed).
// eps > 0 drops sums with |sum| < eps (screening, Sec. 3).
void sigma_sorted(sfci_problem* P, const SigmaLaunch& v, u64 out_cap, u64* out_rank, double* out_amp,
                  u64* out_count_dev, u64* emitted_dev, double eps = 0.0);
// Pass-by-pass form: a pass covers a range [alo, ahi) of target alpha ranks
// (ascending, disjoint).  Before a pass's reduction the sink says where its
// entries go (appended at out[*base_dev ...], *base_dev advanced by their
// number); after it, the sink may consume them.  tup_cap = 0: sized from free
// memory.  Returns the number of passes run.
struct SortPassOut {
    u64* r;
    double* a;
    u64 cap;
    u64* base_dev;
};
struct SortPassSink {
    virtual SortPassOut begin(u64 alo, u64 ahi, u64 tuples) = 0;
    virtual void end(u64 alo, u64 ahi) = 0;
    virtual ~SortPassSink() = default;
};
// Device bytes per sort-path tuple over the emission, sort and reduction buffers.
constexpr u64 SFCI_SORT_TUPLE_BYTES = 2 * (sizeof(u64) + sizeof(double)) + sizeof(double) + sizeof(u64);
u64 sort_tuple_cap(sfci_problem* P);
u64 sigma_sorted_passes(sfci_problem* P, const SigmaLaunch& v, SortPassSink& sink, u64* emitted_dev, u64 tup_cap,
                        double eps);
// The same passes with target-row-driven emission (rowpass.hip): per-row
// tuple counts once per call, then per pass only the (target row, source
// row) pairs that land in it.
u64 sigma_rowpass(sfci_problem* P, const SigmaLaunch& v, SortPassSink& sink, u64* emitted_dev, u64 tup_cap,
                  double eps);
// K = u64 or u32.
template <class K>
void radix_sort_pairs(sfci_problem* P, K* k1, double* v1, K* k2, double* v2, u64 n, int kbits, K** k_out,
                      double** v_out);
int key_bits(u64 maxval);
// Entries per radix-sort tile.
constexpr u64 SFCI_SORT_TILE = 4096;
// Stable sort of pass-local keys (target row - lo) * N_beta + beta rank whose
// entries are already grouped by target row in ascending row order: only the
// beta rank is sorted, inside each row.  tpre / ttile hold the entries and the
// tiles (ceil(entries / SFCI_SORT_TILE)) before every row of the space,
// ntiles = ttile[hi] - ttile[lo]; tile_row has room for ntiles entries.
void radix_sort_rows(sfci_problem* P, u32* k1, double* v1, u32* k2, double* v2, u64 n, const u64* tpre,
                     const u64* ttile, u64 lo, u64 hi, u64 ntiles, u32* tile_row, u32** k_out, double** v_out);
template <class K>
void segmented_sum_append(sfci_problem* P, const K* keys, const double* vals, u64 n, u64 key_base, double eps,
                          u64* out_base_dev, u64 out_cap, u64* out_r, double* out_a);

// ---- Lanczos vector ops (lanczos.hip) ----
void launch_dot_dense(sfci_problem* P, const u64* r, const double* a, const u64* nnz, u64 cap, const double* D,
                      double* out1, double* out2, bool ordered);
// The dots of iteration step j: T_lj = <w_l|y> and S_lj = <w_l|w_j>, l = 0..j,
// written to both triangles of the n_L x n_L matrices.
struct StepDots {
    const u64* Wr;  // basis vector w_l at Wr + l cap, Wa + l cap, nnz[l] entries
    const double* Wa;
    const u64* nnz;
    u64 cap;
    int j, nL;
    const double* y;  // ystride = 0: dense, y[rank]; else y at entry i of w_l is y[l ystride + i]
    u64 ystride;
    double *T, *S;
};
void launch_step_dots(sfci_problem* P, const StepDots& d, bool ordered);
// sum of x[0..*nnz) (ordered: strictly in index order) and sum of squares
void launch_sum(sfci_problem* P, const double* x, const u64* nnz, u64 cap, double* out, bool ordered);
void launch_sumsq(sfci_problem* P, const double* a, const u64* nnz, u64 cap, double* out, bool ordered);
void launch_dot_sparse(sfci_problem* P, const u64* xr, const double* xa, const u64* xn, u64 xcap, const u64* yr,
                       const double* ya, const u64* yn, double* out1, double* out2, bool ordered);
void launch_axpy_scatter(sfci_problem* P, double* D, const u64* r, const double* a, const u64* nnz, u64 cap,
                         const double* coef, double sign);
void launch_normalise(sfci_problem* P, double* a, const u64* nnz, u64 cap, bool ordered, double* part_ws = nullptr);
// doubles of working memory launch_normalise needs (part_ws)
u64 normalise_ws_doubles();
void launch_scatter_set(sfci_problem* P, double* D, const u64* r, const double* a, const u64* nnz, u64 cap);
// energy_slot[blk ? *blk : 0] receives lambda (blk: device block index, may be null)
void launch_geneig_full(sfci_problem* P, int m, const double* T, const double* S, double* lambda, double* x,
                        double* energy_slot, int* status, bool ordered, const int* blk = nullptr);
void launch_inc_int(sfci_problem* P, int* p);
void launch_add_u64(sfci_problem* P, u64* dst, const u64* src);  // *dst += *src
void launch_div_by_sumsq(sfci_problem* P, const double* a, const u64* nnz, u64 cap, double* out);

int sfci_set_error(int code, const std::string& msg);

// ---- host helpers shared by the ABI files (abi.hip) ----
void sfci_sync(sfci_problem* P);
void launch_set_u64(sfci_problem* P, u64* p, u64 v);
void validate_vec(sfci_problem* P, const u64* r, u64 n);  // throws on out-of-range or unsorted ranks
bool ensure_dense(sfci_problem* P);                       // allocates the zeroed N_det accumulator if it fits
void dense_sigma(sfci_problem* P, const SigmaLaunch& sl, int dedup, unsigned long long* emitted, double eps = 0.0);
// Zeroes the N_det array when an error leaves a call while the array holds
// sums (armed, until done): the next call counts on zeros.
void clear_dense(sfci_problem* P, hipStream_t st) noexcept;
struct DenseGuard {
    sfci_problem* P;
    bool armed = true;
    explicit DenseGuard(sfci_problem* P_) : P(P_) {}
    DenseGuard(const DenseGuard&) = delete;
    void done() { armed = false; }
    ~DenseGuard() {
        if (armed) clear_dense(P, P->stream);
    }
};
// Screening (Sec. 3): D[i] = 0 where 0 < |D[i]| < eps.
void launch_screen(sfci_problem* P, double* D, u64 n, double eps);

// Device time of a sequence of bracketed regions on a stream (HIP events).
struct EventTimer {
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
    bool on = false;
    void begin(hipStream_t s) {
        if (!on) return;
        hipEvent_t a, b;
        SFCI_CHECK_HIP(hipEventCreate(&a));
        SFCI_CHECK_HIP(hipEventCreate(&b));
        SFCI_CHECK_HIP(hipEventRecord(a, s));
        ev.push_back({a, b});
    }
    void end(hipStream_t s) {
        if (!on) return;
        SFCI_CHECK_HIP(hipEventRecord(ev.back().second, s));
    }
    double total_ms() {
        double t = 0.0;
        for (auto& p : ev) {
            float ms = 0.f;
            SFCI_CHECK_HIP(hipEventElapsedTime(&ms, p.first, p.second));
            t += ms;
        }
        return t;
    }
    ~EventTimer() {
        for (auto& p : ev) {
            (void)hipEventDestroy(p.first);
            (void)hipEventDestroy(p.second);
        }
    }
};

// ---- list-based iteration and truncated sigma without an N_det array (listlz.hip) ----
// sigma = H v in passes of target alpha rows (the sort path's, or with
// tiles_ok by target rows: tiles for all, or hash tables and tiles);
// the top-M (tie rule) sorted by rank into out when it fits out_cap.  Returns
// the selected count; *distinct_host (may be NULL) receives the number of
// distinct nonzero entries.
u64 sigma_list_topm(sfci_problem* P, const SigmaLaunch& v, u64 M, u64* out_rank, double* out_amp, u64 out_cap,
                    u64* emitted_dev, u64* distinct_host, bool tiles_ok, double eps = 0.0);
// Fast mode's per-sigma choice of the tile kernel for all rows, from the
// input's size (SFCI_LIST_SIGMA=tile|sort forces).
bool list_sigma_tiles(sfci_problem* P, u64 nnz);
// sigma = H v in full through the sort path's passes, no N_det array: the
// nonzero entries sorted by rank in list_ws.Rr / Ra; returns their number.
u64 sigma_list_full(sfci_problem* P, const SigmaLaunch& v, u64* emitted_dev, u64** r, double** a);
// H v in full as a rank-sorted list (zeros dropped): the N_det array (in-order
// rows when deterministic, else the tile kernel) compacted in rank order (it
// is zero again afterwards), or the sort path where those do not apply.
// The list lives in the problem's workspace until the next such call;
// *cnt_dev receives its length, which is also returned.
u64 sigma_full_list(sfci_problem* P, const SigmaLaunch& sl, bool det, u64* emitted, u64** yr, double** ya,
                    u64* cnt_dev);
// The basis and the per-block outputs the iteration writes (device).
struct ListBasis {
    u64 cap;        // entries per basis vector
    u64* Wr;        // n_L x cap ranks
    double* Wa;     // n_L x cap amplitudes
    u64* sc;        // [0, n_L) nnz per vector, [32] emitted-term counter
    double *Td, *Sd, *xd, *lam, *energies_d;
    int* status_d;
    u64* nnz_hist;  // nnz of each sigma input, block after block
};
// w_0 must already hold the normalised start vector.  *psi_n_out receives the
// last Psi's length; it is copied to psi_out when it fits.
void lanczos_list(sfci_problem* P, const sfci_lanczos_opts* o, const ListBasis& B, sfci_svec* psi_out, u64* psi_n_out,
                  u64* sigma_calls, EventTimer& tsig, int* blocks_run);
// Halting test of Sec. 2.1 after block b (energies on the device): true when
// o->conv_eps > 0, b >= 1 and E(b-1) - E(b) < conv_eps.  Synchronises when it
// has to look.
bool halt_after_block(sfci_problem* P, const sfci_lanczos_opts* o, const double* energies_d, int b);

// Device-resident sparse vector with a device nnz (Lanczos basis storage).
struct DVec {
    u64* r = nullptr;
    double* a = nullptr;
    u64* nnz = nullptr;
    u64 cap = 0;
};
