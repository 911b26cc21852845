// Fused RQA engine for gfx950: recurrence predicate, diagonal / vertical /
// white-vertical run extraction and histogram recombination in one pass over
// the upper triangle of the recurrence matrix, which is never stored.
//
// Mapping of the paper's method (Sect. 4):
//  * operator I (similarity of one vector pair) -- evaluated once per unique pair
//    i < j with j - i >= max(theiler, 1): the matrix is symmetric, so the lower
//    triangle is recovered by mirroring (Sect. 4.2 notes that a symmetric matrix
//    needs only N-1 diagonals);
//  * operators II and III (lines along one diagonal / one column) -- run-length
//    state machines over 64-bit bit-words of 64x64 tiles;
//  * divide & recombine with carry-over (Sect. 4.1) -- open runs are carried
//    across tile edges in registers (left to right) and through LDS between the
//    waves of a workgroup (top to bottom); runs that touch the top or bottom edge
//    of a workgroup's strip are summarised and joined by the stitch kernel.
//
// Geometry.  n delay vectors, w' = max(theiler, 1).  U = {(i,j): j - i >= w'}.
// A workgroup of W waves owns a strip of H = 64*W consecutive rows; wave w owns
// rows R = R0 + 64w .. R+63, one row per lane, and walks the 64-column tiles
// c = c0 .. c_last of its strip left to right.  The waves run as a pipeline:
// wave w takes the open runs of a tile's columns and diagonals as wave w-1 left
// them, from state rings in LDS (no workgroup barrier per tile; wave 0 may run
// up to kRing tiles ahead of the last wave).  An open run is kept as the position
// where it began, so a tile that changes no run's colour needs no work at all.
//
// Full-matrix lines from U:
//  * a diagonal k >= w' of U and its mirror -k: each run counted twice;
//  * column j of the full matrix = [column j of U: rows 0..j-w'] ++ [middle] ++
//    [row j of U: columns j+w'..n-1], the middle being the Theiler band (white,
//    theiler >= 1) or the single recurrent cell (j,j) (theiler = 0).  Runs inside
//    either segment are counted where they are found; the trailing run of the
//    column segment, the middle and the leading run of the row segment are
//    merged by the join step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <vector>

#include "rqa_internal.h"

namespace rqa {

KParams make_kparams(const rqa_params &p) {
    KParams k;
    k.m = p.m;
    k.tau = p.tau;
    k.eps = p.eps;
    volatile float e = p.eps;   // one FP32 rounding of eps*eps, no contraction
    k.eps_sq = e * e;
    // First-coordinate bound.  The accumulated distance a never falls below the
    // first coordinate's term (a sum or max of non-negative terms, and rounding
    // is monotone), and that term is monotone in |d_0|, so |d_0| > d0_bound
    // decides "not recurrent" exactly.
    if (p.norm != RQA_NORM_L2) {
        k.d0_bound = p.eps;
    } else if (!std::isfinite(k.eps_sq)) {
        k.d0_bound = std::numeric_limits<float>::infinity();
    } else {
        // Largest t >= 0 with fl32(t*t) <= eps_sq: binary search over the bit
        // patterns of non-negative floats, which are ordered like the values
        // (fl32(0*0) = 0 <= eps_sq; fl32(inf*inf) = inf > eps_sq).
        uint32_t lo = 0u, hi = 0x7F800000u;
        while (hi - lo > 1u) {
            const uint32_t mid = lo + (hi - lo) / 2u;
            float t;
            std::memcpy(&t, &mid, sizeof t);
            volatile float tv = t;
            volatile float sq = tv * tv;
            if (sq <= k.eps_sq) lo = mid; else hi = mid;
        }
        std::memcpy(&k.d0_bound, &lo, sizeof lo);
    }
    k.norm = p.norm;
    k.theiler = p.theiler;
    k.lmin = p.lmin;
    k.vmin = p.vmin;
    k.wmin = p.wmin;
    return k;
}

namespace {

constexpr int kMaxWaves = 8;
constexpr int kCapD = 1024;    // LDS bins for diagonal lengths < kCapD
constexpr int kCapV = 1024;    // LDS bins for vertical lengths < kCapV
constexpr int kCapW = 6016;    // LDS bins for white-vertical lengths < kCapW; a launch whose
                               // jobs have no longer line takes fewer (GroupDesc::capw)
constexpr int kMaxM = 6;       // embedding dimensions held in registers
constexpr int kRing = 32;      // column-state slots: tiles wave 0 may run ahead of the last wave
constexpr int kDiagRing = 64;  // diagonal-state slots (of 64 diagonals each); at most
                               // kRing + kMaxWaves of them are live at once
constexpr int kGroup = 8;      // column tiles classified at a time
constexpr uint32_t kSpinLimit = 1u << 20;   // polls (~28 ms) before a neighbour wait gives up
constexpr int kStitchThreads = 512;
constexpr int kStitchBatch = 8;   // strips whose summaries a stitch thread loads at once
constexpr int kFewRows = 4;       // non-zero rows up to which a tile is not transposed
static_assert(32 % kStitchBatch == 0, "a batch lies in one word of the masks");
constexpr int kStitchCapV = 2048; // stitch LDS bins for vertical lengths < kStitchCapV (the
                                  // stitch joins the runs that cross strip edges: long ones)
constexpr int kStatThreads = 256;
constexpr int kStatMaxBlocks = 60;
constexpr int kStatLengths = 2048;   // lengths per statistics block (8 per thread: the blocks'
                                     // loops are chains of dependent loads)
constexpr int kPrepareBlocks = 64;   // k_prepare blocks per job, at most
constexpr int kPrepareThreads = 256;
constexpr int kCounters = 64;        // work counters of a launch
// Boxes (exact pruning of the predicate, see classify): of every kBoxVecs
// consecutive delay vectors the smallest and the largest of each of the first
// kBoxK coordinates, in planes (minimum, maximum of coordinate 0, 1, 2).  Which
// jobs take them: boxes_pay.
constexpr int kBoxK = 3;
constexpr int kBoxVecs = 8;
constexpr int kBoxHeader = 64;       // floats before the first plane: the samples' counts
constexpr int kSamples = 32;         // pieces sampled per k_prepare block (see sample_piece)

// Device-side description of one job (one series or window).
struct JobDesc {
    const float *s;            // series of the rows (n_points values)
    const float *sb;           // series of the columns (auto: s)
    const uint64_t *bits;      // given matrix: n rows of `words` u64 (bit b of word c = column 64c+b)
    int64_t words;
    int64_t n_points_b;        // points of sb
    const float *tail;         // coordinates of the last column tile, zero padded
    unsigned long long *hd;    // histograms, n+1 entries each
    unsigned long long *hv;
    unsigned long long *hw;
    int *flag;                 // non-finite flag
    uint32_t *lead;            // leading run of each row of U: len | color<<31
    uint32_t *hfirst;          // auto, segments > 1: per (row, segment) first / last run of
    uint32_t *hlast;           // the row's piece in the segment, len | color<<31
    uint16_t *vfirst;          // per (strip, column): first run len | color<<15
    uint16_t *vlast;           // per (strip, column): last run len | color<<15
    uint16_t *dfirst;          // per (strip, diagonal): black run at the top edge
    uint16_t *dlast;           // per (strip, diagonal): black run at the bottom edge
    int64_t n_points;
    int32_t n;                 // delay vectors (rows)
    int32_t nb;                // columns (auto: n)
    int32_t hmax;              // longest possible line; histograms hold hmax+1 entries
    int32_t mode;              // JobMode
    int32_t m, tau, norm, theiler, wp;
    float thr;                 // eps (L1, Linf) or fl32(eps*eps) (L2)
    float thr0;                // first-coordinate bound (KParams::d0_bound)
    int32_t H;                 // strip height
    int32_t nstrips;
    int32_t segs;              // column segments per strip (1: strips are not cut)
    int32_t seg_tiles;         // column tiles per segment; segment g covers the column
                               // tiles [seg_base + g*seg_tiles, seg_base + (g+1)*seg_tiles)
    int32_t seg_base;          // first column tile of segment 0 (auto: wp/64; full: 0)
    int32_t dw;                // diagonal summary slots per (strip, segment) block (segs > 1
                               // or full matrix)
    int32_t c_last;            // last column tile (nb-1)/64
    int32_t tail_len;          // floats in tail
    int32_t strip_base;        // first work item of this job within its group
    int32_t stitch_block0;     // first stitch block of this job
    int32_t mins[3];           // lmin, vmin, wmin
    int32_t stat_blocks;       // blocks of the statistics kernels for this job
    uint8_t *nonfinite;        // kPrepareBlocks bytes: k_prepare block b saw a non-finite value
    uint32_t *stat_done;       // statistics blocks of this job that have finished
    unsigned char *host_info;  // pinned host copy of the info record (nullptr: none)
    uint32_t run;              // number of the run (Job::run)
    unsigned long long *host_hist;   // pinned host copy of the histograms (nullptr: none)
    JobStats *stats;           // device statistics record
    double *ent_part;          // [3][kStatMaxBlocks] entropy partial sums
    float *boxr, *boxc;        // boxes of the rows' and the columns' vectors (one series:
                               // the same), nullptr if none
    int32_t ncr, ncc;          // entries per plane
    uint8_t *decided;          // kPrepareBlocks bytes: of k_prepare block b's kSamples pieces, those
                               // that boxes decide (blocks from sample_blocks on sample none)
    int32_t sample_blocks;
    uint32_t *vmask;           // which summaries were written (process_strip), a bit per strip
    uint32_t *dfmask;          // of the row band: per column tile from seg_base on, and per block
    uint32_t *dlmask;          // of 64 diagonals at a strip's top edge and at its bottom edge
    int32_t mask_words;        // words per tile or block
    int32_t kb_off;            // entry of diagonal block 0
    int64_t mask_total;        // words of the three masks, which lie one after the other
    int32_t spin_limit;        // polls before a neighbour wait gives up (kSpinLimit)
    int32_t wait_bias;         // added to every wait target: 0, or (fault injection
                               // for tests) a bias no counter reaches
    // Row bands (auto mode): the launch walks strips [s_lo, s_hi) of band_strips
    // per band; summary slots are relative to strip s_lo (strip_offset(s_lo) =
    // soff_lo).  With several bands the open run of each column of U and of
    // each diagonal passes to the next band through cstate / dstate.
    int32_t s_lo, s_hi;
    int32_t band_strips, nbands;
    int64_t soff_lo;
    uint32_t *cstate;          // per column: open run len | color<<31 (nbands > 1)
    uint32_t *dstate;          // per diagonal: open black run length (nbands > 1)
};

struct GroupDesc {
    int32_t job0, job1;        // jobs [job0, job1) of the descriptor table
    int32_t items;             // total strips of the group
    int32_t capw;              // LDS bins for white lengths: enough for the longest line, at
                               // most kCapW (short jobs: more workgroups per CU, less to clear)
};

__host__ __device__ inline int64_t strip_offset(int32_t s, int32_t n, int32_t wp, int32_t H) {
    // sum_{s' < s} (n - wp - s' H): entries of the strips before s
    return (int64_t)s * (n - wp) - (int64_t)H * ((int64_t)s * (s - 1) / 2);
}

// ---------------------------------------------------------------------------
// Bit-word helpers (64-bit words split in two VGPRs; bit p = position p along a
// line).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t mk64(uint32_t lo, uint32_t hi) {
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t range_mask(uint32_t lo, uint32_t hi) {
    // bits [lo, hi), 0 <= lo <= hi <= 64
    const uint64_t a = lo >= 64 ? 0ull : (~0ull << lo);
    const uint64_t b = hi >= 64 ? ~0ull : ((1ull << hi) - 1ull);
    return a & b;
}

// Lane exchange within 32-lane halves: lane l reads lane l^D (ds_swizzle in
// xor mode; no VALU work).
template <int D>
__device__ __forceinline__ uint32_t swizzle_xor(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (D << 10));
}

// One butterfly stage of the 64x64 bit transpose, D in {16,8,4,2,1}: lanes l and
// l^D exchange bit blocks.  M marks the bit positions whose D-bit is 0.  The
// lower lane keeps its M positions and takes the partner's M positions moved up
// by D; the upper lane keeps its ~M positions and takes the partner's ~M
// positions moved down by D.  The move is a rotation (v_alignbit); the bits it
// wraps around fall outside the selected positions, so one v_bfi finishes the
// stage.
template <int D, uint32_t M>
__device__ __forceinline__ void transpose_stage(uint32_t &lo, uint32_t &hi, int lane) {
    const bool up = (lane & D) != 0;
    const uint32_t keep = up ? ~M : M;
    const uint32_t amt = up ? (uint32_t)D : (uint32_t)(32 - D);
    const uint32_t rl = swizzle_xor<D>(lo);
    const uint32_t rh = swizzle_xor<D>(hi);
    const uint32_t sl = __builtin_amdgcn_alignbit(rl, rl, amt);
    const uint32_t sh = __builtin_amdgcn_alignbit(rh, rh, amt);
    lo = (keep & lo) | (~keep & sl);
    hi = (keep & hi) | (~keep & sh);
}

// In-register transpose of a 64x64 bit matrix held one row per lane: on return
// lane l holds column l (bit r = old lane r's bit l).  The 32-lane stage is one
// v_permlane32_swap (upper lanes of `lo` <-> lower lanes of `hi`); the other five
// stages are butterflies within 32-lane halves.
__device__ __forceinline__ void transpose64(uint32_t &lo, uint32_t &hi, int lane) {
    const auto sw = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
    lo = sw[0];
    hi = sw[1];
    transpose_stage<16, 0x0000FFFFu>(lo, hi, lane);
    transpose_stage<8, 0x00FF00FFu>(lo, hi, lane);
    transpose_stage<4, 0x0F0F0F0Fu>(lo, hi, lane);
    transpose_stage<2, 0x33333333u>(lo, hi, lane);
    transpose_stage<1, 0x55555555u>(lo, hi, lane);
}

// 64-bit rotate right by r (0..63), branch-free.
__device__ __forceinline__ void rotr64(uint32_t &lo, uint32_t &hi, uint32_t r) {
    const bool sw = (r & 32) != 0;
    const uint32_t a = sw ? hi : lo;
    const uint32_t b = sw ? lo : hi;
    const uint32_t s = r & 31;
    lo = __builtin_amdgcn_alignbit(b, a, s);
    hi = __builtin_amdgcn_alignbit(a, b, s);
}

// ---------------------------------------------------------------------------
// Run state machine.  A line is cut into segments; `Run` is the open run at the
// current position: colour (1 = recurrent), where it began, and whether it is the
// first run of the current segment (then it is recorded instead of counted).
// Keeping the start rather than the length makes a tile without colour changes
// free: nothing is added up for it.
// ---------------------------------------------------------------------------
struct Run {
    uint32_t color;
    uint32_t start;     // position where the run began: column (rows of U), or row within the
                        // strip (columns and diagonals: at most 64 * kMaxWaves, 10 bits)
    uint32_t first;
};

// Column and diagonal states in LDS: 16 bits.
__device__ __forceinline__ uint16_t pack_run(const Run &r) {
    return (uint16_t)((r.start & 0x3FFu) | (r.first << 14) | (r.color << 15));
}
__device__ __forceinline__ Run unpack_run(uint32_t v) {
    return Run{(v >> 15) & 1u, v & 0x3FFu, (v >> 14) & 1u};
}
constexpr uint32_t kFreshColumn = 1u << 14;   // white from row 0 of the strip, the first run
constexpr uint32_t kNoDiagonal = 0u;          // white, not first: nothing to record or count

// Global-memory access through address-space-1 pointers.  The kernels reach
// HBM through pointers held in the job descriptor, which the compiler cannot
// prove global; it would emit flat instructions, and every flat access also
// counts against the LDS/scalar wait counter, so a later wait for a scalar load
// would also wait for outstanding histogram atomics and summary stores.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T *glb(T *p) {
    return (__attribute__((address_space(1))) T *)p;
}
__device__ __forceinline__ void g_add(unsigned long long *p, unsigned long long v) {
    __hip_atomic_fetch_add(glb(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void g_or(int *p, int v) {
    __hip_atomic_fetch_or(glb(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS bins, one after the other: diagonal (kCapD), vertical (kCapV), white
// vertical (kCapW) lengths.
struct Bins {
    uint32_t *d, *v, *w;
    int capw;
};

// Columns (y) and diagonals (z: the rows rotated right by their number, then
// transposed) of a tile in which only the rows `rows` have cells: a row's word is
// the mask of the lanes that get its bit.  Two transposes are ~80 vector
// instructions and two chains of LDS swizzles; a row costs six here.  Without it
// noise and AR(1) series with m = 5, a few recurrences to a tile, are 1-5% slower (300
// windows of 6,000 points 2,522 -> 2,584 us, 9,000 points 174 -> 183), logistic and
// sine windows 1-2% faster, others the same; with limits of 2 or 8 rows 32 calls of
// five kinds of series stayed within 1%.
__device__ __forceinline__ void gather_rows(uint32_t xlo, uint32_t xhi, uint32_t rows, int base,
                                            uint32_t &y, uint32_t &z) {
    y = z = 0u;
    while (rows) {
        const int r = __builtin_ctz(rows);
        rows &= rows - 1u;
        const uint64_t w = mk64((uint32_t)__builtin_amdgcn_readlane((int)xlo, base + r),
                                (uint32_t)__builtin_amdgcn_readlane((int)xhi, base + r));
        const uint64_t turned = (w >> (base + r)) | (w << ((64 - base - r) & 63));
        const uint32_t bit = 1u << r;
        y |= __builtin_amdgcn_inverse_ballot_w64(w) ? bit : 0u;
        z |= __builtin_amdgcn_inverse_ballot_w64(turned) ? bit : 0u;
    }
}

// A length beyond the LDS bins goes to the global histogram; one beyond the
// histogram cannot occur for a correct run and is reported through bit 1 of the
// job flag instead of being written.
__device__ __forceinline__ void emit_global(unsigned long long *glob, uint32_t len, uint32_t wt,
                                            uint32_t n, int *flag) {
    if (len <= n) g_add(glob + len, (unsigned long long)wt);
    else g_or(flag, 2);
}

// Index of the lowest set bit of a non-zero 64-bit word.
__device__ __forceinline__ uint32_t low_bit(uint64_t t) { return (uint32_t)__builtin_ctzll(t); }

// Colour changes of x inside win, a window that begins at bit lo: the set bits of
// x ^ (x shifted by one, with the open run's colour entering at lo).
__device__ __forceinline__ uint64_t changes(uint64_t x, uint64_t win, uint32_t lo, uint32_t color) {
    const uint64_t at = 1ull << (lo & 63u);
    const uint64_t prev = ((x << 1) & ~at) | (color ? at : 0ull);
    return (x ^ prev) & win;
}

// Runs between the changes t of one word (the first of them, at bit sp, begins a
// run of colour c): each lies inside the word, is never a segment's first, and
// is shorter than 64.  Returns the last change and the colour after it.
__device__ __forceinline__ void inner_runs(const Bins &bins, uint64_t t, uint32_t &sp, uint32_t &c) {
    while (t) {
        const uint32_t p = low_bit(t);
        atomicAdd((c ? bins.v : bins.w) + (p - sp), 1u);
        c ^= 1u;
        sp = p;
        t &= t - 1ull;
    }
}

// Advance the open run `st` of a column over the bits of y inside win (from bit 0;
// bit p is row base + p of the strip), counting every run that ends there; the
// strip's first run is recorded in *first (this lane's slot) instead.  Runs of
// a strip are at most 64 * kMaxWaves = 512 long, and no longer than the job's
// longest line, so every one has an LDS bin.  (After a neighbour wait has given up,
// states are arbitrary: the mask then keeps the index inside the workgroup's LDS,
// where a launch of few white bins has the state rings behind them.  The item is
// flagged as failed, and the rings are set anew for the next.)
__device__ __forceinline__ void column_runs(const Bins &bins, uint64_t y, uint64_t win, uint32_t base,
                                            Run &st, uint16_t *first, uint32_t lane) {
    uint64_t t = changes(y, win, 0u, st.color);
    if (t == 0) return;
    uint32_t p = low_bit(t);
    const uint32_t len = (base + p - st.start) & (kCapV - 1);
    if (st.first) glb(first)[lane] = (uint16_t)(len | (st.color << 15));
    else atomicAdd((st.color ? bins.v : bins.w) + len, 1u);
    uint32_t c = st.color ^ 1u;
    t &= t - 1ull;
    inner_runs(bins, t, p, c);
    st = Run{c, base + p, 0u};
}

// A run of a row of U has ended.  Such runs may be long.  A piece's first run is
// recorded in slot[off] instead of counted.
__device__ __forceinline__ void finish_row(const JobDesc &j, const Bins &bins, uint32_t color,
                                           uint32_t len, uint32_t first, uint32_t *slot, uint32_t off) {
    if (first) {
        glb(slot)[off] = len | (color << 31);
    } else if (len < (color ? (uint32_t)kCapV : (uint32_t)bins.capw)) {
        atomicAdd((color ? bins.v : bins.w) + len, 1u);
    } else {
        emit_global(color ? j.hv : j.hw, len, 1u, (uint32_t)j.hmax, j.flag);
    }
}

// As column_runs, for a part of a diagonal: bits of d inside win, from bit lo.
// White runs are not counted (and never a first run), so one trip takes a whole
// black run.  DW: how many lines a diagonal run stands for (2 in the upper triangle
// of a symmetric matrix, whose mirror diagonal repeats it; 1 in a full matrix).
template <int DW>
__device__ __forceinline__ void diagonal_runs(const Bins &bins, uint64_t d, uint64_t win, uint32_t lo,
                                              uint32_t base, Run &st, uint16_t *first, uint32_t lane,
                                              bool slot_ok) {
    const uint64_t t = changes(d, win, lo, st.color);
    if (t == 0) return;
    uint64_t starts = t & d, ends = t & ~d;
    uint32_t s = st.start;                 // where the open or the next black run began
    if (!st.color) {
        s = base + low_bit(starts);        // (t's first change begins a black run)
        starts &= starts - 1ull;
    }
    uint32_t f = st.first;
    bool open = true;
    while (ends) {
        const uint32_t len = (base + low_bit(ends) - s) & (kCapD - 1);
        if (f) { if (slot_ok) glb(first)[lane] = (uint16_t)len; }
        else atomicAdd(bins.d + len, (uint32_t)DW);
        f = 0u;
        ends &= ends - 1ull;
        open = starts != 0ull;
        s = base + low_bit(starts | (1ull << 63));
        starts &= starts - 1ull;
    }
    st = Run{open ? 1u : 0u, open ? s : 0u, open ? f : 0u};
}

// A black run of a diagonal that ends at a border.
template <int DW>
__device__ __forceinline__ void end_diagonal(const Bins &bins, uint32_t len, uint32_t f, uint16_t *first,
                                             uint32_t lane, bool slot_ok) {
    len &= kCapD - 1;
    if (f) { if (slot_ok) glb(first)[lane] = (uint16_t)len; }
    else atomicAdd(bins.d + len, (uint32_t)DW);
}

// Series pointer in the constant address space: loads through it with a
// wave-uniform address become scalar (s_load) loads, so the column coordinates
// arrive in SGPRs and feed the VALU as scalar operands.
typedef const __attribute__((address_space(4))) float *ConstF;

__device__ __forceinline__ ConstF to_const(const float *p) { return (ConstF)(p); }

// ---------------------------------------------------------------------------
// Recurrence predicate for one column against the 64 rows of a wave, with the
// first coordinate's difference d0 = col[0] - xr[0] given.
// Returns a word whose bit 31 is set when the pair is NOT recurrent: the sign of
// fl(thr - a) is set exactly when a > thr (IEEE subtraction of two finite floats
// is zero only for equal operands).  a is accumulated in FP32, coordinates in
// ascending order, no FMA.
// ---------------------------------------------------------------------------
template <int NORM, int M>
__device__ __forceinline__ uint32_t nonrec_sign_d0(float d0, ConstF col, int tau, const float *xr,
                                                   float thr) {
    float a;
    if (NORM == RQA_NORM_L1) {
        a = fabsf(d0);
#pragma unroll
        for (int k = 1; k < M; ++k) a = a + fabsf(col[k * tau] - xr[k]);
    } else if (NORM == RQA_NORM_L2) {
        a = d0 * d0;
#pragma unroll
        for (int k = 1; k < M; ++k) {
            const float e = col[k * tau] - xr[k];
            a = a + e * e;
        }
    } else {
        a = fabsf(d0);
#pragma unroll
        for (int k = 1; k < M; ++k) a = fmaxf(a, fabsf(col[k * tau] - xr[k]));
    }
    return __float_as_uint(thr - a);
}

// The same, for column b of a chunk whose coordinate k starts at ck[k].
template <int NORM, int M>
__device__ __forceinline__ uint32_t nonrec_sign_rows(const ConstF *ck, int b, const float *xr,
                                                     float thr) {
    float a;
    if (NORM == RQA_NORM_L1) {
        a = fabsf(ck[0][b] - xr[0]);
#pragma unroll
        for (int k = 1; k < M; ++k) a = a + fabsf(ck[k][b] - xr[k]);
    } else if (NORM == RQA_NORM_L2) {
        const float d = ck[0][b] - xr[0];
        a = d * d;
#pragma unroll
        for (int k = 1; k < M; ++k) {
            const float e = ck[k][b] - xr[k];
            a = a + e * e;
        }
    } else {
        a = fabsf(ck[0][b] - xr[0]);
#pragma unroll
        for (int k = 1; k < M; ++k) a = fmaxf(a, fabsf(ck[k][b] - xr[k]));
    }
    return __float_as_uint(thr - a);
}

// Generic embedding dimension: row coordinates read from memory.
template <int NORM>
__device__ __forceinline__ uint32_t nonrec_sign_dyn(ConstF col, const float *__restrict__ rowp,
                                                    int m, int tau, float thr) {
    const auto row = glb(rowp);
    float a;
    if (NORM == RQA_NORM_L1) {
        a = fabsf(col[0] - row[0]);
        for (int k = 1; k < m; ++k) a = a + fabsf(col[(int64_t)k * tau] - row[(int64_t)k * tau]);
    } else if (NORM == RQA_NORM_L2) {
        const float d = col[0] - row[0];
        a = d * d;
        for (int k = 1; k < m; ++k) {
            const float e = col[(int64_t)k * tau] - row[(int64_t)k * tau];
            a = a + e * e;
        }
    } else {
        a = fabsf(col[0] - row[0]);
        for (int k = 1; k < m; ++k) a = fmaxf(a, fabsf(col[(int64_t)k * tau] - row[(int64_t)k * tau]));
    }
    return __float_as_uint(thr - a);
}

// Recurrence of eight columns for this lane's row: bit b of the result is set when
// column b of the chunk at `cb` is NOT recurrent (on top of acc << 8).
// m >= 5 takes the first coordinate's differences first: when no lane of the
// wave has |d_0| <= thr0, all 8 x 64 pairs are non-recurrent and the other
// coordinates are not evaluated.  (Their 40-48 column coordinates do not fit
// the SGPRs left otherwise, and without the loads pinned ahead of the test the
// compiler rebuilt their addresses with long chains of 64-bit scalar adds:
// measured 29% slower on the L1, m = 5 windows.)
template <int NORM, int M>
__device__ __forceinline__ uint32_t chunk_nonrec(uint32_t acc, ConstF cb, int tau, const float *xr,
                                                 const float *__restrict__ rowp, int m, float thr,
                                                 float thr0) {
    if (M >= 5) {
        // All of the chunk's coordinates are loaded up front (the empty asm
        // keeps the compiler from sinking the loads of the other coordinates
        // into the branch, which would add a second wait).
        float d0[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            d0[b] = cb[b] - xr[0];
#pragma unroll
            for (int k = 1; k < (M > 0 ? M : 1); ++k) {
                const float ck = cb[b + k * tau];
                asm volatile("" ::"s"(ck));
            }
        }
        const float near =
            fminf(fminf(fminf(fabsf(d0[0]), fabsf(d0[1])), fminf(fabsf(d0[2]), fabsf(d0[3]))),
                  fminf(fminf(fabsf(d0[4]), fabsf(d0[5])), fminf(fabsf(d0[6]), fabsf(d0[7]))));
        if (__builtin_amdgcn_ballot_w64(near <= thr0) == 0ull) return (acc << 8) | 0xFFu;
#pragma unroll
        for (int b = 7; b >= 0; --b)
            acc = __builtin_amdgcn_alignbit(acc, nonrec_sign_d0<NORM, M>(d0[b], cb + b, tau, xr, thr), 31);
    } else if (M > 0) {
        // One uniform pointer per coordinate: each coordinate's 8 columns are
        // then one s_load_dwordx8 at a fixed offset (indexing cb[b + k*tau]
        // instead made the compiler build 8*m addresses with 64-bit adds).
        ConstF ck[M > 0 ? M : 1];
#pragma unroll
        for (int k = 0; k < (M > 0 ? M : 1); ++k) ck[k] = cb + k * tau;
#pragma unroll
        for (int b = 7; b >= 0; --b)
            acc = __builtin_amdgcn_alignbit(acc, nonrec_sign_rows<NORM, M>(ck, b, xr, thr), 31);
    } else {
        for (int b = 7; b >= 0; --b)
            acc = __builtin_amdgcn_alignbit(acc, nonrec_sign_dyn<NORM>(cb + b, rowp, m, tau, thr), 31);
    }
    return acc;
}

// The thresholds are uniform, but as scalar operands they would make the
// subtraction and the compare read an SGPR too; VALU instructions with only
// VGPR operands issue faster on gfx950 (measured: the six-instruction
// L-infinity column sustains ~1.5 instead of ~1.2 wave-instructions per clock
// per CU).  The empty asm pins the copies in VGPRs.
__device__ __forceinline__ float in_vgpr(float v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Recurrence bits of one 64x64 tile for this lane's row: bit b <-> column
// jbase + b.  `cols` points at the coordinate of column jbase (uniform).  The 64
// columns are taken in eight chunks of 8 (highest first), each fully unrolled,
// so that at most 8*m column coordinates are live in SGPRs (chunks of 16 left
// too few SGPRs for the rest of the kernel, which then spilled into VGPR lanes;
// measured 10% slower).
template <int NORM, int M>
__device__ __forceinline__ void tile_bits(ConstF cols, int tau, const float *xr,
                                          const float *__restrict__ rowp, int m, float thr_s,
                                          float thr0_s, uint32_t &lo, uint32_t &hi) {
    const float thr = in_vgpr(thr_s), thr0 = in_vgpr(thr0_s);
#pragma unroll 1
    for (int half = 1; half >= 0; --half) {
        uint32_t acc = 0;
#pragma unroll 1
        for (int sub = 3; sub >= 0; --sub)
            acc = chunk_nonrec<NORM, M>(acc, cols + half * 32 + sub * 8, tau, xr, rowp, m, thr, thr0);
        if (half) hi = ~acc; else lo = ~acc;
    }
}

// Bytes 0..3 = 0xFF where bit 0..3 of `four` is set.
__device__ __forceinline__ uint32_t spread4(uint32_t four) {
    return ((four * 0x00204081u) & 0x01010101u) * 0xFFu;
}

// The same for the chunks in `eval` only (bit q: columns 8q .. 8q+7); all pairs of
// the chunks in `ones` are recurrent, and those of the other chunks are not.
template <int NORM, int M>
__device__ __forceinline__ void tile_bits_some(ConstF cols, int tau, const float *xr,
                                               const float *__restrict__ rowp, int m, float thr_s,
                                               float thr0_s, uint32_t eval, uint32_t ones,
                                               uint32_t &lo, uint32_t &hi) {
    const float thr = in_vgpr(thr_s), thr0 = in_vgpr(thr0_s);
    uint32_t nlo = ~spread4(ones & 15u), nhi = ~spread4(ones >> 4);   // not recurrent
#pragma unroll 1
    while (eval) {
        const int q = __builtin_ctz(eval);
        eval &= eval - 1u;
        // eight bits on top of ones, turned to the chunk's place
        const uint32_t non = chunk_nonrec<NORM, M>(0xFFFFFFu, cols + q * 8, tau, xr, rowp, m, thr, thr0);
        const uint32_t turned = __builtin_amdgcn_alignbit(non, non, (uint32_t)(32 - 8 * q) & 31u);
        if (q < 4) nlo &= turned; else nhi &= turned;
    }
    lo = ~nlo;
    hi = ~nhi;
}

// Exact classes of the kGroup column tiles of group cg against the 64 rows of
// block rb, from the boxes: bit 8*i + q of `act` is clear when no pair of the
// block's rows and columns 8q .. 8q+7 of the group's tile i can be recurrent,
// bit 8*i + q of `full` is set when every such pair is (the predicate need not be
// evaluated for either).  One lane per 8-column box; the block's rows are eight
// boxes of 8 rows, read as scalars.
// Why it is exact: with y in [yn, yx] and x in [xn, xx], FP32 subtraction being
// monotone in each operand, |fl(y - x)| is at least max(fl(yn - xx),
// fl(xn - yx), 0) and at most max(|fl(yn - xx)|, |fl(yx - xn)|); sums, products
// and maxima of such bounds, rounded in the predicate's own order, bound the
// accumulated distance on the same side.  A lower bound over the first
// min(m, kBoxK) coordinates bounds the whole distance (later terms are not
// negative); the upper bound takes every coordinate, so m <= kBoxK only.
// Cost: about 90 VALU instructions per 8 tiles.  On the 1M-point Lorenz series
// 2.0 of 8 chunks per tile are left to evaluate (4.6 with one box per 64
// columns), on the 1M-point sine 0.6.
struct Boxes {
    const float *r, *c;   // planes of the rows' and the columns' boxes
    int64_t nr, nc;       // entries per plane
    float thr;
};
template <int NORM, int M>
__device__ __forceinline__ void classify(const Boxes &bx, int rb, int cg, int lane, uint64_t &act,
                                         uint64_t &full) {
    constexpr int K = M < kBoxK ? M : kBoxK;
    float yn[K], yx[K];
    const auto pc = glb(bx.c) + (int64_t)cg * (kGroup * 8) + lane;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        yn[k] = pc[(2 * k) * bx.nc];
        yx[k] = pc[(2 * k + 1) * bx.nc];
    }
    const ConstF pr = to_const(bx.r) + (int64_t)rb * 8;
    const int64_t ncr = bx.nr;
    float best = INFINITY, worst = 0.0f;
#pragma unroll 1
    for (int r0 = 0; r0 < 8; r0 += 4) {
        float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float xn = pr[(2 * k) * ncr + r0 + r], xx = pr[(2 * k + 1) * ncr + r0 + r];
                const float g = fmaxf(fmaxf(yn[k] - xx, xn - yx[k]), NORM == RQA_NORM_LINF ? a[r] : 0.0f);
                if (NORM == RQA_NORM_LINF) a[r] = g;
                else if (NORM == RQA_NORM_L1) a[r] = a[r] + g;
                else a[r] = a[r] + g * g;
            }
        }
        best = fminf(fminf(best, fminf(a[0], a[1])), fminf(a[2], a[3]));
        if (M <= kBoxK) worst = fmaxf(fmaxf(worst, fmaxf(a[0], a[1])), fmaxf(a[2], a[3]));
    }
    const float thr = bx.thr;
    act = __builtin_amdgcn_ballot_w64(best <= thr);
    full = 0ull;
    if (M <= kBoxK && __builtin_amdgcn_ballot_w64(worst <= thr) != 0ull) {
        float a = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float xn = INFINITY, xx = -INFINITY;   // the whole block's range
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                xn = fminf(xn, pr[(2 * k) * ncr + r]);
                xx = fmaxf(xx, pr[(2 * k + 1) * ncr + r]);
            }
            const float g = fmaxf(fabsf(yn[k] - xx), fabsf(yx[k] - xn));
            if (NORM == RQA_NORM_LINF) a = fmaxf(a, g);
            else if (NORM == RQA_NORM_L1) a = a + g;
            else a = a + g * g;
        }
        full = __builtin_amdgcn_ballot_w64(worst <= thr && a <= thr);
    }
}

// ---------------------------------------------------------------------------
// Kernel 1: per-job preparation -- zero the histograms, the statistics and the
// flag, reset the work counters, look for non-finite input, build the
// zero-padded tail of the last column tile and the boxes, and sample what these
// decide.  grid = (prepare_blocks_of the longest job, jobs).
// Non-finite input is noted per block (a plain store: the flag itself is being
// cleared by block 0 of this kernel) and enters the flag in the statistics.
// ---------------------------------------------------------------------------
// Boxes of `count` delay vectors: one thread per (box, coordinate).  Boxes
// without a vector (the planes are padded to whole groups) get an empty range,
// which every test takes as "no pair recurs".
__device__ __forceinline__ void make_boxes(float *box, int entries, const float *s, int count, int m,
                                           int tau, int64_t tid, int64_t stride) {
    const int K = m < kBoxK ? m : kBoxK;
    for (int64_t t = tid; t < (int64_t)entries * K; t += stride) {
        const int k = (int)(t / entries);
        const int64_t q = t - (int64_t)k * entries;
        float lo = INFINITY, hi = -INFINITY;
        const int64_t first = q * kBoxVecs, last = (int64_t)count - 1;
        if (first <= last) {
            // (past the end: the last vector again, so that no load waits for another)
            const auto x = glb(s) + (int64_t)k * tau;
            float v[kBoxVecs];
#pragma unroll
            for (int u = 0; u < kBoxVecs; ++u) v[u] = x[first + u < last ? first + u : last];
#pragma unroll
            for (int u = 0; u < kBoxVecs; ++u) {
                lo = fminf(lo, v[u]);
                hi = fmaxf(hi, v[u]);
            }
        }
        glb(box)[(int64_t)(2 * k) * entries + q] = lo;
        glb(box)[(int64_t)(2 * k + 1) * entries + q] = hi;
    }
}

// Whether boxes decide a sampled piece (64 rows by 8 columns), as classify would
// say: eight lanes, one per box of 8 rows, from the series itself (the boxes are
// being made).  A fixed sequence of places, even over the triangle or the matrix.
// All lanes of the group return the answer.
__device__ __forceinline__ bool sample_piece(const JobDesc &j, uint32_t piece) {
    const int rblocks = j.n / 64, cblocks = j.nb / kBoxVecs;   // (whole ones: jobs with boxes have some)
    if (rblocks == 0 || cblocks == 0) return false;
    // Halves of a 64-bit mix of the piece's number (splitmix64's finaliser).
    uint64_t h = (piece + 1ull) * 0x9E3779B97F4A7C15ull;
    h = (h ^ (h >> 30)) * 0xBF58476D1CE4E5B9ull;
    h = (h ^ (h >> 27)) * 0x94D049BB133111EBull;
    h ^= h >> 31;
    int rb = (int)(((h >> 32) * (uint64_t)rblocks) >> 32);
    int cq = (int)(((h & 0xFFFFFFFFull) * (uint64_t)cblocks) >> 32);
    if (j.mode == kModeAuto && cq < 8 * rb) {   // mirrored into the upper triangle
        const int r = cq / 8;
        cq = 8 * rb + (cq & 7);
        rb = r;
    }
    const int K = j.m < kBoxK ? j.m : kBoxK;
    const int64_t row = (int64_t)rb * 64 + (threadIdx.x & 7) * kBoxVecs, col = (int64_t)cq * kBoxVecs;
    float least = 0.0f, most = 0.0f;
    for (int k = 0; k < K; ++k) {
        const auto x = glb(j.s) + row + (int64_t)k * j.tau, y = glb(j.sb) + col + (int64_t)k * j.tau;
        float xn = INFINITY, xx = -INFINITY, yn = INFINITY, yx = -INFINITY;
#pragma unroll
        for (int u = 0; u < kBoxVecs; ++u) {
            xn = fminf(xn, x[u]);
            xx = fmaxf(xx, x[u]);
            yn = fminf(yn, y[u]);
            yx = fmaxf(yx, y[u]);
        }
        const float a = fmaxf(fmaxf(yn - xx, xn - yx), 0.0f), b = fmaxf(fabsf(yn - xx), fabsf(yx - xn));
        if (j.norm == RQA_NORM_LINF) {
            least = fmaxf(least, a);
            most = fmaxf(most, b);
        } else {
            least += j.norm == RQA_NORM_L1 ? a : a * a;
            most += j.norm == RQA_NORM_L1 ? b : b * b;
        }
    }
    const uint64_t group = 0xFFull << (threadIdx.x & 56);
    const uint64_t open = __builtin_amdgcn_ballot_w64(least <= j.thr) & group;
    const uint64_t full = __builtin_amdgcn_ballot_w64(j.m <= kBoxK && most <= j.thr) & group;
    return open == 0ull || full == group;
}

__device__ __forceinline__ void prepare_job(const JobDesc &j, int *counters) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t hl = (int64_t)j.hmax + 1;
    if (blockIdx.y == 0 && tid < kCounters) counters[tid] = 0;
    if (tid == 0) {
        *j.flag = 0;
        *j.stat_done = 0u;
    }
    for (int64_t t = tid; t < hl; t += stride) {
        j.hd[t] = 0ull;
        j.hv[t] = 0ull;
        j.hw[t] = 0ull;
    }
    if (tid < (int64_t)(sizeof(JobStats) / 8))
        reinterpret_cast<unsigned long long *>(j.stats)[tid] = 0ull;
    for (int64_t t = tid; t < j.mask_total; t += stride) j.vmask[t] = 0u;
    bool bad = false;
    if (j.mode != kModeMatrix) {   // a given matrix has no series
        for (int64_t t = tid; t < j.n_points; t += stride) bad |= !__builtin_isfinite(j.s[t]);
        if (j.mode == kModeCross)
            for (int64_t t = tid; t < j.n_points_b; t += stride) bad |= !__builtin_isfinite(j.sb[t]);
        // Column coordinates of the last tile, from the columns' series.
        const int64_t base = (int64_t)j.c_last * 64;
        float *tail = const_cast<float *>(j.tail);
        for (int64_t t = tid; t < j.tail_len; t += stride)
            tail[t] = base + t < j.n_points_b ? j.sb[base + t] : 0.0f;
    }
    if (j.boxc != nullptr) {
        make_boxes(j.boxc, j.ncc, j.sb, j.nb, j.m, j.tau, tid, stride);
        if (j.boxr != j.boxc) make_boxes(j.boxr, j.ncr, j.s, j.n, j.m, j.tau, tid, stride);
        int count = 0;
        if ((int)blockIdx.x < j.sample_blocks) {
            const bool yes = sample_piece(j, blockIdx.x * kSamples + threadIdx.x / 8);
            count = __syncthreads_count(yes && (threadIdx.x & 7) == 0 ? 1 : 0);
        }
        if (threadIdx.x == 0) j.decided[blockIdx.x] = (uint8_t)count;
    }
    const int any = __syncthreads_or(bad ? 1 : 0);
    if (threadIdx.x == 0) j.nonfinite[blockIdx.x] = any ? 1 : 0;
    if (blockIdx.x == 0 && threadIdx.x >= gridDim.x && threadIdx.x < kPrepareBlocks) {   // no such blocks
        j.nonfinite[threadIdx.x] = 0;
        if (j.boxc != nullptr) j.decided[threadIdx.x] = 0;
    }
}

__global__ void k_prepare(const JobDesc *__restrict__ jobs, int *counters) {
    prepare_job(jobs[blockIdx.y], counters);
}

// The same for a launch of one job, whose descriptors come as kernel arguments
// and are written to device memory here: nothing to stage on the host, and no
// copy in front of the first kernel.
__global__ void k_prepare_one(const JobDesc d, const GroupDesc g, JobDesc *ddesc, GroupDesc *dgroups,
                              int *counters) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *ddesc = d;
        *dgroups = g;
    }
    prepare_job(d, counters);
}

// Move a one-job launch to row band b: its strips [b K, min((b+1) K, S)), the
// origin of their summary slots, the band's work items, and a fresh work
// counter (K strips per band, S strips in all); and clear the masks.
__global__ void k_band(JobDesc *jobs, GroupDesc *groups, int *counters, int b) {
    JobDesc &j = jobs[0];
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < j.mask_total;
         t += (int64_t)gridDim.x * blockDim.x)
        j.vmask[t] = 0u;
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const int lo = b * j.band_strips;
    const int hi = lo + j.band_strips < j.nstrips ? lo + j.band_strips : j.nstrips;
    j.s_lo = lo;
    j.s_hi = hi;
    j.soff_lo = strip_offset(lo, j.n, j.wp, j.H);
    groups[0].items = (hi - lo) * j.segs;
    counters[0] = 0;
}

// ---------------------------------------------------------------------------
// Kernel 2: the fused tile pass.  Persistent workgroups pull (job, strip) work
// items of one (norm, m) group from a counter.
// ---------------------------------------------------------------------------
// LDS of a tile workgroup (dynamic shared memory): privatised histogram bins; the
// state rings, written in place by one wave after the other:
//  * vst: open runs of the columns of tile c, in slot c mod kRing,
//  * dst: open runs of the 64 diagonals of block k (diagonals 64k .. 64k+63), in
//    slot k mod kDiagRing.  Wave w meets block k as the upper part of tile k + rb
//    (rb its row block) and as the lower part of the tile after; then the block
//    is wave w+1's;
// of wave w, in entry w + 1 of each: the number of tiles it is done with, a note
// per slot on what the states it leaves there hold (kHas*; entry 0 is what wave 0
// finds: fresh columns); which summaries of the 32 tiles at hand were written; the
// current work item.  44 KB.  The kernel is compiled for six waves per SIMD (at
// most 80 VGPRs), i.e. three 8-wave workgroups per CU.
struct StripLds {
    uint32_t *bd, *bv, *bw;
    int capw;           // entries of bw
    uint16_t *vst;      // [kRing][64]
    uint16_t *dst;      // [kDiagRing][64]
    int *prog;          // [kMaxWaves + 1]
    uint8_t *note;      // [kMaxWaves + 1][kRing]
    uint32_t *words;    // columns, top-edge diagonals, bottom-edge diagonals
    int *item;
    int *bad;           // a wait gave up in this item: its bins are not counted
    __device__ uint16_t &vs(int c, int lane) { return vst[(c & (kRing - 1)) * 64 + lane]; }
    __device__ uint16_t &ds(int k, int lane) { return dst[(k & (kDiagRing - 1)) * 64 + lane]; }
};

constexpr int kLeastWhiteBins = 64;   // (white_bins)
static_assert(sizeof(uint32_t) * (kCapV - kLeastWhiteBins) <= sizeof(uint16_t) * 64 * (kRing + kDiagRing),
              "a masked length past the white bins stays in the state rings");

// Notes on a tile's states as a wave leaves them to the wave below: some column
// or (outgoing) diagonal run is open and black / white; some column state is not
// kFreshColumn any more.
constexpr uint32_t kHasBlack = 1u, kHasWhite = 2u, kStored = 4u;

constexpr size_t strip_lds_bytes(int capw) {
    return sizeof(uint32_t) * ((size_t)kCapD + kCapV + capw) + sizeof(uint16_t) * 64 * (kRing + kDiagRing) +
    sizeof(int) * (kMaxWaves + 1) + (size_t)(kMaxWaves + 1) * kRing + 3 * sizeof(uint32_t) + 16;
}

// Wait (wave-uniform) until the counter reaches `target`; returns its value.  Each
// wait is bounded: past j.spin_limit polls it gives up (ok = false), so a wave
// never hangs.
__device__ __forceinline__ int wait_counter(int *ctr, int target, const JobDesc &j, bool &ok) {
    int v = __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
    if (v >= target) return v;
    // The bound is read only when the first poll fails (most waits need none).
    const uint32_t limit = (uint32_t)j.spin_limit;
    for (uint32_t spin = 0; spin < limit; ++spin) {
        __builtin_amdgcn_s_sleep(1);
        v = __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
        if (v >= target) return v;
    }
    ok = false;
    return v;
}

__device__ __forceinline__ void publish_counter(int *ctr, int value) {
    __hip_atomic_store(ctr, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ void flush_bins(const StripLds &L, const JobDesc &j) {
    // No line is longer than hmax.  (Where a wait gave up, the job is flagged as
    // failed, and bins may hold any length: all are cleared.)
    const int bins = j.hmax + 1 < L.capw && !*L.bad ? j.hmax + 1 : L.capw;
    for (int t = threadIdx.x; t < bins || (*L.bad && t < kCapV); t += blockDim.x) {
        if (t < kCapD) {
            const uint32_t v = L.bd[t];
            if (v) { if (t <= j.hmax) g_add(j.hd + t, (unsigned long long)v); L.bd[t] = 0; }
        }
        if (t < kCapV) {
            const uint32_t v = L.bv[t];
            if (v) { if (t <= j.hmax) g_add(j.hv + t, (unsigned long long)v); L.bv[t] = 0; }
        }
        const uint32_t v = t < L.capw ? L.bw[t] : 0u;
        if (v) { if (t <= j.hmax) g_add(j.hw + t, (unsigned long long)v); L.bw[t] = 0; }
    }
}

__device__ __forceinline__ Boxes boxes_of(const JobDesc &j) {
    return Boxes{j.boxr, j.boxc, j.ncr, j.ncc, j.thr};
}

// One (strip, column segment) block of one job.  MODE kModeAuto: the upper
// triangle U of the symmetric recurrence matrix of one series (horizontal runs
// are the row segments of the full columns, joined through the band by the
// stitch).  MODE kModeCross / kModeMatrix: a full n x nb matrix that is not
// symmetric (every diagonal and every column walked once; no horizontal runs).
//
// What bounds it, and how it is cut.  A tile costs its predicate (6-11 VALU
// instructions per column), its run extraction, and bookkeeping.  Smooth
// series leave most tiles without a colour change.  So
//  * the wave classifies kGroup tiles at a time from the boxes, and evaluates
//    only the 8-column chunks that the boxes leave open;
//  * open runs are kept by their start, in place; a tile of one colour in
//    which every open run has that colour is passed over, up to a group of
//    tiles at a time, with no state read or written.
// BOX: classify the tiles (below); without, every tile is evaluated, and the
// code for classes takes no registers from it.
template <int NORM, int M, int MODE, bool BOX>
__device__ void process_strip(const JobDesc &j, int item, StripLds &L) {
    static_assert(kMaxWaves <= 8, "LDS budget assumes at most 8 waves per workgroup");
    constexpr bool FULL = MODE != kModeAuto;
    constexpr int kDW = FULL ? 1 : 2;   // lines per diagonal run found
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
    const int nw = blockDim.x >> 6;
    const bool bottom = wave == nw - 1;                    // records the strip's bottom edge
    const int n = j.n, wp = j.wp, H = j.H, tau = j.tau;   // n: rows
    const float *const sb = j.sb;
    const int nb = FULL ? j.nb : n;                        // columns
    const int64_t band = j.theiler;                        // full matrix: cells |i-j| < band are 0
    const int G = j.segs;
    const bool BLK = FULL || G > 1;              // per-block diagonal summaries
    const int lstrip = item / G;                 // strip within the row band
    const int strip = j.s_lo + lstrip;
    const int seg = item - lstrip * G;
    const int R0 = strip * H;
    const int Rl = 64 * wave;                    // first row of this wave within the strip
    const int R = R0 + Rl;
    const int rb = R >> 6;
    const int i = R + lane;                      // this lane's row
    // Column tiles [ca, cb) of this block: the segment's cut to the strip's.
    // A block that does not start at the strip's first tile begins with the
    // row and diagonal runs that enter through its left edge, of unknown
    // history.
    const int c0 = FULL ? 0 : (R0 + wp) >> 6;
    const int sa = j.seg_base + seg * j.seg_tiles;
    const int ca = sa > c0 ? sa : c0;
    const int cb = sa + j.seg_tiles < j.c_last + 1 ? sa + j.seg_tiles : j.c_last + 1;
    if (ca >= cb) return;                        // the triangle leaves this block empty
    const bool seg_start = ca > c0;
    // The first tile in which this wave has cells (cb: none).
    const bool wave_has_u = FULL ? R <= n - 1 : R + wp <= n - 1;
    int cw = FULL ? ca : (R + wp) >> 6;
    cw = !wave_has_u || cw > cb ? cb : (cw < ca ? ca : cw);
    const int64_t soff = FULL ? 0 : strip_offset(strip, n, wp, H) - j.soff_lo;
    // Summary slots: columns -- per (strip, column), in triangular strip order
    // from the row band's first strip in auto mode; diagonals -- auto with one
    // segment: per (strip, diagonal of U) in the same order; otherwise per
    // work item j.dw slots for the diagonals k = x0-(R0+H-1) .. x1-1-R0 that
    // have a cell in the block's columns [x0, x1).
    const int x0 = ca * 64;
    const int x1 = cb * 64 < nb ? cb * 64 : nb;
    const int64_t vbase = FULL ? (int64_t)lstrip * nb : soff - R0 - wp;
    const int64_t dbase = BLK ? (int64_t)item * j.dw + (R0 + H - 1) - x0 : soff - wp;
    const int kmin = BLK ? (FULL || x0 - (R0 + H - 1) > wp ? x0 - (R0 + H - 1) : wp) : wp;
    const int kmax = BLK ? x1 - 1 - R0 : n - 1 - R0;
    // (Interior tiles have slots for all their diagonals, but for lane 0's lower
    // part in a block's first tile, which is empty.)
    auto dok = [&](int k, bool interior, int c) -> bool {
        return (interior && c > ca) || (k >= kmin && k <= kmax);
    };
    // Interior tiles need no masking, and every column and diagonal of theirs
    // goes on below this wave: tiles [ia, ib), in a full matrix without those
    // that the band touches, [ja, jb).
    int ia, ib, ja = 0x7FFFFFFF, jb = 0x7FFFFFFF;
    if constexpr (FULL) {
        ia = 0;
        ib = R + 64 <= n - 1 ? nb >> 6 : 0;
        if (band > 0) {
            const int64_t a = (int64_t)R - 63 - band, b = (int64_t)R + 63 + band;
            ja = (int)(a < 0 ? 0 : (a >> 6) + 1);
            jb = (int)((b + 63) >> 6 < 0x7FFFFFFF ? (b + 63) >> 6 : 0x7FFFFFFF);
        }
    } else {
        ia = (R + 64 + wp + 63) >> 6;
        ib = n >> 6;
    }

    // Row coordinates of this lane (clamped for rows past the end).
    const int irow = i < n ? i : n - 1;
    const float *rowp = MODE == kModeMatrix ? nullptr : j.s + irow;
    float xr[M > 0 ? M : 1] = {};
    if constexpr (MODE != kModeMatrix) {
#pragma unroll
        for (int k = 0; k < (M > 0 ? M : 1); ++k) xr[k] = M > 0 ? glb(rowp)[(int64_t)k * tau] : 0.0f;
        // Wait for these loads here, once per strip: gfx950 counts outstanding
        // global stores and atomics in the same counter as loads, so a wait
        // for them at their first use inside the tile loop would also wait
        // for every summary store and histogram atomic still in flight.
#pragma unroll
        for (int k = 0; k < (M > 0 ? M : 1); ++k) asm volatile("" : "+v"(xr[k]));
    }

    Bins bins{L.bd, L.bv, L.bw, L.capw};
    // Horizontal runs: with segments, each row's piece in this block records
    // its first and last runs (hfirst / hlast); otherwise the row's first run
    // is its lead.
    auto hslot = [&]() -> uint32_t * {
        return G > 1 ? j.hfirst + ((int64_t)(R - j.s_lo * H) * G + seg) : j.lead + R;
    };
    const uint32_t hoff = (uint32_t)lane * (uint32_t)(G > 1 ? G : 1);
    constexpr uint32_t kNotBegun = 0xFFFFFFFFu;
    Run hs{0, kNotBegun, 0};  // horizontal run of this lane's row (auto)
    // Colours (kHasBlack, kHasWhite) of the open runs of the rows, and of the
    // diagonals that leave this wave's last tile through its right edge.
    uint32_t hown = 0, lown = kHasWhite;

    // Given matrix: the next tile's row word is loaded while the current tile
    // is processed (loading 2, 4 or 8 tiles ahead measured no faster).
    const auto mrow = MODE == kModeMatrix && i < n ? glb(j.bits) + (int64_t)i * j.words : nullptr;
    uint64_t mnext = 0;
    if constexpr (MODE == kModeMatrix) {
        if (mrow && cw < cb) mnext = mrow[cw];
    }

    // Progress.  Tiles [.., ready) may be entered: the wave above is done with
    // them, or (wave 0) their state slots are free again, the last wave being
    // kRing tiles behind.  After one wait has given up the wave stops waiting
    // (the job is flagged as failed), so a strip finishes in bounded time.
    bool sync_ok = true;
    int *const from = &L.prog[wave == 0 ? nw : wave];
    const int lead = wave == 0 ? kRing : 0;
    const int wbias = j.wait_bias;   // 0 (a test injecting give-ups sets it)
    int ready = wbias ? ca : ca + lead;
    uint32_t notes = kHasWhite;      // lane s: the note found for slot s
    int c = ca;
    auto await = [&]() {
        if (c < ready) return;
        ready = ca + lead + wait_counter(from, c - ca - lead + 1 + wbias, j, sync_ok);
        notes = L.note[wave * kRing + (lane & (kRing - 1))];
        if (!sync_ok) ready = 0x7FFFFFFF;
        // A strip goes at the pace of its slowest wave (the one whose rows hold
        // most recurrences); the others wait for it.  So a wave with many tiles
        // ready is issued first: 1M-point Lorenz series 63.2 -> 52.5 ms, 1M-point
        // sine 47.4 -> 34.1, 262,144-point cross recurrence 7.7 -> 6.5.
        const int lag = __builtin_amdgcn_readfirstlane(ready - c);
        if (lag >= 12) __builtin_amdgcn_s_setprio(3);
        else if (lag >= 4) __builtin_amdgcn_s_setprio(2);
        else if (lag >= 2) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
    };
    auto advance = [&](int next) {   // done with the tiles up to `next`
        publish_counter(&L.prog[wave + 1], next - ca);
        // (readfirstlane: the compiler does not see that `next` is uniform, and
        // took the column coordinates as vector loads from here on)
        c = __builtin_amdgcn_readfirstlane(next);
    };
    // A tile whose columns are white from the strip's top edge to its bottom
    // edge, or whose diagonals are white at the edge, writes no summaries.  The
    // others are noted in LDS (columns and bottom-edge diagonals by the bottom
    // wave, top-edge diagonals by wave 0) and, 32 tiles at a time, in the masks
    // (one lane per tile; an atomic per tile in the tile's own path made the
    // bottom wave, which sets the pace, slower: 62.6 -> 69.8 ms on the 1M-point
    // Lorenz series).
    auto note_written = [&](int which) {
        if (lane == 0) atomicOr(&L.words[which], 1u << (c & 31));
    };
    auto flush_written = [&](int window) {   // tiles [32 window, 32 window + 32)
        const int e = 32 * window + lane;
        const int64_t strip_word = lstrip >> 5;
        const uint32_t bit = 1u << (lstrip & 31);
        auto put = [&](int which, uint32_t *mask, int entry) {
            if (lane < 32 && (L.words[which] >> lane & 1u))
                __hip_atomic_fetch_or(glb(mask + ((int64_t)entry * j.mask_words + strip_word)), bit,
                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) L.words[which] = 0u;
        };
        if (wave == 0) put(1, j.dfmask, e - rb + j.kb_off);
        if (bottom) {
            put(0, j.vmask, e - j.seg_base);
            put(2, j.dlmask, e - rb - 1 + j.kb_off);
        }
    };
    int window = wave == 0 || bottom ? ca >> 5 : 0x7FFFFFFF;
    while (c < cw) {   // nothing of this wave here yet: follow the wave above
        await();
        advance(ready < cw ? ready : cw);
    }
    const uint32_t stop_white = kHasBlack | (bottom ? kStored : 0u);
    const uint32_t stop_black = kHasWhite | (bottom ? ~0u : 0u);
    // Plain tiles: interior, and not the first behind a segment edge.
    const int pa = seg_start && ia <= ca ? ca + 1 : ia;
    int group = -1;                  // group of tiles that act / full / kinds describe
    uint64_t act = ~0ull, full = 0ull;
    uint32_t kinds = 0;              // bit i: tile i of the group is empty; bit 8 + i: it is full
    int unsorted = 0;                // groups to take unclassified (boxes decide little here)
    while (c < cb) {
        if ((c >> 5) > window) {
            flush_written(window);
            window = c >> 5;
        }
        const int slot = c & (kRing - 1);
        const int gi = c & (kGroup - 1);
        if constexpr (BOX) {
            if ((c / kGroup) != group) {
                group = c / kGroup;
                if (unsorted > 0) {
                    --unsorted;
                    act = ~0ull;
                    full = 0ull;
                    kinds = 0u;
                } else {
                    classify<NORM, M>(boxes_of(j), rb, group, lane, act, full);
                    const uint32_t b = (uint32_t)((act >> (8 * (lane & 7))) & 0xFFull);
                    const uint32_t f = (uint32_t)((full >> (8 * (lane & 7))) & 0xFFull);
                    kinds = ((uint32_t)__builtin_amdgcn_ballot_w64(b == 0u) & 0xFFu) |
                            (((uint32_t)__builtin_amdgcn_ballot_w64(f == 0xFFu) & 0xFFu) << 8);
                    // Where nearly every chunk stays open, the next seven
                    // groups are not classified: noise pays an eighth of the
                    // cost (1-2% of its predicate) instead of all of it.
                    if (__builtin_popcountll(act & ~full) >= 60) unsorted = 7;
                }
            }
        }
        const bool plain = c >= pa && c < ib && (!FULL || c < ja || c >= jb);
        const uint32_t kind = BOX ? (kinds >> gi) & 0x101u : 0u;   // 1: empty, 0x100: full

        // ---- tiles of one colour, known from the boxes: passed over if every
        // open run has that colour, as many of the group's as are alike, with
        // the same states waiting, and ready ----
        if (plain && kind) {
            await();
            const uint32_t stop = kind == 1u ? stop_white : stop_black;
            const uint32_t note = (uint32_t)__builtin_amdgcn_readlane((int)notes, slot);
            if (((note | hown | lown) & stop) == 0u) {
                uint32_t same = kind == 1u ? kinds : kinds >> 8;
                same &= ~((uint32_t)__builtin_amdgcn_ballot_w64((notes & stop) != 0u) >>
                          (slot & ~(kGroup - 1)));
                int next = c + __builtin_ctz(~(((same & 0xFFu) >> gi) | 1u));   // at least this one
                next = next < ib ? next : ib;
                next = next < cb ? next : cb;
                if (FULL && c < ja) next = next < ja ? next : ja;
                next = next < ready ? next : ready;
                if (((lane - slot) & (kRing - 1)) < next - c && lane < kRing)
                    L.note[(wave + 1) * kRing + lane] =
                        (uint8_t)(kind == 1u ? kHasWhite | (notes & kStored) : kHasBlack | kStored);
                lown = kind == 1u ? kHasWhite : kHasBlack;
                advance(next);
                continue;
            }
        }

        // ---- this lane's row of the tile ----
        const int jbase = c * 64;
        const bool interior = plain || (c >= ia && c < ib && (!FULL || c < ja || c >= jb));
        const bool fresh = seg_start && c == ca;   // first tile behind a segment edge
        uint32_t xlo = kind & 0x100u ? ~0u : 0u, xhi = xlo;
        if constexpr (MODE == kModeMatrix) {
            const uint64_t word = mnext;
            if (mrow && c + 1 < cb) mnext = mrow[c + 1];
            xlo = (uint32_t)word;
            xhi = (uint32_t)(word >> 32);
        } else if (kind == 0u) {
            uint32_t eval = 0xFFu, ones = 0u;
            if (BOX) {
                eval = (uint32_t)(act >> (8 * gi)) & 0xFFu;
                ones = (uint32_t)(full >> (8 * gi)) & 0xFFu;
                eval &= ~ones;
            }
            // The last tile's coordinates end past the series unless it is
            // interior.
            const ConstF cols = to_const(!interior && c == j.c_last ? j.tail : sb + jbase);
            if (!BOX || eval == 0xFFu)
                tile_bits<NORM, M>(cols, tau, xr, rowp, j.m, j.thr, j.thr0, xlo, xhi);
            else
                tile_bits_some<NORM, M>(cols, tau, xr, rowp, j.m, j.thr, j.thr0, eval, ones, xlo, xhi);
        }
        int lo_v = 0;
        uint64_t vmask = ~0ull;
        if (!interior) {
            if constexpr (FULL) {
                // Valid cells of this row: columns [0, nb) outside the band.
                vmask = 0ull;
                if (i < n) {
                    const int hv = nb - jbase < 64 ? nb - jbase : 64;
                    vmask = hv > 0 ? range_mask(0, hv) : 0ull;
                    if (band > 0) {
                        int64_t blo = (int64_t)i - band + 1 - jbase, bhi = (int64_t)i + band - jbase;
                        blo = blo < 0 ? 0 : blo;
                        bhi = bhi > 64 ? 64 : bhi;
                        if (blo < bhi) vmask &= ~range_mask((uint32_t)blo, (uint32_t)bhi);
                    }
                }
            } else {
                // Valid cells of this row: columns [i + wp, n-1], rows < n.
                lo_v = i + wp - jbase;
                lo_v = lo_v < 0 ? 0 : lo_v;
                if (i >= n || lo_v > 64) lo_v = 64;
                int hi_v = n - jbase;
                hi_v = hi_v > 64 ? 64 : hi_v;
                vmask = lo_v < hi_v ? range_mask(lo_v, hi_v) : 0ull;
            }
            xlo &= (uint32_t)vmask;
            xhi &= (uint32_t)(vmask >> 32);
        }
        const uint64_t rows = __builtin_amdgcn_ballot_w64((xlo | xhi) != 0u);
        const bool any = rows != 0ull;
        await();   // the columns' and diagonals' states from the wave above
        if (plain && !any) {   // evaluated, and found empty
            const uint32_t note = (uint32_t)__builtin_amdgcn_readlane((int)notes, slot);
            if (((note | hown | lown) & stop_white) == 0u) {
                if (lane == 0)
                    L.note[(wave + 1) * kRing + slot] = (uint8_t)(kHasWhite | (note & kStored));
                lown = kHasWhite;
                advance(c + 1);
                continue;
            }
        }
        const bool all = any && __builtin_amdgcn_ballot_w64((xlo & xhi) != ~0u) == 0ull;
        const uint64_t X = mk64(xlo, xhi);
        const bool few = __builtin_popcountll(rows) <= kFewRows;
        uint32_t ylo = xlo, yhi = xhi, zlo = xlo, zhi = xhi;
        if (few) {
            gather_rows(xlo, xhi, (uint32_t)rows, 0, ylo, zlo);
            gather_rows(xlo, xhi, (uint32_t)(rows >> 32), 32, yhi, zhi);
        }

        // The diagonals that enter a block through its left edge start a segment
        // there: lane q's lower part (q > 0) begins at cell (R + 64 - q, jbase),
        // bit 0 of lane 64 - q's row word; lane 0's lower part is empty and its
        // diagonal enters the block in the wave below, which starts it.
        const bool fresh_up = wave == 0 || (fresh && lane == 0);

        // ---- horizontal runs (row i of U) ----
        if constexpr (!FULL) {
            if (!plain && vmask != 0ull && hs.start == kNotBegun) {
                hs = Run{(uint32_t)((X >> lo_v) & 1ull), (uint32_t)(jbase + lo_v), 1u};
            }
            uint64_t t = changes(X, vmask, (uint32_t)lo_v, hs.color);
            if (t != 0ull) {
                uint32_t p = low_bit(t), col = hs.color ^ 1u;
                finish_row(j, bins, hs.color, (uint32_t)jbase + p - hs.start, hs.first, hslot(), hoff);
                t &= t - 1ull;
                inner_runs(bins, t, p, col);
                hs = Run{col, (uint32_t)jbase + p, 0u};
            }
            hown = (__builtin_amdgcn_ballot_w64(hs.color != 0u) != 0ull ? kHasBlack : 0u) |
                   (__builtin_amdgcn_ballot_w64(hs.color == 0u) != 0ull ? kHasWhite : 0u);
        }

        // ---- vertical runs (columns) ----
        uint32_t vcolor = 0;   // colours of the columns' open runs below this wave
        {
            if (!few && !all) transpose64(ylo, yhi, lane);
            const uint64_t Y = mk64(ylo, yhi);
            uint16_t *const first = j.vfirst + (vbase + jbase);
            if (plain) {
                Run st = wave == 0 ? Run{(uint32_t)(Y & 1ull), 0u, 1u} : unpack_run(L.vs(slot, lane));
                column_runs(bins, Y, ~0ull, (uint32_t)Rl, st, first, (uint32_t)lane);
                if (bottom) {
                    const uint16_t pk = (uint16_t)(((uint32_t)(Rl + 64) - st.start) | (st.color << 15));
                    uint16_t *const last = j.vlast + (vbase + jbase);
                    glb(st.first ? first : last)[lane] = pk;   // one run: its last is its first
                    st = unpack_run(kFreshColumn);
                }
                L.vs(slot, lane) = pack_run(st);
                vcolor = st.color;
            } else {
                const int jc = jbase + lane;
                // last valid local row of column jc: the band (auto) or the
                // bottom border (full) ends its segment
                const int e = FULL ? n - 1 - R : jc - wp - R;
                if (jc <= nb - 1 && e >= 0) {
                    const uint32_t vhi = e >= 63 ? 64u : (uint32_t)(e + 1);
                    Run st = wave == 0 ? Run{(uint32_t)(Y & 1ull), 0u, 1u} : unpack_run(L.vs(slot, lane));
                    column_runs(bins, Y, vhi >= 64 ? ~0ull : ((1ull << vhi) - 1ull), (uint32_t)Rl, st,
                                first, (uint32_t)lane);
                    if (e <= 63 || bottom) {
                        const uint16_t pk = (uint16_t)((Rl + vhi - st.start) | (st.color << 15));
                        uint16_t *const last = j.vlast + (vbase + jbase);
                        glb(st.first ? first : last)[lane] = pk;
                        st = unpack_run(kFreshColumn);
                    }
                    L.vs(slot, lane) = pack_run(st);
                }
            }
            if (bottom) note_written(0);
        }

        // ---- diagonal runs ----
        {
            if (!few && !all) {
                rotr64(zlo, zhi, (uint32_t)lane);
                transpose64(zlo, zhi, lane);
            }
            const uint64_t D = mk64(zlo, zhi);
            const int q = lane;
            const int kb = c - rb;                  // diagonal block of the upper part
            const int kup = 64 * kb + q;            // diagonal of the upper part
            const int klo = kup - 64;               // diagonal of the lower part
            const uint64_t upwin = ~0ull >> q;
            uint16_t *const ufirst = j.dfirst + (dbase + 64 * kb), *const lfirst = ufirst - 64;
            const bool uok = dok(kup, interior, c), lok = dok(klo, interior, c);
            Run up;
            if (fresh_up) {
                // Segment start on the strip's top row (or the block's left
                // edge).  A white first cell means "no black run at the edge"
                // (white diagonal runs are never counted, so it is not a run
                // to record either).
                const uint32_t b = (uint32_t)(D & 1ull);
                up = Run{b, (uint32_t)Rl, b};
            } else if (jbase + q > nb - 1) {
                up = Run{0u, 0u, 0u};   // starts past the border
            } else {
                up = unpack_run(L.ds(kb, lane));
            }
            if (wave == 0) {
                // On the strip's top row the white diagonals are recorded only
                // beside black ones.
                if (__builtin_amdgcn_ballot_w64(up.color != 0u) != 0ull) {
                    note_written(1);
                    if (up.color == 0u && uok) glb(ufirst)[lane] = 0;
                }
            } else if (fresh && lane == 0 && up.color == 0u && uok) {
                glb(ufirst)[lane] = 0;
            }
            diagonal_runs<kDW>(bins, D, upwin, 0u, (uint32_t)Rl, up, ufirst, (uint32_t)lane, uok);
            L.ds(kb, lane) = pack_run(up);
            lown = (__builtin_amdgcn_ballot_w64(up.color != 0u) != 0ull ? kHasBlack : 0u) |
                   (__builtin_amdgcn_ballot_w64(up.color == 0u) != 0ull ? kHasWhite : 0u);

            Run lw;
            if (fresh) {
                const uint64_t col0 = __builtin_amdgcn_ballot_w64((X & 1ull) != 0ull);
                const uint32_t b = lane == 0 ? 0u : (uint32_t)(col0 >> ((64 - lane) & 63)) & 1u;
                lw = Run{b, (uint32_t)(Rl + 64 - q), b};
                if (lane != 0 && b == 0u && lok) glb(lfirst)[lane] = 0;
            } else {
                lw = unpack_run(L.ds(kb - 1, lane));
            }
            diagonal_runs<kDW>(bins, D, ~upwin, (uint32_t)(64 - q), (uint32_t)Rl, lw, lfirst,
                               (uint32_t)lane, lok);
            // The lower part ends on row R+63.  Diagonals with no cell on the
            // next row end here at the right (or, full matrix, bottom) border;
            // the others go to the wave below or, from the last wave, into the
            // summary.
            const uint32_t len = (uint32_t)(Rl + 64) - lw.start;
            bool ends = false;
            if (!interior) {
                ends = FULL ? (R + 64 > n - 1 || R + 64 + klo > nb - 1) : (R + 64 + klo > n - 1);
                if (ends) {
                    if (lw.color) end_diagonal<kDW>(bins, len, lw.first, lfirst, (uint32_t)lane, lok);
                    lw = Run{0u, 0u, 0u};
                }
            }
            if (bottom) {
                if (__builtin_amdgcn_ballot_w64(lw.color != 0u) != 0ull) {
                    note_written(2);
                    // A black run over the whole piece: the stitch reads only
                    // its first (a white one reads as 0 and needs its last).
                    uint16_t *const llast = j.dlast + (dbase + 64 * kb - 64);
                    if (!ends && lok) glb(lw.first ? lfirst : llast)[lane] = (uint16_t)(lw.color ? len : 0u);
                }
                lw = Run{0u, 0u, 0u};   // the slot is free again
            }
            L.ds(kb - 1, lane) = pack_run(lw);
            if (!bottom) {
                uint32_t mine = kHasBlack | kHasWhite | kStored;   // at a border: not known
                if (plain) {
                    mine = kStored;
                    if (__builtin_amdgcn_ballot_w64((vcolor | lw.color) != 0u) != 0ull) mine |= kHasBlack;
                    if (__builtin_amdgcn_ballot_w64((vcolor & lw.color) == 0u) != 0ull) mine |= kHasWhite;
                }
                if (lane == 0) L.note[(wave + 1) * kRing + slot] = (uint8_t)mine;
            }
        }
        advance(c + 1);
    }
    if (wave == 0 || bottom) flush_written(window);
    if (!sync_ok) {   // a neighbour wait gave up: result invalid
        g_or(j.flag, 8);
        *L.bad = 1;
    }

    if (cw < cb) {
        // Rows end at column n-1: their last run is complete; a block that is
        // not the strip's last records each row's open run as its last.
        if constexpr (!FULL) {
            if (hs.start != kNotBegun) {
                const uint32_t len = (uint32_t)x1 - hs.start;
                uint32_t *const first = hslot();
                if (cb == j.c_last + 1)
                    finish_row(j, bins, hs.color, len, hs.first, first, hoff);
                else
                    glb(hs.first ? first : j.hlast + (first - j.hfirst))[hoff] = len | (hs.color << 31);
            }
        }
        // Upper parts that left the last tile on its right edge end at the
        // border, and so do those whose next cell (one row down, in the next
        // block) lies below the matrix; the others go on in the next block:
        // recorded as the block's last runs.
        const int kb = cb - 1 - rb;
        const bool uok = dok(64 * kb + lane, false, ca);
        const Run left = unpack_run(L.ds(kb, lane));
        const uint32_t len = (uint32_t)(Rl + 64 - lane) - left.start;
        uint16_t *const first = j.dfirst + (dbase + 64 * kb), *const last = j.dlast + (dbase + 64 * kb);
        if (cb == j.c_last + 1 || R + 64 - lane > n - 1) {
            if (left.color) end_diagonal<kDW>(bins, len, left.first, first, (uint32_t)lane, uok);
        } else if (uok) {
            // A black run over the whole piece: the stitch reads only its first.
            glb(left.first ? first : last)[lane] = (uint16_t)(left.color ? len : 0u);
        }
    }
}

// Whether the tiles of a job are classified: where the boxes decide a quarter of its
// sampled pieces (noise: none, or nearly; AR(1) series a few; Lorenz and sine most).
// With the classes in its code the L1, m = 5 kernel ran 4.5% slower on uniform noise
// (400 windows 9.52 -> 9.96 ms); classified for a sixteenth, 362 AR(1) windows of 3,831
// points (m = 5) took 1.43 ms, without 1.39, and 100,000 AR(1) points (m = 3) 2.82, 2.77;
// a line at three eighths gave the same times.  Counted once per job: for each wave to
// try four groups of its part cost two to four memory latencies an item (200 noise
// windows of 9,000 points 3.67 ms, 3.52 this way; the 400 windows 9.58 -> 9.36).
template <int M, int MODE>
__device__ __forceinline__ bool use_boxes(const JobDesc &j) {
    if constexpr (MODE == kModeMatrix || M == 0) {
        return false;
    } else {
        if (j.boxc == nullptr) return false;
        const auto d = (const __attribute__((address_space(4))) uint32_t *)(const uint32_t *)j.decided;
        uint32_t sum = 0;   // two 16-bit halves
#pragma unroll
        for (int q = 0; q < kPrepareBlocks / 4; ++q) sum += (d[q] & 0x00FF00FFu) + ((d[q] >> 8) & 0x00FF00FFu);
        return (int)((sum & 0xFFFFu) + (sum >> 16)) >= kSamples / 4 * j.sample_blocks;
    }
}

template <int NORM, int M, int MODE>
__global__ void __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(6, 6)))
k_tiles(const JobDesc *__restrict__ jobs, const GroupDesc *__restrict__ groups, int g,
        int *counters) {
    extern __shared__ uint32_t lds_words[];
    StripLds L;
    L.bd = lds_words;
    L.bv = L.bd + kCapD;
    L.bw = L.bv + kCapV;
    const GroupDesc gd = groups[g];
    L.capw = gd.capw;
    L.vst = reinterpret_cast<uint16_t *>(L.bw + gd.capw);
    L.dst = L.vst + kRing * 64;
    L.prog = reinterpret_cast<int *>(L.dst + kDiagRing * 64);
    L.note = reinterpret_cast<uint8_t *>(L.prog + kMaxWaves + 1);
    L.words = reinterpret_cast<uint32_t *>(L.note + (kMaxWaves + 1) * kRing);
    L.item = reinterpret_cast<int *>(L.words + 3);
    L.bad = L.item + 1;
    for (int t = threadIdx.x; t < kCapD + kCapV + gd.capw; t += blockDim.x) L.bd[t] = 0;
    __syncthreads();
    while (true) {
        if (threadIdx.x == 0) {
            *L.item = atomicAdd(counters + g, 1);
            *L.bad = 0;
        }
        if (threadIdx.x <= kMaxWaves) L.prog[threadIdx.x] = 0;
        if (threadIdx.x < kRing) L.note[threadIdx.x] = (uint8_t)kHasWhite;
        if (threadIdx.x < 3) L.words[threadIdx.x] = 0u;
        static_assert(kNoDiagonal == 0u, "pairs of 16-bit states");
        uint32_t *rings = reinterpret_cast<uint32_t *>(L.vst);
        for (int t = threadIdx.x; t < 32 * (kRing + kDiagRing); t += blockDim.x)
            rings[t] = t < 32 * kRing ? kFreshColumn * 0x10001u : 0u;
        __syncthreads();
        const int item = *L.item;
        __syncthreads();
        if (item >= gd.items) break;
        // locate the job: largest job index in [job0, job1) with strip_base <= item
        int lo = gd.job0, hi = gd.job1 - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].strip_base <= item) lo = mid; else hi = mid - 1;
        }
        // By reference: fields are re-read with scalar loads where needed
        // instead of occupying SGPRs for the whole strip.
        const JobDesc &j = jobs[lo];
        const int block = item - j.strip_base;
        if constexpr (MODE != kModeMatrix && M > 0) {
            if (use_boxes<M, MODE>(j)) process_strip<NORM, M, MODE, true>(j, block, L);
            else process_strip<NORM, M, MODE, false>(j, block, L);
        } else {
            process_strip<NORM, M, MODE, false>(j, block, L);
        }
        __syncthreads();
        flush_bins(L, j);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Kernel 3: stitch and join.  One thread per line: columns j in [0, n) fold their
// per-strip segment summaries and join the trailing run of column j of U with
// the middle and the leading run of row j of U; diagonals k in [w', n) fold
// their summaries.  Runs crossing strip edges are counted here.
// ---------------------------------------------------------------------------
struct StitchLds {
    uint32_t bd[kCapD];
    uint32_t bv[kStitchCapV];
    uint32_t bw[kCapW];
};

// Global histogram add in which the active lanes of the wave that add to the
// same bin are combined into one atomic (64-bit atomics on one address
// serialise in L2; in the stitch, neighbouring lines of a smooth series end long
// runs of equal length together).
__device__ __forceinline__ void g_add_combined(unsigned long long *p, uint32_t w) {
    const uint64_t a = (uint64_t)(uintptr_t)p;
    // At most 64 rounds: each retires at least the first active lane (its own
    // address matches); the bound keeps a wave from spinning whatever happens.
    for (int round = 0; round < 64; ++round) {
        // readfirstlane returns int: go through uint32_t so that the low half
        // is not sign-extended into the high one.
        const uint32_t lo0 = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a);
        const uint32_t hi0 = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
        const uint64_t a0 = ((uint64_t)hi0 << 32) | (uint64_t)lo0;
        // The ballot is taken by every active lane, before the branch.
        const uint64_t same = __builtin_amdgcn_ballot_w64(a == a0);
        if (a == a0) {
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                       __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            if (below == 0u)
                g_add(p, (unsigned long long)w * (unsigned long long)__builtin_popcountll(same));
            break;
        }
    }
}

// Stitch emission: LDS bin below the cap, else the combined global add.
__device__ __forceinline__ void emit_stitch(uint32_t *bins, int cap, unsigned long long *glob,
                                            uint32_t len, uint32_t wt, uint32_t n, int *flag) {
    if (len < (uint32_t)cap && len <= n)
        atomicAdd(bins + len, wt);
    else if (len <= n)
        g_add_combined(glob + len, wt);
    else
        g_or(flag, 2);
}

__device__ __forceinline__ void emit_line(StitchLds &L, const JobDesc &j, uint32_t color,
                                          uint32_t len) {
    if (len == 0) return;
    if (color) emit_stitch(L.bv, kStitchCapV, j.hv, len, 1u, (uint32_t)j.hmax, j.flag);
    else emit_stitch(L.bw, kCapW, j.hw, len, 1u, (uint32_t)j.hmax, j.flag);
}

// Segment of column x (a column of segment g lies in the column tiles
// [seg_base + g*seg_tiles, seg_base + (g+1)*seg_tiles)).
__device__ __forceinline__ int seg_of(const JobDesc &j, int x) {
    return ((x >> 6) - j.seg_base) / j.seg_tiles;
}

// Row r of U, cut into pieces by the column segments (auto mode, segs > 1):
// fold the pieces' first and last runs in order, count the runs that span
// piece edges and return the row's first (leading) run, which the join with
// column r needs.  Runs inside a piece were counted by the tile kernel, and so
// was the last piece's final run at column n-1 unless it is that piece's
// first.  kStitchBatch pieces are loaded before any is folded.
__device__ void row_pieces(StitchLds &L, const JobDesc &j, int r, uint32_t &lc, uint32_t &ll) {
    const int n = j.n;
    const int a = r + j.wp;                     // first column of the row
    const int W = j.seg_tiles * 64;
    bool lead_open = true, have = false;
    uint32_t oc = 0, ol = 0;
    lc = 0;
    ll = 0;
    auto close = [&](uint32_t c, uint32_t l) {
        if (lead_open) { lc = c; ll = l; lead_open = false; }
        else emit_line(L, j, c, l);
    };
    const int ga = seg_of(j, a), gl = seg_of(j, n - 1);
    const int64_t row = (int64_t)(r - j.s_lo * j.H) * j.segs;   // rows of the band
    for (int gb = ga; gb <= gl; gb += kStitchBatch) {
        uint32_t fv[kStitchBatch], hv[kStitchBatch];
#pragma unroll
        for (int u = 0; u < kStitchBatch; ++u) {
            if (gb + u <= gl) {
                fv[u] = *glb(j.hfirst + row + gb + u);
                hv[u] = *glb(j.hlast + row + gb + u);
            }
        }
#pragma unroll
        for (int u = 0; u < kStitchBatch; ++u) {
            const int g = gb + u;
            if (g > gl) break;
            const int g0 = (j.seg_base + g * j.seg_tiles) * 64;
            const int lo = a > g0 ? a : g0;
            const int hi = n - 1 < g0 + W - 1 ? n - 1 : g0 + W - 1;
            const uint32_t len = (uint32_t)(hi - lo + 1);
            const bool last = g == gl;
            const uint32_t f = fv[u];
            const uint32_t fc = f >> 31, fl = f & 0x7FFFFFFFu;
            if (have && fc == oc) {
                ol += fl;
            } else {
                if (have) close(oc, ol);
                oc = fc;
                ol = fl;
                have = true;
            }
            if (fl == len && !last) continue;       // the piece is one run: it stays open
            close(oc, ol);                          // the open run ends in this piece
            have = false;
            if (!last) {
                oc = hv[u] >> 31;
                ol = hv[u] & 0x7FFFFFFFu;
                have = true;
            }
        }
    }
}

// The written bits (process_strip) of 32 strips of the band, from strip s on (a
// multiple of 32 above the band's first), of a mask entry.
__device__ __forceinline__ uint32_t written32(const JobDesc &j, const uint32_t *mask, int entry, int s) {
    const int word = (s - j.s_lo) >> 5;
    return word < j.mask_words ? *glb(mask + ((int64_t)entry * j.mask_words + word)) : 0u;
}

// The pieces of diagonal k in the (strip, segment) blocks it crosses in strips
// [s, sb], in order, from row ra0 (its first row there): a block's first and
// last black runs are folded across edges.  `open`: the black run that enters.
// r1 is the diagonal's last row.  W is the segment width, g0 the first column of
// segment 0.  FULL: a piece that begins where the diagonal begins, below its
// strip's top row, starts at the matrix's left border: nothing enters it, and
// its runs were counted where they ended.
// Top-edge and bottom-edge summaries exist where the masks say so; those at a
// segment's left or right edge always do.  kStitchBatch pieces are loaded
// before any is folded: one piece at a time cost a memory latency each
// (150 of 740 us of a 65,521-point series).
template <bool FULL>
__device__ __forceinline__ uint32_t fold_diagonal(StitchLds &L, const JobDesc &j, int k, int r0, int r1,
                                                  int s, int sb, uint32_t open, uint32_t wt) {
    const int H = j.H, W = j.seg_tiles * 64, base = j.seg_base * 64;
    int ra = r0 > s * H ? r0 : s * H;          // first row of the next piece
    const int entry = (k >> 6) + j.kb_off;
    uint32_t wf = 0, wl = 0;                   // written bits of strip s's 32
    int have = -1;
    // The segment of the next piece: the one after, where a piece has left at the
    // right edge.  A division per piece stood before every load's address: stitch
    // of a 65,521-point Lorenz series 72 -> 66 us, of the 262,144-point cross
    // recurrence 537 -> 501.
    int g = (ra + k - base) / W;
    while (s <= sb) {
        if ((s - j.s_lo) >> 5 != have) {
            have = (s - j.s_lo) >> 5;
            wf = written32(j, j.dfmask, entry, s);
            wl = written32(j, j.dlmask, entry, s);
        }
        uint32_t fv[kStitchBatch], lv[kStitchBatch], ln[kStitchBatch];   // ln: length, top bits below
        constexpr uint32_t kLast = 1u << 31, kBorder = 1u << 30, kFirst = 1u << 29, kEnd = 1u << 28;
        int count = 0;
#pragma unroll
        for (int u = 0; u < kStitchBatch; ++u) {
            if (s <= sb && (s - j.s_lo) >> 5 == have) {
                const uint32_t bit = 1u << ((s - j.s_lo) & 31);
                const int gend = base + (g + 1) * W - 1;                 // segment's last column
                int rz = r1 < s * H + H - 1 ? r1 : s * H + H - 1;        // last row in the strip
                const bool right = rz + k >= gend;                       // leaves at the right edge
                if (right) rz = gend - k;
                const bool last = rz == r1;
                // the block's first column tile (auto: cut by the strip's)
                const int xs = FULL ? 0 : ((s * H + j.wp) >> 6) * 64;
                const int bx0 = base + g * W > xs ? base + g * W : xs;
                const int64_t idx = (int64_t)((s - j.s_lo) * j.segs + g) * j.dw + (s * H + H - 1 - bx0) + k;
                const bool top = ra == s * H;
                const bool border = FULL && ra == r0 && !top;
                // Every slot is loaded and chosen from at the fold.  Behind conditions
                // per lane the loads went one after the other: stitch of a given
                // 44,915 x 44,915 Lorenz matrix 146 -> 86 us, of 65,516 x 65,516
                // 137 -> 100; where few were written it is no faster (262,144-point
                // cross recurrence 501 -> 512).
                const bool first = !border && (!top || (wf & bit)), end = !last && (right || (wl & bit));
                fv[u] = *glb(j.dfirst + idx);
                lv[u] = *glb(j.dlast + idx);
                ln[u] = (uint32_t)(rz - ra + 1) | (last ? kLast : 0u) | (border ? kBorder : 0u) |
                        (first ? kFirst : 0u) | (end ? kEnd : 0u);
                count = u + 1;
                ra = rz + 1;
                g += right ? 1 : 0;
                if (ra == (s + 1) * H || last) ++s;
                if (last) s = sb + 1;
            }
        }
#pragma unroll
        for (int u = 0; u < kStitchBatch; ++u) {
            if (u >= count) break;
            const uint32_t len = ln[u] & (kEnd - 1u), fb = ln[u] & kFirst ? fv[u] : 0u;
            const bool last = (ln[u] & kLast) != 0u;
            if (!(ln[u] & kBorder)) {
                if (!last && fb == len) { open += len; continue; }
                if (open + fb) emit_stitch(L.bd, kCapD, j.hd, open + fb, wt, (uint32_t)j.hmax, j.flag);
            }
            open = ln[u] & kEnd ? lv[u] : 0u;
        }
    }
    return open;
}

// Lines of a stitch: columns first, then, from here on, diagonals.  Columns and
// diagonals both begin at the first lane of a wave, diagonals so that those of a
// block of 64 (k >> 6) share one: a wave's lines then have one mask entry, and what
// was not written is skipped by whole waves.
__host__ __device__ __forceinline__ int64_t stitch_diag_line(int mode, int64_t n, int64_t nb, int64_t lo) {
    if (mode == kModeAuto) return (n - lo + 63) / 64 * 64;
    return (nb + 63) / 64 * 64 + ((64 - ((n - 1) & 63)) & 63);
}
__device__ __forceinline__ int64_t stitch_diag_line(const JobDesc &j, int64_t lo) {
    return stitch_diag_line(j.mode, j.n, j.nb, lo);
}
__host__ __device__ __forceinline__ int64_t stitch_lines(int mode, int64_t n, int64_t nb, int64_t lo) {
    return stitch_diag_line(mode, n, nb, lo) + (mode == kModeAuto ? n - lo : n + nb - 1);
}

// Stitch of a full (not symmetric) matrix: lines [0, nb) are the columns, lines
// from stitch_diag_line on the diagonals k = -(n-1) .. nb-1.  A diagonal that
// starts inside a strip (at the left border) has no top-edge summary there.
__device__ __forceinline__ void stitch_full(StitchLds &L, const JobDesc &j, int64_t line) {
    const int n = j.n, nb = j.nb, H = j.H, S = j.nstrips;
    // Strips [s_lo, s_hi) of one row band (all strips with one band): a line
    // goes on from the open run an earlier band left in cstate / dstate, and
    // leaves its own there unless its last piece is in this band.
    const int s_lo = j.s_lo, s_hi = j.s_hi;
    const bool first_band = s_lo == 0, last_band = s_hi >= S;
    if (line < nb) {
        const int col = (int)line;
        uint32_t w = 0, wn = written32(j, j.vmask, col >> 6, s_lo);
        uint32_t oc = 0, ol = 0;
        if (!first_band) {
            const uint32_t c = *glb(j.cstate + col);
            oc = c >> 31;
            ol = c & 0x7FFFFFFFu;
        }
        for (int s0 = s_lo; s0 < s_hi; s0 += kStitchBatch) {
            uint32_t fv[kStitchBatch], lv[kStitchBatch];
            if (((s0 - s_lo) & 31) == 0) {   // the next word is loaded one ahead
                w = (uint32_t)__builtin_amdgcn_readfirstlane((int)wn);   // (one tile per wave)
                wn = written32(j, j.vmask, col >> 6, s0 + 32);
            }
#pragma unroll
            for (int u = 0; u < kStitchBatch; ++u) {
                const int s = s0 + u;
                const int64_t idx = (int64_t)(s - s_lo) * nb + col;
                if (s < s_hi) {
                    // The last strip's are always written (its columns end at
                    // the border); another that is not is white from edge to edge.
                    fv[u] = (uint32_t)H;
                    lv[u] = 0u;
                    if (s == S - 1 || (w >> ((s - s_lo) & 31) & 1u)) {
                        fv[u] = *glb(j.vfirst + idx);
                        lv[u] = *glb(j.vlast + idx);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kStitchBatch; ++u) {
                const int s = s0 + u;
                if (s >= s_hi) break;
                const uint32_t Ls = s < S - 1 ? (uint32_t)H : (uint32_t)(n - s * H);
                const uint32_t f = fv[u], l = lv[u];
                const uint32_t fc = f >> 15, fl = f & 0x7FFFu;
                if (fl == Ls) {   // the segment is one run
                    if (ol && oc == fc) ol += Ls;
                    else { emit_line(L, j, oc, ol); oc = fc; ol = Ls; }
                } else {
                    if (ol && oc == fc) emit_line(L, j, fc, ol + fl);
                    else { emit_line(L, j, oc, ol); emit_line(L, j, fc, fl); }
                    oc = l >> 15;
                    ol = l & 0x7FFFu;
                }
            }
        }
        if (last_band) emit_line(L, j, oc, ol);
        else *glb(j.cstate + col) = ol | (oc << 31);
    } else if (line >= stitch_diag_line(j, 0) && line < stitch_diag_line(j, 0) + n + nb - 1) {
        // Diagonal k: its pieces in the (strip, segment) blocks it crosses, in
        // order; a block's first and last black runs are folded across edges.
        const int dk = (int)(line - stitch_diag_line(j, 0));        // carry slot
        const int k = dk - (n - 1);
        const int r0 = k < 0 ? -k : 0;                              // first row
        const int r1 = n - 1 < nb - 1 - k ? n - 1 : nb - 1 - k;     // last row
        const int sa = r0 / H > s_lo ? r0 / H : s_lo;               // its strips in this band
        const int sb = r1 / H < s_hi - 1 ? r1 / H : s_hi - 1;
        if (sa > sb) return;
        uint32_t open = r0 / H < s_lo ? (uint32_t)*glb(j.dstate + dk) : 0u;
        open = fold_diagonal<true>(L, j, k, r0, r1, sa, sb, open, 1u);
        if (r1 / H > sb) *glb(j.dstate + dk) = open;
    }
}

// Stitch of the recurrence matrix of one series over the strips [s_lo, s_hi)
// of one row band (all strips when the job has one band).  Lines of the band:
// the columns [s_lo H, n), then the diagonals k = 0 .. n-1-s_lo H; the other
// lines have no piece in these strips.  A line whose pieces go on in a later
// band keeps its open run in cstate / dstate; column col joins the band and
// row col of U in the band that holds that row (its lead, or its pieces).
__device__ __forceinline__ void stitch_auto(StitchLds &L, const JobDesc &j, int64_t line) {
    const int n = j.n, wp = j.wp, H = j.H;
    const int s_lo = j.s_lo, s_hi = j.s_hi;
    const bool last_band = s_hi >= j.nstrips;
    const bool carried = j.nbands > 1 && s_lo > 0;   // open runs come from earlier bands
    const int64_t lines = (int64_t)n - (int64_t)s_lo * H;
    if (line < lines) {
        // ---- column col of the full matrix ----
        const int col = (int)((int64_t)s_lo * H + line);
        const int s_last = col >= wp ? (col - wp) / H : -1;   // strips holding column col of U
        const int entry = (col >> 6) > j.seg_base ? (col >> 6) - j.seg_base : 0;   // (below: no strips)
        uint32_t w = 0, wn = written32(j, j.vmask, entry, s_lo);
        const int tile = __builtin_amdgcn_readfirstlane(col);   // the wave's first column
        const bool has_row = col + wp <= n - 1;               // row col of U has cells
        const int js = has_row ? col / H : (s_last > 0 ? s_last : 0);
        const bool join = js >= s_lo && (js < s_hi || last_band);
        const int sb = s_last < s_hi - 1 ? s_last : s_hi - 1;   // last strip folded here
        uint32_t oc = 0, ol = 0;   // open run after folding column `col` of U
        if (carried && s_last >= 0 && (join || sb >= s_lo)) {
            const uint32_t c = *glb(j.cstate + col);
            oc = c >> 31;
            ol = c & 0x7FFFFFFFu;
        }
        // The summaries of kStitchBatch strips are loaded before any is
        // folded, so a thread has that many loads in flight.
        for (int s0 = s_lo; s0 <= sb; s0 += kStitchBatch) {
            uint32_t fv[kStitchBatch], lv[kStitchBatch];
            if (((s0 - s_lo) & 31) == 0) {   // the next word is loaded one ahead
                w = (uint32_t)__builtin_amdgcn_readfirstlane((int)wn);   // (one tile per wave)
                wn = written32(j, j.vmask, entry, s0 + 32);
            }
#pragma unroll
            for (int u = 0; u < kStitchBatch; ++u) {
                const int s = s0 + u;
                if (s <= sb) {
                    const int64_t idx = strip_offset(s, n, wp, H) - j.soff_lo + (col - s * H - wp);
                    // A piece that ends inside the strip is always written; one
                    // that is not is white from edge to edge.
                    fv[u] = (uint32_t)H;
                    lv[u] = 0u;
                    const bool bit = w >> ((s - s_lo) & 31) & 1u;
                    if (bit || tile - wp < s * H + H - 1) {   // (of this wave's lanes, see below)
                        fv[u] = *glb(j.vfirst + idx);
                        lv[u] = *glb(j.vlast + idx);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kStitchBatch; ++u) {
                const int s = s0 + u;
                if (s > sb) break;
                const uint32_t Ls = s < s_last ? (uint32_t)H : (uint32_t)(col - wp - s * H + 1);
                // (Chosen here: beside the loads it waited for each pair.  400
                // noise windows 374 -> 335 us, 65,521-point Lorenz series 83 -> 72.)
                const bool there = (w >> ((s - s_lo) & 31) & 1u) || col - wp < s * H + H - 1;
                const uint32_t f = there ? fv[u] : (uint32_t)H, l = there ? lv[u] : 0u;
                const uint32_t fc = f >> 15, fl = f & 0x7FFFu;
                if (fl == Ls) {   // the segment is one run
                    if (ol && oc == fc) ol += Ls;
                    else { emit_line(L, j, oc, ol); oc = fc; ol = Ls; }
                } else {
                    if (ol && oc == fc) emit_line(L, j, fc, ol + fl);
                    else { emit_line(L, j, oc, ol); emit_line(L, j, fc, fl); }
                    oc = l >> 15;
                    ol = l & 0x7FFFu;
                }
            }
        }
        if (!join) {
            if (sb >= s_lo) *glb(j.cstate + col) = ol | (oc << 31);
            return;
        }
        // join: [trailing run of the column of U] [middle] [leading run of row col of U]
        uint32_t mc, ml;
        if (j.theiler == 0) { mc = 1; ml = 1; }
        else {
            const int w = j.theiler;
            const int up = col < w - 1 ? col : w - 1;
            const int dn = (n - 1 - col) < w - 1 ? (n - 1 - col) : w - 1;
            mc = 0;
            ml = (uint32_t)(up + 1 + dn);
        }
        if (ol && oc == mc) ol += ml;
        else { emit_line(L, j, oc, ol); oc = mc; ol = ml; }
        if (has_row) {
            uint32_t hc, hl;
            if (j.segs > 1) {
                row_pieces(L, j, col, hc, hl);
            } else {
                const uint32_t ld = *glb(j.lead + col);
                hc = ld >> 31;
                hl = ld & 0x7FFFFFFFu;
            }
            if (oc == hc) ol += hl;
            else { emit_line(L, j, oc, ol); oc = hc; ol = hl; }
        }
        emit_line(L, j, oc, ol);
    } else if (line >= stitch_diag_line(j, (int64_t)s_lo * H) &&
               line < stitch_diag_line(j, (int64_t)s_lo * H) + lines) {
        // ---- diagonal k of U (and its mirror) ----
        const int k = (int)(line - stitch_diag_line(j, (int64_t)s_lo * H));
        if (k >= wp && j.segs > 1) {
            const int r1 = n - 1 - k;
            const int s_end = r1 / H;                           // >= s_lo
            const int sb = s_end < s_hi - 1 ? s_end : s_hi - 1;
            uint32_t open = carried ? (uint32_t)*glb(j.dstate + k) : 0u;
            open = fold_diagonal<false>(L, j, k, 0, r1, s_lo, sb, open, 2u);
            if (s_end > sb) *glb(j.dstate + k) = open;
        } else if (k >= wp) {
            const int s_last = (n - 1 - k) / H;                 // >= s_lo
            const int sb = s_last < s_hi - 1 ? s_last : s_hi - 1;
            uint32_t open = carried ? (uint32_t)*glb(j.dstate + k) : 0u;
            const int entry = (k >> 6) + j.kb_off;
            uint32_t wf = 0, wl = 0;
            uint32_t wfn = written32(j, j.dfmask, entry, s_lo), wln = written32(j, j.dlmask, entry, s_lo);
            for (int s0 = s_lo; s0 <= sb; s0 += kStitchBatch) {
                uint32_t fv[kStitchBatch], lv[kStitchBatch];
                if (((s0 - s_lo) & 31) == 0) {
                    wf = (uint32_t)__builtin_amdgcn_readfirstlane((int)wfn);
                    wl = (uint32_t)__builtin_amdgcn_readfirstlane((int)wln);
                    wfn = written32(j, j.dfmask, entry, s0 + 32);
                    wln = written32(j, j.dlmask, entry, s0 + 32);
                }
#pragma unroll
                for (int u = 0; u < kStitchBatch; ++u) {
                    const int s = s0 + u;
                    if (s <= sb) {
                        const int64_t idx = strip_offset(s, n, wp, H) - j.soff_lo + (k - wp);
                        fv[u] = 0u;
                        lv[u] = 0u;
                        if (wf >> ((s - s_lo) & 31) & 1u) fv[u] = *glb(j.dfirst + idx);
                        if (wl >> ((s - s_lo) & 31) & 1u) lv[u] = *glb(j.dlast + idx);   // (used if s < s_last)
                    }
                }
#pragma unroll
                for (int u = 0; u < kStitchBatch; ++u) {
                    const int s = s0 + u;
                    if (s > sb) break;
                    const uint32_t fb = fv[u];
                    if (s < s_last && fb == (uint32_t)H) { open += H; continue; }
                    if (open + fb) emit_stitch(L.bd, kCapD, j.hd, open + fb, 2u, (uint32_t)n, j.flag);
                    open = s < s_last ? lv[u] : 0u;
                }
            }
            if (s_last > sb) *glb(j.dstate + k) = open;
        } else if (k == 0 && j.theiler == 0 && s_lo == 0) {
            // main diagonal: every cell (i,i) is recurrent (distance 0 <= eps)
            emit_stitch(L.bd, kCapD, j.hd, (uint32_t)n, 1u, (uint32_t)n, j.flag);
        }
    }
}

__global__ void __launch_bounds__(kStitchThreads) k_stitch(const JobDesc *__restrict__ jobs,
                                                           int njobs) {
    __shared__ StitchLds L;
    static_assert(kStitchCapV <= kCapW, "bins are cleared and flushed in one pass over kCapW");
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].stitch_block0 <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    const JobDesc &j = jobs[lo];
    // No line is longer than hmax, so a short job clears and flushes few bins.
    const int bins = j.hmax + 1 < kCapW ? j.hmax + 1 : kCapW;
    for (int t = threadIdx.x; t < bins; t += blockDim.x) {
        if (t < kCapD) L.bd[t] = 0;
        if (t < kStitchCapV) L.bv[t] = 0;
        L.bw[t] = 0;
    }
    __syncthreads();
    const int64_t line = (int64_t)(blockIdx.x - j.stitch_block0) * blockDim.x + threadIdx.x;
    if (j.mode != kModeAuto) stitch_full(L, j, line);
    else stitch_auto(L, j, line);
    __syncthreads();
    for (int t = threadIdx.x; t < bins; t += blockDim.x) {
        if (t < kCapD && L.bd[t]) g_add(j.hd + t, (unsigned long long)L.bd[t]);
        if (t < kStitchCapV && L.bv[t]) g_add(j.hv + t, (unsigned long long)L.bv[t]);
        if (L.bw[t]) g_add(j.hw + t, (unsigned long long)L.bw[t]);
    }
}

// ---------------------------------------------------------------------------
// Kernels 4 and 5: statistics of the finished histograms (the inputs of the RQA
// measures), so that a result fetch needs only a few hundred bytes.  Integer
// moments are exact (u64); the entropy partial sums use a fixed reduction
// order, so a job's statistics depend only on its own histograms.
// grid = (blocks of the largest job, jobs); block b of a job covers one
// contiguous chunk of lengths.  A job of one block (up to kStatLengths lengths)
// has its moments, its entropies and its flag done by k_stats_moments alone:
// short calls are made of launches, and three kernels of ~10 us (n = 2,000: 14 +
// 8 + 4 us and the gaps between them) become one.  For longer jobs
// k_stats_entropy's last block to finish adds the partial sums up.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void chunk_of(const JobDesc &j, int b, int64_t &lo, int64_t &hi) {
    const int64_t len = (int64_t)j.hmax + 1;
    const int64_t per = (len + j.stat_blocks - 1) / j.stat_blocks;
    lo = (int64_t)b * per;
    hi = lo + per < len ? lo + per : len;
}

constexpr int kStatPer = kStatLengths / kStatThreads;   // lengths a thread takes at a time

// This thread's kStatPer entries of the three histograms from length `base` on,
// all loads issued together (one memory latency; a loop that loads and adds
// pays one per entry: 14 us instead of 5 for a 2,000-point job).
struct StatCounts {
    unsigned long long c[3][kStatPer];
};
__device__ __forceinline__ void load_counts(const JobDesc &j, int64_t base, int64_t hi, StatCounts &s) {
    const unsigned long long *hs[3] = {j.hd, j.hv, j.hw};
#pragma unroll
    for (int h = 0; h < 3; ++h)
#pragma unroll
        for (int u = 0; u < kStatPer; ++u) {
            const int64_t l = base + threadIdx.x + u * kStatThreads;
            s.c[h][u] = l < hi && l > 0 ? *glb(hs[h] + l) : 0ull;
        }
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const unsigned long long o = __shfl_xor(v, d, 64);
        v = o > v ? o : v;
    }
    return v;
}

// This thread's share of -sum p ln p over its loaded lengths >= least.
__device__ __forceinline__ double entropy_part(const unsigned long long *c, int64_t base, int64_t least,
                                               unsigned long long total) {
    double acc = 0.0;
    const double C = (double)total;
#pragma unroll
    for (int u = 0; u < kStatPer; ++u) {
        if (base + threadIdx.x + u * kStatThreads < least || c[u] == 0) continue;
        const double p = (double)c[u] / C;
        acc -= p * log(p);
    }
    return acc;
}

// Sums of three values over the workgroup in a fixed order: lanes by butterfly,
// then the waves (every thread returns with the sums).
__device__ __forceinline__ void block_sums(double (&v)[3], double (*red)[3]) {
#pragma unroll
    for (int h = 0; h < 3; ++h)
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) v[h] = v[h] + __shfl_xor(v[h], d, 64);
    if ((threadIdx.x & 63) == 0)
        for (int h = 0; h < 3; ++h) red[threadIdx.x >> 6][h] = v[h];
    __syncthreads();
    for (int h = 0; h < 3; ++h) {
        v[h] = 0.0;
        for (int w = 0; w < kStatThreads / 64; ++w) v[h] = v[h] + red[w][h];
    }
}

// Called by one whole wave once the statistics are complete: bit 0 of the flag
// (non-finite input), and the info record's copy in pinned host memory, where a
// result fetch finds it after one wait (a copy of its own, and a second wait
// for the histograms, were ~40 us of a 2,000-point call).
__device__ __forceinline__ void finish_job(const JobDesc &j, const double (&ent)[3]) {
    static_assert(kPrepareBlocks == 64, "one k_prepare block per lane");
    const int lane = threadIdx.x & 63;
    const int bad = __ballot(*glb(j.nonfinite + lane) != 0) != 0ull ? 1 : 0;
    if (lane < 3) j.stats->ent[lane] = lane == 0 ? ent[0] : lane == 1 ? ent[1] : ent[2];
    if (lane == 0 && bad) g_or(j.flag, 1);
    if (j.host_info == nullptr) return;
    constexpr int kMoments = offsetof(JobStats, ent) / 8;
    auto *rec = reinterpret_cast<unsigned long long *>(j.host_info + 8);
    const auto *st = reinterpret_cast<const unsigned long long *>(j.stats);
    if (lane < kMoments)
        *glb(rec + lane) = __hip_atomic_load(glb(st + lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else if (lane < kMoments + 3)
        *glb(rec + lane) = (unsigned long long)__double_as_longlong(
            lane == kMoments ? ent[0] : lane == kMoments + 1 ? ent[1] : ent[2]);
    if (lane == 0)
        *glb(rec - 1) = mk64((uint32_t)(bad | __hip_atomic_load(glb(j.flag), __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT)),
                             j.run);
}

__global__ void __launch_bounds__(kStatThreads) k_stats_moments(const JobDesc *__restrict__ jobs) {
    const JobDesc &j = jobs[blockIdx.y];
    if ((int)blockIdx.x >= j.stat_blocks) return;
    const bool alone = j.stat_blocks == 1;
    __shared__ unsigned long long part[kStatThreads / 64][15];
    __shared__ double red[kStatThreads / 64][3];
    int64_t lo, hi;
    chunk_of(j, blockIdx.x, lo, hi);
    // per histogram: count, mass, count and mass from the minimum, longest
    unsigned long long v[3][5] = {};
    StatCounts s;
    for (int64_t base = lo; base < hi; base += kStatLengths) {
        load_counts(j, base, hi, s);
#pragma unroll
        for (int h = 0; h < 3; ++h)
#pragma unroll
            for (int u = 0; u < kStatPer; ++u) {
                const unsigned long long l = (unsigned long long)base + threadIdx.x + u * kStatThreads;
                const unsigned long long c = s.c[h][u];
                if (c == 0) continue;
                v[h][0] += c;
                v[h][1] += c * l;
                if (l >= (unsigned long long)j.mins[h]) {
                    v[h][2] += c;
                    v[h][3] += c * l;
                }
                v[h][4] = l;
            }
    }
#pragma unroll
    for (int h = 0; h < 3; ++h)
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const unsigned long long r = q < 4 ? wave_sum(v[h][q]) : wave_max(v[h][q]);
            if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][h * 5 + q] = r;
        }
    __syncthreads();
    if (threadIdx.x < 15) {
        const int h = threadIdx.x / 5, q = threadIdx.x % 5;
        unsigned long long r = 0;
        for (int w = 0; w < kStatThreads / 64; ++w) {
            const unsigned long long o = part[w][threadIdx.x];
            r = q < 4 ? r + o : (o > r ? o : r);
        }
        part[0][threadIdx.x] = r;
        // JobStats: the five moments are rows of three u64, in the order above.
        static_assert(offsetof(JobStats, longest) == 12 * sizeof(uint64_t), "moment rows");
        unsigned long long *dst = reinterpret_cast<unsigned long long *>(j.stats) + q * 3 + h;
        if (alone) __hip_atomic_store(glb(dst), r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else if (r && q < 4) atomicAdd(dst, r);
        else if (r) atomicMax(dst, r);
    }
    if (!alone) return;
    if (j.host_hist != nullptr) {
        const int64_t hl = (int64_t)j.hmax + 1;
#pragma unroll
        for (int h = 0; h < 3; ++h)
#pragma unroll
            for (int u = 0; u < kStatPer; ++u) {
                const int64_t l = threadIdx.x + u * kStatThreads;
                if (l < hl) glb(j.host_hist)[h * hl + l] = s.c[h][u];
            }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the moments have left (finish_job reads them)
    __syncthreads();
    double e[3];
#pragma unroll
    for (int h = 0; h < 3; ++h) e[h] = entropy_part(s.c[h], lo, j.mins[h], part[0][h * 5 + 2]);
    block_sums(e, red);
    if (threadIdx.x < 64) finish_job(j, e);
}

__global__ void __launch_bounds__(kStatThreads) k_stats_entropy(const JobDesc *__restrict__ jobs) {
    const JobDesc &j = jobs[blockIdx.y];
    if (j.stat_blocks == 1 || (int)blockIdx.x >= j.stat_blocks) return;
    __shared__ double red[kStatThreads / 64][3];
    int64_t lo, hi;
    chunk_of(j, blockIdx.x, lo, hi);
    const unsigned long long *hs[3] = {j.hd, j.hv, j.hw};
    double e[3] = {};
    for (int h = 0; h < 3; ++h) {
        const unsigned long long total = j.stats->cnt_min[h];
        if (!total) continue;
        const double C = (double)total;
        const int64_t from = lo > j.mins[h] ? lo : (int64_t)j.mins[h];
        for (int64_t l = from + threadIdx.x; l < hi; l += kStatThreads) {
            const unsigned long long c = *glb(hs[h] + l);
            if (l == 0 || c == 0) continue;
            const double p = (double)c / C;
            e[h] -= p * log(p);
        }
    }
    if (j.host_hist != nullptr) {
        const int64_t hl = (int64_t)j.hmax + 1;
        for (int h = 0; h < 3; ++h)
            for (int64_t l = lo + threadIdx.x; l < hi; l += kStatThreads)
                glb(j.host_hist)[h * hl + l] = *glb(hs[h] + l);
    }
    block_sums(e, red);
    if (threadIdx.x >= 64) return;
    // The last block's first wave adds the partial sums up, one block per lane,
    // in a fixed order.
    uint32_t done = 0;
    if (threadIdx.x == 0) {
        for (int h = 0; h < 3; ++h)
            __hip_atomic_store(j.ent_part + h * kStatMaxBlocks + blockIdx.x, e[h], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        // The partial sums are agent-scope stores: once they have left (the wait),
        // the count may follow.  (A release at agent scope, which the memory model
        // asks for, writes the whole L2 back, once per block: 74 instead of 36 us for
        // the 400-window batch.  gfx950 keeps the order without it: an agent-scope
        // store is done, and its counter down, when it has reached the level that all
        // CUs share, and the count is added there too.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        done = __hip_atomic_fetch_add(j.stat_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    done = (uint32_t)__builtin_amdgcn_readfirstlane((int)done);
    if (done + 1u != (uint32_t)j.stat_blocks) return;
    // What the other blocks stored before they were counted is read from here on.
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    static_assert(kStatMaxBlocks <= 64, "one statistics block per lane");
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        e[h] = (int)threadIdx.x < j.stat_blocks
                   ? __hip_atomic_load(j.ent_part + h * kStatMaxBlocks + threadIdx.x, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT)
                   : 0.0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) e[h] = e[h] + __shfl_xor(e[h], d, 64);
    }
    finish_job(j, e);
}

// ---------------------------------------------------------------------------
// Recurrence plot output: the masked matrix bit-packed row-major (bit b of word c
// of row i = cell (i, 64c+b)).  A wave owns one 64-row tile row and a chunk of
// column tiles.  For the matrix of one series only tiles on or above the
// diagonal are evaluated; each one above it is also written transposed into the
// mirror tile (the matrix is exactly symmetric).
// ---------------------------------------------------------------------------
struct PlotDesc {
    const float *a;            // rows' series
    const float *b;            // columns' series (one series: a)
    const float *tail;         // coordinates of the last column tile, zero padded
    uint64_t *bits;
    int64_t words;             // 64-bit words per output row
    int64_t nb_points;         // points of b
    int32_t n, nb, m, tau, theiler;
    float thr, thr0;
    int32_t row_tiles, col_tiles, chunks, cross;
    int32_t xchunks;           // column chunks per XCD: ceil(chunks / 8)
    float *boxr, *boxc;        // boxes of the rows' and the columns' vectors (one series: the same)
    int32_t ncr, ncc;          // entries per plane
    int32_t tail_len;
};

constexpr int kPlotChunk = 16;   // column tiles per wave: a 128-byte line of row words

// Boxes of the plot's vectors, and the coordinates of the last column tile.
__global__ void k_plot_prepare(const PlotDesc d) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t base = (int64_t)(d.col_tiles - 1) * 64;
    for (int64_t t = tid; t < d.tail_len; t += stride)
        const_cast<float *>(d.tail)[t] = base + t < d.nb_points ? d.b[base + t] : 0.0f;
    if (d.boxc == nullptr) return;
    make_boxes(d.boxc, d.ncc, d.b, d.nb, d.m, d.tau, tid, stride);
    if (d.boxr != d.boxc) make_boxes(d.boxr, d.ncr, d.a, d.n, d.m, d.tau, tid, stride);
}

template <int NORM, int M>
__global__ void __launch_bounds__(256) k_plot(const PlotDesc d) {
    const int lane = threadIdx.x & 63;
    // Workgroups go to the 8 XCDs in turn (block b to XCD b mod 8), each XCD
    // with its own L2.  XCD x takes the column chunks q = x, x + 8, ... (a
    // balanced share of the triangle), and its consecutive waves take
    // consecutive row tiles of one chunk: the mirror tiles they write are then
    // neighbouring words of the same rows, which meet in that XCD's L2.
    const int x = (int)blockIdx.x & 7;
    const int L = __builtin_amdgcn_readfirstlane((int)(blockIdx.x >> 3) * 4 + (int)(threadIdx.x >> 6));
    const int qq = L / d.row_tiles, r = L - qq * d.row_tiles;
    const int q = qq * 8 + x;
    if (qq >= d.xchunks || q >= d.chunks) return;
    const int n = d.n, nb = d.nb, R = r * 64, i = R + lane;
    const int irow = i < n ? i : n - 1;
    const float *rowp = d.a + irow;
    float xr[M > 0 ? M : 1];
#pragma unroll
    for (int k = 0; k < (M > 0 ? M : 1); ++k) xr[k] = M > 0 ? glb(rowp)[(int64_t)k * d.tau] : 0.0f;
    const int cq = q * kPlotChunk;
    int cbeg = cq;
    const int cend = cbeg + kPlotChunk < d.col_tiles ? cbeg + kPlotChunk : d.col_tiles;
    if (!d.cross && cbeg < r) cbeg = r;
    const int64_t band = d.theiler;
    // Row words go through LDS and out as a row's whole 128-byte line, 16 lanes to
    // a row.  The 35 KB also keep a CU at 16 waves: with 64-byte halves and 28 waves
    // the open lines of the mirror tiles outgrew the XCD's L2 where the boxes leave
    // little to evaluate (60,001 points: sine 342 against 276 us, Lorenz, m = 4, L1,
    // 372 against 295; noise, m = 6, gains from more waves: 546 against 624).
    __shared__ uint64_t words[4][64 * (kPlotChunk + 1)];
    uint64_t *const mine = words[threadIdx.x >> 6];
#pragma unroll 1
    for (int g = 0; g < kPlotChunk / kGroup; ++g) {
        const int cg = cq + g * kGroup;
        if (cg >= cend || cg + kGroup <= cbeg) continue;
        // The tile kernel's classes: only the 8-column pieces that the boxes leave
        // open are evaluated.
        uint64_t act = ~0ull, full = 0ull;
        if constexpr (M > 0)
            classify<NORM, M>(Boxes{d.boxr, d.boxc, d.ncr, d.ncc, d.thr}, r, cg / kGroup, lane, act, full);
        const int u1 = cend - cg < kGroup ? cend - cg : kGroup;
#pragma unroll 1
        for (int u = cbeg > cg ? cbeg - cg : 0; u < u1; ++u) {
            const int c = cg + u;
            const int jbase = c * 64;
            const ConstF cols = to_const(c == d.col_tiles - 1 ? d.tail : d.b + jbase);
            uint32_t xlo, xhi;
            const uint32_t ones = (uint32_t)(full >> (8 * u)) & 0xFFu;
            const uint32_t eval = (uint32_t)(act >> (8 * u)) & 0xFFu & ~ones;
            if (eval == 0xFFu)
                tile_bits<NORM, M>(cols, d.tau, xr, rowp, d.m, d.thr, d.thr0, xlo, xhi);
            else
                tile_bits_some<NORM, M>(cols, d.tau, xr, rowp, d.m, d.thr, d.thr0, eval, ones, xlo, xhi);
            // Cells outside the matrix or inside the Theiler band are 0 (few
            // tiles have any).
            uint64_t vm = ~0ull;
            if (!(R + 64 <= n && jbase + 64 <= nb &&
                  ((int64_t)jbase - (R + 63) >= band || (int64_t)R - (jbase + 63) >= band))) {
                vm = 0ull;
                if (i < n) {
                    const int hv = nb - jbase < 64 ? nb - jbase : 64;
                    vm = range_mask(0, (uint32_t)hv);
                    if (band > 0) {
                        int64_t blo = (int64_t)i - band + 1 - jbase, bhi = (int64_t)i + band - jbase;
                        blo = blo < 0 ? 0 : blo;
                        bhi = bhi > 64 ? 64 : bhi;
                        if (blo < bhi) vm &= ~range_mask((uint32_t)blo, (uint32_t)bhi);
                    }
                }
            }
            const uint64_t X = mk64(xlo, xhi) & vm;
            mine[lane * (kPlotChunk + 1) + (c - cq)] = X;
            if (!d.cross && c > r) {
                uint32_t lo = (uint32_t)X, hi = (uint32_t)(X >> 32);
                if (__builtin_amdgcn_ballot_w64(X != 0ull) != 0ull) transpose64(lo, hi, lane);
                const int jr = jbase + lane;   // row of the mirror tile
                if (jr < n) glb(d.bits)[(int64_t)jr * d.words + r] = mk64(lo, hi);
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's own LDS
#pragma unroll 8
    for (int it = 0; it < kPlotChunk; ++it) {
        const int row = it * 4 + (lane >> 4), c = cq + (lane & 15);
        if (R + row < n && c >= cbeg && c < cend)
            glb(d.bits)[(int64_t)(R + row) * d.words + c] = mine[row * (kPlotChunk + 1) + (lane & 15)];
    }
}

using PlotKernel = void (*)(const PlotDesc);

template <int NORM>
PlotKernel pick_plot(int m) {
    switch (m) {
        case 1: return k_plot<NORM, 1>;
        case 2: return k_plot<NORM, 2>;
        case 3: return k_plot<NORM, 3>;
        case 4: return k_plot<NORM, 4>;
        case 5: return k_plot<NORM, 5>;
        case 6: return k_plot<NORM, 6>;
        default: return k_plot<NORM, 0>;
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
using TileKernel = void (*)(const JobDesc *, const GroupDesc *, int, int *);

template <int NORM, int MODE>
TileKernel pick_kernel(int m) {
    switch (m) {
        case 1: return k_tiles<NORM, 1, MODE>;
        case 2: return k_tiles<NORM, 2, MODE>;
        case 3: return k_tiles<NORM, 3, MODE>;
        case 4: return k_tiles<NORM, 4, MODE>;
        case 5: return k_tiles<NORM, 5, MODE>;
        case 6: return k_tiles<NORM, 6, MODE>;
        default: return k_tiles<NORM, 0, MODE>;
    }
}

template <int MODE>
TileKernel tile_kernel_mode(int norm, int m) {
    if (norm == RQA_NORM_L1) return pick_kernel<RQA_NORM_L1, MODE>(m);
    if (norm == RQA_NORM_L2) return pick_kernel<RQA_NORM_L2, MODE>(m);
    return pick_kernel<RQA_NORM_LINF, MODE>(m);
}

TileKernel tile_kernel(int mode, int norm, int m) {
    if (mode == kModeMatrix) return k_tiles<RQA_NORM_LINF, 1, kModeMatrix>;   // no predicate
    if (mode == kModeCross) return tile_kernel_mode<kModeCross>(norm, m);
    return tile_kernel_mode<kModeAuto>(norm, m);
}

int group_key(const Job &jb) {
    const int nm = jb.mode == kModeMatrix ? 0 : jb.kp.norm * 16 + (jb.kp.m <= kMaxM ? jb.kp.m : 0);
    return ((jb.mode * 64) + nm) * 32 + jb.waves;
}

struct Layout {
    int H, nstrips;
    int band, nbands;      // strips per row band (auto mode) and the number of bands
    int segs, seg_tiles;   // column segments per strip and their width (tiles)
    int seg_base;          // first column tile of segment 0
    int64_t hentries;      // row pieces (auto, segs > 1): rows of one band * segs
    int items;             // work items of the largest band: band * segs
    int64_t blocks;        // its tiles, counted in items of a whole segment
    int dw;                // full matrix: diagonal summary slots per block
    int64_t ventries;      // vertical summary entries per array (first, last), one band
    int64_t dentries;      // diagonal summary entries per array, one band
    int64_t tail_len;
    int ncr, ncc;          // boxes of the rows' and the columns' vectors (0: none)
    int64_t box_floats;    // floats of their planes
    int mask_words;        // words per mask entry
    int64_t vmask_entries, dmask_entries;
    size_t off_tail, off_lead, off_vf, off_vl, off_df, off_dl, off_ent, off_nf, off_hf, off_hl, off_box,
        off_mask, off_cs, off_ds, bytes;
    size_t charge;         // of these, what a limit or a budget counts (below)
};

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

// Work items (strips x column segments) a single series run alone is cut
// into: a few times the workgroups one launch keeps resident (256 CUs x 3).
constexpr int kTargetItems = 2048;
// Work items of a series cut into column segments (per row band when banded)
// and of a full-matrix job: shorter chains of tiles, so that the launch's
// last, partly idle round of items is short (cross recurrence of 2 x 262,144
// points 10.3 -> 9.3 ms, given 65,516^2 matrix 0.72 -> 0.50 ms against 2,048
// items; 16,384 items made the given matrix slower again).
constexpr int kSegItems = 8192;    // (one series alone, one band or several)
constexpr int kFullItems = 8192;
constexpr int kFullFineItems = 1024;

// Offset of the first evaluated diagonal of U, max(theiler, 1), clamped to n:
// every window of n or more masks the whole matrix alike, and the clamp keeps
// the kernels' 32-bit row + offset arithmetic from overflowing.
int effective_wp(int32_t theiler, int64_t n) {
    const int64_t w = theiler > 1 ? theiler : 1;
    return (int)(w < n ? w : (n > 1 ? n : 1));
}

int default_waves_impl(int64_t n) {
    // Eight waves per workgroup measured fastest from about 16,000 vectors on
    // (20,000 Lorenz points, tiles + stitch: 156 us, 177 with four); shorter
    // series use four so that more strips exist.
    if (n >= 16384) return 8;
    return 4;
}

// Column segments of an auto-mode job when it runs alone (`nstrips`: the
// strips of one launch, i.e. of one row band).
//  * Enough for about kSegItems work items, each at least 64 tiles wide, for
//    jobs whose first strip has 128 tiles or more (a 199,873-vector served job at
//    RR 5%: 13.9 ms with 2,048 items, 12.1 with 4,096, 11.5 with 8,192; a
//    300,000-point Lorenz series 9.2 / 8.3 / 7.8 ms).
//  * With `fine` (a handle's own run) up to kFineSegs, however narrow: a short job is
//    its longest chain of tiles (7 us each at RR 12%, for want of other waves to
//    hide their latency), and cutting it into 16 to 20 costs less in the stitch
//    than it saves.  Tile kernel + stitch, whole strips -> cut: 500 points 73 -> 41
//    us, 2,000 (RR 12%) 270 -> 72, 9,973 (AR(1)) 500 -> 149, 20,000 (Lorenz) 254 -> 156.
//    As many of them as give the shortest time if every round of blocks takes
//    that of a whole segment: 20 are no gain where they begin a round that they leave
//    half empty.  Uniform points (RR 19%), 20 segments -> this many: 56,761 with 8
//    waves 3,164 -> 2,850 us (13), 40,000 1,817 -> 1,497 (18), 26,000 with 4 886 -> 802
//    (19); Lorenz and sine 2-6% there.  (A whole round is 740 of the 768 blocks of
//    eight waves that the chip holds, 988 of the 1,024 of four: with 768, the blocks
//    that the diagonal cuts short begin another one, 40,000 points 1,607.)
//    (A served job keeps the first rule, and its footprint.)
//  * 1 for jobs of more than kTargetItems / 2 strips (the 1,048,576-point workload
//    has 2,048): whole strips leave no CU idle there.
constexpr int kFineSegs = 20;
constexpr int kRoundBlocks = 740, kRoundBlocks4 = 988;
// Tiles of the first nstrips strips, of T0 tiles and H/64 fewer each.
int64_t strip_tiles(int T0, int H, int nstrips) {
    return (int64_t)nstrips * T0 - (int64_t)nstrips * (nstrips - 1) / 2 * (H / 64);
}
int auto_segs_max(int64_t n, int wp, int H, int nstrips, bool fine) {
    const int T0 = (int)((n - 1) / 64 - wp / 64 + 1);
    if (nstrips < 1 || 2 * nstrips > kTargetItems) return 1;
    int segs = 1;
    if (T0 >= 128)
        segs = (int)std::max<int64_t>(1, std::min<int64_t>((kSegItems + nstrips - 1) / nstrips, T0 / 64));
    if (fine) {
        const int64_t tiles = strip_tiles(T0, H, nstrips);
        const int whole = H > 64 * 4 ? kRoundBlocks : kRoundBlocks4;   // (white_bins)
        const auto rounds = [&](int t) {   // of blocks, `tiles` in all, a t-th of a strip's T0 each
            return ((tiles * t + T0 - 1) / T0 + whole - 1) / whole;
        };
        const int least = segs, most = std::min(T0, kFineSegs);
        for (int t = least + 1; t <= most; ++t)
            if (rounds(t) * segs <= rounds(segs) * t) segs = t;
    }
    return segs;
}

// Whether a job of these row and column tiles takes boxes.  A run alone of fewer
// than 128 column tiles does not: its time is a chain of tiles too short to fill
// the chip, of which the predicate is a small part.  Jobs that may share a launch
// do from 32 on (190 sine windows of 3,652 points 557 -> 356 us, 200 of 8,000 1.87 ->
// 1.01 ms, 400 noise windows of 3,000 1.12 -> 1.12; 24 tiles: no gain), and so do tall
// cross matrices, whose many row tiles fill the chip (200,000 x 8,000 sine 668 -> 598
// us, Lorenz 750 -> 722; of 50,000 x 8,000, 98,000 tiles, Lorenz gained 1%, noise lost 3).
bool boxes_pay(const Job &jb, int64_t rtiles, int64_t ctiles) {
    if (!jb.boxes || jb.mode == kModeMatrix || jb.kp.m > kMaxM || ctiles < 32) return false;
    return ctiles >= 128 || (jb.mode == kModeAuto ? !jb.fine : rtiles * ctiles >= 131072);
}

Layout layout_of(const Job &jb) {
    Layout L{};
    const int64_t n = jb.n_vec;
    const int wp = effective_wp(jb.kp.theiler, n);
    L.H = 64 * (jb.waves > 0 ? jb.waves : default_waves_impl(n));
    if (jb.mode == kModeAuto) {
        L.nstrips = n - wp > 0 ? (int)((n - wp + L.H - 1) / L.H) : 0;
        // Row bands: the summaries hold the strips of one band (the first,
        // whose strips are the longest); the open runs of every line pass
        // from band to band in per-line carries.
        L.band = jb.band_strips > 0 && jb.band_strips < L.nstrips ? jb.band_strips : L.nstrips;
        L.nbands = L.band > 0 ? (L.nstrips + L.band - 1) / L.band : 1;
        // sum over the band's strips of (n - wp - s H) entries
        L.ventries = strip_offset(L.band, (int32_t)n, wp, L.H);
        // Segments: as set on the job, else the most it could be given.
        const int T0 = (int)((n - 1) / 64 - wp / 64 + 1);
        int segs = jb.segs > 0 ? std::min(jb.segs, std::max(T0, 1)) : auto_segs_max(n, wp, L.H, L.band, jb.fine);
        L.seg_base = wp / 64;
        L.seg_tiles = (T0 + segs - 1) / segs;
        L.segs = segs > 1 ? (T0 + L.seg_tiles - 1) / L.seg_tiles : 1;
        if (L.segs > 1) {
            L.dw = L.seg_tiles * 64 + L.H - 1;
            L.dentries = (int64_t)L.band * L.segs * L.dw;
            L.hentries = std::min<int64_t>(n, (int64_t)L.band * L.H) * L.segs;
        } else {
            L.dw = 0;
            L.dentries = L.ventries;
            L.hentries = 0;
        }
        L.blocks = L.band > 0 ? strip_tiles(T0, L.H, L.band) * L.segs / T0 : 0;
    } else {
        // A strip of a full matrix walks every column tile; its chain of
        // tiles is cut into column segments walked by different workgroups,
        // enough of them for about kFullItems work items, each at least
        // max(8, H/64) tiles wide; in a run alone, narrower where that leaves fewer
        // than kFullFineItems items, down to a kFineSegs-th of the chain (with no
        // such bound the 200,000 x 1,000 uniform cross recurrence, 391 strips, was
        // cut into single tiles: 658 us, 501 in 3 segments, 518 in the 2 wide ones;
        // a bound of 2,048 items: 531).
        const int64_t nb = jb.n_cols;
        L.nstrips = (int)((n + L.H - 1) / L.H);
        // Row bands as in auto mode: summaries for one band's strips.
        L.band = jb.band_strips > 0 && jb.band_strips < L.nstrips ? jb.band_strips : L.nstrips;
        L.nbands = (L.nstrips + L.band - 1) / L.band;
        const int T = (int)((nb - 1) / 64 + 1);
        const int wide = std::max(8, L.H / 64);
        int segs = std::max(1, std::min((kFullItems + L.band - 1) / L.band, T / wide));
        if (jb.fine)
            segs = std::max(segs, std::min((kFullFineItems + L.band - 1) / L.band,
                                           T / std::max(1, std::min(wide, T / kFineSegs))));
        L.seg_base = 0;
        L.seg_tiles = (T + segs - 1) / segs;
        L.segs = (T + L.seg_tiles - 1) / L.seg_tiles;
        L.dw = L.seg_tiles * 64 + L.H - 1;
        L.ventries = (int64_t)L.band * nb;
        L.dentries = (int64_t)L.band * L.segs * L.dw;
        L.hentries = 0;
    }
    L.items = L.band * L.segs;
    if (jb.mode != kModeAuto) L.blocks = L.items;
    if (L.ventries < 1) L.ventries = 1;
    if (L.dentries < 1) L.dentries = 1;
    L.tail_len = jb.mode == kModeMatrix ? 0 : 64 + (int64_t)(jb.kp.m - 1) * jb.kp.tau;
    // Row leads: with whole strips only (with segments the row pieces hold them).
    const int64_t lead = jb.mode == kModeAuto && L.segs == 1 ? n : 1;
    size_t off = 0;
    L.off_tail = off; off += a256(sizeof(float) * (size_t)L.tail_len);
    L.off_lead = off; off += a256(sizeof(uint32_t) * (size_t)lead);
    L.off_vf = off; off += a256(sizeof(uint16_t) * (size_t)L.ventries);
    L.off_vl = off; off += a256(sizeof(uint16_t) * (size_t)L.ventries);
    L.off_df = off; off += a256(sizeof(uint16_t) * (size_t)L.dentries);
    L.off_dl = off; off += a256(sizeof(uint16_t) * (size_t)L.dentries);
    // Statistics: entropy partial sums, the count of finished blocks, and
    // k_prepare's non-finite notes.
    L.off_ent = off;
    L.off_nf = off + sizeof(double) * 3 * kStatMaxBlocks;
    off += a256(sizeof(double) * 3 * kStatMaxBlocks + sizeof(uint32_t) + kPrepareBlocks);
    L.off_hf = off; off += a256(sizeof(uint32_t) * (size_t)L.hentries);
    L.off_hl = off; off += a256(sizeof(uint32_t) * (size_t)L.hentries);
    // Boxes for the modes with a predicate and the embedding dimensions whose
    // row coordinates live in registers.
    const int64_t ncols = jb.mode == kModeAuto ? n : jb.n_cols;
    const int64_t ctiles = (ncols - 1) / 64 + 1;
    if (boxes_pay(jb, (n - 1) / 64 + 1, ctiles)) {
        L.ncc = (int)((ctiles + kGroup - 1) / kGroup * kGroup * (64 / kBoxVecs));
        L.ncr = jb.mode == kModeAuto ? L.ncc : (int)(((n - 1) / 64 + 1) * (64 / kBoxVecs));
        L.box_floats = kBoxHeader + 2 * std::min(jb.kp.m, kBoxK) *
                                        ((int64_t)L.ncc + (jb.mode == kModeAuto ? 0 : L.ncr));
    }
    L.off_box = off; off += a256(sizeof(float) * (size_t)L.box_floats);
    // Masks of what summaries were written: a bit per strip of the band, for
    // every column tile and (twice) every block of 64 diagonals.
    L.mask_words = (L.band + 31) / 32;
    // (Auto mode: from the first with a cell outside the Theiler window.)
    L.vmask_entries = std::max<int64_t>(1, ctiles - L.seg_base);
    L.dmask_entries = L.vmask_entries + 1 + (jb.mode == kModeAuto ? 0 : (n - 1) / 64 + 1);
    L.off_mask = off;
    off += a256(sizeof(uint32_t) * (size_t)((L.vmask_entries + 2 * L.dmask_entries) * L.mask_words));
    // Per-line carries between bands: the open run of each column (of U in
    // auto mode) and of each diagonal (n - 1 + nb of them in a full matrix).
    const bool banded = L.nbands > 1;
    const size_t ccarries = banded ? (size_t)(jb.mode == kModeAuto ? n : jb.n_cols) : 0;
    const size_t dcarries = banded ? (size_t)(jb.mode == kModeAuto ? n : n + jb.n_cols - 1) : 0;
    L.off_cs = off; off += a256(sizeof(uint32_t) * ccarries);
    L.off_ds = off; off += a256(sizeof(uint32_t) * dcarries);
    L.bytes = off;
    // Limits and budgets count the line summaries of strips cut no finer than into
    // wide segments, the tail, the row leads (whether or not the segments hold them)
    // and the carries, and 32 bytes per column tile where there can be boxes.  On top
    // come the boxes and masks themselves (3 bytes per vector at most, and under 0.2%
    // of the summaries) and what a short run's narrow segments add (8 MiB or 4%): a
    // limit then cuts a run into the row bands that its wide cut needs, and no more.
    // (Counted, they cut 2,000 points in 100 KiB into 8 bands: 272 us, one band 74.)
    if (jb.fine) {
        Job wide = jb;
        wide.fine = false;
        L.charge = layout_of(wide).charge;
        return L;
    }
    L.charge = off - a256(sizeof(float) * (size_t)L.box_floats) -
               a256(sizeof(uint32_t) * (size_t)((L.vmask_entries + 2 * L.dmask_entries) * L.mask_words)) +
               (jb.mode == kModeAuto ? a256(sizeof(uint32_t) * (size_t)n) - a256(sizeof(uint32_t) * (size_t)lead) : 0) +
               (jb.mode != kModeMatrix && jb.kp.m <= kMaxM ? a256(sizeof(float) * (size_t)(64 + 8 * ctiles)) : 0);
    return L;
}


// Device descriptor of one job whose work items start at `strip_base` of its
// group and whose stitch blocks start at `stitch_block0`.
JobDesc make_desc(const Job &jb, const Layout &lay, int strip_base, int stitch_block0) {
    const KParams &kp = jb.kp;
    char *scr = static_cast<char *>(jb.scratch);
    JobDesc d{};
    const bool full = jb.mode != kModeAuto;
    const int64_t hlen = jb.hist_len();
    const int64_t stride = jb.hist_stride > 0 ? jb.hist_stride : hlen;
    const int64_t ncols = full ? jb.n_cols : jb.n_vec;
    d.s = jb.series;
    d.sb = jb.mode == kModeCross ? jb.series_b : jb.series;
    d.n_points_b = jb.mode == kModeCross ? jb.n_points_b : jb.n_points;
    d.bits = jb.bits;
    d.words = jb.words;
    d.tail = reinterpret_cast<const float *>(scr + lay.off_tail);
    d.hd = reinterpret_cast<unsigned long long *>(jb.hist);
    d.hv = d.hd + stride;
    d.hw = d.hv + stride;
    d.flag = jb.flag;
    d.lead = reinterpret_cast<uint32_t *>(scr + lay.off_lead);
    d.vfirst = reinterpret_cast<uint16_t *>(scr + lay.off_vf);
    d.vlast = reinterpret_cast<uint16_t *>(scr + lay.off_vl);
    d.dfirst = reinterpret_cast<uint16_t *>(scr + lay.off_df);
    d.dlast = reinterpret_cast<uint16_t *>(scr + lay.off_dl);
    d.n_points = jb.n_points;
    d.n = (int32_t)jb.n_vec;
    d.nb = (int32_t)ncols;
    d.hmax = (int32_t)(hlen - 1);
    d.mode = jb.mode;
    d.m = kp.m;
    d.tau = kp.tau;
    d.norm = kp.norm;
    d.theiler = kp.theiler;
    d.wp = effective_wp(kp.theiler, jb.n_vec);
    d.thr = kp.norm == RQA_NORM_L2 ? kp.eps_sq : kp.eps;
    d.thr0 = kp.d0_bound;
    d.H = lay.H;
    d.nstrips = lay.nstrips;
    d.segs = lay.segs;
    d.seg_tiles = lay.seg_tiles;
    d.seg_base = lay.seg_base;
    d.dw = lay.dw;
    d.hfirst = lay.hentries > 0 ? reinterpret_cast<uint32_t *>(scr + lay.off_hf) : nullptr;
    d.hlast = lay.hentries > 0 ? reinterpret_cast<uint32_t *>(scr + lay.off_hl) : nullptr;
    d.s_lo = 0;
    d.s_hi = lay.band;
    d.band_strips = lay.band;
    d.nbands = lay.nbands;
    d.soff_lo = 0;
    d.cstate = lay.nbands > 1 ? reinterpret_cast<uint32_t *>(scr + lay.off_cs) : nullptr;
    d.dstate = lay.nbands > 1 ? reinterpret_cast<uint32_t *>(scr + lay.off_ds) : nullptr;
    d.c_last = (int32_t)((ncols - 1) / 64);
    d.tail_len = (int32_t)lay.tail_len;
    d.strip_base = strip_base;
    d.stitch_block0 = stitch_block0;
    d.mins[0] = kp.lmin;
    d.mins[1] = kp.vmin;
    d.mins[2] = kp.wmin;
    d.stat_blocks = (int32_t)std::min<int64_t>(
        kStatMaxBlocks, std::max<int64_t>(1, (hlen + kStatLengths - 1) / kStatLengths));
    d.stat_done = reinterpret_cast<uint32_t *>(scr + lay.off_nf);
    d.nonfinite = reinterpret_cast<uint8_t *>(d.stat_done + 1);
    d.stats = jb.stats ? reinterpret_cast<JobStats *>(jb.stats)
                       : reinterpret_cast<JobStats *>(reinterpret_cast<char *>(jb.flag) + 8);
    d.ent_part = reinterpret_cast<double *>(scr + lay.off_ent);
    d.host_info = static_cast<unsigned char *>(jb.host_info);
    d.run = jb.run;
    d.host_hist = static_cast<unsigned long long *>(jb.host_hist);
    d.boxc = lay.box_floats > 0 ? reinterpret_cast<float *>(scr + lay.off_box) + kBoxHeader : nullptr;
    d.decided = reinterpret_cast<uint8_t *>(scr + lay.off_box);
    // 128 pieces of a short job, 2,048 of one of 131,072 vectors (the samples of
    // 400 windows of 3,000 points, 2,048 each, took 70 us).
    d.sample_blocks = (int32_t)std::min<int64_t>(kPrepareBlocks, std::max<int64_t>(4, ncols / 2048));
    d.boxr = jb.mode == kModeAuto || !d.boxc
                 ? d.boxc : d.boxc + (int64_t)2 * std::min(kp.m, kBoxK) * lay.ncc;
    d.ncc = lay.ncc;
    d.ncr = lay.ncr;
    d.mask_words = lay.mask_words;
    d.vmask = reinterpret_cast<uint32_t *>(scr + lay.off_mask);
    d.dfmask = d.vmask + lay.vmask_entries * lay.mask_words;
    d.dlmask = d.dfmask + lay.dmask_entries * lay.mask_words;
    d.mask_total = (lay.vmask_entries + 2 * lay.dmask_entries) * lay.mask_words;
    d.kb_off = 1 + (full ? (int32_t)((jb.n_vec - 1) / 64 + 1) : -lay.seg_base);
    // Fault injection for tests of the give-up path: with
    // RQA_DEBUG_WAIT_GIVEUP=1 in the environment every neighbour wait of the
    // tile kernel aims at a count no wave reaches and gives up after 64
    // polls; the kernels still finish and the job reports RQA_EDEVICE.
    const char *giveup = std::getenv("RQA_DEBUG_WAIT_GIVEUP");
    const bool inject = giveup && giveup[0] == '1';
    d.spin_limit = inject ? 64 : (int32_t)kSpinLimit;
    d.wait_bias = inject ? (1 << 30) : 0;
    return d;
}

// Statistics of njobs jobs, the largest of which has `blocks` statistics blocks.
void launch_stats(const JobDesc *jobs, int blocks, int njobs, hipStream_t st) {
    hipLaunchKernelGGL(k_stats_moments, dim3(blocks, njobs), dim3(kStatThreads), 0, st, jobs);
    if (blocks > 1)
        hipLaunchKernelGGL(k_stats_entropy, dim3(blocks, njobs), dim3(kStatThreads), 0, st, jobs);
}

// k_prepare blocks of a launch: a thread per length or point of its longest job, up
// to kPrepareBlocks (64 for each of 400 windows of 3,000 points: 31 us, 15 so).
int prepare_blocks_of(const Job &jb) {
    const int64_t most = std::max({jb.hist_len(), jb.n_points, jb.n_points_b});
    return (int)std::max<int64_t>(4, std::min<int64_t>(kPrepareBlocks, (most + kPrepareThreads - 1) / kPrepareThreads));
}

// LDS bins for the white lengths of a launch of that many blocks, whose longest line
// has `len` - 1.  Six thousand let three workgroups share a CU.  Of those of up to four
// waves there may be four, with fewer bins, where there are blocks for them: 12 waves
// hide too little (200 windows of 8,000 points, L1, m = 5, 3.82 -> 3.34 ms, sine 1.38 ->
// 1.20, 1,800 x 80,000 uniform cross recurrence 228 -> 206 us).  Blocks of less than a
// round they would pack onto fewer CUs (16,000 uniform points 399 -> 468 us).
constexpr int kCapW4 = 4992;
static_assert(3 * strip_lds_bytes(kCapW) <= 160 * 1024 && 4 * strip_lds_bytes(kCapW4) <= 160 * 1024,
              "workgroups per CU");
int white_bins(int waves, int64_t blocks, int64_t len) {
    return (int)std::min<int64_t>(waves <= 4 && blocks > kRoundBlocks ? kCapW4 : kCapW,
                                  (len + kLeastWhiteBins - 1) / kLeastWhiteBins * kLeastWhiteBins);
}

int stitch_blocks_of(const Job &jb) {
    const bool full = jb.mode != kModeAuto;
    const int64_t lines = stitch_lines(jb.mode, jb.n_vec, full ? jb.n_cols : jb.n_vec, 0);
    return (int)((lines + kStitchThreads - 1) / kStitchThreads);
}

}  // namespace

size_t engine_job_scratch_bytes(const Job &job) { return layout_of(job).bytes; }

int engine_band_strips(const Job &job, size_t limit) {
    if (limit == 0) return 0;
    Job jb = job;
    jb.band_strips = 0;
    const Layout all = layout_of(jb);
    if (all.charge <= limit || all.nstrips <= 1) return 0;
    // The largest band whose scratch fits (the scratch grows with the band,
    // up to the jumps where the column segments per strip change).
    int lo = 1, hi = all.nstrips - 1;
    while (lo < hi) {
        const int mid = lo + (hi - lo + 1) / 2;
        jb.band_strips = mid;
        if (layout_of(jb).charge <= limit) lo = mid; else hi = mid - 1;
    }
    jb.band_strips = lo;
    while (lo > 1 && layout_of(jb).charge > limit) jb.band_strips = --lo;
    return lo;
}

// With strips of 8 waves from 32,768 vectors on, and of 4 below: what a budget
// admits does not follow the default shape.
size_t engine_budget_bytes(Job jb) {
    jb.waves = jb.n_vec >= 32768 ? 8 : 4;
    return layout_of(jb).charge;
}

JobPlan engine_job_plan(const Job &job) {
    const Layout lay = layout_of(job);
    JobPlan p{};
    p.bands = lay.nbands;
    p.band_strips = lay.band;
    p.segs = lay.segs;
    p.strip_rows = lay.H;
    p.scratch_bytes = lay.charge;
    return p;
}

int engine_default_waves(int64_t n) { return default_waves_impl(n); }

// Few windows, or short ones, leave CUs idle as whole strips: the chains of
// tiles are then cut so that the launch has about kBatchItems work items (at
// least two tiles each).
void engine_batch_segs(std::vector<Job> &jobs) {
    constexpr int64_t kBatchItems = 4096;
    int64_t strips = 0;
    for (const Job &jb : jobs) strips += (jb.n_vec + 64 * jb.waves - 1) / (64 * jb.waves);
    const int64_t segs = kBatchItems / std::max<int64_t>(strips, 1);
    for (Job &jb : jobs)
        jb.segs = (int)std::max<int64_t>(1, std::min<int64_t>({segs, jb.n_vec / 128, kFineSegs}));
}

size_t engine_launch_scratch_bytes(size_t njobs) {
    return a256(sizeof(JobDesc) * njobs) + a256(sizeof(GroupDesc) * 64) + 256;
}

int AuxStreams::create(int n) {
    n = n < kMax ? n : kMax;
    for (int k = 0; k < n; ++k) {
        if (hipStreamCreateWithFlags(&s[k], hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&join[k], hipEventDisableTiming) != hipSuccess) {
            count = k;
            destroy();
            return RQA_EDEVICE;
        }
        count = k + 1;
    }
    if (hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess) {
        destroy();
        return RQA_EDEVICE;
    }
    return RQA_OK;
}

void AuxStreams::destroy() {
    for (int k = 0; k < count; ++k) {
        if (s[k]) hipStreamDestroy(s[k]);
        if (join[k]) hipEventDestroy(join[k]);
        s[k] = nullptr;
        join[k] = nullptr;
    }
    if (fork) hipEventDestroy(fork);
    fork = nullptr;
    count = 0;
}

int engine_launch(const std::vector<Job> &jobs_in, void *launch_scratch, void *staging,
                  hipEvent_t staging_free, int groups_req, hipStream_t st,
                  const PhaseEvents *phases, AuxStreams *aux) {
    const int njobs = (int)jobs_in.size();
    if (njobs == 0) return RQA_OK;
    for (const Job &jb : jobs_in)
        if (jb.waves < 1 || jb.waves > kMaxWaves) return RQA_EINVAL;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return RQA_EDEVICE;
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return RQA_EDEVICE;

    // Order: by (norm, m, waves) group, then by decreasing size (largest strips first).
    std::vector<int> order(njobs);
    for (int k = 0; k < njobs; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        const int ga = group_key(jobs_in[a]), gb = group_key(jobs_in[b]);
        if (ga != gb) return ga < gb;
        return jobs_in[a].n_vec > jobs_in[b].n_vec;
    });

    // The descriptors of a launch of one job travel as kernel arguments; those
    // of several are staged and copied.  The previous launch that used
    // `staging` must have consumed it.
    std::vector<JobDesc> one_desc(njobs == 1 ? 1 : 0);
    std::vector<GroupDesc> one_group(njobs == 1 ? 64 : 0);
    if (njobs > 1 && staging_free && hipEventSynchronize(staging_free) != hipSuccess) return RQA_EDEVICE;

    char *dbase = static_cast<char *>(launch_scratch);
    JobDesc *hdesc = njobs == 1 ? one_desc.data() : static_cast<JobDesc *>(staging);
    GroupDesc *hgroups = njobs == 1 ? one_group.data()
                                    : reinterpret_cast<GroupDesc *>(static_cast<char *>(staging) +
                                                                    a256(sizeof(JobDesc) * njobs));
    JobDesc *ddesc = reinterpret_cast<JobDesc *>(dbase);
    GroupDesc *dgroups = reinterpret_cast<GroupDesc *>(dbase + a256(sizeof(JobDesc) * njobs));
    int *dcounters = reinterpret_cast<int *>(dbase + a256(sizeof(JobDesc) * njobs) +
                                             a256(sizeof(GroupDesc) * 64));

    std::vector<int> gkeys;
    int stitch_blocks = 0;
    int stat_grid = 1, prepare_grid = 1;
    int ngroups = 0;
    int strip_acc = 0;
    int64_t blocks = 0, longest = 0;   // of the group
    for (int r = 0; r < njobs; ++r) {
        // A job launched with others keeps whole strips: the launch has work
        // items enough, and its scratch is sized for any choice.
        Job jb = jobs_in[order[r]];
        if (jb.segs == 0 && njobs > 1) jb.segs = 1;   // (or what engine_batch_segs chose)
        const Layout lay = layout_of(jb);
        const int key = group_key(jb);
        if (ngroups == 0 || gkeys.back() != key) {
            if (ngroups == 64) return RQA_EINVAL;
            if (ngroups > 0) hgroups[ngroups - 1].items = strip_acc;
            gkeys.push_back(key);
            hgroups[ngroups] = GroupDesc{r, r + 1, 0, 0};   // items, capw: below
            ++ngroups;
            strip_acc = 0;
            blocks = longest = 0;
        }
        hgroups[ngroups - 1].job1 = r + 1;
        blocks += lay.blocks;
        longest = std::max(longest, jb.hist_len());
        hgroups[ngroups - 1].capw = white_bins(jb.waves, blocks, longest);
        JobDesc d = make_desc(jb, lay, strip_acc, stitch_blocks);
        stat_grid = std::max(stat_grid, (int)d.stat_blocks);
        prepare_grid = std::max(prepare_grid, prepare_blocks_of(jb));
        strip_acc += lay.items;
        stitch_blocks += stitch_blocks_of(jb);
        hdesc[r] = d;
    }
    hgroups[ngroups - 1].items = strip_acc;

    if (njobs > 1) {
        const size_t desc_bytes = a256(sizeof(JobDesc) * njobs) + a256(sizeof(GroupDesc) * 64);
        if (hipMemcpyAsync(dbase, staging, desc_bytes, hipMemcpyHostToDevice, st) != hipSuccess)
            return RQA_EDEVICE;
        if (staging_free && hipEventRecord(staging_free, st) != hipSuccess) return RQA_EDEVICE;
    }

    if (phases) hipEventRecord(phases->ev[0], st);
    if (njobs == 1)
        hipLaunchKernelGGL(k_prepare_one, dim3(prepare_grid), dim3(kPrepareThreads), 0, st, hdesc[0],
                           hgroups[0], ddesc, dgroups, dcounters);
    else
        hipLaunchKernelGGL(k_prepare, dim3(prepare_grid, njobs), dim3(kPrepareThreads), 0, st, ddesc,
                           dcounters);

    if (phases) hipEventRecord(phases->ev[1], st);
    if (njobs == 1 && hdesc[0].nbands > 1) {
        // One job in row bands: per band the tile kernel over the band's
        // strips, then the stitch of the lines those strips cross.
        const JobDesc &d = hdesc[0];
        const Job &jb = jobs_in[0];
        TileKernel kern = tile_kernel(jb.mode, jb.kp.norm, jb.kp.m);
        int occ = 0;
        const size_t lds = strip_lds_bytes(hgroups[0].capw);
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 64 * jb.waves, lds) != hipSuccess ||
            occ < 1)
            occ = 1;
        const int full_grid = groups_req > 0 ? groups_req : ncu * occ;
        for (int b = 0; b < d.nbands; ++b) {
            const int lo = b * d.band_strips;
            const int hi = std::min(lo + d.band_strips, d.nstrips);
            const int items = (hi - lo) * d.segs;
            const int64_t lines = stitch_lines(d.mode, d.n, d.nb, (int64_t)lo * d.H);
            hipLaunchKernelGGL(k_band, dim3(64), dim3(256), 0, st, ddesc, dgroups, dcounters, b);
            if (items > 0)
                hipLaunchKernelGGL(kern, dim3(std::min(full_grid, items)), dim3(64 * jb.waves), lds, st,
                                   ddesc, dgroups, 0, dcounters);
            if (phases && b == d.nbands - 1) hipEventRecord(phases->ev[2], st);
            if (lines > 0)
                hipLaunchKernelGGL(k_stitch, dim3((unsigned)((lines + kStitchThreads - 1) / kStitchThreads)),
                                   dim3(kStitchThreads), 0, st, ddesc, 1);
        }
        launch_stats(ddesc, stat_grid, 1, st);
        if (phases) hipEventRecord(phases->ev[3], st);
        return hipGetLastError() == hipSuccess ? RQA_OK : RQA_EDEVICE;
    }
    int active = 0;
    for (int g = 0; g < ngroups; ++g) active += hgroups[g].items > 0;
    const bool fork = aux && aux->count > 0 && active > 1;
    if (fork) hipEventRecord(aux->fork, st);
    bool used[AuxStreams::kMax] = {};
    int launched = 0;
    for (int g = 0; g < ngroups; ++g) {
        const GroupDesc &gd = hgroups[g];
        if (gd.items == 0) continue;
        const KParams &kp = jobs_in[order[gd.job0]].kp;
        const int w = jobs_in[order[gd.job0]].waves;
        TileKernel kern = tile_kernel(jobs_in[order[gd.job0]].mode, kp.norm, kp.m);
        int occ = 0;
        const size_t lds = strip_lds_bytes(gd.capw);
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 64 * w, lds) != hipSuccess ||
            occ < 1)
            occ = 1;
        int grid = groups_req > 0 ? groups_req : ncu * occ;
        grid = std::min(grid, gd.items);
        // The first group runs on the launch stream; further groups fork.
        hipStream_t gs = st;
        if (fork && launched > 0) {
            const int k = (launched - 1) % aux->count;
            gs = aux->s[k];
            if (!used[k]) hipStreamWaitEvent(gs, aux->fork, 0);
            used[k] = true;
        }
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * w), lds, gs, ddesc, dgroups, g, dcounters);
        ++launched;
    }
    if (fork) {
        for (int k = 0; k < aux->count; ++k) {
            if (!used[k]) continue;
            hipEventRecord(aux->join[k], aux->s[k]);
            hipStreamWaitEvent(st, aux->join[k], 0);
        }
    }
    if (phases) hipEventRecord(phases->ev[2], st);
    if (stitch_blocks > 0)
        hipLaunchKernelGGL(k_stitch, dim3(stitch_blocks), dim3(kStitchThreads), 0, st, ddesc, njobs);
    launch_stats(ddesc, stat_grid, njobs, st);
    if (phases) hipEventRecord(phases->ev[3], st);
    return hipGetLastError() == hipSuccess ? RQA_OK : RQA_EDEVICE;
}

size_t engine_static_bytes(const Job &jb) {
    return engine_launch_scratch_bytes(1) + a256(kInfoBytes) + layout_of(jb).bytes;
}

static_assert(sizeof(JobDesc) <= 512, "counted in what rqa_run_static admits");
size_t engine_static_charge(const Job &jb) {
    return engine_launch_scratch_bytes(1) + a256(kInfoBytes) + engine_budget_bytes(jb);
}

int engine_launch_static(Job jb, void *scratch, hipStream_t st) {
    if (jb.waves < 1 || jb.waves > kMaxWaves || jb.mode != kModeAuto) return RQA_EINVAL;
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return RQA_EDEVICE;
    // [descriptors | groups | counters][statistics record][job scratch]
    char *base = static_cast<char *>(scratch);
    JobDesc *ddesc = reinterpret_cast<JobDesc *>(base);
    GroupDesc *dgroups = reinterpret_cast<GroupDesc *>(base + a256(sizeof(JobDesc)));
    int *dcounters = reinterpret_cast<int *>(base + a256(sizeof(JobDesc)) +
                                             a256(sizeof(GroupDesc) * 64));
    jb.stats = base + engine_launch_scratch_bytes(1);
    jb.scratch = base + engine_launch_scratch_bytes(1) + a256(kInfoBytes);
    const Layout lay = layout_of(jb);
    const JobDesc d = make_desc(jb, lay, 0, 0);
    const GroupDesc g{0, 1, lay.items, white_bins(jb.waves, lay.blocks, jb.hist_len())};
    hipLaunchKernelGGL(k_prepare_one, dim3(prepare_blocks_of(jb)), dim3(kPrepareThreads), 0, st, d, g,
                       ddesc, dgroups, dcounters);
    if (lay.items > 0) {
        TileKernel kern = tile_kernel(kModeAuto, jb.kp.norm, jb.kp.m);
        int occ = 0;
        const size_t lds = strip_lds_bytes(g.capw);
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 64 * jb.waves, lds) != hipSuccess ||
            occ < 1)
            occ = 1;
        const int grid = std::min(ncu * occ, lay.items);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * jb.waves), lds, st, ddesc, dgroups, 0,
                           dcounters);
    }
    hipLaunchKernelGGL(k_stitch, dim3(stitch_blocks_of(jb)), dim3(kStitchThreads), 0, st, ddesc, 1);
    launch_stats(ddesc, d.stat_blocks, 1, st);
    return hipGetLastError() == hipSuccess ? RQA_OK : RQA_EDEVICE;
}

// The last column tile's coordinates, then (256-byte aligned) the boxes.
int64_t engine_plot_tail_floats(const KParams &kp) {
    return (64 + (int64_t)(kp.m - 1) * kp.tau + 63) / 64 * 64;
}
static int64_t plot_box_entries(int64_t vecs) {   // whole groups of tiles
    return ((vecs + 63) / 64 + kGroup - 1) / kGroup * kGroup * (64 / kBoxVecs);
}
int64_t engine_plot_scratch_floats(const KParams &kp, int64_t n, int64_t nb, bool cross) {
    const int64_t entries = plot_box_entries(nb) + (cross ? plot_box_entries(n) : 0);
    return engine_plot_tail_floats(kp) + (kp.m <= kMaxM ? 2 * std::min(kp.m, kBoxK) * entries : 0);
}

int engine_plot(const KParams &kp, const float *a, int64_t na_points, const float *b,
                int64_t nb_points, uint64_t *bits, int64_t words, float *scratch, bool boxes,
                hipStream_t st) {
    const int64_t d = (int64_t)(kp.m - 1) * kp.tau;
    const bool cross = b != nullptr;
    const int64_t n = na_points - d, nb = cross ? nb_points - d : n;
    PlotDesc pd{};
    pd.a = a;
    pd.b = cross ? b : a;
    pd.tail = scratch;
    if (boxes && kp.m <= kMaxM) {
        pd.boxc = scratch + engine_plot_tail_floats(kp);
        pd.ncc = (int32_t)plot_box_entries(nb);
        pd.boxr = cross ? pd.boxc + (int64_t)2 * std::min(kp.m, kBoxK) * pd.ncc : pd.boxc;
        pd.ncr = cross ? (int32_t)plot_box_entries(n) : pd.ncc;
    }
    pd.bits = bits;
    pd.words = words;
    pd.nb_points = cross ? nb_points : na_points;
    pd.n = (int32_t)n;
    pd.nb = (int32_t)nb;
    pd.m = kp.m;
    pd.tau = kp.tau;
    pd.theiler = kp.theiler;
    pd.thr = kp.norm == RQA_NORM_L2 ? kp.eps_sq : kp.eps;
    pd.thr0 = kp.d0_bound;
    pd.row_tiles = (int32_t)((n + 63) / 64);
    pd.col_tiles = (int32_t)((nb + 63) / 64);
    pd.chunks = (pd.col_tiles + kPlotChunk - 1) / kPlotChunk;
    pd.xchunks = (pd.chunks + 7) / 8;
    pd.cross = cross ? 1 : 0;
    pd.tail_len = (int32_t)(64 + (int64_t)(kp.m - 1) * kp.tau);
    const int64_t entries = std::max<int64_t>((int64_t)std::min(kp.m, kBoxK) * (pd.ncc + pd.ncr), pd.tail_len);
    hipLaunchKernelGGL(k_plot_prepare, dim3((unsigned)std::min<int64_t>((entries + 255) / 256, 4096)),
                       dim3(256), 0, st, pd);
    // Without boxes: the kernel of any m, which classifies nothing (a test for them
    // in the others made the 65,516-point Lorenz plot 218 -> 222 us).
    const int m = pd.boxc ? kp.m : 0;
    PlotKernel kern = kp.norm == RQA_NORM_L1 ? pick_plot<RQA_NORM_L1>(m)
                      : kp.norm == RQA_NORM_L2 ? pick_plot<RQA_NORM_L2>(m)
                                               : pick_plot<RQA_NORM_LINF>(m);
    const int64_t xwaves = (int64_t)pd.row_tiles * pd.xchunks;   // waves per XCD
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * ((xwaves + 3) / 4))), dim3(256), 0, st, pd);
    return hipGetLastError() == hipSuccess ? RQA_OK : RQA_EDEVICE;
}

}  // namespace rqa
