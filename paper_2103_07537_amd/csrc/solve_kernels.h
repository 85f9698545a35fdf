// Solve-phase views and launchers (device work in solve_kernels.hip).
#pragma once

#include "common.h"

namespace mbamg {

// Rows of one block on one level, in smoother colour order, cut into slices
// of at most 64 rows that never straddle two colours.
struct SliceView {
    const int32_t* row0;
    const int32_t* nrow;
};

// One matrix part in masked sliced-ELL form.  Slice s has width[s] slots; slot
// t of slice s is global slot coff[s]+t, with a column per lane in
// col[slot*64 + lane] (-1 marks padding) and a bit mask of the block entries
// stored for every lane of the slot.  The values of the slot's set bits follow
// each other as groups of 64 (one per lane) starting at group voff[slot].
constexpr int COL16_NONE = 0xFFFF;   // a padding lane's 16-bit column
template <class T>
struct SellView {
    const int32_t* width;
    const int64_t* coff;
    const int64_t* voff;       // per slot
    const uint32_t* mask;
    const int32_t* col;        // or, where not NULL, 16-bit columns relative to the slot's cbase (0xFFFF: none)
    const uint16_t* col16;
    const int32_t* cbase;
    const T* val;
};

// What every block of a level's four matrix blocks has in common.  Vector fields
// whose components are coupled alike (a vector Laplacian, a component-wise
// coupling) have blocks whose leading (D-1) x (D-1) part is a multiple of the
// identity; where the last column also equals the last row (a gradient and its
// divergence, coarsened with equal transfers) it need not be stored twice.
//   SHAPE_FULL       any block: all D x D entries
//   SHAPE_SCALED     s I in the leading part: s, the last column, the last row, the last entry
//   SHAPE_SYMMETRIC  that, last column = last row: s, the last column, the last entry
// Entries that are zero in a whole slot are left out under every shape.
constexpr int SHAPE_FULL = 0, SHAPE_SCALED = 1, SHAPE_SYMMETRIC = 2;
// waves per slice that the sliced kernels are instantiated for, beyond SHAPE_FULL
constexpr int SHAPE_MAX_SPLIT = 2;

template <class T>
struct GsArgs {
    int shape;
    int s_begin, s_count;      // slices of this colour
    SliceView sl;
    SellView<T> off, cpl, dinv;
    const T* b;                // right-hand side of this block
    const T* x;                // current iterate of this block (unused when starting from zero)
    T* t;                      // undamped Gauss-Seidel iterate x + e
    T* xn;                     // damped result x + omega e
    const T* xg;               // iterate of the other block for the coupling term
    int cstart;                // rows below this index already carry this sweep's update
    T omega;
    const T* w_row;            // per-row damping (NULL: use omega)
    int skip_off;              // nothing processed yet and zero start: the A_ff term vanishes
    int keep_t;                // t is read by a later launch
};

// One colour of the nodal-block Gauss-Seidel over the full node blocks (both
// blocks' rows of a node relaxed together): the two blocks share one colour
// order and slicing; the node inverses are ((d0+d1) x (d0+d1)), masked per
// slice: the entries k set in dmask[s] stored as groups of 64 values (one per
// lane) from group doff[s].
template <class T>
struct GsFcArgs {
    int s_begin, s_count;
    SliceView sl;
    SellView<T> off[2], cpl[2];    // A_ff without its diagonal block; A_fg with it (skipped)
    const T* dinv;
    const uint64_t* dmask;
    const int32_t* doff;
    const T* b[2];
    const T* x[2];                 // current iterates (unused when starting from zero)
    T* t[2];                       // undamped iterates x + e
    T* xn[2];                      // damped results x + omega e
    int cstart;                    // rows below this index already carry this sweep's update
    T omega;
    const T* w_row;                // per-row damping (NULL: use omega)
    int skip_off;                  // nothing processed yet and zero start: the sums vanish
};

// A block row in row form: each row's blocks contiguous (row-major br x bc)
// with columns in the column block's colour order.
template <class T>
struct RowView {
    const int32_t* rp;         // rows + 1
    const int32_t* col;
    const T* val;
};

// One slice of a grouped block row as the sweep and the grouped residual read
// it: its rows, the first row of its colour, and its slots in the two parts.
struct SweepRec {
    int32_t row0, nrow;        // nrow == 0: a launch position with nothing to do
    int32_t cstart;            // first row of the slice's colour
    int32_t off_w, off_c;      // A_ff without its diagonal: slots, first slot
    int32_t cpl_w, cpl_c;      // A_fg: the same (two-block systems)
    int32_t slice;
};

// Slots of a grouped part (see k_sweep): like SellView, but a slice has 64 / G
// rows and G consecutive lanes hold G blocks of one row.
template <class T>
struct GroupView {
    const int64_t* voff;       // per slot
    const uint32_t* mask;
    const int32_t* col;
    const T* val;
};

// One block row's share of a sweep launch in grouped form: the launch positions
// [begin, begin + count) of its record list (whole colours, ascending).
template <class T>
struct SweepArgs {
    const SweepRec* rec;
    int begin, count;
    int lg;                    // log2 of the lanes per row
    GroupView<T> off;
    const T* dinv;             // d x d per row, colour order
    const T* b;
    const T* x;                // current iterate (unused when starting from zero)
    T* t;                      // undamped iterate x + e: written, and awaited for earlier colours
    T* t_reset;                // the other undamped buffer: this launch's rows are set to "not yet written" (NULL: no)
    T* xn;                     // damped result x + omega e
    int inplace;               // a further inner sweep: every neighbour's value comes from t
    T omega;
    const T* w_row;            // per-row damping (NULL: use omega)
};

// The vector a coupling block multiplies: x (t NULL), or the damped result of a
// block relaxed in the same launch, x + omega (t - x) (x NULL: omega t), with t
// awaited.
template <class T>
struct SweepOperand {
    const T* x;
    const T* t;
    const T* w_row;
    T omega;
};

// A wait ends after this many rounds even if the value never comes, with the pauses
// between them about a second.  The launch then finishes, with NaN results, and says
// so in *late (page-locked host memory).
constexpr int SWEEP_MAX_ROUNDS = 1 << 15;
struct SweepWait {
    int rounds;
    uint32_t* late;
};

// Algorithm 1 over two blocks of one size: block 0's positions, then block 1's; or
// one block alone, in the first places (the second count is zero then).
template <class T>
struct Sweep2Args {
    int shape;
    int spread;                // few workgroups per colour: one per compute unit
    SweepArgs<T> s[2];
    GroupView<T> cpl[2];
    SweepOperand<T> xg[2];     // x and t NULL: no coupling term; t: launches of both blocks only
    uint32_t* ticket;          // zero at launch
    uint32_t* ticket_next;     // set to zero for the next launch
    SweepWait wait;
};

// More than two blocks: one coupling block A_fg (any shape up to 4 x 4) in
// grouped form on block f's slices, and the vector it multiplies.
constexpr int SWEEP_MAX_BLOCKS = 4;
struct GroupPart {
    GroupView<double> a;
    const int32_t* width;      // per slice
    const int64_t* coff;       // per slice
    const double* x;
    int bc;
};
struct SweepNArgs {
    SweepArgs<double> s;
    int spread;
    int n_cpl;
    GroupPart cpl[SWEEP_MAX_BLOCKS - 1];
    uint32_t* ticket;
    uint32_t* ticket_next;
    SweepWait wait;
};
// r_f = b_f - sum_g A_fg x_g (b NULL: w_f = sum_g A_fg x_g) for every block f
struct ResidNArgs {
    int nb;
    int count[SWEEP_MAX_BLOCKS];           // launch positions of block f
    const SweepRec* rec[SWEEP_MAX_BLOCKS];
    int lg[SWEEP_MAX_BLOCKS], d[SWEEP_MAX_BLOCKS];
    GroupView<double> off[SWEEP_MAX_BLOCKS];
    const double* diag[SWEEP_MAX_BLOCKS];
    int n_cpl[SWEEP_MAX_BLOCKS];
    GroupPart cpl[SWEEP_MAX_BLOCKS][SWEEP_MAX_BLOCKS - 1];
    const double* b[SWEEP_MAX_BLOCKS];
    const double* x[SWEEP_MAX_BLOCKS];
    double* r[SWEEP_MAX_BLOCKS];
};

template <class T, class TX = T>   // TX: the type x is stored in
struct ResidGroupArgs {
    int shape;
    const SweepRec* rec[2];
    int count[2];
    int lg[2];
    GroupView<T> off[2], cpl[2];
    const T* diag[2];          // d x d per row, colour order
    const T* b[2];             // NULL for a plain operator apply
    const TX* x[2];
    T* r[2];
};

template <class T, class TX = T>
struct ResidArgs {
    int shape;
    int s_count[2];
    SliceView sl[2];
    SellView<T> off[2], cpl[2], diag[2];
    const T* b[2];             // NULL for a plain operator apply
    const TX* x[2];
    T* r[2];
    const int32_t* order[2];   // slice of each launch position (NULL: the position itself)
};

template <class T>
struct TransferArgs {
    int n_rows[2];             // fine rows (prolongation) or coarse rows (restriction) per block
    const int32_t* map[2];     // prolongation: coarse row of each fine row; restriction: member pointer
    const int32_t* idx[2];     // restriction: member rows
    // Weight of P per fine row (prolongation) or per member, in member-list order
    // (restriction).  The transfers start from the constant in every component, so a row's
    // components have one weight; reading it once (8 or 4 bytes) instead of per component
    // took a V-cycle of 128^3 nodes from 1904 to 1874 us.
    const T* q[2];
    const T* in[2];
    T* out[2];
    // restriction: the coarse row each group of lanes takes, in launch order (NULL: row i for
    // group i); the next level's natural order keeps neighbouring aggregates, whose members
    // share the fine rows' cache lines, in neighbouring groups
    const int32_t* order[2];
};

// P: waves per slice (1, 2 or 4); the slice's slots are split among them.
template <class T>
struct XferArgs {
    int s_count[2];
    SliceView sl[2];
    SellView<T> A[2];
    const T* x[2];
    T* y[2];
    int accumulate;
    const int32_t* out_row[2];   // row of y each slice row writes (NULL: the slice row itself)
};

// P waves share each slice's slots (1, 2 or 4)
template <class T>
void launch_xfer(int d, int P, const XferArgs<T>& a, hipStream_t s);

// A transfer in row form: one wavefront per row of P or P^T (rows of block 0,
// then block 1), for few wide rows.
template <class T>
struct XferRowArgs {
    int n[2];
    RowView<T> A[2];
    const T* x[2];
    T* y[2];
    int accumulate;
    const int32_t* out_row[2];   // row of y each matrix row writes (NULL: the row itself)
};
template <class T>
void launch_xfer_rows(int d, const XferRowArgs<T>& a, hipStream_t s);
template <class T>
void launch_gs(int d, int P, bool zero_x, bool has_cpl, const GsArgs<T>& a, hipStream_t s);
template <class T, class TX>
void launch_resid(int d, int P, const ResidArgs<T, TX>& a, hipStream_t s);
template <class T>
void launch_gs_fc(int d, int P, bool zero_x, const GsFcArgs<T>& a, hipStream_t s);
// positions of a record list are taken this many at a time: every colour's are padded to a multiple
constexpr int SWEEP_WAVES = 8;
template <class T>
void launch_sweep(int d, bool zero_x, const Sweep2Args<T>& a, hipStream_t s);
template <class T, class TX>
void launch_resid_group(int d, const ResidGroupArgs<T, TX>& a, hipStream_t s);
void launch_sweep_n(int d, bool zero_x, const SweepNArgs& a, hipStream_t s);
void launch_resid_n(const ResidNArgs& a, hipStream_t s);

template <class T>
// G: lanes per coarse row (4, 8, 16 or 64)
void launch_restrict(int d, const TransferArgs<T>& a, int G, hipStream_t s);
template <class T>
void launch_prolong(int d, const TransferArgs<T>& a, hipStream_t s);
template <class T>
void launch_coarse(int n, const double* inv, const T* x, T* y, hipStream_t s);

// Krylov helpers (FP64).  Reductions are deterministic: per-block partial sums
// stored slot-major (partial[q * KBLOCKS + block]), summed in a fixed order by the
// block that finishes last.  Every launch uses the same number of blocks.
constexpr int KMAXQ = 33;        // basis vectors + 2 slots (a dot with the candidate, a norm)
constexpr int KBLOCKS = 1024;
// layout of the coefficient buffer of the delayed-reorthogonalisation update:
// [0, KMAXQ) a (reorthogonalisation coefficients of the candidate),
// [KMAXQ, 2 KMAXQ) b (projections of the new vector), then 1/nu and c_j
constexpr int KC_A = 0, KC_B = KMAXQ, KC_INV_NU = 2 * KMAXQ, KC_CJ = 2 * KMAXQ + 1, KC_TOTAL = 2 * KMAXQ + 2;
// counters of finished blocks, each in a cache line of its own
constexpr int KCOUNTERS = 16, KCOUNTER_STRIDE = 32, KCOUNTER_WORDS = (1 + KCOUNTERS) * KCOUNTER_STRIDE;
struct KrylovBufs {
    double* partial;             // KBLOCKS * KMAXQ, "unwritten" at launch
    double* partial_next;        // the other set, made so for the next launch:
    int n_next;                  // the sums it holds (at most KMAXQ)
    uint32_t* counter;           // KCOUNTER_WORDS, zero between launches
    double* coef;                // KC_TOTAL, device
    // results (page-locked host memory the device writes, read after the stream is waited for)
    double* d1;                  // dot pass: V_q . w
    double* d2;                  // update pass: the next candidate's a'
    double* nu;                  // update pass: its nu'
    double* nu2;                 // norm: w . w
    SweepWait wait;
};
void launch_norm2(int64_t n, const double* w, const KrylovBufs& kb, hipStream_t s);
void launch_orth(int64_t n, int nq, const double* V, int64_t ldv, const double* w, const KrylovBufs& kb,
                 hipStream_t s);
// One pass of the delayed reorthogonalisation step (see the kernel)
void launch_dcgs_update(int64_t n, int nq, const double* V, int64_t ldv, double* u, const double* w, double* out,
                        float* out32, const KrylovBufs& kb, hipStream_t s);
void launch_combine(int64_t n, int k, const double* Z, int64_t ldz, const double* y, double* x, hipStream_t s);
void launch_combine32(int64_t n, int k, const float* Z, int64_t ldz, const double* y, double* x, hipStream_t s);
void launch_axpby(int64_t n, double a, const double* x, double b, double* y, hipStream_t s);
void launch_seeded(int64_t n, uint64_t seed, double* v, hipStream_t s);
int krylov_blocks(int64_t n);
// all blocks of a vector between the interface's (natural) order and the colour order
struct ReorderArgs {
    int nb;
    int n[SWEEP_MAX_BLOCKS], d[SWEEP_MAX_BLOCKS];
    int64_t off[SWEEP_MAX_BLOCKS];               // first entry of each block
    const int32_t* iperm[SWEEP_MAX_BLOCKS];      // colour position of every natural row
    int blocks[SWEEP_MAX_BLOCKS];                // (set by the launcher)
};
void launch_reorder(bool to_colour, ReorderArgs a, const double* src, double* dst, hipStream_t s);
void launch_cast64to32(int64_t n, const double* a, float* b, hipStream_t s);
void launch_cast32to64(int64_t n, const float* a, double* b, hipStream_t s);

}  // namespace mbamg
