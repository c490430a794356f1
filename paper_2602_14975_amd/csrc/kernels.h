// Launchers and argument blocks of the libnnp kernels (internal).
#pragma once

#include <cmath>
#include <string>
#include <vector>

#include "common.h"
#include "mp.h"

namespace nnp {

// Brackets one launch with HIP events when its site is enabled
// (nnp_timer_enable); otherwise costs one branch.
// With `by_launch`, the events are not recorded around the launch but handed
// to it (hipExtLaunchKernelGGL), which timestamps the kernel itself: the
// interval then excludes dispatch gaps and host-side delays.
struct ScopedTimer {
    const char* name;
    hipStream_t stream;
    hipEvent_t a = nullptr, b = nullptr;
    bool active = false;
    bool by_launch = false;
    ScopedTimer(const char* site, hipStream_t s, bool by_launch = false);
    ~ScopedTimer();
};

// Small tables from the host to the device as kernel arguments: one launch
// for up to 12 tables of 3,840 bytes together, larger ones by pageable
// copies.  Each pageable copy is a launch of its own behind host work: a
// fast-force evaluation of 192 atoms took 24.9 us with its three (16.6
// without: a single replica needs no tables), a list build of 12,288 atoms 225
// us with its nine and the sort behind two of them (174 with one launch here,
// the cell numbers formed on the device and one copy back; now 141).  Sources may go as
// soon as add() returned; flush() before the first use on the stream.
class Uploads {
public:
    explicit Uploads(hipStream_t s) : s_(s) {}
    // bytes: a multiple of 4; src = nullptr: zeros
    void add(void* dst, const void* src, size_t bytes);
    void flush();
    static constexpr int kPieces = 12, kWords = 960;
    struct Args {
        uint32_t* dst[kPieces];
        int end[kPieces];  // last word of each piece, plus one
        int pieces, words;
        uint32_t data[kWords];
    };

private:
    hipStream_t s_;
    Args a_{};
};

// ---------------------------------------------------------------- neighbours
// Cell numbering: the cell at lexicographic position l ((cx m + cy) m + cz)
// of replica r is number code[base_r + l]; lex is the inverse.  Within a
// replica the numbers follow the Morton (bit-interleaved) order of the
// cell coordinates, so consecutive cells, and the atoms the cell order
// puts together, form compact blocks of space.
struct CellPlan {
    std::vector<int> m;     // cells per side per replica (1 = whole replica)
    std::vector<int> base;  // first global cell of each replica
    int n_cells = 0;
};

// Where a cell-order build that succeeds leaves the permutation (order[2n]:
// row -> caller index, then caller index -> row) and the positions and species
// in row order.
struct RowOrder {
    const int* species_in = nullptr;
    int* order = nullptr;
    double* pos = nullptr;
    int* species = nullptr;
};

struct NbrScratch {
    int *grid_m, *grid_base, *cell_code, *cell_lex, *cell_of_atom, *slot_of_atom, *cell_count, *cell_start,
        *cell_atoms, *counts, *tmp_off, *status;
    int* hits;         // [n][kKeptEntries] entries of each row as the count found them (cell positions)
    double* cell_pos;  // [3][n] positions in cell order
};

CellPlan plan_cells(const nnp_system& sys, double radius);
int64_t max_cells(int64_t n_atoms, int32_t n_rep);
// Entries of a row that the fill takes as the count found them.
constexpr int kKeptEntries = 128;
// hits: take room for the kept entries too (else the caller gives it some that
// nothing else uses from a build's count to its fill)
void carve_nbr_scratch(Arena& a, int64_t n, int32_t n_rep, NbrScratch& s, bool hits);
// The plan's tables through `up` (flushed), then the cell numbers on the device
void upload_cell_plan(const CellPlan& plan, NbrScratch& s, Uploads& up, hipStream_t stream);
// cell_rows: rows and entries in the cell order of this list build (s.cell_atoms
// maps them to the caller's indices, s.cell_pos holds the positions in that
// order); each row still ascending in caller index.
void launch_build(int n, const double* pos, const RepGeom& geom, const CellPlan& plan, NbrScratch& s, const int* run,
                  double radius, int64_t capacity, int* offsets, int* nbr, int* rev, double* pos_ref,
                  hipStream_t stream, bool cell_rows = false,
                  const RowOrder& order = {});
// pos: the positions in the order of the input list's rows; key (or
// nullptr): caller's index of a row, for the reverse entries
// src_status (or nullptr): the input list's build status; a failed build
// leaves this list untouched
void launch_filter(int n, const double* pos, const RepGeom& geom, NbrScratch& s, const int* run, const int* off_in,
                   const int* nbr_in, double radius, int64_t capacity, int* offsets, int* nbr, int* rev, int* status,
                   hipStream_t stream, const int* key = nullptr, const int* src_status = nullptr);
// After a build into spare buffers that ran and succeeded (s.status): the
// spare list (and, with order_src, the order and row-ordered positions and
// species) copied over the ones in use.
void launch_adopt_lists(int n, const int* run, const NbrScratch& s, const int* off_src, const int* nbr_src,
                        int64_t capacity, int* off_dst, int* nbr_dst, const int* order_src, int* order_dst,
                        const double* pos_src, double* pos_dst, const int* sp_src, int* sp_dst, hipStream_t stream);
// pos_m / species_m (or nullptr) in row order from the caller's arrays
void launch_gather_rows(int n, const int* order, const double* pos, const int* species, double* pos_m,
                        int* species_m, hipStream_t stream);
// The identity order into order[2n], with pos_m and species_m copied.
void launch_reset_rows(int n, int* order, const double* pos, const int* species, double* pos_m, int* species_m,
                       hipStream_t stream);
void launch_set_flag(int* flag, int value, hipStream_t stream);
void launch_disp_check(int n, const double* pos, const double* ref, double thr, int* flag, hipStream_t stream);
// Ends a (possibly skipped) rebuild: counts it, clears the trigger and, with
// `maxd2`, restarts the displacement record ([0] since the build, [1] at the
// previous decision).
void launch_finish_rebuild(int* flag, long long* n_rebuilds, unsigned* maxd2, hipStream_t stream);
// Per-outer-step decision: set `flag` when the largest displacement since
// the last build, extrapolated over one more outer step from its growth
// during the previous one, may reach `thr`.
void launch_predict_rebuild(unsigned* maxd2, double thr, int* flag, hipStream_t stream);

// --------------------------------------------------------------------- GEMM
enum { EPI_NONE = 0, EPI_SILU = 1, EPI_DSILU = 2 };

struct GemmArgs {
    int M, N, K;
    const float* A;
    int64_t sam, sak;
    const float* B;
    int64_t sbk, sbn;
    float* C;
    int64_t ldc;
    const float* bias;
    int epi;
    float* pre;
    int64_t ldp;
    int accum;
    int64_t chunk_rows;    // > 0: split the K range into chunks along grid.z
    int64_t chunk_stride;  // C offset between chunks
    int bf16;              // operands rounded to bfloat16 (float32 accumulation)
    // B(k, n) = B[n * sbn + k] also as three bfloat16 pieces (hi, mid, lo;
    // hi + mid + lo = B to within 2^-24 relative), piece p at Bx + p * bxs,
    // same [N][K] layout; lets FP32 products run on bfloat16 matrix cores
    const uint16_t* Bx;
    int64_t bxs;
    // float32 register-direct kernel only: rows from b_split on multiply by
    // B2 instead of B (same layout)
    const float* B2;
    int64_t b_split;
    // split-bfloat16 kernel: row tiles from b_split on (a multiple of 128)
    // take the pieces at Bx2 instead of Bx
    const uint16_t* Bx2;
};

void launch_gemm(const GemmArgs& g, hipStream_t s);
void gemm_xwt(int M, int N, int K, const float* X, int ldx, const float* W, const float* b, float* out, int ldo,
              int epi, float* pre, int ldp, bool accum, hipStream_t s, bool bf16 = false,
              const uint16_t* Wx = nullptr, int64_t wx_stride = 0);
// out = X W^T with float32 operands on the matrix cores, rows m >= m_split
// taking W2 (same [N][K] layout) instead of W; m_split a multiple of 32,
// N <= 160, K and the strides multiples of 4.
// The same on the split-bfloat16 kernel (FP32-equivalent): pieces Wx and Wx2
// (piece stride wx_stride), m_split a multiple of 128; false (nothing
// launched) where the kernel cannot take the shapes or the float32 kernels
// are selected.
bool gemm_x3_split(int M, int N, int K, const float* X, int ldx, const uint16_t* Wx, const uint16_t* Wx2,
                   int64_t wx_stride, int m_split, float* out, int ldo, hipStream_t s);
void gemm_xwt_f32_split(int M, int N, int K, const float* X, int ldx, const float* W, const float* W2, int m_split,
                        float* out, int ldo, hipStream_t s);
// ------------------------------------------- per-atom blocks (width 128) --
// Matrices as operand fragments of the per-atom blocks (atom_block.hip).
struct PackFrags {
    static constexpr int kMax = 12;
    struct Mat {
        const float* src;  // [N][K] row-major, or [K][N] with tr
        uint16_t* dst;     // np pieces of N * K
        int N, K, tr;
    } m[kMax];
};
void launch_pack_frags(const PackFrags& P, int count, int np, hipStream_t s);
// Once per device before the first launch of a block.
void atom_block_setup();

// Forward block after a message step: update block, then the next layer's
// phi perceptron (last = false) or the readout with the energy's adjoint of
// s (last = true: W1 = Wo, b1 = bo, W2 = Wo transposed, s_out = the adjoint).
struct AtomFwd {
    int n;
    const float *smid, *vmid;
    const uint16_t *U, *M1, *M2, *W1, *W2;  // packed; U is [U; V]
    const float *m1, *m2, *b1, *b2;
    float *UV, *a1, *pqo, *s_out, *v_out, *h1, *phi, *pv;
    // first layer by species (FP32 models), or nullptr: packed T_0 and T_2;
    // smid and vmid are then the rows E and U, v_keep room for v
    const uint16_t *T0, *T2;
    float* v_keep;
    // last
    const float *wo, *beta;
    const int* species;
    int n_species;
    float* Ei;
    const int* perm;
};
void launch_atom_fwd(const AtomFwd& a, bool last, bool bf16, hipStream_t s);
// Reverse block before a message step's reverse: with top = false the next
// layer's phi adjoint first (gphi, h1, W2t, W1t), then the update block's.
// UV, pqo, a1 and h1 in the order the forward block left them (rows padded to
// a multiple of 32); packed matrices transposed.
struct AtomBwd {
    int n;
    const float *gs_in, *gv_in, *gphi, *h1, *UV, *pqo, *a1;
    const uint16_t *W2t, *W1t, *M2t, *M1t, *Ut, *Vt;
    float *gs_out, *gv_out;
    // first layer by species (FP32 models), or nullptr: packed transposes of
    // T_0 and T_2 (pp rows); P0 and P2 (rows of 128) are written instead of
    // gs_out and gv_out, keep is room for the former ([tile rows][3][F])
    const uint16_t *TT0, *TT2;
    int pp;
    float *P0, *P2, *keep;
};
void launch_atom_bwd(const AtomBwd& a, bool top, bool bf16, hipStream_t s);
// Whether the matrix-core dense kernels are selected (nnp_set_dense_kernels).
bool dense_auto();

// dst[p * piece_stride + e] = piece p (hi, mid, lo) of src[e] as bfloat16
void launch_split3(const float* src, int64_t count, uint16_t* dst, int64_t piece_stride, hipStream_t s);
// 0: FP32 products on split-bfloat16 matrix cores where the shapes allow
// (default); 1: float32-operand kernels only
void set_dense_mode(int mode);
// dst[c][r] = src[r][c] for a rows x cols row-major matrix
void launch_transpose(int rows, int cols, const float* src, float* dst, hipStream_t s);
void gemm_gw(int M, int N, int K, const float* G, int ldg, const float* W, float* out, int ldo, int epi,
             const float* pre, int ldp, bool accum, hipStream_t s, bool bf16 = false);
void gemm_wgrad(int M, int N, int K, const float* G, int ldg, const float* X, int ldx, float* dW, float* scratch,
                int chunk, bool accum, hipStream_t s);
void colsum(int M, int N, const float* G, int ldg, float* db, float* scratch, int chunk, bool accum, hipStream_t s);

// ------------------------------------------------------------ edge kernels
// argument blocks: mp.h
int mp_blocks(int n, int F);
// matrix-core message kernels (F = 128, K = 16, cosine cutoff; forces, no weight adjoints)
bool message_mx_shape(int F, int K, int cut);
// What nnp_set_message_kernels leaves an evaluation of this shape and of n
// atoms: the matrix-core message kernels, and the first layer by neighbour
// species with them.  Read once per evaluation.
struct MessageRoute {
    bool matrix_cores, species_sum;
};
MessageRoute message_route(int F, int K, int cut, int64_t n);
// With Es, also the first conservative layer's edge sums by neighbour species
// (rows Es [n][ep], Ev [3n][ep]; S species, S <= 8; mp_species.hip).
void launch_edge_prep(const MpGeom& mg, int* ecnt, EdgeRec* erec, uint4* ehalf, hipStream_t s, float* Es = nullptr,
                      float* Ev = nullptr, int S = 0, int ep = 0);
// First layer of the conservative message step summed by neighbour species
// (mp_species.hip): row pitches (pp of the per-atom tables P, a multiple of
// 32; ep of the edge sums, 128 or 256), shapes covered, the weight tables
// T [2][F][ep] and TT [2][pp][F] (refreshed with the weights; the forward
// edge sums come from launch_edge_prep) and the reverse edge kernel from
// P0 [n][pp], P2 [3n][pp].
void species_sum_pitches(int n_species, int& pp, int& ep);
bool species_sum_shape(int F, int K, int cut, int n_species);
void launch_sp_tables(int F, int S, const float* Wr, const float* br, const float* phi, const float* emb, float* T,
                      float* TT, hipStream_t s);
void launch_sp_bwd(const MpGeom& mg, int S, const float* P0, const float* P2, float* force, bool accum, float* vir,
                   hipStream_t s);
// The first layer's share of edge_f (see launch_edge_force), written or added
void launch_sp_bwd_own(const MpGeom& mg, int S, int pitch, const float* P0, const float* P2, float* edge_f, bool add,
                       hipStream_t s);
void launch_message_fwd_mx(const MpGeom& mg, const MpFwd& a, hipStream_t s, const ScopedTimer& t);
void launch_message_bwd_mx(const MpGeom& mg, const MpBwd& a, hipStream_t s, const ScopedTimer& t);
void launch_filter_scale(int count, const float* Wr, float* out, hipStream_t s);
// Filter operands of one layer in the order the matrix-core message kernels
// read them (filter_operand_units() units of 16 bytes), after its scale.
int64_t filter_operand_units();
void launch_filter_operands(const float* Wr, const float* br, const float* scale, uint4* out, hipStream_t s);
void launch_message_fwd(int F, int K, int cut, const MpGeom& mg, const MpFwd& a, hipStream_t s);
void launch_message_bwd(int F, int K, int cut, const MpGeom& mg, const MpBwd& a, bool geo, bool wgrad,
                        hipStream_t s);

// ----------------------------------------------------------- block kernels
void launch_embed(int n, int F, int S, const int* species, const float* emb, float* s, float* v, hipStream_t st);
void launch_build_x(int n, int F, const float* smid, const float* UV, float* X, hipStream_t st);
void launch_update_combine(int n, int F, const float* smid, const float* vmid, const float* UV, const float* pqo,
                           float* s_out, float* v_out, hipStream_t st);
void launch_update_combine_bwd(int n, int F, const float* UV, const float* pqo, const float* gs, const float* gv,
                               float* gpqo, float* gUV, hipStream_t st);
void launch_norm_bwd(int n, int F, const float* gs, const float* gX, const float* X, const float* UV, float* gsmid,
                     float* gUV, hipStream_t st);
// perm (or nullptr): E_i of row i stored at Ei[perm[i]]
void launch_readout(int n, int F, int S, const float* z, const float* wo, const float* beta, const int* species, float* Ei,
                    hipStream_t st, const int* perm = nullptr);
void launch_readout_bwd(int n, int F, const float* ao, const float* wo, float* gao, hipStream_t st);
// out[r] = sum of x over the atoms of replica r (rep_start is not read for a
// single replica, of n atoms)
struct RepSum {
    int n_rep = 0;
    const int64_t* rep_start = nullptr;
    int64_t n = 0;
    const float* x = nullptr;
    double* out = nullptr;
};
void launch_rep_sum(const RepSum& a, hipStream_t st);
// The same by the 256 threads of one block, in a fixed order.
__device__ __forceinline__ void rep_sum_block(const RepSum& q, int r, double* red) {
    const int64_t a0 = q.n_rep > 1 ? q.rep_start[r] : 0, a1 = q.n_rep > 1 ? q.rep_start[r + 1] : q.n;
    double s = 0.0;
    int64_t a = a0 + threadIdx.x;
    // eight loads in flight, added in the same order as one at a time
    for (; a + 7 * 256 < a1; a += 8 * 256) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = q.x[a + k * 256];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += double(v[k]);
    }
    for (; a < a1; a += 256) s += double(q.x[a]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) q.out[r] = red[0];
}
// Forces (and virial shares) from the feature sums of the edges' messages; in
// the same launch also the per-replica sums `rs` (the energies).
void launch_edge_force(const MpGeom& mg, const float* edge_f, float* force, float* vir, const RepSum& rs,
                       hipStream_t s);
// scratch: cdiv(n, chunk) x S x F floats
void launch_emb_grad(int n, int F, int S, const int* species, const float* gs0, float* gemb, float* scratch, int chunk,
                     hipStream_t st);
void launch_reduce_chunks(int64_t count, int nchunks, const float* part, int64_t stride, float* out, bool accum,
                          hipStream_t s);
// vir_set / vir_add ([n] or nullptr): per owner i, sum_j F_ij . r_ij (its
// share of the NPT virial proxy), written / added to
void launch_head_fwd_rec(const MpGeom& mg, const int* cnt, const NcEdge* rec, const float* QK, const float* Vh,
                         float* F, bool accum, hipStream_t st, float* vir_set, float* vir_add);
void launch_head_fwd(const MpGeom& mg, const float* QK, const float* Vh, float* F, bool accum, hipStream_t st,
                     float* vir_set = nullptr, float* vir_add = nullptr);
void launch_head_bwd(const MpGeom& mg, const float* QK, const float* Vh, const float* gF, float* gQK, float* gVh,
                     hipStream_t st);

// Embedding of NC models of width 8, 16 or 32: message step, update block and
// q/k/V projections in one kernel (nc_embed.hip).
struct NcEmbedArgs {
    const float *Wr, *br, *phi_tab, *emb;  // filter, phi per species [S][3F], embedding [S][F]
    const float *wt, *m1, *m2;             // packed weights (nc_pack_weights), biases
    NcEdge* edge_out;                      // or nullptr: edge records at the owner's list positions
    int* edge_cnt;                         // or nullptr: edges per atom
    float *QK, *Vh;                        // [n][2 H n_c], [n][3][n_l]
};
void launch_nc_embed(const MpGeom& mg, const NcEmbedArgs& a, int F, bool bf16, hipStream_t s);
// U|V, M1, M2, W_qk and W_V as its matrix operands (rounded to bfloat16 when
// bf16); nc_pack_count(F) floats
void nc_pack_weights(int F, const float* UV, const float* M1, const float* M2, const float* Wqk, const float* WV,
                     bool bf16, float* out, hipStream_t s);
int64_t nc_pack_count(int F);

// -------------------------------------------------------------- integrator
struct BaoaArgs {
    int n;
    double* pos;
    double* vel;
    const double* mass;
    const double* gamma;
    const float* force;
    double dt;
    double temperature;
    const int32_t* rep_of_atom;
    const int64_t* rep_start;
    const uint64_t* seed;
    const uint64_t* stream;
    const uint64_t* step_base;
    uint64_t step_offset;
    const uint64_t* step_dev;  // optional device O-step counter added to step_offset
    int ffl;
    const double* pos_ref;
    double disp_thr2;
    int* flag;         // set when an atom moved more than sqrt(disp_thr2) since the last build
    unsigned* maxd2;   // optional: running maximum of the squared displacement (float bits)
    // 1: the opening kick is B(dt) instead of B(dt/2), standing for the
    // closing B(dt/2) of the previous step with the same force as well
    int full_kick;
    // optional: the new positions also into pos_rows[c * n + row[i]] (the
    // force evaluations' copy in their working row order)
    double* pos_rows;
    const int* row;
};

// v += half_dt * ACC * (Fa - Fb) / m; with `bump`, also advances that O-step
// counter by bump_by (read by the next k_baoa)
void launch_kick(int n, double* vel, const double* mass, const float* Fa, const float* Fb, double half_dt,
                 hipStream_t s, uint64_t* bump = nullptr, uint64_t bump_by = 1);
void launch_set_u64(uint64_t* p, uint64_t value, hipStream_t s);
void launch_disp_record(int n, const double* pos, const double* pos_ref, unsigned* maxd2, hipStream_t s);
// device wall-clock ticks (hipDeviceAttributeWallClockRate) written once the stream reaches it
void launch_stamp(uint64_t* out, hipStream_t s);
// zero fill as a kernel (safe inside recorded graphs); with `run`, only when *run != 0
void launch_zero(void* p, int64_t words, const int* run, hipStream_t s);
void launch_virial_combine(int n, const float* wc, const float* wl, const float* ws, float inv_n, float* out,
                           hipStream_t s);
void launch_add(int n, const float* x, float* y, hipStream_t s);  // y += x
bool timers_active();
void launch_baoa(const BaoaArgs& a, hipStream_t s);
// stochastic cell rescaling (pressures in kcal/mol/A^3, beta in their inverse)
struct ScrArgs {
    double p0, beta, tau, dt, temperature;
    uint64_t seed, stream, step;
};
void launch_scr(int n_rep, const double* ke, const double* virial, double* box, double* mu, const ScrArgs& a,
                hipStream_t s);
void launch_scale(int n, const int32_t* rep_of_atom, const double* mu, double* pos, double* vel, hipStream_t s);
// atoms per block of the chunked kinetic-energy reduction; part: scratch of
// n_rep * chunks doubles, chunks = the largest replica's atom count over
// kKeChunk, rounded up (without it, one block per replica)
constexpr int kKeChunk = 2048;
void launch_kinetic(int n_rep, const int64_t* rep_start, int n, const double* pos, const double* vel,
                    const double* mass, double* ke, int* bad, hipStream_t s,
                    const int32_t* rep_of_atom = nullptr, double* part = nullptr, int chunks = 0);

}  // namespace nnp
