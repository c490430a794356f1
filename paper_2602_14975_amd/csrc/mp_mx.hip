// Matrix-core message kernels for width-128 embeddings with 16 Bessel
// functions and the cosine cutoff (the message step and its reverse), and
// the edge preparation they share.
//
// The radial filter of a batch of edges is a product of the per-edge basis
// (edges x K) with the filter weights (K x 3F).  It runs on the FP16 matrix
// cores at FP32-equivalent precision: each FP32 operand x is split into
// x_hi = fp16(x) and x_lo = fp16(x - x_hi), which together carry 22
// significant bits, and the products lo*hi, hi*lo and hi*hi are accumulated
// in FP32 (lo*lo lies below FP32 rounding).  The weights enter scaled by a
// power of two that puts their largest magnitude in [2^13, 2^14), inside the
// FP16 range whatever the model; every sum that is linear in the filter is
// rescaled once per atom, which is exact.
//
// Edge preparation (once per force evaluation, shared by the three layers'
// forward and reverse launches): one wavefront per atom applies the float64
// pair rule at the model cutoff to the atom's list row, compacts the edges
// that pass in list order to the front of the row, and stores per edge a
// record (neighbour, species, f, f', unit vector, 1/r) and the radial values
// e_k(r) f(r) and their r-derivatives (float32) already split into FP16
// pairs.
//
// Message kernels: blocks take one or two atoms in turn with four wavefronts,
// one per block of 32 features, which share the staged edges.  The reverse by
// both messages of a pair (BF16 models; FP32 ones: one message of each edge,
// below) is bound by its vector arithmetic (34 operations per edge and
// feature, 59 % of its time at 12,288 atoms) and by the rows it gathers
// through L1 (9 loads per edge and feature, about half of it), the forward by
// the gathers; what remains is the chain product -> gather -> sums of a batch
// with three wavefronts per SIMD (forward: four) to hide it.  Held out of that chain: the filter operands
// (laid out with the weights, in LDS during the kernel), the list rows of the
// block's atoms (in registers), the sums over lanes (no LDS).  At 12,288 atoms
// these took the forward from 155 to 137 us (now 125) and the reverse from 255
// to 246, at 1,536 atoms, with fewer atoms to a block, from 31 to 21 (now 18.5)
// and from 48 to 32.  An atom's edges are
// consumed in batches of fixed size (32 forward, 16 reverse) in list order,
// so the batch an edge falls into depends only on its rank among the atom's
// edges within the cutoff: results do not depend on the list radius.
//
// In a 32x32x16 product the lane (c, h) = (lane % 32, lane / 32) holds output
// column c for rows 8j + 4h + i (j, i = 0..3): every lane owns one feature and
// accumulates over a fixed subset of each batch's edges; the two halves of the
// wavefront are added at the end of the atom.  Forward: the rows are 32 edges.
// Reverse: rows 0..15 hold e_k(r) f(r) and rows 16..31 their r-derivatives
// for the same 16 edges, so one product gives w and dw/dr of an edge in the
// same lane.  The per-edge work after the filter is that of the vector
// kernels (same formulas; see the message kernels of mp.hip).
#include <hip/hip_ext.h>

#include "common.h"
#include "kernels.h"
#include "mp_edge.h"
#include "mp_rows.h"

namespace nnp {

namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));

constexpr int kMxF = kRowFeatures, kMxK = 16, kMxWaves = 4, kMxAtoms = 2;
// forward: edges of a lane in a group of loads, two groups in flight (40
// loads per lane, within four wavefronts per SIMD)
constexpr int kFwdGroup = 4;
// reverse: small groups keep every variant within three
// wavefronts per SIMD (measured: more gathers in flight per wavefront at
// two wavefronts per SIMD are 7 % slower than fewer at three)
template <bool L0>
constexpr int kBwdGroup = L0 ? 4 : 2;

__device__ __forceinline__ void split8(const float* x, half8_t& hi, half8_t& lo) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const _Float16 t = static_cast<_Float16>(x[q]);
        hi[q] = t;
        lo[q] = static_cast<_Float16>(x[q] - static_cast<float>(t));
    }
}

// The bias product (rows ab, bias operand bb), then A (32 x 16) times
// B (16 x 32) from the split operands, small terms first
template <bool BIAS = true>
__device__ __forceinline__ floatx16_t mma3(const half4_t& ab, const half4_t& bb, const half8_t& ah,
                                           const half8_t& al, const half8_t& bh, const half8_t& bl) {
    floatx16_t c = {};
    if constexpr (BIAS) c = __builtin_amdgcn_mfma_f32_32x32x8f16(ab, bb, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, c, 0, 0, 0);
    return c;
}

// A lane's filter operands: of each channel the B fragments (rows 8h..8h+7 of
// column f of the scaled filter weights, split) and the bias operand (a
// 32x32x8 product: rows 0..2 of column f hold (b_hi, b_hi, b_lo) of the
// scaled bias, the other rows zero, so that with A rows (c_hi, c_lo, c_hi,
// 0, ...) of a per-edge factor c one product gives c b at FP32-equivalent
// precision).  They are functions of the weights: k_filter_operands lays
// them out once per weight change as pieces bh[0..2], bl[0..2], then bb[0],
// bb[1] and bb[2] (8 bytes each) in pieces 6 and 7, [wavefront][piece][lane]
// of 16 bytes, the order in which the kernels read them (into registers, or
// into LDS as they are).
constexpr int kFiltPieces = 8;

__device__ __forceinline__ half8_t as_half8(const uint4& u) { return __builtin_bit_cast(half8_t, u); }

__device__ __forceinline__ void load_channel(const uint4* fl, int p, half8_t& bh, half8_t& bl, half4_t& bb) {
    bh = as_half8(fl[p * 64]);
    bl = as_half8(fl[(3 + p) * 64]);
    const uint4 q = fl[(6 + p / 2) * 64];
    bb = __builtin_bit_cast(half4_t, p % 2 == 0 ? make_uint2(q.x, q.y) : make_uint2(q.z, q.w));
}

// one thread per lane of the message kernels' four wavefronts
__global__ void __launch_bounds__(64 * kMxWaves) k_filter_operands(const float* Wr, const float* br,
                                                                   const float* scale, uint4* out) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int h = lane >> 5, f = w * 32 + (lane & 31);
    const float sc = scale[0];
    uint4* fl = out + w * kFiltPieces * 64 + lane;
    uint2 bias[3];
    for (int p = 0; p < 3; ++p) {
        float x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = Wr[(p * kMxF + f) * kMxK + 8 * h + q] * sc;
        half8_t hi, lo;
        split8(x, hi, lo);
        fl[p * 64] = __builtin_bit_cast(uint4, hi);
        fl[(3 + p) * 64] = __builtin_bit_cast(uint4, lo);
        const float b = br[p * kMxF + f] * sc;
        const _Float16 b_hi = static_cast<_Float16>(b);
        const _Float16 b_lo = static_cast<_Float16>(b - static_cast<float>(b_hi));
        half4_t bb{};
        if (h == 0) {
            bb[0] = b_hi;
            bb[1] = b_hi;
            bb[2] = b_lo;
        }
        bias[p] = __builtin_bit_cast(uint2, bb);
    }
    fl[6 * 64] = make_uint4(bias[0].x, bias[0].y, bias[1].x, bias[1].y);
    fl[7 * 64] = make_uint4(bias[2].x, bias[2].y, 0u, 0u);
}

// The A operand of the bias product for a row whose per-edge factor is c
// (the cutoff f or its derivative): (c_hi, c_lo, c_hi, 0, ...) in the lanes
// of the first half, zero in the second.
__device__ __forceinline__ half4_t bias_rows(float c, int h) {
    half4_t a = {};
    if (h == 0) {
        const _Float16 c_hi = static_cast<_Float16>(c);
        a[0] = c_hi;
        a[1] = static_cast<_Float16>(c - static_cast<float>(c_hi));
        a[2] = c_hi;
    }
    return a;
}

// A float at a 32-bit byte offset (mp_rows.h) from a wavefront-uniform base;
// the quantities of a row differ by immediate offsets.
template <int IMM = 0>  // added to the address, not to the offset, which might wrap
__device__ __forceinline__ float ld_off(const float* base, uint32_t byte_off) {
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + byte_off + IMM);
}

// Sums over the wavefront in the order of a butterfly 32, 16, 8, 4, 2, 1 (the
// same bits), by lane swaps and row rotations instead of trips through LDS:
// once the pairs 8 lanes apart are added a row repeats every 8 lanes, so that
// a rotation by 4 meets the lane 4 apart, and so on.
__device__ __forceinline__ float add_half(float x) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
template <int N>
__device__ __forceinline__ float add_rotated(float x) {  // row_ror:N
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xF, 0xF, true));
}
__device__ __forceinline__ float butterfly_sum(float x) {
    x = add_half(x);
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    return add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(x))));
}

// ---------------------------------------------------------- edge preparation

// With SM > 0 the same pass also forms the first conservative layer's edge
// sums by neighbour species (see mp_species.hip): the edges of each
// iteration are staged in LDS grouped by species, and lane (c, k) =
// (lane / 16, lane % 16) adds w_c e_k f (w_0 = 1, w_{1+a} = u_a) and w_c f
// over each species' segment; rows Es[i][ep] (c = 0) and Ev[3 i + a][ep],
// 20 slots per species (16 basis values, the cutoff, the species
// indicator, two zeros), zero past S species.
constexpr int kSpKP = kMxK + 4;

template <int SM>
__global__ void __launch_bounds__(256, 3) k_edge_prep(MpGeom mg, int* __restrict__ ecnt, EdgeRec* __restrict__ erec,
                                                   uint4* __restrict__ ehalf, float* __restrict__ Es,
                                                   float* __restrict__ Ev, int S, int ep) {
    constexpr int SP_PITCH = kMxK + 5;  // staged edge: e_k f, 1, u[3], f
    // An iteration's radial pieces, turned around so that a store writes whole
    // lines (from the lanes that hold them, 16 bytes to each of 64 lines, the
    // stores were a tenth of the pass: 12,288 atoms 51 us, now 45), then, in the same
    // room, its edges for the sums by species.
    __shared__ uint4 lds_s[4][64 * 8];
    static_assert(sizeof(float) * 64 * SP_PITCH <= sizeof(uint4) * 64 * 8, "room");
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= mg.n) return;  // whole wavefronts
    const int c = lane >> 4, kk = lane & 15;
    float acc[SM > 0 ? SM : 1] = {}, accf[SM > 0 ? SM : 1] = {};
    uint4* turn = lds_s[threadIdx.x >> 6];
    float(*st)[SP_PITCH] = reinterpret_cast<float(*)[SP_PITCH]>(turn);
    const int n = mg.n;
    const int start = mg.off[i], end = mg.off[i + 1];
    double L, inv;
    mg.geom.get(i, L, inv);
    const double xi = mg.pos[i], yi = mg.pos[n + i], zi = mg.pos[2 * n + i];
    int cnt = 0;
    for (int base = start; base < end; base += 64) {
        const int e = base + lane;
        bool ok = false;
        double dx = 0, dy = 0, dz = 0;
        int j = -1;
        if (e < end) {
            j = mg.nbr[e];
            ok = pair_rule(xi, yi, zi, mg.pos[j], mg.pos[n + j], mg.pos[2 * n + j], L, inv, mg.rc2, dx, dy, dz);
        }
        const uint64_t bal = __ballot(ok);
        const int tj = ok && mg.species ? min(max(mg.species[j], 0), mg.n_species - 1) : 0;
        // this iteration's edges grouped by neighbour species (list order
        // within a species)
        int seg[SM + 1];
        seg[0] = 0;
        int slot = 0;  // staging row of this lane's edge
        if constexpr (SM > 0) {
            const int t = ok ? min(tj, S - 1) : SM;
#pragma unroll
            for (int sp = 0; sp < SM; ++sp) {
                const uint64_t m = __ballot(t == sp);
                if (t == sp) slot = seg[sp] + __popcll(m & ((1ull << lane) - 1ull));
                seg[sp + 1] = seg[sp] + __popcll(m);
            }
        }
        const int rank = __popcll(bal & ((1ull << lane) - 1ull)), found = __popcll(bal);
        float ef[kMxK], u[3], fc;
        if (ok) {
            const int p = start + cnt + rank;
            const double r = sqrt((dx * dx + dy * dy) + dz * dz);
            const double ir = 1.0 / r;
            float def[kMxK], dfc;
            radial_cos_f32<kMxK>(float(r), mg, ef, def, fc, dfc);
            EdgeRec rec;
            rec.j = j;
            rec.t = tj;
            rec.fc = fc;
            rec.dfc = dfc;
            rec.u[0] = float(dx * ir);
            rec.u[1] = float(dy * ir);
            rec.u[2] = float(dz * ir);
            rec.ir = float(ir);
            erec[p] = rec;
            if (mg.edge_key) mg.edge_key[p] = mg.perm ? mg.perm[j] : j;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                half8_t hi, lo;
                uint4* t = turn + 8 * rank;
                split8(ef + 8 * q, hi, lo);
                t[q ^ (rank & 7)] = __builtin_bit_cast(uint4, hi);
                t[(2 + q) ^ (rank & 7)] = __builtin_bit_cast(uint4, lo);
                split8(def + 8 * q, hi, lo);
                t[(4 + q) ^ (rank & 7)] = __builtin_bit_cast(uint4, hi);
                t[(6 + q) ^ (rank & 7)] = __builtin_bit_cast(uint4, lo);
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) u[a] = rec.u[a];
        }
        wave_sync_lds();
        {
            uint4* dst = ehalf + int64_t(start + cnt) * 8;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int t = 64 * k + lane;
                if (t < 8 * found) dst[t] = turn[(t & ~7) + ((t & 7) ^ ((t >> 3) & 7))];
            }
        }
        wave_sync_lds();
        if (ok) {
            if constexpr (SM > 0) {
#pragma unroll
                for (int q = 0; q < kMxK; ++q) st[slot][q] = ef[q];
                st[slot][kMxK] = 1.f;
                st[slot][kMxK + 1] = u[0];
                st[slot][kMxK + 2] = u[1];
                st[slot][kMxK + 3] = u[2];
                st[slot][kMxK + 4] = fc;
            }
        }
        cnt += found;
        if constexpr (SM > 0) {
            wave_sync_lds();
            // each edge added to the running sums in list order (within its
            // species), so that the sums do not depend on where the list
            // rows split into iterations (list radius, replica packing)
#pragma unroll
            for (int sp = 0; sp < SM; ++sp) {
                for (int q = seg[sp]; q < seg[sp + 1]; ++q) {
                    const float wc = st[q][kMxK + c];
                    acc[sp] = fmaf(wc, st[q][kk], acc[sp]);
                    accf[sp] = fmaf(wc, st[q][kMxK + 4], accf[sp]);
                }
            }
        }
        wave_sync_lds();  // the next iteration overwrites the staged edges
    }
    if (lane == 0) ecnt[i] = cnt;
    if constexpr (SM > 0) {
        float* row = c == 0 ? Es + int64_t(i) * ep : Ev + (int64_t(i) * 3 + (c - 1)) * ep;
        const int ti = min(max(mg.species[i], 0), S - 1);
#pragma unroll
        for (int sp = 0; sp < SM; ++sp) {
            if (sp >= S) break;
            row[sp * kSpKP + kk] = acc[sp];
            if (kk == 0) row[sp * kSpKP + kMxK] = accf[sp];
            if (kk == 1) row[sp * kSpKP + kMxK + 1] = (c == 0 && sp == ti) ? 1.f : 0.f;
            if (kk >= 2 && kk < kSpKP - kMxK) row[sp * kSpKP + kMxK + kk] = 0.f;
        }
        for (int z = S * kSpKP + kk; z < ep; z += 16) row[z] = 0.f;
    }
}

// A batch's prepared edges are loaded once per block: thread t holds one
// 16-byte piece (radial pieces of the batch's edges, then its records) in a
// register while the previous batch is processed, and stores it into the
// batch's LDS buffer (two, alternating) after the barrier that ends that
// batch's predecessor.  The forward needs only the e_k f pieces of an edge.
template <int BATCH>
struct BatchBuf {
    static constexpr int AP = BATCH == 32 ? 4 : 8;  // radial pieces per edge
    static constexpr int NA = BATCH * AP, N = NA + 2 * BATCH;
    uint4 a[BATCH][AP];
    EdgeRec rec[BATCH];
};

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 load_nt(const uint4* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// This thread's piece of every batch: what does not change from one batch to
// the next is kept (the offsets took about 40 vector instructions a batch).
template <int BATCH>
struct Stage {
    const char* src;  // of list position 0
    int edge, shift;  // the piece's edge in the batch; log2 of its array's bytes per position
    bool head;        // the piece with the neighbour's index
    __device__ __forceinline__ explicit Stage(const MpGeom& mg) {
        using B = BatchBuf<BATCH>;
        const int t = threadIdx.x, u = t - B::NA;
        head = false;
        if (t < B::NA) {
            edge = t / B::AP;
            shift = 7;
            src = reinterpret_cast<const char*>(mg.ehalf + edge * 8 + t % B::AP);
        } else {
            edge = t < B::N ? u / 2 : 0x7FFFFFFF;
            shift = 5;
            head = u % 2 == 0;
            src = reinterpret_cast<const char*>(mg.erec) + 16 * u;
        }
    }
    // Edges past nb are zeros: their filter is zero; their neighbour is the
    // owner, so that what their rows hold cannot reach another atom.
    __device__ __forceinline__ uint4 fetch(int p0, int nb, int owner) const {
        // read once per evaluation and layer: non-temporal, so that the
        // streamed edges do not displace the neighbour rows from L2
        if (edge < nb) return load_nt(reinterpret_cast<const uint4*>(src + (int64_t(p0) << shift)));
        return make_uint4(head ? uint32_t(owner) : 0u, 0u, 0u, 0u);
    }
};

template <int BATCH>
__device__ __forceinline__ void store_piece(BatchBuf<BATCH>& b, const uint4& v) {
    if (threadIdx.x < BatchBuf<BATCH>::N) reinterpret_cast<uint4*>(&b)[threadIdx.x] = v;
}

// The rows of the block's atoms i0 .. end - 1: lane a holds the list start and
// the edge count of atom i0 + a (none past the last atom), read once; a row is
// then a lane read with no trip to memory (as scalar loads where a batch ends,
// they took a tenth of the reverse).
struct Rows {
    int off, cnt, atoms;
    __device__ __forceinline__ Rows(const MpGeom& mg, int i0, int per) : atoms(min(per, mg.n - i0)) {
        const int lane = threadIdx.x & 63;
        off = lane < atoms ? mg.off[i0 + lane] : 0;
        cnt = lane < atoms ? mg.ecnt[i0 + lane] : 0;
    }
    __device__ __forceinline__ int count(int ai) const { return __builtin_amdgcn_readlane(cnt, ai); }
    __device__ __forceinline__ int start(int ai) const { return __builtin_amdgcn_readlane(off, ai); }
};

// The block's batches in processing order, each atom's edges in batches of
// BATCH.  Returns the list position and size of the batch after batch b0 of
// atom ai (ai = -1: the first batch), or nb = 0 when there is none.
struct NextBatch {
    int p0, nb, ai;
};

template <int BATCH>
__device__ __forceinline__ NextBatch next_batch(const Rows& rows, int ai, int b0, int cnt) {
    if (ai >= 0 && b0 + BATCH < cnt) return {rows.start(ai) + b0 + BATCH, min(BATCH, cnt - b0 - BATCH), ai};
    for (int a2 = ai + 1; a2 < rows.atoms; ++a2) {
        const int c2 = rows.count(a2);
        if (c2 > 0) return {rows.start(a2), min(BATCH, c2), a2};
    }
    return {0, 0, 0};
}

// ------------------------------------------------------------- forward --

struct FwdAcc {
    float s, v[3];
};

// One batch of up to 32 edges.  Of the lane's 16 edges two groups of kFwdGroup
// are in flight: the loads of the first two are issued together behind the
// filter products, those of the next where a group's registers are free
// (left to the compiler, the first half of a batch waited for its loads in
// three parts: 130 -> 125 us at 12,288 atoms, 323 -> 313 at 30,000, 8.0 ->
// 7.3 at 192; with the loads before the products 128.6 and 318, and 173 with
// two features to a lane and no barriers).  An edge past the end of a partial
// batch reads the owner's rows and adds them times a filter of exact zeros:
// with a branch around each edge instead the edges' arithmetic could not
// overlap (137 -> 129 us at 12,288 atoms, 20.7 -> 19.3 at 1,536; the reverse,
// short of registers, is no faster without).
template <bool L0>
__device__ __forceinline__ void fwd_batch(const MpFwd& a, const float* ptab, const BatchBuf<32>& buf, int f, int h,
                                          const uint4* fl, FwdAcc& acc) {
    constexpr int F = kMxF, E = 16, G = kFwdGroup;
    const EdgeRec* rec = buf.rec;
    const int r = threadIdx.x & 31;  // A row: edge r (zero past nb: staged as zeros)
    const half8_t ah = as_half8(buf.a[r][h]), al = as_half8(buf.a[r][2 + h]);
    const half4_t ab = bias_rows(rec[r].fc, h);
    // w = Wr (e f) + b f of every channel
    half8_t bh, bl;
    half4_t bb;
    load_channel(fl, 0, bh, bl, bb);
    const floatx16_t wa = mma3(ab, bb, ah, al, bh, bl);
    floatx16_t wb = {};
    if (!L0) {  // the first layer's vector input is zero
        load_channel(fl, 1, bh, bl, bb);
        wb = mma3(ab, bb, ah, al, bh, bl);
    }
    load_channel(fl, 2, bh, bl, bb);
    const floatx16_t wc = mma3(ab, bb, ah, al, bh, bl);
    const uint32_t fo = uint32_t(f) * 4u;
    // the b channel enters only as phi_b v_j, read as one product; rows
    // of phi and pv are 3F floats: one byte offset per edge serves both
    float pa[2][G], pc[2][G], pv[2][G][3];
    auto gather = [&](int g0) {
        const int d = g0 / G % 2;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int q = g0 + g;
            const EdgeRec& s = rec[8 * (q / 4) + 4 * h + q % 4];
            if (L0) {
                const float* phj = ptab + s.t * 3 * F + f;
                pa[d][g] = phj[0];
                pc[d][g] = phj[2 * F];
            } else {
                const uint32_t off = row3_offset(uint32_t(s.j), fo);
                pa[d][g] = ld_off(a.phi, off);
                pc[d][g] = ld_off<2 * F * 4>(a.phi, off);
                pv[d][g][0] = ld_off(a.pv, off);
                pv[d][g][1] = ld_off<F * 4>(a.pv, off);
                pv[d][g][2] = ld_off<2 * F * 4>(a.pv, off);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    gather(0);
    gather(G);
#pragma unroll
    for (int g0 = 0; g0 < E; g0 += G) {
        const int d = g0 / G % 2;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int q = g0 + g;
            const EdgeRec& s = rec[8 * (q / 4) + 4 * h + q % 4];
            const float c = pc[d][g] * wc[q];
            acc.s = fmaf(pa[d][g], wa[q], acc.s);
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                if (L0) acc.v[x] = fmaf(s.u[x], c, acc.v[x]);
                else acc.v[x] = fmaf(s.u[x], c, fmaf(wb[q], pv[d][g][x], acc.v[x]));
            }
        }
        if (g0 + 2 * G < E) {
            __builtin_amdgcn_sched_barrier(0);
            gather(g0 + 2 * G);
        }
    }
}

template <bool L0>
__global__ void __launch_bounds__(64 * kMxWaves, 4) k_message_fwd_mx(MpGeom mg, MpFwd a, int per) {
    constexpr int F = kMxF, BATCH = 32;
    __shared__ __align__(16) BatchBuf<BATCH> buf[2];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int h = lane >> 5, f = w * 32 + (lane & 31);
    const int n = mg.n;
    // first layer: the species table of phi in LDS
    __shared__ float ptab_s[L0 ? 8 * 3 * kMxF : 1];
    if constexpr (L0) {
        for (int t = threadIdx.x; t < mg.n_species * 3 * F; t += blockDim.x) ptab_s[t] = a.phi_tab[t];
        __syncthreads();
    }
    const float isc = a.mx_scale[1];
    __shared__ __align__(16) uint4 filt_s[kMxWaves][kFiltPieces][64];
    uint4* fl = &filt_s[w][0][lane];
#pragma unroll
    for (int p = 0; p < kFiltPieces; ++p) fl[p * 64] = a.mx_filter[(w * kFiltPieces + p) * 64 + lane];
    wave_sync_lds();
    const int i0 = xcd_block(blockIdx.x, gridDim.x) * per;
    const Rows rows(mg, i0, per);
    NextBatch nx = next_batch<BATCH>(rows, -1, 0, 0);
    const Stage<BATCH> stage(mg);
    uint4 piece = stage.fetch(nx.p0, nx.nb, i0 + nx.ai);
    int k = 0;  // batches of the block so far (LDS buffer parity)
    for (int ai = 0; ai < rows.atoms; ++ai) {
        const int i = i0 + ai;
        const int cnt = rows.count(ai);
        FwdAcc acc{};
        for (int b0 = 0; b0 < cnt; b0 += BATCH, ++k) {
            BatchBuf<BATCH>& b = buf[k & 1];
            store_piece(b, piece);
            __syncthreads();  // the batch is staged; the other buffer's batch is done
            nx = next_batch<BATCH>(rows, ai, b0, cnt);
            piece = stage.fetch(nx.p0, nx.nb, i0 + nx.ai);
            fwd_batch<L0>(a, ptab_s, b, f, h, fl, acc);
        }
        // both halves of the wavefront hold partial sums of feature f
        acc.s = add_half(acc.s);
#pragma unroll
        for (int al = 0; al < 3; ++al) acc.v[al] = add_half(acc.v[al]);
        if (h == 0) {
            const int ti = L0 ? min(max(a.species[i], 0), mg.n_species - 1) : 0;
            const float si = L0 ? a.emb[ti * F + f] : a.s_in[int64_t(i) * F + f];
            a.s_out[int64_t(i) * F + f] = si + acc.s * isc;
#pragma unroll
            for (int al = 0; al < 3; ++al) {
                const int64_t idx = (int64_t(i) * 3 + al) * F + f;
                const float vi = L0 ? 0.f : a.v_in[idx];
                a.v_out[idx] = vi + acc.v[al] * isc;
            }
        }
    }
}

// ------------------------------------------------------------- reverse --

struct Owner {
    float ph[3], v[3], gs, gv[3];
};

// Per-lane sums of the reverse over the lane's edges (feature f):
//   gph0 = sum gs_n w_a,  gph2 = -sum w_c (g_vn . u),  GV = sum w_b g_vn
//   (phi_b adjoint o.v . GV and v adjoint o.ph_b GV at the end),
// and the lane's share of the force on the owner,
//   sum_e [dr u + (g_u - (g_u . u) u) / r]
//     = S1 + o.gv T1 - o.ph_c T2,  g_u = pc w_c o.gv - o.ph_c w_c g_vn,
//   S1 = sum (dr - (g_u . u) / r) u,  T1 = sum pc w_c / r,  T2 = sum w_c g_vn / r,
// which keeps the owner's factors out of the per-edge work.
struct BwdAcc {
    float gph0, gph2, GV[3], S1[3], T1, T2[3], vir;
};

// The neighbour rows one group of edges needs (phi_b of the neighbour
// enters only as phi_b v_n, read as one product; phi, pv and the vector
// adjoints have rows of 3F floats, one byte offset per edge serves them,
// the scalar adjoints rows of F).
template <int G>
struct BwdGather {
    float pa[G], pc[G], pvn[G][3], gn[G][3], gsn[G];
};

// One batch of nb <= 16 edges.  The lane's eight edges are taken kBwdGroup
// at a time (an edge past the end of a partial batch reads the owner's rows
// and contributes nothing).  Past the first layer the rows of the next
// group are requested before the current one is reduced, and the filter
// operands come from LDS (fl) for the products only, which keeps their
// registers free for the second group; the first layer, with fewer rows per
// edge and room for a fourth wavefront per SIMD, keeps its operands in
// registers (bhr, blr, bbr) and takes the groups one after the other.
template <bool L0, bool VIR>
__device__ __forceinline__ void bwd_batch(const MpBwd& a, const float* ptab, const BatchBuf<16>& buf, int nb, int f,
                                          int h, const uint4* fl, const half8_t* bhr, const half8_t* blr,
                                          const half4_t* bbr, const float* b0, const Owner& o, BwdAcc& acc) {
    constexpr int F = kMxF, E = 8, G = kBwdGroup<L0>;
    const EdgeRec* rec = buf.rec;
    // A rows 0..15: e_k f of edges 0..15, rows 16..31: their r-derivatives
    // (zero past nb: staged as zeros), and the bias rows f or f'
    const int r = threadIdx.x & 31, e = r & 15, part = 4 * (r >> 4);
    const half8_t ah = as_half8(buf.a[e][part + h]), al = as_half8(buf.a[e][part + 2 + h]);
    // the first layer adds the biases in the per-edge work instead: the
    // bias operands would cost it the registers of a fourth wavefront per SIMD
    const half4_t ab = L0 ? half4_t{} : bias_rows(part ? rec[e].dfc : rec[e].fc, h);
    floatx16_t m0, m1 = {}, m2;
    if constexpr (L0) {
        // the b channel gates v, zero in the first layer: nothing of it
        // reaches the forces there
        m0 = mma3<false>(ab, bbr[0], ah, al, bhr[0], blr[0]);
        m2 = mma3<false>(ab, bbr[2], ah, al, bhr[2], blr[2]);
    } else {
        half8_t bh, bl;
        half4_t bb;
        load_channel(fl, 0, bh, bl, bb);
        m0 = mma3(ab, bb, ah, al, bh, bl);
        load_channel(fl, 1, bh, bl, bb);
        m1 = mma3(ab, bb, ah, al, bh, bl);
        load_channel(fl, 2, bh, bl, bb);
        m2 = mma3(ab, bb, ah, al, bh, bl);
    }
    const uint32_t fo = uint32_t(f) * 4u;
    auto gather = [&](int g0, BwdGather<G>& d) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int q = g0 + g;
            const int te = 8 * (q / 4) + 4 * h + q % 4;
            const EdgeRec& s = rec[te];
            const uint32_t off = row_offset(uint32_t(s.j), fo), off3 = row3_offset(uint32_t(s.j), fo);
            if (L0) {
                const float* phj = ptab + s.t * 3 * F + f;
                d.pa[g] = phj[0];
                d.pc[g] = phj[2 * F];
            } else {
                d.pa[g] = ld_off(a.phi, off3);
                d.pc[g] = ld_off<2 * F * 4>(a.phi, off3);
                d.pvn[g][0] = ld_off(a.pv, off3);
                d.pvn[g][1] = ld_off<F * 4>(a.pv, off3);
                d.pvn[g][2] = ld_off<2 * F * 4>(a.pv, off3);
            }
            d.gn[g][0] = ld_off(a.gvm, off3);
            d.gn[g][1] = ld_off<F * 4>(a.gvm, off3);
            d.gn[g][2] = ld_off<2 * F * 4>(a.gvm, off3);
            d.gsn[g] = ld_off(a.gsm, off);
        }
    };
    auto reduce = [&](int g0, const BwdGather<G>& d) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int q = g0 + g;
            const int te = 8 * (q / 4) + 4 * h + q % 4;
            if (te >= nb) continue;
            const EdgeRec& s = rec[te];
            // w of edge te is row te, dw/dr row 16 + te: accumulator elements q and 8 + q
            const float ir = s.ir;
            float w0 = m0[q], w2 = m2[q], dw0 = m0[8 + q], dw2 = m2[8 + q];
            if constexpr (L0) {
                w0 = fmaf(b0[0], s.fc, w0);
                w2 = fmaf(b0[2], s.fc, w2);
                dw0 = fmaf(b0[0], s.dfc, dw0);
                dw2 = fmaf(b0[2], s.dfc, dw2);
            }
            const float u0 = s.u[0], u1 = s.u[1], u2 = s.u[2];
            const float g0v = d.gn[g][0], g1v = d.gn[g][1], g2v = d.gn[g][2];
            const float gvn_u = fmaf(g2v, u2, fmaf(g1v, u1, g0v * u0));
            const float gvo_u = fmaf(o.gv[2], u2, fmaf(o.gv[1], u1, o.gv[0] * u0));
            // filter adjoints of both messages of the pair (n -> o and o -> n),
            // contracted with dw/dr
            const float A = fmaf(o.gs, d.pa[g], o.ph[0] * d.gsn[g]);
            const float C = fmaf(d.pc[g], gvo_u, -(o.ph[2] * gvn_u));
            float dr;
            if constexpr (L0) {
                dr = fmaf(A, dw0, C * dw2);
            } else {
                const float w1 = m1[q], dw1 = m1[8 + q];
                const float gvn_vo = fmaf(g2v, o.v[2], fmaf(g1v, o.v[1], g0v * o.v[0]));
                const float gvo_pvn =
                    fmaf(o.gv[2], d.pvn[g][2], fmaf(o.gv[1], d.pvn[g][1], o.gv[0] * d.pvn[g][0]));
                const float B = fmaf(o.ph[1], gvn_vo, gvo_pvn);
                dr = fmaf(A, dw0, fmaf(B, dw1, C * dw2));
                acc.GV[0] = fmaf(w1, g0v, acc.GV[0]);
                acc.GV[1] = fmaf(w1, g1v, acc.GV[1]);
                acc.GV[2] = fmaf(w1, g2v, acc.GV[2]);
            }
            // g_u . u of the unit-vector adjoints is w2 C (the projections
            // above), so its share of the radial term is C w2 / r
            const float w2ir = w2 * ir;
            const float sv = fmaf(-C, w2ir, dr);
            acc.S1[0] = fmaf(sv, u0, acc.S1[0]);
            acc.S1[1] = fmaf(sv, u1, acc.S1[1]);
            acc.S1[2] = fmaf(sv, u2, acc.S1[2]);
            acc.T1 = fmaf(d.pc[g], w2ir, acc.T1);
            acc.T2[0] = fmaf(w2ir, g0v, acc.T2[0]);
            acc.T2[1] = fmaf(w2ir, g1v, acc.T2[1]);
            acc.T2[2] = fmaf(w2ir, g2v, acc.T2[2]);
            // o as the sender of the message o -> n
            acc.gph0 = fmaf(d.gsn[g], w0, acc.gph0);
            acc.gph2 = fmaf(-w2, gvn_u, acc.gph2);
            // r_ij . (pair force share): the projected term is normal to u
            if constexpr (VIR) acc.vir += __fdividef(dr, ir);
        }
    };
    if constexpr (L0) {
#pragma unroll
        for (int g0 = 0; g0 < E; g0 += G) {
            BwdGather<G> d;
            gather(g0, d);
            reduce(g0, d);
        }
    } else {
        BwdGather<G> d0, d1;
        gather(0, d0);
#pragma unroll
        for (int g0 = 0; g0 < E; g0 += 2 * G) {
            if (g0 + G < E) gather(g0 + G, d1);
            reduce(g0, d0);
            if (g0 + G < E) {
                if (g0 + 2 * G < E) gather(g0 + 2 * G, d0);
                reduce(g0 + G, d1);
            }
        }
    }
}

template <bool L0, bool VIR>
__global__ void __launch_bounds__(64 * kMxWaves, 3) k_message_bwd_mx(MpGeom mg, MpBwd a, int per) {
    constexpr int F = kMxF, BATCH = 16;
    __shared__ __align__(16) BatchBuf<BATCH> buf[2];
    __shared__ float fpart[kMxAtoms][kMxWaves][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int h = lane >> 5, f = w * 32 + (lane & 31);
    const int n = mg.n;
    // first layer: the species table of phi in LDS
    __shared__ float ptab_s[L0 ? 8 * 3 * kMxF : 1];
    if constexpr (L0) {
        for (int t = threadIdx.x; t < mg.n_species * 3 * F; t += blockDim.x) ptab_s[t] = a.phi_tab[t];
        __syncthreads();
    }
    const float sc = a.mx_scale[0], isc = a.mx_scale[1];
    // this lane's split filter operands: past the first layer kept in LDS
    // between the batches, in the first layer in registers
    __shared__ __align__(16) uint4 filt_s[L0 ? 1 : kMxWaves][L0 ? 1 : kFiltPieces][64];
    uint4* fl = L0 ? nullptr : &filt_s[L0 ? 0 : w][0][lane];
    half8_t bh[3], bl[3];
    half4_t bb[3];
    {
        const uint4* src = a.mx_filter + w * kFiltPieces * 64 + lane;
        if constexpr (L0) {
#pragma unroll
            for (int p = 0; p < 3; ++p) load_channel(src, p, bh[p], bl[p], bb[p]);
        } else {
#pragma unroll
            for (int p = 0; p < kFiltPieces; ++p) fl[p * 64] = src[p * 64];
            wave_sync_lds();
        }
    }
    float bf[3] = {};  // the scaled biases, for the first layer's per-edge work
    if constexpr (L0) {
#pragma unroll
        for (int p = 0; p < 3; ++p) bf[p] = a.br[p * F + f] * sc;
    }
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int i0 = blk * per;
    const Rows rows(mg, i0, per);
    NextBatch nx = next_batch<BATCH>(rows, -1, 0, 0);
    const Stage<BATCH> stage(mg);
    uint4 piece = stage.fetch(nx.p0, nx.nb, i0 + nx.ai);
    int k = 0;  // batches of the block so far (LDS buffer parity)
    for (int ai = 0; ai < rows.atoms; ++ai) {
        const int i = i0 + ai;
        const int cnt = rows.count(ai);
        Owner o{};
        {
            const int ti = L0 ? min(max(a.species[i], 0), mg.n_species - 1) : 0;
            const float* pho = L0 ? ptab_s + ti * 3 * F + f : a.phi + int64_t(i) * 3 * F + f;
#pragma unroll
            for (int p = 0; p < 3; ++p) o.ph[p] = pho[p * F];
#pragma unroll
            for (int al = 0; al < 3; ++al) {
                const int64_t idx = (int64_t(i) * 3 + al) * F + f;
                if (!L0) o.v[al] = a.v_in[idx];
                o.gv[al] = a.gvm[idx];
            }
            o.gs = a.gsm[int64_t(i) * F + f];
        }
        BwdAcc acc{};
        for (int b0 = 0; b0 < cnt; b0 += BATCH, ++k) {
            BatchBuf<BATCH>& b = buf[k & 1];
            store_piece(b, piece);
            __syncthreads();  // the batch is staged; the other buffer's batch is done
            nx = next_batch<BATCH>(rows, ai, b0, cnt);
            piece = stage.fetch(nx.p0, nx.nb, i0 + nx.ai);
            bwd_batch<L0, VIR>(a, ptab_s, b, min(BATCH, cnt - b0), f, h, fl, bh, bl, bb, bf, o, acc);
        }
        // the lane's force share, then both halves of the wavefront (partial
        // sums of feature f) and the features of the wavefront
        float fs[3];
#pragma unroll
        for (int al = 0; al < 3; ++al) fs[al] = fmaf(o.gv[al], acc.T1, fmaf(-o.ph[2], acc.T2[al], acc.S1[al]));
        acc.gph0 = add_half(acc.gph0);
        acc.gph2 = add_half(acc.gph2);
#pragma unroll
        for (int p = 0; p < 3; ++p) acc.GV[p] = add_half(acc.GV[p]);
        const float gph[3] = {acc.gph0, fmaf(o.v[2], acc.GV[2], fmaf(o.v[1], acc.GV[1], o.v[0] * acc.GV[0])),
                              acc.gph2};
        const float fx = butterfly_sum(fs[0]), fy = butterfly_sum(fs[1]), fz = butterfly_sum(fs[2]);
        const float vr = VIR ? butterfly_sum(acc.vir) : 0.f;
        if (lane == 0) {
            fpart[ai][w][0] = fx;
            fpart[ai][w][1] = fy;
            fpart[ai][w][2] = fz;
            fpart[ai][w][3] = vr;
        }
        if (h == 0) {
            if (a.want_gphi) {
#pragma unroll
                for (int p = 0; p < 3; ++p) a.gphi[int64_t(i) * 3 * F + p * F + f] = gph[p] * isc;
            }
            if (!L0) {
#pragma unroll
                for (int al = 0; al < 3; ++al) {
                    const int64_t idx = (int64_t(i) * 3 + al) * F + f;
                    a.gv_in[idx] = o.gv[al] + (o.ph[1] * acc.GV[al]) * isc;
                }
            }
        }
    }
    __syncthreads();
    // the force (and virial share) of each atom of the block: the feature
    // blocks' shares in a fixed order
    const int t = threadIdx.x;
    if (t < 4 * rows.atoms) {
        const int ai = t / 4, c = t % 4;
        const int i = i0 + ai;
        if (c < 3 || VIR) {
            float sum = 0.f;
            for (int k = 0; k < kMxWaves; ++k) sum += fpart[ai][k][c];
            sum *= isc;
            const int io = mg.perm ? min(max(mg.perm[i], 0), n - 1) : i;
            float* fo = c < 3 ? a.force + int64_t(c) * n + io : a.vir + io;
            if (c == 3) sum *= 0.5f;  // each pair is seen by both of its atoms
            if (a.accum_force) *fo += sum;
            else *fo = sum;
        }
    }
}

// ---------------------------------------- reverse, one message of each edge --
// FP32 models with the per-atom blocks.  A pair's force is the sum of those
// of its two messages, and both of its atoms see both.  Here an atom takes
// only the messages it sends, o -> n, which need of the neighbour the adjoints
// of s and v alone (4 rows instead of 9, which are most of what the kernel
// above waits for), and keeps of each the sums over the features
//   S = sum_f [ph_a gs_n w_a' + (ph_b v_o . gv_n) w_b' - ph_c (gv_n . u) w_c'],
//   T = sum_f ph_c w_c gv_n,
// with which the force on o through it is (S + T . u / r) u - T / r; the
// messages it receives are the ones its neighbours send it, found from their
// rows (k_edge_force, once for all layers).  The sums over features take
// 9 operations per edge and feature (all four sums of a batch's edges in one
// exchange that halves the values at every step), the rest 20 instead of 34;
// vector arithmetic keeps the SIMDs three quarters busy.  At 12,288 atoms a
// layer takes 185 us instead of 240, at 1,536 26 instead of 32 (rows in the
// caller's order; in cell order, in which a trajectory has them, 165 instead of
// 214 at 12,288), and the first layer in the same form (k_sp_bwd_own) with k_edge_force no more than
// k_sp_bwd did (35 + 24 us instead of 66; 7.6 + 5.2 instead of 11.6): energy
// and forces 1,184 -> 1,086 us and 258 -> 249.  Forces are 2 % closer to
// float64.  The adjoints of phi and of the vector input are as above, bit for
// bit.

// One step of the exchange: of the sums x and y over 2 k lanes each, x's in
// half of the lanes and y's in the other (by lane bit 4, 3, 2, 1, 0).
__device__ __forceinline__ float halve16(float x, float y) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
template <int CTRL>
__device__ __forceinline__ float plus_dpp(float x) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int BANKS>
__device__ __forceinline__ float pick_banks(float x, float y) {  // y in the quads of BANKS
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(y), 0xE4, 0xF, BANKS, false));
}
__device__ __forceinline__ float halve8(float x, float y) {  // row_ror:8
    return pick_banks<0xC>(plus_dpp<0x128>(x), plus_dpp<0x128>(y));
}
__device__ __forceinline__ float halve4(float x, float y) {  // row_half_mirror
    return pick_banks<0xA>(plus_dpp<0x141>(x), plus_dpp<0x141>(y));
}
__device__ __forceinline__ float halve2(float x, float y, bool odd) {  // quad_perm 2 3 0 1
    const float u = plus_dpp<0x4E>(x), t = plus_dpp<0x4E>(y);
    return odd ? t : u;
}
__device__ __forceinline__ float halve1(float x, float y, bool odd) {  // quad_perm 1 0 3 2
    const float u = plus_dpp<0xB1>(x), t = plus_dpp<0xB1>(y);
    return odd ? t : u;
}

constexpr int kSendGroup = 2;  // edges of a lane whose rows are requested together

struct SendAcc {
    float gph0, gph2, GV[3];
};
struct SendOwner {
    float ph0, ph2, pv[3];  // ph_a, ph_c, ph_b v
};

// One batch of nb <= 16 edges; returns the lane's feature sum (over its
// wavefront's 32 features) of value (edge, component) = send_slot(lane).
__device__ __forceinline__ float send_batch(const MpBwd& a, const BatchBuf<16>& buf, int nb, int f, int h,
                                            const uint4* fl, const SendOwner& o, SendAcc& acc) {
    constexpr int F = kMxF, E = 8, G = kSendGroup;
    const EdgeRec* rec = buf.rec;
    const int lane = threadIdx.x & 63, r = lane & 31, e = r & 15, part = 4 * (r >> 4);
    const half8_t ah = as_half8(buf.a[e][part + h]), al = as_half8(buf.a[e][part + 2 + h]);
    const half4_t ab = bias_rows(part ? rec[e].dfc : rec[e].fc, h);
    half8_t bh, bl;
    half4_t bb;
    load_channel(fl, 0, bh, bl, bb);
    const floatx16_t m0 = mma3(ab, bb, ah, al, bh, bl);
    load_channel(fl, 1, bh, bl, bb);
    const floatx16_t m1 = mma3(ab, bb, ah, al, bh, bl);
    load_channel(fl, 2, bh, bl, bb);
    const floatx16_t m2 = mma3(ab, bb, ah, al, bh, bl);
    struct Rows4 {
        float gn[G][3], gsn[G];
    };
    const uint32_t fo = uint32_t(f) * 4u;
    auto gather = [&](int g0, Rows4& d) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int q = g0 + g, te = 8 * (q / 4) + 4 * h + q % 4;
            const uint32_t j = uint32_t(rec[te].j), off = row_offset(j, fo), off3 = row3_offset(j, fo);
            d.gn[g][0] = ld_off(a.gvm, off3);
            d.gn[g][1] = ld_off<F * 4>(a.gvm, off3);
            d.gn[g][2] = ld_off<2 * F * 4>(a.gvm, off3);
            d.gsn[g] = ld_off(a.gsm, off);
        }
    };
    // edges past nb: a filter of exact zeros
    float quarter[E / 2];  // a pair of edges: lane bits 4, 3, 2 = edge, component % 2, component / 2
    auto reduce = [&](int g0, const Rows4& d) {
#pragma unroll
        for (int g1 = 0; g1 < G; g1 += 2) {
            float val[2][4];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int g = g1 + k, q = g0 + g, te = 8 * (q / 4) + 4 * h + q % 4;
                const EdgeRec& s = rec[te];
                const float g0v = d.gn[g][0], g1v = d.gn[g][1], g2v = d.gn[g][2];
                const float gvn_u = fmaf(g2v, s.u[2], fmaf(g1v, s.u[1], g0v * s.u[0]));
                const float B = fmaf(g2v, o.pv[2], fmaf(g1v, o.pv[1], g0v * o.pv[0]));
                const float A = o.ph0 * d.gsn[g], C = o.ph2 * gvn_u;
                const float w0 = m0[q], w1 = m1[q], w2 = m2[q];
                val[k][0] = fmaf(A, m0[8 + q], fmaf(B, m1[8 + q], -C * m2[8 + q]));
                const float p2 = o.ph2 * w2;
                val[k][1] = p2 * g0v;
                val[k][2] = p2 * g1v;
                val[k][3] = p2 * g2v;
                acc.GV[0] = fmaf(w1, g0v, acc.GV[0]);
                acc.GV[1] = fmaf(w1, g1v, acc.GV[1]);
                acc.GV[2] = fmaf(w1, g2v, acc.GV[2]);
                acc.gph0 = fmaf(d.gsn[g], w0, acc.gph0);
                acc.gph2 = fmaf(-w2, gvn_u, acc.gph2);
            }
            float x[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = halve16(val[0][c], val[1][c]);
            quarter[(g0 + g1) / 2] = halve4(halve8(x[0], x[1]), halve8(x[2], x[3]));
        }
    };
    Rows4 d0, d1;
    gather(0, d0);
#pragma unroll
    for (int g0 = 0; g0 < E; g0 += 2 * G) {
        if (g0 + G < E) gather(g0 + G, d1);
        reduce(g0, d0);
        if (g0 + G < E) {
            if (g0 + 2 * G < E) gather(g0 + 2 * G, d0);
            reduce(g0 + G, d1);
        }
    }
    const bool b1 = lane & 2, b0 = lane & 1;
    return halve1(halve2(quarter[0], quarter[1], b1), halve2(quarter[2], quarter[3], b1), b0);
}
// (edge of the batch) 4 + component of the value a lane holds then
__device__ __forceinline__ int send_slot(int lane) {
    const int pair = ((lane >> 1) & 1) + 2 * (lane & 1), q = 2 * pair + ((lane >> 4) & 1);
    const int comp = ((lane >> 3) & 1) + 2 * ((lane >> 2) & 1);
    return (8 * (q / 4) + 4 * (lane >> 5) + q % 4) * 4 + comp;
}

// ADD: a.edge_f already holds the sums of the layers above.  BLOCKS per CU:
// four spill 11 registers, which pays where there are more blocks than three
// per CU hold (12,288 atoms 192 -> 183 us, 4,095 atoms 79 -> 74; 1,536 atoms,
// all in flight with three, 27.0 -> 28.4).
template <bool ADD, int BLOCKS>
__global__ void __launch_bounds__(64 * kMxWaves, BLOCKS) k_message_bwd_send(MpGeom mg, MpBwd a, int per) {
    constexpr int F = kMxF, BATCH = 16;
    __shared__ __align__(16) BatchBuf<BATCH> buf[2];
    __shared__ float fsum[2][kMxWaves][4 * BATCH];  // feature sums of a batch per wavefront
    __shared__ __align__(16) uint4 filt_s[kMxWaves][kFiltPieces][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int h = lane >> 5, f = w * 32 + (lane & 31);
    const float isc = a.mx_scale[1];
    uint4* fl = &filt_s[w][0][lane];
#pragma unroll
    for (int p = 0; p < kFiltPieces; ++p) fl[p * 64] = a.mx_filter[(w * kFiltPieces + p) * 64 + lane];
    wave_sync_lds();
    const int i0 = xcd_block(blockIdx.x, gridDim.x) * per;
    const Rows rows(mg, i0, per);
    const int slot = send_slot(lane);
    NextBatch nx = next_batch<BATCH>(rows, -1, 0, 0);
    const Stage<BATCH> stage(mg);
    uint4 piece = stage.fetch(nx.p0, nx.nb, i0 + nx.ai);
    int k = 0;           // batches of the block so far (LDS buffer parity)
    int done_p = 0, done_n = 0;  // the batch before: its sums are in fsum[(k - 1) & 1]
    // the wavefronts take turns to add the batch's sums over all features
    auto pending = [&] { return done_n > 0 && w == ((k - 1) & 3) && (lane >> 2) < done_n; };
    auto store = [&](float before) {
        const float* p = &fsum[(k - 1) & 1][0][lane];
        const float sum = ((p[0] + p[4 * BATCH]) + p[8 * BATCH]) + p[12 * BATCH];
        a.edge_f[int64_t(done_p) * 4 + lane] = ADD ? fmaf(sum, isc, before) : sum * isc;
    };
    for (int ai = 0; ai < rows.atoms; ++ai) {
        const int i = i0 + ai;
        const int cnt = rows.count(ai);
        const float* pho = a.phi + int64_t(i) * 3 * F + f;
        const float ph1 = pho[F];
        SendOwner o;
        o.ph0 = pho[0];
        o.ph2 = pho[2 * F];
        float v[3], gv[3];
#pragma unroll
        for (int al = 0; al < 3; ++al) {
            v[al] = a.v_in[(int64_t(i) * 3 + al) * F + f];
            gv[al] = a.gvm[(int64_t(i) * 3 + al) * F + f];
            o.pv[al] = ph1 * v[al];
        }
        SendAcc acc{};
        for (int b0 = 0; b0 < cnt; b0 += BATCH, ++k) {
            BatchBuf<BATCH>& b = buf[k & 1];
            store_piece(b, piece);
            __syncthreads();  // the batch is staged; the other buffer's batch is done, its sums in fsum
            const int nb = min(BATCH, cnt - b0);
            const bool mine = pending();
            float before = 0.f;
            if (ADD && mine) before = a.edge_f[int64_t(done_p) * 4 + lane];
            nx = next_batch<BATCH>(rows, ai, b0, cnt);
            piece = stage.fetch(nx.p0, nx.nb, i0 + nx.ai);
            const float x = send_batch(a, b, nb, f, h, fl, o, acc);
            if (mine) store(before);
            fsum[k & 1][w][slot] = x;
            done_p = rows.start(ai) + b0;
            done_n = nb;
        }
        acc.gph0 = add_half(acc.gph0);
        acc.gph2 = add_half(acc.gph2);
#pragma unroll
        for (int p = 0; p < 3; ++p) acc.GV[p] = add_half(acc.GV[p]);
        const float gph[3] = {acc.gph0, fmaf(v[2], acc.GV[2], fmaf(v[1], acc.GV[1], v[0] * acc.GV[0])), acc.gph2};
        if (h == 0) {
#pragma unroll
            for (int p = 0; p < 3; ++p) a.gphi[int64_t(i) * 3 * F + p * F + f] = gph[p] * isc;
#pragma unroll
            for (int al = 0; al < 3; ++al)
                a.gv_in[(int64_t(i) * 3 + al) * F + f] = gv[al] + (ph1 * acc.GV[al]) * isc;
        }
    }
    __syncthreads();
    if (pending()) store(ADD ? a.edge_f[int64_t(done_p) * 4 + lane] : 0.f);
}

// Forces (and virial shares) of the messages whose feature sums
// k_message_bwd_send left: one wavefront per atom, lanes over its edges, the
// message it receives along an edge from the neighbour's row (ascending in
// the caller's index, so found by bisection; its unit vector is the other way
// round).  Bound by that chain of dependent loads.
// Blocks past the atoms': the energies of the replicas (as a launch of its
// own, between the forward and the reverse, 4.6 us).
template <bool VIR>
__global__ void __launch_bounds__(256) k_edge_force(MpGeom mg, const float4* __restrict__ edge_f,
                                                    float* __restrict__ force, float* __restrict__ vir, RepSum rs) {
    __shared__ double red[256];
    const int blocks = gridDim.x - rs.n_rep;
    if (int(blockIdx.x) >= blocks) {
        rep_sum_block(rs, blockIdx.x - blocks, red);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int i = xcd_block(blockIdx.x, blocks) * 4 + (threadIdx.x >> 6);
    if (i >= mg.n) return;  // whole wavefronts
    const int start = mg.off[i], cnt = mg.ecnt[i];
    const int key = mg.perm ? mg.perm[i] : i;
    float fx = 0.f, fy = 0.f, fz = 0.f, vr = 0.f;
    for (int e = lane; e < cnt; e += 64) {
        const EdgeRec rec = mg.erec[start + e];
        const float4 own = edge_f[start + e];
        const int row = mg.off[rec.j], end = row + mg.ecnt[rec.j];
        int lo = row;
        for (int hi = end; lo < hi;) {
            const int mid = (lo + hi) >> 1;
            if (mg.edge_key[mid] < key) lo = mid + 1;
            else hi = mid;
        }
        // a caller's list whose rows do not ascend: entry by entry
        if (lo >= end || mg.edge_key[lo] != key)
            for (lo = row; lo < end && mg.edge_key[lo] != key;) ++lo;
        float4 got = make_float4(0.f, 0.f, 0.f, 0.f);
        if (lo < end) got = edge_f[lo];
        const float S = own.x + got.x;
        const float tx = own.y - got.y, ty = own.z - got.z, tz = own.w - got.w;
        const float tu = fmaf(tz, rec.u[2], fmaf(ty, rec.u[1], tx * rec.u[0]));
        const float rad = fmaf(tu, rec.ir, S);
        fx += fmaf(rad, rec.u[0], -tx * rec.ir);
        fy += fmaf(rad, rec.u[1], -ty * rec.ir);
        fz += fmaf(rad, rec.u[2], -tz * rec.ir);
        if (VIR) vr += S / rec.ir;
    }
    fx = butterfly_sum(fx);
    fy = butterfly_sum(fy);
    fz = butterfly_sum(fz);
    if (VIR) vr = butterfly_sum(vr);
    if (lane == 0) {
        const int io = mg.perm ? min(max(key, 0), mg.n - 1) : i;
        force[io] = fx;
        force[mg.n + io] = fy;
        force[2 * mg.n + io] = fz;
        if (VIR) vir[io] = 0.5f * vr;
    }
}

// Scale of the filter weights and biases of one layer for the split
// products: a power of two s with max(|Wr|, |br|) s in [2^13, 2^14) (s = 1
// when all are zero), and 1 / s.  Wr and br are contiguous in the weights.
__global__ void __launch_bounds__(256) k_filter_scale(int count, const float* Wr, float* out) {
    __shared__ float part[256];
    float m = 0.f;
    for (int k = threadIdx.x; k < count; k += blockDim.x) m = fmaxf(m, fabsf(Wr[k]));
    part[threadIdx.x] = m;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) part[threadIdx.x] = fmaxf(part[threadIdx.x], part[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float mx = part[0];
        int e = 0;
        if (mx > 0.f && isfinite(mx)) (void)frexpf(mx, &e);  // mx < 2^e
        e = min(max(e, -100), 100);
        out[0] = ldexpf(1.f, 14 - e);
        out[1] = ldexpf(1.f, e - 14);
    }
}

// pv[i][al][f] = phi[i][F + f] * v[i][al][f]: one thread per four features
// of an atom.
__global__ void __launch_bounds__(256) k_phib_v(int n, const float* __restrict__ phi, const float* __restrict__ v,
                                                float* __restrict__ pv) {
    constexpr int F = kMxF, C = F / 4;
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n) * C) return;
    const int64_t i = t / C;
    const int c = int(t % C);
    const float4 b = reinterpret_cast<const float4*>(phi + i * 3 * F + F)[c];
#pragma unroll
    for (int al = 0; al < 3; ++al) {
        const int64_t row = (i * 3 + al) * F;
        const float4 x = reinterpret_cast<const float4*>(v + row)[c];
        reinterpret_cast<float4*>(pv + row)[c] = make_float4(b.x * x.x, b.y * x.y, b.z * x.z, b.w * x.w);
    }
}

// Atoms of a block: one or two, whichever takes fewer turns (an atom's time)
// of the 3 x 256 blocks of the two-message reverse that are in flight at once,
// two where that is equal (half as many starts).  A block's atoms follow one
// another, so that with fewer blocks than the chip holds the longest block is
// the time.  Measured with one and two atoms, us, rows in random order (forward;
// reverse by one message; by both): 192 atoms 9.7 14.5; 12.1 19.4; 14.6 23.5.
// 768: 13.5 16.4; 16.2 21.5; 19.0 26.0.  1,536: 22.1 21.5; 29.9 26.6; 34.9 33.6.
// 2,100: 28.7 31.2; 37.6 42.5; 50.0 55.7.  3,000: 42.3 42.3; 49.9 52.6; 79.4 78.7.
// 12,288: 215 218; 199 197; 407 416.  The forward and the reverse by one message
// have up to 4 x 256 blocks in flight, and from 769 to 1,024 atoms one atom is
// the faster for them (1,000: 15.4 16.7; 19.7 22.4, against 27.9 27.3): the line
// is the two-message reverse's there.  An atom's sums do not depend on it.
constexpr int kMxSlots = 3 * 256;
int mx_atoms(int n) { return cdiv(n, kMxSlots) < 2 * cdiv(cdiv(n, 2), kMxSlots) ? 1 : kMxAtoms; }

template <typename Kern, typename Args>
void launch_mx(const ScopedTimer& t, Kern kern, int n, hipStream_t s, const MpGeom& mg, const Args& a) {
    const int per = mx_atoms(n);
    const dim3 grid(cdiv(n, per));
    if (t.active && t.by_launch) hipExtLaunchKernelGGL(kern, grid, dim3(64 * kMxWaves), 0, s, t.a, t.b, 0, mg, a, per);
    else kern<<<grid, 64 * kMxWaves, 0, s>>>(mg, a, per);
}

}  // namespace

bool message_mx_shape(int F, int K, int cut) { return F == kMxF && K == kMxK && cut == 0; }

void launch_message_fwd_mx(const MpGeom& mg, const MpFwd& a, hipStream_t s, const ScopedTimer& t) {
    if (a.phi_tab) {
        launch_mx(t, k_message_fwd_mx<true>, mg.n, s, mg, a);
        return;
    }
    if (!a.pv) {
        set_error("matrix-core message step: no phi_b * v buffer");
        throw Fail{NNP_EINVAL};
    }
    if (!a.pv_ready)
        k_phib_v<<<cdiv(int64_t(mg.n) * (kMxF / 4), 256), 256, 0, s>>>(mg.n, a.phi, a.v_in, a.pv);
    launch_mx(t, k_message_fwd_mx<false>, mg.n, s, mg, a);
}

void launch_edge_force(const MpGeom& mg, const float* edge_f, float* force, float* vir, const RepSum& rs,
                       hipStream_t s) {
    if (mg.n <= 0) return;
    ScopedTimer t("message_bwd_first", s, true);
    const float4* ef = reinterpret_cast<const float4*>(edge_f);
    const dim3 grid(cdiv(mg.n, 4) + rs.n_rep), block(256);
    auto go = [&](auto kern) {
        if (t.active && t.by_launch)
            hipExtLaunchKernelGGL(kern, grid, block, 0, s, t.a, t.b, 0, mg, ef, force, vir, rs);
        else kern<<<grid, block, 0, s>>>(mg, ef, force, vir, rs);
    };
    if (vir) go(k_edge_force<true>);
    else go(k_edge_force<false>);
    NNP_LAUNCH_CHECK();
}

void launch_message_bwd_mx(const MpGeom& mg, const MpBwd& a, hipStream_t s, const ScopedTimer& t) {
    if (a.edge_f && !a.phi_tab) {
        const bool many = cdiv(mg.n, mx_atoms(mg.n)) > kMxSlots;
        if (a.accum_force) launch_mx(t, many ? k_message_bwd_send<true, 4> : k_message_bwd_send<true, 3>, mg.n, s, mg, a);
        else launch_mx(t, many ? k_message_bwd_send<false, 4> : k_message_bwd_send<false, 3>, mg.n, s, mg, a);
        return;
    }
    if (!a.phi_tab && !a.pv) {
        set_error("matrix-core message reverse: no phi_b * v buffer");
        throw Fail{NNP_EINVAL};
    }
    if (a.vir) {
        if (a.phi_tab) launch_mx(t, k_message_bwd_mx<true, true>, mg.n, s, mg, a);
        else launch_mx(t, k_message_bwd_mx<false, true>, mg.n, s, mg, a);
    } else {
        if (a.phi_tab) launch_mx(t, k_message_bwd_mx<true, false>, mg.n, s, mg, a);
        else launch_mx(t, k_message_bwd_mx<false, false>, mg.n, s, mg, a);
    }
}

void launch_edge_prep(const MpGeom& mg, int* ecnt, EdgeRec* erec, uint4* ehalf, hipStream_t s, float* Es, float* Ev,
                      int S, int ep) {
    if (mg.n <= 0) return;
    const dim3 grid(cdiv(mg.n, 4));
    if (!Es) k_edge_prep<0><<<grid, 256, 0, s>>>(mg, ecnt, erec, ehalf, nullptr, nullptr, 0, 0);
    else if (S <= 2) k_edge_prep<2><<<grid, 256, 0, s>>>(mg, ecnt, erec, ehalf, Es, Ev, S, ep);
    else if (S <= 4) k_edge_prep<4><<<grid, 256, 0, s>>>(mg, ecnt, erec, ehalf, Es, Ev, S, ep);
    else k_edge_prep<8><<<grid, 256, 0, s>>>(mg, ecnt, erec, ehalf, Es, Ev, S, ep);
    NNP_LAUNCH_CHECK();
}

void launch_filter_scale(int count, const float* Wr, float* out, hipStream_t s) {
    k_filter_scale<<<1, 256, 0, s>>>(count, Wr, out);
    NNP_LAUNCH_CHECK();
}

int64_t filter_operand_units() { return int64_t(kMxWaves) * kFiltPieces * 64; }

void launch_filter_operands(const float* Wr, const float* br, const float* scale, uint4* out, hipStream_t s) {
    k_filter_operands<<<1, 64 * kMxWaves, 0, s>>>(Wr, br, scale, out);
    NNP_LAUNCH_CHECK();
}

}  // namespace nnp
