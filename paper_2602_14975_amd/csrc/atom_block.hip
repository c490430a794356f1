// The per-atom work between two message steps of a width-128 conservative
// model as one kernel each way (forward: update block, then the next layer's
// phi perceptron or the readout; reverse: their adjoints), instead of one
// launch per dense product and elementwise step.
//
// A block of eight wavefronts owns a tile of TA = 16 or 32 atoms.  Every
// product is
//   out[feature][atom] = sum_k W[feature][k] x[atom][k]
// on v_mfma_f32_16x16x32_bf16 with the weights as the first operand, so that
// a lane of wavefront w holds, of atoms a = lane % 16 and a + 16, the features
// 16 w + 4 h + q (h = lane / 16, q < 4) in its accumulators: four consecutive
// features per 16-byte global access, and everything elementwise between the
// products stays in registers, the same features for all of an atom's
// quantities.  The inputs of a product pass through LDS as operand
// fragments (16 bytes per lane and step); the weights are read straight from
// L2 in the packed order of launch_pack_frags, each fragment by one
// wavefront of the block, a few steps ahead.
//
// FP32 models split both operands into three bfloat16 pieces and accumulate
// the six piece products of order >= 2^-18 in float32, smallest first, as
// k_gemm_x3 does (FP32-equivalent); BF16 models take the operands rounded to
// bfloat16 and one product.
//
// What bounds it: of a block alone on its CU the way of 1 MB of packed weights
// from L2 (45 bytes a cycle of at most 64) beside 23,000 cycles (32 atoms;
// half at 16) of matrix instructions per SIMD and the chain from one product
// to the next.  With two blocks on a CU the rows from memory too: a middle
// layer moves 204 MB at 12,288 atoms, 43 us at the rate of a copy, of 65
// (BF16, with a sixth of the matrix work: 42), and the blocks, which start
// together, load, compute and store at the same times.  While a block has a
// CU to itself, 16 atoms take two thirds of the time of 32 (half the matrix
// and elementwise work per lane, the same weights), beyond that they read the
// weights twice as often: see small_tiles.  Eight wavefronts of 16 features
// rather than four of 32: two (and with two blocks four) per SIMD hide each
// other's waits.  Middle layer, reverse / forward, us, four -> eight: tiles of
// 16, 1,536 atoms FP32 22.9 / 21.2 -> 21.5 / 19.6, BF16 15.6 / 14.6 -> 13.3 /
// 12.8; tiles of 32 (there on 32x32x16 products, two wavefronts per SIMD),
// FP32 6,144 41.9 / 42.7 -> 40.4 / 40.6, 12,288 71.8 / 68.4 -> 69.4 / 64.6,
// BF16 23,700 78.5 / 80.9 -> 75.3 / 75.2.  As separate launches the same work
// moved about 40 F floats per atom and layer through memory forward and more
// in reverse, 28 products and 15 elementwise launches per evaluation; the
// blocks move 24 F and are six launches.  Measured, dense products and
// elementwise launches together, per evaluation (3 layers, FP32): 12,288
// atoms 885 -> 378 us (blocks of 43 to 79 us, the first layer's species
// products among them); 1,536 atoms 460 -> 119 us (13 to 24 us each).
#include <algorithm>
#include <numeric>

#include "atom_block_addr.h"
#include "common.h"
#include "kernels.h"

namespace nnp {

namespace {

using namespace atom_block;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kF = kFeatures;
constexpr int kFrag = 1024;      // bytes of one operand fragment (64 lanes x 16)
constexpr int kKsF = kF / 32;    // steps of a product over one width: 32 k each
constexpr int kW = kWaves;
constexpr int kWF = kSliceFeatures;
template <int TA>
constexpr int kTurn = TA * kWF * 4;  // bytes of LDS that turn one slice around
template <int TA>
constexpr int kFragsF = TA * kF / 512;  // operand fragments of one width of the tile's atoms, per piece
// LDS of a block: three regions, each the fragments of F inputs of its atoms
// (or room to turn one slice per wavefront around); 72 KB at three pieces and
// 32 atoms: two blocks per CU
template <int NP, int TA>
constexpr int kRegion = kFragsF<TA> * kFrag * (NP == 1 ? 2 : NP);
template <int NP, int TA>
constexpr int kLdsBytes = 3 * kRegion<NP, TA>;

// Four floats as NP bfloat16 pieces (round to nearest of what the previous
// pieces leave), two packed words per piece.
template <int NP>
__device__ __forceinline__ void split4(const f32x4_t& x, uint2 (&o)[NP]) {
    f32x2_t r0{x.x, x.y}, r1{x.z, x.w};
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        o[p].x = __builtin_bit_cast(uint32_t, __builtin_convertvector(r0, bf16x2_t));
        o[p].y = __builtin_bit_cast(uint32_t, __builtin_convertvector(r1, bf16x2_t));
        if (p + 1 < NP) {  // exact differences
            r0 -= f32x2_t{__uint_as_float(o[p].x << 16), __uint_as_float(o[p].x & 0xFFFF0000u)};
            r1 -= f32x2_t{__uint_as_float(o[p].y << 16), __uint_as_float(o[p].y & 0xFFFF0000u)};
        }
    }
}

// A lane's values of one slice of 16 features: element 4 g + q = feature
// 16 w + 4 h + q of atom a + 16 g.
template <int TA>
struct Slice {
    static constexpr int G = TA / 16;
    f32x4_t v[G];
    __device__ __forceinline__ float operator[](int i) const { return v[i >> 2][i & 3]; }
};

// The sums of one slice of a product, element by element those of Slice
template <int TA>
struct Sums {
    static constexpr int G = TA / 16;
    f32x4_t c[G] = {};
    __device__ __forceinline__ float operator[](int e) const { return c[e >> 2][e & 3]; }
    __device__ __forceinline__ void add(const Sums& o) {
#pragma unroll
        for (int g = 0; g < G; ++g) c[g] += o.c[g];
    }
};

// Global memory through buffer descriptors: a uniform base, a uniform offset
// and one 32-bit lane offset per row stride, so that addresses take no
// vector registers (plain pointers cost these kernels about 60), and rows
// past the last atom, which are out of the bound by the lane offset, are read
// as zero and not stored (atom_block_addr.h).
struct Buf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Buf(const void* p, uint32_t bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000)) {}
    __device__ __forceinline__ u32x4_t load(uint32_t lane_off, uint32_t off) const {
        return __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0);
    }
    // The whole offset in the lane's register: with part of it in an SGPR the
    // compiler leaves no wait between a 16-byte store and the next vector
    // instruction that writes its data registers, and this GPU needs one (the
    // last lanes then stored the new value of the first register).
    __device__ __forceinline__ void store(const u32x4_t& v, uint32_t off) const {
        __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, 0);
    }
};

// This lane's place in the block
template <int TA>
struct Lane {
    int lane, w, a, h;
    int64_t t0;  // first atom of the block's tile
    int rows;    // atoms of the tile
    __device__ __forceinline__ Lane(int n) {
        lane = threadIdx.x & 63;
        w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        a = lane & 15;
        h = lane >> 4;
        t0 = int64_t(xcd_block(blockIdx.x, gridDim.x)) * TA;
        rows = min(TA, n - int(t0));
    }
};

// Row-major float32 of C rows per atom, row width ld: the lane's slice at
// column c0 of row c of its atom.
template <int C, int ld, int TA>
__device__ __forceinline__ Slice<TA> load_slice(const float* p, int c, int c0, const Lane<TA>& L) {
    const Buf b(p + L.t0 * (C * ld), uint32_t(L.rows * (C * ld * 4)));
    const uint32_t o = row_uniform_offset<C, ld>(c, c0, L.w);
    Slice<TA> s;
#pragma unroll
    for (int g = 0; g < s.G; ++g)
        s.v[g] = __builtin_bit_cast(f32x4_t, b.load(row_lane_offset<C, ld>(L.a, g, L.h), o));
    return s;
}
// The slice into row-major rows, turned around through kTurn bytes of LDS
// (`turn`, this wavefront's own) so that four lanes write the 64 bytes of a
// row together: written as held, 16 bytes per lane and row, a store took
// about 100 cycles and the stores a third of the kernel.
template <int C, int ld, int TA>
__device__ __forceinline__ void store_slice(float* p, int c, int c0, const Lane<TA>& L, const Slice<TA>& s,
                                            char* turn) {
    const Buf b(p + L.t0 * (C * ld), uint32_t(L.rows * (C * ld * 4)));
    wave_sync_lds();
#pragma unroll
    for (int g = 0; g < s.G; ++g)
        *reinterpret_cast<f32x4_t*>(turn + (16 * g + L.a) * 64 + (L.h ^ (L.a & 3)) * 16) = s.v[g];
    wave_sync_lds();
    const int row = L.lane >> 2, q = L.lane & 3;
    const uint32_t lo = uint32_t(row * (C * ld * 4) + 16 * q + (c * ld + c0 + kWF * L.w) * 4);
#pragma unroll
    for (int g = 0; g < s.G; ++g)
        b.store(*reinterpret_cast<const u32x4_t*>(turn + (16 * g + row) * 64 + (q ^ (row & 3)) * 16),
                lo + g * (16 * C * ld * 4));
}
// Quantities that only these kernels exchange are kept in lane order: slice
// `c` (of C) of the tile's wavefront w, 1 KB per group of four features.
// Rows past the last atom are part of the buffers.
template <int C, int TA>
__device__ __forceinline__ void keep_slice(float* p, int c, const Lane<TA>& L, const Slice<TA>& s) {
    const Buf b(p + L.t0 * (C * kF), uint32_t(TA * C * kF * 4));
#pragma unroll
    for (int g = 0; g < s.G; ++g)
        b.store(__builtin_bit_cast(u32x4_t, s.v[g]), uint32_t(16 * L.lane + ((c * kW + L.w) * s.G + g) * 1024));
}
template <int C, int TA>
__device__ __forceinline__ Slice<TA> kept_slice(const float* p, int c, const Lane<TA>& L) {
    const Buf b(p + L.t0 * (C * kF), uint32_t(TA * C * kF * 4));
    Slice<TA> s;
#pragma unroll
    for (int g = 0; g < s.G; ++g)
        s.v[g] = __builtin_bit_cast(f32x4_t, b.load(16 * L.lane, uint32_t(((c * kW + L.w) * s.G + g) * 1024)));
    return s;
}
// kF per-feature constants (biases)
template <int TA>
__device__ __forceinline__ Slice<TA> load_feat(const float* p, const Lane<TA>& L) {
    const Buf b(p, kF * 4);
    Slice<TA> s;
    s.v[0] = __builtin_bit_cast(f32x4_t, b.load(16 * L.h, uint32_t(4 * kWF * L.w)));
#pragma unroll
    for (int g = 1; g < s.G; ++g) s.v[g] = s.v[0];
    return s;
}

// The slice as operand fragments.  The 32 features v of wavefronts 2 v and
// 2 v + 1 are four groups of eight k, G0..G3; the products of a sum are
// chained in the order of k_gemm_x3, 32x32x16 products with (G0 G2) and then
// (G1 G3).  Fragment v holds G0 G2 G1 G3 in its quarters: one 16x16x32
// product gives the bits of those two chained (measured on random operands:
// no result differs; any other order of the quarters does).  With `two` (BF16
// models, sums of odd steps apart) fragments 2 u and 2 u + 1 hold (G0 G2) and
// (G1 G3) of the features 2 u and 2 u + 1.  `at`: first fragment at `buf`
// (widths before this one); the atoms a + 16 g of a fragment follow each
// other.
template <int NP, int TA>
__device__ __forceinline__ void put_slice(char* buf, int at, const Lane<TA>& L, const Slice<TA>& s, bool two) {
    const bool apart = NP == 1 && two;
    const int v = L.w >> 1, odd = L.w & 1, half = L.h >> 1;  // group 2 odd + half of v
    const int frag = at + (apart ? (v & 2) + half : v);
    const int unit = (apart ? 2 * (v & 1) + odd : 2 * half + odd) * 16 + L.a;
    char* d = buf + frag * (s.G * NP * kFrag) + unit * 16 + 8 * (L.h & 1);
#pragma unroll
    for (int g = 0; g < s.G; ++g) {
        uint2 o[NP];
        split4<NP>(s.v[g], o);
#pragma unroll
        for (int p = 0; p < NP; ++p) *reinterpret_cast<uint2*>(d + (g * NP + p) * kFrag) = o[p];
    }
}

// Packed weights of one matrix [N][K] (launch_pack_frags): piece p, 16-byte
// unit ((n / 16) K/8 + k / 8) 16 + n % 16 holds W[n][8 (k/8) .. + 7].
// A ring of D steps of the fragments of NT slices of 16 rows: step f is 32 k,
// those of put_slice, of slice f % NT (a ring of whole steps of three slices
// does not fit 128 registers: at 4,800 atoms, where two blocks share CUs, the
// kernels took 41.7 us instead of 39.1).
// KN: steps of 32 k that the product takes (the first of the matrix's KS).
template <int NP, int NT, int KN, int KS, int D, int TA>
struct Weights {
    static constexpr uint32_t kRow = slice_bytes(KS);
    static_assert(KN <= KS, "steps of the matrix");
    Buf b;
    uint32_t ps, off, step, lo;  // bytes: piece, first slice, slice step; lane
    bool apart;
    bf16x8_t r[D][NP];
    // mat: the matrix's pieces, N its rows; slices t0, t0 + st, ...
    __device__ __forceinline__ Weights(const uint16_t* mat, int N, int t0, int st, const Lane<TA>& L, bool two)
        : b(mat, NP * piece_bytes(N, KS)), ps(piece_bytes(N, KS)), off(t0 * kRow), step(st * kRow),
          lo(unit_offset(L.h, L.a, NP == 1 && two)), apart(NP == 1 && two) {
#pragma unroll
        for (int d = 0; d < D - 1; ++d) load(d, d);
    }
    // step f into ring slot d
    __device__ __forceinline__ void load(int f, int d) {
        const uint32_t at = step_offset(f, NT, KN, apart);
#pragma unroll
        for (int p = 0; p < NP; ++p)
            r[d][p] = __builtin_bit_cast(bf16x8_t, b.load(lo, off + (f % NT) * step + p * ps + at));
    }
};

// Steps of weights held: what 128 registers leave room for
template <int NP, int NT, int TA>
constexpr int kDepth = NP == 1 ? 4 * NT : NT == 2 ? 2 : TA == 16 ? 4 : 2;

// acc[t][b] += W_t x_b over all steps; x_b's fragments at buf + b * stride.
// The loads of step f + D - 1 are issued before the products of f and held
// there (left alone, the compiler sinks each load to its use and the chain
// waits for L2 at every step).  A loop over turns of a few steps rather than
// straight-line code: a block walks through its code once, so that code is
// fetched as slowly as data.
//
// FP32 models: where registers allow, the products of the leading pieces are
// summed apart from the five small ones (in `sep`, added by the caller's
// fold), so that a sum is rounded once instead of six times per k-step at
// its full size.
// BF16 models: the sums of k_gemm_x3 bit for bit (its odd k-steps of 16 apart
// in `sep` where it keeps two accumulators, `two`): operands are rounded to
// bfloat16 after every product, and another order would flip some.
template <int NP, int NT, int NB, int TA>
constexpr bool kApart = NP == 3 && (TA == 16 || (NT <= 2 && NT * NB <= 3));

template <int NP, int NT, int NB, int KN, int KS, int D, int TA>
__device__ __forceinline__ void product(Sums<TA> (&acc)[NT][NB], Sums<TA> (&sep)[NT][NB],
                                        Weights<NP, NT, KN, KS, D, TA>& W, const char* buf, int stride,
                                        const Lane<TA>& L) {
    constexpr int G = Sums<TA>::G;
    constexpr int S = KN * NT;                      // steps taken
    // Fragments of x held: with 16 atoms those of all b (and of the next step
    // where there is one b); with 32 atoms one, or with one b the two of an
    // atom pair in turn: more do not fit (the reverse spilled 10 registers).
    constexpr int XD = NB == 1 ? 2 : 1, XB = G > 1 ? 1 : NB;
    constexpr int R0 = std::lcm(D, G > 1 ? NT : XD * NT);  // steps of a turn: whole rings of weights and of x,
    constexpr int R = R0 / NT % 2 ? 2 * R0 : R0;           // an even number of k steps
    static_assert(S % R == 0, "whole rings");
    const char* bl = buf + L.lane * 16;
    bf16x8_t x[XD][XB][NP];
    auto load_x = [&](int k, int u, int d) {  // u: the step's b and g (16 atoms: all b)
#pragma unroll
        for (int b = 0; b < XB; ++b)
#pragma unroll
            for (int p = 0; p < NP; ++p)
                x[d][b][p] = *reinterpret_cast<const bf16x8_t*>(
                    bl + (b + u / G) * stride + ((k * G + u % G) * NP + p) * kFrag);
    };
    if (XD == 2) load_x(0, 0, 0);
    auto step = [&](int f, int d, Sums<TA>(&c)[NT][NB]) {
        W.load(f + D - 1, (d + D - 1) % D);
        const auto& w = W.r[d % D];
        const int t = d % NT;
        // the product of the pieces px of x and pw of w
        auto term = [&](Sums<TA>(&to)[NT][NB], int u, int px, int pw) {
#pragma unroll
            for (int b = 0; b < XB; ++b) {
                auto& o = to[t][b + u / G].c[u % G];
                o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[pw], x[(G > 1 ? u : d / NT) % XD][b][px], o, 0, 0, 0);
            }
        };
#pragma unroll
        for (int u = 0; u < G * (NB / XB); ++u) {
            if (G > 1) {
                const bool last = u + 1 == G * NB;
                if (XD == 1) load_x(f / NT, u, 0);
                else load_x(last ? min((f + 1) / NT, KN - 1) : f / NT, last ? 0 : u + 1, (u + 1) % 2);
            } else if (t == 0) {
                if (XD == 1) load_x(f / NT, 0, 0);
                else load_x(min(f / NT + 1, KN - 1), 0, (d / NT + 1) % 2);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NP == 3) {
                auto& small = kApart<NP, NT, NB, TA> ? sep : c;
                term(small, u, 2, 0);
                term(small, u, 0, 2);
                term(small, u, 1, 1);
                term(small, u, 1, 0);
                term(small, u, 0, 1);
            }
            term(c, u, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (NP == 3 || !W.apart) {
#pragma unroll 1
        for (int k0 = 0; k0 < S; k0 += R)
#pragma unroll
            for (int d = 0; d < R; ++d) step(k0 + d, d, acc);
    } else {
#pragma unroll 1
        for (int k0 = 0; k0 < S; k0 += R)
#pragma unroll
            for (int d = 0; d < R; ++d) step(k0 + d, d, (d / NT) % 2 ? sep : acc);
    }
}

// Whether k_gemm_x3 sums odd k-steps apart in the product [M][N] of K = 128
// (for other K it always does): where it gives a block 32 columns, i.e. where
// 64 would leave fewer than 512 blocks.
__host__ __device__ __forceinline__ bool two_sums(int64_t M, int N) { return (M + 127) / 128 * (N / 64) < 512; }

template <int NT, int NB, int TA>
__device__ __forceinline__ void fold(Sums<TA> (&acc)[NT][NB], const Sums<TA> (&sep)[NT][NB]) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[t][b].add(sep[t][b]);
}
// acc = W x
template <int NP, int NT, int NB, int KN, int KS, int D, int TA>
__device__ __forceinline__ void product(Sums<TA> (&acc)[NT][NB], Weights<NP, NT, KN, KS, D, TA>& W, const char* buf,
                                        int stride, const Lane<TA>& L) {
    Sums<TA> sep[NT][NB];
    product<NP, NT, NB>(acc, sep, W, buf, stride, L);
    if (NP == 1 || kApart<NP, NT, NB, TA>) fold(acc, sep);
}

template <int TA>
__device__ __forceinline__ Slice<TA> as_slice(const Sums<TA>& c) {
    Slice<TA> s;
#pragma unroll
    for (int e = 0; e < 4 * s.G; ++e) s.v[e >> 2][e & 3] = c[e];
    return s;
}
// Biases, and the adjoints that pass a product by, are added to it last:
// started from them, every partial sum is rounded at their size (forces then
// were 1 % further off float64 than with separate products, now 1 % closer),
// and BF16 models would not have the bits of k_gemm_x3.
template <int TA>
__device__ __forceinline__ Slice<TA> added(const Sums<TA>& c, const Slice<TA>& b) {
    Slice<TA> s = as_slice(c);
#pragma unroll
    for (int g = 0; g < s.G; ++g) s.v[g] += b.v[g];
    return s;
}

// ---------------------------------------------------------------- forward --
// smid, vmid (the message step's outputs) -> update block -> s, v; then
//   LAST = false: phi = W2 silu(W1 s + b1) + b2 of the next layer, and
//                 phi_b v for its message kernels;
//   LAST = true:  the readout, the atomic energy and the adjoint of s of the
//                 energy (v is not used past the last layer: not formed).
//   FIRST (FP32 models, first layer by species): smid and vmid are the edge
//   sums by species, rows E and U of 128 slots; s = T_0 E and v = T_2 U come
//   first (v_keep: v, read again later).  As launches of their own this
//   layer's products, here and in the reverse, took 47 us at 12,288 atoms and 16
//   at 1,536 (more where n is not a multiple of 128); in the blocks 20 and 8.
// Kept for the reverse: U v and V v, the M1 pre-activation, q and o (LAST: q
// alone), the W1 pre-activation.
template <int NP, int TA, bool LAST, bool FIRST>
__global__ void __launch_bounds__(64 * kW, 4) k_atom_fwd(AtomFwd A) {
    extern __shared__ __align__(16) char lds[];
    __shared__ float epart[LAST ? 4 : 1][TA], ehalf[LAST ? 8 : 1][TA];
    constexpr int CB = kRegion<NP, TA>, E = 4 * Slice<TA>::G;
    const Lane<TA> L(A.n);
    // (tiles of 32 are for sizes where k_gemm_x3 had one sum in the first two)
    const bool two_uv = TA == 16 && two_sums(3 * int64_t(A.n), 2 * kF);
    const bool two_3 = TA == 16 && two_sums(A.n, 3 * kF), two_1 = two_sums(A.n, kF);
    // free while the rows of s and v (turn) and the outputs (turn2) are written
    char* turn = lds + CB + L.w * kTurn<TA>;
    char* turn2 = lds + 2 * CB + L.w * kTurn<TA>;
    Slice<TA> s0;
    {
        Slice<TA> v0[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) v0[c] = load_slice<3, kF>(A.vmid, c, 0, L);
#pragma unroll
        for (int c = 0; c < 3; ++c) put_slice<NP>(lds + c * CB, 0, L, v0[c], two_uv);
        s0 = load_slice<1, kF>(A.smid, 0, 0, L);
        if constexpr (FIRST) {
            // v = T_2 U, then s = T_0 E, by way of the same regions
            {
                Sums<TA> sums[1][3];
                Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W(A.T2, kF, L.w, 1, L, false);
                __syncthreads();
                product<NP, 1, 3>(sums, W, lds, CB, L);
#pragma unroll
                for (int c = 0; c < 3; ++c) v0[c] = as_slice(sums[0][c]);
            }
            if constexpr (!LAST) {
#pragma unroll
                for (int c = 0; c < 3; ++c) keep_slice<3>(A.v_keep, c, L, v0[c]);
            }
            Sums<TA> sums[1][1];
            Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W(A.T0, kF, L.w, 1, L, false);
            __syncthreads();  // the rows of U are read
            put_slice<NP>(lds, 0, L, s0, false);
#pragma unroll
            for (int c = 1; c < 3; ++c) put_slice<NP>(lds + c * CB, 0, L, v0[c], two_uv);
            __syncthreads();
            product<NP, 1, 1>(sums, W, lds, 0, L);
            s0 = as_slice(sums[0][0]);
            __syncthreads();  // the rows of E are read
            put_slice<NP>(lds, 0, L, v0[0], two_uv);
        }
    }

    // U v, V v: slices w of U and of V, of the adjacent matrices
    Sums<TA> uv[2][3];
    {
        Weights<NP, 2, kKsF, kKsF, kDepth<NP, 2, TA>, TA> W(A.U, 2 * kF, L.w, kW, L, two_uv);
        __syncthreads();
        product<NP, 2, 3>(uv, W, lds, CB, L);
    }
    Slice<TA> nrm, dot;
#pragma unroll
    for (int g = 0; g < E / 4; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = 4 * g + q;
            float nn = 1e-8f, dd = 0.f;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                nn = fmaf(uv[1][c][e], uv[1][c][e], nn);
                dd = fmaf(uv[0][c][e], uv[1][c][e], dd);
            }
            nrm.v[g][q] = sqrtf(nn);
            dot.v[g][q] = dd;
        }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < 2; ++m)
            keep_slice<6>(A.UV, 2 * c + m, L, as_slice(uv[m][c]));
    // [s; |V v|] (k-steps 0..15), then M1; its output behind them (16..23)
    Slice<TA> z;
    {
        Sums<TA> acc[1][1];
        Weights<NP, 1, 2 * kKsF, 2 * kKsF, kDepth<NP, 1, TA>, TA> W(A.M1, kF, L.w, 1, L, true);
        __syncthreads();  // the vector fragments are read
        put_slice<NP>(lds, 0, L, s0, true);
        put_slice<NP>(lds, kKsF, L, nrm, true);
        __syncthreads();
        product<NP, 1, 1>(acc, W, lds, 0, L);
        const Slice<TA> a1 = added(acc[0][0], load_feat(A.m1, L));
        keep_slice<1>(A.a1, 0, L, a1);
#pragma unroll
        for (int e = 0; e < E; ++e) z.v[e >> 2][e & 3] = silu(a1[e]);
    }
    put_slice<NP>(lds + 2 * CB, 0, L, z, two_3);
    // p, q, o
    constexpr int NQ = LAST ? 2 : 3;
    Slice<TA> s1;
    Slice<TA> v1[3];
    {
        Sums<TA> acc[NQ][1];
        Weights<NP, NQ, kKsF, kKsF, kDepth<NP, NQ, TA>, TA> W(A.M2, 3 * kF, L.w, kW, L, two_3);
        __syncthreads();
        product<NP, NQ, 1>(acc, W, lds + 2 * CB, 0, L);
        Slice<TA> h[NQ];
#pragma unroll
        for (int c = 0; c < NQ; ++c) h[c] = added(acc[c][0], load_feat(A.m2 + c * kF, L));
#pragma unroll
        for (int c = 1; c < NQ; ++c) keep_slice<3>(A.pqo, c, L, h[c]);
#pragma unroll
        for (int e = 0; e < E; ++e) s1.v[e >> 2][e & 3] = fmaf(h[1][e], dot[e], s0[e] + h[0][e]);
        if constexpr (!LAST) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                // v and U v are read again rather than held over the products
                // (96 registers)
                Slice<TA> v0;
                if constexpr (FIRST) v0 = kept_slice<3>(A.v_keep, c, L);
                else v0 = load_slice<3, kF>(A.vmid, c, 0, L);
                const Slice<TA> u = kept_slice<6>(A.UV, 2 * c, L);
#pragma unroll
                for (int e = 0; e < E; ++e) v1[c].v[e >> 2][e & 3] = fmaf(h[NQ - 1][e], u[e], v0[e]);
                store_slice<3, kF>(A.v_out, c, 0, L, v1[c], turn);
            }
        }
    }
    // the s fragments of M1 are read (the barrier before M2's product)
    put_slice<NP>(lds, 0, L, s1, two_1);
    Sums<TA> acc1[1][1];
    Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W1(A.W1, kF, L.w, 1, L, two_1);
    __syncthreads();
    product<NP, 1, 1>(acc1, W1, lds, 0, L);
    const Slice<TA> h1 = added(acc1[0][0], load_feat(A.b1, L));
    if constexpr (!LAST) {
        keep_slice<1>(A.h1, 0, L, h1);
#pragma unroll
        for (int e = 0; e < E; ++e) z.v[e >> 2][e & 3] = silu(h1[e]);
        put_slice<NP>(lds + CB, 0, L, z, two_3);
        Sums<TA> acc[3][1];
        Weights<NP, 3, kKsF, kKsF, kDepth<NP, 3, TA>, TA> W2(A.W2, 3 * kF, L.w, kW, L, two_3);
        __syncthreads();
        product<NP, 3, 1>(acc, W2, lds + CB, 0, L);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Slice<TA> ph = added(acc[c][0], load_feat(A.b2 + c * kF, L));
            store_slice<1, 3 * kF>(A.phi, 0, c * kF, L, ph, turn2);
            if (c == 1 && A.pv) {
#pragma unroll
                for (int al = 0; al < 3; ++al) {
                    Slice<TA> t;
#pragma unroll
                    for (int g = 0; g < E / 4; ++g) t.v[g] = ph.v[g] * v1[al].v[g];
                    store_slice<3, kF>(A.pv, al, 0, L, t, turn2);
                }
            }
        }
        store_slice<1, kF>(A.s_out, 0, 0, L, s1, turn2);
    } else {
        // E_i = wo . silu(h1) + beta[t_i]; adjoint of s: Wo^T (wo silu'(h1))
        const Slice<TA> wo = load_feat(A.wo, L);
        Slice<TA> y;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            y.v[e >> 2][e & 3] = silu(h1[e]);
            z.v[e >> 2][e & 3] = wo[e] * silu_grad(h1[e]);
        }
        // The sum over 32 features: the groups of four 0, 2, 4, 6 and 1, 3,
        // 5, 7, then the two sums.  Groups 0 to 3 are in the four lanes of an
        // atom of an even wavefront and 4 to 7 in those of the next one,
        // which takes the two sums over and goes on.
        auto pair_sum = [&](float e0, int g) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                if (r) e0 = __shfl_xor(e0, 32, 64);
#pragma unroll
                for (int q = 0; q < 4; ++q) e0 = fmaf(wo.v[g][q], y.v[g][q], e0);
            }
            return e0;
        };
        if (!(L.w & 1)) {
#pragma unroll
            for (int g = 0; g < E / 4; ++g) {
                const float e0 = pair_sum(0.f, g);
                if (L.h >= 2) ehalf[L.w + L.h - 2][16 * g + L.a] = e0;
            }
        }
        put_slice<NP>(lds + CB, 0, L, z, two_1);
        Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W2(A.W2, kF, L.w, 1, L, two_1);
        __syncthreads();
        if (L.w & 1) {
#pragma unroll
            for (int g = 0; g < E / 4; ++g) {
                float e0 = pair_sum(ehalf[L.w - 1 + (L.h & 1)][16 * g + L.a], g);
                e0 += __shfl_xor(e0, 16, 64);
                if (L.h == 2) epart[L.w >> 1][16 * g + L.a] = e0;
            }
        }
        Sums<TA> acc[1][1];
        product<NP, 1, 1>(acc, W2, lds + CB, 0, L);
        __syncthreads();
        const int r = L.lane, i = int(L.t0) + r;
        if (L.w == 0 && r < L.rows) {
            const int io = A.perm ? min(max(A.perm[i], 0), A.n - 1) : i;
            const float sum = (epart[0][r] + epart[1][r]) + (epart[2][r] + epart[3][r]);
            A.Ei[io] = sum + A.beta[min(max(A.species[i], 0), A.n_species - 1)];
        }
        store_slice<1, kF>(A.s_out, 0, 0, L, as_slice(acc[0][0]), turn2);
    }
}

// ---------------------------------------------------------------- reverse --
// Adjoints of (s, v) after a layer -> adjoints of its message step's outputs
// (gs_out of smid, gv_out of vmid).
//   TOP = false: the adjoint of s is first completed from that of the next
//     layer's phi, gs = gs_in + W1^T (silu'(h1) W2^T gphi); gs_in is the
//     adjoint that passes that layer's message step by.
//   TOP = true (the last layer): gs_in is the adjoint of s, that of v is zero.
//   BOTTOM (with FIRST): instead of gs_out and gv_out the rows P_0 and P_2 (128
//   slots, the first pp used) that k_sp_bwd_own takes (keep: room for g_s).
template <int NP, int TA, bool TOP, bool BOTTOM>
__global__ void __launch_bounds__(64 * kW, 4) k_atom_bwd(AtomBwd A) {
    extern __shared__ __align__(16) char lds[];
    constexpr int CB = kRegion<NP, TA>, E = 4 * Slice<TA>::G;
    const Lane<TA> L(A.n);
    const bool two_1 = two_sums(A.n, kF), two_2 = two_sums(A.n, 2 * kF);
    char* turn = lds + CB + L.w * kTurn<TA>;
    Slice<TA> gs = load_slice<1, kF>(A.gs_in, 0, 0, L);
    if constexpr (!TOP) {
        Weights<NP, 1, 3 * kKsF, 3 * kKsF, kDepth<NP, 1, TA>, TA> W(A.W2t, kF, L.w, 1, L, true);
        const Slice<TA> h1 = kept_slice<1>(A.h1, 0, L);
#pragma unroll
        for (int c = 0; c < 3; ++c)
            put_slice<NP>(lds, c * kKsF, L, load_slice<1, 3 * kF>(A.gphi, 0, c * kF, L), true);
        __syncthreads();
        Sums<TA> acc[1][1];
        product<NP, 1, 1>(acc, W, lds, 0, L);
        Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W1(A.W1t, kF, L.w, 1, L, two_1);
        Slice<TA> g;
#pragma unroll
        for (int e = 0; e < E; ++e) g.v[e >> 2][e & 3] = acc[0][0][e] * silu_grad(h1[e]);
        __syncthreads();
        put_slice<NP>(lds, 0, L, g, two_1);
        __syncthreads();
        Sums<TA> acc1[1][1];
        product<NP, 1, 1>(acc1, W1, lds, 0, L);
        gs = added(acc1[0][0], gs);
    }
    // adjoints of p, q (and o): gs, gs (U v . V v), sum gv U v
    Slice<TA> gsq, o, dot, go;
    Slice<TA> gv[3];
    {
        constexpr int KN = (TOP ? 2 : 3) * kKsF;
        Weights<NP, 1, KN, 3 * kKsF, kDepth<NP, 1, TA>, TA> W(A.M2t, kF, L.w, 1, L, true);
        const Slice<TA> q = kept_slice<3>(A.pqo, 1, L);
        if constexpr (!TOP) o = kept_slice<3>(A.pqo, 2, L);
#pragma unroll
        for (int g = 0; g < E / 4; ++g) gsq.v[g] = gs.v[g] * q.v[g];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Slice<TA> u = kept_slice<6>(A.UV, 2 * c, L), v = kept_slice<6>(A.UV, 2 * c + 1, L);
            if constexpr (!TOP) gv[c] = load_slice<3, kF>(A.gv_in, c, 0, L);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float d = c ? dot[e] : 0.f;
                dot.v[e >> 2][e & 3] = fmaf(u[e], v[e], d);
                if constexpr (!TOP) {
                    const float t = c ? go[e] : 0.f;
                    go.v[e >> 2][e & 3] = fmaf(gv[c][e], u[e], t);
                }
            }
        }
#pragma unroll
        for (int g = 0; g < E / 4; ++g) dot.v[g] = gs.v[g] * dot.v[g];
        if constexpr (!TOP) __syncthreads();  // W1's input is read
        put_slice<NP>(lds, 0, L, gs, true);
        put_slice<NP>(lds, kKsF, L, dot, true);
        if constexpr (!TOP) put_slice<NP>(lds, 2 * kKsF, L, go, true);
        const Slice<TA> a1 = kept_slice<1>(A.a1, 0, L);
        __syncthreads();
        Sums<TA> acc[1][1];
        product<NP, 1, 1>(acc, W, lds, 0, L);
#pragma unroll
        for (int e = 0; e < E; ++e) dot.v[e >> 2][e & 3] = acc[0][0][e] * silu_grad(a1[e]);
    }
    // M1^T: adjoints of s (added to gs) and of |V v|
    Slice<TA> gn;
    {
        Weights<NP, 2, kKsF, kKsF, kDepth<NP, 2, TA>, TA> W(A.M1t, 2 * kF, L.w, kW, L, two_2);
        __syncthreads();
        put_slice<NP>(lds, 0, L, dot, two_2);
        __syncthreads();
        Sums<TA> acc[2][1];
        product<NP, 2, 1>(acc, W, lds, 0, L);
        gn = as_slice(acc[1][0]);
        if constexpr (BOTTOM) keep_slice<3>(A.keep, 0, L, added(acc[0][0], gs));
        else store_slice<1, kF>(A.gs_out, 0, 0, L, added(acc[0][0], gs), turn);
    }
    // adjoints of U v and V v, one after the other through the same regions:
    // g_vmid = gv + [gU gV] [U; V], gv (48 registers) read again at the end
    Sums<TA> sums[1][3], sep[1][3];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W(m ? A.Vt : A.Ut, kF, L.w, 1, L, true);
        __syncthreads();
        Slice<TA> nn;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Slice<TA> v = kept_slice<6>(A.UV, 2 * c + 1, L);
            Slice<TA> t;
            if (m == 0) {
                if constexpr (!TOP && TA == 32) {  // read again rather than held over the products
                    gv[c] = load_slice<3, kF>(A.gv_in, c, 0, L);
                    if (c == 0) o = kept_slice<3>(A.pqo, 2, L);
                }
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    nn.v[e >> 2][e & 3] = fmaf(v[e], v[e], c ? nn[e] : 1e-8f);
                    t.v[e >> 2][e & 3] = TOP ? gsq[e] * v[e] : fmaf(gsq[e], v[e], gv[c][e] * o[e]);
                }
            } else {
                const Slice<TA> u = kept_slice<6>(A.UV, 2 * c, L);
#pragma unroll
                for (int e = 0; e < E; ++e) t.v[e >> 2][e & 3] = fmaf(gn[e], v[e], gsq[e] * u[e]);
            }
            put_slice<NP>(lds + c * CB, 0, L, t, true);
        }
        if (m == 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) gn.v[e >> 2][e & 3] = gn[e] / sqrtf(nn[e]);
        }
        __syncthreads();
        product<NP, 1, 3>(sums, sep, W, lds, CB, L);
    }
    fold(sums, sep);
    __syncthreads();
    Slice<TA> gvo[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        gvo[c] = TOP ? as_slice(sums[0][c]) : added(sums[0][c], load_slice<3, kF>(A.gv_in, c, 0, L));
    if constexpr (!BOTTOM) {
#pragma unroll
        for (int c = 0; c < 3; ++c) store_slice<3, kF>(A.gv_out, c, 0, L, gvo[c], turn);
    } else {
        // P_2 = T_2^T g_v, then P_0 = T_0^T g_s; wavefront w has the slots
        // kWF w .. of the pp ones
        const bool on = kWF * L.w < A.pp;
        const int t = slice_within(L.w, A.pp);
#pragma unroll
        for (int c = 0; c < 3; ++c) put_slice<NP>(lds + c * CB, 0, L, gvo[c], false);
        {
            Sums<TA> p[1][3];
            Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W(A.TT2, A.pp, t, 1, L, false);
            __syncthreads();
            if (on) product<NP, 1, 3>(p, W, lds, CB, L);
            __syncthreads();  // read: region 1 is the room to turn again
            if (on) {
#pragma unroll
                for (int c = 0; c < 3; ++c) store_slice<3, kF>(A.P2, c, 0, L, as_slice(p[0][c]), turn);
            }
        }
        Sums<TA> p[1][1];
        Weights<NP, 1, kKsF, kKsF, kDepth<NP, 1, TA>, TA> W(A.TT0, A.pp, t, 1, L, false);
        put_slice<NP>(lds, 0, L, kept_slice<3>(A.keep, 0, L), false);
        __syncthreads();
        if (on) {
            product<NP, 1, 1>(p, W, lds, 0, L);
            store_slice<1, kF>(A.P0, 0, 0, L, as_slice(p[0][0]), turn);
        }
    }
}

// ---------------------------------------------------------- weight packing --
// One 16-byte unit (eight k of one row) per thread and matrix: dst piece p,
// unit ((n / 16) K/8 + k8) 16 + n % 16.  With `tr` the matrix is the
// transpose of the stored one ([K][N] row-major).
__global__ void __launch_bounds__(256) k_pack_frags(PackFrags P, int np) {
    const PackFrags::Mat m = P.m[blockIdx.y];
    const int k8n = m.K / 8;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= m.N * k8n) return;
    const int n = (t / (16 * k8n)) * 16 + t % 16, k8 = (t / 16) % k8n;
    __bf16* dst = reinterpret_cast<__bf16*>(m.dst) + int64_t(t) * 8;
    const int64_t ps = int64_t(m.N) * m.K;
    for (int q = 0; q < 8; ++q) {
        const int k = 8 * k8 + q;
        float x = m.tr ? m.src[int64_t(k) * m.N + n] : m.src[int64_t(n) * m.K + k];
        for (int p = 0; p < np; ++p) {
            const __bf16 b = __bf16(x);
            dst[p * ps + q] = b;
            x -= float(b);
        }
    }
}

template <int NP, int TA, typename K, typename Args>
void launch_block(K kern, const Args& a, hipStream_t s) {
    kern<<<cdiv(a.n, TA), 64 * kW, kLdsBytes<NP, TA>, s>>>(a);
    NNP_LAUNCH_CHECK();
}

// more than 64 KB of dynamic LDS: raise the limit of each instance once per
// device (the first call of a process on it; an idempotent setting)
template <typename K>
void raise_lds(K kern) {
    NNP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLdsBytes<3, 32>));
}

// 16 atoms to a block or 32.  Measured (reverse / forward of a middle layer,
// us): FP32, 1,536 atoms 21.7 / 19.6 with 16 against 30 / 27 with 32; 4,096:
// 27 / 26 against 32 / 30; 5,121: 39 / 38 with 16, 5,421: 39 / 37 with 32;
// 6,144: 41 / 43 against 40 / 41; 12,288: 72 / 75 against 69 / 65.  BF16, a
// third of the weights: 1,536 13.3 / 12.8 against 21 / 20; 8,192 28 / 31
// against 38 / 36; over an evaluation's blocks 11,100 39 / 41 against 44 / 41,
// 12,288 41.5 / 43.6 against 45.2 / 41.7, 23,700 77 against 72 and 48,000
// 148 against 135.  BF16 results are the same bits
// with both.  FP32 ones are not (the order of the six piece products): they
// change tiles where k_gemm_x3 changed its number of sums for the widest of
// these products, close to where the two are equal, so that replicas give the
// same bits alone and packed up to the same total as with it.
bool small_tiles(int n, bool bf16) { return bf16 ? n <= 3 * 256 * 16 : two_sums(3 * int64_t(n), 2 * kF); }

template <int NP, int TA>
void launch_fwd(const AtomFwd& a, bool last, hipStream_t s) {
    if constexpr (NP == 3) {
        if (a.T0) {
            if (last) launch_block<NP, TA>(k_atom_fwd<NP, TA, true, true>, a, s);
            else launch_block<NP, TA>(k_atom_fwd<NP, TA, false, true>, a, s);
            return;
        }
    }
    if (last) launch_block<NP, TA>(k_atom_fwd<NP, TA, true, false>, a, s);
    else launch_block<NP, TA>(k_atom_fwd<NP, TA, false, false>, a, s);
}
template <int NP, int TA>
void launch_bwd(const AtomBwd& a, bool top, hipStream_t s) {
    if constexpr (NP == 3) {
        if (a.TT0) {
            if (top) launch_block<NP, TA>(k_atom_bwd<NP, TA, true, true>, a, s);
            else launch_block<NP, TA>(k_atom_bwd<NP, TA, false, true>, a, s);
            return;
        }
    }
    if (top) launch_block<NP, TA>(k_atom_bwd<NP, TA, true, false>, a, s);
    else launch_block<NP, TA>(k_atom_bwd<NP, TA, false, false>, a, s);
}

}  // namespace

void launch_pack_frags(const PackFrags& P, int count, int np, hipStream_t s) {
    int most = 0;
    for (int k = 0; k < count; ++k) most = std::max(most, P.m[k].N * P.m[k].K / 8);
    k_pack_frags<<<dim3(cdiv(most, 256), count), 256, 0, s>>>(P, np);
    NNP_LAUNCH_CHECK();
}

void atom_block_setup() {
    raise_lds(k_atom_fwd<3, 32, false, false>);
    raise_lds(k_atom_fwd<3, 32, true, false>);
    raise_lds(k_atom_fwd<3, 32, false, true>);
    raise_lds(k_atom_fwd<3, 32, true, true>);
    raise_lds(k_atom_bwd<3, 32, false, false>);
    raise_lds(k_atom_bwd<3, 32, true, false>);
    raise_lds(k_atom_bwd<3, 32, false, true>);
    raise_lds(k_atom_bwd<3, 32, true, true>);
}

void launch_atom_fwd(const AtomFwd& a, bool last, bool bf16, hipStream_t s) {
    if (a.n <= 0) return;
    ScopedTimer timer("gemm", s);
    if (small_tiles(a.n, bf16)) bf16 ? launch_fwd<1, 16>(a, last, s) : launch_fwd<3, 16>(a, last, s);
    else bf16 ? launch_fwd<1, 32>(a, last, s) : launch_fwd<3, 32>(a, last, s);
}

void launch_atom_bwd(const AtomBwd& a, bool top, bool bf16, hipStream_t s) {
    if (a.n <= 0) return;
    ScopedTimer timer("gemm", s);
    if (small_tiles(a.n, bf16)) bf16 ? launch_bwd<1, 16>(a, top, s) : launch_bwd<3, 16>(a, top, s);
    else bf16 ? launch_bwd<1, 32>(a, top, s) : launch_bwd<3, 32>(a, top, s);
}

}  // namespace nnp
