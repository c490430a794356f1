// Embedding of the NC model (paper, Methods: one message step, the update
// block, then q_ih, k_ih and V_ih), widths up to 32, as one kernel: the first
// layer's message needs only positions and species, so the message, the
// update and the projections of an atom need nothing of its neighbours'
// features.
//
// A block of eight (four up to 16 features) wavefronts owns 16 atoms.
//   Messages (each wavefront its own two or four atoms, whose list rows are
//   one run of entries): in chunks of 64 or 128 entries, the float64 pair rule with lanes
//   over entries, the edges that pass compacted in list order into LDS; their
//   radial values with lanes over edges; then lanes over features, one atom
//   per F lanes, every edge added in list order.
//   Update and projections: on the float32 matrix cores
//   (v_mfma_f32_16x16x4_f32, which adds its four products one after the other
//   in k with one rounding each, like a chain of fused multiply-adds), the
//   weights as the first operand, so that lane (atom a = lane % 16, q = lane / 16)
//   holds features 16 t + 4 q + i (i < 4) of atom a.  Every sum runs over k in
//   increasing order; for BF16 models weights and inputs are rounded to
//   bfloat16 first.
// Bound by the chain of a block's steps (a block alone takes 10 us, vector
// instructions issue a third of the time at 12,288 atoms).  As two kernels (message;
// update with weights and inputs read from LDS for plain multiply-adds) with
// s and v of the message step through memory, 12,288 atoms took 18.0 + 21.9
// us; now 24.6 (192 atoms at width 16: 8.8 + 8.8 -> 8.9).
#include "common.h"
#include "kernels.h"
#include "mp_edge.h"

namespace nnp {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kK = 8;                                    // Bessel functions of the filter
constexpr int kHC = 160, kNl = 2;                        // q and k outputs, vector heads
constexpr int kAtoms = 16;                               // atoms of a block

constexpr int pad16(int x) { return (x + 15) / 16 * 16; }

// Packed weights: row tiles of 16 (zero rows past the last), k in blocks of
// 16 (zero past the last); the 16-byte unit of lane (row r = lane % 16,
// q = lane / 16) holds k = 16 kb + 4 s + q, s < 4, the operands of four
// matrix instructions.  Order of the row tiles: U, V, M1 (k = 2F), p, q, o of
// M2, the projections, the vector heads.
template <int F>
struct Pack {
    static constexpr int T = pad16(F) / 16;              // row tiles of a width
    static constexpr int KB = pad16(F) / 16, KB2 = pad16(2 * F) / 16;
    static constexpr int UNIT = 256;                     // floats per tile and k block
    static constexpr int oU = 0, oV = oU + T * KB, oM1 = oV + T * KB, oM2 = oM1 + T * KB2, oQ = oM2 + 3 * T * KB,
                         oWV = oQ + kHC / 16 * KB, total = oWV + KB;
};

__device__ __forceinline__ float bf16_round(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xFFFF0000u);
}

// Inputs of the products in LDS: element (k, atom) of a K x 16 array, in the
// order the lanes of an instruction read it
__device__ __forceinline__ int at(int k, int atom) { return (((k >> 4) * 4 + (k & 3)) * 16 + atom) * 4 + ((k & 15) >> 2); }

// acc += W_tile x over KB blocks of k
template <int KB, bool BF16>
__device__ __forceinline__ void product(f32x4_t& acc, const f32x4_t* w, const float* x, int lane) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const f32x4_t b = *reinterpret_cast<const f32x4_t*>(x + kb * 256 + lane * 4);
#pragma unroll
        for (int s = 0; s < 4; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[kb][s], BF16 ? bf16_round(b[s]) : b[s], acc, 0, 0, 0);
    }
}

template <int KB>
__device__ __forceinline__ void load_tile(f32x4_t (&w)[KB], const float* wt, int unit, int lane) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
        w[kb] = *reinterpret_cast<const f32x4_t*>(wt + (unit + kb) * 256 + lane * 4);
}

// One edge of the chunk in LDS, 64 bytes: the radial values (before them, in
// their place: dx, dy, dz, r^2 and the neighbour), f, u and the neighbour's
// species; pad.
struct Slot {
    float ef[kK];
    float fc, u[3];
    int t, owner, pad[2];
};

template <int F, bool BF16, int kWaves>
__global__ void __launch_bounds__(64 * kWaves, kWaves == 4 ? 3 : 4) k_nc_embed(MpGeom mg, NcEmbedArgs A) {
    using P = Pack<F>;
    constexpr int kPer = kAtoms / kWaves;                // atoms of a wavefront
    constexpr int kChunk = kWaves == 4 ? 128 : 64;       // list entries per wavefront and chunk
    constexpr int FL = F < 16 ? 16 : F;        // lanes per atom in the feature step
    constexpr int G = 64 / FL, R = kPer > G ? kPer / G : 1;  // atoms at a time, rounds
    constexpr int KV = pad16(F), KX = pad16(2 * F);
    __shared__ __align__(16) Slot slot_s[kWaves][kChunk];
    __shared__ __align__(16) float xs[KX * 16];       // [s; |V v|]; s alone before it
    __shared__ __align__(16) float vs[3][KV * 16];    // v, then v after the update
    __shared__ __align__(16) float zs[KV * 16], ss[KV * 16];  // hidden; s after the update
    __shared__ double own_s[kWaves][kPer][5];         // x, y, z, L, 1/L of the owners
    __shared__ float phi_s[8][2][FL];                 // a and c channels of phi per species
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = mg.n;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int ib = blk * kAtoms, i0 = ib + w * kPer;
    auto rnd = [](float x) { return BF16 ? bf16_round(x) : x; };

    // ---------------------------------------------------------- messages --
    for (int t = threadIdx.x; t < mg.n_species * 2 * FL; t += 64 * kWaves) {
        const int sp = t / (2 * FL), c = t / FL % 2, f = t % FL;
        phi_s[sp][c][f] = f < F ? A.phi_tab[sp * 3 * F + c * 2 * F + f] : 0.f;
    }
    if (lane < kPer) {
        const int i = min(i0 + lane, n - 1);
        double L, inv;
        mg.geom.get(i, L, inv);
        double* o = own_s[w][lane];
        o[0] = mg.pos[i];
        o[1] = mg.pos[n + i];
        o[2] = mg.pos[2 * n + i];
        o[3] = L;
        o[4] = inv;
    }
    int row[kPer + 1];
#pragma unroll
    for (int r = 0; r <= kPer; ++r) row[r] = __builtin_amdgcn_readfirstlane(mg.off[min(i0 + r, n)]);
    const int f = lane % FL, g = lane / FL;
    float wa[kK], wc[kK], ba, bc;
    {
        const int fr = min(f, F - 1);
#pragma unroll
        for (int k = 0; k < kK; ++k) {
            wa[k] = A.Wr[fr * kK + k];
            wc[k] = A.Wr[(2 * F + fr) * kK + k];
        }
        ba = A.br[fr];
        bc = A.br[2 * F + fr];
    }
    __syncthreads();  // the species table
    Slot* slot = slot_s[w];
    float sacc[R] = {}, vacc[R][3] = {};
    int found[kPer] = {};  // edges of each owner in earlier chunks
    for (int cb = row[0]; cb < row[kPer]; cb += kChunk) {
        const int ce = min(row[kPer], cb + kChunk);
        int tot = 0, seg[kPer] = {};  // edges of the chunk up to and including owner r
#pragma unroll
        for (int p = 0; p < kChunk / 64; ++p) {
            const int eb = cb + 64 * p, e = eb + lane;
            bool ok = false;
            double dx = 0, dy = 0, dz = 0;
            int j = -1, r = 0;
            if (e < ce) {
                j = mg.nbr[e];
#pragma unroll
                for (int q = 1; q < kPer; ++q) r += e >= row[q] ? 1 : 0;
                const double* o = own_s[w][r];
                ok = pair_rule(o[0], o[1], o[2], mg.pos[j], mg.pos[n + j], mg.pos[2 * n + j], o[3], o[4], mg.rc2, dx,
                               dy, dz);
            }
            const uint64_t bal = __ballot(ok);
            if (ok) {
                Slot& s = slot[tot + __popcll(bal & ((1ull << lane) - 1ull))];
                const float r2 = float((dx * dx + dy * dy) + dz * dz);
                s.ef[0] = float(dx);
                s.ef[1] = float(dy);
                s.ef[2] = float(dz);
                s.ef[3] = r2;
                s.t = j;
                s.owner = r;
            }
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int nb = min(max(row[q + 1] - eb, 0), 64);
                seg[q] += __popcll(nb == 64 ? bal : bal & ((1ull << nb) - 1ull));
            }
            tot += __popcll(bal);
        }
        wave_sync_lds();
        for (int x = lane; x < tot; x += 64) {
            Slot& s = slot[x];
            const float dx = s.ef[0], dy = s.ef[1], dz = s.ef[2];
            const float r = sqrtf(s.ef[3]);
            const int j = s.t, o = s.owner;
            const float ir = 1.f / r;
            float ef[kK], fc;
            radial_poly_f32<kK>(r * float(mg.inv_rc), float(mg.bessel_norm) * ir, ef, fc);
            const float u[3] = {dx * ir, dy * ir, dz * ir};
#pragma unroll
            for (int k = 0; k < kK; ++k) s.ef[k] = ef[k];
            s.fc = fc;
            s.u[0] = u[0];
            s.u[1] = u[1];
            s.u[2] = u[2];
            s.t = min(max(mg.species[j], 0), mg.n_species - 1);
            if (A.edge_out) {
                // rank among the owner's edges: earlier chunks, then this one
                int rank = x + found[0], start = row[0];
#pragma unroll
                for (int q = 1; q < kPer; ++q)
                    if (o == q) {
                        rank = x - seg[q - 1] + found[q];
                        start = row[q];
                    }
                NcEdge rec;
                rec.j = j;
                rec.r = r;
#pragma unroll
                for (int a = 0; a < 3; ++a) rec.u[a] = u[a];
                rec.pad[0] = rec.pad[1] = rec.pad[2] = 0.f;
#pragma unroll
                for (int k = 0; k < kK; ++k) rec.ef[k] = ef[k];
                A.edge_out[start + rank] = rec;
            }
        }
        wave_sync_lds();
        // lane (g, f): feature f of owners g, G + g, ...
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
            int t0 = 0, t1 = 0;
#pragma unroll
            for (int q = 0; q < kPer; ++q)
                if (q / G == rr && q % G == g) {
                    t0 = q ? seg[q > 0 ? q - 1 : 0] : 0;
                    t1 = seg[q];
                }
#pragma unroll 2
            for (int t = t0; t < t1; ++t) {
                const Slot& s = slot[t];
                const float fc = s.fc;
                const float pa = phi_s[s.t][0][f], pc = phi_s[s.t][1][f];
                float a = ba * fc, c = bc * fc;
#pragma unroll
                for (int k = 0; k < kK; ++k) {
                    a = fmaf(wa[k], s.ef[k], a);
                    c = fmaf(wc[k], s.ef[k], c);
                }
                c = pc * c;
                sacc[rr] = fmaf(pa, a, sacc[rr]);
#pragma unroll
                for (int al = 0; al < 3; ++al) vacc[rr][al] = fmaf(s.u[al], c, vacc[rr][al]);
            }
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) found[q] += seg[q] - (q ? seg[q > 0 ? q - 1 : 0] : 0);
        wave_sync_lds();  // the next chunk overwrites the slots
    }
    if (A.edge_cnt && lane < kPer && i0 + lane < n) {
        int c = found[0];
#pragma unroll
        for (int q = 1; q < kPer; ++q) c = lane == q ? found[q] : c;
        A.edge_cnt[i0 + lane] = c;
    }
    // s and v of the block's atoms (zero rows past the last atom and feature)
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
        if (rr * G + g >= kPer) continue;
        const int a = w * kPer + rr * G + g, i = ib + a;
        const bool on = i < n && f < F;
        const int ti = i < n ? min(max(mg.species[i], 0), mg.n_species - 1) : 0;
        if (f < F) xs[at(f, a)] = on ? A.emb[ti * F + f] + sacc[rr] : 0.f;
#pragma unroll
        for (int al = 0; al < 3; ++al) vs[al][at(f, a)] = on ? 0.f + vacc[rr][al] : 0.f;
    }

    // -------------------------------------------- update and projections --
    const int a = lane & 15, q = lane >> 4;
    const bool main = w < P::T;  // wavefront t < T: features 16 t .. 16 t + 15
    const int t = main ? w : 0, f0 = 16 * t + 4 * q;
    f32x4_t wU[P::KB], wV[P::KB], wM1[P::KB2], wM2[3][P::KB];
    f32x4_t m1 = {}, m2[3] = {};
    if (main) {
        load_tile(wU, A.wt, P::oU + t * P::KB, lane);
        load_tile(wV, A.wt, P::oV + t * P::KB, lane);
        load_tile(wM1, A.wt, P::oM1 + t * P::KB2, lane);
#pragma unroll
        for (int c = 0; c < 3; ++c) load_tile(wM2[c], A.wt, P::oM2 + (c * P::T + t) * P::KB, lane);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (f0 + i < F) {
                m1[i] = A.m1[f0 + i];
#pragma unroll
                for (int c = 0; c < 3; ++c) m2[c][i] = A.m2[c * F + f0 + i];
            }
    }
    __syncthreads();
    f32x4_t Uv[3] = {}, Vv[3] = {};
    float s_own[4], v_own[3][4];
    if (main) {
#pragma unroll
        for (int al = 0; al < 3; ++al) {
            product<P::KB, BF16>(Uv[al], wU, vs[al], lane);
            product<P::KB, BF16>(Vv[al], wV, vs[al], lane);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (f0 + i >= F) continue;
            s_own[i] = xs[at(f0 + i, a)];
#pragma unroll
            for (int al = 0; al < 3; ++al) v_own[al][i] = vs[al][at(f0 + i, a)];
            float nn = 1e-8f;
#pragma unroll
            for (int al = 0; al < 3; ++al) nn = fmaf(Vv[al][i], Vv[al][i], nn);
            xs[at(F + f0 + i, a)] = sqrtf(nn);
        }
    }
    __syncthreads();
    if (main) {
        f32x4_t acc = m1;
        product<P::KB2, BF16>(acc, wM1, xs, lane);
#pragma unroll
        for (int i = 0; i < 4; ++i) zs[at(f0 + i, a)] = f0 + i < F ? silu(acc[i]) : 0.f;
    }
    __syncthreads();
    // the projections' weights, in flight during M2
    constexpr int kTasks = kHC / 16 + 3, kMine = (kTasks + kWaves - 1) / kWaves;
    f32x4_t wQ[kMine][P::KB];
#pragma unroll
    for (int c = 0; c < kMine; ++c) {
        const int task = w + c * kWaves;
        load_tile(wQ[c], A.wt, task < kHC / 16 ? P::oQ + task * P::KB : P::oWV, lane);
    }
    if (main) {
#pragma unroll
        for (int c = 0; c < 3; ++c) product<P::KB, BF16>(m2[c], wM2[c], zs, lane);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool real = f0 + i < F;
            const float dot = Uv[0][i] * Vv[0][i] + Uv[1][i] * Vv[1][i] + Uv[2][i] * Vv[2][i];
            ss[at(f0 + i, a)] = real ? s_own[i] + m2[0][i] + m2[1][i] * dot : 0.f;
#pragma unroll
            for (int al = 0; al < 3; ++al)
                vs[al][at(f0 + i, a)] = real ? v_own[al][i] + m2[2][i] * Uv[al][i] : 0.f;
        }
    }
    __syncthreads();
    const int i = ib + a;
#pragma unroll
    for (int c = 0; c < kMine; ++c) {
        const int task = w + c * kWaves;
        if (task >= kTasks) break;
        f32x4_t acc = {};
        if (task < kHC / 16) {
            product<P::KB, BF16>(acc, wQ[c], ss, lane);
            if (i < n) *reinterpret_cast<f32x4_t*>(A.QK + int64_t(i) * kHC + 16 * task + 4 * q) = acc;
        } else {
            const int al = task - kHC / 16;
            product<P::KB, BF16>(acc, wQ[c], vs[al], lane);
            if (i < n && q == 0)
                *reinterpret_cast<float2*>(A.Vh + (int64_t(i) * 3 + al) * kNl) = make_float2(acc[0], acc[1]);
        }
    }
}

// The packed weights, rounded for BF16 models.
template <int F>
__global__ void __launch_bounds__(256) k_nc_pack(const float* UV, const float* M1, const float* M2, const float* Wqk,
                                                 const float* WV, int bf16, float* out) {
    using P = Pack<F>;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= P::total * P::UNIT) return;
    int unit = t / P::UNIT;
    const int lane = t % P::UNIT / 4, s = t % 4, r = lane & 15;
    const int kk = 4 * s + (lane >> 4);  // k within the block
    const float* W;
    int rows, K, kb, tile;
    if (unit < P::oM1) {
        const int m = unit >= P::oV;
        unit -= m ? P::oV : P::oU;
        W = UV + m * F * F;
        rows = F;
        K = F;
        tile = unit / P::KB;
        kb = unit % P::KB;
    } else if (unit < P::oM2) {
        unit -= P::oM1;
        W = M1;
        rows = F;
        K = 2 * F;
        tile = unit / P::KB2;
        kb = unit % P::KB2;
    } else if (unit < P::oQ) {
        unit -= P::oM2;
        const int c = unit / (P::T * P::KB);
        unit %= P::T * P::KB;
        W = M2 + c * F * F;
        rows = F;
        K = F;
        tile = unit / P::KB;
        kb = unit % P::KB;
    } else if (unit < P::oWV) {
        unit -= P::oQ;
        W = Wqk;
        rows = kHC;
        K = F;
        tile = unit / P::KB;
        kb = unit % P::KB;
    } else {
        W = WV;
        rows = kNl;
        K = F;
        tile = 0;
        kb = unit - P::oWV;
    }
    const int o = tile * 16 + r, k = kb * 16 + kk;
    const float v = o < rows && k < K ? W[o * K + k] : 0.f;
    out[t] = bf16 ? bf16_round(v) : v;
}

}  // namespace

int64_t nc_pack_count(int F) {
    return 256 * int64_t(F == 32 ? Pack<32>::total : F == 16 ? Pack<16>::total : Pack<8>::total);
}

void nc_pack_weights(int F, const float* UV, const float* M1, const float* M2, const float* Wqk, const float* WV,
                     bool bf16, float* out, hipStream_t s) {
    const int blocks = cdiv(nc_pack_count(F), 256);
    if (F == 32) k_nc_pack<32><<<blocks, 256, 0, s>>>(UV, M1, M2, Wqk, WV, bf16, out);
    else if (F == 16) k_nc_pack<16><<<blocks, 256, 0, s>>>(UV, M1, M2, Wqk, WV, bf16, out);
    else k_nc_pack<8><<<blocks, 256, 0, s>>>(UV, M1, M2, Wqk, WV, bf16, out);
    NNP_LAUNCH_CHECK();
}

void launch_nc_embed(const MpGeom& mg, const NcEmbedArgs& a, int F, bool bf16, hipStream_t s) {
    if (mg.n <= 0) return;
    ScopedTimer timer("nc_message_fwd", s);
    const int blocks = cdiv(mg.n, kAtoms);
    // Wavefronts of a block: eight with two atoms each, where these fill their
    // lanes (32 features): 192 atoms 12.3 -> 10.4 us, 4,095 atoms 16.8 -> 13.8,
    // 12,288 atoms 25.1 -> 24.6.  At 16 features a wavefront takes four atoms at
    // a time: 12,288 atoms 19.0 with four wavefronts, 21.7 with eight (192
    // atoms 8.9 and 8.7).
    auto launch = [&](auto kernel, int waves) { kernel<<<blocks, 64 * waves, 0, s>>>(mg, a); };
    if (F == 32) launch(bf16 ? k_nc_embed<32, true, 8> : k_nc_embed<32, false, 8>, 8);
    else if (F == 16) launch(bf16 ? k_nc_embed<16, true, 4> : k_nc_embed<16, false, 4>, 4);
    else launch(bf16 ? k_nc_embed<8, true, 4> : k_nc_embed<8, false, 4>, 4);
    NNP_LAUNCH_CHECK();
}

}  // namespace nnp
