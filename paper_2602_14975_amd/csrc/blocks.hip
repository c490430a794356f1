// Per-atom elementwise pieces of the embedding block and the readout, and
// the non-conservative pair head (paper, Methods: q_ih, k_ih, c_ijh, F_ij,
// F_i = sum_j (F_ij - F_ji)).  The dense contractions around them run in
// gemm.hip; the edge loops of the embedding in mp.hip.
#include "common.h"
#include "kernels.h"
#include "mp_edge.h"

namespace nnp {

// s0[i] = emb[t_i]; v0[i] = 0
__global__ void k_embed(int n, int F, int S, const int* __restrict__ species, const float* __restrict__ emb,
                        float* __restrict__ s, float* __restrict__ v) {
    int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n) * F) return;
    int i = int(t / F), f = int(t % F);
    const int sp = min(max(species[i], 0), S - 1);  // out-of-range species read row 0 or S-1, never past the table
    s[t] = emb[sp * F + f];
    v[(int64_t(i) * 3 + 0) * F + f] = 0.f;
    v[(int64_t(i) * 3 + 1) * F + f] = 0.f;
    v[(int64_t(i) * 3 + 2) * F + f] = 0.f;
}

// X[i] = [smid_i ; sqrt(sum_al Vv[i][al]^2 + 1e-8)], UV rows [Uv (F) | Vv (F)] per component.
__global__ void k_build_x(int n, int F, const float* __restrict__ smid, const float* __restrict__ UV,
                          float* __restrict__ X) {
    int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n) * F) return;
    int i = int(t / F), f = int(t % F);
    float acc = 1e-8f;
#pragma unroll
    for (int al = 0; al < 3; ++al) {
        float vv = UV[(int64_t(i) * 3 + al) * 2 * F + F + f];
        acc = fmaf(vv, vv, acc);
    }
    X[int64_t(i) * 2 * F + f] = smid[t];
    X[int64_t(i) * 2 * F + F + f] = sqrtf(acc);
}

// s_out = smid + p + q * sum_al Uv Vv ; v_out = vmid + o * Uv
__global__ void k_update_combine(int n, int F, const float* __restrict__ smid, const float* __restrict__ vmid,
                                 const float* __restrict__ UV, const float* __restrict__ pqo,
                                 float* __restrict__ s_out, float* __restrict__ v_out) {
    int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n) * F) return;
    int i = int(t / F), f = int(t % F);
    const float* h = pqo + int64_t(i) * 3 * F;
    float dot = 0.f, uv[3];
#pragma unroll
    for (int al = 0; al < 3; ++al) {
        const float* row = UV + (int64_t(i) * 3 + al) * 2 * F;
        uv[al] = row[f];
        dot = fmaf(row[f], row[F + f], dot);
    }
    s_out[t] = smid[t] + h[f] + h[F + f] * dot;
#pragma unroll
    for (int al = 0; al < 3; ++al) {
        int64_t idx = (int64_t(i) * 3 + al) * F + f;
        v_out[idx] = vmid[idx] + h[2 * F + f] * uv[al];
    }
}

// Reverse of k_update_combine: g_pqo and the Uv/Vv adjoints (the norm path
// of Vv is added by k_norm_bwd).
__global__ void k_update_combine_bwd(int n, int F, const float* __restrict__ UV, const float* __restrict__ pqo,
                                     const float* __restrict__ gs, const float* __restrict__ gv,
                                     float* __restrict__ gpqo, float* __restrict__ gUV) {
    int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n) * F) return;
    int i = int(t / F), f = int(t % F);
    const float* h = pqo + int64_t(i) * 3 * F;
    const float q = h[F + f], o = h[2 * F + f];
    const float g = gs[t];
    float dot = 0.f, go = 0.f;
#pragma unroll
    for (int al = 0; al < 3; ++al) {
        const float* row = UV + (int64_t(i) * 3 + al) * 2 * F;
        const float u = row[f], vv = row[F + f];
        const float gva = gv ? gv[(int64_t(i) * 3 + al) * F + f] : 0.f;  // nullptr: zero adjoint
        dot = fmaf(u, vv, dot);
        go = fmaf(gva, u, go);
        float* grow = gUV + (int64_t(i) * 3 + al) * 2 * F;
        grow[f] = g * q * vv + gva * o;
        grow[F + f] = g * q * u;
    }
    float* gh = gpqo + int64_t(i) * 3 * F;
    gh[f] = g;
    gh[F + f] = g * dot;
    gh[2 * F + f] = go;
}

// g_smid = gs + gX[:, :F];  gVv[al] += gX[:, F:] * Vv[al] / nrm
__global__ void k_norm_bwd(int n, int F, const float* __restrict__ gs, const float* __restrict__ gX,
                           const float* __restrict__ X, const float* __restrict__ UV, float* __restrict__ gsmid,
                           float* __restrict__ gUV) {
    int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n) * F) return;
    int i = int(t / F), f = int(t % F);
    gsmid[t] = gs[t] + gX[int64_t(i) * 2 * F + f];
    const float gn = gX[int64_t(i) * 2 * F + F + f] / X[int64_t(i) * 2 * F + F + f];
#pragma unroll
    for (int al = 0; al < 3; ++al) {
        const int64_t idx = (int64_t(i) * 3 + al) * 2 * F + F + f;
        gUV[idx] = fmaf(gn, UV[idx], gUV[idx]);
    }
}

// E_i = wo . z_i + beta[t_i] (z = silu(Wo s + bo) from the GEMM epilogue)
__global__ void k_readout(int n, int F, int S, const float* __restrict__ z, const float* __restrict__ wo,
                          const float* __restrict__ beta, const int* __restrict__ species, float* __restrict__ Ei,
                          const int* __restrict__ perm) {
    int lane = threadIdx.x & 63;
    int i = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (i >= n) return;
    float acc = 0.f;
    for (int f = lane; f < F; f += 64) acc = fmaf(wo[f], z[int64_t(i) * F + f], acc);
    acc = wave_sum(acc);
    if (lane == 0) Ei[perm ? min(max(perm[i], 0), n - 1) : i] = acc + beta[min(max(species[i], 0), S - 1)];
}

// g_ao = wo * silu'(a_o)  (dE/dE_i = 1)
__global__ void k_readout_bwd(int n, int F, const float* __restrict__ ao, const float* __restrict__ wo,
                              float* __restrict__ gao) {
    int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= int64_t(n) * F) return;
    gao[t] = wo[t % F] * silu_grad(ao[t]);
}

// Per-replica sums, one block per replica.
__global__ void __launch_bounds__(256) k_rep_sum(RepSum a) {
    __shared__ double red[256];
    rep_sum_block(a, blockIdx.x, red);
}

// Per-species column sums over a chunk of rows, for the adjoints of
// per-species tables: part[c][t][f] = sum over atoms of species t of x[i][f],
// i in chunk c; launch_reduce_chunks adds the chunks (both in fixed order).
// One block per chunk and 32 columns: thread (row group, column) walks every
// eighth row of the chunk, reads of a row group being contiguous.  Bound by
// the one read of x; one thread per (species, column) walking all rows was a
// serial chain of n loads (4.95 ms per launch for 24,576 rows; with this kernel
// and the reductions of gemm.hip a distillation step of those rows went from
// 12.4 to 0.97 ms).
__global__ void __launch_bounds__(256) k_emb_grad_part(int n, int F, int S, int chunk, const int* __restrict__ species,
                                                       const float* __restrict__ x, float* __restrict__ part) {
    __shared__ float red[8][8][32];  // row group, species, column
    const int col = threadIdx.x & 31, rg = threadIdx.x >> 5;
    const int f = blockIdx.x * 32 + col;
    const int i0 = blockIdx.y * chunk, i1 = min(n, i0 + chunk);
    float acc[8] = {};
    if (f < F) {
        for (int i = i0 + rg; i < i1; i += 8) {
            const int sp = species[i];
            const float v = x[int64_t(i) * F + f];
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] += sp == t ? v : 0.f;
        }
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) red[rg][t][col] = acc[t];
    __syncthreads();
    if (rg < S && f < F) {  // row group rg now adds species rg (S <= 8)
        float s = 0.f;
#pragma unroll
        for (int g = 0; g < 8; ++g) s += red[g][rg][col];
        part[(int64_t(blockIdx.y) * S + rg) * F + f] = s;
    }
}

// ------------------------------------------------------------- NC head ----
// Per owner atom i (one wavefront), lanes over the CSR entries of its row.
// QK rows: [q (H x n_c) | k (H x n_c)]; Vh rows [n][3][n_l].
constexpr int kNs = 8, kNl = 2, kNc = 8, kH = kNs + kNl;

struct HeadEdge {
    float ef[kNs];  // B_h(r) u(r/rc)
    float u[3];
    float r;
    int j;
};

__device__ __forceinline__ bool head_edge(const MpGeom& mg, int i, int e, double xi, double yi, double zi,
                                          double L, double inv, HeadEdge& he) {
    const int n = mg.n;
    const int j = mg.nbr[e];
    double dx, dy, dz;
    if (!pair_rule(xi, yi, zi, mg.pos[j], mg.pos[n + j], mg.pos[2 * n + j], L, inv, mg.rc2, dx, dy, dz)) return false;
    // radial values in float32 (the pair rule above decides in float64)
    const float r = sqrtf(float((dx * dx + dy * dy) + dz * dz));
    const float ir = 1.f / r;
    float env;
    radial_poly_f32<kNs>(r * float(mg.inv_rc), float(mg.bessel_norm) * ir, he.ef, env);
    he.u[0] = float(dx) * ir;
    he.u[1] = float(dy) * ir;
    he.u[2] = float(dz) * ir;
    he.r = r;
    he.j = j;
    return true;
}

__device__ __forceinline__ void head_coeffs(const float* qa, const float* kb, float* c) {
    const float scale = 0.35355339059327373f;  // 1/sqrt(n_c), n_c = 8
#pragma unroll
    for (int h = 0; h < kH; ++h) {
        const float4 a0 = *reinterpret_cast<const float4*>(qa + h * kNc);
        const float4 a1 = *reinterpret_cast<const float4*>(qa + h * kNc + 4);
        const float4 b0 = *reinterpret_cast<const float4*>(kb + h * kNc);
        const float4 b1 = *reinterpret_cast<const float4*>(kb + h * kNc + 4);
        float acc = a0.x * b0.x;
        acc = fmaf(a0.y, b0.y, acc); acc = fmaf(a0.z, b0.z, acc); acc = fmaf(a0.w, b0.w, acc);
        acc = fmaf(a1.x, b1.x, acc); acc = fmaf(a1.y, b1.y, acc); acc = fmaf(a1.z, b1.z, acc);
        acc = fmaf(a1.w, b1.w, acc);
        c[h] = acc * scale;
    }
}

// S = sum_h c_h B_h(r) u(r/rc) over the n_s Bessel heads in one fixed
// order, ((p0 + p4) + (p2 + p6)) + ((p1 + p5) + (p3 + p7)) with rounded
// products p_h: the order a butterfly over eight lanes produces, so that
// the record kernel below, which spreads the heads over lanes, gives the
// same sums bit for bit.
__device__ __forceinline__ float head_sum(const float* c, const float* ef) {
#pragma clang fp contract(off)  // rounded products: no product may fuse into the sums
    float p[kNs];
#pragma unroll
    for (int h = 0; h < kNs; ++h) p[h] = c[h] * ef[h];
    return ((p[0] + p[4]) + (p[2] + p[6])) + ((p[1] + p[5]) + (p[3] + p[7]));
}

// The contribution of edge (i, j) to F_i: F_ij - F_ji = S_ij D_ij - S_ji D_ji
// with D_ij = u + c_ij,s V_i,0 + c_ij,s+1 V_i,1 and D_ji = -u + c_ji,s V_j,0 +
// c_ji,s+1 V_j,1 (s = n_s), and with VIR its share F_ij . r_ij of the virial
// proxy in out[3].  Vi, Vj: [n_l][3].  Explicit fused operations fix the
// rounding.
template <bool VIR>
__device__ __forceinline__ void head_pair(float Sij, float Sji, float ci8, float ci9, float cj8, float cj9,
                                          const float* u, float r, const float (*Vi)[3], const float (*Vj)[3],
                                          float* out) {
    float fu = 0.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float Dij = fmaf(ci9, Vi[1][a], fmaf(ci8, Vi[0][a], u[a]));
        const float Dji = fmaf(cj9, Vj[1][a], fmaf(cj8, Vj[0][a], -u[a]));
        out[a] = fmaf(Sij, Dij, -(Sji * Dji));
        if (VIR) fu = fmaf(Sij * Dij, u[a], fu);
    }
    out[3] = VIR ? fu * r : 0.f;
}

// A group of G lanes per owner atom (64 / G atoms per wavefront); lanes take
// one CSR entry each.  The contributions of the entries that pass the pair
// rule are compacted (ballot) into LDS and added by the group's first lane
// in row order, so the sum does not depend on how many extra Verlet entries
// the row holds or where batch boundaries fall.
template <int G, bool VIR>
__global__ void __launch_bounds__(256) k_head_fwd(MpGeom mg, const float* __restrict__ QK,
                                                  const float* __restrict__ Vh, float* __restrict__ Fout, int accum,
                                                  float* __restrict__ vir_set, float* __restrict__ vir_add) {
    constexpr int APW = 64 / G;
    // force (and F_ij . r_ij) per staged edge, one 16-byte slot each
    __shared__ __align__(16) float contrib[4][APW][G][4];
    // the owner's q and k rows, read by every lane of its group: in LDS
    __shared__ __align__(16) float qk_s[4][APW][2 * kH * kNc];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int g = lane / G, l = lane % G;
    const int i = (xcd_block(blockIdx.x, gridDim.x) * 4 + w) * APW + g;
    const bool active = i < mg.n;
    const int n = mg.n;
    double L = 1, inv = 1, xi = 0, yi = 0, zi = 0;
    int e0 = 0, e1 = 0;
    float Vi[kNl][3] = {};
    if (active) {
        mg.geom.get(i, L, inv);
        xi = mg.pos[i]; yi = mg.pos[n + i]; zi = mg.pos[2 * n + i];
        e0 = mg.off[i];
        e1 = mg.off[i + 1];
#pragma unroll
        for (int t = l; t < 2 * kH * kNc; t += G) qk_s[w][g][t] = QK[int64_t(i) * 2 * kH * kNc + t];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int h = 0; h < kNl; ++h) Vi[h][a] = Vh[(int64_t(i) * 3 + a) * kNl + h];
    }
    wave_sync_lds();
    const float* qi = qk_s[w][g];
    const float* ki = qi + kH * kNc;
    const uint64_t gmask = (G == 64) ? ~0ull : (((1ull << G) - 1ull) << (g * G));
    float fx = 0.f, fy = 0.f, fz = 0.f, vr = 0.f;  // running sums (first lane of the group)
    for (int base = 0; __ballot(e0 + base < e1) != 0ull; base += G) {
        const int e = e0 + base + l;
        HeadEdge he;
        const bool ok = e < e1 && head_edge(mg, i, e, xi, yi, zi, L, inv, he);
        const uint64_t mine = __ballot(ok) & gmask;
        if (ok) {
            const int j = he.j;
            const float* qj = QK + int64_t(j) * 2 * kH * kNc;
            const float* kj = qj + kH * kNc;
            float cij[kH], cji[kH];
            head_coeffs(qi, kj, cij);
            head_coeffs(qj, ki, cji);
            float Vj[kNl][3];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int h = 0; h < kNl; ++h) Vj[h][a] = Vh[(int64_t(j) * 3 + a) * kNl + h];
            const int pre = __popcll(mine & ((1ull << lane) - 1ull));
            float c[4];
            head_pair<VIR>(head_sum(cij, he.ef), head_sum(cji, he.ef), cij[kNs], cij[kNs + 1], cji[kNs],
                           cji[kNs + 1], he.u, he.r, Vi, Vj, c);
            *reinterpret_cast<float4*>(&contrib[w][g][pre][0]) = make_float4(c[0], c[1], c[2], c[3]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (l == 0) {
            const int cnt = __popcll(mine);
            for (int t = 0; t < cnt; ++t) {
                const float4 c = *reinterpret_cast<const float4*>(&contrib[w][g][t][0]);
                fx += c.x;
                fy += c.y;
                fz += c.z;
                if constexpr (VIR) vr += c.w;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
    if (active && l == 0) {
        const int io = mg.perm ? min(max(mg.perm[i], 0), n - 1) : i;
        if (accum) {
            Fout[io] += fx; Fout[n + io] += fy; Fout[2 * n + io] += fz;
        } else {
            Fout[io] = fx; Fout[n + io] = fy; Fout[2 * n + io] = fz;
        }
        if constexpr (VIR) {
            if (vir_set) vir_set[io] = vr;
            if (vir_add) vir_add[io] += vr;
        }
    }
}

// x of another lane of the row of 16 (zero where there is none): kShr + k
// reads lane l - k, kXor1 and kXor2 the lane of the quad.
constexpr int kShr = 0x110, kXor1 = 0xB1, kXor2 = 0x4E;
template <int CTRL>
__device__ __forceinline__ float row_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

// The same head over the records the NC message step left (edges within the
// cutoff in list order, B_h u, u and r in float32): no pair rule or radial
// values here.  One wavefront per four owner atoms, lanes 16 e .. 16 e + 15
// for owner e, over chunks of 32 of its edges in three steps:
//   A  one edge at a time, lane 16 e + h taking head h (h < 10), so that the
//      neighbour's q and k rows are read as 32-byte pieces per lane,
//      contiguous across the heads of an edge, four edges in flight; the
//      sums over heads (the order of head_sum) move between neighbouring
//      lanes by DPP operands and are left in LDS;
//   B  lane 16 e + t taking edge t (two passes of 16): the pair contribution
//      (head_pair) from the sums and the neighbour's V rows, into LDS;
//   C  the owner's force components added over the edges in record order.
// The result is the same, bit for bit, as that of the kernel above.  Bound by
// instruction issue and the latency of the gathers: with step B done for one
// lane of 16 within step A and the sums shuffled through LDS, 12,288 atoms
// took 19.7 us; now 13.6 (192 atoms: 13.8 -> 7.4).
template <bool VIR>
__global__ void __launch_bounds__(256) k_head_fwd_rec(int n, const int* __restrict__ off,
                                                      const int* __restrict__ cnt_in, const NcEdge* __restrict__ rec,
                                                      const float* __restrict__ QK, const float* __restrict__ Vh,
                                                      float* __restrict__ Fout, int accum, float* __restrict__ vir_set,
                                                      float* __restrict__ vir_add, const int* __restrict__ perm) {
    constexpr int HC = 2 * kH * kNc, CH = 32, DEPTH = 4;
    static_assert(kNs == 8 && kNl == 2 && CH % DEPTH == 0 && sizeof(NcEdge) == 64, "lane roles and record layout");
    // per edge: S_ij, S_ji, then c_8 and c_9 of both directions; contributions
    __shared__ __align__(16) float sums_s[4][4][CH][8];
    __shared__ __align__(16) float contrib_s[4][4][CH][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = lane >> 4, h = lane & 15;
    const int iw = (xcd_block(blockIdx.x, gridDim.x) * 4 + w) * 4;
    if (iw >= n) return;  // whole wavefronts
    float(*sums)[8] = sums_s[w][e];
    float(*contrib)[4] = contrib_s[w][e];
    const int i = iw + e;
    const bool own = i < n;
    const int e0 = own ? off[i] : 0, cnt = own ? cnt_in[i] : 0;
    const int hh = h < kH ? h : 0;
    float qi[kNc] = {}, ki[kNc] = {};
    float Vi[kNl][3] = {};
    if (own) {
        const float4* q4 = reinterpret_cast<const float4*>(QK + int64_t(i) * HC + hh * kNc);
        const float4* k4 = reinterpret_cast<const float4*>(QK + int64_t(i) * HC + (kH + hh) * kNc);
        const float4 a0 = q4[0], a1 = q4[1], b0 = k4[0], b1 = k4[1];
        qi[0] = a0.x; qi[1] = a0.y; qi[2] = a0.z; qi[3] = a0.w; qi[4] = a1.x; qi[5] = a1.y; qi[6] = a1.z; qi[7] = a1.w;
        ki[0] = b0.x; ki[1] = b0.y; ki[2] = b0.z; ki[3] = b0.w; ki[4] = b1.x; ki[5] = b1.y; ki[6] = b1.z; ki[7] = b1.w;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int l = 0; l < kNl; ++l) Vi[l][a] = Vh[(int64_t(i) * 3 + a) * kNl + l];
    }
    // the longest row of the four
    int steps = cnt;
#pragma unroll
    for (int m = 16; m <= 32; m <<= 1) steps = max(steps, __shfl_xor(steps, m, 64));
    steps = __builtin_amdgcn_readfirstlane(steps);
    const float scale = 0.35355339059327373f;  // 1/sqrt(n_c), n_c = 8
    // q_a . k_b over the channels in the order of head_coeffs
    auto dot8 = [](const float* a, const float4& b0, const float4& b1) {
        float acc = a[0] * b0.x;
        acc = fmaf(a[1], b0.y, acc); acc = fmaf(a[2], b0.z, acc); acc = fmaf(a[3], b0.w, acc);
        acc = fmaf(a[4], b1.x, acc); acc = fmaf(a[5], b1.y, acc); acc = fmaf(a[6], b1.z, acc);
        acc = fmaf(a[7], b1.w, acc);
        return acc;
    };
    auto dot8r = [](const float4& a0, const float4& a1, const float* b) {
        float acc = a0.x * b[0];
        acc = fmaf(a0.y, b[1], acc); acc = fmaf(a0.z, b[2], acc); acc = fmaf(a0.w, b[3], acc);
        acc = fmaf(a1.x, b[4], acc); acc = fmaf(a1.y, b[5], acc); acc = fmaf(a1.z, b[6], acc);
        acc = fmaf(a1.w, b[7], acc);
        return acc;
    };
    // what one lane holds of an edge in step A: its head's q and k rows of
    // the neighbour and B_h u
    struct Pre {
        float4 q0, q1, k0, k1;
        float ef;
    };
    // what it holds of its two edges of step B
    struct Edge {
        float4 r0;     // j, r, u_0, u_1
        float u2;
        float2 vj[3];  // the neighbour's V
    };
    float sum = 0.f;  // component h of the owner's force (3: of the virial share)
    for (int base = 0; base < steps; base += CH) {
        const int left = cnt - base;  // this owner's edges from here on
        // records of the lane's edges h and 16 + h of the chunk
        Edge ed[2];
        int jl[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int t = 16 * p + h;
            ed[p] = Edge{};
            if (t < left) {
                const NcEdge* re = rec + e0 + base + t;
                ed[p].r0 = *reinterpret_cast<const float4*>(re);
                ed[p].u2 = re->u[2];
            }
            jl[p] = __float_as_int(ed[p].r0.x);
        }
        const float* ef_row = rec[e0 + base].ef + (h < kNs ? h : 0);
        // edge t of the chunk; every lane takes part in the shuffle
        auto fetch = [&](int t, Pre& p) {
            const int j = __shfl(t < 16 ? jl[0] : jl[1], 16 * e + (t & 15), 64);
            if (t >= left || h >= kH) return;
            const char* row = reinterpret_cast<const char*>(QK) + uint32_t(j) * uint64_t(HC * 4);
            const float4* q4 = reinterpret_cast<const float4*>(row) + h * 2;
            p.q0 = q4[0];
            p.q1 = q4[1];
            p.k0 = q4[kH * 2];
            p.k1 = q4[kH * 2 + 1];
            p.ef = ef_row[t * int(sizeof(NcEdge) / 4)];
        };
        // --- A
        auto edge_step = [&](int t, const Pre& cur) {
            float cij = 0.f, cji = 0.f;
            if (h < kH) {
                cij = dot8(qi, cur.k0, cur.k1) * scale;   // q_i . k_j
                cji = dot8r(cur.q0, cur.q1, ki) * scale;  // q_j . k_i
            }
            // S over lanes 0..7 of the owner, in lanes 4..7: pairs four, two,
            // one lane apart (rounded products as in head_sum)
            float pij, pji;
            {
#pragma clang fp contract(off)
                pij = h < kNs ? cij * cur.ef : 0.f;
                pji = h < kNs ? cji * cur.ef : 0.f;
                pij += row_lane<kShr + 4>(pij);
                pji += row_lane<kShr + 4>(pji);
                pij += row_lane<kXor2>(pij);
                pji += row_lane<kXor2>(pji);
                pij += row_lane<kXor1>(pij);
                pji += row_lane<kXor1>(pji);
            }
            // lane 7: the sums; lanes 8 and 9: c_8 and c_9
            if (h >= kNs - 1 && h < kH)
                *reinterpret_cast<float2*>(&sums[t][2 * (h - (kNs - 1))]) =
                    h == kNs - 1 ? make_float2(pij, pji) : make_float2(cij, cji);
        };
        const int ch = min(CH, steps - base);
        Pre pre[DEPTH] = {};
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (d < ch) fetch(d, pre[d]);
        // V rows of the neighbours of step B
#pragma unroll
        for (int p = 0; p < 2; ++p)
            if (16 * p + h < left)
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    ed[p].vj[a] = *reinterpret_cast<const float2*>(Vh + (int64_t(jl[p]) * 3 + a) * kNl);
        for (int t = 0; t < ch; t += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                if (t + d >= ch) break;
                edge_step(t + d, pre[d]);
                if (t + d + DEPTH < ch) fetch(t + d + DEPTH, pre[d]);
            }
        }
        wave_sync_lds();
        // --- B
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int t = 16 * p + h;
            if (t < left) {
                const float4 s0 = *reinterpret_cast<const float4*>(&sums[t][0]);
                const float2 s1 = *reinterpret_cast<const float2*>(&sums[t][4]);
                const Edge& x = ed[p];
                const float u[3] = {x.r0.z, x.r0.w, x.u2};
                const float Vj[kNl][3] = {{x.vj[0].x, x.vj[1].x, x.vj[2].x}, {x.vj[0].y, x.vj[1].y, x.vj[2].y}};
                float c[4];
                head_pair<VIR>(s0.x, s0.y, s0.z, s1.x, s0.w, s1.y, u, x.r0.y, Vi, Vj, c);
                *reinterpret_cast<float4*>(&contrib[t][0]) = make_float4(c[0], c[1], c[2], c[3]);
            }
        }
        wave_sync_lds();
        // --- C
        const int mine = min(CH, left);
        for (int t = 0; t < mine; ++t) sum += contrib[t][h & 3];
        wave_sync_lds();  // the next chunk overwrites both
    }
    if (own && h < 4) {
        const int io = perm ? min(max(perm[i], 0), n - 1) : i;  // outputs under the caller's index
        if (h < 3) {
            if (accum) Fout[int64_t(h) * n + io] += sum;
            else Fout[int64_t(h) * n + io] = sum;
        } else if constexpr (VIR) {
            if (vir_set) vir_set[io] = sum;
            if (vir_add) vir_add[io] += sum;
        }
    }
}

// Reverse of the head for a loss with dL/dF_i = gF_i: each directed edge
// (i, j) carries a_ij = gF_i - gF_j as the adjoint of F_ij.  The owner i
// accumulates only its own adjoints, so no atomics are needed: q_i and V_i
// from its edges (i, j) (first sweep), k_i from the reverse edges (j, i)
// (second sweep).  In each sweep, phase 1 (lanes over edges) forms the
// coefficient adjoints dL/dc and stages them in LDS; phase 2 (lanes over the
// (head, channel) pairs) gathers the neighbour's k or q row.
__global__ void __launch_bounds__(64) k_head_bwd(MpGeom mg, const float* __restrict__ QK, const float* __restrict__ Vh,
                                                 const float* __restrict__ gF, float* __restrict__ gQK,
                                                 float* __restrict__ gVh) {
    __shared__ float gc[64][kH];
    __shared__ int jj[64];
    __shared__ float gvc[64][kNl * 3];  // per-entry V adjoint contributions (sweep 0)
    const int lane = threadIdx.x;
    const int i = xcd_block(blockIdx.x, gridDim.x);
    const int n = mg.n;
    double L, inv;
    mg.geom.get(i, L, inv);
    const double xi = mg.pos[i], yi = mg.pos[n + i], zi = mg.pos[2 * n + i];
    const float* qi = QK + int64_t(i) * 2 * kH * kNc;
    const float* ki = qi + kH * kNc;
    float Vi[kNl][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int h = 0; h < kNl; ++h) Vi[h][a] = Vh[(int64_t(i) * 3 + a) * kNl + h];
    const float gFi[3] = {gF[i], gF[n + i], gF[2 * n + i]};
    const float scale = 0.35355339059327373f;  // 1/sqrt(n_c)
    const int e0 = mg.off[i], e1 = mg.off[i + 1];
    float* gq = gQK + int64_t(i) * 2 * kH * kNc;
    float* gk = gq + kH * kNc;
    float gv_acc = 0.f;  // lane < 6: component (h, a) = (lane / 3, lane % 3)
    for (int sweep = 0; sweep < 2; ++sweep) {
        float acc0 = 0.f, acc1 = 0.f;  // (h, c) = lane and 64 + lane (lane < 16)
        for (int base = e0; base < e1; base += 64) {
            const int e = base + lane;
            HeadEdge he;
            const bool ok = e < e1 && head_edge(mg, i, e, xi, yi, zi, L, inv, he);
            if (ok) {
                const int j = he.j;
                const float* qj = QK + int64_t(j) * 2 * kH * kNc;
                const float* kj = qj + kH * kNc;
                float aij[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) aij[a] = gFi[a] - gF[a * n + j];
                float c[kH];
                if (sweep == 0) {
                    head_coeffs(qi, kj, c);  // c_ijh
                    float S = 0.f;
#pragma unroll
                    for (int h = 0; h < kNs; ++h) S = fmaf(c[h], he.ef[h], S);
                    float D[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) D[a] = he.u[a] + c[kNs] * Vi[0][a] + c[kNs + 1] * Vi[1][a];
                    const float gS = aij[0] * D[0] + aij[1] * D[1] + aij[2] * D[2];
#pragma unroll
                    for (int h = 0; h < kNs; ++h) gc[lane][h] = gS * he.ef[h];
#pragma unroll
                    for (int h = 0; h < kNl; ++h) {
                        gc[lane][kNs + h] = S * (aij[0] * Vi[h][0] + aij[1] * Vi[h][1] + aij[2] * Vi[h][2]);
#pragma unroll
                        for (int a = 0; a < 3; ++a) gvc[lane][h * 3 + a] = aij[a] * S * c[kNs + h];
                    }
                } else {
                    head_coeffs(qj, ki, c);  // c_jih
                    float Vj[kNl][3];
#pragma unroll
                    for (int a = 0; a < 3; ++a)
#pragma unroll
                        for (int h = 0; h < kNl; ++h) Vj[h][a] = Vh[(int64_t(j) * 3 + a) * kNl + h];
                    float S = 0.f;
#pragma unroll
                    for (int h = 0; h < kNs; ++h) S = fmaf(c[h], he.ef[h], S);
                    float D[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) D[a] = -he.u[a] + c[kNs] * Vj[0][a] + c[kNs + 1] * Vj[1][a];
                    // the adjoint of F_ji is -aij
                    const float gS = -(aij[0] * D[0] + aij[1] * D[1] + aij[2] * D[2]);
#pragma unroll
                    for (int h = 0; h < kNs; ++h) gc[lane][h] = gS * he.ef[h];
#pragma unroll
                    for (int h = 0; h < kNl; ++h)
                        gc[lane][kNs + h] = -S * (aij[0] * Vj[h][0] + aij[1] * Vj[h][1] + aij[2] * Vj[h][2]);
                }
                jj[lane] = j;
            } else {
                jj[lane] = -1;
            }
            __syncthreads();
            const int cnt = min(64, e1 - base);
            for (int t = 0; t < cnt; ++t) {
                const int j = jj[t];
                if (j < 0) continue;
                // sweep 0 gathers k_j, sweep 1 gathers q_j
                const float* row = QK + int64_t(j) * 2 * kH * kNc + (sweep == 0 ? kH * kNc : 0);
                acc0 = fmaf(gc[t][lane / kNc] * scale, row[lane], acc0);
                if (lane < 16) acc1 = fmaf(gc[t][(64 + lane) / kNc] * scale, row[64 + lane], acc1);
                if (sweep == 0 && lane < kNl * 3) gv_acc += gvc[t][lane];
            }
            __syncthreads();
        }
        float* out = sweep == 0 ? gq : gk;
        out[lane] = acc0;
        if (lane < 16) out[64 + lane] = acc1;
    }
    if (lane < kNl * 3) {
        const int h = lane / 3, a = lane % 3;
        gVh[(int64_t(i) * 3 + a) * kNl + h] = gv_acc;
    }
}

// ------------------------------------------------------------------- host --
static int ew_blocks(int64_t count) { return cdiv(count, 256); }

void launch_embed(int n, int F, int S, const int* species, const float* emb, float* s, float* v, hipStream_t st) {
    k_embed<<<ew_blocks(int64_t(n) * F), 256, 0, st>>>(n, F, S, species, emb, s, v);
    NNP_LAUNCH_CHECK();
}
void launch_build_x(int n, int F, const float* smid, const float* UV, float* X, hipStream_t st) {
    k_build_x<<<ew_blocks(int64_t(n) * F), 256, 0, st>>>(n, F, smid, UV, X);
    NNP_LAUNCH_CHECK();
}
void launch_update_combine(int n, int F, const float* smid, const float* vmid, const float* UV, const float* pqo,
                           float* s_out, float* v_out, hipStream_t st) {
    k_update_combine<<<ew_blocks(int64_t(n) * F), 256, 0, st>>>(n, F, smid, vmid, UV, pqo, s_out, v_out);
    NNP_LAUNCH_CHECK();
}
void launch_update_combine_bwd(int n, int F, const float* UV, const float* pqo, const float* gs, const float* gv,
                               float* gpqo, float* gUV, hipStream_t st) {
    k_update_combine_bwd<<<ew_blocks(int64_t(n) * F), 256, 0, st>>>(n, F, UV, pqo, gs, gv, gpqo, gUV);
    NNP_LAUNCH_CHECK();
}
void launch_norm_bwd(int n, int F, const float* gs, const float* gX, const float* X, const float* UV, float* gsmid,
                     float* gUV, hipStream_t st) {
    k_norm_bwd<<<ew_blocks(int64_t(n) * F), 256, 0, st>>>(n, F, gs, gX, X, UV, gsmid, gUV);
    NNP_LAUNCH_CHECK();
}
void launch_readout(int n, int F, int S, const float* z, const float* wo, const float* beta, const int* species, float* Ei,
                    hipStream_t st, const int* perm) {
    k_readout<<<cdiv(n, 4), 256, 0, st>>>(n, F, S, z, wo, beta, species, Ei, perm);
    NNP_LAUNCH_CHECK();
}
void launch_readout_bwd(int n, int F, const float* ao, const float* wo, float* gao, hipStream_t st) {
    k_readout_bwd<<<ew_blocks(int64_t(n) * F), 256, 0, st>>>(n, F, ao, wo, gao);
    NNP_LAUNCH_CHECK();
}
void launch_rep_sum(const RepSum& a, hipStream_t st) {
    k_rep_sum<<<a.n_rep, 256, 0, st>>>(a);
    NNP_LAUNCH_CHECK();
}
void launch_emb_grad(int n, int F, int S, const int* species, const float* gs0, float* gemb, float* scratch, int chunk,
                     hipStream_t st) {
    if (n <= 0) return;
    const int nch = cdiv(n, chunk);
    k_emb_grad_part<<<dim3(cdiv(F, 32), nch), 256, 0, st>>>(n, F, S, chunk, species, gs0, scratch);
    NNP_LAUNCH_CHECK();
    const int64_t cnt = int64_t(S) * F;
    launch_reduce_chunks(cnt, nch, scratch, cnt, gemb, false, st);
}
void launch_head_fwd(const MpGeom& mg, const float* QK, const float* Vh, float* F, bool accum, hipStream_t st,
                     float* vir_set, float* vir_add) {
    if (mg.n <= 0) return;
    ScopedTimer timer("head_fwd", st);
    // 16 lanes per atom: rows of the 3.5 A list hold about 40 candidates
    if (vir_set || vir_add) k_head_fwd<16, true><<<cdiv(mg.n, 16), 256, 0, st>>>(mg, QK, Vh, F, accum, vir_set, vir_add);
    else k_head_fwd<16, false><<<cdiv(mg.n, 16), 256, 0, st>>>(mg, QK, Vh, F, accum, nullptr, nullptr);
    NNP_LAUNCH_CHECK();
}
void launch_head_fwd_rec(const MpGeom& mg, const int* cnt, const NcEdge* rec, const float* QK, const float* Vh,
                         float* F, bool accum, hipStream_t st, float* vir_set, float* vir_add) {
    if (mg.n <= 0) return;
    ScopedTimer timer("head_fwd", st);
    // four owner atoms per wavefront
    if (vir_set || vir_add)
        k_head_fwd_rec<true><<<cdiv(mg.n, 16), 256, 0, st>>>(mg.n, mg.off, cnt, rec, QK, Vh, F, accum, vir_set, vir_add,
                                                             mg.perm);
    else
        k_head_fwd_rec<false><<<cdiv(mg.n, 16), 256, 0, st>>>(mg.n, mg.off, cnt, rec, QK, Vh, F, accum, nullptr,
                                                              nullptr, mg.perm);
    NNP_LAUNCH_CHECK();
}
void launch_head_bwd(const MpGeom& mg, const float* QK, const float* Vh, const float* gF, float* gQK, float* gVh,
                     hipStream_t st) {
    if (mg.n <= 0) return;
    k_head_bwd<<<mg.n, 64, 0, st>>>(mg, QK, Vh, gF, gQK, gVh);
    NNP_LAUNCH_CHECK();
}

}  // namespace nnp
