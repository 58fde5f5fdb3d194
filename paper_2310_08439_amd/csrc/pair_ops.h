// Per-pair work shared by the descriptor and adjoint kernels: launch arguments,
// pair geometry, radial functions, the fixed-point force sums, and the adjoint
// of one pair.
#pragma once

#include "tmd_internal.h"
#include "tensor_ops.h"

namespace tmd {

using namespace ops;

struct PathArgs {
    int64_t n;
    int S, K, F, cap, nch_log2;
    float rc2, half_inv_rc, pi_over_rc;
    int rec;
    float rec_a, rec_b, rec_c;
    float rec_m2eta, rec_delta;  // uniform grid: -2 eta and the centre spacing Delta
    float rec_c4;                // rec_c^16, the step of four radial functions (when rec4)
    // radial table (TAB kernels): [(tab_n + 1)][K] cubic coefficients, spacing 1/tab_inv
    const float4* tab;
    float tab_inv;
    int tab_n;
    double L[3];
    // per-atom box edges (x, y, z) when the atoms of several systems share one
    // list (tmd_energy_forces_batch); nullptr: every atom's box is L
    const double4* boxes;
    const double4* xs;
    const int32_t* nbr;
    const int32_t* img;
    const int32_t* cnt;
    // work slot -> sorted atom (nullptr: identity); P is stored by work slot
    const int32_t* wperm;
    const float* mu;
    const float* eta;
    // forward output / backward input; with Gb non-null the forward output is
    // stored there as the bits of (__bf16)G instead (the BF16 MLP's operand)
    float* G;
    uint16_t* Gb;
    const float* dG;
    // P written by the forward pass (if non-null) and read back by the
    // adjoint: [S][K][DR][n] by work slot (VALU kernels); atom by atom,
    // [n][S][K][16], the components in order (row kernels) or as [4][4] with
    // element (set, i) = component kMfmaRow[i][set] (16x16x4 matrix-core
    // adjoint); or, for the matrix-core pair, one tile per 16-atom group g of
    // the work order,
    // [g][S][K/4][4][16][4][4]: element (kk, set, atom, j, i) =
    // P[4 kk + j][kMfmaRow[i][set]]
    float* Pbuf;
    // backward output: virial block partials
    double* vir;
};
// Arguments of a model and list (outputs unset); descriptor.hip.
PathArgs make_args(const tmd_model* m, const tmd_nlist* nl);

// Kernels with many lanes per atom (rows.hip), for lists without a work order
// of the models that row_kernels names: atoms per adjoint workgroup (a power of
// two, at most 256) for at most max_partials workgroups; the launches (a's outputs
// set; segs: the segment of each 256 atoms of a merged list, or null).
int adjoint_rows_atoms(int64_t n, int64_t max_partials);
tmd_status launch_descriptor_rows(tmd_context* ctx, const tmd_model* m, const PathArgs& a);
tmd_status launch_adjoint_rows(tmd_context* ctx, const tmd_model* m, const PathArgs& a, const int2* segs, int atoms,
                               unsigned long long* F);

struct Pair {
    float dx, dy, dz, r2;
    int q;     // neighbour (sorted index)
    int slot;  // where the entry's force goes: its LDS halo slot (LdsPos) or sorted index (GlobalPos)
};

template <int NB>
struct IntVec;
template <>
struct IntVec<2> {
    using T = int2;
    __device__ static void split(const int2& v, int* o) { o[0] = v.x, o[1] = v.y; }
};
template <>
struct IntVec<4> {
    using T = int4;
    __device__ static void split(const int4& v, int* o) { o[0] = v.x, o[1] = v.y, o[2] = v.z, o[3] = v.w; }
};

// Neighbour positions of list entries, in one of two places.  GlobalPos
// reads the sorted FP64 positions from HBM and forms D = (x_q - x_i) + n L in
// FP64.  LdsPos reads a workgroup's LDS copy of its cell block and one-cell
// halo, held as FP32 offsets from each atom's own cell origin: the entry's
// stencil offset (ox, oy, oz), stored as the bit fields ox+1, oy+1, oz+1 of
// its image word, names the halo slot (slot = centre's slot +
// (oz HY + oy) HX + ox; atom q of slot h sits at hoff[h] + q) and the cell
// offset, and D = (x_q - x_i) + o w with w the cell edge.  Both hand D to the
// caller in FP32 (the LDS form carries about 3e-7 A more rounding on |D| < 8 A).
struct GlobalPos {
    const double4* xs;
    double L0, L1, L2;
    double4 xi;
    __device__ double4 fetch(int q, int32_t, int& slot) const {
        slot = q;
        return xs[q];
    }
    __device__ float3 disp(const double4& xj, int32_t im) const {
        int nx, ny, nz;
        unpack_img(im, nx, ny, nz);
        return make_float3((float)((xj.x - xi.x) + (double)nx * L0), (float)((xj.y - xi.y) + (double)ny * L1),
                           (float)((xj.z - xi.z) + (double)nz * L2));
    }
};
struct LdsPos {
    const float* sp;  // [halo slot][3]
    const int32_t* hoff;
    int hp0;           // centre's halo slot minus (HX HY + HX + 1), the slot offset of the bit fields (0, 0, 0)
    int HX, HXY;       // halo cells along x, and per z layer
    float xi, yi, zi;  // centre atom from its cell origin, plus one cell edge
    float wx, wy, wz;  // cell edges
    __device__ float4 fetch(int q, int32_t im, int& slot) const {
        const int i = hoff[hp0 + img_sz(im) * HXY + img_sy(im) * HX + img_sx(im)] + q;
        slot = i;
        return make_float4(sp[3 * i], sp[3 * i + 1], sp[3 * i + 2], 0.0f);
    }
    // (x_q - x_i) + (b - 1) w = x_q - (x_i + w) + b w for the field b = o + 1
    __device__ float3 disp(const float4& xj, int32_t im) const {
        return make_float3(fmaf((float)img_sx(im), wx, xj.x - xi), fmaf((float)img_sy(im), wy, xj.y - yi),
                           fmaf((float)img_sz(im), wz, xj.z - zi));
    }
};

// NB consecutive entries c0 .. c0+NB-1 (c0 a multiple of NB) of a list row of
// nb (>= 1) entries starting at `row` (16-byte aligned): one vector load each
// for indices and image words, then all position loads, so the loads overlap.
// Entries past the row end are replaced by the last valid entry (never a
// stale slot) and marked with r2 = +inf so that every consumer skips them.
template <int NB, class Pos>
__device__ __forceinline__ void load_pairs(const PathArgs& a, int64_t row, int c0, int nb, Pair (&pr)[NB],
                                           const Pos& pos) {
    int q[NB], im[NB];
    IntVec<NB>::split(*reinterpret_cast<const typename IntVec<NB>::T*>(a.nbr + row + c0), q);
    IntVec<NB>::split(*reinterpret_cast<const typename IntVec<NB>::T*>(a.img + row + c0), im);
#pragma unroll
    for (int j = 1; j < NB; ++j)
        if (c0 + j >= nb) {  // entry c0 < nb is always valid
            q[j] = q[0];
            im[j] = im[0];
        }
    int slot[NB];
    decltype(pos.fetch(0, 0, slot[0])) xj[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) xj[j] = pos.fetch(q[j], im[j], slot[j]);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const float3 d = pos.disp(xj[j], im[j]);
        pr[j].dx = d.x;
        pr[j].dy = d.y;
        pr[j].dz = d.z;
        pr[j].r2 = (c0 + j < nb) ? pr[j].dx * pr[j].dx + pr[j].dy * pr[j].dy + pr[j].dz * pr[j].dz
                                 : __builtin_inff();
        pr[j].q = q[j];
        pr[j].slot = slot[j];
    }
}

// The value of the neighbouring lane (lane ^ 1), by a DPP quad permutation
// [1, 0, 3, 2] (no LDS crossbar).
__device__ __forceinline__ float swap_pair(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
}

// load_pairs for an atom whose list is walked by two adjacent lanes (its two
// radial chunks; both lanes see the same row): each lane fetches every other
// neighbour position and forms its displacement, and the two swap results, so
// the row's position gathers and FP64 geometry are done once per atom rather
// than once per lane.  The values are those of load_pairs bit for bit.
template <int NB, class Pos>
__device__ __forceinline__ void load_pairs_split2(const PathArgs& a, int64_t row, int c0, int nb, Pair (&pr)[NB],
                                                  const Pos& pos, int odd) {
    static_assert(NB % 2 == 0, "pairs are shared two at a time");
    int q[NB], im[NB];
    IntVec<NB>::split(*reinterpret_cast<const typename IntVec<NB>::T*>(a.nbr + row + c0), q);
    IntVec<NB>::split(*reinterpret_cast<const typename IntVec<NB>::T*>(a.img + row + c0), im);
#pragma unroll
    for (int j = 1; j < NB; ++j)
        if (c0 + j >= nb) {
            q[j] = q[0];
            im[j] = im[0];
        }
    int slot_unused;
    decltype(pos.fetch(0, 0, slot_unused)) xj[NB / 2];  // entries 2t + odd
#pragma unroll
    for (int t = 0; t < NB / 2; ++t)
        xj[t] = pos.fetch(odd ? q[2 * t + 1] : q[2 * t], odd ? im[2 * t + 1] : im[2 * t], slot_unused);
#pragma unroll
    for (int t = 0; t < NB / 2; ++t) {
        const float3 mine = pos.disp(xj[t], odd ? im[2 * t + 1] : im[2 * t]);
        const float3 other = make_float3(swap_pair(mine.x), swap_pair(mine.y), swap_pair(mine.z));
        const float3 d0 = odd ? other : mine, d1 = odd ? mine : other;
        pr[2 * t].dx = d0.x;
        pr[2 * t].dy = d0.y;
        pr[2 * t].dz = d0.z;
        pr[2 * t + 1].dx = d1.x;
        pr[2 * t + 1].dy = d1.y;
        pr[2 * t + 1].dz = d1.z;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        pr[j].r2 = (c0 + j < nb) ? pr[j].dx * pr[j].dx + pr[j].dy * pr[j].dy + pr[j].dz * pr[j].dz
                                 : __builtin_inff();
        pr[j].q = q[j];
        pr[j].slot = q[j];  // the descriptor has no force sink
    }
}

constexpr int kBatchFwd = 4;
constexpr int kBatchAdj = 2;

// A thread's KC x DR tile of P (its kept components) in the element-major
// buffer [S][K][DR][n]: element (k, r) of work slot w lives at
// ((b*K + k)*DR + r)*n + w, so for a fixed
// element the lanes of a wave (consecutive slots, two chunks) write and read
// whole contiguous cache lines.  P (2 GB at 1 M atoms) is written once and
// read once by the adjoint, far more than the L2 holds.  With at most two
// chunk lanes per atom every store instruction writes whole 128-byte lines,
// and those go out non-temporally (measured: less L2 pollution for the next
// kernel); with more chunks a store covers 32-byte pieces, which must merge in
// L2 (non-temporal stores were up to five times slower there).
template <int KC, int D, bool NT>
__device__ __forceinline__ void store_tile(float* dst, int64_t n, const float (&P)[KC][D]) {
#pragma unroll
    for (int q = 0; q < KC * D; ++q) {
        if constexpr (NT)
            __builtin_nontemporal_store(P[q / D][q % D], dst + (int64_t)q * n);
        else
            dst[(int64_t)q * n] = P[q / D][q % D];
    }
}

// Kept components (reduced index) of the matrix-core kernels' slices:
// entry n of slice q is kMfmaRow[q][n]; column n, (kMfmaRow[0..3][n]), is fold
// set n: the three kept components tied by the unit-norm identity to one
// dropped component, and one more.
__device__ constexpr int kMfmaRow[4][4] = {{0, 1, 2, 3}, {4, 9, 10, 11}, {7, 12, 14, 15}, {5, 6, 8, 13}};

// The same tile (M = 3) in the atom-major layout [n][S][K][4][4] of the
// large-K matrix-core adjoint: per radial function the four fold sets, each a float4 (kMfmaRow[0..3][g]), so that a lane moves its
// fold set with one instruction.
template <int KC, int D>
__device__ __forceinline__ void store_tile_am(float* dst, const float (&P)[KC][D]) {
    static_assert(D == 16, "the 16-component basis");
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(dst + kk * 16 + 4 * g) =
                make_float4(P[kk][kMfmaRow[0][g]], P[kk][kMfmaRow[1][g]], P[kk][kMfmaRow[2][g]], P[kk][kMfmaRow[3][g]]);
}
template <int KC, int D>
__device__ __forceinline__ void load_tile(const float* src, int64_t n, float (&P)[KC][D]) {
#pragma unroll
    for (int q = 0; q < KC * D; ++q) P[q / D][q % D] = src[(int64_t)q * n];
}

// Gaussians exp(-eta_k (R - mu_k)^2) of a chunk of KC radial functions
// (mu, nef = -eta log2 e of the chunk).  On a uniform grid (a.rec) two
// exponentials and a multiplicative recurrence replace the KC exponentials:
// e_{k+1} = e_k r_k, r_k = exp2(rec_a (R - mu_k) + rec_b), r_{k+1} = r_k rec_c.
template <int KC>
__device__ __forceinline__ void gaussians_rec(const PathArgs& a, float R, const float* mu, const float* nef,
                                              float (&e)[KC]) {
    const float t0 = R - mu[0];
    float ek = __builtin_amdgcn_exp2f(nef[0] * t0 * t0);
    float rk = __builtin_amdgcn_exp2f(fmaf(a.rec_a, t0, a.rec_b));
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        e[kk] = ek;
        ek *= rk;
        rk *= a.rec_c;
    }
}
template <int KC>
__device__ __forceinline__ void gaussians_direct(float R, const float* mu, const float* nef, float (&e)[KC]) {
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const float t = R - mu[kk];
        e[kk] = __builtin_amdgcn_exp2f(nef[kk] * t * t);
    }
}
template <int KC>
__device__ __forceinline__ void gaussians(const PathArgs& a, float R, const float* mu, const float* nef,
                                          float (&e)[KC]) {
    if (a.rec) gaussians_rec<KC>(a, R, mu, nef, e);
    else gaussians_direct<KC>(R, mu, nef, e);
}

// How the adjoint kernels evaluate the radial functions (a template
// parameter, so that each instantiation keeps only its own registers):
// directly, by the uniform-grid recurrence, or from the table.
constexpr int kRadDirect = 0, kRadRec = 1, kRadTab = 2;

// Chunk k0 .. k0+KC-1 of the tabulated radial functions at distance R (the
// caller has R < rc): interval j = floor(R / delta), clamped to the zero row
// tab_n, local t = R / delta - j, h = c0 + t(c1 + t(c2 + t c3)) and, with DH,
// h' = (c1 + t(2 c2 + 3 t c3)) / delta.  The KC coefficient quadruples of a
// thread are one contiguous 16*KC-byte run of the table.
template <int KC, bool DH>
__device__ __forceinline__ void tabulated(const PathArgs& a, float R, int k0, float (&h)[KC], float (&dh)[KC]) {
    const float x = R * a.tab_inv;
    const float jf = fminf(floorf(x), (float)a.tab_n);
    const float t = x - jf;
    const float4* row = a.tab + (int64_t)jf * a.K + k0;
    float4 c[KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) c[kk] = row[kk];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        h[kk] = fmaf(t, fmaf(t, fmaf(t, c[kk].w, c[kk].z), c[kk].y), c[kk].x);
        if (DH) dh[kk] = fmaf(t, fmaf(3.0f * t, c[kk].w, 2.0f * c[kk].z), c[kk].y) * a.tab_inv;
    }
}

// ---- adjoint ---------------------------------------------------------------
//
// Force sums.  Each pair's g is added to the neighbour's force (F_j -= g) by
// an atomic add, first into the workgroup's LDS accumulators and then into
// the global ones.  The adds are made on 64-bit fixed-point integers with 32
// fractional bits: integer addition is associative, so the result does not
// depend on the order in which the atomics land and the forces are the same
// bit for bit on every run (float atomics would round in arrival order).
// A contribution g is split as g = hi + fr with hi = floor(g) (an integer,
// exact in FP32 for |g| < 2^31) and fr in [0, 1) (exact); fr 2^32 is exact
// too and converts to the low word (truncating only bits below 2^-32), hi to
// the high word, which together are the two's-complement integer g 2^32.
__device__ __forceinline__ unsigned long long to_fixed(float g) {
    const float hi = floorf(g);
    const unsigned lo = (unsigned)((g - hi) * 4294967296.0f);
    return ((unsigned long long)(unsigned)(int)hi << 32) | lo;
}

// P' = 2 T sigma' P in place for one species' KC x D tile (sigma' = dE/dS
// from dE/dG): for m = 0, G = sqrt(P_k0^2) = |P_k0|, so P'_k0 = G' sign(P_k0)
// (0 where P_k0 = 0; no reciprocal square root of a possibly denormal S).
template <int KC, int M>
__device__ __forceinline__ void tile_adjoint(const float* dGp, float (&P)[KC][Moments<M>::D]) {
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
#pragma unroll
        for (int m = 0; m <= M; ++m) {
            const float gbar = dGp[kk * (M + 1) + m];
            if (m == 0) {
                const float pk = P[kk][0];
                P[kk][0] = pk > 0.0f ? gbar : (pk < 0.0f ? -gbar : 0.0f);
            } else {
#pragma unroll
                for (int d = kOrderStart[m]; d < kOrderStart[m + 1]; ++d) P[kk][d] *= 2.0f * kMult[d] * gbar;
            }
        }
    }
}

// This thread's P' tile of species b in the kept basis: the stored kept
// components of P, expanded, turned into P' and folded back.
template <int KC, int M>
__device__ __forceinline__ void adjoint_tile(const PathArgs& a, int64_t p, int64_t w, int b, int ch,
                                             float (&Pr)[KC][Moments<M>::DR]) {
    constexpr int D = Moments<M>::D, DR = Moments<M>::DR;
    float P[KC][D];
    load_tile<KC, DR>(a.Pbuf + ((int64_t)(b * a.K + ch * KC) * DR) * a.n + w, a.n, Pr);
    expand_P<M, KC>(Pr, P);
    tile_adjoint<KC, M>(a.dG + p * a.F + (b * a.K + ch * KC) * (M + 1), P);
    fold_Pbar<M, KC>(P, Pr);
}

// U += sum_d P_d M_d and V_d += P_d h, d in order.
template <int D>
__device__ __forceinline__ void moment_sums(const float (&P)[D], const float (&Mv)[D], float h, float& U,
                                            float (&V)[D]) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
        U = fmaf(P[d], Mv[d], U);
        V[d] = fmaf(P[d], h, V[d]);
    }
}

// This chunk's share of g = dE/dD for one pair within the cutoff:
// U_k = sum_d P'_kd M_d, V_d = sum_k P'_kd h_k,
// g = (sum_k U_k h'_k) u + (1/R)(sum_d V_d grad_u M_d - u sum_d ord(d) V_d M_d).
// P: the tile P' folded onto the kept basis, indexed [kk] (the rows' own
// moment_sums adds them).  FUSED: the last multiply-add of each
// component is written out (as the compiler forms it in k_adjoint_atomic).
template <int KC, int M, int RAD, bool FUSED = false, class Tile>
__device__ __forceinline__ void pair_grad(const PathArgs& a, float dx, float dy, float dz, float r2, int k0,
                                          const float* mu, const float* nef, const float* m2eta,
                                          const Tile& P, float& gx, float& gy, float& gz) {
    constexpr int D = Moments<M>::DR;
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float R = r2 * rinv;
    const float ux = dx * rinv, uy = dy * rinv, uz = dz * rinv;
    float Mv[D];
    reduced_monomials<M>(ux, uy, uz, Mv);
    float V[D];
#pragma unroll
    for (int d = 0; d < D; ++d) V[d] = 0.0f;
    if constexpr (RAD == kRadRec) {
        // Uniform grid (mu_k = mu_0 + k Delta, one eta): with e_k the bare
        // Gaussians, h_k = e_k f_c and h'_k = e_k (-2 eta (t0 - k Delta) f_c + f_c'),
        // t0 = R - mu_0, so sum_k U_k h'_k = -2 eta f_c (t0 S0 - Delta S1) + f_c' S0
        // with S0 = sum_k U_k e_k and S1 = sum_k k U_k e_k, and f_c, being common
        // to every V_d, factors out of the moment adjoint.
        const float ang = R * a.half_inv_rc;
        const float fc = 0.5f * __builtin_amdgcn_cosf(ang) + 0.5f;
        const float dfc = -0.5f * a.pi_over_rc * __builtin_amdgcn_sinf(ang);
        float e[KC];
        gaussians_rec<KC>(a, R, mu, nef, e);
        float S0 = 0.0f, S1 = 0.0f;
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            float U = 0.0f;
            moment_sums<D>(P[kk], Mv, e[kk], U, V);
            const float Ue = U * e[kk];
            S0 += Ue;
            S1 = fmaf((float)kk, Ue, S1);
        }
        const float t0 = R - mu[0];
        const float s1 = fmaf(a.rec_m2eta * fc, fmaf(-a.rec_delta, S1, t0 * S0), dfc * S0);
        float Ax, Ay, Az, B;
        reduced_moment_adjoint<M>(ux, uy, uz, V, Mv, Ax, Ay, Az, B);
        const float rf = rinv * fc;
        if constexpr (FUSED) {
            gx = fmaf(rf, fmaf(-ux, B, Ax), s1 * ux);
            gy = fmaf(rf, fmaf(-uy, B, Ay), s1 * uy);
            gz = fmaf(rf, fmaf(-uz, B, Az), s1 * uz);
            return;
        }
        gx = s1 * ux + rf * (Ax - ux * B);
        gy = s1 * uy + rf * (Ay - uy * B);
        gz = s1 * uz + rf * (Az - uz * B);
        return;
    }
    float s1 = 0.0f, hv[KC], dhv[KC];
    if constexpr (RAD == kRadTab) {
        tabulated<KC, true>(a, R, k0, hv, dhv);
    } else {
        const float ang = R * a.half_inv_rc;
        const float fc = 0.5f * __builtin_amdgcn_cosf(ang) + 0.5f;
        const float dfc = -0.5f * a.pi_over_rc * __builtin_amdgcn_sinf(ang);
        gaussians_direct<KC>(R, mu, nef, hv);
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            const float e = hv[kk];
            hv[kk] = e * fc;
            dhv[kk] = e * fmaf(m2eta[kk] * (R - mu[kk]), fc, dfc);
        }
    }
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const float h = hv[kk];
        const float dh = dhv[kk];
        float U = 0.0f;
        moment_sums<D>(P[kk], Mv, h, U, V);
        s1 = fmaf(U, dh, s1);
    }
    float Ax, Ay, Az, B;
    reduced_moment_adjoint<M>(ux, uy, uz, V, Mv, Ax, Ay, Az, B);
    if constexpr (FUSED) {
        gx = fmaf(s1, ux, rinv * fmaf(-ux, B, Ax));
        gy = fmaf(s1, uy, rinv * fmaf(-uy, B, Ay));
        gz = fmaf(s1, uz, rinv * fmaf(-uz, B, Az));
        return;
    }
    gx = s1 * ux + rinv * (Ax - ux * B);
    gy = s1 * uy + rinv * (Ay - uy * B);
    gz = s1 * uz + rinv * (Az - uz * B);
}

// Virial of one pair: w6 -= D (x) g, off-diagonals symmetrised.
__device__ __forceinline__ void virial_add(float (&w6)[6], float dx, float dy, float dz, float gx, float gy, float gz) {
    w6[0] -= dx * gx;
    w6[1] -= dy * gy;
    w6[2] -= dz * gz;
    w6[3] -= 0.5f * (dx * gy + dy * gx);
    w6[4] -= 0.5f * (dx * gz + dz * gx);
    w6[5] -= 0.5f * (dy * gz + dz * gy);
}

// Radial parameters of this thread's chunk k0 .. k0+KC-1.
template <int KC>
__device__ __forceinline__ void chunk_params(const PathArgs& a, int k0, float (&mu)[KC], float (&nef)[KC],
                                             float (&m2eta)[KC]) {
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        mu[kk] = a.mu[k0 + kk];
        nef[kk] = -a.eta[k0 + kk] * kLog2e;
        m2eta[kk] = -2.0f * a.eta[k0 + kk];
    }
}

struct CompD {
    double s, c;
};
__device__ __forceinline__ CompD comp_merge_d(CompD a, CompD b) {
    const double t = a.s + b.s;
    if (fabs(a.s) >= fabs(b.s)) a.c += (a.s - t) + b.s;
    else a.c += (b.s - t) + a.s;
    a.s = t;
    a.c += b.c;
    return a;
}

}  // namespace tmd
