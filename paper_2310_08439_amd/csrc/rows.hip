// Descriptor and adjoint with 16 lanes per atom (M = 3, K = 4, 8, 12 or 16
// radial functions), for lists without a work order: systems with a box edge
// below one list cutoff (or a grid that no block shape fits, or rows of more
// than ~2,400 entries), and the merged list of several systems.  A wave walks
// the list rows of its atoms 16 entries at a time.  Every sum (P over the row,
// the atom's force and its virial over the row) runs in the order of the row
// with the roundings of the kernels in descriptor.hip that take one lane per
// atom and chunk, so the two agree bit for bit.
#include "pair_ops.h"

#include <algorithm>

namespace tmd {
namespace {

// Lanes of the wave see each other's LDS writes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// acc_q += (lane i's h_q) m for six or four q: the lane's value comes by row
// broadcast (DPP), an operand modifier of the multiply-add itself.  Written as
// assembly because the compiler turns the builtin into a move of its own per
// element and hoists those out of the loops into registers it does not have.
// Every lane must be active; the s_nop covers a value written just before.
#define TMD_FMAC_ROW(acc, h, m, i) "v_fmac_f32_dpp " acc ", " h ", " m " row_newbcast:" i " row_mask:0xf bank_mask:0xf\n\t"
template <int I>
__device__ __forceinline__ void row_fma(float (&acc)[6], const float (&h)[6], float m) {
    asm("s_nop 1\n\t" TMD_FMAC_ROW("%0", "%6", "%12", "%13") TMD_FMAC_ROW("%1", "%7", "%12", "%13")
            TMD_FMAC_ROW("%2", "%8", "%12", "%13") TMD_FMAC_ROW("%3", "%9", "%12", "%13")
                TMD_FMAC_ROW("%4", "%10", "%12", "%13") TMD_FMAC_ROW("%5", "%11", "%12", "%13")
        : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(acc[4]), "+&v"(acc[5])
        : "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]), "v"(h[4]), "v"(h[5]), "v"(m), "n"(I));
}
template <int I>
__device__ __forceinline__ void row_fma(float (&acc)[4], const float (&h)[4], float m) {
    asm("s_nop 1\n\t" TMD_FMAC_ROW("%0", "%4", "%8", "%9") TMD_FMAC_ROW("%1", "%5", "%8", "%9")
            TMD_FMAC_ROW("%2", "%6", "%8", "%9") TMD_FMAC_ROW("%3", "%7", "%8", "%9")
        : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
        : "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]), "v"(m), "n"(I));
}
template <int I>
__device__ __forceinline__ void row_fma(float& acc, float h, float m) {
    asm("s_nop 1\n\t" TMD_FMAC_ROW("%0", "%1", "%2", "%3") : "+&v"(acc) : "v"(h), "v"(m), "n"(I));
}
// Entry I's terms: P += h M, and P0 += e f_c.
template <int I, int NC, int KC>
__device__ __forceinline__ void add_entry(float (&P)[NC][KC], const float (&h)[NC][KC], float m, float& P0, float fc,
                                          float e) {
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) row_fma<I>(P[ch], h[ch], m);
    row_fma<I>(P0, fc, e);
}
template <int I, int NC, int KC>
__device__ __forceinline__ void add_four(float (&P)[NC][KC], const float (&h)[NC][KC], const float* m, float& P0,
                                         float fc, const float* e) {
    const float4 m4 = *reinterpret_cast<const float4*>(m + I), e4 = *reinterpret_cast<const float4*>(e + I);
    add_entry<I>(P, h, m4.x, P0, fc, e4.x);
    add_entry<I + 1>(P, h, m4.y, P0, fc, e4.y);
    add_entry<I + 2>(P, h, m4.z, P0, fc, e4.z);
    add_entry<I + 3>(P, h, m4.w, P0, fc, e4.w);
}
__device__ __forceinline__ void load_tile_row(const float* src, float (&P)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(src + 4 * q);
        P[4 * q] = v.x, P[4 * q + 1] = v.y, P[4 * q + 2] = v.z, P[4 * q + 3] = v.w;
    }
}

// Stride of a column of 16 values in LDS (16-byte reads of four of them).
constexpr int kCol = 20;

// ---- descriptor --------------------------------------------------------------
//
// 16 lanes per atom, K = KC NC radial functions.  Per 16 entries of the row:
// lane = entry forms the pair's monomials and radial values; then lane = moment
// component d adds h_k M_d of entry after entry to its P_kd, h_k by row
// broadcast from the entry's lane and M_d from a transpose in LDS, so a
// multiply-add is one instruction and 4 entries take one 16-byte read.
// Bound by vector instructions (13 an entry and atom at K = 12, and ~170 per
// 16 entries for the pairs): 40 systems of 54 to 4,096 atoms, K = 12: 48 us
// (a lane per (atom, chunk), rows not pruned to the cutoff 98 us; radial values
// from LDS 52 us).
template <int KC, int NC, bool TAB>
__global__ void __launch_bounds__(256) k_descriptor_rows(PathArgs a, int64_t nblocks) {
    constexpr int K = KC * NC, kAtom = (15 + K) * kCol + 8;  // (+ 8: the four atoms' columns in other banks)
    __shared__ __align__(16) float lds[kBlock / 64][4 * kAtom];
    const int64_t lb = xcd_block(nblocks);
    if (lb < 0) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, al = lane >> 4, l = lane & 15;
    const int64_t w = (lb * (kBlock / 64) + wv) * 4 + al;
    const bool active = w < a.n;
    const int64_t p = active ? w : 0;
    const double4 Lp = a.boxes ? a.boxes[p] : make_double4(a.L[0], a.L[1], a.L[2], 0.0);
    const GlobalPos pos{a.xs, Lp.x, Lp.y, Lp.z, a.xs[p]};
    float* const cm = &lds[wv][al * kAtom];  // monomials 1 .. 15, then the Gaussians
    float* const ce = cm + 15 * kCol;
    const float* const my_m = cm + (max(l, 1) - 1) * kCol;
    const float* const my_e = ce + min(l, K - 1) * kCol;
    for (int b = 0; b < a.S; ++b) {
        const int nb = active ? a.cnt[(int64_t)b * a.n + p] : 0;
        const int64_t base = (p * a.S + b) * a.cap;
        float P[NC][KC], P0 = 0.0f;  // lane d: P_kd; lane k: P_k0
#pragma unroll
        for (int k = 0; k < K; ++k) P[k / KC][k % KC] = 0.0f;
        for (int c0 = 0; __any(c0 < nb); c0 += 16) {
            // the entry's values; zeros past the row's end and beyond the cutoff
            const int c = c0 + l;
            float Mv[16] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            float hv[NC][KC], ev[K], fc = 0.0f;
#pragma unroll
            for (int k = 0; k < K; ++k) hv[k / KC][k % KC] = ev[k] = 0.0f;
            float r2 = __builtin_inff();
            float3 d = make_float3(0.0f, 0.0f, 0.0f);
            if (c < nb) {
                const int32_t im = a.img[base + c];
                int slot;
                d = pos.disp(pos.fetch(a.nbr[base + c], im, slot), im);
                r2 = d.x * d.x + d.y * d.y + d.z * d.z;
            }
            if (!(r2 >= a.rc2)) {  // (a NaN distance is not passed over)
                const float rinv = __builtin_amdgcn_rsqf(r2), R = r2 * rinv;
                reduced_monomials<3>(d.x * rinv, d.y * rinv, d.z * rinv, Mv);
                fc = TAB ? 1.0f : 0.5f * __builtin_amdgcn_cosf(R * a.half_inv_rc) + 0.5f;
#pragma unroll
                for (int ch = 0; ch < NC; ++ch) {
                    float h[KC];
                    if constexpr (TAB) {
                        tabulated<KC, false>(a, R, ch * KC, h, h);
                    } else {
                        // a chunk's first offset R - mu with one rounding, the
                        // others from the rounded R
                        const float t0 = fmaf(r2, rinv, -a.mu[ch * KC]), nef0 = -a.eta[ch * KC] * kLog2e;
                        h[0] = __builtin_amdgcn_exp2f(nef0 * t0 * t0);
                        if (a.rec) {
                            float rk = __builtin_amdgcn_exp2f(fmaf(a.rec_a, t0, a.rec_b));
#pragma unroll
                            for (int kk = 1; kk < KC; ++kk) {
                                h[kk] = h[kk - 1] * rk;
                                rk *= a.rec_c;
                            }
                        } else {
#pragma unroll
                            for (int kk = 1; kk < KC; ++kk) {
                                const float t = __fsub_rn(R, a.mu[ch * KC + kk]);
                                h[kk] = __builtin_amdgcn_exp2f(-a.eta[ch * KC + kk] * kLog2e * t * t);
                            }
                        }
                    }
#pragma unroll
                    for (int kk = 0; kk < KC; ++kk) {
                        ev[ch * KC + kk] = h[kk];
                        hv[ch][kk] = TAB ? h[kk] : h[kk] * fc;
                    }
                }
            }
#pragma unroll
            for (int q = 1; q < 16; ++q) cm[(q - 1) * kCol + l] = Mv[q];
#pragma unroll
            for (int k = 0; k < K; ++k) ce[k * kCol + l] = ev[k];
            wave_sync();
            // past the end of the longest row the entries are zeros
            int left = nb - c0;
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) left = max(left, __shfl_xor(left, off));
            left = __builtin_amdgcn_readfirstlane(left);
            add_four<0>(P, hv, my_m, P0, fc, my_e);
            if (left > 4) add_four<4>(P, hv, my_m, P0, fc, my_e);
            if (left > 8) add_four<8>(P, hv, my_m, P0, fc, my_e);
            if (left > 12) add_four<12>(P, hv, my_m, P0, fc, my_e);
            wave_sync();
        }
        // P by radial function: lane = k
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (l > 0) cm[k * kCol + l] = P[k / KC][k % KC];
        if (l < K) cm[l * kCol] = P0;
        wave_sync();
        if (l < K && active) {
            float Pr[1][16], Pf[1][20];
            load_tile_row(cm + l * kCol, Pr[0]);
            if (a.Pbuf) {
                float4* dst = reinterpret_cast<float4*>(a.Pbuf + ((p * a.S + b) * K + l) * 16);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    dst[q] = make_float4(Pr[0][4 * q], Pr[0][4 * q + 1], Pr[0][4 * q + 2], Pr[0][4 * q + 3]);
            }
            expand_P<3, 1>(Pr, Pf);
            float f[4];
#pragma unroll
            for (int m = 0; m <= 3; ++m) {
                float s = 0.0f;
#pragma unroll
                for (int q = kOrderStart[m]; q < kOrderStart[m + 1]; ++q) s += kMult[q] * Pf[0][q] * Pf[0][q];
                f[m] = (m == 0) ? fabsf(Pf[0][0]) : s;
            }
            const int64_t gi = p * a.F + ((int64_t)b * K + l) * 4;
            if (a.Gb) {
                ushort4 o;
                o.x = __builtin_bit_cast(uint16_t, (__bf16)f[0]);
                o.y = __builtin_bit_cast(uint16_t, (__bf16)f[1]);
                o.z = __builtin_bit_cast(uint16_t, (__bf16)f[2]);
                o.w = __builtin_bit_cast(uint16_t, (__bf16)f[3]);
                *reinterpret_cast<ushort4*>(a.Gb + gi) = o;
            } else {
                *reinterpret_cast<float4*>(a.G + gi) = make_float4(f[0], f[1], f[2], f[3]);
            }
        }
        wave_sync();
    }
}

// ---- adjoint -----------------------------------------------------------------
//
// K = KC NCH <= 16 radial functions, 16 lanes per atom: lane = (entry, chunk of
// KC).  P' is formed by one lane per radial function and read from LDS, the
// same row by all lanes of an atom's chunk.  A pair's g goes to the neighbour
// through the workgroup's LDS window of force accumulators, W consecutive atoms
// (cyclic) of the system around the workgroup's own; what falls outside goes
// to the global ones.  Nine lanes of the atom then add the 16 / NCH pairs'
// virial and force terms in row order.
//
// Bound by vector instructions (about 250 a pair and chunk in pair_grad, half
// as many again around it).  40 systems of 54 to 4,096 atoms, K = 12: 73 us;
// one lane per (atom, chunk) with global atomics (three 8-byte ones a pair,
// ~15 G/s) 362 us.  The window as large as lets two workgroups onto a CU: 512
// atoms 117, 1,024 92, 2,048 (one workgroup) 130 us; 64 atoms per workgroup
// 97 us, 128 110 us.  P' by row broadcast instead of from LDS 89 us.
constexpr int kRowThreads = 512, kRowWaves = kRowThreads / 64, kRowAtoms = 32;
constexpr int row_window(int K) { return K > 12 ? 1280 : 1536; }

struct LdsTile {  // rows of P' fetched one at a time
    struct Row {
        float v[16];
    };
    const float* p;
    __device__ __forceinline__ Row operator[](int kk) const {
        Row r;
        load_tile_row(p + kk * 16, r.v);
        return r;
    }
};
template <int D>
__device__ __forceinline__ void moment_sums(const LdsTile::Row& P, const float (&Mv)[D], float h, float& U,
                                            float (&V)[D]) {
    tmd::moment_sums<D>(P.v, Mv, h, U, V);
}

template <int KC, int NCH, int RAD>
__global__ void __launch_bounds__(kRowThreads, RAD == kRadDirect && KC * NCH == 16 ? 2 : 4)
    k_adjoint_rows(PathArgs a, unsigned long long* F, int atoms, int W, const int2* __restrict__ segs) {
    constexpr int K = KC * NCH, LP = 16 / NCH, kTile = KC * 16 + 4, kPairs = LP + 4;
    constexpr int kAtom = NCH * kTile + 9 * kPairs;
    extern __shared__ __align__(16) unsigned char dyn[];
    unsigned long long* const win = reinterpret_cast<unsigned long long*>(dyn);
    __shared__ __align__(16) float stage[kRowWaves][4 * kAtom];
    __shared__ double red[6][kRowWaves][2];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int al = lane >> 4, l = lane & 15, ch = l & (NCH - 1), pr = l / NCH;
    const int64_t w0 = (int64_t)blockIdx.x * atoms;  // first atom of the workgroup
    // (segments are padded to a multiple of the atoms of a workgroup)
    const int2 seg = segs ? segs[w0 / kBlock] : make_int2(0, (int)a.n);
    const int start = seg.y > W ? (int)(((w0 - seg.x) + atoms / 2 + seg.y - W / 2) % seg.y) : 0;
    const int nwin = 3 * min(W, seg.y);
    for (int i = t; i < nwin; i += kRowThreads) win[i] = 0ull;
    __syncthreads();
    auto slot_of = [&](int q) {
        const int d = q - seg.x - start;
        return d < 0 ? d + seg.y : d;
    };
    float mu[KC], nef[KC], m2eta[KC];
    chunk_params<KC>(a, ch * KC, mu, nef, m2eta);
    // columns of LP pairs: -D (3), g (3), the off-diagonal virial terms (3).
    // Lane j < 9 of an atom sums column B times column A or a constant: the
    // virial (w -= D g, w -= 1/2 (..)), then the force (f += g).
    float* const tile = &stage[wv][al * kAtom];
    float* const sg = tile + NCH * kTile;
    const LdsTile P{tile + ch * kTile};
    const float* const colA = sg + (l < 3 ? l : 0) * kPairs;
    const float* const colB = sg + (l < 6 ? 3 + l : (l < 9 ? l - 3 : 0)) * kPairs;
    const float cA = l < 6 ? -0.5f : 1.0f;
    double Wd = 0.0;
    for (int r = 0; r < atoms; r += 4 * kRowWaves) {
        const int64_t p = w0 + r + wv * 4 + al;
        const bool active = p < a.n;
        const double4 Lp = a.boxes ? a.boxes[active ? p : 0] : make_double4(a.L[0], a.L[1], a.L[2], 0.0);
        const GlobalPos pos{a.xs, Lp.x, Lp.y, Lp.z, a.xs[active ? p : 0]};
        float Fo = 0.0f;
        for (int b = 0; b < a.S; ++b) {
            const int nb = active ? a.cnt[(int64_t)b * a.n + p] : 0;
            if (!__any(nb > 0)) continue;
            const int64_t base = (p * a.S + b) * a.cap;
            if (l < K) {  // lane = radial function
                float Pr[1][16] = {{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}}, Pf[1][20];
                if (nb > 0) {
                    load_tile_row(a.Pbuf + ((p * a.S + b) * K + l) * 16, Pr[0]);
                    expand_P<3, 1>(Pr, Pf);
                    tile_adjoint<1, 3>(a.dG + p * a.F + (b * K + l) * 4, Pf);
                    fold_Pbar<3, 1>(Pf, Pr);
                }
                float4* dst = reinterpret_cast<float4*>(tile + (l / KC) * kTile + (l % KC) * 16);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    dst[q] = make_float4(Pr[0][4 * q], Pr[0][4 * q + 1], Pr[0][4 * q + 2], Pr[0][4 * q + 3]);
            }
            wave_sync();
            float acc = l < 6 ? 0.0f : Fo;
            for (int c0 = 0; __any(c0 < nb); c0 += LP) {
                const int c = c0 + pr;
                // lanes without a pair run a harmless one and drop the result
                float3 d = make_float3(1.0f, 0.0f, 0.0f);
                float r2 = 1.0f;
                int q = 0;
                bool in = false;
                if (c < nb) {
                    const int32_t im = a.img[base + c];
                    const float3 e = pos.disp(pos.fetch(a.nbr[base + c], im, q), im);
                    const float e2 = e.x * e.x + e.y * e.y + e.z * e.z;
                    in = !(e2 >= a.rc2);
                    if (in) d = e, r2 = e2;
                }
                float gx, gy, gz;
                pair_grad<KC, 3, RAD, true>(a, d.x, d.y, d.z, r2, ch * KC, mu, nef, m2eta, P, gx, gy, gz);
                if (NCH == 2) {
                    gx += swap_pair(gx);
                    gy += swap_pair(gy);
                    gz += swap_pair(gz);
                }
                if (!in) {
                    d = make_float3(0.0f, 0.0f, 0.0f);
                    gx = gy = gz = 0.0f;
                }
                // a pair's first lane stages and adds x and y, its last the rest
                if (ch == 0) {
                    sg[0 * kPairs + pr] = -d.x;
                    sg[1 * kPairs + pr] = -d.y;
                    sg[2 * kPairs + pr] = -d.z;
                    sg[3 * kPairs + pr] = gx;
                    sg[4 * kPairs + pr] = gy;
                }
                if (ch == NCH - 1) {
                    sg[5 * kPairs + pr] = gz;
                    sg[6 * kPairs + pr] = fmaf(d.y, gx, d.x * gy);  // (roundings as in virial_add)
                    sg[7 * kPairs + pr] = fmaf(d.z, gx, d.x * gz);
                    sg[8 * kPairs + pr] = fmaf(d.z, gy, d.y * gz);
                }
                if (in) {
                    const bool xy = NCH == 1 || ch == 0;
                    const unsigned long long f0 = to_fixed(xy ? -gx : -gz), f1 = to_fixed(-gy);
                    const unsigned long long f2 = NCH == 1 ? to_fixed(-gz) : 0ull;
                    const int dq = slot_of(q), c0q = xy ? 0 : 2;
                    if (dq < W) {
                        unsigned long long* f = win + 3 * dq;
                        atomicAdd(f + c0q, f0);
                        if (xy) atomicAdd(f + 1, f1);
                        if (NCH == 1) atomicAdd(f + 2, f2);
                    } else {
                        asm volatile("");  // kept apart: one add through a flat pointer would serve neither well
                        unsigned long long* f = F + 3 * (int64_t)q;
                        atomicAdd(f + c0q, f0);
                        if (xy) atomicAdd(f + 1, f1);
                        if (NCH == 1) atomicAdd(f + 2, f2);
                    }
                }
                wave_sync();
#pragma unroll
                for (int i = 0; i < LP; i += 4) {
                    const float4 A = *reinterpret_cast<const float4*>(colA + i);
                    const float4 B = *reinterpret_cast<const float4*>(colB + i);
                    acc = fmaf(l < 3 ? A.x : cA, B.x, acc);
                    acc = fmaf(l < 3 ? A.y : cA, B.y, acc);
                    acc = fmaf(l < 3 ? A.z : cA, B.z, acc);
                    acc = fmaf(l < 3 ? A.w : cA, B.w, acc);
                }
                wave_sync();
            }
            if (l < 6) Wd += (double)acc;
            else Fo = acc;
        }
        if (active && l >= 6 && l < 9) {
            const int dq = slot_of((int)p);
            if (dq < W) {
                atomicAdd(&win[3 * dq + l - 6], to_fixed(Fo));
            } else {
                asm volatile("");
                atomicAdd(&F[3 * p + l - 6], to_fixed(Fo));
            }
        }
    }
    __syncthreads();
    for (int i = t; i < nwin; i += kRowThreads) {
        const unsigned long long f = win[i];
        if (f == 0ull) continue;
        int q = i / 3 + start;
        if (q >= seg.y) q -= seg.y;
        atomicAdd(&F[3 * (int64_t)(seg.x + q) + i % 3], f);
    }
    // the workgroup's virial: the rows of a wave, then the waves in turn
    CompD v{l < 6 ? Wd : 0.0, 0.0};
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
        const CompD o{__shfl_xor(v.s, off), __shfl_xor(v.c, off)};
        v = (lane & off) ? comp_merge_d(o, v) : comp_merge_d(v, o);
    }
    if (lane < 6) {
        red[lane][wv][0] = v.s;
        red[lane][wv][1] = v.c;
    }
    __syncthreads();
    if (t < 6) {
        CompD s{0.0, 0.0};
        for (int q = 0; q < kRowWaves; ++q) s = comp_merge_d(s, CompD{red[t][q][0], red[t][q][1]});
        a.vir[(int64_t)blockIdx.x * kVirDoubles + 2 * t] = s.s;
        a.vir[(int64_t)blockIdx.x * kVirDoubles + 2 * t + 1] = s.c;
    }
}

using DescFn = void (*)(PathArgs, int64_t);
using AdjFn = void (*)(PathArgs, unsigned long long*, int, int, const int2*);

template <bool TAB>
DescFn pick_desc_rows(int K) {
    switch (K) {
        case 4: return k_descriptor_rows<4, 1, TAB>;
        case 8: return k_descriptor_rows<4, 2, TAB>;
        case 12: return k_descriptor_rows<6, 2, TAB>;
        case 16: return k_descriptor_rows<4, 4, TAB>;
        default: return nullptr;
    }
}
template <int RAD>
AdjFn pick_adj_rows(int K) {
    switch (K) {
        case 4: return k_adjoint_rows<4, 1, RAD>;
        case 8: return k_adjoint_rows<8, 1, RAD>;
        case 12: return k_adjoint_rows<6, 2, RAD>;
        case 16: return k_adjoint_rows<8, 2, RAD>;
        default: return nullptr;
    }
}

}  // namespace

bool row_kernels(const tmd_model* m) { return m->M == 3 && pick_adj_rows<kRadDirect>(m->K) != nullptr; }

tmd_status launch_descriptor_rows(tmd_context* ctx, const tmd_model* m, const PathArgs& a) {
    auto fn = m->tab ? pick_desc_rows<true>(m->K) : pick_desc_rows<false>(m->K);
    const int64_t nblocks = (a.n + kBlock / 16 - 1) / (kBlock / 16);
    fn<<<xcd_grid(nblocks), kBlock, 0, ctx->stream>>>(a, nblocks);
    TMD_HIP(ctx, hipGetLastError());
    return TMD_OK;
}

int adjoint_rows_atoms(int64_t n, int64_t max_partials) {
    int atoms = kRowAtoms;
    while (atoms < kBlock && (n + atoms - 1) / atoms > max_partials) atoms *= 2;
    return atoms;
}

tmd_status launch_adjoint_rows(tmd_context* ctx, const tmd_model* m, const PathArgs& a, const int2* segs, int atoms,
                               unsigned long long* F) {
    const int rad = m->tab ? kRadTab : (m->rec ? kRadRec : kRadDirect);
    auto fn = rad == kRadTab ? pick_adj_rows<kRadTab>(m->K)
                             : rad == kRadRec ? pick_adj_rows<kRadRec>(m->K) : pick_adj_rows<kRadDirect>(m->K);
    const int W = (int)std::min<int64_t>(a.n, row_window(m->K));
    fn<<<(unsigned)((a.n + atoms - 1) / atoms), kRowThreads, 24 * (size_t)W, ctx->stream>>>(a, F, atoms, W, segs);
    TMD_HIP(ctx, hipGetLastError());
    return TMD_OK;
}

}  // namespace tmd
