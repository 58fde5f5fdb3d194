// Per-element MLP: atomic energies E_a = NNP_s(G_a) and their input gradient
// dE_a/dG_a by back-propagation (Sec. III.A; the paper fuses forward and
// backward of the dense network into one kernel and keeps both W and W^T,
// which is also done here: the backward GEMMs read stored transposes so that
// every operand row is contiguous).
//
// All GEMMs run on MFMA in the transposed orientation Z^T = W A^T: hidden
// units are the MFMA rows and 16 atoms form the MFMA columns.  With that
// orientation the accumulator layout of one layer (lane = (row group, atom),
// four consecutive rows per lane) is exactly the B-operand layout the next
// layer needs, up to a fixed permutation of the reduction index that is
// applied identically to the weights, so where a wave holds whole layers the activations never leave
// its registers.
//   BF16: v_mfma_f32_16x16x32_bf16, operands rounded to BF16 (nearest-even),
//         FP32 accumulation.  One K-step covers 32 hidden units: for lane
//         group g the 8 operand slots hold units {4g..4g+3, 16+4g..16+4g+3}.
//   FP32: v_mfma_f32_16x16x4_f32.  One K-step covers 4 units, lane group g
//         holding unit 16*blk + 4g + r in step (blk, r).
// Three forms: k_mlp (a layer's rows shared by four waves, weights from L2),
// k_mlp_staged (whole layers per wave, weights through LDS, many atoms) and
// k_mlp_resident (the same, weights kept in LDS, large BF16 systems).  All
// add a unit's products in the same order, so they agree bit for bit.
#include "tmd_internal.h"

#include <type_traits>

namespace tmd {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;


struct MlpArgs {
    int S, F, Fpad;
    int64_t sp_off[kMaxSpecies + 1];
    int64_t tile_off[kMaxSpecies + 1];
    const int32_t* sp_idx;
    const float* G;      // FP32 descriptors (FP32 kernels)
    const uint16_t* Gb;  // BF16 descriptors, the bits of (__bf16)G (BF16 kernels)
    float* Ei;
    float* dG;
    const float* w32;
    const __hip_bfloat16* wbf;
    int64_t wstride;
    int64_t w_off[TMD_MAX_HIDDEN];
    int64_t wt_off[TMD_MAX_HIDDEN];
    const float* bias;  // [S][L][H]
    const float* wout;  // [S][H]
    const float* bout;  // [S]
};

template <int ACT>
__device__ __forceinline__ float act_f(float z) {
    constexpr int act = ACT;
    if constexpr (act == TMD_ACT_SQUAREPLUS) return 0.5f * (z + __builtin_amdgcn_sqrtf(z * z + 4.0f));
    // tanh(z) = 1 - 2/(exp(2z)+1) with the hardware reciprocal (1 ulp); saturates
    // cleanly to +-1 (exp2 overflows to inf, whose reciprocal is 0)
    const float e = __builtin_amdgcn_exp2f(2.8853900817779268f * z);
    return fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
}
template <int ACT>
__device__ __forceinline__ float act_df(float z, float a) {
    constexpr int act = ACT;
    if constexpr (act == TMD_ACT_SQUAREPLUS) return 0.5f * (1.0f + z * __builtin_amdgcn_rsqf(z * z + 4.0f));
    return 1.0f - a * a;
}

__device__ __forceinline__ bf16x8 cat8(bf16x4 lo, bf16x4 hi) {
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ bf16x4 to_bf4(f32x4 v) {
    bf16x4 r;
    r[0] = (__bf16)v[0];
    r[1] = (__bf16)v[1];
    r[2] = (__bf16)v[2];
    r[3] = (__bf16)v[3];
    return r;
}

// n (a multiple of 8) weights to LDS by the whole workgroup; callers synchronise around it.
__device__ __forceinline__ void copy_weights(const __hip_bfloat16* W, int n, __hip_bfloat16* lds) {
    for (int c = threadIdx.x; c < n / 8; c += blockDim.x)
        reinterpret_cast<uint4*>(lds)[c] = reinterpret_cast<const uint4*>(W)[c];
}

// B operand of the first layer: four consecutive features of one atom's
// descriptor row, zero past the row's end.
__device__ __forceinline__ f32x4 load_g4(const float* G, int64_t atom, int F, int g0, bool valid) {
    f32x4 v = {0, 0, 0, 0};
    if (!valid || g0 >= F) return v;
    const float* row = G + atom * F;
    if ((F & 3) == 0) return *reinterpret_cast<const f32x4*>(row + g0);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (g0 + r < F) v[r] = row[g0 + r];
    return v;
}

// The same four features stored as BF16 (rounded by the producer exactly as
// to_bf4 rounds: nearest-even), so the operand bits are those of
// to_bf4(load_g4(...)) on the FP32 row.
__device__ __forceinline__ bf16x4 load_gb4(const uint16_t* Gb, int64_t atom, int F, int g0, bool valid) {
    if (!valid || g0 >= F) return bf16x4{0, 0, 0, 0};
    const uint16_t* row = Gb + atom * F;
    if ((F & 3) == 0) return __builtin_bit_cast(bf16x4, *reinterpret_cast<const uint2*>(row + g0));
    bf16x4 v = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (g0 + r < F) v[r] = __builtin_bit_cast(__bf16, row[g0 + r]);
    return v;
}

__device__ __forceinline__ void store_dg4(float* dG, int64_t atom, int F, int f0, bool valid, f32x4 v) {
    if (!valid || f0 >= F) return;
    float* row = dG + atom * F;
    if ((F & 3) == 0) {
        *reinterpret_cast<f32x4*>(row + f0) = v;
        return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (f0 + r < F) row[f0 + r] = v[r];
}

// The operands of a matrix product Z = W X over a run of reduction blocks (16
// values for FP32, 32 for BF16): W's rows straight from memory, X from LDS
// (activations, [atom][H + pad]) or from the descriptor rows.
template <bool BF16>
struct Op;
template <>
struct Op<false> {
    using A = f32x4;
    static constexpr int kBlock = 16;  // reduction values per block
    static constexpr int kPad = 4;     // floats of row padding of the activations
    using X = float;
    // W's rows 16 rb .., block k of nk
    static __device__ __forceinline__ A load_w(const float* w, int nk, int rb, int k, int lane) {
        return *reinterpret_cast<const f32x4*>(w + ((rb * nk + k) * 64 + lane) * 4);
    }
    static __device__ __forceinline__ A load_x(const float* row, int k, int grp) {
        return *reinterpret_cast<const f32x4*>(row + 16 * k + 4 * grp);
    }
    static __device__ __forceinline__ A load_g(const MlpArgs& a, int64_t atom, int k, int grp, bool valid) {
        return load_g4(a.G, atom, a.F, 16 * k + 4 * grp, valid);
    }
    static __device__ __forceinline__ void store_x(float* row, int o0, f32x4 v) {
        *reinterpret_cast<f32x4*>(row + o0) = v;
    }
    static __device__ __forceinline__ f32x4 mul(A w, A x, f32x4 c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f32_16x16x4f32(w[r], x[r], c, 0, 0, 0);
        return c;
    }
};
template <>
struct Op<true> {
    using A = bf16x8;
    static constexpr int kBlock = 32;
    static constexpr int kPad = 4;
    using X = __bf16;
    static __device__ __forceinline__ A load_w(const __hip_bfloat16* w, int nk, int rb, int k, int lane) {
        return *reinterpret_cast<const bf16x8*>(w + ((rb * nk + k) * 64 + lane) * 8);
    }
    static __device__ __forceinline__ A load_x(const __bf16* row, int k, int grp) {
        const __bf16* p = row + 32 * k + 4 * grp;
        return cat8(*reinterpret_cast<const bf16x4*>(p), *reinterpret_cast<const bf16x4*>(p + 16));
    }
    static __device__ __forceinline__ A load_g(const MlpArgs& a, int64_t atom, int k, int grp, bool valid) {
        const int g0 = 32 * k + 4 * grp;
        return cat8(load_gb4(a.Gb, atom, a.F, g0, valid), load_gb4(a.Gb, atom, a.F, g0 + 16, valid));
    }
    static __device__ __forceinline__ void store_x(__bf16* row, int o0, f32x4 v) {
        *reinterpret_cast<bf16x4*>(row + o0) = to_bf4(v);
    }
    static __device__ __forceinline__ f32x4 mul(A w, A x, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
    }
};

// One workgroup of four waves takes 16 CB atoms of one species.  Wave w owns a
// quarter of every layer's output rows (in both directions, so s' stays in its
// registers) and a quarter of dE/dG's; the activations pass between the waves
// through LDS, one barrier per layer.  A wave's weight rows are nobody else's,
// so they come straight from memory (L2), a whole layer ahead of the barrier it
// needs.
//
// Bound by the chain of layers where atoms are few (32 atoms of 32-64-64: 8 us,
// 16 with one wave per 16 atoms and weights staged in LDS), by the weights' way
// from L2 where layers are many: 23,040 atoms of 512-128-128-128-128 in FP32
// 134 us (staged 315; the products 69), 85,750 of 128-128-128-128 in BF16 61
// (staged 119).  With the weights row-major instead of in operand order those
// are 193 and 157 us.
template <bool BF16, int H, int L, int CB, int ACT>
__global__ void __launch_bounds__(256) k_mlp(MlpArgs a) {
    using O = Op<BF16>;
    using A = typename O::A;
    using X = typename O::X;
    constexpr int NB = H / 16, NW = NB >= 4 ? NB / 4 : 1;  // row blocks, and of one wave
    constexpr int KB = H / O::kBlock;                      // reduction blocks of a hidden layer
    constexpr int XS = H + O::kPad, ES = H + 4, kTile = 16 * CB;
    constexpr int PF = 4;  // reduction blocks of the descriptor in flight
    __shared__ __attribute__((aligned(16))) X xs[2][kTile * XS];
    __shared__ __attribute__((aligned(16))) float last[kTile * ES];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int64_t tile = blockIdx.x;
    int s = 0;
    for (int q = 0; q < a.S; ++q)
        if (tile >= a.tile_off[q] && tile < a.tile_off[q + 1]) s = q;
    const int64_t first = a.sp_off[s] + (tile - a.tile_off[s]) * kTile;
    const int64_t end = a.sp_off[s + 1];
    int64_t atom[CB];
    bool valid[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int64_t r = first + cb * 16 + col;
        valid[cb] = r < end;
        atom[cb] = valid[cb] ? (int64_t)a.sp_idx[r] : 0;
    }
    const auto* wsp = [&] {
        if constexpr (BF16) return a.wbf + s * a.wstride;
        else return a.w32 + s * a.wstride;
    }();
    const float* bias = a.bias + (int64_t)s * L * H;
    const bool mine = wv * NW < NB;  // (H = 32: two waves own rows)
    const int ob0 = mine ? wv * NW : 0;

    f32x4 acc[NW][CB];
    f32x4 dact[L][NW][CB];
    A wr[NW][KB];  // this wave's rows of a hidden layer
    auto load_layer = [&](int64_t off) {
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int k = 0; k < KB; ++k) wr[j][k] = O::load_w(wsp + off, KB, ob0 + j, k, lane);
    };
    auto dense = [&](const X* x) {
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            A xv[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) xv[cb] = O::load_x(x + (16 * cb + col) * XS, k, grp);
#pragma unroll
            for (int j = 0; j < NW; ++j)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[j][cb] = O::mul(wr[j][k], xv[cb], acc[j][cb]);
        }
    };
    auto set_bias = [&](const float* bl) {
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            f32x4 init = {0, 0, 0, 0};
            if (bl) init = *reinterpret_cast<const f32x4*>(bl + 16 * (ob0 + j) + 4 * grp);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[j][cb] = init;
        }
    };
    auto activate = [&](int l) {
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float z = acc[j][cb][r];
                    const float y = act_f<ACT>(z);
                    dact[l][j][cb][r] = act_df<ACT>(z, y);
                    acc[j][cb][r] = y;
                }
    };
    auto give = [&](X* x) {
        if (!mine) return;
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                O::store_x(x + (16 * cb + col) * XS, 16 * (ob0 + j) + 4 * grp, acc[j][cb]);
    };

    // ---- layer 1: W_1 [H][Fpad] times G^T, PF blocks ahead
    set_bias(bias);
    {
        const auto* W = wsp + a.w_off[0];
        const int nk = a.Fpad / O::kBlock;
        A wb[PF][NW], gb[PF][CB];
        auto fetch = [&](int q, int k) {
            k = min(k, nk - 1);
#pragma unroll
            for (int j = 0; j < NW; ++j) wb[q][j] = O::load_w(W, nk, ob0 + j, k, lane);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) gb[q][cb] = O::load_g(a, atom[cb], k, grp, valid[cb]);
        };
#pragma unroll
        for (int q = 0; q < PF; ++q) fetch(q, q);
        for (int k0 = 0; k0 < nk; k0 += PF) {
#pragma unroll
            for (int q = 0; q < PF; ++q) {
                if (k0 + q < nk) {
#pragma unroll
                    for (int j = 0; j < NW; ++j)
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) acc[j][cb] = O::mul(wb[q][j], gb[q][cb], acc[j][cb]);
                }
                if (k0 + q + PF < nk) fetch(q, k0 + q + PF);
            }
        }
    }
    int buf = 0;
    // ---- hidden layers 2..L
#pragma unroll
    for (int l = 0; l < L; ++l) {
        if (l > 0) {
            set_bias(bias + l * H);
            dense(xs[buf]);
            buf ^= 1;
        }
        activate(l);
        if (l < L - 1) {
            give(xs[buf]);
            load_layer(a.w_off[l + 1]);
            __syncthreads();
        }
    }

    // ---- output layer: E = w_out . a_L + b_out; delta_L = w_out * act'(z_L)
    const float* wo = a.wout + (int64_t)s * H;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const f32x4 wv4 = *reinterpret_cast<const f32x4*>(wo + 16 * (ob0 + j) + 4 * grp);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            if (mine) *reinterpret_cast<f32x4*>(last + (16 * cb + col) * ES + 16 * (ob0 + j) + 4 * grp) = acc[j][cb];
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][cb][r] = wv4[r] * dact[L - 1][j][cb][r];
        }
    }
    give(xs[buf]);
    if (L > 1) load_layer(a.wt_off[L - 1]);
    __syncthreads();
    const float bo = a.bout[s];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        if ((cb & 3) != wv) continue;  // one wave per 16 atoms
        float e = 0.0f;
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) {
            const f32x4 w4 = *reinterpret_cast<const f32x4*>(wo + 16 * ob + 4 * grp);
            const f32x4 y = *reinterpret_cast<const f32x4*>(last + (16 * cb + col) * ES + 16 * ob + 4 * grp);
#pragma unroll
            for (int r = 0; r < 4; ++r) e = fmaf(w4[r], y[r], e);
        }
        e += __shfl_xor(e, 16);
        e += __shfl_xor(e, 32);
        if (grp == 0 && valid[cb]) a.Ei[atom[cb]] = e + bo;
    }

    // ---- backward through hidden layers: delta_{l-1} = (W_l^T delta_l) * act'(z_{l-1})
#pragma unroll
    for (int l = L - 1; l >= 1; --l) {
        set_bias(nullptr);
        dense(xs[buf]);
        buf ^= 1;
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[j][cb][r] *= dact[l - 1][j][cb][r];
        give(xs[buf]);
        if (l > 1) load_layer(a.wt_off[l - 1]);
        __syncthreads();
    }

    // ---- dE/dG^T = W_1^T delta_1: Fpad output rows, a block of 16 at a time
    // per wave, the next block's weights in flight
    {
        const auto* W = wsp + a.wt_off[0];
        const int nf = a.Fpad / 16;
        A xv[KB][CB];
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) xv[k][cb] = O::load_x(xs[buf] + (16 * cb + col) * XS, k, grp);
        A wb[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) wb[k] = O::load_w(W, KB, min(wv, nf - 1), k, lane);
        for (int fb = wv; fb < nf; fb += 4) {
            A wn[KB];
#pragma unroll
            for (int k = 0; k < KB; ++k) wn[k] = O::load_w(W, KB, min(fb + 4, nf - 1), k, lane);
            f32x4 out[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) out[cb] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < KB; ++k)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) out[cb] = O::mul(wb[k], xv[k][cb], out[cb]);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) store_dg4(a.dG, atom[cb], a.F, 16 * fb + 4 * grp, valid[cb], out[cb]);
#pragma unroll
            for (int k = 0; k < KB; ++k) wb[k] = wn[k];
        }
    }
}

// Staged form: every wave takes 16 atoms (128 units, eight waves) or 32 (fewer
// units, four waves), activations never leave a wave's registers, and each
// layer's weights pass once per 128 atoms through LDS, panels of four reduction
// blocks at a time.  Bound by the products and, in FP32, their operands' way
// from LDS: 1,000,188 atoms of 32-64-64: 239 us in FP32 (k_mlp, weights from L2
// per 32 atoms: 334), 82 in BF16 (207); of 32-32 73 (192) and 51 (173); 54,000
// of 96-128-128 in BF16 21 (32).  (128 registers where one or two layers allow
// it, so that four waves share a SIMD: with 136 the FP32 form of 128-128 took
// 1,094 us for 877,952 atoms, with 128 892.)
constexpr int staged_waves(int H) { return H == 128 ? 8 : 4; }
constexpr int staged_cols(int H) { return H == 128 ? 1 : 2; }  // 16-atom columns of a wave
// Waves on a SIMD that the registers are to allow (512 / waves each).
constexpr int staged_occupancy(int H, int L, int act) {
    if (H == 32) return 4;
    if (H == 64) return act == TMD_ACT_TANH ? (L <= 2 ? 4 : L == 3 ? 3 : 2) : (L == 1 ? 4 : 2);
    return L == 1 || (L == 2 && act == TMD_ACT_TANH) ? 4 : 2;
}
template <bool BF16, int H, int L, int ACT>
__global__ void __launch_bounds__(64 * staged_waves(H), staged_occupancy(H, L, ACT)) k_mlp_staged(MlpArgs a) {
    using O = Op<BF16>;
    using A = typename O::A;
    using T = std::conditional_t<BF16, __hip_bfloat16, float>;
    constexpr int CB = staged_cols(H), kThreads = 64 * staged_waves(H), kAtoms = kThreads / 4 * CB;
    constexpr int NB = H / 16, KB = H / O::kBlock;
    constexpr int PB = 4;              // reduction blocks of 1 KB per row block in a panel
    constexpr int RB = NB * PB / KB;   // row blocks of W_1^T in a panel
    // BF16: a panel in operand order.  FP32: rows padded by 28 floats (pads of
    // 20 to 36 are alike, 4 or 44 and more a quarter slower).
    constexpr int PS = 16 * PB + 28, FS = H + 28;
    constexpr int kLds = BF16 ? NB * PB * 512 : (H * PS > 16 * RB * FS ? H * PS : 16 * RB * FS);
    __shared__ __attribute__((aligned(16))) T lds[kLds];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int64_t tile = blockIdx.x;
    int s = 0;
    for (int q = 0; q < a.S; ++q)
        if (tile >= a.tile_off[q] && tile < a.tile_off[q + 1]) s = q;
    const int64_t first = a.sp_off[s] + (tile - a.tile_off[s]) * kAtoms + wv * 16 * CB + col;
    bool valid[CB];
    int64_t atom[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        valid[cb] = first + 16 * cb < a.sp_off[s + 1];
        atom[cb] = valid[cb] ? (int64_t)a.sp_idx[first + 16 * cb] : 0;
    }
    const T* wsp;
    if constexpr (BF16) wsp = a.wbf + s * a.wstride;
    else wsp = a.w32 + s * a.wstride;
    const float* bias = a.bias + (int64_t)s * L * H;
    f32x4 acc[NB][CB], x[NB][CB], dact[L][NB][CB];
    auto set_bias = [&](const float* bl) {
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) {
            f32x4 init = {0, 0, 0, 0};
            if (bl) init = *reinterpret_cast<const f32x4*>(bl + 16 * ob + 4 * grp);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[ob][cb] = init;
        }
    };
    auto activate = [&](int l) {
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float z = acc[ob][cb][q];
                    const float y = act_f<ACT>(z);
                    dact[l][ob][cb][q] = act_df<ACT>(z, y);
                    acc[ob][cb][q] = y;
                }
    };
    // blocks c .. c + n - 1 of every row block of a matrix with nk blocks a row
    auto panel = [&](const T* W, int nk, int c, int n) {
        __syncthreads();
        for (int q = threadIdx.x; q < NB * n * 64; q += kThreads) {
            const int ob = q / (n * 64), e = q - ob * (n * 64);
            const uint4 v = reinterpret_cast<const uint4*>(W)[(ob * nk + c) * 64 + e];
            if constexpr (BF16) reinterpret_cast<uint4*>(lds)[q] = v;
            else *reinterpret_cast<uint4*>(lds + (16 * ob + (e & 15)) * PS + 4 * (e >> 4)) = v;
        }
        __syncthreads();
    };
    auto from_panel = [&](int n, int ob, int k) {
        if constexpr (BF16) return O::load_w(lds, n, ob, k, lane);
        else return *reinterpret_cast<const f32x4*>(lds + (16 * ob + col) * PS + 16 * k + 4 * grp);
    };
    auto operand = [&](const f32x4 (&v)[NB][CB], int k, int cb) {
        if constexpr (BF16) return cat8(to_bf4(v[2 * k][cb]), to_bf4(v[2 * k + 1][cb]));
        else return v[k][cb];
    };
    auto dense = [&](const T* W, const float* bl) {
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) x[ob][cb] = acc[ob][cb];
        set_bias(bl);
        constexpr int n = PB < KB ? PB : KB;
#pragma unroll
        for (int c = 0; c < KB; c += n) {
            panel(W, KB, c, n);
#pragma unroll
            for (int k = 0; k < n; ++k) {
                A xv[CB];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) xv[cb] = operand(x, c + k, cb);
#pragma unroll
                for (int ob = 0; ob < NB; ++ob) {
                    const A w = from_panel(n, ob, k);
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) acc[ob][cb] = O::mul(w, xv[cb], acc[ob][cb]);
                }
            }
        }
    };
    // layer 1
    set_bias(bias);
    const int nk = a.Fpad / O::kBlock;
    for (int c = 0; c < nk; c += PB) {
        const int n = min(PB, nk - c);
        panel(wsp + a.w_off[0], nk, c, n);
        for (int k = 0; k < n; ++k) {
            A xv[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) xv[cb] = O::load_g(a, atom[cb], c + k, grp, valid[cb]);
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) {
                const A w = from_panel(n, ob, k);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[ob][cb] = O::mul(w, xv[cb], acc[ob][cb]);
            }
        }
    }
    activate(0);
#pragma unroll
    for (int l = 1; l < L; ++l) {
        dense(wsp + a.w_off[l], bias + l * H);
        activate(l);
    }
    const float* wo = a.wout + (int64_t)s * H;
    float e[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) e[cb] = 0.0f;
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
        const f32x4 w4 = *reinterpret_cast<const f32x4*>(wo + 16 * ob + 4 * grp);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                e[cb] = fmaf(w4[q], acc[ob][cb][q], e[cb]);
                acc[ob][cb][q] = w4[q] * dact[L - 1][ob][cb][q];
            }
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        e[cb] += __shfl_xor(e[cb], 16);
        e[cb] += __shfl_xor(e[cb], 32);
        if (grp == 0 && valid[cb]) a.Ei[atom[cb]] = e[cb] + a.bout[s];
    }
#pragma unroll
    for (int l = L - 1; l >= 1; --l) {
        dense(wsp + a.wt_off[l], nullptr);
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[ob][cb][q] *= dact[l - 1][ob][cb][q];
    }
    A xv[KB][CB];
#pragma unroll
    for (int k = 0; k < KB; ++k)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) xv[k][cb] = operand(acc, k, cb);
    for (int f0 = 0; f0 < a.Fpad / 16; f0 += RB) {
        const int nf = min(RB, a.Fpad / 16 - f0);
        __syncthreads();
        for (int q = threadIdx.x; q < nf * KB * 64; q += kThreads) {
            const uint4 v = reinterpret_cast<const uint4*>(wsp + a.wt_off[0])[f0 * KB * 64 + q];
            if constexpr (BF16) reinterpret_cast<uint4*>(lds)[q] = v;
            else *reinterpret_cast<uint4*>(lds + (q / (KB * 64) * 16 + (q & 15)) * FS + 4 * (q % (KB * 64) >> 4)) = v;
        }
        __syncthreads();
        for (int fb = 0; fb < nf; ++fb) {
            f32x4 out[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) out[cb] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                A w;
                if constexpr (BF16) w = O::load_w(lds, KB, fb, k, lane);
                else w = *reinterpret_cast<const f32x4*>(lds + (16 * fb + col) * FS + 16 * k + 4 * grp);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) out[cb] = O::mul(w, xv[k][cb], out[cb]);
            }
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) store_dg4(a.dG, atom[cb], a.F, 16 * (f0 + fb) + 4 * grp, valid[cb], out[cb]);
        }
    }
}

// Resident-weight form (BF16, networks whose weights fit in LDS): one
// workgroup of 16 waves per CU keeps every matrix of one species in LDS
// (W_1, the hidden W_l, their transposes and W_1^T) and its waves
// take 16-atom tiles independently, with no barrier between layers.  The
// weights are staged once per species and workgroup instead of once per
// 128-atom tile (at 1 M atoms that is ~30 MB of L2 traffic instead of ~0.9 GB).
template <int H, int L, int ACT>
__global__ void __launch_bounds__(1024) k_mlp_resident(MlpArgs a) {
    using T = __hip_bfloat16;
    constexpr int NB = H / 16, KB = H / 32;
    extern __shared__ __attribute__((aligned(16))) T sw[];
    const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4, wv = threadIdx.x >> 6;
    const int nw = blockDim.x >> 6;
    // in operand order, as in memory: a read is 1 KB in a run, free of bank conflicts
    T* W1 = sw;                        // [H][Fpad]
    T* Wh = W1 + H * a.Fpad;           // L-1 x [H][H]
    T* Wt = Wh + (L - 1) * H * H;      // L-1 x [H][H], transposed hidden layers
    T* W1t = Wt + (L - 1) * H * H;     // [Fpad][H]
    for (int s = 0; s < a.S; ++s) {
        const int64_t first_atom = a.sp_off[s], end = a.sp_off[s + 1];
        const int64_t ntiles = (end - first_atom + 15) / 16;
        if (ntiles == 0) continue;  // uniform over the workgroup
        const T* wsp = a.wbf + s * a.wstride;
        __syncthreads();  // the previous species' tiles are done with the LDS copy
        copy_weights(wsp + a.w_off[0], H * a.Fpad, W1);
        for (int l = 1; l < L; ++l) {
            copy_weights(wsp + a.w_off[l], H * H, Wh + (l - 1) * H * H);
            copy_weights(wsp + a.wt_off[l], H * H, Wt + (l - 1) * H * H);
        }
        copy_weights(wsp + a.wt_off[0], H * a.Fpad, W1t);
        __syncthreads();
        const float* bias = a.bias + (int64_t)s * L * H;
        const float* wo = a.wout + (int64_t)s * H;
        const float bo = a.bout[s];
        for (int64_t tile = (int64_t)blockIdx.x * nw + wv; tile < ntiles; tile += (int64_t)gridDim.x * nw) {
            // keep the weight reads inside the tile loop (hoisting them out of
            // it would pin every weight fragment in registers)
            __asm__ volatile("" ::: "memory");
            const int64_t r = first_atom + tile * 16 + col;
            const bool valid = r < end;
            const int64_t atom = valid ? (int64_t)a.sp_idx[r] : 0;
            f32x4 acc[NB], x[NB], dact[L][NB];
            auto set_bias = [&](const float* bl) {
#pragma unroll
                for (int ob = 0; ob < NB; ++ob) {
                    f32x4 init = {0, 0, 0, 0};
                    if (bl) init = *reinterpret_cast<const f32x4*>(bl + 16 * ob + 4 * grp);
                    acc[ob] = init;
                }
            };
            auto activate = [&](int l) {
#pragma unroll
                for (int ob = 0; ob < NB; ++ob)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float z = acc[ob][q];
                        const float y = act_f<ACT>(z);
                        dact[l][ob][q] = act_df<ACT>(z, y);
                        acc[ob][q] = y;
                    }
            };
            // A operand rows of a resident matrix times the B operand held in x
            auto dense = [&](const T* Wm) {
#pragma unroll
                for (int k0 = 0; k0 < H; k0 += 32) {
                    __asm__ volatile("" ::: "memory");  // one block's weights in flight at a time
                    const int blk = k0 / 16;
                    const bf16x8 bop = cat8(to_bf4(x[blk]), to_bf4(x[blk + 1]));
#pragma unroll
                    for (int ob = 0; ob < NB; ++ob) {
                        const bf16x8 av = Op<true>::load_w(Wm, KB, ob, k0 / 32, lane);
                        acc[ob] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bop, acc[ob], 0, 0, 0);
                    }
                }
            };
            // layer 1
            set_bias(bias);
            for (int k0 = 0; k0 < a.Fpad; k0 += 32) {
                const int g0 = k0 + 4 * grp;
                const bf16x8 bop = cat8(load_gb4(a.Gb, atom, a.F, g0, valid), load_gb4(a.Gb, atom, a.F, g0 + 16, valid));
#pragma unroll
                for (int ob = 0; ob < NB; ++ob) {
                    const bf16x8 av = Op<true>::load_w(W1, a.Fpad / 32, ob, k0 / 32, lane);
                    acc[ob] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bop, acc[ob], 0, 0, 0);
                }
            }
            activate(0);
#pragma unroll
            for (int l = 1; l < L; ++l) {
                __asm__ volatile("" ::: "memory");  // one layer's weights in flight at a time
#pragma unroll
                for (int ob = 0; ob < NB; ++ob) x[ob] = acc[ob];
                set_bias(bias + l * H);
                dense(Wh + (l - 1) * H * H);
                activate(l);
            }
            // output layer and its adjoint
            float e = 0.0f;
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) {
                const f32x4 wvv = *reinterpret_cast<const f32x4*>(wo + 16 * ob + 4 * grp);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    e = fmaf(wvv[q], acc[ob][q], e);
                    acc[ob][q] = wvv[q] * dact[L - 1][ob][q];
                }
            }
            e += __shfl_xor(e, 16);
            e += __shfl_xor(e, 32);
            if (grp == 0 && valid) a.Ei[atom] = e + bo;
            // backward through the hidden layers
#pragma unroll
            for (int l = L - 1; l >= 1; --l) {
                __asm__ volatile("" ::: "memory");
#pragma unroll
                for (int ob = 0; ob < NB; ++ob) x[ob] = acc[ob];
                set_bias(nullptr);
                dense(Wt + (l - 1) * H * H);
#pragma unroll
                for (int ob = 0; ob < NB; ++ob)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[ob][q] *= dact[l - 1][ob][q];
            }
            // dE/dG^T = W_1^T delta_1
            __asm__ volatile("" ::: "memory");
            bf16x8 bop[NB / 2];
#pragma unroll
            for (int s2 = 0; s2 < NB / 2; ++s2) bop[s2] = cat8(to_bf4(acc[2 * s2]), to_bf4(acc[2 * s2 + 1]));
            for (int fb = 0; fb < a.Fpad / 16; ++fb) {
                f32x4 out = {0, 0, 0, 0};
#pragma unroll
                for (int s2 = 0; s2 < NB / 2; ++s2) {
                    const bf16x8 av = Op<true>::load_w(W1t, KB, fb, s2, lane);
                    out = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bop[s2], out, 0, 0, 0);
                }
                store_dg4(a.dG, atom, a.F, 16 * fb + 4 * grp, valid, out);
            }
        }
    }
}

using ResidentFn = void (*)(MlpArgs);
template <int ACT>
ResidentFn pick_resident(int H, int L) {
    if (H == 128 && L == 1) return k_mlp_resident<128, 1, ACT>;
    if (H == 128 && L == 2) return k_mlp_resident<128, 2, ACT>;
    if (H == 64 && L == 2) return k_mlp_resident<64, 2, ACT>;
    if (H == 64 && L == 3) return k_mlp_resident<64, 3, ACT>;
    return nullptr;
}
int resident_lds_bytes(int H, int L, int Fpad) { return 2 * (2 * H * Fpad + 2 * (L - 1) * H * H); }
constexpr int kMaxResidentLds = 150 * 1024;

using MlpFn = void (*)(MlpArgs);

template <bool BF16, int H, int ACT, int CB>
MlpFn pick_L(int L) {
    switch (L) {
        case 1: return k_mlp<BF16, H, 1, CB, ACT>;
        case 2: return k_mlp<BF16, H, 2, CB, ACT>;
        case 3: return k_mlp<BF16, H, 3, CB, ACT>;
        default: return k_mlp<BF16, H, 4, CB, ACT>;
    }
}

template <bool BF16, int ACT, int CB>
MlpFn pick_H(int H, int L) {
    switch (H) {
        case 32: return pick_L<BF16, 32, ACT, CB>(L);
        case 64: return pick_L<BF16, 64, ACT, CB>(L);
        default: return pick_L<BF16, 128, ACT, CB>(L);
    }
}

template <bool BF16, int CB>
MlpFn pick_act(int act, int H, int L) {
    return act == TMD_ACT_SQUAREPLUS ? pick_H<BF16, TMD_ACT_SQUAREPLUS, CB>(H, L) : pick_H<BF16, TMD_ACT_TANH, CB>(H, L);
}

template <bool BF16, int H, int ACT>
MlpFn pick_staged_L(int L) {
    switch (L) {
        case 1: return k_mlp_staged<BF16, H, 1, ACT>;
        case 2: return k_mlp_staged<BF16, H, 2, ACT>;
        case 3: return k_mlp_staged<BF16, H, 3, ACT>;
        default: {  // (k_mlp at any size: take_staged's table)
            constexpr bool sp = ACT == TMD_ACT_SQUAREPLUS;
            if constexpr ((H == 128 && (!BF16 || sp)) || (H == 64 && !BF16 && sp)) return nullptr;
            else return k_mlp_staged<BF16, H, 4, ACT>;
        }
    }
}
template <bool BF16, int ACT>
MlpFn pick_staged_H(int H, int L) {
    switch (H) {
        case 32: return pick_staged_L<BF16, 32, ACT>(L);
        case 64: return pick_staged_L<BF16, 64, ACT>(L);
        default: return pick_staged_L<BF16, 128, ACT>(L);
    }
}
template <bool BF16>
MlpFn pick_staged(int act, int H, int L) {
    return act == TMD_ACT_SQUAREPLUS ? pick_staged_H<BF16, TMD_ACT_SQUAREPLUS>(H, L)
                                     : pick_staged_H<BF16, TMD_ACT_TANH>(H, L);
}

// Whether N atoms take the staged form.  k_mlp reads a layer's weights from L2
// for every 16 or 32 atoms, the staged form for every 128 but with a quarter of
// the workgroups, and eight times their work each: it is taken beyond so many
// atoms per CU that its first rounds are filled, later where k_mlp hides the
// weights behind more products (FP32, three and four layers).  Measured at 32,
// 96 and 512 features, 864 to 1,000,188 atoms; us, staged against k_mlp, on
// both sides of the line (256 CUs), 96 features unless noted:
//   FP32  32 wide       16,384 14.8 / 12.0   24,624 15.4 / 16.3   1,000,188 201 / 348 (one layer)
//   FP32  64, 1         32,000 21.2 / 20.6   48,668 27.7 / 27.2   1,000,188 280 / 404
//         64, 2         32,000 27.5 / 25.4   48,668 36.3 / 36.4   1,000,188 406 / 535
//         64, 3         70,304 61.2 / 56.8  256,000 156 / 177
//         64, 4        108,000 108 / 98     442,368 352 / 360
//   FP32 128, 1         16,384 26.0 / 17.5   24,624 26.3 / 26.9   1,000,188 480 / 660
//        128, 2         48,668 73.1 / 70.0  108,000 140 / 149     1,000,188 1,029 / 1,287
//        128, 3, 4   1,000,188 1,897 / 1,736 and 2,538 / 2,407
//   BF16  32 wide       16,384 11.0 / 10.3   24,624 12.5 / 13.0   1,000,188 152 / 263 (one layer)
//   BF16  64, 1         16,384 12.5 / 10.4   24,624 12.8 / 13.4   1,000,188 164 / 284
//         64, 3, 4      32,000 18.6 / 17.3   48,668 20.0 / 23.9 (three)
//   BF16 128, 1, 2      16,384 17.3 / 13.8   24,624 18.7 / 20.4 (two)
//        128, 3         48,668 36.7 / 31.8  442,368 221 / 230
//        128, 4         16,384 25.2 / 18.7   24,624 26.4 / 28.4   1,000,188 618 / 747
// With 128 units and few features (the first layer is cheap, the others
// dominate) a single round of staged workgroups, 96 to 128 atoms per CU, beats
// the second round of k_mlp's: 32,000 atoms of 32-128-128-128 in FP32 58.5 / 66.9.
// Squareplus keeps more registers (its derivative is not formed from its value):
// with four layers the staged form spills and is left out but for few features.
// Few features (up to 64) make k_mlp's first layer, which reads them once per
// wave, no shorter: 32,000 atoms of 18-64-64-64 in BF16 14.9 / 19.3.
bool take_staged(const tmd_model* m, bool bf16, int64_t N, int64_t cus) {
    constexpr int64_t never = INT64_MAX / 1024;
    static const int64_t from[2][2][3][4] = {  // [activation][BF16][units][layers]
        {{{64, 64, 64, 64}, {128, 128, 384, 768}, {96, 256, never, never}},
         {{64, 64, 64, 64}, {64, 64, 128, 128}, {64, 64, 1024, 96}}},
        {{{64, 64, 64, 64}, {128, 384, 768, never}, {96, 256, never, never}},
         {{64, 64, 64, 64}, {64, 64, 128, never}, {64, 64, 1024, never}}}};
    const int h = m->H == 32 ? 0 : m->H == 64 ? 1 : 2, L = m->L;
    const bool sp = m->act == TMD_ACT_SQUAREPLUS;
    int64_t t = from[sp][bf16][h][L - 1];
    if (m->Fpad <= 64) {
        if (h == 1 && (L == 1 || (bf16 && (L == 3 || (L == 4 && !sp && m->F % 4 != 0))))) t = 64;
        if (h == 1 && sp && !bf16 && (L == 2 || L == 3)) t = L == 2 ? 128 : 384;
        if (h == 1 && sp && bf16 && L == 4) t = 384;
        if (h == 2 && !bf16 && (L == 2 || L == 3) && N > 96 * cus && N <= 128 * cus) return true;
    }
    return N > t * cus;
}

// Whether BF16 networks with resident weights take that form (rfn fits in LDS):
// from one 16-atom tile per wave on.  Squareplus with three layers of 64 runs
// out of registers there (70,304 atoms of 96-64-64-64: 38 us, staged 31;
// 256,000: 78 and 71; 1,000,188: 234 and 255).
bool take_resident(const tmd_model* m, int64_t N, int64_t cus) {
    const bool slow = m->act == TMD_ACT_SQUAREPLUS && m->H == 64 && m->L == 3 && m->Fpad > 64;
    return N >= (slow ? 2048 : 256) * cus;
}

}  // namespace

SpeciesGroups species_groups(const tmd_nlist* nl) {
    SpeciesGroups g;
    g.S = nl->S;
    for (int s = 0; s <= nl->S; ++s) g.off[s] = nl->sp_off[s];
    g.idx = nl->sp_idx;
    return g;
}

tmd_status launch_mlp(tmd_context* ctx, const tmd_model* m, const SpeciesGroups& g, tmd_precision prec,
                      const float* G, const uint16_t* Gb, float* Ei, float* dG) {
    if ((prec == TMD_BF16_MLP) != (Gb != nullptr))
        return fail(ctx, TMD_ERR_INVALID_ARGUMENT, "BF16 MLP without BF16 descriptors, or the reverse");
    MlpArgs a{};
    a.S = m->S;
    a.F = m->F;
    a.Fpad = m->Fpad;
    // 16 atoms per workgroup, 32 beyond 96 per CU: 23,040 atoms of
    // 512-128-128-128-128 in FP32 took 134 with 16, 146 us with 32, 32,000 of
    // 32-64-64 19.1 and 18.1, 24,624 of 96-128-128 49 and 47.
    const int64_t N = g.off[m->S], cus = ctx->num_cus;
    const bool wide = N > 96 * cus;
    const bool bf16 = prec == TMD_BF16_MLP;
    const MlpFn staged = take_staged(m, bf16, N, cus)
                             ? (bf16 ? pick_staged<true>(m->act, m->H, m->L) : pick_staged<false>(m->act, m->H, m->L))
                             : nullptr;
    const MlpFn fn = staged ? staged
                     : bf16
                         ? (wide ? pick_act<true, 2>(m->act, m->H, m->L) : pick_act<true, 1>(m->act, m->H, m->L))
                         : (wide ? pick_act<false, 2>(m->act, m->H, m->L) : pick_act<false, 1>(m->act, m->H, m->L));
    const int kTileAtoms = staged ? 128 : wide ? 32 : 16;
    int64_t tiles = 0;
    for (int s = 0; s < m->S; ++s) {
        a.sp_off[s] = g.off[s];
        a.tile_off[s] = tiles;
        tiles += (g.off[s + 1] - g.off[s] + kTileAtoms - 1) / kTileAtoms;
    }
    a.sp_off[m->S] = g.off[m->S];
    a.tile_off[m->S] = tiles;
    a.sp_idx = g.idx;
    a.G = G;
    a.Gb = Gb;
    a.Ei = Ei;
    a.dG = dG;
    a.w32 = m->w32;
    a.wbf = m->wbf;
    a.wstride = m->w_species_stride;
    for (int l = 0; l < m->L; ++l) {
        a.w_off[l] = m->w_off[l];
        a.wt_off[l] = m->wt_off[l];
    }
    a.bias = m->bias;
    a.wout = m->wout;
    a.bout = m->bout;
    if (tiles == 0) return TMD_OK;
    const int rlds = resident_lds_bytes(m->H, m->L, m->Fpad);
    ResidentFn rfn = nullptr;
    if (prec == TMD_BF16_MLP && rlds <= kMaxResidentLds && take_resident(m, N, cus))
        rfn = m->act == TMD_ACT_SQUAREPLUS ? pick_resident<TMD_ACT_SQUAREPLUS>(m->H, m->L)
                                           : pick_resident<TMD_ACT_TANH>(m->H, m->L);
    if (rfn) {
        TMD_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(rfn),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, rlds));
        ProfScope ps_(ctx, "mlp");
        rfn<<<(unsigned)ctx->num_cus, 1024, rlds, ctx->stream>>>(a);
    } else {
        ProfScope ps_(ctx, "mlp");
        fn<<<(unsigned)tiles, staged ? 64 * staged_waves(m->H) : 256, 0, ctx->stream>>>(a);
    }
    TMD_HIP(ctx, hipGetLastError());
    return TMD_OK;
}

}  // namespace tmd
