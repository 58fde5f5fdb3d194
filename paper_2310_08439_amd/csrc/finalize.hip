// Output assembly: forces and atomic energies back to the caller's atom order,
// total energy and virial reduced in FP64 with Neumaier compensation in a fixed
// order (one block, fixed per-thread ranges, fixed tree), so the totals are
// reproducible run to run.
#include "tmd_internal.h"

#include <algorithm>

namespace tmd {
namespace {

struct Comp {
    double s, c;
};

__device__ __forceinline__ void comp_add(Comp& a, double x) {
    const double t = a.s + x;
    if (fabs(a.s) >= fabs(x)) a.c += (a.s - t) + x;
    else a.c += (x - t) + a.s;
    a.s = t;
}

__device__ __forceinline__ Comp comp_merge(Comp a, Comp b) {
    comp_add(a, b.s);
    a.c += b.c;
    return a;
}

// Atoms per summing workgroup: eight per thread, so that up to 2,048 atoms are
// summed by one workgroup without a second stage.
constexpr int64_t kPartAtoms = 2048;

// Compensated sum over the wave's lanes, in a fixed butterfly; every lane gets it.
__device__ __forceinline__ Comp wave_merge(Comp a) {
    const int lane = threadIdx.x & 63;
    for (int off = 32; off > 0; off >>= 1) {
        const Comp o{__shfl_xor(a.s, off), __shfl_xor(a.c, off)};
        a = (lane & off) ? comp_merge(o, a) : comp_merge(a, o);
    }
    return a;
}

// One launch for everything that follows the adjoint.  The first nb workgroups
// each sum a contiguous slice of Ei and of the virial block partials with
// coalesced, thread-strided reads; the last of them to finish merges the nb
// results into totals[0] = sum Ei, totals[1..6] = virial (xx, yy, zz, xy, xz,
// yz), also to host_totals (pinned host memory) when given.  The workgroups
// after them take the forces (fixed point, 32 fractional bits: F = q 2^-32,
// exact in FP64, then rounded to FP32) and atomic energies back to the caller's
// atom order.  As three launches and a copy of the totals these steps took
// 17 us of a small system's evaluation, most of it launch and drain.  The
// counter is zero at the start (k_refresh).
__global__ void __launch_bounds__(256) k_finalize(int64_t n, const int32_t* __restrict__ perm,
                                                  const float* __restrict__ Ei,
                                                  const unsigned long long* __restrict__ Fq,
                                                  float* __restrict__ atom_energy, float* __restrict__ forces, int nb,
                                                  int64_t nvir, const double* __restrict__ vir, double* part,
                                                  unsigned int* counter, double* __restrict__ totals,
                                                  double* __restrict__ host_totals) {
    if ((int)blockIdx.x >= nb) {
        const int64_t p = (int64_t)(blockIdx.x - nb) * blockDim.x + threadIdx.x;
        if (p >= n) return;
        const int64_t i = perm[p];
        constexpr double inv = 1.0 / kForceFixedScale;
        forces[3 * i + 0] = (float)((double)(long long)Fq[3 * p + 0] * inv);
        forces[3 * i + 1] = (float)((double)(long long)Fq[3 * p + 1] * inv);
        forces[3 * i + 2] = (float)((double)(long long)Fq[3 * p + 2] * inv);
        if (atom_energy) atom_energy[i] = Ei[p];
        return;
    }
    // The butterflies are the longest part (about 150 dependent FP64
    // instructions each): every wave sums its share of E, but the six virial
    // components are shared out, one or two to a wave.
    __shared__ Comp wave_e[4], res[7];
    __shared__ bool last;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t per = (n + nb - 1) / nb;
    const int64_t lo = blockIdx.x * per, hi = min<int64_t>(n, lo + per);
    Comp e{0.0, 0.0};
    // unrolled so that a chunk's loads are in flight together (the sums keep
    // their order: each thread adds its values in index order)
#pragma unroll 8
    for (int64_t p = lo + threadIdx.x; p < hi; p += 256) comp_add(e, (double)Ei[p]);
    const int64_t pv = (nvir + nb - 1) / nb;
    const int64_t vlo = blockIdx.x * pv, vhi = min<int64_t>(nvir, vlo + pv);
    for (int j = wv; j < 6; j += 4) {
        Comp w{0.0, 0.0};
#pragma unroll 4
        for (int64_t b = vlo + lane; b < vhi; b += 64)
            w = comp_merge(w, Comp{vir[b * kVirDoubles + 2 * j], vir[b * kVirDoubles + 2 * j + 1]});
        w = wave_merge(w);
        if (lane == 0) res[1 + j] = w;
    }
    e = wave_merge(e);
    if (lane == 0) wave_e[wv] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) e = comp_merge(e, wave_e[w]);
        res[0] = e;
    }
    __syncthreads();
    if (nb > 1) {
        // The slices' sums pass from one XCD's L2 to another's as device-scope
        // atomic stores and loads, which go through the caches; the wave that
        // stored waits for them before it counts.  (__threadfence instead, which
        // writes the whole L2 back, made this launch 45 us at 1,024,000 atoms;
        // now 27.)
        if (threadIdx.x < 7) {
            double* mine = part + (blockIdx.x * 7 + threadIdx.x) * 2;
            __hip_atomic_store(mine, res[threadIdx.x].s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(mine + 1, res[threadIdx.x].c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        if (threadIdx.x == 0) last = atomicInc(counter, nb - 1) == (unsigned)(nb - 1);
        __syncthreads();
        if (!last) return;
        for (int j = wv; j < 7; j += 4) {
            Comp w{0.0, 0.0};
#pragma unroll 4
            for (int b = lane; b < nb; b += 64) {
                const double* p = part + (b * 7 + j) * 2;
                w = comp_merge(w, Comp{__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                                       __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)});
            }
            w = wave_merge(w);
            if (lane == 0) res[j] = w;
        }
        __syncthreads();
    }
    if (threadIdx.x < 7) {
        const double v = res[threadIdx.x].s + res[threadIdx.x].c;
        totals[threadIdx.x] = v;
        if (host_totals) host_totals[threadIdx.x] = v;
    }
}

// out[perm[p] or p][f] = in[p][column of f at the padded radial functions]
// for the model's features f = (b Kabi + k)(M+1) + m.
__global__ void k_permute_rows(int64_t n, int Fabi, int F, int Kabi, int K, int M1, const int32_t* __restrict__ perm,
                               const float* __restrict__ in, float* __restrict__ out) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * Fabi) return;
    const int64_t p = idx / Fabi;
    const int f = (int)(idx - p * Fabi);
    const int per_b = Kabi * M1, b = f / per_b, r = f - b * per_b;
    const int fi = (b * K + r / M1) * M1 + r % M1;
    out[(perm ? (int64_t)perm[p] : p) * Fabi + f] = in[p * F + fi];
}

}  // namespace

tmd_status launch_finalize(tmd_context* ctx, const tmd_nlist* nl, const float* Ei, const unsigned long long* Fs,
                           const double* vir_partials, int nvir, float* atom_energy, float* forces, double* totals7,
                           double* host_totals, double* part) {
    const int64_t n = nl->n;
    const int nb = (int)std::min<int64_t>(kMaxPartials, (n + kPartAtoms - 1) / kPartAtoms);
    {
        ProfScope ps_(ctx, "finalize");
        k_finalize<<<(unsigned)(nb + (n + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
            n, nl->perm, Ei, Fs, atom_energy, forces, nb, nvir, vir_partials, part, finalize_counter(part), totals7,
            host_totals);
    }
    TMD_HIP(ctx, hipGetLastError());
    return TMD_OK;
}

tmd_status launch_permute_rows(tmd_context* ctx, const tmd_nlist* nl, const float* in, const tmd_model* m, float* out) {
    const int64_t total = nl->n * m->Fabi;
    {
        ProfScope ps_(ctx, "permute_rows");
        k_permute_rows<<<(unsigned)((total + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
            nl->n, m->Fabi, m->F, m->Kabi, m->K, m->M + 1, nl->perm, in, out);
    }
    TMD_HIP(ctx, hipGetLastError());
    return TMD_OK;
}

tmd_status launch_compact_features(tmd_context* ctx, int64_t n, const float* in, int F, int Fabi, int K, int Kabi,
                                   int M1, float* out) {
    const int64_t total = n * Fabi;
    if (total == 0) return TMD_OK;
    k_permute_rows<<<(unsigned)((total + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(n, Fabi, F, Kabi, K, M1,
                                                                                         nullptr, in, out);
    TMD_HIP(ctx, hipGetLastError());
    return TMD_OK;
}

}  // namespace tmd
