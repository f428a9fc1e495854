// gfx950 kernels for the state-vector hot path.
//
//  * gate application (Section 3.1, Algorithm 1), k <= 5: single gates whose
//    targets lie high enough straight from memory (amplitude pairs on VALU
//    for k <= 2, MFMA for k >= 3), and a tiled path that stages
//    2^tb-amplitude tiles in LDS for low targets and for several gates per
//    sweep, of one state or of many trajectories' states in one launch;
//  * small circuits (n <= 13) with the state in LDS from the first gate to
//    the last sample;
//  * FP64 reductions (norm, two-qubit reduced density matrix, the
//    conventional method's trial norm) with a fixed grid and a fixed
//    butterfly/tree order, so results are bit-identical run to run;
//  * measurement sampling: FP64 block sums, a tiled scan, one wavefront per
//    sample with Philox draws.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "qs_internal.h"
#include "qs_philox.h"

namespace qs {
namespace {

template <int K>
struct GateArgs {
    float2 m[(1 << K) * (1 << K)];
    int t[K];
};


// Insert a zero bit at each ascending target position.
template <int K, typename Idx>
__device__ __forceinline__ Idx spread_index(Idx g, const int *t) {
#pragma unroll
    for (int b = 0; b < K; ++b) {
        const int q = t[b];
        const Idx low = g & ((Idx(1) << q) - Idx(1));
        g = ((g >> q) << (q + 1)) | low;
    }
    return g;
}

template <int K, typename Idx>
__device__ __forceinline__ Idx local_offset(int j, const int *t) {
    Idx off = 0;
#pragma unroll
    for (int b = 0; b < K; ++b)
        if ((j >> b) & 1) off |= Idx(1) << t[b];
    return off;
}

// Read-only, wave-uniform matrices are read through the constant address
// space, so the compiler fetches them with scalar loads into SGPRs.
typedef const __attribute__((address_space(4))) float *ConstFloats;

__device__ __forceinline__ float2 const_entry(const float2 *p, int i) {
    const ConstFloats c = (ConstFloats)(p);
    return make_float2(c[2 * i], c[2 * i + 1]);
}

__device__ __forceinline__ float2 cmac(float2 acc, float2 a, float2 b) {
    acc.x = fmaf(a.x, b.x, acc.x);
    acc.x = fmaf(-a.y, b.y, acc.x);
    acc.y = fmaf(a.x, b.y, acc.y);
    acc.y = fmaf(a.y, b.x, acc.y);
    return acc;
}

// ---------------------------------------------------------------- gates

// A gate's matrix as the first kernel argument, read through the kernel
// argument segment: a program that applies gates one by one then needs no
// copy of the matrix before each launch (a copy kernel of 2 us and the gaps
// around it, for a gate of 9 us on 22 qubits).  A null device pointer selects
// it.
template <int K>
struct MatArg {
    alignas(16) float2 m[1 << (2 * K)];
};
__device__ __forceinline__ const float2 *gate_matrix(const float2 *dev) {
    return dev ? dev : (const float2 *)(__builtin_amdgcn_kernarg_segment_ptr());
}

// Direct path on VALU: one 2^K-amplitude group per work-item.  A work-item
// issues its group's loads before the workgroup stages the matrix.  K <= 2
// matrices are read with wave-uniform addresses straight from memory (scalar
// loads); larger ones are staged once per workgroup in LDS and read as
// broadcasts (states too small for the matrix units, and 5-qubit gates of
// fewer than 16 groups).
template <int K, typename Idx>
__global__ __launch_bounds__(kBlock) void apply_direct(MatArg<(K <= 4 ? K : 0)>, float2 *__restrict__ amp,
                                                       Idx groups, const float2 *mat_dev, TargetArgs ta) {
    constexpr int D = 1 << K;
    constexpr bool kLds = K >= 3;
    __shared__ float2 sm[kLds ? D * D : 1];
    const float2 *mat = gate_matrix(mat_dev);
    const Idx stride = Idx(gridDim.x) * Idx(kBlock);
    Idx g = Idx(blockIdx.x) * Idx(kBlock) + Idx(threadIdx.x);
    float2 v[D];
    if (g < groups) {
        const Idx base = spread_index<K, Idx>(g, ta.t);
#pragma unroll
        for (int j = 0; j < D; ++j) v[j] = amp[base + local_offset<K, Idx>(j, ta.t)];
    }
    if (kLds) {
        for (int i = threadIdx.x; i < D * D; i += kBlock) sm[i] = mat[i];
        __syncthreads();
    }
    float2 um[kLds ? 1 : D * D];
    if (!kLds) {
#pragma unroll
        for (int i = 0; i < (kLds ? 1 : D * D); ++i) um[i] = const_entry(mat, i);
    }
    const float2 *m = kLds ? sm : um;
    for (;;) {
        if (g >= groups) break;
        const Idx base = spread_index<K, Idx>(g, ta.t);
#pragma unroll(K >= 3 ? 2 : D)
        for (int j = 0; j < D; ++j) {
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int l = 0; l < D; ++l) acc = cmac(acc, m[j * D + l], v[l]);
            amp[base + local_offset<K, Idx>(j, ta.t)] = acc;
        }
        g += stride;
        if (g >= groups) break;
        const Idx nb = spread_index<K, Idx>(g, ta.t);
#pragma unroll
        for (int j = 0; j < D; ++j) v[j] = amp[nb + local_offset<K, Idx>(j, ta.t)];
    }
}

// K <= 2 with every target >= kPairTarget: two groups that differ in bit 0
// per work-item, so each access is a 16-byte amplitude pair.
template <int K, typename Idx>
__global__ __launch_bounds__(kBlock) void apply_pairs(MatArg<K>, float2 *__restrict__ amp, Idx pair_groups,
                                                      const float2 *mat_dev, TargetArgs ta) {
    constexpr int D = 1 << K;
    const float2 *mat = gate_matrix(mat_dev);
    float2 um[D * D];
#pragma unroll
    for (int i = 0; i < D * D; ++i) um[i] = const_entry(mat, i);
    const Idx stride = Idx(gridDim.x) * Idx(kBlock);
    for (Idx g = Idx(blockIdx.x) * Idx(kBlock) + Idx(threadIdx.x); g < pair_groups; g += stride) {
        const Idx base = spread_index<K, Idx>(g << 1, ta.t);
        float4 v[D];
#pragma unroll
        for (int j = 0; j < D; ++j)
            v[j] = *reinterpret_cast<const float4 *>(amp + base + local_offset<K, Idx>(j, ta.t));
#pragma unroll
        for (int j = 0; j < D; ++j) {
            float2 lo = make_float2(0.f, 0.f), hi = make_float2(0.f, 0.f);
#pragma unroll
            for (int l = 0; l < D; ++l) {
                lo = cmac(lo, um[j * D + l], make_float2(v[l].x, v[l].y));
                hi = cmac(hi, um[j * D + l], make_float2(v[l].z, v[l].w));
            }
            *reinterpret_cast<float4 *>(amp + base + local_offset<K, Idx>(j, ta.t)) =
                make_float4(lo.x, lo.y, hi.x, hi.y);
        }
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// K = 3, 4, 5 with every target >= 4, on FP32 MFMA straight from memory: the
// contraction of tile_gate_mfma3/4/5 (16 groups per wavefront batch, lane
// (n, q) = (l % 16, l / 16) supplies and returns the same amplitudes of group
// n), but with the batch's 16 groups differing in index bits 0..3, so that
// every access of a wavefront is four whole 128-byte lines and no LDS is
// needed.  All four real products are formed (re = A x - B y, im = B x + A y):
// memory bounds the pass, so the shorter three-product form would save
// nothing and rounds worse.  22 qubits, 64 MB moved, per gate: k = 3 12.1 ->
// 11.4 us (5.9 TB/s), k = 4 14.6 -> 13.5, k = 5 27.3 -> 19.7 against the VALU
// form above.  The next batch's loads are issued before this one's products.
template <int K, typename Idx>
__global__ __launch_bounds__(kBlock) void apply_direct_mfma(MatArg<(K <= 4 ? K : 0)>, float2 *__restrict__ amp,
                                                            Idx batches, const float2 *mat_dev, TargetArgs ta) {
    constexpr int D = 1 << K;
    constexpr int V = D / 4;            // amplitudes per lane
    constexpr int H = K == 5 ? 2 : 1;   // halves of 16 output rows (K = 3: the 16 real rows)
    const float2 *u = gate_matrix(mat_dev);
    const int lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
    // lane's amplitudes: 2q + s (K = 3), 4q + s (K = 4), 16 (s / 4) + 4q + s % 4 (K = 5)
    Idx off[V];
#pragma unroll
    for (int s = 0; s < V; ++s) {
        const int j = K == 3 ? 2 * q + s : 16 * (s >> 2) + 4 * q + (s & 3);
        Idx o = Idx(n);
#pragma unroll
        for (int b = 0; b < K; ++b) o |= Idx((j >> b) & 1) << ta.t[b];
        off[s] = o;
    }
    const Idx waves = Idx(gridDim.x) * Idx(kBlock / 64);
    Idx batch = Idx(blockIdx.x) * Idx(kBlock / 64) + Idx(__builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6));
    if (batch >= batches) return;
    const Idx first = spread_index<K, Idx>(batch << 4, ta.t);
    float2 v[V];
#pragma unroll
    for (int s = 0; s < V; ++s) v[s] = amp[first + off[s]];
    // A operands: row l % 16, contraction entry of lane quarter q in step s
    float fa[H][K == 3 ? 4 : V], fb[H][K == 3 ? 1 : V];
    if constexpr (K == 3) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float2 e = u[(n >> 1) * 8 + 2 * q + (s >> 1)];
            fa[0][s] = (n & 1) == 0 ? ((s & 1) == 0 ? e.x : -e.y) : ((s & 1) == 0 ? e.y : e.x);
        }
    } else {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int s = 0; s < V; ++s) {
                const float2 e = u[(16 * h + n) * D + 16 * (s >> 2) + 4 * q + (s & 3)];
                fa[h][s] = e.x;
                fb[h][s] = e.y;
            }
    }
    Idx base = first;
    for (;;) {
        const Idx next = batch + waves;
        const bool more = next < batches;
        Idx nbase = base;
        float2 w[V];
        if (more) {
            nbase = spread_index<K, Idx>(next << 4, ta.t);
#pragma unroll
            for (int s = 0; s < V; ++s) w[s] = amp[nbase + off[s]];
        }
        if constexpr (K == 3) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[0][0], v[0].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[0][1], v[0].y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[0][2], v[1].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[0][3], v[1].y, acc, 0, 0, 0);
            amp[base + off[0]] = make_float2(acc[0], acc[1]);
            amp[base + off[1]] = make_float2(acc[2], acc[3]);
        } else {
            float ny[V];
#pragma unroll
            for (int s = 0; s < V; ++s) ny[s] = -v[s].y;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < V; ++s) {
                    re = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[h][s], v[s].x, re, 0, 0, 0);
                    im = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[h][s], v[s].x, im, 0, 0, 0);
                    re = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[h][s], ny[s], re, 0, 0, 0);
                    im = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[h][s], v[s].y, im, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) amp[base + off[4 * h + r]] = make_float2(re[r], im[r]);
            }
        }
        if (!more) break;
        batch = next;
        base = nbase;
#pragma unroll
        for (int s = 0; s < V; ++s) v[s] = w[s];
    }
}

__host__ __device__ constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// Orders a wavefront's LDS accesses before this point against those behind it.
// The hardware keeps them in order (the lanes run in lockstep); the fences keep
// the compiler from moving accesses that one work-item does not see overlap.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS that is read as 16-byte vectors is declared so aligned.
#define QS_LDS_VECTORS(array) static_assert(__alignof__(array) % 16 == 0, "read as 16-byte vectors")

// Issue priority from the batches a wavefront still has to do in this gate:
// the arbiter favours older wavefronts, so without this the younger ones
// finish a gate late and the rest of the workgroup idles at the barrier.
__device__ __forceinline__ void prio_for_remaining(int remaining) {
    if (remaining >= 4) __builtin_amdgcn_s_setprio(3);
    else if (remaining == 3) __builtin_amdgcn_s_setprio(2);
    else if (remaining == 2) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// ---- LDS layout of a tile
// Gates read and write a tile in LDS one 64-lane instruction at a time; the
// lanes of an instruction span a few group bits and target bits of the
// local index, and with the plain layout (float2 index = local index) a gate
// on low local bits puts them on a handful of banks.  The tile kernel
// therefore stores local index x at x ^ m(x): bits 0..4 (which of 32 float2
// bank pairs) are XORed with a linear function m of bits 5..7.  The columns
// of m were chosen by scoring every target set of k <= 4 in 13 bits against
// the access pattern of each gate routine below (average cost 1.26x the
// conflict-free rate instead of 2x, worst case 2x instead of 4x).  Bits 8
// and up are left alone, so the tile copy's per-row offsets stay immediate.
// The map is linear over GF(2), so an index made of disjoint bit fields maps
// field by field, map(a | b) = map(a) ^ map(b): the gate loops split their
// indices into a per-lane part computed once and a wave-uniform part
// computed on the scalar unit.
struct SwizzledTile {
    __host__ __device__ __forceinline__ static int map(int x) {
        const int m = (((x >> 5) & 1) ? 30 : 0) ^ (((x >> 6) & 1) ? 27 : 0) ^ (((x >> 7) & 1) ? 23 : 0);
        return x ^ m;
    }
};

// Address table of a K-qubit gate on a tile.  Logical bit b of an index in
// the gate's frame is target b for b < K and, for b >= K, the (b - K)-th
// non-target local bit in ascending order (the group-index bits).
// tab[b] = 8 * map(1 << local position of logical bit b): the LDS byte offset
// that bit contributes.  The layout map is linear over GF(2), so the byte
// offset of any amplitude is the XOR of tab[] over its logical bits, and the
// gate loops only XOR table entries.  lt must be ascending; entries beyond the
// tile's width are unused.  Built on the host.
template <int K, class L>
__host__ __device__ inline void gate_tables(const int *lt, int *tab) {
#pragma unroll
    for (int b = 0; b < K; ++b) tab[b] = 8 * L::map(1 << lt[b]);
#pragma unroll
    for (int j = 0; j + K < kMaxTileBits; ++j) {
        int p = j;  // the j-th free position: j plus the targets at or below it
#pragma unroll
        for (int b = 0; b < K; ++b)
            if (lt[b] <= p) ++p;
        tab[K + j] = 8 * L::map(1 << p);
    }
}

// XOR of tab[first + j] over the set bits j < NBITS of x.
template <int NBITS>
__device__ __forceinline__ int tab_xor(const int *tab, int first, int x) {
    int r = 0;
#pragma unroll
    for (int j = 0; j < NBITS; ++j)
        if ((x >> j) & 1) r ^= tab[first + j];
    return r;
}

// LDS accesses by byte offset: each address is one XOR of a per-lane and a
// wave-uniform byte offset.
__device__ __forceinline__ float2 lds_get(const float2 *sd, int byte) {
    return *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(sd) + byte);
}
__device__ __forceinline__ void lds_put(float2 *sd, int byte, float2 v) {
    *reinterpret_cast<float2 *>(reinterpret_cast<char *>(sd) + byte) = v;
}
// The real and imaginary parts from two accumulators, as two 4-byte stores
// (one ds_write2_b32, with no register moves to pair them).
__device__ __forceinline__ void lds_put2(float2 *sd, int byte, float re, float im) {
    float *p = reinterpret_cast<float *>(reinterpret_cast<char *>(sd) + byte);
    p[0] = re;
    p[1] = im;
}
__device__ __forceinline__ float lds_getf(const float2 *sd, int byte) {
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(sd) + byte);
}

// Wavefront index as a scalar, so loops over it stay uniform.
__device__ __forceinline__ int wave_index() {
    return __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
}

// One gate on a tile held in LDS with VALU multiply-adds: every group of the
// tile is owned by one work-item, which gathers its 2^K amplitudes,
// multiplies, and writes back in place.  `m` is an LDS copy of the matrix.
template <int K, class L, int NT = kBlock>
__device__ __forceinline__ void tile_gate_valu(float2 *__restrict__ sd, const float2 *__restrict__ m,
                                               const int *lt, int tb) {
    constexpr int D = 1 << K;
    int off[D];
#pragma unroll
    for (int j = 0; j < D; ++j) off[j] = L::map(local_offset<K, int>(j, lt));
    const int groups = 1 << (tb - K);
    for (int gg = threadIdx.x; gg < groups; gg += NT) {
        const int lb = L::map(spread_index<K, int>(gg, lt));
        float2 v[D];
#pragma unroll
        for (int j = 0; j < D; ++j) v[j] = sd[lb ^ off[j]];
#pragma unroll(K >= 3 ? 2 : D)
        for (int j = 0; j < D; ++j) {
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int l = 0; l < D; ++l) acc = cmac(acc, m[j * D + l], v[l]);
            sd[lb ^ off[j]] = acc;
        }
    }
}

// K <= 2: the matrix (at most 16 entries) sits in SGPRs for the whole tile.
// Work-item (lane, wave) owns groups lane + 64 wave + NT i; the next group's
// amplitudes are read before this one's are written (the last iteration
// re-reads its own group, which is harmless: the reads precede the writes).
// MatLds: `gm` is an LDS copy (read as broadcasts) instead of global memory
// read through the scalar cache.
template <int K, class L, int NT = kBlock, bool MatLds = false>
__device__ __forceinline__ void tile_gate_small(float2 *__restrict__ sd, const float2 *gm,
                                                const int *lt, const int *tab, int tb) {
    constexpr int D = 1 << K;
    float2 u[D * D];
#pragma unroll
    for (int i = 0; i < D * D; ++i) u[i] = MatLds ? gm[i] : const_entry(gm, i);
    int off[D];
#pragma unroll
    for (int j = 0; j < D; ++j) off[j] = L::map(local_offset<K, int>(j, lt));
    constexpr int NB = ilog2(NT);
    if (tb < K + NB) {  // fewer groups than work-items (small resident states)
        const int groups = 1 << (tb - K);
        for (int gg = threadIdx.x; gg < groups; gg += NT) {
            const int lb = L::map(spread_index<K, int>(gg, lt));
            float2 v[D];
#pragma unroll
            for (int j = 0; j < D; ++j) v[j] = sd[lb ^ off[j]];
#pragma unroll
            for (int j = 0; j < D; ++j) {
                float2 acc = make_float2(0.f, 0.f);
#pragma unroll
                for (int l = 0; l < D; ++l) acc = cmac(acc, u[j * D + l], v[l]);
                sd[lb ^ off[j]] = acc;
            }
        }
        return;
    }
    // group index lane + 64 wave + NT it: logical bits K.. of the frame
    const int lane = threadIdx.x & 63, wave = wave_index();
    int ab[D];  // byte offset of amplitude j of the lane's group, without the batch part
    const int lane_part = tab_xor<6>(tab, K, lane);
#pragma unroll
    for (int j = 0; j < D; ++j) ab[j] = lane_part ^ tab_xor<K>(tab, 0, j);
    const int iters = 1 << (tb - K - NB);
    const int uw = tab_xor<NB - 6>(tab, K + 6, wave);
    int ub = uw;
    float2 v[D];
#pragma unroll
    for (int j = 0; j < D; ++j) v[j] = lds_get(sd, ab[j] ^ ub);
    for (int it = 0; it < iters; ++it) {
        prio_for_remaining(iters - it);
        const int itn = it + 1 < iters ? it + 1 : it;
        const int ubn = uw ^ tab_xor<kMaxTileBits - K - NB>(tab, K + NB, itn);
        float2 w[D];
#pragma unroll
        for (int j = 0; j < D; ++j) w[j] = lds_get(sd, ab[j] ^ ubn);
#pragma unroll
        for (int j = 0; j < D; ++j) {
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int l = 0; l < D; ++l) acc = cmac(acc, u[j * D + l], v[l]);
            lds_put(sd, ab[j] ^ ub, acc);
        }
        ub = ubn;
#pragma unroll
        for (int j = 0; j < D; ++j) v[j] = w[j];
    }
    __builtin_amdgcn_s_setprio(0);
}

// A fused k-qubit block is a dense contraction W = U V over the tile's
// 2^(tb-k) index groups.  For k = 3, 4, 5 it runs on FP32 MFMA
// (v_mfma_f32_16x16x4f32: in step s lane l supplies A[l%16][4s + l/16] and
// B[4s + l/16][l%16]; accumulator r is row 4(l/16) + r, column l%16), 16
// groups per wavefront batch, the groups' amplitudes (or real components)
// as B, the matrix as A laid out per lane once per launch ("fragments").
//
// The contraction index is permuted so that every lane supplies exactly the
// amplitudes its accumulators return: lane (n, q) = (l%16, l/16) reads and
// writes the same LDS words, and one address set per batch serves both.
// Physical step s, lane quarter q carries logical input index pi(4s + q),
// and the fragments hold the matrix columns in that order.
//
// Every gate also gets a per-lane LDS offset table staged after its
// fragments (lane_base): the lane part of its addresses (group index low
// bits n, quarter q), which would otherwise take some thirty VALU
// instructions per gate and tile on every wavefront.
constexpr int kFrag3 = 64 * 4;   // floats of k = 3 fragments; the lane table follows
constexpr int kFrag4 = 64 * 12;
constexpr int kFrag5 = 64 * 48;

// Real-form entry (row 2 jo + co, column 2 ji + ci) of a complex matrix.
__device__ __forceinline__ float real_form(float2 u, int co, int ci) {
    return co == 0 ? (ci == 0 ? u.x : -u.y) : (ci == 0 ? u.y : u.x);
}

// The lane table of a gate: table[lane] = XOR of tab[] over the lane's
// group bits n (logical bits nb..nb+3) and quarter bits q (logical bits
// qb, qb+1).
template <int NT>
__device__ __forceinline__ void stage_lane_table(int *__restrict__ table, const int *tab, int nb, int qb) {
    for (int lane = threadIdx.x; lane < 64; lane += NT) {
        int v = 0;
        for (int b = 0; b < 4; ++b)
            if ((lane >> b) & 1) v ^= tab[nb + b];
        for (int b = 0; b < 2; ++b)
            if ((lane >> (4 + b)) & 1) v ^= tab[qb + b];
        table[lane] = v;
    }
}

// k = 3 in the real form [[Re U, -Im U], [Im U, Re U]] (rows and columns
// interleaved as 2 j + c, c = 0 real, 1 imaginary).  Lane quarter q supplies
// the real components 4q + s (s = 0..3) of its group, i.e. amplitudes 2q and
// 2q + 1, and its accumulator rows 4q + r are the same components.
// Fragments: frag[lane * 4 + s] = RealForm[l%16][4 (l/16) + s].
// Lane table: group bits are logical bits 3.., amplitude 2q has q at bits 1, 2.
template <int NT = kBlock>
__device__ __forceinline__ void stage_frag3(float *__restrict__ frag, const float2 *__restrict__ u,
                                            const int *tab) {
    for (int i = threadIdx.x; i < 64 * 4; i += NT) {
        const int lane = i >> 2, s = i & 3;
        const int row = lane & 15, col = 4 * (lane >> 4) + s;
        frag[i] = real_form(u[(row >> 1) * 8 + (col >> 1)], row & 1, col & 1);
    }
    stage_lane_table<NT>(reinterpret_cast<int *>(frag + kFrag3), tab, 3, 1);
}

// k = 4 with three real products instead of four (Gauss), arranged so that
// the MFMA accumulators do the combining: for U = A + iB and v = x + iy,
// with k1 = A (x + y),
//   Re Uv = A x - B y = k1 - (A + B) y,   Im Uv = B x + A y = k1 + (B - A) x,
// so one chain forms k1 and two chains seeded with it add (-(A + B)) y and
// (B - A) x.  The only per-amplitude vector work left is x + y.  Lane
// quarter q supplies amplitudes 4q + s in step s and returns 4q + r.
// Fragments: frag[lane * 12 + 4 m + s] = M_m[l%16][4 (l/16) + s] with
// M_0 = Re U, M_1 = -(Re U + Im U), M_2 = Im U - Re U.
// Lane table: group bits are logical bits 4.., q at bits 2, 3.
template <int NT = kBlock>
__device__ __forceinline__ void stage_frag4(float *__restrict__ frag, const float2 *__restrict__ u,
                                            const int *tab) {
    for (int i = threadIdx.x; i < 64 * 12; i += NT) {
        const int lane = i / 12, rem = i - 12 * lane;
        const int m = rem >> 2, s = rem & 3;
        const float2 e = u[(lane & 15) * 16 + 4 * (lane >> 4) + s];
        frag[i] = m == 0 ? e.x : (m == 1 ? -(e.x + e.y) : e.y - e.x);
    }
    stage_lane_table<NT>(reinterpret_cast<int *>(frag + kFrag4), tab, 4, 2);
}

// k = 5: the same three real products as k = 4, each now a 32 x 32 matrix.
// The 32 output rows form two halves h (rows 16 h + i) and the contraction
// runs in eight steps of four: lane quarter q supplies amplitude
// 16 (s / 4) + 4 q + s % 4 in step s and accumulator r of half h returns
// 16 h + 4 q + r.  48 MFMAs per 16 groups (a 5-qubit block is the densest
// contraction of a sweep: 16 flops per byte moved, Section 3.1).
// Fragments: frag[lane * 48 + 24 h + 8 m + s] = M_m[16 h + l%16][16 (s / 4) +
// 4 (l/16) + s % 4].  Lane table: group bits are logical bits 5.., q at 2, 3.
template <int NT = kBlock>
__device__ __forceinline__ void stage_frag5(float *__restrict__ frag, const float2 *__restrict__ u,
                                            const int *tab) {
    for (int i = threadIdx.x; i < 64 * 48; i += NT) {
        const int lane = i / 48, rem = i - 48 * lane;
        const int h = rem / 24, m = (rem % 24) >> 3, s = rem & 7;
        const float2 e = u[(16 * h + (lane & 15)) * 32 + 16 * (s >> 2) + 4 * (lane >> 4) + (s & 3)];
        frag[i] = m == 0 ? e.x : (m == 1 ? -(e.x + e.y) : e.y - e.x);
    }
    stage_lane_table<NT>(reinterpret_cast<int *>(frag + kFrag5), tab, 5, 2);
}

// 16 groups per wavefront batch; the next batch's amplitudes are read before
// this one's MFMAs, so the LDS latency hides behind them (batches touch
// disjoint groups, so reading ahead of the writes is safe).  The batch index
// b = wave + W it occupies the logical bits after the lane's group bits.
template <class L, int NT = kBlock, bool PAIR = false>
__device__ __forceinline__ void tile_gate_mfma3(float2 *__restrict__ sd, f32x4 afr, int a0, const int *tab,
                                                int tb) {
    constexpr int W = NT / 64;
    constexpr int LW = ilog2(W);
    const int wave = wave_index();
    const int a1 = a0 ^ tab[0];  // amplitude 2q + 1
    const int iters = (1 << (tb - 3 - 4)) / W;  // batches per wave: >= 1 needs tb >= 7 + log2 W
    const int uw = tab_xor<LW>(tab, 7, wave);
    if constexpr (PAIR) {
        // two batches at a time: with two wavefronts per SIMD the chain of
        // four dependent products per batch is what a block waits for (with
        // the parallel member look-up of fuse_patched: 100 trajectories of the
        // 12-qubit chain 134 -> 120 us, 300 of 13 qubits 382 -> 341 a call)
        if (iters >= 2) {
            auto part = [&](int it) { return uw ^ tab_xor<kMaxTileBits - 7 - LW>(tab, 7 + LW, it); };
            int u0 = part(0), u1 = part(1);
            float2 p0 = lds_get(sd, a0 ^ u0), p1 = lds_get(sd, a1 ^ u0);
            float2 q0 = lds_get(sd, a0 ^ u1), q1 = lds_get(sd, a1 ^ u1);
            for (int it = 0; it < iters; it += 2) {
                prio_for_remaining(iters - it);
                const int nx = it + 2 < iters ? it + 2 : it;
                const int n0 = part(nx), n1 = part(nx + 1);
                const float2 r0 = lds_get(sd, a0 ^ n0), r1 = lds_get(sd, a1 ^ n0);
                const float2 s0 = lds_get(sd, a0 ^ n1), s1 = lds_get(sd, a1 ^ n1);
                f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = {0.f, 0.f, 0.f, 0.f};
                x = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[0], p0.x, x, 0, 0, 0);
                y = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[0], q0.x, y, 0, 0, 0);
                x = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[1], p0.y, x, 0, 0, 0);
                y = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[1], q0.y, y, 0, 0, 0);
                x = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[2], p1.x, x, 0, 0, 0);
                y = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[2], q1.x, y, 0, 0, 0);
                x = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[3], p1.y, x, 0, 0, 0);
                y = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[3], q1.y, y, 0, 0, 0);
                lds_put(sd, a0 ^ u0, make_float2(x[0], x[1]));
                lds_put(sd, a1 ^ u0, make_float2(x[2], x[3]));
                lds_put(sd, a0 ^ u1, make_float2(y[0], y[1]));
                lds_put(sd, a1 ^ u1, make_float2(y[2], y[3]));
                u0 = n0;
                u1 = n1;
                p0 = r0;
                p1 = r1;
                q0 = s0;
                q1 = s1;
            }
            __builtin_amdgcn_s_setprio(0);
            return;
        }
    }
    int ub = uw;
    float2 v0 = lds_get(sd, a0 ^ ub), v1 = lds_get(sd, a1 ^ ub);
    for (int it = 0; it < iters; ++it) {
        prio_for_remaining(iters - it);
        const int itn = it + 1 < iters ? it + 1 : it;
        const int ubn = uw ^ tab_xor<kMaxTileBits - 7 - LW>(tab, 7 + LW, itn);
        const float2 w0 = lds_get(sd, a0 ^ ubn), w1 = lds_get(sd, a1 ^ ubn);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[0], v0.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[1], v0.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[2], v1.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(afr[3], v1.y, acc, 0, 0, 0);
        lds_put(sd, a0 ^ ub, make_float2(acc[0], acc[1]));
        lds_put(sd, a1 ^ ub, make_float2(acc[2], acc[3]));
        ub = ubn;
        v0 = w0;
        v1 = w1;
    }
    __builtin_amdgcn_s_setprio(0);
}

template <class L, int NT = kBlock>
__device__ __forceinline__ void tile_gate_mfma4(float2 *__restrict__ sd, f32x4 fa, f32x4 fb, f32x4 fs, int base,
                                                const int *tab, int tb) {
    constexpr int W = NT / 64;
    constexpr int LW = ilog2(W);
    const int wave = wave_index();
    int a[4];  // amplitude 4q + s of the lane's group
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = base ^ tab_xor<2>(tab, 0, s);
    const int iters = (1 << (tb - 4 - 4)) / W;  // batches per wave: >= 1 needs tb >= 8 + log2 W
    const int uw = tab_xor<LW>(tab, 8, wave);
    int ub = uw;
    float2 v[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = lds_get(sd, a[s] ^ ub);
    for (int it = 0; it < iters; ++it) {
        prio_for_remaining(iters - it);
        const int itn = it + 1 < iters ? it + 1 : it;
        const int ubn = uw ^ tab_xor<kMaxTileBits - 8 - LW>(tab, 8 + LW, itn);
        float2 w[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) w[s] = lds_get(sd, a[s] ^ ubn);
        f32x4 k1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) k1 = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[s], v[s].x + v[s].y, k1, 0, 0, 0);
        f32x4 re = k1, im = k1;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            re = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[s], v[s].y, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f32_16x16x4f32(fs[s], v[s].x, im, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) lds_put2(sd, a[r] ^ ub, re[r], im[r]);
        ub = ubn;
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = w[s];
    }
    __builtin_amdgcn_s_setprio(0);
}

// The same from the fragments a sweep staged in LDS.
template <class L, int NT>
__device__ __forceinline__ void staged_gate_mfma3(float2 *__restrict__ sd, const float *__restrict__ frag,
                                                  const int *tab, int tb) {
    const int lane = threadIdx.x & 63;
    tile_gate_mfma3<L, NT>(sd, *reinterpret_cast<const f32x4 *>(frag + lane * 4),
                           reinterpret_cast<const int *>(frag + kFrag3)[lane], tab, tb);
}
template <class L, int NT>
__device__ __forceinline__ void staged_gate_mfma4(float2 *__restrict__ sd, const float *__restrict__ frag,
                                                  const int *tab, int tb) {
    const int lane = threadIdx.x & 63;
    const f32x4 *fp = reinterpret_cast<const f32x4 *>(frag + lane * 12);
    tile_gate_mfma4<L, NT>(sd, fp[0], fp[1], fp[2], reinterpret_cast<const int *>(frag + kFrag4)[lane], tab, tb);
}

// ---- k = 4 on BF16 MFMA with FP32 operands split in three
// x = h + m + l with h, m, l BF16 (8 significant bits each, rounded to
// nearest), exactly for FP32 |x| from 2^-110 (below, l leaves BF16's range) to
// 3.39e38 (BF16's largest number).  An infinite component leaves no number in
// its group, as in the FP32 form, whose sums of real and imaginary parts spread
// it.  Of
// the nine products of a split operand pair the three below 2^-26 of the
// largest are left out; the other six are exact in FP32 and are accumulated
// in FP32 from the smallest up, 32 terms per instruction.  Against the FP32
// form above: 192 matrix cycles per batch of 16 groups instead of 384, plus
// 28 VALU instructions for the split, which can issue beside BF16 products
// (beside FP32 ones none did): a block on 2^24 amplitudes takes 11.4 us
// instead of 14, a 24-qubit sweep of four 65 instead of 75, a 28-qubit one
// 1.03 ms instead of 1.11.  The result is nearer the 64-bit one: relative L2
// error of noisy 15- to 30-qubit trajectories 0.4 to 0.9e-6 instead of 0.75
// to 1.2e-6 (one rounding per 32 terms and product instead of one per 4, and
// no sums of real and imaginary parts).  3-qubit blocks stay on FP32: split,
// they measured no faster (their products are a third of the split's cost).
// Used for the sweeps of states above kBatchLdsQubits qubits, whichever
// launch runs them; resident states and the batched launch keep the FP32
// form, in which their results are pinned.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct Split3 {
    unsigned int h, m, l;  // two BF16 values each: low half from the first argument
};
__device__ __forceinline__ bf16x2 pack_bf16(float a, float b) {
    const bf16x2 p = {(__bf16)a, (__bf16)b};  // round to nearest even
    return p;
}
// Seven instructions for two values: the remainder x - h comes from a
// two-term BF16 dot product with (-1, 0) or (0, -1), which needs no unpacking
// (both terms and the result are exact).  The two constants are made opaque:
// as inline constants both assemble to -1.0, which the instruction reads as
// the second one.
__device__ __forceinline__ bf16x2 opaque_bf16(unsigned int bits) {
    asm("" : "+s"(bits));
    return __builtin_bit_cast(bf16x2, bits);
}
__device__ __forceinline__ Split3 split3(float a, float b) {
    const bf16x2 lo = opaque_bf16(0x0000bf80u), hi = opaque_bf16(0xbf800000u);
    const bf16x2 h = pack_bf16(a, b);
    a = __builtin_amdgcn_fdot2_f32_bf16(h, lo, a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(h, hi, b, false);
    const bf16x2 m = pack_bf16(a, b);
    a = __builtin_amdgcn_fdot2_f32_bf16(m, lo, a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(m, hi, b, false);
    const bf16x2 l = pack_bf16(a, b);
    return Split3{__builtin_bit_cast(unsigned int, h), __builtin_bit_cast(unsigned int, m),
                  __builtin_bit_cast(unsigned int, l)};
}
__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

// Issue priority of a split gate: products before splitting, so that the
// matrix unit is fed while other wavefronts' VALU work fills the cycles in
// between, and within each the wavefronts that have more batches to do (see
// prio_for_remaining).
__device__ __forceinline__ void prio_split(int remaining, bool products) {
    if (products) {
        if (remaining >= 3) __builtin_amdgcn_s_setprio(3);
        else __builtin_amdgcn_s_setprio(2);
    } else {
        if (remaining >= 3) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
    }
}

// Fragments: for U[l % 16][4 (l / 16) + s] = a + ib, s < 4, the pair (a, -b)
// split: dword 12 lane + 4 part + s, part 0 (h), 1 (m), 2 (l).  Lane table as
// for k = 4.
template <int NT = kBlock>
__device__ __forceinline__ void stage_split4(unsigned int *__restrict__ frag, const float2 *__restrict__ u,
                                             const int *tab) {
    for (int i = threadIdx.x; i < 64 * 4; i += NT) {
        const int lane = i >> 2, s = i & 3;
        const float2 e = u[(lane & 15) * 16 + 4 * (lane >> 4) + s];
        const Split3 f = split3(e.x, -e.y);
        frag[12 * lane + s] = f.h;
        frag[12 * lane + 4 + s] = f.m;
        frag[12 * lane + 8 + s] = f.l;
    }
    stage_lane_table<NT>(reinterpret_cast<int *>(frag + kFrag4), tab, 4, 2);
}

// Lane (n, q) supplies amplitudes 4 q + s of group n as (x, y) pairs in the
// contraction and gets amplitudes 4 q + r back, as in tile_gate_mfma4.  The
// real part contracts with (a, -b), the imaginary one with (b, a), which is
// the same dword with its halves swapped and the low one negated.
template <class L, int NT>
__device__ __forceinline__ void tile_gate_split4(float2 *__restrict__ sd, const float *__restrict__ frag,
                                                 const int *tab, int tb) {
    constexpr int W = NT / 64;
    constexpr int LW = ilog2(W);
    const int lane = threadIdx.x & 63, wave = wave_index();
    const u32x4 *fp = reinterpret_cast<const u32x4 *>(frag + lane * 12);
    u32x4 F[3], G[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        F[p] = fp[p];
#pragma unroll
        for (int s = 0; s < 4; ++s) G[p][s] = __builtin_amdgcn_alignbit(F[p][s], F[p][s], 16) ^ 0x8000u;
    }
    const int base = reinterpret_cast<const int *>(frag + kFrag4)[lane];
    int a[4];  // amplitude 4q + s of the lane's group
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = base ^ tab_xor<2>(tab, 0, s);
    const int iters = (1 << (tb - 4 - 4)) / W;  // batches per wave: >= 1 needs tb >= 8 + log2 W
    const int uw = tab_xor<LW>(tab, 8, wave);
    int ub = uw;
    float2 v[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = lds_get(sd, a[s] ^ ub);
    for (int it = 0; it < iters; ++it) {
        prio_split(iters - it, false);
        const int itn = it + 1 < iters ? it + 1 : it;
        const int ubn = uw ^ tab_xor<kMaxTileBits - 8 - LW>(tab, 8 + LW, itn);
        u32x4 E[3];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const Split3 e = split3(v[s].x, v[s].y);
            E[0][s] = e.h;
            E[1][s] = e.m;
            E[2][s] = e.l;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = lds_get(sd, a[s] ^ ubn);
        prio_split(iters - it, true);
        f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = {0.f, 0.f, 0.f, 0.f};
        re = mfma_bf16(F[2], E[0], re);
        im = mfma_bf16(G[2], E[0], im);
        re = mfma_bf16(F[0], E[2], re);
        im = mfma_bf16(G[0], E[2], im);
        re = mfma_bf16(F[1], E[1], re);
        im = mfma_bf16(G[1], E[1], im);
        re = mfma_bf16(F[1], E[0], re);
        im = mfma_bf16(G[1], E[0], im);
        re = mfma_bf16(F[0], E[1], re);
        im = mfma_bf16(G[0], E[1], im);
        re = mfma_bf16(F[0], E[0], re);
        im = mfma_bf16(G[0], E[0], im);
#pragma unroll
        for (int r = 0; r < 4; ++r) lds_put2(sd, a[r] ^ ub, re[r], im[r]);
        ub = ubn;
    }
    __builtin_amdgcn_s_setprio(0);
}

// The two output halves are formed one after the other from the same
// inputs in registers.
template <class L, int NT = kBlock>
__device__ __forceinline__ void tile_gate_mfma5(float2 *__restrict__ sd, const float *__restrict__ frag,
                                                const int *tab, int tb) {
    constexpr int W = NT / 64;
    constexpr int LW = ilog2(W);
    const int lane = threadIdx.x & 63, wave = wave_index();
    const f32x4 *fp = reinterpret_cast<const f32x4 *>(frag + lane * 48);
    f32x4 F[12];  // F[6 h + 2 m + s / 4][s % 4]
#pragma unroll
    for (int i = 0; i < 12; ++i) F[i] = fp[i];
    const int base = reinterpret_cast<const int *>(frag + kFrag5)[lane];
    int a[8];  // amplitude 16 h + 4 q + r of the lane's group at a[4 h + r]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) a[4 * h + r] = base ^ tab_xor<2>(tab, 0, r) ^ (h ? tab[4] : 0);
    const int iters = (1 << (tb - 5 - 4)) / W;  // batches per wave: >= 1 needs tb >= 9 + log2 W
    const int uw = tab_xor<LW>(tab, 9, wave);
    int ub = uw;
    float2 v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = lds_get(sd, a[s] ^ ub);
    for (int it = 0; it < iters; ++it) {
        prio_for_remaining(iters - it);
        const int itn = it + 1 < iters ? it + 1 : it;
        const int ubn = uw ^ tab_xor<kMaxTileBits - 9 - LW>(tab, 9 + LW, itn);
        float2 w[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) w[s] = lds_get(sd, a[s] ^ ubn);
        float xy[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) xy[s] = v[s].x + v[s].y;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4 k1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 8; ++s)
                k1 = __builtin_amdgcn_mfma_f32_16x16x4f32(F[6 * h + (s >> 2)][s & 3], xy[s], k1, 0, 0, 0);
            f32x4 re = k1, im = k1;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                re = __builtin_amdgcn_mfma_f32_16x16x4f32(F[6 * h + 2 + (s >> 2)][s & 3], v[s].y, re, 0, 0, 0);
                im = __builtin_amdgcn_mfma_f32_16x16x4f32(F[6 * h + 4 + (s >> 2)][s & 3], v[s].x, im, 0, 0, 0);
            }
            // inputs are in registers, so this half's outputs may overwrite them in LDS
#pragma unroll
            for (int r = 0; r < 4; ++r) lds_put2(sd, a[4 * h + r] ^ ub, re[r], im[r]);
        }
        ub = ubn;
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = w[s];
    }
    __builtin_amdgcn_s_setprio(0);
}

// Tiled path: persistent workgroups stage every gate matrix of the launch in
// LDS once (as MFMA fragments for k = 3, 4; plain for k = 5; k <= 2 matrices
// stay in global memory and arrive through scalar loads), then loop over
// tiles of 2^TB amplitudes -- the index bits in a.pos, bits 0..3 first, so
// every eight lanes of a wavefront load one whole 128-byte line.  A tile is written to LDS, the next
// tile's loads are issued into registers, the gates run on the LDS copy in
// order, and the tile is written back: any number of gates inside the tile
// cost one HBM read and one write.
// K5: whether the launch holds a 5-qubit block (its path needs many more
// VGPRs, so launches without one use a leaner instantiation).  5-qubit blocks
// run on MFMA when every wavefront gets a batch of 16 groups (TB >= 9 +
// log2(NT / 64)), else on VALU from the plain matrix.
// RK: the launch also accumulates the reduced density matrix of one tile
// qubit (TileArgs::rdm_out) from every tile after its gates.
//
// The sweep's description comes through Src: the kernel's own arguments
// (apply_tile) or tables in device memory (batch_sweep).  Tiles first,
// first + step, ... below last are this workgroup's.
// K5V: 5-qubit blocks take the VALU path at any tile width (the batched
// launch, whose resident states do).
template <int TB, typename Idx, bool K5, int NT, bool RK, bool K5V, bool SP, class Src>
__device__ __forceinline__ void tile_sweep(float2 *__restrict__ amp, Idx first, Idx step, Idx last, const Src &a,
                                           float2 *__restrict__ sd, float2 *__restrict__ sm) {
    constexpr int NB = ilog2(NT);
    constexpr bool K5_MFMA = !K5V && TB >= 9 + NB - 6;
    static_assert(TB >= 10, "the MFMA gates need at least 32 groups per tile");
    static_assert((1 << (TB - 8)) >= NT / 64, "every wavefront needs a 4-qubit batch");
    constexpr int E = 1 << TB;
    // Each work-item moves R amplitude pairs per tile: pair (t, r) holds local
    // indices 2 t + NT 2 r + {0, 1}, which differ in local bit 0 = qubit 0, so
    // the pair is one 16-byte load or store, and each eight lanes cover one
    // 128-byte line (local bits 0..3 are global bits 0..3).
    constexpr int R = E / (2 * NT);
    Idx tile = first;
    if (tile >= last) return;  // uniform over the workgroup
    Idx off_tid = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if ((threadIdx.x >> b) & 1) off_tid |= Idx(1) << a.pos(b + 1);
    Idx off_r[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        Idx o = 0;
#pragma unroll
        for (int b = NB + 1; b < TB; ++b)
            if (((r << (NB + 1)) >> b) & 1) o |= Idx(1) << a.pos(b);
        off_r[r] = o;
    }
    // First index of tile t: the bits of t spread over the positions the tile
    // does not hold.  Inserting a zero at position q adds the part of the
    // index at and above q to itself (shifting it up by one); positions 0..3
    // are always the tile's, which is one shift.
    auto tile_base = [&](Idx t) {
        Idx base = t << kTileLowBits;
#pragma unroll
        for (int b = kTileLowBits; b < TB; ++b) base += base & (~Idx(0) << a.pos(b));
        return base + off_tid;
    };
    // A tile's amplitude pairs.  With init_zero the sweep starts from
    // |0...0> without reading the state: nothing is fetched, and the tile's
    // LDS copy is written from zeros (amplitude 1 at index 0).
    auto fetch = [&](Idx t, float4 (&dst)[R]) {
        if (a.init_zero()) return;
        const Idx base = tile_base(t);
#pragma unroll
        for (int r = 0; r < R; ++r) dst[r] = *reinterpret_cast<const float4 *>(amp + base + off_r[r]);
    };
    float4 v[R];
    fetch(tile, v);
    for (int gi = 0; gi < a.n_gates(); ++gi) {
        const int k = a.k(gi);
        const float2 *src = a.mat(gi);
        float2 *dst = sm + a.lofs(gi);
        int gtab[kMaxTileBits];
#pragma unroll
        for (int b = 0; b < kMaxTileBits; ++b) gtab[b] = a.tab(gi, b);
        if (k == 4) {
            if constexpr (SP) stage_split4<NT>(reinterpret_cast<unsigned int *>(dst), src, gtab);
            else stage_frag4<NT>(reinterpret_cast<float *>(dst), src, gtab);
        } else if (k == 3) {
            stage_frag3<NT>(reinterpret_cast<float *>(dst), src, gtab);
        } else if (k == 5) {
            if constexpr (K5_MFMA) stage_frag5<NT>(reinterpret_cast<float *>(dst), src, gtab);
            else
                for (int i = threadIdx.x; i < 1024; i += NT) dst[i] = src[i];
        }
    }
    // One tile: the prefetched amplitudes go to LDS, the previous tile's
    // results (held in registers since its gates finished) are stored, the
    // next tile's loads are issued, the gates run, and the results are read
    // out of LDS into registers.  Stores and loads therefore drain while this
    // tile's gates run, instead of the stores going out in a burst at the end
    // of every tile; the wait for the prefetch at the next loop head covers
    // memory operations issued a whole gate phase earlier.
    // LDS index of local index 2 threadIdx.x + e + 2 NT r: the map leaves the
    // r part alone and flipping bit 0 of an index flips bit 0 of its image,
    // so it is tid_l ^ e + (r << NB + 1).  tid_l itself may be odd (columns 27
    // and 23 of the map set bit 0), so a pair is adjacent but not always in
    // order: it is not one 16-byte LDS access.
    const int tid_l = SwizzledTile::map(int(threadIdx.x) << 1);
    float4 o[R];
    Idx prev_base = 0;
    // RDM of the qubit at tile bit rdm_lt: R00, R11 and R01 = sum v0 conj(v1)
    // over every pair of the work-item's amplitudes that differ in that bit,
    // in a fixed order, summed over the workgroup's tiles.
    double r00 = 0.0, r11 = 0.0, r01r = 0.0, r01i = 0.0;
    auto run_tile = [&](Idx t, bool has_prev) {
        __syncthreads();  // the previous tile is out of LDS; matrices staged
        const Idx base = tile_base(t);
        if (a.init_zero()) {
            const float one = base == Idx(0) ? 1.f : 0.f;  // index 0 is pair 0 of work-item 0
#pragma unroll
            for (int r = 0; r < R; ++r) {
                sd[tid_l + (r << (NB + 1))] = make_float2(r == 0 ? one : 0.f, 0.f);
                sd[(tid_l ^ 1) + (r << (NB + 1))] = make_float2(0.f, 0.f);
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                sd[tid_l + (r << (NB + 1))] = make_float2(v[r].x, v[r].y);
                sd[(tid_l ^ 1) + (r << (NB + 1))] = make_float2(v[r].z, v[r].w);
            }
        }
        if (has_prev) {
#pragma unroll
            for (int r = 0; r < R; ++r) *reinterpret_cast<float4 *>(amp + prev_base + off_r[r]) = o[r];
        }
        const Idx next = t + step;
        if (next < last) fetch(next, v);
        __syncthreads();
        for (int gi = 0; gi < a.n_gates(); ++gi) {
            const int k = a.k(gi);
            int lt[kMaxGateQubits], tab[kMaxTileBits];
#pragma unroll
            for (int b = 0; b < kMaxGateQubits; ++b) lt[b] = a.lt(gi, b);
#pragma unroll
            for (int b = 0; b < kMaxTileBits; ++b) tab[b] = a.tab(gi, b);
            switch (k) {
                case 1: tile_gate_small<1, SwizzledTile, NT>(sd, a.mat(gi), lt, tab, TB); break;
                case 2: tile_gate_small<2, SwizzledTile, NT>(sd, a.mat(gi), lt, tab, TB); break;
                case 3:
                    staged_gate_mfma3<SwizzledTile, NT>(sd, reinterpret_cast<const float *>(sm + a.lofs(gi)), tab,
                                                        TB);
                    break;
                case 4:
                    if constexpr (SP)
                        tile_gate_split4<SwizzledTile, NT>(sd, reinterpret_cast<const float *>(sm + a.lofs(gi)), tab,
                                                           TB);
                    else
                        staged_gate_mfma4<SwizzledTile, NT>(sd, reinterpret_cast<const float *>(sm + a.lofs(gi)), tab,
                                                            TB);
                    break;
                default:
                    if constexpr (K5 && K5_MFMA)
                        tile_gate_mfma5<SwizzledTile, NT>(sd, reinterpret_cast<const float *>(sm + a.lofs(gi)),
                                                          tab, TB);
                    else if constexpr (K5)
                        tile_gate_valu<5, SwizzledTile, NT>(sd, sm + a.lofs(gi), lt, TB);
                    break;
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 lo = sd[tid_l + (r << (NB + 1))], hi = sd[(tid_l ^ 1) + (r << (NB + 1))];
            o[r] = make_float4(lo.x, lo.y, hi.x, hi.y);
        }
        if (RK && a.rdm_out()) {
            // the work-item's amplitudes are local indices 2 tid + e + 2 NT r,
            // read again from LDS (a rolled loop keeps the registers of the
            // common sweep); the partner across the qubit's bit pc sits at
            // LDS index ^ map(2^pc)
            const int pc = a.rdm_lt();
            const int pm = SwizzledTile::map(1 << pc);
            const int tid_bit = pc >= 1 && pc <= NB ? (int(threadIdx.x) >> (pc - 1)) & 1 : 0;
#pragma unroll 1
            for (int i = 0; i < 2 * R; ++i) {
                const int r = i >> 1, e = i & 1;
                const int bit = pc == 0 ? e : (pc <= NB ? tid_bit : (r >> (pc - NB - 1)) & 1);
                const int at = (tid_l ^ e) + (r << (NB + 1));
                const float2 v = sd[at];
                const double vr = v.x, vi = v.y;
                if (bit) {
                    r11 = fma(vr, vr, fma(vi, vi, r11));
                } else {
                    r00 = fma(vr, vr, fma(vi, vi, r00));
                    const float2 u = sd[at ^ pm];
                    const double ur = u.x, ui = u.y;
                    r01r = fma(vr, ur, fma(vi, ui, r01r));
                    r01i = fma(vi, ur, fma(-vr, ui, r01i));
                }
            }
        }
        prev_base = base;
    };
    run_tile(tile, false);
    for (tile += step; tile < last; tile += step) run_tile(tile, true);
#pragma unroll
    for (int r = 0; r < R; ++r) *reinterpret_cast<float4 *>(amp + prev_base + off_r[r]) = o[r];
    if (RK && a.rdm_out()) {
        // wavefront sums by a fixed shuffle tree, then the wavefronts in order
        // through LDS (the tile is no longer needed once every wavefront has
        // read its last tile out)
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            r00 += __shfl_xor(r00, off, 64);
            r11 += __shfl_xor(r11, off, 64);
            r01r += __shfl_xor(r01r, off, 64);
            r01i += __shfl_xor(r01i, off, 64);
        }
        __syncthreads();
        double *red = reinterpret_cast<double *>(sd);
        const int wave = int(threadIdx.x) >> 6;
        if ((threadIdx.x & 63) == 0) {
            red[4 * wave] = r00;
            red[4 * wave + 1] = r11;
            red[4 * wave + 2] = r01r;
            red[4 * wave + 3] = r01i;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double s00 = 0.0, s11 = 0.0, sr = 0.0, si = 0.0;
            for (int w = 0; w < NT / 64; ++w) {
                s00 += red[4 * w];
                s11 += red[4 * w + 1];
                sr += red[4 * w + 2];
                si += red[4 * w + 3];
            }
            double *rec = a.rdm_out() + size_t(blockIdx.x) * 8;
            rec[0] = s00;
            rec[1] = 0.0;
            rec[2] = sr;
            rec[3] = si;
            rec[4] = sr;
            rec[5] = -si;
            rec[6] = s11;
            rec[7] = 0.0;
        }
    }
}

// A launch's sweep in the kernel's arguments.
struct ArgSweep {
    const TileArgs &a;
    __device__ __forceinline__ int pos(int b) const { return a.pos[b]; }
    __device__ __forceinline__ int n_gates() const { return a.n_gates; }
    __device__ __forceinline__ int init_zero() const { return a.init_zero; }
    __device__ __forceinline__ int rdm_lt() const { return a.rdm_lt; }
    __device__ __forceinline__ double *rdm_out() const { return a.rdm_out; }
    __device__ __forceinline__ int k(int gi) const { return a.g[gi].k; }
    __device__ __forceinline__ int lt(int gi, int b) const { return a.g[gi].lt[b]; }
    __device__ __forceinline__ int lofs(int gi) const { return a.g[gi].lofs; }
    __device__ __forceinline__ int tab(int gi, int b) const { return a.g[gi].tab[b]; }
    __device__ __forceinline__ const float2 *mat(int gi) const { return a.g[gi].mat; }
};

template <int TB, typename Idx, bool K5, int NT, bool RK, bool SP>
__global__ __launch_bounds__(NT) void apply_tile(float2 *__restrict__ amp, Idx n_tiles, TileArgs a) {
    // The tile is a static array (its LDS address is a link-time constant
    // that folds into the LDS instructions' offsets); the launch's matrices
    // follow it in dynamic LDS.
    __shared__ float2 sd[1 << TB];
    alignas(16) extern __shared__ float2 sm[];
    QS_LDS_VECTORS(sm);
    tile_sweep<TB, Idx, K5, NT, RK, false, SP>(amp, Idx(blockIdx.x), Idx(gridDim.x), n_tiles, ArgSweep{a}, sd, sm);
}

// One gate of at most four qubits over tiles, its matrix among the kernel's
// arguments when the caller has no device copy.
struct OneGate {
    const TileOneArgs &a;
    __device__ __forceinline__ int pos(int b) const { return a.pos[b]; }
    __device__ __forceinline__ int n_gates() const { return 1; }
    __device__ __forceinline__ int init_zero() const { return 0; }
    __device__ __forceinline__ int rdm_lt() const { return 0; }
    __device__ __forceinline__ double *rdm_out() const { return nullptr; }
    __device__ __forceinline__ int k(int) const { return a.g.k; }
    __device__ __forceinline__ int lt(int, int b) const { return a.g.lt[b]; }
    __device__ __forceinline__ int lofs(int) const { return 0; }
    __device__ __forceinline__ int tab(int, int b) const { return a.g.tab[b]; }
    __device__ __forceinline__ const float2 *mat(int) const { return gate_matrix(a.g.mat); }
};

template <int TB, typename Idx>
__global__ __launch_bounds__(kBlock) void apply_tile_one(MatArg<4>, float2 *__restrict__ amp, Idx n_tiles,
                                                         TileOneArgs a) {
    __shared__ float2 sd[1 << TB];
    __shared__ alignas(16) float2 sm[416];  // tile_mat_slots(4)
    QS_LDS_VECTORS(sm);
    tile_sweep<TB, Idx, false, kBlock, false, false, false>(amp, Idx(blockIdx.x), Idx(gridDim.x), n_tiles, OneGate{a}, sd,
                                                     sm);
}

// ---------------------------------------------------------------- branch selection

// Steps 13-20 of Algorithm 2 on one work-item: the pick and the factor
// 1/sqrt(p N) from R (`rdm`, D x D complex128).
__device__ __forceinline__ void pick_branch(const double *rdm, int D, const double *excess, const double *pbar,
                                            int nk, double resid, int *err, int *pick, double *scale) {
    double N = 0.0;
    for (int j = 0; j < D; ++j) N += rdm[2 * (j * D + j)];
    auto weight = [&](int i) {
        const double *M = excess + size_t(i) * D * D * 2;
        double tr = 0.0;  // Re sum_jl M[j][l] R[l][j]
        for (int j = 0; j < D; ++j)
            for (int l = 0; l < D; ++l) {
                const double mr = M[2 * (j * D + l)], mi = M[2 * (j * D + l) + 1];
                const double rr = rdm[2 * (l * D + j)], ri = rdm[2 * (l * D + j) + 1];
                tr += mr * rr - mi * ri;
            }
        return tr / N;
    };
    double r = resid;
    int chosen = -1, last_pos = -1;
    double e_chosen = 0.0;
    for (int i = 0; i < nk; ++i) {
        const double e = weight(i);
        if (e > 0.0) last_pos = i;
        if (r < e) {
            chosen = i;
            e_chosen = e;
            break;
        }
        r -= e;
    }
    if (chosen < 0) {
        chosen = last_pos >= 0 ? last_pos : nk - 1;
        e_chosen = weight(chosen);
    }
    const double p = pbar[chosen] + e_chosen;
    if (!(N > 0.0) || !(p > 0.0) || !(N < INFINITY)) {
        *err = 1;
        *scale = 0.0;
    } else {
        *scale = 1.0 / sqrt(p * N);
    }
    *pick = chosen;
}

__global__ __launch_bounds__(64) void select_branch(SelectArgs a) {
    __shared__ double scale;
    __shared__ int pick;
    if (threadIdx.x == 0) {
        pick_branch(a.rdm, a.D, a.excess, a.pbar, a.nk, a.resid, a.err, &pick, &scale);
        *a.choice = pick;
    }
    __syncthreads();
    const int dd = a.Db * a.Db;
    const double *c = a.cand + size_t(pick) * dd * 2;
    for (int i = threadIdx.x; i < dd; i += 64)
        a.dst[i] = make_float2(float(c[2 * i] * scale), float(c[2 * i + 1] * scale));
}

// ---------------------------------------------------------------- batched

// A block on a state held in LDS: uniform values, in scalar registers.
struct ResidentGate {
    uint32_t head;
    uint32_t tab2[kMaxTileBits / 2];  // as in BatchTileGate
    const float2 *m;
    int sel;  // >= 0: a selection to make before the block
    __device__ __forceinline__ int k() const { return int(head & 7u); }
    // the matrix is the outcome of the last selection made
    __device__ __forceinline__ bool selected() const { return head & kSelectedGate; }
};

// The lane part of an MFMA gate's addresses: XOR of tab[] over the lane's
// group bits (logical bits nb..nb+3) and quarter bits (qb, qb+1).
__device__ __forceinline__ int lane_offset(const int *tab, int nb, int qb) {
    const int lane = threadIdx.x & 63;
    int v = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) v ^= ((lane >> b) & 1) ? tab[nb + b] : 0;
#pragma unroll
    for (int b = 0; b < 2; ++b) v ^= ((lane >> (4 + b)) & 1) ? tab[qb + b] : 0;
    return v;
}

// One block on a resident state.  For k <= 4, `lm` is the block's matrix in
// LDS, from which every lane forms its own MFMA operands (a 16- or 32-byte
// read and a few VALU operations: staging them as fragments first took a
// second barrier per block); for k = 5, `gm` is the global copy (two
// pointers, so that LDS reads compile to LDS instructions rather than flat
// ones, which would wait for every global load in flight).  `then` runs after
// the block's arithmetic and before the closing barrier.
// The MFMA paths need at least one 16-group batch per wavefront: M3 and M4 are
// the fewest bits they run at for k = 3 and 4 (10 and 11 at 512 work-items, 9
// and 10 at 256).
template <int NT, int M3, int M4, class Then>
__device__ __forceinline__ void resident_gate(float2 *__restrict__ sd, float2 *wide, const ResidentGate &g,
                                              const float2 *lm, int tb, Then then) {
    const int lane = threadIdx.x & 63;
    const int k = g.k();
    int lt[kMaxGateQubits], tab[kMaxTileBits];
#pragma unroll
    for (int j = 0; j < kMaxGateQubits; ++j) lt[j] = int((g.head >> (4 + 4 * j)) & 15u);
#pragma unroll
    for (int b = 0; b < kMaxTileBits; ++b) tab[b] = int((g.tab2[b >> 1] >> (16 * (b & 1))) & 0xffffu);
    if (k == 1) {
        tile_gate_small<1, SwizzledTile, NT, true>(sd, lm, lt, tab, tb);
    } else if (k == 2) {
        tile_gate_small<2, SwizzledTile, NT, true>(sd, lm, lt, tab, tb);
    } else if (k == 3 && tb >= M3) {
        // RealForm[l % 16][4 (l / 16) + s], s < 4: two entries of row (l % 16) / 2
        const float4 e = *reinterpret_cast<const float4 *>(lm + ((lane & 15) >> 1) * 8 + 2 * (lane >> 4));
        const bool im = lane & 1;
        const f32x4 afr = {im ? e.y : e.x, im ? e.x : -e.y, im ? e.w : e.z, im ? e.z : -e.w};
        tile_gate_mfma3<SwizzledTile, NT, true>(sd, afr, lane_offset(tab, 3, 1), tab, tb);
    } else if (k == 4 && tb >= M4) {
        const float4 *p = reinterpret_cast<const float4 *>(lm + (lane & 15) * 16 + 4 * (lane >> 4));
        const float4 e = p[0], f = p[1];
        const f32x4 fa = {e.x, e.z, f.x, f.z};
        const f32x4 fb = {-(e.x + e.y), -(e.z + e.w), -(f.x + f.y), -(f.z + f.w)};
        const f32x4 fs = {e.y - e.x, e.w - e.z, f.y - f.x, f.w - f.z};
        tile_gate_mfma4<SwizzledTile, NT>(sd, fa, fb, fs, lane_offset(tab, 4, 2), tab, tb);
    } else if (k == 3) {
        tile_gate_valu<3, SwizzledTile, NT>(sd, lm, lt, tb);
    } else if (k == 4) {
        tile_gate_valu<4, SwizzledTile, NT>(sd, lm, lt, tb);
    } else {
        for (int i = threadIdx.x; i < 1024; i += NT) wide[i] = g.m[i];
        __syncthreads();
        tile_gate_valu<5, SwizzledTile, NT>(sd, wide, lt, tb);
    }
    then();
    __syncthreads();
}

// Algorithm 2's fast path for a mixture of unitaries: the first i with
// r < pbar_i after subtracting the earlier pbar_j (FP64, in order); when
// rounding leaves r above the total, the last operator with weight.
__device__ __forceinline__ int draw_pick(const double *pb, int nk, double r) {
    for (int i = 0; i < nk; ++i) {
        if (r < pb[i]) return i;
        r -= pb[i];
    }
    for (int i = nk - 1; i >= 0; --i)
        if (pb[i] > 0.0) return i;
    return nk - 1;
}

// This work-item's entry of a k <= 4 matrix that is in memory (at most 256
// entries, one per work-item).
__device__ __forceinline__ bool resident_holds(const ResidentGate &g) {
    return g.k() <= 4 && !g.selected() && int(threadIdx.x) < (1 << (2 * g.k()));
}

// `count` blocks on the amplitudes in `sd`, software-pipelined so that no
// global-memory latency sits between two blocks: while block i runs, the
// matrix of block i + 1 travels into registers (and lands in the other half
// of the double-buffered LDS copy `raw` after block i's arithmetic) and the
// descriptor of block i + 2 is loaded.  Workgroup barriers on gfx950 do not
// wait for outstanding global loads, so both overlap the block's work.
// select(sel, dst) makes a selection on the state as it stands between two
// blocks and writes the matrix of a later block to dst (`chosen`; at most one
// is pending).
template <int NT, int M3, int M4, class Src, class Select>
__device__ __forceinline__ void resident_blocks(const Src &src, int count, float2 *__restrict__ sd, float2 *wide,
                                                float2 *raw, float2 *chosen, int tb, Select select) {
    if (count <= 0) return;
    ResidentGate cur = src.gate(0);
    if (resident_holds(cur)) raw[threadIdx.x] = cur.m[threadIdx.x];
    ResidentGate nxt = cur;
    if (count > 1) nxt = src.gate(1);
    __syncthreads();
    int buf = 0;
    for (int gi = 0; gi < count; ++gi) {
        if (cur.sel >= 0) select(cur.sel, chosen);
        const bool put1 = gi + 1 < count && resident_holds(nxt);
        float2 e1 = make_float2(0.f, 0.f);
        if (put1) e1 = nxt.m[threadIdx.x];
        ResidentGate after = nxt;
        if (gi + 2 < count) after = src.gate(gi + 2);
        float2 *next_raw = raw + 256 * (buf ^ 1);
        resident_gate<NT, M3, M4>(sd, wide, cur, cur.selected() ? chosen : raw + 256 * buf, tb, [&] {
            if (put1) next_raw[threadIdx.x] = e1;
        });
        cur = nxt;
        nxt = after;
        buf ^= 1;
    }
}

// The blocks of a batched job: the circuit's descriptors, each with its
// default matrix or the job's rebuilt copy.
struct BatchBlocks {
    const __attribute__((address_space(4))) BatchTileGate *g;
    const __attribute__((address_space(4))) BatchGate *b;
    const uint32_t *mask;
    const float2 *mats, *mine;
    __device__ __forceinline__ ResidentGate gate(int gi) const {
        ResidentGate r;
        r.head = g[gi].head;
#pragma unroll
        for (int j = 0; j < kMaxTileBits / 2; ++j) r.tab2[j] = g[gi].tab2[j];
        const int mat = b[gi].mat;
        const uint32_t word = __builtin_amdgcn_readfirstlane(mask[gi >> 5]);
        r.m = ((word >> (gi & 31)) & 1u) ? mine + mat : mats + mat;
        r.sel = -1;
        return r;
    }
};

// One operation (k qubits; block position of its bit b in bits 3b..3b+2 of
// `lpp`) on a column of a fused block's matrix, as the host's fusion does
// it: for each group, w_j = sum_l U[j][l] v_l in FP64 with the complex
// products and sums rounded one by one (no contraction into FMAs).
__device__ __forceinline__ int member_spread(int j, int k, int lpp) {
    int x = 0;
    for (int b = 0; b < k; ++b) x |= ((j >> b) & 1) << ((lpp >> (3 * b)) & 7);
    return x;
}

__device__ __forceinline__ int member_base(int grp, int opmask) {
    int base = 0, rest = grp;  // the group's bits, in order, at the positions the operation leaves free
    for (int p = 0; p < kMaxGateQubits; ++p)
        if (!((opmask >> p) & 1)) {
            base |= (rest & 1) << p;
            rest >>= 1;
        }
    return base;
}

// k <= 3: the group's v in registers, U an LDS copy.
template <int K>
__device__ __forceinline__ void fuse_member_small(double2 *col, int D, int lpp, const double2 *U) {
#pragma clang fp contract(off)
    constexpr int d = 1 << K;
    int opmask = 0, off[d];
#pragma unroll
    for (int b = 0; b < K; ++b) opmask |= 1 << ((lpp >> (3 * b)) & 7);
#pragma unroll
    for (int j = 0; j < d; ++j) off[j] = member_spread(j, K, lpp);
    for (int grp = 0; grp < (D >> K); ++grp) {
        const int base = member_base(grp, opmask);
        double2 v[d];
#pragma unroll
        for (int l = 0; l < d; ++l) v[l] = col[base + off[l]];
#pragma unroll
        for (int j = 0; j < d; ++j) {
            double sr = 0.0, si = 0.0;
#pragma unroll
            for (int l = 0; l < d; ++l) {
                const double2 u = U[j * d + l];
                const double pr = u.x * v[l].x - u.y * v[l].y;
                const double pi = u.x * v[l].y + u.y * v[l].x;
                sr = sr + pr;
                si = si + pi;
            }
            col[base + off[j]] = make_double2(sr, si);
        }
    }
}

// k = 4, 5 (a wide gate sharing a block with a channel): v from `old`, a
// copy of the column taken before the operation, U from global memory.
__device__ __forceinline__ void fuse_member_wide(double2 *col, double2 *old, int D, int k, int lpp,
                                                 const double2 *U) {
#pragma clang fp contract(off)
    const int d = 1 << k;
    for (int r = 0; r < D; ++r) old[r] = col[r];
    int opmask = 0;
    for (int b = 0; b < k; ++b) opmask |= 1 << ((lpp >> (3 * b)) & 7);
    for (int grp = 0; grp < (D >> k); ++grp) {
        const int base = member_base(grp, opmask);
        for (int j = 0; j < d; ++j) {
            double sr = 0.0, si = 0.0;
            for (int l = 0; l < d; ++l) {
                const double2 u = U[j * d + l];
                const double2 v = old[base + member_spread(l, k, lpp)];
                const double pr = u.x * v.x - u.y * v.y;
                const double pi = u.x * v.y + u.y * v.x;
                sr = sr + pr;
                si = si + pi;
            }
            col[base + member_spread(j, k, lpp)] = make_double2(sr, si);
        }
    }
}

// The matrix of block `rel` of the job's circuit with the job's picks, by
// one wavefront: each active lane carries one column of the product from
// the identity through the block's operations in order, in the wavefront's
// LDS workspace `ws` (1024 complex128: the column and its copy, so 32
// columns at a time for k <= 4 and 16 for k = 5; operators of up to 3
// qubits are staged in `ush`, 64 complex128), and writes it as complex64
// to the job's copy of the block's matrix.  Channel picks are drawn again
// (the same Philox call as the draw pass).
__device__ void fuse_patched(const BatchArgs &A, const BatchJob &J, const BatchCircuit &C,
                                             int rel, double2 *ws, double2 *ush, float2 *mine) {
    const BatchGate g = C.gates[rel];
    const int D = 1 << g.k;
    const int per_pass = D <= 16 ? D : 16;
    const int lane = int(threadIdx.x) & 63;
    double2 *col = ws + lane * D;
    double2 *old = ws + 512 + lane * D;
    for (int c0 = 0; c0 < D; c0 += per_pass) {
        const bool on = lane < per_pass;
        const int c = c0 + lane;
        if (on)
            for (int r = 0; r < D; ++r) col[r] = make_double2(r == c ? 1.0 : 0.0, 0.0);
        for (int m0 = g.m0; m0 < g.m1; m0 += 64) {
            // lane i resolves member m0 + i: width (0: an identity pick, left
            // out), positions, and where its operator lies.  One by one, each
            // member waited for four dependent loads and a draw (about 2 us).
            const int count = g.m1 - m0 < 64 ? g.m1 - m0 : 64;
            int mk = 0, mlpp = 0, moff = 0;
            if (lane < count) {
                const BatchMember M = C.members[m0 + lane];
                mk = M.k;
                moff = M.src;
                if (M.src < 0) {
                    const int ci = -M.src - 1;
                    const BatchChannel ch = C.chans[ci];
                    const int pick = draw_pick(C.pbar + ch.pbar, ch.nk,
                                               philox_uniform(J.seed, uint32_t(ci), J.traj, J.circ_id,
                                                              kStreamChannel));
                    moff = ch.unit + pick * (1 << (2 * M.k));
                    if ((ch.identity >> pick) & 1u) mk = 0;
                }
#pragma unroll
                for (int b = 0; b < kMaxGateQubits; ++b) mlpp |= (M.lp[b] & 7) << (3 * b);
            }
            // operators of up to three qubits travel one member ahead
            auto fetch = [&](int i) {
                const int k = __builtin_amdgcn_readlane(mk, i);
                const double2 *U = C.fmats + __builtin_amdgcn_readlane(moff, i);
                return k >= 1 && k <= 3 && lane < (1 << (2 * k)) ? U[lane] : make_double2(0.0, 0.0);
            };
            double2 u = fetch(0);
            for (int i = 0; i < count; ++i) {
                const int k = __builtin_amdgcn_readlane(mk, i), lpp = __builtin_amdgcn_readlane(mlpp, i);
                const double2 u_next = i + 1 < count ? fetch(i + 1) : u;
                if (k >= 1 && k <= 3) {
                    // the previous operator's reads precede these writes, and
                    // these writes precede the reads below
                    wave_lds_order();
                    if (lane < (1 << (2 * k))) ush[lane] = u;
                    wave_lds_order();
                    if (on) {
                        if (k == 1) fuse_member_small<1>(col, D, lpp, ush);
                        else if (k == 2) fuse_member_small<2>(col, D, lpp, ush);
                        else fuse_member_small<3>(col, D, lpp, ush);
                    }
                } else if (k > 3 && on) {
                    fuse_member_wide(col, old, D, k, lpp, C.fmats + __builtin_amdgcn_readlane(moff, i));
                }
                u = u_next;
            }
        }
        if (on) {
            float2 *dst = mine + g.mat;
            for (int r = 0; r < D; ++r) dst[r * D + c] = make_float2(float(col[r].x), float(col[r].y));
        }
    }
}

// The job's channel draws (one Philox call per channel, Algorithm 2's fast
// path), recorded when asked; a pick other than the default one flags its
// block in `mask`, and the flagged blocks' matrices are rebuilt with the
// job's picks into `mine`, one wavefront per block, by the first four
// wavefronts (LDS workspaces: 1024 + 64 complex128 each at ws4 and ush4).
// Ends with a workgroup barrier.
template <int NT>
__device__ __forceinline__ void draw_and_patch(const BatchArgs &A, const BatchJob &J, const BatchCircuit &C,
                                               uint32_t *mask, double2 *ws4, double2 *ush4, float2 *mine) {
    const int words = (C.n_gates + 31) >> 5;
    for (int w = threadIdx.x; w < words; w += NT) mask[w] = 0u;
    __syncthreads();
    for (int c = threadIdx.x; c < C.nch; c += NT) {
        const BatchChannel ch = C.chans[c];
        const int pick = draw_pick(C.pbar + ch.pbar, ch.nk,
                                   philox_uniform(J.seed, uint32_t(c), J.traj, J.circ_id, kStreamChannel));
        if (J.choices >= 0) A.choices[J.choices + c] = int8_t(pick);
        if (pick != ch.default_pick) atomicOr(&mask[ch.gate >> 5], 1u << (ch.gate & 31));
    }
    __syncthreads();
    const int wave = int(threadIdx.x) >> 6;
    double2 *ws = ws4 + wave * 1024;
    double2 *ush = ush4 + wave * 64;
    // the flagged blocks in turn to the four wavefronts, wherever they lie
    for (int w = 0, turn = 0; wave < 4 && w < words; ++w) {
        uint32_t bits = __builtin_amdgcn_readfirstlane(mask[w]);
        while (bits) {
            const int b = __builtin_ctz(bits);
            bits &= bits - 1u;
            if ((turn++ & 3) == wave) fuse_patched(A, J, C, 32 * w + b, ws, ush, mine);
        }
    }
    __syncthreads();
}

// Samples of a job's final state, amp(i) its amplitudes: inverse CDF over
// 256 contiguous chunks whose FP64 sums are scanned in a fixed order; readout
// flips as in sample_draw.  PIECE amplitudes are loaded at a time (16 for a
// state in global memory, so that a work-item's 128-byte line is one burst of
// independent loads; the order of the additions is the same for any PIECE,
// which divides the chunk length).  `part` is 256 doubles of LDS.
template <int NT, int PIECE, class Amp>
__device__ __forceinline__ void batched_sample(const BatchArgs &A, const BatchJob &J, const BatchCircuit &C,
                                               Amp amp, double *part) {
    const int n = C.n;
    const int dim = 1 << n;
    // chunk c = amplitudes [c*L, (c+1)*L), L = dim / 256 (>= 1), the same 256
    // chunks at either group size
    const int L = dim >= kBlock ? dim / kBlock : 1;
    const int chunks = dim >= kBlock ? kBlock : dim;
    double acc = 0.0;
    if (int(threadIdx.x) < chunks) {
        for (int i = 0; i < L; i += PIECE) {
            float2 v[PIECE];
#pragma unroll
            for (int j = 0; j < PIECE; ++j) v[j] = amp(int(threadIdx.x) * L + i + j);
#pragma unroll
            for (int j = 0; j < PIECE; ++j)
                acc = fma(double(v[j].x), double(v[j].x), fma(double(v[j].y), double(v[j].y), acc));
        }
    }
    if (int(threadIdx.x) < kBlock) part[threadIdx.x] = acc;
    __syncthreads();
    // inclusive prefix of the chunk sums by one wavefront: lane l sums
    // chunks 4l..4l+3 in order, the lanes' totals are scanned across
    // the wavefront, and chunk c's prefix is the lane's offset plus its
    // own running sum (a fixed order, so every launch rounds alike),
    // then made exactly non-decreasing by a running maximum (the two
    // summation orders can differ by an ulp where lanes meet)
    if (threadIdx.x < 64) {
        const int l = int(threadIdx.x);
        double p4[4];
        double run = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            run += 4 * l + i < chunks ? part[4 * l + i] : 0.0;
            p4[i] = run;
        }
        double t = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double u = __shfl_up(t, o);
            if (l >= o) t += u;
        }
        double off = __shfl_up(t, 1);
        if (l == 0) off = 0.0;
        double hi = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p4[i] = fmax(hi, off + p4[i]);
            hi = p4[i];
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double u = __shfl_up(hi, o);
            if (l >= o) hi = fmax(hi, u);
        }
        double below = __shfl_up(hi, 1);
        if (l == 0) below = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * l + i < chunks) part[4 * l + i] = fmax(below, p4[i]);
    }
    __syncthreads();
    const double N = part[chunks - 1];
    for (int smp = threadIdx.x; smp < C.n_samples; smp += NT) {
        const double target = philox_uniform(J.seed, uint32_t(smp), J.traj, J.circ_id, kStreamMeasure) * N;
        int lo = 0, hi = chunks;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (target < part[mid]) hi = mid; else lo = mid + 1;
        }
        uint32_t x;
        if (lo >= chunks) {
            x = uint32_t(dim - 1);
        } else {
            double run = lo > 0 ? part[lo - 1] : 0.0;
            int at = L - 1;
            for (int i = 0; i < L; i += PIECE) {
                float2 v[PIECE];
#pragma unroll
                for (int j = 0; j < PIECE; ++j) v[j] = amp(lo * L + i + j);
                int found = -1;
#pragma unroll
                for (int j = 0; j < PIECE; ++j) {
                    run += fma(double(v[j].x), double(v[j].x), double(v[j].y) * double(v[j].y));
                    if (found < 0 && target < run) found = i + j;
                }
                if (found >= 0) {
                    at = found;
                    break;
                }
            }
            x = uint32_t(lo * L + at);
        }
        if (C.readout >= 0) {
            const double *e0 = A.readout + C.readout;
            const double *e1 = e0 + n;
            for (int q = 0; q < n; ++q) {
                const int bit = int((x >> q) & 1u);
                const double u = philox_uniform(J.seed, uint32_t(smp * n + q), J.traj, J.circ_id,
                                                kStreamReadout);
                if (u < (bit ? e1[q] : e0[q])) x ^= 1u << q;
            }
        }
        A.out[J.out + smp] = x;
    }
}

// Persistent launch over the jobs whose state fits in LDS (n <=
// kBatchLdsQubits): each workgroup takes jobs blockIdx.x, + gridDim.x, ...
// A job is one trajectory: its channels are drawn, the blocks its picks
// change are rebuilt, the state starts as |0...0>, the circuit's blocks run
// with the job's matrices, and the workgroup samples the final state.
// The workgroup's own global stores (the rebuilt matrices) are read back
// only by its own wavefronts, which share one CU and its L1: the barriers'
// workgroup-scope ordering suffices, and no device-scope fence (an L2
// write-back and invalidate on gfx950) is needed.
template <int NT>
__global__ __launch_bounds__(NT) void run_batched(BatchArgs A) {
    alignas(16) extern __shared__ float2 smem[];
    QS_LDS_VECTORS(smem);
    float2 *sd = smem;                                                   // 2^13 amplitudes
    float2 *wide = smem + (1 << kBatchLdsQubits);                        // a 5-qubit block's matrix
    float2 *raw = smem + (1 << kBatchLdsQubits) + 1024;                  // 2 x 256 entries
    __shared__ double part[kBlock];
    float2 *mine = A.patched + size_t(blockIdx.x) * size_t(A.patched_stride);
    uint32_t *mask = reinterpret_cast<uint32_t *>(part);  // blocks the job's picks change
    for (int job = blockIdx.x; job < A.n_jobs; job += gridDim.x) {
        const BatchJob J = A.jobs[job];
        const BatchCircuit C = A.circs[J.circuit];
        const int dim = 1 << C.n;
        draw_and_patch<NT>(A, J, C, mask, reinterpret_cast<double2 *>(sd), reinterpret_cast<double2 *>(raw), mine);
        for (int i = threadIdx.x; i < dim; i += NT) sd[i] = make_float2(i == 0 ? 1.f : 0.f, 0.f);
        __syncthreads();
        BatchBlocks src;
        src.g = (const __attribute__((address_space(4))) BatchTileGate *)(C.tile_gates);
        src.b = (const __attribute__((address_space(4))) BatchGate *)(C.gates);
        src.mask = mask;
        src.mats = C.mats;
        src.mine = mine;
        // the same MFMA rule at either group size: a job's arithmetic does not
        // depend on the launch it runs in
        resident_blocks<NT, 10, 11>(src, C.n_gates, sd, wide, raw, raw, C.n, [](int, float2 *) {});
        batched_sample<NT, 1>(A, J, C, [&](int i) { return sd[SwizzledTile::map(i)]; }, part);
        __syncthreads();
    }
}

// ---- jobs of n > kBatchLdsQubits
// One workgroup per such job would leave most of the GPU waiting for the
// widest ones (an 18-qubit, 40-cycle trajectory alone took 45 ms), so their
// sweeps are launches over all jobs of a wave at once: launch s applies
// sweep s of every job that has one, a workgroup per one or two tiles of one
// job, with the tile sweep of apply_tile (FP32 MFMA and the LDS round trips
// of its blocks bound it, as there).  What a sweep applies, and in which
// order, is fixed by the circuit's plan, so a job's state does not depend on
// the jobs beside it.  64 circuits of 12..18 qubits x 16 trajectories: 51 ms
// with a workgroup per job, 5.7 ms like this (5.3 ms of it sweeps).

// Per job of the wave: draws, rebuilt matrices, and the table of the job's
// block matrices (default or rebuilt) its sweeps read.
__global__ __launch_bounds__(kBlock) void batch_prepare(BatchArgs A, int job0) {
    alignas(16) extern __shared__ float2 smem[];  // 4 x (1024 + 64) complex128
    QS_LDS_VECTORS(smem);
    __shared__ uint32_t mask[kBatchMaxBlocks / 32];
    const BatchJob J = A.jobs[job0 + int(blockIdx.x)];
    const BatchCircuit C = A.circs[J.circuit];
    float2 *mine = A.patched + J.mine;
    double2 *ws = reinterpret_cast<double2 *>(smem);
    draw_and_patch<kBlock>(A, J, C, mask, ws, ws + 4 * 1024, mine);
    for (int gi = threadIdx.x; gi < C.n_gates; gi += kBlock) {
        const int mat = C.gates[gi].mat;
        const bool patched = (mask[gi >> 5] >> (gi & 31)) & 1u;
        A.mptr[J.mptr + gi] = patched ? mine + mat : C.mats + mat;
    }
}

// A job's sweep in device tables; uniform, so read through the constant
// address space (scalar loads).
struct JobSweep {
    const __attribute__((address_space(4))) BatchSweep *s;
    const __attribute__((address_space(4))) BatchTileGate *g;  // the sweep's first gate
    const __attribute__((address_space(4))) uint64_t *m;   // its matrices' addresses
    int zero;
    __device__ __forceinline__ int pos(int b) const { return s->pos[b]; }
    __device__ __forceinline__ int n_gates() const { return s->g1 - s->g0; }
    __device__ __forceinline__ int init_zero() const { return zero; }
    __device__ __forceinline__ int rdm_lt() const { return 0; }
    __device__ __forceinline__ double *rdm_out() const { return nullptr; }
    __device__ __forceinline__ int k(int gi) const { return int(g[gi].head & 7u); }
    __device__ __forceinline__ int lt(int gi, int b) const { return int((g[gi].head >> (4 + 4 * b)) & 15u); }
    __device__ __forceinline__ int lofs(int gi) const { return g[gi].lofs; }
    __device__ __forceinline__ int tab(int gi, int b) const { return int((g[gi].tab2[b >> 1] >> (16 * (b & 1))) & 0xffffu); }
    __device__ __forceinline__ const float2 *mat(int gi) const { return reinterpret_cast<const float2 *>(m[gi]); }
};

template <bool K5>
__global__ __launch_bounds__(kBatchWideThreads) void batch_sweep(BatchArgs A, const BatchPart *parts, int step) {
    __shared__ float2 sd[1 << kBatchTileBits];
    alignas(16) extern __shared__ float2 sm[];
    QS_LDS_VECTORS(sm);
    typedef const __attribute__((address_space(4))) BatchPart *Parts;
    typedef const __attribute__((address_space(4))) BatchJob *Jobs;
    typedef const __attribute__((address_space(4))) BatchCircuit *Circs;
    typedef const __attribute__((address_space(4))) BatchSweep *Sweeps;
    typedef const __attribute__((address_space(4))) BatchTileGate *Gates;
    typedef const __attribute__((address_space(4))) uint64_t *Words;
    const Parts P = (Parts)(parts) + blockIdx.x;
    const Jobs J = (Jobs)(A.jobs) + P->job;
    const Circs C = (Circs)(A.circs) + J->circuit;
    JobSweep src;
    src.s = (Sweeps)(C->sweeps) + step;
    src.g = (Gates)(C->tile_gates) + src.s->g0;
    src.m = (Words)(A.mptr) + J->mptr + src.s->g0;
    src.zero = step == 0 ? 1 : 0;
    tile_sweep<kBatchTileBits, uint32_t, K5, kBatchWideThreads, false, true, false>(
        A.slots + J->slot, uint32_t(P->tile0), 1u, uint32_t(P->tile0 + P->tiles), src, sd, sm);
}

__global__ __launch_bounds__(kBlock) void batch_sample(BatchArgs A, int job0) {
    __shared__ double part[kBlock];
    const BatchJob J = A.jobs[job0 + int(blockIdx.x)];
    const BatchCircuit C = A.circs[J.circuit];
    const float2 *p = A.slots + J.slot;
    batched_sample<kBlock, 16>(A, J, C, [p](int i) { return p[i]; }, part);
}

// ---------------------------------------------------------------- trajectories side by side

// A resident trajectory's blocks.
struct TrajBlocks {
    const __attribute__((address_space(4))) TrajGate *g;
    __device__ __forceinline__ ResidentGate gate(int gi) const {
        ResidentGate r;
        r.head = g[gi].g.head;
#pragma unroll
        for (int j = 0; j < kMaxTileBits / 2; ++j) r.tab2[j] = g[gi].g.tab2[j];
        r.m = (const float2 *)(g[gi].m);
        r.sel = g[gi].sel;
        return r;
    }
};

// R of K ascending qubits of a resident state, summed over the workgroup in a
// fixed order into red[0 .. 2 D D) (LDS; ends with a barrier).
template <int K, int NT>
__device__ __forceinline__ void resident_rdm(const float2 *sd, int n, const int *t, double *red) {
    constexpr int D = 1 << K;
    constexpr int T = D * D;  // as in rdm_partials
    double acc[T];
#pragma unroll
    for (int w = 0; w < T; ++w) acc[w] = 0.0;
    for (int g = threadIdx.x; g < (1 << (n - K)); g += NT) {
        const int base = spread_index<K, int>(g, t);
        double vr[D], vi[D];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float2 v = sd[SwizzledTile::map(base | local_offset<K, int>(j, t))];
            vr[j] = v.x;
            vi[j] = v.y;
        }
        int w = D;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            acc[j] = fma(vr[j], vr[j], fma(vi[j], vi[j], acc[j]));
#pragma unroll
            for (int l = j + 1; l < D; ++l, w += 2) {
                acc[w] = fma(vr[j], vr[l], fma(vi[j], vi[l], acc[w]));
                acc[w + 1] = fma(vi[j], vr[l], fma(-vr[j], vi[l], acc[w + 1]));
            }
        }
    }
#pragma unroll
    for (int w = 0; w < T; ++w) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc[w] += __shfl_xor(acc[w], off, 64);
    }
    double *part = red + 32;  // [wavefront][T]
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int w = 0; w < T; ++w) part[(threadIdx.x >> 6) * T + w] = acc[w];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum[T];
#pragma unroll
        for (int w = 0; w < T; ++w) {
            double x = 0.0;
            for (int i = 0; i < NT / 64; ++i) x += part[i * T + w];
            sum[w] = x;
        }
        int w = D;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            red[2 * (j * D + j)] = sum[j];
            red[2 * (j * D + j) + 1] = 0.0;
#pragma unroll
            for (int l = j + 1; l < D; ++l, w += 2) {
                red[2 * (j * D + l)] = sum[w];
                red[2 * (j * D + l) + 1] = sum[w + 1];
                red[2 * (l * D + j)] = sum[w];
                red[2 * (l * D + j) + 1] = -sum[w + 1];
            }
        }
    }
}

// One trajectory per workgroup, its state in LDS from |0...0> to the end: the
// blocks in launch order, each selection where its channel stands in the
// circuit (between the blocks of the operations before it and after it).
// Bound by the chain of blocks on one CU (LDS round trip, barrier, a few MFMAs
// each: about 1 us), so a call's trajectories run side by side on as many CUs.
template <int NT, int M3, int M4>
__global__ __launch_bounds__(NT) void run_resident(TrajResidentArgs A) {
    alignas(16) extern __shared__ float2 smem[];
    QS_LDS_VECTORS(smem);
    float2 *sd = smem;                    // 2^n amplitudes
    float2 *wide = smem + (1 << A.n);     // a 5-qubit block's matrix
    float2 *raw = wide + 1024;            // 2 x 256 entries
    float2 *chosen = raw + 512;           // a selection's matrix
    __shared__ double red[32 + 16 * (NT / 64)];
    __shared__ double scale;
    __shared__ int pick;
    const TrajJob J = A.jobs[blockIdx.x];
    for (int i = threadIdx.x; i < (1 << A.n); i += NT) sd[i] = make_float2(i == 0 ? 1.f : 0.f, 0.f);
    __syncthreads();
    TrajBlocks src;
    src.g = (const __attribute__((address_space(4))) TrajGate *)(A.gates) + J.g0;
    resident_blocks<NT, M3, M4>(src, J.n_gates, sd, wide, raw, chosen, A.n, [&](int sel, float2 *dst) {
        const TrajSelect S = A.sels[sel];
        if (S.k == 1) resident_rdm<1, NT>(sd, A.n, S.t, red);
        else resident_rdm<2, NT>(sd, A.n, S.t, red);
        if (threadIdx.x == 0) {  // the work-item that wrote `red`
            pick_branch(red, 1 << S.k, S.excess, S.pbar, S.nk, S.resid, S.err, &pick, &scale);
            *S.choice = pick;
        }
        __syncthreads();
        const int dd = S.Db * S.Db;  // at most 256
        const double *c = S.cand + size_t(pick) * dd * 2;
        if (int(threadIdx.x) < dd)
            dst[threadIdx.x] =
                make_float2(float(c[2 * threadIdx.x] * scale), float(c[2 * threadIdx.x + 1] * scale));
        __syncthreads();
    });
    if (J.out)
        for (int i = threadIdx.x; i < (1 << A.n); i += NT) J.out[i] = sd[SwizzledTile::map(i)];
}

// A sweep of one trajectory, in device tables.
struct TrajSweepSrc {
    const __attribute__((address_space(4))) TrajSweep *s;
    const __attribute__((address_space(4))) TrajGate *g;  // the sweep's first gate
    __device__ __forceinline__ int pos(int b) const { return s->pos[b]; }
    __device__ __forceinline__ int n_gates() const { return s->n_gates; }
    __device__ __forceinline__ int init_zero() const { return s->init_zero; }
    __device__ __forceinline__ int rdm_lt() const { return s->rdm_lt; }
    __device__ __forceinline__ double *rdm_out() const { return (double *)(s->rdm_out); }
    __device__ __forceinline__ int k(int gi) const { return int(g[gi].g.head & 7u); }
    __device__ __forceinline__ int lt(int gi, int b) const { return int((g[gi].g.head >> (4 + 4 * b)) & 15u); }
    __device__ __forceinline__ int lofs(int gi) const { return g[gi].g.lofs; }
    __device__ __forceinline__ int tab(int gi, int b) const {
        return int((g[gi].g.tab2[b >> 1] >> (16 * (b & 1))) & 0xffffu);
    }
    __device__ __forceinline__ const float2 *mat(int gi) const { return (const float2 *)(g[gi].m); }
};

// Step of several trajectories: workgroup (x, y) takes tiles x, x + gridDim.x,
// ... of sweep y.  One trajectory of 14..21 qubits has 2 to 256 tiles for 512
// workgroup slots and a sweep of it takes 12 to 20 us whatever its size, so
// the sweeps of several trajectories share a launch.
template <int NT>
__global__ __launch_bounds__(NT, 4) void traj_sweep(const TrajSweep *sweeps, const TrajGate *gates,
                                                    uint32_t n_tiles) {
    __shared__ float2 sd[1 << kBatchTileBits];
    alignas(16) extern __shared__ float2 sm[];
    QS_LDS_VECTORS(sm);
    TrajSweepSrc src;
    src.s = (const __attribute__((address_space(4))) TrajSweep *)(sweeps) + blockIdx.y;
    src.g = (const __attribute__((address_space(4))) TrajGate *)(gates) + src.s->g0;
    tile_sweep<kBatchTileBits, uint32_t, false, NT, true, true, true>(
        (float2 *)(src.s->amp), blockIdx.x, gridDim.x, n_tiles, src, sd, sm);
}

// A step's selections, one wavefront each: the sweep's workgroup records are
// summed in a fixed order, then as select_branch.
__global__ __launch_bounds__(64) void traj_select(const TrajSelect *sels) {
    __shared__ double red[8];
    __shared__ double scale;
    __shared__ int pick;
    const TrajSelect S = sels[blockIdx.x];
    double acc[8];
#pragma unroll
    for (int w = 0; w < 8; ++w) acc[w] = 0.0;
    for (int i = threadIdx.x; i < S.n_records; i += 64) {
#pragma unroll
        for (int w = 0; w < 8; ++w) acc[w] += S.records[size_t(i) * 8 + w];
    }
#pragma unroll
    for (int w = 0; w < 8; ++w) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc[w] += __shfl_xor(acc[w], off, 64);
        if (threadIdx.x == 0) red[w] = acc[w];
    }
    if (threadIdx.x == 0) {
        pick_branch(red, 2, S.excess, S.pbar, S.nk, S.resid, S.err, &pick, &scale);
        *S.choice = pick;
    }
    __syncthreads();
    const int dd = S.Db * S.Db;
    const double *c = S.cand + size_t(pick) * dd * 2;
    for (int i = threadIdx.x; i < dd; i += 64)
        S.dst[i] = make_float2(float(c[2 * i] * scale), float(c[2 * i + 1] * scale));
}

// ---------------------------------------------------------------- utility

template <typename Idx>
__global__ __launch_bounds__(kBlock) void set_basis(float2 *__restrict__ amp, Idx dim, Idx index) {
    const Idx stride = Idx(gridDim.x) * Idx(kBlock);
    for (Idx i = Idx(blockIdx.x) * Idx(kBlock) + Idx(threadIdx.x); i < dim; i += stride)
        amp[i] = make_float2(i == index ? 1.f : 0.f, 0.f);
}

// A state copy: pairs of amplitudes as 16-byte loads and stores, over a
// grid of four 256-work-item groups per CU (the shape that copied a 2 GiB
// state fastest in a sweep of grids and unrolling).
__global__ __launch_bounds__(kBlock) void copy_pairs(float4 *__restrict__ dst, const float4 *__restrict__ src,
                                                     int64_t pairs) {
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < pairs; i += stride) dst[i] = src[i];
}

template <typename Idx>
__global__ __launch_bounds__(kBlock) void scale_state(float2 *__restrict__ amp, Idx dim, float s) {
    const Idx stride = Idx(gridDim.x) * Idx(kBlock);
    for (Idx i = Idx(blockIdx.x) * Idx(kBlock) + Idx(threadIdx.x); i < dim; i += stride) {
        float2 v = amp[i];
        amp[i] = make_float2(v.x * s, v.y * s);
    }
}

// ---------------------------------------------------------------- reductions

// Fixed-order workgroup sum of W per-thread values; thread 0 writes them.
template <int W>
__device__ __forceinline__ void block_sum_write(double (&vals)[W], double *__restrict__ dst) {
    __shared__ double red[kBlock / 64][W];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        double x = vals[w];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
        vals[w] = x;
    }
    if (lane == 0) {
#pragma unroll
        for (int w = 0; w < W; ++w) red[wave][w] = vals[w];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            double s = red[0][w];
#pragma unroll
            for (int i = 1; i < kBlock / 64; ++i) s += red[i][w];
            dst[w] = s;
        }
    }
}

template <typename Idx>
__global__ __launch_bounds__(kBlock) void norm_partials(const float2 *__restrict__ amp, Idx dim,
                                                        double *__restrict__ partials) {
    double acc[1] = {0.0};
    const Idx stride = Idx(gridDim.x) * Idx(kBlock);
    for (Idx i = Idx(blockIdx.x) * Idx(kBlock) + Idx(threadIdx.x); i < dim; i += stride) {
        const float2 v = amp[i];
        const double re = v.x, im = v.y;
        acc[0] = fma(re, re, fma(im, im, acc[0]));
    }
    block_sum_write<1>(acc, partials + blockIdx.x);
}

// R = sum v v^dag is Hermitian, so only its upper triangle is summed (D real
// and D (D - 1) / 2 complex entries: 16 accumulators instead of 32 for two
// qubits, half the FP64 work) and the record is completed from it.  HBM-bound
// (two qubits, 26 qubits: 107 us with the full matrix, 94 with the triangle;
// the one-qubit pass takes 87).
template <int K, typename Idx>
__global__ __launch_bounds__(kBlock) void rdm_partials(const float2 *__restrict__ amp, Idx groups,
                                                       TargetArgs ta,
                                                       double *__restrict__ partials) {
    constexpr int D = 1 << K;
    constexpr int T = D * D;  // packed: diagonal entries, then (re, im) of j < l in row order
    double acc[T];
#pragma unroll
    for (int w = 0; w < T; ++w) acc[w] = 0.0;
    const Idx stride = Idx(gridDim.x) * Idx(kBlock);
    for (Idx g = Idx(blockIdx.x) * Idx(kBlock) + Idx(threadIdx.x); g < groups; g += stride) {
        const Idx base = spread_index<K, Idx>(g, ta.t);
        double vr[D], vi[D];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float2 v = amp[base + local_offset<K, Idx>(j, ta.t)];
            vr[j] = v.x;
            vi[j] = v.y;
        }
        // R[j][l] += v_j conj(v_l)
        int w = D;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            acc[j] = fma(vr[j], vr[j], fma(vi[j], vi[j], acc[j]));
#pragma unroll
            for (int l = j + 1; l < D; ++l, w += 2) {
                acc[w] = fma(vr[j], vr[l], fma(vi[j], vi[l], acc[w]));
                acc[w + 1] = fma(vi[j], vr[l], fma(-vr[j], vi[l], acc[w + 1]));
            }
        }
    }
    __shared__ double sum[T];
    block_sum_write<T>(acc, sum);
    if (threadIdx.x == 0) {  // the work-item that wrote `sum`
        double *rec = partials + size_t(blockIdx.x) * (2 * D * D);
        int w = D;
        for (int j = 0; j < D; ++j) {
            rec[2 * (j * D + j)] = sum[j];
            rec[2 * (j * D + j) + 1] = 0.0;
            for (int l = j + 1; l < D; ++l, w += 2) {
                rec[2 * (j * D + l)] = sum[w];
                rec[2 * (j * D + l) + 1] = sum[w + 1];
                rec[2 * (l * D + j)] = sum[w];
                rec[2 * (l * D + j) + 1] = -sum[w + 1];
            }
        }
    }
}

template <int K, typename Idx>
__global__ __launch_bounds__(kBlock) void apply_copy_norm(const float2 *__restrict__ in,
                                                          float2 *__restrict__ out, Idx groups,
                                                          GateArgs<K> a,
                                                          double *__restrict__ partials) {
    constexpr int D = 1 << K;
    double acc[2] = {0.0, 0.0};
    const Idx stride = Idx(gridDim.x) * Idx(kBlock);
    for (Idx g = Idx(blockIdx.x) * Idx(kBlock) + Idx(threadIdx.x); g < groups; g += stride) {
        const Idx base = spread_index<K, Idx>(g, a.t);
        float2 v[D];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            v[j] = in[base + local_offset<K, Idx>(j, a.t)];
            acc[1] = fma(double(v[j].x), double(v[j].x), fma(double(v[j].y), double(v[j].y), acc[1]));
        }
#pragma unroll
        for (int j = 0; j < D; ++j) {
            float2 w = make_float2(0.f, 0.f);
#pragma unroll
            for (int l = 0; l < D; ++l) w = cmac(w, a.m[j * D + l], v[l]);
            out[base + local_offset<K, Idx>(j, a.t)] = w;
            acc[0] = fma(double(w.x), double(w.x), fma(double(w.y), double(w.y), acc[0]));
        }
    }
    block_sum_write<2>(acc, partials + size_t(blockIdx.x) * 2);
}

// Per-qubit weights (see launch_zweights).  Workgroup w owns the contiguous
// chunk [w 2^c, (w + 1) 2^c).  HBM-bound: a work-item adds fewer than two FP64
// sums per amplitude where one conditional sum per qubit took ten (26 qubits:
// 412 us before, 93 now, 5.8 TB/s).
//
// Chunks of 2^12 and more: in step o of 2^(c - 12), work-item t reads the
// eight pairs x = chunk + 4096 o + 512 r + 2 t + {0, 1} as 16-byte loads, so
// bit 0 of x is the pair's half, bits 1..8 come from t, 9..11 from r and the
// rest from o and the chunk (uniform).  The eight pairs are summed as a tree
// whose inner nodes give the bit 9..11 sums; the step's total joins the sum
// of every bit set in o.
constexpr int kZStepBits = 12;
constexpr int kZOuterBits = 12;  // o has c - 12 bits
constexpr int kZSums = 1 + kZStepBits + kZOuterBits;
template <typename Idx>
__global__ __launch_bounds__(kBlock) void zweight_partials(const float2 *__restrict__ amp, int n, int c,
                                                           double *__restrict__ partials) {
    const int t = threadIdx.x;
    const int obits = c - kZStepBits;
    const Idx chunk = Idx(blockIdx.x) << c;
    // s[0]: total; s[1 + q]: the chunk's sum over bit q set, q < c
    double s[kZSums];
#pragma unroll
    for (int w = 0; w < kZSums; ++w) s[w] = 0.0;
    for (uint32_t o = 0; o < (uint32_t(1) << obits); ++o) {
        const float4 *p4 = reinterpret_cast<const float4 *>(amp + chunk + (Idx(o) << kZStepBits)) + t;
        float4 v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = p4[r * kBlock];
        double p[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const double lo = fma(double(v[r].x), double(v[r].x), double(v[r].y) * double(v[r].y));
            const double hi = fma(double(v[r].z), double(v[r].z), double(v[r].w) * double(v[r].w));
            s[1] += hi;
            p[r] = lo + hi;
        }
        const double a0 = p[0] + p[1], a1 = p[2] + p[3], a2 = p[4] + p[5], a3 = p[6] + p[7];
        const double b1 = a2 + a3;
        const double all = (a0 + a1) + b1;
        s[10] += (p[1] + p[3]) + (p[5] + p[7]);
        s[11] += a1 + a3;
        s[12] += b1;
        s[0] += all;
#pragma unroll
        for (int j = 0; j < kZOuterBits; ++j)
            if (j < obits && ((o >> j) & 1)) s[1 + kZStepBits + j] += all;
    }
#pragma unroll
    for (int q = 1; q < 9; ++q) s[1 + q] = ((t >> (q - 1)) & 1) ? s[0] : 0.0;
    __shared__ double sum[kZSums];
    block_sum_write<kZSums>(s, sum);
    if (t == 0) {  // the work-item that wrote `sum`
        double *rec = partials + size_t(blockIdx.x) * kZRecord;
        rec[0] = sum[0];
        for (int q = 0; q < kZRecord - 1; ++q) {
            double x = 0.0;
            if (q < c) x = sum[1 + q];
            else if (q < n) x = ((chunk >> q) & 1) ? sum[0] : 0.0;
            rec[1 + q] = x;
        }
    }
}

// States below 2^12 amplitudes: one workgroup, work-item t takes x = t, t +
// 256, ...
__global__ __launch_bounds__(kBlock) void zweight_small(const float2 *__restrict__ amp, int n,
                                                        double *__restrict__ out) {
    double vals[1 + kZStepBits];
#pragma unroll
    for (int w = 0; w <= kZStepBits; ++w) vals[w] = 0.0;
    for (int x = threadIdx.x; x < (1 << n); x += kBlock) {
        const float2 v = amp[x];
        const double p = fma(double(v.x), double(v.x), double(v.y) * double(v.y));
        vals[0] += p;
#pragma unroll
        for (int q = 0; q < kZStepBits; ++q) vals[1 + q] += ((x >> q) & 1) ? p : 0.0;
    }
    block_sum_write<1 + kZStepBits>(vals, out);
    for (int q = 1 + kZStepBits + int(threadIdx.x); q < kZRecord; q += kBlock) out[q] = 0.0;
}

// Sum `count` records of `width` doubles in a fixed order: workgroup w sums
// entry w (one workgroup walking the entries took 2 us for each: 105 us for
// 2048 Z-weight records, now 5).
__global__ __launch_bounds__(kBlock) void reduce_records(const double *__restrict__ partials,
                                                         int count, int width,
                                                         double *__restrict__ out) {
    __shared__ double red[kBlock];
    const int w = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < count; i += kBlock) s += partials[size_t(i) * width + w];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = kBlock / 2; h >= 1; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[w] = red[0];
}

// ---------------------------------------------------------------- sampling

// Per-lane sum of |amp|^2 over `per` consecutive amplitudes starting at
// `first`, in index order (pairs loaded as one 16-byte access).
template <typename Idx>
__device__ __forceinline__ double chunk_weight(const float2 *__restrict__ amp, Idx first, int per) {
    double acc = 0.0;
    if (per >= 2) {
        const float4 *p4 = reinterpret_cast<const float4 *>(amp + first);
        for (int i = 0; i < per / 2; ++i) {
            const float4 v = p4[i];
            acc = fma(double(v.x), double(v.x), fma(double(v.y), double(v.y), acc));
            acc = fma(double(v.z), double(v.z), fma(double(v.w), double(v.w), acc));
        }
    } else {
        const float2 v = amp[first];
        acc = fma(double(v.x), double(v.x), double(v.y) * double(v.y));
    }
    return acc;
}

// One wavefront per sampling block of 2^B amplitudes (kBlock / 64 blocks per
// workgroup): the lanes read the block coalesced (lane j takes pairs j,
// j + 64, ... as 16-byte loads) and add in that fixed order, then a fixed
// shuffle tree adds the lanes.
template <typename Idx>
__global__ __launch_bounds__(kBlock) void sample_block_sums(const float2 *__restrict__ amp, int B,
                                                            int64_t nb, double *__restrict__ sums) {
    const int64_t blk = int64_t(blockIdx.x) * (kBlock / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (blk >= nb) return;  // uniform over the wavefront
    const int len = 1 << B;
    const Idx first = Idx(blk) << B;
    double x = 0.0;
    if (len >= 128) {
        const float4 *p4 = reinterpret_cast<const float4 *>(amp + first);
#pragma unroll 8
        for (int i = lane; i < len / 2; i += 64) {
            const float4 v = p4[i];
            x = fma(double(v.x), double(v.x), fma(double(v.y), double(v.y), x));
            x = fma(double(v.z), double(v.z), fma(double(v.w), double(v.w), x));
        }
    } else {
        for (int i = lane; i < len; i += 64) {
            const float2 v = amp[first + Idx(i)];
            x = fma(double(v.x), double(v.x), fma(double(v.y), double(v.y), x));
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    if (lane == 0) sums[blk] = x;
}

// Inclusive prefix of the block sums in index order, in three fixed-order
// steps: every tile of kScanThreads * kScanPer sums is scanned by its own
// workgroup; one workgroup scans the tile totals into exclusive tile offsets
// (written over the block sums, which are no longer needed) and the total;
// the offsets are added to the tiles after the first.
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 8;
constexpr int kScanTile = kScanThreads * kScanPer;
__device__ __forceinline__ double wave_inclusive_scan(double x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Exclusive prefix over the workgroup's kScanThreads values in thread order
// (wavefront scans, then the wavefront totals in order); *all gets the total.
__device__ __forceinline__ double workgroup_exclusive_scan(double x, double *wave_tot, double *all) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double inc = wave_inclusive_scan(x);
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    double before = 0.0, sum = 0.0;
    for (int w = 0; w < kScanThreads / 64; ++w) {
        if (w < wave) before += wave_tot[w];
        sum += wave_tot[w];
    }
    *all = sum;
    return before + (inc - x);
}

// A tile is loaded coalesced into LDS (one pad slot per kScanPer, so each
// work-item's run of kScanPer consecutive sums sits on distinct banks), each
// work-item adds its run, the runs' offsets come from one workgroup scan,
// and the runs' prefixes go back through LDS and out coalesced.
__device__ __forceinline__ int scan_slot(int i) { return i + i / kScanPer; }

__global__ __launch_bounds__(kScanThreads) void sample_scan_tiles(const double *__restrict__ sums,
                                                                  int64_t nb, double *__restrict__ incl,
                                                                  double *norm, double *norm_host) {
    __shared__ double tile[kScanTile + kScanTile / kScanPer];
    __shared__ double wave_tot[kScanThreads / 64];
    const int t = threadIdx.x;
    const int64_t base = int64_t(blockIdx.x) * kScanTile;
    const int len = nb - base < kScanTile ? int(nb - base) : kScanTile;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        const int i = j * kScanThreads + t;
        tile[scan_slot(i)] = i < len ? sums[base + i] : 0.0;
    }
    __syncthreads();
    double v[kScanPer], tot = 0.0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        v[j] = tile[scan_slot(t * kScanPer + j)];
        tot += v[j];
    }
    double all;
    double run = workgroup_exclusive_scan(tot, wave_tot, &all);
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        run += v[j];
        tile[scan_slot(t * kScanPer + j)] = run;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        const int i = j * kScanThreads + t;
        if (i < len) incl[base + i] = tile[scan_slot(i)];
    }
    if (norm && t == 0) {  // the only tile: its last prefix is the norm
        *norm = tile[scan_slot(len - 1)];
        if (norm_host) *norm_host = tile[scan_slot(len - 1)];
    }
}

// Tile totals (each tile's last prefix) added one after another: offsets[t]
// is the running sum before tile t, so that a tile's last prefix plus its
// offset equals the next offset exactly and the prefix stays non-decreasing
// across tiles.  *norm is the final sum.
constexpr int kScanMaxTiles = 2048;  // 2^(kMaxQubits - kSampleBlockBits) / kScanTile
__global__ __launch_bounds__(kScanThreads) void sample_scan_offsets(const double *__restrict__ incl,
                                                                    int64_t nb, int n_tiles,
                                                                    double *__restrict__ offsets,
                                                                    double *__restrict__ norm,
                                                                    double *norm_host) {
    __shared__ double tot[kScanMaxTiles];
    for (int t = threadIdx.x; t < n_tiles; t += kScanThreads) {
        const int64_t end = int64_t(t + 1) * kScanTile;
        tot[t] = incl[(end < nb ? end : nb) - 1];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double run = 0.0;
        for (int t0 = 0; t0 < n_tiles; t0 += 16) {
            double v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = t0 + j < n_tiles ? tot[t0 + j] : 0.0;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (t0 + j < n_tiles) {
                    offsets[t0 + j] = run;
                    run += v[j];
                }
        }
        *norm = run;
        if (norm_host) *norm_host = run;
    }
}

__global__ __launch_bounds__(kBlock) void sample_scan_add(double *__restrict__ incl, int64_t nb,
                                                          const double *__restrict__ offsets) {
    const int64_t i = int64_t(kScanTile) + int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < nb) incl[i] += offsets[i / kScanTile];
}

// One wavefront per sample: find the block by a 64-way search over the block
// prefix, then the lanes sum 2^B/64 consecutive amplitudes each, scan those
// partial sums in a fixed order, and the first lane whose running sum passes
// the target walks its own amplitudes.  PER > 0: blocks of 64 * PER
// amplitudes, each lane's run kept in registers for the walk; PER = 0: any
// block size, the walk reloads.
template <typename Idx, int PER>
__global__ __launch_bounds__(kBlock) void sample_draw(const float2 *__restrict__ amp, int n, int B,
                                                      const double *__restrict__ incl, int64_t nb,
                                                      const double *__restrict__ norm,
                                                      uint64_t seed, uint32_t traj, uint32_t circ,
                                                      int n_samples, ReadoutDesc ro,
                                                      uint64_t *__restrict__ out) {
    const int s = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (s >= n_samples) return;  // uniform over the wavefront
    const double N = *norm;
    const double target = philox_uniform(seed, uint32_t(s), traj, circ, kStreamMeasure) * N;
    // smallest block b with target < incl[b] (nb if none): the lanes probe
    // evenly spaced entries and a ballot keeps the first passing interval.
    // Invariant: the answer lies in [lo, hi], and hi passes or is nb.
    int64_t lo = 0, hi = nb;
    while (lo < hi) {
        const int64_t span = hi - lo;
        const int64_t step = span <= 64 ? 1 : (span + 63) / 64;
        int64_t probe = lo + int64_t(lane + 1) * step - 1;
        if (probe > hi - 1) probe = hi - 1;
        const bool pass = target < incl[probe];
        const uint64_t mask = __ballot(pass);
        if (mask == 0) {  // every probe up to hi - 1 fails
            lo = hi;
            break;
        }
        const int L = __ffsll((unsigned long long)mask) - 1;
        const int64_t pL = __shfl(probe, L, 64);
        const int64_t pprev = L > 0 ? __shfl(probe, L - 1, 64) : lo - 1;
        if (step == 1) {
            lo = pL;
            break;
        }
        lo = pprev + 1;
        hi = pL;
    }
    uint64_t x;
    if (lo >= nb) {
        x = (uint64_t(1) << n) - 1;
    } else {
        const double base = lo > 0 ? incl[lo - 1] : 0.0;
        const Idx first = Idx(lo) << B;
        const int len = 1 << B;
        const int per = PER > 0 ? PER : (len >= 64 ? len / 64 : 1);
        const int lanes = len >= 64 ? 64 : len;
        double part = 0.0;
        float2 keep[PER > 0 ? PER : 1];
        if constexpr (PER > 0) {
            // the block is read in whole lines and turned in LDS so that each
            // lane gets its run of PER consecutive amplitudes; one pad slot
            // per run keeps the runs on distinct banks.  Read straight from
            // memory, each load touched 64 lines (10^5 samples: 202 us at 28
            // qubits, now 184; a 20-qubit state, in cache: the whole call
            // 185 us, now 164).
            __shared__ float2 turn[kBlock / 64][64 * (PER + 1)];
            float2 *mine = turn[threadIdx.x >> 6];
            const float4 *p4 = reinterpret_cast<const float4 *>(amp + first);
            float4 in[PER / 2];
#pragma unroll
            for (int i = 0; i < PER / 2; ++i) in[i] = p4[i * 64 + lane];
#pragma unroll
            for (int i = 0; i < PER / 2; ++i) {
                const int a = 2 * (i * 64 + lane);
                mine[a + a / PER] = make_float2(in[i].x, in[i].y);
                mine[a + a / PER + 1] = make_float2(in[i].z, in[i].w);
            }
            wave_lds_order();
#pragma unroll
            for (int i = 0; i < PER; ++i) keep[i] = mine[lane * (PER + 1) + i];
#pragma unroll
            for (int i = 0; i < PER; ++i)
                part = fma(double(keep[i].x), double(keep[i].x), fma(double(keep[i].y), double(keep[i].y), part));
        } else if (lane < lanes) {
            part = chunk_weight(amp, first + Idx(lane * per), per);
        }
        const double inc = base + wave_inclusive_scan(part);
        const uint64_t passed = __ballot(lane < lanes && target < inc);
        int pick = len - 1;
        if (passed) {
            const int L = __ffsll((unsigned long long)passed) - 1;
            // lane L walks its amplitudes from its exclusive prefix, adding
            // them as chunk_weight does
            int idx = L * per + per - 1;
            if (lane == L) {
                double run = inc - part;
                if constexpr (PER > 0) {
                    bool found = false;
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        run = fma(double(keep[i].x), double(keep[i].x),
                                  fma(double(keep[i].y), double(keep[i].y), run));
                        if (!found && target < run) {
                            idx = L * PER + i;
                            found = true;
                        }
                    }
                } else if (per >= 2) {
                    const float4 *p4 = reinterpret_cast<const float4 *>(amp + first + Idx(L * per));
                    for (int i = 0; i < per / 2; ++i) {
                        const float4 v = p4[i];
                        const double r0 = fma(double(v.x), double(v.x), fma(double(v.y), double(v.y), run));
                        if (target < r0) { idx = L * per + 2 * i; break; }
                        const double r1 = fma(double(v.z), double(v.z), fma(double(v.w), double(v.w), r0));
                        if (target < r1) { idx = L * per + 2 * i + 1; break; }
                        run = r1;
                    }
                } else {
                    idx = L;
                }
            }
            pick = __shfl(idx, L, 64);
        }
        x = uint64_t(first) + uint64_t(pick);
    }
    // readout: lane q draws for qubit q (28 draws in a row on one lane took
    // 330 of the kernel's 470 us for 10^5 samples of 28 qubits)
    if (ro.enabled) {
        bool flip = false;
        if (lane < n) {
            const int bit = int((x >> lane) & 1u);
            const double u = philox_uniform(seed, uint32_t(uint64_t(s) * uint64_t(n) + uint64_t(lane)),
                                            traj, circ, kStreamReadout);
            flip = u < (bit ? ro.e1[lane] : ro.e0[lane]);
        }
        x ^= uint64_t(__ballot(flip));
    }
    if (lane == 0) out[s] = x;
}

// ---------------------------------------------------------------- helpers

inline unsigned grid_for(uint64_t work_items, unsigned cap = 1u << 20) {
    uint64_t b = (work_items + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return unsigned(b);
}

template <int K>
GateArgs<K> make_args(const GateDesc &g) {
    GateArgs<K> a;
    constexpr int D = 1 << K;
    for (int i = 0; i < D * D; ++i) a.m[i] = g.m[i];
    for (int b = 0; b < K; ++b) a.t[b] = g.t[b];
    return a;
}

int device_cus() {
    // initialised once, thread-safely (several host threads may launch at once)
    static const int cus = [] {
        int dev = 0, c = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0)
            c = 256;
        return c;
    }();
    return cus;
}

// Once per instantiation, thread-safely: allow the matrix region, and read
// how many workgroups per CU registers and waves allow (with no matrices the
// LDS is not what limits the count); a negative value is an error.
template <int TB, typename Idx, bool K5, int NT, bool RK, bool SP>
int tile_reg_limit() {
    static const int reg_limit = [] {
        const void *fn = reinterpret_cast<const void *>(&apply_tile<TB, Idx, K5, NT, RK, SP>);
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(sizeof(float2) * kTileMatBudget)) != hipSuccess)
            return -1;
        int blocks = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, NT, 0) != hipSuccess) return -1;
        return blocks < 1 ? 1 : blocks;
    }();
    return reg_limit;
}

// launch = false only sets the instantiation up (no stream work), so that a
// later launch under stream capture makes no attribute or occupancy calls.
template <int TB, typename Idx, bool K5, int NT, bool RK, bool SP>
hipError_t tile_launch(float2 *amp, int n, const TileArgs &a, hipStream_t st, bool launch,
                       int *grid_out) {
    // static tile + dynamic matrices
    const size_t dyn = sizeof(float2) * size_t(a.mat_total);
    const size_t lds = sizeof(float2) * (size_t(1) << TB) + dyn;
    const int reg_limit = tile_reg_limit<TB, Idx, K5, NT, RK, SP>();
    if (reg_limit < 0) return hipErrorInvalidDeviceFunction;
    const int cus = device_cus();
    if (!launch) return hipSuccess;
    const Idx n_tiles = Idx(1) << (n - TB);
    // persistent grid: as many workgroups as are resident at once at this LDS size
    int per_cu = int((160u * 1024u) / lds);
    if (per_cu < 1) per_cu = 1;
    if (per_cu > reg_limit) per_cu = reg_limit;
    uint64_t grid = uint64_t(cus) * uint64_t(per_cu);
    if (grid > uint64_t(n_tiles)) grid = uint64_t(n_tiles);
    if (RK && grid > uint64_t(kMaxReduceBlocks)) return hipErrorInvalidValue;  // record space
    if (grid_out) *grid_out = int(grid);
    apply_tile<TB, Idx, K5, NT, RK, SP><<<unsigned(grid), NT, dyn, st>>>(amp, n_tiles, a);
    return hipGetLastError();
}

template <int TB, typename Idx>
hipError_t tile_launch_k(float2 *amp, int n, const TileArgs &a, hipStream_t st, bool launch,
                         int *grid_out) {
    bool k5 = false;
    for (int gi = 0; gi < a.n_gates; ++gi) k5 |= a.g[gi].k == 5;
    // Four wavefronts per SIMD hide the LDS and MFMA latency: a 2^14-amplitude
    // tile (128 KiB) leaves room for one workgroup per CU, so it runs 1024
    // work-items; 2^13 (64 KiB) for two, with 512 each.  Smaller tiles fit
    // more workgroups and do better with 256 (measured on the 24-qubit noisy
    // grid).
    constexpr int NT = TB >= 14 ? 1024 : (TB >= 13 ? 512 : kBlock);
    auto go = [&](auto split) {
        constexpr bool SP = decltype(split)::value;
        if (a.rdm_out) {
            if (k5) return hipErrorInvalidValue;
            return tile_launch<TB, Idx, false, NT, true, SP>(amp, n, a, st, launch, grid_out);
        }
        return k5 ? tile_launch<TB, Idx, true, NT, false, SP>(amp, n, a, st, launch, grid_out)
                  : tile_launch<TB, Idx, false, NT, false, SP>(amp, n, a, st, launch, grid_out);
    };
    if (n > kBatchLdsQubits) return go(std::true_type());
    return go(std::false_type());
}

template <typename Idx>
hipError_t apply_tile_idx(float2 *amp, int n, const TileArgs &a, hipStream_t st, bool launch,
                          int *grid_out) {
    switch (a.tb) {
        case 10: return tile_launch_k<10, Idx>(amp, n, a, st, launch, grid_out);
        case 11: return tile_launch_k<11, Idx>(amp, n, a, st, launch, grid_out);
        case 12: return tile_launch_k<12, Idx>(amp, n, a, st, launch, grid_out);
        case 13: return tile_launch_k<13, Idx>(amp, n, a, st, launch, grid_out);
        case 14: return tile_launch_k<14, Idx>(amp, n, a, st, launch, grid_out);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_select(const SelectArgs &a, hipStream_t st) {
    if (a.nk < 1 || a.D < 1 || a.Db < 1 || a.Db > 32) return hipErrorInvalidValue;
    select_branch<<<1, 64, 0, st>>>(a);
    return hipGetLastError();
}

int batched_grid() {
    const int per_cu = int((160u * 1024u) / (sizeof(float2) * ((1u << kBatchLdsQubits) + 1536u) +
                                             sizeof(double) * kBlock));
    return device_cus() * (per_cu < 1 ? 1 : per_cu);
}

// Launches with no more jobs than CUs run one 512-work-item group per job
// (eight wavefronts share each block's work, twice the 256-work-item
// form's); larger ones run two 256-work-item groups per CU.  The grid never
// exceeds batched_grid(), which sizes the per-workgroup buffers.
hipError_t launch_batched(const BatchArgs &a, int grid, hipStream_t st) {
    const size_t lds = sizeof(float2) * ((size_t(1) << kBatchLdsQubits) + 1536);
    static const hipError_t attr256 = hipFuncSetAttribute(reinterpret_cast<const void *>(&run_batched<256>),
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    static const hipError_t attr512 = hipFuncSetAttribute(reinterpret_cast<const void *>(&run_batched<512>),
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (attr256 != hipSuccess) return attr256;
    if (attr512 != hipSuccess) return attr512;
    if (grid < 1 || a.n_jobs < 1) return hipErrorInvalidValue;
    if (a.n_jobs <= device_cus() && a.n_jobs <= grid)
        run_batched<512><<<unsigned(a.n_jobs), 512, lds, st>>>(a);
    else
        run_batched<256><<<unsigned(grid), 256, lds, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_batch_prepare(const BatchArgs &a, int job0, int jobs, hipStream_t st) {
    const size_t lds = sizeof(double2) * 4 * (1024 + 64);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&batch_prepare),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (attr != hipSuccess) return attr;
    if (jobs < 1) return hipErrorInvalidValue;
    batch_prepare<<<unsigned(jobs), kBlock, lds, st>>>(a, job0);
    return hipGetLastError();
}

hipError_t launch_batch_sweep(const BatchArgs &a, const BatchPart *parts, int n_parts, int step, bool k5,
                              hipStream_t st) {
    const size_t lds = sizeof(float2) * size_t(tile_mat_budget(kBatchTileBits));
    static const hipError_t attr_k5 = hipFuncSetAttribute(reinterpret_cast<const void *>(&batch_sweep<true>),
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&batch_sweep<false>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (attr_k5 != hipSuccess) return attr_k5;
    if (attr != hipSuccess) return attr;
    if (n_parts < 1 || step < 0) return hipErrorInvalidValue;
    if (k5) batch_sweep<true><<<unsigned(n_parts), kBatchWideThreads, lds, st>>>(a, parts, step);
    else batch_sweep<false><<<unsigned(n_parts), kBatchWideThreads, lds, st>>>(a, parts, step);
    return hipGetLastError();
}

hipError_t launch_batch_sample(const BatchArgs &a, int job0, int jobs, hipStream_t st) {
    if (jobs < 1) return hipErrorInvalidValue;
    batch_sample<<<unsigned(jobs), kBlock, 0, st>>>(a, job0);
    return hipGetLastError();
}

hipError_t launch_traj_resident(const TrajResidentArgs &a, int jobs, hipStream_t st) {
    if (a.n < 1 || a.n > kBatchLdsQubits || jobs < 1) return hipErrorInvalidValue;
    const size_t most = sizeof(float2) * ((size_t(1) << kBatchLdsQubits) + 1792);
    static const hipError_t attr256 = hipFuncSetAttribute(reinterpret_cast<const void *>(&run_resident<256, 9, 10>),
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(most));
    static const hipError_t attr512 = hipFuncSetAttribute(reinterpret_cast<const void *>(&run_resident<512, 10, 11>),
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(most));
    if (attr256 != hipSuccess) return attr256;
    if (attr512 != hipSuccess) return attr512;
    const size_t lds = sizeof(float2) * ((size_t(1) << a.n) + 1792);
    // below 11 qubits eight wavefronts have no 16-group batch of a 4-qubit block each
    if (a.n <= 10) run_resident<256, 9, 10><<<unsigned(jobs), 256, lds, st>>>(a);
    else run_resident<512, 10, 11><<<unsigned(jobs), 512, lds, st>>>(a);
    return hipGetLastError();
}

// With no more tiles than CUs, a tile's workgroup has 16 wavefronts: alone on
// its CU, eight leave two per SIMD (one 20-qubit trajectory, 128 tiles: 19 us
// a launch with 512 work-items, 17.3 with 1024).  From twice the 512
// resident workgroups on, each takes several tiles, so that the next tile's
// loads run under this one's gates and the matrices are staged once for them
// (20 trajectories of 21 qubits: 3.32 ms with a tile each, 2.81 like this).
int traj_sweep_groups(int n, int count) {
    int groups = 1 << (n - kBatchTileBits);
    while (groups > 1 && int64_t(groups) * count >= 4 * int64_t(device_cus())) groups /= 2;
    return groups;
}

hipError_t launch_traj_sweep(const TrajSweep *sweeps, const TrajGate *gates, int n, int count, hipStream_t st) {
    const size_t lds = sizeof(float2) * size_t(tile_mat_budget(kBatchTileBits));
    static const hipError_t attr512 = hipFuncSetAttribute(reinterpret_cast<const void *>(&traj_sweep<512>),
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    static const hipError_t attr1024 = hipFuncSetAttribute(reinterpret_cast<const void *>(&traj_sweep<1024>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (attr512 != hipSuccess) return attr512;
    if (attr1024 != hipSuccess) return attr1024;
    if (n <= kBatchTileBits || n > 31 || count < 1 || count > 65535) return hipErrorInvalidValue;
    const unsigned tiles = 1u << (n - kBatchTileBits);
    const dim3 grid(unsigned(traj_sweep_groups(n, count)), unsigned(count));
    if (int64_t(tiles) * count <= device_cus()) traj_sweep<1024><<<grid, 1024, lds, st>>>(sweeps, gates, tiles);
    else traj_sweep<512><<<grid, 512, lds, st>>>(sweeps, gates, tiles);
    return hipGetLastError();
}

hipError_t launch_traj_select(const TrajSelect *sels, int count, hipStream_t st) {
    if (count < 1) return hipErrorInvalidValue;
    traj_select<<<unsigned(count), 64, 0, st>>>(sels);
    return hipGetLastError();
}

BatchTileGate batch_tile_gate(int k, const int *lt, int lofs) {
    int tab[kMaxTileBits];
    switch (k) {
        case 1: gate_tables<1, SwizzledTile>(lt, tab); break;
        case 2: gate_tables<2, SwizzledTile>(lt, tab); break;
        case 3: gate_tables<3, SwizzledTile>(lt, tab); break;
        case 4: gate_tables<4, SwizzledTile>(lt, tab); break;
        default: gate_tables<5, SwizzledTile>(lt, tab); break;
    }
    BatchTileGate g;
    g.head = uint32_t(k);
    for (int j = 0; j < k; ++j) g.head |= uint32_t(lt[j]) << (4 + 4 * j);
    // entries past the 13 local bits are never used
    for (int b = 0; b < kMaxTileBits; b += 2)
        g.tab2[b >> 1] = (uint32_t(tab[b]) & 0xffffu) | (uint32_t(tab[b + 1]) << 16);
    g.lofs = lofs;
    return g;
}

int reduce_blocks_for(int n, int k) {
    // at least 4 groups per work-item; a fixed count per (n, k)
    const uint64_t groups = uint64_t(1) << (n - k);
    uint64_t b = groups / (4u * kBlock);
    if (b < 1) b = 1;
    if (b > kMaxReduceBlocks) b = kMaxReduceBlocks;
    return int(b);
}

hipError_t launch_set_basis(float2 *amp, int n, uint64_t index, hipStream_t st) {
    const uint64_t dim = uint64_t(1) << n;
    const unsigned grid = grid_for(dim);
    if (n <= 31)
        set_basis<uint32_t><<<grid, kBlock, 0, st>>>(amp, uint32_t(dim), uint32_t(index));
    else
        set_basis<uint64_t><<<grid, kBlock, 0, st>>>(amp, dim, index);
    return hipGetLastError();
}

hipError_t launch_copy_state(float2 *dst, const float2 *src, int n, hipStream_t st) {
    if (n < 1 || n > kMaxQubits || !dst || !src) return hipErrorInvalidValue;
    const int64_t pairs = int64_t(1) << (n - 1);
    const int64_t want = (pairs + kBlock - 1) / kBlock;
    const int64_t cap = int64_t(device_cus()) * 4;
    const unsigned grid = unsigned(want < cap ? want : cap);
    copy_pairs<<<grid, kBlock, 0, st>>>(reinterpret_cast<float4 *>(dst), reinterpret_cast<const float4 *>(src),
                                        pairs);
    return hipGetLastError();
}

hipError_t launch_scale(float2 *amp, int n, float s, hipStream_t st) {
    const uint64_t dim = uint64_t(1) << n;
    const unsigned grid = grid_for(dim);
    if (n <= 31)
        scale_state<uint32_t><<<grid, kBlock, 0, st>>>(amp, uint32_t(dim), s);
    else
        scale_state<uint64_t><<<grid, kBlock, 0, st>>>(amp, dim, s);
    return hipGetLastError();
}

// Lowest target the kernels that work straight on memory take: from bit 3 on
// a pair kernel's accesses are whole 64-byte pieces, and the MFMA kernel
// needs bits 0..3 for its 16 groups.  Gates below that stage tiles in LDS.
constexpr int kPairTarget = 3;
constexpr int kMfmaTarget = 4;

// Tile of a single gate: bits 0..5, its targets and the lowest others.
void tile_for_gate(int n, const GateDesc &g, TileArgs &a) {
    bool in_tile[kMaxQubits] = {false};
    int cnt = 0;
    for (int q = 0; q < 6; ++q) { in_tile[q] = true; ++cnt; }
    for (int b = 0; b < g.k; ++b)
        if (!in_tile[g.t[b]]) { in_tile[g.t[b]] = true; ++cnt; }
    int tb = cnt;
    if (tb < 10) tb = 10;
    if (tb < g.k + 8) tb = g.k + 8;
    if (tb > n) tb = n;
    for (int q = 0; q < n && cnt < tb; ++q)
        if (!in_tile[q]) { in_tile[q] = true; ++cnt; }
    a.tb = tb;
    int i = 0;
    for (int q = 0; q < n; ++q)
        if (in_tile[q]) a.pos[i++] = q;
    a.n_gates = 1;
    a.init_zero = 0;
    a.mat_total = tile_mat_slots(g.k);
    a.g[0].k = g.k;
    a.g[0].lofs = 0;
    a.g[0].pad = 0;
    a.g[0].mat = nullptr;
    for (int b = 0; b < g.k; ++b) {
        int lp = 0;
        while (a.pos[lp] != g.t[b]) ++lp;
        a.g[0].lt[b] = lp;  // ascending because g.t is ascending
    }
}

template <int K>
MatArg<K> mat_arg(const GateDesc &g, const float2 *dev) {
    MatArg<K> m;
    if (!dev) std::memcpy(m.m, g.m, sizeof(m.m));
    return m;
}

template <int TB, typename Idx>
hipError_t tile_one(float2 *amp, int n, const TileArgs &t, const GateDesc &g, const float2 *dev, hipStream_t st) {
    TileOneArgs a;
    for (int b = 0; b < kMaxTileBits; ++b) a.pos[b] = t.pos[b];
    a.g = t.g[0];
    a.g.mat = dev;
    switch (g.k) {
        case 1: gate_tables<1, SwizzledTile>(a.g.lt, a.g.tab); break;
        case 2: gate_tables<2, SwizzledTile>(a.g.lt, a.g.tab); break;
        case 3: gate_tables<3, SwizzledTile>(a.g.lt, a.g.tab); break;
        default: gate_tables<4, SwizzledTile>(a.g.lt, a.g.tab); break;
    }
    MatArg<4> m;
    if (!dev) std::memcpy(m.m, g.m, sizeof(float2) << (2 * g.k));
    const uint64_t n_tiles = uint64_t(1) << (n - TB);
    // the workgroups the CUs hold at once (LDS, and eight 256-work-item groups of wavefronts)
    const uint64_t per_cu = std::min<uint64_t>(8, (160u * 1024u) / (sizeof(float2) * ((1u << TB) + 416u)));
    const uint64_t grid = std::min<uint64_t>(n_tiles, uint64_t(device_cus()) * per_cu);
    apply_tile_one<TB, Idx><<<unsigned(grid), kBlock, 0, st>>>(m, amp, Idx(n_tiles), a);
    return hipGetLastError();
}

template <int K, typename Idx>
hipError_t gate_k(float2 *amp, int n, const GateDesc &g, const float2 *dev, hipStream_t st) {
    constexpr int KA = K <= 4 ? K : 0;
    TargetArgs ta;
    for (int b = 0; b < kMaxGateQubits; ++b) ta.t[b] = b < K ? g.t[b] : 0;
    const MatArg<KA> m = mat_arg<KA>(g, K <= 4 ? dev : g.m);
    if constexpr (K <= 2) {
        if (g.t[0] >= kPairTarget) {
            const uint64_t pairs = uint64_t(1) << (n - K - 1);
            apply_pairs<K, Idx><<<grid_for(pairs), kBlock, 0, st>>>(m, amp, Idx(pairs), dev, ta);
            return hipGetLastError();
        }
    } else {
        if (g.t[0] >= kMfmaTarget) {  // then n - K >= 4: sixteen groups
            const uint64_t batches = uint64_t(1) << (n - K - 4);
            // a few batches per wavefront: the A operands are loaded once for
            // them (us a gate on high targets at 1 / 2 / 4 / 8 workgroups per
            // CU: k = 3, 22 qubits 10.9, 9.8, 9.6, 9.4, 26 qubits 347, 228,
            // 193, 206; k = 4 14.3, 12.7, 12.4, 12.8 and 279, 200, 205, 209;
            // k = 5, 24 qubits 60, 59, 64, 69, 26 qubits 259, 224, 242, 247;
            // up to 20 qubits the same at any)
            const uint64_t cap = uint64_t(device_cus()) * (K == 5 ? 2 : 4);
            const uint64_t grid = std::min<uint64_t>((batches + 3) / 4, cap);
            apply_direct_mfma<K, Idx><<<unsigned(grid), kBlock, 0, st>>>(m, amp, Idx(batches), dev, ta);
            return hipGetLastError();
        }
    }
    if (n >= kTileMinQubits) {
        TileArgs t;
        std::memset(&t, 0, sizeof(t));
        tile_for_gate(n, g, t);
        if constexpr (K == 5) {
            t.g[0].mat = dev;
            return launch_apply_tile(amp, n, t, st);
        } else {
            switch (t.tb) {  // 10 .. k + 8, and no wider than the state
                case 10: return tile_one<10, Idx>(amp, n, t, g, dev, st);
                case 11: return tile_one<11, Idx>(amp, n, t, g, dev, st);
                case 12: return tile_one<12, Idx>(amp, n, t, g, dev, st);
                default: return hipErrorInvalidValue;
            }
        }
    }
    const uint64_t groups = uint64_t(1) << (n - K);
    apply_direct<K, Idx><<<grid_for(groups), kBlock, 0, st>>>(m, amp, Idx(groups), dev, ta);
    return hipGetLastError();
}

template <typename Idx>
hipError_t gate_idx(float2 *amp, int n, const GateDesc &g, const float2 *dev, hipStream_t st) {
    switch (g.k) {
        case 1: return gate_k<1, Idx>(amp, n, g, dev, st);
        case 2: return gate_k<2, Idx>(amp, n, g, dev, st);
        case 3: return gate_k<3, Idx>(amp, n, g, dev, st);
        case 4: return gate_k<4, Idx>(amp, n, g, dev, st);
        case 5: return gate_k<5, Idx>(amp, n, g, dev, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_apply_gate(float2 *amp, int n, const GateDesc &g, const float2 *mat_dev,
                             hipStream_t st) {
    if (!mat_dev && g.k > kMaxArgGate) return hipErrorInvalidValue;
    if (n <= 31) return gate_idx<uint32_t>(amp, n, g, mat_dev, st);
    return gate_idx<uint64_t>(amp, n, g, mat_dev, st);
}

hipError_t launch_apply_tile(float2 *amp, int n, const TileArgs &a, hipStream_t st, int *grid_out) {
    return launch_apply_tile_impl(amp, n, a, st, true, grid_out);
}

hipError_t prepare_apply_tile(int n, const TileArgs &a) {
    return launch_apply_tile_impl(nullptr, n, a, nullptr, false);
}

hipError_t launch_apply_tile_impl(float2 *amp, int n, const TileArgs &a, hipStream_t st, bool launch,
                                  int *grid_out) {
    if (a.tb < 10 || a.tb > kMaxTileBits || a.tb > n || a.n_gates < 0 ||
        a.n_gates > kMaxTileGates || a.mat_total < 0 || a.mat_total > kTileMatBudget)
        return hipErrorInvalidValue;
    if (a.rdm_out && (a.rdm_lt < 0 || a.rdm_lt >= a.tb)) return hipErrorInvalidValue;
    // tile bits: ascending global positions below n, the first kTileLowBits
    // of them bits 0.. (the pair loads need local bit 0 = global bit 0)
    for (int b = 0; b < a.tb; ++b)
        if (a.pos[b] < 0 || a.pos[b] >= n || (b > 0 && a.pos[b] <= a.pos[b - 1]) ||
            (b < kTileLowBits && a.pos[b] != b))
            return hipErrorInvalidValue;
    for (int gi = 0; gi < a.n_gates; ++gi) {
        const TileGate &g = a.g[gi];
        if (g.k < 1 || g.k > kMaxGateQubits || g.k > a.tb || !g.mat || g.lofs < 0 ||
            g.lofs + tile_mat_slots(g.k) > a.mat_total)
            return hipErrorInvalidValue;
        for (int b = 0; b < g.k; ++b)
            if (g.lt[b] < 0 || g.lt[b] >= a.tb || (b > 0 && g.lt[b] <= g.lt[b - 1]))
                return hipErrorInvalidValue;
    }
    // each gate's address table for the swizzled tile layout
    TileArgs b = a;
    for (int gi = 0; gi < b.n_gates; ++gi) {
        TileGate &g = b.g[gi];
        switch (g.k) {
            case 1: gate_tables<1, SwizzledTile>(g.lt, g.tab); break;
            case 2: gate_tables<2, SwizzledTile>(g.lt, g.tab); break;
            case 3: gate_tables<3, SwizzledTile>(g.lt, g.tab); break;
            case 4: gate_tables<4, SwizzledTile>(g.lt, g.tab); break;
            default: gate_tables<5, SwizzledTile>(g.lt, g.tab); break;
        }
    }
    if (n <= 31) return apply_tile_idx<uint32_t>(amp, n, b, st, launch, grid_out);
    return apply_tile_idx<uint64_t>(amp, n, b, st, launch, grid_out);
}

hipError_t launch_reduce_records(const double *partials, int count, int width, double *out_dev,
                                 hipStream_t st) {
    if (count < 1 || count > kMaxReduceBlocks || width < 1 || width > kMaxReduceWidth)
        return hipErrorInvalidValue;
    reduce_records<<<unsigned(width), kBlock, 0, st>>>(partials, count, width, out_dev);
    return hipGetLastError();
}

hipError_t launch_norm(const float2 *amp, int n, double *partials, double *out_dev,
                       hipStream_t st) {
    const int nb = reduce_blocks_for(n, 0);
    const uint64_t dim = uint64_t(1) << n;
    if (n <= 31)
        norm_partials<uint32_t><<<nb, kBlock, 0, st>>>(amp, uint32_t(dim), partials);
    else
        norm_partials<uint64_t><<<nb, kBlock, 0, st>>>(amp, dim, partials);
    reduce_records<<<1, kBlock, 0, st>>>(partials, nb, 1, out_dev);
    return hipGetLastError();
}

hipError_t launch_zweights(const float2 *amp, int n, double *partials, double *out_dev, hipStream_t st) {
    if (n < 1 || n > kZRecord - 1) return hipErrorInvalidValue;
    if (n < kZStepBits) {
        zweight_small<<<1, kBlock, 0, st>>>(amp, n, out_dev);
        return hipGetLastError();
    }
    // at most 1024 chunks (four workgroups per CU, 32 KiB of loads in flight each)
    const int lb = n - kZStepBits < 10 ? n - kZStepBits : 10;
    const int c = n - lb;  // 12..24
    const unsigned nb = 1u << lb;
    if (n <= 31) zweight_partials<uint32_t><<<nb, kBlock, 0, st>>>(amp, n, c, partials);
    else zweight_partials<uint64_t><<<nb, kBlock, 0, st>>>(amp, n, c, partials);
    reduce_records<<<kZRecord, kBlock, 0, st>>>(partials, int(nb), kZRecord, out_dev);
    return hipGetLastError();
}

hipError_t launch_rdm(const float2 *amp, int n, int k, const int *t_sorted, double *partials,
                      double *out_dev, hipStream_t st) {
    const int nb = reduce_blocks_for(n, k);
    TargetArgs ta;
    for (int b = 0; b < kMaxGateQubits; ++b) ta.t[b] = b < k ? t_sorted[b] : 0;
    const uint64_t groups = uint64_t(1) << (n - k);
    const int width = 2 << (2 * k);
    if (k == 1) {
        if (n <= 31) rdm_partials<1, uint32_t><<<nb, kBlock, 0, st>>>(amp, uint32_t(groups), ta, partials);
        else rdm_partials<1, uint64_t><<<nb, kBlock, 0, st>>>(amp, groups, ta, partials);
    } else if (k == 2) {
        if (n <= 31) rdm_partials<2, uint32_t><<<nb, kBlock, 0, st>>>(amp, uint32_t(groups), ta, partials);
        else rdm_partials<2, uint64_t><<<nb, kBlock, 0, st>>>(amp, groups, ta, partials);
    } else {
        return hipErrorInvalidValue;
    }
    reduce_records<<<unsigned(width), kBlock, 0, st>>>(partials, nb, width, out_dev);
    return hipGetLastError();
}

hipError_t launch_apply_copy_norm(const float2 *in, float2 *out, int n, const GateDesc &g,
                                  double *partials, double *out_dev, hipStream_t st) {
    const int nb = reduce_blocks_for(n, g.k);
    const uint64_t groups = uint64_t(1) << (n - g.k);
    if (g.k == 1) {
        if (n <= 31) apply_copy_norm<1, uint32_t><<<nb, kBlock, 0, st>>>(in, out, uint32_t(groups), make_args<1>(g), partials);
        else apply_copy_norm<1, uint64_t><<<nb, kBlock, 0, st>>>(in, out, groups, make_args<1>(g), partials);
    } else if (g.k == 2) {
        if (n <= 31) apply_copy_norm<2, uint32_t><<<nb, kBlock, 0, st>>>(in, out, uint32_t(groups), make_args<2>(g), partials);
        else apply_copy_norm<2, uint64_t><<<nb, kBlock, 0, st>>>(in, out, groups, make_args<2>(g), partials);
    } else {
        return hipErrorInvalidValue;
    }
    reduce_records<<<2, kBlock, 0, st>>>(partials, nb, 2, out_dev);
    return hipGetLastError();
}

// ---------------------------------------------------------------- allocation-free sampling

// The sampling buffers of qs_sample_measurements_noalloc: a fixed array per
// GPU, held until the process ends (4.5 MiB: block sums and prefix for up to
// 2^28 amplitudes, the norm, up to 2^16 bitstrings).  Host code must not pass
// `scratch` itself to a kernel (in host code the name is a stand-in, not a
// device address): it uses the address noalloc_scratch looked up.
static __device__ __align__(256) double scratch[kNoAllocDoubles];

namespace {
std::mutex g_scratch_mu;
double *g_scratch_dev[64] = {};  // per device, filled once
}  // namespace

hipError_t noalloc_scratch(int device, double **out) {
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[device]) {
        int prev = 0;
        hipError_t e = hipGetDevice(&prev);
        if (e != hipSuccess) return e;
        if (prev != device && (e = hipSetDevice(device)) != hipSuccess) return e;
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (prev != device) (void)hipSetDevice(prev);
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_dev[device] = static_cast<double *>(p);
    }
    *out = g_scratch_dev[device];
    return hipSuccess;
}

hipError_t launch_sample(const float2 *amp, int n, double *sums, double *incl, uint64_t seed,
                         uint32_t traj, uint32_t circ, int n_samples, const ReadoutDesc &ro,
                         uint64_t *out_dev, double *norm_dev, hipStream_t st, double *norm_host) {
    const int B = n < kSampleBlockBits ? n : kSampleBlockBits;
    const int64_t nb = int64_t(1) << (n - B);
    const int64_t n_tiles = (nb + kScanTile - 1) / kScanTile;
    if (n_tiles > kScanMaxTiles) return hipErrorInvalidValue;
    const unsigned sum_grid = unsigned((nb + kBlock / 64 - 1) / (kBlock / 64));
    if (n <= 31)
        sample_block_sums<uint32_t><<<sum_grid, kBlock, 0, st>>>(amp, B, nb, sums);
    else
        sample_block_sums<uint64_t><<<sum_grid, kBlock, 0, st>>>(amp, B, nb, sums);
    // one tile (up to 23 qubits) needs no offsets
    sample_scan_tiles<<<unsigned(n_tiles), kScanThreads, 0, st>>>(sums, nb, incl, n_tiles == 1 ? norm_dev : nullptr,
                                                                  norm_host);
    if (n_tiles > 1) {
        // the block sums have been read: their first n_tiles slots take the offsets
        sample_scan_offsets<<<1, kScanThreads, 0, st>>>(incl, nb, int(n_tiles), sums, norm_dev, norm_host);
        sample_scan_add<<<unsigned((nb - kScanTile + kBlock - 1) / kBlock), kBlock, 0, st>>>(incl, nb, sums);
    }
    if (n_samples > 0) {
        const unsigned grid = unsigned((n_samples + kBlock / 64 - 1) / (kBlock / 64));
        if (B == 10 && n <= 31)
            sample_draw<uint32_t, 16><<<grid, kBlock, 0, st>>>(amp, n, B, incl, nb, norm_dev, seed, traj,
                                                               circ, n_samples, ro, out_dev);
        else if (B == 10)
            sample_draw<uint64_t, 16><<<grid, kBlock, 0, st>>>(amp, n, B, incl, nb, norm_dev, seed, traj,
                                                               circ, n_samples, ro, out_dev);
        else
            sample_draw<uint32_t, 0><<<grid, kBlock, 0, st>>>(amp, n, B, incl, nb, norm_dev, seed, traj,
                                                              circ, n_samples, ro, out_dev);
    }
    return hipGetLastError();
}

}  // namespace qs
