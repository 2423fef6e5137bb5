// SDF network: forward + analytic input gradient, and the backward pass with the
// second-order term, fused per 32-point tile on the matrix cores (fp32 values as sums of bf16
// terms, see mfma_tile.h).
//
// Paper: Eq. 1 ((d,g) = f_Theta(e)), Definition 1 (bias-free ReLU MLP, masks G_l, vectors
// P_l^j and S_l^i), Eq. 2 (n = grad_x d), supplement Sec. B (dy/dx = H_L G_L ... G_2 H_1),
// Theorem 1 (d(dy/dx)_(i,j)/dH_l = (P_l^j S_l^i)^T, second input derivative zero) and
// Eqs. 7-8 (what is left of the chain rule).
//
// With i = 0 (the SDF output), S_l is the reverse sweep from row 0 of the last matrix and
// the sum over j of P_l^j weighted by (de/dx) dL/dn is ONE forward-mode sweep t_l, so
//     dL/dH_l = delta_l a_{l-1}^T  +  S_l^T t_{l-1}^T        (first + second order)
// Both products contract over points and run as MFMA outer-product accumulations.
// Activations and masks are recomputed in the backward kernel from the encoding (cheaper
// than storing and re-reading four 64-wide vectors per point).
#include <type_traits>

#include "common.h"
#include "mfma_tile.h"

namespace neus2 {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

struct SdfArgs {
    const float* enc; const float* jac; const float* H[3];
    const float* d_y; const float* d_normal;
    float* y; float* q; float* normal;
    float* dH[3]; float* d_enc; float* d_pos;
    uint32_t* masks;           // optional [2][n][2]: written by the forward kernel, read by the backward kernel
    int64_t n; int active_levels;
    bool stream_q;             // q (forward kernel) and dL/de (backward kernel) with non-temporal stores
};

// The ReLU masks of a point as the kernels keep them: one word per hidden layer and lane half h,
// bit 16 b + r for neuron 32 b + neuron_of(r, h); word (layer * n + i) * 2 + h of the buffer.
__device__ __forceinline__ int64_t mask_word(int layer, int64_t n, int64_t i, int h) { return ((int64_t)layer * n + i) * 2 + h; }

// LDS copies of the matrices, split into bf16 terms (see mfma_tile.h), in the orientations a
// kernel needs ("f": rows = outputs, "t": rows = inputs).  Everything the forward kernel
// computes, and the forward pass where the backward kernel recomputes it, uses three terms per
// factor and six products: as accurate as fp32 arithmetic, and the same arithmetic in both
// kernels, so the ReLU masks agree.  The adjoint, S and t sweeps of the backward kernel use
// two terms and three products.
// PF: terms of the matrices of the forward direction.
template <int D, int K, bool BWD, int PF = 3>
struct SdfWeights {
    static constexpr int KS1 = D / 16;
    typedef SplitMatrix<KS1, PF> M1f;              // [64][D]
    typedef SplitMatrix<4, PF> M2f;                // [64][64]
    typedef SplitMatrix<4, 3> MLf;                 // last matrix [16 -> 32][64]
    typedef SplitMatrix<4, BWD ? 2 : 3> M1t;       // [D -> 32][64]
    typedef SplitMatrix<4, BWD ? 2 : 3> M2t;
    typedef SplitMatrix<1, 2> MLt;                 // [64][16]
    alignas(16) unsigned char H1f[64 * M1f::kLd];
    alignas(16) unsigned char H1t[32 * M1t::kLd];
    alignas(16) unsigned char H2f[K == 3 ? 64 * M2f::kLd : 16];
    alignas(16) unsigned char H2t[K == 3 ? 64 * M2t::kLd : 16];
    alignas(16) unsigned char HLf[BWD ? 16 : 32 * MLf::kLd];
    alignas(16) unsigned char HLt[BWD ? 64 * MLt::kLd : 16];
    // Row 0 of the last matrix (the SDF output), already split and packed as a lane holds it
    // (Split<2, 3>): [lane half][term][word 8 b + p]
    alignas(16) uint32_t HLrow0[2][3][16];
};

// Every matrix is fetched from global memory before the first is written to LDS, so the fetches
// are in flight together; the copies cover every slot a product reads, so nothing is cleared.
template <int D, int K, bool BWD, int THREADS, int PF = 3>
__device__ void load_weights(SdfWeights<D, K, BWD, PF>& w, const SdfArgs& a) {
    typedef SdfWeights<D, K, BWD, PF> W;
    const int tid = threadIdx.x;
    const float* __restrict__ H1 = a.H[0];
    const float* __restrict__ H2 = a.H[1];
    const float* __restrict__ HL = a.H[K - 1];
    typename W::M1f::template Fill<64, THREADS, false> f1;
    typename W::M1t::template Fill<32, THREADS, true> t1;
    typename W::M2f::template Fill<K == 3 ? 64 : 0, THREADS, false> f2;
    typename W::M2t::template Fill<K == 3 ? 64 : 0, THREADS, true> t2;
    typename W::MLf::template Fill<BWD ? 0 : 32, THREADS, false> fl;
    typename W::MLt::template Fill<BWD ? 64 : 0, THREADS, true> tl;
    f1.load(tid, [&](int o, int i) { return H1[o * D + i]; });
    t1.load(tid, [&](int i, int o) { return i < D ? H1[o * D + i] : 0.f; });
    f2.load(tid, [&](int o, int i) { return H2[o * 64 + i]; });
    t2.load(tid, [&](int i, int o) { return H2[o * 64 + i]; });
    fl.load(tid, [&](int o, int i) { return o < 16 ? HL[o * 64 + i] : 0.f; });
    tl.load(tid, [&](int i, int o) { return HL[o * 64 + i]; });
    // thread 16 h + 8 b + p < 32 splits the pair of row-0 elements that word p of block b of lane
    // half h holds: registers 2p and 2p + 1
    float row0[2] = {0.f, 0.f};
    if (tid < 32) {
        const int hh = tid >> 4, b = (tid >> 3) & 1, p = tid & 7;
        row0[0] = HL[32 * b + neuron_of(2 * p, hh)];
        row0[1] = HL[32 * b + neuron_of(2 * p + 1, hh)];
    }
    f1.store(w.H1f, tid);
    t1.store(w.H1t, tid);
    f2.store(w.H2f, tid);
    t2.store(w.H2t, tid);
    fl.store(w.HLf, tid);
    tl.store(w.HLt, tid);
    if (tid < 32) {
        typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
        typedef float f2 __attribute__((ext_vector_type(2)));
        float x0 = row0[0], x1 = row0[1];
#pragma unroll
        for (int term = 0; term < 3; ++term) {
            const uint32_t word = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x0, x1}, bf2));
            w.HLrow0[tid >> 4][term][tid & 15] = word;
            x0 -= __builtin_bit_cast(float, word << 16);
            x1 -= __builtin_bit_cast(float, word & 0xffff0000u);
        }
    }
    __syncthreads();
}

// level-major [L][n][2] <-> register vector of width D.  Register r = 4g + 2u + f of lane half h
// is feature f of level 4g + 2h + u.
template <int D>
__device__ __forceinline__ v16f load_levels(const float* __restrict__ src, int64_t n, int64_t i, bool valid,
                                            int active, int h) {
    v16f x = zero16();
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int level = 4 * g + 2 * h + u;
            if (valid && level < active) {
                const float2 v = reinterpret_cast<const float2*>(src)[(int64_t)level * n + i];
                x[4 * g + 2 * u] = v.x;
                x[4 * g + 2 * u + 1] = v.y;
            }
        }
    return x;
}

template <int D, bool STREAM = false>
__device__ __forceinline__ void store_levels(float* __restrict__ dst, int64_t n, int64_t i, bool valid,
                                             const v16f& x, int h) {
    if (!valid) return;
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int level = 4 * g + 2 * h + u;
            if (STREAM) {
                typedef float f2v __attribute__((ext_vector_type(2)));
                __builtin_nontemporal_store(f2v{x[4 * g + 2 * u], x[4 * g + 2 * u + 1]}, reinterpret_cast<f2v*>(dst) + (int64_t)level * n + i);
            } else {
                reinterpret_cast<float2*>(dst)[(int64_t)level * n + i] = make_float2(x[4 * g + 2 * u], x[4 * g + 2 * u + 1]);
            }
        }
}

// the levels below active only (an array of a narrower encoding has no more)
__device__ __forceinline__ void store_levels_active(float* __restrict__ dst, int64_t n, int64_t i, bool valid, int active, int h,
                                                    const v16f& x) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int level = 4 * g + 2 * h + u;
            if (valid && level < active)
                reinterpret_cast<float2*>(dst)[(int64_t)level * n + i] = make_float2(x[4 * g + 2 * u], x[4 * g + 2 * u + 1]);
        }
}

// out_a = sum over this lane's features of x_k * J[k][a]   (J = de/dx; per level three planes [n] of
// pairs: (J00,J01), (J02,J10), (J11,J12))
template <int D>
__device__ __forceinline__ void contract_jac(const float* __restrict__ jac, int64_t n, int64_t i, bool valid,
                                             int active, int h, const v16f& x, float out[3]) {
    out[0] = out[1] = out[2] = 0.f;
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int level = 4 * g + 2 * h + u;
            if (valid && level < active) {
                const float2* J = reinterpret_cast<const float2*>(jac) + (int64_t)level * 3 * n + i;
                const float2 a = J[0], b = J[n], c = J[2 * n];     // (J00,J01) (J02,J10) (J11,J12)
                const float x0 = x[4 * g + 2 * u], x1 = x[4 * g + 2 * u + 1];
                out[0] += x0 * a.x + x1 * b.y;
                out[1] += x0 * a.y + x1 * c.x;
                out[2] += x0 * b.x + x1 * c.y;
            }
        }
}

// t_k = sum_a J[k][a] * v_a
template <int D>
__device__ __forceinline__ v16f apply_jac(const float* __restrict__ jac, int64_t n, int64_t i, bool valid,
                                          int active, int h, const float v[3]) {
    v16f t = zero16();
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int level = 4 * g + 2 * h + u;
            if (valid && level < active) {
                const float2* J = reinterpret_cast<const float2*>(jac) + (int64_t)level * 3 * n + i;
                const float2 a = J[0], b = J[n], c = J[2 * n];
                t[4 * g + 2 * u] = a.x * v[0] + a.y * v[1] + b.x * v[2];
                t[4 * g + 2 * u + 1] = b.y * v[0] + c.x * v[1] + c.y * v[2];
            }
        }
    return t;
}

// The Jacobian rows of this lane's features, held in registers so that the loads can be issued
// long before they are needed.
template <int D>
struct JacRegs {
    float2 v[D / 4][3];        // per level of this lane: (J00,J01) (J02,J10) (J11,J12)
};

template <int D>
__device__ __forceinline__ JacRegs<D> load_jac(const float* __restrict__ jac, int64_t n, int64_t i, bool valid,
                                               int active, int h) {
    JacRegs<D> J;
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int level = 4 * g + 2 * h + u;
            const bool on = valid && level < active;
            const float2* p = reinterpret_cast<const float2*>(jac) + (int64_t)(on ? level : 0) * 3 * n + (on ? i : 0);
#pragma unroll
            // the Jacobian is the widest stream of the network kernels and is not read again before the
            // other kernel's turn, a whole batch later: non-temporal loads (5 us of the step)
            for (int c = 0; c < 3; ++c) {
                typedef float f2v __attribute__((ext_vector_type(2)));
                J.v[2 * g + u][c] = make_float2(0.f, 0.f);
                if (on) {
                    const f2v w = __builtin_nontemporal_load(reinterpret_cast<const f2v*>(p) + c * n);
                    J.v[2 * g + u][c] = make_float2(w.x, w.y);
                }
            }
        }
    return J;
}

template <int D>
__device__ __forceinline__ v16f apply_jac_regs(const JacRegs<D>& J, const float v[3]) {
    v16f t = zero16();
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float2 a = J.v[2 * g + u][0], b = J.v[2 * g + u][1], c = J.v[2 * g + u][2];
            t[4 * g + 2 * u] = a.x * v[0] + a.y * v[1] + b.x * v[2];
            t[4 * g + 2 * u + 1] = b.y * v[0] + c.x * v[1] + c.y * v[2];
        }
    return t;
}

// Row 0 of the last matrix, masked (S_{K-1} of Definition 1 for output 0), as a split vector: the
// terms were split when the matrix was copied to LDS, and masking a packed pair is an AND with a
// word that has ones in the halves whose mask bit is set (bit 16 b + r for register r of block b;
// word p holds registers 2p and 2p + 1).  The same values as splitting the masked row.
template <int P>
__device__ __forceinline__ void last_row_masked(const uint32_t (*row0)[3][16], uint32_t m, int h, Split<2, P>& out) {
    const uint32_t one = opaque<1u>();
    uint32_t keep[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int bit = 16 * (k >> 3) + 2 * (k & 7);
        const uint32_t lo = mask_bit(m, bit, one), hi = mask_bit(m, bit + 1, one);
        keep[k] = (lo & 0xffffu) | (hi & 0xffff0000u);
    }
#pragma unroll
    for (int term = 0; term < P; ++term)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const u32x4 words = *reinterpret_cast<const u32x4*>(&row0[h][term][4 * g]);
#pragma unroll
            for (int e = 0; e < 4; ++e) out.t[term][g >> 1][4 * (g & 1) + e] = words[e] & keep[4 * g + e];
        }
}

// 16-wide per-point rows ([n][16]) <-> register vector: registers 0..7 of lane half h hold
// columns 4h..4h+3 and 8+4h..8+4h+3.
__device__ __forceinline__ v16f load_rows16(const float* __restrict__ src, int64_t i, bool valid, int h) {
    v16f x = zero16();
    if (valid) {
        const float4 a = *reinterpret_cast<const float4*>(src + i * 16 + 4 * h);
        const float4 b = *reinterpret_cast<const float4*>(src + i * 16 + 8 + 4 * h);
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    }
    return x;
}

__device__ __forceinline__ void store_rows16(float* __restrict__ dst, int64_t i, bool valid, int h, const v16f& x) {
    if (!valid) return;
    *reinterpret_cast<float4*>(dst + i * 16 + 4 * h) = make_float4(x[0], x[1], x[2], x[3]);
    *reinterpret_cast<float4*>(dst + i * 16 + 8 + 4 * h) = make_float4(x[4], x[5], x[6], x[7]);
}

// ------------------------------------------------------------------------------------------
// The forward kernel runs 1024 threads per workgroup: its 90 KB of matrices are shared by sixteen wavefronts, four per
// SIMD with 128 registers each, so that one wavefront's waits for memory, LDS and matrix results are filled by the others.
// Nothing is requested ahead: two wavefronts per SIMD that prefetched the next encoding and this tile's Jacobian (221
// registers) took 60 us at 2^18 points and 199 at 2^20, four take 51 and 168 (4.5 TB/s: its streams are 732 bytes a point),
// at 32576 points 15.7 and 12.8.  The first layer leaves out the k-step of levels that are not read.
constexpr int kFwdThreads = 1024;
constexpr int kFwdWaves = kFwdThreads / 64;
constexpr int kValueThreads = 512;
constexpr int kValueWaves = kValueThreads / 64;

// Accesses of a tile: a uniform address (scalar registers: array, tile, level) plus a byte offset of the lane.  Written
// with one 64-bit index per lane, the compiler kept two dozen addresses in vector registers through the whole loop and spilled
// them.  The largest lane offset is 48 n bytes (upper lane half, Jacobian): 32 bits below kTileMaxPoints, 64 (WIDE) from there on,
// where an access takes an addition of its own: 2^26 points forward 12.1 ms narrow, 13.2 wide, backward 19.0 and 18.9.
constexpr int64_t kTileMaxPoints = (int64_t)1 << 26;

template <bool WIDE>
using LaneOffset = std::conditional_t<WIDE, uint64_t, uint32_t>;

typedef float f2v __attribute__((ext_vector_type(2)));

// Levels 4 g + 2 h + u of the tile's points as in load_levels, store_levels and load_jac, first: the tile's first point.
// Loads are unconditional within the groups of four levels that a kernel reads: a lane without a point reads the tile's last
// one, the upper lane half reads the lower half's level where its own is not active, and what does not count is replaced by
// zeros afterwards.  So one level beyond the active ones is read at most (5, 9 or 13 of them; in bounds: the arrays hold every
// level).  A branch per level instead kept 48 zeroed registers alive across the loads.
__device__ __forceinline__ int last_point(int64_t n, int64_t first) { return n - first < 32 ? (int)(n - first) - 1 : 31; }

template <int D, bool WIDE>
__device__ __forceinline__ v16f load_levels_tile(const float* __restrict__ src, int64_t n, int64_t first, int active, int j, int h) {
    v16f x = zero16();
    const f2v* tile = reinterpret_cast<const f2v*>(src) + first;
    typedef LaneOffset<WIDE> Offset;
    const int64_t plane = again(n);
    const int last = last_point(n, first);
    const Offset off = (Offset)8 * min(j, last), upper = again(h ? (Offset)16 * (Offset)n : (Offset)0);
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bool on = 4 * g + 2 * h + u < active;
            const f2v v = *lane_address(tile + (4 * g + u) * plane, off + (on ? upper : (Offset)0));
            x[4 * g + 2 * u] = on && j <= last ? v.x : 0.f;
            x[4 * g + 2 * u + 1] = on && j <= last ? v.y : 0.f;
        }
    return x;
}

template <int D, bool WIDE, bool STREAM>
__device__ __forceinline__ void store_levels_tile(float* __restrict__ dst, int64_t n, int64_t first, bool valid, const v16f& x, int j, int h) {
    if (!valid) return;
    f2v* tile = reinterpret_cast<f2v*>(dst) + first;
    typedef LaneOffset<WIDE> Offset;
    const int64_t plane = again(n);
    const Offset off = again((Offset)8 * ((Offset)j + (Offset)2 * (Offset)h * (Offset)n));
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const f2v v = {x[4 * g + 2 * u], x[4 * g + 2 * u + 1]};
            if (STREAM) __builtin_nontemporal_store(v, lane_address(tile + (4 * g + u) * plane, off));
            else *lane_address(tile + (4 * g + u) * plane, off) = v;
        }
}

// (de/dx)^T dL/de of the tile's points: this lane's levels
template <int D, bool WIDE, bool STREAM>
__device__ __forceinline__ void contract_jac_tile(const float* __restrict__ jac, int64_t n, int64_t first, int active, int j, int h,
                                                  const v16f& x, float out[3]) {
    out[0] = out[1] = out[2] = 0.f;
    const f2v* tile = reinterpret_cast<const f2v*>(jac) + first;
    typedef LaneOffset<WIDE> Offset;
    const int64_t plane = again(n);
    const int last = last_point(n, first);
    const Offset off = (Offset)8 * min(j, last), upper = again(h ? (Offset)48 * (Offset)n : (Offset)0);
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bool on = 4 * g + 2 * h + u < active;
            f2v J[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const f2v* p = lane_address(tile + (3 * (4 * g + u) + c) * plane, off + (on ? upper : (Offset)0));
                J[c] = STREAM ? __builtin_nontemporal_load(p) : *p;
            }
            const float x0 = x[4 * g + 2 * u], x1 = x[4 * g + 2 * u + 1];
            out[0] += on ? x0 * J[0].x + x1 * J[1].y : 0.f;
            out[1] += on ? x0 * J[0].y + x1 * J[2].x : 0.f;
            out[2] += on ? x0 * J[1].x + x1 * J[2].y : 0.f;
        }
}

// t_0 = (de/dx) dL/dn of the tile's points
template <int D, bool WIDE>
__device__ __forceinline__ v16f apply_jac_tile(const float* __restrict__ jac, int64_t n, int64_t first, int active, int j, int h,
                                               const float v[3]) {
    f2v J[D / 4][3];           // (J00,J01) (J02,J10) (J11,J12) per level of this lane
    const f2v* tile = reinterpret_cast<const f2v*>(jac) + first;
    typedef LaneOffset<WIDE> Offset;
    const int64_t plane = again(n);
    const int last = last_point(n, first);
    const Offset off = (Offset)8 * min(j, last), upper = again(h ? (Offset)48 * (Offset)n : (Offset)0);
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bool on = 4 * g + 2 * h + u < active;
            const Offset o = off + (on ? upper : (Offset)0);
#pragma unroll
            for (int c = 0; c < 3; ++c) J[2 * g + u][c] = __builtin_nontemporal_load(lane_address(tile + (3 * (4 * g + u) + c) * plane, o));
        }
    v16f t = zero16();
#pragma unroll
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bool on = 4 * g + 2 * h + u < active && j <= last;
            const f2v a = J[2 * g + u][0], b = J[2 * g + u][1], c = J[2 * g + u][2];
            const float t0 = a.x * v[0] + a.y * v[1] + b.x * v[2], t1 = b.y * v[0] + c.x * v[1] + c.y * v[2];
            t[4 * g + 2 * u] = on ? t0 : 0.f;
            t[4 * g + 2 * u + 1] = on ? t1 : 0.f;
        }
    return t;
}

// G: groups of four levels that are read (those with an active one); WIDE: from kTileMaxPoints points on
template <int D, int K, int G, bool WIDE>
__global__ __launch_bounds__(kFwdThreads) void sdf_fwd_kernel(SdfArgs a) {
    __shared__ SdfWeights<D, K, false> w;
    load_weights<D, K, false, kFwdThreads>(w, a);
    constexpr int KS1 = SdfWeights<D, K, false>::KS1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // the same for all lanes: keeps tile indices and addresses scalar
    const int j = lane & 31, h = lane >> 5;
    const int64_t tiles = (a.n + 31) / 32;
    const int64_t stride = (int64_t)gridDim.x * kFwdWaves;
    // tiles go to the workgroups first and then to their wavefronts: a small batch has every compute unit at work
    for (int64_t tile = (int64_t)wave * gridDim.x + blockIdx.x; tile < tiles; tile += stride) {
        const bool valid = tile * 32 + j < a.n;
        v16f x0[1] = {load_levels_tile<8 * G, WIDE>(a.enc, a.n, tile * 32, a.active_levels, j, h)};
        v16f a1[2], yv[1];
        Split<1, 3> px;
        Split<2, 3> pv;
        split(x0, px);
        matvec_split<2, (8 * G + 15) / 16, 3, 3, KS1>(w.H1f, px, a1, lane);
        const uint32_t m1 = relu_mask<2>(a1);
        uint32_t m_last = m1;
        split(a1, pv);
        if (K == 3) {
            v16f a2[2];
            matvec_split<2, 4, 3, 3>(w.H2f, pv, a2, lane);
            m_last = relu_mask<2>(a2);
            split(a2, pv);
        }
        matvec_split<1, 4, 3, 3>(w.HLf, pv, yv, lane);
        if (valid) {
            float4* row = lane_address(reinterpret_cast<float4*>(a.y) + tile * 128, 64u * j + 16u * h);
            row[0] = make_float4(yv[0][0], yv[0][1], yv[0][2], yv[0][3]);
            row[2] = make_float4(yv[0][4], yv[0][5], yv[0][6], yv[0][7]);
            if (a.masks) {
                uint32_t* words = a.masks + tile * 64;
                *lane_address(words, 8u * j + 4u * h) = m1;
                if (K == 3) *lane_address(words + 2 * a.n, 8u * j + 4u * h) = m_last;
            }
        }
        // reverse sweep for dd/de
        v16f s1[2];
        last_row_masked(w.HLrow0, m_last, h, pv);
        if (K == 3) {
            matvec_split<2, 4, 3, 3>(w.H2t, pv, s1, lane);
            apply_mask<2>(s1, m1);
            split(s1, pv);
        }
        v16f qv[1];
        matvec_split<1, 4, 3, 3>(w.H1t, pv, qv, lane);
        // dd/de is read next by the scatter-add, four kernels later: for a batch whose per-point arrays
        // exceed the caches it is written with non-temporal stores (25 us of the step at 2^20 points; at
        // 2^18 points the cached store is the faster one)
        if (a.stream_q) store_levels_tile<D, WIDE, true>(a.q, a.n, tile * 32, valid, qv[0], j, h);
        else store_levels_tile<D, WIDE, false>(a.q, a.n, tile * 32, valid, qv[0], j, h);
        float nrm[3];
        contract_jac_tile<8 * G, WIDE, true>(a.jac, a.n, tile * 32, a.active_levels, j, h, qv[0], nrm);
#pragma unroll
        for (int c = 0; c < 3; ++c) nrm[c] += __shfl_xor(nrm[c], 32);
        if (valid && h == 0) {
            float* out = lane_address(a.normal + tile * 96, 12u * j);
            out[0] = nrm[0]; out[1] = nrm[1]; out[2] = nrm[2];
        }
    }
}

// ------------------------------------------------------------------------------------------
// The SDF value alone (a refresh of the occupancy grid wants no normals): the forward kernel's arithmetic without its
// reverse sweep, 128 bytes of input a point instead of 512 and 4 of output instead of 220.  Four wavefronts per SIMD.
// 2^20 points: 73 us, the forward kernel 177.
template <int D, int K>
struct SdfValueWeights {
    typedef SplitMatrix<D / 16, 3> M1;
    typedef SplitMatrix<4, 3> M2;
    alignas(16) unsigned char H1[64 * M1::kLd];
    alignas(16) unsigned char H2[K == 3 ? 64 * M2::kLd : 16];
    alignas(16) unsigned char HL[32 * M2::kLd];
};

template <int D, int K>
__global__ __launch_bounds__(kValueThreads, 4) void sdf_value_kernel(SdfArgs a) {
    typedef SdfValueWeights<D, K> W;
    __shared__ W w;
    {
        typename W::M1::template Fill<64, kValueThreads, false> f1;
        typename W::M2::template Fill<K == 3 ? 64 : 0, kValueThreads, false> f2;
        typename W::M2::template Fill<32, kValueThreads, false> fl;
        const float* __restrict__ H1 = a.H[0];
        const float* __restrict__ H2 = a.H[1];
        const float* __restrict__ HL = a.H[K - 1];
        f1.load(threadIdx.x, [&](int o, int i) { return H1[o * D + i]; });
        f2.load(threadIdx.x, [&](int o, int i) { return H2[o * 64 + i]; });
        fl.load(threadIdx.x, [&](int o, int i) { return o < 16 ? HL[o * 64 + i] : 0.f; });
        f1.store(w.H1, threadIdx.x);
        f2.store(w.H2, threadIdx.x);
        fl.store(w.HL, threadIdx.x);
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 31, h = lane >> 5;
    const int64_t tiles = (a.n + 31) / 32;
    for (int64_t tile = (int64_t)blockIdx.x * kValueWaves + wave; tile < tiles; tile += (int64_t)gridDim.x * kValueWaves) {
        const int64_t i = tile * 32 + j;
        const bool valid = i < a.n;
        v16f x0[1] = {load_levels<D>(a.enc, a.n, i, valid, a.active_levels, h)};
        v16f z[2], yv[1];
        Split<1, 3> px;
        Split<2, 3> pv;
        split(x0, px);
        matvec_split<2, D / 16, 3, 3>(w.H1, px, z, lane);
        relu<2>(z);
        split(z, pv);
        if (K == 3) {
            matvec_split<2, 4, 3, 3>(w.H2, pv, z, lane);
            relu<2>(z);
            split(z, pv);
        }
        matvec_split<1, 4, 3, 3>(w.HL, pv, yv, lane);
        if (valid && h == 0) a.y[i] = yv[0][0];
    }
}

// ------------------------------------------------------------------------------------------
template <int D, int K>
struct SdfBwdSmem {
    SdfWeights<D, K, true> w;
    float tiles[kWaves][2][kTileWords];
};

// Without masks from the forward kernel: the forward pass is recomputed in the forward kernel's own arithmetic, which
// yields the same masks bit for bit, and one wavefront carries a tile through both orders.
template <int D, int K>
__global__ __launch_bounds__(kThreads) void sdf_bwd_kernel(SdfArgs a) {
    __shared__ SdfBwdSmem<D, K> sm;
    SdfWeights<D, K, true>& w = sm.w;
    load_weights<D, K, true, kThreads>(w, a);
    constexpr int KS1 = SdfWeights<D, K, true>::KS1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // the same for all lanes: keeps tile indices and addresses scalar
    const int j = lane & 31, h = lane >> 5;
    float* Zt = sm.tiles[wave][0];
    float* Xt = sm.tiles[wave][1];
    uint32_t* Zs = reinterpret_cast<uint32_t*>(Zt);     // the same tiles in the transposed split layout
    uint32_t* Xs = reinterpret_cast<uint32_t*>(Xt);

    v16f G1[2][1], G2[2][2], tsum[2];
    v4f GL[4];                 // gradient of the last matrix [16][64]: four blocks of 16 columns
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        G1[mb][0] = zero16();
        G2[mb][0] = zero16(); G2[mb][1] = zero16();
        tsum[mb] = zero16();
    }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) GL[cb] = v4f{0.f, 0.f, 0.f, 0.f};

    const int64_t tiles = (a.n + 31) / 32;
    const int64_t stride = (int64_t)gridDim.x * kWaves;
    int64_t tile = (int64_t)blockIdx.x * kWaves + wave;
    // every global input of a tile is requested at its top (the next tile's encoding as well),
    // so that HBM latency hides behind the matrix work
    v16f x_next = load_levels<D>(a.enc, a.n, tile * 32 + j, tile < tiles && tile * 32 + j < a.n, a.active_levels, h);
    for (; tile < tiles; tile += stride) {
        const int64_t i = tile * 32 + j;
        const bool valid = i < a.n;
        v16f x0[1] = {x_next};
        v16f dK[1] = {zero16()};
        if (valid) {
            typedef float f4v __attribute__((ext_vector_type(4)));
            const f4v a_ = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(a.d_y + i * 16 + 4 * h));
            const f4v b_ = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(a.d_y + i * 16 + 8 + 4 * h));
            dK[0][0] = a_.x; dK[0][1] = a_.y; dK[0][2] = a_.z; dK[0][3] = a_.w;
            dK[0][4] = b_.x; dK[0][5] = b_.y; dK[0][6] = b_.z; dK[0][7] = b_.w;
        }
        uint32_t m1, m_last;
        float nb3[3] = {0.f, 0.f, 0.f};
        if (valid) { nb3[0] = a.d_normal[3 * i]; nb3[1] = a.d_normal[3 * i + 1]; nb3[2] = a.d_normal[3 * i + 2]; }
        const JacRegs<D> J = load_jac<D>(a.jac, a.n, i, valid, a.active_levels, h);
        {
            const int64_t in = (tile + stride) * 32 + j;
            x_next = load_levels<D>(a.enc, a.n, in, tile + stride < tiles && in < a.n, a.active_levels, h);
        }
        // ---- forward pass again
        constexpr int PF = 3;
        v16f a1[2], a2[2];
        Split<1, PF> px;         // x0: input of the first layer, factor of its weight gradient
        Split<2, PF> p1;         // a1 likewise for the second layer
        split(x0, px);
        matvec_split<2, KS1, 3, PF>(w.H1f, px, a1, lane);
        m_last = m1 = relu_mask<2>(a1);
        split(a1, p1);
        if (K == 3) {
            matvec_split<2, 4, 3, PF>(w.H2f, p1, a2, lane);
            m_last = relu_mask<2>(a2);
        }
        // t_0 = (de/dx) dL/dn, computed now so that the Jacobian's registers are free again
        v16f t0[1] = {apply_jac_regs<D>(J, nb3)};
        // ---- first-order chain delta_K .. delta_1 (two terms, three products from here on),
        // weight gradients as they appear
        v16f d2[2], d1[2];
        Split<1, 2> pk;
        Split<2, 2> pd;
        stage<1, kLd64>(Zt, dK, j, h);
        stage<2, kLd64>(Xt, K == 3 ? a2 : a1, j, h);
        wave_lds_fence();
        outer_accumulate16<2, kLd64, kLd64>(GL, Zt, Xt, lane);
        split(dK, pk);
        matvec_split<2, 1, 2, 2>(w.HLt, pk, d2, lane);
        apply_mask<2>(d2, m_last);
        if (K == 3) {
            split(d2, pd);
            wave_lds_fence();
            stage_split(Zs, pd, j, h);
            stage_split(Xs, p1, j, h);
            wave_lds_fence();
            outer_accumulate_split<2, 2>(G2, Zs, Xs, lane);
            matvec_split<2, 4, 2, 2>(w.H2t, pd, d1, lane);
            apply_mask<2>(d1, m1);
        } else {
            d1[0] = d2[0]; d1[1] = d2[1];
        }
        split(d1, pd);
        wave_lds_fence();
        stage_split(Zs, pd, j, h);
        stage_split(Xs, px, j, h);
        wave_lds_fence();
        outer_accumulate_split<2, 1>(G1, Zs, Xs, lane);
        v16f de[1];
        matvec_split<1, 4, 2, 2>(w.H1t, pd, de, lane);
        if (a.stream_q) store_levels<D, true>(a.d_enc, a.n, i, valid, de[0], h);      // as for q in the forward kernel
        else store_levels<D>(a.d_enc, a.n, i, valid, de[0], h);
        if (a.d_pos) {
            float dp[3];
            contract_jac<D>(a.jac, a.n, i, valid, a.active_levels, h, de[0], dp);
#pragma unroll
            for (int c = 0; c < 3; ++c) dp[c] += __shfl_xor(dp[c], 32);
            if (valid && h == 0) {
                a.d_pos[3 * i + 0] += dp[0]; a.d_pos[3 * i + 1] += dp[1]; a.d_pos[3 * i + 2] += dp[2];
            }
        }
        // ---- second order: S sweep (reverse) and t sweep (forward mode), Theorem 1
        v16f s1[2];
        Split<2, 2> ps2;
        Split<1, 2> pt;
        last_row_masked(w.HLrow0, m_last, h, ps2);
        if (K == 3) {
            matvec_split<2, 4, 2, 2>(w.H2t, ps2, s1, lane);
            apply_mask<2>(s1, m1);
            split(s1, pd);
        } else {
            pd = ps2;
        }
        split(t0, pt);
        wave_lds_fence();
        stage_split(Zs, pd, j, h);
        stage_split(Xs, pt, j, h);
        wave_lds_fence();
        outer_accumulate_split<2, 1>(G1, Zs, Xs, lane);
        v16f t1[2], t2[2];
        matvec_split<2, KS1, 3, 2>(w.H1f, pt, t1, lane);
        apply_mask<2>(t1, m1);
        if (K == 3) {
            split(t1, pd);
            wave_lds_fence();
            stage_split(Zs, ps2, j, h);
            stage_split(Xs, pd, j, h);
            wave_lds_fence();
            outer_accumulate_split<2, 2>(G2, Zs, Xs, lane);
            matvec_split<2, 4, 3, 2>(w.H2f, pd, t2, lane);
            apply_mask<2>(t2, m_last);
            tsum[0] += t2[0]; tsum[1] += t2[1];
        } else {
            tsum[0] += t1[0]; tsum[1] += t1[1];
        }
        wave_lds_fence();
    }
    // S_K is the unit row selecting the SDF output: row 0 of the last matrix's gradient gets
    // the sum of t_{K-1} over points.  One outer product with a one-hot factor does the
    // cross-lane sum of the per-lane partials.
    {
        v16f onehot[1] = {zero16()};
        if (h == 0) onehot[0][0] = 1.f;
        stage<1, kLd64>(Zt, onehot, j, h);
        stage<2, kLd64>(Xt, tsum, j, h);
        wave_lds_fence();
        outer_accumulate16<2, kLd64, kLd64>(GL, Zt, Xt, lane);
    }
    __syncthreads();
    // ---- the block's sums go to global memory in the gradients' own order
    float* scratch = reinterpret_cast<float*>(&sm);
    constexpr int kVecs = K == 3 ? 7 : 3;
    static_assert(sizeof(sm) >= kWaves * kVecs * 1024 * sizeof(float), "scratch for the block sum");
    v16f gl;                   // the four 16-column blocks of GL side by side
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) gl[4 * cb + v] = GL[cb][v];
    if constexpr (K == 3) {
        const v16f* const all[7] = {&G1[0][0], &G1[1][0], &gl, &G2[0][0], &G2[0][1], &G2[1][0], &G2[1][1]};
        block_store<7>(scratch, all, wave, lane);
    } else {
        const v16f* const all[3] = {&G1[0][0], &G1[1][0], &gl};
        block_store<3>(scratch, all, wave, lane);
    }
    __syncthreads();
    constexpr int kOf1 = 64 * D, kOf2 = K == 3 ? 64 * 64 : 0, kOfL = 16 * 64;
    constexpr int kChunks = (kOf1 + kOf2 + kOfL) / kThreads;
    static_assert((kOf1 + kOf2 + kOfL) % kThreads == 0, "whole chunks");
    for (int k = 0; k < kChunks; ++k) {
        const int x = rotated_chunk<kChunks>(k) * kThreads + threadIdx.x;
        if (x < kOf1) {
            atomicAdd(a.dH[0] + x, block_element<kWaves, kVecs, 1>(scratch, 0, x / D, x % D));
        } else if (x < kOf1 + kOf2) {
            const int e = x - kOf1;
            atomicAdd(a.dH[1] + e, block_element<kWaves, kVecs, 2>(scratch, 3, e >> 6, e & 63));
        } else {
            const int e = x - kOf1 - kOf2;
            atomicAdd(a.dH[K - 1] + e, block_element16<kWaves, kVecs>(scratch, 2, e >> 6, e & 63));
        }
    }
}

// ------------------------------------------------------------------------------------------
// With the masks from the forward kernel (a.masks) the two orders of a tile have nothing in common but the masks: the
// first-order chain (activations, delta sweep) reads enc and dL/d(d,g), the second-order one (S and t sweeps) the
// Jacobian and dL/dn.  So two wavefronts share a tile, one per order, and each needs only its own working registers beside
// its copy of the weight gradients: 256 registers instead of 512, eight wavefronts a workgroup, two per SIMD (waves w and
// w + 4 share a SIMD, so every SIMD holds one of each), and one's waits for LDS, memory and matrix results are filled by
// the other.  The chains are about equally long: 114 and 96 matrix instructions of 32 clocks.
// Everything that depends on the lane alone (its offsets into LDS and into the arrays) is worked out again for every tile:
// kept through the loop those values took 31 registers that were not there, and fetching them back from memory was 20 % of
// the time (2^18 points 105 -> 84 us, 2^20 points 318 -> 270).
// Everything here is at gradient tolerance: two terms and three products, a plain ReLU for the recomputed
// activations (where its sign differs from the given mask the value is within rounding of zero).
constexpr int kPairThreads = 512;
constexpr int kPairs = kPairThreads / 128;        // tiles a workgroup works on

template <int D, int K>
struct SdfPairSmem {
    SdfWeights<D, K, true, 2> w;
    alignas(16) unsigned char tiles[2 * kPairs][kTilesPerWave * kBlockTile];
};

template <int D, int K, int G, bool WIDE>
__device__ __forceinline__ void sdf_first_order(const SdfArgs& a, const SdfWeights<D, K, true, 2>& w, unsigned char* tile_mem,
                                                int slot, int lane_in, v16f (*G1)[1], v16f (*G2)[2], v4f* GL) {
    constexpr int KS1 = D / 16;
    float* Xt = reinterpret_cast<float*>(tile_mem);
    float* Zt = Xt + 32 * kLd64;
    static_assert((32 * kLd64 + 32 * kLd16) * 4 <= kTilesPerWave * kBlockTile, "fp32 tiles fit the wave's memory");
    const int64_t tiles = (a.n + 31) / 32;
    const int64_t stride = (int64_t)gridDim.x * kPairs;
    for (int64_t tile = (int64_t)blockIdx.x * kPairs + slot; tile < tiles; tile += stride) {
        const int lane = (int)again((uint32_t)lane_in), j = lane & 31, h = lane >> 5;
        const int64_t i = tile * 32 + j;
        const bool valid = i < a.n;
        v16f x0[1] = {load_levels_tile<8 * G, WIDE>(a.enc, a.n, tile * 32, a.active_levels, j, h)};
        v16f dK[1] = {zero16()};
        uint32_t m1 = 0u, m_last = 0u;
        if (valid) {
            // read here for the last time in the step: non-temporal loads
            typedef float f4v __attribute__((ext_vector_type(4)));
            const f4v* row = lane_address(reinterpret_cast<const f4v*>(a.d_y) + tile * 128, 64u * j + 16u * h);
            const f4v a_ = __builtin_nontemporal_load(row), b_ = __builtin_nontemporal_load(row + 2);
            dK[0][0] = a_.x; dK[0][1] = a_.y; dK[0][2] = a_.z; dK[0][3] = a_.w;
            dK[0][4] = b_.x; dK[0][5] = b_.y; dK[0][6] = b_.z; dK[0][7] = b_.w;
            const uint32_t* words = a.masks + tile * 64;
            m1 = *lane_address(words, 8u * j + 4u * h);
            m_last = K == 3 ? *lane_address(words + 2 * a.n, 8u * j + 4u * h) : m1;
        }
        v16f a1[2], a2[2], d2[2], d1[2], de[1];
        Split<1, 2> px, pk;      // x0: input of the first layer, factor of its weight gradient
        Split<2, 2> p1, pd;      // a1 likewise for the second layer
        split(x0, px);
        matvec_split<2, (8 * G + 15) / 16, 2, 2, KS1>(w.H1f, px, a1, lane);
        relu<2>(a1);
        if (K == 3) {
            split(a1, p1);
            matvec_split<2, 4, 2, 2>(w.H2f, p1, a2, lane);
            relu<2>(a2);
        }
        wave_lds_fence();
        stage16<kLd16>(Zt, dK[0], j, h);
        stage<2, kLd64>(Xt, K == 3 ? a2 : a1, j, h);
        wave_lds_fence();
        outer_accumulate16<2, kLd16, kLd64>(GL, Zt, Xt, lane);
        split(dK, pk);
        matvec_split<2, 1, 2, 2>(w.HLt, pk, d2, lane);
        apply_mask<2>(d2, m_last);
        if (K == 3) {
            split(d2, pd);
            outer_accumulate_points<2, 2>(G2, pd, p1, tile_mem, lane);
            matvec_split<2, 4, 2, 2>(w.H2t, pd, d1, lane);
            apply_mask<2>(d1, m1);
        } else {
            d1[0] = d2[0]; d1[1] = d2[1];
        }
        split(d1, pd);
        outer_accumulate_points<2, 1>(G1, pd, px, tile_mem, lane);
        matvec_split<1, 4, 2, 2>(w.H1t, pd, de, lane);
        if (a.stream_q) store_levels_tile<D, WIDE, true>(a.d_enc, a.n, tile * 32, valid, de[0], j, h);      // as for q in the forward kernel
        else store_levels_tile<D, WIDE, false>(a.d_enc, a.n, tile * 32, valid, de[0], j, h);
        if (a.d_pos) {
            float dp[3];
            contract_jac_tile<8 * G, WIDE, false>(a.jac, a.n, tile * 32, a.active_levels, j, h, de[0], dp);
#pragma unroll
            for (int c = 0; c < 3; ++c) dp[c] += __shfl_xor(dp[c], 32);
            if (valid && h == 0) {
                a.d_pos[3 * i + 0] += dp[0]; a.d_pos[3 * i + 1] += dp[1]; a.d_pos[3 * i + 2] += dp[2];
            }
        }
    }
}

template <int D, int K, int G, bool WIDE>
__device__ __forceinline__ void sdf_second_order(const SdfArgs& a, const SdfWeights<D, K, true, 2>& w, unsigned char* tile_mem,
                                                 int slot, int lane_in, v16f (*G1)[1], v16f (*G2)[2], v4f* GL) {
    constexpr int KS1 = D / 16;
    v16f tsum[2] = {zero16(), zero16()};
    const int64_t tiles = (a.n + 31) / 32;
    const int64_t stride = (int64_t)gridDim.x * kPairs;
    for (int64_t tile = (int64_t)blockIdx.x * kPairs + slot; tile < tiles; tile += stride) {
        const int lane = (int)again((uint32_t)lane_in), j = lane & 31, h = lane >> 5;
        const int64_t i = tile * 32 + j;
        const bool valid = i < a.n;
        uint32_t m1 = 0u, m_last = 0u;
        float nb3[3] = {0.f, 0.f, 0.f};
        if (valid) {
            const uint32_t* words = a.masks + tile * 64;
            m1 = *lane_address(words, 8u * j + 4u * h);
            m_last = K == 3 ? *lane_address(words + 2 * a.n, 8u * j + 4u * h) : m1;
            const float* nb = lane_address(a.d_normal + tile * 96, 12u * j);
            nb3[0] = nb[0]; nb3[1] = nb[1]; nb3[2] = nb[2];
        }
        // The t sweep first: of its vectors only t_0 outlives the product with S_{K-1}, and S_{K-1} does not outlive the
        // product that turns it into S_1.
        v16f t0[1] = {apply_jac_tile<8 * G, WIDE>(a.jac, a.n, tile * 32, a.active_levels, j, h, nb3)};
        v16f s1[2], t1[2], t2[2];
        Split<1, 2> pt;
        Split<2, 2> ps, pd;
        split(t0, pt);
        __builtin_amdgcn_sched_barrier(0);
        matvec_split<2, (8 * G + 15) / 16, 2, 2, KS1>(w.H1f, pt, t1, lane);
        apply_mask<2>(t1, m1);
        if (K == 3) {
            split(t1, pd);
            __builtin_amdgcn_sched_barrier(0);
            matvec_split<2, 4, 2, 2>(w.H2f, pd, t2, lane);
            apply_mask<2>(t2, m_last);
            tsum[0] += t2[0]; tsum[1] += t2[1];
            __builtin_amdgcn_sched_barrier(0);
            last_row_masked(w.HLrow0, again(m_last), h, ps);
            outer_accumulate_points<2, 2>(G2, ps, pd, tile_mem, lane);
            matvec_split<2, 4, 2, 2>(w.H2t, ps, s1, lane);
            apply_mask<2>(s1, again(m1));
            split(s1, ps);
        } else {
            tsum[0] += t1[0]; tsum[1] += t1[1];
            last_row_masked(w.HLrow0, m_last, h, ps);
        }
        outer_accumulate_points<2, 1>(G1, ps, pt, tile_mem, lane);
    }
    // S_K is the unit row selecting the SDF output: row 0 of the last matrix's gradient gets the sum of t_{K-1} over
    // points, through one outer product with a one-hot factor
    float* Xt = reinterpret_cast<float*>(tile_mem);
    float* Zt = Xt + 32 * kLd64;
    const int lane = lane_in, j = lane & 31, h = lane >> 5;
    v16f onehot = zero16();
    if (h == 0) onehot[0] = 1.f;
    wave_lds_fence();
    stage16<kLd16>(Zt, onehot, j, h);
    stage<2, kLd64>(Xt, tsum, j, h);
    wave_lds_fence();
    outer_accumulate16<2, kLd16, kLd64>(GL, Zt, Xt, lane);
}

template <int D, int K, int G, bool WIDE>
__global__ __launch_bounds__(kPairThreads) void sdf_bwd_pair_kernel(SdfArgs a) {
    __shared__ SdfPairSmem<D, K> sm;
    load_weights<D, K, true, kPairThreads, 2>(sm.w, a);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // the same for all lanes: keeps tile indices and addresses scalar
    const int slot = wave % kPairs;
    const bool second = wave >= kPairs;
    v16f G1[2][1], G2[2][2];
    v4f GL[4];                 // gradient of the last matrix [16][64]: four blocks of 16 columns
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        G1[mb][0] = zero16();
        G2[mb][0] = zero16(); G2[mb][1] = zero16();
    }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) GL[cb] = v4f{0.f, 0.f, 0.f, 0.f};
    if (second) sdf_second_order<D, K, G, WIDE>(a, sm.w, sm.tiles[wave], slot, lane, G1, G2, GL);
    else sdf_first_order<D, K, G, WIDE>(a, sm.w, sm.tiles[wave], slot, lane, G1, G2, GL);
    __syncthreads();
    // ---- the waves of the second order leave their sums in LDS, their partners add their own, and the block's sums go
    // to global memory in the gradients' own order
    float* scratch = reinterpret_cast<float*>(&sm);
    constexpr int kVecs = K == 3 ? 7 : 3;
    static_assert(sizeof(sm) >= kPairs * kVecs * 1024 * sizeof(float), "scratch for the block sum");
    v16f gl;                   // the four 16-column blocks of GL side by side
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) gl[4 * cb + v] = GL[cb][v];
    const v16f* all[kVecs];
    all[0] = &G1[0][0]; all[1] = &G1[1][0]; all[2] = &gl;
    if constexpr (K == 3) { all[3] = &G2[0][0]; all[4] = &G2[0][1]; all[5] = &G2[1][0]; all[6] = &G2[1][1]; }
    float* own = scratch + slot * kVecs * 1024 + lane;
    if (second) {
#pragma unroll
        for (int k = 0; k < kVecs; ++k)
#pragma unroll
            for (int r = 0; r < 16; ++r) own[(k * 16 + r) * 64] = (*all[k])[r];
    }
    __syncthreads();
    if (!second) {
#pragma unroll
        for (int k = 0; k < kVecs; ++k)
#pragma unroll
            for (int r = 0; r < 16; ++r) own[(k * 16 + r) * 64] += (*all[k])[r];
    }
    __syncthreads();
    constexpr int kOf1 = 64 * D, kOf2 = K == 3 ? 64 * 64 : 0, kOfL = 16 * 64;
    constexpr int kChunks = (kOf1 + kOf2 + kOfL) / kPairThreads;
    static_assert((kOf1 + kOf2 + kOfL) % kPairThreads == 0, "whole chunks");
    for (int k = 0; k < kChunks; ++k) {
        const int x = rotated_chunk<kChunks>(k) * kPairThreads + threadIdx.x;
        if (x < kOf1) {
            atomicAdd(a.dH[0] + x, block_element_points<kPairs, kVecs, 1>(scratch, 0, x / D, x % D));
        } else if (x < kOf1 + kOf2) {
            const int e = x - kOf1;
            atomicAdd(a.dH[1] + e, block_element_points<kPairs, kVecs, 2>(scratch, 3, e >> 6, e & 63));
        } else {
            const int e = x - kOf1 - kOf2;
            atomicAdd(a.dH[K - 1] + e, block_element16<kPairs, kVecs>(scratch, 2, e >> 6, e & 63));
        }
    }
}

typedef void (*SdfKernel)(SdfArgs);

// The variant that reads the groups of levels with an active one, from kTileMaxPoints points on the one that reads all.  With
// one variant for all, levels that the training step leaves unwritten were fetched (half of the levels active, 2^20 points,
// forward and backward: 169 and 251 us, now 155 and 243); picking level 0 for them in scalar registers, or a branch round
// every load, cost up to 6 % forward and 8 % backward with all levels active.
template <int D, int K>
SdfKernel fwd_kernel(const SdfArgs& a) {
    if (a.n >= kTileMaxPoints) return sdf_fwd_kernel<D, K, D / 8, true>;
    if (a.active_levels <= 4) return sdf_fwd_kernel<D, K, 1, false>;
    if (D == 16 || a.active_levels <= 8) return sdf_fwd_kernel<D, K, 2, false>;
    return a.active_levels <= 12 ? sdf_fwd_kernel<D, K, D == 32 ? 3 : 2, false> : sdf_fwd_kernel<D, K, D / 8, false>;
}

template <int D, int K>
SdfKernel bwd_kernel(const SdfArgs& a) {
    if (a.n >= kTileMaxPoints) return sdf_bwd_pair_kernel<D, K, D / 8, true>;
    if (a.active_levels <= 4) return sdf_bwd_pair_kernel<D, K, 1, false>;
    if (D == 16 || a.active_levels <= 8) return sdf_bwd_pair_kernel<D, K, 2, false>;
    return a.active_levels <= 12 ? sdf_bwd_pair_kernel<D, K, D == 32 ? 3 : 2, false> : sdf_bwd_pair_kernel<D, K, D / 8, false>;
}

template <int D, int K>
int run_fwd(const SdfArgs& a, hipStream_t st) {
    const int64_t tiles = (a.n + 31) / 32;
    const SdfKernel kernel = fwd_kernel<D, K>(a);
    const int blocks = persistent_blocks((const void*)kernel, kFwdThreads, tiles);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kFwdThreads), 0, st, a);
    return check_launch("sdf forward");
}

template <int D, int K>
int run_values(const SdfArgs& a, hipStream_t st) {
    const int64_t tiles = (a.n + 31) / 32;
    const int blocks = persistent_blocks((const void*)sdf_value_kernel<D, K>, kValueThreads, (tiles + kValueWaves - 1) / kValueWaves);
    hipLaunchKernelGGL((sdf_value_kernel<D, K>), dim3(blocks), dim3(kValueThreads), 0, st, a);
    return check_launch("sdf values");
}

template <int D, int K>
int run_bwd(const SdfArgs& a, hipStream_t st) {
    const int64_t tiles = (a.n + 31) / 32;
    if (a.masks) {
        const SdfKernel kernel = bwd_kernel<D, K>(a);
        const int blocks = persistent_blocks((const void*)kernel, kPairThreads, (tiles + kPairs - 1) / kPairs);
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kPairThreads), 0, st, a);
    } else {
        const int blocks = persistent_blocks((const void*)sdf_bwd_kernel<D, K>, kThreads, (tiles + kWaves - 1) / kWaves);
        hipLaunchKernelGGL((sdf_bwd_kernel<D, K>), dim3(blocks), dim3(kThreads), 0, st, a);
    }
    return check_launch("sdf backward");
}

// ------------------------------------------------------------------------------------------
// Networks deeper than the fused kernels hold (up to eight hidden layers of 64: the depths of the
// paper's Fig. 7), in runs of consecutive layers: a launch keeps the matrices of its run in LDS (six of three terms at
// most) and a tile's vectors in registers from layer to layer; between launches they pass through a workspace in HBM.
// One layer a launch instead, each lane writing its 32 registers as 128 consecutive bytes, moved 4.2 GB where 2.2 are
// needed, every access instruction in 64 cache lines: eight hidden layers at 2^17 points, forward and backward, took
// 1243 us, runs of layers 617 and without spilled registers 556.  Bound by the vectors that the backward call stores and
// reads back.
// Every matrix is stored as 64 x 64 (the first one's missing columns and the last one's missing rows are zeros; the products leave
// their k-steps and blocks of rows out), so one kernel serves every layer.
//   forward run:   a_l = G_l H_l a_{l-1}  (six-product arithmetic, writes the mask words)
//                  t_l = G_l H_l t_{l-1}  (WITH_T; t_0 = (de/dx) dL/dn)
//   reverse run:   S_{l-1} = (H_l^T S_l) G_{l-1}, down to dd/de and the normal
//   gradient run:  dH_l += delta_l a_{l-1}^T + S_l^T t_{l-1}^T
//                  S_{l-1} as above, delta_{l-1} = G_{l-1} H_l^T delta_l
// with S_K = the unit row of the SDF output and delta_K = dL/d(d,g): Theorem 1 and Eqs. 7-8 as in
// the fused kernels, Definition 1's vectors.
constexpr int kDeepThreads = 512;                  // two wavefronts per SIMD: one's memory waits under the other's products
constexpr int kDeepWaves = kDeepThreads / 64;
constexpr int kDeepRun = 6;                        // layers a run holds at most
constexpr int kDeepGradRun = 2;                    // of a gradient run: their sums take 64 registers a layer

// The workspace: vectors of 32 floats per lane, two lanes a point, in the order [tile][register quad][lane][4], so that
// an access instruction covers 1 KB on end: t_0, a_1, t_1, ..., a_{K-1}, t_{K-1}, two vectors that runs hand on (one of each
// order), then the mask words of the hidden layers [layer][tile * 64 + lane].  (a_0 is the encoding itself; the upper 16 of
// t_0's 32 registers are empty and left unwritten.)
struct DeepArgs {
    const float* H[NEUS2_DEEP_MAX_MATS];
    int n_mats, enc_dim;
    int first, count;                      // layers first .. first + count - 1 (numbered from 0); reverse kinds start at the last
    int64_t n, vec;                        // points; floats of a workspace vector
    float* ws;
    const float* enc; const float* jac; const float* d_normal; const float* d_y;
    float* y; float* q; float* normal; float* d_enc;
    float* dH[NEUS2_DEEP_MAX_MATS];

    __device__ __forceinline__ int in_dim(int l) const { return l == 0 ? enc_dim : 64; }
    __device__ __forceinline__ int out_dim(int l) const { return l == n_mats - 1 ? 16 : 64; }
    __device__ __forceinline__ float* a_vec(int l) const { return ws + (2 * l - 1) * vec; }          // l > 0
    __device__ __forceinline__ float* t_vec(int l) const { return ws + 2 * l * vec; }
    __device__ __forceinline__ float* passed(int k) const { return ws + (2 * n_mats - 1 + k) * vec; }
    __device__ __forceinline__ uint32_t* masks(int l, int64_t tile) const {
        return reinterpret_cast<uint32_t*>(ws + (2 * n_mats + 1) * vec) + ((int64_t)l * ((n + 31) / 32) + tile) * 64;
    }
};

template <int NB>
__device__ __forceinline__ void load_lane(const float* base, int64_t tile, int lane, v16f* v) {
    const float4* p = lane_address(reinterpret_cast<const float4*>(base) + tile * 512, 16u * lane);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (b >= NB) { v[b] = zero16(); continue; }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 f = p[64 * (4 * b + k)];
            v[b][4 * k] = f.x; v[b][4 * k + 1] = f.y; v[b][4 * k + 2] = f.z; v[b][4 * k + 3] = f.w;
        }
    }
}

template <int NB>
__device__ __forceinline__ void store_lane(float* base, int64_t tile, int lane, const v16f* v) {
    float4* p = lane_address(reinterpret_cast<float4*>(base) + tile * 512, 16u * lane);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int k = 0; k < 4; ++k) p[64 * (4 * b + k)] = make_float4(v[b][4 * k], v[b][4 * k + 1], v[b][4 * k + 2], v[b][4 * k + 3]);
}

// The matrices of layers l0, l0 + step, ... (COUNT at most, count of them) side by side in LDS; ROW_FASTEST: transposed.
// All are fetched before the first is stored.
template <int P, int COUNT, bool TRANSPOSED>
__device__ __forceinline__ void deep_matrices(const DeepArgs& a, int l0, int step, int count, unsigned char* mats) {
    typedef SplitMatrix<4, P> M;
    typename M::template Fill<64, kDeepThreads, TRANSPOSED> f[COUNT];
#pragma unroll
    for (int k = 0; k < COUNT; ++k) {
        if (k >= count) break;
        const int l = l0 + k * step, od = a.out_dim(l), id = a.in_dim(l);
        const float* __restrict__ W = a.H[l];
        f[k].load(threadIdx.x, [&](int r, int c) {
            const int o = TRANSPOSED ? c : r, i = TRANSPOSED ? r : c;
            return o < od && i < id ? W[o * id + i] : 0.f;
        });
    }
#pragma unroll
    for (int k = 0; k < COUNT; ++k) {
        if (k >= count) break;
        f[k].store(mats + k * 64 * M::kLd, threadIdx.x);
    }
    __syncthreads();
}

template <bool WITH_T>
__global__ __launch_bounds__(kDeepThreads) void deep_forward_kernel(DeepArgs a) {
    constexpr int kMatrix = 64 * SplitMatrix<4, 3>::kLd;
    __shared__ alignas(16) unsigned char mats[kDeepRun * kMatrix];
    deep_matrices<3, kDeepRun, false>(a, a.first, 1, a.count, mats);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 31, h = lane >> 5;
    const int64_t tiles = (a.n + 31) / 32;
    for (int64_t tile = (int64_t)blockIdx.x * kDeepWaves + wave; tile < tiles; tile += (int64_t)gridDim.x * kDeepWaves) {
        const int64_t i = tile * 32 + j;
        const bool valid = i < a.n;
        v16f x[2], t[2];
        if (a.first == 0) {
            x[0] = load_levels<32>(a.enc, a.n, i, valid, a.enc_dim / 2, h);
            x[1] = zero16();
            if (WITH_T) {
                float nb3[3] = {0.f, 0.f, 0.f};
                if (valid) { nb3[0] = a.d_normal[3 * i]; nb3[1] = a.d_normal[3 * i + 1]; nb3[2] = a.d_normal[3 * i + 2]; }
                t[0] = apply_jac<32>(a.jac, a.n, i, valid, a.enc_dim / 2, h, nb3);
                t[1] = zero16();
                store_lane<1>(a.t_vec(0), tile, lane, t);
            }
        } else {
            load_lane<2>(a.a_vec(a.first), tile, lane, x);
            if (WITH_T) load_lane<2>(a.t_vec(a.first), tile, lane, t);
        }
#pragma unroll 1
        for (int k = 0; k < a.count; ++k) {
            const int l = a.first + k;
            const unsigned char* W = mats + k * kMatrix;
            v16f z[2];
            Split<2, 3> px;
            split(x, px);
            uint32_t m = 0xffffffffu;
            if (l == a.n_mats - 1) {                             // 16 outputs: one block of rows
                matvec_split<1, 4, 3, 3>(W, px, z, lane);
                store_rows16(a.y, i, valid, h, z[0]);
                break;
            } else {
                if (l == 0) matvec_split<2, 2, 3, 3, 4>(W, px, z, lane);      // 32 inputs at most
                else matvec_split<2, 4, 3, 3>(W, px, z, lane);
                m = relu_mask<2>(z);
                if (WITH_T || k == a.count - 1) store_lane<2>(a.a_vec(l + 1), tile, lane, z);
                a.masks(l, tile)[lane] = m;
            }
            x[0] = z[0]; x[1] = z[1];
            if (WITH_T) {
                Split<2, 2> pt;
                split(t, pt);
                if (l == 0) matvec_split<2, 2, 3, 2, 4>(W, pt, t, lane);
                else matvec_split<2, 4, 3, 2>(W, pt, t, lane);
                apply_mask<2>(t, m);
                store_lane<2>(a.t_vec(l + 1), tile, lane, t);
            }
        }
    }
}

// dd/de and the normal (Eq. 2): S downwards from row 0 of the last matrix, three terms per factor (compared at forward tolerance),
// the transposed matrices of a run in LDS.  Forward call at 2^17 points: eight hidden layers 152 -> 141 us against a product with
// the last matrix too (two runs either way), six 119 -> 100 (one run instead of two), two 46 -> 40; sixteen wavefronts
// instead of eight spill 8 registers: 138, 100 and 41.  (Two scaled fp16 terms, whose eight matrices fit LDS at once, took 107, 82 and 38
// but lose the small elements of a vector or a matrix beside large ones.)
struct DeepReverseSmem {
    alignas(16) unsigned char mats[kDeepRun * 64 * SplitMatrix<4, 3>::kLd];
    alignas(16) float row0[2][32];                          // [lane half][16 b + r]
};

__global__ __launch_bounds__(kDeepThreads) void deep_reverse_kernel(DeepArgs a) {
    constexpr int kMatrix = 64 * SplitMatrix<4, 3>::kLd;
    __shared__ DeepReverseSmem sm;
    const bool from_top = a.first == a.n_mats - 2;
    if (from_top && threadIdx.x < 64) {
        const int k = threadIdx.x & 31;
        sm.row0[threadIdx.x >> 5][k] = a.H[a.n_mats - 1][32 * (k >> 4) + neuron_of(k & 15, threadIdx.x >> 5)];
    }
    deep_matrices<3, kDeepRun, true>(a, a.first, -1, a.count, sm.mats);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 31, h = lane >> 5;
    const int64_t tiles = (a.n + 31) / 32;
    for (int64_t tile = (int64_t)wave * gridDim.x + blockIdx.x; tile < tiles; tile += (int64_t)gridDim.x * kDeepWaves) {
        const int64_t i = tile * 32 + j;
        const bool valid = i < a.n;
        v16f s[2];
        if (from_top) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[b][r] = sm.row0[h][16 * b + r];
            apply_mask<2>(s, a.masks(a.n_mats - 2, tile)[lane]);
        } else {
            load_lane<2>(a.passed(0), tile, lane, s);
        }
        Split<2, 3> ps;
        const int products = a.first - a.count >= 0 ? a.count : a.count - 1;       // the first layer's has another end
#pragma unroll 1
        for (int k = 0; k < products; ++k) {
            const uint32_t m = a.masks(a.first - k - 1, tile)[lane];
            split(s, ps);
            matvec_split<2, 4, 3, 3>(sm.mats + k * kMatrix, ps, s, lane);
            apply_mask<2>(s, m);
        }
        if (products == a.count) {
            store_lane<2>(a.passed(0), tile, lane, s);
            continue;
        }
        v16f de[1];
        split(s, ps);
        matvec_split<1, 4, 3, 3>(sm.mats + products * kMatrix, ps, de, lane);
        store_levels_active(a.q, a.n, i, valid, a.enc_dim / 2, h, de[0]);
        float nrm[3];
        contract_jac<32>(a.jac, a.n, i, valid, a.enc_dim / 2, h, de[0], nrm);
#pragma unroll
        for (int c = 0; c < 3; ++c) nrm[c] += __shfl_xor(nrm[c], 32);
        if (valid && h == 0) { a.normal[3 * i] = nrm[0]; a.normal[3 * i + 1] = nrm[1]; a.normal[3 * i + 2] = nrm[2]; }
    }
}

// Both orders of a layer are the same work on other vectors (delta and a; S and t), so a wavefront takes one order of a
// tile at a time and keeps the weight gradients of LAYERS layers, both orders' together, in registers.
// What depends on the lane alone is worked out again for every layer: kept, it was 34 registers spilled (eight hidden layers
// at 2^17 points, forward and backward: 622 -> 556 us).
template <int LAYERS>
struct DeepGradSmem {
    alignas(16) unsigned char mats[LAYERS * 64 * SplitMatrix<4, 2>::kLd];
    alignas(16) unsigned char tiles[kDeepWaves][kTilesPerWave * kBlockTile];
};

template <int LAYERS>
__global__ __launch_bounds__(kDeepThreads) void deep_gradient_kernel(DeepArgs a) {
    constexpr int kMatrix = 64 * SplitMatrix<4, 2>::kLd;
    __shared__ DeepGradSmem<LAYERS> sm;
    deep_matrices<2, LAYERS, true>(a, a.first, -1, LAYERS, sm.mats);
    const int lane_in = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char* tile_mem = sm.tiles[wave];
    v16f G[LAYERS][2][2];
#pragma unroll
    for (int k = 0; k < LAYERS; ++k)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) { G[k][mb][0] = zero16(); G[k][mb][1] = zero16(); }
    const int64_t items = 2 * ((a.n + 31) / 32);
    for (int64_t item = (int64_t)blockIdx.x * kDeepWaves + wave; item < items; item += (int64_t)gridDim.x * kDeepWaves) {
        const int lane = (int)again((uint32_t)lane_in), j = lane & 31, h = lane >> 5;
        const int64_t tile = item >> 1;
        const bool second = item & 1;
        const int64_t i = tile * 32 + j;
        const bool valid = i < a.n;
        v16f z[2];
        if (a.first == a.n_mats - 1) {
            // S_K: the unit row of output 0; delta_K: the adjoint of the 16 outputs
            z[1] = zero16();
            if (second) {
                z[0] = zero16();
                if (h == 0 && valid) z[0][0] = 1.f;
            } else {
                z[0] = load_rows16(a.d_y, i, valid, h);
            }
        } else {
            load_lane<2>(a.passed(second), tile, lane, z);
        }
#pragma unroll
        for (int k = 0; k < LAYERS; ++k) {
            const int l = a.first - k;
            const int lane = (int)again((uint32_t)lane_in), j = lane & 31, h = lane >> 5;
            v16f x[2];
            uint32_t m = 0u;
            if (l > 0) {
                load_lane<2>(second ? a.t_vec(l) : a.a_vec(l), tile, lane, x);
                m = a.masks(l - 1, tile)[lane];
            } else if (second) {
                load_lane<1>(a.t_vec(0), tile, lane, x);
            } else {
                x[0] = load_levels<32>(a.enc, a.n, i, valid, a.enc_dim / 2, h);
                x[1] = zero16();
            }
            Split<2, 2> pz, px;
            split(z, pz);
            split(x, px);
            outer_accumulate_points<2, 2>(G[k], pz, px, tile_mem, lane);
            if (l > 0) {
                matvec_split<2, 4, 2, 2>(sm.mats + k * kMatrix, pz, z, lane);
                apply_mask<2>(z, m);
                if (k == LAYERS - 1) store_lane<2>(a.passed(second), tile, lane, z);
            } else if (!second) {
                v16f de[1];
                matvec_split<1, 4, 2, 2>(sm.mats + k * kMatrix, pz, de, lane);
                store_levels_active(a.d_enc, a.n, i, valid, a.enc_dim / 2, h, de[0]);
            }
        }
    }
    // ---- half of the waves leave their sums in LDS, the other half adds its own, and the block's sums go to global
    // memory in the gradients' own order
    __syncthreads();
    float* scratch = reinterpret_cast<float*>(&sm);
    constexpr int kVecs = 4 * LAYERS, kSlots = kDeepWaves / 2;
    static_assert(sizeof(sm) >= kSlots * kVecs * 1024 * sizeof(float), "scratch for the block sum");
    float* own = scratch + (wave % kSlots) * kVecs * 1024 + lane_in;
    const v16f* all[kVecs];
#pragma unroll
    for (int k = 0; k < LAYERS; ++k)
#pragma unroll
        for (int b = 0; b < 4; ++b) all[4 * k + b] = &G[k][b >> 1][b & 1];
    if (wave >= kSlots) {
#pragma unroll
        for (int k = 0; k < kVecs; ++k)
#pragma unroll
            for (int r = 0; r < 16; ++r) own[(k * 16 + r) * 64] = (*all[k])[r];
    }
    __syncthreads();
    if (wave < kSlots) {
#pragma unroll
        for (int k = 0; k < kVecs; ++k)
#pragma unroll
            for (int r = 0; r < 16; ++r) own[(k * 16 + r) * 64] += (*all[k])[r];
    }
    __syncthreads();
    for (int k = 0; k < LAYERS; ++k) {
        const int l = a.first - k, id = a.in_dim(l), count = a.out_dim(l) * id;       // a multiple of kDeepThreads
        const int shift = id == 64 ? 6 : id == 32 ? 5 : 4;
        for (int c = 0; c < count; c += kDeepThreads) {
            const int e = (c + (int)blockIdx.x / 8 * kDeepThreads) % count + threadIdx.x;   // workgroups start at different places
            atomicAdd(a.dH[l] + e, block_element_points<kSlots, kVecs, 2>(scratch, 4 * k, e >> shift, e & (id - 1)));
        }
    }
}

SdfArgs base_args(const neus2_config* cfg, const float* enc, const float* jac, const float* const* H, int64_t n) {
    SdfArgs a = {};
    a.enc = enc; a.jac = jac; a.n = n; a.active_levels = cfg->active_levels;
    for (int l = 0; l < cfg->n_sdf_mats; ++l) a.H[l] = H[l];
    return a;
}

}  // namespace

int launch_sdf_fwd(const neus2_config* cfg, const float* enc, const float* jac, const float* const* H,
                   int64_t n, float* y, float* q, float* normal, uint32_t* masks, hipStream_t st) {
    if (n == 0) return NEUS2_OK;
    SdfArgs a = base_args(cfg, enc, jac, H, n);
    a.y = y; a.q = q; a.normal = normal; a.masks = masks;
    a.stream_q = n >= ((int64_t)1 << 20);
    const int D = cfg->sdf_dims[0], K = cfg->n_sdf_mats;
    if (D == 32 && K == 3) return run_fwd<32, 3>(a, st);
    if (D == 32 && K == 2) return run_fwd<32, 2>(a, st);
    if (D == 16 && K == 3) return run_fwd<16, 3>(a, st);
    if (D == 16 && K == 2) return run_fwd<16, 2>(a, st);
    return fail(NEUS2_ERR_UNSUPPORTED, "sdf network: input width %d with %d matrices has no kernel", D, K);
}

int launch_sdf_values(const neus2_config* cfg, const float* enc, const float* const* H, int64_t n, float* sdf, hipStream_t st) {
    if (n == 0) return NEUS2_OK;
    SdfArgs a = base_args(cfg, enc, nullptr, H, n);
    a.y = sdf;
    const int D = cfg->sdf_dims[0], K = cfg->n_sdf_mats;
    if (D == 32 && K == 3) return run_values<32, 3>(a, st);
    if (D == 32 && K == 2) return run_values<32, 2>(a, st);
    if (D == 16 && K == 3) return run_values<16, 3>(a, st);
    if (D == 16 && K == 2) return run_values<16, 2>(a, st);
    return fail(NEUS2_ERR_UNSUPPORTED, "sdf network: input width %d with %d matrices has no kernel", D, K);
}

// Workspace of the deeper networks: see DeepArgs.
static int64_t deep_vector_floats(int64_t n) { return ((n + 31) / 32) * 64 * 32; }

int64_t sdf_deep_workspace_bytes(int n_mats, int64_t n) {
    const int64_t vec = deep_vector_floats(n) * 4, words = ((n + 31) / 32) * 64 * 4;
    return (2 * (int64_t)n_mats + 1) * vec + ((int64_t)n_mats - 1) * words;
}

namespace {

DeepArgs deep_args(int n_mats, int enc_dim, const float* enc, const float* jac, const float* const* H, int64_t n, void* workspace) {
    DeepArgs a = {};
    for (int l = 0; l < n_mats; ++l) a.H[l] = H[l];
    a.n_mats = n_mats; a.enc_dim = enc_dim; a.n = n; a.vec = deep_vector_floats(n);
    a.ws = reinterpret_cast<float*>(workspace);
    a.enc = enc; a.jac = jac;
    return a;
}

// items: pieces of work of a wavefront
template <typename Kernel>
void deep_launch(Kernel kernel, const DeepArgs& a, int64_t items, hipStream_t st) {
    const int blocks = persistent_blocks((const void*)kernel, kDeepThreads, (items + kDeepWaves - 1) / kDeepWaves);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kDeepThreads), 0, st, a);
}

// layers 0 .. n - 1 in as few runs as possible, of sizes that differ by one at most: [start[r], start[r + 1])
int deep_runs(int n, int* start) {
    const int runs = (n + kDeepRun - 1) / kDeepRun;
    for (int r = 0; r <= runs; ++r) start[r] = r * n / runs;
    return runs;
}

}  // namespace

int launch_sdf_deep_fwd(int n_mats, int enc_dim, const float* enc, const float* jac, const float* const* H, int64_t n,
                        float* y, float* q, float* normal, void* workspace, hipStream_t st) {
    if (n == 0) return NEUS2_OK;
    DeepArgs a = deep_args(n_mats, enc_dim, enc, jac, H, n, workspace);
    a.y = y; a.q = q; a.normal = normal;
    const int64_t tiles = (n + 31) / 32;
    int start[NEUS2_DEEP_MAX_MATS + 1];
    const int runs = deep_runs(n_mats, start);
    for (int r = 0; r < runs; ++r) {                             // a_1 .. a_{K-1}, y
        a.first = start[r]; a.count = start[r + 1] - start[r];
        deep_launch(deep_forward_kernel<false>, a, tiles, st);
    }
    const int back = deep_runs(n_mats - 1, start);
    for (int r = back - 1; r >= 0; --r) {                        // S_{K-1} .. S_1, dd/de
        a.first = start[r + 1] - 1; a.count = start[r + 1] - start[r];
        const int blocks = persistent_blocks((const void*)deep_reverse_kernel, kDeepThreads, tiles);
        hipLaunchKernelGGL(deep_reverse_kernel, dim3(blocks), dim3(kDeepThreads), 0, st, a);
    }
    return check_launch("sdf forward (deeper network)");
}

int launch_sdf_deep_bwd(int n_mats, int enc_dim, const float* enc, const float* jac, const float* const* H,
                        const float* d_y, const float* d_normal, int64_t n, float* const* dH, float* d_enc,
                        void* workspace, hipStream_t st) {
    if (n == 0) return NEUS2_OK;
    DeepArgs a = deep_args(n_mats, enc_dim, enc, jac, H, n, workspace);
    a.d_y = d_y; a.d_normal = d_normal; a.d_enc = d_enc;
    for (int l = 0; l < n_mats; ++l) a.dH[l] = dH[l];
    const int64_t tiles = (n + 31) / 32;
    int start[NEUS2_DEEP_MAX_MATS + 1];
    const int runs = deep_runs(n_mats - 1, start);
    for (int r = 0; r < runs; ++r) {                             // a_l and t_l of every hidden layer
        a.first = start[r]; a.count = start[r + 1] - start[r];
        deep_launch(deep_forward_kernel<true>, a, tiles, st);
    }
    for (int l = n_mats - 1; l >= 0; l -= kDeepGradRun) {
        a.first = l;
        if (l > 0) deep_launch(deep_gradient_kernel<kDeepGradRun>, a, 2 * tiles, st);
        else deep_launch(deep_gradient_kernel<1>, a, 2 * tiles, st);
    }
    return check_launch("sdf backward (deeper network)");
}

int launch_sdf_bwd(const neus2_config* cfg, const float* enc, const float* jac, const float* const* H,
                   const float* d_y, const float* d_normal, int64_t n, float* const* dH, float* d_enc,
                   float* d_pos, const uint32_t* masks, hipStream_t st) {
    if (n == 0) return NEUS2_OK;
    SdfArgs a = base_args(cfg, enc, jac, H, n);
    a.d_y = d_y; a.d_normal = d_normal; a.d_enc = d_enc; a.d_pos = d_pos;
    a.stream_q = n >= ((int64_t)1 << 20);
    a.masks = const_cast<uint32_t*>(masks);              // the backward kernel only reads them
    for (int l = 0; l < cfg->n_sdf_mats; ++l) a.dH[l] = dH[l];
    const int D = cfg->sdf_dims[0], K = cfg->n_sdf_mats;
    if (D == 32 && K == 3) return run_bwd<32, 3>(a, st);
    if (D == 32 && K == 2) return run_bwd<32, 2>(a, st);
    if (D == 16 && K == 3) return run_bwd<16, 3>(a, st);
    if (D == 16 && K == 2) return run_bwd<16, 2>(a, st);
    return fail(NEUS2_ERR_UNSUPPORTED, "sdf network: input width %d with %d matrices has no kernel", D, K);
}

}  // namespace neus2
