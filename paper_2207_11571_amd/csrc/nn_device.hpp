// Device code of the forcing network shared by the network kernels and the
// fused BR1-and-network kernel of the stage: bf16 rounding, activations, the
// 16-row MFMA layer product (v_mfma_f32_16x16x32_bf16, float32
// accumulation) and the forward pass of one 16-row block whose normalised
// inputs are in LDS.
#pragma once

#include "dgnn_internal.hpp"

namespace dgnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Global-memory views of pointers taken from the argument structs: indexed
// by a run-time layer number they reach the kernel as generic pointers, and
// generic (flat) accesses count against the LDS counter as well, so LDS
// accesses would wait for the global traffic in flight.
template <class T>
using global_t = __attribute__((address_space(1))) T;
template <class T>
__device__ __forceinline__ global_t<T>* gmem(T* p) { return (global_t<T>*)p; }

constexpr int kRows = 16;      // rows (elements / samples) per block
constexpr int kRowWaves = 16;     // row-block kernels: sixteen wavefronts share the column tiles
constexpr int kRowThreads = 64 * kRowWaves;
constexpr int kLdPad = 8;      // LDS row padding (bf16 elements)

// Weight fragments are read with buffer loads through a resource over one
// layer's bf16 weights [Np][Kp]: one vector offset per lane, the 1 KB steps
// of a tile as scalar offsets.  Plain global loads need an address register
// of their own for every step past the 4 KB immediate offset.
constexpr int kBufferWord3 = 0x00020000;   // fourth resource word, gfx9 family (32-bit data format)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_rsrc(const __attribute__((address_space(1))) uint16_t* W,
                                                               int Kp, int Np) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(const uint16_t*)W, 0, Np * Kp * 2, kBufferWord3);
}

// fragment step s of the tile whose lane offset (bytes) is vo
__device__ __forceinline__ bf16x8 weight_frag(__amdgpu_buffer_rsrc_t rs, int vo, int s) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, vo, s * 1024, 0));
}

// float32 -> bfloat16, round to nearest even (NaN kept quiet); a select,
// not a branch, for the NaN case
__device__ __forceinline__ uint16_t f2bf(float x) {
    const uint32_t u = __float_as_uint(x);
    const uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    const uint32_t qnan = (u >> 16) | 0x0040u;
    return (uint16_t)((u & 0x7FFFFFFFu) > 0x7F800000u ? qnan : r);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

__device__ __forceinline__ float act_fwd(float z, int act) { return act == 0 ? tanhf(z) : fmaxf(z, 0.0f); }
// derivative through the output h = act(z)
__device__ __forceinline__ float act_bwd(float h, int act) { return act == 0 ? 1.0f - h * h : (h > 0.0f ? 1.0f : 0.0f); }

// Position of W[n][k] (n < Np, k < Kp, both padded to multiples of 32) in
// the bf16 weight copies: the fragment order of the B operand of
// v_mfma_f32_16x16x32_bf16 as tile_mma loads it.  Each 16-column tile and
// 32-wide K step is one 1 KB block in which lane r + 16 q holds
// W[16 tile + r][32 s + 8 q, + 8), so that a wavefront's fragment load reads
// one contiguous kilobyte instead of 64-byte pieces of sixteen rows (half
// the time of a row-major layout for the chain of layers, measured).
__host__ __device__ __forceinline__ int64_t wfrag_index(int n, int k, int Kp) {
    const int tile = n >> 4, r = n & 15, s = k >> 5, q = (k & 31) >> 3, j = k & 7;
    return ((((int64_t)tile * (Kp >> 5) + s) * 64 + r + 16 * q) << 3) + j;
}

// C[16][Np] = A[16][Kp] W^T with W [Np][Kp] bf16 in global memory, in the
// fragment order of wfrag_index.
// Wave w computes the 16-column tiles w, w + kRowWaves, ...; epi(m, n, value)
// per output.  For the common widths the K loop is unrolled so that all of a
// tile's weight fragments are in flight at once: the weights come from L2 and
// their latency, not the matrix cores, bounds this product, so sixteen
// wavefronts (one or two tiles each) beat fewer wavefronts with prefetching.
template <int KP, class Epi>
__device__ __forceinline__ void tile_mma_fixed(const uint16_t* __restrict__ sA, int ldA,
                                               const global_t<uint16_t>* __restrict__ W, int Np, int wave, int lane,
                                               Epi& epi) {
    constexpr int KS = KP / 32;
    const int kq = 8 * (lane >> 4);
    const int r = lane & 15;
    const uint16_t* arow = sA + r * ldA + kq;
    const __amdgpu_buffer_rsrc_t rs = weight_rsrc(W, KP, Np);
    for (int tile = wave; tile < Np / 16; tile += kRowWaves) {
        const int vo = (tile * KS * 64 + lane) * 16;
        bf16x8 b[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) b[s] = weight_frag(rs, vo, s);
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8 a = *(const bf16x8*)(arow + 32 * s);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[s], acc, 0, 0, 0);
        }
        const int n = tile * 16 + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) epi(4 * (lane >> 4) + i, n, acc[i]);
    }
}

template <class Epi>
__device__ __forceinline__ void tile_mma(const uint16_t* __restrict__ sA, int ldA,
                                         const global_t<uint16_t>* __restrict__ W, int Kp, int Np, int wave, int lane,
                                         Epi epi) {
    if (Kp == 256) {
        tile_mma_fixed<256>(sA, ldA, W, Np, wave, lane, epi);
        return;
    }
    if (Kp == 320) {
        tile_mma_fixed<320>(sA, ldA, W, Np, wave, lane, epi);
        return;
    }
    const int kq = 8 * (lane >> 4);
    const int r = lane & 15;
    for (int tile = wave; tile < Np / 16; tile += kRowWaves) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        const int n = tile * 16 + r;
        const global_t<uint16_t>* wt = W + ((int64_t)tile * (Kp / 32) * 64 + lane) * 8;
        const uint16_t* arow = sA + r * ldA + kq;
        for (int k0 = 0; k0 < Kp; k0 += 32) {
            const bf16x8 a = *(const bf16x8*)(arow + k0);
            const bf16x8 b = *(const global_t<bf16x8>*)(wt + (k0 / 32) * 512);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) epi(4 * (lane >> 4) + i, n, acc[i]);
    }
}

// Layers with K <= 32 * kMaxKS = 320 keep a wavefront's whole weight tile in
// registers, so the next layer's tile can be loaded while the current one's
// outputs are formed (below).
constexpr int kMaxKS = 10;

// issue the loads of this wavefront's fragments of column tile `tile` of W
// [Np][Kp].  (Each load sits under its own branch, the count being known at
// run time; with global loads and their per-step address registers the
// compiler waited for all loads in flight before each step past the first
// four, which the buffer loads avoid.)
__device__ __forceinline__ void load_frags(bf16x8 (&b)[kMaxKS], const global_t<uint16_t>* W, int Kp, int Np, int tile,
                                           int lane) {
    const int KS = Kp >> 5;
    const __amdgpu_buffer_rsrc_t rs = weight_rsrc(W, Kp, Np);
    const int vo = (tile * KS * 64 + lane) * 16;
#pragma unroll
    for (int s = 0; s < kMaxKS; ++s)
        if (s < KS) b[s] = weight_frag(rs, vo, s);
}

// C tile = A[16][Kp] (LDS rows from arow) times the fragments b
__device__ __forceinline__ floatx4 mma_frags(const bf16x8 (&b)[kMaxKS], const uint16_t* arow, int Kp) {
    const int KS = Kp >> 5;
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < kMaxKS; ++s)
        if (s < KS) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8*)(arow + 32 * s), b[s], acc, 0, 0, 0);
    return acc;
}

// normalised network input of node n of the j-th variable read, value qv
// (Sec. 2.2: per-variable, or per-node when the model carries column
// statistics)
__device__ __forceinline__ float net_input(const NetArgs& na, int NP, int j, int n, double qv) {
    if (na.col) {
        const int cc = na.in_var[j] * NP + n;
        return (float)((qv - gmem(na.col)[cc]) / gmem(na.col)[5 * NP + cc]);
    }
    return (float)((qv - na.in_mu[j]) * na.in_isig[j]);
}

// write mode: the variables the network does not force get s = 0 (rows
// e0 .. e0 + 15 of target T)
__device__ __forceinline__ void net_zero_unforced(const NetArgs& na, int NP, const NetTarget& T, int e0, int t) {
    if (na.n_out >= 5) return;
    const size_t vs = (size_t)T.E * NP;
    for (int idx = t; idx < kRows * 5 * NP; idx += kRowThreads) {
        const int r = idx / (5 * NP), c = idx - r * (5 * NP);
        const int v = c / NP, n = c - v * NP;
        const int e = e0 + r;
        bool forced = false;
        for (int j = 0; j < na.n_out; ++j) forced = forced || na.out_var[j] == v;
        if (e < T.E && !forced) gmem(T.out)[v * vs + (size_t)e * NP + n] = 0.0;
    }
}

// ---- networks whose hidden layers are all 256 wide, as the ones of the
// accuracy studies and the throughput workload: one column tile of each
// hidden layer for each of the sixteen wavefronts, eight K steps.
//
// What a launch takes is one block's chain: states, dependent layers, the
// forcing, and the 590 KB of weights that each block reads from L2 at 64 B a
// clock (9200 clocks).  The general form below spent 40 k clocks on it (512
// elements, 320-256-256-256-320: 18.3 us a launch; 12.1 k until the rows were
// in LDS, entry after entry with two divisions each; 2 k a layer issuing the
// next tile's loads in one run, all sixteen wavefronts at once, before 1.9 k
// of epilogue; 1.3 k a layer of products, each behind its own LDS read).
// Here the loads are issued between the rows of the epilogue, and the step
// counts are template arguments: counts known at run time put a branch around
// each load and copies of registers in flight where the branches meet.
// 12.3 us a launch; with the BR1 pass of 16^3 elements 25.2 -> 19.8 us.

// The loads are scheduled as written between these.
__device__ __forceinline__ void net_fence() { __builtin_amdgcn_sched_barrier(0); }

// waits until a loaded value is in its register
template <class V>
__device__ __forceinline__ void arrived(V& x) {
    asm volatile("" : "+v"(x));
}

// fragments [S0, S1) of the tile whose lane offset is vo
template <int S0, int S1, int N>
__device__ __forceinline__ void load_steps(bf16x8 (&b)[N], __amdgpu_buffer_rsrc_t rs, int vo) {
#pragma unroll
    for (int s = S0; s < S1; ++s) b[s] = weight_frag(rs, vo, s);
}

// C tile = A[16][32 KS] (LDS rows from arow) times the fragments b
template <int KS, int N>
__device__ __forceinline__ floatx4 mma_steps(const bf16x8 (&b)[N], const uint16_t* arow) {
    bf16x8 a[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) a[s] = *(const bf16x8*)(arow + 32 * s);
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[s], acc, 0, 0, 0);
    return acc;
}

// input steps K0 (dims[0] padded to 32 K0) that have kernels of their own
inline int net256_steps(const NetArgs& na) {
    if (na.n_layers < 2) return 0;
    for (int l = 1; l < na.n_layers; ++l)
        if (na.dims[l] != 256) return 0;
    const int k0 = na.pdims[0] / 32;
    if (na.pdims[na.n_layers] > 32 * kMaxKS) return 0;
    return k0 == 3 || k0 == 5 || k0 == 6 || k0 == 10 ? k0 : 0;
}

// A wavefront's tile of the first layer, loaded behind the states it is
// applied to.
template <int K0>
struct FirstTile {
    bf16x8 b[K0];
    float bias;
    __device__ __forceinline__ void load(const NetArgs& na, int wave, int lane) {
        load_steps<0, K0>(b, weight_rsrc(gmem(na.W[0]), 32 * K0, 256), (wave * K0 * 64 + lane) * 16);
        bias = gmem(na.b[0])[wave * 16 + (lane & 15)];
    }
};

// A five-entry array of the arguments in scalar registers, entry j by selects:
// indexed by a lane's value the array would be read from memory, a round trip
// each (and the compiler turns selects of its loads into that).
template <class V>
struct Five {
    V a, b, c, d, e;
    __device__ __forceinline__ explicit Five(const V* p) : a(p[0]), b(p[1]), c(p[2]), d(p[3]), e(p[4]) {
        asm volatile("" : "+s"(a), "+s"(b), "+s"(c), "+s"(d), "+s"(e));
    }
    __device__ __forceinline__ V at(int j) const { return j == 0 ? a : (j == 1 ? b : (j == 2 ? c : (j == 3 ? d : e))); }
};

// Gather + normalise + bf16 of a block's sixteen rows (elements e0 ...):
// wavefront w row w, a lane a node (zero rows beyond E and columns beyond
// dims[0]).  The first tile of weights (K0 > 0) is asked for when the states
// are there: all wavefronts' loads go through one queue, and the last one's
// states would wait for the others' weights.
template <int K0>
__device__ __forceinline__ void net_gather(const NetArgs& na, const int (&in_var)[5], int NP, const NetTarget& T, int e0,
                                           uint16_t* bufA, int ld, int wave, int lane, FirstTile<K0 ? K0 : 1>& first) {
    const size_t vs = (size_t)T.E * NP;
    const int din = na.dims[0], pin = na.pdims[0];
    const int e = e0 + wave;
    uint16_t* row = bufA + wave * ld;
    const bool in = e < T.E;
    const global_t<const double>* q = gmem(T.q) + (size_t)(in ? e : e0) * NP;
    size_t var[5];   // beyond n_in: variable 0, read and not used
#pragma unroll
    for (int j = 0; j < 5; ++j) var[j] = in_var[j] * vs;
    for (int n0 = 0; n0 < NP; n0 += 64) {
        const int n = n0 + lane;
        const int nc = n < NP ? n : NP - 1;
        double x[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) x[j] = q[var[j] + nc];
        if constexpr (K0 > 0)
            if (n0 == 0) {
#pragma unroll
                for (int j = 0; j < 5; ++j) arrived(x[j]);
                first.load(na, wave, lane);
            }
#pragma unroll
        for (int j = 0; j < 5; ++j)
            if (j < na.n_in) {
                const float v = net_input(na, NP, j, nc, x[j]);
                if (n < NP) row[j * NP + n] = f2bf(in ? v : 0.0f);
            }
    }
    for (int c = din + lane; c < pin; c += 64) row[c] = f2bf(0.0f);
}

// The layers of one 16-row block, as net_block_forward below.
template <int K0, int ACT>
__device__ __forceinline__ void net256_forward(const NetArgs& na, int NP, const NetTarget& T, int e0, int accumulate,
                                               uint16_t* bufA, uint16_t* bufB, int ld, int wave, int lane,
                                               FirstTile<K0>& first) {
    const size_t vs = (size_t)T.E * NP;
    const int L = na.n_layers;
    const int r = lane & 15, g = lane >> 4;
    const int Np = na.pdims[L], Nd = na.dims[L], nt = Np / 16;
    bf16x8 b[8];
    float bn = first.bias;
    floatx4 acc = mma_steps<K0>(first.b, bufA + r * ld + 8 * g);
    for (int l = 0; l + 1 < L; ++l) {
        // layer l's products are in acc; its epilogue with layer l + 1's loads
        const bool out = l + 2 == L;
        const __amdgpu_buffer_rsrc_t rs = weight_rsrc(gmem(na.W[l + 1]), 256, out ? Np : 256);
        const int tile = out && wave >= nt ? nt - 1 : wave;
        const int vo = (tile * 8 * 64 + lane) * 16;
        const int n1 = tile * 16 + r;
        const float bnext = gmem(na.b[l + 1])[out && n1 >= Nd ? Nd - 1 : n1];
        uint16_t* o = bufB + 4 * g * ld + wave * 16 + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i == 0) load_steps<0, 2>(b, rs, vo);
            if (i == 1) load_steps<2, 4>(b, rs, vo);
            if (i == 2) load_steps<4, 6>(b, rs, vo);
            if (i == 3) load_steps<6, 8>(b, rs, vo);
            net_fence();
            o[i * ld] = f2bf(act_fwd(acc[i] + bn, ACT));
            net_fence();
        }
        bn = bnext;
        __syncthreads();
        uint16_t* tmp = bufA;
        bufA = bufB;
        bufB = tmp;
        acc = mma_steps<8>(b, bufA + r * ld + 8 * g);
    }
    // the output layer: its first tile's products are in acc
    const Five<int> out_var(na.out_var);
    const Five<double> out_scale(na.out_scale), out_shift(na.out_shift);
    const __amdgpu_buffer_rsrc_t rs = weight_rsrc(gmem(na.W[L - 1]), 256, Np);
    for (int tile = wave; tile < nt; tile += kRowWaves) {
        const int n = tile * 16 + r;
        const bool more = tile + kRowWaves < nt;
        const int nc = n < Nd ? n : Nd - 1;
        const int j = (nc >= NP) + (nc >= 2 * NP) + (nc >= 3 * NP) + (nc >= 4 * NP), node = nc - j * NP;
        const int vv = out_var.at(j);
        double sc = out_scale.at(j), sh = out_shift.at(j);
        if (na.col) {
            const int cc = vv * NP + node;
            const double mask = na.mask[vv];
            sc = mask * gmem(na.col)[15 * NP + cc];
            sh = mask * gmem(na.col)[10 * NP + cc];
        }
        arrived(sc);   // ahead of the next tile's loads, which return behind it
        arrived(sh);
        arrived(bn);
        if (more) load_steps<0, 8>(b, rs, ((tile + kRowWaves) * 8 * 64 + lane) * 16);
        if (n < Nd) {
            global_t<double>* o = gmem(T.out) + vv * vs + (size_t)(e0 + 4 * g) * NP + node;
            double s[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = sc * (double)(acc[i] + bn) + sh;
            if (accumulate) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e0 + 4 * g + i < T.E) s[i] += o[i * NP];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (e0 + 4 * g + i < T.E) o[i * NP] = s[i];
        }
        if (more) {
            const int n1 = n + 16 * kRowWaves;
            bn = gmem(na.b[L - 1])[n1 < Nd ? n1 : Nd - 1];
            acc = mma_steps<8>(b, bufA + r * ld + 8 * g);
        }
    }
}

// The layers of one 16-row block: bufA holds the rows' normalised bf16
// inputs (zero beyond dims[0] and for rows past the target's end), bufB is
// scratch of the same shape; hidden layers apply bias and activation, the
// last layer de-normalises and writes (or adds) s for rows e0 .. e0 + 15 of
// T.  Ends with a block barrier.
__device__ __forceinline__ void net_block_forward(const NetArgs& na, int NP, const NetTarget& T, int e0, int accumulate,
                                                  uint16_t* bufA, uint16_t* bufB, int ld, int wave, int lane) {
    const size_t vs = (size_t)T.E * NP;
    const int L = na.n_layers;
    // Narrow layers: each wavefront's weight tile of the next layer is
    // loaded as soon as the products of its last tile of this layer are
    // issued, so the load latency overlaps the bias / activation epilogue
    // and the block barrier instead of starting after them.
    bool narrow = true;
    for (int l = 0; l < L; ++l) narrow = narrow && na.pdims[l] <= 32 * kMaxKS;
    if (narrow) {
        const int r = lane & 15;
        const int kq = 8 * (lane >> 4);
        bf16x8 b[kMaxKS];
        if (wave < na.pdims[1] / 16) load_frags(b, gmem(na.W[0]), na.pdims[0], na.pdims[1], wave, lane);
        for (int l = 0; l < L; ++l) {
            const int Kp = na.pdims[l], Np = na.pdims[l + 1], Nd = na.dims[l + 1];
            const global_t<const float>* bias = gmem(na.b[l]);
            const uint16_t* arow = bufA + r * ld + kq;
            // a wavefront with no tile in this layer but one in the next
            if (l + 1 < L && wave >= Np / 16 && wave < na.pdims[l + 2] / 16)
                load_frags(b, gmem(na.W[l + 1]), Np, na.pdims[l + 2], wave, lane);
            for (int tile = wave; tile < Np / 16; tile += kRowWaves) {
                if (tile != wave) load_frags(b, gmem(na.W[l]), Kp, Np, tile, lane);
                const floatx4 acc = mma_frags(b, arow, Kp);
                if (tile + kRowWaves >= Np / 16 && l + 1 < L && wave < na.pdims[l + 2] / 16)
                    load_frags(b, gmem(na.W[l + 1]), Np, na.pdims[l + 2], wave, lane);
                const int n = tile * 16 + r;
                if (l < L - 1) {
                    const float bn = n < Nd ? bias[n] : 0.0f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int m = 4 * (lane >> 4) + i;
                        bufB[m * ld + n] = f2bf(n < Nd ? act_fwd(acc[i] + bn, na.act) : 0.0f);
                    }
                } else if (n < Nd) {
                    const float bn = bias[n];
                    const int j = n / NP, node = n - j * NP;
                    const int vv = na.out_var[j];
                    const int cc = vv * NP + node;
                    const double sc = na.col ? na.mask[vv] * na.col[15 * NP + cc] : na.mask[vv] * na.sig_out[vv];
                    const double sh = na.col ? na.mask[vv] * na.col[10 * NP + cc] : na.mask[vv] * na.mu_out[vv];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int e = e0 + 4 * (lane >> 4) + i;
                        if (e < T.E) {
                            const double s = sc * (double)(acc[i] + bn) + sh;
                            global_t<double>* o = gmem(T.out) + vv * vs + (size_t)e * NP + node;
                            *o = accumulate ? *o + s : s;
                        }
                    }
                }
            }
            __syncthreads();
            uint16_t* tmp = bufA;
            bufA = bufB;
            bufB = tmp;
        }
        return;
    }
    for (int l = 0; l < L; ++l) {
        const int Kp = na.pdims[l], Np = na.pdims[l + 1], Nd = na.dims[l + 1];
        const global_t<const float>* bias = gmem(na.b[l]);
        if (l < L - 1) {
            const int act = na.act;
            tile_mma(bufA, ld, gmem(na.W[l]), Kp, Np, wave, lane, [&](int m, int n, float v) {
                const float z = v + (n < Nd ? bias[n] : 0.0f);
                bufB[m * ld + n] = f2bf(n < Nd ? act_fwd(z, act) : 0.0f);
            });
        } else {
            tile_mma(bufA, ld, gmem(na.W[l]), Kp, Np, wave, lane, [&](int m, int n, float v) {
                const int e = e0 + m;
                if (e < T.E && n < Nd) {
                    const float y = v + bias[n];
                    const int j = n / NP, node = n - j * NP;
                    const int vv = na.out_var[j];
                    const int cc = vv * NP + node;
                    const double s = na.col ? na.mask[vv] * (na.col[15 * NP + cc] * (double)y + na.col[10 * NP + cc])
                                            : na.mask[vv] * (na.sig_out[vv] * (double)y + na.mu_out[vv]);
                    global_t<double>* o = gmem(T.out) + vv * vs + (size_t)e * NP + node;
                    *o = accumulate ? *o + s : s;
                }
            });
        }
        __syncthreads();
        uint16_t* tmp = bufA;
        bufA = bufB;
        bufB = tmp;
    }
}

}  // namespace dgnn
