// Forcing network kernels for gfx950: bf16 MFMA (v_mfma_f32_16x16x32_bf16)
// with float32 accumulation.
//
// Inference (Sec. 2.2, Eq. (4)): one block of sixteen wavefronts takes 16
// elements; their states are gathered from the DG layout q[v][e][n],
// normalised and rounded to bf16 in LDS; every layer is a 16 x N x K product
// of the LDS-resident activations with the bf16 weights read from L2, with
// bias and activation fused into the epilogue; the last layer writes the
// de-normalised forcing straight into the float64 field.  Activations never
// leave LDS.
//
// Training (MSE loss, Adam): the same row blocks run forward, loss and the
// backward data chain with all activations LDS-resident, and write the
// transposed activations and output gradients needed by the weight-gradient
// products dW_l = dz_l^T h_l, which reduce over the batch in a second kernel
// that also updates the weights.
#include "nn_device.hpp"

namespace dgnn {

int net_rows_per_block() { return kRows; }
int net_row_pad() { return kLdPad; }

struct NetTargets {
    NetTarget t[16];
    int n;
};

// ------------------------------------------------------------------ inference

// K0 > 0: hidden layers of 256 (net256_forward), K0 steps of input; 0: any
template <int K0, int ACT>
__global__ void __launch_bounds__(kRowThreads) k_net_forcing(NetArgs na, int NP, NetTargets tg, int accumulate) {
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    const int ld = na.ld;
    uint16_t* bufA = smem;
    uint16_t* bufB = smem + kRows * ld;

    const int b = blockIdx.x;
    int ti = 0;
    for (int i = 1; i < tg.n; ++i)
        if (tg.t[i].blk_begin <= b) ti = i;
    const NetTarget T = tg.t[ti];
    const int e0 = (b - T.blk_begin) * kRows;
    const int E = T.E;
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const size_t vs = (size_t)E * NP;

    FirstTile<K0 ? K0 : 1> first;
    net_gather<K0>(na, na.in_var, NP, T, e0, bufA, ld, wave, lane, first);
    if (!accumulate) net_zero_unforced(na, NP, T, e0, t);
    __syncthreads();
    if constexpr (K0 > 0) net256_forward<K0, ACT>(na, NP, T, e0, accumulate, bufA, bufB, ld, wave, lane, first);
    else net_block_forward(na, NP, T, e0, accumulate, bufA, bufB, ld, wave, lane);
}

// ------------------------------------------------------------------- weights

// bf16 copies of W_l ([pout][pin]) and W_l^T ([pin][pout]), zero padded, in
// the fragment order of wfrag_index
__global__ void __launch_bounds__(256) k_net_refresh(NetArgs na, const float* __restrict__ params,
                                                    uint16_t* __restrict__ wbf,
                                                    int64_t woff0, int l, int64_t wbf_off, int64_t wtbf_off) {
    const int din = na.dims[l], dout = na.dims[l + 1];
    const int pin = na.pdims[l], pout = na.pdims[l + 1];
    const int total = pin * pout;
    for (int idx = blockIdx.x * 256 + threadIdx.x; idx < total; idx += gridDim.x * 256) {
        const int o = idx / pin, i = idx - o * pin;
        const float w = (o < dout && i < din) ? params[woff0 + (int64_t)o * din + i] : 0.0f;
        const uint16_t h = f2bf(w);
        wbf[wbf_off + wfrag_index(o, i, pin)] = h;
        wbf[wtbf_off + wfrag_index(i, o, pout)] = h;
    }
}

__global__ void __launch_bounds__(256) k_fill_f32(float* p, float v, size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = v;
}

// ------------------------------------------------------------------- training

typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

// Columns c < pd of the block's 16 LDS rows (rows r0 .. r0 + 15 of the
// batch) to dst in fragment order over the batch (wfrag_index with K = Bp):
// eight consecutive rows of a column are sixteen contiguous bytes there, so
// each thread packs eight LDS values into one store.
__device__ __forceinline__ void store_transposed(const uint16_t* src, int ld, int pd, global_t<uint16_t>* dst, int r0,
                                                 int Bp, int t) {
    for (int idx = t; idx < pd * 2; idx += kRowThreads) {
        const int c = idx >> 1, g = 8 * (idx & 1);
        u16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = src[(g + j) * ld + c];
        *(global_t<u16x8>*)(dst + wfrag_index(c, r0 + g, Bp)) = v;
    }
}

// One row block: forward with LDS-resident activations, MSE loss in
// normalised space, backward data chain dz_{l-1} = (dz_l W_l) * act'(h_l).
// Writes transposed activations and output gradients for the weight products,
// in fragment order over the batch (wfrag_index with K = Bp).
__global__ void __launch_bounds__(kRowThreads) k_train_rows(NetArgs na, TrainArgs ta) {
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    const int L = na.n_layers;
    const int ld = na.ld;
    // act(0..L-1) then two gradient buffers
    auto act = [&](int l) { return smem + l * kRows * ld; };
    uint16_t* g0 = smem + L * kRows * ld;
    uint16_t* g1 = g0 + kRows * ld;
    __shared__ float red[kRowWaves];

    const int r0 = blockIdx.x * kRows;
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int B = ta.B, Bp = ta.Bp;
    const int din = na.dims[0], pin = na.pdims[0];
    const int npv_in = din / na.n_in;
    const size_t xw = (size_t)5 * npv_in;
    for (int idx = t; idx < kRows * pin; idx += kRowThreads) {
        const int r = idx / pin, c = idx - r * pin;
        const int row = r0 + r;
        float x = 0.0f;
        if (row < B && c < din) {
            const int j = c / npv_in, n = c - j * npv_in;
            const int v = na.in_var[j];
            const size_t src = ta.idx ? (size_t)ta.idx[row] : (size_t)row;
            const double xv = ta.x[src * xw + (size_t)v * npv_in + n];
            if (na.col) {
                const int cc = v * npv_in + n;
                x = (float)((xv - na.col[cc]) / na.col[5 * npv_in + cc]);
            } else {
                x = (float)((xv - na.mu_in[v]) / na.sig_in[v]);
            }
        }
        act(0)[r * ld + c] = f2bf(x);
    }
    __syncthreads();
    // forward through the hidden layers
    for (int l = 0; l < L - 1; ++l) {
        const int Kp = na.pdims[l], Np = na.pdims[l + 1], Nd = na.dims[l + 1];
        const global_t<const float>* bias = gmem(na.b[l]);
        uint16_t* out = act(l + 1);
        const int a = na.act;
        tile_mma(act(l), ld, gmem(na.W[l]), Kp, Np, wave, lane, [&](int m, int n, float v) {
            const float z = v + (n < Nd ? bias[n] : 0.0f);
            out[m * ld + n] = f2bf(n < Nd ? act_fwd(z, a) : 0.0f);
        });
        __syncthreads();
    }
    // output layer + loss gradient dY = scale (yhat - ytilde)
    float lsum = 0.0f;
    {
        const int l = L - 1;
        const int Kp = na.pdims[l], Np = na.pdims[l + 1], Nd = na.dims[l + 1];
        const int npv_out = Nd / na.n_out;
        const size_t yw = (size_t)5 * npv_out;
        const global_t<const float>* bias = gmem(na.b[l]);
        tile_mma(act(l), ld, gmem(na.W[l]), Kp, Np, wave, lane, [&](int m, int n, float v) {
            const int row = r0 + m;
            float dy = 0.0f;
            if (row < B && n < Nd) {
                const int j = n / npv_out, nn = n - j * npv_out;
                const int vv = na.out_var[j];
                const size_t src = ta.idx ? (size_t)ta.idx[row] : (size_t)row;
                const double yv = ta.y[src * yw + (size_t)vv * npv_out + nn];
                const int cc = vv * npv_out + nn;
                const float yt = na.col ? (float)((yv - na.col[10 * npv_out + cc]) / na.col[15 * npv_out + cc])
                                        : (float)((yv - na.mu_out[vv]) / na.sig_out[vv]);
                const float diff = v + bias[n] - yt;
                lsum += diff * diff;
                dy = ta.grad_scale * diff;
            }
            g0[m * ld + n] = f2bf(dy);
        });
    }
    // the block's loss: a fixed butterfly within each wavefront, then
    // wavefront 0 sums the sixteen partial sums in order (one barrier)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off);
    if (lane == 0) red[wave] = lsum;
    __syncthreads();
    if (t == 0) {
        float sum = 0.0f;
        for (int w = 0; w < kRowWaves; ++w) sum += red[w];
        ta.loss_part[blockIdx.x] = sum;
    }
    // row-block sums of dz for the bias gradients (g0 is complete after the barrier above)
    for (int c = t; c < na.pdims[L]; c += kRowThreads) {
        float sacc = 0.0f;
        for (int rr = 0; rr < kRows; ++rr) sacc += bf2f(g0[rr * ld + c]);
        gmem(ta.bias_part[L - 1])[(size_t)blockIdx.x * na.pdims[L] + c] = sacc;
    }
    // transposed activations and dz_{L-1}
    for (int l = 0; l < L; ++l) store_transposed(act(l), ld, na.pdims[l], gmem(ta.actT[l]), r0, Bp, t);
    store_transposed(g0, ld, na.pdims[L], gmem(ta.dzT[L - 1]), r0, Bp, t);
    // backward data chain
    uint16_t* gin = g0;
    uint16_t* gout = g1;
    for (int l = L - 1; l >= 1; --l) {
        const int Kp = na.pdims[l + 1], Np = na.pdims[l], Nd = na.dims[l];
        const uint16_t* h = act(l);
        const int a = na.act;
        tile_mma(gin, ld, gmem(na.WT[l]), Kp, Np, wave, lane, [&](int m, int n, float v) {
            const float d = (n < Nd) ? v * act_bwd(bf2f(h[m * ld + n]), a) : 0.0f;
            gout[m * ld + n] = f2bf(r0 + m < B ? d : 0.0f);
        });
        __syncthreads();
        store_transposed(gout, ld, Np, gmem(ta.dzT[l - 1]), r0, Bp, t);
        for (int c = t; c < Np; c += kRowThreads) {
            float sacc = 0.0f;
            for (int rr = 0; rr < kRows; ++rr) sacc += bf2f(gout[rr * ld + c]);
            gmem(ta.bias_part[l - 1])[(size_t)blockIdx.x * Np + c] = sacc;
        }
        uint16_t* tmp = gin;
        gin = gout;
        gout = tmp;
        __syncthreads();
    }
}

// Touches every line of the weights that a row block reads after its input
// layer, in that order, so that they are in the L2 of this block's XCD.  The
// last step's update left them in other XCDs', and with few row blocks each
// layer would wait for them again: batch 64 19.4 -> 17.9 us, 512 19.6 -> 18.7.
__device__ __forceinline__ void warm_weights(const NetArgs& na, int t) {
    const int L = na.n_layers;
    uint32_t sum = 0;
    for (int i = 1; i < 2 * L - 1; ++i) {
        const int l = i < L ? i : 2 * L - 1 - i;
        const global_t<const uint32_t>* w = gmem((const uint32_t*)(i < L ? na.W[l] : na.WT[l]));
        const int lines = na.pdims[l] * na.pdims[l + 1] / 64;
        for (int x = t; x < lines; x += kRowThreads) sum += w[x * 32];
    }
    asm volatile("" ::"v"(sum));
}

// k_train_rows for networks with hidden layers of 256 (net256_steps), K0 steps of
// input and nt column tiles of output.  Each wavefront owns the same column
// tile of every hidden layer, forward and backward, and the lane that forms
// rows 4 g .. 4 g + 3 of a column holds four consecutive batch entries of it,
// so activations and output gradients go to their transposed arrays straight
// from the epilogues, 8 bytes a lane, and the bias sums of a column are three
// additions and a butterfly over its four lanes; only the input's transpose
// goes through LDS.  Weights are loaded ahead as in net256_forward, the
// targets before the output layer.
// What a block's first loads need is ahead of the structures: the first sixteen
// words of a kernel's arguments are in scalar registers when it starts.
template <int K0, int ACT>
__global__ void __launch_bounds__(kRowThreads)
k_train256(const float* rows, const int32_t* idx, int B, int Bp, int npv, int v0, int v1, int v2, int v3, int v4, NetArgs na,
           TrainArgs ta) {
    if ((int)blockIdx.x >= Bp / kRows) return warm_weights(na, threadIdx.x);
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    const int L = na.n_layers, ld = na.ld;
    auto act = [&](int l) { return smem + l * kRows * ld; };
    uint16_t* g0 = smem + L * kRows * ld;
    uint16_t* g1 = g0 + kRows * ld;
    __shared__ float red[kRowWaves];

    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int r = lane & 15, g = lane >> 4;
    const int r0 = blockIdx.x * kRows;
    const int in_var[5] = {v0, v1, v2, v3, v4};
    const int Np = na.pdims[L], Nd = na.dims[L], nt = Np / 16;
    const size_t rw = (size_t)5 * npv;

    // gather + normalise + bf16: wavefront w row w
    FirstTile<K0> first;
    {
        const int din = na.dims[0];
        const int row = r0 + wave;
        const bool in = row < B;
        const int rc = in ? row : B - 1;
        const size_t src = idx ? (size_t)gmem(idx)[rc] : (size_t)rc;
        const global_t<const float>* x = gmem(rows) + src * rw;
        uint16_t* o = act(0) + wave * ld;
        float xv[5];
        for (int n0 = 0; n0 < npv; n0 += 64) {
            const int n = n0 + lane;
            const int nc = n < npv ? n : npv - 1;
#pragma unroll
            for (int j = 0; j < 5; ++j) xv[j] = x[in_var[j] * npv + nc];
            if (n0 == 0) {
#pragma unroll
                for (int j = 0; j < 5; ++j) arrived(xv[j]);
                first.load(na, wave, lane);
            }
#pragma unroll
            for (int j = 0; j < 5; ++j)
                if (j < na.n_in) {
                    const float v = net_input(na, npv, j, nc, (double)xv[j]);
                    if (n < npv) o[j * npv + n] = f2bf(in ? v : 0.0f);
                }
        }
        for (int c = din + lane; c < 32 * K0; c += 64) o[c] = f2bf(0.0f);
    }
    // the lane's four rows of the targets
    size_t ysrc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = r0 + 4 * g + i < B ? r0 + 4 * g + i : B - 1;
        ysrc[i] = (idx ? (size_t)gmem(idx)[row] : (size_t)row) * rw;
    }
    __syncthreads();
    // its place in the transposed arrays, in column tile 0: batch rows
    // r0 + 4 g .. + 3 of column r
    const int64_t tile_step = (int64_t)(Bp >> 5) * 512;
    const int64_t tr = wfrag_index(r, r0 + 4 * g, Bp);

    bf16x8 b[K0 > 8 ? K0 : 8];
    float bn = first.bias;
    floatx4 acc = mma_steps<K0>(first.b, act(0) + r * ld + 8 * g);
    store_transposed(act(0), ld, 32 * K0, gmem(ta.actT[0]), r0, Bp, t);
    float yv[2][4];
    const Five<int> out_var(na.out_var);
    for (int l = 0; l + 1 < L; ++l) {
        const bool out = l + 2 == L;
        const __amdgpu_buffer_rsrc_t rs = weight_rsrc(gmem(na.W[l + 1]), 256, out ? Np : 256);
        const int tile = out && wave >= nt ? nt - 1 : wave;
        const int vo = (tile * 8 * 64 + lane) * 16;
        const int n1 = tile * 16 + r;
        const float bnext = gmem(na.b[l + 1])[out && n1 >= Nd ? Nd - 1 : n1];
        uint16_t* o = act(l + 1) + 4 * g * ld + wave * 16 + r;
        u16x4 h;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i == 0) load_steps<0, 2>(b, rs, vo);
            if (i == 1) load_steps<2, 4>(b, rs, vo);
            if (i == 2) load_steps<4, 6>(b, rs, vo);
            if (i == 3) load_steps<6, 8>(b, rs, vo);
            net_fence();
            h[i] = f2bf(act_fwd(acc[i] + bn, ACT));
            o[i * ld] = h[i];
            net_fence();
        }
        *(global_t<u16x4>*)(gmem(ta.actT[l + 1]) + wave * tile_step + tr) = h;
        if (out) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int n = (wave + s * kRowWaves) * 16 + r;
                const int nc = n < Nd ? n : Nd - 1;
                const int j = (nc >= npv) + (nc >= 2 * npv) + (nc >= 3 * npv) + (nc >= 4 * npv);
                const int c = out_var.at(j) * npv + nc - j * npv;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    yv[s][i] = gmem(ta.y)[ysrc[i] + c];
            }
        }
        bn = bnext;
        __syncthreads();
        acc = mma_steps<8>(b, act(l + 1) + r * ld + 8 * g);
    }
    // output layer: loss gradient dY = scale (yhat - ytilde); its first tile's
    // products are in acc
    float lsum = 0.0f;
    const Five<double> out_mu(na.out_mu), out_isig(na.out_isig);
    auto output_tile = [&](int tile, const float (&y)[4]) {
        const int n = tile * 16 + r;
        const int nc = n < Nd ? n : Nd - 1;
        const int j = (nc >= npv) + (nc >= 2 * npv) + (nc >= 3 * npv) + (nc >= 4 * npv);
        const double mu = out_mu.at(j), isig = out_isig.at(j);
        u16x4 d;
        float bsum = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float dy = 0.0f;
            if (r0 + 4 * g + i < B && n < Nd) {
                float yt;
                if (na.col) {
                    const int cc = out_var.at(j) * npv + nc - j * npv;
                    yt = (float)(((double)y[i] - gmem(na.col)[10 * npv + cc]) / gmem(na.col)[15 * npv + cc]);
                } else {
                    yt = (float)(((double)y[i] - mu) * isig);
                }
                const float diff = acc[i] + bn - yt;
                lsum += diff * diff;
                dy = ta.grad_scale * diff;
            }
            d[i] = f2bf(dy);
            g0[(4 * g + i) * ld + n] = d[i];
            bsum += bf2f(d[i]);
        }
        *(global_t<u16x4>*)(gmem(ta.dzT[L - 1]) + tile * tile_step + tr) = d;
        bsum += __shfl_xor(bsum, 16);
        bsum += __shfl_xor(bsum, 32);
        if (g == 0) gmem(ta.bias_part[L - 1])[(size_t)blockIdx.x * Np + n] = bsum;
    };
    if (wave + kRowWaves < nt) {
        const int n1 = (wave + kRowWaves) * 16 + r;
        load_steps<0, 8>(b, weight_rsrc(gmem(na.W[L - 1]), 256, Np), ((wave + kRowWaves) * 8 * 64 + lane) * 16);
        const float bnext = gmem(na.b[L - 1])[n1 < Nd ? n1 : Nd - 1];
        output_tile(wave, yv[0]);
        bn = bnext;
        acc = mma_steps<8>(b, act(L - 1) + r * ld + 8 * g);
        output_tile(wave + kRowWaves, yv[1]);
    } else if (wave < nt) {
        output_tile(wave, yv[0]);
    }
    // the first backward product's weights: K0 steps, as the input has
    load_steps<0, K0>(b, weight_rsrc(gmem(na.WT[L - 1]), 32 * K0, 256), (wave * K0 * 64 + lane) * 16);
    // the block's loss: a fixed butterfly within each wavefront, then
    // wavefront 0 sums the sixteen partial sums in order
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off);
    if (lane == 0) red[wave] = lsum;
    __syncthreads();
    if (t == 0) {
        float sum = 0.0f;
        for (int w = 0; w < kRowWaves; ++w) sum += red[w];
        ta.loss_part[blockIdx.x] = sum;
    }
    // backward data chain
    uint16_t* gin = g0;
    uint16_t* gout = g1;
    acc = mma_steps<K0>(b, gin + r * ld + 8 * g);
    for (int l = L - 1; l >= 1; --l) {
        const uint16_t* h = act(l) + 4 * g * ld + wave * 16 + r;
        uint16_t* o = gout + 4 * g * ld + wave * 16 + r;
        const bool more = l > 1;
        const __amdgpu_buffer_rsrc_t rs = weight_rsrc(gmem(na.WT[more ? l - 1 : l]), 256, 256);
        const int vo = (wave * 8 * 64 + lane) * 16;
        u16x4 d;
        float bsum = 0.0f;
        if (more) load_steps<0, 8>(b, rs, vo);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = acc[i] * act_bwd(bf2f(h[i * ld]), ACT);
            d[i] = f2bf(r0 + 4 * g + i < B ? v : 0.0f);
            o[i * ld] = d[i];
            bsum += bf2f(d[i]);
        }
        *(global_t<u16x4>*)(gmem(ta.dzT[l - 1]) + wave * tile_step + tr) = d;
        bsum += __shfl_xor(bsum, 16);
        bsum += __shfl_xor(bsum, 32);
        if (g == 0) gmem(ta.bias_part[l - 1])[(size_t)blockIdx.x * 256 + wave * 16 + r] = bsum;
        if (more) {
            __syncthreads();
            uint16_t* tmp = gin;
            gin = gout;
            gout = tmp;
            acc = mma_steps<8>(b, gin + r * ld + 8 * g);
        }
    }
}

// Adam update of parameter i (flat index) with gradient gi and its old moments
// and value, loaded by the caller; returns the new value
struct AdamState {
    float m, v, p;
};
__device__ __forceinline__ AdamState adam_load(const AdamArgs& aa, int64_t i) {
    return {gmem(aa.m)[i], gmem(aa.v)[i], gmem(aa.p)[i]};
}
__device__ __forceinline__ float adam_one(const AdamArgs& aa, int64_t i, float gi, const AdamState& s) {
    const float mi = aa.b1 * s.m + (1.0f - aa.b1) * gi;
    const float vi = aa.b2 * s.v + (1.0f - aa.b2) * gi * gi;
    gmem(aa.m)[i] = mi;
    gmem(aa.v)[i] = vi;
    const float pi = s.p - aa.lr * (mi / aa.bc1) / (sqrtf(vi / aa.bc2) + aa.eps);
    gmem(aa.p)[i] = pi;
    return pi;
}

// layer of entry x of a list whose layers end at end[l + 1] (one load of the
// ends, where a search would wait for one after the other)
__device__ __forceinline__ int layer_of(const int (&end)[kMaxLayers + 1], int n_layers, int x) {
    int l = 0;
#pragma unroll
    for (int i = 1; i < kMaxLayers; ++i) l += i < n_layers && x >= end[i];
    return l;
}

// The end of a training step in one launch.  Blocks [0, gtiles) take one
// 32 x 32 tile of a layer's weights each: gradient dz^T h over the whole
// batch, Adam, and the tile's share of the bf16 copies W_l [pout][pin] and
// W_l^T [pin][pout].  Eight wavefronts split the batch; each computes 2 x 2
// MFMA tiles (every fragment it loads feeds two products), and their sums are
// added in LDS in a fixed order.  Then bias blocks (32 biases each: the sums
// of the row blocks), then, with a loss output, one block for the loss.
// Bound by the reads of h and dz: tiles that share rows go to one XCD (the
// hardware deals blocks out to the eight in turn), whose L2 then takes 3.5 of
// the 19 MB at a batch of 4096 instead of all of them (21.2 -> 14.5 us;
// 64 x 32 tiles, which read a quarter less from L2, 15.8).
// With the split over blocks, the partial sums in memory and Adam in a launch
// of its own: 320-256-256-256-320, batch 512 6.2 + 6.6 us, 4096 13.0 + 9.3;
// so 6.6 and 14.4.
constexpr int kGradWaves = 8;
__global__ void __launch_bounds__(64 * kGradWaves) k_grad_adam(GradArgs ga, ParamMap pm, AdamArgs aa, int nbias) {
    constexpr int LDR = 36;    // floats a row of a partial tile: the four row groups of a store use other banks
    constexpr int LDH = 40;    // bf16 a row of the new weights, rows 16 bytes aligned
    constexpr int T = 64 * kGradWaves, NE = 1024 / T;
    __shared__ float red[kGradWaves][32 * LDR];
    __shared__ __attribute__((aligned(16))) uint16_t hw[2][32 * LDH];
    const int t = threadIdx.x;
    const int b = blockIdx.x;
    if (b < ga.gtiles) {
        const int tile = (b % 8) * (ga.gtiles / 8) + b / 8;
        if (tile >= ga.tblk[ga.n_layers]) return;
        const int l = layer_of(ga.tblk, ga.n_layers, tile);
        const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
        const int pout = ga.pout[l], pin = ga.pin[l], dout = ga.dout[l], din = ga.din[l];
        const int tiles_i = pin / 32;
        const int to = (tile - ga.tblk[l]) / tiles_i, ti = (tile - ga.tblk[l]) - to * tiles_i;
        // the weights of this thread
        int64_t at[NE];
        bool in[NE];
        AdamState old[NE];
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int o = to * 32 + t / 32 + j * (T / 32), i = ti * 32 + (t & 31);
            in[j] = o < dout && i < din;
            at[j] = in[j] ? (int64_t)o * din + i : 0;
            old[j] = adam_load(aa, pm.woff[l] + at[j]);
        }
        // dzT and actT are in fragment order over the batch (wfrag_index with
        // K = Bp): the 32-batch step s of 16-row tile t is the 1 KB block
        // t * Bp / 32 + s, lane-major
        const int ksteps = ga.Bp / 32;
        const int kn = (ksteps + kGradWaves - 1) / kGradWaves;
        const int kb = wave * kn, ke = kb + kn < ksteps ? kb + kn : ksteps;
        const global_t<bf16x8>* a0 = (const global_t<bf16x8>*)gmem(ga.dzT[l]) + (int64_t)2 * to * ksteps * 64 + lane;
        const global_t<bf16x8>* a1 = a0 + (int64_t)ksteps * 64;
        const global_t<bf16x8>* b0 = (const global_t<bf16x8>*)gmem(ga.actT[l]) + (int64_t)2 * ti * ksteps * 64 + lane;
        const global_t<bf16x8>* b1 = b0 + (int64_t)ksteps * 64;
        floatx4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
        for (int k = kb; k < ke; ++k) {
            const bf16x8 x0 = a0[k * 64], x1 = a1[k * 64], y0 = b0[k * 64], y1 = b1[k * 64];
            acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, y0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, y1, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, y0, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, y1, acc[1][1], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    red[wave][(16 * i + 4 * (lane >> 4) + v) * LDR + 16 * j + (lane & 15)] = acc[i][j][v];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int o = t / 32 + j * (T / 32), i = t & 31;
            float g = red[0][o * LDR + i];
#pragma unroll
            for (int w = 1; w < kGradWaves; ++w) g += red[w][o * LDR + i];
            uint16_t h = 0;   // past the true sizes the copies hold zeros
            if (in[j]) {
                gmem(ga.gW[l])[at[j]] = g;
                h = f2bf(adam_one(aa, pm.woff[l] + at[j], g, old[j]));
            }
            hw[0][o * LDH + i] = h;
            hw[1][i * LDH + o] = h;
        }
        __syncthreads();
        // two 1 KB fragments (16 rows, 32 columns) of each copy
        if (wave < 4) {
            const int c = wave >> 1, half = wave & 1;   // W or W^T
            const int64_t frag = c ? (int64_t)(2 * ti + half) * (pout / 32) + to : (int64_t)(2 * to + half) * (pin / 32) + ti;
            ((global_t<bf16x8>*)(gmem(aa.wbf) + (c ? pm.wtbo[l] : pm.wbo[l])))[frag * 64 + lane] =
                *(const bf16x8*)(hw[c] + (16 * half + (lane & 15)) * LDH + 8 * (lane >> 4));
        }
        return;
    }
    float(*sum)[33] = (float(*)[33])red;
    const int bblk = (nbias + 31) / 32;
    if (b < ga.gtiles + bblk) {
        const int n = (b - ga.gtiles) * 32 + (t & 31);   // bias n of all layers'
        int l = 0, o = n;
        while (l + 1 < ga.n_layers && o >= ga.dout[l]) {
            o -= ga.dout[l];
            ++l;
        }
        const bool in = n < nbias;
        AdamState old{};
        if (in && t < 32) old = adam_load(aa, pm.boff[l] + o);
        float s = 0.0f;
        if (in) {
            const global_t<float>* part = gmem(ga.bias_part[l]) + o;
            const int pout = ga.pout[l];
#pragma unroll 8
            for (int k = t / 32; k < ga.nrb; k += T / 32) s += part[(size_t)k * pout];
        }
        sum[t / 32][t & 31] = s;
        __syncthreads();
        if (in && t < 32) {
            s = sum[0][t];
            for (int w = 1; w < T / 32; ++w) s += sum[w][t];
            gmem(ga.gb[l])[o] = s;
            adam_one(aa, pm.boff[l] + o, s, old);
        }
        return;
    }
    // the loss: sum of the row-block partials
    float s = 0.0f;
    for (int i = t; i < aa.n_loss; i += T) s += aa.loss_part[i];
    red[0][t] = s;
    __syncthreads();
    for (int w = T / 2; w > 0; w >>= 1) {
        if (t < w) red[0][t] += red[0][t + w];
        __syncthreads();
    }
    if (t == 0) aa.loss[0] = red[0][0] * aa.inv_count;
}

// Per-variable statistics of a training set (rows of 5 n_p floats).  Pass 0
// sums values, pass 1 squared deviations from the pass-0 means; each block
// reduces a contiguous chunk of rows, the final kernel sums the block
// partials in order.
__global__ void __launch_bounds__(256) k_stats_partial(const float* __restrict__ x, const float* __restrict__ y,
                                                      int64_t rows, int n_p, const double* __restrict__ mean,
                                                      double* __restrict__ part) {
    __shared__ double red[10][256];
    const int t = threadIdx.x;
    const int64_t per = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = (int64_t)blockIdx.x * per;
    const int64_t r1 = r0 + per < rows ? r0 + per : rows;
    const int width = 5 * n_p;
    double acc[10];
    for (int c = 0; c < 10; ++c) acc[c] = 0.0;
    for (int64_t r = r0; r < r1; ++r)
        for (int c = t; c < width; c += 256) {
            const int v = c / n_p;
            const double a = x[r * width + c], b = y[r * width + c];
            if (mean) {
                const double da = a - mean[v], db = b - mean[5 + v];
                acc[v] += da * da;
                acc[5 + v] += db * db;
            } else {
                acc[v] += a;
                acc[5 + v] += b;
            }
        }
    for (int c = 0; c < 10; ++c) red[c][t] = acc[c];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w)
            for (int c = 0; c < 10; ++c) red[c][t] += red[c][t + w];
        __syncthreads();
    }
    if (t < 10) part[(size_t)blockIdx.x * 10 + t] = red[t][0];
}

__global__ void k_stats_means(const double* __restrict__ out, double* __restrict__ mean) {
    const int c = threadIdx.x;
    if (c < 10) mean[c] = out[10 * (c / 5) + (c % 5)];
}

// out layout: mu_x[5], sigma_x[5], mu_y[5], sigma_y[5]
__global__ void k_stats_final(const double* __restrict__ part, int nblocks, double count, int pass,
                              double* __restrict__ out) {
    const int c = threadIdx.x;
    if (c >= 10) return;
    double s = 0.0;
    for (int b = 0; b < nblocks; ++b) s += part[(size_t)b * 10 + c];
    const int v = c % 5, which = c / 5;          // which: 0 x, 1 y
    if (pass == 0) {
        out[10 * which + v] = s / count;
    } else {
        const double mu = out[10 * which + v];
        const double floor_v = 1e-12 * fmax(1.0, fabs(mu));
        out[10 * which + 5 + v] = fmax(sqrt(s / count), floor_v);
    }
}

// Per-column statistics of a training set (x and y rows of ncols floats):
// block b sums its contiguous chunk of rows for every column (pass 0 values,
// pass 1 squared deviations from the pass-0 means), the final kernel sums the
// block partials in order.  out: [4][ncols] = mu_x, sigma_x, mu_y, sigma_y.
__global__ void __launch_bounds__(256) k_colstats_partial(const float* __restrict__ x, const float* __restrict__ y,
                                                         int64_t rows, int ncols, const double* __restrict__ out,
                                                         int pass, double* __restrict__ part) {
    const int64_t per = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = (int64_t)blockIdx.x * per;
    const int64_t r1 = r0 + per < rows ? r0 + per : rows;
    for (int c = threadIdx.x; c < 2 * ncols; c += 256) {
        const float* A = c < ncols ? x : y;
        const int cc = c < ncols ? c : c - ncols;
        const double mu = pass ? out[(c < ncols ? 0 : 2 * ncols) + cc] : 0.0;
        double s = 0.0;
        for (int64_t r = r0; r < r1; ++r) {
            const double v = (double)A[r * ncols + cc] - mu;
            s += pass ? v * v : v;
        }
        part[(size_t)blockIdx.x * 2 * ncols + c] = s;
    }
}

__global__ void __launch_bounds__(256) k_colstats_final(const double* __restrict__ part, int nblocks, int ncols,
                                                       double count, int pass, double* __restrict__ out) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= 2 * ncols) return;
    double s = 0.0;
    for (int b = 0; b < nblocks; ++b) s += part[(size_t)b * 2 * ncols + c];
    const int base = c < ncols ? 0 : 2 * ncols, cc = c < ncols ? c : c - ncols;
    if (pass == 0) {
        out[base + cc] = s / count;
    } else {
        const double mu = out[base + cc];
        out[base + ncols + cc] = fmax(sqrt(s / count), 1e-12 * fmax(1.0, fabs(mu)));
    }
}

// ------------------------------------------------------------ host launchers

hipError_t launch_data_stats(const float* x, const float* y, int64_t rows, int n_p, double* part, int nblocks,
                             double* out, hipStream_t st) {
    const double count = (double)rows * n_p;
    hipLaunchKernelGGL(k_stats_partial, dim3(nblocks), dim3(256), 0, st, x, y, rows, n_p, (const double*)nullptr,
                       part);
    hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(64), 0, st, part, nblocks, count, 0, out);
    // pass 1 needs the means in the layout mean[v] (x) and mean[5 + v] (y): gather them
    hipLaunchKernelGGL(k_stats_means, dim3(1), dim3(64), 0, st, out, out + 20);
    hipLaunchKernelGGL(k_stats_partial, dim3(nblocks), dim3(256), 0, st, x, y, rows, n_p, out + 20, part);
    hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(64), 0, st, part, nblocks, count, 1, out);
    return hipGetLastError();
}

static size_t net_smem_bytes(const NetArgs& na, int nbuf) {
    return (size_t)nbuf * kRows * na.ld * sizeof(uint16_t);
}

static hipError_t launch_forcing(const NetArgs& na, int n_p, const NetTarget* targets, int nt, int nblocks,
                                 int accumulate, hipStream_t st) {
    if (nt < 1 || nt > 16) return hipErrorInvalidValue;
    NetTargets tg;
    for (int i = 0; i < nt; ++i) tg.t[i] = targets[i];
    tg.n = nt;
    const size_t smem = net_smem_bytes(na, 2);
    auto kernel = k_net_forcing<0, 0>;
    switch (net256_steps(na)) {
        case 3: kernel = na.act ? k_net_forcing<3, 1> : k_net_forcing<3, 0>; break;
        case 5: kernel = na.act ? k_net_forcing<5, 1> : k_net_forcing<5, 0>; break;
        case 6: kernel = na.act ? k_net_forcing<6, 1> : k_net_forcing<6, 0>; break;
        case 10: kernel = na.act ? k_net_forcing<10, 1> : k_net_forcing<10, 0>; break;
        default: break;
    }
    if (smem > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(kRowThreads), smem, st, na, n_p, tg, accumulate);
    return hipGetLastError();
}

hipError_t launch_net_forcing(const NetArgs& na, int n_p, const NetTarget* targets, int nt, int nblocks,
                              hipStream_t st) {
    return launch_forcing(na, n_p, targets, nt, nblocks, 1, st);
}

hipError_t launch_net_forcing_write(const NetArgs& na, int n_p, const NetTarget* targets, int nt, int nblocks,
                                    hipStream_t st) {
    return launch_forcing(na, n_p, targets, nt, nblocks, 0, st);
}

hipError_t launch_net_refresh_layer(const NetArgs& na, const float* params, int64_t woff, int l, uint16_t* wbf,
                                    int64_t wbf_off, int64_t wtbf_off, hipStream_t st) {
    const int total = na.pdims[l] * na.pdims[l + 1];
    int blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_net_refresh, dim3(blocks), dim3(256), 0, st, na, params, wbf, woff, l, wbf_off,
                       wtbf_off);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, float v, size_t n, hipStream_t st) {
    int blocks = (int)((n + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_fill_f32, dim3(blocks), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

size_t train_smem_bytes(const NetArgs& na) { return net_smem_bytes(na, na.n_layers + 2); }

template <int K0>
static hipError_t launch_train256(const NetArgs& na, const TrainArgs& ta, int blocks, size_t smem, hipStream_t st) {
    const auto kernel = na.act ? k_train256<K0, 1> : k_train256<K0, 0>;
    if (smem > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
    }
    const int* v = na.in_var;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kRowThreads), smem, st, ta.x, ta.idx, ta.B, ta.Bp,
                       na.dims[0] / na.n_in, v[0], v[1], v[2], v[3], v[4], na, ta);
    return hipGetLastError();
}

hipError_t launch_train_rows(const NetArgs& na, const TrainArgs& ta, int nblocks, hipStream_t st) {
    const size_t smem = train_smem_bytes(na);
    // one block on each XCD reads the weights ahead of the row blocks (batch
    // 1024, eight row blocks an XCD: no change; 2048 21.6 -> 21.9 us)
    const int ahead = nblocks + (8 * nblocks <= cu_count() ? 8 : 0);
    // the backward chain starts with as many steps as the forward one where
    // the network reads as many columns as it forces
    if (na.pdims[na.n_layers] == na.pdims[0]) switch (net256_steps(na)) {
        case 3: return launch_train256<3>(na, ta, ahead, smem, st);
        case 5: return launch_train256<5>(na, ta, ahead, smem, st);
        case 6: return launch_train256<6>(na, ta, ahead, smem, st);
        case 10: return launch_train256<10>(na, ta, ahead, smem, st);
        default: break;
    }
    if (smem > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)k_train_rows, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_train_rows, dim3(nblocks), dim3(kRowThreads), smem, st, na, ta);
    return hipGetLastError();
}

hipError_t launch_grad_adam(const GradArgs& ga, const ParamMap& pm, const AdamArgs& aa, hipStream_t st) {
    int nbias = 0;
    for (int l = 0; l < ga.n_layers; ++l) nbias += ga.dout[l];
    const int blocks = ga.gtiles + (nbias + 31) / 32 + (aa.loss ? 1 : 0);
    hipLaunchKernelGGL(k_grad_adam, dim3(blocks), dim3(64 * kGradWaves), 0, st, ga, pm, aa, nbias);
    return hipGetLastError();
}

hipError_t launch_column_stats(const float* x, const float* y, int64_t rows, int ncols, double* part, int nblocks,
                               double* out, hipStream_t st) {
    const int fb = (2 * ncols + 255) / 256;
    const double count = (double)rows;
    for (int pass = 0; pass < 2; ++pass) {
        hipLaunchKernelGGL(k_colstats_partial, dim3(nblocks), dim3(256), 0, st, x, y, rows, ncols,
                           (const double*)out, pass, part);
        hipLaunchKernelGGL(k_colstats_final, dim3(fb), dim3(256), 0, st, part, nblocks, ncols, count, pass, out);
    }
    return hipGetLastError();
}

}  // namespace dgnn
