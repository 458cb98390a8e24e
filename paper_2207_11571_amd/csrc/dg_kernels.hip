// FP64 DGSEM kernels for gfx950: face traces, BR1 gradient pass, residual and
// Runge-Kutta stage update, Taylor-Green initial condition, diagnostics,
// filter G and training-pair packing.
//
// Discretisation (Sec. 2.6, Sec. 3.1, App. A): weak-form nodal DGSEM on
// Gauss-Legendre points, Roe interface flux, BR1 gradients of (u, v, w, T)
// and viscous fluxes, optional Smagorinsky closure, on uniform periodic
// hexahedra.
//
// Per Runge-Kutta stage two kernels run (BR1 needs neighbours' gradients,
// which need their neighbours' traces); their device code is in dg_lines.hpp:
//   k_grad  : q, neighbour q traces -> BR1 gradient -> one-sided viscous normal
//             flux on the element's six faces (fv);
//   k_resid : q, neighbour q traces, fv of both sides -> Roe minus averaged
//             viscous interface flux, volume flux divergence, forcing ->
//             residual, or the low-storage stage update of q and k plus the
//             face traces of the new q for the next stage.
#include <mutex>

#include "dgnn_internal.hpp"
#include "nn_device.hpp"

namespace dgnn {

__constant__ BasisTab c_basis[DG_MAX_ORDER];
__constant__ FilterTab c_filter[DG_MAX_ORDER * DG_MAX_ORDER];

// The arrays a solve descriptor points to are addressed through gmem()
// (global memory): read from a descriptor in memory they are generic
// pointers, and generic (flat) accesses count against the LDS counter as
// well, so every LDS access would wait for the element's global loads and
// stores in flight.
using gdouble = global_t<double>;

__device__ __forceinline__ int find_solve(const DescList& dl, int b) {
    int s = 0;
    for (int i = 1; i < dl.n; ++i)
        if (dl.blk[i] <= b) s = i;
    return s;
}

// --------------------------------------------------------------- physics

// 1/x for x > 0 normal: hardware estimate refined by two Newton-Raphson
// steps r <- r + r (1 - x r), each doubling the correct bits
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// sqrt(x) for x > 0 normal: hardware 1/sqrt estimate y, then Goldschmidt's
// coupled iteration on g ~ sqrt(x), h ~ 1/(2 sqrt(x)) and a final residual
// correction g + h (x - g^2)
__device__ __forceinline__ double sqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    const double d = fma(-g, g, x);
    return fma(d, h, g);
}

}  // namespace dgnn

#include "dg_lines.hpp"

namespace dgnn {

// ---------------------------------------------------------------- kernels
//
// Order in which a launch takes the groups of a solve.  The hardware deals
// workgroups out to the eight XCDs in turn, and each XCD has an L2 of its own.
// kRange gives each XCD a contiguous range of the groups, the same in every
// launch: most neighbours' traces and fluxes, and what the launch before left,
// are in its own L2.  kTurn follows the workgroups, kBack in reverse.
enum Order { kTurn, kRange, kBack };

// groups of the elements of one solve
template <int PP>
__host__ __device__ __forceinline__ int groups(int E) {
    return (E + Line<PP>::EPG - 1) / Line<PP>::EPG;
}

__device__ __forceinline__ int xcd_range(int b, int n) {
    const int x = b & 7, each = n >> 3, more = n & 7;
    return x * each + (x < more ? x : more) + (b >> 3);
}
template <int PP, Order ORDER>
__device__ __forceinline__ int group_of_block(int E) {
    return ORDER == kRange  ? xcd_range(blockIdx.x, groups<PP>(E))
           : ORDER == kBack ? (int)(gridDim.x - 1 - blockIdx.x)
                            : (int)blockIdx.x;
}

// k_grad and k_resid exist twice: for one solve with its descriptor in the
// kernel arguments (two dependent loads fewer before a block's first data
// load), and for a list of solves whose descriptors are in device memory.

// What a block's first loads need comes as arguments of its own ahead of the
// descriptor: the first sixteen words of a kernel's arguments are in scalar
// registers when its wavefronts start (the build asks for that), where a load
// of them would be the first of three dependent ones.  A step of a long call:
// 4^3 P=3 24.3 -> 21.5 us, 8^3 P=3 27.9 -> 25.9, 8^3 P=6 57.0 -> 55.0, 16^3 P=3
// 76.8 -> 73.1.  (A call of one step takes the trace launch more, 8 % and
// above; of small meshes it is bound by the host's enqueueing.)
__device__ __forceinline__ SolveDesc with_head(const SolveDesc& D, const double* state, const double* qtr_in, double* fv, int N,
                                               int E) {
    SolveDesc S = D;
    S.q = const_cast<double*>(state);
    S.qtr_in = qtr_in;
    S.fv = fv;
    S.N = N;
    S.E = E;
    return S;
}

template <int PP, Order ORDER>
__global__ void __launch_bounds__(Line<PP>::NT) k_traces(const double* state, int N, int E, SolveDesc D) {
    __shared__ double sh[7 * Line<PP>::FS];
    const SolveDesc S = with_head(D, state, nullptr, nullptr, N, E);
    traces_group<PP>(S, group_of_block<PP, ORDER>(S.E), threadIdx.x, sh);
}

template <int PP, Order ORDER>
__global__ void __launch_bounds__(Line<PP>::NT) __attribute__((amdgpu_waves_per_eu(line_waves<GradLds<PP>, Line<PP>::NT>()))) k_grad1(const double* state, const double* qtr_in, double* fv, int N, int E, SolveDesc D) {
    const SolveDesc S = with_head(D, state, qtr_in, fv, N, E);
    __shared__ double sh[GradLds<PP>::N];
    double q[Line<PP>::NN][5];
    grad_group<PP>(S, group_of_block<PP, ORDER>(S.E), threadIdx.x, sh, q);
}

template <int PP>
__global__ void __launch_bounds__(Line<PP>::NT) __attribute__((amdgpu_waves_per_eu(line_waves<GradLds<PP>, Line<PP>::NT>()))) k_grad(DescList dl) {
    __shared__ double sh[GradLds<PP>::N];
    const int block = blockIdx.x;
    const int si = find_solve(dl, block);
    double q[Line<PP>::NN][5];
    grad_group<PP>(*dl.d[si], block - dl.blk[si], threadIdx.x, sh, q);
}

// P = 3 with the forcing network at every stage (Eq. (4)): the BR1 pass of
// sixteen elements, one per wavefront, and the network on the same sixteen
// rows in one launch.  Each wavefront works on its own element in its own
// LDS area, so between the BR1 pass's phases it waits for itself only, not
// for the block.  After the BR1 pass each wavefront holds its
// element's state in registers (node n in lane n), so it writes the
// element's normalised network input row straight into LDS instead of the
// network gathering the state from HBM again, and the layers follow in the
// same block.  The same device code as k_grad and k_net_forcing, so the same
// numbers.  One solve per launch (its descriptor in the kernel arguments),
// E a multiple of 16.
template <int PP, int K0, int ACT>
__global__ void __launch_bounds__(kRowThreads) k_grad_net(const double* state, const double* qtr_in, double* fv, int N, int E, SolveDesc D, NetArgs na, NetTarget T) {
    const SolveDesc S = with_head(D, state, qtr_in, fv, N, E);
    using L = Line<PP>;
    static_assert(L::NT == 64 && L::NP == 64 && L::EPG == 1, "one element per wavefront, one node per lane");
    constexpr int NP = L::NP;
    extern __shared__ __attribute__((aligned(16))) double gsm[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ld = na.ld;
    uint16_t* bufA = (uint16_t*)(gsm + kRowWaves * GradLds<PP>::N);
    uint16_t* bufB = bufA + kRows * ld;
    const int e0 = xcd_range(blockIdx.x, S.E / kRows) * kRows;

    double q[1][5];
    grad_group<PP>(S, __builtin_amdgcn_readfirstlane(e0 + wave), lane, gsm + wave * GradLds<PP>::N, q);

    FirstTile<K0 ? K0 : 1> first;
    if constexpr (K0 > 0) first.load(na, wave, lane);
    // row `wave` of the network input: column j NP + n is node n of
    // variable in_var[j]
    const int din = na.dims[0], pin = na.pdims[0];
    uint16_t* row = bufA + wave * ld;
    for (int j = 0; j < na.n_in; ++j) {
        const int v = na.in_var[j];
        const double qv = v == 0 ? q[0][0] : (v == 1 ? q[0][1] : (v == 2 ? q[0][2] : (v == 3 ? q[0][3] : q[0][4])));
        row[j * NP + lane] = f2bf(net_input(na, NP, j, lane, qv));
    }
    for (int c = din + lane; c < pin; c += 64) row[c] = f2bf(0.0f);
    net_zero_unforced(na, NP, T, e0, threadIdx.x);
    __syncthreads();
    if constexpr (K0 > 0) net256_forward<K0, ACT>(na, NP, T, e0, 0, bufA, bufB, ld, wave, lane, first);
    else net_block_forward(na, NP, T, e0, 0, bufA, bufB, ld, wave, lane);
}

// The same two on a mesh that does not fill the GPU with such blocks: the
// first blocks do the network of sixteen elements each, the others the BR1
// pass of sixteen elements, side by side on different CUs in one launch
// (512 elements: 12.3 us, against 12.3 us for the network and 4.0 us for the
// BR1 pass).
template <int PP, int K0, int ACT>
__global__ void __launch_bounds__(kRowThreads) k_grad_beside_net(const double* state, const double* qtr_in, double* fv, int N, int E, int v0, int v1, int v2, int v3, int v4,
                  int net_blocks, SolveDesc D, NetArgs na, double* forcing) {
    const SolveDesc S = with_head(D, state, qtr_in, fv, N, E);
    const NetTarget T = {state, forcing, E, 0};
    using L = Line<PP>;
    static_assert(L::NT == 64 && L::EPG == 1, "one element per wavefront");
    extern __shared__ __attribute__((aligned(16))) double gsm[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if ((int)blockIdx.x >= net_blocks) {
        const int e = xcd_range((int)blockIdx.x - net_blocks, net_blocks) * kRowWaves + wave;
        double q[1][5];
        if (e < S.E) grad_group<PP>(S, e, lane, gsm + wave * GradLds<PP>::N, q);
        return;
    }
    const int ld = na.ld, e0 = xcd_range(blockIdx.x, net_blocks) * kRows;
    uint16_t* bufA = (uint16_t*)gsm;
    uint16_t* bufB = bufA + kRows * ld;
    FirstTile<K0> first;
    const int in_var[5] = {v0, v1, v2, v3, v4};
    net_gather<K0>(na, in_var, L::NP, T, e0, bufA, ld, wave, lane, first);
    net_zero_unforced(na, L::NP, T, e0, threadIdx.x);
    __syncthreads();
    net256_forward<K0, ACT>(na, L::NP, T, e0, 0, bufA, bufB, ld, wave, lane, first);
}

// kBack (see streams()): the launch begins with what the BR1 pass left in the
// cache, and ends where the next begins; the register passes by the caches.
template <int PP, int UPDATE, int VISC, Order ORDER>
__global__ void __launch_bounds__(Line<PP>::NT) __attribute__((amdgpu_waves_per_eu(line_waves<ResidLds<PP>, Line<PP>::NT>())))
k_resid1(const double* state, const double* qtr_in, double* fv, int N, int E, int first_stage, SolveDesc D, double rkA,
         double rkB) {
    const SolveDesc S = with_head(D, state, qtr_in, fv, N, E);
    __shared__ double sh[ResidLds<PP>::N];
    resid_group<PP, UPDATE, VISC, ORDER == kBack>(S, group_of_block<PP, ORDER>(S.E), threadIdx.x, sh, rkA, rkB, first_stage);
}

// the stage update of a list of solves, all with viscous fluxes
template <int PP, bool STREAM>
__global__ void __launch_bounds__(Line<PP>::NT) __attribute__((amdgpu_waves_per_eu(line_waves<ResidLds<PP>, Line<PP>::NT>())))
k_resid(DescList dl, double rkA, double rkB, int first_stage) {
    __shared__ double sh[ResidLds<PP>::N];
    const int block = STREAM ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
    const int si = find_solve(dl, block);
    resid_group<PP, 1, 1, STREAM>(*dl.d[si], block - dl.blk[si], threadIdx.x, sh, rkA, rkB, first_stage);
}

// Taylor-Green vortex initial condition, Eq. (11), on [0, L]^3.
template <int PP>
__global__ void __launch_bounds__(768) k_tgv(Phys ph, int N, double* __restrict__ q) {
    constexpr int NP = PP * PP * PP;
    const int e = blockIdx.x;
    const int t = threadIdx.x;
    if (t >= NP) return;
    const BasisTab& B = c_basis[PP - 2];
    const int i = t % PP, j = (t / PP) % PP, k = t / (PP * PP);
    const int ex = e % N, ey = (e / N) % N, ez = e / (N * N);
    const double h = ph.h;
    const double x = ex * h + (B.nodes[i] + 1.0) * h * 0.5;
    const double y = ey * h + (B.nodes[j] + 1.0) * h * 0.5;
    const double z = ez * h + (B.nodes[k] + 1.0) * h * 0.5;
    const double u = sin(x) * cos(y) * cos(z);
    const double v = -cos(x) * sin(y) * cos(z);
    const double p = ph.p0 + (cos(2.0 * x) + cos(2.0 * y)) * (cos(2.0 * z) + 2.0) / 16.0;
    const size_t vs = (size_t)N * N * N * NP;
    const size_t n = (size_t)e * NP + t;
    q[n] = 1.0;
    q[vs + n] = u;
    q[2 * vs + n] = v;
    q[3 * vs + n] = 0.0;
    q[4 * vs + n] = p / ph.gm1 + 0.5 * (u * u + v * v);
}

// fmax and fmin drop a NaN, and a state that has blown up would show the values
// of its finite nodes.  NaN is noted beside the joins and takes the joined
// value's place at their end: by the high words, of which a NaN's is the
// largest, or by sums that it enters.  (us a call at 32^3 P=6, joins that drop
// it / that keep it / so: diagnostics 85.9 / 87.3 / 86.3, error norm 87.5 / 88.6
// / 87.8.)
constexpr uint32_t kInfWord = 0x7ff00000;
__device__ __forceinline__ uint32_t high_word(double x) { return (uint32_t)__double2hiint(fabs(x)); }

// Reduction of eight values over 256 threads, in an order that depends on
// nothing but the thread numbers: value 1 by maximum, 2 by minimum, the others
// by sum.  In LDS red[c][x]; thread 32 c returns value c.
constexpr int kReduceRow = 257;   // row stride of red: the writers of one x use different banks
__device__ __forceinline__ double diag_join(int c, double a, double b) {
    return c == 1 ? fmax(a, b) : (c == 2 ? fmin(a, b) : a + b);
}
template <int COUNT>
__device__ __forceinline__ double reduce_rows(const double (&red)[8][kReduceRow], int t) {
    const int c = t >> 5, x = t & 31;
    double r = red[c][x];
    bool nan = r != r;
#pragma unroll
    for (int i = 1; i < COUNT / 32; ++i) {
        const double v = red[c][x + 32 * i];
        nan |= v != v;
        r = diag_join(c, r, v);
    }
#pragma unroll
    for (int w = 16; w > 0; w >>= 1) r = diag_join(c, r, __shfl_xor(r, w));
    return (uint32_t)(__ballot(nan) >> (t & 32)) ? NAN : r;
}

// Diagnostics, first launch: per block the kinetic-energy integrand's sum,
// max(|v| + c), min rho, and the integrals of the five conserved variables
// (quadrature-weighted) of the nodes it strides over.  Bound by its launch on
// small meshes and by reading the state on large ones; a fixed number of
// blocks, at most kDiagBlocks, so that the second launch stays short.  The
// launches take, with a block per element and a third launch for the mean ->
// so: 4^3 P=3 8.4 -> 6.5 us, 8^3 P=6 10.0 -> 9.8 and a launch gap, 16^3 P=6
// 25 -> 17.5, 32^3 P=6 160 -> 86 (450 MB).
constexpr int kDiagBlocks = 512;
static int diag_blocks(int E, int NP) {
    const size_t b = ((size_t)E * NP + 255) / 256;
    const size_t most = E < kDiagBlocks ? E : kDiagBlocks;   // the workspace holds a row an element
    return (int)(b < most ? b : most);
}

template <int PP>
__global__ void __launch_bounds__(256) k_diag_partial(Phys ph, int E, const double* __restrict__ q,
                                                     double* __restrict__ part) {
    constexpr int NP = PP * PP * PP;
    __shared__ double red[8][kReduceRow];
    const int t = threadIdx.x;
    const BasisTab& B = c_basis[PP - 2];
    double val[8] = {0.0, 0.0, 1e300, 0.0, 0.0, 0.0, 0.0, 0.0};
    double c2 = 0.0;   // smallest squared speed of sound
    const size_t vs = (size_t)E * NP, step = (size_t)gridDim.x * 256;
    const int advance = (int)(step % NP);
    int m = (int)(((size_t)blockIdx.x * 256 + t) % NP);   // node of the element
    for (size_t n = (size_t)blockIdx.x * 256 + t; n < vs; n += step, m = m + advance < NP ? m + advance : m + advance - NP) {
        const int i = m % PP, j = (m / PP) % PP, k = m / (PP * PP);
        const double wq = B.w[i] * B.w[j] * B.w[k];
        double qq[5];
        for (int v = 0; v < 5; ++v) qq[v] = q[v * vs + n];
        const double ir = 1.0 / qq[0];
        const double m2 = qq[1] * qq[1] + qq[2] * qq[2] + qq[3] * qq[3];
        val[0] += wq * 0.5 * m2 * ir;
        const double p = ph.gm1 * (qq[4] - 0.5 * m2 * ir);
        const double cc = ph.gamma * p * ir;
        c2 = fmin(c2, cc);
        val[1] = fmax(val[1], sqrt(m2) * ir + sqrt(cc));
        val[2] = fmin(val[2], qq[0]);
        for (int v = 0; v < 5; ++v) val[3 + v] += wq * qq[v];
    }
    // a NaN of the state is one of the sums', too
    const double state = val[0] + val[7];
    if (c2 < 0.0 || state != state) val[1] = NAN;
    if (val[3] != val[3]) val[2] = NAN;
    for (int c = 0; c < 8; ++c) red[c][t] = val[c];
    __syncthreads();
    const double r = reduce_rows<256>(red, t);
    if ((t & 31) == 0) part[(size_t)blockIdx.x * 8 + (t >> 5)] = r;
}

// Second launch, one block: the rows of the first, times the Jacobian
// (integrals) or its share of the volume (the mean kinetic energy).
__global__ void __launch_bounds__(256) k_diag_final(int rows, double mean_factor, double vol_factor,
                                                   const double* __restrict__ part, double* __restrict__ out) {
    __shared__ double red[8][kReduceRow];
    const int t = threadIdx.x, c = t & 7;
    // eight loads in flight; past the last row, the last once more, not joined
    double r = c == 2 ? 1e300 : 0.0;
    bool nan = false;
    for (int x0 = t >> 3; x0 < rows; x0 += 256) {
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int x = x0 + 32 * i;
            v[i] = part[(x < rows ? x : rows - 1) * 8 + c];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (x0 + 32 * i < rows) {
                nan |= v[i] != v[i];
                r = diag_join(c, r, v[i]);
            }
    }
    red[c][t >> 3] = nan ? NAN : r;
    __syncthreads();
    r = reduce_rows<32>(red, t);
    const int o = t >> 5;
    if ((t & 31) == 0) out[o] = o == 0 ? r * mean_factor : (o < 3 ? r : r * vol_factor);
}

// maximum of four numbers that are not negative, or NaN
__device__ __forceinline__ double join_waves(double a, double b, double c, double d) {
    const double m = fmax(fmax(a, b), fmax(c, d)), sum = (a + b) + (c + d);
    return sum != sum ? sum : m;
}

// Eq. (9): max |q_v - qref_v| of the three momenta, per block (rows of four)
__global__ void __launch_bounds__(256) k_err_partial(size_t vs, const double* __restrict__ q,
                                                    const double* __restrict__ qr, double* __restrict__ part) {
    __shared__ double red[4][3];
    const int t = threadIdx.x;
    double m[3] = {0.0, 0.0, 0.0};
    uint32_t high[3] = {0, 0, 0};
    const size_t step = (size_t)gridDim.x * 256;
    for (size_t n = (size_t)blockIdx.x * 256 + t; n < vs; n += step)
        for (int c = 0; c < 3; ++c) {
            const size_t idx = (1 + c) * vs + n;
            const double d = q[idx] - qr[idx];
            high[c] = max(high[c], high_word(d));
            m[c] = fmax(m[c], fabs(d));
        }
    for (int c = 0; c < 3; ++c) {
        for (int w = 32; w > 0; w >>= 1) m[c] = fmax(m[c], __shfl_xor(m[c], w));
        if (__ballot(high[c] > kInfWord)) m[c] = NAN;
    }
    if ((t & 63) == 0)
        for (int c = 0; c < 3; ++c) red[t >> 6][c] = m[c];
    __syncthreads();
    if (t < 3) part[(size_t)blockIdx.x * 4 + t] = join_waves(red[0][t], red[1][t], red[2][t], red[3][t]);
}

__global__ void __launch_bounds__(256) k_err_final(int rows, const double* __restrict__ part, double* __restrict__ out) {
    __shared__ double red[4][4];
    const int t = threadIdx.x;
    double m = 0.0;
    uint32_t high = 0;
    if ((t & 3) < 3)
        for (int x = t; x < rows * 4; x += 256) {
            const double v = part[x];
            high = max(high, high_word(v));
            m = fmax(m, v);
        }
    for (int w = 32; w > 3; w >>= 1) m = fmax(m, __shfl_xor(m, w));
    if (__ballot(high > kInfWord) >> (t & 3) & 0x1111111111111111ull) m = NAN;
    if ((t & 63) < 4) red[t >> 6][t & 3] = m;
    __syncthreads();
    if (t < 3) out[t] = join_waves(red[0][t], red[1][t], red[2][t], red[3][t]);
}

// Filter G: tensor-product 1D projection, one element per block, five
// variables.  A thread takes a line along x (straight from memory), then along
// y, then along z, each line's PPS entries to its PPD; the matrix is the same
// for all threads, in scalar registers.  Latency-bound on small meshes: 8^3
// elements, P = 8 to 3, with the matrix in the kernel's arguments, read lane by
// lane, and a thread per result 7.7 us, 5.5 so.  Pairs are packed
// in the same launch (5 us, and the projection in memory, less).
template <int PPS>
constexpr int kProjectThreads = (5 * PPS * PPS + 63) / 64 * 64;

template <int PPS, int PPD>
__global__ void __launch_bounds__(kProjectThreads<PPS>) k_project(int E, const double* __restrict__ src, ProjectOut out) {
    constexpr int NS = PPS * PPS * PPS, ND = PPD * PPD * PPD;
    __shared__ double b1[5 * PPS * PPS * PPD];   // [v][k][j][i']
    __shared__ double b2[5 * PPS * PPD * PPD];   // [v][k][j'][i']
    const int e = blockIdx.x, t = threadIdx.x;
    const double* G = c_filter[(PPS - 2) * DG_MAX_ORDER + PPD - 2].G;
    const auto line = [&](const double (&a)[PPS], double (&r)[PPD]) {
#pragma unroll
        for (int o = 0; o < PPD; ++o) {
            double acc = 0.0;
#pragma unroll
            for (int i = 0; i < PPS; ++i) acc += G[o * PPS + i] * a[i];
            r[o] = acc;
        }
    };
    double a[PPS], r[PPD];
    if (t < 5 * PPS * PPS) {
        const int v = t / (PPS * PPS), kj = t - v * PPS * PPS;
        const double* s = src + (size_t)v * E * NS + (size_t)e * NS + kj * PPS;
#pragma unroll
        for (int i = 0; i < PPS; ++i) a[i] = s[i];
        line(a, r);
#pragma unroll
        for (int o = 0; o < PPD; ++o) b1[t * PPD + o] = r[o];
    }
    __syncthreads();
    if (t < 5 * PPS * PPD) {
        const int vk = t / PPD, ip = t - vk * PPD;
#pragma unroll
        for (int j = 0; j < PPS; ++j) a[j] = b1[(vk * PPS + j) * PPD + ip];
        line(a, r);
#pragma unroll
        for (int o = 0; o < PPD; ++o) b2[(vk * PPD + o) * PPD + ip] = r[o];
    }
    __syncthreads();
    if (t < 5 * PPD * PPD) {
        const int v = t / (PPD * PPD), ji = t - v * PPD * PPD;
#pragma unroll
        for (int k = 0; k < PPS; ++k) a[k] = b2[(v * PPS + k) * PPD * PPD + ji];
        line(a, r);
        const size_t at = (size_t)v * E * ND + (size_t)e * ND + ji;
        const size_t row = (size_t)e * (5 * ND) + v * ND + ji;
#pragma unroll
        for (int o = 0; o < PPD; ++o) {
            const size_t n = o * PPD * PPD;
            if (out.y) {
                out.x[row + n] = (float)out.first[at + n];
                out.y[row + n] = (float)((r[o] - out.minus[at + n]) / out.div);
            } else {
                out.dst[at + n] = r[o];
                if (out.dst2) out.dst2[at + n] = r[o];
            }
        }
    }
}

struct DescBatch {
    SolveDesc d[4];
};

__global__ void k_write_descs(DescBatch b, int n, SolveDesc* dev) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (threadIdx.x == 0 && i < n) dev[i] = b.d[i];
}

// ------------------------------------------- scratch of the no-alloc stepper

// Workspace of dg_rk_step_noalloc: one array per GPU, loaded with the code
// object.  Host code never passes the array's name to a kernel or a copy (on
// the host it is a stand-in, not a device address); it uses the address that
// scratch_setup looks up per device.
static __device__ __align__(256) unsigned char scratch[DG_NOALLOC_SCRATCH_BYTES];

static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices];

hipError_t scratch_setup(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[dev]) return hipSuccess;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
    return hipSuccess;
}

void* scratch_device_ptr(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_scratch_ptr[dev];
}

// ------------------------------------------------------------ host launchers

hipError_t upload_basis_tables(const BasisTab* host_tabs, const FilterTab* host_filters) {
    const hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_filter), host_filters, sizeof(c_filter));
    if (e != hipSuccess) return e;
    return hipMemcpyToSymbol(HIP_SYMBOL(c_basis), host_tabs, sizeof(BasisTab) * DG_MAX_ORDER);
}

hipError_t launch_write_descs(const SolveDesc* host, int n, SolveDesc* dev, hipStream_t st) {
    if (n < 1 || n > 4) return hipErrorInvalidValue;
    DescBatch b;
    for (int i = 0; i < 4; ++i) b.d[i] = host[i < n ? i : 0];
    hipLaunchKernelGGL(k_write_descs, dim3(1), dim3(64), 0, st, b, n, dev);
    return hipGetLastError();
}

#define DG_DISPATCH_PP(PPV, CALL)           \
    switch (PPV) {                          \
        case 2: { constexpr int PP = 2; CALL; } break; \
        case 3: { constexpr int PP = 3; CALL; } break; \
        case 4: { constexpr int PP = 4; CALL; } break; \
        case 5: { constexpr int PP = 5; CALL; } break; \
        case 6: { constexpr int PP = 6; CALL; } break; \
        case 7: { constexpr int PP = 7; CALL; } break; \
        case 8: { constexpr int PP = 8; CALL; } break; \
        case 9: { constexpr int PP = 9; CALL; } break; \
        default: return hipErrorInvalidValue;          \
    }

// the list's first blocks (given in elements) in groups
template <int PP>
static DescList in_groups(const DescList& dl) {
    DescList g = dl;
    for (int i = 0; i < dl.n; ++i) g.blk[i + 1] = g.blk[i] + groups<PP>(dl.blk[i + 1] - dl.blk[i]);
    return g;
}

// Whether what a stage goes through (state, register, two sets of traces,
// viscous fluxes) exceeds the 256 MiB of the memory-side cache: then the
// register is kept out of it, and the stage update takes the groups in
// reverse.  A step of a long call, us, without -> with: 16^3 P=7 (328 MiB) 446
// -> 424, 16^3 P=8 605 -> 565, 20^3 P=5 (316 MiB) 392 -> 372, 24^3 P=6 1030 ->
// 974, 32^3 P=6 2389 -> 2266; below, 24^3 P=3 (209 MiB) 223 -> 234, 16^3 P=6
// (236 MiB) 298 -> 304.
template <int PP>
static bool streams(int E) {
    using L = Line<PP>;
    return (size_t)E * (2 * 5 * L::NP + 6 * (5 + 5 + 4) * L::NF) * sizeof(double) > ((size_t)256 << 20);
}

// Where the single solves' launches take the groups in ranges: while the data
// fit the memory-side cache, a step of a long call, us: 11^3 P=5 91.5 -> 83.3, 12^3 P=6 143 ->
// 136, 14^3 P=7 302 -> 286, two of 8^3 P=3 with the network (whose blocks take
// sixteen elements in a row) 111 -> 100.  With N a multiple of eight, groups in
// turn have their y and z neighbours on the same XCD already, and ranges gain
// nothing (16^3 P=6 300.5 -> 301.0, three of 8^3 P=8 324 -> 326): there only
// P = 3 takes them.  Beyond the cache, eight ranges far apart cost more than
// they save (24^3 P=6 962 -> 1120, 32^3 P=6 2310 -> 2540).
template <int PP>
static bool in_ranges(const SolveDesc& S) {
    return !streams<PP>(S.E) && (PP == 4 || S.N % 8 != 0);
}

hipError_t launch_traces(int PPv, const SolveDesc& S, hipStream_t st) {
    DG_DISPATCH_PP(PPv, hipLaunchKernelGGL((in_ranges<PP>(S) ? k_traces<PP, kRange> : k_traces<PP, kTurn>),
                                           dim3(groups<PP>(S.E)), dim3(Line<PP>::NT), 0, st, S.q, S.N, S.E, S));
    return hipGetLastError();
}

hipError_t launch_grad(int PPv, const SolveDesc& S, hipStream_t st) {
    DG_DISPATCH_PP(PPv, hipLaunchKernelGGL((in_ranges<PP>(S) ? k_grad1<PP, kRange> : k_grad1<PP, kTurn>),
                                           dim3(groups<PP>(S.E)), dim3(Line<PP>::NT), 0, st, S.q, S.qtr_in,
                                           S.fv, S.N, S.E, S));
    return hipGetLastError();
}

hipError_t launch_grad(int PPv, const DescList& dl, hipStream_t st) {
    DG_DISPATCH_PP(PPv, const DescList g = in_groups<PP>(dl);
                   hipLaunchKernelGGL(k_grad<PP>, dim3(g.blk[g.n]), dim3(Line<PP>::NT), 0, st, g));
    return hipGetLastError();
}

// compute units of the current device (persistent launches size their grid
// by it), looked up once per device
int cu_count() {
    static std::mutex mu;
    static int cus[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
    std::lock_guard<std::mutex> lk(mu);
    if (cus[dev] <= 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev] = n;
    }
    return cus[dev];
}

// the dynamic LDS limit of a kernel, raised once per device to the largest
// size asked; `slot` names the kernel
constexpr int kNetKernels = 9;
static hipError_t allow_lds(const void* kernel, int slot, size_t smem) {
    static std::mutex mu;
    static size_t set_for[kNetKernels][kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (set_for[slot][dev] < smem) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        set_for[slot][dev] = smem;
    }
    return hipSuccess;
}

// Two corrected steps of 8^3 elements took 130 us apart and 114 us beside (96 us
// with what came after); 16^3 elements fill every CU with one fused block (one
// step 112 us).  In between,
// blocks of both kinds would take more than one round of the CUs.
GradNetForm grad_net_form(const NetArgs& na, int E) {
    if (E % kRows == 0 && E / kRows >= cu_count()) return kGradNetFused;
    const int k0 = net256_steps(na);
    const int blocks = (E + kRows - 1) / kRows;
    return (k0 == 6 || k0 == 10) && 2 * blocks <= cu_count() ? kGradNetBeside : kGradNetApart;
}

hipError_t launch_grad_net(int PPv, const SolveDesc& S, const NetArgs& na, const NetTarget& T, hipStream_t st) {
    const GradNetForm form = grad_net_form(na, T.E);
    if (PPv != 4 || form == kGradNetApart || na.dims[0] != na.n_in * 64) return hipErrorInvalidValue;
    const size_t rows = (size_t)2 * kRows * na.ld * sizeof(uint16_t);
    const size_t grad = (size_t)kRowWaves * GradLds<4>::N * sizeof(double);
    const int k0 = net256_steps(na);
    const int nw = k0 == 10 ? (na.act ? 1 : 2) : (k0 == 6 ? (na.act ? 3 : 4) : 0);
    if (form == kGradNetBeside) {
        const size_t smem = rows > grad ? rows : grad;
        const auto kernel = nw == 1   ? k_grad_beside_net<4, 10, 1>
                            : nw == 2 ? k_grad_beside_net<4, 10, 0>
                            : nw == 3 ? k_grad_beside_net<4, 6, 1>
                                      : k_grad_beside_net<4, 6, 0>;
        const hipError_t e = allow_lds((const void*)kernel, 4 + nw, smem);
        if (e != hipSuccess) return e;
        const int blocks = (T.E + kRows - 1) / kRows;
        const int* v = na.in_var;
        hipLaunchKernelGGL(kernel, dim3(2 * blocks), dim3(kRowThreads), smem, st, S.q, S.qtr_in, S.fv, S.N, S.E, v[0], v[1],
                           v[2], v[3], v[4], blocks, S, na, T.out);
        return hipGetLastError();
    }
    const size_t smem = grad + rows;
    const auto kernel = nw == 1   ? k_grad_net<4, 10, 1>
                        : nw == 2 ? k_grad_net<4, 10, 0>
                        : nw == 3 ? k_grad_net<4, 6, 1>
                        : nw == 4 ? k_grad_net<4, 6, 0>
                                  : k_grad_net<4, 0, 0>;
    const hipError_t e = allow_lds((const void*)kernel, nw, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(T.E / kRows), dim3(kRowThreads), smem, st, S.q, S.qtr_in, S.fv, S.N, S.E, S, na, T);
    return hipGetLastError();
}

template <int PP, int UPDATE, int VISC>
static void launch_resid1(const SolveDesc& S, double rkA, double rkB, int first_stage, hipStream_t st) {
    const auto kernel = UPDATE && streams<PP>(S.E) ? k_resid1<PP, UPDATE, VISC, UPDATE ? kBack : kTurn>
                        : in_ranges<PP>(S)         ? k_resid1<PP, UPDATE, VISC, kRange>
                                                   : k_resid1<PP, UPDATE, VISC, kTurn>;
    hipLaunchKernelGGL(kernel, dim3(groups<PP>(S.E)), dim3(Line<PP>::NT), 0, st, S.q, S.qtr_in, S.fv, S.N, S.E,
                       first_stage, S, rkA, rkB);
}

template <int PP, int UPDATE>
static void launch_resid1(const SolveDesc& S, double rkA, double rkB, int first_stage, hipStream_t st) {
    if (S.ph.viscous) launch_resid1<PP, UPDATE, 1>(S, rkA, rkB, first_stage, st);
    else launch_resid1<PP, UPDATE, 0>(S, rkA, rkB, first_stage, st);
}

hipError_t launch_resid(int PPv, int update, const SolveDesc& S, double rkA, double rkB, int first_stage,
                        hipStream_t st) {
    if (update) {
        DG_DISPATCH_PP(PPv, (launch_resid1<PP, 1>(S, rkA, rkB, first_stage, st)));
    } else {
        DG_DISPATCH_PP(PPv, (launch_resid1<PP, 0>(S, rkA, rkB, first_stage, st)));
    }
    return hipGetLastError();
}

hipError_t launch_resid(int PPv, const DescList& dl, double rkA, double rkB, int first_stage, hipStream_t st) {
    DG_DISPATCH_PP(PPv, const DescList g = in_groups<PP>(dl);
                   hipLaunchKernelGGL((streams<PP>(dl.blk[dl.n]) ? k_resid<PP, true> : k_resid<PP, false>),
                                      dim3(g.blk[g.n]), dim3(Line<PP>::NT), 0, st, g, rkA, rkB, first_stage));
    return hipGetLastError();
}

hipError_t launch_tgv(int PPv, const Phys& ph, int N, double* q, hipStream_t st) {
    DG_DISPATCH_PP(PPv, hipLaunchKernelGGL(k_tgv<PP>, dim3(N * N * N), dim3((PP * PP * PP + 63) / 64 * 64), 0, st, ph, N, q));
    return hipGetLastError();
}

hipError_t launch_diag(int PPv, const Phys& ph, int N, const double* q, double* partial, double* out,
                       hipStream_t st) {
    const int E = N * N * N;
    const int blocks = diag_blocks(E, PPv * PPv * PPv);
    DG_DISPATCH_PP(PPv, hipLaunchKernelGGL(k_diag_partial<PP>, dim3(blocks), dim3(256), 0, st, ph, E, q, partial));
    const double J = (ph.h * 0.5) * (ph.h * 0.5) * (ph.h * 0.5);
    hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(256), 0, st, blocks, J / (ph.L * ph.L * ph.L), J, partial, out);
    return hipGetLastError();
}

hipError_t launch_err_inf(int PPv, int E, const double* q, const double* qref, double* partial, double* out,
                          hipStream_t st) {
    const int NP = PPv * PPv * PPv;
    const int blocks = diag_blocks(E, NP);
    hipLaunchKernelGGL(k_err_partial, dim3(blocks), dim3(256), 0, st, (size_t)E * NP, q, qref, partial);
    hipLaunchKernelGGL(k_err_final, dim3(1), dim3(256), 0, st, blocks, partial, out);
    return hipGetLastError();
}

template <int PPS>
static hipError_t launch_project_s(int PPd, int E, const double* src, const ProjectOut& out, hipStream_t st) {
    switch (PPd) {
#define DG_PROJ_CASE(V)                                                                                      \
    case V:                                                                                                  \
        if constexpr (V <= PPS)                                                                              \
            hipLaunchKernelGGL((k_project<PPS, V>), dim3(E), dim3(kProjectThreads<PPS>), 0, st, E, src, out); \
        else                                                                                                 \
            return hipErrorInvalidValue;                                                                     \
        break;
        DG_PROJ_CASE(2) DG_PROJ_CASE(3) DG_PROJ_CASE(4) DG_PROJ_CASE(5) DG_PROJ_CASE(6) DG_PROJ_CASE(7)
        DG_PROJ_CASE(8) DG_PROJ_CASE(9)
#undef DG_PROJ_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_project(int PPs, int PPd, int E, const double* src, const ProjectOut& out, hipStream_t st) {
    DG_DISPATCH_PP(PPs, return launch_project_s<PP>(PPd, E, src, out, st));
    return hipErrorInvalidValue;
}

}  // namespace dgnn
