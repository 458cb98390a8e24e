// Internal declarations shared by the HIP kernels (dg_kernels.hip,
// nn_kernels.hip) and the host side of the library (api.cpp, nn_api.cpp,
// server.cpp).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "../../include/dgnn.h"

namespace dgnn {

constexpr int kMaxPP = DG_MAX_ORDER + 1;   // nodes per direction at the highest order
constexpr int kMaxHalf = (kMaxPP + 1) / 2;   // of them, up to and with the middle one
constexpr int kMaxLayers = 8;               // weight layers of the forcing network
constexpr int kMaxDevices = 64;             // GPUs a process can build meshes on

// Gauss-Legendre nodal basis of one order (Sec. 2.6): nodes and quadrature
// weights, and the operators along a line of nodes.
struct BasisTab {
    double nodes[kMaxPP];
    double w[kMaxPP];
    // With D[i][j] = l_j'(xi_i) and bp[j] = l_j(1): the weak derivative
    // Dhat[i][m] = D[m][i] w[m] / w[i], the weights bpw[i] = bp[i] / w[i] that lift
    // interface values into the line, and the end values' weights bp, split by
    // parity about the middle of the line (the nodes are symmetric): with
    // H = PP / 2 pairs, M = (PP + 1) / 2, mirrored index i' = P - i,
    //   nS[i*H + m] = -(Dhat[i][m] - Dhat[i][m']) / 2,  nT[i*M + m] = -(Dhat[i][m] + Dhat[i][m']) / 2
    // (-Dhat[i][m] at the middle m), lS[i] = (bpw[i] + bpw[i']) / 2, lT[i] = (bpw[i] - bpw[i']) / 2
    // (lS = bpw at the middle i), iE[m] = (bp[m] + bp[m']) / 2 (bp at the middle), iO[m] = (bp[m] - bp[m']) / 2
    double nS[kMaxHalf * (kMaxHalf - 1)];
    double nT[kMaxHalf * (kMaxHalf - 1)];
    double lS[kMaxHalf], lT[kMaxHalf];
    double iE[kMaxHalf], iO[kMaxHalf];
};

// Per-solve physical constants, in the form the kernels use them.
struct Phys {
    double gamma, gm1;      // gamma, gamma - 1
    double p_ref;           // subtracted from the momentum fluxes
    double mu, kappa;       // molecular viscosity and conductivity
    double les_c;           // (Cs * h / (P + 1))^2, 0 without the closure
    double kt;              // gamma / ((gamma - 1) Pr_t): mu_t -> kappa_t
    double s;               // 2 / h: d/dx = s d/dxi
    double h, L;            // element size and box side
    double p0;              // background pressure of the TGV state
    int viscous;            // BR1 gradients and viscous fluxes
    int les;                // Smagorinsky closure
};

// One solve as the batched stage kernels see it (device memory).
struct SolveDesc {
    double* q;              // state [5][E][n_p]
    double* k;              // Runge-Kutta register [5][E][n_p]
    double* out;            // residual output [5][E][n_p] (residual mode)
    const double* forcing;  // s(q) [5][E][n_p] added to the residual, or null
    const double* post;     // update mode: q += dt post after the stage update
                            // (a post-step correction), or null
    const double* qtr_in;   // face traces of q   [E][6][5][n_f], in the frame of the face
    double* qtr_out;        // face traces of the updated q (update mode)
    double* fv;             // one-sided viscous normal fluxes [E][6][4][n_f], likewise
    int N, E;
    double dt;
    Phys ph;
};

// The solves one stage launch works on (by value, in the kernel arguments):
// elements [blk[i], blk[i+1]) are *d[i]'s.
constexpr int kMaxDescs = 32;
struct DescList {
    const SolveDesc* d[kMaxDescs];
    int blk[kMaxDescs + 1];
    int n;
};

// Forcing-network description passed by value to the network kernels.
struct NetArgs {
    int n_layers;
    int act;                         // 0 tanh, 1 relu
    int dims[kMaxLayers + 1];        // true sizes
    int pdims[kMaxLayers + 1];       // sizes rounded up to 32
    const uint16_t* W[kMaxLayers];   // bf16 [pdims[l+1]][pdims[l]], zero padded
    const uint16_t* WT[kMaxLayers];  // bf16 [pdims[l]][pdims[l+1]], zero padded
    const float* b[kMaxLayers];      // float32 [dims[l+1]]
    double mu_in[5], sig_in[5], mu_out[5], sig_out[5], mask[5];
    // per input variable j: mean and 1 / sigma (per-variable normalisation)
    double in_mu[5], in_isig[5];
    // per output variable: s = out_scale[j] yhat + out_shift[j] (mask applied)
    double out_scale[5], out_shift[5];
    // and of the targets: mean and 1 / sigma
    double out_mu[5], out_isig[5];
    // the network reads variables in_var[0..n_in) (input column j n_p + n is
    // node n of variable in_var[j]) and forces out_var[0..n_out) likewise
    int n_in, n_out;
    int in_var[5], out_var[5];
    int ld;                          // row length of activations in LDS: widest layer, padded
    // per-node normalisation (null: per variable): device [4][5 col_np] doubles,
    // mu_in, sigma_in, mu_out, sigma_out of row column v col_np + n
    const double* col;
    int col_np;
};

// One network application target for the batched forcing kernel: the
// elements of one solve, in blocks of rows.
struct NetTarget {
    const double* q;        // [5][E][n_p]
    double* out;            // [5][E][n_p], out += s(q)
    int E;
    int blk_begin;
};

struct Mesh {
    dg_params prm;
    int N, P, PP, E, n_p, n_f;
    Phys ph;
    int device;
};

}  // namespace dgnn

struct dg_mesh {
    dgnn::Mesh m;
};

namespace dgnn {

// workspace layout of one mesh, in bytes from the workspace base
struct WsLayout {
    size_t qtr0, qtr1, fv, forcing, partial, total;
};
WsLayout ws_layout(const Mesh& m);

void fill_phys(const dg_params& p, Phys& ph);

// ----------------------------------------------------------- host launchers
// All return hipSuccess or the launch error.  `descs` is device memory.
// filter matrices G1 [PPd][PPs], at (Ps - 1) * DG_MAX_ORDER + Pd - 1, Pd <= Ps
struct FilterTab {
    double G[kMaxPP * kMaxPP];
};
hipError_t upload_basis_tables(const BasisTab* host_tabs /* index P-1 */, const FilterTab* host_filters);
// address of the no-alloc stepper's scratch on device dev (looked up once, by
// scratch_setup with dev current); null before the set-up
hipError_t scratch_setup(int dev);
void* scratch_device_ptr(int dev);
hipError_t launch_write_descs(const SolveDesc* host, int n, SolveDesc* dev, hipStream_t st);
hipError_t launch_traces(int PP, const SolveDesc& S, hipStream_t st);
// compute units of the current device
int cu_count();
hipError_t launch_grad(int PP, const SolveDesc& S, hipStream_t st);
hipError_t launch_grad(int PP, const DescList& dl, hipStream_t st);
// How the BR1 pass and the forcing network of a P = 3 stage run on E elements:
// in one block per sixteen elements where those fill the GPU (one per CU),
// side by side in one launch where both together leave CUs free, else in two
// launches.
enum GradNetForm { kGradNetApart, kGradNetBeside, kGradNetFused };
GradNetForm grad_net_form(const NetArgs& na, int E);
// k_grad and the forcing network in one launch (P = 3, one solve, the network
// reading all n_p nodes of its variables); hipErrorInvalidValue where the form
// is apart
hipError_t launch_grad_net(int PP, const SolveDesc& S, const NetArgs& na, const NetTarget& T, hipStream_t st);
hipError_t launch_resid(int PP, int update, const SolveDesc& S, double rkA, double rkB, int first_stage,
                        hipStream_t st);
// the stage update of a list of solves, all viscous
hipError_t launch_resid(int PP, const DescList& dl, double rkA, double rkB, int first_stage, hipStream_t st);
hipError_t launch_tgv(int PP, const Phys& ph, int N, double* q, hipStream_t st);
hipError_t launch_diag(int PP, const Phys& ph, int N, const double* q, double* partial,
                       double* out, hipStream_t st);
hipError_t launch_err_inf(int PP, int E, const double* q, const double* qref, double* partial,
                          double* out, hipStream_t st);
// filter G of a field: into dst (and dst2, if given), or, with y given, its
// row of the pair (first, (G field - minus) / div) as float rows x, y
struct ProjectOut {
    double* dst;
    double* dst2;
    const double* first;
    const double* minus;
    double div;
    float* x;
    float* y;
};
hipError_t launch_project(int PPs, int PPd, int E, const double* src, const ProjectOut& out, hipStream_t st);

hipError_t launch_net_forcing(const NetArgs& na, int n_p, const NetTarget* targets, int nt,
                              int nblocks, hipStream_t st);             // out += s(q)
hipError_t launch_net_forcing_write(const NetArgs& na, int n_p, const NetTarget* targets, int nt,
                                    int nblocks, hipStream_t st);       // out = s(q)
hipError_t launch_net_refresh_layer(const NetArgs& na, const float* params, int64_t woff, int l,
                                    uint16_t* wbf, int64_t wbf_off, int64_t wtbf_off, hipStream_t st);
hipError_t launch_fill_f32(float* p, float v, size_t n, hipStream_t st);
int net_rows_per_block();
int net_row_pad();

// training: per-row-block forward / loss / backward data chain, then the
// weight-gradient products reduced over the batch, then Adam
struct TrainArgs {
    const float* x;                   // [rows][5 n_p] (all variables)
    const float* y;                   // [rows][5 n_p]
    const int32_t* idx;               // batch row b is row idx[b] (null: row b)
    int B, Bp;                        // batch, batch rounded up to 32
    float grad_scale;                 // 2 / (B * dims[L])
    uint16_t* actT[kMaxLayers];       // [pdims[l]][Bp]  (act[0] = xhat)
    uint16_t* dzT[kMaxLayers];        // [pdims[l+1]][Bp]
    float* bias_part[kMaxLayers];     // [Bp / 16][pdims[l+1]] row-block sums of dz_l
    float* loss_part;                 // [Bp / 16]
};

// All layers' weight and bias gradients of one training step.
struct GradArgs {
    const uint16_t* dzT[kMaxLayers];
    const uint16_t* actT[kMaxLayers];
    const float* bias_part[kMaxLayers];
    float* gW[kMaxLayers];
    float* gb[kMaxLayers];
    int pout[kMaxLayers], pin[kMaxLayers], dout[kMaxLayers], din[kMaxLayers];
    int tblk[kMaxLayers + 1];         // 32 x 32 tiles before layer l
    int gtiles;                       // blocks for all tiles: their number, a multiple of eight
    int n_layers, Bp, nrb;
};

// Adam on the float32 master weights with the bf16 copies W_l, W_l^T written
// in the same pass.
struct ParamMap {
    int64_t woff[kMaxLayers], boff[kMaxLayers], wbo[kMaxLayers], wtbo[kMaxLayers];
};
// Adam step of the whole parameter vector (and the loss output, when loss is
// not null), for the fused end-of-step launch
struct AdamArgs {
    float* p;
    float* m;
    float* v;
    uint16_t* wbf;
    float lr, b1, b2, eps, bc1, bc2;
    const float* loss_part;
    int n_loss;
    float inv_count;
    float* loss;
};
size_t train_smem_bytes(const NetArgs& na);
hipError_t launch_train_rows(const NetArgs& na, const TrainArgs& ta, int nblocks, hipStream_t st);
// gradients, Adam update and loss, in one launch
hipError_t launch_grad_adam(const GradArgs& ga, const ParamMap& pm, const AdamArgs& aa, hipStream_t st);
hipError_t launch_data_stats(const float* x, const float* y, int64_t rows, int n_p, double* part, int nblocks,
                             double* out_dev, hipStream_t st);
hipError_t launch_column_stats(const float* x, const float* y, int64_t rows, int ncols, double* part, int nblocks,
                               double* out_dev, hipStream_t st);

// error reporting (thread-local)
int set_error(int code, const char* fmt, ...);

// host-side building blocks shared by the C ABI and the solve server
extern const double kRkA[3];
extern const double kRkB[3];
int make_mesh(const dg_params* prm, Mesh& M);
int residual_impl(const Mesh& m, const double* q, double* dqdt, char* ws, hipStream_t st);
int diag_impl(const Mesh& m, const double* q, double* out_dev, char* ws, hipStream_t st);
int project_impl(const Mesh& src, const Mesh& dst, const double* f_src, double* f_dst, hipStream_t st,
                 double* f_dst2 = nullptr);
int init_tgv_impl(const Mesh& m, double* q, hipStream_t st);
double stable_dt_from_diag(const Mesh& m, const double* diag_host, double cfl);

}  // namespace dgnn
