// The stage kernels: a group of threads owns one element (or a few small
// ones), each thread one line of nodes and one or a few nodes.
//
// An element has 3 PP^2 lines of PP nodes.  Line (d, r), r = (a, b), runs
// along axis d through the face nodes r of the two faces normal to d, so one
// thread forms the interface values of a line's two ends from the traces and
// keeps them in registers, and contracts the line in registers with the
// operator's entries as scalar operands.  LDS only transposes fields between
// the nodes and the lines of the three directions: PP reads and PP writes a
// line and component, instead of the PP reads for each node that a
// contraction by one thread per node makes.
//
// Everything that belongs to a line or a face is in the frame of its axis:
// vectors are ordered (d, d + 1, d + 2) mod 3.  The face traces (rho, m_d,
// m_d+1, m_d+2, rho e) and the one-sided viscous fluxes (tau_dd, tau_d+1,d,
// tau_d+2,d, energy) are stored in that order too, and the fields in LDS lie
// so that a line reaches the entry it needs of its own frame at one address
// with a constant offset.  So threads of all three directions run the same
// instructions, in the same wavefront, without selects.
//
// What bounds the stage kernels is the traffic to memory.  16^3 elements,
// against one thread a node and one element a block (mean launch, BR1 pass /
// residual and update): P = 3 17.1 -> 8.3 / 19.8 -> 17.3 us, P = 5 38.6 ->
// 21.5 / 57.8 -> 45.3 us, P = 6 57.6 -> 27 / 112 -> 64 us (102 and 257
// bytes a node, with neighbours' traces and fluxes from the caches: 5.3 / 5.6
// TB/s), P = 8 124 -> 50 / 244 -> 137 us; 32^3 elements at P = 6 455 -> 222 /
// 985 -> 530 us (5.1 / 5.4 TB/s; a large copy reaches 4.95).  The
// kernels before were bound by latency: an element of 343 nodes took six
// wavefronts through ten barriers, each with a few contractions between them,
// and 950 instructions a wavefront where this form takes 3 x 1300 for the
// element.  A whole column of nodes a thread, one
// wavefront an element, was measured too: it needs 450 registers, so one
// wavefront a SIMD, and nothing covers its loads (P = 6 37 / 87 us).
#pragma once

#include "dgnn_internal.hpp"
#include "nn_device.hpp"

namespace dgnn {

template <int PP>
struct Line {
    static constexpr int NP = PP * PP * PP;
    static constexpr int NF = PP * PP;
    static constexpr int H = PP / 2;            // pairs of nodes of a line
    static constexpr int M = (PP + 1) / 2;      // pairs and the middle node
    static constexpr int NL = 3 * NF;           // lines of an element
    // elements of a group: one, or as many as fill a wavefront at P = 1, 2
    static constexpr int EPG = PP == 2 ? 5 : (PP == 3 ? 2 : 1);
    // threads: a line each; where a direction's lines nearly fill a
    // wavefront (P = 6, 7) one wavefront a direction, else packed
    static constexpr bool WD = PP == 7;
    static constexpr int NT = WD ? 192 : 64 * ((EPG * NL + 63) / 64);
    static constexpr bool XOR = PP == 8 || PP == 4;       // permuted LDS order (lds_index)
    static constexpr int NN = (EPG * NP + NT - 1) / NT;   // nodes of a thread
    static constexpr int FS = EPG * NP;         // stride of the fields in LDS
};

using Tab = const __attribute__((address_space(4))) BasisTab*;

template <int PP>
__device__ __forceinline__ Tab basis_tab() {
    return (Tab)&c_basis[PP - 2];
}

// The table's address made opaque at each use for the highest orders: its
// entries do not fit the scalar registers, and kept across phases they are
// spilled to vector lanes, two moves a use, where a scalar load brings eight.
template <int PP>
__device__ __forceinline__ Tab tab_again(Tab p) {
    if constexpr (PP >= 8) asm volatile("" : "+s"(p));
    return p;
}

// Keeps the compiler from moving instructions across: loads issued before it
// stay in flight while the arithmetic behind it runs.
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Has the value formed here: without it the compiler moves a value's whole
// computation to a later branch that alone uses it, and keeps the inputs in
// registers until then.
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }

// barrier of a group; a group of one wavefront waits for itself only (its LDS
// operations complete in order, the fences keep the compiler's order)
template <int PP>
__device__ __forceinline__ void group_sync() {
    if constexpr (Line<PP>::NT == 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// Weak derivative along a line, without the factor 2 / h: lifted interface
// values fm, fp of its ends minus the volume operator.  The nodes are
// symmetric about the middle, so the operator splits into an even and an odd
// half (M H + H M products instead of PP^2).
template <int PP>
__device__ __forceinline__ void line_weak(Tab p, const double (&x)[PP], double fm, double fp,
                                          double (&out)[PP]) {
    constexpr int H = Line<PP>::H, M = Line<PP>::M;
    const Tab B = tab_again<PP>(p);
    double e[M], o[H];
#pragma unroll
    for (int m = 0; m < H; ++m) {
        e[m] = x[m] + x[PP - 1 - m];
        o[m] = x[m] - x[PP - 1 - m];
    }
    if constexpr (M > H) e[H] = x[H];
    const double df = fp - fm, sf = fp + fm;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        double S = B->lS[i] * df;
#pragma unroll
        for (int m = 0; m < H; ++m) S = fma(B->nS[i * H + m], o[m], S);
        if (i < H) {
            double T = B->lT[i] * sf;
#pragma unroll
            for (int m = 0; m < M; ++m) T = fma(B->nT[i * M + m], e[m], T);
            out[i] = S + T;
            out[PP - 1 - i] = S - T;
        } else {
            out[i] = S;
        }
    }
}

// values at the two ends of a line
template <int PP>
__device__ __forceinline__ void line_ends(Tab p, const double (&x)[PP], double& om, double& op) {
    constexpr int H = Line<PP>::H, M = Line<PP>::M;
    const Tab B = tab_again<PP>(p);
    double E = 0.0, O = 0.0;
    if constexpr (M > H) E = B->iE[H] * x[H];
#pragma unroll
    for (int m = 0; m < H; ++m) {
        E = fma(B->iE[m], x[m] + x[PP - 1 - m], E);
        O = fma(B->iO[m], x[m] - x[PP - 1 - m], O);
    }
    om = E - O;
    op = E + O;
}

// velocity, pressure and 1 / rho of a state
struct Prim {
    double v[3], p, ir;
};

__device__ __forceinline__ Prim prim_of(const double q[5], double gm1) {
    Prim w;
    w.ir = recip(q[0]);
    w.v[0] = q[1] * w.ir;
    w.v[1] = q[2] * w.ir;
    w.v[2] = q[3] * w.ir;
    w.p = gm1 * (q[4] - 0.5 * (q[1] * w.v[0] + q[2] * w.v[1] + q[3] * w.v[2]));
    return w;
}

// Roe flux (Roe 1981) along the first axis of the frame the states are given
// in, L on the lower side, from the states and their primitive values
__device__ __forceinline__ void roe_flux(const double qL[5], const Prim& L, const double qR[5], const Prim& R,
                                         const Phys& ph, double F[5]) {
    const double gm1 = ph.gm1;
    const double sL = sqrt_pos(qL[0]), sR = sqrt_pos(qR[0]);
    const double rt = sL * sR;
    const double isum = recip(sL + sR);
    const double aL = sL * isum, aR = sR * isum;
    double vt[3], dv[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        vt[a] = aL * L.v[a] + aR * R.v[a];
        dv[a] = R.v[a] - L.v[a];
    }
    const double hL = qL[4] + L.p, hR = qR[4] + R.p;       // rho H
    const double Ht = aL * (hL * L.ir) + aR * (hR * R.ir);
    const double v2 = vt[0] * vt[0] + vt[1] * vt[1] + vt[2] * vt[2];
    const double c2 = gm1 * (Ht - 0.5 * v2);
    const double ct = sqrt_pos(c2);
    const double ic2 = recip(c2);
    const double vn = vt[0], l0 = fabs(vn);
    const double dr = qR[0] - qL[0], dp = R.p - L.p;
    const double rcd = rt * ct * dv[0];
    // wave strengths times |eigenvalue|
    const double wm = fabs(vn - ct) * (dp - rcd) * (0.5 * ic2);
    const double wp = fabs(vn + ct) * (dp + rcd) * (0.5 * ic2);
    const double we = l0 * (dr - dp * ic2);
    const double ws = wm + we + wp, wd = (wp - wm) * ct;
    double diss[5];
    diss[0] = ws;
    double de = (wm + wp) * Ht + wd * vn + we * (0.5 * v2);
    const double lr = l0 * rt;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (a == 0) {
            diss[1 + a] = ws * vt[a] + wd;
        } else {
            const double sh = lr * dv[a];          // shear wave
            diss[1 + a] = ws * vt[a] + sh;
            de += sh * vt[a];
        }
    }
    diss[4] = de;
    const double vL = L.v[0], vR = R.v[0];
    F[0] = 0.5 * (qL[1] + qR[1] - diss[0]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double s = qL[1 + a] * vL + qR[1 + a] * vR;
        if (a == 0) s += (L.p - ph.p_ref) + (R.p - ph.p_ref);
        F[1 + a] = 0.5 * (s - diss[1 + a]);
    }
    F[4] = 0.5 * (hL * vL + hR * vR - diss[4]);
}

// S:S of the strain rate, gradient g[j][c]
__device__ __forceinline__ double strain_square(const double g[3][4]) {
    double SS = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        SS += g[a][a] * g[a][a];
#pragma unroll
        for (int b = a + 1; b < 3; ++b) {
            const double t = g[a][b] + g[b][a];
            SS += 0.5 * t * t;
        }
    }
    return SS;
}


// LDS index of node (i, j, k) where PP is a power of two: rows and entries
// permuted by the coordinates above them, so that the lines of each direction
// spread over all banks (in node order, lines along x are PP entries apart).
// 16^3 P=7: BR1 pass 47 -> 41 us, residual 127 -> 110, a step of a long call
// 511 -> 440; 8^3 P=3: 29.0 -> 27.9.  Odd PP has no conflicts in node order, and
// PP = 6 a two-way one along x alone.
template <int PP>
__device__ __forceinline__ int lds_index(int i, int j, int k) {
    return (k * PP + (j ^ k)) * PP + (i ^ j);
}

// One thread's place in its group: its line and its nodes.  A thread without a
// line, or without its last node, takes another's, and does everything but
// the stores: loads under a branch would make the compiler wait for all of
// them wherever the branches meet.
template <int PP>
struct Place {
    int e0, n_el;       // first element of the group, elements in it
    int t;
    bool line;          // whether the thread has a line
    int e, d, r;        // element, axis and face node of the line
    int nbm, nbp;       // neighbours at its lower and upper end
    int at[PP];         // LDS index of its nodes, field 0
};

template <int PP>
__device__ __forceinline__ Place<PP> place_of(int group, int t, int N, int E) {
    using L = Line<PP>;
    Place<PP> p;
    p.t = t;
    p.e0 = group * L::EPG;
    p.n_el = E - p.e0 < L::EPG ? E - p.e0 : L::EPG;
    int el = 0, q = t;
    if constexpr (L::EPG > 1) {
        el = t / L::NL;
        q = t - el * L::NL;
        p.line = el < p.n_el;
        el = p.line ? el : 0;
    }
    if constexpr (L::WD) {
        p.d = __builtin_amdgcn_readfirstlane(t >> 6);
        p.r = t & 63;
        p.line = p.r < L::NF;
        p.r = p.line ? p.r : 0;
    } else {
        if constexpr (L::EPG == 1) p.line = q < L::NL;
        q = p.line ? q : 0;
        p.d = q / L::NF;
        p.r = q - p.d * L::NF;
    }
    p.e = p.e0 + el;
    const int ez = p.e / (N * N), rem = p.e - ez * N * N, ey = rem / N, ex = rem - ey * N;
    const int c = p.d == 0 ? ex : (p.d == 1 ? ey : ez);
    const int st = p.d == 0 ? 1 : (p.d == 1 ? N : N * N);
    p.nbp = p.e + (c + 1 == N ? 1 - N : 1) * st;
    p.nbm = p.e + (c == 0 ? N - 1 : -1) * st;
    const int a = p.r % PP, b = p.r / PP;
    if constexpr (L::XOR) {
#pragma unroll
        for (int m = 0; m < PP; ++m) {
            const int i = p.d == 0 ? m : a, j = p.d == 0 ? a : (p.d == 1 ? m : b), k = p.d == 2 ? m : b;
            p.at[m] = lds_index<PP>(i, j, k);
        }
    } else {
        const int base = p.d == 0 ? PP * p.r : (p.d == 1 ? a + L::NF * b : p.r);
        const int ns = p.d == 0 ? 1 : (p.d == 1 ? PP : L::NF);
#pragma unroll
        for (int m = 0; m < PP; ++m) p.at[m] = el * L::NP + base + m * ns;
    }
    return p;
}

// index of the thread's i-th node in the group, and whether it exists
template <int PP>
__device__ __forceinline__ bool node_of(const Place<PP>& p, int i, int& n) {
    using L = Line<PP>;
    const int last = (L::EPG > 1 ? p.n_el * L::NP : L::NP) - 1;
    n = p.t + i * L::NT;
    if ((i + 1) * L::NT <= L::NP && L::EPG == 1) return true;
    const bool in = n <= last;
    n = in ? n : last;
    return in;
}

// LDS index of node n of the group
template <int PP>
__device__ __forceinline__ int node_lds(int n) {
    if constexpr (Line<PP>::XOR) return lds_index<PP>(n % PP, (n / PP) % PP, n / (PP * PP));
    else return n;
}

// the traces that the two ends of a line need: own and neighbour's
struct EndStates {
    double qi[2][5], qo[2][5];
};

template <int PP>
__device__ __forceinline__ void load_ends(const Place<PP>& p, const double* tr, EndStates& f) {
    constexpr int NF = Line<PP>::NF;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const gdouble* ti = gmem(tr) + (size_t)(p.e * 6 + 2 * p.d + s) * 5 * NF + p.r;
        const gdouble* to = gmem(tr) + (size_t)((s ? p.nbp : p.nbm) * 6 + 2 * p.d + (s ^ 1)) * 5 * NF + p.r;
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            f.qi[s][v] = ti[v * NF];
            f.qo[s][v] = to[v * NF];
        }
    }
}

// state of the thread's nodes: load, and w = (u, v, w, T) into the fields
// 0 .. 7 of LDS as u, v, w, u, v, T, T, T (a line of axis d finds the velocity
// of its frame at fields d .. d + 2, T at d + 5)
template <int PP, bool STREAM = false>
__device__ __forceinline__ void load_nodes(const Place<PP>& p, const double* f, size_t vs, double (&q)[Line<PP>::NN][5]) {
    using L = Line<PP>;
#pragma unroll
    for (int i = 0; i < L::NN; ++i) {
        int n;
        node_of<PP>(p, i, n);
        const gdouble* g = gmem(f) + ((size_t)p.e0 * L::NP + n);
#pragma unroll
        for (int v = 0; v < 5; ++v) q[i][v] = STREAM ? __builtin_nontemporal_load(g + v * vs) : g[v * vs];
    }
}

template <int PP>
__device__ __forceinline__ void nodes_to_w(const Place<PP>& p, const double (&q)[Line<PP>::NN][5], double gm1,
                                           double* sh) {
    using L = Line<PP>;
    constexpr int FS = L::FS;
#pragma unroll
    for (int i = 0; i < L::NN; ++i) {
        const Prim a = prim_of(q[i], gm1);
        const double T = a.p * a.ir;
        int n;
        if (node_of<PP>(p, i, n)) {
            n = node_lds<PP>(n);
            sh[n] = a.v[0];
            sh[FS + n] = a.v[1];
            sh[2 * FS + n] = a.v[2];
            sh[3 * FS + n] = a.v[0];
            sh[4 * FS + n] = a.v[1];
            sh[5 * FS + n] = T;
            sh[6 * FS + n] = T;
            sh[7 * FS + n] = T;
        }
    }
}

// the thread's line of the field at f
template <int PP>
__device__ __forceinline__ void read_line(const Place<PP>& p, const double* f, double (&x)[PP]) {
#pragma unroll
    for (int m = 0; m < PP; ++m) x[m] = f[p.at[m]];
}

template <int PP>
__device__ __forceinline__ void write_line(const Place<PP>& p, double* f, const double (&x)[PP]) {
#pragma unroll
    for (int m = 0; m < PP; ++m) f[p.at[m]] = x[m];
}

// The derivative of w along the line, in the frame of its axis: from the
// fields that nodes_to_w wrote.
template <int PP>
__device__ __forceinline__ void line_gradient(const Place<PP>& p, Tab B, const double* sh, const double (&wh)[2][4],
                                              double (&o)[4][PP]) {
    constexpr int FS = Line<PP>::FS;
    const double* f = sh + p.d * FS;
    double x[4][PP];
#pragma unroll
    for (int c = 0; c < 4; ++c) read_line<PP>(p, f + (c < 3 ? c : 5) * FS, x[c]);
#pragma unroll
    for (int c = 0; c < 4; ++c) line_weak<PP>(B, x[c], wh[0][c], wh[1][c], o[c]);
}

// New traces of the state of the thread's nodes: through LDS (rho, rho e at
// fields f0, f0 + 1, the momenta m0, m1, m2, m0, m1 behind them) to the lines.
template <int PP>
__device__ __forceinline__ void nodes_to_traces(const Place<PP>& p, Tab B, const double (&q)[Line<PP>::NN][5], double* sh,
                                                gdouble* out) {
    using L = Line<PP>;
    constexpr int FS = L::FS, NF = L::NF;
#pragma unroll
    for (int i = 0; i < L::NN; ++i) {
        int n;
        if (node_of<PP>(p, i, n)) {
            n = node_lds<PP>(n);
            sh[n] = q[i][0];
            sh[FS + n] = q[i][4];
            sh[2 * FS + n] = q[i][1];
            sh[3 * FS + n] = q[i][2];
            sh[4 * FS + n] = q[i][3];
            sh[5 * FS + n] = q[i][1];
            sh[6 * FS + n] = q[i][2];
        }
    }
    group_sync<PP>();
    if (p.line) {
        gdouble* o = out + (size_t)(p.e * 6 + 2 * p.d) * 5 * NF + p.r;
        double x[5][PP];
        read_line<PP>(p, sh, x[0]);
        read_line<PP>(p, sh + FS, x[4]);
#pragma unroll
        for (int a = 0; a < 3; ++a) read_line<PP>(p, sh + (p.d + 2 + a) * FS, x[1 + a]);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            double lo, hi;
            line_ends<PP>(B, x[v], lo, hi);
            o[v * NF] = lo;
            o[(5 + v) * NF] = hi;
        }
    }
}

// Wavefronts per SIMD that a stage kernel is compiled for: as many as its LDS
// area lets share a CU (160 KB), at most three (four at P = 3, in 128
// registers: spills, a 16^3 step 79 -> 90 us).
template <class Lds, int NT>
constexpr int line_waves() {
    constexpr int groups = (160 * 1024) / (Lds::N * 8);
    constexpr int waves = groups * (NT / 64) / 4;
    return waves < 1 ? 1 : (waves > 3 ? 3 : waves);
}

// --------------------------------------------------------------- BR1 pass

template <int PP>
struct GradLds {
    static constexpr int N = 9 * Line<PP>::FS;
};

// One-sided viscous flux normal to a face, in the frame of the face: from
// rho, v and the gradient g[j][c] = d_j w_c / s (g[1][3] and g[2][3] not used;
// g[1][2] and g[2][1] by the closure only)
__device__ __forceinline__ void viscous_normal(double rho, const double v[3], const double g[3][4], const Phys& ph,
                                               double Fv[4]) {
    double mu = ph.mu, kappa = ph.kappa;
    if (ph.les) {
        const double mut = rho * ph.les_c * ph.s * sqrt(2.0 * strain_square(g));
        mu += mut;
        kappa += mut * ph.kt;
    }
    mu *= ph.s;
    kappa *= ph.s;
    const double div = g[0][0] + g[1][1] + g[2][2];
    Fv[0] = mu * (g[0][0] + g[0][0]) - (2.0 / 3.0) * mu * div;
    Fv[1] = mu * (g[0][1] + g[1][0]);
    Fv[2] = mu * (g[0][2] + g[2][0]);
    Fv[3] = kappa * g[0][3] + v[0] * Fv[0] + v[1] * Fv[1] + v[2] * Fv[2];
}

// BR1 pass of a group's elements: the one-sided viscous normal fluxes on
// their faces.  The nodes' state is left in q.
template <int PP>
__device__ __forceinline__ void grad_group(const SolveDesc& S, int group, int t, double* sh,
                                           double (&q)[Line<PP>::NN][5]) {
    using L = Line<PP>;
    constexpr int FS = L::FS, NF = L::NF;
    const Phys ph = S.ph;
    const Tab B = basis_tab<PP>();
    const Place<PP> p = place_of<PP>(group, t, S.N, S.E);
    const size_t vs = (size_t)S.E * L::NP;
    load_nodes<PP>(p, S.q, vs, q);
    EndStates f;
    load_ends<PP>(p, S.qtr_in, f);
    sched_fence();
    nodes_to_w<PP>(p, q, ph.gm1, sh);
    double own[2][4], wh[2][4];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const Prim a = prim_of(f.qi[s], ph.gm1), b = prim_of(f.qo[s], ph.gm1);
        own[s][0] = f.qi[s][0];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            own[s][1 + c] = a.v[c];
            wh[s][c] = 0.5 * (a.v[c] + b.v[c]);
        }
        wh[s][3] = 0.5 * (a.p * a.ir + b.p * b.ir);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            pin(own[s][c]);
            pin(wh[s][c]);
        }
    }
    group_sync<PP>();
    double g[2][3][4], o[4][PP];
    if (p.line) {
        line_gradient<PP>(p, B, sh, wh, o);
#pragma unroll
        for (int c = 0; c < 4; ++c) line_ends<PP>(B, o[c], g[0][0][c], g[1][0][c]);
    }
    group_sync<PP>();
    if (p.line) {
        // the velocity's derivatives along axis d to fields 3 d .. 3 d + 2
        double* f0 = sh + 3 * p.d * FS;
#pragma unroll
        for (int c = 0; c < 3; ++c) write_line<PP>(p, f0 + c * FS, o[c]);
    }
    group_sync<PP>();
    if (!p.line) return;
    // entry (j, c) of the frame is component c - j of axis d + j's frame
    const int d1 = p.d == 2 ? 0 : p.d + 1, d2 = p.d == 0 ? 2 : p.d - 1;
    const double* f1 = sh + 3 * d1 * FS;
    const double* f2 = sh + 3 * d2 * FS;
    double x[4][PP];
    read_line<PP>(p, f1 + 2 * FS, x[0]);
    read_line<PP>(p, f1, x[1]);
    read_line<PP>(p, f2 + FS, x[2]);
    read_line<PP>(p, f2, x[3]);
    line_ends<PP>(B, x[0], g[0][1][0], g[1][1][0]);
    line_ends<PP>(B, x[1], g[0][1][1], g[1][1][1]);
    line_ends<PP>(B, x[2], g[0][2][0], g[1][2][0]);
    line_ends<PP>(B, x[3], g[0][2][2], g[1][2][2]);
    if (ph.les) {
        read_line<PP>(p, f1 + FS, x[0]);
        read_line<PP>(p, f2 + 2 * FS, x[1]);
        line_ends<PP>(B, x[0], g[0][1][2], g[1][1][2]);
        line_ends<PP>(B, x[1], g[0][2][1], g[1][2][1]);
    }
    double Fv[2][4];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const double v[3] = {own[s][1], own[s][2], own[s][3]};
        viscous_normal(own[s][0], v, g[s], ph, Fv[s]);
    }
    gdouble* out = gmem(S.fv) + (size_t)(p.e * 6 + 2 * p.d) * 4 * NF + p.r;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) out[(4 * s + c) * NF] = Fv[s][c];
}

// ------------------------------------------- residual and stage update

template <int PP>
struct ResidLds {
    static constexpr int N = 13 * Line<PP>::FS;
};

// Net volume fluxes (inviscid minus viscous) of one node from its state
// and the gradient g[j][c] = d_j w_c / s: the momentum flux is symmetric, so twelve entries serve the three directions.
struct NodeFlux {
    double m[3], e[3], t[3], t01, t12, t20;
};

template <int VISC>
__device__ __forceinline__ NodeFlux node_flux(const double q[5], const double g[3][4], const Phys& ph) {
    NodeFlux G;
    const Prim a = prim_of(q, ph.gm1);
    const double* w = a.v;
    const double pt = a.p - ph.p_ref, pe = q[4] + a.p;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        G.m[d] = q[1 + d];
        G.t[d] = q[1 + d] * w[d] + pt;
        G.e[d] = pe * w[d];
    }
    G.t01 = q[1] * w[1];
    G.t12 = q[2] * w[2];
    G.t20 = q[3] * w[0];
    if constexpr (VISC) {
        double mu = ph.mu, kappa = ph.kappa;
        if (ph.les) {
            const double mut = q[0] * ph.les_c * ph.s * sqrt(2.0 * strain_square(g));
            mu += mut;
            kappa += mut * ph.kt;
        }
        mu *= ph.s;
        kappa *= ph.s;
        const double lam = (2.0 / 3.0) * mu * (g[0][0] + g[1][1] + g[2][2]);
        const double t0 = mu * (g[0][0] + g[0][0]) - lam, t1 = mu * (g[1][1] + g[1][1]) - lam,
                     t2 = mu * (g[2][2] + g[2][2]) - lam;
        const double t01 = mu * (g[0][1] + g[1][0]), t12 = mu * (g[1][2] + g[2][1]), t20 = mu * (g[0][2] + g[2][0]);
        G.t[0] -= t0;
        G.t[1] -= t1;
        G.t[2] -= t2;
        G.t01 -= t01;
        G.t12 -= t12;
        G.t20 -= t20;
        G.e[0] -= w[0] * t0 + w[1] * t01 + w[2] * t20 + kappa * g[0][3];
        G.e[1] -= w[0] * t01 + w[1] * t1 + w[2] * t12 + kappa * g[1][3];
        G.e[2] -= w[0] * t20 + w[1] * t12 + w[2] * t2 + kappa * g[2][3];
    }
    return G;
}

// Residual (out = p(q) + forcing), or Runge-Kutta stage (UPDATE: k <- A k +
// dt R, q <- q + B k, the traces of the new q), of a group's elements.
// STREAM: the register, which nothing else of a step reads, passes by the
// caches.
template <int PP, int UPDATE, int VISC, bool STREAM = false>
__device__ __forceinline__ void resid_group(const SolveDesc& S, int group, int t, double* sh, double rkA, double rkB,
                                            int first_stage) {
    using L = Line<PP>;
    constexpr int FS = L::FS, NF = L::NF, NN = L::NN;
    const Phys ph = S.ph;
    const Tab B = basis_tab<PP>();
    const Place<PP> p = place_of<PP>(group, t, S.N, S.E);
    const size_t vs = (size_t)S.E * L::NP;
    const double dt = S.dt;
    const double* const fo = S.forcing;
    const double* const po = S.post;
    gdouble* const qtr_out = gmem(S.qtr_out);

    double q[NN][5], k[NN][5];
    load_nodes<PP>(p, S.q, vs, q);
    EndStates f;
    double fi[2][4], fn[2][4];
    load_ends<PP>(p, S.qtr_in, f);
    if constexpr (VISC) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const gdouble* a = gmem(S.fv) + (size_t)(p.e * 6 + 2 * p.d + s) * 4 * NF + p.r;
            const gdouble* b = gmem(S.fv) + (size_t)((s ? p.nbp : p.nbm) * 6 + 2 * p.d + (s ^ 1)) * 4 * NF + p.r;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                fi[s][c] = a[c * NF];
                fn[s][c] = b[c * NF];
            }
        }
    }
    sched_fence();
    if constexpr (VISC) nodes_to_w<PP>(p, q, ph.gm1, sh);
    double F[2][5], wh[2][4];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const Prim a = prim_of(f.qi[s], ph.gm1), b = prim_of(f.qo[s], ph.gm1);
        if (s) roe_flux(f.qi[s], a, f.qo[s], b, ph, F[s]);
        else roe_flux(f.qo[s], b, f.qi[s], a, ph, F[s]);
        if constexpr (VISC) {
#pragma unroll
            for (int c = 0; c < 3; ++c) wh[s][c] = 0.5 * (a.v[c] + b.v[c]);
            wh[s][3] = 0.5 * (a.p * a.ir + b.p * b.ir);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                F[s][1 + c] -= 0.5 * (fi[s][c] + fn[s][c]);
                pin(wh[s][c]);
            }
        }
#pragma unroll
        for (int v = 0; v < 5; ++v) pin(F[s][v]);
    }
    if constexpr (VISC) {
        group_sync<PP>();
        double o[4][PP];
        if (p.line) line_gradient<PP>(p, B, sh, wh, o);
        group_sync<PP>();
        if (p.line) {
            // to fields 4 d .. 4 d + 3
            double* f0 = sh + 4 * p.d * FS;
#pragma unroll
            for (int c = 0; c < 4; ++c) write_line<PP>(p, f0 + c * FS, o[c]);
        }
        group_sync<PP>();
    }
    // node fluxes, in place: mass 0 - 2, energy 3 - 5, momentum: diagonal
    // 6 - 8, then t20, t01, t12, t20
#pragma unroll
    for (int i = 0; i < NN; ++i) {
        int n;
        const bool in = node_of<PP>(p, i, n);
        n = node_lds<PP>(n);
        // the primitive values are formed again: kept from above they would
        // not fit the registers beside the faces' data
        pin(q[i][0]);
        double g[3][4];
        if constexpr (VISC) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
#pragma unroll
                for (int c = 0; c < 3; ++c) g[j][c] = sh[(4 * j + (c - j + 3) % 3) * FS + n];
                g[j][3] = sh[(4 * j + 3) * FS + n];
            }
        }
        const NodeFlux G = node_flux<VISC>(q[i], g, ph);
        if (in) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                sh[d * FS + n] = G.m[d];
                sh[(3 + d) * FS + n] = G.e[d];
                sh[(6 + d) * FS + n] = G.t[d];
            }
            sh[9 * FS + n] = G.t20;
            sh[10 * FS + n] = G.t01;
            sh[11 * FS + n] = G.t12;
            sh[12 * FS + n] = G.t20;
        }
    }
    // the Runge-Kutta register, in flight until the update
    if (UPDATE && !first_stage) load_nodes<PP, STREAM>(p, S.k, vs, k);
    sched_fence();
    group_sync<PP>();
    double o[5][PP];
    if (p.line) {
        const double* f0 = sh + p.d * FS;
        double x[3][PP];
        read_line<PP>(p, f0, x[0]);
        read_line<PP>(p, f0 + 6 * FS, x[1]);
        read_line<PP>(p, f0 + 10 * FS, x[2]);
#pragma unroll
        for (int v = 0; v < 3; ++v) line_weak<PP>(B, x[v], F[0][v], F[1][v], o[v]);
        sched_fence();   // two batches: all five lines at once do not fit the registers
        read_line<PP>(p, f0 + 9 * FS, x[0]);
        read_line<PP>(p, f0 + 3 * FS, x[1]);
#pragma unroll
        for (int v = 3; v < 5; ++v) line_weak<PP>(B, x[v - 3], F[0][v], F[1][v], o[v]);
    }
    group_sync<PP>();
    // back to the nodes: mass and momentum of axis d at fields 4 d .. 4 d + 3,
    // then the energy at field d
    if (p.line) {
        double* f0 = sh + 4 * p.d * FS;
#pragma unroll
        for (int v = 0; v < 4; ++v) write_line<PP>(p, f0 + v * FS, o[v]);
    }
    group_sync<PP>();
    double R[NN][5];
#pragma unroll
    for (int i = 0; i < NN; ++i) {
        int n;
        node_of<PP>(p, i, n);
        n = node_lds<PP>(n);
        R[i][0] = sh[n] + sh[4 * FS + n] + sh[8 * FS + n];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            R[i][1 + a] = sh[(1 + a) * FS + n] + sh[(5 + (a + 2) % 3) * FS + n] + sh[(9 + (a + 1) % 3) * FS + n];
    }
    group_sync<PP>();
    if (p.line) write_line<PP>(p, sh + p.d * FS, o[4]);
    group_sync<PP>();
#pragma unroll
    for (int i = 0; i < NN; ++i) {
        int n;
        node_of<PP>(p, i, n);
        n = node_lds<PP>(n);
        R[i][4] = sh[n] + sh[FS + n] + sh[2 * FS + n];
#pragma unroll
        for (int v = 0; v < 5; ++v) R[i][v] *= -ph.s;
    }
    if (fo) {
        double x[NN][5];
        load_nodes<PP>(p, fo, vs, x);
#pragma unroll
        for (int i = 0; i < NN; ++i)
#pragma unroll
            for (int v = 0; v < 5; ++v) R[i][v] += x[i][v];
    }
    if constexpr (!UPDATE) {
#pragma unroll
        for (int i = 0; i < NN; ++i) {
            int n;
            if (node_of<PP>(p, i, n)) {
                gdouble* out = gmem(S.out) + ((size_t)p.e0 * L::NP + n);
#pragma unroll
                for (int v = 0; v < 5; ++v) out[v * vs] = R[i][v];
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < NN; ++i)
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                k[i][v] = first_stage ? dt * R[i][v] : rkA * k[i][v] + dt * R[i][v];
                q[i][v] += rkB * k[i][v];
            }
        if (po) {
            double x[NN][5];
            load_nodes<PP>(p, po, vs, x);
#pragma unroll
            for (int i = 0; i < NN; ++i)
#pragma unroll
                for (int v = 0; v < 5; ++v) q[i][v] += dt * x[i][v];
        }
        gdouble* const qg = gmem(S.q);
        gdouble* const kg = gmem(S.k);
#pragma unroll
        for (int i = 0; i < NN; ++i) {
            int n;
            if (node_of<PP>(p, i, n)) {
                const size_t at = (size_t)p.e0 * L::NP + n;
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    if constexpr (STREAM) __builtin_nontemporal_store(k[i][v], kg + at + v * vs);
                    else kg[at + v * vs] = k[i][v];
                    qg[at + v * vs] = q[i][v];
                }
            }
        }
        // above the fields that other threads may still read (0 - 2)
        nodes_to_traces<PP>(p, B, q, sh + 3 * FS, qtr_out);
    }
}

// face traces of the state of a group's elements
template <int PP>
__device__ __forceinline__ void traces_group(const SolveDesc& S, int group, int t, double* sh) {
    using L = Line<PP>;
    const Place<PP> p = place_of<PP>(group, t, S.N, S.E);
    double q[L::NN][5];
    load_nodes<PP>(p, S.q, (size_t)S.E * L::NP, q);
    nodes_to_traces<PP>(p, basis_tab<PP>(), q, sh, gmem(S.qtr_out));
}

}  // namespace dgnn
