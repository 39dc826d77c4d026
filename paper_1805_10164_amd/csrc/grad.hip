// Gradient of the DIRECT current I = sum_k w_k T_k with respect to the onsite potentials V_i
// and the dephasing rates gamma_i (Sigma_s,ii = -(i/2) gamma_i, Sec. III A, Eq. (77)).
//
// With injection from lead p and collection at q (f_p = 1, f_q = 0), Sec. III C, Eq. (79)
// read as the diagonal of Eq. (8):
//   T = T_qp + c^T M^{-1} b,  M = diag(gamma_j A_jj) - T_PP,  b_j = gamma_j w_p(j),
//   c_j = gamma_j w_q(j),  T_PP,ij = gamma_i gamma_j |G_ij|^2,  A_jj = -2 Im G_jj,
//   w_r(j) = (G Gamma_r G^+)_jj,  T_qp = Tr Gamma_q G_qp Gamma_p G_qp^+.
// Adjoint: x = M^{-1} b, lambda = M^{-1} c (M is symmetric), u = gamma lambda, v = gamma x.
// At fixed gamma, dT = Re sum_ab Psi_ab dG_ab with
//   Psi_ab   = 2 u_a v_b conj(G_ab)                              (|G_ab|^2 in M)
//   Psi_jj  += -2i u_j x_j                                       (A_jj in M)
//   Psi_ja  += 2 u_j sum_c Gamma_p,ac conj(G_jc),  a, c in slice p   (w_p in b)
//   Psi_ja  += 2 v_j sum_c Gamma_q,ac conj(G_jc),  a, c in slice q   (w_q in c)
//   Psi_ab  += 2 (Gamma_p G_qp^+ Gamma_q)_ba,  a in slice q, b in slice p   (T_qp)
// and dG = G dV G (dA = -dV), so dT/dV_i = Re K_i with K = diag(G Psi G); a change of
// gamma_i changes A by (i/2) e_i e_i^T, giving Im K_i / 2, plus the explicit terms
//   lambda_i w_p(i) + x_i w_q(i) - lambda_i A_ii x_i + lambda_i (P v)_i + x_i (P u)_i.
// G is complex symmetric (G_ij = G_ji), so with Q = conj(G) diag(v) G and R = conj(G) diag(u) G
//   dense part of K_i = 2 sum_a G_ia u_a Q_ai,
//   lead parts:  sum_j G_ij u_j conj(G_{j,sp+b}) = conj(R_{i,sp+b}),
//                sum_j G_ij v_j conj(G_{j,sq+b}) = conj(Q_{i,sq+b}).
// A column of Q or R is conj(A)^{-1} applied to d o G_{:,c} (A = E - H - Sigma, block
// tridiagonal with off-diagonal blocks t I), by the block LDL^T of A that the stored
// left-connected blocks gL_k provide (A is complex symmetric: D_k = gL_k^{-1}):
//   forward   w_k = h_k - t y_{k-1},  y_k = conj(gL_k) w_k,
//   backward  q_k = y_k - t conj(gL_k) q_{k+1}.
// The dense part is a quadratic form of column c alone, with h^u = u o G_{:,c}, h^v = v o G_{:,c}
//   sum_a G_ac u_a Q_ac = (h^u)^T conj(A)^{-1} h^v = sum_k (w^u_k)^T y^v_k,
// so two forward eliminations in one pass over G give it, O(N W) per column and nothing stored;
// only the 2 W lead columns take the backward sweep.  (A full solve per column read G twice and
// wrote and read its forward result: four times the traffic.)
#include "common.h"

namespace mcnegf {

__device__ inline int perm16(int j) { return (j & ~15) + 4 * (j & 3) + ((j >> 2) & 3); }

__device__ inline double readlane_dbl(double v, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// L^T xt = y and L^T lt = z with L the Cholesky factor of the bordered scaled probe system
// (lower part, columns of each 16-block stored permuted, logical row and column i being site
// perm16(i)) and y, z its bordered rows Np and Np + 1; then x = s xt and lambda = s lt
// (s_j = M_jj^{-1/2}, vector slot 3).  One workgroup of 1024 threads per energy, right-looking over
// block rows of 64 from the last one down:
//   solve  L_II^T x_I = r_I       (diagonal block staged in LDS, one wavefront, lane per row)
//   update r_j -= sum_{i in I} L_ij x_i   for every j < 64 I
// Thread tid owns the stored positions p = tid + 1024 q of r (in registers), so the update
// reads the rows of block I coalesced with 64 independent loads per position.
constexpr int BSV_THREADS = 1024;

// BSV_Q: positions per thread (Np <= BSV_THREADS * BSV_Q)
template <int BSV_Q>
__global__ void __launch_bounds__(BSV_THREADS) backsolve_kernel(const double* __restrict__ Lall,
                                                                const double* __restrict__ vec,
                                                                int N, int Np, int64_t ld,
                                                                double* __restrict__ xl) {
    __shared__ double dg[64][65];
    __shared__ double rI[2][64];
    __shared__ double xI[2][64];
    const int e = blockIdx.x;
    const int tid = threadIdx.x;
    const double* Le = Lall + (size_t)e * (Np + 2) * ld;
    const double* s = vec + (size_t)e * 4 * N + 3 * N;
    double* xo = xl + (size_t)e * 2 * ld;
    double rx[BSV_Q], rl[BSV_Q];
#pragma unroll
    for (int q = 0; q < BSV_Q; ++q) {
        const int p = tid + BSV_THREADS * q;
        rx[q] = p < Np ? Le[(size_t)Np * ld + p] : 0.0;
        rl[q] = p < Np ? Le[(size_t)(Np + 1) * ld + p] : 0.0;
    }
    const int nJ = (Np + 63) / 64;
    for (int I = nJ - 1; I >= 0; --I) {
        const int c0 = 64 * I;
        const int wI = min(64, Np - c0);  // a multiple of 16
        for (int t = tid; t < 64 * 64; t += BSV_THREADS) {
            const int i = t >> 6, pp = t & 63;
            dg[i][pp] = (i < wI && pp < wI) ? Le[(size_t)(c0 + i) * ld + c0 + pp] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < BSV_Q; ++q) {
            const int p = tid + BSV_THREADS * q;
            if (p >= c0 && p < c0 + wI) {  // logical column perm16(p), row perm16(p) - c0
                const int m = perm16(p) - c0;
                rI[0][m] = rx[q];
                rI[1][m] = rl[q];
            }
        }
        __syncthreads();
        if (tid < 64) {
            const int m = tid;         // logical column c0 + m of the block
            const int pm = perm16(m);  // its stored position
            double ax = m < wI ? rI[0][m] : 0.0, al = m < wI ? rI[1][m] : 0.0;
            // lane m holds 1 / L_mm, so the sequential loop below only multiplies
            const double inv = m < wI ? 1.0 / dg[m][pm] : 0.0;
            for (int k = wI - 1; k >= 0; --k) {  // uniform loop, whole wavefront active
                const double ik = readlane_dbl(inv, k);
                const double xk = readlane_dbl(ax, k) * ik;
                const double lk = readlane_dbl(al, k) * ik;
                const double lkm = (m < k) ? dg[k][pm] : 0.0;
                ax = (m == k) ? xk : fma(-lkm, xk, ax);
                al = (m == k) ? lk : fma(-lkm, lk, al);
            }
            if (m < wI) {
                xI[0][m] = ax;
                xI[1][m] = al;
                const int site = c0 + pm;  // the factor takes the sites in stored order
                if (site < N) {
                    xo[site] = s[site] * ax;
                    xo[ld + site] = s[site] * al;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < BSV_Q; ++q) {
            const int p = tid + BSV_THREADS * q;
            if (p < c0) {
                double ax = 0.0, al = 0.0;
                for (int i0 = 0; i0 < wI; i0 += 16) {  // 16 independent loads, then use
                    double lip[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) lip[i] = Le[(size_t)(c0 + i0 + i) * ld + p];
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        ax = fma(lip[i], xI[0][i0 + i], ax);
                        al = fma(lip[i], xI[1][i0 + i], al);
                    }
                }
                rx[q] -= ax;
                rl[q] -= al;
            }
        }
        __syncthreads();  // dg, rI and xI are rewritten for the next block
    }
}

typedef __attribute__((address_space(3))) double lds_double;

// out = conj(M) in for a W x W complex block M (row-major, (re, im) pairs in LDS; the same
// address on every lane, so each read is a broadcast).
template <int W>
__device__ inline void conj_block_matvec(double2 (&out)[W], const double2 (&in)[W],
                                         const lds_double* M) {
#pragma unroll
    for (int y = 0; y < W; ++y) {
        double2 acc = cmk(0.0, 0.0);
#pragma unroll
        for (int x = 0; x < W; ++x)
            cfma(acc, cmk(M[2 * (y * W + x)], -M[2 * (y * W + x) + 1]), in[x]);
        out[y] = acc;
    }
}

// The W x W block src into the LDS buffer dst by NT threads.
template <int W, int NT>
__device__ inline void stage_block(lds_double* dst, const double2* __restrict__ src, int tid) {
#pragma unroll
    for (int i = tid; i < W * W; i += NT) {
        const double2 v = src[i];
        dst[2 * i] = v.x;
        dst[2 * i + 1] = v.y;
    }
}

struct AdjointArgs {
    const double2* gL;     // [nE][L][W][W]
    const double2* G;      // [nE][N][ld]
    const double* xl;      // [nE][2][ld] x, lambda
    const double* gamma;   // [N]
    double2* Y;            // [nE][N][ldY]: columns sq .. of Q and N .. of R
    double2* part_k;       // [nE][2][N]
    double* part_p;        // [nE][2][N]
    int L;
    double t;
    int64_t ld, ldY;
    uint32_t inject_lead;
};

// The lead columns of one energy, on one wavefront: right-hand side c < W is
// column sq + c of Q (d = v), c = W + b is column sp + b of R (d = u), one lane each; y goes to Y
// and q replaces it.  A chain of 2 L slices: it shares its launch with the dense columns.
template <int W>
__device__ inline void adjoint_lead_columns(const AdjointArgs& a, int e, lds_double* Ms) {
    constexpr int BS = 2 * W * W;
    const int N = W * a.L;
    const int tid = threadIdx.x;
    const bool on = tid < 2 * W;
    const int sp = a.inject_lead == 0 ? 0 : N - W;
    const int sq = a.inject_lead == 0 ? N - W : 0;
    const bool isq = tid < W;
    const int col = isq ? sq + tid : sp + tid - W;  // column of G
    const int yc = isq ? sq + tid : N + tid - W;    // column of Y
    const double2* Ge = a.G + (size_t)e * N * a.ld;
    double2* Ye = a.Y + (size_t)e * N * a.ldY;
    const double* xe = a.xl + (size_t)e * 2 * a.ld;
    const double* de = isq ? xe : xe + a.ld;
    const double2* gLe = a.gL + (size_t)e * a.L * W * W;
    double2 y[W], z[W];
#pragma unroll
    for (int r = 0; r < W; ++r) y[r] = cmk(0.0, 0.0);
    stage_block<W, 64>(Ms, gLe, tid);
    for (int k = 0; k < a.L; ++k) {
        __syncthreads();  // block k visible in buffer k & 1; the other is no longer read
        if (k + 1 < a.L)
            stage_block<W, 64>(Ms + ((k + 1) & 1) * BS, gLe + (size_t)(k + 1) * W * W, tid);
        if (on) {
#pragma unroll
            for (int r = 0; r < W; ++r) {
                const int row = k * W + r;
                const double d = a.gamma[row] * de[row];
                const double2 g = Ge[(size_t)row * a.ld + col];
                z[r] = cmk(fma(d, g.x, -a.t * y[r].x), fma(d, g.y, -a.t * y[r].y));
            }
            conj_block_matvec<W>(y, z, Ms + (k & 1) * BS);
#pragma unroll
            for (int r = 0; r < W; ++r) Ye[(size_t)(k * W + r) * a.ldY + yc] = y[r];
        }
    }
    // y now holds y_{L-1} = q_{L-1}; the backward sweep stages gL_{L-2}, gL_{L-3}, ...
    __syncthreads();
    if (a.L > 1) stage_block<W, 64>(Ms, gLe + (size_t)(a.L - 2) * W * W, tid);
    for (int k = a.L - 2; k >= 0; --k) {
        const int j = a.L - 2 - k;  // 0, 1, ... : buffer parity
        __syncthreads();
        if (k > 0)
            stage_block<W, 64>(Ms + ((j + 1) & 1) * BS, gLe + (size_t)(k - 1) * W * W, tid);
        if (on) {
            conj_block_matvec<W>(z, y, Ms + (j & 1) * BS);
#pragma unroll
            for (int r = 0; r < W; ++r) {
                double2* at = Ye + (size_t)(k * W + r) * a.ldY + yc;
                y[r] = cmk(fma(-a.t, z[r].x, at->x), fma(-a.t, z[r].y, at->y));
                *at = y[r];
            }
        }
    }
}

__device__ inline double other_half(double v) {  // of lane + 32, in lanes 0 .. 31
    auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[1], lo[1]);
}

// Dense columns on the VALU (up to W = 15): a wavefront owns 32 columns, lanes 0 .. 31 eliminate
// h^v, lanes 32 .. 63 h^u, and the blocks gL_k are broadcast from LDS to both (double-buffered, one
// slice ahead).  Per column
//   kd = sum_k (w^u_k)^T y^v_k,  kg = sum_a G_ac^2 u_a x_a,  pv = sum_a |G_ac|^2 v_a,  pu (u).
// The first workgroup of an energy takes the lead columns instead.
// Above W = 12 the registers are held to two wavefronts per SIMD, no fewer and no more, and the
// rows of G and of the final sums are taken four at a time (all at once, they cost a wavefront at
// W = 15; held to three, the LDS operands come too late): W = 15, N = 2400, 16 energies 4.46 ->
// 2.46 ms, W = 14 2.48 -> 2.38.
template <int W>
__global__ void __launch_bounds__(64)
    __attribute__((amdgpu_waves_per_eu(W > 12 ? 2 : 1, W > 12 ? 2 : 8)))
    adjoint_solve_kernel(AdjointArgs a) {
    constexpr int BS = 2 * W * W;  // doubles per buffer
    __shared__ double Ms_raw[2 * BS];
    lds_double* Ms = (lds_double*)Ms_raw;
    const int e = blockIdx.y;
    if (blockIdx.x == 0) {
        adjoint_lead_columns<W>(a, e, Ms);
        return;
    }
    const int N = W * a.L;
    const int lane = threadIdx.x;
    const bool half_u = lane >= 32;
    const int c = (blockIdx.x - 1) * 32 + (lane & 31);
    const int col = min(c, N - 1);
    const double2* Ge = a.G + (size_t)e * N * a.ld;
    const double* xe = a.xl + (size_t)e * 2 * a.ld;
    const double* le = xe + a.ld;
    const double2* gLe = a.gL + (size_t)e * a.L * W * W;
    double2 y[W], w[W];
#pragma unroll
    for (int r = 0; r < W; ++r) y[r] = cmk(0.0, 0.0);
    double2 kd = cmk(0.0, 0.0), kg = cmk(0.0, 0.0);
    double pv = 0.0, pu = 0.0;
    stage_block<W, 64>(Ms, gLe, lane);
    for (int k = 0; k < a.L; ++k) {
        __syncthreads();
        if (k + 1 < a.L)
            stage_block<W, 64>(Ms + ((k + 1) & 1) * BS, gLe + (size_t)(k + 1) * W * W, lane);
#pragma unroll
        for (int r = 0; r < W; ++r) {
            const int row = k * W + r;
            const double gm = a.gamma[row], x = xe[row];
            const double ua = gm * le[row], va = gm * x;
            const double d = half_u ? ua : va;
            const double2 g = Ge[(size_t)row * a.ld + col];
            w[r] = cmk(fma(d, g.x, -a.t * y[r].x), fma(d, g.y, -a.t * y[r].y));
            kg = cadd(kg, cscale(cmul(g, g), ua * x));
            const double p = cabs2(g);
            pv = fma(p, va, pv);
            pu = fma(p, ua, pu);
            if (W > 12 && r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        if (W > 12) __builtin_amdgcn_sched_barrier(0);
        conj_block_matvec<W>(y, w, Ms + (k & 1) * BS);
        if (W > 12) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < W; ++r) {
            cfma(kd, cmk(other_half(w[r].x), other_half(w[r].y)), y[r]);
            if (W > 12 && r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (!half_u && c < N) {
        a.part_k[((size_t)e * 2 + 0) * N + c] = kd;
        a.part_k[((size_t)e * 2 + 1) * N + c] = kg;
        a.part_p[((size_t)e * 2 + 0) * N + c] = pv;
        a.part_p[((size_t)e * 2 + 1) * N + c] = pu;
    }
}

// Dense columns from W = 16 on, on the FP64 matrix cores: a wavefront owns TC tiles of 16
// columns and both eliminations of each; lane (n, g) holds the rows 16 rt + 4 r + g of column n,
// which is the accumulator layout of one product and the B operand of the next, so w and y
// never leave registers; the staged block is the A operand (NW wavefronts share it).  G is read
// one slice ahead, under the products (64 clocks each, 4 (W / 4) (W / 16) per complex tile).
// N = 3200, 128 energies: 22.9 -> 7.6 ms (44 TFLOP/s; G read at 2.8 TB/s); W = 32, N = 4160,
// 16 energies 25.5 -> 4.1 ms.
// Widths between 16 and 32 are padded to 32 rows of zeros (a padded row reads a row of its block
// and multiplies it by a zero rate; steps of four padded columns are left out).  On the VALU both
// eliminations of a column take 8 W registers at once, which from W = 17 on leaves one wavefront
// per SIMD: N = 2400, 16 energies, W = 17 5.04 -> 1.74 ms, W = 24 6.39 -> 1.45 ms, W = 31 11.3 ->
// 1.84 ms (with a full solve per column 2.7, 4.4 and 7.3 ms).
typedef double dmfma4 __attribute__((ext_vector_type(4)));

// Rows a block of width W takes on the matrix cores.
constexpr int padded(int W) { return (W + 15) / 16 * 16; }
// Padded row y: whether the block has it, and a row of the block to read in its place.
template <int W>
__device__ inline bool has_row(int y) {
    return W == padded(W) || y < W;
}
template <int W>
__device__ inline int row_in_block(int y) {
    return W == padded(W) ? y : min(y, W - 1);
}

// The block src into the LDS buffer dst of padded rows; the padding stays zero.
template <int W, int NT>
__device__ inline void stage_padded(lds_double* dst, const double2* __restrict__ src, int tid) {
    if constexpr (W == padded(W)) {
        stage_block<W, NT>(dst, src, tid);
    } else {
#pragma unroll
        for (int i = tid; i < W * W; i += NT) {
            const double2 v = src[i];
            const int at = 2 * (i / W * padded(W) + i % W);
            dst[at] = v.x;
            dst[at + 1] = v.y;
        }
    }
}

// (yr, yi)[i] = conj(M) (wr, wi)[i] for V vectors, M staged in LDS.
template <int W, int V>
__device__ inline void conj_product(dmfma4 (&yr)[V][padded(W) / 16], dmfma4 (&yi)[V][padded(W) / 16],
                                    const dmfma4 (&wr)[V][padded(W) / 16],
                                    const dmfma4 (&wi)[V][padded(W) / 16], const lds_double* M,
                                    int n, int g) {
#pragma unroll
    for (int rt = 0; rt < padded(W) / 16; ++rt) {
#pragma unroll
        for (int i = 0; i < V; ++i) yr[i][rt] = yi[i][rt] = dmfma4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < (W + 3) / 4; ++s) {
            const int at = 2 * ((16 * rt + n) * padded(W) + 4 * s + g);
            const double ar = M[at], ai = M[at + 1];  // conj: ar - i ai
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const double br = wr[i][s >> 2][s & 3], bi = wi[i][s >> 2][s & 3];
                yr[i][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, yr[i][rt], 0, 0, 0);
                yi[i][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, yi[i][rt], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const double br = wr[i][s >> 2][s & 3], bi = wi[i][s >> 2][s & 3];
                yr[i][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, bi, yr[i][rt], 0, 0, 0);
                yi[i][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, br, yi[i][rt], 0, 0, 0);
            }
        }
    }
}

// The lead columns of one energy (see adjoint_lead_columns), 16 per wavefront.
template <int W>
__device__ inline void adjoint_lead_mfma(const AdjointArgs& a, int e, lds_double* Ms) {
    constexpr int P = padded(W), RT = P / 16, BS = 2 * P * P;
    constexpr int NT = 8 * P;  // 2 W columns, 16 per wavefront
    const int N = W * a.L;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int sp = a.inject_lead == 0 ? 0 : N - W;
    const int sq = a.inject_lead == 0 ? N - W : 0;
    const int lc = 16 * (tid >> 6) + n;
    const bool on = W == P || lc < 2 * W;
    const int c = on ? lc : 0;
    const bool isq = c < W;
    const int col = isq ? sq + c : sp + c - W;  // column of G
    const int yc = isq ? sq + c : N + c - W;    // column of Y
    const double2* Ge = a.G + (size_t)e * N * a.ld;
    double2* Ye = a.Y + (size_t)e * N * a.ldY;
    const double* xe = a.xl + (size_t)e * 2 * a.ld;
    const double* de = isq ? xe : xe + a.ld;
    const double2* gLe = a.gL + (size_t)e * a.L * W * W;
    dmfma4 yr[1][RT], yi[1][RT], wr[1][RT], wi[1][RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) yr[0][rt] = yi[0][rt] = dmfma4{0, 0, 0, 0};
    stage_padded<W, NT>(Ms, gLe, tid);
    for (int k = 0; k < a.L; ++k) {
        __syncthreads();
        if (k + 1 < a.L)
            stage_padded<W, NT>(Ms + ((k + 1) & 1) * BS, gLe + (size_t)(k + 1) * W * W, tid);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int y = 16 * rt + 4 * r + g;
                const int row = k * W + row_in_block<W>(y);
                const double d = has_row<W>(y) ? a.gamma[row] * de[row] : 0.0;
                const double2 v = Ge[(size_t)row * a.ld + col];
                wr[0][rt][r] = fma(d, v.x, -a.t * yr[0][rt][r]);
                wi[0][rt][r] = fma(d, v.y, -a.t * yi[0][rt][r]);
            }
        conj_product<W, 1>(yr, yi, wr, wi, Ms + (k & 1) * BS, n, g);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int y = 16 * rt + 4 * r + g;
                if (on && has_row<W>(y))
                    Ye[(size_t)(k * W + y) * a.ldY + yc] = cmk(yr[0][rt][r], yi[0][rt][r]);
            }
    }
    __syncthreads();
    if (a.L > 1) stage_padded<W, NT>(Ms, gLe + (size_t)(a.L - 2) * W * W, tid);
    for (int k = a.L - 2; k >= 0; --k) {
        const int j = a.L - 2 - k;
        __syncthreads();
        if (k > 0)
            stage_padded<W, NT>(Ms + ((j + 1) & 1) * BS, gLe + (size_t)(k - 1) * W * W, tid);
        conj_product<W, 1>(wr, wi, yr, yi, Ms + (j & 1) * BS, n, g);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int y = 16 * rt + 4 * r + g;
                double2* at = Ye + (size_t)(k * W + row_in_block<W>(y)) * a.ldY + yc;
                const double2 v = *at;
                yr[0][rt][r] = has_row<W>(y) ? fma(-a.t, wr[0][rt][r], v.x) : 0.0;
                yi[0][rt][r] = has_row<W>(y) ? fma(-a.t, wi[0][rt][r], v.y) : 0.0;
                if (on && has_row<W>(y)) *at = cmk(yr[0][rt][r], yi[0][rt][r]);
            }
    }
}

// One workgroup of P / 8 wavefronts (P the padded width): the lead columns (first workgroup of an
// energy), else 16 TC dense columns per wavefront, TC = 32 / P.
template <int W>
__global__ void __launch_bounds__(8 * padded(W), 2) adjoint_mfma_kernel(AdjointArgs a) {
    constexpr int P = padded(W), TC = 32 / P, NW = P / 8;
    constexpr int RT = P / 16, BS = 2 * P * P, NT = 64 * NW;
    __shared__ double Ms_raw[2 * BS];
    lds_double* Ms = (lds_double*)Ms_raw;
    const int e = blockIdx.y;
    if constexpr (W != P) {
        for (int i = threadIdx.x; i < 2 * BS; i += NT) Ms[i] = 0.0;
        __syncthreads();
    }
    if (blockIdx.x == 0) {
        adjoint_lead_mfma<W>(a, e, Ms);
        return;
    }
    const int N = W * a.L;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int c0 = ((blockIdx.x - 1) * NW + (tid >> 6)) * 16 * TC;
    const double2* Ge = a.G + (size_t)e * N * a.ld;
    const double* xe = a.xl + (size_t)e * 2 * a.ld;
    const double* le = xe + a.ld;
    const double2* gLe = a.gL + (size_t)e * a.L * W * W;
    int col[TC];
    double2 kd[TC], kg[TC];
    double pv[TC], pu[TC];
#pragma unroll
    for (int tc = 0; tc < TC; ++tc) {
        col[tc] = min(c0 + 16 * tc + n, N - 1);
        kd[tc] = kg[tc] = cmk(0.0, 0.0);
        pv[tc] = pu[tc] = 0.0;
    }
    // [2 tile + (0: u, 1: v)][row tile]: y of the previous slice, then w of this one
    dmfma4 wr[2 * TC][RT], wi[2 * TC][RT];
#pragma unroll
    for (int i = 0; i < 2 * TC; ++i)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) wr[i][rt] = wi[i][rt] = dmfma4{0, 0, 0, 0};
    dmfma4 gr[TC][RT], gi[TC][RT], gam[RT], xk[RT], lk[RT];
    auto read = [&](int k) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int y = 16 * rt + 4 * r + g;
                const int row = k * W + row_in_block<W>(y);
                gam[rt][r] = has_row<W>(y) ? a.gamma[row] : 0.0;
                xk[rt][r] = xe[row];
                lk[rt][r] = le[row];
#pragma unroll
                for (int tc = 0; tc < TC; ++tc) {
                    const double2 v = Ge[(size_t)row * a.ld + col[tc]];
                    gr[tc][rt][r] = v.x;
                    gi[tc][rt][r] = v.y;
                }
            }
    };
    read(0);
    stage_padded<W, NT>(Ms, gLe, tid);
    for (int k = 0; k < a.L; ++k) {
        __syncthreads();
        if (k + 1 < a.L)
            stage_padded<W, NT>(Ms + ((k + 1) & 1) * BS, gLe + (size_t)(k + 1) * W * W, tid);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double ua = gam[rt][r] * lk[rt][r], va = gam[rt][r] * xk[rt][r];
                const double ux = ua * xk[rt][r];
#pragma unroll
                for (int tc = 0; tc < TC; ++tc) {
                    const double2 v = cmk(gr[tc][rt][r], gi[tc][rt][r]);
                    wr[2 * tc][rt][r] = fma(ua, v.x, -a.t * wr[2 * tc][rt][r]);
                    wi[2 * tc][rt][r] = fma(ua, v.y, -a.t * wi[2 * tc][rt][r]);
                    wr[2 * tc + 1][rt][r] = fma(va, v.x, -a.t * wr[2 * tc + 1][rt][r]);
                    wi[2 * tc + 1][rt][r] = fma(va, v.y, -a.t * wi[2 * tc + 1][rt][r]);
                    kg[tc] = cadd(kg[tc], cscale(cmul(v, v), ux));
                    const double p = cabs2(v);
                    pv[tc] = fma(p, va, pv[tc]);
                    pu[tc] = fma(p, ua, pu[tc]);
                }
            }
        read(min(k + 1, a.L - 1));
        __builtin_amdgcn_sched_barrier(0);  // the loads go ahead of the products
        dmfma4 yr[2 * TC][RT], yi[2 * TC][RT];
        conj_product<W, 2 * TC>(yr, yi, wr, wi, Ms + (k & 1) * BS, n, g);
#pragma unroll
        for (int tc = 0; tc < TC; ++tc)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    cfma(kd[tc], cmk(wr[2 * tc][rt][r], wi[2 * tc][rt][r]),
                         cmk(yr[2 * tc + 1][rt][r], yi[2 * tc + 1][rt][r]));
#pragma unroll
        for (int i = 0; i < 2 * TC; ++i)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                wr[i][rt] = yr[i][rt];
                wi[i][rt] = yi[i][rt];
            }
    }
    auto over_groups = [](double v) {  // the four lanes of a column
        v += __shfl_xor(v, 16, 64);
        return v + __shfl_xor(v, 32, 64);
    };
#pragma unroll
    for (int tc = 0; tc < TC; ++tc) {
        const double2 d = cmk(over_groups(kd[tc].x), over_groups(kd[tc].y));
        const double2 q = cmk(over_groups(kg[tc].x), over_groups(kg[tc].y));
        const double sv = over_groups(pv[tc]), su = over_groups(pu[tc]);
        const int c = c0 + 16 * tc + n;
        if (g == 0 && c < N) {
            a.part_k[((size_t)e * 2 + 0) * N + c] = d;
            a.part_k[((size_t)e * 2 + 1) * N + c] = q;
            a.part_p[((size_t)e * 2 + 0) * N + c] = sv;
            a.part_p[((size_t)e * 2 + 1) * N + c] = su;
        }
    }
}

// Per energy and site i: K_i and the explicit gamma terms (see the top of the file), from
// the column partials of adjoint_solve_kernel, the rows i of Q (columns sq..) and R
// (columns N..) in Y, and the slice entries G_{sp+c,i}, G_{sq+c,i}.
template <int W>
__global__ void __launch_bounds__(256) grad_assemble_kernel(
    const double2* __restrict__ Gc, const double2* __restrict__ Y, const double* __restrict__ xl,
    const double* __restrict__ gamma, const double* __restrict__ wL, const double* __restrict__ wR,
    const double* __restrict__ Adiag, const double* __restrict__ gam_lead,
    const double2* __restrict__ corner, const double2* __restrict__ part_k,
    const double* __restrict__ part_p, int L, int64_t ld, int64_t ldY, uint32_t inject_lead,
    double* __restrict__ gV, double* __restrict__ gG) {
    constexpr int WW = W * W;
    __shared__ double2 psi5[WW];  // Psi5[a][b], a in slice q, b in slice p
    const int N = W * L;
    const int e = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int sp = inject_lead == 0 ? 0 : (L - 1) * W;  // first site of slice p
    const int sq = inject_lead == 0 ? (L - 1) * W : 0;  // first site of slice q
    const double* gm = gam_lead + (size_t)e * WW;       // Gamma_p = Gamma_q (identical leads)
    // corner C = G_{q,p}: G_{L-1,0} for injection from L, G_{0,L-1} from R
    const double2* C = corner + (size_t)e * 2 * WW + (inject_lead == 0 ? 0 : WW);
    for (int t = threadIdx.x; t < WW; t += blockDim.x) {
        const int a = t / W, b = t % W;
        // Psi5[a][b] = 2 (Gamma_p C^+ Gamma_q)[b][a] = 2 sum_{c,d} Gp[b][c] conj(C[d][c]) Gq[d][a]
        double2 acc = cmk(0.0, 0.0);
        for (int c = 0; c < W; ++c)
            for (int d = 0; d < W; ++d) {
                const double f = 2.0 * gm[b * W + c] * gm[d * W + a];
                const double2 cc = C[d * W + c];
                acc = cadd(acc, cmk(f * cc.x, -f * cc.y));
            }
        psi5[t] = acc;
    }
    __syncthreads();
    if (i >= N) return;
    const double2* Ge = Gc + (size_t)e * N * ld;
    const double2* Yi = Y + ((size_t)e * N + i) * ldY;
    const double* xe = xl + (size_t)e * 2 * ld;
    const double* le = xe + ld;
    const double2 kd = part_k[((size_t)e * 2 + 0) * N + i];
    const double2 kg = part_k[((size_t)e * 2 + 1) * N + i];
    const double pv = part_p[((size_t)e * 2 + 0) * N + i];
    const double pu = part_p[((size_t)e * 2 + 1) * N + i];
    double2 K = cadd(cscale(kd, 2.0), cmk(2.0 * kg.y, -2.0 * kg.x));  // 2 kd - 2i kg
    // lead terms: 2 sum_b al_b (Gamma_p G_{p,i})_b + 2 sum_b be_b (Gamma_q G_{q,i})_b with
    // al_b = conj(R_{i,sp+b}), be_b = conj(Q_{i,sq+b})
    double2 gpi[W], gqi[W];
#pragma unroll
    for (int c = 0; c < W; ++c) {
        gpi[c] = Ge[(size_t)(sp + c) * ld + i];
        gqi[c] = Ge[(size_t)(sq + c) * ld + i];
    }
#pragma unroll 1
    for (int b = 0; b < W; ++b) {
        double2 tp = cmk(0.0, 0.0), tq = cmk(0.0, 0.0);
#pragma unroll
        for (int c = 0; c < W; ++c) {
            tp = cadd(tp, cscale(gpi[c], gm[b * W + c]));
            tq = cadd(tq, cscale(gqi[c], gm[b * W + c]));
        }
        const double2 al = cconj(Yi[N + b]);
        const double2 be = cconj(Yi[sq + b]);
        K = cadd(K, cscale(cadd(cmul(al, tp), cmul(be, tq)), 2.0));
    }
    // T_qp term: sum_{a in q, b in p} G_ia Psi5_ab G_bi
#pragma unroll 1
    for (int a = 0; a < W; ++a) {
        double2 s = cmk(0.0, 0.0);
#pragma unroll
        for (int b = 0; b < W; ++b) s = cadd(s, cmul(psi5[a * W + b], gpi[b]));
        K = cadd(K, cmul(Ge[(size_t)(sq + a) * ld + i], s));
    }
    const double wp = inject_lead == 0 ? wL[(size_t)e * N + i] : wR[(size_t)e * N + i];
    const double wq = inject_lead == 0 ? wR[(size_t)e * N + i] : wL[(size_t)e * N + i];
    const double Aii = Adiag[(size_t)e * N + i];
    double lam = le[i], x = xe[i];
    if (gamma[i] == 0.0) {
        // The site is absent from the probe system (its row of M vanishes), but x_i and
        // lambda_i have finite limits as gamma_i -> 0: row i of M x = b divided by gamma_i.
        x = (wp + pv) / Aii;
        lam = (wq + pu) / Aii;
    }
    gV[(size_t)e * N + i] = K.x;
    gG[(size_t)e * N + i] = 0.5 * K.y + lam * wp + x * wq - lam * Aii * x + lam * pv + x * pu;
}

// dI/dV_i = sum_k w_k gV[k][i], dI/dgamma_i likewise (fixed order over k).
__global__ void grad_reduce_kernel(const double* __restrict__ gV, const double* __restrict__ gG,
                                   const double* __restrict__ w, int nE, int N,
                                   double* __restrict__ dV, double* __restrict__ dG) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    double a = 0.0, b = 0.0;
    for (int k = 0; k < nE; ++k) {
        a = fma(w[k], gV[(size_t)k * N + i], a);
        b = fma(w[k], gG[(size_t)k * N + i], b);
    }
    dV[i] = a;
    dG[i] = b;
}

template <int W>
static hipError_t launch_adjoint_w(const mcnegf_kernel& k, const GradBuffers& gb,
                                   uint32_t inject_lead, hipStream_t s) {
    const AdjointArgs a = {reinterpret_cast<const double2*>(k.gL), gb.G, gb.xl, k.gamma, gb.Y,
                           gb.part_k, gb.part_p, k.L, k.t, gb.ld, gb.ldY, inject_lead};
    {
        // one workgroup of lead columns, then the dense ones
        MCNEGF_TIMED("adjoint_solve_kernel", s);
        if constexpr (W >= 16) {
            // 64 columns per workgroup: P / 8 wavefronts of 32 / P tiles of 16.  Ahead of the
            // VALU at every width it pads, by the least at 17 (2.69 -> 1.74 ms, see above, with
            // the VALU's registers held to two wavefronts).
            hipLaunchKernelGGL(adjoint_mfma_kernel<W>, dim3(1 + (k.N + 63) / 64, k.nE),
                               dim3(8 * padded(W)), 0, s, a);
        } else {
            hipLaunchKernelGGL(adjoint_solve_kernel<W>, dim3(1 + (k.N + 31) / 32, k.nE), dim3(64),
                               0, s, a);
        }
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    {
        MCNEGF_TIMED("grad_assemble_kernel", s);
        hipLaunchKernelGGL(grad_assemble_kernel<W>, dim3((k.N + 255) / 256, k.nE), dim3(256), 0,
                           s, gb.G, gb.Y, gb.xl, k.gamma, k.wL, k.wR, k.Adiag, k.gam_lead,
                           reinterpret_cast<const double2*>(k.corner), gb.part_k, gb.part_p, k.L,
                           gb.ld, gb.ldY, inject_lead, gb.gV, gb.gG);
    }
    return hipGetLastError();
}

static hipError_t launch_backsolve(const mcnegf_kernel& k, double* xl, hipStream_t s) {
    const int N = k.N, nE = k.nE;
    const int Np = (int)k.p_pitch;
    {
        MCNEGF_TIMED("backsolve_kernel", s);
        if (Np <= BSV_THREADS * 4)
            hipLaunchKernelGGL(backsolve_kernel<4>, dim3(nE), dim3(BSV_THREADS), 0, s, k.direct,
                               k.direct_vec, N, Np, k.p_pitch, xl);
        else if (Np <= BSV_THREADS * 8)
            hipLaunchKernelGGL(backsolve_kernel<8>, dim3(nE), dim3(BSV_THREADS), 0, s, k.direct,
                               k.direct_vec, N, Np, k.p_pitch, xl);
        else
            hipLaunchKernelGGL(backsolve_kernel<16>, dim3(nE), dim3(BSV_THREADS), 0, s, k.direct,
                               k.direct_vec, N, Np, k.p_pitch, xl);
    }
    return hipGetLastError();
}

// Energies are processed in chunks of `chunk`: the complex G, the adjoint solves and the
// per-site partials of one chunk live in the workspace at a time (the stored RGF blocks of
// every energy regenerate each chunk's G); gV, gG hold every energy for the final sum.
hipError_t launch_grad(const mcnegf_kernel& k, const GradBuffers& gb, uint32_t inject_lead,
                       const double* weights, double* dI_dV, double* dI_dgamma, int chunk,
                       hipStream_t s) {
    const int N = k.N, nE = k.nE;
    hipError_t err;
    for (int e0 = 0; e0 < nE; e0 += chunk) {
        const int nc = min(chunk, nE - e0);
        const mcnegf_kernel kc = energy_slice(k, e0, nc);
        GradBuffers g = gb;
        g.gV = gb.gV + (size_t)e0 * N;
        g.gG = gb.gG + (size_t)e0 * N;
        if ((err = launch_backsolve(kc, g.xl, s)) != hipSuccess) return err;
        if ((err = launch_fullinv_store_g(kc, g.G, g.ld, s)) != hipSuccess) return err;
        switch (k.W) {
#define MCNEGF_CASE(w)                                                         \
    case w:                                                                    \
        if ((err = launch_adjoint_w<w>(kc, g, inject_lead, s)) != hipSuccess) \
            return err;                                                        \
        break;
            MCNEGF_CASE(1) MCNEGF_CASE(2) MCNEGF_CASE(3) MCNEGF_CASE(4) MCNEGF_CASE(5)
            MCNEGF_CASE(6) MCNEGF_CASE(7) MCNEGF_CASE(8) MCNEGF_CASE(9) MCNEGF_CASE(10)
            MCNEGF_CASE(11) MCNEGF_CASE(12) MCNEGF_CASE(13) MCNEGF_CASE(14) MCNEGF_CASE(15)
            MCNEGF_CASE(16) MCNEGF_CASE(17) MCNEGF_CASE(18) MCNEGF_CASE(19) MCNEGF_CASE(20)
            MCNEGF_CASE(21) MCNEGF_CASE(22) MCNEGF_CASE(23) MCNEGF_CASE(24) MCNEGF_CASE(25)
            MCNEGF_CASE(26) MCNEGF_CASE(27) MCNEGF_CASE(28) MCNEGF_CASE(29) MCNEGF_CASE(30)
            MCNEGF_CASE(31) MCNEGF_CASE(32)
#undef MCNEGF_CASE
            default:
                return hipErrorInvalidValue;
        }
    }
    return launch_grad_reduce(gb, weights, nE, N, dI_dV, dI_dgamma, s);
}

hipError_t launch_grad_reduce(const GradBuffers& gb, const double* weights, int nE, int N,
                              double* dI_dV, double* dI_dgamma, hipStream_t s) {
    {
        MCNEGF_TIMED("grad_reduce_kernel", s);
        hipLaunchKernelGGL(grad_reduce_kernel, dim3((N + 255) / 256), dim3(256), 0, s, gb.gV,
                           gb.gG, weights, nE, N, dI_dV, dI_dgamma);
    }
    return hipGetLastError();
}

}  // namespace mcnegf
