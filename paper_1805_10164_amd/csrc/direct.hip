// Effective transmissions and the current.
//
// MC (Sec. II E, Eq. (66); relative deviation as in Sec. IV A): with injection at lead p,
//   p_k = exits at the other lead q / walkers,  T_k = c_p p_k,
//   sigma_k = c_p sqrt(p_k (1 - p_k) / (walkers - 1)),  c_p = total of injection row p.
// DIRECT (Sec. III C, Eq. (79)): the diagonal of G^< = G Sigma^< G^+ (Eq. (8)) with
// Buttiker lesser self-energies gamma_i n_i gives, per probe j,
//   gamma_j A_jj n_j - sum_i T_ji n_i = T_jp   (f_p = 1, f_q = 0),  T_ji = gamma_j gamma_i |G_ji|^2,
// a symmetric, weakly diagonally dominant system with positive diagonal (its row sums are
// the probe's couplings to the leads), so Cholesky without pivoting applies.  It is solved
// in the symmetrically scaled form S M S = L L^T with S = diag(M_jj^{-1/2}); probes with
// gamma_j = 0 decouple (identity row).  Then
//   T_k = T_qp + sum_j T_qj n_j = T_qp + (L^{-1} S T_q) . (L^{-1} S T_p),
// so only forward substitutions are needed; they come out of the factorization itself when
// the two vectors (S T_p)^T and (S T_q)^T are appended below the matrix as two extra rows.
// Current: I = sum_k w_k T_k (midpoint quadrature, Sec. III C), sigma_I^2 = sum_k w_k^2 sigma_k^2.
#include <algorithm>

#include "common.h"

namespace mcnegf {

__device__ inline double block_reduce256(double v, double* red) {
    const int tid = threadIdx.x;
    red[tid] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// The weighted sums over energies of a workgroup of 256 (fixed order): reduce[0] = sum w T,
// reduce[1] = sum w^2 s^2, and I, sigma_I for the caller if I_sigma is given.
__device__ inline void store_current(double a, double b, double* red, double* __restrict__ reduce,
                                     double* __restrict__ I_sigma) {
    a = block_reduce256(a, red);
    b = block_reduce256(b, red);
    if (threadIdx.x == 0) {
        reduce[0] = a;
        reduce[1] = b;
        if (I_sigma) {
            I_sigma[0] = a;
            I_sigma[1] = sqrt(b > 0.0 ? b : 0.0);
        }
    }
}

__global__ void __launch_bounds__(256) current_sum_kernel(const double* __restrict__ T,
                                                          const double* __restrict__ sig,
                                                          const double* __restrict__ w, int nE,
                                                          double* __restrict__ reduce,
                                                          double* __restrict__ I_sigma) {
    __shared__ double red[256];
    double a = 0.0, b = 0.0;
    for (int k = threadIdx.x; k < nE; k += 256) {
        a += w[k] * T[k];
        b += w[k] * w[k] * sig[k] * sig[k];
    }
    store_current(a, b, red, reduce, I_sigma);
}

struct McCurrentArgs {
    const int64_t* tallies;
    const double* lead;
    int nE;
    uint32_t inject_lead;
    double* T;
    double* sig;
};

// T_k and sigma_k of energy k's tallies, stored and returned.
__device__ inline double2 mc_current_entry(const McCurrentArgs& m, int k) {
    const int64_t* t = m.tallies + (size_t)k * MCNEGF_TALLY_N;
    const double walkers =
        (double)(t[MCNEGF_TALLY_EXIT_L] + t[MCNEGF_TALLY_EXIT_R] + t[MCNEGF_TALLY_TRUNC]);
    const double hits =
        (double)(m.inject_lead == 0 ? t[MCNEGF_TALLY_EXIT_R] : t[MCNEGF_TALLY_EXIT_L]);
    const double c = m.lead[(size_t)k * MCNEGF_LEAD_NTERMS +
                            (m.inject_lead == 0 ? MCNEGF_LEAD_CL : MCNEGF_LEAD_CR)];
    const double p = walkers > 0.0 ? hits / walkers : 0.0;
    const double Tk = walkers > 0.0 ? c * p : 0.0;
    const double sk = walkers > 1.0 ? c * sqrt(p * (1.0 - p) / (walkers - 1.0)) : 0.0;
    m.T[k] = Tk;
    m.sig[k] = sk;
    return cmk(Tk, sk);
}

// The entries and their weighted sums in one workgroup: with few energies what a call costs is
// launches (three of them, 18 us between events, before).
__global__ void __launch_bounds__(256) mc_current_kernel(McCurrentArgs m,
                                                         const double* __restrict__ w,
                                                         double* __restrict__ reduce,
                                                         double* __restrict__ I_sigma) {
    __shared__ double red[256];
    double a = 0.0, b = 0.0;
#pragma unroll 4
    for (int k = threadIdx.x; k < m.nE; k += 256) {
        const double2 Ts = mc_current_entry(m, k);
        a += w[k] * Ts.x;
        b += w[k] * w[k] * Ts.y * Ts.y;
    }
    store_current(a, b, red, reduce, I_sigma);
}

__global__ void __launch_bounds__(256) mc_entries_kernel(McCurrentArgs m) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < m.nE) mc_current_entry(m, k);
}

// One workgroup for entries and sums up to 8192 energies (4096: 13.6 us between events, 16.5 as
// launches of their own; 16384: 26 both ways), above that the entries over the whole chip, then
// the sums (70000: 154 us in one workgroup, 81 here).  Both add in the same order.
constexpr int kOneGroupEnergies = 8192;

hipError_t launch_mc_current(const mcnegf_kernel& k, uint32_t inject_lead, const int64_t* tallies,
                             const double* weights, double* T, double* sigmaT, double* I_sigma,
                             hipStream_t s) {
    const McCurrentArgs m = {tallies, k.lead, k.nE, inject_lead, T, sigmaT};
    if (k.nE <= kOneGroupEnergies) {
        MCNEGF_TIMED("mc_current_kernel", s);
        hipLaunchKernelGGL(mc_current_kernel, dim3(1), dim3(256), 0, s, m, weights, k.reduce,
                           I_sigma);
        return hipGetLastError();
    }
    {
        MCNEGF_TIMED("mc_current_kernel", s);
        hipLaunchKernelGGL(mc_entries_kernel, dim3((k.nE + 255) / 256), dim3(256), 0, s, m);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    {
        MCNEGF_TIMED("current_sum_kernel", s);
        hipLaunchKernelGGL(current_sum_kernel, dim3(1), dim3(256), 0, s, T, sigmaT, weights, k.nE,
                           k.reduce, I_sigma);
    }
    return hipGetLastError();
}

// Energy-resolved current of inelastic walks (step 7'): a walker injected at lead p at energy
// e0 scores c_p(e0) at its exit, so the exits at lead r with energy e give
//   S[r][e] = sum_e0 w_e0 c_p(e0) hist[r][e0][e] / N_e0
// (N_e0 the walkers injected at e0, truncated ones included); sum_e S[q][e] is the current of
// the tallies.  A workgroup takes 16 entries of one lead: 16 threads per entry sum every 16th e0,
// the partial sums are added in a fixed order (one thread per entry, a chain of nE loads, took
// 135 us at 256 energies).
__global__ void __launch_bounds__(256) spectrum_kernel(const int64_t* __restrict__ tallies,
                                                       const int64_t* __restrict__ hist,
                                                       const double* __restrict__ lead,
                                                       const double* __restrict__ weights,
                                                       int nE, uint32_t inject_lead,
                                                       double* __restrict__ S) {
    __shared__ double part[16][17];
    const int r = blockIdx.y;
    const int ce = threadIdx.x & 15, ch = threadIdx.x >> 4;
    const int e = blockIdx.x * 16 + ce;
    const int slot = inject_lead == 0 ? MCNEGF_LEAD_CL : MCNEGF_LEAD_CR;
    double acc = 0.0;
    if (e < nE) {
#pragma unroll 4
        for (int e0 = ch; e0 < nE; e0 += 16) {
            const int64_t* t = tallies + (size_t)e0 * MCNEGF_TALLY_N;
            const int64_t nw =
                t[MCNEGF_TALLY_EXIT_L] + t[MCNEGF_TALLY_EXIT_R] + t[MCNEGF_TALLY_TRUNC];
            const int64_t h = hist[((size_t)r * nE + e0) * nE + e];
            const double c = lead[(size_t)e0 * MCNEGF_LEAD_NTERMS + slot];
            acc += nw > 0 && h != 0 ? weights[e0] * c / (double)nw * (double)h : 0.0;
        }
    }
    part[ch][ce] = acc;
    __syncthreads();
    if (threadIdx.x < 16 && e < nE) {
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += part[i][ce];
        S[(size_t)r * nE + e] = sum;
    }
}

hipError_t launch_spectrum(const mcnegf_kernel& k, uint32_t inject_lead, const int64_t* tallies,
                           const int64_t* hist, const double* weights, double* spectrum,
                           hipStream_t s) {
    {
        MCNEGF_TIMED("spectrum_kernel", s);
        hipLaunchKernelGGL(spectrum_kernel, dim3((k.nE + 15) / 16, 2), dim3(256), 0, s, tallies,
                           hist, k.lead, weights, k.nE, inject_lead, spectrum);
    }
    return hipGetLastError();
}

// Importance-sampled walks (Sec. V A, "Improved estimator"): per energy the N_k walkers'
// scores (path likelihood ratios at an exit at q, else 0) have sums S1, S2; then
//   T_k = c_p S1 / N_k,  sigma_k = c_p sqrt(s^2 / N_k),  s^2 = (S2 - S1^2 / N_k) / (N_k - 1).
__global__ void weighted_current_kernel(const int64_t* __restrict__ tallies,
                                        const double* __restrict__ wsum,
                                        const double* __restrict__ lead, int nE,
                                        uint32_t inject_lead, double* __restrict__ T,
                                        double* __restrict__ sig) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nE) return;
    const int64_t* t = tallies + (size_t)k * MCNEGF_TALLY_N;
    const double walkers =
        (double)(t[MCNEGF_TALLY_EXIT_L] + t[MCNEGF_TALLY_EXIT_R] + t[MCNEGF_TALLY_TRUNC]);
    const double c = lead[(size_t)k * MCNEGF_LEAD_NTERMS +
                          (inject_lead == 0 ? MCNEGF_LEAD_CL : MCNEGF_LEAD_CR)];
    if (walkers <= 0.0) {
        T[k] = 0.0;
        sig[k] = 0.0;
        return;
    }
    const double s1 = wsum[2 * (size_t)k], s2 = wsum[2 * (size_t)k + 1];
    T[k] = c * s1 / walkers;
    const double var = walkers > 1.0 ? fmax(s2 - s1 * s1 / walkers, 0.0) / (walkers - 1.0) : 0.0;
    sig[k] = c * sqrt(var / walkers);
}

hipError_t launch_weighted_current(const mcnegf_kernel& k, uint32_t inject_lead,
                                   const int64_t* tallies, const double* wsum,
                                   const double* weights, double* T, double* sigmaT,
                                   hipStream_t s) {
    {
        MCNEGF_TIMED("weighted_current_kernel", s);
        hipLaunchKernelGGL(weighted_current_kernel, dim3((k.nE + 255) / 256), dim3(256), 0, s,
                           tallies, wsum, k.lead, k.nE, inject_lead, T, sigmaT);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    {
        MCNEGF_TIMED("current_sum_kernel", s);
        hipLaunchKernelGGL(current_sum_kernel, dim3(1), dim3(256), 0, s, T, sigmaT, weights, k.nE,
                           k.reduce, nullptr);
    }
    return hipGetLastError();
}

// Interpolated walks (Sec. V A, "Interpolation"): fine energy f between the built energies
// E_lo and E_hi with mixture weight alpha = a32 / 2^32 (the one its walks used); the row total
// that scales the estimator is interpolated like the rows, c = (1 - alpha) c_lo + alpha c_hi,
// then T_f and sigma_f as in MC mode.
__global__ void interp_current_kernel(const int64_t* __restrict__ tallies,
                                      const double* __restrict__ lead,
                                      const double* __restrict__ nodes, uint32_t nE,
                                      const double* __restrict__ fine, int nF,
                                      uint32_t inject_lead, double* __restrict__ T,
                                      double* __restrict__ sig, uint32_t* __restrict__ status) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nF) return;
    uint32_t lo, a32;
    bool bad;
    interp_bracket(nodes, nE, fine[f], lo, a32, bad);
    if (bad) atomicOr(status, MCNEGF_FLAG_RANGE);
    const uint32_t hi = lo + 1 < nE ? lo + 1 : lo;
    const int slot = inject_lead == 0 ? MCNEGF_LEAD_CL : MCNEGF_LEAD_CR;
    const double alpha = (double)a32 * 0x1.0p-32;
    const double c = (1.0 - alpha) * lead[(size_t)lo * MCNEGF_LEAD_NTERMS + slot] +
                     alpha * lead[(size_t)hi * MCNEGF_LEAD_NTERMS + slot];
    const int64_t* t = tallies + (size_t)f * MCNEGF_TALLY_N;
    const double walkers =
        (double)(t[MCNEGF_TALLY_EXIT_L] + t[MCNEGF_TALLY_EXIT_R] + t[MCNEGF_TALLY_TRUNC]);
    const double hits = (double)(inject_lead == 0 ? t[MCNEGF_TALLY_EXIT_R] : t[MCNEGF_TALLY_EXIT_L]);
    if (walkers <= 0.0) {
        T[f] = 0.0;
        sig[f] = 0.0;
        return;
    }
    const double p = hits / walkers;
    T[f] = c * p;
    sig[f] = walkers > 1.0 ? c * sqrt(p * (1.0 - p) / (walkers - 1.0)) : 0.0;
}

hipError_t launch_interp_current(const mcnegf_kernel& k, const double* fine, uint32_t nF,
                                 uint32_t inject_lead, const int64_t* tallies,
                                 const double* weights, double* T, double* sigmaT,
                                 hipStream_t s) {
    {
        MCNEGF_TIMED("interp_current_kernel", s);
        hipLaunchKernelGGL(interp_current_kernel, dim3((nF + 255) / 256), dim3(256), 0, s,
                           tallies, k.lead, k.energies, (uint32_t)k.nE, fine, (int)nF,
                           inject_lead, T, sigmaT, k.status);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    {
        MCNEGF_TIMED("current_sum_kernel", s);
        hipLaunchKernelGGL(current_sum_kernel, dim3(1), dim3(256), 0, s, T, sigmaT, weights,
                           (int)nF, k.reduce, nullptr);
    }
    return hipGetLastError();
}

// Energies drawn with probability w_k / W (W = sum_k w_k, Sec. II F step 2 with h = w / W)
// and the estimator of the linear-response transmission with h proportional to the weight
// (Sec. II G, Eq. (66) read with f -> w): X = W c_p(E_k) for an exit at q, else 0, so that
// E[X] = sum_k w_k T_k.  Over the N walkers of the tallies: I = W S1 / N with
// S1 = sum_k c_k R_k (R_k exits at q), and sigma_I^2 = (W^2 S2 / N - I^2) / (N - 1) with
// S2 = sum_k c_k^2 R_k (the sample variance of X over N).  T_k and sigma_k are the per-energy
// ratios as in MC mode.  out[0] = I, out[1] = sigma_I^2.
__global__ void __launch_bounds__(256) sampled_current_kernel(const int64_t* __restrict__ tallies,
                                                              const double* __restrict__ lead,
                                                              const double* __restrict__ w,
                                                              int nE, uint32_t inject_lead,
                                                              double* __restrict__ T,
                                                              double* __restrict__ sig,
                                                              double* __restrict__ out) {
    __shared__ double red[256];
    double sw = 0.0, s1 = 0.0, s2 = 0.0, nw = 0.0;
    for (int k = threadIdx.x; k < nE; k += 256) {
        const int64_t* t = tallies + (size_t)k * MCNEGF_TALLY_N;
        const double walkers =
            (double)(t[MCNEGF_TALLY_EXIT_L] + t[MCNEGF_TALLY_EXIT_R] + t[MCNEGF_TALLY_TRUNC]);
        const double hits =
            (double)(inject_lead == 0 ? t[MCNEGF_TALLY_EXIT_R] : t[MCNEGF_TALLY_EXIT_L]);
        const double c = lead[(size_t)k * MCNEGF_LEAD_NTERMS +
                              (inject_lead == 0 ? MCNEGF_LEAD_CL : MCNEGF_LEAD_CR)];
        sw += w[k];
        s1 += c * hits;
        s2 += c * c * hits;
        nw += walkers;
        const double p = walkers > 0.0 ? hits / walkers : 0.0;
        T[k] = c * p;
        sig[k] = walkers > 1.0 ? c * sqrt(p * (1.0 - p) / (walkers - 1.0)) : 0.0;
    }
    sw = block_reduce256(sw, red);
    s1 = block_reduce256(s1, red);
    s2 = block_reduce256(s2, red);
    nw = block_reduce256(nw, red);
    if (threadIdx.x == 0) {
        const double I = nw > 0.0 ? sw * s1 / nw : 0.0;
        const double m2 = nw > 0.0 ? sw * sw * s2 / nw : 0.0;
        const double var = nw > 1.0 ? (m2 - I * I) / (nw - 1.0) : 0.0;
        out[0] = I;
        out[1] = var > 0.0 ? var : 0.0;
    }
}

hipError_t launch_sampled_current(const mcnegf_kernel& k, uint32_t inject_lead,
                                  const int64_t* tallies, const double* weights, double* T,
                                  double* sigmaT, hipStream_t s) {
    {
        MCNEGF_TIMED("sampled_current_kernel", s);
        hipLaunchKernelGGL(sampled_current_kernel, dim3(1), dim3(256), 0, s, tallies, k.lead,
                           weights, k.nE, inject_lead, T, sigmaT, k.reduce);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- DIRECT
// vec layout per energy: [0] u_j = gamma_j s_j, [1] u_j w_p(j), [2] u_j w_q(j), [3] s_j,
// with s_j = M_jj^{-1/2} (0 for a decoupled probe) and w_p, w_q the exit weights of the
// injecting and the collecting lead.  Scaled matrix: 1 on the diagonal, -u_i u_j |G_ij|^2 off it;
// scaled right-hand sides: u_j w_p(j) and u_j w_q(j).
__global__ void direct_prep_kernel(const double* __restrict__ P, const double* __restrict__ Adiag,
                                   const double* __restrict__ wL, const double* __restrict__ wR,
                                   const double* __restrict__ gamma, int N, int64_t ldP,
                                   uint32_t inject_lead, double* __restrict__ vec) {
    const int e = blockIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= N) return;
    const double g = gamma[j];
    const double Pjj = P[((size_t)e * N + j) * ldP + j];
    const double mjj = g * Adiag[(size_t)e * N + j] - g * g * Pjj;
    const double sj = (g > 0.0 && mjj > 0.0) ? 1.0 / sqrt(mjj) : 0.0;
    const double wp = inject_lead == 0 ? wL[(size_t)e * N + j] : wR[(size_t)e * N + j];
    const double wq = inject_lead == 0 ? wR[(size_t)e * N + j] : wL[(size_t)e * N + j];
    const double u = g * sj;
    double* v = vec + (size_t)e * 4 * N;
    v[j] = u;
    v[N + j] = u * wp;
    v[2 * N + j] = u * wq;
    v[3 * N + j] = sj;
}

// ---- Recursive blocked Cholesky of the bordered probe system on FP64 matrix cores.
//
// Per energy, logical rows 0..Np-1 are the scaled matrix padded with identity rows up to
// Np = round_up(N, 16), rows Np and Np+1 are the two scaled right-hand sides; columns
// 0..Np-1 are factored in panels of 128 columns.  Panel J (first column c0 = 128 J), all
// energies of a launch together:
//   factor  L_JJ = chol(V_JJ) and the inverses Z_b of its 16 x 16 diagonal sub-blocks,
//           one workgroup per energy (the last panel's two bordered rows included);
//   solve   L[below, J] = V[below, J] L_JJ^{-T};
//   update  with m the largest power of two that divides J + 1, the next m panels get the
//           contribution of the last m: V[i, j] -= sum_k L[i, k] L[j, k] over the 128 m
//           columns k before column c1 = 128 (J + 1), for j in [c1, c1 + 128 m) and rows i >= j.
//           m = 1 (odd panels) has no launch: the next factor and solve take that product.
// The powers of two are the recursion V_22 - L_21 L_21^T by halves: each entry is read and
// written once per set bit of its panel's index instead of once per panel, the products'
// inner lengths are as long as their outer ones (a left-looking panel has few tiles of full
// length at the end, a right-looking one a whole pass over the matrix per panel), and every
// update has rows / 128 x m tiles per energy, enough to fill the chip with few energies.
// Panel j >= 2 is first touched by the update with J + 1 = m, which reads the matrix itself
// (panels 0 and 1 by their factor and solve).
// The launch boundaries order the steps; no workgroup waits for another.
// Measured against one workgroup per energy going left-looking through 64-column panels (split
// over workgroups by panel rows with few energies), ms per factorization:
//   N = 16000, 8 energies    418 -> 171  (64 TFLOP/s)     N = 4000, 64 energies   39.4 -> 26.2
//   N = 3200, 128 energies  35.3 -> 28.2                  N = 1000, 256 energies  2.85 -> 2.36
// (the split formed each diagonal block, a product over all previous columns, in every
// workgroup, and the factor's serial chain of pivots took 24 us per 64 columns).
//
// v_mfma_f64_16x16x4f64 operand layouts (lane l, g = l / 16, n = l % 16):
//   A[m][k]: m = n, k = g;   B[k][c]: k = g, c = n;   D[i][c] (item r): i = 4 r + g, c = n.
// Column rows are the A operand and tile rows the B operand, so an accumulator holds the
// transposed block: lane (n, g) has row n, columns 4 r + g, which is the B operand of the
// next product.  Rows of L are stored with the columns of every 16-column block permuted so
// that these four items are contiguous (logical column 4 r + g at position 4 g + r, an
// involution): the update contracts over stored positions of two rows of L, which any common
// column permutation leaves unchanged, and the two bordered rows enter only through their dot
// product, which it leaves unchanged too.
typedef double dmfma4 __attribute__((ext_vector_type(4)));
typedef double dmfma4u __attribute__((ext_vector_type(4), aligned(8)));  // four of any row
typedef double dvec2 __attribute__((ext_vector_type(2)));

constexpr int CH_NB = 128;            // panel width
constexpr int CH_SB = CH_NB / 16;     // 16-column sub-blocks of a panel
constexpr int CH_NBLK = CH_SB * (CH_SB + 1) / 2;
constexpr int CH_WAVES = 8;           // wavefronts of the factor and solve workgroups

struct CholArgs {
    const double* P;      // [nE][N][ld] |G_ij|^2
    const double* vec;    // [nE][4][N]
    const double* lead;   // [nE][8]
    double* Lall;         // [nE][Np + 2][ld]
    double* T;
    double* sig;
    uint32_t* status;
    int N, Np;
    int64_t ld;
    uint32_t inject_lead;
    int nE;
    int J;      // panel
    int m;      // update: panels per side
    int tiles;  // solve: workgroups per energy; update: tiles per energy
    int rows;   // solve: 16-row tiles per wavefront
};

// The factored matrix takes the sites of every 16-site block in the order of the involution
// 4 r + g <-> 4 g + r (rows and columns alike), so that the four columns 4 r + g of a lane are
// four consecutive sites, one 32-byte load of a row of P.
__device__ inline int ch_site(int i) { return (i & ~15) + 4 * (i & 3) + ((i >> 2) & 3); }

// Entries (i, cb + 4 r + g), r = 0..3, of the bordered scaled matrix (cb a multiple of 16).
__device__ inline dmfma4 aorig4(const CholArgs& a, const double* Pe, const double* ve, int i,
                                int cb, int g) {
    const int N = a.N;
    const int j = cb + 4 * g;  // the first of the four sites
    dmfma4 out = dmfma4{0.0, 0.0, 0.0, 0.0};
    if (i < a.Np) {
        const int si = ch_site(i);
        if (si < N) {
            const double4 p = *reinterpret_cast<const double4*>(Pe + (size_t)si * a.ld + j);
            const dmfma4 pv = dmfma4{p.x, p.y, p.z, p.w};
            const double ui = ve[si];
            // beyond N the other vectors of this energy are read and not used; with fewer than
            // four sites those end before the padded columns do
            const double* uj = ve + min(j, 4 * N - 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) out[r] = j + r < N ? -ui * uj[r] * pv[r] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = j + r == si ? 1.0 : out[r];
    } else if (i < a.Np + 2) {
        const double* rhs = ve + (size_t)(i - a.Np + 1) * N;
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = j + r < N ? rhs[j + r] : 0.0;
    }
    return out;
}

__device__ inline dmfma4 load4(const double* p) {
    const double4 v = *reinterpret_cast<const double4*>(p);
    return dmfma4{v.x, v.y, v.z, v.w};
}
__device__ inline void store4(double* p, dmfma4 v) {
    *reinterpret_cast<double4*>(p) = double4{v[0], v[1], v[2], v[3]};
}

// c + A B for 16 x 16 blocks: one operand item per K-step.
__device__ inline dmfma4 mfma16(dmfma4 a, dmfma4 b, dmfma4 c) {
#pragma unroll
    for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b[r], c, 0, 0, 0);
    return c;
}

// The lower 16 x 16 sub-blocks (mb, kb) of a panel's diagonal block in LDS, without padding:
// row n keeps its four 32-byte chunks (the columns 4 r + g of lane group g) rotated by n / 2,
// which spreads the eight lanes of a 16-byte read over all banks.  The LDS address space is
// carried in the type so that every access is a DS instruction.
typedef __attribute__((address_space(3))) double lds_double;
__device__ inline int ch_blk(int mb, int kb) { return (mb * (mb + 1) / 2 + kb) * 256; }
__device__ inline int ch_at(int n, int g) { return n * 16 + 4 * ((g + (n >> 1)) & 3); }
__device__ inline dmfma4 lds_load4(const lds_double* p) { return dmfma4{p[0], p[1], p[2], p[3]}; }
__device__ inline void lds_store4(lds_double* p, dmfma4 v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = v[r];
}

// Forward substitution of one 16-row tile with the panel in LDS (Z_b in the diagonal
// sub-blocks): y[b], block b of the tile's transposed rows, becomes block b of L.
__device__ inline void panel_solve(const lds_double* S, dmfma4 (&y)[CH_SB], int nsb, int n, int g) {
    const int at = ch_at(n, g);
#pragma unroll
    for (int kb = 0; kb < CH_SB; ++kb) {
        if (kb < nsb) {
            const dmfma4 x =
                mfma16(lds_load4(S + ch_blk(kb, kb) + at), y[kb], dmfma4{0.0, 0.0, 0.0, 0.0});
            y[kb] = x;
            const dmfma4 xn = -x;
#pragma unroll
            for (int mb = kb + 1; mb < CH_SB; ++mb)
                if (mb < nsb) y[mb] = mfma16(lds_load4(S + ch_blk(mb, kb) + at), xn, y[mb]);
        }
    }
}

// Position of Z_b among the unused upper sub-blocks of a full diagonal block.
__device__ inline void z_home(int b, int& rb, int& cb) {
    rb = b < CH_SB - 1 ? 0 : 1;
    cb = b < CH_SB - 1 ? b + 1 : 2;
}

// Lane N of every row of 16 lanes, in all of them (one DPP move, no scalar registers).
template <int N>
__device__ inline double bcast16(double v) {
    return __builtin_amdgcn_update_dpp(v, v, 0x150 + N, 0xF, 0xF, true);  // row_newbcast
}

// Pivots K .. 15 of a 16 x 16 sub-block: lane n of each row of 16 holds row n of the
// sub-block (rw) and column n of the inverse of its factor (z).
template <int K, int J>
__device__ inline void factor_columns(double (&rw)[16], double (&z)[16], double lik) {
    if constexpr (J < 16) {
        const double ljk = bcast16<J>(lik);
        rw[J] = fma(-lik, ljk, rw[J]);
        z[J] = fma(-ljk, z[K], z[J]);
        // the updates stay with their pivot: put off, the broadcasts would pile up and spill
        asm volatile("" : "+v"(rw[J]), "+v"(z[J]));
        factor_columns<K, J + 1>(rw, z, lik);
    }
}
template <int K>
__device__ inline void factor_pivots(double (&rw)[16], double (&z)[16], int n, bool& bad) {
    if constexpr (K < 16) {
        double piv = bcast16<K>(rw[K]);
        const bool good = piv > 0.0 && isfinite(piv);
        bad |= !good;
        piv = good ? piv : 1.0;
        // one reciprocal square root and products: a shorter dependent chain per pivot than a
        // square root followed by divisions
        const double rs = rsqrt(piv);
        const double lik = n >= K ? rw[K] * rs : 0.0;
        rw[K] = lik;
        z[K] *= rs;
        factor_columns<K, K + 1>(rw, z, lik);
        factor_pivots<K + 1>(rw, z, n, bad);
    }
}

// Cholesky factor of the diagonal block of panel J, one workgroup per energy.  Bound by the
// serial chain of 128 pivots: wavefront 0 factors the 16 x 16 sub-blocks (lane per row, the
// pivot column's entries by DPP broadcasts, which also feed the inverse's columns) while the
// other wavefronts apply the previous sub-block's products to the rest.
__global__ void __launch_bounds__(64 * CH_WAVES) cholesky_factor_kernel(CholArgs a) {
    __shared__ double S_raw[CH_NBLK * 256];
    lds_double* S = (lds_double*)S_raw;
    const int e = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int at = ch_at(n, g);
    const int R = a.Np + 2;
    const int64_t ld = a.ld;
    const int c0 = a.J * CH_NB;
    const int nsb = min(CH_SB, (a.Np - c0) >> 4);
    const bool last = c0 + CH_NB >= a.Np;
    const double* Pe = a.P + (size_t)e * a.N * ld;
    const double* ve = a.vec + (size_t)e * 4 * a.N;
    double* Le = a.Lall + (size_t)e * R * ld;
    double* Ld = Le + (size_t)c0 * ld + c0;
    for (int q = wave; q < CH_NBLK; q += CH_WAVES) {
        int mb = 0;
        while ((mb + 1) * (mb + 2) / 2 <= q) ++mb;
        const int kb = q - mb * (mb + 1) / 2;
        if (mb < nsb) {
            dmfma4 v = a.J <= 1 ? aorig4(a, Pe, ve, c0 + 16 * mb + n, c0 + 16 * kb, g)
                                : load4(Ld + (size_t)(16 * mb + n) * ld + 16 * kb + 4 * g);
            if (a.J & 1) {
                const double* xr = Ld + (size_t)(16 * mb + n) * ld + 4 * g - CH_NB;
                const double* xc = Ld + (size_t)(16 * kb + n) * ld + 4 * g - CH_NB;
                dmfma4 acc = dmfma4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < CH_SB; ++k) acc = mfma16(load4(xc + 16 * k), load4(xr + 16 * k), acc);
                v -= acc;
            }
            lds_store4(S + q * 256 + at, v);
        }
    }
    __syncthreads();
    bool bad = false;
    for (int b = 0; b < nsb; ++b) {
        if (wave == 0) {
            lds_double* D = S + ch_blk(b, b);
            if (b > 0) {  // the last product of this sub-block, then its factor
                const dmfma4 x = lds_load4(S + ch_blk(b, b - 1) + at);
                lds_store4(D + at, mfma16(x, -x, lds_load4(D + at)));
            }
            // lane n (and its copies n + 16 g) holds row n of the sub-block and column n of
            // the inverse
            double rw[16], z[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                rw[j] = D[ch_at(n, j & 3) + (j >> 2)];
                z[j] = j == n ? 1.0 : 0.0;
            }
            factor_pivots<0>(rw, z, n, bad);
            if (lane < 16) {
                double* Lg = Ld + (size_t)(16 * b + n) * ld + 16 * b;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    if (j <= n) Lg[4 * (j & 3) + (j >> 2)] = rw[j];
                    D[ch_at(j, n & 3) + (n >> 2)] = z[j];  // Z[j][n]
                }
            }
            if (!last) {  // Z_b for the solve launch
                int rb, cb;
                z_home(b, rb, cb);
                store4(Ld + (size_t)(16 * rb + n) * ld + 16 * cb + 4 * g, lds_load4(D + at));
            }
        } else if (b > 0) {
            // products of sub-block column b - 1 with the rest of the block
            const int q = nsb - b;  // rows and columns b .. nsb - 1, without (b, b)
            for (int t = wave; t < q * (q + 1) / 2; t += CH_WAVES - 1) {
                int tb = 0;
                while ((tb + 1) * (tb + 2) / 2 <= t) ++tb;
                const int cb = t - tb * (tb + 1) / 2;
                lds_double* V = S + ch_blk(b + tb, b + cb) + at;
                const dmfma4 xc = lds_load4(S + ch_blk(b + cb, b - 1) + at);
                const dmfma4 xt = lds_load4(S + ch_blk(b + tb, b - 1) + at);
                lds_store4(V, mfma16(xc, -xt, lds_load4(V)));
            }
        }
        __syncthreads();
        // the sub-blocks below the factored one
        for (int mb = b + 1 + wave; mb < nsb; mb += CH_WAVES) {
            lds_double* V = S + ch_blk(mb, b) + at;
            const dmfma4 x = mfma16(lds_load4(S + ch_blk(b, b) + at), lds_load4(V),
                                    dmfma4{0.0, 0.0, 0.0, 0.0});
            lds_store4(V, x);
            store4(Ld + (size_t)(16 * mb + n) * ld + 16 * b + 4 * g, x);
        }
        __syncthreads();
    }
    if (bad && threadIdx.x == 0) atomicOr(a.status, MCNEGF_FLAG_NOTSPD);
    if (last && wave == 0) {  // the two bordered rows
        const int row = a.Np + (n & 1);
        dmfma4 y[CH_SB];
#pragma unroll
        for (int kb = 0; kb < CH_SB; ++kb) {
            y[kb] = dmfma4{0.0, 0.0, 0.0, 0.0};
            if (kb < nsb) {
                y[kb] = a.J <= 1 ? aorig4(a, Pe, ve, row, c0 + 16 * kb, g)
                                 : load4(Le + (size_t)row * ld + c0 + 16 * kb + 4 * g);
                if (a.J & 1) {
                    const double* xr = Le + (size_t)row * ld + c0 + 4 * g - CH_NB;
                    const double* xc = Ld + (size_t)(16 * kb + n) * ld + 4 * g - CH_NB;
                    dmfma4 acc = dmfma4{0.0, 0.0, 0.0, 0.0};
                    for (int k = 0; k < CH_SB; ++k) acc = mfma16(load4(xc + 16 * k), load4(xr + 16 * k), acc);
                    y[kb] -= acc;
                }
            }
        }
        panel_solve(S, y, nsb, n, g);
#pragma unroll
        for (int kb = 0; kb < CH_SB; ++kb)
            if (kb < nsb && n < 2) store4(Le + (size_t)row * ld + c0 + 16 * kb + 4 * g, y[kb]);
    }
}

// Work index of a workgroup: consecutive workgroups are dealt to the eight XCDs in turn, so
// each XCD takes one contiguous eighth of the (energy, tile) list and its L2 serves the rows
// that neighbouring tiles share.  The grid is 8 x ceil(total / 8).
__device__ inline int xcd_contiguous(int total) {
    return (blockIdx.x & 7) * ((total + 7) >> 3) + (blockIdx.x >> 3);
}

// Rows below a full panel: V L_JJ^{-T}, two 16-row tiles per wavefront at a time, `rows` times.
// An odd panel (UPD) first takes the product with the previous panel's 128 columns: its rows
// and the panel's come from L2, and V is read once instead of being written by a launch of its
// own and read again.  The steps of a tile are a serial chain of products, so its reads are what
// can be hidden: V's entries are loaded a tile ahead and before the stores of the tile at hand,
// the product's operands a block column ahead (N = 1000, 256 energies: the seven launches
// 1022 -> 809 us, the first 240 -> 152 us at 3.0 TB/s).
constexpr int CH_SOLVE_WAVES = 4;
constexpr int CH_SOLVE_ROWS = 32 * CH_SOLVE_WAVES;  // rows per workgroup and pass

template <bool UPD>
__global__ void __launch_bounds__(64 * CH_SOLVE_WAVES, 2) cholesky_solve_kernel(CholArgs a) {
    __shared__ double S_raw[CH_NBLK * 256 + CH_NB];
    lds_double* S = (lds_double*)S_raw;
    lds_double* us = S + CH_NBLK * 256;  // the scales of the panel's columns
    const int idx = xcd_contiguous(a.nE * a.tiles);
    if (idx >= a.nE * a.tiles) return;
    const int e = idx / a.tiles, part = idx - e * a.tiles;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int at = ch_at(n, g);
    const int R = a.Np + 2;
    const int64_t ld = a.ld;
    const int c0 = a.J * CH_NB;
    const double* Pe = a.P + (size_t)e * a.N * ld;
    const double* ve = a.vec + (size_t)e * 4 * a.N;
    double* Le = a.Lall + (size_t)e * R * ld;
    const double* Ld = Le + (size_t)c0 * ld + c0;
    for (int q = wave; q < CH_NBLK; q += CH_SOLVE_WAVES) {
        int mb = 0;
        while ((mb + 1) * (mb + 2) / 2 <= q) ++mb;
        int kb = q - mb * (mb + 1) / 2;
        if (kb == mb) z_home(mb, mb, kb);
        lds_store4(S + q * 256 + at, load4(Ld + (size_t)(16 * mb + n) * ld + 16 * kb + 4 * g));
    }
    // a full panel's columns are below N, and no row below it meets the diagonal there: an entry is
    // one of V's (J >= 2), a scaled one of P or one of a bordered row, 32 bytes of one row each way
    const bool orig = a.J <= 1;
    if (threadIdx.x < CH_NB) us[threadIdx.x] = orig ? ve[c0 + threadIdx.x] : 0.0;
    __syncthreads();
    auto load_v = [&](dmfma4 (&v)[CH_SB], double& ui, int row) {
        const int i = min(row + n, R - 1);
        const int si = min(ch_site(i), a.N - 1);
        const double* src = !orig ? Le + (size_t)i * ld
                            : i < a.Np ? Pe + (size_t)si * ld : ve + (size_t)(i - a.Np + 1) * a.N;
        src += c0 + 4 * g;
        ui = ve[si];
#pragma unroll
        for (int kb = 0; kb < CH_SB; ++kb) {
            const dmfma4u x = *reinterpret_cast<const dmfma4u*>(src + 16 * kb);
            v[kb] = dmfma4{x[0], x[1], x[2], x[3]};
        }
    };
    auto entry = [&](dmfma4 v, double ui, int row, int kb) {
        const int i = min(row + n, R - 1);
        if (!orig || i >= a.Np) return v;
        const dmfma4 uj = lds_load4(us + 16 * kb + 4 * g);
        dmfma4 out;
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = ch_site(i) < a.N ? -ui * uj[r] * v[r] : 0.0;
        return out;
    };
    const int pass = CH_SOLVE_ROWS;
    const int first = c0 + CH_NB + part * a.rows * pass + 32 * wave;
    const int last = min(first + (a.rows - 1) * pass + 32, R);
    // The loads of a tile's entries are issued before the stores of the tile before it: loads
    // and stores are counted in order, and behind the stores they would wait for those too.
    dmfma4 v[CH_SB];
    double ui = 0.0;
    if (!UPD) {
        if (first < last) load_v(v, ui, first);
        for (int row = first; row < last; row += (row - first) % pass ? pass - 16 : 16) {
            dmfma4 y[CH_SB];
#pragma unroll
            for (int kb = 0; kb < CH_SB; ++kb) y[kb] = entry(v[kb], ui, row, kb);
            __builtin_amdgcn_sched_barrier(0);
            const int next = row + ((row - first) % pass ? pass - 16 : 16);
            if (next < last) load_v(v, ui, next);
            __builtin_amdgcn_sched_barrier(0);
            panel_solve(S, y, CH_SB, n, g);
            if (row + n < R) {
                double* dst = Le + (size_t)(row + n) * ld + c0 + 4 * g;
#pragma unroll
                for (int kb = 0; kb < CH_SB; ++kb) store4(dst + 16 * kb, y[kb]);
            }
        }
        return;
    }
    for (int row0 = first; row0 < last; row0 += pass) {
        dmfma4 y[2][CH_SB];
        double* dst[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            dst[h] = Le + (size_t)min(row0 + 16 * h + n, R - 1) * ld + c0 + 4 * g;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int kb = 0; kb < CH_SB; ++kb) y[h][kb] = dmfma4{0.0, 0.0, 0.0, 0.0};
        const double* xc = Ld + (size_t)n * ld + 4 * g - CH_NB;
        // the operands of block column k + 1 take the place of those of k as they are used
        dmfma4 x0 = load4(dst[0] - CH_NB), x1 = load4(dst[1] - CH_NB);
#pragma unroll
        for (int kb = 0; kb < CH_SB; ++kb) v[kb] = load4(xc + (size_t)(16 * kb) * ld);
        for (int k = 0; k < CH_SB; ++k) {
            const int kn = 16 * min(k + 1, CH_SB - 1);
            const dmfma4 x0n = load4(dst[0] - CH_NB + kn), x1n = load4(dst[1] - CH_NB + kn);
#pragma unroll
            for (int kb = 0; kb < CH_SB; ++kb) {
                y[0][kb] = mfma16(v[kb], x0, y[0][kb]);
                y[1][kb] = mfma16(v[kb], x1, y[1][kb]);
                __builtin_amdgcn_sched_barrier(0);
                v[kb] = load4(xc + (size_t)(16 * kb) * ld + kn);
                __builtin_amdgcn_sched_barrier(0);
            }
            x0 = x0n;
            x1 = x1n;
        }
        load_v(v, ui, row0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int kb = 0; kb < CH_SB; ++kb)
                y[h][kb] = entry(v[kb], ui, row0 + 16 * h, kb) - y[h][kb];
            __builtin_amdgcn_sched_barrier(0);
            if (h == 0) load_v(v, ui, row0 + 16);
            __builtin_amdgcn_sched_barrier(0);
            panel_solve(S, y[h], CH_SB, n, g);
            if (row0 + 16 * h + n < R) {
#pragma unroll
                for (int kb = 0; kb < CH_SB; ++kb) store4(dst[h] + 16 * kb, y[h][kb]);
            }
        }
    }
}

// Update: one workgroup per tile of 32 F x 32 F entries, four wavefronts of F x F
// accumulators (16 F x 16 F entries) each.  A 16x16x4 product occupies a SIMD for 64 clocks,
// so a 128 x 128 tile, 32 products per SIMD and 8 columns, needs 16 KB of operands per 2048
// clocks: bandwidth is not short, latency is.  The 8-column steps are staged in LDS
// (double-buffered, one barrier per step) from registers loaded four steps ahead; two workgroups
// share a CU (four of 64 x 64, which need twice the operands but are less often all at their reads
// and writes of V at once; the launch takes the one that is faster).  In a step lane group g takes
// the positions 2 g, 2 g + 1 of both operands (the same permutation of the contracted columns on
// both sides); a staged row is 64 bytes, its 16-byte pieces swizzled by the row so that eight rows
// spread over all banks.
template <int F>
__global__ void __launch_bounds__(256, F == 4 ? 2 : 4) cholesky_update_kernel(CholArgs a) {
    constexpr int TS = 32 * F;  // tile side
    __shared__ double X[2][2 * TS * 8];
    const int idx = xcd_contiguous(a.nE * a.tiles);
    if (idx >= a.nE * a.tiles) return;
    const int e = idx / a.tiles;
    int t = idx - e * a.tiles;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int Np = a.Np, R = Np + 2;
    const int64_t ld = a.ld;
    const int c1 = (a.J + 1) * CH_NB;
    const int wide = min(a.m * CH_NB, Np - c1);  // columns of the update
    const int nct = (wide + TS - 1) / TS, nrt = (R - c1 + TS - 1) / TS;
    // tiles in groups of eight tile columns, row by row within a group (tile row >= tile
    // column): the tiles that run together share their rows
    int g0 = 0, ct = 0, rt = 0;
    for (; g0 < nct; g0 += 8) {
        const int w = min(8, nct - g0);
        // rows g0 .. g0 + w - 1 hold 1 .. w tiles, the rest w
        const int tri = w * (w + 1) / 2;
        const int cnt = tri + (nrt - g0 - w) * w;
        if (t >= cnt) {
            t -= cnt;
            continue;
        }
        if (t < tri) {
            int q = 0;
            while ((q + 1) * (q + 2) / 2 <= t) ++q;
            rt = g0 + q;
            ct = g0 + t - q * (q + 1) / 2;
        } else {
            rt = g0 + w + (t - tri) / w;
            ct = g0 + (t - tri) % w;
        }
        break;
    }
    const int i0 = c1 + rt * TS + (wave & 1) * 16 * F;   // this wavefront's rows
    const int j0 = c1 + ct * TS + (wave >> 1) * 16 * F;  // and columns
    // a wavefront above the diagonal or outside the matrix stages and multiplies for nothing
    const bool on = i0 + 16 * F > j0 && i0 < R && j0 < c1 + wide;
    double* Le = a.Lall + (size_t)e * R * ld;
    // [row tile][column block].  The products are summed by themselves and subtracted once: added
    // one by one to entries near 1 the small ones would be lost, always on the same side
    dmfma4 acc[F][F];
#pragma unroll
    for (int tb = 0; tb < F; ++tb)
#pragma unroll
        for (int cb = 0; cb < F; ++cb) acc[tb][cb] = dmfma4{0.0, 0.0, 0.0, 0.0};
    const int K = a.m * CH_NB;
    const char* base = reinterpret_cast<const char*>(Le + (c1 - K));
    // staging: thread (r, q) = (tid / 4, tid % 4) copies piece q of the tile's rows r + 64 u and
    // (u >= F / 2) of its columns' rows; byte offsets of one energy's factor are below 2^32
    const int sr = threadIdx.x >> 2, sq = threadIdx.x & 3;
    uint32_t off[F];
#pragma unroll
    for (int u = 0; u < F; ++u) {
        const int row = (u < F / 2 ? c1 + rt * TS + 64 * u : c1 + ct * TS + 64 * (u - F / 2)) + sr;
        off[u] = (uint32_t)((size_t)min(row, R - 1) * ld * 8) + 16u * (sq ^ ((sr >> 2) & 3));
    }
    dvec2 s0[F], s1[F];
    auto load = [&](dvec2 (&st)[F], int k) {
        const char* b = base + (size_t)k * 64;
#pragma unroll
        for (int u = 0; u < F; ++u) st[u] = *reinterpret_cast<const dvec2*>(b + off[u]);
    };
    auto put = [&](const dvec2 (&st)[F], int buf) {
#pragma unroll
        for (int u = 0; u < F; ++u)
            *reinterpret_cast<dvec2*>(&X[buf][(64 * u + sr) * 8 + 2 * sq]) = st[u];
    };
    const int piece = 2 * (g ^ ((n >> 2) & 3));
    const int xi = ((wave & 1) * 16 * F + n) * 8 + piece;
    const int xj = (TS + (wave >> 1) * 16 * F + n) * 8 + piece;
    auto take = [&](dvec2 (&v)[2 * F], int buf) {
#pragma unroll
        for (int q = 0; q < F; ++q) {
            v[q] = *reinterpret_cast<const dvec2*>(&X[buf][xi + 128 * q]);
            v[F + q] = *reinterpret_cast<const dvec2*>(&X[buf][xj + 128 * q]);
        }
    };
    auto mult = [&](const dvec2 (&v)[2 * F]) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int tb = 0; tb < F; ++tb)
#pragma unroll
                for (int cb = 0; cb < F; ++cb)
                    acc[tb][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[F + cb][r], v[tb][r],
                                                                       acc[tb][cb], 0, 0, 0);
    };
    // While step k is multiplied from registers, step k + 1 is read from its buffer, step k + 2
    // written to the other one and step k + 4 loaded, so a wavefront has its next products
    // ready when it leaves the barrier.  Loads past the end re-read the last step, unused.
    // The scheduling barriers keep the memory accesses ahead of the products.
    const int nk = K / 8;  // a multiple of 32
    dvec2 fa[2 * F], fb[2 * F];
    load(s0, 0);
    load(s1, 1);
    __builtin_amdgcn_sched_barrier(0);
    put(s0, 0);
    load(s0, 2);
    __builtin_amdgcn_sched_barrier(0);
    put(s1, 1);
    load(s1, 3);
    __syncthreads();
    take(fa, 0);
    __syncthreads();
    for (int k = 0; k < nk; k += 2) {
        take(fb, 1);
        put(s0, 0);
        load(s0, min(k + 4, nk - 1));
        __builtin_amdgcn_sched_barrier(0);
        mult(fa);
        __syncthreads();
        take(fa, 0);
        put(s1, 1);
        load(s1, min(k + 5, nk - 1));
        __builtin_amdgcn_sched_barrier(0);
        mult(fb);
        __syncthreads();
    }
    if (!on) return;
    const bool first = a.J + 1 == a.m;
    const double* Pe = a.P + (size_t)e * a.N * ld;
    const double* ve = a.vec + (size_t)e * 4 * a.N;
    // one row of blocks is loaded before the one ahead of it is stored (loads behind stores wait
    // for them)
    dmfma4 v[2][F];
    auto load_row = [&](int tb) {
        const int row = min(i0 + 16 * tb + n, R - 1);
#pragma unroll
        for (int cb = 0; cb < F; ++cb) {
            const int col = min(j0 + 16 * cb, Np - 16);
            v[tb & 1][cb] = first ? aorig4(a, Pe, ve, row, col, g)
                                  : load4(Le + (size_t)row * ld + col + 4 * g);
        }
    };
    load_row(0);
#pragma unroll
    for (int tb = 0; tb < F; ++tb) {
        if (tb + 1 < F) load_row(tb + 1);
        __builtin_amdgcn_sched_barrier(0);
        const int row = i0 + 16 * tb + n;
#pragma unroll
        for (int cb = 0; cb < F; ++cb) {
            const int col = j0 + 16 * cb;
            if (row < R && col < Np)
                store4(Le + (size_t)row * ld + col + 4 * g, v[tb & 1][cb] - acc[tb][cb]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// T_k = T_qp + (row Np of L) . (row Np + 1 of L) after a factorization in several launches
// (fixed-order sum; both rows carry the same column permutation).
__global__ void __launch_bounds__(256) direct_dot_kernel(CholArgs a) {
    __shared__ double red[256];
    const int e = blockIdx.x;
    const int Np = a.Np;
    const double* Le = a.Lall + (size_t)e * (Np + 2) * a.ld;
    const double* y = Le + (size_t)Np * a.ld;
    const double* z = y + a.ld;
    double part = 0.0;
    for (int j = threadIdx.x; j < Np; j += 256) part = fma(y[j], z[j], part);
    const double dot = block_reduce256(part, red);
    if (threadIdx.x == 0) {
        const double* ld_ = a.lead + (size_t)e * MCNEGF_LEAD_NTERMS;
        const double tqp = a.inject_lead == 0 ? ld_[MCNEGF_LEAD_TRL] : ld_[MCNEGF_LEAD_TLR];
        const double Tk = tqp + dot;
        a.T[e] = Tk;
        a.sig[e] = 0.0;
        if (!isfinite(Tk)) atomicOr(a.status, MCNEGF_FLAG_NONFINITE);
    }
}

// d_I_sigma[0] = I, d_I_sigma[1] = sqrt(sum_k w_k^2 sigma_k^2), from the weighted sums.
__global__ void current_out_kernel(const double* __restrict__ reduce, double* __restrict__ out) {
    if (threadIdx.x == 0) {
        out[0] = reduce[0];
        out[1] = sqrt(reduce[1] > 0.0 ? reduce[1] : 0.0);
    }
}

hipError_t launch_current_out(const mcnegf_kernel& k, double* d_I_sigma, hipStream_t s) {
    {
        MCNEGF_TIMED("current_out_kernel", s);
        hipLaunchKernelGGL(current_out_kernel, dim3(1), dim3(64), 0, s, k.reduce, d_I_sigma);
    }
    return hipGetLastError();
}

// The factorization's launches, under one timer record.
static hipError_t factorize(CholArgs a, int cus, hipStream_t s) {
    MCNEGF_TIMED("cholesky_kernel", s);
    const int R = a.Np + 2;
    const int nJ = (a.Np + CH_NB - 1) / CH_NB;
    auto grid = [&] { return dim3(8u * (unsigned)(((int64_t)a.nE * a.tiles + 7) / 8)); };
    hipError_t err;
    for (int J = 0; J < nJ; ++J) {
        a.J = J;
        hipLaunchKernelGGL(cholesky_factor_kernel, dim3(a.nE), dim3(64 * CH_WAVES), 0, s, a);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        if (J + 1 == nJ) break;
        // solve: at most about two workgroups per CU (each loads the whole panel block)
        const int below = (R - (J + 1) * CH_NB + CH_SOLVE_ROWS - 1) / CH_SOLVE_ROWS;
        const int per = std::min(std::max(2 * cus / a.nE, 1), below);
        a.rows = (below + per - 1) / per;
        a.tiles = (below + a.rows - 1) / a.rows;
        const dim3 block(64 * CH_SOLVE_WAVES);
        if (J & 1) hipLaunchKernelGGL(cholesky_solve_kernel<true>, grid(), block, 0, s, a);
        else hipLaunchKernelGGL(cholesky_solve_kernel<false>, grid(), block, 0, s, a);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        if ((J & 1) == 0) continue;
        // update of the next m panels.  Tiles of 64 x 64 leave four workgroups on a CU whose
        // reads and writes of V overlap the others' products: with K = 128 m = 256 or 512
        // columns they are ahead of 128 x 128 (N = 1000, 256 energies: 561 -> 481 and 800 ->
        // 675 us).  From K = 1024 the larger tiles multiply 4 .. 7 % faster (N = 16000, 8
        // energies, K = 2048: 13.8 -> 12.6 ms) unless their rounded edges cost more than that
        // (N = 4000, 64 energies, K = 2048: 8.1 ms with 64, 8.8 with 128) or they are too few.
        a.m = (J + 1) & -(J + 1);
        const int c1 = (J + 1) * CH_NB;
        const int wide = std::min(a.m * CH_NB, a.Np - c1);
        auto tiles = [&](int side) {
            const int nct = (wide + side - 1) / side, nrt = (R - c1 + side - 1) / side;
            return nct * (nct + 1) / 2 + (nrt - nct) * nct;
        };
        const int64_t t128 = tiles(128), t64 = tiles(64);
        const bool big = a.m >= 8 && t128 * a.nE >= cus && 100 * t128 <= 26 * t64;
        a.tiles = (int)(big ? t128 : t64);
        if (big) hipLaunchKernelGGL(cholesky_update_kernel<4>, grid(), dim3(256), 0, s, a);
        else hipLaunchKernelGGL(cholesky_update_kernel<2>, grid(), dim3(256), 0, s, a);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    return hipSuccess;
}

hipError_t launch_direct_current(const mcnegf_kernel& k, uint32_t inject_lead,
                                 const double* weights, double* T, double* sigmaT,
                                 double* I_sigma, hipStream_t s) {
    const int N = k.N;
    {
        MCNEGF_TIMED("direct_prep_kernel", s);
        hipLaunchKernelGGL(direct_prep_kernel, dim3((N + 255) / 256, k.nE), dim3(256), 0, s, k.P,
                           k.Adiag, k.wL, k.wR, k.gamma, N, k.p_pitch, inject_lead, k.direct_vec);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    CholArgs a;
    a.P = k.P;
    a.vec = k.direct_vec;
    a.lead = k.lead;
    a.Lall = k.direct;
    a.T = T;
    a.sig = sigmaT;
    a.status = k.status;
    a.N = N;
    a.Np = (int)k.p_pitch;
    a.ld = k.p_pitch;
    a.inject_lead = inject_lead;
    a.nE = k.nE;
    int dev = 0, cus = 0;
    if ((err = hipGetDevice(&dev)) != hipSuccess) return err;
    if ((err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
        hipSuccess)
        return err;
    if ((err = factorize(a, cus, s)) != hipSuccess) return err;
    {
        MCNEGF_TIMED("direct_dot_kernel", s);
        hipLaunchKernelGGL(direct_dot_kernel, dim3(k.nE), dim3(256), 0, s, a);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
    {
        MCNEGF_TIMED("current_sum_kernel", s);
        hipLaunchKernelGGL(current_sum_kernel, dim3(1), dim3(256), 0, s, T, sigmaT, weights, k.nE,
                           k.reduce, I_sigma);
    }
    return hipGetLastError();
}

}  // namespace mcnegf
