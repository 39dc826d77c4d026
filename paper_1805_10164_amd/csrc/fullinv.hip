// All blocks of G^r from the RGF blocks, streamed straight into the walker's weights.
//
// For a column l (slice of the column), the blocks of G obey (E - H - Sigma) G = I with
// off-diagonal blocks t I, which below the diagonal gives
//   G_{k,l} = -t gR_k G_{k-1,l}   (k > l),
// starting from the diagonal block G_{l,l}.  G is complex symmetric (real H, symmetric lead
// self-energies), so the blocks above the diagonal are their transposes: only the lower half is
// computed, and every entry below the diagonal blocks is stored twice.  Each lane owns one
// column j of G (a workgroup is one wavefront owning 64 consecutive columns) and keeps its
// W-vector G_{k, j} in registers while the wavefront sweeps k down the wire; the W x W factors
// gR_k are the same for every lane: the wavefront stages them in LDS one slice ahead
// (double-buffered) and every lane reads the same address (a broadcast), which keeps the block
// operands off the scalar path and the texture units.  Nothing of G is written except
//   P[i][j]  = |G_ij|^2                      (probe-to-probe weights, step 6', Eq. (75)),
//   wL[j]    = <psi_j|Gamma_L|psi_j>, wR[j]  (psi_j = G|j>, exit weights, Eq. (76)),
//   corner   = G_{L-1,0} and G_{0,L-1}       (lead-to-lead transmissions).
// Rows of P are written by 64 lanes at consecutive columns (coalesced 512-byte segments), the
// transposed entries through LDS by whole aligned 128-byte lines (W = 10: 0.79 ms by 64-byte
// sectors, 0.99 ms by the 80 bytes of a slice).
// wL[j] needs G_{0,j}, i.e. row j of the columns of slice 0 (exit_left_chain; on the matrix
// cores the first workgroup of an energy forms them from its columns as it passes).
// Half the block products and one sweep instead of two: 0.75 -> 0.54 ms at W = 10, N = 1000,
// 256 energies (3.8 TB/s of |G|^2 written), 2.82 -> 2.32 ms over six W = 8 wires.  With few
// wavefronts the chain of slices bounds it, and a slice of the chain has become longer (the ring,
// two waits): W = 7, 61 slices, 37 energies 0.102 -> 0.106 ms, W = 1, N = 2400, 4 energies 0.51 ->
// 0.60 ms.
// The block products run on the FP64 VALU: the operands live in registers and LDS, and
// gfx950's FP64 matrix-core rate equals its FP64 FMA rate, so padding W up to a 16x16x4 MFMA
// shape would only add work.  Up to W = 27 the column and the product fit the register file (from
// W = 19 on a SIMD holds one wavefront); from W = 28 on values spill, 0.5 KB per lane at W = 31.
#include <type_traits>

#include "common.h"

namespace mcnegf {

typedef __attribute__((address_space(3))) double lds_double;

// v <- mt * M v for a W x W complex block M staged in LDS as (re, im) pairs, row-major, in the
// lanes where on is set.
template <int W>
__device__ inline void block_matvec(double2 (&v)[W], const lds_double* M, double mt, bool on) {
    double2 nv[W];
#pragma unroll
    for (int y = 0; y < W; ++y) {
        double2 acc = cmk(0.0, 0.0);
#pragma unroll
        for (int x = 0; x < W; ++x) cfma(acc, cmk(M[2 * (y * W + x)], M[2 * (y * W + x) + 1]), v[x]);
        nv[y] = cscale(acc, mt);
        // keeps the products here: sunk into a branch on `on`, they would leave the whole block
        // in registers (affordable, and faster with few wavefronts, for narrow blocks)
        if constexpr (W > 5) asm volatile("" : "+v"(nv[y].x), "+v"(nv[y].y));
    }
#pragma unroll
    for (int y = 0; y < W; ++y) v[y] = cmk(on ? nv[y].x : v[y].x, on ? nv[y].y : v[y].y);
}

// A W x W block on its way from memory to LDS by NT threads: loaded into registers one slice
// before it is written to LDS, so that the wait for the loads does not include the stores of
// the slice in between (the memory counter retires them in order).
template <int W, int NT>
struct StagedBlock {
    static constexpr int n = (W * W + NT - 1) / NT;
    typedef double dvec2 __attribute__((ext_vector_type(2)));
    dvec2 r[n];
    __device__ inline void load(const double2* __restrict__ src, int tid) {
#pragma unroll
        for (int i = 0; i < n; ++i)
            r[i] = reinterpret_cast<const dvec2*>(src)[min(tid + i * NT, W * W - 1)];
    }
    __device__ inline void write(lds_double* dst, int tid) const {
#pragma unroll
        for (int i = 0; i < n; ++i)
            if (W * W % NT == 0 || tid + i * NT < W * W) {
                dst[2 * (tid + i * NT)] = r[i].x;
                dst[2 * (tid + i * NT) + 1] = r[i].y;
            }
    }
};

// Whether the LDS of whole slices and two staged blocks would hold fewer wavefronts than the
// registers do, and cost time by it.  Then a slice goes through the ring a few rows at a time and
// one block is staged, the next waiting in registers (a wavefront's LDS accesses are in order, so
// it may overwrite a block that it has read).  |G|^2, N = 2400, 64 energies: W = 26 2.50 -> 2.01
// ms, W = 31 4.69 -> 2.73 ms, but W = 17 1.16 -> 1.27 and W = 20 1.53 -> 1.61 ms, where four to six
// wavefronts per CU fit the LDS.  Complex G, 16 energies: W = 20 1.67 -> 1.08 ms (two sweeps 1.35),
// W = 17 .. 19 1 to 2 % slower, W = 21 .. 31 equal within 2 %.
template <int W, bool STORE_G>
constexpr bool kSmallLds = W >= (STORE_G ? 20 : 26);

// Exit weights into L of one energy, on one wavefront: the columns of slice 0, X = G_{k,0} (W x W
// in LDS, lanes over its entries), go down the wire by themselves, and row y of slice k weighs
// sum_a Re conj(X_ya) (Gamma X^T)_ay.  As a chain of its own it stays off the wavefront that
// stores those columns (the longest one).
template <int W, bool ONE>
__device__ inline void exit_left_chain(lds_double* Ms, lds_double* X,
                                       const double2* __restrict__ gRe,
                                       const double2* __restrict__ Gde,
                                       const double* __restrict__ gme, int L, double mt,
                                       double* __restrict__ wLe) {
    constexpr int BS = 2 * W * W;
    constexpr int PN = (W * W + 63) / 64;  // entries per lane
    constexpr int UW = W <= 16 ? W : 4;    // unrolling of the inner products
    lds_double* terms = X + 2 * W * W;
    lds_double* Gs = X + 3 * W * W;  // (W <= 16; wider blocks read Gamma from memory)
    const int lane = threadIdx.x;
    int y[PN], a[PN];
#pragma unroll
    for (int i = 0; i < PN; ++i) {
        const int p = min(lane + 64 * i, W * W - 1);
        y[i] = p / W;
        a[i] = p - y[i] * W;
        const double2 x = Gde[p];
        X[2 * p] = x.x;
        X[2 * p + 1] = x.y;
        if constexpr (W <= 16) Gs[p] = gme[p];
    }
    StagedBlock<W, 64> st;
    st.load(gRe + (size_t)min(1, L - 1) * W * W, lane);
    for (int k = 0; k < L; ++k) {
        lds_double* M = Ms + (ONE ? 0 : (k & 1) * BS);
        st.write(M, lane);  // block k + 1
        st.load(gRe + (size_t)min(k + 2, L - 1) * W * W, lane);
        __syncthreads();  // one wavefront: orders the LDS accesses
        double2 nx[PN];
#pragma unroll
        for (int i = 0; i < PN; ++i) {
            double2 u = cmk(0.0, 0.0), acc = cmk(0.0, 0.0);
            const lds_double* xr = X + 2 * (y[i] * W);
            const lds_double* xc = X + 2 * a[i];
            const lds_double* m = M + 2 * (y[i] * W);
#pragma unroll UW
            for (int b = 0; b < W; ++b) {
                const double gab = W <= 16 ? Gs[a[i] * W + b] : gme[a[i] * W + b];
                u = cadd(u, cscale(cmk(xr[2 * b], xr[2 * b + 1]), gab));
                cfma(acc, cmk(m[2 * b], m[2 * b + 1]), cmk(xc[2 * b * W], xc[2 * b * W + 1]));
            }
            terms[y[i] * W + a[i]] = fma(xr[2 * a[i]], u.x, xr[2 * a[i] + 1] * u.y);
            nx[i] = cscale(acc, mt);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PN; ++i) {
            X[2 * (y[i] * W + a[i])] = nx[i].x;
            X[2 * (y[i] * W + a[i]) + 1] = nx[i].y;
        }
        if (lane < W) {
            double sum = 0.0;
#pragma unroll UW
            for (int b = 0; b < W; ++b) sum += terms[lane * W + b];
            wLe[k * W + lane] = sum;
        }
        __syncthreads();
    }
}

// STORE_G: write the complex blocks of G (row-major, pitch ldG, Gc) instead of |G_ij|^2,
// the exit weights and the corners.
template <int W, bool STORE_G>
__global__ void __launch_bounds__(64) fullinv_kernel(const double2* __restrict__ gR,
                                                      const double2* __restrict__ Gd,
                                                      const double* __restrict__ gam_lead,
                                                      int L, double t, int64_t ldP,
                                                      double* __restrict__ P,
                                                      double* __restrict__ wL,
                                                      double* __restrict__ wR,
                                                      double2* __restrict__ corner,
                                                      double2* __restrict__ Gc, int64_t ldG,
                                                      int nE) {
    const int N = W * L;
    // XCD-aware order: workgroups are dealt to the eight XCDs in turn (workgroup b on XCD
    // b % 8); every column tile of energy e runs on XCD e % 8, whose L2 then serves that
    // energy's RGF blocks to all its tiles.  Tile by tile over the energies, so that the long
    // tiles (the first columns) start first and are dealt evenly to the CUs.
    const int per_xcd = (nE + 7) / 8;
    const int xcd = blockIdx.x & 7, jb = blockIdx.x >> 3;
    const int e = xcd + 8 * (jb % per_xcd);
    if (e >= nE) return;  // padding of the last round (whole workgroup)
    const int lane = threadIdx.x;
    // index 0 is the chain of the exit weights into L, index t + 1 the t-th 64 columns
    const int tile = jb / per_xcd - (STORE_G ? 0 : 1);
    const int wave_first = tile * 64;
    const int col = wave_first + lane;
    const bool valid = col < N;
    const int colc = valid ? col : N - 1;
    const int l = colc / W;
    const int y0 = colc - l * W;
    const int kmin = wave_first / W;
    const size_t eb = (size_t)e * L * W * W;
    const double2* gRe = gR + eb;
    const double2* Gde = Gd + eb;
    const double* gme = gam_lead + (size_t)e * W * W;
    const double mt = -t;
    constexpr int BS = 2 * W * W;  // doubles per staged block
    constexpr bool SMALL = kSmallLds<W, STORE_G>;
    constexpr int NB = SMALL ? 1 : 2;
    __shared__ double Ms_raw[NB * BS];
    lds_double* Ms = (lds_double*)Ms_raw;
    // what is stored per entry, and a ring of rows whose transposed entries wait until FR
    // aligned rows (whole 128-byte lines of the transposed row) are there, PR rows of a slice
    // at a time
    typedef typename std::conditional<STORE_G, double2, double>::type Entry;
    constexpr int FR = 128 / sizeof(Entry);
    constexpr int PR = !SMALL ? W : STORE_G ? 4 : 8;
    constexpr int RB = FR + PR - 1;
    constexpr int CH = STORE_G ? 0 : (W <= 16 ? 4 : 3) * W * W;  // the chain's blocks (doubles)
    constexpr int RS = RB * 65 < CH ? (CH + 64) / 65 : RB;
    __shared__ Entry Tr[RS][65];
    static_assert(!SMALL || sizeof(Ms_raw) + sizeof(Tr) <= 160 * 1024 / (STORE_G && W <= 23 ? 8 : 4),
                  "the LDS holds as many wavefronts as the registers: eight, or four, per CU");
    if constexpr (!STORE_G) {
        if (tile < 0) {
            lds_double* X = (lds_double*)&Tr[0][0];
            exit_left_chain<W, SMALL>(Ms, X, gRe, Gde, gme, L, mt, wL + (size_t)e * N);
            return;  // the whole workgroup
        }
    }
    Entry* Oe = STORE_G ? (Entry*)Gc + (size_t)e * N * ldG : (Entry*)P + (size_t)e * N * ldP;
    const int64_t ldO = STORE_G ? ldG : ldP;
    const int tc = lane / FR, tr = lane % FR;  // transposed store: column and row of a pass
    int pending = (kmin * W) & ~(FR - 1);      // first row not stored transposed
    // from this row on every column of the tile is stored transposed (none: ragged last tile)
    const int below = wave_first + 64 <= N ? ((wave_first + 63) / W + 1) * W : N;
    // the column of the diagonal block, kept until the sweep has passed its slice
    double2 v[W];
#pragma unroll
    for (int y = 0; y < W; ++y) v[y] = Gde[((size_t)l * W + y) * W + y0];
    // block k + 1 (with one buffer block k) at the top of slice k; the last one again past the end
    StagedBlock<W, 64> st;
    st.load(gRe + (size_t)kmin * W * W, lane);
    if constexpr (NB == 2) {
        st.write(Ms, lane);
        st.load(gRe + (size_t)min(kmin + 1, L - 1) * W * W, lane);
    }
    for (int k = kmin; k < L; ++k) {
        __syncthreads();  // the buffer that is written next is free
        const int b = NB == 2 ? (k - kmin) & 1 : 0;
        st.write(Ms + (NB == 2 ? (b ^ 1) * BS : 0), lane);
        st.load(gRe + (size_t)min(k + NB, L - 1) * W * W, lane);
        if constexpr (NB == 1) __syncthreads();
        block_matvec<W>(v, Ms + b * BS, mt, k > l);
#pragma unroll
        for (int p = 0; p < W; p += PR) {
            const int base = (k * W + p) % RB;
#pragma unroll
            for (int y = p; y < (p + PR < W ? p + PR : W); ++y) {
                Entry o;
                if constexpr (STORE_G) o = v[y];
                else o = cabs2(v[y]);
                if (valid && k >= l) Oe[(size_t)(k * W + y) * ldO + col] = o;
                Tr[base + y - p < RB ? base + y - p : base + y - p - RB][lane] = o;
            }
            __syncthreads();  // one wavefront: orders the LDS accesses
            const int end = k * W + (p + PR < W ? p + PR : W);
            while (pending + FR <= end || (end == N && pending < end)) {
                const int r = pending + tr;
                const int at = pending % RB + tr;
                const Entry* row = Tr[at < RB ? at : at - RB];
                Entry* dst = Oe + (size_t)(wave_first + tc) * ldO + r;
                if (pending >= below && pending + FR <= end) {  // every entry is stored
#pragma unroll 8
                    for (int c = 0; c < 64; c += 64 / FR) dst[(size_t)c * ldO] = row[c + tc];
                } else {
#pragma unroll 1
                    for (int c = 0; c < 64; c += 64 / FR) {
                        const int j = wave_first + c + tc;
                        if (j < N && r < end && r >= (j / W + 1) * W)
                            dst[(size_t)c * ldO] = row[c + tc];
                    }
                }
                pending += FR;
            }
            if (p + PR < W) __syncthreads();
        }
    }
    if (STORE_G) return;
    // k = L-1 now: exit weight into R and, for the columns of slice 0, the corner blocks
    if (valid) {
        double acc = 0.0;
#pragma unroll
        for (int a = 0; a < W; ++a) {
#pragma unroll
            for (int bb = 0; bb < W; ++bb)
                acc = fma(gme[a * W + bb], v[a].x * v[bb].x + v[a].y * v[bb].y, acc);
        }
        wR[(size_t)e * N + col] = acc;
        if (l == 0) {
            double2* cRL = corner + (size_t)e * 2 * W * W;
            double2* cLR = cRL + W * W;
#pragma unroll
            for (int y = 0; y < W; ++y) {
                cRL[y * W + y0] = v[y];
                cLR[y0 * W + y] = v[y];
            }
        }
    }
}

template <int W, bool STORE_G>
static hipError_t launch_fullinv_w(const mcnegf_kernel& k, double2* Gc, int64_t ldG,
                                   hipStream_t s) {
    const unsigned tiles = (unsigned)((k.N + 63) / 64) + (STORE_G ? 0 : 1);  // and the chain
    dim3 grid(8u * tiles * (unsigned)((k.nE + 7) / 8));
    {
        MCNEGF_TIMED(STORE_G ? "fullinv_store_g_kernel" : "fullinv_kernel", s);
        hipLaunchKernelGGL((fullinv_kernel<W, STORE_G>), grid, dim3(64), 0, s,
                           reinterpret_cast<const double2*>(k.gR),
                           reinterpret_cast<const double2*>(k.Gd), k.gam_lead, k.L, k.t, k.p_pitch,
                           k.P, k.wL, k.wR, reinterpret_cast<double2*>(k.corner), Gc, ldG,
                           k.nE);
    }
    return hipGetLastError();
}

// ---- W = 16 and W = 32 on FP64 matrix cores ----------------------------------------------
//
// The same sweep, with the block products on v_mfma_f64_16x16x4f64 (no padding at these
// widths).  A workgroup of NW wavefronts shares one double-buffered staged block (so the LDS of
// a workgroup does not limit the wavefronts a CU holds) and sweeps from its first column's
// slice; a wavefront's columns hold their diagonal block's column until it is passed.  A
// wavefront owns TC tiles of 16 consecutive columns; lane (n, g) = (l % 16, l / 16)
// holds, for tile t and row tile rt, the rows 16 rt + 4 r + g (r = 0..3) of column n, which is
// both the accumulator layout of the product (item r of lane n + 16 g is row 4 r + g) and the
// B-operand layout of the next product (K-step s takes rows 4 s + g from lane n + 16 g), so the
// columns stay in registers from slice to slice.  The A operand of K-step s and row tile rt,
// lane (m, g): (-t) M[16 rt + m][4 s + g], read from the LDS-staged block.  A complex product
// is four real products (re re, -im im into the real part; re im, im re into the imaginary).
// With the lower half only: W = 16, N = 3200, 128 energies 5.33 -> 2.36 ms (|G|^2; 4.5 TB/s
// written) and 6.97 -> 4.96 ms (complex G); W = 32, N = 16000, 8 energies 11.2 -> 7.5 ms.
typedef double dmfma4 __attribute__((ext_vector_type(4)));
typedef float fmfma4 __attribute__((ext_vector_type(4)));

// One 16x16x4 product on the matrix cores in the column state's precision.
__device__ inline dmfma4 mfma4(double a, double b, dmfma4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline fmfma4 mfma4(float a, float b, fmfma4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <typename T> struct Mfma4;
template <> struct Mfma4<double> { typedef dmfma4 type; };
template <> struct Mfma4<float> { typedef fmfma4 type; };

// Row of item r in lane group g within a 16-row tile: the FP64 product returns row 4 r + g,
// the FP32 product row 4 g + r.  In both cases K-step s of the next product takes item
// s & 3 of tile s >> 2 from every lane group, i.e. the contraction runs over the rows in the
// order the accumulator holds them, and the A operand is read in that column order.
template <typename T>
__device__ inline int tile_row(int r, int g) {
    return sizeof(T) == 8 ? 4 * r + g : 4 * g + r;
}

// x[r] of lane group g becomes x[g] of lane group r (a 4 x 4 transpose across the groups of 16
// lanes): exchange half wavefronts between items 0, 2 and 1, 3, then neighbouring groups
// between items 0, 1 and 2, 3.  Every lane must be active.
__device__ inline void swap_halves(double& a, double& b) {
    auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
}
__device__ inline void swap_groups(double& a, double& b) {
    auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
}
__device__ inline void transpose_groups(double (&x)[4]) {
    swap_halves(x[0], x[2]);
    swap_halves(x[1], x[3]);
    swap_groups(x[0], x[1]);
    swap_groups(x[2], x[3]);
}

// T = double: FP64 products throughout.  T = float (a build with FP32 block products): the
// column state and the products are FP32 (the staged FP64 blocks are rounded as they are
// read), |G|^2, the exit weights and the corners are formed from the FP32 state in FP64.
// FP32 products form both halves, the upper one by a second sweep G_{k,l} = -t gL_k G_{k+1,l}
// (k < l) up the wire, with the exit weights into L and G_{0,L-1} at its end: the two halves'
// roundings are then independent of each other, as the sums over a probe's row and column expect.
// A mirrored lower half has one rounding for both: the rms error of T_eff grew from 6.6e-8 to 8.4e-8
// (W = 32, L = 50) and from 9.4e-8 to 1.5e-7 (W = 16, L = 120), the current's from 1.8e-8 to 3.3e-8,
// that of |G|^2 after refinement by a quarter.  Nor is it faster: |G|^2, N = 3200, 16 energies
// 0.47 ms at W = 16 (mirrored 0.61) and 0.64 ms at W = 32 (0.78).
template <int W, int TC, int NW, bool STORE_G, typename T = double>
__global__ void __launch_bounds__(64 * NW, 2) fullinv_mfma_kernel(const double2* __restrict__ gL,
                                                          const double2* __restrict__ gR,
                                                          const double2* __restrict__ Gd,
                                                          const double* __restrict__ gam_lead,
                                                          int L, double t, int64_t ldP,
                                                          double* __restrict__ P,
                                                          double* __restrict__ wL,
                                                          double* __restrict__ wR,
                                                          double2* __restrict__ corner,
                                                          double2* __restrict__ Gc, int64_t ldG) {
    constexpr int RT = W / 16;  // row tiles
    constexpr int S = W / 4;    // K-steps
    constexpr int BS = 2 * W * W;
    __shared__ double Ms_raw[2 * BS];
    lds_double* Ms = (lds_double*)Ms_raw;
    constexpr bool BOTH = sizeof(T) == 4;  // both halves by their own sweeps
    // (first workgroup of an energy) Gamma and, double-buffered, the columns of slice 0 at the
    // current slice, [column][row]
    constexpr int XN = STORE_G || BOTH ? 1 : W * W;
    __shared__ double Gs[XN];
    __shared__ double2 X[2][XN];
    const int N = W * L;
    const int e = blockIdx.x;  // tile by tile over the energies: the long tiles start first
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int cg0 = blockIdx.y * NW * 16 * TC;  // the workgroup's first column
    const int c0 = cg0 + (tid >> 6) * 16 * TC;  // this wavefront's first column
    const int kmin = cg0 / W;
    // the workgroup whose first wavefront holds the columns of slice 0
    const bool slice0 = !STORE_G && !BOTH && cg0 == 0;
    const size_t eb = (size_t)e * L * W * W;
    const double2* gLe = gL + eb;
    const double2* gRe = gR + eb;
    const double2* Gde = Gd + eb;
    const double* gme = gam_lead + (size_t)e * W * W;
    double* Pe = P + (size_t)e * N * ldP;
    double2* Ge = Gc + (size_t)e * N * ldG;
    const double mt = -t;

    int col[TC], l[TC], y0[TC];
    bool valid[TC];
#pragma unroll
    for (int tc = 0; tc < TC; ++tc) {
        col[tc] = c0 + 16 * tc + n;
        valid[tc] = col[tc] < N;
        const int cc = valid[tc] ? col[tc] : N - 1;
        l[tc] = cc / W;
        y0[tc] = cc - l[tc] * W;
    }
    typedef typename Mfma4<T>::type acc4;
    T vr[TC][RT][4], vi[TC][RT][4];

    // one slice: v <- (-t) M v with M the block staged at buf, for the columns whose slice the
    // sweep has passed (the others keep their diagonal block's column)
    auto product = [&](const lds_double* buf, int k, bool down = true) {
        acc4 cr[TC][RT], ci[TC][RT];
#pragma unroll
        for (int tc = 0; tc < TC; ++tc)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                cr[tc][rt] = acc4{0, 0, 0, 0};
                ci[tc][rt] = acc4{0, 0, 0, 0};
            }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                // column of M that K-step s pairs with lane group g (see tile_row)
                const int kc = 16 * (s >> 2) + tile_row<T>(s & 3, g);
                const int at = 2 * ((16 * rt + n) * W + kc);
                const T ar = (T)(mt * buf[at]), ai = (T)(mt * buf[at + 1]);
                // consecutive products go to different accumulators (2 TC independent chains)
#pragma unroll
                for (int tc = 0; tc < TC; ++tc) {
                    cr[tc][rt] = mfma4(ar, vr[tc][s >> 2][s & 3], cr[tc][rt]);
                    ci[tc][rt] = mfma4(ar, vi[tc][s >> 2][s & 3], ci[tc][rt]);
                }
#pragma unroll
                for (int tc = 0; tc < TC; ++tc) {
                    cr[tc][rt] = mfma4(-ai, vi[tc][s >> 2][s & 3], cr[tc][rt]);
                    ci[tc][rt] = mfma4(ai, vr[tc][s >> 2][s & 3], ci[tc][rt]);
                }
            }
        }
#pragma unroll
        for (int tc = 0; tc < TC; ++tc)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool on = down ? k > l[tc] : k < l[tc];
                    vr[tc][rt][r] = on ? cr[tc][rt][r] : vr[tc][rt][r];
                    vi[tc][rt][r] = on ? ci[tc][rt][r] : vi[tc][rt][r];
                }
    };
    // entry (row, column) and, below the diagonal block (with one sweep), its transpose: four
    // consecutive rows per lane, so that the four lane groups fill a 128-byte line of the transposed
    // row
    auto store = [&](int k, bool down = true) {
#pragma unroll
        for (int tc = 0; tc < TC; ++tc)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                double xr[4], xi[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    xr[r] = vr[tc][rt][r];
                    xi[r] = vi[tc][rt][r];
                    if (!STORE_G) xr[r] = xr[r] * xr[r] + xi[r] * xi[r];
                    const size_t row = k * W + 16 * rt + tile_row<T>(r, g);
                    if (valid[tc] && (down ? k >= l[tc] : k < l[tc])) {
                        if (STORE_G) Ge[row * ldG + col[tc]] = cmk(xr[r], xi[r]);
                        else Pe[row * ldP + col[tc]] = xr[r];
                    }
                }
                if (!BOTH) {
                    transpose_groups(xr);
                    if (STORE_G) transpose_groups(xi);
                }
                if (!BOTH && valid[tc] && k > l[tc]) {
                    const size_t c4 = k * W + 16 * rt + 4 * g;
                    if (STORE_G) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            Ge[(size_t)col[tc] * ldG + c4 + r] = cmk(xr[r], xi[r]);
                    } else {
                        *reinterpret_cast<double4*>(Pe + (size_t)col[tc] * ldP + c4) =
                            double4{xr[0], xr[1], xr[2], xr[3]};
                    }
                }
            }
    };
    // Exit weights into L of the rows of slice k, from the columns of slice 0 in X: wavefront w
    // takes YPW rows, the lanes of a row AC of the W terms Re conj(x_a) (Gamma x)_a each.
    constexpr int YPW = W / NW, AC = W * YPW / 64;
    auto exit_left = [&](int k) {
        const double2* x = X[k & 1];
        const int y = YPW * (tid >> 6) + lane % YPW, a0 = AC * (lane / YPW);
        double acc = 0.0;
#pragma unroll
        for (int a = 0; a < AC; ++a) {
            double2 u = cmk(0.0, 0.0);
#pragma unroll 8
            for (int b = 0; b < W; ++b) u = cadd(u, cscale(x[b * W + y], Gs[(a0 + a) * W + b]));
            const double2 xa = x[(a0 + a) * W + y];
            acc = fma(xa.x, u.x, fma(xa.y, u.y, acc));
        }
#pragma unroll
        for (int o = YPW; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
        if (lane < YPW) wL[(size_t)e * N + k * W + y] = acc;
    };
    // Re v^+ Gamma v per column (Gamma real symmetric): u = Gamma v on the matrix cores, the
    // row sum of Re(conj(v) u) over the four lanes of each column; lane g = 0 gets the result.
    auto quad = [&](int tc) -> double {
        acc4 ur[RT], ui[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            ur[rt] = acc4{0, 0, 0, 0};
            ui[rt] = acc4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const T a = (T)gme[(16 * rt + n) * W + 16 * (s >> 2) + tile_row<T>(s & 3, g)];
                ur[rt] = mfma4(a, vr[tc][s >> 2][s & 3], ur[rt]);
                ui[rt] = mfma4(a, vi[tc][s >> 2][s & 3], ui[rt]);
            }
        }
        double q = 0.0;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                q = fma((double)vr[tc][rt][r], (double)ur[rt][r],
                        fma((double)vi[tc][rt][r], (double)ui[rt][r], q));
        q += __shfl_xor(q, 16, 64);
        q += __shfl_xor(q, 32, 64);
        return q;
    };

    auto start = [&] {
#pragma unroll
        for (int tc = 0; tc < TC; ++tc)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double2 d =
                        Gde[((size_t)l[tc] * W + 16 * rt + tile_row<T>(r, g)) * W + y0[tc]];
                    vr[tc][rt][r] = (T)d.x;
                    vi[tc][rt][r] = (T)d.y;
                }
    };
    start();
    if (slice0)
        for (int i = tid; i < W * W; i += 64 * NW) Gs[i] = gme[i];
    StagedBlock<W, 64 * NW> st;  // block k + 1 at the top of slice k
    st.load(gRe + (size_t)kmin * W * W, tid);
    st.write(Ms, tid);
    st.load(gRe + (size_t)min(kmin + 1, L - 1) * W * W, tid);
    for (int k = kmin; k < L; ++k) {
        __syncthreads();
        const int b = (k - kmin) & 1;
        st.write(Ms + (b ^ 1) * BS, tid);
        st.load(gRe + (size_t)min(k + 2, L - 1) * W * W, tid);
        if (slice0 && k > 0) exit_left(k - 1);
        product(Ms + b * BS, k);
        store(k);
        if (slice0 && tid < 64) {
#pragma unroll
            for (int tc = 0; tc < W / 16; ++tc)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        X[k & 1][(16 * tc + n) * W + 16 * rt + tile_row<T>(r, g)] =
                            cmk(vr[tc][rt][r], vi[tc][rt][r]);
        }
    }
    if (slice0) {  // the whole workgroup
        __syncthreads();
        exit_left(L - 1);
    }
    // the exit weights at the end of a sweep and, for the columns of the opposite end slice, the
    // corner block; with one sweep the other corner block is its transpose
    auto finish = [&](bool down) {
#pragma unroll
        for (int tc = 0; tc < TC; ++tc) {
            const double q = quad(tc);
            if (valid[tc] && g == 0) (down ? wR : wL)[(size_t)e * N + col[tc]] = q;
            if (valid[tc] && l[tc] == (down ? 0 : L - 1)) {
                double2* c = corner + ((size_t)e * 2 + (down ? 0 : 1)) * W * W;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int y = 16 * rt + tile_row<T>(r, g);
                        c[y * W + y0[tc]] = cmk(vr[tc][rt][r], vi[tc][rt][r]);
                        if (!BOTH) c[W * W + y0[tc] * W + y] = cmk(vr[tc][rt][r], vi[tc][rt][r]);
                    }
            }
        }
    };
    if (!STORE_G) finish(true);
    if constexpr (BOTH) {
        const int kmax = (min(cg0 + NW * 16 * TC, N) - 1) / W;
        start();
        __syncthreads();  // the downward sweep's reads are done
        st.load(gLe + (size_t)kmax * W * W, tid);
        st.write(Ms, tid);
        st.load(gLe + (size_t)max(kmax - 1, 0) * W * W, tid);
        for (int k = kmax; k >= 0; --k) {
            __syncthreads();
            const int b = (kmax - k) & 1;
            st.write(Ms + (b ^ 1) * BS, tid);
            st.load(gLe + (size_t)max(k - 2, 0) * W * W, tid);
            product(Ms + b * BS, k, false);
            store(k, false);
        }
        if (!STORE_G) finish(false);
    }
}

template <int W, int TC, int NW, bool STORE_G, typename T = double>
static hipError_t launch_fullinv_mfma(const mcnegf_kernel& k, double2* Gc, int64_t ldG,
                                      hipStream_t s) {
    dim3 grid(k.nE, (k.N + 16 * TC * NW - 1) / (16 * TC * NW));
    {
        MCNEGF_TIMED(STORE_G ? "fullinv_store_g_kernel" : "fullinv_kernel", s);
        hipLaunchKernelGGL((fullinv_mfma_kernel<W, TC, NW, STORE_G, T>), grid, dim3(64 * NW), 0, s,
                           reinterpret_cast<const double2*>(k.gL),
                           reinterpret_cast<const double2*>(k.gR),
                           reinterpret_cast<const double2*>(k.Gd), k.gam_lead, k.L, k.t, k.p_pitch,
                           k.P, k.wL, k.wR, reinterpret_cast<double2*>(k.corner), Gc, ldG);
    }
    return hipGetLastError();
}

// wavefronts per workgroup sharing one staged block
constexpr int kFullinvWaves16 = 1;
constexpr int kFullinvWaves32 = 4;

template <bool STORE_G>
static hipError_t launch_fullinv_any(const mcnegf_kernel& k, double2* Gc, int64_t ldG,
                                     hipStream_t s) {
    if (k.W == 16) return launch_fullinv_mfma<16, 4, kFullinvWaves16, STORE_G>(k, Gc, ldG, s);
    if (k.W == 32) return launch_fullinv_mfma<32, 2, kFullinvWaves32, STORE_G>(k, Gc, ldG, s);
    switch (k.W) {
#define MCNEGF_CASE(w) \
    case w:            \
        return launch_fullinv_w<w, STORE_G>(k, Gc, ldG, s);
        MCNEGF_CASE(1) MCNEGF_CASE(2) MCNEGF_CASE(3) MCNEGF_CASE(4) MCNEGF_CASE(5)
        MCNEGF_CASE(6) MCNEGF_CASE(7) MCNEGF_CASE(8) MCNEGF_CASE(9) MCNEGF_CASE(10)
        MCNEGF_CASE(11) MCNEGF_CASE(12) MCNEGF_CASE(13) MCNEGF_CASE(14) MCNEGF_CASE(15)
        MCNEGF_CASE(17) MCNEGF_CASE(18) MCNEGF_CASE(19) MCNEGF_CASE(20)
        MCNEGF_CASE(21) MCNEGF_CASE(22) MCNEGF_CASE(23) MCNEGF_CASE(24) MCNEGF_CASE(25)
        MCNEGF_CASE(26) MCNEGF_CASE(27) MCNEGF_CASE(28) MCNEGF_CASE(29) MCNEGF_CASE(30)
        MCNEGF_CASE(31)
#undef MCNEGF_CASE
        default:
            return hipErrorInvalidValue;
    }
}

hipError_t launch_fullinv(const mcnegf_kernel& k, hipStream_t s) {
    return launch_fullinv_any<false>(k, nullptr, 0, s);
}

// The full inverse with FP32 block products (W = 16 and 32 only; any other width is refused).
hipError_t launch_fullinv_fp32(const mcnegf_kernel& k, hipStream_t s) {
    if (k.W == 16) return launch_fullinv_mfma<16, 4, kFullinvWaves16, false, float>(k, nullptr, 0, s);
    if (k.W == 32) return launch_fullinv_mfma<32, 2, kFullinvWaves32, false, float>(k, nullptr, 0, s);
    return hipErrorInvalidValue;
}

hipError_t launch_fullinv_fp32_store_g(const mcnegf_kernel& k, double2* Gc, int64_t ldG,
                                       hipStream_t s) {
    if (k.W == 16) return launch_fullinv_mfma<16, 4, kFullinvWaves16, true, float>(k, Gc, ldG, s);
    if (k.W == 32) return launch_fullinv_mfma<32, 2, kFullinvWaves32, true, float>(k, Gc, ldG, s);
    return hipErrorInvalidValue;
}

hipError_t launch_fullinv_store_g(const mcnegf_kernel& k, double2* Gc, int64_t ldG,
                                  hipStream_t s) {
    return launch_fullinv_any<true>(k, Gc, ldG, s);
}

}  // namespace mcnegf
