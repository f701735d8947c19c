// Backpropagation: adjoint of the IF synthesis (Eqs. 11-12) per path, then
// the reverse sweep through the ray geometry of every ray (Eq. 13 chain rule)
// with per-bounce recomputation, scattering dL/dverts.
#include <vector>

#include "sbr_internal.h"
#include "sbr_device.h"

namespace sbr {

namespace {

struct AdjArgs {
    const int32_t *count;
    PathSoA rec;
    const float2 *G;       // [V][C][S]
    int32_t V, C, S;
    int32_t rows;          // G rows per LDS stage (direct form)
    int32_t Sp;            // S rounded up to a multiple of 8
    int32_t v_per;         // antennas per y-block
    int32_t nvs;           // y-blocks
    int32_t tile;          // paths per work item of the kernel that runs this request
    float fcf, sl_fs, tc;  // fc, slope / fs, chirp period
    float *tau_bar;        // [V][cap]
    float2 *abar_part;     // [nvs][cap]
    float *tdb_part;       // [nvs][cap] dL/d taudot partials
    const float4 *nu_rows; // non-uniform FFT rows of 2S + 8 points (NULL: direct form):
                           // [V][C] of the chirp-row form, [V][q] of the node form
    float *nu_corr;        // [S] 1/Psi table of the chirp-row form
    float2 *td_rows;       // [V][q][2S + 8] node form: rows of the taudot sums
    double *acc;           // sums over rays to clear (NULL: none)
    int32_t n_acc;
    NodePlan nd;           // nd.q = 0: not the node form
};

constexpr int kAdjRowsMax = 8;   // G rows staged in LDS at a time
constexpr int kAdjPPL = 2;       // paths per lane, direct form
constexpr int kNuPPL = 4;        // paths per lane, non-uniform FFT form
constexpr int kAdjQueueDirect = 32;   // work counters: of the direct form, of the chirp-row
constexpr int kAdjQueueNode = 48;     // form (queue[0]) and of the node form
constexpr int kNodeThreads = 512;     // threads of a node-form block
constexpr int kNodePPL = 2;           // its paths per lane

// ---- Eqs. 11-12 by a type-2 non-uniform FFT -------------------------------
// For each (v, c) the two sums of the adjoint are finite Fourier series of one
// G row evaluated at a path's beat frequency g (cycles per sample, reduced to
// [-1/2, 1/2]):
//   P(g) = sum_s h1_s e^{2 pi j s g},  h1_s = conj(G_s)
//   Q(g) = sum_s h2_s e^{2 pi j s g},  h2_s = conj(G_s) (fc + (slope/fs) s)
// (Q = fc P + (slope/fs) x P'(x) of the direct form).  By the identity of the
// non-uniform FFT forms (sbr_internal.h),
//   P(g) = e^{2 pi j g S/2} sum_l u_l psi(gM - l),
//   u_l  = sum_s' (h_{s'+S/2} / Psi(s'/M)) e^{2 pi j s' l / M}:
// the rows u (one per (v, c), shared by every path) cost one dense DFT each,
// and a path then needs kNuW taps per (v, c) instead of S terms; the error
// stays below 1e-6 of sum_s |h_s| at every g (two orders of magnitude under
// the FP32 rounding of a 256-term direct sum).
// float4's layout for address-space-qualified 16-byte loads of the rows
struct alignas(16) F4 {
    float x, y, z, w;
};
__device__ __forceinline__ SBR_GLOBAL_AS const F4 *gmem4(const float4 *p) { return (SBR_GLOBAL_AS const F4 *)p; }

// Chirp rows per LDS stage of the non-uniform FFT adjoint: about 36 KiB
// (4 rows at S = 256), 1 .. 8 rows.
__host__ __device__ inline int nu_stage(int S) { return max(1, min(8, 36864 / (nu_row_len(S) * 16))); }

// frac(n f) for an integer-valued n < 2^24: the product is exact inside the fma
__device__ __forceinline__ float frac_of_product(float n, float f) { return fmaf(n, f, -rintf(n * f)); }

// 1 / Psi((s - S/2) / 2S) for s < S (nu_corr_value) of request blockIdx.y of an
// adjoint batch, blocks of 256 modes.
__global__ __launch_bounds__(256) void k_nu_corr_adj(const AdjArgs *__restrict__ args) {
    __shared__ double kn[kNuTaps];
    if (threadIdx.x < kNuTaps) kn[threadIdx.x] = nu_kernel_sample((int)threadIdx.x);
    __syncthreads();
    const AdjArgs &a = args[blockIdx.y];
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < a.S) a.nu_corr[s] = nu_corr_value(a.S, s, kn);
}


// Gradient row (v, c) of a request of the batch (blocks [first[j], first[j + 1])
// are request j's rows, v major): u1_l, u2_l (float4: u1.re, u1.im, u2.re, u2.im)
// for l = -M/2 - 3 .. M/2 + 3 at index l + M/2 + 3, the DFT of the S
// deconvolved modes (mode s' = s - S/2 at position s' mod M of an M-point
// sequence, zero elsewhere) with twiddles e^{2 pi j k / M} from an
// exact-index LDS table: for M a power of two an in-place radix-2 FFT in LDS
// (both sequences in the same butterflies), otherwise a direct sum per
// output; the last entry of the row is zero padding.
__global__ __launch_bounds__(256) void k_nu_rows(const AdjArgs *__restrict__ args, const int32_t *__restrict__ first,
                                                 int m) {
    extern __shared__ float4 nsh[];
    // request j of the batch owns blocks (rows) [first[j], first[j + 1])
    int j = 0, hi = m;
    while (hi - j > 1) {
        const int mid = (j + hi) >> 1;
        if (first[mid] <= (int)blockIdx.x) j = mid;
        else hi = mid;
    }
    const AdjArgs &a = args[j];
    const float2 *__restrict__ G = a.G;
    const float *__restrict__ corr = a.nu_corr;
    float4 *__restrict__ rows = const_cast<float4 *>(a.nu_rows);
    const int S = a.S;
    const float fcf = a.fcf, sl_fs = a.sl_fs;
    const int M = 2 * S, RL = nu_row_len(S);
    float2 *tw = reinterpret_cast<float2 *>(nsh + M);        // [M], after the M-point sequence
    const size_t row = (size_t)((int)blockIdx.x - first[j]);
    for (int k = threadIdx.x; k < M; k += blockDim.x) {
        double sn, cs;
        sincospi(2.0 * k / M, &sn, &cs);
        tw[k] = make_float2((float)cs, (float)sn);
    }
    const float2 *g = G + row * S;
    float4 *out = rows + row * RL;
    if ((M & (M - 1)) == 0) {
        // a[n] = h_{s}, n = (s - S/2) mod M (zero for the other half), stored
        // at bit-reversed positions; X[l] = sum_n a[n] e^{2 pi j n l / M}
        float4 *a4 = nsh;   // [M]
        const int lg = 31 - __clz(M);
        for (int n = threadIdx.x; n < M; n += blockDim.x) {
            const int s = (n + S / 2) % M;
            float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
            if (s < S) {
                const float2 v = g[s];
                const float r = corr[s];
                const float w2 = fmaf(sl_fs, (float)s, fcf);
                const float hr = v.x * r, hi = -v.y * r;   // conj(G_s) / Psi
                h = make_float4(hr, hi, hr * w2, hi * w2);
            }
            a4[__brev((uint32_t)n) >> (32 - lg)] = h;
        }
        __syncthreads();
        for (int half = 1; half < M; half <<= 1) {
            const int tstep = M / (2 * half);
            for (int i = threadIdx.x; i < M / 2; i += blockDim.x) {
                const int pos = i & (half - 1), j0 = ((i - pos) << 1) + pos, j1 = j0 + half;
                const float2 w = tw[pos * tstep];
                const float4 u = a4[j0], v = a4[j1];
                const float4 vw = make_float4(v.x * w.x - v.y * w.y, v.x * w.y + v.y * w.x,
                                              v.z * w.x - v.w * w.y, v.z * w.y + v.w * w.x);
                a4[j0] = make_float4(u.x + vw.x, u.y + vw.y, u.z + vw.z, u.w + vw.w);
                a4[j1] = make_float4(u.x - vw.x, u.y - vw.y, u.z - vw.z, u.w - vw.w);
            }
            __syncthreads();
        }
        for (int i = threadIdx.x; i < RL; i += blockDim.x) {
            if (i < RL - 1) {
                int lm = (i - (M / 2 + kNuHalf)) % M;   // l mod M
                if (lm < 0) lm += M;
                out[i] = a4[lm];
            } else {
                out[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        return;
    }
    float4 *hb = nsh;   // [S] h1, h2 over Psi
    for (int s = threadIdx.x; s < S; s += blockDim.x) {
        const float2 v = g[s];
        const float r = corr[s];
        const float w2 = fmaf(sl_fs, (float)s, fcf);
        const float hr = v.x * r, hi = -v.y * r;   // conj(G_s) / Psi
        hb[s] = make_float4(hr, hi, hr * w2, hi * w2);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < RL; i += blockDim.x) {
        float ar = 0.f, ai = 0.f, br = 0.f, bi = 0.f;
        if (i < RL - 1) {
            int lm = (i - (M / 2 + kNuHalf)) % M;   // l mod M
            if (lm < 0) lm += M;
            int k = (int)(((long long)(M - S / 2) * lm) % M);   // (s - S/2) l mod M at s = 0
            for (int s = 0; s < S; s++) {
                const float2 t = tw[k];
                const float4 h = hb[s];
                ar = fmaf(h.x, t.x, fmaf(-h.y, t.y, ar));
                ai = fmaf(h.x, t.y, fmaf(h.y, t.x, ai));
                br = fmaf(h.z, t.x, fmaf(-h.w, t.y, br));
                bi = fmaf(h.z, t.y, fmaf(h.w, t.x, bi));
                k += lm;
                if (k >= M) k -= M;
            }
        }
        out[i] = make_float4(ar, ai, br, bi);
    }
}

// One work item of the non-uniform FFT form: per path and (v, c) the taps
// l0 .. l0 + 6 around x = gM (l0 = rint(x) - 3) of both rows, kernel weights
// from their polynomial forms (nu_weights), and the same accumulation as the
// direct form with z0 e^{2 pi j g S/2} as the phase factor.  That phase is
// alpha + c beta + (S/2) g = alpha + (S/2) gamma + c (beta + (S/2) eps) up to
// an integer ((S/2) times the integer that reduces g), so from one chirp to
// the next the factor turns by r = e^{2 pi j (beta + (S/2) eps)}: it is
// computed exactly at the first chirp of each stage and rotated by r for the
// others (at most 7 rotations).  The rows of `stage` chirps at a time are
// copied to LDS by the whole block (coalesced 16-byte loads), so that each
// row read from L2 serves the item's 256 PPL paths, and paths of similar beat
// frequency read the same LDS words.
template <int PPL>
__device__ __forceinline__ void adj_item_nu(const AdjArgs &a, float4 *rsh, const int stage, const int P,
                                            const int grp, const int blk_p0) {
    const auto amp = gmem(a.rec.amp);
    const auto bet = gmem(a.rec.beta);
    const auto eps = gmem(a.rec.epsd);
    const auto alp = gmem(a.rec.alpha);
    const auto gam = gmem(a.rec.gamma);
    const auto tbar = gmem(a.tau_bar);
    int pp[PPL];
    bool act[PPL];
    float Ax[PPL], Ay[PPL], beta[PPL], epsd[PPL], abr[PPL], abi[PPL], tdb[PPL], rc[PPL], rs[PPL];
    const int S = a.S, M = 2 * S, RL = nu_row_len(S);
    const float Mf = (float)M, halfS = (float)(S / 2);
#pragma unroll
    for (int i = 0; i < PPL; i++) {
        pp[i] = blk_p0 + i * 256 + threadIdx.x;
        act[i] = pp[i] < P;
        const int pc = act[i] ? pp[i] : blk_p0;
        const F2 A = amp[pc];
        Ax[i] = A.x;
        Ay[i] = A.y;
        beta[i] = bet[pc];
        epsd[i] = eps[pc];
        abr[i] = abi[i] = tdb[i] = 0.0f;
        pp[i] = pc;
        float rt = beta[i] + frac_of_product(halfS, epsd[i]);   // turn per chirp
        rt -= rintf(rt);
        rs[i] = __builtin_amdgcn_sinf(rt);
        rc[i] = __builtin_amdgcn_cosf(rt);
    }
    const int v0 = grp * a.v_per, v1 = min(a.V, v0 + a.v_per);
    for (int v = v0; v < v1; v++) {
        float alpha[PPL], gamma[PPL], tb[PPL];
#pragma unroll
        for (int i = 0; i < PPL; i++) {
            alpha[i] = alp[(size_t)v * a.rec.cap + pp[i]];
            gamma[i] = gam[(size_t)v * a.rec.cap + pp[i]];
            tb[i] = 0.0f;
        }
        const auto rows_v = gmem4(a.nu_rows) + (size_t)v * a.C * RL;
        for (int c0 = 0; c0 < a.C; c0 += stage) {
            const int nr = min(stage, a.C - c0);
            __syncthreads();   // the previous stage has been read
            for (int i = threadIdx.x; i < nr * RL; i += 256) {
                const F4 u = rows_v[(size_t)c0 * RL + i];
                rsh[i] = make_float4(u.x, u.y, u.z, u.w);
            }
            __syncthreads();
            float zc[PPL], zs[PPL];   // phase factor of the current chirp
            for (int cc = 0; cc < nr; cc++) {
                const float cf = (float)(c0 + cc);
                const float4 *row = rsh + cc * RL;
#pragma unroll
                for (int i = 0; i < PPL; i++) {
                    const float f = fmaf(cf, epsd[i], gamma[i]);
                    const float g = f - rintf(f);   // [-1/2, 1/2]
                    const float x = g * Mf;         // exact
                    const float xr = rintf(x);
                    const int i0 = min(max((int)xr + M / 2, 0), M);   // row index of l0 = xr - 3 (clamped: NaN-safe)
                    float w[kNuW];
                    nu_weights(x - xr, w);
                    float pr = 0.f, pi = 0.f, qr = 0.f, qi = 0.f;
#pragma unroll
                    for (int t = 0; t < kNuW; t++) {
                        const float4 u = row[i0 + t];
                        pr = fmaf(w[t], u.x, pr);
                        pi = fmaf(w[t], u.y, pi);
                        qr = fmaf(w[t], u.z, qr);
                        qi = fmaf(w[t], u.w, qi);
                    }
                    if (cc == 0) {   // block-uniform
                        float th = alpha[i] + frac_of_product(cf, beta[i]) + frac_of_product(halfS, g);
                        th -= rintf(th);
                        zs[i] = __builtin_amdgcn_sinf(th);
                        zc[i] = __builtin_amdgcn_cosf(th);
                    } else {
                        const float tc = zc[i] * rc[i] - zs[i] * rs[i];
                        zs[i] = zc[i] * rs[i] + zs[i] * rc[i];
                        zc[i] = tc;
                    }
                    // Q0 = z0 P, m = z0 Q (z0 including e^{2 pi j g S/2})
                    const float q0r = zc[i] * pr - zs[i] * pi, q0i = zc[i] * pi + zs[i] * pr;
                    const float mr = zc[i] * qr - zs[i] * qi, mi = zc[i] * qi + zs[i] * qr;
                    abr[i] += q0r;
                    abi[i] -= q0i;
                    const float dq = -2.0f * (float)kPi * (Ax[i] * mi + Ay[i] * mr);
                    tb[i] += dq;
                    tdb[i] = fmaf(dq, cf * a.tc, tdb[i]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < PPL; i++)
            if (act[i]) tbar[(size_t)v * a.rec.cap + pp[i]] = tb[i];
    }
#pragma unroll
    for (int i = 0; i < PPL; i++)
        if (act[i]) {
            gmem(a.abar_part)[(size_t)grp * a.rec.cap + pp[i]] = F2{abr[i], abi[i]};
            gmem(a.tdb_part)[(size_t)grp * a.rec.cap + pp[i]] = tdb[i];
        }
}

// ---- the node form of the adjoint (type-2 transform over Doppler nodes) -----
// The kernel is one tap wider than the synthesis' (aliasing 9e-8 instead of
// 8e-7 of the terms' RMS): the gradients of the pose, the medium and the
// materials sum over all paths with cancellation and show that error.
// Against 64 bits they come out 0.4 times as far off as with the chirp rows
// (geometric mean over 40 scenes of 320^2 rays).
// The transpose of the synthesis' node form (NodePlan, sbr_internal.h): per
// (v, j) one row of the node sums
//   H_j[s] = sum_c conj(G[v][c][s]) e^{2 pi j (c - cbar)(1 + s kappa) nu_j}
// is transformed like a gradient row of the chirp-row form, and a path reads
// kNu8W taps of q rows instead of one row per chirp; its chirp-weighted sum (the
// taudot adjoint, Q with the weight c t_chirp) has rows of its own, made and
// read only where a gradient that depends on it is asked for.

// Node row (v, j) = blockIdx.x: the chirps summed against the node's phase
// (thread groups take every groups-th chirp), weighted and deconvolved, then
// the DFT as in k_nu_rows with the taudot sequence beside.  All of it in FP64:
// a path reads a few node rows where it read one row per chirp, so rounding in
// a row no longer averages over the chirps, and there are only V q rows (84 at
// 12 antennas and 7 nodes: the launch is bound by its longest chain).
constexpr int kNodeRowThreads = 512;
struct D4 {
    double x, y, z, w;
};

template <bool TD>
__global__ __launch_bounds__(kNodeRowThreads) void k_node_adj_rows(const AdjArgs *__restrict__ args,
                                                                   const int32_t *__restrict__ first, int m) {
    extern __shared__ double nsd[];
    __shared__ double kn[kNu8Taps];
    int j = 0, hi = m;
    while (hi - j > 1) {
        const int mid = (j + hi) >> 1;
        if (first[mid] <= (int)blockIdx.x) j = mid;
        else hi = mid;
    }
    const AdjArgs &a = args[j];
    const int S = a.S, M = 2 * S, RL = nu_row_len(S), Q = a.nd.q, C = a.C;
    D4 *seq = reinterpret_cast<D4 *>(nsd);                    // [M] (P, Q) sequence
    double2 *tw = reinterpret_cast<double2 *>(seq + M);       // [M]
    double2 *sq2 = tw + M;                                    // [M] taudot sequence (TD)
    D4 *part = reinterpret_cast<D4 *>(TD ? sq2 + M : sq2);    // [groups][cols], one per thread
    const int row = (int)blockIdx.x - first[j], v = row / Q, k = row - v * Q;
    const bool pow2 = (M & (M - 1)) == 0;
    const int lg = 31 - __clz(M);
    const double nu = a.nd.nu0 + a.nd.h * cospi((2.0 * k + 1.0) / (2.0 * Q));
    if (threadIdx.x < kNu8Taps) kn[threadIdx.x] = nu8_kernel_sample((int)threadIdx.x);
    for (int i = threadIdx.x; i < M; i += kNodeRowThreads) {
        double sn, cs;
        sincospi(2.0 * i / M, &sn, &cs);
        tw[i] = make_double2(cs, sn);
    }
    __syncthreads();
    // chirp sums of column s by the groups' threads, partial sums through LDS
    const int cols = min(S, kNodeRowThreads), groups = kNodeRowThreads / cols;
    const int g = (int)threadIdx.x / cols, col = (int)threadIdx.x % cols;
    const auto G = gmem(a.G) + (size_t)v * C * S;
    for (int s0 = 0; s0 < S; s0 += cols) {
        const int s = s0 + col;
        double pr = 0.0, pi = 0.0, tr = 0.0, ti = 0.0;
        if (g < groups && s < S) {
            const double rate = (1.0 + s * a.nd.kappa) * nu;
#pragma unroll 4
            for (int c = g; c < C; c += groups) {
                const F2 x = G[(size_t)c * S + s];
                const double ph = (double)(c - a.nd.cbar) * rate;
                float sn, cs;
                sincospif(2.0f * (float)(ph - rint(ph)), &sn, &cs);
                const float zr = fmaf(x.x, cs, x.y * sn), zi = fmaf(x.x, sn, -x.y * cs);   // conj(G) e^{...}
                pr += zr;
                pi += zi;
                if (TD) {
                    tr += (double)c * zr;
                    ti += (double)c * zi;
                }
            }
        }
        if (groups > 1) {
            if (g < groups) part[g * cols + col] = D4{pr, pi, tr, ti};
            __syncthreads();
            if (g == 0) {
                for (int q = 1; q < groups; q++) {
                    const D4 x = part[q * cols + col];
                    pr += x.x;
                    pi += x.y;
                    tr += x.z;
                    ti += x.w;
                }
            }
        }
        if (g == 0 && s < S) {
            const double r = nu8_corr_value(S, s, kn);
            const double w2 = (double)a.sl_fs * s + (double)a.fcf;
            const double hr = pr * r, hi2 = pi * r;
            const int n = pow2 ? (s - S / 2) & (M - 1) : s;                      // mode s - S/2
            const int pos = pow2 ? (int)(__brev((uint32_t)n) >> (32 - lg)) : s;
            seq[pos] = D4{hr, hi2, hr * w2, hi2 * w2};
            if (TD) sq2[pos] = make_double2(tr * (r * w2 * a.tc), ti * (r * w2 * a.tc));
        }
    }
    if (pow2) {
        // the other S modes are zero
        for (int i = threadIdx.x; i < S; i += kNodeRowThreads) {
            const int n = (i + S - S / 2) & (M - 1);
            const int pos = (int)(__brev((uint32_t)n) >> (32 - lg));
            seq[pos] = D4{0.0, 0.0, 0.0, 0.0};
            if (TD) sq2[pos] = make_double2(0.0, 0.0);
        }
    }
    __syncthreads();
    float4 *out = const_cast<float4 *>(a.nu_rows) + (size_t)row * RL;
    float2 *out2 = a.td_rows + (size_t)row * RL;
    if (pow2) {
        for (int half = 1; half < M; half <<= 1) {
            const int tstep = M / (2 * half);
            for (int i = threadIdx.x; i < M / 2; i += kNodeRowThreads) {
                const int pos = i & (half - 1), j0 = ((i - pos) << 1) + pos, j1 = j0 + half;
                const double2 w = tw[pos * tstep];
                const D4 u = seq[j0], x = seq[j1];
                const D4 vw = {x.x * w.x - x.y * w.y, x.x * w.y + x.y * w.x, x.z * w.x - x.w * w.y,
                               x.z * w.y + x.w * w.x};
                seq[j0] = D4{u.x + vw.x, u.y + vw.y, u.z + vw.z, u.w + vw.w};
                seq[j1] = D4{u.x - vw.x, u.y - vw.y, u.z - vw.z, u.w - vw.w};
                if (TD) {
                    const double2 u2 = sq2[j0], x2 = sq2[j1];
                    const double2 t = make_double2(x2.x * w.x - x2.y * w.y, x2.x * w.y + x2.y * w.x);
                    sq2[j0] = make_double2(u2.x + t.x, u2.y + t.y);
                    sq2[j1] = make_double2(u2.x - t.x, u2.y - t.y);
                }
            }
            __syncthreads();
        }
    }
    for (int i = threadIdx.x; i < RL; i += kNodeRowThreads) {
        D4 o = {0.0, 0.0, 0.0, 0.0};
        double2 o2 = make_double2(0.0, 0.0);
        int lm = (i - (M / 2 + kNuHalf)) % M;   // l mod M, l = -M/2 - 3 .. M/2 + 4
        if (lm < 0) lm += M;
        if (pow2) {
            o = seq[lm];
            if (TD) o2 = sq2[lm];
        } else {
            int kk = (int)(((long long)(M - S / 2) * lm) % M);   // (s - S/2) l mod M at s = 0
            for (int s = 0; s < S; s++) {
                const double2 t = tw[kk];
                const D4 h = seq[s];
                o.x = fma(h.x, t.x, fma(-h.y, t.y, o.x));
                o.y = fma(h.x, t.y, fma(h.y, t.x, o.y));
                o.z = fma(h.z, t.x, fma(-h.w, t.y, o.z));
                o.w = fma(h.z, t.y, fma(h.w, t.x, o.w));
                if (TD) {
                    const double2 h2 = sq2[s];
                    o2.x = fma(h2.x, t.x, fma(-h2.y, t.y, o2.x));
                    o2.y = fma(h2.x, t.y, fma(h2.y, t.x, o2.y));
                }
                kk += lm;
                if (kk >= M) kk -= M;
            }
        }
        out[i] = make_float4((float)o.x, (float)o.y, (float)o.z, (float)o.w);
        if (TD) out2[i] = make_float2((float)o2.x, (float)o2.y);
    }
}

// Node rows per LDS stage: at most 60 KiB (all 6 or 7 rows at 256 samples
// without taudot rows), so that two blocks share a CU.
__host__ __device__ inline int node_stage(int S, int q, bool td) {
    return max(1, min(q, 61440 / (nu_row_len(S) * (td ? 24 : 16))));
}

// One work item of the node form: a.tile paths from blk_p0 on, kNodePPL per lane
// at a time; per antenna the tap weights and the phase factor once, then per
// node the kNu8W taps (16-byte LDS reads, 8 more for the taudot rows) times the
// node's Lagrange polynomial.  Bound by those LDS reads: 8 q (16 or 24) bytes
// per path and antenna.  An item of one antenna whose rows are all in LDS keeps
// them for all its paths.
template <bool TD>
__device__ __forceinline__ void adj_part_node(const AdjArgs &a, float4 *rsh, const int P, const int grp,
                                              const int blk_p0, const bool have_rows) {
    constexpr int PPL = kNodePPL;
    const auto amp = gmem(a.rec.amp);
    const auto bet = gmem(a.rec.beta);
    const auto eps = gmem(a.rec.epsd);
    const auto alp = gmem(a.rec.alpha);
    const auto gam = gmem(a.rec.gamma);
    const auto tbar = gmem(a.tau_bar);
    int pp[PPL];
    bool act[PPL];
    float Ax[PPL], Ay[PPL], beta[PPL], epsd[PPL], abr[PPL], abi[PPL], tdb[PPL], tau[PPL], lp[PPL];
    const int S = a.S, RL = nu_row_len(S), Q = a.nd.q;
    const double cb = (double)a.nd.cbar;
    const int stage = node_stage(S, Q, TD);
    float2 *rs2 = reinterpret_cast<float2 *>(rsh + stage * RL);
#pragma unroll
    for (int i = 0; i < PPL; i++) {
        pp[i] = blk_p0 + i * kNodeThreads + (int)threadIdx.x;
        act[i] = pp[i] < P;
        const int pc = act[i] ? pp[i] : blk_p0;
        const F2 A = amp[pc];
        Ax[i] = A.x;
        Ay[i] = A.y;
        beta[i] = bet[pc];
        epsd[i] = eps[pc];
        abr[i] = abi[i] = tdb[i] = 0.0f;
        pp[i] = pc;
        tau[i] = node_offset(beta[i], a.nd.nu0f, a.nd.inv_h);   // [-1, 1]
        lp[i] = 1.0f;
        for (int k = 0; k < Q; k++) lp[i] *= node_factor(tau[i], a.nd.node[k].x);
    }
    const int v0 = grp * a.v_per, v1 = min(a.V, v0 + a.v_per);
    for (int v = v0; v < v1; v++) {
        float zc[PPL], zs[PPL], w[PPL][kNu8W], pr[PPL], pi[PPL], qr[PPL], qi[PPL], tr[PPL], ti[PPL];
        int i0[PPL];
#pragma unroll
        for (int i = 0; i < PPL; i++) {
            const float alpha = alp[(size_t)v * a.rec.cap + pp[i]];
            const float gamma = gam[(size_t)v * a.rec.cap + pp[i]];
            const NodePoint pt = node_point(alpha, exact_gamma(alpha, gamma, a.nd.kappa, a.nd.inv_kappa), beta[i],
                                            epsd[i], cb, S);
            const double xf = floor(pt.x);
            i0[i] = min(max((int)xf + S, 0), 2 * S);   // row index of the first tap xf - 3 (clamped: NaN-safe)
            nu8_weights((float)(pt.x - xf - 0.5), w[i]);
            zs[i] = pt.zi;
            zc[i] = pt.zr;
            pr[i] = pi[i] = qr[i] = qi[i] = tr[i] = ti[i] = 0.0f;
        }
        const auto rows_v = gmem4(a.nu_rows) + (size_t)v * Q * RL;
        for (int q0 = 0; q0 < Q; q0 += stage) {
            const int nr = min(stage, Q - q0);
            if (!have_rows) {   // uniform over the block
                __syncthreads();   // the previous stage has been read
                for (int i = threadIdx.x; i < nr * RL; i += kNodeThreads) {
                    const F4 u = rows_v[(size_t)q0 * RL + i];
                    rsh[i] = make_float4(u.x, u.y, u.z, u.w);
                }
                if (TD) {
                    const auto t_v = gmem(a.td_rows) + ((size_t)v * Q + q0) * RL;
                    for (int i = threadIdx.x; i < nr * RL; i += kNodeThreads) {
                        const F2 u = t_v[i];
                        rs2[i] = make_float2(u.x, u.y);
                    }
                }
                __syncthreads();
            }
            for (int k = 0; k < nr; k++) {
                const float2 nd = a.nd.node[q0 + k];
#pragma unroll
                for (int i = 0; i < PPL; i++) {
                    const float4 *row = rsh + k * RL + i0[i];
                    float sx = 0.f, sy = 0.f, sz = 0.f, sw = 0.f, tx = 0.f, ty = 0.f;
#pragma unroll
                    for (int t = 0; t < kNu8W; t++) {
                        const float4 u = row[t];
                        sx = fmaf(w[i][t], u.x, sx);
                        sy = fmaf(w[i][t], u.y, sy);
                        sz = fmaf(w[i][t], u.z, sz);
                        sw = fmaf(w[i][t], u.w, sw);
                    }
                    if (TD) {
                        const float2 *row2 = rs2 + k * RL + i0[i];
#pragma unroll
                        for (int t = 0; t < kNu8W; t++) {
                            const float2 u = row2[t];
                            tx = fmaf(w[i][t], u.x, tx);
                            ty = fmaf(w[i][t], u.y, ty);
                        }
                    }
                    const float Lq = lp[i] * nd.y * __builtin_amdgcn_rcpf(0.5f * node_factor(tau[i], nd.x));
                    pr[i] = fmaf(Lq, sx, pr[i]);
                    pi[i] = fmaf(Lq, sy, pi[i]);
                    qr[i] = fmaf(Lq, sz, qr[i]);
                    qi[i] = fmaf(Lq, sw, qi[i]);
                    if (TD) {
                        tr[i] = fmaf(Lq, tx, tr[i]);
                        ti[i] = fmaf(Lq, ty, ti[i]);
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < PPL; i++) {
            // Q0 = z P, m = z Q (z = e^{2 pi j (alpha + cbar nu + g S/2)})
            const float q0r = zc[i] * pr[i] - zs[i] * pi[i], q0i = zc[i] * pi[i] + zs[i] * pr[i];
            const float mr = zc[i] * qr[i] - zs[i] * qi[i], mi = zc[i] * qi[i] + zs[i] * qr[i];
            abr[i] += q0r;
            abi[i] -= q0i;
            if (act[i]) tbar[(size_t)v * a.rec.cap + pp[i]] = -2.0f * (float)kPi * (Ax[i] * mi + Ay[i] * mr);
            if (TD) {
                const float nr2 = zc[i] * tr[i] - zs[i] * ti[i], ni = zc[i] * ti[i] + zs[i] * tr[i];
                tdb[i] = fmaf(-2.0f * (float)kPi, Ax[i] * ni + Ay[i] * nr2, tdb[i]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < PPL; i++)
        if (act[i]) {
            gmem(a.abar_part)[(size_t)grp * a.rec.cap + pp[i]] = F2{abr[i], abi[i]};
            if (TD) gmem(a.tdb_part)[(size_t)grp * a.rec.cap + pp[i]] = tdb[i];
        }
}

template <bool TD>
__device__ __forceinline__ void adj_item_node(const AdjArgs &a, float4 *rsh, const int P, const int grp,
                                              const int blk_p0) {
    const bool keep = a.v_per == 1 && node_stage(a.S, a.nd.q, TD) >= a.nd.q;
    const int end = min(P, blk_p0 + a.tile);
    for (int p0 = blk_p0; p0 < end; p0 += kNodeThreads * kNodePPL)
        adj_part_node<TD>(a, rsh, P, grp, p0, keep && p0 > blk_p0);
}

// Path-stationary adjoint of Eq. (8).  For each (path, v, c) the sums
//   P(x) = sum_s conj(G_s) x^s,  P'(x)   with x = e^{2 pi j delta}
// run by Horner's rule; with z0 = e^{2 pi j phi0}:
//   sum_s w_s = z0 P(x),  sum_s s w_s = z0 x P'(x),  w_s = conj(G_s) e^{j phi_s}
//   dL/dA    += conj(z0 P(x))                                  (Eq. 12)
//   dL/dtau  += -2 pi Im(A (fc z0 P + (slope/fs) z0 x P'))       (Eq. 11)
// Each lane carries PPL paths (256 apart) so every G sample read from LDS
// feeds 8 * PPL fused multiply-adds.
//
// Work items are (antenna group, tile of 256 * PPL paths) pairs, antenna group
// major; the number of live paths is only known on the device, so a grid of
// about one device-full of blocks takes items from an atomic counter until
// they run out (no blocks are launched for the empty path slots).
template <int PPL>
__device__ __forceinline__ void adj_item(const AdjArgs &a, float2 *gsh, const int P, const int grp,
                                         const int blk_p0) {
    const auto amp = gmem(a.rec.amp);
    const auto bet = gmem(a.rec.beta);
    const auto eps = gmem(a.rec.epsd);
    const auto alp = gmem(a.rec.alpha);
    const auto gam = gmem(a.rec.gamma);
    const auto tbar = gmem(a.tau_bar);
    int pp[PPL];
    bool act[PPL];
    float2 A[PPL];
    float beta[PPL], epsd[PPL], abr[PPL], abi[PPL], tdb[PPL];
#pragma unroll
    for (int i = 0; i < PPL; i++) {
        pp[i] = blk_p0 + i * 256 + threadIdx.x;
        act[i] = pp[i] < P;
        const int pc = act[i] ? pp[i] : blk_p0;
        A[i] = make_float2(amp[pc].x, amp[pc].y);
        beta[i] = bet[pc];
        epsd[i] = eps[pc];
        abr[i] = 0.0f;
        abi[i] = 0.0f;
        tdb[i] = 0.0f;
        pp[i] = pc;
    }
    const int v0 = grp * a.v_per, v1 = min(a.V, v0 + a.v_per);
    const int S = a.S;
    for (int v = v0; v < v1; v++) {
        float alpha[PPL], gamma[PPL], tb[PPL];
#pragma unroll
        for (int i = 0; i < PPL; i++) {
            alpha[i] = alp[(size_t)v * a.rec.cap + pp[i]];
            gamma[i] = gam[(size_t)v * a.rec.cap + pp[i]];
            tb[i] = 0.0f;
        }
        for (int c0 = 0; c0 < a.C; c0 += a.rows) {
            const int nr = min(a.rows, a.C - c0);
            __syncthreads();
            // rows padded with zeros to Sp = S rounded up to 8: leading zero
            // coefficients leave Horner's recurrences unchanged
            const auto src = gmem(a.G) + ((size_t)v * a.C + c0) * S;
            for (int i = threadIdx.x; i < nr * a.Sp; i += 256) {
                const int rr = i / a.Sp, ss = i - rr * a.Sp;
                if (ss < S) {
                    const F2 g = src[(size_t)rr * S + ss];
                    gsh[i] = make_float2(g.x, g.y);
                } else {
                    gsh[i] = make_float2(0.0f, 0.0f);
                }
            }
            __syncthreads();
            for (int cc = 0; cc < nr; cc++) {
                const int c = c0 + cc;
                const float cf = (float)c;
                float zs[PPL], zc[PPL], xs[PPL], xc[PPL], pr[PPL], pi[PPL], qr[PPL], qi[PPL];
#pragma unroll
                for (int i = 0; i < PPL; i++) {
                    const float delta = fmaf(cf, epsd[i], gamma[i]);
                    const float cb = cf * beta[i];
                    float ph = alpha[i] + fmaf(cf, beta[i], -rintf(cb));
                    ph -= rintf(ph);
                    zs[i] = __builtin_amdgcn_sinf(ph);
                    zc[i] = __builtin_amdgcn_cosf(ph);
                    const float dd = delta - rintf(delta);
                    xs[i] = __builtin_amdgcn_sinf(dd);
                    xc[i] = __builtin_amdgcn_cosf(dd);
                    pr[i] = pi[i] = qr[i] = qi[i] = 0.0f;
                }
                const float4 *g4 = reinterpret_cast<const float4 *>(gsh + cc * a.Sp);
                // q = q x + p ;  p = p x + conj(g_s), s descending
#define SBR_HORNER_STEP(GR, GI)                                                 \
    _Pragma("unroll") for (int i = 0; i < PPL; i++) {                          \
        float nqr = fmaf(qr[i], xc[i], fmaf(-qi[i], xs[i], pr[i]));            \
        float nqi = fmaf(qr[i], xs[i], fmaf(qi[i], xc[i], pi[i]));             \
        float npr = fmaf(pr[i], xc[i], fmaf(-pi[i], xs[i], (GR)));             \
        float npi = fmaf(pr[i], xs[i], fmaf(pi[i], xc[i], -(GI)));             \
        qr[i] = nqr;                                                           \
        qi[i] = nqi;                                                           \
        pr[i] = npr;                                                           \
        pi[i] = npi;                                                           \
    }
                for (int j = a.Sp / 2 - 4; j >= 0; j -= 4) {
                    const float4 h3 = g4[j + 3], h2 = g4[j + 2], h1 = g4[j + 1], h0 = g4[j];
                    SBR_HORNER_STEP(h3.z, h3.w)
                    SBR_HORNER_STEP(h3.x, h3.y)
                    SBR_HORNER_STEP(h2.z, h2.w)
                    SBR_HORNER_STEP(h2.x, h2.y)
                    SBR_HORNER_STEP(h1.z, h1.w)
                    SBR_HORNER_STEP(h1.x, h1.y)
                    SBR_HORNER_STEP(h0.z, h0.w)
                    SBR_HORNER_STEP(h0.x, h0.y)
                }
#undef SBR_HORNER_STEP
#pragma unroll
                for (int i = 0; i < PPL; i++) {
                    // Q0 = z0 P, Q1 = z0 x P'
                    const float q0r = zc[i] * pr[i] - zs[i] * pi[i], q0i = zc[i] * pi[i] + zs[i] * pr[i];
                    const float xqr = xc[i] * qr[i] - xs[i] * qi[i], xqi = xc[i] * qi[i] + xs[i] * qr[i];
                    const float q1r = zc[i] * xqr - zs[i] * xqi, q1i = zc[i] * xqi + zs[i] * xqr;
                    abr[i] += q0r;
                    abi[i] -= q0i;
                    const float mr = a.fcf * q0r + a.sl_fs * q1r;
                    const float mi = a.fcf * q0i + a.sl_fs * q1i;
                    const float dq = -2.0f * (float)kPi * (A[i].x * mi + A[i].y * mr);
                    tb[i] += dq;
                    tdb[i] += dq * (cf * a.tc);   // tau(c) = tau + c t_chirp taudot
                }
            }
        }
#pragma unroll
        for (int i = 0; i < PPL; i++)
            if (act[i]) tbar[(size_t)v * a.rec.cap + pp[i]] = tb[i];
    }
#pragma unroll
    for (int i = 0; i < PPL; i++)
        if (act[i]) {
            gmem(a.abar_part)[(size_t)grp * a.rec.cap + pp[i]] = F2{abr[i], abi[i]};
            gmem(a.tdb_part)[(size_t)grp * a.rec.cap + pp[i]] = tdb[i];
        }
}

// Work items of each request of a batch: (antenna groups) x (path tiles of
// args[i].tile paths) for its device-side path count; item_first[i] = first
// item of request i, item_first[n] = total.  Also clears the work counters of
// the adjoint forms and the requests' sums over rays.  One block.
__global__ __launch_bounds__(1024) void k_adj_items(const AdjArgs *args, int n, uint32_t *item_first,
                                                    uint32_t *queue) {
    __shared__ uint32_t part[1024];
    const int t = threadIdx.x;
    const int chunk = (n + 1023) / 1024;
    const int b = t * chunk, e = min(n, b + chunk);
    for (int i = 0; i < n; i++)
        if (args[i].acc && t < args[i].n_acc) args[i].acc[t] = 0.0;
    uint32_t sum = 0;
    for (int i = b; i < e; i++) {
        const uint32_t P = (uint32_t)args[i].count[0], tile = (uint32_t)args[i].tile;
        sum += (P + tile - 1u) / tile * (uint32_t)args[i].nvs;
    }
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    uint32_t run = part[t] - sum;
    for (int i = b; i < e; i++) {
        item_first[i] = run;
        const uint32_t P = (uint32_t)args[i].count[0], tile = (uint32_t)args[i].tile;
        run += (P + tile - 1u) / tile * (uint32_t)args[i].nvs;
    }
    if (t == 1023) item_first[n] = part[1023];
    if (t == 0) {
        queue[0] = 0u;
        queue[kAdjQueueDirect] = 0u;
        queue[kAdjQueueNode] = 0u;
    }
}

// Request of a work item: binary search over item_first[lo .. hi).
__device__ __forceinline__ int adj_request(const uint32_t *item_first, int lo, int hi, uint32_t item) {
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (item_first[mid] <= item) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Work items of requests [r0, r1) of a batch (one request for sbr_backward)
// are taken from one atomic counter by about one device-full of blocks; an
// item is mapped to its request by binary search over item_first, then to
// (antenna group, path tile) exactly as in a launch of its own.  `slot` is
// the LDS float2 offset of the work-item word (after the largest G-row stage).
template <int PPL>
__global__ __launch_bounds__(256) void k_synth_adj(const AdjArgs *__restrict__ args,
                                                   const uint32_t *__restrict__ item_first, int r0, int r1,
                                                   uint32_t *queue, int slot) {
    // [rows][Sp] G rows, then the current work item.  No static LDS: it would
    // shift the dynamic area off the 16-byte alignment of the row reads.
    extern __shared__ float2 gsh[];
    uint32_t &s_item = *reinterpret_cast<uint32_t *>(gsh + slot);
    const uint32_t first = item_first[r0], total = item_first[r1];
    for (;;) {
        __syncthreads();   // the previous item is done with s_item and gsh
        if (threadIdx.x == 0) s_item = first + atomicAdd(queue, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= total) break;   // uniform over the block
        const int lo = adj_request(item_first, r0, r1, item);
        const AdjArgs &a = args[lo];
        const int P = __builtin_amdgcn_readfirstlane(*gmem(a.count));
        const uint32_t tiles = (uint32_t)((P + 256 * PPL - 1) / (256 * PPL));
        const uint32_t local = item - item_first[lo];
        adj_item<PPL>(a, gsh, P, (int)(local / tiles), (int)(local % tiles) * 256 * PPL);
    }
}

// The same work queue over requests [r0, r1) for the non-uniform FFT form;
// `stage` rows of nu_row_len(S) float4 per LDS stage, the work-item word
// after the largest stage (float4 offset `slot`).
template <int PPL>
__global__ __launch_bounds__(256) void k_synth_adj_nu(const AdjArgs *__restrict__ args,
                                                      const uint32_t *__restrict__ item_first, int r0, int r1,
                                                      uint32_t *queue, int slot) {
    extern __shared__ float4 rsh[];
    uint32_t &s_item = *reinterpret_cast<uint32_t *>(rsh + slot);
    const uint32_t first = item_first[r0], total = item_first[r1];
    for (;;) {
        __syncthreads();   // the previous item is done with s_item and the rows
        if (threadIdx.x == 0) s_item = first + atomicAdd(queue, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= total) break;   // uniform over the block
        const int lo = adj_request(item_first, r0, r1, item);
        const AdjArgs &a = args[lo];
        const int P = __builtin_amdgcn_readfirstlane(*gmem(a.count));
        const uint32_t tiles = (uint32_t)((P + 256 * PPL - 1) / (256 * PPL));
        const uint32_t local = item - item_first[lo];
        adj_item_nu<PPL>(a, rsh, nu_stage(a.S), P, (int)(local / tiles), (int)(local % tiles) * 256 * PPL);
    }
}

// The same work queue over requests [r0, r1) for the node form; the work-item
// word lies after the largest stage (float4 offset `slot`).
template <bool TD>
__global__ __launch_bounds__(kNodeThreads) void k_synth_adj_node(const AdjArgs *__restrict__ args,
                                                                 const uint32_t *__restrict__ item_first, int r0,
                                                                 int r1, uint32_t *queue, int slot) {
    extern __shared__ float4 rsh[];
    uint32_t &s_item = *reinterpret_cast<uint32_t *>(rsh + slot);
    const uint32_t first = item_first[r0], total = item_first[r1];
    for (;;) {
        __syncthreads();   // the previous item is done with s_item and the rows
        if (threadIdx.x == 0) s_item = first + atomicAdd(queue, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= total) break;   // uniform over the block
        const int lo = adj_request(item_first, r0, r1, item);
        const AdjArgs &a = args[lo];
        const int P = __builtin_amdgcn_readfirstlane(*gmem(a.count));
        const uint32_t tiles = (uint32_t)((P + a.tile - 1) / a.tile);
        const uint32_t local = item - item_first[lo];
        adj_item_node<TD>(a, rsh, P, (int)(local / tiles), (int)(local % tiles) * a.tile);
    }
}

// For kSplitAntennas or more, per path: the partial sums of Abar (and
// taudot_bar where tpart is given) of the nvs antenna groups in their order, and
// the delay adjoints tau_bar[t n_rx + m] summed over m (rows 0 .. n_tx - 1) and
// over t (rows n_tx ..), all that the geometry adjoint needs of them, written
// over the path's column of tau_bar.  A block takes 64 paths, its wavefronts the
// n_tx + n_rx + 1 sums in turn (at most kSumsPer each).  A ray's lane in the
// geometry adjoint would walk the n_tx n_rx rows twice: 0.44 ms of it at 400
// antennas, 0.07 ms here; at 12 antennas the lane's own sums are the cheaper
// (0.15 ms where this kernel took 0.45 on the 2048^2-ray scene).
constexpr int kSumsWaves = 8;
constexpr int kSumsPer = (SBR_MAX_TX + SBR_MAX_RX + kSumsWaves) / kSumsWaves;

__global__ __launch_bounds__(64 * kSumsWaves) void k_path_sums(const int32_t *count, const float2 *part,
                                                               const float *tpart, int nvs, int cap, float2 *abar,
                                                               float *tdbar, float *tau_bar, int ntx, int nrx) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int P = count[0];
    if ((int)blockIdx.x * 64 >= P) return;   // uniform over the block
    const int p = (int)blockIdx.x * 64 + lane;
    const bool live = p < P;
    const int n_out = ntx + nrx;
    float out[kSumsPer];
#pragma unroll
    for (int i = 0; i < kSumsPer; i++) {
        const int o = w + i * kSumsWaves;
        float s = 0.0f;
        if (live && o < n_out) {
            const int n = o < ntx ? nrx : ntx, first = o < ntx ? o * nrx : o - ntx, step = o < ntx ? 1 : nrx;
            const float *src = tau_bar + (size_t)first * cap + p;
#pragma unroll 4
            for (int q = 0; q < n; q++) s += src[(size_t)q * step * cap];
        } else if (live && o == n_out) {
            float r = 0.0f, im = 0.0f, t = 0.0f;
#pragma unroll 4
            for (int q = 0; q < nvs; q++) {
                const float2 x = part[(size_t)q * cap + p];
                r += x.x;
                im += x.y;
                if (tpart) t += tpart[(size_t)q * cap + p];
            }
            abar[p] = make_float2(r, im);
            if (tpart) tdbar[p] = t;
        }
        out[i] = s;
    }
    __syncthreads();   // the columns have been read
#pragma unroll
    for (int i = 0; i < kSumsPer; i++) {
        const int o = w + i * kSumsWaves;
        if (live && o < n_out) tau_bar[(size_t)o * cap + p] = out[i];
    }
}

constexpr int kParamSums = 16;

// Blocks of the geometry adjoint from which on each takes several tiles of rays.
constexpr int kGeomBlocks = 2048;

struct GeomArgs {
    const float *verts;
    const int32_t *faces;
    const uint16_t *mat_id;
    const int32_t *tri;
    int32_t R;
    int32_t nf;
    MatTable mt;
    int32_t any_fresnel;
    RadarDev rd;
    GridDev g;
    ChirpDev ch;
    const int32_t *wave_first, *blk;   // path stage
    int32_t by_ray;                    // paths_by_ray
    const uint8_t *flags;
    int32_t drop, exit_only;
    // dL/dA: the sum of `parts` rows [cap]; dL/d taudot likewise, or NULL (no
    // wanted gradient depends on it)
    const float2 *abar;
    const float *tdbar;
    int32_t parts;
    // dL/dtau, rows of cap paths: TX t's leg takes the sum of the tx_n rows from
    // t tx_n, RX m's leg that of the rx_n rows rx_first + m + i n_rx
    const float *tau_bar;
    int32_t tx_n, rx_n, rx_first;
    int32_t tiles;          // tiles of 256 rays per block
    int32_t cap;
    float *grad;            // [nv][3]
    double *acc;            // [kParamSums + 2 n_mats] sums over rays: origin (3), velocity
                            // (3), rot (9), attenuation, materials; NULL: none wanted
    int32_t want_mats, want_rot;
    int32_t attached;       // 1: first hits follow their triangle (Eqs. 6-7)
    float txl[SBR_MAX_TX][3];   // antenna positions in the radar frame
    float rxl[SBR_MAX_RX][3];
};

__device__ __forceinline__ float3 f3(float x, float y, float z) { return make_float3(x, y, z); }
__device__ __forceinline__ float3 operator+(float3 a, float3 b) { return f3(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ __forceinline__ float3 operator-(float3 a, float3 b) { return f3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ float3 operator*(float s, float3 a) { return f3(s * a.x, s * a.y, s * a.z); }
__device__ __forceinline__ float dot3(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ float3 cross3(float3 a, float3 b) {
    return f3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ float len3(float3 a) { return sqrtf(dot3(a, a)); }
__device__ __forceinline__ float3 vload3(const float *v, int i) { return f3(v[3 * i], v[3 * i + 1], v[3 * i + 2]); }

// A block's vertex gradients, collected in LDS and added to global memory once
// per block and vertex: the large faces of a scene are hit by every wavefront,
// and atomics on the same few lines of memory are served one after another
// (1.4 of 1.8 ms on the 2048^2-ray scene).  Open addressing over kVtxSlots
// slots; a vertex that finds none in kVtxProbes goes to global memory.
constexpr int kVtxSlots = 1024;
constexpr int kVtxProbes = 4;

struct VtxTable {
    int key[kVtxSlots];
    float g[kVtxSlots][3];
};

__device__ __forceinline__ void atomic_add3(VtxTable &tab, float *g, int vi, float3 x) {
    float *dst = nullptr;
    uint32_t slot = (uint32_t)vi * 2654435761u >> 22;   // 10 bits
#pragma unroll
    for (int i = 0; i < kVtxProbes; i++) {
        if (!dst) {
            int k = tab.key[slot];
            if (k < 0) {
                k = atomicCAS(&tab.key[slot], -1, vi);
                if (k < 0) k = vi;
            }
            if (k == vi) dst = tab.g[slot];
            slot = (slot + 1) & (kVtxSlots - 1);
        }
    }
    if (dst) {
        atomicAdd(&dst[0], x.x);
        atomicAdd(&dst[1], x.y);
        atomicAdd(&dst[2], x.z);
        return;
    }
    atomicAdd(&g[3 * vi], x.x);
    atomicAdd(&g[3 * vi + 1], x.y);
    atomicAdd(&g[3 * vi + 2], x.z);
}

// x of the lane N below in the same row of 16 lanes, 0 past the row's start.
template <int N>
__device__ __forceinline__ int row_up(int x) {
    return __builtin_amdgcn_update_dpp(0, x, 0x110 | N, 0xf, 0xf, true);   // row_shr:N
}

// Sum of x over the lanes of its row from the start of the run on (in[i]: the
// lane 2^i below is in the run); complete in the last lane of the run.
__device__ __forceinline__ float run_sum(float x, const bool (&in)[4]) {
    float y = __int_as_float(row_up<1>(__float_as_int(x)));
    x += in[0] ? y : 0.0f;
    y = __int_as_float(row_up<2>(__float_as_int(x)));
    x += in[1] ? y : 0.0f;
    y = __int_as_float(row_up<4>(__float_as_int(x)));
    x += in[2] ? y : 0.0f;
    y = __int_as_float(row_up<8>(__float_as_int(x)));
    return x + (in[3] ? y : 0.0f);
}

// Per ray: single-precision forward recompute of its bounces from the face
// ids (nothing is stored per path), path adjoints -> dL/dx_j and dL/dcos_j,
// then one reverse sweep through x = o + t d, t = N.(a - o)/(N.d), the
// specular reflection, the normalisation and the cross product, Fresnel
// coefficients included.  Rays of a wavefront are consecutive in a grid row,
// so neighbouring lanes often hit the same face: their vertex gradients are
// summed over runs of equal face ids first and added by one atomic per run.
// The gradients summed over all rays (origin, velocity, rotation,
// attenuation) are returned in sum[16] where wanted.
template <int K, bool FULL>
__device__ __forceinline__ void geom_ray(const GeomArgs &a, VtxTable &tab, const int r, const int lane,
                                         float (&sum)[kParamSums]) {
    int n = 0;                          // bounces to recompute (last returning one + 1)
    uint32_t mask = 0;                  // bounces that return a path
    if (r < a.R) {
        mask = ray_path_mask(a.tri, a.flags, (size_t)a.R, (size_t)r, a.g.K, a.nf, a.drop != 0, a.exit_only != 0, &n);
    }
    if (__ballot(n > 0) == 0) return;   // uniform over the wavefront
    const int wave = __builtin_amdgcn_readfirstlane(r / kPathWave);
    const int first = a.wave_first[wave] + a.blk[wave / (kPathBlock / kPathWave)];
    PathRank rank(mask, K, a.by_ray != 0);
    const int ix = r % a.g.nx, iy = r / a.g.nx;
    double d0[3], dl[3], dwd;
    grid_dir_local(a.g, ix, iy, dl, &dwd);
    for (int i = 0; i < 3; i++) d0[i] = a.rd.rot[3 * i] * dl[0] + a.rd.rot[3 * i + 1] * dl[1] + a.rd.rot[3 * i + 2] * dl[2];
    const float dw = (float)dwd;
    const float3 O = f3((float)a.rd.o[0], (float)a.rd.o[1], (float)a.rd.o[2]);
    // ---- forward recompute, cached per bounce
    float3 X[K], D[K];
    float T[K], CI[K], SG[K], LC[K];
    float2 RC[K], DRC[K], DEPS[K];
    int F[K], MAT[K];
    // FULL = false: conductors only (r = -1 at every bounce, no derivatives) and
    // no gradients but the vertices'
    const bool fresnel = FULL && a.any_fresnel;
    float3 dir = f3((float)d0[0], (float)d0[1], (float)d0[2]);
    float3 o = O;
    float L = 0.0f;
#pragma unroll
    for (int k = 0; k < K; k++) {
        F[k] = -1;
        MAT[k] = -1;
        if (k < n) {
            const int f = a.tri[(size_t)k * a.R + r];
            const float3 va = vload3(a.verts, a.faces[3 * f]);
            const float3 e1 = vload3(a.verts, a.faces[3 * f + 1]) - va;
            const float3 e2 = vload3(a.verts, a.faces[3 * f + 2]) - va;
            const float3 N = cross3(e1, e2);
            const float den = dot3(N, dir);
            const float t = dot3(N, va - o) / den;
            const float3 x = o + t * dir;
            L += len3(x - o);
            const float nl = len3(N);
            const float dn = den / nl;
            X[k] = x;
            D[k] = dir;
            T[k] = t;
            LC[k] = L;
            F[k] = f;
            CI[k] = fabsf(dn);
            SG[k] = dn >= 0.0f ? 1.0f : -1.0f;
            cd rc = {-1.0, 0.0}, drc = {0.0, 0.0}, de = {0.0, 0.0};
            const int mi = a.mat_id ? (int)a.mat_id[f] : 0;
            if (fresnel) {
                reflect_coef(a.mt, mi, a.ch.fc, (double)CI[k], rc, drc);
                if (a.want_mats) de = reflect_deps(a.mt, mi, a.ch.fc, (double)CI[k]);
                if (mi < a.mt.n && a.mt.mode[mi] != 0) MAT[k] = mi;
            }
            RC[k] = make_float2((float)rc.re, (float)rc.im);
            DRC[k] = make_float2((float)drc.re, (float)drc.im);
            DEPS[k] = make_float2((float)de.re, (float)de.im);
            dir = dir - (2.0f * dn / nl) * N;
            o = x;
        }
    }
    // ---- path adjoints -> dL/dx_j, dL/dcos_j
    float3 xb[K];
    float cib[K];
    float2 gm[K];                           // dL/d (eps_r, sigma) of the material at bounce j
    float3 go = f3(0.f, 0.f, 0.f);          // dL/d radar origin
    float3 gu = f3(0.f, 0.f, 0.f);          // dL/d scene velocity
    float3 gd0 = f3(0.f, 0.f, 0.f);         // dL/d first ray direction (Doppler part)
    float gR[9];                            // dL/d rot from the antenna positions
#pragma unroll
    for (int q = 0; q < 9; q++) gR[q] = 0.0f;
    const bool want_rot = FULL && a.want_rot != 0;
    float wJ = 0.0f;                        // sum over the ray's paths of Re(conj(Abar) A)
    const float atn = (float)a.rd.atten;
    float ga_atn = 0.0f;                    // dL/d attenuation
    // directional gains F(d_0) G(x_k - o) of Eq. 1, cos^n about the boresight zb
    const float ntg = (float)a.rd.n_tg, nrg = (float)a.rd.n_rg;
    const float3 ZB = f3((float)a.rd.rot[2], (float)a.rd.rot[5], (float)a.rd.rot[8]);
    const float3 D0 = f3((float)d0[0], (float)d0[1], (float)d0[2]);
    const float ctx = dot3(D0, ZB);
    const float Fg = ntg == 0.0f ? 1.0f : (ctx > 0.0f ? __powf(ctx, ntg) : 0.0f);
    float3 gZ = f3(0.f, 0.f, 0.f);          // dL/d boresight vector (world)
    const float3 U = f3((float)a.rd.vel[0], (float)a.rd.vel[1], (float)a.rd.vel[2]);
#pragma unroll
    for (int k = 0; k < K; k++) {
        xb[k] = f3(0.f, 0.f, 0.f);
        cib[k] = 0.0f;
        gm[k] = make_float2(0.f, 0.f);
    }
    const float inv_we0 = (float)(1.0 / (2.0 * kPi * a.ch.fc * kEps0));
    const int ntx = a.rd.n_tx, nrx = a.rd.n_rx;
    const float ic0 = (float)(1.0 / kC0);
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int p = first + rank.next(k);
        if ((mask >> k) & 1u) {
            float2 ab = make_float2(0.f, 0.f);
#pragma unroll 4
            for (int i = 0; i < a.parts; i++) {
                const float2 x = a.abar[(size_t)i * a.cap + p];
                ab.x += x.x;
                ab.y += x.y;
            }
            float2 prod = make_float2(k & 1 ? 1.0f : -1.0f, 0.0f);
            if (FULL) prod = make_float2(1.0f, 0.0f);
#pragma unroll
            for (int j = 0; j <= k; j++)
                if (FULL) prod = make_float2(prod.x * RC[j].x - prod.y * RC[j].y, prod.x * RC[j].y + prod.y * RC[j].x);
            const float3 qk = X[k] - O;
            const float Rk = len3(qk);
            const float qz = dot3(qk, ZB);
            const float Gg = nrg == 0.0f ? 1.0f : (qz > 0.0f ? __powf(qz / Rk, nrg) : 0.0f);
            // A = dw prod ci_k exp(-a (L + R)) F G / (L R);  u = Re(conj(Abar) A / ci_k)
            const float sc = dw / (LC[k] * Rk) * __expf(-atn * (LC[k] + Rk)) * (Fg * Gg);
            const float u = sc * (ab.x * prod.x + ab.y * prod.y);
            const float gk = u * CI[k];
            wJ += gk;                               // Re(conj(Abar) A): dL/d log(cell weight)
            cib[k] += u;
            const float Lb = -gk / LC[k] - atn * gk, Rb = -gk / Rk - atn * gk;
            ga_atn -= gk * (LC[k] + Rk);            // d A / d a = -(L + R) A
            if (nrg != 0.0f && qz > 0.0f) {         // log G = n (log(q.zb) - log |q|)
                const float3 t = nrg * ((1.0f / qz) * ZB - (1.0f / (Rk * Rk)) * qk);
                xb[k] = xb[k] + gk * t;
                go = go - gk * t;
                gZ = gZ + (gk * nrg / qz) * qk;
            }
            if (ntg != 0.0f && ctx > 0.0f) {        // log F = n log(d_0.zb)
                gd0 = gd0 + (gk * ntg / ctx) * ZB;
                gZ = gZ + (gk * ntg / ctx) * D0;
            }
            if (fresnel) {
#pragma unroll
                for (int j = 0; j <= k; j++) {
                    float2 ex = make_float2(sc * CI[k], 0.0f);
#pragma unroll
                    for (int i = 0; i <= k; i++)
                        if (i != j) ex = make_float2(ex.x * RC[i].x - ex.y * RC[i].y, ex.x * RC[i].y + ex.y * RC[i].x);
                    const float2 dA = make_float2(ex.x * DRC[j].x - ex.y * DRC[j].y, ex.x * DRC[j].y + ex.y * DRC[j].x);
                    cib[j] += ab.x * dA.x + ab.y * dA.y;
                    if (a.want_mats) {
                        // eps_c = eps_r - j sigma / (omega eps_0): d/deps_r = d/deps_c,
                        // d/dsigma = -j / (omega eps_0) d/deps_c
                        const float2 W = make_float2(ex.x * DEPS[j].x - ex.y * DEPS[j].y,
                                                     ex.x * DEPS[j].y + ex.y * DEPS[j].x);
                        gm[j].x += ab.x * W.x + ab.y * W.y;
                        gm[j].y += (ab.x * W.y - ab.y * W.x) * inv_we0;
                    }
                }
            }
            float3 prv = O;
#pragma unroll
            for (int j = 0; j <= k; j++) {
                const float3 sg = X[j] - prv;
                const float3 uj = (Lb / len3(sg)) * sg;
                xb[j] = xb[j] + uj;
                if (j > 0) xb[j - 1] = xb[j - 1] - uj;
                else go = go - uj;                  // first segment starts at the origin
                prv = X[j];
            }
            xb[k] = xb[k] + (Rb / Rk) * (X[k] - O);
            // the TX leg of antenna (t, m) moves with the sum over m of its
            // delay adjoints, the RX leg with the sum over t
            const float *tbp = a.tau_bar + p;
            float Tt = 0.0f;
            auto tx_leg = [&](int t, float ts) {
                const float3 q = X[0] - f3((float)a.rd.tx[t][0], (float)a.rd.tx[t][1], (float)a.rd.tx[t][2]);
                const float3 gq = (ts * ic0 / len3(q)) * q;
                xb[0] = xb[0] + gq;
                go = go - gq;                       // TX positions move with the origin
                if (want_rot) {                     // tx_world = origin + rot tx_local
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        gR[c] -= gq.x * a.txl[t][c];
                        gR[3 + c] -= gq.y * a.txl[t][c];
                        gR[6 + c] -= gq.z * a.txl[t][c];
                    }
                }
            };
            auto rx_leg = [&](int m, float rs) {
                const float3 q = X[k] - f3((float)a.rd.rx[m][0], (float)a.rd.rx[m][1], (float)a.rd.rx[m][2]);
                const float3 gq = (rs * ic0 / len3(q)) * q;
                xb[k] = xb[k] + gq;
                go = go - gq;                       // RX positions move with the origin
                if (want_rot) {
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        gR[c] -= gq.x * a.rxl[m][c];
                        gR[3 + c] -= gq.y * a.rxl[m][c];
                        gR[6 + c] -= gq.z * a.rxl[m][c];
                    }
                }
            };
            for (int t = 0; t < ntx; t++) {
                float ts = 0.0f;
#pragma unroll 4
                for (int i = 0; i < a.tx_n; i++) ts += tbp[(size_t)(t * a.tx_n + i) * a.cap];
                Tt += ts;
                tx_leg(t, ts);
            }
            for (int m = 0; m < nrx; m++) {
                float rs = 0.0f;
#pragma unroll 4
                for (int i = 0; i < a.rx_n; i++) rs += tbp[(size_t)(a.rx_first + m + i * nrx) * a.cap];
                rx_leg(m, rs);
            }
            go = go - (Rb / Rk) * (X[k] - O);        // R_k = |x_k - origin|
            // taudot = 2 (u . d_1) / c
            float tdq = 0.0f;
            if (a.tdbar) {
                for (int i = 0; i < a.parts; i++) tdq += a.tdbar[(size_t)i * a.cap + p];
                tdq *= 2.0f * ic0;
            }
            gu = gu + tdq * f3((float)d0[0], (float)d0[1], (float)d0[2]);
            gd0 = gd0 + tdq * U;
#pragma unroll
            for (int j = 1; j <= k; j++) {
                const float3 sg = X[j] - X[j - 1];
                const float3 uj = (Tt * ic0 / len3(sg)) * sg;
                xb[j] = xb[j] + uj;
                xb[j - 1] = xb[j - 1] - uj;
            }
        }
    }
    // ---- reverse sweep over bounces
    float3 dnext = f3(0.f, 0.f, 0.f);   // dL/d d_{j+1}
#pragma unroll
    for (int j = K - 1; j >= 0; j--) {
        const bool act = j < n;
        float3 ga = f3(0.f, 0.f, 0.f), gb = ga, gc = ga;
        if (act && j == 0 && a.attached) {
            // Eqs. 6-7 with T attached to the first hit: x_0 = a + b1 e1 + b2 e2 at
            // fixed (b1, b2), d_0 = (x_0 - o) / |x_0 - o|, cell weight times
            // D / D_0 with D = |N . (x_0 - o)| / |x_0 - o|^3
            const float3 va = vload3(a.verts, a.faces[3 * F[0]]);
            const float3 e1 = vload3(a.verts, a.faces[3 * F[0] + 1]) - va;
            const float3 e2 = vload3(a.verts, a.faces[3 * F[0] + 2]) - va;
            const float3 N = cross3(e1, e2);
            const float nl = len3(N);
            const float3 nh = (1.0f / nl) * N;
            const float3 d = D[0];
            const float dn = dot3(d, nh);
            const float3 q = X[0] - O;
            const float r0 = len3(q);
            const float nn = dot3(N, N);
            const float3 w0 = X[0] - va;
            const float b1 = dot3(cross3(w0, e2), N) / nn, b2 = dot3(cross3(e1, w0), N) / nn;
            float3 db = (cib[0] * SG[0]) * nh + gd0;   // cos_0 = |d_0 . n|, Doppler 2 u.d_0 / c
            float3 nhb = (cib[0] * SG[0]) * d;
            const float ndn = dot3(nh, dnext);          // d_1 = d_0 - 2 (d_0.n) n
            db = db + dnext - (2.0f * ndn) * nh;
            nhb = nhb - 2.0f * (dn * dnext + ndn * d);
            const float3 dq = (1.0f / r0) * (db - dot3(db, d) * d);
            const float sN = dot3(N, q);
            const float3 lj = wJ * ((1.0f / sN) * N - (3.0f / (r0 * r0)) * q);
            const float3 xb0 = xb[0] + dq + lj;
            go = go - dq - lj;
            const float3 Nb = (wJ / sN) * q + (1.0f / nl) * (nhb - dot3(nhb, nh) * nh);
            const float3 gbN = cross3(e2, Nb), gcN = cross3(Nb, e1);
            ga = (1.0f - b1 - b2) * xb0 - gbN - gcN;
            gb = b1 * xb0 + gbN;
            gc = b2 * xb0 + gcN;
            dnext = f3(0.f, 0.f, 0.f);                  // d_0 no longer depends on the grid
            gd0 = f3(0.f, 0.f, 0.f);
        } else if (act) {
            const float3 va = vload3(a.verts, a.faces[3 * F[j]]);
            const float3 e1 = vload3(a.verts, a.faces[3 * F[j] + 1]) - va;
            const float3 e2 = vload3(a.verts, a.faces[3 * F[j] + 2]) - va;
            const float3 N = cross3(e1, e2);
            const float nl = len3(N);
            const float3 nh = (1.0f / nl) * N;
            const float3 d = D[j];
            const float dn = dot3(d, nh);
            const float t = T[j];
            float3 ob = xb[j];                     // x = o + t d
            const float tbar = dot3(xb[j], d);
            float3 db = t * xb[j];
            float3 nhb = (cib[j] * SG[j]) * d;      // cos = |d . n|
            db = db + (cib[j] * SG[j]) * nh;
            const float ndn = dot3(nh, dnext);      // d_{j+1} = d - 2 (d.n) n
            db = db + dnext - (2.0f * ndn) * nh;
            nhb = nhb - 2.0f * (dn * dnext + ndn * d);
            const float den = dot3(N, d);           // t = N.(a - o) / (N.d)
            const float w = tbar / den;
            float3 Nb = w * (va - X[j]);
            ga = w * N;
            ob = ob - w * N;
            db = db - (w * t) * N;
            Nb = Nb + (1.0f / nl) * (nhb - dot3(nhb, nh) * nh);   // n = N / |N|
            gb = cross3(e2, Nb);                    // N = e1 x e2
            gc = cross3(Nb, e1);
            ga = ga - gb - gc;
            if (j > 0) xb[j - 1] = xb[j - 1] + ob;
            else go = go + ob;                      // rays start at the origin
            dnext = db;
        }
        // sum over runs of lanes of a 16-lane row that hit the same face (DPP moves:
        // no LDS traffic), one addition to the table per run
        const int key = act ? F[j] : -1;
        const int l16 = lane & 15;
        const int kprev = row_up<1>(key);   // with all lanes active
        int s0 = (l16 == 0 || kprev != key) ? l16 : 0;
        s0 = max(s0, row_up<1>(s0));
        s0 = max(s0, row_up<2>(s0));
        s0 = max(s0, row_up<4>(s0));
        s0 = max(s0, row_up<8>(s0));
        const bool in[4] = {l16 - 1 >= s0, l16 - 2 >= s0, l16 - 4 >= s0, l16 - 8 >= s0};
        const int knext = __builtin_amdgcn_update_dpp(0, key, 0x101, 0xf, 0xf, true);   // row_shl:1
        const bool tail = act && (l16 == 15 || knext != key);
        float v9[9] = {ga.x, ga.y, ga.z, gb.x, gb.y, gb.z, gc.x, gc.y, gc.z};
#pragma unroll
        for (int q = 0; q < 9; q++) v9[q] = run_sum(v9[q], in);
        if (tail) {
            const int f = F[j];
            atomic_add3(tab, a.grad, a.faces[3 * f], f3(v9[0], v9[1], v9[2]));
            atomic_add3(tab, a.grad, a.faces[3 * f + 1], f3(v9[3], v9[4], v9[5]));
            atomic_add3(tab, a.grad, a.faces[3 * f + 2], f3(v9[6], v9[7], v9[8]));
        }
        if (FULL && a.want_mats) {
            // one wavefront sum per distinct material of this bounce
            const int km = act ? MAT[j] : -1;
            uint64_t pending = __ballot(km >= 0);
            while (pending) {
                const int leader = __ffsll((unsigned long long)pending) - 1;
                const int m = __shfl(km, leader);
                const bool mine = km == m;
                double e0 = mine ? (double)gm[j].x : 0.0, e1 = mine ? (double)gm[j].y : 0.0;
                for (int off = 32; off >= 1; off >>= 1) {
                    e0 += __shfl_xor(e0, off);
                    e1 += __shfl_xor(e1, off);
                }
                if (lane == leader) {
                    atomicAdd(&a.acc[kParamSums + 2 * m], e0);
                    atomicAdd(&a.acc[kParamSums + 2 * m + 1], e1);
                }
                pending &= ~__ballot(mine);
            }
        }
    }
    if (FULL && a.acc) {
        // d_0 = rot d_local: dL/drot += (dL/dd_0) d_local^T, where dL/dd_0 is
        // what the reverse sweep left for the first segment plus the Doppler part;
        // zb = rot e_z: the gains add dL/dzb to the third column
        const float3 g0 = dnext + gd0;
        const float l0 = (float)dl[0], l1 = (float)dl[1], l2 = (float)dl[2];
        const float v16[kParamSums] = {go.x, go.y, go.z, gu.x, gu.y, gu.z,
                                       gR[0] + g0.x * l0, gR[1] + g0.x * l1, gR[2] + g0.x * l2 + gZ.x,
                                       gR[3] + g0.y * l0, gR[4] + g0.y * l1, gR[5] + g0.y * l2 + gZ.y,
                                       gR[6] + g0.z * l0, gR[7] + g0.z * l1, gR[8] + g0.z * l2 + gZ.z, ga_atn};
#pragma unroll
        for (int q = 0; q < kParamSums; q++) sum[q] = v16[q];
    }
}

// A block takes a.tiles consecutive tiles of 256 rays, so that its vertex table
// holds what many wavefronts add to the same vertices.  The sums over rays are
// taken in FP64 (wavefronts, the block, then one atomic per block and sum into
// a.acc): they cancel, and in FP32 their value depended on the order of the
// atomics at 1e-6.
template <int K, bool FULL>
__global__ __launch_bounds__(256) void k_geom_adj(GeomArgs a) {
    __shared__ VtxTable tab;
    __shared__ double sh[4][kParamSums];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int i = tid; i < kVtxSlots; i += 256) {
        tab.key[i] = -1;
        tab.g[i][0] = tab.g[i][1] = tab.g[i][2] = 0.0f;
    }
    __syncthreads();
    const bool sums = FULL && a.acc;   // uniform over the grid
    double acc = 0.0;
    for (int i = 0; i < a.tiles; i++) {
        const int tile = (int)blockIdx.x * a.tiles + i;
        if (tile * 256LL >= a.R) break;
        float sum[kParamSums];
#pragma unroll
        for (int q = 0; q < kParamSums; q++) sum[q] = 0.0f;
        geom_ray<K, FULL>(a, tab, tile * 256 + tid, lane, sum);
        if (!sums) continue;
#pragma unroll
        for (int q = 0; q < kParamSums; q++) {
            double d = (double)sum[q];
            for (int off = 32; off >= 1; off >>= 1) d += __shfl_xor(d, off);
            if (lane == 0) sh[w][q] = d;
        }
        __syncthreads();
        if (tid < kParamSums) acc += (sh[0][tid] + sh[1][tid]) + (sh[2][tid] + sh[3][tid]);
        __syncthreads();
    }
    if (sums && tid < kParamSums) atomicAdd(&a.acc[tid], acc);
    __syncthreads();
    for (int i = tid; i < kVtxSlots; i += 256) {
        const int v = tab.key[i];
        if (v < 0) continue;
#pragma unroll
        for (int c = 0; c < 3; c++) atomicAdd(&a.grad[3 * v + c], tab.g[i][c]);
    }
}

// The parameter gradients wanted += the sums over rays.
__global__ void k_param_add(const double *acc, int n_mats, float *g_mats, float *g_radar, float *g_rot,
                            float *g_atten) {
    const int q = threadIdx.x;
    if (q < 6) {
        if (g_radar) g_radar[q] += (float)acc[q];
    } else if (q < 15) {
        if (g_rot) g_rot[q - 6] += (float)acc[q];
    } else if (q == 15) {
        if (g_atten) g_atten[0] += (float)acc[q];
    } else if (q < kParamSums + 2 * n_mats) {
        if (g_mats) g_mats[q - kParamSums] += (float)acc[q];
    }
}

}  // namespace

struct BackPlan {
    int nvs, v_per;
};

// One antenna per block row (grid.y) unless the per-row partial sums of Abar
// and taudot_bar (12 bytes per path and row) would pass 4 GiB: the number of
// live paths is only known on the device, and splitting over antennas keeps
// the launch full when few of the `cap` slots hold paths.
static BackPlan back_plan(long long cap, int V) {
    const long long budget = 4LL << 30;
    int v_per = 1;
    while (v_per < V && (long long)((V + v_per - 1) / v_per) * cap * 12 > budget) v_per++;
    const int nvs = (V + v_per - 1) / v_per;
    return {nvs, v_per};
}

// Whether a request's adjoint sums run as the non-uniform FFT form.
static bool use_nu(int32_t S, int32_t flags) { return nu_size(S) && !(flags & SBR_DIRECT_SUMS); }

// Adjoint buffers after the path stage: tau_bar, Abar and taudot_bar partials
// and sums, then (for chirps of kNuMinS .. kNuMaxS samples, whatever the
// flags) the 1/Psi table and the non-uniform FFT rows.
struct BackExtra {
    float *tau_bar;
    float2 *part, *abar;
    float *tpart, *tdbar;
    double *acc;
    float *corr;
    float4 *rows;
    size_t bytes;
};

static BackExtra back_extra(void *buf, int32_t R, int32_t K, int32_t V, int32_t C, int32_t S) {
    const long long cap = (long long)R * K;
    const BackPlan bp = back_plan(cap, V);
    const bool sums = V >= kSplitAntennas;
    Carver cv(buf);
    BackExtra e;
    e.tau_bar = cv.take<float>((size_t)V * cap);
    e.part = cv.take<float2>((size_t)bp.nvs * cap);
    e.abar = cv.take<float2>(sums ? cap : 0);
    e.tpart = cv.take<float>((size_t)bp.nvs * cap);
    e.tdbar = cv.take<float>(sums ? cap : 0);
    e.acc = cv.take<double>(kParamSums + 2 * SBR_MAX_MATERIALS);
    e.corr = nullptr;
    e.rows = nullptr;
    if (nu_size(S)) {
        e.corr = cv.take<float>((size_t)S);
        e.rows = cv.take<float4>((size_t)V * C * nu_row_len(S));
    }
    e.bytes = align_up(cv.off, 256);
    return e;
}

size_t backward_extra_bytes(int32_t R, int32_t K, int32_t V, int32_t C, int32_t S) {
    return back_extra(nullptr, R, K, V, C, S).bytes;
}

// Device table of a batched adjoint: the requests' arguments, their first
// work items and the work counter.
struct AdjTable {
    AdjArgs *args;
    uint32_t *item_first;
    uint32_t *queue;
    int32_t *row_first;   // first G row of each request of the chirp-row form
    int32_t *node_first;  // first node row of each request of the node form
};

static AdjTable adj_table(void *buf, int n, size_t *bytes) {
    Carver cv(buf);
    AdjTable t;
    t.args = cv.take<AdjArgs>(n);
    t.item_first = cv.take<uint32_t>((size_t)n + 1);
    t.queue = cv.take<uint32_t>(64);
    t.row_first = cv.take<int32_t>((size_t)n + 1);
    t.node_first = cv.take<int32_t>((size_t)n + 1);
    if (bytes) *bytes = align_up(cv.off, 256);
    return t;
}

size_t adj_table_bytes(int n) {
    size_t b = 0;
    adj_table(nullptr, n, &b);
    return b;
}

// G rows per LDS stage of a request with S samples, with the 16-byte
// work-item slot after them, within 64 KiB of LDS per block.
static int adj_rows(int Sp) { return std::max(1, std::min<int>(kAdjRowsMax, (65536 - 16) / (int)(sizeof(float2) * Sp))); }

template <int K = 1>
static void launch_geom(const GeomArgs &g, dim3 grid, hipStream_t s) {
    if constexpr (K < SBR_MAX_BOUNCES) {
        if (g.g.K != K) return launch_geom<K + 1>(g, grid, s);
    }
    if (g.any_fresnel || g.acc) hipLaunchKernelGGL((k_geom_adj<K, true>), grid, dim3(256), 0, s, g);
    else hipLaunchKernelGGL((k_geom_adj<K, false>), grid, dim3(256), 0, s, g);
}

// Paths per work item of the node form: 1024, and up to eight times as many
// while the path slots give 16384 items (a tenth of the slots may hold paths,
// and about 512 blocks take the items).  An item's rows cost as much to load as
// a few hundred of its paths: 2048^2 rays, 12 antennas, 16.8M slots 1.77 -> 1.44
// ms (four times: 1.46), 1024^2 rays, 3.1M slots 97 -> 86 us (twice).
static int node_tile(long long cap, int nvs) {
    constexpr int part = kNodeThreads * kNodePPL;
    return part * (int)std::max(1LL, std::min(8LL, cap * nvs / part / 16384));
}

int launch_backward_batch(const BackwardReq *reqs, int n, void *table, hipStream_t s) {
    if (n <= 0) return SBR_OK;
    // requests of the node form first, then those of the chirp-row form, then
    // those of the direct one
    std::vector<NodePlan> plans(n);
    std::vector<int> order;
    for (int r = 0; r < n; r++)
        if (use_nu(reqs[r].cd.S, reqs[r].flags)) plans[r] = node_plan(reqs[r].rd, reqs[r].gd, reqs[r].cd);
    for (int r = 0; r < n; r++)
        if (plans[r].q) order.push_back(r);
    const int n_node = (int)order.size();
    for (int r = 0; r < n; r++)
        if (!plans[r].q && use_nu(reqs[r].cd.S, reqs[r].flags)) order.push_back(r);
    const int n_nu = (int)order.size();
    for (int r = 0; r < n; r++)
        if (!use_nu(reqs[r].cd.S, reqs[r].flags)) order.push_back(r);
    std::vector<AdjArgs> aa(n);
    std::vector<GeomArgs> gg(n);
    size_t lds_f2 = 0;   // float2 words of the largest G-row stage
    long long items_node = 0, items_nu = 0, items_direct = 0;
    bool any_td = false;
    for (int r = 0; r < n; r++) {
        const BackwardReq &q = reqs[order[r]];
        const RadarDev &rd = q.rd;
        const int V = rd.n_tx * rd.n_rx;
        const long long cap = q.st.rec.cap;
        const bool node = r < n_node, nu = r < n_nu;
        // the taudot adjoint reaches the velocity, the ray directions and,
        // through the attached first hit, the vertices
        const bool td = (q.flags & SBR_ATTACHED) || (q.params && (q.params->radar || q.params->rot));
        BackPlan bp = back_plan(cap, V);
        const BackExtra e = back_extra(q.extra, q.gd.nx * q.gd.ny, q.gd.K, V, q.cd.C, q.cd.S);
        AdjArgs &a = aa[r];
        a.count = q.st.count;
        a.rec = q.st.rec;
        a.G = q.G;
        a.V = V;
        a.C = q.cd.C;
        a.S = q.cd.S;
        a.v_per = bp.v_per;
        a.nvs = bp.nvs;
        a.tile = node ? node_tile(cap, bp.nvs) : nu ? 256 * kNuPPL : 256 * kAdjPPL;
        a.fcf = (float)q.cd.fc;
        a.sl_fs = (float)(q.cd.slope / q.cd.fs);
        a.tc = (float)q.cd.tc;
        a.tau_bar = e.tau_bar;
        a.abar_part = e.part;
        a.tdb_part = e.tpart;
        a.nu_rows = nu ? e.rows : nullptr;
        a.nu_corr = nu ? e.corr : nullptr;
        a.nd = plans[order[r]];
        // node rows with taudot sums take 24 bytes per point of q <= C / 2 rows:
        // within the chirp rows' 16 bytes of C rows
        a.td_rows = node ? reinterpret_cast<float2 *>(e.rows + (size_t)V * a.nd.q * nu_row_len(a.S)) : nullptr;
        if (node && td) any_td = true;   // then made for every node-form request of the batch
        a.Sp = (q.cd.S + 7) / 8 * 8;
        a.rows = adj_rows(a.Sp);
        const long long items = (cap + a.tile - 1) / a.tile * bp.nvs;
        if (node) {
            items_node += items;
        } else if (nu) {
            items_nu += items;
        } else {
            lds_f2 = std::max(lds_f2, (size_t)a.rows * a.Sp);
            items_direct += items;
        }
        GeomArgs &g = gg[r];
        const sbr_mesh *m = q.mesh;
        g.verts = m->verts;
        g.faces = m->faces;
        g.mat_id = m->mat_id;
        g.tri = q.hits->tri;
        g.R = q.gd.nx * q.gd.ny;
        g.nf = m->nf;
        g.mt = q.mt;
        g.any_fresnel = 0;
        for (int i = 0; i < q.mt.n; i++)
            if (q.mt.mode[i] != 0) g.any_fresnel = 1;
        g.rd = rd;
        g.g = q.gd;
        g.ch = q.cd;
        g.wave_first = q.st.wave_first;
        g.blk = q.st.blk;
        g.by_ray = paths_by_ray(rd, q.gd, q.cd) ? 1 : 0;
        g.flags = q.hits->flags;
        g.drop = (q.flags & SBR_DROP_FLAGGED) ? 1 : 0;
        g.exit_only = (q.flags & SBR_EXIT_ONLY) ? 1 : 0;
        const bool sums = V >= kSplitAntennas;   // k_path_sums
        g.abar = sums ? e.abar : e.part;
        g.tdbar = !td ? nullptr : sums ? e.tdbar : e.tpart;
        g.parts = sums ? 1 : bp.nvs;
        g.tau_bar = e.tau_bar;
        g.tx_n = sums ? 1 : rd.n_rx;
        g.rx_n = sums ? 1 : rd.n_tx;
        g.rx_first = sums ? rd.n_tx : 0;
        g.tiles = std::min(std::max(g.R / (256 * kGeomBlocks), 1), 16);
        g.cap = (int32_t)cap;
        g.grad = q.grad;
        const bool want = q.params && (q.params->materials || q.params->radar || q.params->rot || q.params->attenuation);
        g.acc = want ? e.acc : nullptr;
        g.want_mats = q.params && q.params->materials;
        g.want_rot = q.params && q.params->rot;
        a.acc = g.acc;
        a.n_acc = kParamSums + 2 * q.mt.n;
        g.attached = (q.flags & SBR_ATTACHED) ? 1 : 0;
        for (int t = 0; t < SBR_MAX_TX; t++)
            for (int c = 0; c < 3; c++) g.txl[t][c] = t < q.radar->n_tx ? (float)q.radar->tx[t][c] : 0.0f;
        for (int k = 0; k < SBR_MAX_RX; k++)
            for (int c = 0; c < 3; c++) g.rxl[k][c] = k < q.radar->n_rx ? (float)q.radar->rx[k][c] : 0.0f;
    }
    AdjTable t = adj_table(table, n, nullptr);
    int rc = put_table(t.args, aa.data(), sizeof(AdjArgs) * n, s);
    if (rc) return rc;
    hipLaunchKernelGGL(k_adj_items, dim3(1), dim3(1024), 0, s, t.args, n, t.item_first, t.queue);
    SBR_LAUNCHED();
    // gradient rows of requests [r0, r1) of one of the FFT forms in row_first[0..]
    auto put_rows = [&](int r0, int r1, int32_t *dst, unsigned *total, int *max_s) {
        std::vector<int32_t> row_first(1, 0);
        *max_s = 0;
        for (int r = r0; r < r1; r++) {
            const long long rows = (long long)aa[r].V * (aa[r].nd.q ? aa[r].nd.q : aa[r].C);
            if (row_first.back() + rows > 0x7fffffffLL) {
                set_error("batched backward: more than 2^31 gradient rows in one launch");
                return (int)SBR_E_ARG;
            }
            row_first.push_back(row_first.back() + (int32_t)rows);
            *max_s = std::max(*max_s, (int)aa[r].S);
        }
        *total = (unsigned)row_first.back();
        return put_table(dst, row_first.data(), sizeof(int32_t) * row_first.size(), s);
    };
    if (n_node > 0) {
        unsigned rows = 0;
        int max_s = 0;
        if ((rc = put_rows(0, n_node, t.node_first, &rows, &max_s))) return rc;
        ProfScope ps(kProfSynthAdj, s);
        // sequences and twiddles, and the chirp groups' partial sums where a
        // row has fewer columns than the block threads (at most 144 KiB)
        const size_t lds_rows = (size_t)2 * max_s * (any_td ? 64 : 48) + kNodeRowThreads * 32;
        size_t slot = 0;   // float4 words of the largest stage
        for (int r = 0; r < n_node; r++) {
            const int RL = nu_row_len(aa[r].S);
            slot = std::max(slot, (size_t)(node_stage(aa[r].S, aa[r].nd.q, any_td) * RL * (any_td ? 24 : 16) + 15) / 16);
        }
        const size_t lds = sizeof(float4) * slot + 16;
        const void *kr = any_td ? (const void *)k_node_adj_rows<true> : (const void *)k_node_adj_rows<false>;
        const void *kt = any_td ? (const void *)k_synth_adj_node<true> : (const void *)k_synth_adj_node<false>;
        if (lds_rows > 65536 - 1024)
            SBR_HIP(hipFuncSetAttribute(kr, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_rows));
        const dim3 grid((unsigned)std::max(1LL, std::min<long long>(items_node,
                                                                   resident_blocks(kt, kNodeThreads, lds, 256 * 2))));
        if (any_td)
            hipLaunchKernelGGL(k_node_adj_rows<true>, dim3(rows), dim3(kNodeRowThreads), lds_rows, s, t.args,
                               t.node_first, n_node);
        else
            hipLaunchKernelGGL(k_node_adj_rows<false>, dim3(rows), dim3(kNodeRowThreads), lds_rows, s, t.args,
                               t.node_first, n_node);
        SBR_LAUNCHED();
        ProfScope pk(kProfNuTaps, s);
        if (any_td)
            hipLaunchKernelGGL(k_synth_adj_node<true>, grid, dim3(kNodeThreads), lds, s, t.args, t.item_first, 0,
                               n_node, t.queue + kAdjQueueNode, (int)slot);
        else
            hipLaunchKernelGGL(k_synth_adj_node<false>, grid, dim3(kNodeThreads), lds, s, t.args, t.item_first, 0,
                               n_node, t.queue + kAdjQueueNode, (int)slot);
    }
    SBR_LAUNCHED();
    if (n_nu > n_node) {
        // all requests of the chirp-row form: 1/Psi tables, then the row transforms
        unsigned rows = 0;
        int max_s = 0;
        if ((rc = put_rows(n_node, n_nu, t.row_first, &rows, &max_s))) return rc;
        ProfScope ps(kProfSynthAdj, s);
        hipLaunchKernelGGL(k_nu_corr_adj, dim3((unsigned)((max_s + 255) / 256), (unsigned)(n_nu - n_node)), dim3(256),
                           0, s, t.args + n_node);
        const size_t lds_rows = sizeof(float4) * 2 * max_s + sizeof(float2) * 2 * max_s;   // sequence + twiddles
        hipLaunchKernelGGL(k_nu_rows, dim3(rows), dim3(256), lds_rows, s, t.args + n_node, t.row_first,
                           n_nu - n_node);
        SBR_LAUNCHED();
        size_t slot = 0;   // float4 words of the largest row stage
        for (int r = n_node; r < n_nu; r++) slot = std::max(slot, (size_t)nu_stage(aa[r].S) * nu_row_len(aa[r].S));
        const size_t lds = sizeof(float4) * slot + 16;
        dim3 grid((unsigned)std::max(1LL, std::min<long long>(items_nu, resident_blocks((const void *)k_synth_adj_nu<kNuPPL>,
                                                                                         256, lds, 256 * 2))));
        ProfScope pk(kProfNuTaps, s);
        hipLaunchKernelGGL(k_synth_adj_nu<kNuPPL>, grid, dim3(256), lds, s, t.args, t.item_first, n_node, n_nu,
                           t.queue, (int)slot);
    }
    SBR_LAUNCHED();
    if (n_nu < n) {
        const size_t lds = sizeof(float2) * lds_f2 + 16;
        // one device-full of blocks, or fewer if the path slots cannot fill it
        dim3 grid((unsigned)std::max(1LL, std::min<long long>(items_direct, resident_blocks((const void *)k_synth_adj<kAdjPPL>,
                                                                                             256, lds, 256 * 2))));
        ProfScope ps(kProfSynthAdj, s);
        hipLaunchKernelGGL(k_synth_adj<kAdjPPL>, grid, dim3(256), lds, s, t.args, t.item_first, n_nu, n,
                           t.queue + kAdjQueueDirect, (int)lds_f2);
    }
    SBR_LAUNCHED();
    for (int r = 0; r < n; r++) {
        const AdjArgs &a = aa[r];
        const GeomArgs &g = gg[r];
        const long long cap = a.rec.cap;
        if (g.R == 0 || g.nf == 0) continue;
        if (a.V >= kSplitAntennas) {
            hipLaunchKernelGGL(k_path_sums, dim3((unsigned)((cap + 63) / 64)), dim3(64 * kSumsWaves), 0, s, a.count,
                               a.abar_part, g.tdbar ? a.tdb_part : nullptr, a.nvs, (int)cap,
                               const_cast<float2 *>(g.abar), const_cast<float *>(g.tdbar), a.tau_bar, g.rd.n_tx,
                               g.rd.n_rx);
            SBR_LAUNCHED();
        }
        dim3 gb((unsigned)((g.R + 256LL * g.tiles - 1) / (256LL * g.tiles)));
        launch_geom(g, gb, s);
        if (g.acc) {
            const sbr_param_grads &pg = *reqs[order[r]].params;
            hipLaunchKernelGGL(k_param_add, dim3(1), dim3(256), 0, s, g.acc, g.mt.n, pg.materials, pg.radar, pg.rot,
                               pg.attenuation);
        }
        SBR_LAUNCHED();
    }
    return SBR_OK;
}

}  // namespace sbr
