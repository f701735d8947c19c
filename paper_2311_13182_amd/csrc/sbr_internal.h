// Internal definitions shared by the libsbr HIP sources (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include <algorithm>
#include <string>

#include "sbr.h"

namespace sbr {

// ----------------------------------------------------------------- errors
void set_error(const char *fmt, ...);
void clear_error();

#define SBR_CHECK_ARG(cond, ...)              \
    do {                                      \
        if (!(cond)) {                        \
            ::sbr::set_error(__VA_ARGS__);    \
            return SBR_E_ARG;                 \
        }                                     \
    } while (0)

#define SBR_HIP(call)                                                              \
    do {                                                                           \
        hipError_t e_ = (call);                                                    \
        if (e_ != hipSuccess) {                                                    \
            ::sbr::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), \
                             __FILE__, __LINE__);                                  \
            return SBR_E_HIP;                                                      \
        }                                                                          \
    } while (0)

#define SBR_LAUNCHED()                                                                \
    do {                                                                              \
        hipError_t e_ = hipGetLastError();                                            \
        if (e_ != hipSuccess) {                                                       \
            ::sbr::set_error("kernel launch failed: %s (%s:%d)", hipGetErrorString(e_), \
                             __FILE__, __LINE__);                                     \
            return SBR_E_HIP;                                                         \
        }                                                                             \
    } while (0)

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Carve sub-buffers out of a caller-provided byte buffer.
struct Carver {
    char *base;
    size_t off = 0;
    explicit Carver(void *b) : base(static_cast<char *>(b)) {}
    template <class T>
    T *take(size_t count) {
        off = align_up(off, 256);
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

// ----------------------------------------------------------------- BVH
// Node of the depth-first layout, 16 bytes: the box in 16-bit steps of the
// mesh's bounds (low half lo, high half hi, rounded outwards), and the link: an
// internal node's escape index (next node after its subtree; == node count
// ends traversal; its left child is the next node), a leaf's kLeafBit | slot
// (its escape is the next node).
struct __align__(16) BvhNode {
    uint32_t x, y, z, link;
};
constexpr uint32_t kLeafBit = 0x80000000u;

// Triangle of a leaf: three vertices, .w of the first = original face id bits.
struct __align__(16) LeafTri {
    float4 a, b, c;
};

// Box of a run of leaves.
struct Box {
    float lo[3], hi[3];
};

struct BvhView {
    int32_t n;          // triangles
    int32_t n_nodes;    // 2n - 1
    BvhNode *nodes;     // [n_nodes], depth-first order
    LeafTri *tris;      // [n], Morton order (leaf slot order)
    int32_t *order;     // [n] leaf slot -> original face
    int32_t *other;     // [n - 1] internal node i covers the leaf slots from i to other[i]
    int32_t *dfs_of;    // [n_nodes] radix-tree index (internal i, leaf n - 1 + slot) -> depth-first index
    Box *prefix;        // [n] union of the leaves of the slot's block of kBoxBlock up to the slot
    Box *suffix;        // [n] union from the slot to the end of its block
    uint32_t *part;     // [kBoundsBlocks][12] partial bounds of the centroids and of the vertices
    int32_t *header;    // [16] [0] n, [1] kBvhMagic once a BUILD of n faces has
                        // finished, [2] set to 1 by a REFIT that found no such BUILD;
                        // [4..6] origin and [8..10] step of the nodes' boxes (floats)
};
constexpr int kBoundsBlocks = 256;
constexpr int kBoxBlock = 256;

// Seal of a built BVH buffer (header[1]); refit and traversal check it
// together with header[0] == face count before they follow any stored index.
constexpr int32_t kBvhMagic = 0x48564253;

BvhView bvh_view(void *buf, int32_t nf, size_t *bytes_out);

// ----------------------------------------------------------------- constants
constexpr double kC0 = 299792458.0;
constexpr double kEps0 = 8.8541878128e-12;
constexpr double kPi = 3.14159265358979323846;

// Arguments of the path stage, passed by value to kernels.
struct MatTable {
    int32_t n;
    int32_t mode[SBR_MAX_MATERIALS];
    double eps_r[SBR_MAX_MATERIALS];
    double sigma[SBR_MAX_MATERIALS];
};

struct RadarDev {
    double o[3];
    double rot[9];
    int32_t n_tx, n_rx;
    double tx[SBR_MAX_TX][3];   // world frame
    double rx[SBR_MAX_RX][3];   // world frame
    double vel[3];
    double atten;               // amplitude attenuation of the medium, 1/m
    double n_tg, n_rg;          // TX / RX gain exponents (cos^n about boresight)
};

struct GridDev {
    int32_t nx, ny, K, options;
    double thx, thy, t_min;
    uint32_t seed_lo, seed_hi;
};

struct ChirpDev {
    double fc, slope, fs, tc;
    int32_t S, C;
};

// Device-side path records (structure of arrays, capacity = K * R).
struct PathSoA {
    int32_t cap;
    int32_t V;
    float *alpha;     // [V][cap] frac(fc * tau_v), cycles
    float *gamma;     // [V][cap] slope * tau_v / fs, cycles per sample
    float2 *amp;      // [cap] I^s
    float *beta;      // [cap] frac(fc * tc * taudot), cycles per chirp
    float *epsd;      // [cap] slope * tc * taudot / fs, cycles per sample per chirp
};

// Scratch layout of the path stage (compaction + records).  Paths lie wavefront
// by wavefront of kPathWave consecutive rays.  Within one, requests of the node
// form have them bounce by bounce: the wavefront's first returns in ray order,
// then its second ones, and so on.  Neighbouring paths then come from
// neighbouring rays at the same bounce, so a wavefront of a kernel over rays
// meets a run of paths per bounce (coalesced: path stage 0.57 -> 0.47 ms at 2048^2
// rays), and one of a kernel over paths meets similar beat frequencies.  The
// chirp rows' phase recurrences start at a chirp that depends on the lane, and
// their contributions are rounded to 19 bits, so there the order of the paths
// shows in the cube (5e-6, and 3e-3 of the RMS at the peaks of a 400-antenna
// image): those requests have them ray by ray, and so have many antennas, where
// kernels over paths do most of the work.
struct PathStage {
    int32_t *count;       // [0] = number of paths P, [1] = float bits of the largest
                          // max(|Re A|, |Im A|) over them
    int32_t *wave_first;  // [nwave] first path of each wavefront of rays, from its block's first
    int32_t *blk;         // [nblk] first path of each block of kPathBlock rays
    int32_t nwave, nblk;
    PathSoA rec;
};

constexpr int kPathWave = 64;
constexpr int kPathBlock = 1024;   // rays per block of the counting kernel

// Antennas (TX times RX) from which on a path's delays are written, and their
// adjoints summed, by kernels of their own rather than by the path's lane.
// Measured at 12 (path stage and geometry adjoint 1.32 ms together at 2048^2 rays,
// with the summing kernel alone 0.45 ms more) and at 400 (0.65 ms, 0.16 with the
// kernels); the line is drawn between them.
constexpr int kSplitAntennas = 32;

// Doppler nodes of the node form of the non-uniform FFT sums.  With nu =
// fc t_chirp taudot (cycles per chirp) and kappa = slope / (fs fc), the phase
// of Eq. (8) in cycles is
//   alpha + c nu + s gamma + c s eps,  eps = kappa nu
//     = [alpha + cbar nu] + s [gamma + cbar eps] + (c - cbar)(1 + s kappa) nu.
// Only the last term couples the chirps to a path, and every path of a request
// has nu = (2 fc t_chirp / c0) u . d within the range that the ray grid's
// directions d span: for a scene speed u of a few m/s the term turns by less
// than a cycle between the ends of that range.  So it is interpolated in nu
// from q Chebyshev nodes nu_j = nu0 + h x_j: a path spreads into (or reads) q
// grid rows instead of one row per chirp, and the chirps are formed from the
// q rows at the end with the exact factor e^{2 pi j (c - cbar)(1 + s kappa) nu_j}.
constexpr int kMaxNodes = 32;
struct NodePlan {
    int32_t q;       // nodes; 0: the chirp-row form is used
    int32_t cbar;    // C / 2
    double nu0, h;   // centre and half width of the range of nu
    double kappa;
    double inv_kappa;   // 1 / kappa (0 with no slope)
    float nu0f;      // nu0 modulo 1
    float inv_h;     // 1 / h (0 with one node)
    float2 node[kMaxNodes];   // x_j and the weight (-1)^j sin(theta_j) / (2 q) of its Lagrange polynomial
};

// Launch shape of the IF synthesis: L samples per lane, SB sample blocks per
// chirp row, tiles_per_v wavefronts per antenna, n_chunks path chunks.
struct SynthPlan {
    int32_t L, SB, tiles_per_v, n_chunks;
    int32_t nu, cg;      // non-uniform FFT form (L = 0): chirps (nodes) per spreading block
    int32_t q;           // node form: nodes (0: chirp rows)
};

// A pointer read from a device table is generic; marking it global lets the
// compiler use scalar or global (not flat) loads through it.  The qualifier
// exists in the device pass only (the host pass merely parses these bodies).
#if defined(__HIP_DEVICE_COMPILE__)
#define SBR_GLOBAL_AS __attribute__((address_space(1)))
#else
#define SBR_GLOBAL_AS
#endif
template <class T>
__device__ __forceinline__ SBR_GLOBAL_AS T *gmem(T *p) {
    return (SBR_GLOBAL_AS T *)p;
}
// plain pair of floats with float2's layout, for address-space-qualified access
struct F2 {
    float x, y;
};
__device__ __forceinline__ SBR_GLOBAL_AS const F2 *gmem(const float2 *p) { return (SBR_GLOBAL_AS const F2 *)p; }
__device__ __forceinline__ SBR_GLOBAL_AS F2 *gmem(float2 *p) { return (SBR_GLOBAL_AS F2 *)p; }
struct alignas(16) D2 {
    double x, y;
};
__device__ __forceinline__ SBR_GLOBAL_AS D2 *gmem2(double2 *p) { return (SBR_GLOBAL_AS D2 *)p; }

// Arguments of one request's IF synthesis (device-table entry of a batch).
struct SynthArgs {
    const int32_t *count;
    PathSoA rec;
    int32_t V, C, S;
    int32_t SB;          // sample blocks per chirp row
    int32_t tiles_per_v; // wavefront tiles per antenna
    int32_t n_chunks;
    int32_t gx;          // blocks per chunk (4 wavefronts each)
    float2 *partial;     // [n_chunks][V][C][S] (direct forms)
    // non-uniform FFT form (nu = 1): chirps per spreading block, chirp groups;
    // the max-amplitude word, the 1/Psi table and the fixed-point grids
    int32_t nu, cg, ncg;
    uint32_t *amax;      // [kNuMaxChunks] per path chunk: max over its paths of max(|Re A|, |Im A|), float bits
    float *corr;         // [S]
    long long *grid;     // [n_chunks][V][C][re, im][nu_row_len(S)]
    float2 *out;         // [V][C][S] the IF cube (set by launch_synth_batch)
    // node form (nd.q > 0): cg nodes per spreading block, ncg node groups, the
    // fixed-point bits below the largest amplitude, the transformed rows; the
    // grids are [n_chunks][V][q][re, im][nu_row_len(S)]
    int32_t bits;
    double2 *modes;      // [V][q][S] deconvolved modes of each node row
    NodePlan nd;
};

PathStage carve_path_stage(Carver &cv, int32_t R, int32_t K, int32_t V);
// The Doppler nodes of a request; q = 0 where the chirp-row form is used.
NodePlan node_plan(const RadarDev &rd, const GridDev &g, const ChirpDev &ch);
// The synthesis' nodes: those of node_plan where it takes the node form, q = 0
// where it takes chirp rows.
NodePlan synth_nodes(const RadarDev &rd, const GridDev &g, const ChirpDev &ch);
// Whether a request's paths lie ray by ray within a wavefront of rays (else
// bounce by bounce); see PathStage.
bool paths_by_ray(const RadarDev &rd, const GridDev &g, const ChirpDev &ch);
SynthPlan synth_plan(int32_t R, int32_t K, int32_t V, int32_t C, int32_t S, bool nu);
// The node form's plan: never more grid words than synth_plan(..., true) asks for.
SynthPlan synth_node_plan(int32_t R, int32_t K, int32_t V, int32_t C, int32_t S, int32_t q);
size_t synth_partial_elems(const SynthPlan &p, int32_t V, int32_t C, int32_t S);
// Fixed-point grid words (long long) of the non-uniform FFT form.
size_t synth_grid_words(const SynthPlan &p, int32_t V, int32_t C, int32_t S);
SynthArgs synth_args(const PathStage &st, const SynthPlan &p, const NodePlan &nd, int32_t V, int32_t C, int32_t S,
                     float2 *partial, long long *grid, float *corr, uint32_t *amax);
// Device-table bytes of a batch of n syntheses.
size_t synth_table_bytes(int n);
// IF synthesis of n requests whose path stages are enqueued: one launch per
// sample-run length over all their blocks (args[i] and L[i] = synth_plan's L),
// then each request's fixed-order chunk reduction into out[i]; requests of the
// non-uniform FFT form (L[i] = 0) run their own spreading and row launches.
int launch_synth_batch(const SynthArgs *args, const int *L, int n, void *table, float2 *const *out,
                       hipStream_t s);

// One request of a (batched) backward pass: validated arguments, path stage
// enqueued into st, `extra` = its scratch after the path stage.
struct BackwardReq {
    const sbr_mesh *mesh;
    MatTable mt;
    RadarDev rd;
    GridDev gd;
    ChirpDev cd;
    const sbr_hits *hits;
    PathStage st;
    void *extra;
    const float2 *G;
    float *grad;
    const sbr_radar *radar;
    const sbr_param_grads *params;
    int32_t flags;
};
size_t backward_extra_bytes(int32_t R, int32_t K, int32_t V, int32_t C, int32_t S);
// Device-table bytes of a batch of n adjoints.
size_t adj_table_bytes(int n);
// Synthesis adjoint of n requests as one work-queue launch over all their
// (antenna group, path tile) items, then each request's reduction and
// geometry adjoint.
int launch_backward_batch(const BackwardReq *reqs, int n, void *table, hipStream_t s);

// ---- non-uniform FFT forms of Eq. (8) (type 1) and Eqs. (11)-(12) (type 2)
// A sum over the S samples of a chirp, sum_s h_s e^{2 pi j s g}, is a finite
// Fourier series at the beat frequency g of a path.  With the modes centred
// (s' = s - S/2), a grid of M = 2S points and a kernel psi of width kNuW grid
// points whose Fourier transform is Psi:
//   e^{2 pi j s' g} Psi(s'/M) = sum_l e^{2 pi j s' l / M} psi(gM - l)
// up to the kernel's aliasing error, which is below 1e-6 of the sum of the
// magnitudes of the terms for the exponential-of-semicircle kernel
// psi(z) = exp(beta (sqrt(1 - (2z/W)^2) - 1)), W = 7, beta = 2.3 W.  Rows of
// grid values hold l = -M/2 - 3 .. M/2 + 3 at index l + M/2 + 3, plus one
// padding entry.
constexpr int kNuW = 7;
constexpr int kNuHalf = (kNuW - 1) / 2;
constexpr double kNuBeta = 2.30 * kNuW;
constexpr int kNuMinS = 16;     // shorter chirps use the direct forms (cheap there)
constexpr int kNuMaxS = 1024;   // longer chirps use the direct forms
constexpr int kNuMaxChunks = 256;   // path chunks of a spreading launch, each with its own scale
__host__ __device__ constexpr int nu_row_len(int S) { return 2 * S + 8; }
static inline bool nu_size(int S) { return S >= kNuMinS && S <= kNuMaxS; }

// Copy `bytes` (a multiple of 4) of host data into device memory on stream s
// with fill kernels that carry the data as kernel arguments: no memcpy node,
// and the host data need not outlive the call.
int put_table(void *dst, const void *src, size_t bytes, hipStream_t s);

// host-side conversions / validation shared by the entry points
int check_mesh(const sbr_mesh *m);
int check_common(const sbr_mesh *m, const sbr_material *mats, int32_t n_mats,
                 const sbr_radar *r, const sbr_rays *g, const sbr_hits *h,
                 const sbr_chirp *ch);
MatTable make_mats(const sbr_material *mats, int32_t n_mats);
RadarDev make_radar(const sbr_radar *r);
GridDev make_grid(const sbr_rays *g);
ChirpDev make_chirp(const sbr_chirp *c);

// Brackets one kernel launch with HIP events while sbr_profile(1) is on.
class ProfScope {
   public:
    ProfScope(int id, hipStream_t s);
    ~ProfScope();

   private:
    int id_;
    hipStream_t s_;
    bool active_;
    hipEvent_t a_{}, b_{};
};
enum { kProfSynth = 0, kProfSynthAdj = 1, kProfTrace = 2, kProfNuSpread = 3, kProfNuTaps = 4, kProfIds = 5 };

// Blocks of `kernel` (launched with `threads` threads and `lds` bytes of
// dynamic LDS) the current device holds at once: CUs times the occupancy the
// runtime reports for the compiled kernel, cached per (device, kernel,
// threads, lds); `fallback` where the runtime cannot answer.
int resident_blocks(const void *kernel, int threads, size_t lds, int fallback);

// zero n floats with a fill kernel on stream s (no memset node, so the call
// can sit in a captured graph)
int fill_zero_f32(float *p, size_t n, hipStream_t s);

// enqueue path compaction + FP64 refinement; records go to st.rec
int launch_paths(const sbr_mesh *m, const MatTable &mt, const RadarDev &rd, const GridDev &gd,
                 const ChirpDev &cd, const sbr_hits *h, int32_t flags, const PathStage &st,
                 hipStream_t s);

}  // namespace sbr
