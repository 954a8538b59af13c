// Implicit diffusion (Sec. II.B.3b, Scheme 2): per diffusing pool, solve
// (I + a L_w) y = x with the conjugate gradient method preconditioned by the
// inverse diagonal of the system matrix (Sec. III).  Matrix-free: the
// Laplacian is applied as a gather over the neighbours (the explicit step's
// neighbour source: table or packed).  Vectors,
// dot products and scalars are FP64 whatever the field type.
//
// Both kernels of an iteration are bound by memory, so the iteration is cut
// to move as few bytes as it can:
//  - k_cg_dot: the partials of (z, B z), a gather of z and the neighbour
//    words and nothing else (12.5 B per voxel).  (p, B p) follows from it:
//    with p = z + beta p_old and q_old = B p_old,
//    (p, B p) = (z, B z) + 2 beta (z, q_old) + beta^2 (p_old, q_old),
//    whose last two products the step before sums where z and q_old are in
//    registers.  (The orthogonality of z and r_old would give them for free
//    as -beta (r.z) / alpha_old together - Chronopoulos and Gear, J. Comput.
//    Appl. Math. 25, 1989 - but rounding loses it on ill-conditioned systems:
//    a 12^3 cube at a = 1e12 never converged and a chain of 400 at a = 1e6
//    took 1.3 times the iterations.  The summed products keep the iteration
//    counts of a directly summed (p, B p), and cost nothing measurable beside
//    the recurrence.)
//  - k_cg_step: p = z + beta p_old for the voxel and its neighbours, so that
//    q = B p is formed in registers and never stored; z <- z - alpha M^-1 q
//    into the other z buffer (r = M z is not stored: r_i is z_i times the
//    diagonal), p into the other p buffer, and every second iteration
//    x += alpha_old p_old + alpha p (a last odd direction is added on
//    write-back); the partials of r.z, r.r, (p, q) and (z, q).  20.5 B read,
//    16 B written per voxel and 16 B for x every second iteration.
// 57 B per voxel and iteration on average.  (The form before it stored q, r
// and updated x each time: 93.5 B; 512^3, 22.8 M voxels: see k_cg_step.)
// There is no kernel for the scalars: each block of the kernel that needs
// them adds up the partials of the kernel before it, in a fixed order, and
// block 0 keeps the results for later kernels in slots no other block of the
// same kernel reads.  That holds for the convergence flag too: the kernels
// that check convergence do not look at it but repeat the check, whose
// partials stay as they are once the flag is up; the others return on it at
// once.  The host reads the scalars only every few iterations (the number
// follows the convergence seen so far).
//
// Multigrid option (not in the paper, whose preconditioner is the diagonal):
// M^-1 is one V-cycle over a hierarchy of aggregates.  Level l+1 has one cell
// per occupied 2x2x2 block of level l's grid and the piecewise-constant
// prolongation P; its operator P^T B_l P keeps the form mass + a L_w (the
// mass of a cell is its number of voxels, the weight between two cells the
// sum of the weights of the level-l edges between them), so every level
// runs the same kind of kernel.  Pre-smoothing is one damped Jacobi sweep
// from zero, x = w D^-1 r, post-smoothing the same sweep after the coarse
// correction, and the coarsest level gets kMgSweeps damped Jacobi sweeps:
// a fixed linear map, symmetric (the post-smoother is the transpose of the
// pre-smoother; k Jacobi sweeps from zero are D^-1/2 p(D^-1/2 B D^-1/2)
// D^-1/2 for a polynomial p) and positive definite (w times the largest
// eigenvalue of D^-1 B stays below 2 because every row's weights sum to less
// than its diagonal).  The restriction is computed per coarse cell from its
// children (found with the level's rank index in a fixed order) and the
// prolongation per fine cell from its parent, so no sum depends on
// scheduling.  Three kernels per level: residual, restriction (sum over the
// children), then prolongation and post-smoothing in one; one thread per cell,
// the fine level's residual and last kernel in grid strides of several voxels.  With t = r - B x the residual of the pre-smoothed x, and P e the
// prolongated coarse solution, the post-smoothed result is
//   y + w D^-1 (r - B y) = x + P e + w D^-1 (t - B P e),  y = x + P e,
// and P e is constant on every 2x2x2 block: of a cell's six neighbours three
// lie in its own block (their terms vanish) and the others in the three
// coarse neighbours on its side, so this kernel gathers only from the four
// times smaller coarse solution.  With the multigrid r is kept (in place of
// the z update: 28.5 B read by k_cg_step) and the V-cycle writes z and the r.z
// partials.  z comes after the step that holds q_old, but the V-cycle M^-1 is
// symmetric: (z, q_old) = (z, r_old - r) / alpha_old, and (z, r_old) =
// (r, z_old), which that step sums.  (As (B z, p_old) in k_cg_dot it took
// another vector's stream, 2 % of a solve.)
#include <type_traits>

#include "vg_internal.h"

namespace vg {
namespace {

// Scalars on the device: r.z and alpha of the current and the previous
// iteration (slot = iteration & 1), r.r, b.b, the convergence flag, the
// iterations done, the squared tolerance, and (p, q) and (z, q) of the
// iteration before (z the one after it).
enum { S_RZ = 0, S_ALPHA = 2, S_RR = 4, S_BB, S_DONE, S_ITER, S_RTOL2, S_PQ, S_ZQ, S_NSCAL };
// Partials per block, one array of CgArgs::ldp each: r.z, (z, q) (MG: (r, z) of
// the new r and the old z), (p, q), r.r (k_cg_step's, in this order), b.b,
// z.Bz.
enum { P_RZ = 0, P_ZQ, P_PQ, P_RR, P_BB, P_ZBZ, P_N };
static_assert(S_NSCAL <= kCgScal && P_N == kCgParts, "the workspace layout's sizes");

// The gathering kernels come in two forms.  A 64-lane load of doubles takes
// the vector cache 16 cycles whatever its addresses (measured: 17.8 accesses
// per load), so a voxel's seven values of one vector cost more than their
// memory traffic.  The staged form puts a block's tile of kCgTileV * kBlock
// consecutive voxels and a halo of kCgHalo voxels on each side into LDS by
// contiguous loads, reads the x and y neighbours there (4 cycles per wave)
// and gathers only the z neighbours; it needs the x and y distances to fit
// the halo, enough voxels that every CU has tiles (kCgStagedMin) and unit
// weights (cg_staged).  The direct form, one voxel per thread, serves the rest.
constexpr int kCgTileV = 4;
constexpr int kMgPostV = 2;      // voxels per thread of the V-cycle's last kernel
constexpr int kCgHalo = 256;
constexpr int64_t kCgStagedMin = (int64_t)1 << 20;
constexpr int kCgMaxBlocks = 2048;      // partials per slot at most (vg_sim::cg_blocks)

// multigrid V-cycle
constexpr double kMgOmega = 0.8;        // damping of the Jacobi smoother
constexpr int64_t kMgCoarsest = 1024;   // a level this small is solved by sweeps alone
constexpr int kMgSweeps = 8;            // damped Jacobi sweeps on the coarsest level
constexpr int kMgCoarseThreads = 1024;  // the coarsest level's single block
constexpr int kMgCoarseMax = 4096;      // cells the coarsest kernel holds in LDS

__device__ __forceinline__ double weight(const uint16_t *rcode, const double *cl, int64_t i, int k,
                                         bool reg) {
    if (!reg) return 1.0;
    const uint32_t code = rcode[i];
    const uint32_t own = code & 7u;
    const uint32_t other = own ^ (((code >> (3 + k)) & 1u) << (k >> 1));
    return 0.5 * (cl[own] + cl[other]);
}

struct CgArgs {
    const int32_t *nbr = nullptr;
    const uint16_t *rcode = nullptr;
    PackedNbr pk;                // packed neighbour sources (when built)
    int64_t n = 0;
    int64_t ntiles = 0;
    double a = 0;
    double c[VG_NREG] = {};
    int ldp = 0;                 // partials per slot
    uint32_t run = kXcdRun;      // block tiles per XCD run (xcd_run)
};

// Neighbour sources of the CG kernels (the explicit step's): the table, or
// a packed source; an absent neighbour comes back as the voxel itself.
// NS_WIDE: a packed source whose FP64 vectors outgrow 32-bit byte offsets.
enum { NS_TABLE = 0, NS_REL = 1, NS_OFF = 2, NS_WIDE = 4 };
template <int NS>
constexpr bool kRel = (NS & ~NS_WIDE) == NS_REL;

template <int NS>
__device__ __forceinline__ void cg_neighbours(const CgArgs &A, int64_t i, int64_t (&j)[6], bool (&pres)[6]) {
    if constexpr (NS == NS_TABLE) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const int32_t jk = A.nbr[(int64_t)k * A.n + i];
            pres[k] = jk >= 0;
            j[k] = pres[k] ? (int64_t)jk : i;
        }
    } else {
        uint32_t jp[6];
        const PackedWords W = packed_words<kRel<NS>>(A.pk, (uint32_t)i);
        packed_decode<kRel<NS>>(A.pk, (uint32_t)i, W, jp);
#pragma unroll
        for (int k = 0; k < 6; k++) {
            j[k] = (int64_t)jp[k];
            pres[k] = j[k] != i;      // no periodic wrap: a neighbour is never the voxel itself
        }
    }
}

// Index type: 32 bits with a packed source (one address register per lane
// beside the array's base), 64 where n doubles do not fit 2^32 bytes and with
// the table.
template <int NS>
using CgIdx = std::conditional_t<NS == NS_TABLE || (NS & NS_WIDE) != 0, int64_t, uint32_t>;
template <typename T>
__device__ __forceinline__ T &el(T *b, uint32_t i) {
    return at(b, i);
}
template <typename T>
__device__ __forceinline__ T &el(T *b, int64_t i) {
    return b[i];
}

// What the kernels load ahead of a voxel's gathers: its neighbour words (the
// table's six indices, or the packed words and, for relative codes, the six
// base distances of its group of 64: the same for the wave's lanes).
template <int NS>
struct CgWords {
    int32_t jt[NS == NS_TABLE ? 6 : 1];
    PackedWords W;
    uint32_t base[kRel<NS> ? 6 : 1];
};

template <int NS>
__device__ __forceinline__ void cg_words(const CgArgs &A, CgIdx<NS> i, CgWords<NS> &w) {
    w.W = PackedWords{0, 0};
    if constexpr (NS == NS_TABLE) {
#pragma unroll
        for (int k = 0; k < 6; k++) w.jt[k] = A.nbr[(int64_t)k * A.n + i];
    } else {
        w.W = packed_words<kRel<NS>>(A.pk, (uint32_t)i);
        if constexpr (kRel<NS>) {
            const uint32_t grp = __builtin_amdgcn_readfirstlane((uint32_t)i / (uint32_t)kGroup);
            const uint32_t *bp = A.pk.rel_base + (size_t)grp * 8;
#pragma unroll
            for (int k = 0; k < 6; k++) w.base[k] = *(const __attribute__((address_space(4))) uint32_t *)(bp + k);
        }
    }
}

// The neighbours (an absent one is the voxel itself).
template <int NS>
__device__ __forceinline__ void cg_decode(const CgArgs &A, CgIdx<NS> i, const CgWords<NS> &w, CgIdx<NS> (&j)[6],
                                          bool (&pres)[6]) {
    if constexpr (NS == NS_TABLE) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            pres[k] = w.jt[k] >= 0;
            j[k] = pres[k] ? (int64_t)w.jt[k] : i;
        }
    } else if constexpr (kRel<NS>) {
        const uint32_t u = (uint32_t)i;
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const uint32_t c = (w.W.a >> A.pk.rl.sh[k]) & A.pk.rl.mk[k];
            const uint32_t d = w.base[k] + (c ? c - 1u : 0u), last = (uint32_t)A.n - 1u;
            j[k] = (CgIdx<NS>)((k & 1) ? min(u + d, last) : u - min(d, u));
            pres[k] = c != 0;
        }
    } else {
        uint32_t jp[6];
        packed_decode<false>(A.pk, (uint32_t)i, w.W, jp);
#pragma unroll
        for (int k = 0; k < 6; k++) {
            j[k] = (CgIdx<NS>)jp[k];
            pres[k] = j[k] != i;
        }
    }
}

// The voxels of a thread in block tile t (clamped to the last voxel).
template <int V, typename I>
__device__ __forceinline__ void cg_own(const CgArgs &A, int64_t t, I (&i)[V], bool (&act)[V]) {
#pragma unroll
    for (int v = 0; v < V; v++) {
        const int64_t x = (t * V + v) * kBlock + threadIdx.x;
        act[v] = x < A.n;
        i[v] = (I)(act[v] ? x : A.n - 1);
    }
}

// Staged form: the window of a tile in LDS, win[q] = voxel t0 - kCgHalo + q;
// a thread's halo voxels (clamped into the volume: a clamped one is nobody's
// neighbour).
constexpr int kCgWin = kCgTileV * kBlock + 2 * kCgHalo;
static_assert(kCgHalo == kBlock, "one halo voxel per thread and side");
__device__ __forceinline__ void cg_halo(const CgArgs &A, int64_t t, uint32_t (&hi)[2]) {
    const int64_t t0 = t * kCgTileV * kBlock, lo = t0 - kCgHalo + threadIdx.x,
                  up = t0 + kCgTileV * kBlock + threadIdx.x;
    hi[0] = (uint32_t)(lo > 0 ? lo : 0);
    hi[1] = (uint32_t)(up < A.n ? up : A.n - 1);
}
__device__ __forceinline__ void cg_stage(double *win, const double (&own)[kCgTileV], const double (&halo)[2]) {
    win[threadIdx.x] = halo[0];
#pragma unroll
    for (int v = 0; v < kCgTileV; v++) win[kCgHalo + v * kBlock + threadIdx.x] = own[v];
    win[kCgHalo + kCgTileV * kBlock + threadIdx.x] = halo[1];
    lds_barrier();
}

// Sums of the G[m] per-block partials of M slots, the same in every thread of
// the block, in a fixed order.  lds: kWaves * M doubles.
template <int M>
__device__ __forceinline__ void reduce_parts(const double *const (&part)[M], const int (&G)[M], double *lds,
                                             double (&out)[M]) {
    // all loads in flight at once (one after the other they cost the start of
    // the kernel a memory latency each)
    constexpr int U = kCgMaxBlocks / kBlock;
    double x[M][U];
#pragma unroll
    for (int m = 0; m < M; m++)
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int b = u * kBlock + (int)threadIdx.x;
            x[m][u] = b < G[m] ? part[m][b] : 0.0;
        }
#pragma unroll
    for (int m = 0; m < M; m++) {
        double v = x[m][0];
#pragma unroll
        for (int u = 1; u < U; u++) v += x[m][u];
        v = wave_sum(v);
        if ((threadIdx.x & 63) == 0) lds[m * kWaves + (threadIdx.x >> 6)] = v;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; m++) {
        out[m] = lds[m * kWaves];
        for (int w = 1; w < kWaves; w++) out[m] += lds[m * kWaves + w];
    }
    __syncthreads();
}
__device__ __forceinline__ double reduce_parts(const double *__restrict__ part, int G, double *lds) {
    const double *const p[1] = {part};
    const int g[1] = {G};
    double v[1];
    reduce_parts<1>(p, g, lds, v);
    return v[0];
}

// Convergence of iterate k (k iterations done) from its r.r; block 0 keeps the
// scalars, once.  True in every thread of every block once converged.
__device__ __forceinline__ bool cg_check(double rr, int k, double bb, double *__restrict__ scal) {
    const bool done = rr <= scal[S_RTOL2] * bb;
    if (blockIdx.x == 0 && threadIdx.x == 0 && scal[S_DONE] == 0.0) {
        scal[S_RR] = rr;
        scal[S_ITER] = (double)k;
        if (done) scal[S_DONE] = 1.0;
    }
    return done;
}

// Start: y = b, r = b - B b; z = M^-1 r (Jacobi), or r for the V-cycle.
template <typename F, bool REG, int NS, bool MG>
__global__ __launch_bounds__(kBlock) void k_cg_init(CgArgs A, F field, double *__restrict__ y,
                                                    double *__restrict__ rz, double *__restrict__ m,
                                                    double *__restrict__ part) {
    __shared__ double lds[kWaves * 3];
    __shared__ double cl[VG_NREG];
    if (threadIdx.x < VG_NREG) cl[threadIdx.x] = A.c[threadIdx.x];
    __syncthreads();
    double acc[3] = {0.0, 0.0, 0.0};   // r.z, r.r, b.b
    for (int64_t it = 0;; it++) {
        const int64_t t = xcd_stride_tile(blockIdx.x, gridDim.x, it, A.ntiles);
        if (t >= A.ntiles) break;
        const int64_t i = t * kTile + threadIdx.x;
        if (i >= A.n) continue;
        const double b = field.get(i);
        int64_t j[6];
        bool pres[6];
        cg_neighbours<NS>(A, i, j, pres);
        double fj[6];
#pragma unroll
        for (int k = 0; k < 6; k++) fj[k] = field.get(j[k]);
        double s = 0.0, deg = 0.0;
#pragma unroll
        for (int k = 0; k < 6; k++) {
            if (!pres[k]) continue;
            const double w = weight(A.rcode, cl, i, k, REG);
            deg += w;
            s += w * (b - fj[k]);
        }
        const double mi = 1.0 / (1.0 + A.a * deg);
        const double ri = b - (b + A.a * s);
        y[i] = b;
        rz[i] = MG ? ri : mi * ri;
        if (REG) m[i] = mi;
        else ((uint8_t *)m)[i] = (uint8_t)deg;   // 1/diag is then one of 7 values
        acc[0] += ri * (mi * ri);
        acc[1] += ri * ri;
        acc[2] += b * b;
    }
    block_sum<3>(acc, lds);
    if (threadIdx.x == 0) {
        if (!MG) part[P_RZ * A.ldp + (int)blockIdx.x] = acc[0];
        part[P_RR * A.ldp + (int)blockIdx.x] = acc[1];
        part[P_BB * A.ldp + (int)blockIdx.x] = acc[2];
    }
}

// Partials of (z, B z) of iteration k; before that r.z of iterate k from its
// Gp partials, (p, q) and (z, q) of the iteration before from its Gs, and for
// Jacobi the convergence check (the V-cycle has done it).
// In every gathering kernel a tile's neighbour words are loaded one tile
// ahead, so that its gathers wait for nothing; the staged window is double
// buffered (one barrier per tile).
// 512^3 (22.8 M voxels): 125 us direct, 92 us staged (12.5 B per voxel).
template <bool REG, int NS, bool MG, int V>
__global__ __launch_bounds__(kBlock) void k_cg_dot(CgArgs A, int k, int Gp, int Gs, const double *__restrict__ z,
                                                   double *__restrict__ scal, double *__restrict__ part) {
    if (MG && scal[S_DONE] != 0.0) return;   // (Jacobi: this kernel's own check below)
    constexpr bool ST = V > 1;
    __shared__ double win[ST ? 2 : 1][ST ? kCgWin : 1];
    __shared__ double lds[kWaves * 3];
    __shared__ double cl[VG_NREG];
    if (threadIdx.x < VG_NREG) cl[threadIdx.x] = A.c[threadIdx.x];
    __syncthreads();
    // block 0 adds up what the next kernel needs, in one go (one sum after the
    // other would hold up the kernel; before the first direction (z, q) and
    // (p, q) hold nothing and are not used)
    if (blockIdx.x == 0) {
        const double *const p[3] = {part + P_RZ * A.ldp, part + P_ZQ * A.ldp, part + P_PQ * A.ldp};
        const int Gq = k == 0 ? 0 : Gs, G[3] = {Gp, Gq, Gq};
        double v[3];
        reduce_parts<3>(p, G, lds, v);
        if (threadIdx.x == 0) {
            scal[S_RZ + (k & 1)] = v[0];
            scal[S_ZQ] = MG ? (v[1] - v[0]) / scal[S_ALPHA + ((k & 1) ^ 1)] : v[1];
            scal[S_PQ] = v[2];
        }
    }
    if (!MG && cg_check(reduce_parts(part + P_RR * A.ldp, Gp, lds), k, scal[S_BB], scal)) return;
    const int64_t nt = (A.n + kBlock * V - 1) / (kBlock * V);
    double acc[1] = {0.0};
    int64_t t = xcd_stride_tile(blockIdx.x, gridDim.x, 0, nt, A.run);
    CgIdx<NS> i[V];
    bool act[V];
    CgWords<NS> w[V];
    cg_own(A, t, i, act);
#pragma unroll
    for (int v = 0; v < V; v++) cg_words<NS>(A, i[v], w[v]);
    for (int64_t it = 1; t < nt; it++) {
        bool pres[V][6];
        double zi[V], zj[V][6];
        [[maybe_unused]] uint32_t q[V][4];
        [[maybe_unused]] double hz[2];
#pragma unroll
        for (int v = 0; v < V; v++) {
            CgIdx<NS> j[6];
            cg_decode<NS>(A, i[v], w[v], j, pres[v]);
            zi[v] = el(z, i[v]);
#pragma unroll
            for (int k6 = ST ? 4 : 0; k6 < 6; k6++) zj[v][k6] = el(z, j[k6]);
            if constexpr (ST) {
#pragma unroll
                for (int k4 = 0; k4 < 4; k4++) q[v][k4] = (uint32_t)(j[k4] - (uint32_t)(t * V * kBlock)) + kCgHalo;
            }
        }
        if constexpr (ST) {
            uint32_t hi[2];
            cg_halo(A, t, hi);
            hz[0] = el(z, hi[0]);
            hz[1] = el(z, hi[1]);
        }
        t = xcd_stride_tile(blockIdx.x, gridDim.x, it, nt, A.run);
        CgIdx<NS> in[V];
        bool an[V];
        cg_own(A, t, in, an);
#pragma unroll
        for (int v = 0; v < V; v++) cg_words<NS>(A, in[v], w[v]);
        if constexpr (ST) {
            double *wb = win[it & 1];
            cg_stage(wb, zi, hz);
#pragma unroll
            for (int v = 0; v < V; v++)
#pragma unroll
                for (int k4 = 0; k4 < 4; k4++) zj[v][k4] = wb[q[v][k4]];
        }
#pragma unroll
        for (int v = 0; v < V; v++) {
            double s = 0.0;
#pragma unroll
            for (int k6 = 0; k6 < 6; k6++) {
                const double wt = weight(A.rcode, cl, i[v], k6, REG);
                s += pres[v][k6] ? wt * (zi[v] - zj[v][k6]) : 0.0;
            }
            acc[0] += act[v] ? zi[v] * (zi[v] + A.a * s) : 0.0;
            i[v] = in[v];
            act[v] = an[v];
        }
    }
    block_sum<1>(acc, lds);
    if (threadIdx.x == 0) part[P_ZBZ * A.ldp + (int)blockIdx.x] = acc[0];
}

// Iteration k's update: alpha and beta from the Gp partials of (z, B z),
// p = z + beta p_old (for the neighbours too), q = B p, then z' = z - alpha
// M^-1 q (Jacobi, into zr) or r -= alpha q (MG, zr in place).  Odd k also add
// the last two directions to y.  512^3: 325 us direct, 255 us staged (44.5 B
// per voxel on average); the two kernels that stored q and r took 343 and
// 151 us.
template <bool REG, int NS, bool MG, int V>
__global__ __launch_bounds__(kBlock) void k_cg_step(CgArgs A, int k, int Gp, const double *__restrict__ z,
                                                    const double *__restrict__ pold, double *__restrict__ pnew,
                                                    double *__restrict__ y, double *__restrict__ zr,
                                                    double *__restrict__ scal, double *__restrict__ part) {
    if (scal[S_DONE] != 0.0) return;
    constexpr bool ST = V > 1;
    __shared__ double win[ST ? 2 : 1][ST ? kCgWin : 1];
    __shared__ double lds[kWaves * 2];
    __shared__ double sum[kQuads * (MG ? 3 : 4)];
    __shared__ double cl[VG_NREG];
    __shared__ double mtab[8];
    if (threadIdx.x < VG_NREG) cl[threadIdx.x] = A.c[threadIdx.x];
    if (!MG && !REG && threadIdx.x < 7) mtab[threadIdx.x] = 1.0 / (1.0 + A.a * (double)threadIdx.x);
    __syncthreads();
    const double zbz = reduce_parts(part + P_ZBZ * A.ldp, Gp, lds);
    const double rz = scal[S_RZ + (k & 1)];
    const double aold = k > 0 ? scal[S_ALPHA + ((k & 1) ^ 1)] : 0.0;
    double beta = k > 0 ? rz / scal[S_RZ + ((k & 1) ^ 1)] : 0.0;
    double pbp = k > 0 ? zbz + beta * (2.0 * scal[S_ZQ] + beta * scal[S_PQ]) : zbz;
    if (pbp <= 0.0) {   // lost to rounding (B is positive definite): restart from p = z
        beta = 0.0;
        pbp = zbz;
    }
    const double alpha = rz / pbp;
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[S_ALPHA + (k & 1)] = alpha;
    const bool add = (k & 1) != 0, first = k == 0;   // p_old holds nothing before the first direction
    const int64_t nt = (A.n + kBlock * V - 1) / (kBlock * V);
    constexpr int M = MG ? 3 : 4;
    double acc[M] = {};   // (Jacobi: r.z,) (z, q) or (r, z_old), (p, q), r.r
    int64_t t = xcd_stride_tile(blockIdx.x, gridDim.x, 0, nt, A.run);
    CgIdx<NS> i[V];
    bool act[V];
    CgWords<NS> w[V];
    cg_own(A, t, i, act);
#pragma unroll
    for (int v = 0; v < V; v++) cg_words<NS>(A, i[v], w[v]);
    for (int64_t it = 1; t < nt; it++) {
        constexpr int K0 = ST ? 4 : 0;   // the slots gathered from memory
        bool pres[V][6];
        double zi[V], po[V], zj[V][6], oj[V][6], yi[V], ri[V];
        [[maybe_unused]] uint32_t q[V][4];
        [[maybe_unused]] double hz[2], ho[2];
#pragma unroll
        for (int v = 0; v < V; v++) {
            CgIdx<NS> j[6];
            cg_decode<NS>(A, i[v], w[v], j, pres[v]);
            zi[v] = el(z, i[v]);
            po[v] = first ? 0.0 : el(pold, i[v]);
#pragma unroll
            for (int k6 = K0; k6 < 6; k6++) zj[v][k6] = el(z, j[k6]);
#pragma unroll
            for (int k6 = K0; k6 < 6; k6++) oj[v][k6] = first ? 0.0 : el(pold, j[k6]);
            yi[v] = add ? el(y, i[v]) : 0.0;
            ri[v] = MG ? el(zr, i[v]) : 0.0;
            if constexpr (ST) {
#pragma unroll
                for (int k4 = 0; k4 < 4; k4++) q[v][k4] = (uint32_t)(j[k4] - (uint32_t)(t * V * kBlock)) + kCgHalo;
            }
        }
        if constexpr (ST) {
            uint32_t hi[2];
            cg_halo(A, t, hi);
#pragma unroll
            for (int u = 0; u < 2; u++) {
                hz[u] = el(z, hi[u]);
                ho[u] = first ? 0.0 : el(pold, hi[u]);
            }
        }
        t = xcd_stride_tile(blockIdx.x, gridDim.x, it, nt, A.run);
        CgIdx<NS> in[V];
        bool an[V];
        cg_own(A, t, in, an);
#pragma unroll
        for (int v = 0; v < V; v++) cg_words<NS>(A, in[v], w[v]);
        // p = z + beta p_old of the voxel (po becomes it below) and its neighbours
        double pi[V];
#pragma unroll
        for (int v = 0; v < V; v++) {
            pi[v] = zi[v] + beta * po[v];
#pragma unroll
            for (int k6 = K0; k6 < 6; k6++) zj[v][k6] += beta * oj[v][k6];
        }
        if constexpr (ST) {
#pragma unroll
            for (int u = 0; u < 2; u++) hz[u] += beta * ho[u];
            double *wb = win[it & 1];
            cg_stage(wb, pi, hz);
#pragma unroll
            for (int v = 0; v < V; v++)
#pragma unroll
                for (int k4 = 0; k4 < 4; k4++) zj[v][k4] = wb[q[v][k4]];
        }
#pragma unroll
        for (int v = 0; v < V; v++) {
            double s = 0.0, deg = 0.0;
#pragma unroll
            for (int k6 = 0; k6 < 6; k6++) {
                const double wt = weight(A.rcode, cl, i[v], k6, REG);
                deg += pres[v][k6] ? wt : 0.0;
                s += pres[v][k6] ? wt * (pi[v] - zj[v][k6]) : 0.0;
            }
            const double qi = pi[v] + A.a * s;
            double rn, zn = 0.0;
            if (MG) {
                rn = ri[v] - alpha * qi;
            } else {
                const double di = 1.0 + A.a * deg;
                const double mi = REG ? 1.0 / di : mtab[(int)deg];
                zn = zi[v] - alpha * (mi * qi);
                rn = di * zn;
            }
            if (act[v]) {
                el(pnew, i[v]) = pi[v];
                if (add) el(y, i[v]) = yi[v] + (aold * po[v] + alpha * pi[v]);
                el(zr, i[v]) = MG ? rn : zn;
                if constexpr (!MG) acc[0] += rn * zn;
                acc[M - 3] += MG ? rn * zi[v] : zn * qi;
                acc[M - 2] += pi[v] * qi;
                acc[M - 1] += rn * rn;
            }
            i[v] = in[v];
            act[v] = an[v];
        }
    }
    tile_sum_to<M>(acc, sum, part + (MG ? P_ZQ : P_RZ) * A.ldp + (int)blockIdx.x, A.ldp);   // (MG: the V-cycle writes r.z)
}

// The scalars of iterate k for the host (one block); k = 0: b.b too.
__global__ __launch_bounds__(kBlock) void k_cg_status(int ldp, int Gp, int k, double *__restrict__ scal,
                                                      const double *__restrict__ part) {
    if (scal[S_DONE] != 0.0) return;
    __shared__ double lds[kWaves];
    double bb = scal[S_BB];
    if (k == 0) {
        bb = reduce_parts(part + P_BB * ldp, Gp, lds);
        if (threadIdx.x == 0) scal[S_BB] = bb;
    }
    cg_check(reduce_parts(part + P_RR * ldp, Gp, lds), k, bb, scal);
}

// The solution, rounded to the field storage; an odd number of iterations
// leaves the last direction to add (p: the buffer that holds it).
template <typename F>
__global__ __launch_bounds__(kBlock) void k_cg_writeback(int64_t n, const double *__restrict__ y,
                                                         const double *__restrict__ p, int add,
                                                         const double *__restrict__ scal, F field) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) field.put(i, add ? y[i] + scal[S_ALPHA] * p[i] : y[i]);
}

// ---------------------------------------------------------------- multigrid

// One level of the hierarchy as the kernels see it (levels >= 1).
struct MgView {
    const int32_t *nbr;
    const float *w, *mass;
    const double *invd;
    double *r, *x, *e;
    const uint32_t *parent;
    const RankWord *rank;
    const int32_t *vox;
    int64_t n, ld;
    Geom g;
};

// Diagonal inverse of the fine level, 1 / (1 + a sum_j w_ij): from the
// vector the init kernel wrote (region weights) or from the neighbour count.
template <bool REG, typename I>
__device__ __forceinline__ double fine_minv(const double *m, const double *mtab, I i) {
    return REG ? el(m, i) : mtab[el((const uint8_t *)m, i)];
}

// Calls f(i, d) for the cells i of level l inside cell (X, Y, Z) of level
// l + 1, in the fixed order z, y, x ascending; d = dx | dy << 1 | dz << 2 is
// the child's offset inside the 2x2x2 block.
template <typename Fn>
__device__ __forceinline__ void mg_children(const RankWord *rank, const Geom &g, int X, int Y, int Z, Fn &&f) {
    for (int dz = 0; dz < 2; dz++) {
        const int z = 2 * Z + dz;
        if (z >= g.nz) break;
        for (int dy = 0; dy < 2; dy++) {
            const int y = 2 * Y + dy;
            if (y >= g.ny) break;
            for (int dx = 0; dx < 2; dx++) {
                const int x = 2 * X + dx;
                if (x >= g.nx) break;
                const int64_t p = geom_pos(g, x, y, z);
                const int32_t i = rank_lookup(rank[p >> 5], (uint32_t)p);
                if (i >= 0) f((int64_t)i, dx | (dy << 1) | (dz << 2));
            }
        }
    }
}

__device__ __forceinline__ void mg_cell_xyz(const int32_t *vox, int64_t i, int nx, int ny, int &x, int &y, int &z) {
    const int v = vox[i];
    x = v % nx;
    y = (v / nx) % ny;
    z = v / (nx * ny);
}

// set-up: occupancy of the next grid (every writer writes 1)
__global__ __launch_bounds__(kBlock) void k_mg_mark(const int32_t *__restrict__ vox, int64_t n, int nx, int ny,
                                                    int cnx, int cny, uint8_t *__restrict__ mask) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    int x, y, z;
    mg_cell_xyz(vox, i, nx, ny, x, y, z);
    mask[(x >> 1) + (int64_t)cnx * ((y >> 1) + (int64_t)cny * (z >> 1))] = 1;
}

// set-up: the cell of the next level that holds each cell, in the low 27
// bits (the grids are at most 1024^3, so a coarse one has at most 2^27
// cells), and above them the cell's outer neighbours (those outside its
// 2x2x2 block, one per axis) as a base-3 number, x first: per axis 0 absent,
// 1 on the minus side (even coordinate), 2 on the plus side.
constexpr int kParentBits = 27;
__global__ __launch_bounds__(kBlock) void k_mg_parent(const int32_t *__restrict__ vox, int64_t n, int nx, int ny,
                                                      const RankWord *__restrict__ crank, Geom cg,
                                                      const int32_t *__restrict__ nbr, int64_t ld,
                                                      uint32_t *__restrict__ parent) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    int x, y, z;
    mg_cell_xyz(vox, i, nx, ny, x, y, z);
    const int64_t p = geom_pos(cg, x >> 1, y >> 1, z >> 1);
    const int odd[3] = {x & 1, y & 1, z & 1};
    uint32_t c = 0, unit = 1;
#pragma unroll
    for (int axis = 0; axis < 3; axis++) {
        if (nbr[(int64_t)(2 * axis + odd[axis]) * ld + i] >= 0) c += unit * (uint32_t)(1 + odd[axis]);
        unit *= 3;
    }
    parent[i] = (uint32_t)rank_lookup(crank[p >> 5], (uint32_t)p) | c << kParentBits;
}

// A parent word's cell, and the slot of the outer neighbour of each axis (-1 absent).
__device__ __forceinline__ int64_t mg_parent_cell(uint32_t w, int (&slot)[3]) {
    const uint32_t c = w >> kParentBits;
    const uint32_t s2 = (c * 57u) >> 9, r = c - 9u * s2, s1 = (r * 11u) >> 5, s0 = r - 3u * s1;   // c / 9, r / 3
    slot[0] = (int)s0 - 1;
    slot[1] = s1 ? 1 + (int)s1 : -1;
    slot[2] = s2 ? 3 + (int)s2 : -1;
    return (int64_t)(w & ((1u << kParentBits) - 1u));
}

// set-up: mass and face weights of the cells of level l + 1 from level l
// (fine level: unit masses and the step's edge weights).  The weight of face
// k sums, over the children on that face (fixed order), the weight of their
// edge in direction k; the neighbour cell sums the same edges in the same
// order from its side, so both ends hold the same float.
template <bool FINE, bool REG>
__global__ __launch_bounds__(kBlock) void k_mg_coarse_op(const RankWord *__restrict__ rank, Geom g,
                                                         const int32_t *__restrict__ nbr, int64_t ld,
                                                         const float *__restrict__ w, const float *__restrict__ mass,
                                                         const uint16_t *__restrict__ rcode, CgArgs A,
                                                         const int32_t *__restrict__ cvox, int64_t cn, int cnx,
                                                         int cny, float *__restrict__ cmass,
                                                         float *__restrict__ cw, int64_t cld) {
    __shared__ double cl[VG_NREG];
    if (threadIdx.x < VG_NREG) cl[threadIdx.x] = A.c[threadIdx.x];
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= cn) return;
    int X, Y, Z;
    mg_cell_xyz(cvox, c, cnx, cny, X, Y, Z);
    double m = 0.0, wk[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    mg_children(rank, g, X, Y, Z, [&](int64_t i, int d) {
        m += FINE ? 1.0 : (double)mass[i];
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const int axis = k >> 1, plus = k & 1;
            if (((d >> axis) & 1) != plus) continue;   // not on face k of the block
            if (nbr[(int64_t)k * ld + i] < 0) continue;
            if (FINE) wk[k] += weight(rcode, cl, i, k, REG);
            else wk[k] += (double)w[(int64_t)k * ld + i];
        }
    });
    cmass[c] = (float)m;
#pragma unroll
    for (int k = 0; k < 6; k++) cw[(int64_t)k * cld + c] = (float)wk[k];
}

// per solve: 1 / diag of every cell, mass + a sum_k w_k
__global__ __launch_bounds__(kBlock) void k_mg_invd(const float *__restrict__ w, const float *__restrict__ mass,
                                                    int64_t n, int64_t ld, double a, double *__restrict__ invd) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 6; k++) s += (double)w[(int64_t)k * ld + i];
    invd[i] = 1.0 / ((double)mass[i] + a * s);
}

// Fine-level residual of the pre-smoothed iterate x0 = w D^-1 r, which is
// formed in registers for the voxel and its neighbours: t = r - B x0, V voxels
// per thread (staged form: kCgTileV).  With rr_part, first the convergence check of iterate k
// from its Gp residual partials.
template <bool REG, int NS, int V>
__global__ __launch_bounds__(kBlock) void k_mg_res0(CgArgs A, int k, const double *__restrict__ r,
                                                    const double *__restrict__ m, double *__restrict__ t,
                                                    double *__restrict__ scal,
                                                    const double *__restrict__ rr_part, int Gp) {
    if (!rr_part && scal[S_DONE] != 0.0) return;   // (with rr_part: this kernel's own check below)
    constexpr bool ST = V > 1;
    __shared__ double win[ST ? 2 : 1][ST ? kCgWin : 1];
    __shared__ double lds[kWaves];
    __shared__ double cl[VG_NREG];
    __shared__ double mtab[8];
    if (threadIdx.x < VG_NREG) cl[threadIdx.x] = A.c[threadIdx.x];
    if (!REG && threadIdx.x < 7) mtab[threadIdx.x] = 1.0 / (1.0 + A.a * (double)threadIdx.x);
    __syncthreads();
    if (rr_part && cg_check(reduce_parts(rr_part, Gp, lds), k, scal[S_BB], scal)) return;
    const int64_t nt = (A.n + kBlock * V - 1) / (kBlock * V);
    int64_t tl = xcd_stride_tile(blockIdx.x, gridDim.x, 0, nt, A.run);
    CgIdx<NS> i[V];
    bool act[V];
    CgWords<NS> w[V];
    cg_own(A, tl, i, act);
#pragma unroll
    for (int v = 0; v < V; v++) cg_words<NS>(A, i[v], w[v]);
    for (int64_t it = 1; tl < nt; it++) {
        constexpr int K0 = ST ? 4 : 0;   // the slots gathered from memory
        bool pres[V][6];
        double ri[V], mi[V], xj[V][6], mj[V][6];
        [[maybe_unused]] uint32_t q[V][4];
        [[maybe_unused]] double hx[2], hm[2];
#pragma unroll
        for (int v = 0; v < V; v++) {
            CgIdx<NS> j[6];
            cg_decode<NS>(A, i[v], w[v], j, pres[v]);
            ri[v] = el(r, i[v]);
#pragma unroll
            for (int k6 = K0; k6 < 6; k6++) xj[v][k6] = el(r, j[k6]);
            mi[v] = fine_minv<REG>(m, mtab, i[v]);
#pragma unroll
            for (int k6 = K0; k6 < 6; k6++) mj[v][k6] = fine_minv<REG>(m, mtab, j[k6]);
            if constexpr (ST) {
#pragma unroll
                for (int k4 = 0; k4 < 4; k4++) q[v][k4] = (uint32_t)(j[k4] - (uint32_t)(tl * V * kBlock)) + kCgHalo;
            }
        }
        if constexpr (ST) {
            uint32_t hi[2];
            cg_halo(A, tl, hi);
#pragma unroll
            for (int u = 0; u < 2; u++) {
                hx[u] = el(r, hi[u]);
                hm[u] = fine_minv<REG>(m, mtab, hi[u]);
            }
        }
        tl = xcd_stride_tile(blockIdx.x, gridDim.x, it, nt, A.run);
        CgIdx<NS> in[V];
        bool an[V];
        cg_own(A, tl, in, an);
#pragma unroll
        for (int v = 0; v < V; v++) cg_words<NS>(A, in[v], w[v]);
        double xi[V];
#pragma unroll
        for (int v = 0; v < V; v++) {
            xi[v] = kMgOmega * ri[v] * mi[v];
#pragma unroll
            for (int k6 = K0; k6 < 6; k6++) xj[v][k6] = kMgOmega * xj[v][k6] * mj[v][k6];
        }
        if constexpr (ST) {
#pragma unroll
            for (int u = 0; u < 2; u++) hx[u] = kMgOmega * hx[u] * hm[u];
            double *wb = win[it & 1];
            cg_stage(wb, xi, hx);
#pragma unroll
            for (int v = 0; v < V; v++)
#pragma unroll
                for (int k4 = 0; k4 < 4; k4++) xj[v][k4] = wb[q[v][k4]];
        }
#pragma unroll
        for (int v = 0; v < V; v++) {
            double s = 0.0;
#pragma unroll
            for (int k6 = 0; k6 < 6; k6++) {
                const double wt = weight(A.rcode, cl, i[v], k6, REG);
                s += pres[v][k6] ? wt * (xi[v] - xj[v][k6]) : 0.0;
            }
            if (act[v]) el(t, i[v]) = ri[v] - (xi[v] + A.a * s);
            i[v] = in[v];
            act[v] = an[v];
        }
    }
}

// Residual on level l >= 1 (into e): r - B x.
__global__ __launch_bounds__(kBlock) void k_mg_res(MgView L, double a, const double *__restrict__ scal) {
    if (scal[S_DONE] != 0.0) return;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= L.n) return;
    const double xi = L.x[i];
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const int32_t j = L.nbr[(int64_t)k * L.ld + i];
        if (j >= 0) s += (double)L.w[(int64_t)k * L.ld + i] * (xi - L.x[j]);
    }
    L.e[i] = L.r[i] - ((double)L.mass[i] * xi + a * s);
}

// Restriction, one thread per cell of the coarser level C: the sum of the
// finer level's residuals over its children (fixed order); also C's
// pre-smoothed iterate w D^-1 r.  (Eight lanes per cell with a butterfly sum
// measured twice as slow at 512^3.)
__global__ __launch_bounds__(kBlock) void k_mg_sum(const RankWord *__restrict__ rank, Geom g,
                                                   const double *__restrict__ res, MgView C,
                                                   const double *__restrict__ scal) {
    if (scal[S_DONE] != 0.0) return;
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= C.n) return;
    int X, Y, Z;
    mg_cell_xyz(C.vox, c, C.g.nx, C.g.ny, X, Y, Z);
    double sum = 0.0;
    mg_children(rank, g, X, Y, Z, [&](int64_t i, int) { sum += res[i]; });
    C.r[c] = sum;
    C.x[c] = kMgOmega * sum * C.invd[c];
}

// The coarsest level (at most kMgCoarseMax cells): kMgSweeps damped Jacobi
// sweeps from zero (the first is the x the restriction wrote) in one block,
// the iterate in LDS; the result replaces x.
__global__ __launch_bounds__(kMgCoarseThreads) void k_mg_coarsest(MgView L, double a,
                                                                  const double *__restrict__ scal) {
    if (scal[S_DONE] != 0.0) return;
    __shared__ double xs[2][kMgCoarseMax];
    constexpr int kPer = kMgCoarseMax / kMgCoarseThreads;
    for (int u = 0; u < kPer; u++) {
        const int64_t i = threadIdx.x + (int64_t)u * kMgCoarseThreads;
        if (i < L.n) xs[0][i] = L.x[i];
    }
    __syncthreads();
    int src = 0;
    for (int sweep = 1; sweep < kMgSweeps; sweep++) {
        for (int u = 0; u < kPer; u++) {
            const int64_t i = threadIdx.x + (int64_t)u * kMgCoarseThreads;
            if (i >= L.n) continue;
            const double xi = xs[src][i];
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < 6; k++) {
                const int32_t j = L.nbr[(int64_t)k * L.ld + i];
                if (j >= 0) s += (double)L.w[(int64_t)k * L.ld + i] * (xi - xs[src][j]);
            }
            xs[src ^ 1][i] = xi + kMgOmega * (L.r[i] - ((double)L.mass[i] * xi + a * s)) * L.invd[i];
        }
        __syncthreads();
        src ^= 1;
    }
    for (int u = 0; u < kPer; u++) {
        const int64_t i = threadIdx.x + (int64_t)u * kMgCoarseThreads;
        if (i < L.n) L.x[i] = xs[src][i];
    }
}

// The coarse solution's part of B P e at a cell: sum over the cell's outer
// neighbours of w (e_I - e_J), I its parent and J the parent's neighbour on
// that side.
template <typename W>
__device__ __forceinline__ double mg_outer(const int32_t *__restrict__ cnbr, int64_t cld,
                                           const double *__restrict__ e, int64_t I, double eI, const int (&slot)[3],
                                           W &&w) {
    int64_t J[3];
    double eJ[3];
#pragma unroll
    for (int axis = 0; axis < 3; axis++) J[axis] = slot[axis] >= 0 ? (int64_t)cnbr[(int64_t)slot[axis] * cld + I] : I;
#pragma unroll
    for (int axis = 0; axis < 3; axis++) eJ[axis] = e[J[axis]];
    double s = 0.0;
#pragma unroll
    for (int axis = 0; axis < 3; axis++)
        if (slot[axis] >= 0) s += w(slot[axis]) * (eI - eJ[axis]);
    return s;
}

// Prolongation and post-smoothing on level l >= 1 (see the top): x <- x +
// P e + w D^-1 (t - B P e), t the residual in e, the coarse solution in C.x.
__global__ __launch_bounds__(kBlock) void k_mg_post(MgView L, MgView C, double a, const double *__restrict__ scal) {
    if (scal[S_DONE] != 0.0) return;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= L.n) return;
    int slot[3];
    const int64_t I = mg_parent_cell(L.parent[i], slot);
    const double eI = C.x[I];
    const double s = mg_outer(C.nbr, C.ld, C.x, I, eI, slot,
                              [&](int q) { return (double)L.w[(int64_t)q * L.ld + i]; });
    L.x[i] += eI + kMgOmega * (L.e[i] - ((double)L.mass[i] * eI + a * s)) * L.invd[i];
}

// The same on the fine level, x = w D^-1 r formed from r (512^3: 178 us; as a
// prolongation and a smoothing kernel that gathered the fine iterate 130 +
// 170 us): writes z and the
// per-block r.z partials (the grid-stride blocks of the other CG kernels).
template <bool REG, int NS>
__global__ __launch_bounds__(kBlock) void k_mg_post0(CgArgs A, const double *__restrict__ r,
                                                     const double *__restrict__ m, const double *__restrict__ t,
                                                     const uint32_t *__restrict__ parent, MgView C,
                                                     double *__restrict__ z, const double *__restrict__ scal,
                                                     double *__restrict__ part) {
    if (scal[S_DONE] != 0.0) return;
    __shared__ double lds[kWaves];
    __shared__ double cl[VG_NREG];
    __shared__ double mtab[8];
    if (threadIdx.x < VG_NREG) cl[threadIdx.x] = A.c[threadIdx.x];
    if (!REG && threadIdx.x < 7) mtab[threadIdx.x] = 1.0 / (1.0 + A.a * (double)threadIdx.x);
    __syncthreads();
    constexpr int V = kMgPostV;
    const int64_t nt = (A.n + kBlock * V - 1) / (kBlock * V);
    double acc[1] = {0.0};
    int64_t tl = xcd_stride_tile(blockIdx.x, gridDim.x, 0, nt, A.run);
    CgIdx<NS> i[V];
    uint32_t pw[V];
    bool act[V];
    cg_own(A, tl, i, act);
#pragma unroll
    for (int v = 0; v < V; v++) pw[v] = el(parent, i[v]);
    for (int64_t it = 1; tl < nt; it++) {
        double ri[V], ti[V], mi[V], eI[V], s[V];
#pragma unroll
        for (int v = 0; v < V; v++) {
            ri[v] = el(r, i[v]);
            ti[v] = el(t, i[v]);
            mi[v] = fine_minv<REG>(m, mtab, i[v]);
            int slot[3];
            const int64_t I = mg_parent_cell(pw[v], slot);
            eI[v] = C.x[I];
            s[v] = mg_outer(C.nbr, C.ld, C.x, I, eI[v], slot,
                            [&](int q) { return weight(A.rcode, cl, i[v], q, REG); });
        }
        tl = xcd_stride_tile(blockIdx.x, gridDim.x, it, nt, A.run);
        CgIdx<NS> in[V];
        bool an[V];
        cg_own(A, tl, in, an);
#pragma unroll
        for (int v = 0; v < V; v++) pw[v] = el(parent, in[v]);
#pragma unroll
        for (int v = 0; v < V; v++) {
            const double zi = kMgOmega * ri[v] * mi[v] + eI[v] + kMgOmega * (ti[v] - (eI[v] + A.a * s[v])) * mi[v];
            if (act[v]) {
                el(z, i[v]) = zi;
                acc[0] += ri[v] * zi;
            }
            i[v] = in[v];
            act[v] = an[v];
        }
    }
    block_sum<1>(acc, lds);
    if (threadIdx.x == 0) part[P_RZ * A.ldp + (int)blockIdx.x] = acc[0];
}

// Jacobi as a separate map (vg_precondition): z = D^-1 r.
template <bool REG>
__global__ __launch_bounds__(kBlock) void k_mg_jacobi(int64_t n, double a, const double *__restrict__ r,
                                                      const double *__restrict__ m, double *__restrict__ z) {
    __shared__ double mtab[8];
    if (!REG && threadIdx.x < 7) mtab[threadIdx.x] = 1.0 / (1.0 + a * (double)threadIdx.x);
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) z[i] = fine_minv<REG>(m, mtab, i) * r[i];
}

// The fine diagonal for a given a (what the init kernel writes into m).
template <bool REG, int NS>
__global__ __launch_bounds__(kBlock) void k_mg_fine_diag(CgArgs A, double *__restrict__ m) {
    __shared__ double cl[VG_NREG];
    if (threadIdx.x < VG_NREG) cl[threadIdx.x] = A.c[threadIdx.x];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= A.n) return;
    int64_t j[6];
    bool pres[6];
    cg_neighbours<NS>(A, i, j, pres);
    double deg = 0.0;
#pragma unroll
    for (int k = 0; k < 6; k++)
        if (pres[k]) deg += weight(A.rcode, cl, i, k, REG);
    if (REG) m[i] = 1.0 / (1.0 + A.a * deg);
    else ((uint8_t *)m)[i] = (uint8_t)deg;
}

inline unsigned mg_grid(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

MgView mg_view(vg_sim *h, int l) {
    vg_sim::MgLevel &L = h->mg[l];
    MgView v;
    v.nbr = L.nbr;
    v.w = L.w;
    v.mass = L.mass;
    v.invd = L.invd;
    v.r = L.r;
    v.x = L.x;
    v.e = L.e;
    v.parent = L.parent;
    v.rank = L.rank;
    v.vox = L.vox;
    v.n = L.n;
    v.ld = L.cap;
    make_geom(L.nx, L.ny, L.nz, 0, &v.g);
    return v;
}

Geom fine_geom(const vg_sim *h) {
    Geom g;
    make_geom(h->nx, h->ny, h->nz, h->brick, &g);
    return g;
}

CgArgs cg_args(const vg_sim *h, double a, int V = 1) {
    CgArgs A;
    A.nbr = h->nbr;
    A.rcode = h->rcode;
    A.pk = packed_of(h);
    A.n = h->n;
    A.ntiles = h->ntiles;
    A.a = a;
    A.ldp = h->cg_blocks;
    A.run = xcd_run(h, V);
    for (int k = 0; k < VG_NREG; k++) A.c[k] = h->c[k];
    return A;
}

// coarse weights for the current region factors (the structure is fixed)
int mg_weights(vg_sim *h, hipStream_t s) {
    const bool reg = h->rcode != nullptr;
    const CgArgs A = cg_args(h, 0.0);
    const Geom g0 = fine_geom(h);
    for (int l = 0; l + 1 < h->mg_levels; l++) {
        const vg_sim::MgLevel &F = h->mg[l];
        vg_sim::MgLevel &C = h->mg[l + 1];
        if (l == 0) {
            if (reg) hipLaunchKernelGGL((k_mg_coarse_op<true, true>), dim3(mg_grid(C.n)), dim3(kBlock), 0, s,
                                        (const RankWord *)h->rank, g0, h->nbr, h->n, nullptr, nullptr, h->rcode, A,
                                        C.vox, C.n, C.nx, C.ny, C.mass, C.w, C.cap);
            else hipLaunchKernelGGL((k_mg_coarse_op<true, false>), dim3(mg_grid(C.n)), dim3(kBlock), 0, s,
                                    (const RankWord *)h->rank, g0, h->nbr, h->n, nullptr, nullptr, h->rcode, A,
                                    C.vox, C.n, C.nx, C.ny, C.mass, C.w, C.cap);
        } else {
            const MgView fv = mg_view(h, l);
            hipLaunchKernelGGL((k_mg_coarse_op<false, false>), dim3(mg_grid(C.n)), dim3(kBlock), 0, s, F.rank, fv.g,
                               F.nbr, F.cap, F.w, F.mass, nullptr, A, C.vox, C.n, C.nx, C.ny, C.mass, C.w, C.cap);
        }
        int rc = launch_status("k_mg_coarse_op");
        if (rc) return rc;
    }
    h->mg_wdone = true;
    return VG_OK;
}

// 1 / diag of every coarse level for this a (and the weights if stale)
int mg_prepare(vg_sim *h, double a, hipStream_t s) {
    int rc;
    if (!h->mg_wdone && (rc = mg_weights(h, s))) return rc;
    for (int l = 1; l < h->mg_levels; l++) {
        vg_sim::MgLevel &L = h->mg[l];
        hipLaunchKernelGGL(k_mg_invd, dim3(mg_grid(L.n)), dim3(kBlock), 0, s, L.w, L.mass, L.n, L.cap, a, L.invd);
        if ((rc = launch_status("k_mg_invd"))) return rc;
    }
    return VG_OK;
}

// Blocks of a grid-stride kernel over the voxels, V per thread: as many as
// are resident, no more than there is work for, within the partials.
int cg_grid(const vg_sim *h, const void *kernel, int V) {
    const int64_t nt = (h->n + kBlock * V - 1) / (kBlock * V);
    return resident_blocks(kernel, (int)(nt < h->cg_blocks ? nt : h->cg_blocks));
}

template <bool REG, int NS>
int mg_rz_blocks(const vg_sim *h) {
    return cg_grid(h, (const void *)k_mg_post0<REG, NS>, kMgPostV);
}

// z = V-cycle(r) on the fine level, m the fine diagonal as the init kernel
// wrote it; the r.z partials go to slot P_RZ (mg_rz_blocks of them).  Each
// level's result is in x.  Gp > 0: the first kernel also checks the
// convergence of iterate k from its Gp residual partials.
template <bool REG, int NS, int V>
int mg_vcycle(vg_sim *h, const CgArgs &A, int k, int Gp, const double *r, const double *m, double *z,
              hipStream_t s) {
    const int L = h->mg_levels;
    const double a = A.a;
    double *t = h->mg[0].e;   // fine residual
    int rc;
    hipLaunchKernelGGL((k_mg_res0<REG, NS, V>), dim3(cg_grid(h, (const void *)k_mg_res0<REG, NS, V>, V)), dim3(kBlock), 0, s, A,
                       k, r, m, t, h->cg_scal, Gp > 0 ? (const double *)h->cg_part + P_RR * A.ldp : nullptr, Gp);
    if ((rc = launch_status("k_mg_res0"))) return rc;
    hipLaunchKernelGGL(k_mg_sum, dim3(mg_grid(h->mg[1].n)), dim3(kBlock), 0, s, (const RankWord *)h->rank,
                       fine_geom(h), (const double *)t, mg_view(h, 1), h->cg_scal);
    if ((rc = launch_status("k_mg_sum"))) return rc;
    for (int l = 1; l + 1 < L; l++) {
        const MgView F = mg_view(h, l);
        hipLaunchKernelGGL(k_mg_res, dim3(mg_grid(F.n)), dim3(kBlock), 0, s, F, a, h->cg_scal);
        if ((rc = launch_status("k_mg_res"))) return rc;
        hipLaunchKernelGGL(k_mg_sum, dim3(mg_grid(h->mg[l + 1].n)), dim3(kBlock), 0, s, F.rank, F.g,
                           (const double *)F.e, mg_view(h, l + 1), h->cg_scal);
        if ((rc = launch_status("k_mg_sum"))) return rc;
    }
    hipLaunchKernelGGL(k_mg_coarsest, dim3(1), dim3(kMgCoarseThreads), 0, s, mg_view(h, L - 1), a, h->cg_scal);
    if ((rc = launch_status("k_mg_coarsest"))) return rc;
    for (int l = L - 2; l >= 1; l--) {
        hipLaunchKernelGGL(k_mg_post, dim3(mg_grid(h->mg[l].n)), dim3(kBlock), 0, s, mg_view(h, l), mg_view(h, l + 1),
                           a, h->cg_scal);
        if ((rc = launch_status("k_mg_post"))) return rc;
    }
    hipLaunchKernelGGL((k_mg_post0<REG, NS>), dim3(mg_rz_blocks<REG, NS>(h)), dim3(kBlock), 0, s,
                       cg_args(h, a, kMgPostV), r, m, (const double *)t,
                       (const uint32_t *)h->mg[0].parent, mg_view(h, 1), z, h->cg_scal,
                       h->cg_part);
    return launch_status("k_mg_post0");
}

// storage of one pool of the bound fields
template <typename F>
F pool_acc(vg_sim *h, int pool);
template <>
PlainAcc<float> pool_acc<PlainAcc<float>>(vg_sim *h, int pool) {
    return PlainAcc<float>{(float *)h->fields + (int64_t)pool * h->n};
}
template <>
PlainAcc<double> pool_acc<PlainAcc<double>>(vg_sim *h, int pool) {
    return PlainAcc<double>{(double *)h->fields + (int64_t)pool * h->n};
}
template <>
CompAcc pool_acc<CompAcc>(vg_sim *h, int pool) {
    return CompAcc{(float *)h->fields + (int64_t)pool * h->n, h->lo + (int64_t)pool * h->n};
}

template <typename F, int NS, bool REG, bool MG, int V>
int cg_solve_t(vg_sim *h, int pool, double a, double rtol, int max_iter, int *iters, double *relres,
               hipStream_t s) {
    const CgArgs A = cg_args(h, a, V);
    const int Gi = cg_grid(h, (const void *)k_cg_init<F, REG, NS, MG>, 1);
    const int Gd = cg_grid(h, (const void *)k_cg_dot<REG, NS, MG, V>, V);
    const int Gs = cg_grid(h, (const void *)k_cg_step<REG, NS, MG, V>, V);
    const F field = pool_acc<F>(h, pool);
    int rc;
    // squared tolerance (compared with squared norms; rtol^2 is exact enough)
    double host_scal[S_NSCAL] = {};
    host_scal[S_RTOL2] = rtol * rtol;
    if ((rc = hip_status(hipMemcpyAsync(h->cg_scal, host_scal, sizeof(host_scal), hipMemcpyHostToDevice, s),
                         "cg scalars"))) return rc;
    if (MG && (rc = mg_prepare(h, a, s))) return rc;
    // Jacobi: z ping-pongs (iterate k in zb[k & 1]); MG: z and r
    double *zb[2] = {h->cg_z, MG ? h->cg_z : h->cg_r};
    hipLaunchKernelGGL((k_cg_init<F, REG, NS, MG>), dim3(Gi), dim3(kBlock), 0, s, A, field, h->cg_y,
                       MG ? h->cg_r : zb[0], h->cg_m, h->cg_part);
    if ((rc = launch_status("k_cg_init"))) return rc;
    hipLaunchKernelGGL(k_cg_status, dim3(1), dim3(kBlock), 0, s, A.ldp, Gi, 0, h->cg_scal, (const double *)h->cg_part);
    if ((rc = launch_status("k_cg_status"))) return rc;
    if (MG && (rc = mg_vcycle<REG, NS, V>(h, A, 0, 0, h->cg_r, h->cg_m, h->cg_z, s))) return rc;

    int launched = 0, todo = 8;
    double back[S_NSCAL], rr0 = 0.0;
    int it0 = 0;
    for (;;) {
        if (launched > 0) {
            hipLaunchKernelGGL(k_cg_status, dim3(1), dim3(kBlock), 0, s, A.ldp, Gs, launched, h->cg_scal,
                               (const double *)h->cg_part);
            if ((rc = launch_status("k_cg_status"))) return rc;
        }
        if ((rc = hip_status(hipMemcpyAsync(back, h->cg_scal, sizeof(back), hipMemcpyDeviceToHost, s),
                             "cg scalars back"))) return rc;
        if ((rc = hip_status(hipStreamSynchronize(s), "cg sync"))) return rc;
        if (back[S_DONE] != 0.0 || launched >= max_iter) break;
        // the next batch: the iterations the convergence so far says are
        // left (kernels past convergence cost a few microseconds each, a
        // host round trip more than that)
        if (launched > 0 && back[S_RR] < rr0 && back[S_RTOL2] * back[S_BB] > 0.0) {
            const double per = (__builtin_log(rr0) - __builtin_log(back[S_RR])) / (double)(launched - it0);
            const double left = (__builtin_log(back[S_RR]) - __builtin_log(back[S_RTOL2] * back[S_BB])) / per;
            todo = left < 2.0 ? 2 : (left < 32.0 ? (int)left + 1 : 32);
        } else {
            todo = 8;
        }
        rr0 = back[S_RR];
        it0 = launched;
        if (todo > max_iter - launched) todo = max_iter - launched;
        for (int it = 0; it < todo; it++) {
            const int k = launched + it;
            hipLaunchKernelGGL((k_cg_dot<REG, NS, MG, V>), dim3(Gd), dim3(kBlock), 0, s, A, k,
                               MG ? mg_rz_blocks<REG, NS>(h) : (k > 0 ? Gs : Gi), Gs, (const double *)zb[k & 1],
                               h->cg_scal, h->cg_part);
            if ((rc = launch_status("k_cg_dot"))) return rc;
            hipLaunchKernelGGL((k_cg_step<REG, NS, MG, V>), dim3(Gs), dim3(kBlock), 0, s, A, k, Gd,
                               (const double *)zb[k & 1], (const double *)h->cg_p[(k & 1) ^ 1], h->cg_p[k & 1], h->cg_y,
                               MG ? h->cg_r : zb[(k & 1) ^ 1], h->cg_scal, h->cg_part);
            if ((rc = launch_status("k_cg_step"))) return rc;
            if (MG && (rc = mg_vcycle<REG, NS, V>(h, A, k + 1, Gs, h->cg_r, h->cg_m, h->cg_z, s))) return rc;
        }
        launched += todo;
    }
    // direction k is in p[k & 1]; after an odd number of iterations the last one (even k) is still to add
    const int done = (int)back[S_ITER];
    hipLaunchKernelGGL((k_cg_writeback<F>), dim3((unsigned)((h->n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       h->n, (const double *)h->cg_y, (const double *)h->cg_p[0], done & 1,
                       (const double *)h->cg_scal, field);
    if ((rc = launch_status("k_cg_writeback"))) return rc;
    if (iters) *iters = done;
    if (relres) *relres = back[S_BB] > 0.0 ? __builtin_sqrt(back[S_RR] / back[S_BB]) : 0.0;
    return back[S_DONE] != 0.0 ? VG_OK : VG_ENOCONV;
}

template <typename F, int NS, int V>
int cg_solve_ns(vg_sim *h, int pool, double a, double rtol, int max_iter, int *iters, double *relres,
                hipStream_t s) {
    const bool mg = h->precond == VG_PRECOND_MG && h->mg_levels >= 2;
    if constexpr (V == 1) {   // (staged: unit weights, see cg_staged)
        if (h->rcode) return mg ? cg_solve_t<F, NS, true, true, V>(h, pool, a, rtol, max_iter, iters, relres, s)
                                : cg_solve_t<F, NS, true, false, V>(h, pool, a, rtol, max_iter, iters, relres, s);
    }
    return mg ? cg_solve_t<F, NS, false, true, V>(h, pool, a, rtol, max_iter, iters, relres, s)
              : cg_solve_t<F, NS, false, false, V>(h, pool, a, rtol, max_iter, iters, relres, s);
}

template <int NS, int V>
int mg_apply_ns(vg_sim *h, double a, const double *r, double *z, hipStream_t s) {
    const CgArgs A = cg_args(h, a, V);
    const bool reg = h->rcode != nullptr;
    const bool mg = h->precond == VG_PRECOND_MG && h->mg_levels >= 2;
    int rc;
    if (reg) hipLaunchKernelGGL((k_mg_fine_diag<true, NS>), dim3(mg_grid(h->n)), dim3(kBlock), 0, s, A, h->cg_m);
    else hipLaunchKernelGGL((k_mg_fine_diag<false, NS>), dim3(mg_grid(h->n)), dim3(kBlock), 0, s, A, h->cg_m);
    if ((rc = launch_status("k_mg_fine_diag"))) return rc;
    if (!mg) {
        if (reg) hipLaunchKernelGGL(k_mg_jacobi<true>, dim3(mg_grid(h->n)), dim3(kBlock), 0, s, h->n, a, r, h->cg_m, z);
        else hipLaunchKernelGGL(k_mg_jacobi<false>, dim3(mg_grid(h->n)), dim3(kBlock), 0, s, h->n, a, r, h->cg_m, z);
        return launch_status("k_mg_jacobi");
    }
    // the V-cycle's kernels check the convergence flag: clear it
    if ((rc = hip_status(hipMemsetAsync(h->cg_scal, 0, sizeof(double) * S_NSCAL, s), "cg scalars"))) return rc;
    if ((rc = mg_prepare(h, a, s))) return rc;
    if constexpr (V == 1) {
        if (reg) return mg_vcycle<true, NS, V>(h, A, 0, 0, r, h->cg_m, z, s);
    }
    return mg_vcycle<false, NS, V>(h, A, 0, 0, r, h->cg_m, z, s);
}

// The FP64 vectors outgrow 32-bit byte offsets.  (A packed source then means
// FP32 fields of 2^29 voxels and more: their codes still fit, and the table
// reads 24 B per voxel and kernel for the codes' 4.5.  560 M voxels: 16.9 ms
// an iteration with the table, 13.8 with codes and 64-bit indices.)
bool cg_wide(const vg_sim *h) { return (uint64_t)h->n * sizeof(double) >= ((uint64_t)1 << 32); }

// The staged kernels: relative codes, x and y distances within the halo,
// enough voxels (see kCgTileV) and unit weights.  Measured, 16 iterations,
// direct over staged: unit weights 1 - 2 M voxels 0.97-1.20, 4 M and more
// 1.00-1.35 (Jacobi), 0.99-1.15 (multigrid); with region weights, whose table
// reads the registers of four voxels leave no waves to hide, 0.76-0.93 and
// 0.84-0.89 at every size from 1 to 16 M.
bool cg_staged(const vg_sim *h) {
    return use_relative(h) && !h->rcode && h->xy_dist >= 0 && h->xy_dist <= kCgHalo && h->n >= kCgStagedMin;
}

template <typename F>
int cg_solve(vg_sim *h, int pool, double a, double rtol, int max_iter, int *iters, double *relres,
             hipStream_t s) {
    if (cg_wide(h)) {
        if constexpr (!std::is_same_v<F, PlainAcc<double>>) {
            if (use_relative(h)) return cg_solve_ns<F, NS_REL | NS_WIDE, 1>(h, pool, a, rtol, max_iter, iters, relres, s);
            if (use_offsets(h)) return cg_solve_ns<F, NS_OFF | NS_WIDE, 1>(h, pool, a, rtol, max_iter, iters, relres, s);
        }
        return cg_solve_ns<F, NS_TABLE, 1>(h, pool, a, rtol, max_iter, iters, relres, s);
    }
    if (cg_staged(h)) return cg_solve_ns<F, NS_REL, kCgTileV>(h, pool, a, rtol, max_iter, iters, relres, s);
    if (use_relative(h)) return cg_solve_ns<F, NS_REL, 1>(h, pool, a, rtol, max_iter, iters, relres, s);
    if (use_offsets(h)) return cg_solve_ns<F, NS_OFF, 1>(h, pool, a, rtol, max_iter, iters, relres, s);
    return cg_solve_ns<F, NS_TABLE, 1>(h, pool, a, rtol, max_iter, iters, relres, s);
}

}  // namespace

void mg_plan(vg_sim *h) {
    h->mg[0].nx = h->nx;
    h->mg[0].ny = h->ny;
    h->mg[0].nz = h->nz;
    h->mg[0].cap = h->n;
    int l = 0;
    while (l + 1 < VG_MG_MAX_LEVELS) {
        const vg_sim::MgLevel &F = h->mg[l];
        if (F.nx <= 1 && F.ny <= 1 && F.nz <= 1) break;
        vg_sim::MgLevel &C = h->mg[l + 1];
        C.nx = (F.nx + 1) / 2;
        C.ny = (F.ny + 1) / 2;
        C.nz = (F.nz + 1) / 2;
        const int64_t cells = (int64_t)C.nx * C.ny * C.nz;
        C.cap = cells < F.cap ? cells : F.cap;   // every cell holds at least one cell of the level below
        l++;
    }
    h->mg_plan_levels = l + 1;
}

int mg_build(vg_sim *h, hipStream_t s) {
    h->mg_levels = 0;
    h->mg_wdone = false;
    if (h->n == 0) return VG_OK;
    h->mg[0].n = h->n;
    int l = 0, rc;
    while (l + 1 < h->mg_plan_levels) {
        const vg_sim::MgLevel &F = h->mg[l];
        if (l > 0 && F.n <= kMgCoarsest) break;
        vg_sim::MgLevel &C = h->mg[l + 1];
        const int32_t *fvox = l == 0 ? h->vox : F.vox;
        uint32_t *fparent = F.parent;
        const size_t cells = (size_t)C.nx * C.ny * C.nz;
        if ((rc = hip_status(hipMemsetAsync(h->mg_mask, 0, cells, s), "clear occupancy"))) return rc;
        hipLaunchKernelGGL(k_mg_mark, dim3(mg_grid(F.n)), dim3(kBlock), 0, s, fvox, F.n, F.nx, F.ny, C.nx, C.ny,
                           h->mg_mask);
        if ((rc = launch_status("k_mg_mark"))) return rc;
        int64_t cn = 0;
        if ((rc = vg_count_pores(h->mg_mask, C.nx, C.ny, C.nz, 0, C.rank, &cn, s))) return rc;
        if (cn < 1 || cn > C.cap) { set_error("multigrid level %d: %lld cells", l + 1, (long long)cn); return VG_EHIP; }
        C.n = cn;
        if ((rc = vg_build_graph(C.rank, C.nx, C.ny, C.nz, 0, 0u, 0, cn, C.cap, C.vox, C.nbr, s))) return rc;
        Geom cg;
        make_geom(C.nx, C.ny, C.nz, 0, &cg);
        hipLaunchKernelGGL(k_mg_parent, dim3(mg_grid(F.n)), dim3(kBlock), 0, s, fvox, F.n, F.nx, F.ny,
                           (const RankWord *)C.rank, cg, l == 0 ? h->nbr : (const int32_t *)F.nbr,
                           l == 0 ? h->n : F.cap, fparent);
        if ((rc = launch_status("k_mg_parent"))) return rc;
        l++;
    }
    h->mg_levels = l + 1;
    if (h->mg_levels >= 2 && h->mg[l].n > kMgCoarseMax) {
        set_error("multigrid: coarsest level of %lld cells", (long long)h->mg[l].n);
        return VG_EINVAL;
    }
    return mg_weights(h, s);
}

int mg_apply(vg_sim *h, double a, const double *r, double *z, hipStream_t s) {
    if (h->n == 0) return VG_OK;
    if (cg_wide(h)) {
        if (use_relative(h)) return mg_apply_ns<NS_REL | NS_WIDE, 1>(h, a, r, z, s);
        if (use_offsets(h)) return mg_apply_ns<NS_OFF | NS_WIDE, 1>(h, a, r, z, s);
        return mg_apply_ns<NS_TABLE, 1>(h, a, r, z, s);
    }
    if (cg_staged(h)) return mg_apply_ns<NS_REL, kCgTileV>(h, a, r, z, s);
    if (use_relative(h)) return mg_apply_ns<NS_REL, 1>(h, a, r, z, s);
    if (use_offsets(h)) return mg_apply_ns<NS_OFF, 1>(h, a, r, z, s);
    return mg_apply_ns<NS_TABLE, 1>(h, a, r, z, s);
}

int run_cg(vg_sim *h, int pool, double a, double rtol, int max_iter, int *iters, double *relres,
           hipStream_t s) {
    if (h->n == 0) {
        if (iters) *iters = 0;
        if (relres) *relres = 0.0;
        return VG_OK;
    }
    if (h->prec == VG_F32C) return cg_solve<CompAcc>(h, pool, a, rtol, max_iter, iters, relres, s);
    if (h->prec == VG_F64) return cg_solve<PlainAcc<double>>(h, pool, a, rtol, max_iter, iters, relres, s);
    return cg_solve<PlainAcc<float>>(h, pool, a, rtol, max_iter, iters, relres, s);
}

}  // namespace vg
