// Explicit time stepping: the per-voxel transformation (Sec. II.C eq. (3) with
// the clamps of Appendix A, Algorithm 1) and explicit diffusion on the voxel
// graph (Sec. II.B.3a, Scheme 1), fused into one bandwidth-bound pass over
// the compacted pore list, plus the FP64 mass totals.
//
// One pass reads each pool of a voxel once, gathers the mobile pools of its
// six neighbours (mostly cache hits: +-x are adjacent entries, +-y and +-z lie
// one row / one plane away in the enumeration), and writes each pool once.
// Immobile pools are updated in place; mobile pools ping-pong between the
// caller's field buffer and its alt buffer because neighbours read them.
//
// Two ways to find the neighbours of compact voxel i:
//   table  the 6-slot int32 table nbr[6][n] (24 B per voxel and pass);
//   rank   a 32-bit geometry word per voxel (packed coordinates, and in raster
//          order the -x / +x neighbours, which are i - 1 / i + 1) plus the rank
//          index of the enumeration: a neighbour's compact index is the rank of
//          its position (pore-bitmap word + popcount; the words are cache
//          hits), so a pass moves ~46 B per voxel instead of 64 B.  Single
//          volume, no periodic axis, every dimension <= 1024.
//   offset two 32-bit words per voxel holding the distances i - j (minus side)
//          and j - i (plus side) to its neighbours in the enumeration, packed
//          by axis (48 B per voxel and pass, and the neighbour loads depend on
//          one load only).  Any volume or batch without periodic wrap whose
//          largest distances fit the packing.
//   relative  one 32-bit word per voxel of per-slot codes relative to base
//          distances shared by each group of 64 voxels (one wave): 44.5 B per
//          voxel and pass.  The default where it fits.
//
// The band kernel (k_band2, below) applies two fused passes per launch to
// bands of rows marching along z, keeping the first pass's DOM in LDS, for a
// single raster volume with relative codes.
//
// The paper's step is T then D.  The pass computes K = T o D (diffuse, then
// transform), so n paper steps run as T, K^(n-1), D.  Inside a K pass the
// state between its D and T halves is exactly the paper state after a full
// step, which is where the totals of that step are taken.
#include <algorithm>

#include "vg_internal.h"

#pragma clang fp contract(off)

namespace vg {
namespace {

// Transformation of one voxel, Appendix A Algorithm 2 (sequential): uptake,
// mortality, respiration, SOM and FOM turnover update the masses one after
// the other, each from what the previous left; a process that would take
// more than its source holds takes all of it.  The printed algorithm's slips
// are read as corrected (each turnover against its own pool, the pool moved
// to DOM before it is zeroed, MB zeroed when it all dies).
template <typename R>
__device__ __forceinline__ void transform_seq(const Coef<R> &C, R &m1, R &m2, R &m3, R &m4, R &m5) {
    if (m1 > R(0)) {
        if (m2 > R(0)) {
            const R uptake = C.v_dom * m2 / (C.k_dom + m2) * m1 * C.dt;
            if (uptake < m2) {
                m1 = m1 + uptake;
                m2 = m2 - uptake;
            } else {
                m1 = m1 + m2;
                m2 = R(0);
            }
        }
        const R morta = C.mu * m1 * C.dt;
        const R dead = morta < m1 ? morta : m1;
        m1 = morta < m1 ? m1 - morta : R(0);
        if (C.route == 0) {
            m2 = m2 + C.beta * dead;
            m3 = m3 + C.omb * dead;
        } else {
            m4 = m4 + dead;
        }
        const R resp = C.rho * m1 * C.dt;
        if (resp < m1) {
            m1 = m1 - resp;
            m5 = m5 + resp;
        } else {
            m5 = m5 + m1;
            m1 = R(0);
        }
    }
    if (m3 > R(0)) {
        const R turn = C.v_som * m3 * C.dt;
        if (turn < m3) {
            m3 = m3 - turn;
            m2 = m2 + turn;
        } else {
            m2 = m2 + m3;
            m3 = R(0);
        }
    }
    if (m4 > R(0)) {
        const R turn = C.v_p4 * m4 * C.dt;
        if (turn < m4) {
            m4 = m4 - turn;
            m2 = m2 + turn;
        } else {
            m2 = m2 + m4;
            m4 = R(0);
        }
    }
}

// Transformation of one voxel, Appendix A Algorithm 1: fluxes from the
// pre-step masses, each clamped to what its source pool holds, then applied.
template <typename R>
__device__ __forceinline__ void transform_flux(const Coef<R> &C, R &m1, R &m2, R &m3, R &m4, R &m5) {
    R uptake = C.v_dom * m2 / (C.k_dom + m2) * m1 * C.dt;
    if (uptake > m2) uptake = m2;
    R resp = C.rho * m1 * C.dt;
    R morta = C.mu * m1 * C.dt;
    if (resp + morta > m1) {
        if (morta > m1) {
            morta = m1;
            resp = R(0);
        } else {
            resp = m1 - morta;
        }
    }
    R turn_p4 = C.v_p4 * m4 * C.dt;
    if (turn_p4 > m4) turn_p4 = m4;
    R turn_som = C.v_som * m3 * C.dt;
    if (turn_som > m3) turn_som = m3;
    const R n1 = m1 + (uptake - morta - resp);
    R n2, n3, n4;
    if (C.route == 0) {
        const R to_som = C.omb * morta;
        const R to_dom = C.beta * morta;
        n2 = m2 + (to_dom - uptake + turn_p4 + turn_som);
        n3 = m3 + (to_som - turn_som);
        n4 = m4 - turn_p4;
    } else {
        n2 = m2 + (R(0) - uptake + turn_p4 + turn_som);
        n3 = m3 + (R(0) - turn_som);
        n4 = m4 + (morta - turn_p4);
    }
    m1 = n1;
    m2 = n2;
    m3 = n3;
    m4 = n4;
    m5 = m5 + resp;
}

// The algorithm chosen at compile time (the hot pass) or by C.seq.
template <bool SEQ, typename R>
__device__ __forceinline__ void transform_alg(const Coef<R> &C, R &m1, R &m2, R &m3, R &m4, R &m5) {
    if constexpr (SEQ) transform_seq(C, m1, m2, m3, m4, m5);
    else transform_flux(C, m1, m2, m3, m4, m5);
}

template <typename R>
__device__ __forceinline__ void transform(const Coef<R> &C, R &m1, R &m2, R &m3, R &m4, R &m5) {
    if (C.seq) transform_seq(C, m1, m2, m3, m4, m5);
    else transform_flux(C, m1, m2, m3, m4, m5);
}

template <typename R>
struct StepBufs {
    const int32_t *nbr = nullptr;       // [6][n]
    const uint16_t *rcode = nullptr;    // [n] or null
    PackedNbr pk;                       // packed neighbour sources (when built)
    const R *src[VG_NPOOL] = {};
    R *dst[VG_NPOOL] = {};
    // when set (a recording pass of the adjoint that keeps the diffused
    // DOM): a fused pass also writes each voxel's DOM after the diffusion
    // half, before the transformation, here
    R *xdom = nullptr;
    int64_t n = 0;
};

// The graph-side members of a pass's buffers, all taken from the handle (the
// pool pointers are the caller's).
template <typename R>
StepBufs<R> graph_bufs(const vg_sim *h) {
    StepBufs<R> B;
    B.nbr = h->nbr;
    B.rcode = h->rcode;
    B.pk = packed_of(h);
    B.n = h->n;
    return B;
}


// Loads and stores of data used once per pass (the neighbour table, the
// immobile pools); plain accesses (nontemporal ones measured no faster).
template <typename T>
__device__ __forceinline__ T ld_once(const T *p) {
    return *p;
}
template <typename T>
__device__ __forceinline__ void st_once(T *p, T v) {
    *p = v;
}

// MOB: 1 = only DOM diffuses, 2 = every pool diffuses (a_s may be 0).
template <int MOB>
__device__ __forceinline__ constexpr bool mobile(int s) {
    return MOB == 2 || (MOB == 1 && s == 1);
}

template <int MODE, int MOB, int TOT>
__device__ __forceinline__ constexpr bool reads(int s) {
    // a diffusion-only pass reads the immobile pools only to total them
    return MODE != MODE_D || mobile<MOB>(s) || TOT != TOT_NONE;
}

// Scheme 1 for the mobile pools of one voxel: x_s += a_s * sum_k w_k (x_s,j - x_s,i),
// slot terms added as ((d0+d1)+(d2+d3))+(d4+d5).
template <typename R, int MOB, bool REG>
__device__ __forceinline__ void diffuse_voxel(const StepBufs<R> &B, const Coef<R> &C, int64_t i, const int32_t (&j)[6],
                                              const R (&w)[6], R (&x)[VG_NPOOL]) {
#pragma unroll
    for (int s = 0; s < VG_NPOOL; s++) {
        if (!mobile<MOB>(s)) continue;
        const R xi = x[s];
        // all six loads are issued before any is used (an absent neighbour
        // reads the voxel itself and contributes 0), so their latencies overlap
        R v[6];
#pragma unroll
        for (int k = 0; k < 6; k++) v[k] = B.src[s][j[k] >= 0 ? (int64_t)j[k] : i];
        R d[6];
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const R diff = v[k] - xi;
            d[k] = j[k] >= 0 ? (REG ? w[k] * diff : diff) : R(0);
        }
        const R sum = ((d[0] + d[1]) + (d[2] + d[3])) + (d[4] + d[5]);
        x[s] = xi + C.a[s] * sum;
    }
}

// A thread handles kVPT voxels of its tile.  The work is split into phases
// over all of them (indices, own loads, neighbour loads, arithmetic and
// stores) so that every load of the thread is in flight before the first
// result is needed; no store precedes a load of the same thread.

// own pools of every voxel of the thread (inactive lanes read a valid index)
template <typename R, int MODE, int MOB, int TOT>
__device__ __forceinline__ void load_own(const StepBufs<R> &B, const int64_t (&ic)[kVPT], R (&x)[kVPT][VG_NPOOL]) {
#pragma unroll
    for (int v = 0; v < kVPT; v++)
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++)
            x[v][s] = reads<MODE, MOB, TOT>(s) ? (mobile<MOB>(s) ? B.src[s][ic[v]] : ld_once(&B.src[s][ic[v]])) : R(0);
}

// Scheme 1 for DOM only, all gathers first: x_1 += a_1 * sum_k w_k (x_1,j - x_1,i).
template <typename R, bool REG>
__device__ __forceinline__ void diffuse_dom(const StepBufs<R> &B, const Coef<R> &C, const int64_t (&ic)[kVPT],
                                            const int32_t (&j)[kVPT][6], const R (&w)[kVPT][6],
                                            R (&x)[kVPT][VG_NPOOL]) {
    R g[kVPT][6];
#pragma unroll
    for (int v = 0; v < kVPT; v++)
#pragma unroll
        for (int k = 0; k < 6; k++) g[v][k] = B.src[1][j[v][k] >= 0 ? (int64_t)j[v][k] : ic[v]];
#pragma unroll
    for (int v = 0; v < kVPT; v++) {
        const R xi = x[v][1];
        R d[6];
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const R diff = g[v][k] - xi;
            d[k] = j[v][k] >= 0 ? (REG ? w[v][k] * diff : diff) : R(0);
        }
        const R sum = ((d[0] + d[1]) + (d[2] + d[3])) + (d[4] + d[5]);
        x[v][1] = xi + C.a[1] * sum;
    }
}

// After the neighbours are known: diffuse, total, transform, store.
template <typename R, int MODE, int MOB, bool REG, int TOT>
__device__ __forceinline__ void finish(const StepBufs<R> &B, const Coef<R> &C, const int64_t (&ic)[kVPT],
                                       const bool (&act)[kVPT], const int32_t (&j)[kVPT][6], const R (&w)[kVPT][6],
                                       R (&x)[kVPT][VG_NPOOL], double (&acc)[kVPT][VG_NPOOL]) {
    constexpr bool do_d = MODE == MODE_D || MODE == MODE_DT;
    constexpr bool do_t = MODE == MODE_T || MODE == MODE_DT;
#pragma unroll
    for (int v = 0; v < kVPT; v++)
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) acc[v][s] = (TOT == TOT_IN && act[v]) ? (double)x[v][s] : 0.0;
    if (do_d) {
        if (MOB == 1) {
            diffuse_dom<R, REG>(B, C, ic, j, w, x);
        } else {
#pragma unroll
            for (int v = 0; v < kVPT; v++) diffuse_voxel<R, MOB, REG>(B, C, ic[v], j[v], w[v], x[v]);
        }
    }
    if (MODE == MODE_DT && MOB == 1 && B.xdom) {
#pragma unroll
        for (int v = 0; v < kVPT; v++)
            if (act[v]) B.xdom[ic[v]] = x[v][1];
    }
#pragma unroll
    for (int v = 0; v < kVPT; v++) {
        if (TOT == TOT_MID && act[v]) {
#pragma unroll
            for (int s = 0; s < VG_NPOOL; s++) acc[v][s] = (double)x[v][s];
        }
        if (do_t) transform(C, x[v][0], x[v][1], x[v][2], x[v][3], x[v][4]);
        if (TOT == TOT_OUT && act[v]) {
#pragma unroll
            for (int s = 0; s < VG_NPOOL; s++) acc[v][s] = (double)x[v][s];
        }
    }
    if (MODE != MODE_NONE) {
#pragma unroll
        for (int v = 0; v < kVPT; v++) {
            if (!act[v]) continue;
#pragma unroll
            for (int s = 0; s < VG_NPOOL; s++) {
                if (mobile<MOB>(s)) B.dst[s][ic[v]] = x[v][s];
                else if (MODE != MODE_D) st_once(&B.dst[s][ic[v]], x[v][s]);
            }
        }
    }
}

// Per-piece sums of the thread's accumulators (a piece is the part of a tile
// inside one segment), written to part[piece][pool] in a fixed order; `lds`
// holds kQuads * 5 doubles.
__device__ __forceinline__ void tile_totals(const Pieces &pc, int64_t tile, const double (&acc)[kVPT][VG_NPOOL],
                                            double *__restrict__ part, double *lds) {
    const int32_t p0 = pc.piece_first[tile], p1 = pc.piece_first[tile + 1];
    for (int32_t p = p0; p < p1; p++) {
        const int64_t lo = pc.piece_lo[p], hi = pc.piece_lo[p + 1];
        double v5[VG_NPOOL] = {0, 0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < kVPT; v++) {
            const int64_t i = tile * kTile + v * kBlock + threadIdx.x;
            const bool in = i >= lo && i < hi;
#pragma unroll
            for (int s = 0; s < VG_NPOOL; s++) v5[s] += in ? acc[v][s] : 0.0;
        }
        tile_sum_to<VG_NPOOL>(v5, lds, part + (int64_t)p * VG_NPOOL);
    }
}

template <typename R, int MODE, int MOB, bool REG, int TOT>
__global__ __launch_bounds__(kBlock) void k_step(StepBufs<R> B, Coef<R> C, Pieces pc, double *__restrict__ part) {
    __shared__ double lds[kQuads * VG_NPOOL];
    __shared__ R cl[VG_NREG];
    constexpr bool do_d = MODE == MODE_D || MODE == MODE_DT;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    if (REG) {
        if (threadIdx.x < VG_NREG) cl[threadIdx.x] = C.c[threadIdx.x];
        __syncthreads();
    }
    int64_t ic[kVPT];
    bool act[kVPT];
#pragma unroll
    for (int v = 0; v < kVPT; v++) {
        const int64_t i = tile * kTile + v * kBlock + threadIdx.x;
        act[v] = i < B.n;
        ic[v] = act[v] ? i : B.n - 1;
    }
    int32_t j[kVPT][6];
    R w[kVPT][6];
    if (do_d) {
#pragma unroll
        for (int v = 0; v < kVPT; v++) {
#pragma unroll
            for (int k = 0; k < 6; k++) j[v][k] = ld_once(&B.nbr[(int64_t)k * B.n + ic[v]]);
            if (REG) {
                region_weights<R>(cl, B.rcode[ic[v]], w[v]);
            }
        }
    }
    R x[kVPT][VG_NPOOL];
    load_own<R, MODE, MOB, TOT>(B, ic, x);
    double acc[kVPT][VG_NPOOL];
    finish<R, MODE, MOB, REG, TOT>(B, C, ic, act, j, w, x, acc);
    if (TOT != TOT_NONE) tile_totals(pc, tile, acc, part, lds);
}

// Packed-offset variant of the diffusing passes (D and DT).  Neighbour j of
// voxel i is i - d or i + d with d unpacked from the voxel's two offset words;
// an absent neighbour has d = 0 and so reads the voxel itself, whose
// difference x_i - x_i is exactly +0 (the absent slot's zero) for finite
// values, so no selects are needed.  All indices are 32-bit.
template <typename R, int MODE, int MOB, bool REG, int TOT, bool RELC, bool SEQ, int V = kVPT>
__global__ __launch_bounds__(kBlock) void k_step_off(StepBufs<R> B, Coef<R> C, Pieces pc, double *__restrict__ part) {
    static_assert(MODE == MODE_D || MODE == MODE_DT, "diffusing passes only");
    __shared__ double lds[kQuads * VG_NPOOL];
    __shared__ R cl[VG_NREG];
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t n = (uint32_t)B.n;
    if (REG) {
        if (threadIdx.x < VG_NREG) cl[threadIdx.x] = C.c[threadIdx.x];
        __syncthreads();
    }
    uint32_t ic[V];
    bool act[V];
#pragma unroll
    for (int v = 0; v < V; v++) {
        const uint32_t i = (uint32_t)tile * (uint32_t)(kBlock * V) + (uint32_t)(v * kBlock) + threadIdx.x;
        act[v] = i < n;
        ic[v] = act[v] ? i : n - 1;
    }
    // the neighbour words first (the gathers depend on them), then the pools
    PackedWords pw[V];
#pragma unroll
    for (int v = 0; v < V; v++) pw[v] = packed_words<RELC>(B.pk, ic[v]);
    R x[V][VG_NPOOL];
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++)
            x[v][s] = reads<MODE, MOB, TOT>(s) ? (mobile<MOB>(s) ? at(B.src[s], ic[v]) : ld_once(&at(B.src[s], ic[v])))
                                               : R(0);
    uint32_t j[V][6], pres[V];
#pragma unroll
    for (int v = 0; v < V; v++) pres[v] = packed_decode_near<RELC>(B.pk, ic[v], n, pw[v], j[v]);   // lanes past n hold n - 1
    R w[V][6];
#pragma unroll
    for (int v = 0; v < V; v++) {
        if (REG) {
            region_weights<R>(cl, at(B.rcode, ic[v]), w[v]);
        }
    }
    double acc[V][VG_NPOOL];
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) acc[v][s] = (TOT == TOT_IN && act[v]) ? (double)x[v][s] : 0.0;
    // Scheme 1: every gather of the thread first, then the sums
    constexpr int NM = MOB == 2 ? VG_NPOOL : 1;
    R g[V][NM][6];
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
        for (int m = 0; m < NM; m++)
#pragma unroll
            for (int k = 0; k < 6; k++) g[v][m][k] = at(B.src[NM == 1 ? 1 : m], j[v][k]);
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
        for (int m = 0; m < NM; m++) {
            const int s = NM == 1 ? 1 : m;
            const R xi = x[v][s];
            R d[6];
#pragma unroll
            for (int k = 0; k < 6; k++) {
                const R gk = ((pres[v] >> k) & 1u) ? g[v][m][k] : xi;
                d[k] = REG ? w[v][k] * (gk - xi) : gk - xi;
            }
            const R sum = ((d[0] + d[1]) + (d[2] + d[3])) + (d[4] + d[5]);
            x[v][s] = xi + C.a[s] * sum;
        }
    if (MODE == MODE_DT && MOB == 1 && B.xdom) {
#pragma unroll
        for (int v = 0; v < V; v++)
            if (act[v]) at(B.xdom, ic[v]) = x[v][1];
    }
#pragma unroll
    for (int v = 0; v < V; v++) {
        if (TOT == TOT_MID && act[v]) {
#pragma unroll
            for (int s = 0; s < VG_NPOOL; s++) acc[v][s] = (double)x[v][s];
        }
        if (MODE == MODE_DT) transform_alg<SEQ>(C, x[v][0], x[v][1], x[v][2], x[v][3], x[v][4]);
        if (TOT == TOT_OUT && act[v]) {
#pragma unroll
            for (int s = 0; s < VG_NPOOL; s++) acc[v][s] = (double)x[v][s];
        }
    }
#pragma unroll
    for (int v = 0; v < V; v++) {
        if (!act[v]) continue;
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) {
            if (mobile<MOB>(s)) at(B.dst[s], ic[v]) = x[v][s];
            else if (MODE != MODE_D) st_once(&at(B.dst[s], ic[v]), x[v][s]);
        }
    }
    if constexpr (TOT != TOT_NONE) {
        // totals per reduction tile of kTile voxels: the thread's voxel v
        // lies in tile tile * V + v (uniform over the block)
        static_assert(kVPT == 1, "one voxel per thread and reduction tile");
#pragma unroll
        for (int v = 0; v < V; v++) {
            const int64_t tv = tile * V + v;
            if (tv * kTile < (int64_t)n) tile_totals(pc, tv, reinterpret_cast<const double(&)[1][VG_NPOOL]>(acc[v]), part, lds);
        }
    }
}

// Compensated float32 fields (VG_F32C): every pool is a float hi and an
// int16 compensation word lo (6 B per value, a 39-bit significand, see
// comp_get / comp_put).  The pass decodes to FP64, diffuses and transforms in
// FP64 with the operations of the FP64 pass in the same order, and rounds
// each value once on the way out.  Neighbours come from the table or a packed
// source, chosen at run time (uniform branch); region weights and the
// algorithm likewise.
struct CompBufs {
    const int32_t *nbr = nullptr;       // [6][n]
    const uint16_t *rcode = nullptr;    // [n] or null
    PackedNbr pk;
    int ns = 0;                         // 0 table, 1 relative codes, 2 packed offsets
    const float *src[VG_NPOOL] = {};
    const int16_t *slo[VG_NPOOL] = {};
    float *dst[VG_NPOOL] = {};
    int16_t *dlo[VG_NPOOL] = {};
    int64_t n = 0;
    TileRange tr;                       // the tiles the pass covers (t1 = 0: all)
};

__device__ __forceinline__ double comp_at(const float *hi, const int16_t *lo, uint32_t i) {
    return comp_get(at(hi, i), at(lo, i));
}

// SLAB: the pass covers the tiles B.tr (see the slabs of vg_api.cpp).
template <int MODE, int MOB, int TOT, bool SLAB>
__global__ __launch_bounds__(kBlock) void k_step_c(CompBufs B, Coef<double> C, Pieces pc,
                                                   double *__restrict__ part) {
    __shared__ double lds[kQuads * VG_NPOOL];
    __shared__ double cl[VG_NREG];
    constexpr bool do_d = MODE == MODE_D || MODE == MODE_DT;
    constexpr bool do_t = MODE == MODE_T || MODE == MODE_DT;
    const int64_t tile = SLAB ? B.tr.t0 + xcd_tile_run(blockIdx.x, gridDim.x, B.tr.run)
                              : xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t n = (uint32_t)B.n;
    const bool reg = B.rcode != nullptr;
    if (reg) {   // uniform over the block
        if (threadIdx.x < VG_NREG) cl[threadIdx.x] = C.c[threadIdx.x];
        __syncthreads();
    }
    const uint32_t i0 = (uint32_t)tile * (uint32_t)kBlock + threadIdx.x;
    const bool act = i0 < n;
    const uint32_t i = act ? i0 : n - 1;
    // neighbours: an absent one is the voxel itself (its difference is +0)
    uint32_t j[6];
    bool pres[6];
    if (do_d) {
        if (B.ns == 0) {
#pragma unroll
            for (int k = 0; k < 6; k++) {
                const int32_t jk = B.nbr[(int64_t)k * B.n + i];
                pres[k] = jk >= 0;
                j[k] = pres[k] ? (uint32_t)jk : i;
            }
        } else {
            const bool relc = B.ns == 1;
            const PackedWords W = relc ? packed_words<true>(B.pk, i) : packed_words<false>(B.pk, i);
            if (relc) packed_decode<true>(B.pk, i, W, j);
            else packed_decode<false>(B.pk, i, W, j);
#pragma unroll
            for (int k = 0; k < 6; k++) pres[k] = j[k] != i;   // no periodic wrap in packed sources
        }
    }
    double x[VG_NPOOL];
#pragma unroll
    for (int s = 0; s < VG_NPOOL; s++)
        x[s] = reads<MODE, MOB, TOT>(s) ? comp_at(B.src[s], B.slo[s], i) : 0.0;
    double acc[1][VG_NPOOL];
#pragma unroll
    for (int s = 0; s < VG_NPOOL; s++) acc[0][s] = (TOT == TOT_IN && act) ? x[s] : 0.0;
    if (do_d) {
        double w[6] = {1.0, 1.0, 1.0, 1.0, 1.0, 1.0};
        if (reg) {
            region_weights<double>(cl, at(B.rcode, i), w);
        }
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) {
            if (!mobile<MOB>(s)) continue;
            const double xi = x[s];
            double v[6];
#pragma unroll
            for (int k = 0; k < 6; k++) v[k] = comp_at(B.src[s], B.slo[s], j[k]);
            double d[6];
#pragma unroll
            for (int k = 0; k < 6; k++) d[k] = pres[k] ? (reg ? w[k] * (v[k] - xi) : v[k] - xi) : 0.0;
            const double sum = ((d[0] + d[1]) + (d[2] + d[3])) + (d[4] + d[5]);
            x[s] = xi + C.a[s] * sum;
        }
    }
    if (TOT == TOT_MID && act) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) acc[0][s] = x[s];
    }
    if (do_t) transform(C, x[0], x[1], x[2], x[3], x[4]);
    if (TOT == TOT_OUT && act) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) acc[0][s] = x[s];
    }
    if (MODE != MODE_NONE && act) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) {
            if (mobile<MOB>(s) || MODE != MODE_D) {
                float hi;
                int16_t lo;
                comp_put(x[s], hi, lo);
                at(B.dst[s], i) = hi;
                at(B.dlo[s], i) = lo;
            }
        }
    }
    if constexpr (TOT != TOT_NONE) tile_totals(pc, tile, acc, part, lds);
}

// Rank-index variant (single volume: one piece per tile).  Each voxel has a
// 32-bit geometry word (x | y << 10 | z << 20, and in raster order whether
// its -x / +x neighbours are pore in bits 30 / 31: their compact indices are
// then i - 1 / i + 1).  The other neighbours' compact indices are ranks of
// their positions: one pore-bitmap word (8 B, a cache hit) and a popcount.
// Per voxel and pass this reads 4 B of geometry instead of 24 B of table.
// Neighbours of one thread's voxels from their geometry words (rank index).
template <typename R, bool REG, bool RASTER>
__device__ __forceinline__ void geo_neighbours(const RGeom &G, const R *cl, const int64_t (&ic)[kVPT],
                                               const uint32_t (&gw)[kVPT], int32_t (&j)[kVPT][6],
                                               R (&w)[kVPT][6]) {
    constexpr int NW = RASTER ? 4 : 6;        // neighbours found through the bitmap
    const uint32_t nx = G.fnx.d, plane = G.fnx.d * G.fny.d;
    uint32_t pq[kVPT][NW];
    bool ok[kVPT][NW];
#pragma unroll
    for (int v = 0; v < kVPT; v++) {
        const uint32_t c = gw[v];
        const int xx = (int)(c & 1023u), yy = (int)((c >> 10) & 1023u), zz = (int)((c >> 20) & 1023u);
        if (RASTER) {
            const uint32_t p = (uint32_t)xx + nx * ((uint32_t)yy + G.fny.d * (uint32_t)zz);
            j[v][0] = ((c >> 30) & 1u) ? (int32_t)ic[v] - 1 : -1;
            j[v][1] = (c >> 31) ? (int32_t)ic[v] + 1 : -1;
            ok[v][0] = yy > 0;
            ok[v][1] = yy + 1 < G.g.ny;
            ok[v][2] = zz > 0;
            ok[v][3] = zz + 1 < G.g.nz;
            pq[v][0] = ok[v][0] ? p - nx : p;
            pq[v][1] = ok[v][1] ? p + nx : p;
            pq[v][2] = ok[v][2] ? p - plane : p;
            pq[v][3] = ok[v][3] ? p + plane : p;
        } else {
            const int xyz[3] = {xx, yy, zz};
            const int dims[3] = {G.g.nx, G.g.ny, G.g.nz};
            const uint32_t p = rg_pos(G, xx, yy, zz);
#pragma unroll
            for (int k = 0; k < 6; k++) {
                const int axis = k >> 1;
                int q[3] = {xyz[0], xyz[1], xyz[2]};
                q[axis] += (k & 1) ? 1 : -1;
                ok[v][k % NW] = q[axis] >= 0 && q[axis] < dims[axis];
                pq[v][k % NW] = ok[v][k % NW] ? rg_pos(G, q[0], q[1], q[2]) : p;
            }
        }
        if (REG) {
            const int hx = G.g.nx / 2, hy = G.g.ny / 2, hz = G.g.nz / 2;
            const int oct = 4 * (zz >= hz) + 2 * (yy >= hy) + (xx >= hx);
            const int nb[6] = {oct ^ ((xx - 1 >= hx) != (xx >= hx)), oct ^ ((xx + 1 >= hx) != (xx >= hx)),
                               oct ^ (2 * ((yy - 1 >= hy) != (yy >= hy))), oct ^ (2 * ((yy + 1 >= hy) != (yy >= hy))),
                               oct ^ (4 * ((zz - 1 >= hz) != (zz >= hz))), oct ^ (4 * ((zz + 1 >= hz) != (zz >= hz)))};
#pragma unroll
            for (int k = 0; k < 6; k++) w[v][k] = R(0.5) * (cl[oct] + cl[nb[k]]);
        }
    }
    // all bitmap words of the thread are loaded before any is used
    uint32_t wb[kVPT][NW], wbefore[kVPT][NW];
#pragma unroll
    for (int v = 0; v < kVPT; v++)
#pragma unroll
        for (int k = 0; k < NW; k++) {
            const RankWord t = G.rank[pq[v][k] >> 5];
            wb[v][k] = t.bits;
            wbefore[v][k] = t.before;
        }
#pragma unroll
    for (int v = 0; v < kVPT; v++)
#pragma unroll
        for (int k = 0; k < NW; k++) {
            const uint32_t bit = pq[v][k] & 31u;
            const bool pore = ok[v][k] && ((wb[v][k] >> bit) & 1u);
            j[v][k + 6 - NW] = pore ? (int32_t)(wbefore[v][k] + (uint32_t)__popc(wb[v][k] & ((1u << bit) - 1u))) : -1;
        }
}

// Rank-index variant (single volume, one tile per block).  Each voxel has a
// 32-bit geometry word (x | y << 10 | z << 20, and in raster order whether its
// -x / +x neighbours are pore in bits 30 / 31: their compact indices are then
// i - 1 / i + 1).  The other neighbours' compact indices are ranks of their
// positions: one pore-bitmap word (8 B, a cache hit) and a popcount.  Per
// voxel and pass this reads 4 B of geometry instead of 24 B of table.
// (A persistent, software-pipelined form of this kernel measured slower.)
template <typename R, int MODE, int MOB, bool REG, int TOT, bool RASTER>
__global__ __launch_bounds__(kBlock) void k_step_geo(StepBufs<R> B, Coef<R> C, RGeom G,
                                                     const uint32_t *__restrict__ geo, double *__restrict__ part) {
    __shared__ double lds[kQuads * VG_NPOOL];
    __shared__ R cl[VG_NREG];
    constexpr bool do_d = MODE == MODE_D || MODE == MODE_DT;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t n = B.n;
    if (REG) {
        if (threadIdx.x < VG_NREG) cl[threadIdx.x] = C.c[threadIdx.x];
        __syncthreads();
    }
    int64_t ic[kVPT];
    bool act[kVPT];
#pragma unroll
    for (int v = 0; v < kVPT; v++) {
        const int64_t i = tile * kTile + v * kBlock + threadIdx.x;
        act[v] = i < n;
        ic[v] = act[v] ? i : n - 1;
    }
    uint32_t gw[kVPT];
    if (do_d) {
#pragma unroll
        for (int v = 0; v < kVPT; v++) gw[v] = ld_once(&geo[ic[v]]);
    }
    R x[kVPT][VG_NPOOL];
    load_own<R, MODE, MOB, TOT>(B, ic, x);
    int32_t j[kVPT][6];
    R w[kVPT][6];
    if (do_d) geo_neighbours<R, REG, RASTER>(G, cl, ic, gw, j, w);
    double acc[kVPT][VG_NPOOL];
    finish<R, MODE, MOB, REG, TOT>(B, C, ic, act, j, w, x, acc);
    if (TOT != TOT_NONE) {
        double a5[VG_NPOOL] = {0, 0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < kVPT; v++)
#pragma unroll
            for (int s = 0; s < VG_NPOOL; s++) a5[s] += acc[v][s];
        tile_sum_to<VG_NPOOL>(a5, lds, part + tile * VG_NPOOL);
    }
}

// Geometry words of the rank-index kernel, from the compacted list.
__global__ __launch_bounds__(kBlock) void k_geometry(const int32_t *__restrict__ vox, int64_t n, RGeom G,
                                                     uint32_t *__restrict__ geo) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const uint32_t v = (uint32_t)vox[i];
    const uint32_t q1 = G.fnx.div(v);
    const uint32_t z = G.fny.div(q1);
    const uint32_t x = v - q1 * G.fnx.d, y = q1 - z * G.fny.d;
    uint32_t c = x | (y << 10) | (z << 20);
    if (G.g.b <= 0) {
        // raster: the -x / +x neighbours, when pore, are compact voxels i -/+ 1
        if (x > 0) {
            const RankWord wd = G.rank[(v - 1) >> 5];
            if ((wd.bits >> ((v - 1) & 31u)) & 1u) c |= 1u << 30;
        }
        if (x + 1 < G.fnx.d) {
            const RankWord wd = G.rank[(v + 1) >> 5];
            if ((wd.bits >> ((v + 1) & 31u)) & 1u) c |= 1u << 31;
        }
    }
    geo[i] = c;
}

// Packed offsets, pass 2: the two words of every voxel.
__global__ __launch_bounds__(kBlock) void k_offsets(const int32_t *__restrict__ nbr, int64_t n, DLayout L,
                                                    uint32_t *__restrict__ off_m, uint32_t *__restrict__ off_p) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const uint32_t shift[3] = {L.sx, L.bz, 0};
    uint32_t wm = 0, wp = 0;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const int32_t j = nbr[(int64_t)k * n + i];
        if (j < 0) continue;
        const uint32_t d = (k & 1) ? (uint32_t)((int64_t)j - i) : (uint32_t)(i - (int64_t)j);
        if (k & 1) wp |= d << shift[k >> 1];
        else wm |= d << shift[k >> 1];
    }
    off_m[i] = wm;
    off_p[i] = wp;
}

// Neighbour distances, one pass over the table (both packings): per group of
// 64 voxels (one wave) and slot the smallest distance, base[g][k]; over the
// graph the largest distance per axis (stat[0..2]), a flag when a minus-side
// neighbour does not precede the voxel or a plus-side one does not follow it
// (stat[3], as across a periodic wrap) and the largest spread + 1 of a slot's
// distances within a group, per axis (stat[4..6]).  A bounded grid strides
// over the voxels and each block adds its maxima with one atomic per value.
__global__ __launch_bounds__(kBlock) void k_neighbour_stat(const int32_t *__restrict__ nbr, int64_t n,
                                                           uint32_t *__restrict__ base, uint32_t *__restrict__ stat) {
    static_assert(kGroup == 64, "a group is one wave");
    __shared__ uint32_t red[kWaves][7];
    uint32_t acc[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock; i0 < n; i0 += (int64_t)gridDim.x * kBlock) {
        const int64_t i = i0 + threadIdx.x;
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const int32_t j = i < n ? nbr[(int64_t)k * n + i] : -1;
            const int64_t d64 = (k & 1) ? (int64_t)j - i : i - (int64_t)j;
            if (j >= 0 && d64 <= 0) acc[3] = 1;
            const bool pres = j >= 0 && d64 > 0;
            const uint32_t d = pres ? (uint32_t)d64 : 0u;
            acc[k >> 1] = max(acc[k >> 1], d);
            uint32_t lo = pres ? d : 0xffffffffu, hi = d;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
                hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
            }
            if ((threadIdx.x & 63) == 0 && i < n) base[(i / kGroup) * 8 + k] = lo == 0xffffffffu ? 0u : lo;
            if (lo != 0xffffffffu) acc[4 + (k >> 1)] = max(acc[4 + (k >> 1)], hi - lo + 1u);
        }
    }
#pragma unroll
    for (int q = 0; q < 7; q++)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[q] = max(acc[q], (uint32_t)__shfl_xor((int)acc[q], o, 64));
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < 7; q++) red[threadIdx.x >> 6][q] = acc[q];
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        uint32_t v = red[0][threadIdx.x];
        for (int w = 1; w < kWaves; w++) v = max(v, red[w][threadIdx.x]);
        if (v) atomicMax(&stat[threadIdx.x], v);
    }
}

// Relative codes, pass 2: the code word of every voxel.
__global__ __launch_bounds__(kBlock) void k_rel_pack(const int32_t *__restrict__ nbr, int64_t n,
                                                     const uint32_t *__restrict__ base, RLayout L,
                                                     uint32_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const uint32_t *bp = base + (i / kGroup) * 8;
    uint32_t w = 0;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const int32_t j = nbr[(int64_t)k * n + i];
        if (j < 0) continue;
        const uint32_t d = (uint32_t)((k & 1) ? (int64_t)j - i : i - (int64_t)j);
        w |= (d - bp[k] + 1u) << L.sh[k];
    }
    out[i] = w;
}

// Totals, stage 1: chunks of up to kChunk pieces of one segment (blockIdx.y:
// the logged pass; part and chunk_part advance by their row strides).
__global__ __launch_bounds__(kBlock) void k_tot_chunks(const double *__restrict__ part,
                                                       const int32_t *__restrict__ chunk_first,
                                                       double *__restrict__ chunk_part, int64_t part_stride,
                                                       int64_t chunk_stride) {
    __shared__ double lds[kWaves * VG_NPOOL];
    const int c = blockIdx.x;
    part += blockIdx.y * part_stride;
    chunk_part += blockIdx.y * chunk_stride;
    const int32_t p = chunk_first[c] + (int32_t)threadIdx.x;
    double v[VG_NPOOL] = {0, 0, 0, 0, 0};
    if (p < chunk_first[c + 1]) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) v[s] = part[(int64_t)p * VG_NPOOL + s];
    }
    block_sum<VG_NPOOL>(v, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) chunk_part[(int64_t)c * VG_NPOOL + s] = v[s];
    }
}

// Totals, stage 2: one block per segment sums its chunks in a fixed order,
// then the five pool totals into total carbon.
__global__ __launch_bounds__(kBlock) void k_tot_segments(const double *__restrict__ chunk_part,
                                                         const int32_t *__restrict__ seg_chunk,
                                                         double *__restrict__ out, int64_t chunk_stride,
                                                         int64_t out_stride) {
    __shared__ double lds[kWaves * VG_NPOOL];
    const int g = blockIdx.x;
    chunk_part += blockIdx.y * chunk_stride;
    out += blockIdx.y * out_stride;
    double v[VG_NPOOL] = {0, 0, 0, 0, 0};
    for (int32_t c = seg_chunk[g] + (int32_t)threadIdx.x; c < seg_chunk[g + 1]; c += kBlock) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) v[s] += chunk_part[(int64_t)c * VG_NPOOL + s];
    }
    block_sum<VG_NPOOL>(v, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) out[g * 6 + s] = v[s];
        out[g * 6 + 5] = ((v[0] + v[1]) + (v[2] + v[3])) + v[4];
    }
}

// Totals in one stage, for segments of at most kDirectPieces pieces: one
// block per segment sums its pieces (thread t: pieces t, t + 256, ... in
// order, then the block in a fixed order), then the five pool totals into
// total carbon.
constexpr int32_t kDirectPieces = 4096;

__global__ __launch_bounds__(kBlock) void k_tot_direct(const double *__restrict__ part,
                                                       const int32_t *__restrict__ seg_first,
                                                       double *__restrict__ out, int64_t part_stride,
                                                       int64_t out_stride) {
    __shared__ double lds[kWaves * VG_NPOOL];
    const int g = blockIdx.x;
    part += blockIdx.y * part_stride;
    out += blockIdx.y * out_stride;
    double v[VG_NPOOL] = {0, 0, 0, 0, 0};
    for (int32_t p = seg_first[g] + (int32_t)threadIdx.x; p < seg_first[g + 1]; p += kBlock) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) v[s] += part[(int64_t)p * VG_NPOOL + s];
    }
    block_sum<VG_NPOOL>(v, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int s = 0; s < VG_NPOOL; s++) out[g * 6 + s] = v[s];
        out[g * 6 + 5] = ((v[0] + v[1]) + (v[2] + v[3])) + v[4];
    }
}

RGeom make_rgeom(const vg_sim *h) {
    RGeom G;
    make_geom(h->nx, h->ny, h->nz, h->brick, &G.g);
    G.fnx.init((uint32_t)h->nx);
    G.fny.init((uint32_t)h->ny);
    const uint32_t b = h->brick > 0 ? (uint32_t)h->brick : 1u;
    G.fb.init(b);
    G.fb2.init(b * b);
    G.fb3.init(b * b * b);
    G.fnbx.init(G.g.nbx > 0 ? (uint32_t)G.g.nbx : 1u);
    G.fnby.init(G.g.nby > 0 ? (uint32_t)G.g.nby : 1u);
    G.periodic = h->periodic;
    G.rank = (const RankWord *)h->rank;
    return G;
}

template <typename R, int MODE, int MOB, bool REG, int TOT>
int launch_one(vg_sim *h, const StepBufs<R> &B, const Coef<R> &C, hipStream_t s) {
    Pieces pc{h->piece_first, h->piece_lo, h->piece_seg, h->npieces};
    if constexpr (MODE == MODE_D || MODE == MODE_DT) {
        // the algorithm is a template argument of the packed-source pass
        // (Algorithm 2 instances only where a transformation runs)
        const bool seq = MODE == MODE_DT && C.seq;
        if constexpr (MODE == MODE_D) {
            // diffusion-only passes move 12.5 B per voxel (28.5 with totals):
            // two voxels per thread keep more loads in flight (measured 6.5 %
            // faster sub-cycled runs; the fused pass is faster with one)
            constexpr int V2 = 2;
            const unsigned grid = (unsigned)((h->n + kBlock * V2 - 1) / (kBlock * V2));
            if (use_relative(h)) {
                hipLaunchKernelGGL((k_step_off<R, MODE, MOB, REG, TOT, true, false, V2>), dim3(grid), dim3(kBlock),
                                   0, s, B, C, pc, part_of(h));
                return launch_status("k_step_off relative");
            }
            if (use_offsets(h)) {
                hipLaunchKernelGGL((k_step_off<R, MODE, MOB, REG, TOT, false, false, V2>), dim3(grid), dim3(kBlock),
                                   0, s, B, C, pc, part_of(h));
                return launch_status("k_step_off");
            }
        }
        if (use_relative(h)) {
            if (seq)
                hipLaunchKernelGGL((k_step_off<R, MODE, MOB, REG, TOT, true, MODE == MODE_DT>),
                                   dim3((unsigned)h->ntiles), dim3(kBlock), 0, s, B, C, pc, part_of(h));
            else
                hipLaunchKernelGGL((k_step_off<R, MODE, MOB, REG, TOT, true, false>), dim3((unsigned)h->ntiles),
                                   dim3(kBlock), 0, s, B, C, pc, part_of(h));
            return launch_status("k_step_off relative");
        }
        if (use_offsets(h)) {
            if (seq)
                hipLaunchKernelGGL((k_step_off<R, MODE, MOB, REG, TOT, false, MODE == MODE_DT>),
                                   dim3((unsigned)h->ntiles), dim3(kBlock), 0, s, B, C, pc, part_of(h));
            else
                hipLaunchKernelGGL((k_step_off<R, MODE, MOB, REG, TOT, false, false>), dim3((unsigned)h->ntiles),
                                   dim3(kBlock), 0, s, B, C, pc, part_of(h));
            return launch_status("k_step_off");
        }
    }
    if (use_rank(h) && MODE != MODE_NONE) {
        if (h->brick == 0)
            hipLaunchKernelGGL((k_step_geo<R, MODE, MOB, REG, TOT, true>), dim3((unsigned)h->ntiles), dim3(kBlock), 0,
                               s, B, C, make_rgeom(h), h->geo, part_of(h));
        else
            hipLaunchKernelGGL((k_step_geo<R, MODE, MOB, REG, TOT, false>), dim3((unsigned)h->ntiles), dim3(kBlock), 0,
                               s, B, C, make_rgeom(h), h->geo, part_of(h));
        return launch_status("k_step_geo");
    }
    hipLaunchKernelGGL((k_step<R, MODE, MOB, REG, TOT>), dim3((unsigned)h->ntiles), dim3(kBlock), 0, s, B,
                       C, pc, part_of(h));
    return launch_status("k_step");
}

template <typename R, int MODE, int MOB, bool REG>
int pick_tot(vg_sim *h, int tot, const StepBufs<R> &B, const Coef<R> &C, hipStream_t s) {
    switch (tot) {
        case TOT_NONE: return launch_one<R, MODE, MOB, REG, TOT_NONE>(h, B, C, s);
        case TOT_IN: return launch_one<R, MODE, MOB, REG, TOT_IN>(h, B, C, s);
        case TOT_MID: return launch_one<R, MODE, MOB, REG, TOT_MID>(h, B, C, s);
        default: return launch_one<R, MODE, MOB, REG, TOT_OUT>(h, B, C, s);
    }
}

template <typename R, int MODE, int MOB>
int pick_reg(vg_sim *h, int tot, const StepBufs<R> &B, const Coef<R> &C, hipStream_t s) {
    if (B.rcode) return pick_tot<R, MODE, MOB, true>(h, tot, B, C, s);
    return pick_tot<R, MODE, MOB, false>(h, tot, B, C, s);
}

template <typename R>
int dispatch_bufs(vg_sim *h, int mode, int tot, double dt_t, double dt_d, const StepBufs<R> &B, hipStream_t s) {
    const Coef<R> C = make_coef2<R>(h, dt_t, dt_d);
    const int mob = h->mobile_mode();
    if (mode == MODE_T) return pick_tot<R, MODE_T, 1, false>(h, tot, B, C, s);
    if (mode == MODE_NONE) return launch_one<R, MODE_NONE, 1, false, TOT_IN>(h, B, C, s);
    if (mode == MODE_D) return mob == 2 ? pick_reg<R, MODE_D, 2>(h, tot, B, C, s)
                                        : pick_reg<R, MODE_D, 1>(h, tot, B, C, s);
    return mob == 2 ? pick_reg<R, MODE_DT, 2>(h, tot, B, C, s) : pick_reg<R, MODE_DT, 1>(h, tot, B, C, s);
}

// ---------------------------------------------------------------- band kernel
// Two fused passes (x <- T(D(x)), twice) in one launch, for a single volume
// in raster order with relative neighbour codes, only DOM diffusing, unit
// weights and Algorithm 1.  Block (band, chunk) owns the rows
// [y0, y0 + H) of the planes [z0, z0 + Z) and marches along z.  At plane p
// it applies the first pass to the rows [y0 - 1, y0 + H] (the band and one
// neighbour row on each side: one contiguous range of the compact list) and
// the second pass to the band rows of plane p - 1.  LDS rings hold the DOM
// before the first pass (rows [y0 - 2, y0 + H + 1], four planes) and after
// it (four planes), so that every neighbour of both passes is an LDS read;
// what else the second pass needs of a voxel (the other pools after the
// first pass, its code) stays in the registers of the thread that computed
// it.  So every load of the kernel is a contiguous stream whose address only
// needs the row index: a plane's pools and codes are loaded while the plane
// before it is computed, its DOM two planes ahead, and one barrier per plane
// suffices.  Inputs and outputs are separate field sets, since neighbouring
// blocks read the inputs next to their rows and planes.  Same operations in
// the same order as two single passes, so the result is bit-identical.
// (A gather of 64 lanes costs the vector cache up to 26 accesses where a
// contiguous load costs 4, and a pass that gathers waits for the codes
// first; the kernel before this one gathered the first pass's neighbours,
// read the pools twice and took 388 us for a pass pair of 512^3 FP32, the
// single passes 2 x 200.)
struct BandGeom {
    int ny, nz, H, Z, nbands;   // H rows and Z planes per block
    uint32_t capf, cape;   // widest ranges of a plane: band and two / one neighbour rows on each side
};

// rs[r] = compact index of the first pore voxel at or after the start of
// row r = z * ny + y (vox ascending: the raster-order compact list).
__global__ __launch_bounds__(kBlock) void k_band_rows(const int32_t *__restrict__ vox, int64_t n, int nx,
                                                      int64_t nrows, int32_t *__restrict__ rs) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r > nrows) return;
    const int64_t target = r * nx;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)vox[mid] < target) lo = mid + 1;
        else hi = mid;
    }
    rs[r] = (int32_t)lo;
}

// Threads and slots per thread: a plane's range with one neighbour row on
// each side has at most kBandSlots voxels counted from the 64-voxel group it
// starts in.  (The rows' pore counts vary twofold, so the slots are sized by
// the widest plane and those past a plane's range are skipped.  Measured on
// the 512^3 FP32 and a 331x257x403 FP64 call: 768 x 3 threads x slots 2.89
// and 2.41 ms, 1024 x 2 3.69 and 2.41, 512 x 4 3.14 and 2.53; with the pools
// loaded after the first pass instead of a plane ahead 3.28 and 2.79.)
constexpr int kBandThreads = 768;
constexpr int kBandU = 3;
constexpr int kBandSlots = kBandThreads * kBandU;
constexpr int kBandRaw = kBandU + 1;                       // loads per thread of a plane's DOM
constexpr int kBandGroupWords = kBandSlots / kGroup * 8;   // base distances of a plane's groups

// The two field sets of a launch.
template <typename R>
struct BandBufs {
    const R *src[VG_NPOOL];
    R *dst[VG_NPOOL];
};

// LDS of a block: [4][capf] DOM before, [4][cape] after the first pass, [4]
// planes of base distances.
template <typename R>
size_t band_lds_bytes(int64_t capf, int64_t cape) {
    return (size_t)4 * (size_t)(capf + cape) * sizeof(R) + (size_t)4 * kBandGroupWords * sizeof(uint32_t);
}

// Compact ranges of a plane's rows: the band (b), with one (e) and two (f)
// neighbour rows on each side; empty outside the volume.
struct BandRange {
    uint32_t fs, fe, es, ee, bs, be;
};

template <typename R>
__global__ __launch_bounds__(kBandThreads) void k_band2(BandBufs<R> F, const uint32_t *__restrict__ rel_w,
                                                        const uint32_t *__restrict__ rel_base, RLayout L, Coef<R> C,
                                                        BandGeom G, const int32_t *__restrict__ rs) {
    extern __shared__ __align__(16) unsigned char band_lds[];
    R *raw = reinterpret_cast<R *>(band_lds);
    R *dom1 = raw + 4 * G.capf;
    uint32_t *bas = reinterpret_cast<uint32_t *>(dom1 + 4 * G.cape);
    constexpr int U = kBandU, NT = kBandThreads;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wb0 = __builtin_amdgcn_readfirstlane(tid & ~63u);   // the wave's first voxel of a slot
    const int blk = (int)xcd_split(blockIdx.x, gridDim.x);      // neighbouring bands on one XCD
    const int band = blk % G.nbands, chunk = blk / G.nbands;
    const int y0 = band * G.H, y1 = min(y0 + G.H, G.ny);
    const int ey0 = max(y0 - 1, 0), ey1 = min(y1 + 1, G.ny);
    const int fy0 = max(y0 - 2, 0), fy1 = min(y1 + 2, G.ny);
    const int z0 = chunk * G.Z, z1 = min(z0 + G.Z, G.nz);
    auto range = [&](int p) {
        BandRange r{0, 0, 0, 0, 0, 0};
        if (p >= 0 && p < G.nz) {
            const int32_t *row = rs + (int64_t)p * G.ny;
            r.fs = (uint32_t)row[fy0];
            r.fe = (uint32_t)row[fy1];
            r.es = (uint32_t)row[ey0];
            r.ee = (uint32_t)row[ey1];
            r.bs = (uint32_t)row[y0];
            r.be = (uint32_t)row[y1];
            if (r.es == r.ee) r.es = r.ee = r.bs = r.be = 0;   // no voxels: no slot is taken
        }
        return r;
    };
    // the DOM of a plane's f range: thread t's voxels fs + t, fs + NT + t, ...
    auto load_raw = [&](const BandRange &r, R (&v)[kBandRaw]) {
#pragma unroll
        for (int k = 0; k < kBandRaw; k++) {
            const uint32_t w0 = r.fs + wb0 + (uint32_t)(k * NT);
            if (w0 < r.fe) v[k] = at(F.src[1], min(w0 + lane, r.fe - 1u));   // uniform over the wave
        }
    };
    auto put_raw = [&](int p, const BandRange &r, const R (&v)[kBandRaw]) {
        R *d = raw + (uint32_t)(p & 3) * G.capf;
#pragma unroll
        for (int k = 0; k < kBandRaw; k++) {
            const uint32_t q0 = wb0 + (uint32_t)(k * NT), m = r.fe - r.fs;
            if (q0 < m) d[min(q0 + lane, m - 1u)] = v[k];   // (lanes past the end hold the last value)
        }
    };
    // base distances (less one) of the groups the e range touches, one word
    // per thread, the y and z slots' first (one 16-byte read)
    static_assert(kBandGroupWords <= NT, "one word per thread");
    auto load_bas = [&](const BandRange &r) -> uint32_t {
        const uint32_t g0 = r.es / kGroup * 8u, ng = r.ee > r.es ? (r.ee - 1u) / kGroup * 8u + 8u - g0 : 0u;
        return tid < ng ? rel_base[g0 + tid] - 1u : 0u;
    };
    const uint32_t bpos = (tid & ~7u) | ((tid + 6u) & 7u);
    auto put_bas = [&](int p, uint32_t v) {
        if (tid < (uint32_t)kBandGroupWords) bas[(uint32_t)(p & 3) * kBandGroupWords + bpos] = v;
    };
    // a thread's slots of a plane: voxel e = first + u * NT, clamped to the range
    // (the pools of the second pass are the first pass's results, in place)
    struct Slots {
        R m1[U], m3[U], m4[U], m5[U];
        uint32_t w[U];
    };
    auto load_slots = [&](const BandRange &r, Slots &s) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t wb = (r.es & ~63u) + wb0 + (uint32_t)(u * NT);
            if (wb < r.ee) {   // uniform over the wave
                const uint32_t e = wb + lane, i = e < r.es ? r.es : (e < r.ee ? e : r.ee - 1u);
                s.w[u] = at(rel_w, i);
                s.m1[u] = at(F.src[0], i);
                s.m3[u] = at(F.src[2], i);
                s.m4[u] = at(F.src[3], i);
                s.m5[u] = at(F.src[4], i);
            }
        }
    };
    // LDS offsets (in elements of a ring) of the six neighbours of voxel i:
    // own plane at oc - sc, below at om - sm, above at op - sp; an absent
    // neighbour is the voxel itself
    auto neighbours = [&](uint32_t w, const uint32_t *b, uint32_t i, uint32_t oc, uint32_t sc, uint32_t om,
                          uint32_t sm, uint32_t op, uint32_t sp, uint32_t (&q)[6]) {
        const uint32_t own = oc + (i - sc);
        const uint4 bd = *reinterpret_cast<const uint4 *>(b);
        uint32_t c[6];
#pragma unroll
        for (int k = 0; k < 6; k++) c[k] = (w >> L.sh[k]) & L.mk[k];
        q[0] = own - c[0];   // raster order: an x neighbour is the voxel before or after (code 1)
        q[1] = own + c[1];
        const uint32_t ym = own - bd.x - c[2], yp = own + bd.y + c[3], zm = om + i - sm - bd.z - c[4],
                       zp = op + i - sp + bd.w + c[5];
        q[2] = c[2] ? ym : own;
        q[3] = c[3] ? yp : own;
        q[4] = c[4] ? zm : own;
        q[5] = c[5] ? zp : own;
    };

    BandRange rm = range(z0 - 3), rq = range(z0 - 2), rp = range(z0 - 1), rn = range(z0), rn2 = range(z0 + 1);
    (void)rm;
    // march start: DOM of planes z0 - 2 .. z0, the first plane's slots
    R v[kBandRaw];
    {
        R a0[kBandRaw], a1[kBandRaw];
        load_raw(rq, a0);
        load_raw(rp, a1);
        load_raw(rn, v);
        put_raw(z0 + 2, rq, a0);   // plane z0 - 2 (the ring position of z0 + 2)
        put_raw(z0 + 3, rp, a1);
        put_raw(z0, rn, v);
    }
    Slots nxt, cur, old;
    load_slots(rp, nxt);
    put_bas(z0 + 3, load_bas(rp));
    load_raw(rn2, v);
    uint32_t bv = load_bas(rn);
    __syncthreads();
    for (int p = z0 - 1; p <= z1; p++) {
        const BandRange rn3 = range(p + 3);
        cur = nxt;
        if (p < z1) load_slots(rn, nxt);
        // first pass on plane p, e range
        const uint32_t fm = (uint32_t)((p + 3) & 3) * G.capf, fc = (uint32_t)(p & 3) * G.capf,
                       fp = (uint32_t)((p + 1) & 3) * G.capf;
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t wb = (rp.es & ~63u) + wb0 + (uint32_t)(u * NT);
            if (wb < rp.ee) {
                const uint32_t e = wb + lane, i = e < rp.es ? rp.es : (e < rp.ee ? e : rp.ee - 1u);
                const uint32_t *bp = bas + (uint32_t)(p & 3) * kBandGroupWords + (wb / kGroup - rp.es / kGroup) * 8u;
                uint32_t q[6];
                neighbours(cur.w[u], bp, i, fc, rp.fs, fm, rq.fs, fp, rn.fs, q);
                R x2 = raw[fc + (i - rp.fs)];
                R g[6], d[6];
#pragma unroll
                for (int k = 0; k < 6; k++) g[k] = raw[q[k]];
#pragma unroll
                for (int k = 0; k < 6; k++) d[k] = g[k] - x2;
                x2 = x2 + C.a[1] * (((d[0] + d[1]) + (d[2] + d[3])) + (d[4] + d[5]));
                transform_alg<false>(C, cur.m1[u], x2, cur.m3[u], cur.m4[u], cur.m5[u]);
                if (e >= rp.es && e < rp.ee) dom1[(uint32_t)(p & 3) * G.cape + (e - rp.es)] = x2;
            }
        }
        if (p < z1) {
            put_raw(p + 2, rn2, v);
            put_bas(p + 1, bv);
            load_raw(rn3, v);
            bv = load_bas(rn2);
        }
        lds_barrier();
        // second pass on plane p - 1, band rows
        if (p - 1 >= z0) {
            const uint32_t dm = (uint32_t)((p + 2) & 3) * G.cape, dc = (uint32_t)((p + 3) & 3) * G.cape,
                           dp = (uint32_t)(p & 3) * G.cape;
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint32_t wb = (rq.es & ~63u) + wb0 + (uint32_t)(u * NT);
                if (wb < rq.be && wb + 64u > rq.bs) {
                    const uint32_t e = wb + lane, i = e < rq.es ? rq.es : (e < rq.ee ? e : rq.ee - 1u);
                    const uint32_t *bp =
                        bas + (uint32_t)((p + 3) & 3) * kBandGroupWords + (wb / kGroup - rq.es / kGroup) * 8u;
                    const bool act = e >= rq.bs && e < rq.be;
                    // (the neighbour rows' outer neighbours are not held: lanes outside the band read the voxel itself)
                    uint32_t q[6];
                    neighbours(act ? old.w[u] : 0u, bp, i, dc, rq.es, dm, rm.es, dp, rp.es, q);
                    R x1 = old.m1[u], x2 = dom1[dc + (i - rq.es)], x3 = old.m3[u], x4 = old.m4[u], x5 = old.m5[u];
                    R g[6], d[6];
#pragma unroll
                    for (int k = 0; k < 6; k++) g[k] = dom1[q[k]];
#pragma unroll
                    for (int k = 0; k < 6; k++) d[k] = g[k] - x2;
                    x2 = x2 + C.a[1] * (((d[0] + d[1]) + (d[2] + d[3])) + (d[4] + d[5]));
                    transform_alg<false>(C, x1, x2, x3, x4, x5);
                    if (act) {
                        at(F.dst[0], i) = x1;
                        at(F.dst[1], i) = x2;
                        at(F.dst[2], i) = x3;
                        at(F.dst[3], i) = x4;
                        at(F.dst[4], i) = x5;
                    }
                }
            }
        }
        old = cur;
        rm = rq;
        rq = rp;
        rp = rn;
        rn = rn2;
        rn2 = rn3;
    }
}

template <int MODE, int MOB, int TOT>
int launch_c(vg_sim *h, const CompBufs &B, const Coef<double> &C, hipStream_t s) {
    Pieces pc{h->piece_first, h->piece_lo, h->piece_seg, h->npieces};
    if (B.tr.t1 > 0)
        hipLaunchKernelGGL((k_step_c<MODE, MOB, TOT, true>), dim3((unsigned)(B.tr.t1 - B.tr.t0)), dim3(kBlock), 0, s, B,
                           C, pc, part_of(h));
    else
        hipLaunchKernelGGL((k_step_c<MODE, MOB, TOT, false>), dim3((unsigned)h->ntiles), dim3(kBlock), 0, s, B, C, pc,
                           part_of(h));
    return launch_status("k_step_c");
}

template <int MODE, int MOB>
int pick_tot_c(vg_sim *h, int tot, const CompBufs &B, const Coef<double> &C, hipStream_t s) {
    switch (tot) {
        case TOT_NONE: return launch_c<MODE, MOB, TOT_NONE>(h, B, C, s);
        case TOT_IN: return launch_c<MODE, MOB, TOT_IN>(h, B, C, s);
        case TOT_MID: return launch_c<MODE, MOB, TOT_MID>(h, B, C, s);
        default: return launch_c<MODE, MOB, TOT_OUT>(h, B, C, s);
    }
}

// A pass on compensated fields: the same buffer rotation as dispatch<R>, for
// the float parts and the compensation words alike.
int dispatch_c(vg_sim *h, int mode, int tot, double dt_t, double dt_d, const TileRange *tr, hipStream_t s) {
    CompBufs B;
    if (tr) B.tr = *tr;
    B.nbr = h->nbr;
    B.rcode = h->rcode;
    B.pk = packed_of(h);
    B.ns = use_relative(h) ? 1 : (use_offsets(h) ? 2 : 0);
    B.n = h->n;
    const int mob = h->mobile_mode();
    for (int p = 0; p < VG_NPOOL; p++) {
        const bool mob_p = mob == 2 || p == 1;
        const int64_t off = (int64_t)p * h->n;
        float *here = (float *)h->fields + off;
        int16_t *here_lo = h->lo + off;
        float *there = nullptr;
        int16_t *there_lo = nullptr;
        if (mob_p) {
            there = (float *)h->alt + (mob == 2 ? off : 0);
            there_lo = h->lo_alt + (mob == 2 ? off : 0);
        }
        const bool flip = mob_p && h->cur;
        float *cur = flip ? there : here, *oth = flip ? here : there;
        int16_t *cur_lo = flip ? there_lo : here_lo, *oth_lo = flip ? here_lo : there_lo;
        const bool moves = mob_p && (mode == MODE_D || mode == MODE_DT);
        B.src[p] = cur;
        B.slo[p] = cur_lo;
        B.dst[p] = moves ? oth : cur;
        B.dlo[p] = moves ? oth_lo : cur_lo;
    }
    const Coef<double> C = make_coef2<double>(h, dt_t, dt_d);
    int rc;
    if (mode == MODE_T) rc = pick_tot_c<MODE_T, 1>(h, tot, B, C, s);
    else if (mode == MODE_NONE) rc = launch_c<MODE_NONE, 1, TOT_IN>(h, B, C, s);
    else if (mode == MODE_D) rc = mob == 2 ? pick_tot_c<MODE_D, 2>(h, tot, B, C, s) : pick_tot_c<MODE_D, 1>(h, tot, B, C, s);
    else rc = mob == 2 ? pick_tot_c<MODE_DT, 2>(h, tot, B, C, s) : pick_tot_c<MODE_DT, 1>(h, tot, B, C, s);
    if (rc) return rc;
    if (mode == MODE_D || mode == MODE_DT) h->cur ^= 1;
    return VG_OK;
}

// State conversions: x [5][n] of type X into the bound fields, or back.
template <typename X, typename F>
__global__ __launch_bounds__(kBlock) void k_load_state(const X *__restrict__ x, int64_t m, F f) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < m) f.put(i, (double)x[i]);
}

template <typename X, typename F>
__global__ __launch_bounds__(kBlock) void k_store_state(X *__restrict__ x, int64_t m, F f) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < m) x[i] = (X)f.get(i);
}

// float parts of compensated fields as float (the exact values, no rounding)
__global__ __launch_bounds__(kBlock) void k_store_hi(float *__restrict__ x, int64_t m, const float *__restrict__ hi) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < m) x[i] = hi[i];
}

template <typename R>
int dispatch(vg_sim *h, int mode, int tot, double dt_t, double dt_d, hipStream_t s) {
    StepBufs<R> B = graph_bufs<R>(h);
    const int mob = h->mobile_mode();
    R *canon = (R *)h->fields;
    R *alt = (R *)h->alt;
    for (int p = 0; p < VG_NPOOL; p++) {
        const bool mob_p = mob == 2 || p == 1;
        R *here = canon + (int64_t)p * h->n;
        R *there = nullptr;
        if (mob_p) there = (mob == 2) ? alt + (int64_t)p * h->n : alt;
        R *cur = (mob_p && h->cur) ? there : here;
        R *oth = (mob_p && h->cur) ? here : there;
        B.src[p] = cur;
        // a pass that diffuses writes mobile pools to the other buffer
        B.dst[p] = (mob_p && (mode == MODE_D || mode == MODE_DT)) ? oth : cur;
        if (h->band_mid) {   // a fused pass that takes the state back from the band kernel's set
            B.src[p] = (R *)h->band_alt + (int64_t)p * h->n;
            B.dst[p] = cur;
        }
    }
    if (h->band_mid) {
        if (mode != MODE_DT) {
            set_error("only a fused pass takes the state back from the band kernel's field set");
            return VG_ESTATE;
        }
        const int rc = dispatch_bufs<R>(h, mode, tot, dt_t, dt_d, B, s);
        if (!rc) h->band_mid = 0;
        return rc;
    }
    const int rc = dispatch_bufs<R>(h, mode, tot, dt_t, dt_d, B, s);
    if (rc) return rc;
    if (mode == MODE_D || mode == MODE_DT) h->cur ^= 1;
    return VG_OK;
}

}  // namespace

// Neighbour source: an explicit choice, else packed offsets when they fit,
// else the rank index when there is one, else the table.
PackedNbr packed_of(const vg_sim *h) {
    PackedNbr P;
    P.rel_w = h->rel_w;
    P.rel_base = h->rel_base;
    P.rl = h->rel_layout;
    P.off_m = h->off_m;
    P.off_p = h->off_p;
    P.dl = h->off_layout;
    return P;
}

bool use_relative(const vg_sim *h) {
    return h->rel_ok &&
           (h->kernel == VG_KERNEL_AUTO || h->kernel == VG_KERNEL_RELATIVE || h->kernel == VG_KERNEL_BAND);
}

bool band_geometry(const vg_sim *h) {
    return (h->features & VG_FEAT_BAND) && h->nseg == 1 && h->vox != nullptr && h->brick == 0 &&
           h->periodic == 0 && h->n > 0 && h->prec != VG_F32C;
}

// AUTO takes the band kernel when its chunks are long enough (build_band).
bool use_band(const vg_sim *h) {
    return h->band_ok && h->rel_ok && h->prec != VG_F32C &&
           (h->kernel == VG_KERNEL_BAND || (h->kernel == VG_KERNEL_AUTO && h->band_auto)) &&
           !h->mobile_all && h->rcode == nullptr && h->params.sequential == 0;
}

// Row index, band height and chunk length.  The band height is the largest
// whose widest plane fits the kernel's slots and whose LDS fits a CU, for
// FP32 twice (taller bands recompute fewer neighbour rows; a march step costs
// about 3 us whatever its width, so lower ones only add steps); the chunks
// are sized so that every block is resident at once.
// AUTO takes the kernel where two things hold.  The chunks have at least 8
// planes: shorter ones spend too much on their two extra planes.  Measured, 33
// steps, single passes over pairs: FP32 chunks of 4-6 planes (200^3, 256^3)
// 0.69-1.03, 8-9 (300^3; 500x120x500) 1.07-1.20, 24 and more (420^3 and up)
// 1.39-1.51; FP64 6 planes (200^3) 0.99, 10-18 (256^3, 300^3) 1.13-1.30, 28
// and more 1.57-1.66.
// And the single passes' bytes over the band kernel's own, times the share of
// the resident blocks that its launch fills and the planes of a chunk over
// those it marches, reach a break-even: where rows are full the slots leave
// bands of one to three rows, whose pools are read (H + 2) / H times, and
// their number may leave many CUs without a block.  Measured as above, with
// that estimate in brackets, the fields larger than the last-level cache
// (neighbour rows come from caches in part, so bands gain from 0.85 on):
// 400x400x600 full FP32 0.82 [0.68], FP64 0.90 [0.69]; 300x300x800 at porosity
// 0.4 FP64 0.85 [0.72]; 400^3 at 0.8 FP64 (134 blocks on 256 CUs) 0.92 [0.74],
// full 1.02 [0.74]; 512^3 full FP64 1.08-1.14 [0.89]; 330x400x450 full FP32
// 1.08 [0.94]; 450^3 at 0.8 1.15 [1.06], 1.26 [1.08]; 300^3 - 512^3 at 0.3 -
// 0.7 1.34-1.79 [1.18 and more].  Within that cache single passes reread at
// its rate: 120x120x1000 at 0.45 FP32 0.70 [0.77], 150x150x1000 at 0.35 FP32
// 0.89-0.92 [1.00], 160x160x900 at 0.4 FP32 0.95-1.01 [1.07], 200x200x1000 at
// 0.3 FP32 1.03-1.07 [1.14].  An FP32 block alone on its CU has too few loads
// in flight: 20x512x512 full 0.87-0.90 [1.11], 300x480x500 at 0.9 0.97 [1.14],
// 300x500x500 full 1.06 [1.18], 512^3 full 1.16 [1.22].
// In FP32 one-row bands are not taken for the sake of two blocks on a CU (512^3
// full: one row 1126 us a step, two rows 966, single passes 1123).
constexpr double kBandGain = 0.85, kBandGainCached = 1.05, kBandGainAlone = 1.15, kBandCached = 256e6;

int build_band(vg_sim *h, hipStream_t s) {
    h->band_ok = false;
    h->band_auto = false;
    if (!band_geometry(h) || !h->rel_ok) return VG_OK;
    const int64_t nrows = (int64_t)h->nz * h->ny;
    hipLaunchKernelGGL(k_band_rows, dim3((unsigned)((nrows + 1 + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, h->vox,
                       h->n, h->nx, nrows, h->band_rs);
    int rc = launch_status("k_band_rows");
    if (rc) return rc;
    std::vector<int32_t> rs((size_t)nrows + 1);
    if ((rc = hip_status(hipMemcpyAsync(rs.data(), h->band_rs, sizeof(int32_t) * rs.size(), hipMemcpyDeviceToHost, s),
                         "band rows"))) return rc;
    if ((rc = hip_status(hipStreamSynchronize(s), "band rows"))) return rc;
    if (rs[(size_t)nrows] != h->n) { set_error("row index does not cover the compact list"); return VG_EINVAL; }
    const size_t lds_cu = (size_t)160 * 1024;
    static const int hs[] = {32, 28, 24, 20, 18, 16, 14, 12, 11, 10, 9, 8, 7, 6, 5, 4, 3, 2, 1};
    for (size_t lds_max = h->prec == VG_F64 ? lds_cu : lds_cu / 2; lds_max <= lds_cu; lds_max *= 2) {
        for (int H : hs) {
            int64_t capf = 1, cape = 1, sumf = 0, sume = 0;   // widest ranges and sums over the bands and planes
            bool fits = true;
            for (int z = 0; z < h->nz && fits; z++)
                for (int y0 = 0; y0 < h->ny; y0 += H) {
                    const int32_t *row = rs.data() + (size_t)z * h->ny;
                    const int y1 = std::min(y0 + H, h->ny);
                    const int64_t es = row[std::max(y0 - 1, 0)], ee = row[std::min(y1 + 1, h->ny)];
                    const int64_t f = (int64_t)row[std::min(y1 + 2, h->ny)] - row[std::max(y0 - 2, 0)];
                    capf = std::max(capf, f);
                    cape = std::max(cape, ee - es);
                    sumf += f;
                    sume += ee - es;
                    if (ee - es / kGroup * kGroup > kBandSlots || f > (int64_t)kBandThreads * kBandRaw) {
                        fits = false;
                        break;
                    }
                }
            if (!fits) continue;
            const size_t lds = h->prec == VG_F64 ? band_lds_bytes<double>(capf, cape) : band_lds_bytes<float>(capf, cape);
            if (lds > lds_max || (H < 2 && lds_max < lds_cu)) continue;
            // blocks resident at once (registers and this LDS size) on the
            // device.  The attribute belongs to the kernel, not to the handle,
            // so every handle sets the same value; a device that refuses it,
            // or that holds no such block, gets single passes.
            int per = 0, cus = 0, dev = 0;
            const void *kern = h->prec == VG_F64 ? (const void *)k_band2<double> : (const void *)k_band2<float>;
            if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_cu) != hipSuccess ||
                hipGetDevice(&dev) != hipSuccess ||
                hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
                hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, kBandThreads, lds) != hipSuccess ||
                per < 1 || cus < 1) {
                (void)hipGetLastError();
                return VG_OK;
            }
            h->band_h = H;
            h->band_capf = capf;
            h->band_cape = cape;
            h->band_nbands = (h->ny + H - 1) / H;
            const int chunks = std::max(1, std::min(per * cus / h->band_nbands, (h->nz + 3) / 4));
            h->band_z = (h->nz + chunks - 1) / chunks;
            h->band_ok = true;
            // bytes of two passes: DOM of the f ranges, the other pools and the codes of the e ranges, the output;
            // against two single passes
            const double R = (double)h->elem(), codes = 4.5, n = (double)h->n;
            const double pair = R * (double)sumf + (4.0 * R + codes) * (double)sume + 5.0 * R * n;
            const double singles = 2.0 * (10.0 * R + codes) * n;
            const int64_t resident = (int64_t)per * cus;
            const int64_t blocks = (int64_t)h->band_nbands * ((h->nz + h->band_z - 1) / h->band_z);
            const int64_t rounds = (blocks + resident - 1) / resident;
            const double filled = (double)blocks / (double)(rounds * resident);
            const double planes = (double)h->band_z / (double)(h->band_z + 2);
            const double gain = h->prec == VG_F32 && per == 1 ? kBandGainAlone
                                : 5.0 * R * n <= kBandCached  ? kBandGainCached
                                                              : kBandGain;
            h->band_auto = h->band_z >= 8 && filled * planes * singles >= gain * pair;
            return VG_OK;
        }
    }
    return VG_OK;
}

namespace {
template <typename R>
int band_launch(vg_sim *h, double dt, hipStream_t s) {
    const Coef<R> C = make_coef2<R>(h, dt, dt);
    const BandGeom G{h->ny, h->nz, h->band_h, h->band_z, h->band_nbands, (uint32_t)h->band_capf, (uint32_t)h->band_cape};
    BandBufs<R> F;
    for (int p = 0; p < VG_NPOOL; p++) {
        R *here = (p == 1 && h->cur) ? (R *)h->alt : (R *)h->fields + (int64_t)p * h->n;
        R *mid = (R *)h->band_alt + (int64_t)p * h->n;
        F.src[p] = h->band_mid ? mid : here;
        F.dst[p] = h->band_mid ? here : mid;
    }
    const int blocks = h->band_nbands * ((h->nz + h->band_z - 1) / h->band_z);
    hipLaunchKernelGGL(k_band2<R>, dim3((unsigned)blocks), dim3(kBandThreads),
                       band_lds_bytes<R>(h->band_capf, h->band_cape), s, F, (const uint32_t *)h->rel_w,
                       (const uint32_t *)h->rel_base, h->rel_layout, C, G, (const int32_t *)h->band_rs);
    return launch_status("k_band2");
}
}  // namespace

// Two fused passes: from where the state is (the bound fields, or the
// intermediate set: h->band_mid) into the other set.
int launch_band_pair(vg_sim *h, double dt, hipStream_t s) {
    const int rc = h->prec == VG_F64 ? band_launch<double>(h, dt, s) : band_launch<float>(h, dt, s);
    if (!rc) h->band_mid ^= 1;
    return rc;
}

bool use_offsets(const vg_sim *h) {
    if (h->kernel == VG_KERNEL_OFFSET) return h->off_ok;
    return h->off_ok && h->kernel == VG_KERNEL_AUTO && !h->rel_ok;
}

bool use_rank(const vg_sim *h) {
    const bool ok = h->rank != nullptr && h->geo != nullptr && h->nseg == 1 && h->prec != VG_F32C;
    if (h->kernel == VG_KERNEL_RANK) return ok;
    return ok && h->kernel == VG_KERNEL_AUTO && !h->off_ok && !h->rel_ok;
}

static uint32_t bit_width(uint32_t v) {
    uint32_t b = 0;
    while (v) { b++; v >>= 1; }
    return b;
}

// Measures the neighbour distances and, when they fit, writes the packed
// offsets.  Synchronises the stream (the layout is chosen on the host).
int build_offsets(vg_sim *h, hipStream_t s) {
    h->off_ok = false;
    h->rel_ok = false;
    h->xy_dist = h->z_dist = -1;
    if (h->n == 0 || !h->off_m || !h->rel_w || !h->nbr) return VG_OK;
    int rc;
    if ((rc = hip_status(hipMemsetAsync(h->off_stat, 0, 8 * sizeof(uint32_t), s), "clear offset statistics")))
        return rc;
    const unsigned blocks = (unsigned)((h->n + kBlock - 1) / kBlock);
    const unsigned stat_blocks = blocks < 2048u ? blocks : 2048u;
    hipLaunchKernelGGL(k_neighbour_stat, dim3(stat_blocks), dim3(kBlock), 0, s, h->nbr, h->n, h->rel_base,
                       h->off_stat);
    if ((rc = launch_status("k_neighbour_stat"))) return rc;
    uint32_t st[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if ((rc = hip_status(hipMemcpyAsync(st, h->off_stat, sizeof(st), hipMemcpyDeviceToHost, s), "read offsets")))
        return rc;
    if ((rc = hip_status(hipStreamSynchronize(s), "synchronise"))) return rc;
    if (!st[3]) {
        h->xy_dist = st[0] > st[1] ? st[0] : st[1];
        h->z_dist = st[2];
    }
    const uint32_t bx = bit_width(st[0]), by = bit_width(st[1]), bz = bit_width(st[2]);
    // periodic wrap or byte offsets beyond 32 bits: neither packing
    if (st[3] || (uint64_t)h->n * h->elem() >= ((uint64_t)1 << 32)) return VG_OK;
    auto mask = [](uint32_t b) { return b >= 32 ? 0xffffffffu : (1u << b) - 1u; };
    // relative codes: widths from the largest spread + 1 per axis
    const uint32_t cx = bit_width(st[4]), cy = bit_width(st[5]), cz = bit_width(st[6]);
    if (2 * (cx + cy + cz) <= 32) {
        RLayout R;
        const uint32_t width[6] = {cx, cx, cy, cy, cz, cz};
        const uint32_t order[6] = {4, 5, 2, 3, 0, 1};      // z-, z+, y-, y+, x-, x+ from bit 0 up
        uint32_t at_bit = 0;
        for (int q = 0; q < 6; q++) {
            const uint32_t k = order[q];
            R.sh[k] = at_bit & 31u;                         // a zero-width field's shift is never used
            R.mk[k] = mask(width[k]);
            at_bit += width[k];
        }
        hipLaunchKernelGGL(k_rel_pack, dim3(blocks), dim3(kBlock), 0, s, h->nbr, h->n, h->rel_base, R, h->rel_w);
        if ((rc = launch_status("k_rel_pack"))) return rc;
        h->rel_layout = R;
        h->rel_ok = true;
    }
    // neighbours too far apart: no packed offsets
    if (bx + by + bz > 32) return VG_OK;
    DLayout L;
    L.bz = bz & 31u;                     // an empty field's shift is never used
    L.by = by;
    L.sx = (bz + by) & 31u;
    L.mz = mask(bz);
    L.my = mask(by);
    L.mx = mask(bx);
    hipLaunchKernelGGL(k_offsets, dim3(blocks), dim3(kBlock), 0, s, h->nbr, h->n, L, h->off_m, h->off_p);
    if ((rc = launch_status("k_offsets"))) return rc;
    h->off_layout = L;
    h->off_ok = true;
    return VG_OK;
}

int launch_geometry(vg_sim *h, hipStream_t s) {
    if (!h->rank || h->n == 0) return VG_OK;
    hipLaunchKernelGGL(k_geometry, dim3((unsigned)((h->n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, h->vox, h->n,
                       make_rgeom(h), h->geo);
    return launch_status("k_geometry");
}

int launch_pass2(vg_sim *h, int mode, int tot, double dt_t, double dt_d, hipStream_t s, const TileRange *tr) {
    if (h->n == 0) return VG_OK;
    if (h->prec == VG_F32C) return dispatch_c(h, mode, tot, dt_t, dt_d, tr, s);
    if (h->prec == VG_F64) return dispatch<double>(h, mode, tot, dt_t, dt_d, s);
    return dispatch<float>(h, mode, tot, dt_t, dt_d, s);
}

int launch_pass(vg_sim *h, int mode, int tot, double dt, hipStream_t s) {
    return launch_pass2(h, mode, tot, dt, dt, s);
}

// A pass between explicit buffers (pool s read from src[s], written to
// dst[s]); used by the adjoint's forward recording.  xdom: see StepBufs
// (fused passes, only DOM diffusing; a row the pass does not read).
int launch_pass_bufs(vg_sim *h, int mode, int tot, double dt, const void *const src[VG_NPOOL],
                     void *const dst[VG_NPOOL], hipStream_t s, void *xdom) {
    if (h->n == 0) return VG_OK;
    if (h->prec == VG_F64) {
        StepBufs<double> B = graph_bufs<double>(h);
        for (int p = 0; p < VG_NPOOL; p++) { B.src[p] = (const double *)src[p]; B.dst[p] = (double *)dst[p]; }
        B.xdom = (double *)xdom;
        return dispatch_bufs<double>(h, mode, tot, dt, dt, B, s);
    }
    StepBufs<float> B = graph_bufs<float>(h);
    for (int p = 0; p < VG_NPOOL; p++) { B.src[p] = (const float *)src[p]; B.dst[p] = (float *)dst[p]; }
    B.xdom = (float *)xdom;
    return dispatch_bufs<float>(h, mode, tot, dt, dt, B, s);
}

int launch_totals_finalize(vg_sim *h, double *out_rows, int rows, hipStream_t s) {
    if (h->nseg == 0 || h->n == 0 || rows <= 0) return VG_OK;
    const int64_t part_stride = (int64_t)VG_NPOOL * h->npieces, out_stride = (int64_t)h->nseg * 6;
    const int64_t chunk_stride = (int64_t)VG_NPOOL * h->nchunks;
    if (h->max_seg_pieces <= kDirectPieces) {
        hipLaunchKernelGGL(k_tot_direct, dim3((unsigned)h->nseg, (unsigned)rows), dim3(kBlock), 0, s, h->part,
                           h->seg_first, out_rows, part_stride, out_stride);
        return launch_status("k_tot_direct");
    }
    hipLaunchKernelGGL(k_tot_chunks, dim3((unsigned)h->nchunks, (unsigned)rows), dim3(kBlock), 0, s, h->part,
                       h->chunk_first, h->chunk_part, part_stride, chunk_stride);
    int rc = launch_status("k_tot_chunks");
    if (rc) return rc;
    hipLaunchKernelGGL(k_tot_segments, dim3((unsigned)h->nseg, (unsigned)rows), dim3(kBlock), 0, s, h->chunk_part,
                       h->seg_chunk, out_rows, chunk_stride, out_stride);
    return launch_status("k_tot_segments");
}

int launch_load_state(vg_sim *h, const void *x, int xprec, hipStream_t s) {
    const int64_t m = (int64_t)VG_NPOOL * h->n;
    if (m == 0) return VG_OK;
    const dim3 grid((unsigned)((m + kBlock - 1) / kBlock));
    if (h->prec == VG_F32C) {
        const CompAcc f{(float *)h->fields, h->lo};
        if (xprec == VG_F64) hipLaunchKernelGGL((k_load_state<double, CompAcc>), grid, dim3(kBlock), 0, s, (const double *)x, m, f);
        else hipLaunchKernelGGL((k_load_state<float, CompAcc>), grid, dim3(kBlock), 0, s, (const float *)x, m, f);
    } else if (h->prec == VG_F64) {
        const PlainAcc<double> f{(double *)h->fields};
        if (xprec == VG_F64) hipLaunchKernelGGL((k_load_state<double, PlainAcc<double>>), grid, dim3(kBlock), 0, s, (const double *)x, m, f);
        else hipLaunchKernelGGL((k_load_state<float, PlainAcc<double>>), grid, dim3(kBlock), 0, s, (const float *)x, m, f);
    } else {
        const PlainAcc<float> f{(float *)h->fields};
        if (xprec == VG_F64) hipLaunchKernelGGL((k_load_state<double, PlainAcc<float>>), grid, dim3(kBlock), 0, s, (const double *)x, m, f);
        else hipLaunchKernelGGL((k_load_state<float, PlainAcc<float>>), grid, dim3(kBlock), 0, s, (const float *)x, m, f);
    }
    return launch_status("k_load_state");
}

int launch_store_state(vg_sim *h, void *x, int xprec, hipStream_t s) {
    const int64_t m = (int64_t)VG_NPOOL * h->n;
    if (m == 0) return VG_OK;
    const dim3 grid((unsigned)((m + kBlock - 1) / kBlock));
    if (h->prec == VG_F32C) {
        const CompAcc f{(float *)h->fields, h->lo};
        if (xprec == VG_F64) hipLaunchKernelGGL((k_store_state<double, CompAcc>), grid, dim3(kBlock), 0, s, (double *)x, m, f);
        else hipLaunchKernelGGL(k_store_hi, grid, dim3(kBlock), 0, s, (float *)x, m, (const float *)h->fields);
    } else if (h->prec == VG_F64) {
        const PlainAcc<double> f{(double *)h->fields};
        if (xprec == VG_F64) hipLaunchKernelGGL((k_store_state<double, PlainAcc<double>>), grid, dim3(kBlock), 0, s, (double *)x, m, f);
        else hipLaunchKernelGGL((k_store_state<float, PlainAcc<double>>), grid, dim3(kBlock), 0, s, (float *)x, m, f);
    } else {
        const PlainAcc<float> f{(float *)h->fields};
        if (xprec == VG_F64) hipLaunchKernelGGL((k_store_state<double, PlainAcc<float>>), grid, dim3(kBlock), 0, s, (double *)x, m, f);
        else hipLaunchKernelGGL((k_store_state<float, PlainAcc<float>>), grid, dim3(kBlock), 0, s, (float *)x, m, f);
    }
    return launch_status("k_store_state");
}

// Mobile pools that currently live in the alt buffer are copied back to the
// caller's field buffer, so the fields hold the state between calls.
int restore_canonical(vg_sim *h, hipStream_t s) {
    if (!h->cur) return VG_OK;
    const size_t e = h->elem();
    const int mob = h->mobile_mode();
    int rc;
    if (h->prec == VG_F32C) {
        const size_t cnt = (mob == 2 ? VG_NPOOL : 1) * (size_t)h->n;
        const size_t at0 = mob == 2 ? 0 : (size_t)h->n;
        if ((rc = hip_status(hipMemcpyAsync(h->lo + at0, h->lo_alt, sizeof(int16_t) * cnt, hipMemcpyDeviceToDevice, s),
                             "restore compensation words")))
            return rc;
    }
    if (mob == 2) {
        rc = hip_status(hipMemcpyAsync(h->fields, h->alt, e * VG_NPOOL * (size_t)h->n, hipMemcpyDeviceToDevice, s),
                        "restore fields");
    } else {
        rc = hip_status(hipMemcpyAsync(h->fields + e * (size_t)h->n, h->alt, e * (size_t)h->n,
                                       hipMemcpyDeviceToDevice, s),
                        "restore DOM");
    }
    if (rc) return rc;
    h->cur = 0;
    return VG_OK;
}

}  // namespace vg
