// sigma_abl.hip -- the alpha-beta part sigma_3 (Eq. 8) of one-block (CAS) spaces of
// up to 10 orbitals in FP64, with the beta-side scatter through a sorted list (abx.h).
//
// The contraction is that of sigma_abx.hip: one workgroup per output alpha string Ia
// keeps its sigma row in LDS and visits the beta strings in 32-column tiles,
//   R(a, Jb)  = C(Ja_a, Jb)        a = the single alpha excitations Ja_a of Ia, plus Ia itself
//   W(kl, Jb) = sum_a A(kl, a) R(a, Jb),  A(kl, a) = s_a (i_a j_a|kl),  A(kl, Ia) = sum_{j in Ia} (jj|kl)
//   sigma(Ia, Ib) += sum_{(kl, Jb): Ib = E_kl Jb} <Ib|E_kl|Jb> W(kl, Jb);
// Ia's own row takes a k slot (SELF) or starts the accumulators as a rank-1 term.
//
// Why it stays beside the quad form: its sums run in list order, as ever, so FP64 results
// of these spaces are what they were, bit for bit -- the signs of the vectors of a Davidson
// at its 1e-12 hang on the last bits of sigma (with the quad form's sums 8 of 18 came out
// negated) -- and little time is lost: with at most 252 strings a launch is one workgroup
// per compute unit and a handful of tiles, and a call's other launches take most of its
// time (CAS(10,10): 26 us here and 15 in the quad form, of ~50 for a sigma).  From 11
// orbitals on the quad form takes 0.6 of a sigma's time and the sums did change order; the
// vectors' signs there are as arbitrary as they were.
#include "internal.h"
#include "mfma.h"
#include "bufio.h"
#include "abx.h"

#include <algorithm>

namespace cis {
namespace {

using T = double;
using acc_t = Mfma<T>::acc_t;
using vec_t = Mfma<T>::vec_t;

struct AbxArgs {
    const T *cp;           // C, alpha-major padded (row stride ld)
    T *sp;                 // sigma accumulator, same layout (read, then overwritten)
    const uint32_t *aexc;  // [Na][anexc]
    const uint32_t *astr;  // [Na]
    const T *gp;           // [n*n][kp]
    const uint32_t *plan;  // [ntile][4 waves][EW][64 lanes]
    uint32_t cp_bytes;     // bytes of C including the zero row (< 2^31)
    uint32_t plan_bytes;   // bytes of the plan (< 2^31)
    int anexc, n, kp, npair, Na, ld;
};

// KS: k steps over the gathered rows (4*KS >= anexc+1); RB: 16-row blocks of kl
// (16*RB >= npair); RBW: row blocks per producing wave; EW: plan entries per
// lane and tile.  A producing wave owns one 16-column half of the 32-column
// tile (cb) and a run of row blocks [rb0, rb0 + nrb).

// A(m, Ia) = sum_{j in Ia} (jj|kl) for the kl pair of row m
__device__ __forceinline__ T abx_self_coef(const AbxArgs &p, uint32_t xa, int m) {
    T val = 0;
    for (uint32_t b = xa; b; b &= b - 1) {
        const int j = __ffs(b) - 1;
        val += p.gp[int64_t(j * p.n + j) * p.kp + m];
    }
    return val;
}

// A fragments of Ia for the wave's row blocks -- row m (kl) = 16*(rb0 + r) +
// lane%16, column k = 4t + lane/16 -- and the byte offsets of the gathered rows
// (missing excitations read the zero row Na).  With SELF, column anexc is Ia's
// own row.
template <int KS, int RBW, bool SELF>
__device__ __forceinline__ void abx_fragments(const AbxArgs &p, int Ia, int lane, int cb, int rb0, int nrb,
                                              T (&A)[RBW][KS], uint32_t (&boff)[KS]) {
    const uint32_t xa = p.astr[Ia];
    const uint32_t col = uint32_t(cb * 16 + (lane & 15));
#pragma unroll
    for (int t = 0; t < KS; ++t) {
        const int k = 4 * t + (lane >> 4);
        int J = p.Na;
        const T *g = nullptr;
        T sg = 0;
        if (k < p.anexc) {
            const uint32_t e = p.aexc[int64_t(Ia) * p.anexc + k];
            if (e != kExcNone) {
                J = int(e >> 11);
                const int i = (e >> 6) & 31, j = (e >> 1) & 31;   // <Ia|E_ij|Ja>, Ja = Ia - i + j
                g = p.gp + int64_t(i * p.n + j) * p.kp;
                sg = (e & 1) ? T(-1) : T(1);
            }
        } else if (SELF && k == p.anexc) {
            J = Ia;
        }
        boff[t] = (uint32_t(J) * uint32_t(p.ld) + col) * uint32_t(sizeof(T));   // < cp_bytes
#pragma unroll
        for (int r = 0; r < RBW; ++r) {
            const int m = (rb0 + r) * 16 + (lane & 15);
            T val = 0;
            if (r < nrb && m < p.npair) {
                if (g) {
                    val = sg * g[m];
                } else if (SELF && k == p.anexc) {
                    val = abx_self_coef(p, xa, m);
                }
            }
            A[r][t] = val;
        }
    }
}

// Without SELF: A(m, Ia) for the lane's accumulator rows m = 16*(rb0 + r) +
// out_row(lane, i), and the byte offset of C(Ia, column) of the lane's column
template <int RBW>
__device__ __forceinline__ void abx_self_fragments(const AbxArgs &p, int Ia, int lane, int cb, int rb0, int nrb,
                                                   T (&dI)[RBW][4], uint32_t &boffI) {
    using M = Mfma<T>;
    const uint32_t xa = p.astr[Ia];
#pragma unroll
    for (int r = 0; r < RBW; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = (rb0 + r) * 16 + M::out_row(lane, i);
            dI[r][i] = (r < nrb && m < p.npair) ? abx_self_coef(p, xa, m) : T(0);
        }
    boffI = (uint32_t(Ia) * uint32_t(p.ld) + uint32_t(cb * 16 + (lane & 15))) * uint32_t(sizeof(T));   // < cp_bytes
}

template <int KS>
__device__ __forceinline__ void abx_load(__amdgpu_buffer_rsrc_t cr, const uint32_t (&boff)[KS], int tile, T (&b)[KS]) {
    const uint32_t soff = uint32_t(tile) * uint32_t(kAbxNT * sizeof(T));
#pragma unroll
    for (int t = 0; t < KS; ++t) buffer_ld(b[t], cr, boff[t], soff);
}

// W = A R on the matrix cores for the rows held in b; as each k step is
// consumed, b[t] is reloaded with the rows of tile `next` (always a valid
// tile), so the loads stay in flight for a whole tile.  Without SELF the
// accumulators start from A(kl, Ia) C(Ia, Jb), cI holding C(Ia, Jb) of this
// tile (reloaded likewise).
template <int KS, int RBW, bool SELF>
__device__ __forceinline__ void abx_products(__amdgpu_buffer_rsrc_t cr, const T (&A)[RBW][KS],
                                             const uint32_t (&boff)[KS], int next, T (&b)[KS],
                                             acc_t (&acc)[RBW], const T (&dI)[RBW][4],
                                             uint32_t boffI, T &cI) {
    using M = Mfma<T>;
    const uint32_t soff = uint32_t(next) * uint32_t(kAbxNT * sizeof(T));
    if constexpr (SELF) {
#pragma unroll
        for (int r = 0; r < RBW; ++r) acc[r] = acc_t{0, 0, 0, 0};
    } else {
#pragma unroll
        for (int r = 0; r < RBW; ++r)
            acc[r] = acc_t{dI[r][0] * cI, dI[r][1] * cI, dI[r][2] * cI, dI[r][3] * cI};
        buffer_ld(cI, cr, boffI, soff);
    }
#pragma unroll
    for (int t = 0; t < KS; ++t) {
#pragma unroll
        for (int r = 0; r < RBW; ++r) acc[r] = M::op(A[r][t], b[t], acc[r]);
        buffer_ld(b[t], cr, boff[t], soff);
        __builtin_amdgcn_sched_barrier(0);   // keep the reload next to its k step
    }
}

template <int RBW>
__device__ __forceinline__ void abx_store_w(T *W, const acc_t (&acc)[RBW], int lane, int cb,
                                            int rb0, int nrb) {
    using M = Mfma<T>;
#pragma unroll
    for (int r = 0; r < RBW; ++r)
        if (r < nrb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                W[((rb0 + r) * 16 + M::out_row(lane, i)) * kAbxWS + cb * 16 + (lane & 15)] = acc[r][i];
}

// On gfx950 an FP64 MFMA keeps its SIMD from issuing vector instructions of
// other waves, so a scatter wave that shares a SIMD with a producing wave waits
// out every matrix instruction.  The roles are therefore split by SIMD: the
// eight waves of a workgroup are placed on the four SIMDs in turn (wave w on
// SIMD w mod 4), waves 3 and 7 scatter (the four plan ranges of a tile, two
// each) and share one SIMD, and the other six multiply -- three 16-row-block
// groups x two 16-column halves -- on the other three SIMDs.  The sigma row
// leaves room for one W tile: the producing waves compute the next tile's W in
// registers while the scatter waves consume this tile's, and store it between
// two barriers.
template <int KS, int RB, int EW, bool SELF>
__global__ __launch_bounds__(512, 1) void k_sigma_ab_l(AbxArgs p) {
    constexpr int VEC = 16 / sizeof(T);
    constexpr int RBW = (RB + 2) / 3;
    constexpr int MP = 16 * RB;
    constexpr int PW = (EW + 1) * 64;                      // plan words per range and tile
    constexpr int PT = 4 * PW;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *W = reinterpret_cast<T *>(smem_raw);                // [MP][WS]
    T *sig = W + MP * kAbxWS;                              // [ld + 64]: slots ld.. take discarded writes

    const int Ia = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: the roles branch per wave
    const int64_t rowoff = int64_t(Ia) * p.ld;
    for (int c = tid * VEC; c < p.ld; c += 512 * VEC)
        *reinterpret_cast<vec_t *>(sig + c) = *reinterpret_cast<const vec_t *>(p.sp + rowoff + c);
    for (int r = tid; r < MP; r += 512) W[r * kAbxWS + kAbxNT] = T(0);   // pad column: plan padding reads it
    const int ntile = p.ld / kAbxNT;
    if ((wave & 3) != 3) {
        const int m = (wave >> 2) * 3 + (wave & 3);        // 0..5
        const int cb = m & 1, rb0 = (m >> 1) * RBW;
        const int nrb = RB - rb0 < RBW ? RB - rb0 : RBW;   // may be <= 0 for small RB
        T A[RBW][KS];
        uint32_t boff[KS];
        abx_fragments<KS, RBW, SELF>(p, Ia, lane, cb, rb0, nrb, A, boff);
        T dI[RBW][4] = {};
        uint32_t boffI = 0;
        if constexpr (!SELF) abx_self_fragments<RBW>(p, Ia, lane, cb, rb0, nrb, dI, boffI);
        const __amdgpu_buffer_rsrc_t cr = buffer_of(p.cp, p.cp_bytes);
        T b[KS];
        T cI = 0;
        acc_t acc[RBW];
        abx_load<KS>(cr, boff, 0, b);
        if constexpr (!SELF) buffer_ld(cI, cr, boffI, 0u);
        abx_products<KS, RBW, SELF>(cr, A, boff, ntile > 1 ? 1 : 0, b, acc, dI, boffI, cI);
        __syncthreads();                       // the sigma row is in LDS
        abx_store_w<RBW>(W, acc, lane, cb, rb0, nrb);
        __syncthreads();                       // W of tile 0 ready
        for (int tile = 0; tile < ntile; ++tile) {
            if (tile + 1 < ntile) {
                const int t2 = tile + 2 < ntile ? tile + 2 : ntile - 1;
                abx_products<KS, RBW, SELF>(cr, A, boff, t2, b, acc, dI, boffI, cI);
            }
            __syncthreads();                   // W of this tile consumed
            if (tile + 1 < ntile) abx_store_w<RBW>(W, acc, lane, cb, rb0, nrb);
            __syncthreads();                   // W of the next tile ready
        }
    } else {
        const __amdgpu_buffer_rsrc_t pr = buffer_of(p.plan, p.plan_bytes);
        const int sw = wave >> 2;                          // plan ranges sw and sw + 2
        const uint32_t pl0 = uint32_t(sw * PW + lane) * 4u, pl1 = uint32_t((sw + 2) * PW + lane) * 4u;
        const uint32_t spare = uint32_t(p.ld + lane) * uint32_t(sizeof(T));
        uint32_t pa0[EW], ha0, pa1[EW], ha1, pb0[EW], hb0, pb1[EW], hb1;
        abx_plan_load<EW>(pr, pl0, 0u, pa0, ha0);
        abx_plan_load<EW>(pr, pl1, 0u, pa1, ha1);
        __syncthreads();                       // the sigma row is in LDS
        __syncthreads();                       // W of tile 0 ready
        for (int tile = 0; tile < ntile; tile += 2) {
            const int t1 = tile + 1 < ntile ? tile + 1 : tile, t2 = tile + 2 < ntile ? tile + 2 : t1;
            abx_plan_load<EW>(pr, pl0, uint32_t(t1) * (PT * 4u), pb0, hb0);
            abx_plan_load<EW>(pr, pl1, uint32_t(t1) * (PT * 4u), pb1, hb1);
            abx_scatter<T, EW>(W, sig, pa0, ha0, spare);
            abx_scatter<T, EW>(W, sig, pa1, ha1, spare);
            __syncthreads();                   // W of this tile consumed
            __syncthreads();                   // W of the next tile ready
            if (tile + 1 < ntile) {
                abx_plan_load<EW>(pr, pl0, uint32_t(t2) * (PT * 4u), pa0, ha0);
                abx_plan_load<EW>(pr, pl1, uint32_t(t2) * (PT * 4u), pa1, ha1);
                abx_scatter<T, EW>(W, sig, pb0, hb0, spare);
                abx_scatter<T, EW>(W, sig, pb1, hb1, spare);
                __syncthreads();
                __syncthreads();
            }
        }
    }
    for (int cc = tid * VEC; cc < p.ld; cc += 512 * VEC)
        *reinterpret_cast<vec_t *>(p.sp + rowoff + cc) = *reinterpret_cast<const vec_t *>(sig + cc);
}

// LDS bytes: the W tile and the sigma row with its 64 discard slots
size_t abx_lds(int ld, int rb) {
    return (size_t(16) * rb * kAbxWS + ld + 64) * sizeof(T);
}

template <int KS, int RB, int EW, bool SELF>
hipError_t run_abx(const AbxArgs &a, hipStream_t s) {
    const size_t lds = abx_lds(a.ld, RB);
    if (lds > 160 * 1024 || 16 * RB < a.npair || 4 * KS < a.anexc + (SELF ? 1 : 0)) return hipErrorInvalidValue;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_sigma_ab_l<KS, RB, EW, SELF>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_sigma_ab_l<KS, RB, EW, SELF>), dim3(a.Na), dim3(512), lds, s, a);
    return hipGetLastError();
}

int ks_of(int anexc) { return (anexc + 1 + 3) / 4; }
int rb_of(int npair) { return (npair + 15) / 16; }

// The compiled (KS, RB, EW) shapes: for each (KS, RB) of the CAS(n, n/2)
// spaces n = 4..10 and their open-shell neighbours, the plan width of
// CAS(n, n/2) and a wider one.
#define CIS_ABX_SHAPES(X)                                                                              \
    X(2, 1, 2) X(2, 1, 16) X(3, 2, 2) X(3, 2, 16) X(4, 2, 4) X(4, 2, 16) X(4, 3, 4) X(4, 3, 16)         \
    X(5, 3, 4) X(5, 3, 16) X(6, 3, 4) X(6, 3, 16) X(6, 4, 4) X(6, 4, 16) X(7, 4, 4) X(7, 4, 16)

// Shapes with Ia's row as the rank-1 start of the accumulators, for the
// CAS(n, n/2) spaces of even n and their neighbours whose excitation count is
// a multiple of 4 (there it saves a k step; elsewhere the row fills padding).
// The 16-entry plan width serves spaces whose target groups would span more
// than four lanes at the narrow width (CAS(8,8) and smaller).
#define CIS_ABX_SHAPES_R1(X)                                                                            \
    X(1, 1, 2) X(1, 1, 16) X(2, 2, 2) X(2, 2, 16) X(4, 3, 4) X(4, 3, 16) X(6, 4, 4) X(6, 4, 16)

// shape[4] receives {KS, RB, EW, 1: row in a k step, 2: rank-1 start}
bool dispatch_abx(const AbxArgs &a, int ew, hipStream_t s, hipError_t *err, int *shape, const char **name) {
    const int rb = rb_of(a.npair);
    if (a.anexc > 0 && a.anexc % 4 == 0) {
        const int ks1 = a.anexc / 4;
#define CIS_RUN1(K, R, E)                                           \
    if (ks1 == K && rb == R && ew == E) {                           \
        *err = run_abx<K, R, E, false>(a, s);                    \
        shape[0] = K; shape[1] = R; shape[2] = E; shape[3] = 2;     \
        *name = "k_sigma_ab_l<" #K ", " #R ", " #E ", rank1>";      \
        return true;                                                \
    }
        CIS_ABX_SHAPES_R1(CIS_RUN1)
#undef CIS_RUN1
    }
    const int ks = ks_of(a.anexc);
#define CIS_RUN(K, R, E)                                            \
    if (ks == K && rb == R && ew == E) {                            \
        *err = run_abx<K, R, E, true>(a, s);                     \
        shape[0] = K; shape[1] = R; shape[2] = E; shape[3] = 1;     \
        *name = "k_sigma_ab_l<" #K ", " #R ", " #E ", self>";       \
        return true;                                                \
    }
    CIS_ABX_SHAPES(CIS_RUN)
#undef CIS_RUN
    return false;
}

bool owner_t(const cisigma_ctx *ctx, const void *cp, void *sp, hipStream_t s, hipError_t *err) {
    const ScatterPlan &P = ctx->plan;
    const uint32_t *plan = P.d_entries[0];
    if (!plan || P.ew == 0) return false;
    const auto &A = ctx->sp[0];
    AbxArgs x{};
    x.cp = static_cast<const T *>(cp);
    x.sp = static_cast<T *>(sp);
    x.aexc = A.d_exc;
    x.astr = A.d_str;
    x.gp = ctx->d_gp64;
    x.plan = plan;
    x.anexc = A.nexc;
    x.n = ctx->n;
    x.kp = ctx->kp;
    x.npair = ctx->npair;
    x.Na = A.nstr;
    x.ld = ctx->pl[0].ld[0];
    if (abx_lds(x.ld, rb_of(x.npair)) > 160 * 1024) return false;
    // 32-bit byte offsets of the gathered rows (the zero row Na included) and of the plan
    const uint64_t cpb = (uint64_t(x.Na) + 1) * uint64_t(x.ld) * sizeof(T);
    const uint64_t plb = uint64_t(P.ntile) * 4 * (P.ew + 1) * 64 * sizeof(uint32_t);
    if (cpb >= (uint64_t(1) << 31) || plb >= (uint64_t(1) << 31)) return false;
    x.cp_bytes = uint32_t(cpb);
    x.plan_bytes = uint32_t(plb);
    auto *c = const_cast<cisigma_ctx *>(ctx);
    return dispatch_abx(x, P.ew, s, err, c->last_shape[0], &c->last_kernel[0]);
}

}  // namespace

bool launch_sigma_ab_list(const cisigma_ctx *ctx, const void *cp, void *sp, hipStream_t s, hipError_t *err) {
    return owner_t(ctx, cp, sp, s, err);
}

}  // namespace cis
