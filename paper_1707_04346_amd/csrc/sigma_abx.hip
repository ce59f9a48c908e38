// sigma_abx.hip -- the alpha-beta part sigma_3 (Eq. 8) of one-block (CAS) spaces
// of up to 16 orbitals, in FP64: owner-computes rows (FP32: sigma_abs.hip; up to 10
// orbitals mostly sigma_abl.hip).
//
// One workgroup per output alpha string Ia keeps the whole sigma row of Ia in
// LDS and visits the beta strings in 32-column tiles:
//
//   R(a, Jb)  = C(Ja_a, Jb)        a = the single alpha excitations Ja_a of Ia, plus Ia itself
//   W(kl, Jb) = sum_a A(kl, a) R(a, Jb),  A(kl, a) = s_a (i_a j_a|kl),  A(kl, Ia) = sum_{j in Ia} (jj|kl)
//
// Ia's own row either takes a k slot of the matrix product (SELF) or, when the
// excitations alone fill whole k steps, starts the accumulators as the rank-1
// term A(kl, Ia) C(Ia, Jb) (one k step fewer: 16 instead of 17 at CAS(16,16)).
//   sigma(Ia, Ib) += sum_{(kl, Jb): Ib = E_kl Jb} <Ib|E_kl|Jb> W(kl, Jb)
//
// (kl runs over unordered pairs k >= l: E_kl and E_lk share the integral.)
// The gathered rows R are coalesced row reads of C; W comes from the matrix
// cores; the beta-side scatter stays in LDS, so no global atomics are made and
// every sigma row is written once.  The scatter is the program of rounds of
// scatter_prog.h, the same words as in FP32 (offsets doubled).
//
// What bounds it: the FP64 matrix instructions.  A 16x16x4 one holds its SIMD for
// 64 cycles and lets no vector instruction of any wave of that SIMD issue meanwhile,
// so products and scatter add up whatever wave runs them; what can be shaped is how
// evenly the four SIMDs are loaded.  W's rows are therefore dealt in quads of four:
// four quads are one 16x16x4 instruction per k step, a single quad one 4x4x4
// (four blocks, all columns of the half tile: the same operand registers of C, a
// quarter of the time).  A pair of waves w, w + 4 shares a SIMD (wave w is placed on
// SIMD w mod 4); every SIMD gets half the quads of one 16-column half.  At CAS(16,16)
// that is 4.25 blocks per SIMD and k step where whole 16-row blocks on three SIMDs, the
// fourth scattering alone, took 6.
//
// A vector instruction between two matrix ones costs their SIMD ~12 cycles besides its
// own.  From 13 orbitals on scatter and products are therefore kept apart: per tile the
// eight waves scatter, meet, multiply the next tile's rows, and store each its W as soon
// as it is done.  CAS(16,16): 51.5 ms; with four waves scattering beside the products of
// the other four 54.2, with the stores between two barriers at the end 58.0; 15 orbitals
// 11.7 against 12.3, 14 2.94 both, 13 0.57 against 0.67.  Up to 12 orbitals two workgroups
// share a compute unit either way, the one's products fill the other's waits, and the
// fewer partial sums of four scattering waves count: CAS(12,12) 286 us a sigma, 291 with
// all eight.
//
// CAS(16,16) sigma_3 64.1 -> 51.5 ms (the products alone 42.6, their instructions 39, the
// stores of W 1.7), a whole sigma of CAS(12,12) 472 -> 286 us.
#include "internal.h"
#include "mfma.h"
#include "bufio.h"
#include "scatter_prog_dev.h"
#include "slices.h"

#include <algorithm>

namespace cis {
namespace {

constexpr int kNT = 32;      // tile columns
constexpr int kWS = 36;      // W row stride (the scatter program's)

struct AbxArgs {
    const double *cp;        // C, alpha-major padded (row stride ld); row Na is zero
    double *sp;              // sigma accumulator, same layout (read, then overwritten)
    const uint32_t *aexc;    // [Na][anexc]
    const uint32_t *astr;    // [Na]
    const double *gp;        // [n*n][kp]
    const uint32_t *plan;    // [ntile][4 waves][words][64 lanes]
    uint32_t cp_bytes, plan_bytes;   // < 2^31
    int anexc, n, kp, npair, Na, ld;
    int ntile;               // tiles with a beta string (rows are padded to 64 columns)
    double *part;            // [slices - 1][Na][ld]: the sums of the later slices of the tiles
    size_t part_bytes;       // (host)
};

// Quads of wave group g (waves 2g and 2g + 1: the two column halves) of q in all.
// Groups g and g + 2 share SIMDs: half the quads each pair, whole 16-row blocks to
// the first (a little more than half of them).
constexpr int group_quads(int q, int g) {
    const int s = (g & 1) ? q / 2 : (q + 1) / 2;
    const int a = 4 * ((s + 9) / 8), b = 4 * (s / 4);
    const int first = a < b ? a : b;
    return g < 2 ? first : s - first;
}
constexpr int group_quad0(int q, int g) { return g == 0 ? 0 : group_quad0(q, g - 1) + group_quads(q, g - 1); }

// A(m, Ia) = sum_{j in Ia} (jj|kl) for the kl pair of row m
__device__ __forceinline__ double self_coef(const AbxArgs &p, uint32_t xa, int m) {
    double val = 0;
    for (uint32_t b = xa; b; b &= b - 1) {
        const int j = __ffs(b) - 1;
        val += p.gp[int64_t(j * p.n + j) * p.kp + m];
    }
    return val;
}

// One wave: KS k steps of four gathered rows, NQ quads of W rows from row m0 on,
// column half cb; rounds R0 .. R1 - 1 of scatter quarter sw.  A wave without rounds
// meets the scattering ones ("W of this tile consumed") half way through its products.
template <int KS, int NQ, int RB, int PG, bool SELF, bool SL, int R0, int R1>
__device__ __forceinline__ void abx_body(const AbxArgs &p, int Ia, int cb, int m0, int sw, int lane) {
    constexpr int NB = NQ / 4, NS = NQ % 4, NF = NB + NS > 0 ? NB + NS : 1;   // whole blocks, single quads, fragments
    constexpr uint32_t SC = 16 * RB * kWS * 8u, SIG = SC + kProgWaves * 64 * 8u;
    const int lr = lane & 15, lk = lane >> 4;
    const uint32_t xa = p.astr[Ia];
    const uint32_t col = uint32_t(cb * 16 + lr);
    // fragment f, lane: row m0 + 16 f + lane % 16 of a block; of a single quad row
    // lane % 4 of it (repeated for the four column blocks); k = 4t + lane / 16
    auto row_a = [&](int f) { return f < NB ? m0 + 16 * f + lr : m0 + 16 * NB + 4 * (f - NB) + (lane & 3); };
    double A[NF][KS];
    uint32_t boff[KS];
#pragma unroll
    for (int t = 0; t < KS; ++t) {
        const int k = 4 * t + lk;
        int J = p.Na;
        const double *g = nullptr;
        double sg = 0;
        if (k < p.anexc) {
            const uint32_t e = p.aexc[int64_t(Ia) * p.anexc + k];
            if (e != kExcNone) {
                J = int(e >> 11);
                const int i = (e >> 6) & 31, j = (e >> 1) & 31;   // <Ia|E_ij|Ja>, Ja = Ia - i + j
                g = p.gp + int64_t(i * p.n + j) * p.kp;
                sg = (e & 1) ? -1.0 : 1.0;
            }
        } else if (SELF && k == p.anexc) {
            J = Ia;
        }
        boff[t] = (uint32_t(J) * uint32_t(p.ld) + col) * 8u;   // < cp_bytes
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int m = row_a(f);
            double val = 0;
            if (f < NB + NS && m < p.npair) {
                if (g) val = sg * g[m];
                else if (SELF && k == p.anexc) val = self_coef(p, xa, m);
            }
            A[f][t] = val;
        }
    }
    // without SELF: A(m, Ia) of the lane's accumulator rows
    double dB[NB > 0 ? NB : 1][4] = {}, dQ[NS > 0 ? NS : 1] = {};
    uint32_t boffI = 0;
    if constexpr (!SELF) {
#pragma unroll
        for (int f = 0; f < NB; ++f)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = m0 + 16 * f + Mfma<double>::out_row(lane, i);
                dB[f][i] = m < p.npair ? self_coef(p, xa, m) : 0.0;
            }
#pragma unroll
        for (int f = 0; f < NS; ++f) {
            const int m = m0 + 16 * NB + 4 * f + lk;
            dQ[f] = m < p.npair ? self_coef(p, xa, m) : 0.0;
        }
        boffI = (uint32_t(Ia) * uint32_t(p.ld) + col) * 8u;   // < cp_bytes
    }
    int ntile = p.ntile;
    const double *cp = p.cp;
    const uint32_t *plan = p.plan;
    uint32_t cp_bytes = p.cp_bytes, plan_bytes = p.plan_bytes;
    if constexpr (SL) {                  // from this slice's first tile on
        const SliceTiles sl(ntile);
        const uint32_t poff = uint32_t(sl.t0) * uint32_t(kProgWaves * ProgWords<double, PG, R0, R1>::NW * 64);
        ntile = sl.t1 - sl.t0;
        cp += sl.t0 * kNT;
        cp_bytes -= uint32_t(sl.t0) * (kNT * 8u);
        plan += poff;
        plan_bytes -= poff * 4u;
    }
    const __amdgpu_buffer_rsrc_t cr = buffer_of(cp, cp_bytes);
    const __amdgpu_buffer_rsrc_t pr = buffer_of(plan, plan_bytes);
    double b[KS], cI = 0;
    doublex4 acc[NB > 0 ? NB : 1];
    double accq[NS > 0 ? NS : 1];
    // W of the rows held in b; as each k step is consumed, b[t] is reloaded with the
    // rows of tile `next`, so the loads stay in flight for a whole tile
    auto products = [&](int next, bool meet) {
        const uint32_t so = uint32_t(next) * (kNT * 8u);
        if constexpr (SELF) {
#pragma unroll
            for (int f = 0; f < NB; ++f) acc[f] = doublex4{0, 0, 0, 0};
#pragma unroll
            for (int f = 0; f < NS; ++f) accq[f] = 0;
        } else {
#pragma unroll
            for (int f = 0; f < NB; ++f) acc[f] = doublex4{dB[f][0] * cI, dB[f][1] * cI, dB[f][2] * cI, dB[f][3] * cI};
#pragma unroll
            for (int f = 0; f < NS; ++f) accq[f] = dQ[f] * cI;
            buffer_ld(cI, cr, boffI, so);
        }
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            if (meet && t == KS / 2) lds_barrier();
#pragma unroll
            for (int f = 0; f < NB; ++f) acc[f] = Mfma<double>::op(A[f][t], b[t], acc[f]);
#pragma unroll
            for (int f = 0; f < NS; ++f) accq[f] = mfma_quad(A[NB + f][t], b[t], accq[f]);
            buffer_ld(b[t], cr, boff[t], so);
            __builtin_amdgcn_sched_barrier(0);   // keep the reload next to its k step
        }
    };
    auto store_w = [&]() {
        const uint32_t o = uint32_t((m0 + lk) * kWS + int(col)) * 8u;
#pragma unroll
        for (int f = 0; f < NB; ++f)
#pragma unroll
            for (int i = 0; i < 4; ++i) lds_st<double>(o + uint32_t((16 * f + 4 * i) * kWS) * 8u, acc[f][i]);
#pragma unroll
        for (int f = 0; f < NS; ++f) lds_st<double>(o + uint32_t((16 * NB + 4 * f) * kWS) * 8u, accq[f]);
    };
    // this wave's part of a tile's groups: the words, then their sums
    ProgWords<double, PG, R0, R1> pw;
    const uint32_t pl = uint32_t(sw * pw.NW * 64 + lane) * 4u, mine = uint32_t(sw * 64 + lane) * 8u;
#pragma unroll
    for (int t = 0; t < KS; ++t) buffer_ld(b[t], cr, boff[t], 0u);
    if constexpr (!SELF) buffer_ld(cI, cr, boffI, 0u);
    if constexpr (R0 < R1) pw.load(pr, pl, 0);
    products(ntile > 1 ? 1 : 0, false);
    lds_barrier();                       // the sigma row and the zeros of W's pad columns are in LDS
    store_w();
    lds_barrier();                       // W of tile 0 ready
    for (int tile = 0; tile + 1 < ntile; ++tile) {
        if constexpr (R0 < R1) {
            // beside the products of other waves: first (CAS(12,12) 287 us, without 291)
            constexpr bool BESIDE = R0 == 0 && R1 == kProgs[PG].nr;
            if constexpr (BESIDE) __builtin_amdgcn_s_setprio(3);
            prog_run<SC, SIG>(pw, mine);
            pw.load(pr, pl, tile + 1);
            if constexpr (BESIDE) __builtin_amdgcn_s_setprio(0);
            lds_barrier();               // W of this tile consumed
        }
        products(tile + 2 < ntile ? tile + 2 : ntile - 1, R0 == R1);
        store_w();
        lds_barrier();                   // W of the next tile ready
    }
    prog_run<SC, SIG>(pw, mine);
}

// KS: k steps (4*KS >= excitations, plus one with SELF); Q: quads of W rows (4*Q >=
// npair); RB: 16-row blocks that the program's W has room for; PG: program
template <int KS, int Q, int RB, int PG, bool SELF, bool SL>
__global__ __launch_bounds__(512, 2) void k_sigma_ab_x(AbxArgs p) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double *W = reinterpret_cast<double *>(smem_raw);      // [16 RB][kWS], then the waves' scratch
    double *sig = W + 16 * RB * kWS + kProgWaves * 64;     // [ld + 64]: slots ld.. take discarded writes
    const int Ia = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = wave >> 1, cb = wave & 1;
    // the first slice adds to the sigma row, the others to zeros
    double *row = SL ? slice_row(p.sp, p.part, Ia, p.Na, p.ld) : p.sp + int64_t(Ia) * p.ld;
    for (int c = tid * 2; c < p.ld; c += 1024)
        *reinterpret_cast<double2_t *>(sig + c) =
            !SL || blockIdx.y == 0 ? *reinterpret_cast<const double2_t *>(row + c) : double2_t{0, 0};
    for (int r = tid; r < 16 * RB; r += 512) W[r * kWS + kNT] = 0.0;   // pad column: unused references read it
    static_assert(group_quad0(Q, 3) + group_quads(Q, 3) == Q && 4 * Q <= 16 * RB, "every quad has a wave");
    constexpr int NR = kProgs[PG].nr;
    const int sw = wave & 3;
    // all waves scatter, w and w + 4 the first round and the others of a quarter, or
    // waves 4 to 7 do, beside the products of the others (see above)
    constexpr int LO = RB > 5 ? 1 : 0;
    if (g == 0) abx_body<KS, group_quads(Q, 0), RB, PG, SELF, SL, 0, LO>(p, Ia, cb, 0, sw, lane);
    else if (g == 1) abx_body<KS, group_quads(Q, 1), RB, PG, SELF, SL, 0, LO>(p, Ia, cb, 4 * group_quad0(Q, 1), sw, lane);
    else if (g == 2) abx_body<KS, group_quads(Q, 2), RB, PG, SELF, SL, LO, NR>(p, Ia, cb, 4 * group_quad0(Q, 2), sw, lane);
    else abx_body<KS, group_quads(Q, 3), RB, PG, SELF, SL, LO, NR>(p, Ia, cb, 4 * group_quad0(Q, 3), sw, lane);
    __syncthreads();
    for (int c = tid * 2; c < p.ld; c += 1024)
        *reinterpret_cast<double2_t *>(row + c) = *reinterpret_cast<const double2_t *>(sig + c);
}

size_t abx_lds(int ld, int rb) { return (size_t(16) * rb * kWS + kProgWaves * 64 + ld + 64) * sizeof(double); }

// (the slices in a kernel of their own: their bounds cost the others 1 to 4%)
template <int KS, int Q, int RB, int PG, bool SELF, bool SL>
hipError_t run_abx_sl(const AbxArgs &a, int ns, hipStream_t s) {
    const size_t lds = abx_lds(a.ld, RB);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_sigma_ab_x<KS, Q, RB, PG, SELF, SL>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_sigma_ab_x<KS, Q, RB, PG, SELF, SL>), dim3(a.Na, ns), dim3(512), lds, s, a);
    return add_slices<double>(a.sp, a.part, int64_t(a.Na) * a.ld, ns, s);
}

template <int KS, int Q, int RB, int PG, bool SELF>
hipError_t run_abx(const AbxArgs &a, hipStream_t s) {
    if (4 * Q < a.npair || 4 * KS < a.anexc + (SELF ? 1 : 0)) return hipErrorInvalidValue;
    const int ns = slices(a.Na, a.ntile, a.ld, sizeof(double), a.part_bytes, kPlaces64);
    return ns > 1 ? run_abx_sl<KS, Q, RB, PG, SELF, true>(a, ns, s) : run_abx_sl<KS, Q, RB, PG, SELF, false>(a, 1, s);
}

// Compiled (KS, Q, RB, program), by ascending KS: for each RB = ceil(n(n+1)/32) the
// quads of the largest n, the k steps of the half-filled spaces (and, for the larger
// n, of the low fillings), and the programs of the FP32 kernel's table.
#define CIS_ABX_SHAPES(X) \
    X(2, 4, 1, 0) X(3, 7, 2, 0) X(4, 7, 2, 0) X(4, 12, 3, 0) X(4, 12, 3, 1) X(6, 12, 3, 0) X(6, 12, 3, 1) \
    X(4, 14, 4, 0) X(4, 14, 4, 1) X(7, 14, 4, 0) X(7, 14, 4, 1) \
    X(5, 20, 5, 1) X(5, 20, 5, 4) X(8, 17, 5, 1) X(8, 17, 5, 4) X(9, 20, 5, 1) X(9, 20, 5, 4) \
    X(8, 23, 6, 2) X(8, 23, 6, 4) X(11, 23, 6, 2) X(11, 23, 6, 4) \
    X(9, 27, 7, 2) X(9, 27, 7, 4) X(13, 27, 7, 2) X(13, 27, 7, 4) \
    X(10, 30, 8, 3) X(10, 30, 8, 4) X(15, 30, 8, 3) X(15, 30, 8, 4) \
    X(10, 34, 9, 3) X(10, 34, 9, 4) X(16, 34, 9, 3) X(16, 34, 9, 4)
// With Ia's row as the rank-1 start of the accumulators, where the excitations
// fill the k steps: 8, 12 and 16 half-filled orbitals.
#define CIS_ABX_SHAPES_R1(X) \
    X(4, 12, 3, 0) X(4, 12, 3, 1) X(9, 20, 5, 1) X(9, 20, 5, 4) X(16, 34, 9, 3) X(16, 34, 9, 4)

// Size classes of one-block spaces: k steps of four gathered rows, row blocks and the
// entries per lane of a scatter plan in equal runs, by the spaces CAS(n, n/2) and their
// open-shell neighbours.  Up to 10 orbitals they are the list kernel's compiled shapes
// (sigma_abl.hip); for the others they only say how large a space is.
#define CIS_ABX_NAMES(X)                                                                               \
    X(2, 1, 2) X(2, 1, 16) X(3, 2, 2) X(3, 2, 16) X(4, 2, 4) X(4, 2, 16) X(4, 3, 4) X(4, 3, 16)         \
    X(5, 3, 4) X(5, 3, 16) X(6, 3, 4) X(6, 3, 16) X(6, 4, 4) X(6, 4, 16) X(7, 4, 4) X(7, 4, 16)         \
    X(8, 5, 6) X(8, 5, 16) X(10, 5, 6) X(10, 5, 16) X(11, 6, 8) X(11, 6, 16) X(13, 7, 8) X(13, 7, 16)   \
    X(15, 8, 10) X(15, 8, 16) X(17, 9, 10) X(17, 9, 16)
// Those whose excitations fill the k steps.
#define CIS_ABX_NAMES_R1(X)                                                                            \
    X(1, 1, 2) X(1, 1, 16) X(2, 2, 2) X(2, 2, 16) X(4, 3, 4) X(4, 3, 16) X(6, 4, 4) X(6, 4, 16)         \
    X(9, 5, 6) X(9, 5, 16) X(12, 7, 8) X(12, 7, 16) X(16, 9, 10) X(16, 9, 16)

int ks_of(int anexc) { return (anexc + 1 + 3) / 4; }
int rb_of(int npair) { return (npair + 15) / 16; }

}  // namespace

int sigma_ab_owner_width(int anexc, int npair, int need) {
    const int ks = ks_of(anexc), rb = rb_of(npair);
    int best = 0;
#define CIS_W(K, R, E) if (ks == K && rb == R && E >= need && (best == 0 || E < best)) best = E;
    CIS_ABX_NAMES(CIS_W)
#undef CIS_W
    return best;
}

void sigma_ab_owner_shape(int anexc, int npair, int ew, int *shape) {
    const int rb = rb_of(npair);
    shape[0] = ks_of(anexc);
    shape[1] = rb;
    shape[2] = ew;
    shape[3] = 1;
#define CIS_R1(K, R, E) if (anexc == 4 * K && rb == R && ew == E) { shape[0] = K; shape[3] = 2; }
    CIS_ABX_NAMES_R1(CIS_R1)
#undef CIS_R1
}

bool launch_sigma_ab_owner(const cisigma_ctx *ctx, const void *cp, void *sp, const AbScratch &scratch, hipStream_t s,
                           hipError_t *err) {
    if (launch_sigma_ab_list(ctx, cp, sp, s, err)) return true;
    const ProgPlan &P = ctx->prog;
    if (!P.d_words) return false;
    const auto &A = ctx->sp[0];
    AbxArgs x{};
    x.cp = static_cast<const double *>(cp);
    x.sp = static_cast<double *>(sp);
    x.aexc = A.d_exc;
    x.astr = A.d_str;
    x.gp = ctx->d_gp64;
    x.plan = P.d_words;
    x.part = static_cast<double *>(scratch.p);
    x.part_bytes = scratch.bytes;
    x.anexc = A.nexc;
    x.n = ctx->n;
    x.kp = ctx->kp;
    x.npair = ctx->npair;
    x.Na = A.nstr;
    x.ld = ctx->pl[0].ld[0];
    x.ntile = (ctx->sp[1].nstr + kNT - 1) / kNT;
    const int rb = rb_of(x.npair);
    if (abx_lds(x.ld, rb) > 160 * 1024) return false;
    // 32-bit byte offsets of the gathered rows (the zero row Na included) and of the plan
    const uint64_t cpb = (uint64_t(x.Na) + 1) * uint64_t(x.ld) * sizeof(double);
    const uint64_t plb = uint64_t(P.ntile) * kProgWaves * kProgs[P.prog].words() * 64 * sizeof(uint32_t);
    if (cpb >= (uint64_t(1) << 31) || plb >= (uint64_t(1) << 31)) return false;
    x.cp_bytes = uint32_t(cpb);
    x.plan_bytes = uint32_t(plb);
    const char *ran = nullptr;
#define CIS_RUN1(K, Q, R, G)                                                                   \
    if (!ran && x.anexc == 4 * K && rb == R && P.prog == G) {                                  \
        *err = run_abx<K, Q, R, G, false>(x, s);                                               \
        ran = "k_sigma_ab_x<" #K ", " #Q ", " #R ", " #G ", rank1>";                           \
    }
    CIS_ABX_SHAPES_R1(CIS_RUN1)
#undef CIS_RUN1
    // the fewest k steps and quads that hold the space
#define CIS_RUN(K, Q, R, G)                                                                    \
    if (!ran && 4 * K >= x.anexc + 1 && 4 * Q >= x.npair && rb == R && P.prog == G) {          \
        *err = run_abx<K, Q, R, G, true>(x, s);                                                \
        ran = "k_sigma_ab_x<" #K ", " #Q ", " #R ", " #G ", self>";                            \
    }
    CIS_ABX_SHAPES(CIS_RUN)
#undef CIS_RUN
    if (!ran) return false;
    auto *c = const_cast<cisigma_ctx *>(ctx);
    for (int i = 0; i < 4; ++i) c->last_shape[0][i] = P.shape[i];
    c->last_kernel[0] = ran;
    return true;
}

}  // namespace cis
