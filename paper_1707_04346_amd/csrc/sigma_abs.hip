// sigma_abs.hip -- the alpha-beta part sigma_3 (Eq. 8) of one-block (CAS) spaces
// of up to 16 orbitals in FP32: owner-computes rows as in sigma_abx.hip, with the
// contraction on the bf16 matrix cores (split.h) and the beta-side scatter as a
// program of rounds (scatter_prog.h).
//
//   W(kl, Jb) = sum_a A(kl, a) C(Ja_a, Jb)                 one 32-column tile at a time
//   sigma(Ia, Ib) += sum_{(kl, Jb): Ib = E_kl Jb} <Ib|E_kl|Jb> W(kl, Jb)
//
// A workgroup of four waves owns one alpha string Ia: its sigma row and one W tile
// in LDS.  Wave (g, cb) holds the split A of half of the 16-row kl blocks in
// registers and multiplies the tile's column half cb; all four then scatter a
// quarter of the tile's groups each.  Between two barriers a wave computes the
// next tile's W in registers and scatters this tile's; two workgroups share a
// compute unit (72 KB of LDS, at most 256 registers), so one's matrix
// instructions run while the other scatters.
//
// What bounds it (CAS(16,16), 21.1 to 21.8 ms; the FP32 instructions took 31.9): 72 matrix
// instructions of 16 cycles and ~170 vector instructions per wave and tile.  Beside
// a matrix instruction about three vector ones issue free of charge; the scatter,
// alone 11 ms (a third of it bank conflicts), hides behind the other workgroup's
// products only in part.  With six products instead of eight 18.6 ms, and single
// products less exact than in FP32 (split.h).  Four waves that multiply and four that
// scatter in one workgroup, with two W tiles, were slower (six products: 22 ms): one
// wave per SIMD does not hide its own latencies.
//
// A C with elements outside the split's range (infinities, NaN, tiny or huge ones:
// split.h) is multiplied by the FP32 instructions in the same frame, and so is any C
// where integrals are (CAS(16,16) 29.8 instead of 21.8 ms, CAS(12,12) 130 us instead of
// 108).  The kernel that copies C in looks at its elements on the way, which its memory
// traffic hides, and leaves the answer in p.wide.
#include "internal.h"
#include "bufio.h"
#include "scatter_prog_dev.h"
#include "slices.h"
#include "split.h"

#include <algorithm>
#include <cmath>

namespace cis {
namespace {

constexpr int kNT = 32;      // tile columns
constexpr int kWS = 36;      // W row stride: 16-byte rows, a lane's four columns in one store

struct AbsArgs {
    const float *cp;         // C, alpha-major padded (row stride ld); row Na is zero
    float *sp;               // sigma accumulator, same layout (read, then overwritten)
    const uint32_t *aexc;    // [Na][anexc]
    const uint32_t *astr;    // [Na]
    const float *gp;         // [n*n][kp]
    const uint32_t *plan;    // [ntile][4 waves][words][64 lanes]
    float *part;             // [slices - 1][Na][ld]: the sums of the later slices of the tiles
    const int *wide;         // nonzero: C has elements outside the split's range
    int exact;               // nonzero: the integrals have
    size_t part_bytes;       // (host)
    uint32_t cp_bytes, plan_bytes;   // < 2^31
    int anexc, n, kp, npair, Na, ld;
    int ntile;               // tiles with a beta string (rows are padded to 64 columns)
};

// sum_{j in Ia} (jj|kl) for the kl pair of row m < npair: all loads at once
__device__ __forceinline__ float self_coef(const AbsArgs &p, uint32_t xa, int m) {
    float x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = p.gp[(j < p.n ? j * p.n + j : 0) * p.kp + m];
    float val = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) val += (xa >> j) & 1u ? x[j] : 0.0f;
    return val;
}

// KS: 32-row steps over the gathered rows; NR: row blocks of this wave, from rb0;
// SELF: Ia's own row takes a slot of the steps, else it is added in FP32 (rank 1);
// EX: products by the FP32 instruction
template <int KS, int NR, int RB, int PG, bool SELF, bool EX>
__device__ __forceinline__ void abs_body(const AbsArgs &p, float *W, int Ia, int cb, int rb0, int wave, int lane) {
    constexpr int NRA = NR > 0 ? NR : 1;
    constexpr int MP = 16 * RB;
    const int lr = lane & 15, lk = lane >> 4;
    const uint32_t xa = p.astr[Ia];
    // gathered rows of this lane: k = 32 s + 8 (lane / 16) + j
    Split8 A[EX ? 1 : NRA][EX ? 1 : KS];
    float A32[EX ? NRA : 1][EX ? KS : 1][8];
    uint32_t boff[KS][8];
    const uint32_t col = uint32_t(cb * 16 + lr);
    // (without branches, so that the loads are in flight together: CAS(12,12) 107 -> 103 us,
    // 8 alpha and 1 beta electrons in 16 orbitals, a tile a workgroup, 476 -> 397)
    uint32_t ex[KS][8];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = 32 * s + 8 * lk + j;
            ex[s][j] = kExcNone;
            if (p.anexc > 0) {                     // (uniform)
                const uint32_t e = p.aexc[int64_t(Ia) * p.anexc + (k < p.anexc ? k : 0)];
                if (k < p.anexc) ex[s][j] = e;
            }
        }
    float self[NRA];
#pragma unroll
    for (int r = 0; r < NRA; ++r) {
        const int m = (rb0 + r) * 16 + lr;
        const float v = self_coef(p, xa, m < p.npair ? m : 0);
        self[r] = r < NR && m < p.npair ? v : 0.0f;
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        float a[NRA][8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = 32 * s + 8 * lk + j;
            const uint32_t e = ex[s][j];
            const bool ok = e != kExcNone, own = SELF && k == p.anexc;
            const int i = (e >> 6) & 31, jj = (e >> 1) & 31;   // <Ia|E_ij|Ja>, Ja = Ia - i + j
            const int g = ok ? (i * p.n + jj) * p.kp : 0;
            const int J = ok ? int(e >> 11) : own ? Ia : p.Na;
            boff[s][j] = (uint32_t(J) * uint32_t(p.ld) + col) * 4u;   // < cp_bytes
#pragma unroll
            for (int r = 0; r < NRA; ++r) {
                const int m = (rb0 + r) * 16 + lr;
                const bool row = r < NR && m < p.npair;
                const float v = p.gp[g + (row ? m : 0)];
                a[r][j] = ok && row ? ((e & 1) ? -v : v) : own ? self[r] : 0.0f;
            }
        }
#pragma unroll
        for (int r = 0; r < NRA; ++r) {
            if constexpr (EX) {
#pragma unroll
                for (int j = 0; j < 8; ++j) A32[r][s][j] = a[r][j];
            } else {
                A[r][s] = split_round(a[r]);
            }
        }
    }
    uint32_t boffI = 0;
    if constexpr (!SELF) boffI = (uint32_t(Ia) * uint32_t(p.ld) + uint32_t(cb * 16 + 4 * lk)) * 4u;
    // from this slice's first tile on
    const SliceTiles sl(p.ntile);
    const int ntile = sl.t1 - sl.t0;
    const uint32_t coff = uint32_t(sl.t0) * kNT, poff = uint32_t(sl.t0) * uint32_t(kProgWaves * ProgWords<float, PG>::NW * 64);
    const __amdgpu_buffer_rsrc_t cr = buffer_of(p.cp + coff, p.cp_bytes - coff * 4u);
    const __amdgpu_buffer_rsrc_t pr = buffer_of(p.plan + poff, p.plan_bytes - poff * 4u);
    float b[KS][8];
    bf_floatx4 cI{}, cN{};
    floatx4 acc[NRA];
    auto load_step = [&](int s, uint32_t so) {
#pragma unroll
        for (int j = 0; j < 8; ++j) buffer_ld(b[s][j], cr, boff[s][j], so);
    };
    auto load_self = [&](uint32_t so) {
        if constexpr (!SELF) {
            cI = cN;
            buffer_ld(cN, cr, boffI, so);
        }
    };
    // W of the rows held in b, then the rows of tile `next` into b.  D[Jb][kl]:
    // a lane ends with four columns Jb of one kl row.
    auto products_split = [&](uint32_t so) {
        bf16x8 h[KS];
        Split8 c[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            c[s] = split_round(b[s]);
            load_step(s, so);
        }
        load_self(so);
#pragma unroll
        for (int r = 0; r < NRA; ++r) acc[r] = floatx4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            h[s] = c[s].h;
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(c[s].l, A[r][s].m, acc[r]);
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(c[s].m, A[r][s].l, acc[r]);
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(c[s].l, A[r][s].h, acc[r]);
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(c[s].h, A[r][s].l, acc[r]);
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(c[s].m, A[r][s].m, acc[r]);
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(c[s].h, A[r][s].m, acc[r]);
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(c[s].m, A[r][s].h, acc[r]);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] = mfma_bf16(h[s], A[r][s].h, acc[r]);
    };
    // the same layouts: four rows k = 32 s + 8 (lane / 16) + j per instruction
    auto products_fp32 = [&](uint32_t so) {
#pragma unroll
        for (int r = 0; r < NRA; ++r) acc[r] = floatx4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int r = 0; r < NR; ++r) acc[r] = Mfma<float>::op(b[s][j], A32[r][s][j], acc[r]);
            load_step(s, so);
        }
        load_self(so);
    };
    auto products = [&](int next) {
        const uint32_t so = uint32_t(next) * (kNT * 4u);
        if constexpr (EX) products_fp32(so);
        else products_split(so);
    };
    auto store_w = [&]() {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            floatx4 v = acc[r];
            if constexpr (!SELF)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = __builtin_fmaf(self[r], cI[i], v[i]);
            *reinterpret_cast<floatx4 *>(W + ((rb0 + r) * 16 + lr) * kWS + cb * 16 + 4 * lk) = v;
        }
    };
    // this wave's quarter of a tile's groups: the words, then their sums
    ProgWords<float, PG> pw;
    const uint32_t pl = uint32_t(wave * pw.NW * 64 + lane) * 4u, mine = uint32_t(wave * 64 + lane) * 4u;
    constexpr uint32_t SC = MP * kWS * 4u, SIG = SC + kProgWaves * 64 * 4u;
    auto plan_load = [&](int tile) { pw.load(pr, pl, tile); };
    auto scatter = [&]() { prog_run<SC, SIG>(pw, mine); };
#pragma unroll
    for (int s = 0; s < KS; ++s) load_step(s, 0u);
    if constexpr (!SELF) buffer_ld(cN, cr, boffI, 0u);
    plan_load(0);
    products(ntile > 1 ? 1 : 0);
    lds_barrier();                       // the sigma row and the zeros of W's pad columns are in LDS
    store_w();
    lds_barrier();                       // W of tile 0 ready
    for (int tile = 0; tile + 1 < ntile; ++tile) {
        products(tile + 2 < ntile ? tile + 2 : ntile - 1);
        __builtin_amdgcn_sched_barrier(0);   // (mixed into the products the scatter is slower; with six products 19.1 against 18.4 ms)
        scatter();
        plan_load(tile + 1);
        lds_barrier();                   // W of this tile consumed
        store_w();
        lds_barrier();                   // W of the next tile ready
    }
    scatter();
}

template <int KS, int RB, int PG, bool SELF>
__global__ __launch_bounds__(256, 2) void k_sigma_ab_s(AbsArgs p) {
    constexpr int MP = 16 * RB;
    constexpr int R0 = (RB + 1) / 2, R1 = RB - R0;         // row blocks of the two wave pairs
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float *W = reinterpret_cast<float *>(smem_raw);        // [MP][kWS], then the waves' scratch
    float *sig = W + MP * kWS + kProgWaves * 64;           // [ld + 64]: slots ld.. take discarded writes
    const int Ia = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wide = *p.wide;                              // (in flight while the row is read)
    // the first slice adds to the sigma row, the others to zeros
    float *row = slice_row(p.sp, p.part, Ia, p.Na, p.ld);
    for (int c = tid * 4; c < p.ld; c += 1024)
        *reinterpret_cast<floatx4 *>(sig + c) =
            blockIdx.y == 0 ? *reinterpret_cast<const floatx4 *>(row + c) : floatx4{0, 0, 0, 0};
    for (int r = tid; r < MP; r += 256) W[r * kWS + kNT] = 0.0f;   // pad column: unused references read it
    if (p.exact | __builtin_amdgcn_readfirstlane(wide)) {   // one answer for the whole launch
        if (wave < 2) abs_body<KS, R0, RB, PG, SELF, true>(p, W, Ia, wave & 1, 0, wave, lane);
        else abs_body<KS, R1, RB, PG, SELF, true>(p, W, Ia, wave & 1, R0, wave, lane);
    } else {
        if (wave < 2) abs_body<KS, R0, RB, PG, SELF, false>(p, W, Ia, wave & 1, 0, wave, lane);
        else abs_body<KS, R1, RB, PG, SELF, false>(p, W, Ia, wave & 1, R0, wave, lane);
    }
    __syncthreads();
    for (int c = tid * 4; c < p.ld; c += 1024)
        *reinterpret_cast<floatx4 *>(row + c) = *reinterpret_cast<const floatx4 *>(sig + c);
}

size_t abs_lds(int ld, int rb) { return (size_t(16) * rb * kWS + kProgWaves * 64 + ld + 64) * sizeof(float); }

// alone: pad the LDS so that a compute unit holds one workgroup
template <int KS, int RB, int PG, bool SELF>
hipError_t run_abs(const AbsArgs &a, hipStream_t s, bool alone) {
    size_t lds = abs_lds(a.ld, RB);
    if (alone) lds = std::max<size_t>(lds, 81 * 1024);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_sigma_ab_s<KS, RB, PG, SELF>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        if (e != hipSuccess) return e;
    }
    const int ns = slices(a.Na, a.ntile, a.ld, sizeof(float), a.part_bytes, kPlaces32);
    hipLaunchKernelGGL((k_sigma_ab_s<KS, RB, PG, SELF>), dim3(a.Na, ns), dim3(256), lds, s, a);
    return add_slices<float>(a.sp, a.part, int64_t(a.Na) * a.ld, ns, s);
}

// Compiled (KS, RB, program): a space of n orbitals has RB = ceil(n(n+1)/32) and
// KS = 1 while its alpha excitations and own row fit 32 rows (always up to 10
// orbitals), else 2.  Two programs per size: the one CAS(n, n/2) needs and the one
// every filling fits.
#define CIS_ABS_SHAPES(X) \
    X(1, 1, 0) X(1, 2, 0) X(1, 3, 0) X(1, 3, 1) X(1, 4, 0) X(1, 4, 1) \
    X(1, 5, 1) X(1, 5, 4) X(2, 5, 1) X(2, 5, 4) X(1, 6, 2) X(1, 6, 4) X(2, 6, 2) X(2, 6, 4) \
    X(1, 7, 2) X(1, 7, 4) X(2, 7, 2) X(2, 7, 4) X(1, 8, 3) X(1, 8, 4) X(2, 8, 3) X(2, 8, 4) \
    X(1, 9, 3) X(1, 9, 4) X(2, 9, 3) X(2, 9, 4)

}  // namespace

bool sigma_ab_split_prog(int rb, int prog) {
#define CIS_HAS(K, R, P) if (rb == R && prog == P) return true;
    CIS_ABS_SHAPES(CIS_HAS)
#undef CIS_HAS
    return false;
}

bool split_integrals_exact(const std::vector<float> &g) {
    for (float v : g)
        if (v != 0.0f && !(std::fabs(v) >= kSplitMinA && std::fabs(v) < kSplitMax)) return false;
    return true;
}

bool launch_sigma_ab_split(const cisigma_ctx *ctx, const void *cp, void *sp, const int *wide, const AbScratch &scratch,
                           hipStream_t s, hipError_t *err) {
    const ProgPlan &P = ctx->prog;
    if (!P.d_words || !wide) return false;
    const auto &A = ctx->sp[0];
    AbsArgs x{};
    x.cp = static_cast<const float *>(cp);
    x.sp = static_cast<float *>(sp);
    x.aexc = A.d_exc;
    x.astr = A.d_str;
    x.gp = ctx->d_gp32;
    x.plan = P.d_words;
    x.wide = wide;
    x.part = static_cast<float *>(scratch.p);
    x.part_bytes = scratch.bytes;
    x.exact = ctx->split_exact ? 0 : 1;
    x.anexc = A.nexc;
    x.n = ctx->n;
    x.kp = ctx->kp;
    x.npair = ctx->npair;
    x.Na = A.nstr;
    x.ld = ctx->pl[0].ld[0];
    x.ntile = (ctx->sp[1].nstr + kNT - 1) / kNT;
    const int rb = (x.npair + 15) / 16;
    if (abs_lds(x.ld, rb) > 160 * 1024) return false;
    // 32-bit byte offsets of the gathered rows (the zero row Na included) and of the plan
    const uint64_t cpb = (uint64_t(x.Na) + 1) * uint64_t(x.ld) * sizeof(float);
    const uint64_t plb = uint64_t(P.ntile) * kProgWaves * kProgs[P.prog].words() * 64 * sizeof(uint32_t);
    if (cpb >= (uint64_t(1) << 31) || plb >= (uint64_t(1) << 31)) return false;
    x.cp_bytes = uint32_t(cpb);
    x.plan_bytes = uint32_t(plb);
    const bool alone = ctx->ab_mode == 3;
    const int ks = (x.anexc + 1 + 31) / 32;
    auto *c = const_cast<cisigma_ctx *>(ctx);
    const char *ran = nullptr;
    // 64 excitations (8 of 16 orbitals) fill two steps: the own row as a rank-1 term
    if (x.anexc == 64 && rb == 9) {
        if (P.prog == 3) { *err = run_abs<2, 9, 3, false>(x, s, alone); ran = "k_sigma_ab_s<2, 9, 3, rank1>"; }
        if (P.prog == 4) { *err = run_abs<2, 9, 4, false>(x, s, alone); ran = "k_sigma_ab_s<2, 9, 4, rank1>"; }
    }
#define CIS_RUN(K, R, G) \
    if (!ran && ks == K && rb == R && P.prog == G) {                         \
        *err = run_abs<K, R, G, true>(x, s, alone);                          \
        ran = "k_sigma_ab_s<" #K ", " #R ", " #G ", self>";                  \
    }
    CIS_ABS_SHAPES(CIS_RUN)
#undef CIS_RUN
    if (!ran) return false;
    c->ab_shared = !alone && abs_lds(x.ld, rb) <= 80 * 1024;
    for (int i = 0; i < 4; ++i) c->last_shape[1][i] = P.shape[i];
    c->last_kernel[1] = ran;
    return true;
}

}  // namespace cis
