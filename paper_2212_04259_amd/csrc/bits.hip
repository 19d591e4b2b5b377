// Depth 1 of the skeleton search from bit planes.
//
// With X_a, Y_b, Z_c the bit planes of the categories a < r_X - 1, b < r_Y - 1,
// c < r_Z - 1 (one bit per sample, made for the depth-0 contraction),
//   N_abc = sum over words of popcount(X_a & Y_b & Z_c),
// and the cells of a last category follow from the pairwise tables, which
// depth 0 has formed for every pair of variables (Section IV-B) and are the
// test's marginals N_x+z and N_+yz:
//   N(a, b, last) = N_ab - sum_c N_abc,  N(a, last, z) = N_az - sum_b N_abz,
//   N(last, y, z) = N_yz - sum_a N_ayz.
// (r_X - 1)(r_Y - 1)(r_Z - 1) ands and popcounts of 32 samples replace one
// LDS increment per sample: 0.5 vector operations per sample at three
// categories, where an increment instruction of a wave takes ~4.7 LDS cycles
// per compute unit, and a test reads (r - 1) / 8 instead of 1 byte per column
// and sample.  All counts are exact.
//
// A pass counts up to kBitUnit consecutive ranks of one edge (one wave): they
// share the planes of X and Y, whose conjunctions are formed once per word.
// The epilogue completes the pass's tables in LDS, one cell per lane,
// sums the statistic over half-waves, and compares it with the two critical
// values beyond which its FP64 decision is certain; between them it is formed
// again in FP64 and compared with the quantile of alpha itself (a tail is
// evaluated only there).
#include <hip/hip_ext.h>

#include <algorithm>

#include "device_ci.h"
#include "gram.h"
#include "kernels.h"

namespace bns {

// Accumulators per lane: conjunctions of X and Y planes times planes of Z.
constexpr int kBitAcc = 64;
constexpr int kBitZ = 16;       // planes of Z per pass at most
constexpr int kBitRow = kBitAcc + 4;  // LDS words per lane: 16-byte aligned, lanes on different banks
constexpr int kBitSlots = 16;   // half-waves of cells per pass at most
constexpr int kBitWords = 448;  // LDS words for a pass's tables and marginals

// Sum over each half-wave (32 lanes), in every lane of it.
BNS_INLINE float half_sum(float v) {
#define BNS_DPP_ADD(ctrl) \
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xf, 0xf, true))
    BNS_DPP_ADD(0xb1);
    BNS_DPP_ADD(0x4e);
    BNS_DPP_ADD(0x141);
    BNS_DPP_ADD(0x140);  // row_mirror
#undef BNS_DPP_ADD
    return v + __shfl_xor(v, 16, 64);
}
BNS_INLINE double half_sum(double v) {
#pragma unroll 1
    for (int off = 1; off < 32; off <<= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Per-wave state of a pass.
struct BitSh {
    uint32_t M[kBitAcc];          // counts N_abc: [plane of Z][b][a]
    uint32_t xy[16];              // N_ab: [b][a]
    double g2[kBitSlots];         // statistic of each half-wave of cells
    double st[kBitUnit];          // statistic of each test
    int32_t df[kBitUnit];
    uint32_t zcat[kBitUnit];      // first category of Z in the pairwise tables
    uint32_t rz[kBitUnit];
    uint32_t zs[kBitUnit];        // first row of the test in M
    uint32_t toff[kBitUnit];      // first word of the test in tab
    uint32_t slot0[kBitUnit];     // first half-wave of the test
    uint32_t zo[kBitZ];           // byte offset of each plane of Z
    uint8_t slot_t[kBitSlots], slot_c[kBitSlots];  // half-wave -> test, first cell / 32
    union {
        alignas(16) uint32_t part[64 * kBitRow];   // each lane's counts, until they are summed into M
        uint32_t tab[kBitWords];                   // then, per test: cells and marginals
    };
};

// Planes read through a buffer descriptor: one scalar byte offset per plane,
// one lane offset for all of them, so an address costs no vector operation.
typedef __amdgpu_buffer_rsrc_t plane_rsrc;
BNS_INLINE u32x4 plane_words(plane_rsrc rs, uint32_t lane_off, uint32_t plane_off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)lane_off, (int)plane_off, 0));
}

// acc + popcount(v) in one instruction (left to itself the compiler counts
// two words and adds both: three instructions for two words).
BNS_INLINE void bcnt_add(uint32_t &acc, uint32_t v) { asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"(v)); }

// Counts of NZ planes of Z (byte offsets zo) against the NX x NY conjunctions
// over n groups of four words per plane.  Every loop is straight-line code (a
// branch per plane made the compiler copy every word of a step); few planes
// take two groups per lane and step, for the loads in flight.
template <int NX, int NY, int NZ>
BNS_INLINE void bit_count(uint32_t *row, plane_rsrc rs, uint32_t xo, uint32_t yo, uint32_t sb,
                          const uint32_t (&zo)[kBitZ], uint32_t n) {
    constexpr int P = NX * NY, L = NX + NY + NZ;
    constexpr int U = L <= 5 ? 2 : 1;
    static_assert(P * NZ <= kBitAcc && NZ <= kBitZ, "accumulators");
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t acc[(P * NZ + 3) / 4 * 4];
#pragma unroll
    for (int k = 0; k < (P * NZ + 3) / 4 * 4; ++k) acc[k] = 0u;
    for (uint32_t w0 = 0; w0 < n; w0 += 64u * U) {  // uniform
        u32x4 x[U][NX], y[U][NY], z[U][NZ];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // (past the end: the last group, with X cleared below)
            const uint32_t o = 16u * min(w0 + 64u * u + lane, n - 1u);
#pragma unroll
            for (int a = 0; a < NX; ++a) x[u][a] = plane_words(rs, o, xo + a * sb);
#pragma unroll
            for (int b = 0; b < NY; ++b) y[u][b] = plane_words(rs, o, yo + b * sb);
#pragma unroll
            for (int k = 0; k < NZ; ++k) z[u][k] = plane_words(rs, o, zo[k]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = w0 + 64u * u + lane < n;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t t[P];
#pragma unroll
                for (int a = 0; a < NX; ++a) {
                    const uint32_t xa = in ? x[u][a][q] : 0u;
#pragma unroll
                    for (int b = 0; b < NY; ++b) t[b * NX + a] = xa & y[u][b][q];
                }
#pragma unroll
                for (int k = 0; k < NZ; ++k)
#pragma unroll
                    for (int p = 0; p < P; ++p) bcnt_add(acc[k * P + p], t[p] & z[u][k][q]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < P * NZ; k += 4) *(u32x4 *)(row + k) = u32x4{acc[k], acc[k + 1], acc[k + 2], acc[k + 3]};
}

// nzp planes of Z, rounded up to the next instance (the planes past nzp
// repeat the first; their counts are not used).
template <int NX, int NY>
BNS_INLINE void bit_count_z(uint32_t *row, plane_rsrc rs, uint32_t xo, uint32_t yo, uint32_t sb,
                            const uint32_t (&zo)[kBitZ], uint32_t n, int nzp) {
    constexpr int ZB = (kBitAcc / (NX * NY)) < kBitZ ? (kBitAcc / (NX * NY)) : kBitZ;
    if (nzp == 1) return bit_count<NX, NY, 1>(row, rs, xo, yo, sb, zo, n);
    if (nzp == 2) return bit_count<NX, NY, 2>(row, rs, xo, yo, sb, zo, n);
    if (nzp <= 4) return bit_count<NX, NY, 4>(row, rs, xo, yo, sb, zo, n);
    if constexpr (ZB > 8) {
        if (nzp <= 8) return bit_count<NX, NY, 8>(row, rs, xo, yo, sb, zo, n);
    }
    if constexpr (ZB > 12) {
        if (nzp <= 12) return bit_count<NX, NY, 12>(row, rs, xo, yo, sb, zo, n);
    }
    if constexpr (ZB > 4) bit_count<NX, NY, ZB>(row, rs, xo, yo, sb, zo, n);
}

// Sum of the lanes' counts: M[k] for k < nm.  2^lg lanes (consecutive values)
// per row slice; slices are combined with lane exchanges.
BNS_INLINE void bit_reduce(BitSh &s, uint32_t nm) {
    const int lane = threadIdx.x & 63;
    int lg = 3;
    while (lg < 6 && (1u << lg) < nm) ++lg;
    const int k = lane & ((1 << lg) - 1), rows = 1 << lg;  // 64 lanes' rows over 64 >> lg slices
    const uint32_t *p = s.part + (lane >> lg) * rows * kBitRow + k;
    uint32_t v = 0;
    for (int r = 0; r < rows; r += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) v += p[(r + u) * kBitRow];
    }
    for (int off = 1 << lg; off < 64; off <<= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
    if ((uint32_t)lane < nm) s.M[lane] = v;
}

// Cell (x, y, z) of lane `cell` of a table of rx by ry strata.
struct BitCell {
    uint32_t x, y, z;
};
BNS_INLINE BitCell bit_cell(uint32_t cell, uint32_t rx, uint32_t ry, float inv_rx, float inv_ry) {
    const uint32_t rho = fast_div(cell, rx, inv_rx);
    const uint32_t z = fast_div(rho, ry, inv_ry);
    return BitCell{cell - rho * rx, rho - z * ry, z};
}

// g2_half_term<float> for products below 2^53 (the path takes fewer than 2^26
// samples), without the 64-bit form for larger ones.
BNS_INLINE float bit_g2_term(uint32_t N, uint32_t nxz, uint32_t nyz, uint32_t nzz) {
    const double a = (double)N * (double)nzz;
    const double b = (double)nxz * (double)nyz;
    const float t = (float)(a - b) * __builtin_amdgcn_rcpf((float)(a + b));
    const float u = t * t;
    float sr = 1.0f / (float)(2 * TermCfg<float>::terms + 1);
#pragma unroll
    for (int k = TermCfg<float>::terms - 1; k >= 1; --k) sr = sr * u + 1.0f / (float)(2 * k + 1);
    const float near = 2.0f * u * __builtin_amdgcn_rcpf(1.0f + t) + 2.0f * t * u * sr;
    const float w = (float)b * __builtin_amdgcn_rcpf((float)a);
    const float far = w - 1.0f - __logf(w);
    const float E = (float)nxz * (float)nyz * __builtin_amdgcn_rcpf((float)nzz);
    return N == 0 ? E : (float)N * (fabsf(t) <= TermCfg<float>::tau ? near : far);
}

// A test that its statistic's critical values leave open: an FP32 statistic is
// formed again in FP64 (in the band or the error bound of alpha: with alpha
// below the band every dependent test), and a tail is evaluated only where the
// FP64 statistic is at the quantile of alpha itself.  Out of line: its code
// would push the counting loops out of the instruction cache.
static __device__ __noinline__ bool bit_near(const uint32_t *tab, uint32_t rx, uint32_t ry, uint32_t rz, double st,
                                             int64_t df, double alpha, double x64, double y64, int stat, bool fp64) {
    if (!fp64) {
        const uint32_t T = rx * ry * rz;
        const float inv_rx = 1.0f / (float)rx, inv_ry = 1.0f / (float)ry;
        double part = 0.0;
        for (uint32_t c = threadIdx.x & 63u; c < T; c += 64u) {
            const BitCell q = bit_cell(c, rx, ry, inv_rx, inv_ry);
            const uint32_t *mz = tab + T + q.z * (rx + ry + 1u);
            const uint32_t nzz = mz[rx + ry];
            if (nzz)
                part += stat ? x2_term<double>(tab[c], mz[q.x], mz[rx + q.y], nzz)
                             : g2_half_term<double>(tab[c], mz[q.x], mz[rx + q.y], nzz);
        }
        part = wave_sum(part);
        st = stat ? part : 2.0 * part;
    }
    if (st < x64) return true;
    if (st > y64) return false;
    return chi2_tail_wave(df, st).p > alpha;
}

// A decoded work unit: ranks r .. r1 - 1 of edge e (depth 1: at most
// 2 (n - 2) ranks, 32 bits).
struct BitItem1 {
    uint32_t e, r, r1, nA;
    int32_t prob, i, j, posj, posi;
};

// One unit: its tests in order, up to kBitUnit per pass (two in the first
// pass of an edge, twice as many in each later one), until the pass with the
// first acceptance.  Returns the first accepting rank (or ~0) and counts the
// tests run and re-checked.
template <bool GENERAL>
BNS_INLINE uint32_t bit_unit(const DepthArgs &A, BitSh &s, const CritVal *crit, const ProbDev &P, const BitProb &B,
                             const BitItem1 &rec, uint32_t &exec, uint32_t &rechecks) {
    const int lane = threadIdx.x & 63;
    const Grp g = Grp::wave();
    const uint32_t e = uni(rec.e), r0 = uni(rec.r), r1 = uni(rec.r1), nA = uni(rec.nA);
    const VarRec *vars = A.bits.var + uni(P.var_off);
    // conditioning variables of 64 ranks from rb on (lane l: rank rb + l)
    VarRec vz{2, 0, 0, 0};
    auto load_z = [&](uint32_t rb) {
        const uint32_t r = rb + (uint32_t)lane;
        if (r < r1) {
            const bool sideA = r < nA;
            const int owner = sideA ? rec.i : rec.j;
            const int skip = sideA ? rec.posj : rec.posi;
            const int pos = (int)(sideA ? r : r - nA);
            vz = vars[A.nbr[P.adj_off + (int64_t)owner * P.n + pos + (pos >= skip ? 1 : 0)]];
        }
    };
    load_z(r0);
    // X has no more categories than Y (the table is symmetric in them)
    VarRec vx = vars[uni(rec.i)], vy = vars[uni(rec.j)];
    if (vx.card > vy.card) {
        const VarRec t = vx;
        vx = vy;
        vy = t;
    }
    const uint32_t rx = uni((uint32_t)vx.card), ry = uni((uint32_t)vy.card), rxy = rx * ry;
    const uint32_t nx = rx - 1u, ny = ry - 1u, np = nx * ny;
    const uint32_t R = uni((uint32_t)B.R);
    const int32_t *gram = uni(B.gram);
    // (a problem's planes take less than 4 GiB: 32-bit byte offsets)
    const uint32_t sb = uni(B.plane_bytes);
    const uint32_t xo = uni((uint32_t)vx.plane) * sb, yo = uni((uint32_t)vy.plane) * sb;
    const plane_rsrc rs = __builtin_amdgcn_make_buffer_rsrc((void *)uni(B.planes), 0, (int)uni(B.bytes), 0x00020000);
    const uint32_t cx = uni((uint32_t)vx.cat), cy = uni((uint32_t)vy.cat);
    const float inv_rx = 1.0f / (float)rx, inv_ry = 1.0f / (float)ry;
    const uint32_t mw = rx + ry + 1u;  // marginals of a stratum: N_x+z, N_+yz, N_++z
    const uint32_t zmax = min((uint32_t)kBitZ, (uint32_t)kBitAcc / np);
    const int stat = GENERAL ? A.tile.stat : 0;
    const bool adj = GENERAL && A.tile.df_rule != 0, fp64 = GENERAL && A.tile.fp64 != 0;
    // stratum and kind of this lane's marginal (the same for every test)
    const uint32_t ez = fast_div((uint32_t)lane, mw, 1.0f / (float)mw), es = (uint32_t)lane - ez * mw;
    const uint32_t erow = es < rx ? cx + es : cy + (es - rx);
    // this unit's N_ab
    uint32_t vxy = 0;
    if ((uint32_t)lane < np) {
        const uint32_t b = fast_div((uint32_t)lane, nx, 1.0f / (float)nx);
        vxy = (uint32_t)gram[(cx + (uint32_t)lane - b * nx) * R + cy + b];
    }
    uint32_t zb = r0;                    // rank of lane 0's conditioning variable
    int kp = r0 == 0u ? 2 : kBitUnit;    // tests of the next pass at most
    for (uint32_t rb = r0; rb < r1;) {
        // has a lower rank of the edge accepted meanwhile?  (looked at after
        // this pass's counting)
        const unsigned long long ma =
            __hip_atomic_load(&A.min_accept[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (rb + (uint32_t)kp > zb + 64u && r1 > zb + 64u) {
            zb = rb;
            load_z(rb);
        }
        // tests of the pass: those whose planes, words and half-waves fit
        const int t = lane - (int)(rb - zb);
        const bool in = t >= 0 && t < kp && zb + (uint32_t)lane < r1;
        const uint32_t rz = (uint32_t)vz.card;
        const uint32_t T = rxy * rz, need = T + mw * rz, sl = (T + 31u) >> 5;
        // inclusive prefix sums over the pass's lanes: planes, words, half-waves
        uint32_t pzs = in ? (rz - 1u) | (sl << 16) : 0u, pw = in ? need : 0u;
#pragma unroll
        for (int off = 1; off < kBitUnit; off <<= 1) {
            const uint32_t o0 = __shfl_up(pzs, off, 64), o1 = __shfl_up(pw, off, 64);
            if (lane >= off) {
                pzs += o0;
                pw += o1;
            }
        }
        const uint32_t pz = pzs & 0xffffu, ps = pzs >> 16;
        const bool fits = in && pz <= zmax && pw <= (uint32_t)kBitWords && ps <= (uint32_t)kBitSlots;
        const int kb = __popcll(__ballot(fits));  // (a prefix: the sums grow)
        if (fits) {
            s.zcat[t] = (uint32_t)vz.cat;
            s.rz[t] = rz;
            s.zs[t] = pz - (rz - 1u);
            s.toff[t] = pw - need;
            s.slot0[t] = ps - sl;
            s.df[t] = (int)(nx * ny * rz);
            for (uint32_t i = 0; i + 1u < rz; ++i) s.zo[pz - (rz - 1u) + i] = ((uint32_t)vz.plane + i) * sb;
            for (uint32_t i = 0; i < sl; ++i) {
                s.slot_t[ps - sl + i] = (uint8_t)t;
                s.slot_c[ps - sl + i] = (uint8_t)i;
            }
        }
        const uint32_t tot = uni((uint32_t)__shfl(pzs, (int)(rb - zb) + kb - 1, 64));
        const int nzp = (int)(tot & 0xffffu), nsl = (int)(tot >> 16);
        if ((uint32_t)lane < np) s.xy[lane] = vxy;
        g.sync();
        // marginals: requested before the counting, stored after it
        uint32_t mg[kBitUnit];
#pragma unroll
        for (int i = 0; i < kBitUnit; ++i)
            if (i < kb && ez < s.rz[i]) {
                const uint32_t zc = s.zcat[i] + ez;
                mg[i] = (uint32_t)gram[(es == rx + ry ? zc : erow) * R + zc];
            }
        uint32_t zo[kBitZ];
        uint32_t *row = s.part + lane * kBitRow;
#pragma unroll
        for (int i = 0; i < kBitZ; ++i) zo[i] = uni(s.zo[i < nzp ? i : 0]);
        const uint32_t n = (uni(B.words) + 3u) >> 2;  // groups of four words
        switch (nx * 4u + ny) {
            case 5: bit_count_z<1, 1>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 6: bit_count_z<1, 2>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 7: bit_count_z<1, 3>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 8: bit_count_z<1, 4>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 10: bit_count_z<2, 2>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 11: bit_count_z<2, 3>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 12: bit_count_z<2, 4>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 15: bit_count_z<3, 3>(row, rs, xo, yo, sb, zo, n, nzp); break;
            case 16: bit_count_z<3, 4>(row, rs, xo, yo, sb, zo, n, nzp); break;
            default: bit_count_z<4, 4>(row, rs, xo, yo, sb, zo, n, nzp); break;
        }
        g.sync();
        bit_reduce(s, (uint32_t)nzp * np);
#pragma unroll
        for (int i = 0; i < kBitUnit; ++i)
            if (i < kb && ez < s.rz[i]) s.tab[s.toff[i] + rxy * s.rz[i] + (uint32_t)lane] = mg[i];
        g.sync();
        // Two half-waves of cells at a time, one cell per lane: the counts,
        // the last categories in the order z, y, x (each from lower cells,
        // which an earlier step or round has stored), the terms.
        for (int j = 0; j < nsl; j += 2) {
            const int si = j + (lane >> 5);
            float v32 = 0.0f;
            double v64 = 0.0;
            const int ti = s.slot_t[si < nsl ? si : 0];
            const uint32_t rzi = s.rz[ti];
            const uint32_t c = 32u * s.slot_c[si < nsl ? si : 0] + (uint32_t)(lane & 31);
            const bool live = si < nsl && c < rxy * rzi;
            const BitCell q = bit_cell(live ? c : 0u, rx, ry, inv_rx, inv_ry);
            uint32_t *tab = s.tab + s.toff[ti];
            const uint32_t *mz = tab + rxy * rzi + q.z * mw;
            const uint32_t nxz = mz[q.x], nyz = mz[rx + q.y], nzz = mz[rx + ry];
            const bool lx = q.x == nx, ly = q.y == ny, lz = q.z == rzi - 1u;
            const uint32_t ab = q.y * nx + q.x;
            uint32_t v = lx ? nyz : ly ? nxz : lz ? s.xy[ab] : s.M[(s.zs[ti] + q.z) * np + ab];
            if (live && !lx && !ly && !lz) tab[c] = v;
            g.sync();
            if (live && lz && !lx && !ly) {
                for (uint32_t i = 1; i < rzi; ++i) v -= tab[c - i * rxy];
                tab[c] = v;
            }
            g.sync();
            if (live && ly && !lx) {
                for (uint32_t i = 1; i <= ny; ++i) v -= tab[c - i * rx];
                tab[c] = v;
            }
            g.sync();
            if (live && lx) {
                for (uint32_t i = 1; i <= nx; ++i) v -= tab[c - i];
                tab[c] = v;
            }
            if (live && nzz) {
                if (!GENERAL) v32 = bit_g2_term(v, nxz, nyz, nzz);
                else if (fp64) v64 = stat ? x2_term<double>(v, nxz, nyz, nzz) : g2_half_term<double>(v, nxz, nyz, nzz);
                else v32 = stat ? x2_term<float>(v, nxz, nyz, nzz) : bit_g2_term(v, nxz, nyz, nzz);
            }
            v64 = fp64 ? half_sum(v64) : (double)half_sum(v32);
            if ((lane & 31) == 0 && si < nsl) s.g2[si] = v64;
        }
        g.sync();
        // decisions, lane i for test i
        bool acc_t = false, near = false;
        if (lane < kb) {
            const uint32_t rzi = s.rz[lane];
            const uint32_t Ti = rxy * rzi;
            double st = 0.0;
            for (uint32_t i = 0; i < ((Ti + 31u) >> 5); ++i) st += s.g2[s.slot0[lane] + i];
            st = stat ? st : 2.0 * st;
            int df = s.df[lane];
            if (adj) {
                df = 0;
                const uint32_t *mz = s.tab + s.toff[lane] + Ti;
                for (uint32_t z = 0; z < rzi; ++z, mz += mw) {
                    if (mz[rx + ry] == 0u) continue;
                    int na = 0, nb = 0;
                    for (uint32_t x = 0; x < rx; ++x) na += mz[x] > 0u ? 1 : 0;
                    for (uint32_t y = 0; y < ry; ++y) nb += mz[rx + y] > 0u ? 1 : 0;
                    df += (na - 1) * (nb - 1);
                }
                s.df[lane] = df;
            }
            s.st[lane] = st;
            const CritVal &cr = crit[df];  // (df <= (kBitCards - 1)^2 kBitCards)
            acc_t = df <= 0 || st < cr.x;
            near = df > 0 && !(st < cr.x) && !(st > cr.y);
        }
        g.sync();
        uint64_t am = __ballot(acc_t), todo = __ballot(near);
        while (todo) {
            const int ti = __ffsll((long long)todo) - 1;
            todo &= todo - 1ull;
            const CritVal &cr = crit[s.df[ti]];
            if (bit_near(s.tab + s.toff[ti], rx, ry, s.rz[ti], s.st[ti], s.df[ti], P.alpha, cr.x64, cr.y64, stat, fp64))
                am |= 1ull << ti;
            rechecks += fp64 ? 0u : 1u;
        }
        exec += (uint32_t)kb;
        g.sync();  // the tables are rewritten by the next pass
        if (am) return rb + (uint32_t)__ffsll((long long)am) - 1u;
        rb += (uint32_t)kb;
        kp = min(2 * kp, kBitUnit);
        if (uni(ma) < (unsigned long long)rb) break;
    }
    return ~0u;
}

// Units of counter p below `units` when dealt in runs of 2^lgb.
BNS_INLINE unsigned long long bit_units(unsigned long long units, int p, int lgb) {
    const int lrow = 3 + lgb;
    const unsigned long long full = units >> lrow, rem = units - (full << lrow);
    const unsigned long long lo = (unsigned long long)p << lgb;
    return (full << lgb) + (rem > lo ? min(rem - lo, 1ull << lgb) : 0ull);
}

// A work unit is an edge, or one of several consecutive segments of its ranks
// when there are fewer edges than waves.  A wave runs a unit's tests in order
// and stops at the first acceptance (or when a lower segment of the edge has
// accepted), so hardly a test is run in vain.  Unit i of counter p (p =
// blockIdx mod 8, about one per XCD) is the i-th of the runs of 2^run_log2
// consecutive units dealt to p; a wave's first unit is static, the rest are
// grabbed, from the counter with the most left once its own is used up.
// What bounds it: the words of X, Y and Z on their way from the L2s (20 to 29
// bytes per clock and compute unit, with two waves per SIMD to wait for them;
// the vector ALU is ~45% busy on 1,000 variables x 200,000 samples), so a pass takes as many tests of one edge as
// its counts fit registers, and 16-byte loads.  Against one LDS increment per
// sample (k_depth_tests): that search's depth 1 15.1 -> 3.0 ms, 220 x 100,000
// 1.42 -> 0.46 ms, the 64-dataset batch 7.4 -> 2.2 ms, 60 x 50,000 161 -> 98
// us, 20 x 5,000 52 -> 27 us.
template <bool GENERAL>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(2))) void k_depth1_bits(DepthArgs A) {
    __shared__ BitSh sh[kWaves];
    __shared__ CritVal crit_sh[kCritDf];
    __shared__ ProbDev prob_sh;   // searches of one problem
    __shared__ BitProb bprob_sh;
    __shared__ BitItem1 items_sh[kWaves];
    __shared__ unsigned int tal[2];
    __shared__ double tal_bytes;
    __shared__ int hdr_quit;
    Ctl *c = A.ctl;
    const unsigned long long t_enter = wall_clock64();
    if (threadIdx.x == 0) {
        hdr_quit = (c->done | c->error) != 0;
        if (c->xy != 2) {
            hdr_quit = 1;
            if (!c->done) c->error = kDevUnitMismatch;
        }
        tal[0] = tal[1] = 0u;
        tal_bytes = 0.0;
    }
    const bool one_crit = A.bits.n_crit == 1;
    if (one_crit)
        for (int i = threadIdx.x; i < kCritDf; i += kWG) crit_sh[i] = A.bits.crit[i];
    const bool one_prob = A.n_probs == 1;
    if (threadIdx.x == 64) prob_sh = A.probs[0];
    if (threadIdx.x == 128) bprob_sh = A.bits.prob[0];
    const unsigned long long units = uni(c->total_units);
    const unsigned long long edges = uni(c->level_cnt[0]);
    const uint32_t segs = (uint32_t)uni(c->unit_segs);
    __syncthreads();
    if (uni(hdr_quit)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) c->stats[1].t_start = t_enter;
    const int lane = threadIdx.x & 63;
    const int w = uni((int)(threadIdx.x >> 6));
    BitSh &s = sh[w];
    const int nb = (int)gridDim.x;
    BitItem1 &u = items_sh[w];
    const int lgb = A.bits.run_log2;
    int part = (int)(blockIdx.x & 7u);
    unsigned long long bi = (unsigned long long)(blockIdx.x >> 3) * kWaves + (unsigned)w;
    bool fresh = true;  // bi is this wave's static unit
    uint32_t exec = 0, rechecks = 0;
    double bytes = 0.0;
    for (;;) {
        if (!fresh) {
            unsigned long long k = 0;
            if (lane == 0) k = atomicAdd(&c->grab_ctr[part * kGrabStride], 1ull);
            bi = (unsigned long long)kWaves * (unsigned)((nb - part + 7) / 8) + uni(k);
        }
        fresh = false;
        if (bi >= bit_units(units, part, lgb)) {
            // the counter with the most units left, or stop
            unsigned long long key = 0;
            if (lane < kGrabParts) {
                const unsigned long long n = bit_units(units, lane, lgb);
                const unsigned long long u =
                    (unsigned long long)kWaves * (unsigned)((nb - lane + 7) / 8) +
                    __hip_atomic_load(&c->grab_ctr[lane * kGrabStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (n > u) key = ((n - u) << 3) | (unsigned)lane;
            }
#pragma unroll
            for (int off = 1; off < kGrabParts; off <<= 1) {
                const unsigned lo = __shfl_xor((unsigned)(key & 0xffffffffull), off, 64);
                const unsigned hi = __shfl_xor((unsigned)(key >> 32), off, 64);
                const unsigned long long o = ((unsigned long long)hi << 32) | lo;
                key = o > key ? o : key;
            }
            key = uni(key);  // (lane 0's: the largest over lanes 0..7)
            if (key == 0) break;
            part = (int)(key & 7ull);
            continue;
        }
        // segment-major: the low ranks of all edges first
        const unsigned long long tk = ((((bi >> lgb) << 3) + (unsigned)part) << lgb) + (bi & ((1ull << lgb) - 1ull));
        const uint32_t seg = (uint32_t)(tk / edges), e = (uint32_t)(tk - (unsigned long long)seg * edges);
        if (lane == 0) {
            const EdgeRec rec = A.edges[e];
            const uint32_t n = (uint32_t)rec.n, per = (n + segs - 1u) / segs;
            u.e = e;
            u.r = min(n, seg * per);
            u.r1 = min(n, (seg + 1u) * per);
            u.nA = (uint32_t)rec.nA;
            u.prob = rec.prob;
            u.i = rec.i;
            u.j = rec.j;
            u.posj = rec.posj;
            u.posi = rec.posi;
            if (seg > 0 && __hip_atomic_load(&A.min_accept[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < u.r) u.r1 = u.r;
        }
        Grp::wave().sync();
        if (uni(u.r) >= uni(u.r1)) continue;
        const ProbDev &P = one_prob ? prob_sh : A.probs[uni(u.prob)];
        const BitProb &B = one_prob ? bprob_sh : A.bits.prob[uni(u.prob)];
        const CritVal *crit = one_crit ? crit_sh : A.bits.crit + (int64_t)uni(B.crit_row) * kCritDf;
        uint32_t ex = 0, re = 0;
        const uint32_t first = bit_unit<GENERAL>(A, s, crit, P, B, u, ex, re);
        if (lane == 0) {
            if (first != ~0u) atomicMin(&A.min_accept[e], (unsigned long long)first);
            if (A.per_prob && ex) {
                __hip_atomic_fetch_add(&A.ecnt[2 * (uint64_t)e], ex, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (re)
                    __hip_atomic_fetch_add(&A.ecnt[2 * (uint64_t)e + 1], re, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        exec += ex;
        rechecks += re;
        bytes += 3.0 * (double)ex * (double)P.m;
    }
    if (lane == 0) {
        if (exec) atomicAdd(&tal[0], exec);
        if (rechecks) atomicAdd(&tal[1], rechecks);
        if (exec) atomicAdd(&tal_bytes, bytes);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (tal[0]) atomicAdd(&c->stats[1].executed, (unsigned long long)tal[0]);
        if (tal[1]) atomicAdd(&c->stats[1].rechecks, (unsigned long long)tal[1]);
        if (tal_bytes > 0.0) atomicAdd(&c->stats[1].operand_bytes, tal_bytes);
        atomicMax(&c->stats[1].t_end, (unsigned long long)wall_clock64());
    }
}

// ---------------------------------------------------------------------------
// Depth 0 of a search that runs depth 1 from bit planes: one workgroup per
// block of 16 x 16 pairs, one lane per pair.  The lane sums its cells over
// the chunks of the Gram tiles, completes the table, leaves it and its
// transpose in the pairwise tables, and decides the pair by its statistic
// against the critical values: in FP64 where the caller asks for it or the
// contraction is asked for or chosen by the amount of work (BitArgs.fp64), else
// in FP32, and again in FP64 within the critical values' reach.  The block
// writes the adjacency, the removal depths and, for small searches, its
// 16-bit pieces of the adjacency bit rows.  Every pair is tested once, so the
// depth needs no edge list (records, level order and removals of half a
// million edges).  What bounds it: a few dependent loads per lane, and the
// FP64 terms at many pairs.  With the chunk sum and the FP64 pair kernel in
// its place, depth 0 and its preparation took 210 us more at 1,000 variables,
// 185 us at 220 (one workgroup's edge list) and 30 us at 20; this kernel takes
// 92, 28 (FP64) and 13 us (FP32) there.
// ---------------------------------------------------------------------------
constexpr int kPairSide = 16;
constexpr int kBitPlanes = kBitCards - 1;

__global__ __launch_bounds__(kWG) void k_depth0_bits(DepthArgs A, int small) {
    __shared__ uint32_t cnt[2][kPairSide][kBitCards];  // category counts of the block's rows and columns
    __shared__ uint8_t keep_sh[kPairSide][kPairSide + 4];
    __shared__ uint32_t cell_sh[kWG * kBitCards * kBitCards];  // tables of the pairs decided in FP64 (an odd stride)
    __shared__ uint32_t near_sh[kWG];                          // those pairs: lane, r_i, r_j, df
    __shared__ unsigned int near_n, removed_sh;
    const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
    const PairArgs &PA = A.pairs;
    int lo = 0, hi = A.n_probs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (A.bits.prob[mid].block_base <= (int)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const BitProb B = A.bits.prob[lo];
    const ProbDev P = A.probs[lo];
    const GramProb gp = PA.gp[lo];
    int ib = 0, rem = (int)blockIdx.x - B.block_base;
    while (rem >= B.nb16 - ib) {
        rem -= B.nb16 - ib;
        ++ib;
    }
    const int jb = ib + rem;
    const VarRec *vars = A.bits.var + P.var_off;
    const uint32_t m = (uint32_t)P.m;
    const uint32_t R = (uint32_t)B.R;
    // entry (a, b) of the Gram matrix summed over the chunks
    const int nch = gp.nchunks;
    const int64_t tile_words = (int64_t)kGramT * kGramT;
    auto entry = [&](int a, int b) {
        int off;
        const int64_t t = gram_tile(gp, a, b, &off);
        return PA.part + (gp.item_base + t * nch) * tile_words + off;
    };
    if (tid == 0) removed_sh = near_n = 0u;
    // category counts: two lanes' worth of variables, one plane per lane
    if (tid < 2 * kPairSide * kBitPlanes) {
        const int side = tid / (kPairSide * kBitPlanes), q = tid - side * kPairSide * kBitPlanes;
        const int k = q / kBitPlanes, x = q - k * kBitPlanes;
        const int v = kPairSide * (side ? jb : ib) + k;
        uint32_t s = 0;
        if (v < P.n && x < vars[v].card - 1) {
            const int32_t *e = entry(vars[v].plane + x, vars[v].plane + x);
            for (int c = 0; c < nch; c += 8) {
                uint32_t u[8];
#pragma unroll
                for (int k8 = 0; k8 < 8; ++k8) u[k8] = (uint32_t)e[(c + k8 < nch ? c + k8 : 0) * tile_words];
#pragma unroll
                for (int k8 = 0; k8 < 8; ++k8) s += c + k8 < nch ? u[k8] : 0u;
            }
        }
        cnt[side][k][x] = s;
    }
    __syncthreads();
    if (tid < 2 * kPairSide) {
        const int side = tid / kPairSide, k = tid - side * kPairSide;
        const int v = kPairSide * (side ? jb : ib) + k;
        if (v < P.n) {
            const int r = vars[v].card;
            uint32_t s = m;
            for (int x = 0; x < r - 1; ++x) s -= cnt[side][k][x];
            cnt[side][k][r - 1] = s;
            // (the diagonal blocks leave the category counts in the tables)
            if (ib == jb && side == 0)
                for (int x = 0; x < r; ++x) {
                    const uint32_t d = (uint32_t)(vars[v].cat + x);
                    B.gram[d * (R + 1u)] = (int32_t)cnt[0][k][x];
                }
        }
    }
    __syncthreads();
    const int i = kPairSide * ib + ti, j = kPairSide * jb + tj;
    bool kept = false, near = false;
    const bool all64 = A.bits.fp64 != 0;
    int df = 0, ri = 1, rj = 1;
    uint32_t N[kBitCards][kBitCards];
    if (i < j && j < P.n) {
        const VarRec vi = vars[i], vj = vars[j];
        const int pi = vi.card - 1, pj = vj.card - 1;
        ri = vi.card;
        rj = vj.card;
#pragma unroll
        for (int x = 0; x < kBitCards; ++x)
#pragma unroll
            for (int y = 0; y < kBitCards; ++y) N[x][y] = 0u;
        {
            const int32_t *e[kBitPlanes][kBitPlanes];
#pragma unroll
            for (int x = 0; x < kBitPlanes; ++x)
#pragma unroll
                for (int y = 0; y < kBitPlanes; ++y)
                    e[x][y] = entry(vi.plane + (x < pi ? x : 0), vj.plane + (y < pj ? y : 0));
            if (pi > 0 && pj > 0)
                for (int c = 0; c < nch; c += 4) {
                    // four chunks' entries in flight (past the end: the first
                    // chunk's, not added)
                    uint32_t v[4][kBitPlanes][kBitPlanes];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int x = 0; x < kBitPlanes; ++x)
#pragma unroll
                            for (int y = 0; y < kBitPlanes; ++y)
                                if (x < pi && y < pj)
                                    v[u][x][y] = (uint32_t)e[x][y][(c + u < nch ? c + u : 0) * tile_words];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int x = 0; x < kBitPlanes; ++x)
#pragma unroll
                            for (int y = 0; y < kBitPlanes; ++y)
                                if (x < pi && y < pj && c + u < nch) N[x][y] += v[u][x][y];
                }
        }
        // last column, then last row
#pragma unroll
        for (int x = 0; x < kBitCards; ++x) {
            uint32_t rest = cnt[0][ti][x <= pi ? x : 0];
#pragma unroll
            for (int y = 0; y < kBitPlanes; ++y) rest -= N[x][y];
#pragma unroll
            for (int y = 0; y < kBitCards; ++y)
                if (y == pj && x < pi) N[x][y] = rest;
        }
#pragma unroll
        for (int y = 0; y < kBitCards; ++y) {
            uint32_t rest = cnt[1][tj][y <= pj ? y : 0];
#pragma unroll
            for (int x = 0; x < kBitPlanes; ++x) rest -= N[x][y];
#pragma unroll
            for (int x = 0; x < kBitCards; ++x)
                if (x == pi && y <= pj) N[x][y] = rest;
        }
        const uint32_t ci = (uint32_t)vi.cat, cj = (uint32_t)vj.cat;
        const bool x2 = A.tile.stat != 0;
        float st = 0.0f;
        int na = 0, nb = 0;
#pragma unroll
        for (int y = 0; y < kBitCards; ++y) nb += y <= pj && cnt[1][tj][y] > 0u ? 1 : 0;
#pragma unroll
        for (int x = 0; x < kBitCards; ++x) {
            if (x > pi) continue;
            const uint32_t nx = cnt[0][ti][x];
            na += nx > 0u ? 1 : 0;
#pragma unroll
            for (int y = 0; y < kBitCards; ++y) {
                if (y > pj) continue;
                B.gram[(ci + x) * R + cj + y] = (int32_t)N[x][y];
                B.gram[(cj + y) * R + ci + x] = (int32_t)N[x][y];
                const uint32_t ny = cnt[1][tj][y];
                if (!all64) st += x2 ? x2_term<float>(N[x][y], nx, ny, m) : bit_g2_term(N[x][y], nx, ny, m);
            }
        }
        const double stat = x2 ? (double)st : 2.0 * (double)st;
        df = A.tile.df_rule ? (na - 1) * (nb - 1) : pi * pj;
        const CritVal &cr = A.bits.crit[(int64_t)B.crit_row * kCritDf + df];
        kept = df > 0 && !all64 && stat > cr.y;
        near = df > 0 && (all64 || (!(stat < cr.x) && !kept));
    }
    if (near) {
#pragma unroll
        for (int x = 0; x < kBitCards; ++x)
#pragma unroll
            for (int y = 0; y < kBitCards; ++y) cell_sh[(tid * kBitCards + x) * kBitCards + y] = N[x][y];
        near_sh[atomicAdd(&near_n, 1u)] = (uint32_t)(tid | ri << 8 | rj << 12 | df << 16);
    }
    keep_sh[ti][tj] = kept ? 1 : 0;
    __syncthreads();
    // These pairs' statistics in FP64, four lanes each (a chain of 16 cells of
    // one lane takes 13 us; and one loop: unrolled from registers its code
    // would be 20 KB).
    const uint32_t nn = near_n;
    for (uint32_t q0 = 0; q0 < 4u * nn; q0 += kWG) {
        const uint32_t it = q0 + (uint32_t)tid;
        const bool on = it < 4u * nn;
        const uint32_t rec = near_sh[on ? it >> 2 : 0u];
        const uint32_t pt = rec & 255u, a = (rec >> 8) & 15u, b = (rec >> 12) & 15u, d = rec >> 16;
        const uint32_t pi = pt >> 4, pj = pt & 15u;
        const float inv_b = 1.0f / (float)b;
        double s = 0.0;
#pragma unroll 1
        for (uint32_t c = it & 3u; c < a * b; c += 4u) {
            const uint32_t x = fast_div(c, b, inv_b), y = c - x * b;
            const uint32_t v = cell_sh[(pt * kBitCards + x) * kBitCards + y], nx = cnt[0][pi][x], ny = cnt[1][pj][y];
            s += A.tile.stat ? x2_term<double>(v, nx, ny, m) : g2_half_term<double>(v, nx, ny, m);
        }
        s += __shfl_xor(s, 1, 64);
        s += __shfl_xor(s, 2, 64);
        if (on && (it & 3u) == 0u) {
            const double stat = A.tile.stat ? s : 2.0 * s;
            const CritVal &cr = A.bits.crit[(int64_t)B.crit_row * kCritDf + d];
            bool k = stat > cr.y64;
            if (!k && !(stat < cr.x64)) k = !(chi2_tail_lane(d, stat) > P.alpha);
            keep_sh[pi][pj] = k ? 1 : 0;
        }
    }
    __syncthreads();
    kept = keep_sh[ti][tj] != 0;
    // both orders of every pair of the block; (row, column) of the block's own
    // and of its transpose
    unsigned int gone = i < j && j < P.n && !kept ? 1u : 0u;
    const int8_t dep = 0;
    if (ib != jb) {
        if (i < P.n && j < P.n) {
            A.adj[P.adj_off + (int64_t)i * P.n + j] = kept ? 1 : 0;
            A.rdepth[P.adj_off + (int64_t)i * P.n + j] = kept ? (int8_t)-1 : dep;
        }
        const int i2 = kPairSide * jb + ti, j2 = kPairSide * ib + tj;  // transposed
        if (i2 < P.n && j2 < P.n) {
            const bool k2 = keep_sh[tj][ti] != 0;
            A.adj[P.adj_off + (int64_t)i2 * P.n + j2] = k2 ? 1 : 0;
            A.rdepth[P.adj_off + (int64_t)i2 * P.n + j2] = k2 ? (int8_t)-1 : dep;
        }
    } else if (i < P.n && j < P.n) {
        const bool k2 = (i < j ? keep_sh[ti][tj] : keep_sh[tj][ti]) != 0;
        A.adj[P.adj_off + (int64_t)i * P.n + j] = k2 && i != j ? 1 : 0;
        A.rdepth[P.adj_off + (int64_t)i * P.n + j] = k2 || i == j ? (int8_t)-1 : dep;
    }
    if (small && tid < 2 * kPairSide) {
        // 16-bit pieces of the bit rows (rows beyond n have none; a piece
        // beyond n is 0)
        const int side = tid / kPairSide, k = tid - side * kPairSide;
        const int v = kPairSide * (side ? jb : ib) + k, piece = side ? ib : jb;
        if (v < P.n && !(side && ib == jb)) {
            uint32_t bits = 0;
            for (int q = 0; q < kPairSide; ++q) {
                const bool on = ib == jb ? (k < q ? keep_sh[k][q] : keep_sh[q][k]) != 0 && k != q
                                         : (side ? keep_sh[q][k] : keep_sh[k][q]) != 0;
                bits |= on ? 1u << q : 0u;
            }
            const int W = (P.n + 63) >> 6;
            ((uint16_t *)(A.adjbits + P.bit_off + (int64_t)v * W))[piece] = (uint16_t)bits;
        }
    }
    for (int off = 32; off > 0; off >>= 1) gone += __shfl_xor(gone, off, 64);
    if ((tid & 63) == 0 && gone) atomicAdd(&removed_sh, gone);
    __syncthreads();
    if (tid == 0) {
        Ctl *c = A.ctl;
        const unsigned long long np = (unsigned long long)P.n * (unsigned long long)(P.n - 1) / 2ull;
        if (removed_sh) atomicAdd(&c->stats[0].removed, (unsigned long long)removed_sh);
        if (nn && !all64) atomicAdd(&c->stats[0].rechecks, (unsigned long long)nn);
        if (A.per_prob) {
            PStatDev &ps = A.pstat[(int64_t)lo * kMaxDepths];
            if (removed_sh) atomicAdd(&ps.removed, (unsigned long long)removed_sh);
            if (nn && !all64) atomicAdd(&ps.rechecks, (unsigned long long)nn);
            if ((int)blockIdx.x == B.block_base) ps.edges = ps.tickets = ps.required = ps.executed = np;
        }
        if ((int)blockIdx.x == B.block_base) atomicAdd(&c->stats[0].operand_bytes, 2.0 * (double)np * (double)P.m);
        if (blockIdx.x == 0) {
            const unsigned long long all = (unsigned long long)A.n_pairs;
            c->stats[0].edges = c->stats[0].tickets = c->stats[0].required = c->stats[0].executed = all;
            c->depth = 1;
        }
        atomicMax(&c->stats[0].t_end, (unsigned long long)wall_clock64());
    }
}

hipError_t launch_depth0_bits(const DepthArgs &a, hipStream_t s) {
    const bool small = small_search(a);
    hipError_t e = launch_gram_tiles(a, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_depth0_bits, dim3(a.bits.blocks), dim3(kWG), 0, s, a, small ? 1 : 0);
    e = hipGetLastError();
    return e == hipSuccess && small ? launch_prepare_small(a, s) : e;
}

hipError_t launch_depth1_bits(const DepthArgs &a, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    auto kern = a.tile.stat != 0 || a.tile.df_rule != 0 || a.tile.fp64 != 0 ? &k_depth1_bits<true> : &k_depth1_bits<false>;
    if (start && stop) hipExtLaunchKernelGGL(kern, dim3(a.bits.grid), dim3(kWG), 0, s, start, stop, 0, a);
    else hipLaunchKernelGGL(kern, dim3(a.bits.grid), dim3(kWG), 0, s, a);
    return hipGetLastError();
}

int bits_max_wg_per_cu() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_depth1_bits<false>, kWG, 0) != hipSuccess) return 1;
    return nb > 0 ? nb : 1;
}

}  // namespace bns
