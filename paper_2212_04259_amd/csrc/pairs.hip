// Depth 0 of the skeleton search (Section IV-B: every pair is tested once,
// with no conditioning set) as one dense contraction on gfx950 int8 MFMA.
//
// With one-hot columns A[s][(v, x)] = [X_v(s) = x] (m samples by R = sum of
// the cardinalities), the Gram matrix A^T A holds every pairwise contingency
// table: N_ij[x][y] = (A^T A)[(i, x)][(j, y)], and its diagonal the count of
// each category, which are the marginals N_x+ and N_+y of every pair table.
// The products of 0/1 bytes summed in int32 are exact (m < 2^31).
//
// The contraction's work items are T x T tiles of the upper triangle of tile
// blocks of one problem's Gram matrix over one chunk of samples; each writes
// its partial tile.
// k_planes, k_gram_planes: the columns become bit planes (one bit per sample
// for each category but the last), and the contraction forms its int8
// operands from plane words in registers, with no LDS in its loop.
// k_gram: the byte form, for problems of mostly wide variables; a workgroup
// (2 x 2 waves, each a (T/2) x (T/2) block of 32 x 32 MFMA tiles) expands the
// tile's one-hot columns for 64 samples at a time into LDS (double-buffered:
// the global loads of the next step are in flight during the MFMAs of this
// one).
// k_gram_reduce: sums each tile's partials over its problem's chunks.
// k_depth0_pairs: one lane per edge of the depth reads the pair's block of the
// summed tiles, forms the statistic in FP64, its own chi-square tail and the
// decision.
#include <algorithm>

#include "device_ci.h"
#include "gram.h"
#include "kernels.h"

namespace bns {

constexpr int kGramKS = 64;             // samples per pipeline step
constexpr int kGramRow = kGramKS + 16;  // LDS bytes per one-hot column and step
constexpr int kGramQS = kGramKS / 16;   // 16-sample groups per column and step

// Start of the depth-0 span and its launch shape (c: the search's control
// block, or null for the all-pairs entry point); true when the search is done.
BNS_INLINE bool gram_enter(const PairArgs &P, Ctl *c, int *quit) {
    if (threadIdx.x == 0) {
        *quit = c ? c->done : 0;
        if (c && blockIdx.x == 0) {
            // (with planes the span starts in k_planes)
            if (!P.planes) c->stats[0].t_start = wall_clock64();
            c->stats[0].mode = 2;  // depth 0 as the pair contraction
            c->stats[0].chunks = 0;
            c->stats[0].chunk_len = P.chunk;
        }
    }
    __syncthreads();
    return *quit != 0;
}

// Work item -> problem, tile (tr <= tc), chunk of samples.
struct GramItem {
    GramProb gp;
    int tr, tc;
    int64_t s0, s1;
};
BNS_INLINE GramItem gram_item(const PairArgs &P, int64_t item) {
    int lo = 0, hi = P.n_gp - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (P.gp[mid].item_base <= item) lo = mid;
        else hi = mid - 1;
    }
    GramItem it;
    it.gp = P.gp[lo];
    const int64_t rel = item - it.gp.item_base;
    const int64_t t = rel / it.gp.nchunks;
    const int kc = (int)(rel - t * it.gp.nchunks);
    it.tr = 0;
    int64_t rem = t;
    while (rem >= it.gp.nb - it.tr) {
        rem -= it.gp.nb - it.tr;
        ++it.tr;
    }
    it.tc = it.tr + (int)rem;
    it.s0 = (int64_t)kc * P.chunk;
    it.s1 = min(it.gp.m, it.s0 + P.chunk);
    return it;
}

// ---------------------------------------------------------------------------
// Bit planes.  A lane takes 32 samples of one variable (two 16-byte loads)
// and forms their word of each plane: first one word per bit of the value,
// bit k of dword j's four bytes going to bits j, 8 + j, 16 + j, 24 + j (one
// shift and one and-or per dword and bit), then category c's word as the
// conjunction of the value bits of c or their complements.  The samples are
// permuted within a word, the same way in every plane, which no count can
// see.  0.5 vector operations per sample and value bit (comparing bytes
// across the wave took 3 per sample and category), so reading the columns
// bounds it: 1,000 variables x 200,000 samples in 42 us, 250 MB at 5.9 TB/s
// (89 us with the wave compares).  Bits of samples past m are 0.
// ---------------------------------------------------------------------------
template <int NB>
BNS_INLINE void plane_words(const u32x4 (&x)[2], uint32_t valid, int r, uint32_t *out, uint32_t *val,
                            int64_t stride) {
    uint32_t bit[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        uint32_t wd = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t d = x[j >> 2][j & 3];
            wd |= (j >= k ? d << (j - k) : d >> (k - j)) & (0x01010101u << j);
        }
        bit[k] = wd;
    }
    for (int cat = 0; cat < r - 1; ++cat) {
        uint32_t wd = valid;
#pragma unroll
        for (int k = 0; k < NB; ++k) wd &= ((cat >> k) & 1) ? bit[k] : ~bit[k];
        out[(int64_t)cat * stride] = wd;
    }
    if (val)
        for (int k = 0; k < NB && (1 << k) < r; ++k) val[(int64_t)k * stride] = bit[k] & valid;
}

// reset: the kernel is the first of a search (depths 0 and 1 from bit planes)
// and clears the control block and the per-problem counters.
__global__ __launch_bounds__(kWG) void k_planes(PairArgs P, const uint8_t *cards, Ctl *c, PStatDev *pstat, int reset) {
    if (c && blockIdx.x == 0) {
        if (reset) {
            if (threadIdx.x == 0) reset_search(c);
            for (int i = threadIdx.x; i < kMaxDepths; i += kWG) c->stats[i] = DepthStatDev{};
            __syncthreads();
        }
        if (threadIdx.x == 0) c->stats[0].t_start = wall_clock64();
    }
    if (reset && pstat)
        for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < (int64_t)P.n_gp * kMaxDepths;
             i += (int64_t)gridDim.x * kWG)
            pstat[i] = PStatDev{};
    const int lane = threadIdx.x & 63;
    const int w = uni((int)(threadIdx.x >> 6));
    for (int64_t item = (int64_t)blockIdx.x * kWaves + w; item < P.plane_items; item += (int64_t)gridDim.x * kWaves) {
        int lo = 0, hi = P.n_gp - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (P.gp[mid].plane_item <= item) lo = mid;
            else hi = mid - 1;
        }
        const GramProb &gp = P.gp[lo];
        const int64_t m = uni(gp.m), stride = uni(gp.plane_stride);
        const int64_t nq = (stride + kPlaneItem * 64 - 1) / (kPlaneItem * 64);
        const int64_t rel = item - uni(gp.plane_item);
        const int v = (int)(rel / nq);
        const int64_t w0 = (rel - (int64_t)v * nq) * (kPlaneItem * 64) + lane;  // this lane's first word
        const int g = uni(gp.var_off) + v;
        const int r = uni((int)cards[g]);
        if (r < 2) continue;
        const uint8_t *col = gp.data + (int64_t)v * uni(gp.ld);
        u32x4 x[kPlaneItem][2];
#pragma unroll
        for (int u = 0; u < kPlaneItem; ++u) {
            const int64_t s = 32 * (w0 + 64 * u);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                x[u][q] = u32x4{0u, 0u, 0u, 0u};
                if (s + 16 * q < m) x[u][q] = *(const gvec4 *)(col + s + 16 * q);
            }
        }
        uint32_t *out = P.planes + uni(gp.plane_off) + (int64_t)uni(P.var_oh[g]) * stride;
        uint32_t *val = P.var && value_planes(r) > 0 ? P.planes + uni(gp.plane_off) + (int64_t)uni(P.var[g].val) * stride
                                                     : nullptr;
#pragma unroll
        for (int u = 0; u < kPlaneItem; ++u) {
            const int64_t wi = w0 + 64 * u;
            if (wi >= stride) continue;
            uint32_t valid = ~0u;
            const int64_t left = m - 32 * wi;
            if (left < 32) {  // sample i of the word is bit 8 (i mod 4) + i / 4
                valid = 0u;
                for (int i = 0; i < (int)left; ++i) valid |= 1u << (8 * (i & 3) + (i >> 2));
            }
            if (r <= 2) plane_words<1>(x[u], valid, r, out + wi, nullptr, stride);
            else if (r <= 4) plane_words<2>(x[u], valid, r, out + wi, val ? val + wi : nullptr, stride);
            else if (r <= 8) plane_words<3>(x[u], valid, r, out + wi, val ? val + wi : nullptr, stride);
            else plane_words<8>(x[u], valid, r, out + wi, val ? val + wi : nullptr, stride);
        }
    }
}

// ---------------------------------------------------------------------------
// Gram tiles from bit planes.  The four waves of a workgroup compute the same
// 64 x 64 tile over interleaved 256-sample steps of the chunk (the waves'
// 32-byte pieces of a plane share its 128-byte lines) and add their tiles in
// LDS.  A lane of an operand holds one plane's 32-bit word: bytes k, k + 8,
// k + 16, k + 24 of the samples come from one shift and one mask, (w >> k) &
// 0x01010101, so 32 samples cost 15 vector operations and feed two MFMA steps
// (the sample order inside a step does not matter as long as both operands
// use the same).  Per step and wave 240 vector operations meet 32 MFMAs of 32
// cycles: about balanced, against forming one-hot bytes from the columns in
// LDS (k_gram), which is bound by that forming and reads 8 times the bytes.
// 1,000 variables x 200,000 samples (2,000 planes): 305 us, 2.6e15 int8
// operations/s over the upper triangle; k_gram's 3,000 one-hot columns took
// 2,050 us, the planes included 347.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kGramWG) void k_gram_planes(PairArgs P, Ctl *c) {
    constexpr int T = kGramT;
    __shared__ int32_t red[T * T];
    __shared__ int quit;
    if (gram_enter(P, c, &quit)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = uni(tid >> 6);
    const int h = lane >> 5;
    for (int64_t item = blockIdx.x; item < P.items; item += gridDim.x) {
        const GramItem it = gram_item(P, item);
        const GramProb &gp = it.gp;
        const uint32_t *base = P.planes + gp.plane_off;
        // rows past the last plane read the last one; their entries are not used
        const uint32_t *row[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int rr = min((f < 2 ? it.tr : it.tc) * T + 32 * (f & 1) + (lane & 31), gp.R - 1);
            row[f] = base + (int64_t)rr * gp.plane_stride + 4 * h;
        }
        for (int i = tid; i < T * T; i += kGramWG) red[i] = 0;
        v16i acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
        // 256-sample steps of the chunk (whole blocks: the planes are padded)
        const int64_t st0 = it.s0 >> 8;
        const int64_t st1 = (it.s1 + kPlaneBlock - 1) / kPlaneBlock * (kPlaneBlock >> 8);
        u32x4 nx[4];
        int64_t st = st0 + w;
        if (st < st1) {
#pragma unroll
            for (int f = 0; f < 4; ++f) nx[f] = *(const gvec4 *)(row[f] + 8 * st);
        }
        while (st < st1) {
            u32x4 x[4];
#pragma unroll
            for (int f = 0; f < 4; ++f) x[f] = nx[f];
            const int64_t sn = st + kWaves;
            if (sn < st1) {
#pragma unroll
                for (int f = 0; f < 4; ++f) nx[f] = *(const gvec4 *)(row[f] + 8 * sn);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    v4i o[4];
#pragma unroll
                    for (int f = 0; f < 4; ++f)
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[f][e] = (int)((x[f][q] >> (4 * kk + e)) & 0x01010101u);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o[i], o[2 + j], acc[i][j], 0, 0, 0);
                }
            }
            st = sn;
        }
        __syncthreads();  // red is clear
        // register r of lane l holds row (r % 4) + 4 (l / 32) + 8 (r / 4),
        // column l % 32 of a 32 x 32 tile
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int rr = 32 * i + (r & 3) + 4 * h + 8 * (r >> 2);
                    const int cc = 32 * j + (lane & 31);
                    atomicAdd(&red[rr * T + cc], acc[i][j][r]);
                }
        __syncthreads();
        int4 *out = (int4 *)(P.part + item * (int64_t)(T * T));
        for (int i = tid; i < T * T / 4; i += kGramWG) out[i] = ((const int4 *)red)[i];
        __syncthreads();  // red is cleared for the next item
    }
}

template <int T>
__global__ __launch_bounds__(kGramWG) void k_gram(PairArgs P, Ctl *c) {
    constexpr int WT = T / 2;              // rows (and columns) of a wave's block
    constexpr int NF = WT / 32;            // 32 x 32 MFMA tiles per side of a wave's block
    constexpr int kTasks = 2 * T * kGramQS;  // (operand, column, 16-sample group) per step
    constexpr int kPer = kTasks / kGramWG;
    static_assert(kPer * kGramWG == kTasks, "tasks split evenly");
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][2 * T * kGramRow];  // [buffer][operand][column][sample]
    __shared__ int quit;
    if (gram_enter(P, c, &quit)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = w >> 1, wc = w & 1;
    for (int64_t item = blockIdx.x; item < P.items; item += gridDim.x) {
        const GramItem it = gram_item(P, item);
        const GramProb &gp = it.gp;
        const int tr = it.tr, tc = it.tc;
        const int64_t s0 = it.s0, s1 = it.s1;
        const bool diag = tr == tc;  // the second operand is the first
        const int nsteps = (int)((s1 - s0 + kGramKS - 1) / kGramKS);
        // this thread's expansion tasks for every step of the item
        const uint8_t *colp[kPer];
        uint32_t plo[kPer], phi[kPer], cat[kPer];
        int dst[kPer];
        bool act[kPer], wide[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int id = tid + kGramWG * r;
            const int op = id / (T * kGramQS);
            const int rest = id - op * T * kGramQS;
            const int col = rest / kGramQS, q = rest % kGramQS;
            act[r] = !(diag && op == 1);
            dst[r] = op * T * kGramRow + col * kGramRow + 16 * q;
            const int gcol = (op ? tc : tr) * T + col;
            const int v = P.oh_var[gp.oh_base + gcol];
            const uint32_t cb = P.oh_cat[gp.oh_base + gcol];
            wide[r] = (cb & 0x100u) != 0;
            cat[r] = cb & 0xffu;
            plo[r] = cat[r] < 4 ? 1u << (8 * cat[r]) : 0u;
            phi[r] = (cat[r] >= 4 && cat[r] < 8) ? 1u << (8 * (cat[r] - 4)) : 0u;
            colp[r] = v >= 0 ? gp.data + (int64_t)v * gp.ld + 16 * q : nullptr;
        }
        u32x4 pv[kPer];
        int pn[kPer];
        auto load = [&](int64_t s) {
            // samples left from s (uniform; at most a step and a group matter)
            const int left = (int)min(s1 - s, (int64_t)(kGramKS + 16));
#pragma unroll
            for (int r = 0; r < kPer; ++r) {
                pn[r] = min(16, max(0, left - 16 * ((tid + kGramWG * r) % kGramQS)));
                pv[r] = u32x4{0u, 0u, 0u, 0u};
                // (a global load: a flat one would also count against the
                // LDS counter, and the step's LDS reads would wait for it)
                if (act[r] && colp[r] && pn[r] > 0) pv[r] = *(const gvec4 *)(colp[r] + s);
            }
        };
        auto store = [&](int buf) {
#pragma unroll
            for (int r = 0; r < kPer; ++r) {
                if (!act[r]) continue;
                u32x4 o = u32x4{0u, 0u, 0u, 0u};
                if (colp[r]) o = onehot16(pv[r], plo[r], phi[r], cat[r], wide[r], pn[r]);
                *(u32x4 *)(&lds[buf][dst[r]]) = o;
            }
        };
        v16i acc[NF][NF];
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
        load(s0);
        store(0);
        __syncthreads();
        for (int st = 0; st < nsteps; ++st) {
            const int buf = st & 1;
            const bool more = st + 1 < nsteps;
            if (more) load(s0 + (int64_t)(st + 1) * kGramKS);
            const uint8_t *La = &lds[buf][0];
            const uint8_t *Lb = diag ? La : &lds[buf][T * kGramRow];
#pragma unroll
            for (int kk = 0; kk < kGramKS / 32; ++kk) {
                const int koff = 32 * kk + 16 * (lane >> 5);
                v4i af[NF], bf[NF];
#pragma unroll
                for (int i = 0; i < NF; ++i)
                    af[i] = *(const v4i *)(La + (wr * WT + 32 * i + (lane & 31)) * kGramRow + koff);
#pragma unroll
                for (int j = 0; j < NF; ++j)
                    bf[j] = *(const v4i *)(Lb + (wc * WT + 32 * j + (lane & 31)) * kGramRow + koff);
#pragma unroll
                for (int i = 0; i < NF; ++i)
#pragma unroll
                    for (int j = 0; j < NF; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[i], bf[j], acc[i][j], 0, 0, 0);
            }
            if (more) store(buf ^ 1);
            __syncthreads();
        }
        // partial tile of the item: register r of lane l holds row
        // (r % 4) + 4 (l / 32) + 8 (r / 4), column l % 32 of a 32 x 32 tile
        int32_t *out = P.part + item * (int64_t)(T * T);
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = wr * WT + 32 * i + (r & 3) + 4 * (lane >> 5) + 8 * (r >> 2);
                    const int col = wc * WT + 32 * j + (lane & 31);
                    out[row * T + col] = acc[i][j][r];
                }
    }
}

// Sums each tile's partials over its problem's chunks (coalesced, four
// entries per lane): gram[tile] = sum_k part[item of (tile, k)].
__global__ __launch_bounds__(kWG) void k_gram_reduce(PairArgs P) {
    const int64_t tq = (int64_t)P.T * P.T / 4;  // int4 words per tile
    const int64_t total = P.tiles * tq;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < total; i += (int64_t)gridDim.x * kWG) {
        const int64_t tile = i / tq, w = i - tile * tq;
        int lo = 0, hi = P.n_gp - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (P.gp[mid].tile_base <= tile) lo = mid;
            else hi = mid - 1;
        }
        const GramProb &gp = P.gp[lo];
        const int4 *src = (const int4 *)P.part + (gp.item_base + (tile - gp.tile_base) * gp.nchunks) * tq + w;
        int4 s = src[0];
        for (int k = 1; k < gp.nchunks; ++k) {
            const int4 v = src[(int64_t)k * tq];
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
        ((int4 *)P.gram)[i] = s;
    }
}

// Statistic (G^2 or X^2, FP64) and df of a pair with ri and rj categories
// over m samples from its cells and category counts (the marginals N_x+ and
// N_+y; N_++ = m).
template <typename CellF, typename RowF, typename ColF>
BNS_INLINE void pair_terms(int ri, int rj, int64_t m, int stat_kind, bool adj, double &stat, int64_t &df, CellF cell,
                           RowF cnt_i, ColF cnt_j) {
    int na = 0, nb = 0;
    stat = 0.0;
    for (int y = 0; y < rj; ++y) nb += cnt_j(y) > 0u ? 1 : 0;
    for (int x = 0; x < ri; ++x) {
        const uint32_t nx = cnt_i(x);  // N_x+
        na += nx > 0u ? 1 : 0;
        for (int y = 0; y < rj; ++y) {
            const uint32_t ny = cnt_j(y);  // N_+y
            const uint32_t N = cell(x, y);
            if (stat_kind) stat += x2_term<double>(N, nx, ny, (uint32_t)m);
            else stat += g2_half_term<double>(N, nx, ny, (uint32_t)m);
        }
    }
    if (!stat_kind) stat *= 2.0;
    df = adj ? (int64_t)(na - 1) * (int64_t)(nb - 1) : (int64_t)(ri - 1) * (int64_t)(rj - 1);
}

// The same for the pair of variables whose rows of the Gram matrix start at
// oi and oj (oi < oj).  The diagonal entries are the category counts.  With
// planes only the cells of neither variable's last category are entries; the
// last column is what the other columns leave of N_x+, the last row what the
// other rows leave of N_+y.  Up to kPairCats categories (the usual networks) the
// table is completed in the lane's column of `cell` (kPairCats^2 words,
// kPairWG apart): the loads of four rows are in flight together, and one copy
// of the term's code serves every cell.  (25 cells unrolled in registers were
// 20 KB of code, which a call of a few hundred pairs spent longer fetching
// than on its tests: all pairs of 20 x 100,000 of up to six categories 184 us
// a call with them, 141 with this; of 300 x 50,000 239 and 214.)
constexpr int kPairCats = 8;
constexpr int kPairWG = 64;

BNS_INLINE void pair_stat(const PairArgs &P, const GramProb &gp, int oi, int oj, int ri, int rj, int64_t m,
                          int stat_kind, bool adj, double &stat, int64_t &df, uint32_t *cell) {
    // categories that have entries
    const int pi = P.planes ? ri - 1 : ri, pj = P.planes ? rj - 1 : rj;
    if (ri <= kPairCats && rj <= kPairCats) {
        auto at = [&](int x, int y) -> uint32_t & { return cell[(x * kPairCats + y) * kPairWG]; };
        uint32_t ni[kPairCats], nj[kPairCats], li = (uint32_t)m, lj = (uint32_t)m;
#pragma unroll
        for (int x = 0; x < kPairCats; ++x) ni[x] = x < pi ? gram_entry(P, gp, oi + x, oi + x) : 0u;
#pragma unroll
        for (int y = 0; y < kPairCats; ++y) nj[y] = y < pj ? gram_entry(P, gp, oj + y, oj + y) : 0u;
        for (int x0 = 0; x0 < pi; x0 += 4) {
            uint32_t v[4][kPairCats];
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < kPairCats; ++y)
                    v[x][y] = x0 + x < pi && y < pj ? gram_entry(P, gp, oi + x0 + x, oj + y) : 0u;
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < kPairCats; ++y)
                    if (x0 + x < pi && y < pj) at(x0 + x, y) = v[x][y];
        }
#pragma unroll
        for (int x = 0; x < kPairCats; ++x) li -= ni[x];
#pragma unroll
        for (int y = 0; y < kPairCats; ++y) lj -= nj[y];
        // counts of a category (registers are not indexed: eight selects)
        auto pick = [](const uint32_t (&n)[kPairCats], int k, int last, uint32_t rest) {
            uint32_t r = rest;
#pragma unroll
            for (int q = 0; q < kPairCats; ++q)
                if (q == k && k < last) r = n[q];
            return r;
        };
        uint32_t left_row = 0;
        pair_terms(ri, rj, m, stat_kind, adj, stat, df,
                   [&](int x, int y) {
                       if (y == 0) left_row = pick(ni, x, pi, li);
                       uint32_t N;
                       if (y == pj) {
                           N = left_row;
                       } else if (x < pi) {
                           N = at(x, y);
                       } else {
                           N = pick(nj, y, pj, lj);
                           for (int a = 0; a < pi; ++a) N -= at(a, y);
                       }
                       left_row -= N;
                       return N;
                   },
                   [&](int x) { return pick(ni, x, pi, li); }, [&](int y) { return pick(nj, y, pj, lj); });
        return;
    }
    if (!P.planes) {
        pair_terms(ri, rj, m, stat_kind, adj, stat, df, [&](int x, int y) { return gram_entry(P, gp, oi + x, oj + y); },
                   [&](int x) { return gram_entry(P, gp, oi + x, oi + x); },
                   [&](int y) { return gram_entry(P, gp, oj + y, oj + y); });
        return;
    }
    uint32_t li = (uint32_t)m, lj = (uint32_t)m;
    for (int x = 0; x < pi; ++x) li -= gram_entry(P, gp, oi + x, oi + x);
    for (int y = 0; y < pj; ++y) lj -= gram_entry(P, gp, oj + y, oj + y);
    auto cnt_i = [&](int x) { return x < pi ? gram_entry(P, gp, oi + x, oi + x) : li; };
    auto cnt_j = [&](int y) { return y < pj ? gram_entry(P, gp, oj + y, oj + y) : lj; };
    uint32_t left_row = 0;  // what is left of row x
    pair_terms(ri, rj, m, stat_kind, adj, stat, df,
               [&](int x, int y) {
                   if (y == 0) left_row = cnt_i(x);
                   uint32_t N;
                   if (y == pj) {
                       N = left_row;  // (the last row's too: its other cells have been taken off)
                   } else if (x < pi) {
                       N = gram_entry(P, gp, oi + x, oj + y);
                   } else {
                       N = cnt_j(y);
                       for (int a = 0; a < pi; ++a) N -= gram_entry(P, gp, oi + a, oj + y);
                   }
                   left_row -= N;
                   return N;
               },
               cnt_i, cnt_j);
}

// The depth-0 tests of a skeleton search: one lane per edge of the depth.
__global__ __launch_bounds__(kPairWG) void k_depth0_pairs(DepthArgs A) {
    __shared__ uint32_t cells[kPairCats * kPairCats * kPairWG];
    Ctl *c = A.ctl;
    __shared__ int quit;
    if (threadIdx.x == 0) quit = c->done;
    __syncthreads();
    if (quit) return;
    const PairArgs &P = A.pairs;
    const unsigned long long E = c->n_edges;
    const int lane = threadIdx.x & 63;
    unsigned long long ex = 0;
    double ob = 0.0;
    for (unsigned long long e = (unsigned long long)blockIdx.x * kPairWG + threadIdx.x; e < E;
         e += (unsigned long long)gridDim.x * kPairWG) {
        const EdgeRec rec = A.edges[e];
        const ProbDev pd = A.probs[rec.prob];
        const GramProb gp = P.gp[rec.prob];
        const int gi = pd.var_off + rec.i, gj = pd.var_off + rec.j;
        double stat;
        int64_t df;
        pair_stat(P, gp, P.var_oh[gi], P.var_oh[gj], A.cards[gi], A.cards[gj], pd.m, A.tile.stat,
                  A.tile.df_rule != 0, stat, df, cells + threadIdx.x);
        if (chi2_tail_lane(df, stat) > pd.alpha) A.min_accept[e] = 0ull;  // the depth's only test accepted
        ++ex;
        ob += 2.0 * (double)pd.m;
        if (A.per_prob) A.ecnt[2 * e] = 1u;
    }
    ex = wave_sum(ex);
    ob = wave_sum(ob);
    if (lane == 0) {
        if (ex) atomicAdd(&c->stats[0].executed, ex);
        if (ob > 0.0) atomicAdd(&c->stats[0].operand_bytes, ob);
        atomicMax(&c->stats[0].t_end, (unsigned long long)wall_clock64());
    }
}

// Every pair i < j of one dataset (all-pairs entry point): pair index
// i n - i (i + 1) / 2 + j - i - 1.
__global__ __launch_bounds__(kPairWG) void k_ci_pairs(PairArgs P, const uint8_t *cards, int32_t n, double alpha,
                                                  int stat_kind, int df_rule, double *stat_out, int64_t *df_out,
                                                  double *p_out, int32_t *flags_out) {
    const GramProb gp = P.gp[0];
    __shared__ uint32_t cells[kPairCats * kPairCats * kPairWG];
    const int64_t npairs = (int64_t)n * (n - 1) / 2;
    for (int64_t q = (int64_t)blockIdx.x * kPairWG + threadIdx.x; q < npairs; q += (int64_t)gridDim.x * kPairWG) {
        // row i: the largest i with i n - i (i + 1) / 2 <= q
        int lo = 0, hi = n - 2;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if ((int64_t)mid * n - (int64_t)mid * (mid + 1) / 2 <= q) lo = mid;
            else hi = mid - 1;
        }
        const int i = lo;
        const int j = (int)(q - ((int64_t)i * n - (int64_t)i * (i + 1) / 2)) + i + 1;
        double stat;
        int64_t df;
        pair_stat(P, gp, P.var_oh[i], P.var_oh[j], cards[i], cards[j], gp.m, stat_kind, df_rule != 0, stat, df,
                  cells + threadIdx.x);
        const double p = chi2_tail_lane(df, stat);
        if (stat_out) stat_out[q] = stat;
        if (df_out) df_out[q] = df;
        if (p_out) p_out[q] = p;
        if (flags_out) flags_out[q] = p > alpha ? 1 : 0;
    }
}

int gram_max_wg_per_cu(bool planes) {
    int nb = 0;
    const hipError_t e = planes ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_gram_planes, kGramWG, 0)
                                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_gram<kGramT>, kGramWG, 0);
    return (e == hipSuccess && nb > 0) ? nb : 1;
}

// The Gram tiles of every problem; cards: per global variable, first: see
// k_planes.
static void launch_tiles(const PairArgs &p, const uint8_t *cards, Ctl *c, PStatDev *pstat, int first, hipStream_t s) {
    const dim3 grid(p.gram_grid);
    if (p.planes) {
        hipLaunchKernelGGL(k_planes, dim3(p.plane_grid), dim3(kWG), 0, s, p, cards, c, pstat, first);
        hipLaunchKernelGGL(k_gram_planes, grid, dim3(kGramWG), 0, s, p, c);
    } else {
        hipLaunchKernelGGL(k_gram<kGramT>, grid, dim3(kGramWG), 0, s, p, c);
    }
}

// The Gram tiles and their sum over chunks.
static void launch_gram(const PairArgs &p, const uint8_t *cards, Ctl *c, hipStream_t s) {
    launch_tiles(p, cards, c, nullptr, 0, s);
    if (p.gram != p.part) {
        const int64_t words = p.tiles * p.T * p.T / 4;
        const int rg = (int)std::max<int64_t>(1, std::min<int64_t>(4096, (words + kWG - 1) / kWG));
        hipLaunchKernelGGL(k_gram_reduce, dim3(rg), dim3(kWG), 0, s, p);
    }
}

hipError_t launch_gram_tiles(const DepthArgs &a, hipStream_t s) {
    launch_tiles(a.pairs, a.cards, a.ctl, a.per_prob ? a.pstat : nullptr, 1, s);
    return hipGetLastError();
}

hipError_t launch_depth0_pairs(const DepthArgs &a, hipStream_t s) {
    launch_gram(a.pairs, a.cards, a.ctl, s);
    hipLaunchKernelGGL(k_depth0_pairs, dim3(a.edge_grid * (kWG / kPairWG)), dim3(kPairWG), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ci_pairs(const PairArgs &p, const uint8_t *cards, int32_t n, double alpha, int stat,
                           int df_rule, double *stat_out, int64_t *df_out, double *p_out, int32_t *flags_out,
                           hipStream_t s) {
    launch_gram(p, cards, nullptr, s);
    const int64_t npairs = (int64_t)n * (n - 1) / 2;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(8192, (npairs + kPairWG - 1) / kPairWG));
    hipLaunchKernelGGL(k_ci_pairs, dim3(grid), dim3(kPairWG), 0, s, p, cards, n, alpha, stat, df_rule, stat_out,
                       df_out, p_out, flags_out);
    return hipGetLastError();
}

}  // namespace bns
