// Drives the host side of the Fokker-Planck doubling tree (stages, node
// matrices in fragment order, the waves' unit records) for a build with
// AddressSanitizer and UndefinedBehaviorSanitizer.  For every slab it
//   - checks that each fragment and row that a unit names exists, and that
//     the units of a phase cover its rows and column tiles once each;
//   - walks the records as the kernels do, in plain loops, and compares the
//     corrected moments with the eliminations' matrices of the same slab.
// Exit status 0 when everything held.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "setup_math.hpp"

using namespace snfpsa;

#define CHECK(cond)                                                                  \
    do {                                                                             \
        if (!(cond)) {                                                               \
            std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond);  \
            return 1;                                                                \
        }                                                                            \
    } while (0)

struct Unit {
    int off, first, rows, tile;
};

// The correction by the eliminations' matrices: phi [K][2 (L + 1)].
static dvec eliminate(const FPFactors &F, const dvec &diff) {
    const int K = F.K, N = F.N, NH = F.NH, L2 = 2 * (F.L + 1);
    const size_t M2 = (size_t)NH * NH;
    std::vector<int> type(K);
    for (size_t s = 0; s + 1 < F.seg_begin.size(); ++s)
        for (int j = F.seg_begin[s]; j < F.seg_begin[s + 1]; ++j) type[j] = F.seg_type[s];
    dvec s((size_t)K * N, 0.0);
    for (int j = 0; j < K; ++j)
        for (int k = 0; k < L2; ++k)
            for (int c = 0; c < N; ++c)
                s[(size_t)j * N + c] += diff[(size_t)j * L2 + k] * F.EsrcT[((size_t)type[j] * L2 + k) * N + c];
    auto mul = [&](int j, int m, const double *x, double *y) {
        const double *A = &F.cellmats[((size_t)j * FP_CELL_MATS + m) * M2];
        for (int r = 0; r < NH; ++r)
            for (int c = 0; c < NH; ++c) y[r] += A[(size_t)r * NH + c] * x[c];
    };
    dvec p((size_t)(K + 1) * NH, 0.0), q((size_t)(K + 1) * NH, 0.0), a = p, b = p;
    for (int j = 0; j < K; ++j) {
        double *y = &p[(size_t)(j + 1) * NH];
        mul(j, 0, &p[(size_t)j * NH], y);
        mul(j, 1, &s[(size_t)j * N + NH], y);
        for (int i = 0; i < NH; ++i) y[i] += s[(size_t)j * N + i];
    }
    for (int j = K - 1; j >= 0; --j) {
        double *y = &q[(size_t)j * NH];
        mul(j, 2, &q[(size_t)(j + 1) * NH], y);
        mul(j, 3, &s[(size_t)j * N], y);
        for (int i = 0; i < NH; ++i) y[i] += s[(size_t)j * N + NH + i];
    }
    for (int k = 0; k < K; ++k) {  // (a_K is the outflow, which no cell reads)
        if (k > 0) {
            mul(k, 4, &p[(size_t)k * NH], &a[(size_t)k * NH]);
            mul(k, 5, &q[(size_t)k * NH], &a[(size_t)k * NH]);
        }
        mul(k, 6, &a[(size_t)k * NH], &b[(size_t)k * NH]);
        for (int i = 0; i < NH; ++i) b[(size_t)k * NH + i] += q[(size_t)k * NH + i];
    }
    dvec out((size_t)K * L2, 0.0);
    for (int j = 0; j < K; ++j)
        for (int c = 0; c < L2; ++c) {
            double v = 0.0;
            for (int k = 0; k < L2; ++k) v += diff[(size_t)j * L2 + k] * F.PhisrcT[((size_t)type[j] * L2 + k) * L2 + c];
            for (int k = 0; k < NH; ++k) {
                v += a[(size_t)j * NH + k] * F.PhiinfT[((size_t)type[j] * N + k) * L2 + c];
                v += b[(size_t)(j + 1) * NH + k] * F.PhiinfT[((size_t)type[j] * N + NH + k) * L2 + c];
            }
            out[(size_t)j * L2 + c] = v;
        }
    return out;
}

// The same by the tree's records.
static int by_tree(const FPFactors &F, const dvec &diff, dvec &out) {
    const FPTree &T = F.tree;
    const int K = F.K, N = F.N, NH = F.NH, L2 = 2 * (F.L + 1), nb = F.tree.nb, KB = 4 * nb;
    const int ksN = (N + KB - 1) / KB * nb, ksL = (L2 + KB - 1) / KB * nb;
    const int ctN = (N + 15) / 16, ctU = (2 * N + 15) / 16, ctL = (L2 + 15) / 16;
    const int S = (int)T.stages.size();
    CHECK(S >= 1 && S <= kTreeMaxStages);
    out.assign((size_t)K * L2, 0.0);
    // interfaces: the cells' take K rows of N, the later stages' share (K + 1) N / 2
    std::vector<dvec> Y(S + 1);
    size_t later = 0;
    int n = K;
    for (int i = 0; i < S; ++i) {
        const FPTreeStage &s = T.stages[i];
        CHECK(s.n == n && s.c == 1 << s.levels && s.chunks == (n + s.c - 1) / s.c && (s.leaf != 0) == (i == 0));
        CHECK(std::min(s.c, s.n) <= kTreeMaxRows && 2 * s.levels + 2 <= kTreeHdr);
        const size_t rows = std::min(s.c, s.n), root = i == S - 1;
        const size_t lds = (1 + root) * (rows + 1) * fp_tree_ld(nb, N) + (s.leaf ? rows * fp_tree_ld(nb, L2) : 0);
        CHECK(lds * sizeof(double) <= (160u << 10));
        CHECK(s.rec0 + (size_t)s.chunks * kTreeWaves * s.rec_stride <= T.records.size());
        CHECK(s.rec_stride >= kTreeHdr + 4 && (s.rec_stride - kTreeHdr) % 2 == 0 && s.rec_stride - kTreeHdr <= 2 * kTreeMaxUnits);
        Y[i].assign((size_t)(n + 1) * N, 0.0);
        if (i) later += (size_t)(n + 1) * N;
        n = s.chunks;
    }
    CHECK(n == 1 && later <= (size_t)(K + 1) * NH);
    Y[S].assign((size_t)2 * N, 0.0);
    int bad = 0;
    auto B = [&](int off, int k, int col) { return T.frag[(size_t)off * 64 + ((size_t)(k / 8) * 64 + (k % 4) * 16 + col) * 2 + (k % 8) / 4]; };
    // units of a phase of a chunk, checked against its rows (count) and tiles
    auto phase = [&](const FPTreeStage &s, int chunk, int ph, int count, int tiles, int entries, int ks0, int ks1, auto &&body) {
        std::vector<int> seen((size_t)count * tiles, 0);
        for (int w = 0; w < kTreeWaves; ++w) {
            const int *rec = &T.records[s.rec0 + ((size_t)chunk * kTreeWaves + w) * s.rec_stride];
            const int u0 = ph ? rec[ph - 1] : 0, u1 = rec[ph], all = (s.rec_stride - kTreeHdr) / 2;
            if (u0 < 0 || u1 < u0 || (u1 - u0) % entries || u1 >= all) ++bad;
            for (int u = u0; u < u1 && !bad; u += entries) {
                Unit x[2];
                for (int e = 0; e < entries; ++e) {
                    const int off = rec[kTreeHdr + 2 * (u + e)], d = rec[kTreeHdr + 2 * (u + e) + 1];
                    x[e] = Unit{off, d & 0xff, (d >> 8) & 0xff, d >> 16};
                    if (off < 0 || (size_t)(off + (e ? ks1 : ks0)) * 64 > T.frag.size()) ++bad;
                    if (x[e].rows < 1 || x[e].rows > 16 || x[e].first + x[e].rows > count || x[e].tile < 0 || x[e].tile >= tiles) ++bad;
                    if (e && (x[1].first != x[0].first || x[1].rows != x[0].rows || x[1].tile != x[0].tile)) ++bad;
                }
                // the unit after it, of which the first batch is requested
                const int next = rec[kTreeHdr + 2 * (u + entries)];
                if (next < 0 || (size_t)(next + nb) * 64 > T.frag.size()) ++bad;
                if (bad) return;
                for (int r = x[0].first; r < x[0].first + x[0].rows; ++r) {
                    ++seen[(size_t)r * tiles + x[0].tile];
                    for (int c = 0; c < 16; ++c) body(x[0].off, x[entries - 1].off, r, 16 * x[0].tile + c, c);
                }
            }
        }
        for (int v : seen) bad += v != 1;
    };
    auto interfaces = [&](const FPTreeStage &s, int nc, int l) {
        const int half = 1 << (l - 1), step = 1 << l;
        (void)s;
        return nc > half ? (nc - half + step - 1) / step : 0;
    };
    for (int i = 0; i < S; ++i) {  // up
        const FPTreeStage &s = T.stages[i];
        for (int p = 0; p < s.chunks; ++p) {
            const int c0 = p * s.c, nc = std::min(s.c, s.n - c0);
            dvec R((size_t)(nc + 1) * N, 0.0), X = R;
            auto at = [&](dvec &v, int r, int k) -> double & { return v[(size_t)r * N + k]; };
            if (s.leaf)
                phase(s, p, 0, nc, ctN, 1, ksL, 0, [&](int off, int, int r, int col, int c) {
                    if (col >= N) return;
                    double v = 0.0;
                    for (int k = 0; k < L2; ++k) v += diff[(size_t)(c0 + r) * L2 + k] * B(off, k, c);
                    at(R, r + (col < NH), col) = v;
                });
            else
                for (int r = 0; r <= nc; ++r)
                    for (int k = 0; k < N; ++k)
                        if ((r > 0 || k >= NH) && (r < nc || k < NH)) at(R, r, k) = Y[i][(size_t)(c0 + r) * N + k];
            if (bad) break;
            for (int l = 1; l <= s.levels; ++l) {
                const int half = 1 << (l - 1);
                phase(s, p, l, interfaces(s, nc, l), ctU, 1, ksN, 0, [&](int off, int, int r, int col, int c) {
                    if (col >= 2 * N) return;
                    const int j = half + (r << l);
                    double v = 0.0;
                    for (int k = 0; k < N; ++k) v += at(R, j, k) * B(off, k, c);
                    if (col < N)
                        at(X, j, col) = v;
                    else
                        at(R, col - N < NH ? std::min(j + half, nc) : j - half, col - N) += v;
                });
                if (bad) break;
            }
            if (bad) break;
            for (int j = 1; j < nc; ++j)  // zero-inflow values, for the descent
                for (int k = 0; k < N; ++k) Y[i][(size_t)(c0 + j) * N + k] = at(X, j, k);
            for (int k = 0; k < NH; ++k) {
                Y[i + 1][(size_t)(p + 1) * N + k] = at(R, nc, k);
                Y[i + 1][(size_t)p * N + NH + k] = at(R, 0, NH + k);
            }
        }
        CHECK(!bad);
    }
    std::fill(Y[S].begin(), Y[S].end(), 0.0);  // no inflow
    for (int i = S - 1; i >= 0; --i) {  // down
        const FPTreeStage &s = T.stages[i];
        dvec V((size_t)(s.n + 1) * N, 0.0);
        for (int p = 0; p < s.chunks; ++p) {
            const int c0 = p * s.c, nc = std::min(s.c, s.n - c0);
            dvec X((size_t)(nc + 1) * N, 0.0);
            auto at = [&](int r, int k) -> double & { return X[(size_t)r * N + k]; };
            for (int j = 1; j < nc; ++j)
                for (int k = 0; k < N; ++k) at(j, k) = Y[i][(size_t)(c0 + j) * N + k];
            for (int k = 0; k < NH; ++k) {
                at(0, k) = Y[i + 1][(size_t)p * N + k];
                at(nc, NH + k) = Y[i + 1][(size_t)(p + 1) * N + NH + k];
            }
            for (int l = s.levels; l >= 1; --l) {
                const int half = 1 << (l - 1);
                phase(s, p, 2 * s.levels + 1 - l, interfaces(s, nc, l), ctN, 1, ksN, 0, [&](int off, int, int r, int col, int c) {
                    if (col >= N) return;
                    const int j = half + (r << l), j1 = std::min(j + half, nc);
                    double v = 0.0;
                    for (int k = 0; k < N; ++k) v += (k < NH ? at(j - half, k) : at(j1, k)) * B(off, k, c);
                    at(j, col) += v;
                });
                if (bad) break;
            }
            if (bad) break;
            if (s.leaf)
                phase(s, p, 2 * s.levels + 1, nc, ctL, 2, ksL, ksN, [&](int off, int inf, int r, int col, int c) {
                    if (col >= L2) return;
                    double v = 0.0;
                    for (int k = 0; k < L2; ++k) v += diff[(size_t)(c0 + r) * L2 + k] * B(off, k, c);
                    for (int k = 0; k < N; ++k) v += (k < NH ? at(r, k) : at(r + 1, k)) * B(inf, k, c);
                    out[(size_t)(c0 + r) * L2 + col] = v;
                });
            // a at a chunk's left face, b at its right one
            for (int j = 0; j <= nc; ++j)
                for (int k = 0; k < N; ++k)
                    if ((j > 0 || k < NH) && (j < nc || k >= NH)) V[(size_t)(c0 + j) * N + k] = at(j, k);
        }
        CHECK(!bad);
        Y[i] = V;
    }
    return 0;
}

static int one(int K, int N, int L, int regions, int scheme, int slabs, bool fold) {
    dvec mu, w;
    gauss_legendre(N, mu, w);
    const dvec A = scheme == 0 ? wfd_laplacian(N, mu, w) : mpd_laplacian(N, mu, w);
    std::vector<double> h(K), st(K), ss((size_t)K * (L + 1)), sa(K), str(K);
    for (int k = 0; k < K; ++k) {
        const int reg = (int)((long long)k * regions / K);
        h[k] = 0.05 + 0.001 * (reg % 17);
        st[k] = 0.5 + 0.01 * reg;
        double gl = 1.0;
        for (int l = 0; l <= L; ++l, gl *= 0.9) ss[(size_t)k * (L + 1) + l] = (0.99 - 0.002 * (reg % 10)) * st[k] * gl;
        sa[k] = st[k] - ss[(size_t)k * (L + 1)];
        str[k] = ss[(size_t)k * (L + 1)] - (L >= 1 ? ss[(size_t)k * (L + 1) + 1] : 0.0);
    }
    auto build = [&](FPFactors &F, int ts) {
        return fold ? build_fp_factors(K, N, L, h.data(), st.data(), ss.data(), mu, w, A, F, 0, ts)
                    : build_fp_factors_coef(K, N, L, h.data(), sa.data(), str.data(), nullptr, mu, w, A, F, 0, ts);
    };
    FPFactors E, F;
    CHECK(build(E, 0) && build(F, slabs));
    CHECK(E.tree.stages.empty() && !E.cellmats.empty());
    CHECK(!F.tree.stages.empty() && F.cellmats.empty() && F.EsrcT.empty());
    CHECK(F.chunk == E.chunk && F.nchunks == E.nchunks && F.seg_begin == E.seg_begin && F.seg_type == E.seg_type);
    std::mt19937 rng(K * 1000 + N);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    dvec diff((size_t)K * 2 * (L + 1)), got;
    for (double &v : diff) v = u(rng);
    const dvec ref = eliminate(E, diff);
    if (by_tree(F, diff, got)) return 1;
    double err = 0.0, top = 0.0;
    for (size_t i = 0; i < ref.size(); ++i) {
        err = std::max(err, std::fabs(got[i] - ref[i]));
        top = std::max(top, std::fabs(ref[i]));
    }
    std::printf("K=%d N=%d L=%d regions=%d slabs=%d: %zu stages, off by %.1e of %.1e\n", K, N, L, regions, slabs,
                F.tree.stages.size(), err, top);
    // both compose the cells' responses in FP64, as tests of the kernels
    CHECK(err <= 1e-10 * top);
    return 0;
}

int main() {
    struct Case {
        int K, N, L, regions, scheme, slabs;
        bool fold;
    };
    // no level, one, a ragged last node, one chunk at its largest and past it;
    // two to five stages; passes cut by regions; column tiles below, at and
    // past 16; no two cells alike; many slabs; both sides of the sizes that
    // keep the eliminations
    const Case cases[] = {
        {1, 2, 0, 1, 0, 1, true},      {2, 2, 1, 2, 1, 1, true},     {1, 16, 15, 1, 0, 4, false},
        {3, 4, 3, 1, 1, 1, true},      {5, 2, 1, 2, 0, 1, true},     {17, 16, 15, 1, 0, 1, false},
        {33, 18, 6, 4, 1, 1, true},    {64, 8, 7, 64, 0, 1, true},   {255, 8, 7, 1, 0, 1, true},
        {256, 8, 7, 1, 0, 1, true},    {257, 8, 4, 1, 1, 1, true},   {257, 8, 4, 3, 1, 64, true},
        {515, 24, 15, 5, 1, 1, true},  {515, 24, 15, 5, 1, 32, true}, {300, 10, 9, 300, 0, 1, true},
        {1100, 6, 5, 4, 0, 1, true},   {4097, 4, 3, 2, 0, 1, true},  {20000, 2, 1, 3, 0, 1, true},
        {140000, 2, 0, 1, 0, 1, false}, {70, 34, 33, 70, 0, 2, true}, {130, 64, 40, 3, 0, 1, true},
        {200, 64, 63, 1, 0, 256, false}, {20, 34, 33, 2, 0, 1, true}, {50, 80, 70, 3, 0, 2, true},
        {40, 66, 65, 1, 1, 1, true},   {36, 104, 103, 2, 0, 1, true}, {40, 128, 40, 2, 0, 1, true},
        {66, 114, 20, 1, 0, 1, false}, {20, 130, 9, 1, 0, 1, true},  {9, 256, 255, 2, 1, 1, true},
        {70, 20, 19, 3, 0, 400, true}, {70, 20, 19, 3, 0, 500, true}, {90, 46, 45, 2, 0, 1, true},
    };
    // the handles that keep the eliminations: cells, widths and runs at their
    // ends, one slab, several, and of two padded widths
    auto keeps = [](std::vector<FPSlabShape> v) { return fp_keeps_eliminations(v); };
    CHECK(!keeps({}) && keeps({{65, 106, 1}}) && !keeps({{64, 106, 1}}) && !keeps({{65, 104, 1}}) && !keeps({{65, 130, 1}}));
    CHECK(keeps({{700, 98, 2}}) && !keeps({{701, 98, 2}}) && !keeps({{100, 96, 2}}) && keeps({{100, 126, 3}}) && !keeps({{100, 124, 3}}));
    CHECK(!keeps({{100, 128, 4}}) && !keeps({{200, 128, 200}}));
    CHECK(keeps({{300, 128, 1}, {300, 106, 1}}) && !keeps({{300, 128, 1}, {301, 106, 1}}) && !keeps({{30, 128, 1}, {30, 104, 1}}));
    CHECK(keeps({{500, 66, 2}, {500, 128, 1}}) && !keeps({{500, 66, 2}, {501, 128, 1}}) && keeps({{40, 80, 8}, {30, 70, 1}}) && !keeps({{40, 80, 9}, {30, 70, 1}}));
    CHECK(keeps({{800, 50, 4}, {800, 64, 4}}) && !keeps({{800, 50, 3}, {800, 64, 3}}) && !keeps({{801, 50, 4}, {800, 64, 4}}) && !keeps({{80, 48, 8}, {80, 64, 8}}));
    CHECK(!keeps({{80, 64, 8}, {80, 66, 8}}) && !keeps({{80, 128, 2}, {80, 130, 2}}));
    CHECK(!keeps({{2000000000, 128, 2}, {2000000000, 128, 2}, {2000000000, 128, 2}}));
    const double w[] = {1, 1, 2, 2, 1, 1}, t[] = {3, 3, 3, 3, 3, 4}, f[] = {1, 2, 1, 2, 1, 2, 1, 3, 1, 3, 1, 3};
    CHECK(fp_runs(6, 2, w, nullptr, nullptr) == 3 && fp_runs(6, 2, w, t, nullptr) == 4 && fp_runs(6, 2, w, t, f) == 5);
    CHECK(fp_runs(1, 2, w, t, f) == 1 && fp_runs(2, 2, w, t, f) == 1);
    for (const Case &c : cases)
        if (one(c.K, c.N, c.L, c.regions, c.scheme, c.slabs, c.fold)) {
            std::fprintf(stderr, "K=%d N=%d L=%d regions=%d slabs=%d\n", c.K, c.N, c.L, c.regions, c.slabs);
            return 1;
        }
    std::printf("tree driver ok\n");
    return 0;
}
