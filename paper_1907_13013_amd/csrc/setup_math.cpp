// Host FP64 setup math: quadrature, Legendre tables, WFD/MPD Laplacians and
// the two-sided interface (Riccati) factorisation of the LD x S_N
// Fokker-Planck operator.  See setup_math.hpp for the formulation.
#include "setup_math.hpp"

#include <algorithm>
#include <cmath>
#include <map>
#include <stdexcept>

namespace snfpsa {

namespace {

constexpr double kPi = 3.14159265358979323846;

// P_n(x) and P_{n-1}(x) by the three-term recurrence.
void legendre_pair(int n, double x, double &pn, double &pnm1) {
    double a = 1.0, b = x;
    if (n == 0) { pn = 1.0; pnm1 = 0.0; return; }
    for (int k = 2; k <= n; ++k) {
        double c = ((2 * k - 1) * x * b - (k - 1) * a) / k;
        a = b;
        b = c;
    }
    pn = b;
    pnm1 = a;
}

// Row-major dense helpers on n x n (or general) matrices.
void matmul(int m, int k, int n, const double *A, const double *B, double *C) {
    for (int i = 0; i < m; ++i)
        for (int j = 0; j < n; ++j) {
            double s = 0.0;
            for (int t = 0; t < k; ++t) s += A[(size_t)i * k + t] * B[(size_t)t * n + j];
            C[(size_t)i * n + j] = s;
        }
}

// In-place inverse by Gauss-Jordan elimination with partial pivoting.
bool invert(int n, double *A) {
    std::vector<double> M((size_t)n * 2 * n, 0.0);
    for (int i = 0; i < n; ++i) {
        for (int j = 0; j < n; ++j) M[(size_t)i * 2 * n + j] = A[(size_t)i * n + j];
        M[(size_t)i * 2 * n + n + i] = 1.0;
    }
    const int w2 = 2 * n;
    for (int c = 0; c < n; ++c) {
        int piv = c;
        double best = std::fabs(M[(size_t)c * w2 + c]);
        for (int r = c + 1; r < n; ++r) {
            double v = std::fabs(M[(size_t)r * w2 + c]);
            if (v > best) { best = v; piv = r; }
        }
        if (!(best > 0.0)) return false;
        if (piv != c)
            for (int j = 0; j < w2; ++j) std::swap(M[(size_t)c * w2 + j], M[(size_t)piv * w2 + j]);
        const double inv = 1.0 / M[(size_t)c * w2 + c];
        for (int j = 0; j < w2; ++j) M[(size_t)c * w2 + j] *= inv;
        for (int r = 0; r < n; ++r) {
            if (r == c) continue;
            const double f = M[(size_t)r * w2 + c];
            if (f == 0.0) continue;
            for (int j = 0; j < w2; ++j) M[(size_t)r * w2 + j] -= f * M[(size_t)c * w2 + j];
        }
    }
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) A[(size_t)i * n + j] = M[(size_t)i * w2 + n + j];
    return true;
}

}  // namespace

void gauss_legendre(int N, dvec &mu, dvec &w) {
    mu.assign(N, 0.0);
    w.assign(N, 0.0);
    for (int i = 1; i <= N; ++i) {
        // Tricomi's asymptotic guess for the i-th largest root, then Newton.
        double x = (1.0 - 1.0 / (8.0 * N * N) + 1.0 / (8.0 * N * N * N)) *
                   std::cos(kPi * (4.0 * i - 1.0) / (4.0 * N + 2.0));
        double pn = 0, pm = 0, dp = 1;
        for (int it = 0; it < 60; ++it) {
            legendre_pair(N, x, pn, pm);
            dp = N * (pm - x * pn) / (1.0 - x * x);
            const double dx = pn / dp;
            x -= dx;
            if (std::fabs(dx) <= 1e-17 * std::fabs(x) + 1e-300) break;
        }
        legendre_pair(N, x, pn, pm);
        const double one_m_x2 = (1.0 - x) * (1.0 + x);  // accurate near |x| = 1
        dp = N * (pm - x * pn) / one_m_x2;
        mu[N - i] = x;
        w[N - i] = 2.0 / (one_m_x2 * dp * dp);
    }
    // symmetrise: the rule is exactly symmetric about 0
    for (int i = 0; i < N / 2; ++i) {
        const double m = 0.5 * (mu[N - 1 - i] - mu[i]);
        const double ww = 0.5 * (w[N - 1 - i] + w[i]);
        mu[i] = -m;
        mu[N - 1 - i] = m;
        w[i] = w[N - 1 - i] = ww;
    }
    if (N % 2) mu[N / 2] = 0.0;
}

dvec legendre_table(int N, int L, const dvec &mu) {
    dvec P((size_t)(L + 1) * N);
    for (int n = 0; n < N; ++n) {
        double a = 1.0, b = mu[n];
        P[n] = 1.0;
        if (L >= 1) P[(size_t)N + n] = b;
        for (int l = 2; l <= L; ++l) {
            double c = ((2 * l - 1) * mu[n] * b - (l - 1) * a) / l;
            P[(size_t)l * N + n] = c;
            a = b;
            b = c;
        }
    }
    return P;
}

dvec wfd_laplacian(int N, const dvec &mu, const dvec &w) {
    // gamma[i] = gamma_{i+1/2} in 1-based notation: gamma[0] = gamma_{1/2} = 0
    dvec gamma(N + 1, 0.0);
    for (int n = 0; n < N; ++n) gamma[n + 1] = gamma[n] - 2.0 * mu[n] * w[n];
    gamma[N] = 0.0;
    dvec W((size_t)N * N, 0.0);
    for (int n = 0; n < N; ++n) {
        const double down = (n > 0) ? gamma[n] / (mu[n] - mu[n - 1]) : 0.0;
        const double up = (n + 1 < N) ? gamma[n + 1] / (mu[n + 1] - mu[n]) : 0.0;
        if (n > 0) W[(size_t)n * N + n - 1] = down / w[n];
        if (n + 1 < N) W[(size_t)n * N + n + 1] = up / w[n];
        W[(size_t)n * N + n] = -(down + up) / w[n];
    }
    return W;
}

dvec mpd_laplacian(int N, const dvec &mu, const dvec &w) {
    dvec P = legendre_table(N, N - 1, mu);
    dvec F((size_t)N * N, 0.0);
    // F[n][m] = sum_l (2l+1)/2 P_l(mu_n) (-l(l+1)) P_l(mu_m) w_m
    for (int n = 0; n < N; ++n)
        for (int m = 0; m < N; ++m) {
            double s = 0.0;
            for (int l = 0; l < N; ++l)
                s += 0.5 * (2 * l + 1) * P[(size_t)l * N + n] * (-(double)l * (l + 1)) * P[(size_t)l * N + m];
            F[(size_t)n * N + m] = s * w[m];
        }
    return F;
}

bool build_fp_factors(int K, int N, int L, const double *h, const double *sigma_t,
                      const double *sigma_s, const dvec &mu, const dvec &w, const dvec &A,
                      FPFactors &out, int chunk_hint, int tree_slabs) {
    const int L1 = L + 1;
    dvec sa(K), str(K);
    for (int j = 0; j < K; ++j) {
        const double *ss = sigma_s + (size_t)j * L1;
        sa[j] = sigma_t[j] - ss[0];
        str[j] = ss[0] - (L1 > 1 ? ss[1] : 0.0);
    }
    return build_fp_factors_coef(K, N, L, h, sa.data(), str.data(), sigma_s, mu, w, A, out, chunk_hint, tree_slabs);
}

// Cell types and their maps: the interface responses T, R, R', T' of each
// type (into ct) and its source and moment maps (into out).
static bool fp_cell_types(int K, int N, int L, const double *h, const double *sigma_a, const double *sigma_tr,
                          const double *sigma_s, const dvec &mu, const dvec &w, const dvec &A, FPFactors &out,
                          FPCellTypes &ct) {
    const int NH = N / 2, N2 = 2 * N, L1 = L + 1, L2 = 2 * L1;
    out.K = K; out.N = N; out.L = L; out.NH = NH;
    out.folded_sigma_s = sigma_s != nullptr;
    dvec P = legendre_table(N, L, mu);

    // ---- cell types: runs of cells with identical (h, sigma_a, sigma_tr and,
    // when it is folded into the source maps, sigma_s row)
    std::map<std::vector<double>, int> type_of;
    std::vector<std::vector<double>> keys;
    out.seg_begin.clear();
    out.seg_type.clear();
    std::vector<int> &cell_type = ct.cell_type;
    cell_type.assign(K, 0);
    const int nkey = 3 + (sigma_s ? L1 : 0);
    for (int j = 0; j < K; ++j) {
        std::vector<double> key(nkey);
        key[0] = h[j];
        key[1] = sigma_a[j];
        key[2] = sigma_tr[j];
        if (sigma_s)
            for (int l = 0; l < L1; ++l) key[3 + l] = sigma_s[(size_t)j * L1 + l];
        auto it = type_of.find(key);
        int t;
        if (it == type_of.end()) {
            t = (int)keys.size();
            type_of.emplace(key, t);
            keys.push_back(key);
        } else {
            t = it->second;
        }
        cell_type[j] = t;
        if (j == 0 || cell_type[j - 1] != t) {
            out.seg_begin.push_back(j);
            out.seg_type.push_back(t);
        }
    }
    out.seg_begin.push_back(K);
    const int ntypes = (int)keys.size();
    out.ntypes = ntypes;

    // ---- per type: cell block, responses, source and moment maps
    std::vector<dvec> &Tc = ct.T, &Rc = ct.R, &Rpc = ct.Rp, &Tpc = ct.Tp;
    for (std::vector<dvec> *v : {&Tc, &Rc, &Rpc, &Tpc}) v->assign(ntypes, dvec());
    out.EsrcT.assign((size_t)ntypes * L2 * N, 0.0);
    out.PhisrcT.assign((size_t)ntypes * L2 * L2, 0.0);
    out.PhiinfT.assign((size_t)ntypes * N * L2, 0.0);
    dvec D((size_t)N2 * N2), Pm((size_t)N2 * N), Q((size_t)N2 * N2), Qp((size_t)N2 * L2);
    for (int t = 0; t < ntypes; ++t) {
        const double hh = keys[t][0], sa = keys[t][1], str = keys[t][2];
        // D: LD cell block with removal T = sa I - (str/2) A
        for (int n = 0; n < N; ++n)
            for (int m = 0; m < N; ++m) {
                const double T = (n == m ? sa : 0.0) - 0.5 * str * A[(size_t)n * N + m];
                D[(size_t)n * N2 + m] = hh / 3.0 * T;
                D[(size_t)n * N2 + N + m] = hh / 6.0 * T;
                D[(size_t)(N + n) * N2 + m] = hh / 6.0 * T;
                D[(size_t)(N + n) * N2 + N + m] = hh / 3.0 * T;
            }
        for (int n = 0; n < N; ++n) {
            const double m = mu[n];
            D[(size_t)n * N2 + n] += std::fabs(m) / 2.0;
            D[(size_t)n * N2 + N + n] += m / 2.0;
            D[(size_t)(N + n) * N2 + n] -= m / 2.0;
            D[(size_t)(N + n) * N2 + N + n] += std::fabs(m) / 2.0;
        }
        if (!invert(N2, D.data())) return false;  // D now holds D^{-1}
        // Pm = D^{-1} J: inflow columns [a (angles NH..N-1) ; b (angles 0..NH-1)]
        for (int r = 0; r < N2; ++r) {
            for (int i = 0; i < NH; ++i) {
                const int na = NH + i, nb = i;
                Pm[(size_t)r * N + i] = D[(size_t)r * N2 + na] * mu[na];            // row L_na, +mu
                Pm[(size_t)r * N + NH + i] = D[(size_t)r * N2 + N + nb] * (-mu[nb]); // row R_nb, |mu|
            }
        }
        // Q = D^{-1} Mass, Mass per angle (h/6)[[2,1],[1,2]] on (L,R)
        for (int r = 0; r < N2; ++r)
            for (int n = 0; n < N; ++n) {
                const double dl = D[(size_t)r * N2 + n], dr = D[(size_t)r * N2 + N + n];
                Q[(size_t)r * N2 + n] = hh / 6.0 * (2.0 * dl + dr);
                Q[(size_t)r * N2 + N + n] = hh / 6.0 * (dl + 2.0 * dr);
            }
        // Qp = Q (I2 x M Sigma): column (nu, l)
        for (int r = 0; r < N2; ++r)
            for (int nu = 0; nu < 2; ++nu)
                for (int l = 0; l < L1; ++l) {
                    double s = 0.0;
                    for (int n = 0; n < N; ++n)
                        s += Q[(size_t)r * N2 + nu * N + n] * 0.5 * (2 * l + 1) * P[(size_t)l * N + n];
                    Qp[(size_t)r * L2 + nu * L1 + l] = sigma_s ? s * keys[t][3 + l] : s;
                }
        // interface responses; outgoing rows: a_out = U_R at angles NH..N-1,
        // b_out = U_L at angles 0..NH-1
        Tc[t].assign((size_t)NH * NH, 0); Rc[t].assign((size_t)NH * NH, 0);
        Rpc[t].assign((size_t)NH * NH, 0); Tpc[t].assign((size_t)NH * NH, 0);
        for (int i = 0; i < NH; ++i) {
            const int ra = N + NH + i, rb = i;
            for (int c = 0; c < NH; ++c) {
                Tc[t][(size_t)i * NH + c] = Pm[(size_t)ra * N + c];
                Rc[t][(size_t)i * NH + c] = Pm[(size_t)ra * N + NH + c];
                Rpc[t][(size_t)i * NH + c] = Pm[(size_t)rb * N + c];
                Tpc[t][(size_t)i * NH + c] = Pm[(size_t)rb * N + NH + c];
            }
        }
        double *Es = &out.EsrcT[(size_t)t * L2 * N];
        for (int i = 0; i < NH; ++i)
            for (int col = 0; col < L2; ++col) {
                Es[(size_t)col * N + i] = Qp[(size_t)(N + NH + i) * L2 + col];
                Es[(size_t)col * N + NH + i] = Qp[(size_t)i * L2 + col];
            }
        double *Ps = &out.PhisrcT[(size_t)t * L2 * L2];
        double *Pi = &out.PhiinfT[(size_t)t * N * L2];
        for (int nu = 0; nu < 2; ++nu)
            for (int l = 0; l < L1; ++l) {
                const int row = nu * L1 + l;
                for (int col = 0; col < L2; ++col) {
                    double s = 0.0;
                    for (int n = 0; n < N; ++n)
                        s += P[(size_t)l * N + n] * w[n] * Qp[(size_t)(nu * N + n) * L2 + col];
                    Ps[(size_t)col * L2 + row] = s;
                }
                for (int col = 0; col < N; ++col) {
                    double s = 0.0;
                    for (int n = 0; n < N; ++n)
                        s += P[(size_t)l * N + n] * w[n] * Pm[(size_t)(nu * N + n) * N + col];
                    Pi[(size_t)col * L2 + row] = s;
                }
            }
    }

    return true;
}

bool build_fp_factors_coef(int K, int N, int L, const double *h, const double *sigma_a,
                           const double *sigma_tr, const double *sigma_s, const dvec &mu, const dvec &w,
                           const dvec &A, FPFactors &out, int chunk_hint, int tree_slabs) {
    FPCellTypes ct;
    if (!fp_cell_types(K, N, L, h, sigma_a, sigma_tr, sigma_s, mu, w, A, out, ct)) return false;
    const int NH = N / 2;
    const std::vector<int> &cell_type = ct.cell_type;
    const std::vector<dvec> &Tc = ct.T, &Rc = ct.R, &Rpc = ct.Rp, &Tpc = ct.Tp;
    // chunk length ~ sqrt(K/2) balances the local pass (chunk steps) against
    // the fix pass (up to K/chunk fold steps + chunk steps)
    int chunk = chunk_hint > 0 ? chunk_hint : (int)std::lround(std::sqrt(0.5 * K));
    if (chunk < 4) chunk = 4;
    if (chunk > K) chunk = K;
    out.chunk = chunk;
    out.nchunks = (K + chunk - 1) / chunk;
    if (tree_slabs > 0 && build_fp_tree(K, N, L, tree_slabs, ct, out, out.tree)) {
        // all in out.tree.frag now
        for (dvec *v : {&out.tree.mats, &out.EsrcT, &out.PhisrcT, &out.PhiinfT}) dvec().swap(*v);
        return true;
    }
    out.tree = FPTree();

    // ---- Riccati eliminations from both faces
    const size_t M2 = (size_t)NH * NH;
    const size_t CM = FP_CELL_MATS * M2;
    out.cellmats.assign((size_t)K * CM, 0.0);
    dvec rho_all((size_t)(K + 1) * M2, 0.0), sig(M2, 0.0), tmp(M2), tmp2(M2), Mg(M2);
    for (int j = 0; j < K; ++j) {
        const int t = cell_type[j];
        const double *rho = &rho_all[(size_t)j * M2];
        double *G = &out.cellmats[(size_t)j * CM], *Hm = G + M2;
        // G = T (I - rho R')^{-1}, Hm = G rho, rho_{j+1} = R + Hm T'
        matmul(NH, NH, NH, rho, Rpc[t].data(), tmp.data());
        for (size_t e = 0; e < M2; ++e) Mg[e] = -tmp[e];
        for (int i = 0; i < NH; ++i) Mg[(size_t)i * NH + i] += 1.0;
        if (!invert(NH, Mg.data())) return false;
        matmul(NH, NH, NH, Tc[t].data(), Mg.data(), G);
        matmul(NH, NH, NH, G, rho, Hm);
        matmul(NH, NH, NH, Hm, Tpc[t].data(), tmp.data());
        double *rn = &rho_all[(size_t)(j + 1) * M2];
        for (size_t e = 0; e < M2; ++e) rn[e] = Rc[t][e] + tmp[e];
    }
    for (int j = K - 1; j >= 0; --j) {
        const int t = cell_type[j];
        double *cm = &out.cellmats[(size_t)j * CM];
        double *Gb = cm + 2 * M2, *Hb = cm + 3 * M2, *W = cm + 4 * M2, *Wr = cm + 5 * M2, *S = cm + 6 * M2;
        // sig holds sig_{j+1}: Gb = T' (I - sig R)^{-1}, Hb = Gb sig, sig_j = R' + Hb T
        matmul(NH, NH, NH, sig.data(), Rc[t].data(), tmp.data());
        for (size_t e = 0; e < M2; ++e) Mg[e] = -tmp[e];
        for (int i = 0; i < NH; ++i) Mg[(size_t)i * NH + i] += 1.0;
        if (!invert(NH, Mg.data())) return false;
        matmul(NH, NH, NH, Tpc[t].data(), Mg.data(), Gb);
        matmul(NH, NH, NH, Gb, sig.data(), Hb);
        matmul(NH, NH, NH, Hb, Tc[t].data(), tmp.data());
        for (size_t e = 0; e < M2; ++e) sig[e] = Rpc[t][e] + tmp[e];
        // interface j: W = (I - rho_j sig_j)^{-1}, W rho_j, sig_j
        const double *rho = &rho_all[(size_t)j * M2];
        matmul(NH, NH, NH, rho, sig.data(), tmp.data());
        for (size_t e = 0; e < M2; ++e) W[e] = -tmp[e];
        for (int i = 0; i < NH; ++i) W[(size_t)i * NH + i] += 1.0;
        if (!invert(NH, W)) return false;
        matmul(NH, NH, NH, W, rho, Wr);
        std::copy(sig.begin(), sig.end(), S);
    }

    // ---- chunk products for the chunked recurrences
    out.chunk_fwd.assign((size_t)out.nchunks * M2, 0.0);
    out.chunk_bwd.assign((size_t)out.nchunks * M2, 0.0);
    for (int c = 0; c < out.nchunks; ++c) {
        const int j0 = c * chunk, j1 = std::min(K, j0 + chunk) - 1;
        dvec F(M2, 0.0), B(M2, 0.0);
        for (int i = 0; i < NH; ++i) F[(size_t)i * NH + i] = B[(size_t)i * NH + i] = 1.0;
        for (int j = j0; j <= j1; ++j) {
            matmul(NH, NH, NH, &out.cellmats[(size_t)j * CM], F.data(), tmp.data());
            F.swap(tmp);
        }
        for (int j = j1; j >= j0; --j) {
            matmul(NH, NH, NH, &out.cellmats[(size_t)j * CM + 2 * M2], B.data(), tmp2.data());
            B.swap(tmp2);
        }
        std::copy(F.begin(), F.end(), out.chunk_fwd.begin() + (size_t)c * M2);
        std::copy(B.begin(), B.end(), out.chunk_bwd.begin() + (size_t)c * M2);
    }

    // ---- within-chunk prefix products
    out.psi_fwd.assign((size_t)K * M2, 0.0);
    out.psi_bwd.assign((size_t)K * M2, 0.0);
    for (int c = 0; c < out.nchunks; ++c) {
        const int j0 = c * chunk, j1 = std::min(K, j0 + chunk);
        dvec Pf(M2, 0.0);
        for (int i = 0; i < NH; ++i) Pf[(size_t)i * NH + i] = 1.0;
        for (int j = j0; j < j1; ++j) {
            std::copy(Pf.begin(), Pf.end(), out.psi_fwd.begin() + (size_t)j * M2);
            matmul(NH, NH, NH, &out.cellmats[(size_t)j * CM], Pf.data(), tmp.data());
            Pf.swap(tmp);
        }
        dvec Pb(M2, 0.0);
        for (int i = 0; i < NH; ++i) Pb[(size_t)i * NH + i] = 1.0;
        for (int j = j1 - 1; j >= j0; --j) {
            matmul(NH, NH, NH, &out.cellmats[(size_t)j * CM + 2 * M2], Pb.data(), tmp.data());
            Pb.swap(tmp);
            std::copy(Pb.begin(), Pb.end(), out.psi_bwd.begin() + (size_t)j * M2);
        }
    }

    // ---- chunk-to-chunk transfer products
    // forward: carry_c for c = 0..NC (carry_P = p_K).  ThF_{c,c'} for c' <= c-2.
    const int NC = out.nchunks;
    auto tri = [](int a) { return (size_t)(a - 1) * (a - 2) / 2; };  // first index of row a
    out.theta_fwd.assign(tri(NC + 1) * M2, 0.0);
    for (int c = 2; c <= NC; ++c) {
        // ThF_{c,c'} = Phi_{c-1} ... Phi_{c'+1}; build from c' = c-2 downwards
        dvec Th(M2);
        std::copy(out.chunk_fwd.begin() + (size_t)(c - 1) * M2, out.chunk_fwd.begin() + (size_t)c * M2,
                  Th.begin());
        for (int cp = c - 2; cp >= 0; --cp) {
            std::copy(Th.begin(), Th.end(), out.theta_fwd.begin() + (tri(c) + cp) * M2);
            if (cp > 0) {
                matmul(NH, NH, NH, Th.data(), &out.chunk_fwd[(size_t)cp * M2], tmp.data());
                Th.swap(tmp);
            }
        }
    }
    // backward: carry'_c for c = -1..NC-1 (carry'_{NC-1} = b_K = 0, carry'_{-1} = b_0).
    // Mirror index a = NC-1-c (a = 0..NC): ThB_{c,c'} for c' >= c+2 stored at
    // tri(a) + (NC-1-c') with c' from c+2 .. NC-1.
    out.theta_bwd.assign(tri(NC + 1) * M2, 0.0);
    for (int c = -1; c <= NC - 3; ++c) {
        const int a = NC - 1 - c;
        // ThB_{c,c'} = Phi'_{c+1} ... Phi'_{c'-1}; build from c' = c+2 upwards
        dvec Th(M2);
        std::copy(out.chunk_bwd.begin() + (size_t)(c + 1) * M2, out.chunk_bwd.begin() + (size_t)(c + 2) * M2,
                  Th.begin());
        for (int cp = c + 2; cp <= NC - 1; ++cp) {
            std::copy(Th.begin(), Th.end(), out.theta_bwd.begin() + (tri(a) + (NC - 1 - cp)) * M2);
            if (cp < NC - 1) {
                matmul(NH, NH, NH, Th.data(), &out.chunk_bwd[(size_t)cp * M2], tmp.data());
                Th.swap(tmp);
            }
        }
    }
    return true;
}

// ---------------------------------------------------------------------------
// Doubling tree (see FPTree)
// ---------------------------------------------------------------------------

// A slab alone.  The eliminations take one source and one update launch a run
// on all CUs, a level of the tree is one CU's stream of matrices: few runs and
// cells, past 96 angles (where a level's stream is as long as 128's) and at
// most 128 (past it the eliminations' chains leave LDS).  us an iteration,
// eliminations / tree (two and three runs: means over three cuts):
//   K                   100        150        240        400        640        760
//   N = 104, 1 run    97 / 88   100 / 96  102 / 104  111 / 111  118 / 118  121 / 132
//            2       118 / 122 120 / 123  122 / 129  131 / 141  143 / 146  150 / 149
//   N = 116, 1        97 / 99  101 / 102  103 / 108  112 / 116  120 / 122  125 / 128
//            2       118 / 129 120 / 132  122 / 136  131 / 149  146 / 152  153 / 149
//            3       139 / 131 142 / 137  145 / 142  153 / 156  167 / 166  174 / 161
//   N = 128, 1        91 / 98   93 / 101   96 / 108  104 / 115  111 / 120  127 / 126
//            2       111 / 128 113 / 132  115 / 135  121 / 147  134 / 149  150 / 147
//            3       132 / 131 134 / 134  135 / 139  143 / 155  160 / 165  173 / 159
// K = 64, N = 128, 1 to 3 runs 91 / 75, 111 / 111, 131 / 113; N = 96, K = 240,
// two runs 116 / 106; N = 130, K = 240, two runs 222 / 178.
//
// Slabs together.  A run costs the eliminations no launch then (one for all
// slabs), but they move nine N/2 x N/2 matrices a cell, and slabs of which
// some keep them and some take the tree would run one after the other: all of
// a handle or none, of one padded half-width (one launch).  us an iteration:
//   slabs x K           2 x 70    2 x 200    2 x 500    4 x 70    4 x 200    8 x 70    8 x 200
//   N = 64, 1 run     65 / 57    77 / 62    84 / 88    72 / 58   79 / 63    79 / 61  100 / 77
//           2         69 / 65    80 / 72    86 / 88    78 / 71   82 / 74    82 / 83  103 / 93
//           4         70 / 74    79 / 107   87 / 96    78 / 78   83 / 114   82 / 87  102 / 106
//           8         69 / 81    79 / 89    86 / 107   78 / 85   83 / 94    82 / 99  105 / 129
//   N = 96, 1        106 / 82   117 / 125  145 / 125  107 / 84  132 / 131  118 / 104 225 / 146
//           2        108 / 116  120 / 122  147 / 151  111 / 128 133 / 138  122 / 136 235 / 164
//           4        108 / 136  120 / 136  147 / 152  110 / 142 134 / 137  122 / 162 237 / 156
//   N = 128, 1       103 / 112  112 / 123  170 / 152  104 / 139 146 / 125  134 / 153 250 / 154
//            2       105 / 164  114 / 154  174 / 180  107 / 168 150 / 173  140 / 184 256 / 184
//            8       107 / 144  116 / 165  180 / 207  109 / 147 159 / 178  151 / 155 272 / 281
// N = 48 with 4 runs 77 / 68 (2 x 70) to 92 / 83 (4 x 200); N = 144 with 2
// runs 190 / 187 (2 x 70).  Past eight runs nothing was measured.
bool fp_keeps_eliminations(const std::vector<FPSlabShape> &slabs) {
    if (slabs.empty()) return false;
    const bool wide = slabs[0].N > 64;
    long long cells = 0;
    int runs = 0, least = slabs[0].N;
    for (const FPSlabShape &s : slabs) {
        if (s.N <= 48 || s.N > 128 || (s.N > 64) != wide) return false;
        cells += s.K;
        runs = std::max(runs, s.runs);
        least = std::min(least, s.N);
    }
    if (slabs.size() == 1) {
        const int past = runs == 1 ? 104 : runs == 2 ? 96 : 124;
        return runs <= 3 && least > past && cells > 64 && cells <= 700;
    }
    if (runs > 8) return false;
    if (!wide) return runs >= 4 && cells <= 1600;
    return runs == 1 ? least > 104 && cells <= 600 : cells <= 1000;
}

int fp_runs(int K, int L1, const double *h, const double *sigma_t, const double *sigma_s) {
    int runs = 1;
    for (int j = 1; j < K; ++j)
        if (h[j] != h[j - 1] || (sigma_t && sigma_t[j] != sigma_t[j - 1]) ||
            (sigma_s && !std::equal(sigma_s + (size_t)j * L1, sigma_s + (size_t)(j + 1) * L1, sigma_s + (size_t)(j - 1) * L1)))
            ++runs;
    return runs;
}

// A wave waits for one batch of right operands while the next travels, so a
// product of few rows is as long as its batches are many, and padding to whole
// batches costs less than shorter ones, until the padding is work that fills
// the part.  us a correction in batches of 2, 4 and 8: K = 300, one type,
// N = 10 24.0 / 21.7 / 23.4, N = 20 28.1 / 26.3 / 25.0, N = 34 39.4 / 34.8 /
// 35.5, N = 48 44 / 35.2 / 35.7, N = 72 78 / 59 / 54, N = 104 108 / 84 / 77,
// N = 130 317 / 186 / 132.  Large batches, an iteration, 64 slabs of 300 cells:
// N = 24 122 / 119 / 116, N = 40 199 / 182 / 209, N = 48 263 / 217 / 233, N = 72
// 531 / 437 / 413; 32 of 2048: N = 24 185 / 194 / 192, N = 40 362 / 341 / 388,
// N = 48 394 / 363 / 400, N = 72 986 / 872 / 852.
int fp_tree_nb(int N, long long cells) {
    if (N <= 8) return 2;
    if (N <= 16) return 4;
    if (N <= 24) return cells <= 32768 ? 8 : 2;
    return N > 32 && N <= 48 ? 4 : 8;
}
size_t fp_tree_ld(int nb, int cols) {
    const int kb = 4 * nb;
    return (size_t)(cols + kb - 1) / kb * kb + 1;
}

dvec fp_tree_fragments(const double *B, int K, int cols, int nb) {
    const int KS = (K + 4 * nb - 1) / (4 * nb) * nb, CT = (cols + 15) / 16;
    dvec out((size_t)CT * KS * 64, 0.0);
    for (int c = 0; c < CT; ++c)
        for (int p = 0; p < KS / 2; ++p)
            for (int l = 0; l < 64; ++l)
                for (int e = 0; e < 2; ++e) {
                    const int k = 8 * p + 4 * e + l / 16, col = 16 * c + l % 16;
                    if (k < K && col < cols)
                        out[(((size_t)c * (KS / 2) + p) * 64 + l) * 2 + e] = B[(size_t)k * cols + col];
                }
    return out;
}

// doubles of LDS of a chunk of c leaves: interface rows, the second set of
// rows of a root chunk, and the moment-difference rows of a leaf stage
static size_t tree_lds(int nb, int N, int L2, int c, bool leaf, bool root) {
    return (size_t)(root ? 2 : 1) * (c + 1) * fp_tree_ld(nb, N) + (leaf ? (size_t)c * fp_tree_ld(nb, L2) : 0);
}

// Fragments and per-wave unit lists of a built tree.
static bool tree_records(int N, int L2, const FPFactors &maps, FPTree &out) {
    const int nb = out.nb, nt = maps.ntypes;
    const int ksN = (N + 4 * nb - 1) / (4 * nb) * nb, ksL = (L2 + 4 * nb - 1) / (4 * nb) * nb;
    const int ctN = (N + 15) / 16, ctU = (2 * N + 15) / 16, ctL = (L2 + 15) / 16;
    // fragment offsets, in blocks of 64 doubles
    const size_t up = (size_t)ctU * ksN, dn = (size_t)ctN * ksN;
    const size_t src0 = (size_t)out.nclasses * (up + dn), upd0 = src0 + (size_t)nt * ctN * ksL;
    const size_t inf0 = upd0 + (size_t)nt * ctL * ksL, all = inf0 + (size_t)nt * ctL * ksN;
    if (all > 0x7fffffffu) return false;
    out.frag.clear();
    out.frag.reserve(all * 64);
    auto put = [&](const double *B, int K, int cols) {
        const dvec v = fp_tree_fragments(B, K, cols, nb);
        out.frag.insert(out.frag.end(), v.begin(), v.end());
    };
    const size_t N2 = (size_t)N * N;
    for (int k = 0; k < out.nclasses; ++k) {
        put(&out.mats[k * 3 * N2], N, 2 * N);
        put(&out.mats[k * 3 * N2 + 2 * N2], N, N);
    }
    for (int t = 0; t < nt; ++t) put(&maps.EsrcT[(size_t)t * L2 * N], L2, N);
    for (int t = 0; t < nt; ++t) put(&maps.PhisrcT[(size_t)t * L2 * L2], L2, L2);
    for (int t = 0; t < nt; ++t) put(&maps.PhiinfT[(size_t)t * N * L2], N, L2);
    for (FPTreeStage &s : out.stages) {
        std::vector<std::vector<int>> recs((size_t)s.chunks * kTreeWaves);
        size_t most = 0;
        for (int p = 0; p < s.chunks; ++p) {
            const int *lv = &out.lv[(size_t)out.chunk_list[s.first_chunk + p] * kTreeLv];
            for (int w = 0; w < kTreeWaves; ++w) {
                std::vector<int> ends, units;
                // the units (pass, column tile) of a phase, dealt to the waves in turn
                auto phase = [&](int l, int ct, auto &&offset, int entries) {
                    int u = 0;
                    for (int q = lv[l]; q < lv[l + 1]; ++q)
                        for (int c = 0; c < ct; ++c, ++u) {
                            if (u % kTreeWaves != w) continue;
                            const FPPass &ps = out.passes[q];
                            for (int e = 0; e < entries; ++e) {
                                units.push_back((int)offset(ps.cls, c, e));
                                units.push_back(ps.first | (ps.rows << 8) | (c << 16));
                            }
                        }
                    ends.push_back((int)units.size() / 2);
                };
                if (s.leaf)
                    phase(0, ctN, [&](int cls, int c, int) { return src0 + ((size_t)cls * ctN + c) * ksL; }, 1);
                else
                    ends.push_back(0);
                for (int l = 1; l <= s.levels; ++l)
                    phase(l, ctU, [&](int cls, int c, int) { return cls * (up + dn) + (size_t)c * ksN; }, 1);
                for (int l = s.levels; l >= 1; --l)
                    phase(l, ctN, [&](int cls, int c, int) { return cls * (up + dn) + up + (size_t)c * ksN; }, 1);
                if (s.leaf)
                    phase(0, ctL, [&](int cls, int c, int e) {
                        return e == 0 ? upd0 + ((size_t)cls * ctL + c) * ksL : inf0 + ((size_t)cls * ctL + c) * ksN;
                    }, 2);
                else
                    ends.push_back((int)units.size() / 2);
                if (units.empty()) units = {0, 1 << 8};
                // one more entry, so that the last unit has a successor to request
                units.push_back(units[units.size() - 2]);
                units.push_back(units[units.size() - 2]);
                if ((int)ends.size() > kTreeHdr || units.size() / 2 > (size_t)kTreeMaxUnits) return false;
                std::vector<int> &r = recs[(size_t)p * kTreeWaves + w];
                for (int i = 0; i < kTreeHdr; ++i) r.push_back(ends[std::min<size_t>(i, ends.size() - 1)]);
                r.insert(r.end(), units.begin(), units.end());
                most = std::max(most, units.size());
            }
        }
        s.rec_stride = kTreeHdr + (int)most;
        s.rec0 = out.records.size();
        out.records.resize(s.rec0 + recs.size() * s.rec_stride, 0);
        for (size_t i = 0; i < recs.size(); ++i)
            std::copy(recs[i].begin(), recs[i].end(), out.records.begin() + s.rec0 + i * s.rec_stride);
    }
    return true;
}

// Cuts the levels into stages.  cls0: the cells' types, icls[l]: the classes
// of level l's interfaces.
static bool tree_stages(int K, int N, int L2, int slabs, const std::vector<int> &cls0,
                        const std::vector<std::vector<int>> &icls, FPTree &out) {
    const int nb = out.nb, top = (int)icls.size() - 1;
    const int ksN = (N + 4 * nb - 1) / (4 * nb) * nb, ksL = (L2 + 4 * nb - 1) / (4 * nb) * nb;
    const int ctN = (N + 15) / 16, ctU = (2 * N + 15) / 16, ctL = (L2 + 15) / 16;
    // a product of so many rows with ct column tiles over ks k-steps
    auto product = [](int rows, int ct, int ks) {
        const double mfma = (double)ct * ks * (rows > 8 ? 150 : rows > 4 ? 60 : 40) * kTreeUsPerMfmaClk;
        return std::max(mfma, (double)ct * ks * 64 * 8 * kTreeUsPerByte);
    };
    // one launch's time over levels lo + 1 .. hi: the longest chunk, times the
    // rounds of blocks when there are more chunks than CUs; < 0: not possible
    auto stage = [&](int lo, int hi) -> double {
        const bool leaf = lo == 0, root = hi == top;
        const int n = (int)(((size_t)K + ((size_t)1 << lo) - 1) >> lo), c = 1 << (hi - lo);
        const int chunks = (n + c - 1) / c, rows = std::min(c, n);
        if (rows > kTreeMaxRows || 2 * (hi - lo) + 2 > kTreeHdr) return -1.0;
        if (tree_lds(nb, N, L2, rows, leaf, root) * sizeof(double) > kTreeLdsBytes) return -1.0;
        double up = 0.0, down = 0.0, whole = 0.0;
        for (int p = 0; p < chunks; ++p) {
            double u = 0.0, d = 0.0;
            int units = 0, passes = 0;
            auto level = [&](const std::vector<int> &cls, int i0, int i1, auto &&add) {
                for (int i = i0; i < i1;) {
                    int e = i + 1;
                    while (e < i1 && e - i < 16 && cls[e] == cls[i]) ++e;
                    add(e - i);
                    ++passes;
                    i = e;
                }
            };
            for (int l = leaf ? 0 : lo + 1; l <= hi; ++l) {
                const size_t per = (size_t)1 << (hi - l), all = l ? icls[l].size() : cls0.size();
                const std::vector<int> &cls = l ? icls[l] : cls0;
                const int i0 = (int)std::min(all, p * per);
                int i1 = (int)std::min(all, (p + 1) * per);
                if (l && i1 > i0 && cls[i1 - 1] < 0) --i1;  // the last node has one child
                u += kTreeUsPerLevel;
                d += kTreeUsPerLevel;
                level(cls, i0, i1, [&](int r) {
                    u += l ? product(r, ctU, ksN) : product(r, ctN, ksL);
                    d += l ? product(r, ctN, ksN) : product(r, ctL, ksL + ksN);
                    units += l ? ctU + ctN : ctN + 2 * ctL;
                });
            }
            if (passes > kTreeMaxPasses || (units + 7 * (2 * (hi - lo) + 2)) / kTreeWaves + 2 > kTreeMaxUnits) return -1.0;
            up = std::max(up, u);
            down = std::max(down, d);
            whole = std::max(whole, u + d);
        }
        const double rows_us = (double)rows * (N + (leaf ? 2 * L2 : 0)) * 8 * kTreeUsPerByte;
        // more chunks than CUs: rounds, which overlap where two blocks fit a CU
        const bool two = tree_lds(nb, N, L2, rows, leaf, root) * sizeof(double) <= kTreeLdsTwo;
        const double rounds = std::max(1.0, (double)chunks * slabs / kTreeCus * (two ? 0.7 : 1.0));
        return root ? kTreeUsPerLaunch + rounds * (whole + rows_us)
                    : 2 * kTreeUsPerLaunch + rounds * (up + down + 2 * rows_us);
    };
    // best[s][lo]: the levels above lo in at most s + 1 stages, the next one up to cut[s][lo]
    std::vector<std::vector<double>> best(kTreeMaxStages, std::vector<double>(top + 1, -1.0));
    std::vector<std::vector<int>> cut(kTreeMaxStages, std::vector<int>(top + 1, top));
    // (at least two levels a stage: the later stages' interfaces fit the work array)
    for (int lo = top ? top - 1 : 0; lo >= 0; --lo)
        for (int hi = std::min(top, lo + 2); hi <= std::min(top, lo + kTreeMaxLevels); ++hi) {
            const double t = stage(lo, hi);
            if (t < 0.0) continue;
            for (int s = 0; s < kTreeMaxStages; ++s) {
                if (hi < top && (s == 0 || best[s - 1][hi] < 0.0)) continue;
                const double all = t + (hi < top ? best[s - 1][hi] : 0.0);
                if (best[s][lo] < 0.0 || all < best[s][lo]) {
                    best[s][lo] = all;
                    cut[s][lo] = hi;
                }
            }
        }
    if (best[kTreeMaxStages - 1][0] < 0.0) return false;
    size_t later = 0;
    for (int lo = 0, s = kTreeMaxStages - 1;; --s) {
        FPTreeStage g;
        const int hi = cut[s][lo];
        g.n = (int)(((size_t)K + ((size_t)1 << lo) - 1) >> lo);
        g.leaf = lo == 0;
        g.levels = hi - lo;
        g.c = 1 << g.levels;
        g.chunks = (g.n + g.c - 1) / g.c;
        if (lo) later += (size_t)(g.n + 1) * N;
        out.stages.push_back(g);
        lo = hi;
        if (hi == top) break;
    }
    // the later stages' interfaces share one (K + 1) N / 2 work array
    return later <= (size_t)(K + 1) * (N / 2);
}

bool build_fp_tree(int K, int N, int L, int slabs, const FPCellTypes &ct, const FPFactors &maps, FPTree &out) {
    const int NH = N / 2, L2 = 2 * (L + 1);
    const size_t M2 = (size_t)NH * NH, N2 = (size_t)N * N;
    out = FPTree();
    out.nb = fp_tree_nb(N, (long long)slabs * K);
    const int ntypes = (int)ct.T.size();
    // node classes: operators (T, R, R', T') per class, classes of equal
    // child pairs shared
    struct Node {
        dvec T, R, Rp, Tp;
    };
    std::vector<Node> ops;
    for (int t = 0; t < ntypes; ++t) ops.push_back(Node{ct.T[t], ct.R[t], ct.Rp[t], ct.Tp[t]});
    std::map<std::pair<int, int>, int> pair_of;  // (left, right) -> node class
    std::map<std::vector<int>, int> list_of;
    dvec X(M2), t0(M2), t1(M2), t2(M2), t3(M2);
    auto combine = [&](int a, int b) -> int {
        auto it = pair_of.find({a, b});
        if (it != pair_of.end()) return it->second;
        Node nw;
        for (dvec *v : {&nw.T, &nw.R, &nw.Rp, &nw.Tp}) v->assign(M2, 0.0);
        const Node &A = ops[a], &B = ops[b];
        // X = (I - R_A R'_B)^{-1}
        matmul(NH, NH, NH, A.R.data(), B.Rp.data(), t0.data());
        for (size_t e = 0; e < M2; ++e) X[e] = -t0[e];
        for (int i = 0; i < NH; ++i) X[(size_t)i * NH + i] += 1.0;
        if (!invert(NH, X.data())) return -1;
        // M1 = [[X, X R_A], [R'_B X, I + R'_B X R_A]]
        dvec XR(M2), RX(M2), RXR(M2);
        matmul(NH, NH, NH, X.data(), A.R.data(), XR.data());
        matmul(NH, NH, NH, B.Rp.data(), X.data(), RX.data());
        matmul(NH, NH, NH, RX.data(), A.R.data(), RXR.data());
        for (int i = 0; i < NH; ++i) RXR[(size_t)i * NH + i] += 1.0;
        // right operands: up [N][2N] = [M1^T | (diag(T_B, T'_A) M1)^T], down [N][N] = (M1 diag(T_A, T'_B))^T
        const size_t base = out.mats.size();
        out.mats.resize(base + 3 * N2);
        double *U = &out.mats[base], *D = U + 2 * N2;
        auto put_up = [&](const dvec &M, int r0, int c0, int off) {  // rows r0.. of M1 block at columns c0..
            for (int r = 0; r < NH; ++r)
                for (int c = 0; c < NH; ++c) U[(size_t)(c0 + c) * 2 * N + off + r0 + r] = M[(size_t)r * NH + c];
        };
        put_up(X, 0, 0, 0);
        put_up(XR, 0, NH, 0);
        put_up(RX, NH, 0, 0);
        put_up(RXR, NH, NH, 0);
        dvec P(M2);
        auto put_dn = [&](const dvec &M, int r0, int c0) {
            for (int r = 0; r < NH; ++r)
                for (int c = 0; c < NH; ++c) D[(size_t)(c0 + c) * N + r0 + r] = M[(size_t)r * NH + c];
        };
        matmul(NH, NH, NH, B.T.data(), X.data(), t0.data());     // T_B X
        put_up(t0, 0, 0, N);
        matmul(NH, NH, NH, B.T.data(), XR.data(), P.data());     // T_B X R_A
        put_up(P, 0, NH, N);
        matmul(NH, NH, NH, A.Tp.data(), RX.data(), t1.data());   // T'_A R'_B X
        put_up(t1, NH, 0, N);
        matmul(NH, NH, NH, A.Tp.data(), RXR.data(), t2.data());  // T'_A (I + R'_B X R_A)
        put_up(t2, NH, NH, N);
        // the node's operators
        matmul(NH, NH, NH, t0.data(), A.T.data(), nw.T.data());
        matmul(NH, NH, NH, P.data(), B.Tp.data(), t3.data());
        for (size_t e = 0; e < M2; ++e) nw.R[e] = B.R[e] + t3[e];
        matmul(NH, NH, NH, t1.data(), A.T.data(), t3.data());
        for (size_t e = 0; e < M2; ++e) nw.Rp[e] = A.Rp[e] + t3[e];
        matmul(NH, NH, NH, t2.data(), B.Tp.data(), nw.Tp.data());
        matmul(NH, NH, NH, X.data(), A.T.data(), P.data());
        put_dn(P, 0, 0);
        matmul(NH, NH, NH, XR.data(), B.Tp.data(), P.data());
        put_dn(P, 0, NH);
        matmul(NH, NH, NH, RX.data(), A.T.data(), P.data());
        put_dn(P, NH, 0);
        matmul(NH, NH, NH, RXR.data(), B.Tp.data(), P.data());
        put_dn(P, NH, NH);
        ops.push_back(std::move(nw));
        const int id = (int)ops.size() - 1;
        pair_of.emplace(std::make_pair(a, b), id);
        return id;
    };
    // class of the interface inside each node, level by level (icls[l][i]);
    // the node classes of level l are cls_at[l]
    int top = 0;
    while (((size_t)1 << top) < (size_t)K) ++top;
    std::vector<std::vector<int>> icls(top + 1), cls_at(top + 1);
    cls_at[0] = ct.cell_type;
    for (int l = 1; l <= top; ++l) {
        const std::vector<int> &cur = cls_at[l - 1];
        const int m = (int)cur.size();
        std::vector<int> &up = cls_at[l];
        up.assign((m + 1) / 2, 0);
        icls[l].assign((m + 1) / 2, -1);
        for (int i = 0; i < (m + 1) / 2; ++i) {
            if (2 * i + 1 < m) {
                const int id = combine(cur[2 * i], cur[2 * i + 1]);
                if (id < 0) return false;
                up[i] = id;
                icls[l][i] = id - ntypes;
            } else {
                up[i] = cur[2 * i];
            }
        }
    }
    if (!tree_stages(K, N, L2, slabs, cls_at[0], icls, out)) return false;
    int lo = 0;
    for (FPTreeStage &s : out.stages) {
        const int n = s.n;
        // passes per chunk: runs of at most 16 rows of one class, by level
        // (level 0: the leaf cells by type)
        s.first_chunk = (int)out.chunk_list.size();
        for (int p = 0; p < s.chunks; ++p) {
            const int c0 = p * s.c, nc = std::min(s.c, n - c0);
            std::vector<int> key;
            std::vector<FPPass> ps;
            std::vector<int> lv;
            for (int l = 0; l <= s.levels; ++l) {
                lv.push_back((int)ps.size());
                if (l == 0 && !s.leaf) continue;
                const int half = l ? 1 << (l - 1) : 0, step = 1 << l;
                for (int r = 0; half + step * r < nc; ++r) {
                    const int c = l ? icls[lo + l][(c0 >> l) + r] : cls_at[0][c0 + r];
                    if ((int)ps.size() > lv[l] && ps.back().cls == c && ps.back().rows < 16)
                        ++ps.back().rows;
                    else
                        ps.push_back(FPPass{(short)r, 1, c});
                }
            }
            lv.push_back((int)ps.size());
            if (ps.size() > (size_t)kTreeMaxPasses) return false;
            for (const FPPass &q : ps) {
                key.push_back(q.first);
                key.push_back(q.rows);
                key.push_back(q.cls);
            }
            key.insert(key.end(), lv.begin(), lv.end());
            auto it = list_of.find(key);
            if (it == list_of.end()) {
                it = list_of.emplace(key, (int)list_of.size()).first;
                const int base = (int)out.passes.size();
                out.passes.insert(out.passes.end(), ps.begin(), ps.end());
                for (int l = 0; l < kTreeLv; ++l) out.lv.push_back(base + lv[std::min<size_t>(l, lv.size() - 1)]);
            }
            out.chunk_list.push_back(it->second);
        }
        lo += s.levels;  // the chunks are the next stage's leaves
    }
    out.nclasses = (int)pair_of.size();
    return tree_records(N, L2, maps, out);
}

}  // namespace snfpsa
