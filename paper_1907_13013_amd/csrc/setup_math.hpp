// Host-side FP64 setup math of the slab S_N / FPSA library: quadrature,
// Legendre tables, angular Laplacians and the factorisation of the LD x S_N
// Fokker-Planck correction operator.  Runs once per sn_setup (the paper
// excludes this setup from its solver timings, Sec. 4).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace snfpsa {

using dvec = std::vector<double>;

// Gauss-Legendre rule on [-1,1], nodes ascending, weights summing to 2.
void gauss_legendre(int N, dvec &mu, dvec &w);

// P[l*N + n] = P_l(mu_n) for l = 0..L.
dvec legendre_table(int N, int L, const dvec &mu);

// Angular Laplacians of Sec. 2.2 (row-major N x N).
//   WFD: eq:fp-wdd / eq:sph-weights / eq:w_wfd with gamma_{1/2} = 0 and the
//        normalisation nu = -2 (so gamma_{N+1/2} = 0 and gamma > 0 inside).
//   MPD: eq:fp-mpd, F = V^{-1} diag(-l(l+1)) V; for Gauss-Legendre V^{-1} is
//        the moment-to-discrete map M_{n,l} = (2l+1)/2 P_l(mu_n) exactly.
dvec wfd_laplacian(int N, const dvec &mu, const dvec &w);
dvec mpd_laplacian(int N, const dvec &mu, const dvec &w);

// Factorised LD x S_N Fokker-Planck operator of one slab.
//
// Cell equations (both LD test functions, all N angles at once):
//   D_j u_j = Mass_j r_j + J [a_j ; b_{j+1}],   u_j = [U_L(0..N-1); U_R(0..N-1)]
// with removal T = sigma_a I - (sigma_tr/2) A and inflows a_j (the N/2
// positive-cosine fluxes entering cell j through its left face) and b_{j+1}
// (the N/2 negative-cosine fluxes entering through its right face); zero
// inflow at both slab faces (a_0 = 0, b_K = 0).  Eliminating the cell
// interiors leaves, per cell, the interface relations
//   a_{j+1} = T_j a_j + R_j b_{j+1} + s+_j,   b_j = R'_j a_j + T'_j b_{j+1} + s-_j.
// They are solved by two independent Riccati eliminations and a local
// combination at each interface k:
//   from the left   a_k = rho_k b_k + p_k,    p_{j+1} = G_j p_j + Hm_j s-_j + s+_j
//   from the right  b_k = sig_k a_k + q_k,    q_j = Gb_j q_{j+1} + Hb_j s+_j + s-_j
//   a_k = W_k p_k + (W rho)_k q_k,  b_k = sig_k a_k + q_k,  W_k = (I - rho_k sig_k)^{-1}
// with rho_0 = 0, p_0 = 0, sig_K = 0, q_K = 0 and
//   G_j = T_j (I - rho_j R'_j)^{-1},   Hm_j = G_j rho_j,   rho_{j+1} = R_j + Hm_j T'_j,
//   Gb_j = T'_j (I - sig_{j+1} R_j)^{-1}, Hb_j = Gb_j sig_{j+1}, sig_j = R'_j + Hb_j T_j.
// All matrices are fixed by the operator and precomputed here; only the
// vectors change per application.
constexpr int FP_CELL_MATS = 7;  // per cell: G, Hm, Gb, Hb, W, W rho, sig

// Doubling tree.  The interface relations of a
// run of cells compose like those of one cell: for neighbouring runs A, B
// with responses (T, R, R', T') and outgoing sources (s+, s-) under zero
// inflow, the interface between them carries
//   [a; b] = M1 [s+_A; s-_B] + M1 diag(T_A, T'_B) [a_in; b_in],
//   M1 = [[X, X R_A], [R'_B X, I + R'_B X R_A]],  X = (I - R_A R'_B)^{-1},
// and the pair's outgoing sources are s+_B + T_B a and s-_A + T'_A b (zero
// inflow).  Going up a binary tree over the cells gives every interface's
// zero-inflow value and the slab's outgoing flux, going down adds each
// node's inflow.  Nodes with equal children share their matrices, so a slab
// of one cell type needs about two matrix sets per level where the
// eliminations above need nine N/2 x N/2 matrices per cell, and every level
// is a product of all its interfaces' rows with shared matrices (a slab whose
// cells all differ has a matrix set per node: three N x N).  The dependent
// chain is two products a level where the eliminations' is sqrt(K) steps, and
// every launch takes all cell types at once.
//
// The tree is cut into stages of chunks (c leaves each, a power of two): a
// chunk goes up its levels on its own, the chunks are the next stage's
// leaves, and the last stage is one chunk (the root).  The cut is the one of
// the least predicted time (kTreeUs...): short chunks spread the levels over
// the CUs, long ones save launches, and each level of a chunk streams its
// classes' matrices into one CU.
struct FPCellTypes {
    std::vector<int> cell_type;
    std::vector<dvec> T, R, Rp, Tp;   // [ntypes] NH x NH interface responses
};
// Work of one chunk: at level l (0: the leaf cells), `rows` rows from row
// `first` on take the matrices of class (level 0: cell type) cls.  Row i of
// level l is the interface 2^(l-1) + 2^l i of the chunk.
struct FPPass {
    short first, rows;
    int cls;
};
struct FPTreeStage {
    int n = 0, c = 0, chunks = 0, levels = 0, leaf = 0;
    int first_chunk = 0;              // into FPTree::chunk_list
    size_t rec0 = 0;                  // the stage's records (FPTree::records), ints
    int rec_stride = 0;
};
constexpr int kTreeMaxStages = 5, kTreeLv = 12, kTreeMaxPasses = 128;
constexpr int kTreeWaves = 8;         // waves of a chunk's block
constexpr int kTreeHdr = 20, kTreeMaxUnits = 128;
constexpr int kTreeMaxRows = 255, kTreeMaxLevels = 8;
constexpr size_t kTreeLdsBytes = 148 << 10, kTreeLdsTwo = 78 << 10;
// Cost model of the cut into stages (microseconds): a launch with its gap, a
// level's barriers and bookkeeping, a byte of matrices into one CU (measured
// 100 to 134 GB/s), a cycle of FP64 MFMA on one of a CU's four SIMDs at 2.39 GHz.
constexpr double kTreeUsPerLaunch = 4.5, kTreeUsPerLevel = 0.7, kTreeUsPerByte = 1.0 / 110e3,
                 kTreeUsPerMfmaClk = 1.0 / (4 * 2390.0);
constexpr int kTreeCus = 256;
struct FPTree {
    std::vector<FPTreeStage> stages;  // empty: no tree
    int nb = 0;                       // fp_tree_nb
    int nclasses = 0;
    dvec mats;                        // [nclasses]: up [N][2N], then down [N][N]
    std::vector<FPPass> passes;
    std::vector<int> lv;              // [lists][kTreeLv] first pass of each level
    std::vector<int> chunk_list;      // per stage and chunk: its list
    // right operands in the kernels' fragment order: per class up [N][2N] and
    // down [N][N], then per cell type the source, moment and inflow maps
    dvec frag;
    // per stage, chunk and wave: the ends of the wave's units by phase (cells,
    // up 1 .. levels, down levels .. 1, update; kTreeHdr ints), then the
    // units (fragment offset in 64 doubles, first row | rows << 8 | column
    // tile << 16), one unit (pass, column tile) after the other
    std::vector<int> records;
};
int fp_tree_nb(int N, long long cells);  // k-steps of 4 per batch of right operands; cells: of all slabs
size_t fp_tree_ld(int nb, int cols);     // LDS row stride of left operands of so many columns
// [K][cols] in the kernels' fragment order (see FPTreeArgs)
dvec fp_tree_fragments(const double *B, int K, int cols, int nb);

struct FPFactors {
    int K = 0, N = 0, L = 0, NH = 0;
    int chunk = 0, nchunks = 0;
    bool folded_sigma_s = true;       // EsrcT / PhisrcT include the cell's sigma_s
    // per cell j (interface j for W, W rho, sig): FP_CELL_MATS matrices NH x NH
    dvec cellmats;                    // [K][FP_CELL_MATS][NH][NH]
    // chunk products: forward G_{j1}...G_{j0}, backward Gb_{j0}...Gb_{j1}
    dvec chunk_fwd, chunk_bwd;        // [nchunks][NH][NH]
    // Parallel completion of the chunked recurrences.  With p_loc / q_loc
    // the chain values of a chunk started from a zero carry:
    //   p_j = p_loc_j + PsiF_j carry_c,  PsiF_j = G_{j-1} ... G_{j0} (I at j0)
    //   q_j = q_loc_j + PsiB_j carry'_c, PsiB_j = Gb_j ... Gb_{j1-1}
    //   carry_c  = sum_{c'<c} ThF_{c,c'} e_{c'},  ThF_{c,c'} = Phi_{c-1}...Phi_{c'+1}
    //   carry'_c = sum_{c'>c} ThB_{c,c'} e'_{c'}, ThB_{c,c'} = Phi'_{c+1}...Phi'_{c'-1}
    // (carry_c = p at the first interface of chunk c, carry'_c = q at the
    // interface after its last cell; the nearest-neighbour terms are I).
    dvec psi_fwd, psi_bwd;            // [K][NH][NH]
    dvec theta_fwd;                   // ThF_{c,c'} for 0 <= c' <= c-2, c = 2..nchunks,
                                      //   at index (c-1)(c-2)/2 + c'
    dvec theta_bwd;                   // ThB_{c,c'} for c+2 <= c' <= nchunks-1, c = -1..nchunks-3,
                                      //   stored like ThF with c -> nchunks-1-c
    // cell types (runs of identical cells): type index + per-type matrices
    std::vector<int32_t> seg_begin;   // [nseg+1] cell ranges of equal type
    std::vector<int32_t> seg_type;    // [nseg]
    int ntypes = 0;
    // per type, stored as GEMM right operands (row-major K x Ncols):
    //   EsrcT  [2(L+1)][N]     source of the interface problem: s = [s+; s-]
    //   PhisrcT[2(L+1)][2(L+1)] moments of the zero-inflow cell solution
    //   PhiinfT[N][2(L+1)]      moments of the response to [a_j; b_{j+1}]
    dvec EsrcT, PhisrcT, PhiinfT;
    FPTree tree;
};

// A slab of a handle for the choice between the two: cells, angles, and runs
// of equal cells (fp_runs; slab-mean coefficients: of equal widths, sigma_t
// and sigma_s null).
struct FPSlabShape {
    int K, N, runs;
};
int fp_runs(int K, int L1, const double *h, const double *sigma_t, const double *sigma_s);
// Whether the slabs of a handle keep the eliminations (tree_slabs = 0 below).
bool fp_keeps_eliminations(const std::vector<FPSlabShape> &slabs);

// false: use the eliminations (a singular pair, or no cut fits).
// maps: the cell maps of the types (FPFactors::EsrcT, PhisrcT, PhiinfT).
bool build_fp_tree(int K, int N, int L, int slabs, const FPCellTypes &ct, const FPFactors &maps, FPTree &out);

// sigma_s is [K][L+1] for this slab; sigma_a = sigma_t - sigma_s0,
// sigma_tr = sigma_s0 - sigma_s1.  Returns false if a cell block is
// singular.  The FPSA residual's scattering matrix is folded into the
// source maps (EsrcT, PhisrcT act on phi_half - phi_old).  With
// tree_slabs > 0 (slabs solved together), a slab gets its doubling tree,
// whose frag holds all matrices and cell maps (the other arrays are given
// back), instead of the eliminations' matrices (tree.stages is empty otherwise).
bool build_fp_factors(int K, int N, int L, const double *h, const double *sigma_t,
                      const double *sigma_s, const dvec &mu, const dvec &w,
                      const dvec &A, FPFactors &out, int chunk_hint = 0,
                      int tree_slabs = 0);

// The same from the removal coefficients of F directly: sigma_a, sigma_tr
// [K].  sigma_s (nullable) as above; null leaves the scattering out of the
// source maps, which then act on Sigma (phi_half - phi_old) formed by the
// caller, and cell types depend on (h, sigma_a, sigma_tr) only.
bool build_fp_factors_coef(int K, int N, int L, const double *h, const double *sigma_a,
                           const double *sigma_tr, const double *sigma_s, const dvec &mu,
                           const dvec &w, const dvec &A, FPFactors &out, int chunk_hint = 0,
                           int tree_slabs = 0);

}  // namespace snfpsa
