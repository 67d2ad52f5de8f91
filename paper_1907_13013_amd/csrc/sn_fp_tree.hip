// Fokker-Planck correction by the doubling tree of setup_math.hpp
// (eq:correct with F of eq:fpop):
//
//   s = ((phi_half - phi_old) [.* sigma]) E          leaf sources, per cell
//   up the levels: every interface's zero-inflow value, the chunk's outgoing flux
//   down the levels: the interfaces' values
//   phi_new = phi_half + (...) Phi_src + (a_j | b_{j+1}) Phi_inf  (+ stopping test)
//
// An interface's row is (a_j | b_j), N doubles: while going up, row j holds
// the outgoing sources that meet there (s+ of the run ending at j, s- of the
// run starting at j), which is exactly the left operand of the interface's
// own level; its products are the interface's zero-inflow value and what the
// node adds to the rows at its two ends.  So a chunk's whole ascent runs in
// one LDS array with one barrier per level, and no operand is ever copied.
// All products are FP64 MFMA 16x16x4 (operand layout as in gemm_f64_mfma) of
// 16 interface rows with matrices shared by every node of a class, read from
// L2: a level of a pass of 16 rows takes N / 4 products per 16 columns.
//
// What bounds it: a level is a barrier, its bookkeeping and a stream of N x 2N
// (up) or N x N (down) doubles per class into the chunk's one CU, about 1.3
// and 1.0 us for one class at N = 64; a launch is about 3 us more.  Large
// batches are bounded by issue (7 vector and 4 scalar instructions per MFMA)
// and latency: two blocks of 8 waves per CU, the matrix cores busy a quarter
// of the time.  32 slabs of 2048 cells, N = 64 (us, all launches): 326 in
// chunks of 16 cells, 308 of 64 (one block per CU), 272 of 32.
// Measured per correction against the eliminations' kernels (us): K = 200,
// N = 8 17 (25); K = 2000, N = 64 48 (57); K = 2500, N = 64, 8 types 85
// (153); K = 512, N = 64, 24 types 71 (310); 2000 cells of N = 64, no two
// alike, 197 (25000).
#include <algorithm>

#include "sn_device.hpp"

namespace snfpsa {

constexpr int FPT_W = kFptWaves, FPT_T = 64 * FPT_W;

enum : int {
    FPT_LEAF = 1,    // the leaves are cells: their sources from the moment differences
    FPT_UP = 2,
    FPT_ROOT = 4,    // the chunk is the slab: zero inflow, straight down again
    FPT_DOWN = 8,
    FPT_UPDATE = 16  // the corrected moments (and the stopping test)
};

// Right operands are stored in fragment order (see FPTreeArgs): the lane's
// values of two k-steps are one 16-byte word, a step pair of a column tile
// 1 KB contiguous over the wave.
typedef double d2 __attribute__((ext_vector_type(2)));

// step pairs [p, p + NB / 2) of a column tile's fragments (frag: the lane's
// first word)
template <int NB>
__device__ __forceinline__ void fpt_fetch(const d2 *frag, int p, d2 (&b)[NB / 2]) {
#pragma unroll
    for (int u = 0; u < NB / 2; ++u) b[u] = frag[(p + u) * 64];
}

// NB k-steps of a left operand row from k-step u0 on: columns below split
// from pa, the others from pb.
template <int NB>
__device__ __forceinline__ void fpt_row(const double *pa, const double *pb, int split, int u0, double (&a)[NB]) {
    const int kl = (threadIdx.x & 63) >> 4;
    const double *p = 4 * u0 >= split ? pb : pa;
    if (4 * u0 >= split || 4 * (u0 + NB) <= split) {
        p += 4 * u0 + kl;
#pragma unroll
        for (int u = 0; u < NB; ++u) a[u] = p[4 * u];
    } else {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int k = 4 * (u0 + u) + kl;
            a[u] = (k < split ? pa : pb)[k];
        }
    }
}

// acc += the rows (pa, pb) times a column tile's fragments over KS k-steps (a
// multiple of NB).  b holds the fragments' first batch on entry and the
// first batch of `next` on exit: each product ends by requesting what follows
// it, so operands travel while results are stored and the block meets.
template <int NB>
__device__ __forceinline__ void fpt_mma(d4 &acc, const double *pa, const double *pb, int split, int KS,
                                        const d2 *frag, const d2 *next, d2 (&b)[NB / 2]) {
    for (int u0 = 0; u0 < KS; u0 += NB) {
        double a[NB];
        fpt_row<NB>(pa, pb, split, u0, a);
#pragma unroll
        for (int u = 0; u < NB; ++u)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], (u & 1) ? b[u / 2].y : b[u / 2].x, acc, 0, 0, 0);
        const bool more = u0 + NB < KS;
        fpt_fetch<NB>(more ? frag : next, more ? (u0 + NB) / 2 : 0, b);
    }
}

// The same for up to eight rows (pa0, pb0), (pa1, pb1: rows 4 .. 7, with two)
// in MFMA 4x4x4, its four blocks on four columns each, which reads the same
// fragments and A lanes (row r in the lanes l with l % 4 = r).  A result is
// 48 cycles away, so the k-steps go round the accumulators.
template <int NB>
__device__ __forceinline__ void fpt_mma_few(double (&s0)[2], double (&s1)[2], bool two, const double *pa0,
                                            const double *pb0, const double *pa1, const double *pb1, int split, int KS,
                                            const d2 *frag, const d2 *next, d2 (&b)[NB / 2]) {
    for (int u0 = 0; u0 < KS; u0 += NB) {
        double a0[NB];
        fpt_row<NB>(pa0, pb0, split, u0, a0);
        if (two) {
            double a1[NB];
            fpt_row<NB>(pa1, pb1, split, u0, a1);
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const double bu = (u & 1) ? b[u / 2].y : b[u / 2].x;
                s0[u & 1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a0[u], bu, s0[u & 1], 0, 0, 0);
                s1[u & 1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a1[u], bu, s1[u & 1], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const double bu = (u & 1) ? b[u / 2].y : b[u / 2].x;
                double &s = (u & 2) ? s1[u & 1] : s0[u & 1];
                s = __builtin_amdgcn_mfma_f64_4x4x4f64(a0[u], bu, s, 0, 0, 0);
            }
        }
        const bool more = u0 + NB < KS;
        fpt_fetch<NB>(more ? frag : next, more ? (u0 + NB) / 2 : 0, b);
    }
}

// Products of nr (1 .. 16) rows with a column tile's fragments: row r from
// rowa(r) (columns below split) and rowb(r), zero past the operand's columns.
// init(r) is requested before the products, out(r, v, init) called for the
// lane's rows; frag, next and b as in fpt_mma.
//
// More than eight rows take MFMA 16x16x4 (64 cycles a k-step), up to eight
// 4x4x4 (16 for each four rows): the upper levels have few rows.
template <int NB, class RowA, class RowB, class Init, class Out>
__device__ __forceinline__ void fpt_product(int nr, int split, int KS, const d2 *frag, const d2 *next,
                                            d2 (&b)[NB / 2], RowA &&rowa, RowB &&rowb, Init &&init, Out &&out) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, kl = lane >> 4;
    if (nr > 8) {
        const int ra = min(r16, nr - 1);
        double y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = init(min(kl + 4 * r, nr - 1));
        d4 acc = {0.0, 0.0, 0.0, 0.0};
        fpt_mma<NB>(acc, rowa(ra), rowb(ra), split, KS, frag, next, b);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (kl + 4 * r < nr) out(kl + 4 * r, acc[r], y[r]);
        return;
    }
    const bool two = nr > 4;
    const int ra = min(r16 & 3, nr - 1), rb = min(4 + (r16 & 3), nr - 1);
    const double *pa0 = rowa(ra), *pb0 = rowb(ra), *pa1 = rowa(rb), *pb1 = rowb(rb);
    const double y0 = init(min(kl, nr - 1)), y1 = init(min(4 + kl, nr - 1));
    double s0[2] = {0.0, 0.0}, s1[2] = {0.0, 0.0};
    fpt_mma_few<NB>(s0, s1, two, pa0, pb0, pa1, pb1, split, KS, frag, next, b);
    const double v0 = s0[0] + s0[1], v1 = s1[0] + s1[1];
    if (kl < nr) out(kl, two ? v0 : v0 + v1, y0);
    if (4 + kl < nr) out(4 + kl, v1, y1);
}

// Barrier between levels: LDS accesses are complete, loads from memory may
// stay in flight (a __syncthreads would wait for the operands just requested).
__device__ __forceinline__ void level_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One chunk of one stage.  LDS: the interface rows Y [rows + 1][ldy], for a
// root chunk the zero-inflow values X (the same shape), for leaf chunks the
// moment differences [rows][lda].
template <int MODE, int NB>
__device__ __forceinline__ void fpt_body(const FPTreeArgs &f, const int chunk) {
    extern __shared__ double fpt_sm[];
    constexpr bool LEAF = MODE & FPT_LEAF, UP = MODE & FPT_UP, ROOT = MODE & FPT_ROOT, DOWN = MODE & FPT_DOWN,
                   UPDATE = MODE & FPT_UPDATE;
    const int N = f.N, NH = N / 2, L2 = f.L2, ldy = f.ldy, lda = f.lda;
    const int c0 = chunk * f.c, nc = min(f.c, f.n - c0);
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *Y = fpt_sm;
    double *X = ROOT ? Y + (size_t)(f.rows + 1) * ldy : Y;
    double *A = X + (size_t)(f.rows + 1) * ldy;
    // k-steps and column tiles of the products, and their fragments' sizes
    constexpr int KB = 4 * NB;
    const int npk = (N + KB - 1) / KB * KB, l2p = (L2 + KB - 1) / KB * KB;
    const int ksN = npk / 4, ksL = l2p / 4;
    // this wave's record: the ends of its units by phase, then the units,
    // all of it in registers (an entry per lane), so that finding the next
    // unit takes a few scalar instructions and no LDS or memory round trip
    const int *rec = f.recs + ((size_t)chunk * FPT_W + wv) * f.rec_stride;
    const int ends = rec[min(lane, kFptHdr - 1)];
    const int2 *recu = reinterpret_cast<const int2 *>(rec + kFptHdr);
    const int lastu = (f.rec_stride - kFptHdr) / 2 - 1;
    const int2 units0 = recu[min(lane, lastu)], units1 = recu[min(64 + lane, lastu)];
    // moment differences: the first loads go before the convergence gate
    // is resolved
    if constexpr (LEAF || UPDATE) {
        // two moments at a time: L2 is even (a caller's arrays are aligned to
        // 8 bytes only, which a 16-byte load takes)
        typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
        const int n2 = nc * L2 / 2;
        const size_t g0 = (size_t)c0 * L2;
        const d2u *half2 = reinterpret_cast<const d2u *>(f.half + g0), *old2 = reinterpret_cast<const d2u *>(f.old + g0);
        auto moments = [&](auto &&scale) {
            for (int base = 0; base < n2; base += FPT_T * 4) {
                d2 h[4], o[4], sg[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (base + FPT_T * u >= n2) break;
                    const int e = min(base + tid + FPT_T * u, n2 - 1);
                    h[u] = half2[e];
                    o[u] = old2[e];
                    sg[u] = scale(e);
                }
                if (base == 0 && skipped(f.skip)) return false;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (base + FPT_T * u >= n2) break;
                    const int e = base + tid + FPT_T * u;
                    const int r = (int)__umulhi((unsigned)(2 * e), f.rcpL2);
                    if (e < n2) {
                        double *a = A + r * lda + 2 * e - r * L2;
                        a[0] = (h[u].x - o[u].x) * sg[u].x;
                        a[1] = (h[u].y - o[u].y) * sg[u].y;
                    }
                }
            }
            return true;
        };
        if (f.sigma) {
            const d2u *sigma2 = reinterpret_cast<const d2u *>(f.sigma + g0);
            if (!moments([&](int e) -> d2 { return sigma2[e]; })) return;
        } else {
            if (!moments([&](int) { return d2{1.0, 1.0}; })) return;
        }
        if (l2p > L2)
            for (int i = tid; i < nc * (l2p - L2); i += FPT_T) A[(i / (l2p - L2)) * lda + L2 + i % (l2p - L2)] = 0.0;
    } else {
        if (skipped(f.skip)) return;
    }
    // interface rows: zero where nothing else is stored (padding columns and
    // the inflow halves of the end rows)
    if (npk > N)
        for (int i = tid; i < (nc + 1) * (npk - N); i += FPT_T) {
            const int r = i / (npk - N), k = N + i % (npk - N);
            Y[r * ldy + k] = 0.0;
            if (ROOT) X[r * ldy + k] = 0.0;
        }
    if constexpr (UP) {
        for (int k = tid; k < NH; k += FPT_T) {
            Y[k] = 0.0;
            Y[nc * ldy + NH + k] = 0.0;
            if (ROOT) {
                X[k] = 0.0;
                X[nc * ldy + NH + k] = 0.0;
            }
        }
        if constexpr (!LEAF) {
            const double *g = f.Yin + (size_t)c0 * N;
            const int n = (nc + 1) * N;
            for (int base = tid; base < n; base += FPT_T * 4) {
                double v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = g[min(base + FPT_T * u, n - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = base + FPT_T * u, r = (int)__umulhi((unsigned)i, f.rcpN), k = i - r * N;
                    if (i < n && (r > 0 || k >= NH) && (r < nc || k < NH)) Y[r * ldy + k] = v[u];
                }
            }
        }
    } else {
        // the ascent's zero-inflow values and the chunk's inflow
        const double *g = f.Yin + (size_t)c0 * N;
        for (int base = tid + N; base < nc * N; base += FPT_T * 4) {
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = g[min(base + FPT_T * u, nc * N - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = base + FPT_T * u, r = (int)__umulhi((unsigned)i, f.rcpN);
                if (i < nc * N) Y[r * ldy + i - r * N] = v[u];
            }
        }
        for (int k = tid; k < N; k += FPT_T) {
            if (k < NH)
                Y[k] = f.Yout[(size_t)chunk * N + k];
            else
                Y[nc * ldy + k] = f.Yout[(size_t)(chunk + 1) * N + k];
        }
    }
    __syncthreads();
    const int nlev = f.levels;
    const d2 *frag0 = reinterpret_cast<const d2 *>(f.frag) + lane;
    auto entry = [](int x0, int x1, int u) {
        const int a = __builtin_amdgcn_readlane(x0, u & 63), b = __builtin_amdgcn_readlane(x1, u & 63);
        return u < 64 ? a : b;
    };
    auto frag_of = [&](int u) { return frag0 + (size_t)(unsigned)entry(units0.x, units1.x, u) * 32; };
    // every unit of a phase: body(first row, rows, column tile, fragments,
    // the fragments to request next).  b always holds the first batch of the
    // next unit, whichever phase it belongs to.
    d2 b[NB / 2];
    int u = (UP || nlev == 0) ? 0 : __builtin_amdgcn_readlane(ends, nlev);
    fpt_fetch<NB>(frag_of(u), 0, b);
    auto phase = [&](int ph, int entries, auto &&body) {
        const int end = __builtin_amdgcn_readlane(ends, ph);
        for (; u < end; u += entries) {
            const int d = entry(units0.y, units1.y, u);
            body(d & 0xff, (d >> 8) & 0xff, d >> 16, frag_of(u), frag_of(u + 1));
        }
    };
    const auto none = [](int) { return 0.0; };
    if constexpr (LEAF) {
        // cell sources: s+ to the cell's right face, s- to its left
        phase(0, 1, [&](int t0, int nr, int c, const d2 *fr, const d2 *nx) {
            const int col = 16 * c + r16, o = (t0 + (col < NH ? 1 : 0)) * ldy + col;
            auto row = [&](int r) { return A + __mul24(t0 + r, lda); };
            fpt_product<NB>(nr, 0, ksL, fr, nx, b, row, row, none, [&](int r, double v, double) {
                if (col < N) Y[o + __mul24(r, ldy)] = v;
            });
        });
        level_barrier();
    }
    if constexpr (UP) {
        for (int l = 1; l <= nlev; ++l) {
            const int half = 1 << (l - 1);
            const int sl = ldy << l;  // LDS distance of two of the level's interfaces
            phase(l, 1, [&](int t0, int nr, int c, const d2 *fr, const d2 *nx) {
                const int col = 16 * c + r16, base = half * ldy + t0 * sl;
                double *g = f.Yin + (size_t)(c0 + half + (t0 << l)) * N + col;
                auto row = [&](int r) { return Y + base + __mul24(r, sl); };
                auto value = [&](int r, double v) {
                    if (ROOT)
                        X[base + __mul24(r, sl) + col] = v;
                    else
                        g[(size_t)(r << l) * N] = v;
                };
                if (16 * c + 16 <= N) {
                    // the interface's zero-inflow value
                    fpt_product<NB>(nr, 0, ksN, fr, nx, b, row, row, none, [&](int r, double v, double) { value(r, v); });
                    return;
                }
                // what the node adds to the rows at its ends (in a column
                // tile across both parts, also the value)
                const int cy = max(col - N, 0), cz = min(cy, N - 1);
                auto end = [&](int r) {
                    const int j = half + ((t0 + r) << l);
                    return __mul24(cy < NH ? min(j + half, nc) : j - half, ldy) + cz;
                };
                fpt_product<NB>(nr, 0, ksN, fr, nx, b, row, row, [&](int r) { return Y[end(r)]; },
                                [&](int r, double v, double y) {
                                    if (col >= 2 * N) return;
                                    if (col >= N)
                                        Y[end(r)] = y + v;
                                    else
                                        value(r, v);
                                });
            });
            level_barrier();
        }
        if constexpr (ROOT) {
            // the slab's outgoing fluxes (b_0 | a_K)
            for (int k = tid; k < NH; k += FPT_T) {
                f.exit_b0[k] = Y[NH + k];
                f.exit_aK[k] = Y[nc * ldy + k];
            }
        } else {
            for (int k = tid; k < NH; k += FPT_T) {
                f.Yout[(size_t)(chunk + 1) * N + k] = Y[nc * ldy + k];
                f.Yout[(size_t)chunk * N + NH + k] = Y[NH + k];
            }
        }
    }
    if constexpr (DOWN) {
        for (int l = nlev; l >= 1; --l) {
            const int half = 1 << (l - 1);
            const int sl = ldy << l;
            phase(2 * nlev + 1 - l, 1, [&](int t0, int nr, int c, const d2 *fr, const d2 *nx) {
                const int col = 16 * c + r16, cc = min(col, N - 1), base = half * ldy + t0 * sl;
                auto right = [&](int r) { return __mul24(min(half + ((t0 + r) << l) + half, nc), ldy); };
                fpt_product<NB>(nr, NH, ksN, fr, nx, b, [&](int r) { return X + base - half * ldy + __mul24(r, sl); },
                                [&](int r) { return X + right(r); }, [&](int r) { return X[base + __mul24(r, sl) + cc]; },
                                [&](int r, double v, double x) {
                                    if (col < N) X[base + __mul24(r, sl) + col] = x + v;
                                });
            });
            level_barrier();
        }
        if constexpr (!UPDATE) {
            // the next stage down reads a at each chunk's left face and b at
            // its right one; a root chunk has no inflow
            double *g = f.Yin + (size_t)c0 * N;
            for (int i = tid; i < (nc + 1) * N; i += FPT_T) {
                const int r = (int)__umulhi((unsigned)i, f.rcpN), k = i - r * N;
                if ((r > 0 || k < NH) && (r < nc || k >= NH)) g[i] = X[r * ldy + k];
            }
        }
    }
    if constexpr (UPDATE) {
        unsigned long long dmax = 0ull;
        const bool stop = f.stop_slot != nullptr;
        phase(2 * nlev + 1, 2, [&](int t0, int nr, int c, const d2 *fr, const d2 *fi) {
            const int col = 16 * c + r16, kl = lane >> 4, cc = min(col, L2 - 1);
            // r-th row of the lane's results
            auto cell = [&](int r) { return (size_t)(c0 + t0 + min(kl + 4 * r, nr - 1)) * L2 + cc; };
            auto put = [&](int r, double v, double old) {
                if (col >= L2 || kl + 4 * r >= nr) return;
                f.out[cell(r)] = v;
                const unsigned long long d = absdiff_bits(v, old);
                dmax = d > dmax ? d : dmax;
            };
            const d2 *after = frag_of(u + 2);
            // the moments' part, then the inflow's
            if (nr > 8) {
                double hv[4], ov[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    hv[r] = f.half[cell(r)];
                    ov[r] = f.old[cell(r)];
                }
                const int row = t0 + min(r16, nr - 1);
                const double *pa = A + row * lda, *pi = X + row * ldy;
                d4 acc = {0.0, 0.0, 0.0, 0.0};
                fpt_mma<NB>(acc, pa, pa, 0, ksL, fr, fi, b);
                fpt_mma<NB>(acc, pi, pi + ldy, NH, ksN, fi, after, b);
#pragma unroll
                for (int r = 0; r < 4; ++r) put(r, acc[r] + hv[r], ov[r]);
            } else {
                const double h0 = f.half[cell(0)], h1 = f.half[cell(1)], o0 = f.old[cell(0)], o1 = f.old[cell(1)];
                const bool two = nr > 4;
                const int r0 = t0 + min(r16 & 3, nr - 1), r1 = t0 + min(4 + (r16 & 3), nr - 1);
                const double *pa0 = A + r0 * lda, *pa1 = A + r1 * lda, *pi0 = X + r0 * ldy, *pi1 = X + r1 * ldy;
                double s0[2] = {0.0, 0.0}, s1[2] = {0.0, 0.0};
                fpt_mma_few<NB>(s0, s1, two, pa0, pa0, pa1, pa1, 0, ksL, fr, fi, b);
                fpt_mma_few<NB>(s0, s1, two, pi0, pi0 + ldy, pi1, pi1 + ldy, NH, ksN, fi, after, b);
                const double v0 = s0[0] + s0[1], v1 = s1[0] + s1[1];
                put(0, (two ? v0 : v0 + v1) + h0, o0);
                if (two) put(1, v1 + h1, o1);
            }
        });
        if (stop) stop_block_reduce(dmax, f.stop_slot);
    }
}

template <int MODE, int NB>
__global__ void __launch_bounds__(FPT_T) fpt_kernel(FPTreeArgs f) {
    fpt_body<MODE, NB>(f, (int)blockIdx.x);
}

__device__ __forceinline__ void apply_patch(FPTreeArgs &a, const IterPatch &p, int m) {
    patch_skip(a.skip, p, m);
    if (p.flags & PATCH_A1SUB_CUR) a.old = iter_buf(p, m - 1);
    if (p.flags & PATCH_C_NXT) a.out = iter_buf(p, m);
    if (p.flags & PATCH_STOP) a.stop_slot = iter_slot(p, m);
}

template <int MODE, int NB>
__global__ void __launch_bounds__(FPT_T) fpt_kernel_multi(const MultiEntry<FPTreeArgs> *E, const BlockRef *br, const int *iter) {
    const BlockRef r = br[blockIdx.x];
    const MultiEntry<FPTreeArgs> &e = E[r.entry];
    FPTreeArgs a = e.a;
    apply_patch(a, e.p, *iter);
    fpt_body<MODE, NB>(a, r.local);
}

// Entries of several widths in one launch (kMixedBlocks).
template <int MODE>
__global__ void __launch_bounds__(FPT_T) fpt_kernel_mixed(const MultiEntry<FPTreeArgs> *E, const BlockRef *br, const int *iter) {
    const BlockRef r = br[blockIdx.x];
    const MultiEntry<FPTreeArgs> &e = E[r.entry];
    FPTreeArgs a = e.a;
    apply_patch(a, e.p, *iter);
    switch (e.v1) {
        case 2: fpt_body<MODE, 2>(a, r.local); break;
        case 4: fpt_body<MODE, 4>(a, r.local); break;
        default: fpt_body<MODE, 8>(a, r.local); break;
    }
}

constexpr int kFptModes[] = {FPT_LEAF | FPT_UP, FPT_UP, FPT_UP | FPT_ROOT | FPT_DOWN, FPT_DOWN, FPT_DOWN | FPT_UPDATE,
                             FPT_LEAF | FPT_UP | FPT_ROOT | FPT_DOWN | FPT_UPDATE};

LaunchShape fpt_shape(const FPTreeArgs &f, int mode) {
    LaunchShape sh;
    sh.kernel = MK_FPT;
    sh.v1 = f.nb;
    sh.v2 = mode;
    sh.gx = f.chunks;
    sh.block = FPT_T;
    const int m = kFptModes[mode];
    sh.kid = (m & FPT_UPDATE) ? KID_FP_TREE_UPDATE : ((m & FPT_LEAF) ? KID_FP_TREE_UP : KID_FP_TREE_MID);
    size_t d = (size_t)((m & FPT_ROOT) ? 2 : 1) * (f.rows + 1) * f.ldy;
    if (m & (FPT_LEAF | FPT_UPDATE)) d += (size_t)f.rows * f.lda;
    sh.lds = (unsigned)(d * sizeof(double));
    return sh;
}

template <int M, int NB>
static void fpt_launch_m(const LaunchShape &sh, const FPTreeArgs &f, hipStream_t s, KernelTimer *t) {
    LAUNCH(sh.kid, t, (fpt_kernel<M, NB>), dim3(sh.gx), dim3(FPT_T), sh.lds, s, f);
}

template <int NB>
static void fpt_launch_nb(const LaunchShape &sh, const FPTreeArgs &f, hipStream_t s, KernelTimer *t) {
    switch (sh.v2) {
        case 0: fpt_launch_m<kFptModes[0], NB>(sh, f, s, t); break;
        case 1: fpt_launch_m<kFptModes[1], NB>(sh, f, s, t); break;
        case 2: fpt_launch_m<kFptModes[2], NB>(sh, f, s, t); break;
        case 3: fpt_launch_m<kFptModes[3], NB>(sh, f, s, t); break;
        case 4: fpt_launch_m<kFptModes[4], NB>(sh, f, s, t); break;
        default: fpt_launch_m<kFptModes[5], NB>(sh, f, s, t); break;
    }
}

void launch_fpt(const FPTreeArgs &f, int mode, hipStream_t s, KernelTimer *t) {
    if (f.chunks <= 0) return;
    const LaunchShape sh = fpt_shape(f, mode);
    switch (sh.v1) {
        case 2: fpt_launch_nb<2>(sh, f, s, t); break;
        case 4: fpt_launch_nb<4>(sh, f, s, t); break;
        default: fpt_launch_nb<8>(sh, f, s, t); break;
    }
}

template <int M, int NB>
static void fpt_multi_m(const MultiLaunch &L, const int *iter, hipStream_t s, KernelTimer *t) {
    const MultiEntry<FPTreeArgs> *E = static_cast<const MultiEntry<FPTreeArgs> *>(L.entries);
    if constexpr (NB == kMixedWidths)
        LAUNCH(L.shape.kid, t, fpt_kernel_mixed<M>, dim3(L.nblocks), dim3(FPT_T), L.lds, s, E, L.refs, iter);
    else
        LAUNCH(L.shape.kid, t, (fpt_kernel_multi<M, NB>), dim3(L.nblocks), dim3(FPT_T), L.lds, s, E, L.refs, iter);
}

template <int NB>
static void fpt_multi_nb(const MultiLaunch &L, const int *iter, hipStream_t s, KernelTimer *t) {
    switch (L.shape.v2) {
        case 0: fpt_multi_m<kFptModes[0], NB>(L, iter, s, t); break;
        case 1: fpt_multi_m<kFptModes[1], NB>(L, iter, s, t); break;
        case 2: fpt_multi_m<kFptModes[2], NB>(L, iter, s, t); break;
        case 3: fpt_multi_m<kFptModes[3], NB>(L, iter, s, t); break;
        case 4: fpt_multi_m<kFptModes[4], NB>(L, iter, s, t); break;
        default: fpt_multi_m<kFptModes[5], NB>(L, iter, s, t); break;
    }
}

void launch_fpt_multi(const MultiLaunch &L, const int *iter, hipStream_t s, KernelTimer *t) {
    switch (L.shape.v1) {
        case 2: fpt_multi_nb<2>(L, iter, s, t); break;
        case 4: fpt_multi_nb<4>(L, iter, s, t); break;
        case kMixedWidths: fpt_multi_nb<kMixedWidths>(L, iter, s, t); break;
        default: fpt_multi_nb<8>(L, iter, s, t); break;
    }
}

}  // namespace snfpsa
