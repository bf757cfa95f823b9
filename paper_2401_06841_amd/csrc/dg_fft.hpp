// dg_fft.hpp -- the velocity spectrum's Fourier transform in three passes over memory: the point
// velocities of whole x lines are evaluated and transformed in a block, then the y lines are
// transformed in place, and the transform along z ends in the shell sums, so that neither the grid
// of point values nor the finished spectrum is written.
//
// Lines of up to 512 points with no prime factor above 5, by mixed-radix decimation in frequency in
// place: a butterfly of radix r of a sub-line of m points reads its points j + q m / r, q < r, and
// leaves output p, turned by w_m^(p j), at j + p m / r, which begins the sub-line of the frequencies
// k = p mod r.  No pass needs its output in order of frequency, so nothing is reordered: `freq`
// gives the frequency at a position.  Each butterfly owns its points and a stage needs one barrier;
// the first stage of the y and z lines reads memory and the last one of the y lines writes it
// directly, so that a line of 8 x 6 x 8 = 384 points goes through LDS twice.
#pragma once

#include "dg_kernels.hpp"

namespace dg {

constexpr int FFT_MAX_LINE = 512;   // points of a line
constexpr int FFT_MAX_STAGES = 7;   // 2 3^5 = 486: radices 6 3 3 3 3; 512: 8 8 8; 500: 5 5 5 4
constexpr int FFT_COLS = 8;         // x frequencies side by side in memory (128 bytes)
constexpr int FFT_MAX_SHELLS = 448; // shells of a grid of 512 points a side (444)

// one axis: radix, points between a butterfly's points and twiddle step of each stage; q / sub for
// q < 512 is q * magic >> 20
struct FftAxis {
    int n, nst;
    int radix[FFT_MAX_STAGES], sub[FFT_MAX_STAGES], step[FFT_MAX_STAGES];
    unsigned magic[FFT_MAX_STAGES];
};

// the axes' twiddles e^(-2 pi i t / n), frequencies by position and positions by frequency, and the
// Legendre values of the p sub-points of a cell, in device memory
struct FftTables {
    double2 *tw[3];
    int *freq[3], *pos[3];
    double *leg;        // [p][4]
};

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
// a - i s b and a + i s b
__device__ __forceinline__ double2 sub_i(double2 a, double s, double2 b)
{
    return make_double2(fma(s, b.y, a.x), fma(-s, b.x, a.y));
}
__device__ __forceinline__ double2 add_i(double2 a, double s, double2 b)
{
    return make_double2(fma(-s, b.y, a.x), fma(s, b.x, a.y));
}
__device__ __forceinline__ double2 axpy(double s, double2 a, double2 b)
{
    return make_double2(fma(s, a.x, b.x), fma(s, a.y, b.y));
}

constexpr double FFT_S3 = 0.86602540378443864676;   // sin 60
constexpr double FFT_C5A = 0.30901699437494742410, FFT_C5B = -0.80901699437494742410;   // cos 72, cos 144
constexpr double FFT_S5A = 0.95105651629515357212, FFT_S5B = 0.58778525229247312917;    // sin 72, sin 144
constexpr double FFT_R2 = 0.70710678118654752440;

__device__ __forceinline__ void dft3(double2 &a, double2 &b, double2 &c)
{
    const double2 t = cadd(b, c), d = csub(b, c), m = axpy(-0.5, t, a);
    a = cadd(a, t);
    b = sub_i(m, FFT_S3, d);
    c = add_i(m, FFT_S3, d);
}

__device__ __forceinline__ void dft4(double2 &a, double2 &b, double2 &c, double2 &d)
{
    const double2 s0 = cadd(a, c), d0 = csub(a, c), s1 = cadd(b, d), d1 = csub(b, d);
    a = cadd(s0, s1);
    b = sub_i(d0, 1.0, d1);
    c = csub(s0, s1);
    d = add_i(d0, 1.0, d1);
}

// the discrete Fourier transform of R points, in order
template <int R>
__device__ __forceinline__ void dft(double2 (&a)[R])
{
    static_assert(R == 1 || R == 2 || R == 3 || R == 4 || R == 5 || R == 6 || R == 8, "radix");
    if constexpr (R == 2) {
        const double2 t = a[1];
        a[1] = csub(a[0], t);
        a[0] = cadd(a[0], t);
    } else if constexpr (R == 3) {
        dft3(a[0], a[1], a[2]);
    } else if constexpr (R == 4) {
        dft4(a[0], a[1], a[2], a[3]);
    } else if constexpr (R == 5) {
        const double2 t1 = cadd(a[1], a[4]), t2 = cadd(a[2], a[3]), t3 = csub(a[1], a[4]), t4 = csub(a[2], a[3]);
        const double2 m1 = axpy(FFT_C5B, t2, axpy(FFT_C5A, t1, a[0])), m2 = axpy(FFT_C5A, t2, axpy(FFT_C5B, t1, a[0]));
        a[0] = cadd(a[0], cadd(t1, t2));
        a[1] = sub_i(sub_i(m1, FFT_S5A, t3), FFT_S5B, t4);
        a[4] = add_i(add_i(m1, FFT_S5A, t3), FFT_S5B, t4);
        a[2] = add_i(sub_i(m2, FFT_S5B, t3), FFT_S5A, t4);
        a[3] = sub_i(add_i(m2, FFT_S5B, t3), FFT_S5A, t4);
    } else if constexpr (R == 6) {
        dft3(a[0], a[2], a[4]);
        dft3(a[1], a[3], a[5]);
        // w_6^k times the odd points' output k
        const double2 o1 = make_double2(fma(0.5, a[3].x, FFT_S3 * a[3].y), fma(0.5, a[3].y, -FFT_S3 * a[3].x));
        const double2 o2 = make_double2(fma(-0.5, a[5].x, FFT_S3 * a[5].y), fma(-0.5, a[5].y, -FFT_S3 * a[5].x));
        const double2 e0 = a[0], e1 = a[2], e2 = a[4], o0 = a[1];
        a[0] = cadd(e0, o0);
        a[1] = cadd(e1, o1);
        a[2] = cadd(e2, o2);
        a[3] = csub(e0, o0);
        a[4] = csub(e1, o1);
        a[5] = csub(e2, o2);
    } else if constexpr (R == 8) {
        dft4(a[0], a[2], a[4], a[6]);
        dft4(a[1], a[3], a[5], a[7]);
        const double2 o0 = a[1], o2 = make_double2(a[5].y, -a[5].x);
        const double2 o1 = make_double2(FFT_R2 * (a[3].x + a[3].y), FFT_R2 * (a[3].y - a[3].x));
        const double2 o3 = make_double2(FFT_R2 * (a[7].y - a[7].x), -FFT_R2 * (a[7].x + a[7].y));
        const double2 e0 = a[0], e1 = a[2], e2 = a[4], e3 = a[6];
        a[0] = cadd(e0, o0);
        a[1] = cadd(e1, o1);
        a[2] = cadd(e2, o2);
        a[3] = cadd(e3, o3);
        a[4] = csub(e0, o0);
        a[5] = csub(e1, o1);
        a[6] = csub(e2, o2);
        a[7] = csub(e3, o3);
    }
}

// One stage over ncol lines side by side, its butterflies strided over the block's nt threads: ld(pos, col)
// reads a point, st(i, p, pos, col, value) takes output p of the thread's butterfly i.  A
// stage of radix 1 copies.
template <int R, int COLS, typename LD, typename ST>
__device__ __forceinline__ void fft_stage(const FftAxis &ax, int s, const double2 *tw, int ncol, int nt, LD &&ld, ST &&st)
{
    const int nq = R > 1 ? ax.n / R : ax.n, nbf = nq * ncol;
    const int sub = ax.sub[s], step = ax.step[s];
    const unsigned magic = ax.magic[s];
    // (opaque, or the addresses of every radix would be kept in registers across the lines)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    auto butterfly = [&](int i, int b) {
        // columns side by side, or one line's butterflies after the other's
        const int c = COLS ? b % (COLS ? COLS : 1) : b / nq, q = COLS ? b / (COLS ? COLS : 1) : b - c * nq;
        int j = q, pos = q;
        if constexpr (R > 1) {
            const int blk = (int)(((unsigned)q * magic) >> 20);
            j = q - blk * sub;
            pos = blk * sub * R + j;
        }
        double2 a[R];
#pragma unroll
        for (int p = 0; p < R; ++p) a[p] = ld(pos + p * sub, c);
        dft<R>(a);
        if (R > 1 && sub > 1) {
            const int t = j * step;
#pragma unroll
            for (int p = 1; p < R; ++p) a[p] = cmul(a[p], tw[p * t]);
        }
#pragma unroll
        for (int p = 0; p < R; ++p) st(i, p, pos + p * sub, c, a[p]);
    };
    if constexpr (COLS != 0) {
        // nt >= n: at most COLS / R butterflies a thread
        constexpr int NI = (COLS + R - 1) / R;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int b = tid + i * nt;
            if (b < nbf) butterfly(i, b);
        }
    } else {
        for (int b = tid; b < nbf; b += nt) butterfly(0, b);
    }
}

template <int COLS, typename LD, typename ST>
__device__ __forceinline__ void fft_any(const FftAxis &ax, int s, const double2 *tw, int ncol, int nt, LD &&ld, ST &&st)
{
    switch (ax.radix[s]) {
    case 1: fft_stage<1, COLS>(ax, s, tw, ncol, nt, ld, st); break;
    case 2: fft_stage<2, COLS>(ax, s, tw, ncol, nt, ld, st); break;
    case 3: fft_stage<3, COLS>(ax, s, tw, ncol, nt, ld, st); break;
    case 4: fft_stage<4, COLS>(ax, s, tw, ncol, nt, ld, st); break;
    case 5: fft_stage<5, COLS>(ax, s, tw, ncol, nt, ld, st); break;
    case 6: fft_stage<6, COLS>(ax, s, tw, ncol, nt, ld, st); break;
    default: fft_stage<8, COLS>(ax, s, tw, ncol, nt, ld, st); break;
    }
}

// Legendre values by upward recurrence, orthonormal for the mean: sqrt(2n+1) P_n
template <int K>
__device__ __forceinline__ void legendre_row(double x, double (&L)[K + 1]);

static __global__ void __launch_bounds__(BLOCK) k_fft_tables(FftAxis x, FftAxis y, FftAxis z, int p, FftTables tb)
{
    const FftAxis *ax[3] = {&x, &y, &z};
    for (int a = 0; a < 3; ++a) {
        const FftAxis &A = *ax[a];
        for (int t = threadIdx.x; t < A.n; t += BLOCK) {
            double s, c;
            sincospi(2.0 * (double)t / (double)A.n, &s, &c);
            tb.tw[a][t] = make_double2(c, -s);
            // position t: digit p_i of stage i is the frequency's digit of weight r_1 ... r_(i-1)
            int f = 0, w = 1, rest = t;
            for (int s2 = 0; s2 < A.nst; ++s2)
                if (A.radix[s2] > 1) {
                    const int d = rest / A.sub[s2];
                    rest -= d * A.sub[s2];
                    f += d * w;
                    w *= A.radix[s2];
                }
            tb.freq[a][t] = f;
            tb.pos[a][f] = t;
        }
    }
    for (int t = threadIdx.x; t < p; t += BLOCK) {
        double L[4];
        legendre_row<3>(-1.0 + (2.0 * (double)t + 1.0) / p, L);
        for (int n = 0; n < 4; ++n) tb.leg[4 * t + n] = L[n];
    }
}

// points of a line in LDS, whole groups of 8
__host__ __device__ inline int fft_pad(int n) { return (n + 7) / 8 * 8; }

// x lines: the velocities of the points of yl lines of one z and their transforms,
// F[d][tile of 8 x frequencies][z][y][8].  Two real lines of one component, neighbours in y, make a
// complex line (of two components, the larger one's rounding would pass into the smaller).
// Bound about half by the vector units (some 250 instructions a point: the three FP64 quotients, the
// collapse of the weights, the transform) and half by the writes of 128-byte pieces: on 384^3 points
// 0.745 ms (1.37 GB written, 0.34 GB read; averages of one trace, like the two other passes': 1.92 ms
// the whole call), where the evaluation alone took 0.78 ms with the grid written.
// SPLIT: the points of a cell's line are shared by as many threads as the block has for it
template <typename T, int K, bool SPLIT>
__global__ void __launch_bounds__(BLOCK) k_fft_x(const void *u_, int nx, int ny, int nz, double floor_, int p, int yl,
                                                 FftAxis ax, FftTables tb, int ntile, double2 *F)
{
    extern __shared__ double2 shx[];
    constexpr Modes<K> M = make_modes<K>();
    constexpr int NB = Shape<K>::NB, N1 = K + 1, NXY = Shape<K>::NB2;
    const int X = nx * p, Y = ny * p, Z = nz * p;
    const int nt = blockDim.x;
    const int nch = (Y + yl - 1) / yl;
    // a cell row's points of all z and y in neighbouring blocks of one XCD: its weights are read from
    // memory once
    int b = xcd_remap(blockIdx.x, gridDim.x);
    const int iz = b % p; b /= p;
    const int ck = b / nch, y0 = (b - ck * nch) * yl, nyl = min(yl, Y - y0);     // lines y0 .. y0 + nyl - 1
    const int nlc = (nyl + 1) / 2, nl = 3 * nlc;                                  // complex lines
    double2 *tw = shx, *line = shx + X;
    // point x of line l: every group of 8 points in an order of its own, so that points 4 or 8 apart
    // (neighbouring cells', the last stage's butterflies) lie in different LDS banks
    const int XP = fft_pad(X);
    auto at = [&](int x, int l) { return l * XP + (x ^ ((x >> 3) & 7)); };
    double *re = (double *)line;                        // line iy of component d: part iy % 2 of line d nlc + iy / 2
    for (int t = threadIdx.x; t < X; t += nt) tw[t] = tb.tw[0][t];
    const size_t nc = (size_t)nx * ny * nz;
    const T *u = (const T *)u_ + (size_t)nx * ny * ck;
    const double *lz = tb.leg + 4 * iz;
    // a cell's points a0, a0 + na, .. of one line from the line's Legendre coefficients
    auto points = [&](int i, int iy, int a0, int na, const double (&c)[4][N1]) {
        for (int a = a0; a < p; a += na) {
            const double *lx = tb.leg + 4 * a;
            double w[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                w[v] = c[v][0] * lx[0];
#pragma unroll
                for (int n = 1; n < N1; ++n) w[v] = fma(c[v][n], lx[n], w[v]);
            }
            const double rho = fmax(w[0], floor_);
            const int x = i * p + a;
#pragma unroll
            for (int d = 0; d < 3; ++d) re[2 * at(x, d * nlc + (iy >> 1)) + (iy & 1)] = w[1 + d] / rho;
        }
    };
    // weight of cell i of the plane (i < nx ny)
    auto weight = [&](int v, int l, int i) {
        return *(const T *)((const char *)(u + (size_t)(v * NB + l) * nc) + (unsigned)i * sizeof(T));
    };
    // A thread takes one line of a cell, and reads the cell's weights for it; with the 80 weights of
    // degree 3 (at most nt / nx threads a cell) it first sums them over z, for all of its lines.
    // Forms of a thread's work compared, a line at a time against the sums over z first: on 384^3 points,
    // degree 2, FP32, 0.78 and 0.85 ms, on 512^3 points, degree 3, 3.1 and 2.1 ms.
    if constexpr (K < 3) {
        const int na = SPLIT ? max(1, nt / (nx * nyl)) : 1;
        for (int it = threadIdx.x; it < nx * nyl * na; it += nt) {
            const int i = it % nx, q = it / nx, a0 = SPLIT ? q / nyl : 0, iy = q - a0 * nyl, cj = (y0 + iy) / p;
            const double *ly = tb.leg + 4 * (y0 + iy - cj * p);
            double c[4][N1], lyz[NXY];
#pragma unroll
            for (int l = 0; l < NB; ++l)
                if (M.e[l][0] == 0) lyz[M.d2[0][l]] = ly[M.e[l][1]] * lz[M.e[l][2]];
            // (all loads first where the compiler would otherwise send them one at a time: 256^3 cells
            // on 512^3 points 6.7 -> 5.2 ms)
            constexpr bool AHEAD = sizeof(T) == 8 && K == 2;
            T w[4][NB];
            if constexpr (AHEAD) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int l = 0; l < NB; ++l) w[v][l] = weight(v, l, cj * nx + i);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int a = 0; a < N1; ++a) c[v][a] = 0.0;
#pragma unroll
                for (int l = 0; l < NB; ++l)
                    c[v][M.e[l][0]] = fma((double)(AHEAD ? w[v][l] : weight(v, l, cj * nx + i)), lyz[M.d2[0][l]], c[v][M.e[l][0]]);
            }
            points(i, iy, a0, na, c);
        }
    } else {
        const int cj0 = y0 / p, nrow = (y0 + nyl - 1) / p - cj0 + 1;       // the lines' cell rows
        const int ng = max(1, min(min(p, nyl), nt / (nx * nrow)));
        const int na = SPLIT ? max(1, nt / (nx * nrow * ng)) : 1;
        for (int it = threadIdx.x; it < nx * nrow * ng * na; it += nt) {
            const int i = it % nx, q = it / nx, h = q / nrow, cj = cj0 + q - h * nrow;
            const int a0 = SPLIT ? h / ng : 0, g = h - a0 * ng;
            const int ya = max(cj * p, y0) - y0, yb = min((cj + 1) * p, y0 + nyl) - y0;
            double cz[4][NXY];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int l = 0; l < NXY; ++l) cz[v][l] = 0.0;
                T w[NB];
#pragma unroll
                for (int l = 0; l < NB; ++l) w[l] = weight(v, l, cj * nx + i);
                // (FP64 is faster with the compiler's order on all grids below 512^3, 7 % on 256^3, and 5 % slower there)
                if constexpr (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int l = 0; l < NB; ++l) cz[v][M.d2[2][l]] = fma((double)w[l], lz[M.e[l][2]], cz[v][M.d2[2][l]]);
            }
            for (int iy = ya + g; iy < yb; iy += ng) {
                const double *ly = tb.leg + 4 * (y0 + iy - cj * p);
                double c[4][N1];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
#pragma unroll
                    for (int a = 0; a < N1; ++a) c[v][a] = 0.0;
#pragma unroll
                    for (int l = 0; l < NB; ++l)
                        if (M.e[l][2] == 0) c[v][M.e[l][0]] = fma(cz[v][M.d2[2][l]], ly[M.e[l][1]], c[v][M.e[l][0]]);
                }
                points(i, iy, a0, na, c);
            }
        }
    }
    if (nyl & 1)
        for (int x = threadIdx.x; x < X; x += nt)
#pragma unroll
            for (int d = 0; d < 3; ++d) re[2 * at(x, d * nlc + nlc - 1) + 1] = 0.0;
    __syncthreads();
    for (int s = 0; s < ax.nst; ++s) {
        fft_any<0>(ax, s, tw, nl, nt, [&](int pos, int cc) { return line[at(pos, cc)]; },
                   [&](int, int, int pos, int cc, double2 v) { line[at(pos, cc)] = v; });
        __syncthreads();
    }
    // the transforms of the two real lines of a complex one, from frequencies f and X - f
    const int Xh = X / 2 + 1;
    const int zz = ck * p + iz;
    const size_t tstr = (size_t)Z * Y * FFT_COLS;       // between tiles of x frequencies
    for (int f = threadIdx.x; f < Xh; f += nt) {
        const int t = f / FFT_COLS, pf = tb.pos[0][f], pb = tb.pos[0][f ? X - f : 0];
        double2 *G = F + t * tstr + ((size_t)zz * Y + y0) * FFT_COLS + (f - t * FFT_COLS);
        for (int d = 0; d < 3; ++d, G += ntile * tstr)
            for (int j = 0; j < nlc; ++j) {
                const double2 g = line[at(pf, d * nlc + j)], h = line[at(pb, d * nlc + j)];
                G[2 * j * FFT_COLS] = make_double2(0.5 * (g.x + h.x), 0.5 * (g.y - h.y));
                if (2 * j + 1 < nyl) G[(2 * j + 1) * FFT_COLS] = make_double2(0.5 * (g.y + h.y), 0.5 * (h.x - g.x));
            }
    }
}

// the block's threads for lines of n points: n, rounded up to whole waves
__host__ __device__ inline int fft_threads(int n) { return (n + 63) / 64 * 64; }

// y lines, in place: one tile of 8 columns, contiguous, a block.  Bound by memory: 2.83 GB in 0.606 ms
// on 384^3 points (4.7 TB/s; a large copy runs at 4.4)
template <int TN>
__global__ void __launch_bounds__(TN) k_fft_y(FftAxis ax, FftTables tb, double2 *F)
{
    __shared__ double2 tile[TN * FFT_COLS];
    __shared__ double2 tw[TN];
    const int nt = blockDim.x;
    for (int t = threadIdx.x; t < ax.n; t += nt) tw[t] = tb.tw[1][t];
    double2 *G = F + (size_t)blockIdx.x * ax.n * FFT_COLS;
    auto ldg = [&](int pos, int c) { return G[pos * FFT_COLS + c]; };
    auto stg = [&](int, int, int pos, int c, double2 v) { G[pos * FFT_COLS + c] = v; };
    auto lds = [&](int pos, int c) { return tile[pos * FFT_COLS + c]; };
    auto sts = [&](int, int, int pos, int c, double2 v) { tile[pos * FFT_COLS + c] = v; };
    __syncthreads();
    fft_any<FFT_COLS>(ax, 0, tw, FFT_COLS, nt, ldg, sts);
    __syncthreads();
    for (int s = 1; s < ax.nst - 1; ++s) {
        fft_any<FFT_COLS>(ax, s, tw, FFT_COLS, nt, lds, sts);
        __syncthreads();
    }
    fft_any<FFT_COLS>(ax, ax.nst - 1, tw, FFT_COLS, nt, lds, stg);
}

// sqrt(s) to the nearest integer k, k^2 - k < s <= k^2 + k
__device__ __forceinline__ int shell_of(int s)
{
    int k = (int)(__builtin_amdgcn_sqrtf((float)s) + 0.5f);
    if (k * k + k < s) ++k;
    if (k > 0 && k * k - k >= s) --k;
    return k;
}

// z lines and the shell sums of 1/2 |F / npts|^2 (the x frequencies 0 < f < X / 2 stand for
// themselves and their mirror images): one (tile, y) after another, the three components' squares
// added in registers before the one addition to the block's histogram in LDS.  1.42 GB in 0.603 ms on
// 384^3 points and 3.3 GB in 0.85 ms on 512^3; without the histogram 0.61 and 0.83, with three
// resident blocks a compute unit instead of two (twiddles read from memory) 0.62 and 0.98, with the
// next lines fetched ahead in registers 0.54 and 1.07
template <int TN>
__global__ void __launch_bounds__(TN) k_fft_z(FftAxis ax, FftTables tb, const double2 *F, int X, int Y, int ntile,
                                              int nshell, double *part)
{
    __shared__ double2 tile[TN * FFT_COLS];
    __shared__ double2 tw[TN];
    __shared__ double hist[FFT_MAX_SHELLS];
    const int nt = blockDim.x, Z = ax.n;
    for (int t = threadIdx.x; t < Z; t += nt) tw[t] = tb.tw[2][t];
    for (int s = threadIdx.x; s < nshell; s += nt) hist[s] = 0.0;
    const int Xh = X / 2 + 1, ntiles = ntile * Y;
    auto lds = [&](int pos, int c) { return tile[pos * FFT_COLS + c]; };
    auto sts = [&](int, int, int pos, int c, double2 v) { tile[pos * FFT_COLS + c] = v; };
    constexpr int NE = 12;      // squares of a thread: at most ceil(8 / R) R
    for (int b = blockIdx.x; b < ntiles; b += gridDim.x) {
        const int t = b / Y, yp = b - t * Y;
        double e[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) e[i] = 0.0;
        for (int d = 0; d < 3; ++d) {
            const double2 *G = F + (((size_t)d * ntile + t) * Z * Y + yp) * FFT_COLS;
            auto ldg = [&](int pos, int c) { return G[(size_t)pos * Y * FFT_COLS + c]; };
            __syncthreads();
            fft_any<FFT_COLS>(ax, 0, tw, FFT_COLS, nt, ldg, sts);
            __syncthreads();
            for (int s = 1; s < ax.nst - 1; ++s) {
                fft_any<FFT_COLS>(ax, s, tw, FFT_COLS, nt, lds, sts);
                __syncthreads();
            }
            auto last = [&](auto rc) {
                constexpr int R = decltype(rc)::value;
                fft_stage<R, FFT_COLS>(ax, ax.nst - 1, tw, FFT_COLS, nt, lds,
                                       [&](int i, int p, int, int, double2 v) {
                                           e[i * R + p] += v.x * v.x + v.y * v.y;
                                       });
            };
            switch (ax.radix[ax.nst - 1]) {
            case 2: last(std::integral_constant<int, 2>{}); break;
            case 3: last(std::integral_constant<int, 3>{}); break;
            case 4: last(std::integral_constant<int, 4>{}); break;
            case 5: last(std::integral_constant<int, 5>{}); break;
            case 6: last(std::integral_constant<int, 6>{}); break;
            default: last(std::integral_constant<int, 8>{}); break;
            }
        }
        const int iy = tb.freq[1][yp], fy = iy < (Y + 1) / 2 ? iy : iy - Y;
        auto bin = [&](auto rc) {
            constexpr int R = decltype(rc)::value;
            constexpr int NI = (FFT_COLS + R - 1) / R;
            const int nbf = Z / R * FFT_COLS;
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int q = tid + i * nt;
                const int ix = t * FFT_COLS + q % FFT_COLS;
                if (q < nbf && ix < Xh) {
                    const double w = (ix == 0 || (X % 2 == 0 && ix == X / 2)) ? 0.5 : 1.0;
#pragma unroll
                    for (int p = 0; p < R; ++p) {
                        // the last stage's sub-lines are single points
                        const int iz = tb.freq[2][q / FFT_COLS * R + p], fz = iz < (Z + 1) / 2 ? iz : iz - Z;
                        const int shell = shell_of(ix * ix + fy * fy + fz * fz);
                        atomicAdd(&hist[shell], w * e[i * R + p]);
                    }
                }
            }
        };
        switch (ax.radix[ax.nst - 1]) {
        case 2: bin(std::integral_constant<int, 2>{}); break;
        case 3: bin(std::integral_constant<int, 3>{}); break;
        case 4: bin(std::integral_constant<int, 4>{}); break;
        case 5: bin(std::integral_constant<int, 5>{}); break;
        case 6: bin(std::integral_constant<int, 6>{}); break;
        default: bin(std::integral_constant<int, 8>{}); break;
        }
    }
    __syncthreads();
    // (the sums by the square of the point count, at once: its reciprocal's rounding, squared, would
    // stand in every shell)
    const double npts = (double)X * (double)Y * (double)Z;
    for (int s = threadIdx.x; s < nshell; s += nt) part[(size_t)blockIdx.x * nshell + s] = hist[s] / (npts * npts);
}

// The fewest stages of radices 8 6 5 4 3 2 for a line of n points, largest last (the last stage has
// the most work left per butterfly); none if n is too long or has another prime factor.  One stage
// alone is preceded by a copy into LDS.
inline bool fft_radices(int n, int stages, int most, int *r)
{
    if (n == 1) return true;
    if (stages == 0) return false;
    for (int q : {8, 6, 5, 4, 3, 2})
        if (q <= most && n % q == 0) {
            r[0] = q;
            if (fft_radices(n / q, stages - 1, q, r + 1)) return true;
        }
    return false;
}

inline bool fft_axis(long long n, FftAxis *ax)
{
    if (n < 2 || n > FFT_MAX_LINE) return false;
    int r[FFT_MAX_STAGES] = {};
    int ns = 1;
    while (ns < FFT_MAX_STAGES && !fft_radices((int)n, ns, 8, r)) ++ns;
    if (!fft_radices((int)n, ns, 8, r)) return false;
    *ax = FftAxis{};
    ax->n = (int)n;
    int s = 0;
    if (ns == 1) ax->radix[s++] = 1;
    int m = (int)n;
    for (int i = 0; i < ns; ++i, ++s) {
        ax->radix[s] = r[ns - 1 - i];
        ax->step[s] = (int)n / m;
        m /= ax->radix[s];
        ax->sub[s] = m;
        ax->magic[s] = ((1u << 20) + m - 1) / m;
    }
    ax->nst = s;
    return true;
}

}  // namespace dg
