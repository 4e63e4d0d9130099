// plane.hpp -- zebra (r, phi)-plane relaxation for the 7-point operator with
// phi-invariant metrics.  Included by cps.hip after kernels.hpp.
//
// A half-sweep of parity k relaxes every theta row b = k (mod 2): each row's
// (r, phi) plane is solved exactly with the rows of the other parity held
// fixed (their theta fluxes go to the right-hand side), i.e. block
// Gauss-Seidel with the theta rows as blocks.  On a plane the metrics do not
// depend on phi, so the periodic phi coupling is diagonalised by a Fourier
// transform along phi and every azimuthal mode m leaves a tridiagonal system
// in r (the Thomas algorithm):
//
//   grl_a X_{a-1} + (-(grl_a + grh_a + gtl_a + gth_a) + gpp_a lam_m) X_a
//     + grh_a X_{a+1} = R_a,       lam_m = 2 cos(2 pi m / n_phi) - 2,
//
// R = FFT_phi(b - gtl x_{b-1} - gth x_{b+1}).  Three launches per half-sweep:
//  - k_plane_fwd: right-hand side of each (r, row) ring and its real Fourier
//    transform.  A ring of n_phi reals is the complex sequence
//    z_j = x_{2j} + i x_{2j+1}, exactly the two parity planes of the split
//    layout; a Stockham radix-4 transform of length n_phi/2 in LDS and the
//    usual even/odd recombination give the n_phi/2 + 1 modes.  The lanes of
//    a ring lie in one wavefront, so the stages need no block barrier;
//  - k_plane_tri: forward elimination and back substitution down and up the
//    r-line of every (row, mode), real and imaginary parts on two lanes.  The
//    inverse pivots and the off-diagonals depend on the operator only and
//    are computed once per set-up (k_plane_factor).  An r-line is split over
//    the wavefronts of a block, 16 cells each in registers, so the spectra
//    and the pivots cross memory once and the serial chain is 16 steps long
//    instead of n_r;
//  - k_plane_inv: the inverse transform back into the rows.
// Rows whose plane is small take one launch, k_plane_row, a block per row.  The
// first half-sweep from a zero iterate does not read it.
// Spectra and pivots are laid out [a][row][mode], so the r-line solves read
// and write consecutive modes across a wavefront.  The modes 0 and n_phi / 2
// of a real ring are real: they share slot 0 (real and imaginary part), so
// a ring's spectrum is n_phi reals, whole wavefronts and aligned rows.
//
// CROSS: the r-theta cross metrics of an axisymmetric map with cross terms
// (the oblate shell; G_r.phi = G_theta.phi = 0, so phi still decouples).  The
// theta-face cross terms couple a row's own r-neighbours, and where a theta
// wall mirrors row b -/+ 1 onto row b the r-face cross terms do too: the
// r-line stays tridiagonal (not symmetric) with phi-invariant coefficients
// (plane_row).  The cross terms that reach rows b -/+ 1 go to the
// right-hand side.

namespace cps {

template <typename T>
__device__ __forceinline__ Vec2<T> cmul(Vec2<T> a, Vec2<T> b)
{
    Vec2<T> r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}

template <typename T>
__device__ __forceinline__ Vec2<T> conjv(Vec2<T> a)
{
    a.y = -a.y;
    return a;
}

constexpr int kPlaneLds = 1024; // complex values per LDS buffer (rings x length)
constexpr int kTriBlock = 64;
constexpr int kTriBatch = 8;   // r-steps whose loads a lane issues together
constexpr int kLdBatch = 4;    // ring positions whose loads a lane issues together
constexpr int kSmallRing = 256; // ring-size class of the paper-scale shell

// Orders the LDS accesses of the lanes of one wavefront (no block barrier).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Where value i of a ring is held in LDS: the low bits of its index XORed with
// the two above a row of banks (16 complex FP64 values, 32 FP32 ones), in both
// pairs of bits, so that the first two radix-4 stages, whose lanes write 4 and
// 16 values apart, hit every bank as evenly as contiguous accesses do.  Not for
// the longer rings, whose registers do not hold the addresses.  With the stage's
// index division gone as well, paper-scale transforms and back: 103 -> 99 us
// (plane smoother), 147 -> 136 (phi-lines).
template <typename T, int NMAX>
__device__ __forceinline__ int sw(int i)
{
    if (NMAX > kSmallRing) return i;
    return i ^ (((i >> (sizeof(T) == 8 ? 4 : 5)) & 3) * 5);
}

// In-place Stockham transform of length n (a power of 2, <= kPlaneLds) of
// one ring held at A (value i at sw(i)), tpr lanes of one wavefront per ring: a radix-2 stage
// when log2 n is odd, then radix-4 stages.  A stage reads all of its inputs
// into registers before any lane writes, so one buffer serves; the lanes of
// a ring are one wavefront, so the stages need no block barrier.  tw[q] =
// exp(-2 pi i q / n) for q < n / 2 (in LDS); inverse: conjugate twiddles and
// rotations, no scaling.  NMAX bounds n (the register staging of a stage
// is sized for it: kernels are built for rings up to 256 and up to
// kPlaneLds).
//
// A radix-4 stage of span Ls merges the four length-Ls transforms at block
// offsets q n / 4 (q = 0..3, the residues q of the index mod 4 Ls / Ls) into
// one of length 4 Ls: y_{j + p Ls} = sum_q (-i)^{pq} W^{qj} X_q[j],
// W = exp(-2 pi i / (4 Ls)); W^{qj} = tw[q j n / (4 Ls)], and for an index
// past n / 2, tw[s] = -tw[s - n / 2].
template <typename T, int NMAX>
__device__ void wave_fft(Vec2<T>* A, int n, int tr, int tpr, const Vec2<T>* tw, bool inverse)
{
    // butterflies per lane of a radix-2 and a radix-4 stage
    constexpr int kB2 = NMAX / 128 > 0 ? NMAX / 128 : 1, kB4 = NMAX / 256 > 0 ? NMAX / 256 : 1;
    int Ls = 1;
    if (__builtin_ctz(n) & 1) {
        Vec2<T> u[kB2], v[kB2];
#pragma unroll
        for (int i = 0; i < kB2; ++i) {
            const int t = tr + i * tpr;
            if (t < n / 2) {
                u[i] = A[sw<T, NMAX>(t)];
                v[i] = A[sw<T, NMAX>(t + n / 2)];
            }
        }
        wave_sync();
#pragma unroll
        for (int i = 0; i < kB2; ++i) {
            const int t = tr + i * tpr;
            if (t < n / 2) {
                A[sw<T, NMAX>(2 * t)] = u[i] + v[i];
                A[sw<T, NMAX>(2 * t + 1)] = u[i] - v[i];
            }
        }
        wave_sync();
        Ls = 2;
    }
    for (; Ls < n; Ls *= 4) {
        const int stride = n / (4 * Ls);
        Vec2<T> c[kB4][4];
#pragma unroll
        for (int i = 0; i < kB4; ++i) {
            const int t = tr + i * tpr;
            if (t < n / 4) {
#pragma unroll
                for (int q = 0; q < 4; ++q) c[i][q] = A[sw<T, NMAX>(t + q * (n / 4))];
            }
        }
        wave_sync();
#pragma unroll
        for (int i = 0; i < kB4; ++i) {
            const int t = tr + i * tpr;
            if (t < n / 4) {
                const int j = t & (Ls - 1);
                const int s1 = j * stride, s3 = 3 * j * stride;
                Vec2<T> w1 = tw[s1], w2 = tw[2 * s1];
                Vec2<T> w3 = s3 < n / 2 ? tw[s3] : -tw[s3 - n / 2];
                if (inverse) {
                    w1.y = -w1.y;
                    w2.y = -w2.y;
                    w3.y = -w3.y;
                }
                const Vec2<T> c0 = c[i][0], c1 = cmul(w1, c[i][1]), c2 = cmul(w2, c[i][2]),
                              c3 = cmul(w3, c[i][3]);
                const Vec2<T> s02 = c0 + c2, d02 = c0 - c2, s13 = c1 + c3, d13 = c1 - c3;
                Vec2<T> rot; // -i d13 (forward), +i d13 (inverse)
                rot.x = inverse ? -d13.y : d13.y;
                rot.y = inverse ? d13.x : -d13.x;
                const int o = 4 * t - 3 * j; // 4 Ls (t / Ls) + j
                A[sw<T, NMAX>(o)] = s02 + s13;
                A[sw<T, NMAX>(o + Ls)] = d02 + rot;
                A[sw<T, NMAX>(o + 2 * Ls)] = s02 - s13;
                A[sw<T, NMAX>(o + 3 * Ls)] = d02 - rot;
            }
        }
        wave_sync();
    }
}

struct PlaneLaunch {
    int tpr, rb, threads, rows, rings, blocks;
};

// rows of parity k; lanes per ring (a power of two <= 64, so a ring never
// straddles wavefronts; four values of a ring a lane, so that a radix-4 stage
// keeps every lane busy: against two, a batch of 16 with rings of 128 to 256
// cells 34.1 -> 32.9 ms), rings per block (<= 256 lanes, <= kPlaneLds values;
// rb > 0 asks for at most that many: the autotuner's choice)
__host__ __device__ inline PlaneLaunch plane_launch(const Geo& g, int parity, int rb = 0)
{
    PlaneLaunch p;
    p.rows = (g.nt - parity + 1) / 2;
    p.tpr = g.nh < 8 ? 1 : (g.nh / 4 < 64 ? g.nh / 4 : 64);
    p.rb = kBlock / p.tpr;
    if (p.rb * g.nh > kPlaneLds) p.rb = kPlaneLds / g.nh;
    if (rb > 0 && rb < p.rb) p.rb = rb;
    p.threads = p.rb * p.tpr;
    p.rings = g.nr * p.rows;
    p.blocks = (p.rings + p.rb - 1) / p.rb;
    return p;
}

// The elimination's tables of one parity, in one array of nr rows (nh + 3)
// values: inverse pivots P[a][row][mode <= nh], and the r-line's sub- and
// super-diagonal off[a][row].
template <typename T>
struct TriTab {
    T* P;
    Vec2<T>* off;
};

template <typename T>
__host__ __device__ inline TriTab<T> tri_tab(const Geo& g, int parity, T* base)
{
    const long long n = (long long)g.nr * ((g.nt - parity + 1) / 2);
    TriTab<T> t;
    t.off = reinterpret_cast<Vec2<T>*>(base); // first: its pairs stay aligned
    t.P = base + 2 * n;
    return t;
}

// values of n rings' tables, rounded up to whole pairs
__host__ __device__ inline long long plane_pivots_of(long long n, int nh)
{
    return (n * (nh + 3) + 1) & ~1LL;
}
// values of a level's tables (both parities), and where parity k's begin
__host__ __device__ inline long long plane_pivots(const Geo& g)
{
    return plane_pivots_of((long long)g.nr * ((g.nt + 1) / 2), g.nh) +
           plane_pivots_of((long long)g.nr * (g.nt / 2), g.nh);
}
__host__ __device__ inline long long plane_pivot_offset(const Geo& g, int parity)
{
    return parity ? plane_pivots_of((long long)g.nr * ((g.nt + 1) / 2), g.nh) : 0;
}

// Right-hand sides of the rings of parity k and their real transforms:
// S[(a rows + bi) nh + m], m < nh; slot 0 holds (mode 0, mode nh), both real.
// The r-line of row b at a: sub x_{a-1} + (dia + G_pp lam_m) x_a + sup x_{a+1},
// with walls (zero metrics on wall faces, mirrored reads) included.
template <typename T, bool CROSS>
__device__ __forceinline__ void plane_row(const Geo& g, const T* __restrict__ G, long long gk,
                                          int a, int b, T& sub, T& dia, T& sup)
{
    const long long ci = (long long)a * g.nt + b;
    const T grl = G[ci];
    const T grh = a < g.nr - 1 ? G[ci + g.nt] : T(0);
    const T gtl = G[4 * gk + ci];
    const T gth = b < g.nt - 1 ? G[4 * gk + ci + 1] : T(0);
    sub = grl;
    sup = grh;
    dia = -(grl + grh + gtl + gth);
    if (CROSS) {
        // r-face cross terms whose row b -/+ 1 the theta walls mirror onto b
        const T qrl = T(0.25) * G[gk + ci];
        const T qrh = a < g.nr - 1 ? T(0.25) * G[gk + ci + g.nt] : T(0);
        if (b == g.nt - 1) {
            sup += qrh;
            dia += qrh - qrl;
            sub -= qrl;
        }
        if (b == 0) {
            sup -= qrh;
            dia += qrl - qrh;
            sub += qrl;
        }
        // theta-face cross terms on this row: (qth - qtl)(x_{a+1} - x_{a-1})
        const T qtl = T(0.25) * G[3 * gk + ci];
        const T qth = b < g.nt - 1 ? T(0.25) * G[3 * gk + ci + 1] : T(0);
        const T s = qth - qtl;
        if (a < g.nr - 1) sup += s;
        else dia += s;
        if (a > 0) sub -= s;
        else dia -= s;
    }
}

// Mode m < nh of a real ring from its half-length transform Z: zm = Z[m],
// zr = Z[nh - m] (Z[0] for m = 0), w = exp(-2 pi i m / n_phi).  Slot 0: modes 0
// and nh.
template <typename T>
__device__ __forceinline__ Vec2<T> ring_mode(int m, Vec2<T> zm, Vec2<T> zr, Vec2<T> w)
{
    const Vec2<T> zc = conjv(zr);
    // even part E = (zm + zc) / 2, odd part O = (zm - zc) / (2i)
    Vec2<T> E, O;
    E.x = T(0.5) * (zm.x + zc.x);
    E.y = T(0.5) * (zm.y + zc.y);
    O.x = T(0.5) * (zm.y - zc.y);
    O.y = -T(0.5) * (zm.x - zc.x);
    Vec2<T> X = E + cmul(w, O);
    if (m == 0) { // E + O and E - O, both real
        X.x = zm.x + zm.y;
        X.y = zm.x - zm.y;
    }
    return X;
}

// and back: Z[m] from xm = X[m], xr = X[nh - m] (X[0] for m = 0)
template <typename T>
__device__ __forceinline__ Vec2<T> ring_value(int m, Vec2<T> xm, Vec2<T> xr, Vec2<T> w)
{
    const Vec2<T> xc = conjv(xr);
    // E = (xm + xc) / 2, O = (xm - xc) conj(w) / 2, Z = E + i O
    Vec2<T> E, D;
    E.x = T(0.5) * (xm.x + xc.x);
    E.y = T(0.5) * (xm.y + xc.y);
    D.x = T(0.5) * (xm.x - xc.x);
    D.y = T(0.5) * (xm.y - xc.y);
    const Vec2<T> O = cmul(conjv(w), D);
    Vec2<T> z;
    z.x = E.x - O.y;
    z.y = E.y + O.x;
    if (m == 0) {
        z.x = T(0.5) * (xm.x + xm.y);
        z.y = T(0.5) * (xm.x - xm.y);
    }
    return z;
}

// Right-hand side of the ring (a, b) into A: b minus the terms of rows b -/+ 1;
// zero: the iterate is zero, so x is not read.
template <typename T, int NMAX, bool CROSS>
__device__ __forceinline__ void plane_rhs(const Geo& g, const T* __restrict__ G, long long gk,
                                          const T* __restrict__ bv, const T* __restrict__ x, int a,
                                          int b, int tr, int tpr, bool zero, Vec2<T>* A)
{
    const int nh = g.nh;
    if constexpr (CROSS) {
        // b + sum over rows b -/+ 1 at a - 1, a, a + 1 (mirrored in r) of
        // coefficient x value: the theta-face metrics and both faces' cross
        // terms (a mirrored position carries a zero metric or folds onto a)
        const long long ci = (long long)a * g.nt + b;
        const bool lo = b > 0 && !zero, hi = b < g.nt - 1;
        const bool up = hi && !zero;
        const T gtl = G[4 * gk + ci], gth = hi ? G[4 * gk + ci + 1] : T(0);
        const T qrl = T(0.25) * G[gk + ci];
        const T qrh = a < g.nr - 1 ? T(0.25) * G[gk + ci + g.nt] : T(0);
        const T qtl = T(0.25) * G[3 * gk + ci], qth = hi ? T(0.25) * G[3 * gk + ci + 1] : T(0);
        const T ch0 = -gth - qrh + qrl, chp = -qrh - qth, chm = qrl + qth;
        const T cl0 = -gtl + qrh - qrl, clp = qrh + qtl, clm = -qrl - qtl;
        const long long base = (long long)a * g.rowlen + (long long)b * nh;
        const long long dp = a < g.nr - 1 ? g.rowlen : 0, dm = a > 0 ? g.rowlen : 0;
        for (int j = tr; j < nh; j += tpr) {
            Vec2<T> z;
            z.x = ld_once(bv + base + j);
            z.y = ld_once(bv + g.P + base + j);
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const bool on = side ? up : lo;
                if (!on) continue;
                const long long r0 = base + (side ? nh : -nh) + j;
                const T c0 = side ? ch0 : cl0, cp = side ? chp : clp, cm = side ? chm : clm;
                z.x += c0 * x[r0] + cp * x[r0 + dp] + cm * x[r0 - dm];
                z.y += c0 * x[g.P + r0] + cp * x[g.P + r0 + dp] + cm * x[g.P + r0 - dm];
            }
            A[sw<T, NMAX>(j)] = z;
        }
    } else {
        const long long ci = (long long)a * g.nt + b;
        const T gtl = G[4 * gk + ci];
        const T gth = b < g.nt - 1 ? G[4 * gk + ci + 1] : T(0);
        const long long base = (long long)a * g.rowlen + (long long)b * nh;
        const bool lo = b > 0 && !zero, hi = b < g.nt - 1 && !zero;
        for (int j0 = tr; j0 < nh; j0 += kLdBatch * tpr) {
            // the loads of a batch are all issued before any is used
            T e[kLdBatch], o[kLdBatch], el[kLdBatch], ol[kLdBatch], eh[kLdBatch], oh[kLdBatch];
#pragma unroll
            for (int u = 0; u < kLdBatch; ++u) {
                const int j = j0 + u * tpr;
                if (j < nh) {
                    e[u] = ld_once(bv + base + j);
                    o[u] = ld_once(bv + g.P + base + j);
                    el[u] = lo ? x[base - nh + j] : T(0);
                    ol[u] = lo ? x[g.P + base - nh + j] : T(0);
                    eh[u] = hi ? x[base + nh + j] : T(0);
                    oh[u] = hi ? x[g.P + base + nh + j] : T(0);
                }
            }
#pragma unroll
            for (int u = 0; u < kLdBatch; ++u) {
                const int j = j0 + u * tpr;
                if (j < nh) {
                    Vec2<T> z;
                    z.x = e[u];
                    z.y = o[u];
                    if (lo) {
                        z.x -= gtl * el[u];
                        z.y -= gtl * ol[u];
                    }
                    if (hi) {
                        z.x -= gth * eh[u];
                        z.y -= gth * oh[u];
                    }
                    A[sw<T, NMAX>(j)] = z;
                }
            }
        }
    }
}

// Bodies take the logical block index (the batched form maps its blocks to
// problems); buf and twS are the block's LDS.
template <typename T, int NMAX, bool CROSS = false>
__device__ __forceinline__ void d_plane_fwd(unsigned blk, Vec2<T>* buf, Vec2<T>* twS, Geo g,
                                            const T* __restrict__ G, long long gk,
                                            const T* __restrict__ bv, const T* __restrict__ x,
                                            int parity, const Vec2<T>* __restrict__ tw,
                                            const Vec2<T>* __restrict__ twN,
                                            Vec2<T>* __restrict__ S, int rb, bool zero)
{
    const PlaneLaunch pl = plane_launch(g, parity, rb);
    const int nh = g.nh;
    for (int q = (int)threadIdx.x; q < nh / 2; q += pl.threads) twS[q] = tw[q];
    const int rl = (int)threadIdx.x / pl.tpr, tr = (int)threadIdx.x - rl * pl.tpr;
    const int ring = (int)blk * pl.rb + rl;
    // threads past the block's rings (a batched launch of a fixed block
    // size) only take part in the barrier
    const bool live = rl < pl.rb && ring < pl.rings;
    const int a = live ? ring / pl.rows : 0, bi = live ? ring - a * pl.rows : 0;
    const int b = 2 * bi + parity;
    Vec2<T>* A = buf + rl * nh;
    if (live) plane_rhs<T, NMAX, CROSS>(g, G, gk, bv, x, a, b, tr, pl.tpr, zero, A);
    __syncthreads(); // twiddles of the block (the ring's values are wave-local)
    if (!live) return;
    wave_fft<T, NMAX>(A, nh, tr, pl.tpr, twS, false);
    const Vec2<T>* Z = A;
    Vec2<T>* out = S + (long long)ring * nh;
    for (int m0 = tr; m0 < nh; m0 += kLdBatch * pl.tpr) {
        Vec2<T> w[kLdBatch];
#pragma unroll
        for (int u = 0; u < kLdBatch; ++u) {
            const int m = m0 + u * pl.tpr;
            if (m < nh) w[u] = twN[m];
        }
#pragma unroll
        for (int u = 0; u < kLdBatch; ++u) {
            const int m = m0 + u * pl.tpr;
            if (m < nh) {
                out[m] = ring_mode<T>(m, Z[sw<T, NMAX>(m)], Z[sw<T, NMAX>(m == 0 ? 0 : nh - m)], w[u]);
            }
        }
    }
}

template <typename T, int NMAX, bool CROSS>
__global__ void __launch_bounds__(kBlock) k_plane_fwd(Geo g, const T* __restrict__ G, long long gk,
                                                      const T* __restrict__ bv,
                                                      const T* __restrict__ x, int parity,
                                                      const Vec2<T>* __restrict__ tw,
                                                      const Vec2<T>* __restrict__ twN,
                                                      Vec2<T>* __restrict__ S, int rb, int zero)
{
    __shared__ Vec2<T> buf[kPlaneLds], twS[kPlaneLds / 2];
    d_plane_fwd<T, NMAX, CROSS>(blockIdx.x, buf, twS, g, G, gk, bv, x, parity, tw, twN, S, rb,
                                zero != 0);
}

// Inverse pivots of the Thomas elimination of every (row, mode) r-line of
// parity k, P = 1 / (diag - sub c_{a-1}) with c_a = sup_a P_a, and the
// off-diagonals (TriTab).  One thread per (row, mode); set-up only.
template <typename T, bool CROSS>
__global__ void __launch_bounds__(kBlock) k_plane_factor(Geo g, const T* __restrict__ G,
                                                         long long gk, int parity,
                                                         const T* __restrict__ lam,
                                                         T* __restrict__ base)
{
    const int rows = (g.nt - parity + 1) / 2;
    const int nm = g.nh + 1;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long long)rows * nm) return;
    const TriTab<T> tab = tri_tab(g, parity, base);
    const int bi = (int)(t / nm), m = (int)(t - (long long)bi * nm);
    const int b = 2 * bi + parity;
    const T lm = lam[m];
    T c = T(0);
    for (int a = 0; a < g.nr; ++a) {
        const long long ci = (long long)a * g.nt + b, row = (long long)a * rows + bi;
        T sub, dia, sup;
        plane_row<T, CROSS>(g, G, gk, a, b, sub, dia, sup);
        const T diag = dia + G[8 * gk + ci] * lm;
        const T inv = T(1) / (diag - sub * c);
        tab.P[row * nm + m] = inv;
        if (m == 0) {
            tab.off[row].x = sub;
            tab.off[row].y = sup;
        }
        c = sup * inv;
    }
}

// The r-line solves of every (row, mode) of parity k, in place in the spectra
// S (read as reals: lane u of a plane's 2 rows nh), with the tables of
// k_plane_factor.  Two forms, chosen by n_r:
//
// Chunked (n_r <= 256, tri_chunked): an r-line is split over nw = ceil(n_r / 16)
// wavefronts of one block, 16 cells each in registers, every load of a thread
// issued at once.  Each wavefront eliminates its chunk from a zero value
// below and forms how the chunk's last value depends on that value (the
// product of its factors -sub P); after one barrier it finds the value below
// from the chunks before it, one fma a chunk, and eliminates once more from
// there.  The back substitution does the same from above.  The factors are
// below 1 in magnitude (the pivots of a diagonally dominant line), so neither
// the products nor the carried values grow.  Bound by memory: spectra in and
// out and the pivots once, where the streaming form below reads spectra and
// pivots twice and waits on 2 n_r dependent steps.  Finest level of the
// 192 x 256 x 512 shell, FP64: 56.8 us (252 MB, 4.4 TB/s) against 97.2 us
// streaming; of the oblate 128 x 128 x 256 shell, FP32, where the streaming
// form has 258 wavefronts in all: 8.7 against 82.6 us.  16 cells a thread
// keep the FP64 form at 116 VGPRs (16 wavefronts a CU); lines of more than
// 256 cells would need more than one block of 1024 threads.
//
// Streaming (longer lines): Thomas down and up a whole line per thread, TB
// r-steps of loads in flight.
constexpr int kTriChunk = 16; // r-cells a thread of the chunked form holds
constexpr int kTriWaves = 16; // wavefronts of its largest block

// (32-bit byte offsets: spectra and pivots below 4 GiB in FP64)
__host__ __device__ inline bool tri_chunked(const Geo& g)
{
    return g.nr <= kTriChunk * kTriWaves &&
           8LL * g.nr * ((g.nt + 1) / 2) * (2LL * g.nh + 2) < (1LL << 32);
}

// Blocks of the elimination: nw wavefronts a line, gpb groups of 64 lines a
// block.  waves: the block's wavefronts (0: as many as the lines need, at
// least four).  Neither the grouping nor the block size changes a bit.
struct TriLaunch {
    int nw, gpb, threads;
    long long lanes;
    unsigned blocks;
};

__host__ __device__ inline TriLaunch tri_launch(const Geo& g, int parity, int waves = 0)
{
    TriLaunch t;
    t.lanes = 2LL * ((g.nt - parity + 1) / 2) * g.nh;
    t.nw = tri_chunked(g) ? (g.nr + kTriChunk - 1) / kTriChunk : 1;
    if (waves) t.gpb = waves / t.nw;
    else if (tri_chunked(g)) t.gpb = t.nw < 4 ? 4 / t.nw : 1;
    else t.gpb = 1;
    t.threads = 64 * (waves ? waves : t.nw * t.gpb);
    t.blocks = (unsigned)((t.lanes + 64 * t.gpb - 1) / (64 * t.gpb));
    return t;
}

// The wavefronts [lo, hi) of a block that hold the line of wavefront wv: it
// takes the values of the chunks below from [lo, wv), of those above from
// (wv, hi).  Wavefronts past a block's whole groups (a batched block is of one
// size whatever its lines need) hold no line and take none.
struct TriLine {
    int lo, hi;
    bool live;
};

__host__ __device__ inline TriLine tri_line(const TriLaunch& t, int wv)
{
    const int grp = wv / t.nw;
    if (grp >= t.gpb) return TriLine{wv, wv + 1, false};
    return TriLine{grp * t.nw, (grp + 1) * t.nw, true};
}

template <typename T>
struct TriLds {
    Vec2<T> f[kTriWaves][64], b[kTriWaves][64]; // a chunk's end value and its factor
};

// UNI: nh >= 32, so a wavefront's lines are of one row (its off-diagonals
// become scalar loads).
// INLDS: S is the plane of theta row ldsrow alone, [a][2 nh], in LDS, its
// complex values at sw().
template <typename T, bool UNI, bool INLDS = false>
__device__ __forceinline__ void d_tri_chunk(unsigned blk, const TriLaunch& tl, const Geo& g,
                                            int parity, const TriTab<T>& tab,
                                            T* __restrict__ S, TriLds<T>& sh,
                                            unsigned ldsrow = 0)
{
    constexpr int K = kTriChunk;
    const int rows = (g.nt - parity + 1) / 2, nh = g.nh, nr = g.nr;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    const TriLine ln = tri_line(tl, wv);
    const int grp = wv / tl.nw, c = wv - ln.lo; // the line's chunk c
    const unsigned u = (blk * (unsigned)tl.gpb + (unsigned)grp) * 64u + (unsigned)lane;
    const bool live = ln.live && u < (unsigned)tl.lanes;
    const unsigned t = live ? u >> 1 : 0u; // line
    const unsigned bl = INLDS ? ldsrow : t / (unsigned)nh;
    const unsigned m = INLDS ? t : t - bl * (unsigned)nh;
    const unsigned bi = UNI ? (unsigned)__builtin_amdgcn_readfirstlane((int)bl) : bl;
    // slot 0's imaginary lane carries mode nh
    const unsigned mp = m == 0 && (u & 1) ? (unsigned)nh : m;
    const int a0 = c * K, us = 2 * sw<T, kSmallRing>((int)(u >> 1)) + (int)(u & 1);
    // byte offsets of a lane's values at plane a0, and of a plane
    const unsigned ss = (unsigned)tl.lanes * sizeof(T), sp = (unsigned)rows * (nh + 1) * sizeof(T);
    const unsigned so = a0 * ss + u * (unsigned)sizeof(T);
    const unsigned po = a0 * sp + (bl * (unsigned)(nh + 1) + mp) * (unsigned)sizeof(T);
    T d[K], f[K], e[K]; // right-hand side x pivot, -sub x pivot, -sup x pivot
#pragma unroll
    for (int k = 0; k < K; ++k) {
        d[k] = T(0);
        e[k] = T(0);
        if (a0 + k < nr && live) {
            if constexpr (INLDS) d[k] = S[(a0 + k) * 2 * nh + us];
            else d[k] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(S) + (so + k * ss));
            e[k] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(tab.P) +
                                               (po + k * sp));
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        // a few of the per-lane pairs in flight at a time (registers)
        if (!UNI && k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        Vec2<T> o;
        o.x = o.y = T(0);
        if (a0 + k < nr) o = tab.off[(unsigned)(a0 + k) * (unsigned)rows + bi];
        d[k] *= e[k];
        f[k] = -o.x * e[k];
        e[k] *= -o.y;
    }
    T below = T(0);
    if (tl.nw > 1) {
        Vec2<T> v;
        v.x = T(0);
        v.y = T(1);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            v.x = fma_t(f[k], v.x, d[k]);
            v.y *= f[k];
        }
        sh.f[wv][lane] = v;
        __syncthreads();
        for (int w = ln.lo; w < wv; ++w) {
            const Vec2<T> q = sh.f[w][lane];
            below = fma_t(q.y, below, q.x);
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        below = fma_t(f[k], below, d[k]);
        d[k] = below;
    }
    T above = T(0);
    if (tl.nw > 1) {
        Vec2<T> v;
        v.x = T(0);
        v.y = T(1);
#pragma unroll
        for (int k = K - 1; k >= 0; --k) {
            v.x = fma_t(e[k], v.x, d[k]);
            v.y *= e[k];
        }
        sh.b[wv][lane] = v;
        __syncthreads();
        for (int w = ln.hi - 1; w > wv; --w) {
            const Vec2<T> q = sh.b[w][lane];
            above = fma_t(q.y, above, q.x);
        }
    }
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        above = fma_t(e[k], above, d[k]);
        if (a0 + k < nr && live) {
            if constexpr (INLDS) S[(a0 + k) * 2 * nh + us] = above;
            else *reinterpret_cast<T*>(reinterpret_cast<char*>(S) + (so + k * ss)) = above;
        }
    }
}

template <typename T, int TB = kTriBatch>
__device__ __forceinline__ void d_tri_stream(long long u, const Geo& g, int parity,
                                             const TriTab<T>& tab, T* __restrict__ S)
{
    const int rows = (g.nt - parity + 1) / 2;
    const int nh = g.nh, nr = g.nr;
    const long long lanes = 2LL * rows * nh; // one r-plane of spectra
    if (u >= lanes) return;
    const long long t = u >> 1;
    const int bi = (int)(t / nh);
    // slot 0's imaginary lane carries mode nh
    const bool nyq = t == (long long)bi * nh && (u & 1);
    const T* pb = tab.P + t + bi + (nyq ? nh : 0);
    const long long ps = (long long)rows * (nh + 1);
    T d = T(0);
    for (int a0 = 0; a0 < nr; a0 += TB) {
        T r[TB], p[TB], gl[TB];
#pragma unroll
        for (int k = 0; k < TB; ++k) {
            const int a = a0 + k;
            if (a < nr) {
                r[k] = S[a * lanes + u];
                p[k] = pb[a * ps];
                gl[k] = tab.off[(long long)a * rows + bi].x;
            }
        }
#pragma unroll
        for (int k = 0; k < TB; ++k) {
            const int a = a0 + k;
            if (a < nr) {
                d = (r[k] - gl[k] * d) * p[k];
                S[a * lanes + u] = d;
            }
        }
    }
    T xn = d; // X at a = nr - 1
    for (int a0 = nr - 2; a0 >= 0; a0 -= TB) {
        T s[TB], p[TB], gh[TB];
#pragma unroll
        for (int k = 0; k < TB; ++k) {
            const int a = a0 - k;
            if (a >= 0) {
                s[k] = S[a * lanes + u];
                p[k] = pb[a * ps];
                gh[k] = tab.off[(long long)a * rows + bi].y;
            }
        }
#pragma unroll
        for (int k = 0; k < TB; ++k) {
            const int a = a0 - k;
            if (a >= 0) {
                const T c = gh[k] * p[k];
                xn = s[k] - c * xn;
                S[a * lanes + u] = xn;
            }
        }
    }
}

template <typename T, bool UNI>
__global__ void __launch_bounds__(64 * kTriWaves) k_plane_tri(Geo g, int parity,
                                                              const T* __restrict__ piv,
                                                              T* __restrict__ S)
{
    __shared__ TriLds<T> sh;
    d_tri_chunk<T, UNI>(blockIdx.x, tri_launch(g, parity), g, parity,
                        tri_tab<T>(g, parity, const_cast<T*>(piv)), S, sh);
}

template <typename T, int TB>
__global__ void __launch_bounds__(kTriBlock) k_plane_tri_stream(Geo g, int parity,
                                                                const T* __restrict__ piv,
                                                                T* __restrict__ S)
{
    d_tri_stream<T, TB>((long long)blockIdx.x * blockDim.x + threadIdx.x, g, parity,
                        tri_tab<T>(g, parity, const_cast<T*>(piv)), S);
}

// r-steps in flight per lane of the streaming elimination: the candidates the
// autotuner times (the same arithmetic in the same order for each)
__host__ __device__ inline int tri_batch_of(int tb) { return tb == 4 || tb == 16 ? tb : kTriBatch; }


// Inverse transforms of the solved spectra into the rows of parity k.
template <typename T, int NMAX>
__device__ __forceinline__ void d_plane_inv(unsigned blk, Vec2<T>* buf, Vec2<T>* twS, Geo g,
                                            int parity, const Vec2<T>* __restrict__ tw,
                                            const Vec2<T>* __restrict__ twN,
                                            const Vec2<T>* __restrict__ S, T* __restrict__ x,
                                            int rb = 0)
{
    const PlaneLaunch pl = plane_launch(g, parity, rb);
    const int nh = g.nh;
    for (int q = (int)threadIdx.x; q < nh / 2; q += pl.threads) twS[q] = tw[q];
    const int rl = (int)threadIdx.x / pl.tpr, tr = (int)threadIdx.x - rl * pl.tpr;
    const int ring = (int)blk * pl.rb + rl;
    const bool live = rl < pl.rb && ring < pl.rings;
    Vec2<T>* A = buf + rl * nh;
    if (live) {
        const Vec2<T>* X = S + (long long)ring * nh;
        for (int m0 = tr; m0 < nh; m0 += kLdBatch * pl.tpr) {
            Vec2<T> xm[kLdBatch], xc[kLdBatch], w[kLdBatch];
#pragma unroll
            for (int u = 0; u < kLdBatch; ++u) {
                const int m = m0 + u * pl.tpr;
                if (m < nh) {
                    xm[u] = X[m];
                    xc[u] = X[m == 0 ? 0 : nh - m];
                    w[u] = twN[m];
                }
            }
#pragma unroll
            for (int u = 0; u < kLdBatch; ++u) {
                const int m = m0 + u * pl.tpr;
                if (m < nh) {
                    A[sw<T, NMAX>(m)] = ring_value<T>(m, xm[u], xc[u], w[u]);
                }
            }
        }
    }
    __syncthreads(); // twiddles of the block (the ring's values are wave-local)
    if (!live) return;
    wave_fft<T, NMAX>(A, nh, tr, pl.tpr, twS, true);
    const Vec2<T>* z = A;
    const int a = ring / pl.rows, bi = ring - a * pl.rows;
    const int b = 2 * bi + parity;
    const long long base = (long long)a * g.rowlen + (long long)b * nh;
    const T s = T(1) / T(nh);
    for (int j = tr; j < nh; j += pl.tpr) {
        const Vec2<T> v = z[sw<T, NMAX>(j)];
        x[base + j] = v.x * s;
        x[g.P + base + j] = v.y * s;
    }
}

template <typename T, int NMAX>
__global__ void __launch_bounds__(kBlock) k_plane_inv(Geo g, int parity,
                                                      const Vec2<T>* __restrict__ tw,
                                                      const Vec2<T>* __restrict__ twN,
                                                      const Vec2<T>* __restrict__ S,
                                                      T* __restrict__ x, int rb)
{
    __shared__ Vec2<T> buf[kPlaneLds], twS[kPlaneLds / 2];
    d_plane_inv<T, NMAX>(blockIdx.x, buf, twS, g, parity, tw, twN, S, x, rb);
}

// ---------------------------------------------------------------------------
// A half-sweep in one launch, where a row's (r, phi) plane is small: a block
// per relaxed theta row makes its right-hand side, transforms the rings,
// solves the r-lines and transforms back without leaving LDS; the arithmetic
// is that of the three kernels.  Bound by latency: three launches take 4 to
// 6 us each whatever a small level holds, one takes the sum of their chains.
// Measured, a half-sweep (n_r x n_phi/2 a row, three launches -> one): FP32
// 16 x 16 12.0 -> 9.1 us, 32 x 32 13.0 -> 10.9, but 64 x 64 15.5 -> 24 and
// 128 x 128 33 -> 75; FP64 12 x 16 17.0 -> 8.4, 24 x 32 13.2 -> 11.3, but
// 48 x 64 15.8 -> 22: a larger plane gives one block per row too long a chain,
// on few CUs.  The line lies at the largest square plane that gained.
// ---------------------------------------------------------------------------

constexpr int kRowCells = 1024; // complex values of the largest plane

__host__ __device__ inline bool plane_row_fits(const Geo& g)
{
    return tri_chunked(g) && g.nh <= kSmallRing && (long long)g.nr * g.nh <= kRowCells;
}

// threads of a row's block: a ring's lanes for every r (or all that fit), and
// the wavefronts of an r-line
__host__ __device__ inline int plane_row_threads(const Geo& g)
{
    const int tpr = g.nh / 2 < 64 ? g.nh / 2 : 64;
    const int nw = (g.nr + kTriChunk - 1) / kTriChunk, groups = (2 * g.nh + 63) / 64;
    int t = (g.nr * tpr + 63) / 64;
    if (t < nw * groups) t = nw * groups;
    return 64 * (t < kTriWaves ? t : kTriWaves);
}

template <typename T>
struct PlaneRowLds {
    Vec2<T> A[kRowCells], tw[kSmallRing / 2], twN[kSmallRing];
    TriLds<T> tri;
};

template <typename T, bool CROSS>
__device__ __forceinline__ void d_plane_row(unsigned bi, PlaneRowLds<T>& sh, const Geo& g,
                                            const T* __restrict__ G, long long gk,
                                            const T* __restrict__ bv, T* __restrict__ x, int parity,
                                            const Vec2<T>* __restrict__ tw,
                                            const Vec2<T>* __restrict__ twN,
                                            const T* __restrict__ piv, bool zero)
{
    constexpr int V = kSmallRing / 64; // values of a ring per lane, at most
    const int nh = g.nh, nr = g.nr, b = 2 * (int)bi + parity;
    const int tpr = nh / 2 < 64 ? nh / 2 : 64, threads = (int)blockDim.x;
    for (int q = (int)threadIdx.x; q < nh; q += threads) {
        if (q < nh / 2) sh.tw[q] = tw[q];
        sh.twN[q] = twN[q];
    }
    // the lanes of a ring are of one wavefront: rings go by wavefronts' worths
    const int rl = (int)threadIdx.x / tpr, tr = (int)threadIdx.x - rl * tpr, rings = threads / tpr;
    for (int a = rl; a < nr; a += rings)
        plane_rhs<T, kSmallRing, CROSS>(g, G, gk, bv, x, a, b, tr, tpr, zero, sh.A + a * nh);
    __syncthreads(); // twiddles
    for (int a = rl; a < nr; a += rings) {
        Vec2<T>* A = sh.A + a * nh;
        wave_sync();
        wave_fft<T, kSmallRing>(A, nh, tr, tpr, sh.tw, false);
        Vec2<T> X[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int m = tr + i * tpr;
            if (m < nh)
                X[i] = ring_mode<T>(m, A[sw<T, kSmallRing>(m)],
                                    A[sw<T, kSmallRing>(m == 0 ? 0 : nh - m)], sh.twN[m]);
        }
        wave_sync();
#pragma unroll
        for (int i = 0; i < V; ++i)
            if (tr + i * tpr < nh) A[sw<T, kSmallRing>(tr + i * tpr)] = X[i];
    }
    __syncthreads();
    // the r-lines, as many groups of 64 at a time as the block has wavefronts for
    TriLaunch tl;
    tl.lanes = 2 * nh;
    tl.nw = (nr + kTriChunk - 1) / kTriChunk;
    tl.gpb = (threads >> 6) / tl.nw;
    const TriTab<T> tab = tri_tab<T>(g, parity, const_cast<T*>(piv));
    for (unsigned k = 0; k * 64u * (unsigned)tl.gpb < (unsigned)tl.lanes; ++k) {
        d_tri_chunk<T, true, true>(k, tl, g, parity, tab, reinterpret_cast<T*>(sh.A), sh.tri, bi);
        __syncthreads();
    }
    const T s = T(1) / T(nh);
    for (int a = rl; a < nr; a += rings) {
        Vec2<T>* A = sh.A + a * nh;
        Vec2<T> Z[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int m = tr + i * tpr;
            if (m < nh)
                Z[i] = ring_value<T>(m, A[sw<T, kSmallRing>(m)],
                                     A[sw<T, kSmallRing>(m == 0 ? 0 : nh - m)], sh.twN[m]);
        }
        wave_sync();
#pragma unroll
        for (int i = 0; i < V; ++i)
            if (tr + i * tpr < nh) A[sw<T, kSmallRing>(tr + i * tpr)] = Z[i];
        wave_sync();
        wave_fft<T, kSmallRing>(A, nh, tr, tpr, sh.tw, true);
        const long long base = (long long)a * g.rowlen + (long long)b * nh;
        for (int j = tr; j < nh; j += tpr) {
            const Vec2<T> v = A[sw<T, kSmallRing>(j)];
            x[base + j] = v.x * s;
            x[g.P + base + j] = v.y * s;
        }
    }
}

template <typename T, bool CROSS>
__global__ void __launch_bounds__(64 * kTriWaves)
    k_plane_row(Geo g, const T* __restrict__ G, long long gk, const T* __restrict__ bv,
                T* __restrict__ x, int parity, const Vec2<T>* __restrict__ tw,
                const Vec2<T>* __restrict__ twN, const T* __restrict__ piv, int zero)
{
    __shared__ PlaneRowLds<T> sh;
    d_plane_row<T, CROSS>(blockIdx.x, sh, g, G, gk, bv, x, parity, tw, twN, piv, zero != 0);
}

} // namespace cps
