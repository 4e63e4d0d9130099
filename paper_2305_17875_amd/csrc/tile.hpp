// tile.hpp -- the V-cycle's small levels in two launches each.  Included by
// cps.hip after kernels.hpp.
//
// On a small level (a few hundred thousand cells or fewer) every kernel of
// the cycle is short and its launch dominates: 11 launches a level (4
// pre-smoothing passes, residual, restriction, prolongation, 4
// post-smoothing passes).  Here the cycle's work on such a level is two
// launches, each block owning one 8 x 8 x 8 tile of cells and working in LDS:
//  - pre: red-black Gauss-Seidel from a zero iterate (colours 0, 1, 0, 1),
//    the residual of the smoothed iterate, and its full-weighting
//    restriction onto the tile's 4 x 4 x 4 coarse cells;
//  - post: the trilinear prolongation of the coarse correction added to the
//    iterate, then the colours 1, 0, 1, 0.
// Same operator, smoother, transfers and wall treatment as the per-kernel
// path (7-point stencil with phi-invariant metrics, Sec. on the multigrid
// solver): the results agree with it to rounding.  The sums are formed in
// another order, so the bits differ; the single and batched forms share
// these bodies, so they agree with each other bit for bit.
//
// A pass on a tile needs the other colour one cell beyond the cells it
// updates, so the tile is loaded with a halo and the passes shrink the
// region they update by one cell each: pre loads a halo of 5 (the zero pass
// reads no neighbour; three more passes; the residual one cell beyond the
// tile; its neighbours one beyond that), post a halo of 4.  Halo cells are
// recomputed by every tile that loads them and written only by their own
// tile; post reads the iterate of one buffer and writes another, so no
// block reads a cell another block has already overwritten.  Cells past the
// r- and theta-walls are zero in LDS and meet a zero wall metric; phi
// wraps.
//
// Pre ends on the black pass, so the black residual is zero (to rounding):
// only the red residual is formed and restricted, as on the row-pair
// levels of the per-kernel path.

namespace cps {

constexpr int kTile = 8;            // owned cells per dimension
constexpr int kTileThreads = 1024;  // threads per tile block
constexpr int kPreHalo = 5, kPostHalo = 4;
constexpr int kPreR = kTile + 2 * kPreHalo;   // 18
constexpr int kPostR = kTile + 2 * kPostHalo; // 16
constexpr int kCoarseR = kTile / 2 + 6;       // coarse correction box of post

// A level takes the tile path when it is small enough that its launches
// dominate (the finest level only in cycles from a zero iterate); its rings
// need not be whole tiles.  FP32: up to 512 K cells (48 x 64 x 128 in two
// rounds of blocks: 28 us against 52 of eleven per-kernel launches).  FP64:
// up to 64 K cells (24 x 32 x 64: 15 us against 46), and coarse levels whose
// rows are not whole wavefronts, which the per-kernel passes take a cell a
// thread, up to 256 K (40 x 48 x 72: 21 us against 45; 20 x 24 x 36: 15
// against 45).  The other FP64 levels above 64 K keep the passes although
// tiles are faster there too up to 512 K (whole cycles, passes / tiles:
// finest level 16 x 32 x 160 58 / 37 us, 40 x 48 x 72 66 / 48, 48 x 64 x 128
// 75 / 60, 64 x 64 x 128 77 / 67; as the level below 96 x 128 x 256
// 145 / 127): the profiling classes of a finest level of that size time its
// passes one by one, and the coarse limit is that of the finest level.
constexpr long long kTileMaxCells = 1LL << 16;
constexpr long long kTileMaxRagged = 1LL << 18;
constexpr long long kTileMaxCells32 = 1LL << 19;

// level l of the hierarchy
__host__ __device__ inline bool tile_fits(const Geo& g, int l, bool fp32)
{
    const long long most = fp32 ? kTileMaxCells32
                                : (l > 0 && g.nh % 64 != 0 ? kTileMaxRagged : kTileMaxCells);
    return g.nr % 2 == 0 && g.nt % 2 == 0 && (long long)g.nr * g.nt * g.np <= most;
}

__host__ __device__ inline int tile_count(const Geo& g)
{
    return cdiv(g.nr, kTile) * cdiv(g.nt, kTile) * cdiv(g.np, kTile);
}

__device__ __forceinline__ void tile_origin(const Geo& g, int t, int& A0, int& B0, int& C0)
{
    const int nc = cdiv(g.np, kTile), nb = cdiv(g.nt, kTile);
    C0 = (t % nc) * kTile;
    t /= nc;
    B0 = (t % nb) * kTile;
    A0 = (t / nb) * kTile;
}

// offset of cell (a, b, c) in the parity-split layout
__device__ __forceinline__ long long tile_at(const Geo& g, int a, int b, int c)
{
    return (long long)(c & 1) * g.P + (long long)a * g.rowlen + (long long)b * g.nh + (c >> 1);
}

__device__ __forceinline__ int wrapi(int c, int n)
{
    c %= n;
    return c < 0 ? c + n : c;
}

// metrics of row (a, b): the five face values and 1 / D (D: minus the sum
// of all six; a product in the passes, not a division on their dependent
// chain)
template <typename T>
__device__ __forceinline__ void tile_metrics(const Geo& g, const T* __restrict__ G, long long gk,
                                             int a, int b, T m[6])
{
    const long long ci = (long long)a * g.nt + b;
    m[0] = G[ci];                                  // r low
    m[1] = a < g.nr - 1 ? G[ci + g.nt] : T(0);     // r high
    m[2] = G[4 * gk + ci];                         // theta low
    m[3] = b < g.nt - 1 ? G[4 * gk + ci + 1] : T(0); // theta high
    m[4] = G[8 * gk + ci];                         // phi (both faces)
    m[5] = T(1) / -(m[0] + m[1] + m[2] + m[3] + m[4] + m[4]);
}

// Both kernels: a thread owns NP phi pairs of one row (a, b) of the box (a pair
// is one red and one black cell), pair t of the row's thread j being number u
// with t = j + u STEP.  Indices are formed once; the row's metrics, the right-
// hand sides and the thread's own values stay in registers, and a pass reads
// from LDS only the five neighbours that other threads own.  x in LDS is
// [colour][u][thread], so that every read and write of a wavefront is of
// consecutive words: the r and theta neighbours of a pair's cell of one colour
// are the other colour's cells of the pairs of the rows around, at a fixed
// thread distance.
// Bound by the chain of a launch: about 2 us to start, 2 to the first values,
// 0.5 to 0.9 an LDS exchange, one write.  Measured against one cell per thread
// and pass with indices, metrics and b in LDS, FP64 pre + post: 32 x 32 x 32
// 10.4 + 8.6 -> 8.6 + 7.3 us, 24 x 32 x 64 9.7 + 7.3 -> 7.8 + 6.7; FP32
// 48 x 64 x 128 17.1 + 13.7 -> 15.1 + 12.5.  48 KB of LDS and 62 registers let
// two FP64 blocks share a CU (before: one, of 117 KB).

// tile_metrics of a thread's row in registers; all zero past the walls
template <typename T>
struct TileRow {
    T rl, rh, tl, th, p, inv;
    bool in;
};

template <typename T>
__device__ __forceinline__ TileRow<T> tile_row(const Geo& g, const T* __restrict__ G, long long gk,
                                               int a, int b, bool in)
{
    TileRow<T> m;
    m.in = in;
    m.rl = m.rh = m.tl = m.th = m.p = m.inv = T(0);
    if (in) {
        T v[6];
        tile_metrics(g, G, gk, a, b, v);
        m.rl = v[0];
        m.rh = v[1];
        m.tl = v[2];
        m.th = v[3];
        m.p = v[4];
        m.inv = v[5];
    }
    return m;
}

// phi index c of a box cell (no more than 13 past either end of the ring) on the ring
__device__ __forceinline__ int wrap_near(int c, int np)
{
    if (np < 16) return wrapi(c, np);
    return c < 0 ? c + np : (c >= np ? c - np : c);
}

template <typename T>
struct TilePreLds {
    T x[2][3][kTileThreads];
};

template <typename T>
struct TilePostLds {
    T x[2][2][kTileThreads];
    T e[kCoarseR * kCoarseR * kCoarseR];
};

// a thread's place in the box: its row, its pairs t = j + u STEP, and the
// distance in LDS from a pair to the one whose cell is the phi neighbour of
// the pair's red cell (the other phi neighbour is the pair's own black cell);
// of its black cell the neighbour is on the other side
template <int R, int NP>
struct TilePos {
    static constexpr int STEP = R / 2 / NP;
    int aa, bb, j, red, dn[2];

    __device__ __forceinline__ TilePos(int ra, int rb, int rc)
    {
        const int tid = (int)threadIdx.x, row = tid / STEP;
        j = tid - row * STEP;
        aa = row / R;
        bb = row - aa * R;
        // box parity (cc & 1) of the row's red cells
        red = (ra + aa + rb + bb + rc) & 1;
        const int up = j == STEP - 1 ? kTileThreads - (STEP - 1) : 1;
        const int lo = j == 0 ? STEP - 1 - kTileThreads : -1;
        dn[0] = red ? up : lo;
        dn[1] = red ? lo : up;
    }
    __device__ __forceinline__ bool rows(int s) const // row in [s, R - s)^2
    {
        return aa >= s && aa < R - s && bb >= s && bb < R - s;
    }
    __device__ __forceinline__ bool cell(int u, int col, int s) const // cell in [s, R - s)
    {
        const int cc = 2 * (j + u * STEP) + (red ^ col);
        return cc >= s && cc < R - s;
    }
};

// One pass of colour COL over the region [s, R - s)^3 of a tile's LDS copy:
// each cell takes x = (b - S) / D from its six neighbours.
template <int COL, int R, int NP, typename T>
__device__ __forceinline__ void tile_pass(const TileRow<T>& m, const TilePos<R, NP>& p, int s,
                                          T (&x)[2][NP], const T (&bw)[2][NP],
                                          T (&X)[2][NP][kTileThreads])
{
    constexpr int STEP = TilePos<R, NP>::STEP;
    if (!m.in || !p.rows(s)) return;
    const int tid = (int)threadIdx.x;
#pragma unroll
    for (int u = 0; u < NP; ++u)
        if (p.cell(u, COL, s)) {
            const T* n = &X[1 - COL][u][tid];
            const T S = m.rh * n[R * STEP] + m.rl * n[-R * STEP] + m.th * n[STEP] +
                        m.tl * n[-STEP] + m.p * (x[1 - COL][u] + n[p.dn[COL]]);
            x[COL][u] = (bw[COL][u] - S) * m.inv;
            X[COL][u][tid] = x[COL][u];
        }
}

// Pre: bc (the tile's coarse cells) = R r, r = b - A x, x = 2 red-black
// sweeps from zero of A x = b; x is written on the tile's cells.
template <typename T>
__device__ __forceinline__ void d_vpre_tile(Blk bk, Geo f, const T* __restrict__ G, long long gk,
                                            const T* __restrict__ bv, T* __restrict__ x,
                                            Geo c, T* __restrict__ bc, TilePreLds<T>& sh)
{
    constexpr int R = kPreR, H = kPreHalo, NP = 3, STEP = TilePos<R, NP>::STEP;
    static_assert(R * R * STEP <= kTileThreads, "threads of a tile");
    if ((int)bk.L >= tile_count(f)) return; // whole block
    int A0, B0, C0;
    tile_origin(f, (int)bk.L, A0, B0, C0);
    const int ra = A0 - H, rb = B0 - H, rc = C0 - H;
    const TilePos<R, NP> p(ra, rb, rc);
    const int tid = (int)threadIdx.x, a = ra + p.aa, b = rb + p.bb;
    const bool live = p.aa < R && a >= 0 && a < f.nr && b >= 0 && b < f.nt;
    const int ro = a * f.rowlen + b * f.nh, P = (int)f.P;
    T bw[2][NP], xv[2][NP]; // [colour][pair]
#pragma unroll
    for (int u = 0; u < NP; ++u)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int cg = wrap_near(rc + 2 * (p.j + u * STEP) + (p.red ^ q), f.np);
            bw[q][u] = T(0);
            if (live) bw[q][u] = bv[ro + (cg & 1) * P + (cg >> 1)];
        }
    const TileRow<T> m = tile_row<T>(f, G, gk, a, b, live);
    // the first pass from zero reads no neighbour: x = b / D on the red cells
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        sh.x[0][u][tid] = xv[0][u] = bw[0][u] * m.inv;
        sh.x[1][u][tid] = xv[1][u] = T(0);
    }
    __syncthreads();
    tile_pass<1, R, NP>(m, p, 1, xv, bw, sh.x);
    __syncthreads();
    tile_pass<0, R, NP>(m, p, 2, xv, bw, sh.x);
    __syncthreads();
    tile_pass<1, R, NP>(m, p, 3, xv, bw, sh.x);
    __syncthreads();
    // the red residual on the tile +- 1, in place of the red cells in LDS
    // (which only their own thread still needs); the tile's cells of x
    if (live && p.rows(H - 1)) {
        const bool wr = p.rows(H);
#pragma unroll
        for (int u = 0; u < NP; ++u) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int cg = rc + 2 * (p.j + u * STEP) + (p.red ^ q);
                if (wr && p.cell(u, q, H) && cg < f.np) x[ro + (cg & 1) * P + (cg >> 1)] = xv[q][u];
            }
            if (!p.cell(u, 0, H - 1)) continue;
            const T* n = &sh.x[1][u][tid];
            const T v = xv[0][u];
            const T y = m.rh * (n[R * STEP] - v) - m.rl * (v - n[-R * STEP]) + m.th * (n[STEP] - v) -
                        m.tl * (v - n[-STEP]) + m.p * ((xv[1][u] - v) + (n[p.dn[0]] - v));
            sh.x[0][u][tid] = bw[0][u] - y;
        }
    }
    __syncthreads();
    // full weighting onto the coarse cells I = A0/2 .. +3 (weights 1 3 3 1
    // over fine 2I-1 .. 2I+2 in each direction, rows and planes clamped at
    // the walls, phi wrapped): 16 lanes a coarse cell, one of the 4 x 4 fine
    // rows each, of which two cells are red
    constexpr int K4 = kTile / 2;
    const int q = tid & 15, cell = tid >> 4;
    const int kk = cell % K4, jj = (cell / K4) % K4, ii = cell / (K4 * K4);
    const int I = A0 / 2 + ii, J = B0 / 2 + jj, K = C0 / 2 + kk;
    const bool on = I < c.nr && J < c.nt && K < c.np;
    const T w0 = T(0.25), w1 = T(0.75);
    const int qa = q >> 2, qb = q & 3;
    T sum = T(0);
    if (on) {
        const int fa = clampi(2 * I - 1 + qa, f.nr - 1) - ra, fb = clampi(2 * J - 1 + qb, f.nt - 1) - rb;
        const int rd = (ra + fa + rb + fb + rc) & 1;
        // fine c = 2K - 1 .. 2K + 2 at cc = 2t .. 2t + 3, t = kk + (H - 1) / 2:
        // red are the first and third of a row of red parity 0, else the
        // second and fourth
        const int t0 = kk + (H - 1) / 2, t1 = t0 + 1, row = fa * R + fb;
        const T* r = &sh.x[0][0][row * STEP];
        const T r0 = r[t0 / STEP * kTileThreads + t0 % STEP];
        const T r1 = r[t1 / STEP * kTileThreads + t1 % STEP];
        const T ph = (rd ? w1 : w0) * r0 + (rd ? w0 : w1) * r1;
        sum = ((qa == 0 || qa == 3 ? w0 : w1) * (qb == 0 || qb == 3 ? w0 : w1)) * ph;
    }
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) sum += __shfl_xor(sum, d);
    if (on && q == 0) bc[tile_at(c, I, J, K)] = sum;
}

// Post: xo = 2 red-black sweeps (colours 1, 0, 1, 0) of A x = b from
// xi + P e on the tile's cells.  The first pass overwrites every black cell
// unread, so only xi's red cells are read and corrected.  Returns the
// thread's part of the sum of b . xo.
template <typename T>
__device__ __forceinline__ double d_vpost_tile(Blk bk, Geo f, const T* __restrict__ G, long long gk,
                                               const T* __restrict__ bv, const T* __restrict__ xi,
                                               T* __restrict__ xo, Geo c, const T* __restrict__ e,
                                               TilePostLds<T>& sh)
{
    constexpr int R = kPostR, H = kPostHalo, E = kCoarseR, NP = 2, STEP = TilePos<R, NP>::STEP;
    static_assert(R * R * STEP == kTileThreads && E * E * E <= kTileThreads, "threads of a tile");
    if ((int)bk.L >= tile_count(f)) return 0.0; // whole block
    int A0, B0, C0;
    tile_origin(f, (int)bk.L, A0, B0, C0);
    const int ra = A0 - H, rb = B0 - H, rc = C0 - H;
    // coarse box: I = A0/2 - 3 .. A0/2 + 6 (rows and planes clamped, phi wrapped)
    const int ea = A0 / 2 - 3, eb = B0 / 2 - 3, ec = C0 / 2 - 3;
    const TilePos<R, NP> p(ra, rb, rc);
    const int tid = (int)threadIdx.x, a = ra + p.aa, b = rb + p.bb;
    const bool live = a >= 0 && a < f.nr && b >= 0 && b < f.nt;
    const int ro = a * f.rowlen + b * f.nh, P = (int)f.P;
    T ev = T(0);
    if (tid < E * E * E) {
        const int kc = tid % E, kb = (tid / E) % E, ka = tid / (E * E);
        const int cg = wrap_near(ec + kc, c.np);
        ev = e[(cg & 1) * (int)c.P + clampi(ea + ka, c.nr - 1) * c.rowlen +
               clampi(eb + kb, c.nt - 1) * c.nh + (cg >> 1)];
    }
    T bw[2][NP], xv[2][NP], xr[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        xr[u] = bw[0][u] = bw[1][u] = T(0);
        if (live) {
            // rc is even: a pair's two cells are at one index of both planes
            const int o = ro + (wrap_near(rc + 2 * (p.j + u * STEP), f.np) >> 1);
            const int or_ = o + (p.red ? P : 0), ob = o + (p.red ? 0 : P);
            bw[0][u] = bv[or_];
            bw[1][u] = bv[ob];
            xr[u] = xi[or_];
        }
    }
    const TileRow<T> m = tile_row<T>(f, G, gk, a, b, live);
    if (tid < E * E * E) sh.e[tid] = ev;
    __syncthreads();
    const T w0 = T(0.75), w1 = T(0.25);
    // fine 2I takes 3/4 of coarse I and 1/4 of I - 1, fine 2I + 1 of I and
    // I + 1, in each direction: theta, then phi, then r
    const int da = (a & 1) ? E * E : -E * E, db = (b & 1) ? E : -E, dc = p.red ? 1 : -1;
    const T* e0 = sh.e + ((a >> 1) - ea) * E * E + ((b >> 1) - eb) * E + rc / 2 - ec + p.j;
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        T v = T(0);
        if (live) {
            const T* ee = e0 + u * STEP;
            T tr[2];
#pragma unroll
            for (int pa = 0; pa < 2; ++pa) {
                T tp[2];
#pragma unroll
                for (int pc = 0; pc < 2; ++pc) {
                    const T* q = ee + (pa ? da : 0) + (pc ? dc : 0);
                    tp[pc] = w0 * q[0] + w1 * q[db];
                }
                tr[pa] = w0 * tp[0] + w1 * tp[1];
            }
            v = xr[u] + (w0 * tr[0] + w1 * tr[1]);
        }
        sh.x[0][u][tid] = xv[0][u] = v;
        sh.x[1][u][tid] = xv[1][u] = T(0);
    }
    __syncthreads();
    // colours 1, 0, 1, 0, each on a region one cell smaller
    tile_pass<1, R, NP>(m, p, 1, xv, bw, sh.x);
    __syncthreads();
    tile_pass<0, R, NP>(m, p, 2, xv, bw, sh.x);
    __syncthreads();
    tile_pass<1, R, NP>(m, p, 3, xv, bw, sh.x);
    __syncthreads();
    tile_pass<0, R, NP>(m, p, 4, xv, bw, sh.x);
    double dot = 0.0;
    if (live && p.rows(H)) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int cc = 2 * (p.j + u * STEP);
            if (cc < H || cc >= R - H || rc + cc >= f.np) continue;
            const int o = ro + ((rc + cc) >> 1);
            xo[o + (p.red ? P : 0)] = xv[0][u];
            xo[o + (p.red ? 0 : P)] = xv[1][u];
            dot = __builtin_fma((double)bw[0][u], (double)xv[0][u], dot);
            dot = __builtin_fma((double)bw[1][u], (double)xv[1][u], dot);
        }
    }
    return dot;
}

template <typename T>
__global__ void __launch_bounds__(kTileThreads) k_vpre_tile(Geo f, const T* __restrict__ G,
                                                            long long gk, const T* __restrict__ bv,
                                                            T* __restrict__ x, Geo c,
                                                            T* __restrict__ bc)
{
    __shared__ TilePreLds<T> sh;
    d_vpre_tile<T>(self_blk(), f, G, gk, bv, x, c, bc, sh);
}

template <typename T>
__global__ void __launch_bounds__(kTileThreads) k_vpost_tile(Geo f, const T* __restrict__ G,
                                                             long long gk,
                                                             const T* __restrict__ bv,
                                                             const T* __restrict__ xi,
                                                             T* __restrict__ xo, Geo c,
                                                             const T* __restrict__ e,
                                                             double* __restrict__ partial)
{
    __shared__ TilePostLds<T> sh;
    const double dot = d_vpost_tile<T>(self_blk(), f, G, gk, bv, xi, xo, c, e, sh);
    if (partial) {
        __shared__ double s[kTileThreads / 64];
        const double w = wave_sum(dot);
        const int tid = (int)threadIdx.x;
        if ((tid & 63) == 0) s[tid >> 6] = w;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int i = 0; i < kTileThreads / 64; ++i) t += s[i];
            partial[blockIdx.x] = t;
        }
    }
}

// Batched forms: one block per (problem, tile) of the work table.
template <typename T>
__global__ void __launch_bounds__(kTileThreads) kb_vpre_tile(const BItem* __restrict__ items,
                                                             const int* __restrict__ active,
                                                             const PDesc<T>* __restrict__ pd,
                                                             int level)
{
    CPS_BATCH_BLOCK
    __shared__ TilePreLds<T> sh;
    const LDesc<T>& d = pd[it.prob].lv[level];
    const LDesc<T>& c = pd[it.prob].lv[level + 1];
    // as vcycle(): the finest level's pre-smoothed iterate goes to xt
    d_vpre_tile<T>(bk, d.g, d.G, d.gk, d.b, level == 0 ? d.xt : d.x, c.g, c.b, sh);
}

template <typename T>
__global__ void __launch_bounds__(kTileThreads) kb_vpost_tile(const BItem* __restrict__ items,
                                                              const int* __restrict__ active,
                                                              const PDesc<T>* __restrict__ pd,
                                                              int level)
{
    CPS_BATCH_BLOCK
    __shared__ TilePostLds<T> sh;
    const LDesc<T>& d = pd[it.prob].lv[level];
    const LDesc<T>& c = pd[it.prob].lv[level + 1];
    // the finest level reads xt and writes x; the others read x, write xt
    d_vpost_tile<T>(bk, d.g, d.G, d.gk, d.b, level == 0 ? d.xt : d.x, level == 0 ? d.x : d.xt,
                    c.g, level_result(c), sh);
}

// A four-colour Gauss-Seidel sweep (operators with cross terms) of a small
// level in one launch, out of place: a block owns an 8 x 8 x 8 tile, loads it
// with a halo of 4 into LDS and makes the four colour passes, each on a region
// one cell smaller; halo cells are recomputed by every tile that loads them.
// A thread takes at most one cell of a pass, and loads its metrics and right-
// hand side one pass ahead.  The arithmetic of a cell is that of the colour
// passes (stencil_sum), so the bits are too.  zero: xi is taken as zero and
// not read.  rev: colours 3 .. 0.
// Bound by the chain of its loads and passes.  Measured, FP32 with 19 points,
// against four launches a sweep: 32 x 32 x 64 17.6 -> 10.2 us, 16 x 16 x 32
// 16.8 -> 8.4; 64 x 64 x 128 21 -> 35 (its 2.9-fold reads of the metrics, in
// pieces of seven cells, then count), so the line lies between.
constexpr int kSweepThreads = 704, kSweepHalo = 4, kSweepR = kTile + 2 * kSweepHalo;
constexpr long long kSweepMaxCells = 1LL << 17;

__host__ __device__ inline bool sweep_fits(const Geo& g)
{
    return 2 * g.P <= kSweepMaxCells;
}

// a thread's cell of one pass: its place in LDS (-1: none), the domain's ends
template <typename T>
struct SweepCell {
    int at;
    bool rlo, rhi, tlo, thi;
    T b;
    FaceMetrics<T> m;
};

// cell i of pass k, the colour's cells of the region [k + 1, R - k - 1)^3
template <typename T, int MODE, bool AXI>
__device__ __forceinline__ SweepCell<T> sweep_cell(const Geo& g, const T* __restrict__ G,
                                                   long long gk, const T* __restrict__ bv, int ra,
                                                   int rb, int rc, int k, int rev)
{
    constexpr int R = kSweepR;
    const int s = k + 1, n = R - 2 * s, hn = n / 2, i = (int)threadIdx.x;
    const int colour = rev ? 3 - k : k, k1 = colour >> 1, k0 = colour & 1;
    const int aa = s + i / (hn * hn), a = ra + aa;
    // the colour's theta rows and, of them, cells (d_gs)
    const int bb = s + 2 * (i / hn % hn) + ((k0 + k1 + a + rb + s) & 1), b = rb + bb;
    const int cc = s + 2 * (i % hn) + ((k1 + a + rc + s) & 1);
    SweepCell<T> c;
    c.at = -1;
    c.rlo = a > 0;
    c.rhi = a < g.nr - 1;
    c.tlo = b > 0;
    c.thi = b < g.nt - 1;
    if (i >= n * hn * hn || a < 0 || a >= g.nr || b < 0 || b >= g.nt) return c;
    c.at = (aa * R + bb) * R + cc;
    const int cg = wrap_near(rc + cc, g.np), j = cg >> 1, P = (int)g.P;
    const int row = a * g.rowlen + b * g.nh;
    const int i0 = (cg & 1) * P + row + j;
    if (AXI) {
        const long long ci = a * g.nt + b;
        c.m = face_metrics<T, MODE>(G, gk, ci, ci + g.nt, ci + 1, ci, c.rhi, c.thi);
    } else {
        const int cp = (cg & 1) == 0 ? P + row + j : row + (j == g.nh - 1 ? 0 : j + 1);
        c.m = face_metrics<T, MODE>(G, gk, i0, i0 + g.rowlen, i0 + g.nh, cp, c.rhi, c.thi);
    }
    c.b = bv[i0];
    return c;
}

template <typename T, int MODE, bool AXI>
__global__ void __launch_bounds__(kSweepThreads)
    k_sweep_tile(Geo g, const T* __restrict__ G, long long gk, const T* __restrict__ bv,
                 const T* __restrict__ xi, T* __restrict__ xo, int rev, int zero)
{
    constexpr int R = kSweepR, H = kSweepHalo, NX = (R * R * R + kSweepThreads - 1) / kSweepThreads;
    static_assert((R - 2) * (R / 2 - 1) * (R / 2 - 1) <= kSweepThreads, "cells of the first pass");
    __shared__ T X[NX * kSweepThreads];
    int A0, B0, C0;
    tile_origin(g, (int)xcd_block(), A0, B0, C0);
    const int ra = A0 - H, rb = B0 - H, rc = C0 - H, tid = (int)threadIdx.x;
    const int P = (int)g.P;
    SweepCell<T> c = sweep_cell<T, MODE, AXI>(g, G, gk, bv, ra, rb, rc, 0, rev);
    T v[NX];
#pragma unroll
    for (int k = 0; k < NX; ++k) {
        const int i = tid + k * kSweepThreads, a = ra + i / (R * R), b = rb + i / R % R;
        const int cg = wrap_near(rc + i % R, g.np);
        v[k] = T(0);
        if (!zero && i < R * R * R && a >= 0 && a < g.nr && b >= 0 && b < g.nt)
            v[k] = xi[(cg & 1) * P + a * g.rowlen + b * g.nh + (cg >> 1)];
    }
#pragma unroll
    for (int k = 0; k < NX; ++k) X[tid + k * kSweepThreads] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        SweepCell<T> next;
        if (k < 3) next = sweep_cell<T, MODE, AXI>(g, G, gk, bv, ra, rb, rc, k + 1, rev);
        if (c.at >= 0) {
            T D;
            const T S = stencil_sum<T, MODE, true>(
                c.m, [&](int q) { return X[q]; }, c.at, c.rlo ? -R * R : 0, c.rhi ? R * R : 0,
                c.tlo ? -R : 0, c.thi ? R : 0, -1, 1, D);
            X[c.at] = (c.b - S) / D;
        }
        __syncthreads();
        if (k < 3) c = next;
    }
    if (tid >= kTile * kTile * kTile) return;
    const int cc = tid % kTile, bb = tid / kTile % kTile, aa = tid / (kTile * kTile);
    const int a = A0 + aa, b = B0 + bb, cg = C0 + cc;
    if (a < g.nr && b < g.nt && cg < g.np)
        xo[(cg & 1) * P + a * g.rowlen + b * g.nh + (cg >> 1)] =
            X[((aa + H) * R + bb + H) * R + cc + H];
}

} // namespace cps
