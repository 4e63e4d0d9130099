// march.hpp -- the point smoother's V-cycle on a large level in two launches.
// Included by cps.hip after kernels.hpp and tile.hpp.
//
// One V(2,2) cycle's work on a level is 4 red-black passes, the residual and
// the restriction on the way down, and the prolongation and 4 passes on the
// way up.  Pass by pass that moves 12 to 14 fields of the level through
// memory; read once and written once it is the right-hand side in, the red
// iterate and the coarse right-hand side out (1.625 words a cell) and the red
// iterate, the correction and the right-hand side in, the iterate out (2.625
// words).  Here every pass of a way is one stage of a pipeline along r:
//  - a block owns kMOwn theta rows x one segment of phi x a chunk of r-planes
//    and marches over r; at step a, stage s works on plane a - s, on values
//    that stage s - 1 left there one step before.  A stage needs its
//    neighbours of the stage before at planes p - 1, p and p + 1: along r
//    they are the thread's own registers (p + 1 of the same step), along phi
//    the adjacent lane's register, along theta the adjacent rows' values,
//    handed over through LDS (double-buffered: one barrier a plane serves all
//    stages);
//  - every stage needs one row, one cell of phi and one plane more than the
//    next, so a block also computes 4 halo rows on either side, 3 halo lanes
//    (6 cells) at either end of its segment and up to 5 halo planes.  Halo
//    cells are recomputed by each block that needs them and written only by
//    their owner; post reads one buffer and writes another, so no block reads
//    what another has overwritten.
//
// Layout of the work: a wavefront holds one pair of theta rows (2J, 2J + 1)
// x 64 phi pairs, lane j the cells 2j and 2j + 1.  In a row all cells of one
// colour of a plane have one phi parity, so a stage updates one cell per row
// and lane.  12 wavefronts make 24 rows (16 owned).  A ring of 64 pairs is
// one whole segment (the lanes wrap); others split into segments of at most
// 58 owned pairs.
//
// Pre ends on the black pass, so the black residual is zero and only the red
// one is formed and restricted; post starts with the black pass, which reads
// red values only, so pre writes the red cells of its iterate alone.
//
// The passes multiply by 1 / D from a table instead of dividing (as the tile
// path does), and the sums are explicit fma chains: the single and the
// batched forms share these bodies and agree bit for bit.

namespace cps {

constexpr int kMHalo = 4; // halo theta rows on either side
constexpr int kMSide = 3; // halo lanes at a segment's ends
// A block: owned theta rows, a wavefront per row pair, rows in LDS (one of
// zeros at either end).
constexpr int kMOwn = 16, kMWaves = (kMOwn + 2 * kMHalo) / 2, kMThreads = 64 * kMWaves,
              kMSlots = 2 * kMWaves + 2;
constexpr int kMPreStages = 5, kMPostStages = 4;

// The level rule: more than 2^20 cells (and fields below 2 GiB, see kMSkip).
// Whole cycle, two launches against one a pass on such levels: 192 x 256 x 512
// FP64 428 against 746 us, FP32 255 against 457; 96 x 128 x 256 148 / 179 and
// 111 / 145; 80 x 96 x 144 (1.1 M cells) 135 / 148 and 105 / 114.  The gain
// shrinks with the level (a block's chunk approaches its 11 halo planes), and
// up to 2^20 cells the launches of a level stay those of its passes.
constexpr long long kMarchCells = 1LL << 20;

__host__ __device__ inline bool march_fits(const Geo& g)
{
    const long long n = (long long)g.nr * g.nt * g.np;
    return n > kMarchCells && n < (1LL << 28) && g.nr % 2 == 0 && g.nt % 2 == 0 && g.nh % 2 == 0;
}

// Blocks of a level: strips of theta rows x segments of `own` phi pairs x
// chunks of ch planes.  The chunk count makes the time least: rounds of
// resident blocks x the planes a block walks (its chunk and 11 halo planes).
// One FP64 block (133 KB of LDS) has a CU to itself; two FP32 blocks share
// one, and a plane then takes both 1.5 times as long (192 x 256 x 512, pre:
// 82 us in 480 blocks against 97 us in 240; 96 x 128 x 256: 31 us in 288
// against 26 us in 240).
inline MarchGrid march_grid(const Geo& g, bool fp32)
{
    MarchGrid m;
    m.strips = cdiv(g.nt, kMOwn);
    const int most = 64 - 2 * kMSide;
    m.segs = g.nh == 64 ? 1 : cdiv(g.nh, most);
    // whole groups of 8 pairs: a segment's stores end on 64-byte boundaries
    m.own = g.nh == 64 ? 64 : std::min(cdiv(cdiv(g.nh, m.segs), 8) * 8, most);
    const int units = m.strips * m.segs, cus = 256, cap = fp32 ? 2 * cus : cus;
    long long best = -1;
    m.ch = g.nr;
    for (int n = 1; 8 * n <= g.nr || n == 1; ++n) {
        const int ch = 2 * cdiv(g.nr / 2, n);
        const long long blocks = (long long)units * n;
        const long long cost = (long long)cdiv(blocks, cap) * (ch + 11) * (blocks > cus && fp32 ? 3 : 2);
        if (best < 0 || cost < best) {
            best = cost;
            m.ch = ch;
        }
    }
    m.chunks = cdiv(g.nr, m.ch);
    m.blocks = units * m.chunks;
    return m;
}

// The level's face metrics as the stages read them, by scalar loads: for each
// plane and row pair (b0, b0 + 1) one 64-byte record (FP64; the window of six
// planes of a block's pairs has to stay in the scalar cache): low r-faces of
// both rows, low theta-faces, phi-faces, 1 / D.  High r-faces are the next
// plane's record, the high theta-face of row b0 + 1 the next pair's.  kMPad
// planes of zeros lie past either r-wall and a pair of zeros past the high
// theta-wall: a face there carries no flux, and 1 / D = 0 keeps cells beyond
// at zero.
constexpr int kMRec = 8, kMPad = 10;

inline long long march_table_words(const Geo& g)
{
    return (long long)kMRec * (g.nr + 2 * kMPad) * (g.nt / 2 + 1);
}

template <typename T>
__global__ void __launch_bounds__(kBlock) k_march_table(Geo g, const T* __restrict__ G,
                                                        long long gk, T* __restrict__ M)
{
    const int pairs = (g.nt / 2 + 1);
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= (g.nr + 2 * kMPad) * pairs) return;
    const int a = i / pairs - kMPad, b = 2 * (i % pairs);
    T v[kMRec];
    for (int q = 0; q < kMRec; ++q) v[q] = T(0);
    if (a >= 0 && a < g.nr && b < g.nt) {
        T m0[6], m1[6]; // r low, r high, theta low, theta high, phi, 1 / D
        tile_metrics<T>(g, G, gk, a, b, m0);
        tile_metrics<T>(g, G, gk, a, b + 1, m1);
        const T w[kMRec] = {m0[0], m1[0], m0[2], m1[2], m0[4], m1[4], m0[5], m1[5]};
        for (int q = 0; q < kMRec; ++q) v[q] = w[q];
    }
    for (int q = 0; q < kMRec; ++q) M[(long long)kMRec * i + q] = v[q];
}

// the value of the lane below (lane i gets lane i - 1's) / above, wrapping
// around the wavefront
template <int CTRL>
__device__ __forceinline__ float lane_rot(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double lane_rot(double v)
{
    struct I2 {
        int lo, hi;
    } w = __builtin_bit_cast(I2, v);
    w.lo = __builtin_amdgcn_mov_dpp(w.lo, CTRL, 0xf, 0xf, false);
    w.hi = __builtin_amdgcn_mov_dpp(w.hi, CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, w);
}
// the phi neighbour of a cell of phi parity Q that is not of its own pair:
// parity 0 (c = 2j) has c - 1 in lane j - 1, parity 1 has c + 1 in lane j + 1
template <int Q, typename T>
__device__ __forceinline__ T phi_beyond(T v)
{
    return Q == 0 ? lane_rot<0x13C>(v) : lane_rot<0x134>(v); // wave_ror:1 / wave_rol:1
}

template <typename T, int STAGES>
struct MarchLds {
    T v[2][STAGES][kMSlots][64]; // [buffer][stage][row slot][lane]
};

// A thread's column in one buffer, from the row below its pair: the value of
// stage s, row d - 1 of the pair, is at(s, d).  One address register a buffer;
// every access is a constant offset from it (the asm keeps the compiler from
// forming an address register for each).
template <typename T>
struct MarchCol {
    typedef __attribute__((address_space(3))) T* P;
    P p;
    __device__ __forceinline__ explicit MarchCol(T* first)
    {
        unsigned u = (unsigned)(uintptr_t)(P)first;
        asm("" : "+v"(u));
        p = (P)(uintptr_t)u;
    }
    __device__ __forceinline__ T ld(int s, int d) const { return p[(s * kMSlots + d) * 64]; }
    __device__ __forceinline__ void st(int s, int d, T v) const { p[(s * kMSlots + d) * 64] = v; }
};

// What a wavefront works on.
struct MarchPos {
    int w, lane, b0, B0; // wavefront, first row of its pair, first owned row of the block
    int a0, a1;          // owned planes
    unsigned j;          // the lane's phi pair (wrapped)
    bool rows;           // the pair lies in the domain
    bool own_lane;
};

__device__ __forceinline__ MarchPos march_at(Blk bk, const Geo& g, const MarchGrid& mg)
{
    MarchPos p;
    const int units = mg.strips * mg.segs;
    const int chunk = (int)bk.L / units, unit = (int)bk.L - chunk * units;
    const int strip = unit / mg.segs, seg = unit - strip * mg.segs;
    p.w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    p.lane = (int)threadIdx.x & 63;
    p.B0 = strip * kMOwn;
    p.b0 = p.B0 - kMHalo + 2 * p.w;
    p.rows = p.b0 >= 0 && p.b0 < g.nt;
    p.a0 = chunk * mg.ch;
    p.a1 = min(g.nr, p.a0 + mg.ch);
    const int side = g.nh == 64 ? 0 : kMSide;
    const int jj = seg * mg.own + p.lane - side;
    p.j = (unsigned)wrapi(jj, g.nh);
    p.own_lane = p.lane >= side && p.lane < side + mg.own && jj < g.nh;
    return p;
}

// metrics of a row pair at one plane (wavefront-uniform: scalar loads)
template <typename T>
struct MarchM {
    T rl[2], rh[2], t[3], p[2], i[2]; // r low / high, theta faces b0, b1, b1 + 1, phi, 1 / D
};

// The table is read through the constant address space: no kernel that reads
// it writes it, and its wavefront-uniform reads stay scalar loads.
template <typename T>
using MTab = const __attribute__((address_space(4))) T*;

template <typename T>
__device__ __forceinline__ MTab<T> tab_at(MTab<T> m, unsigned bytes)
{
    return (MTab<T>)((const __attribute__((address_space(4))) char*)m + bytes);
}

// s: byte offset of the wanted record, ms: bytes of a plane
template <typename T>
__device__ __forceinline__ MarchM<T> march_m(MTab<T> tab, unsigned s, unsigned ms)
{
    s = (unsigned)__builtin_amdgcn_readfirstlane((int)s);
    const MTab<T> p = tab_at<T>(tab, s), h = tab_at<T>(tab, s + ms);
    return MarchM<T>{{p[0], p[1]}, {h[0], h[1]}, {p[2], p[3], p[kMRec + 2]}, {p[4], p[5]},
                     {p[6], p[7]}};
}

// One Gauss-Seidel update of row k of the pair, x = (b - S) / D: dn, up the
// column's other-colour values at p - 1 and p + 1, tl, th those of the rows
// below and above, c0 the row's other-colour cell of the same phi pair and
// cb the one beyond it.  up comes last: it is the value the stage before has
// just made.
template <typename T>
__device__ __forceinline__ T march_gs(const MarchM<T>& m, int k, T b, T dn, T up, T tl, T th, T c0,
                                      T cb)
{
    T s = mul_t(m.rl[k], dn);
    s = fma_t(m.t[k + 1], th, s);
    s = fma_t(m.t[k], tl, s);
    s = fma_t(m.p[k], c0 + cb, s);
    s = fma_t(m.rh[k], up, s);
    return mul_t(b - s, m.i[k]);
}

// A field as a buffer: a lane's value at its 32-bit byte offset within a row
// and the row's (wavefront-uniform) byte offset.  A lane whose offset is
// kMSkip is out of the buffer's range: its store is dropped, so a stage's
// stores need no branch.  Every memory operation of a step is then issued by
// every wavefront alike, which lets the compiler count them: a wait for a load
// of two steps ago does not also wait for the stores and loads since (with
// branches around the stores each step waited for the one before's).
constexpr unsigned kMSkip = 0x80000000u; // fields are below 2 GiB (march_fits)

typedef unsigned MU2 __attribute__((ext_vector_type(2)));

template <typename T>
struct MarchBuf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ MarchBuf(const T* p, const Geo& g)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0,
                                              (int)(2 * g.P * (long long)sizeof(T)), 0x00020000))
    {
    }
    __device__ __forceinline__ T ld(unsigned off, unsigned plane) const
    {
        if constexpr (sizeof(T) == 8)
            return __builtin_bit_cast(
                T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)plane, 0));
        else
            return __builtin_bit_cast(
                T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, (int)plane, 0));
    }
    __device__ __forceinline__ void st(T v, unsigned off, unsigned plane) const
    {
        if constexpr (sizeof(T) == 8)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(MU2, v), r, (int)off,
                                                  (int)plane, 2);
        else
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off,
                                                  (int)plane, 2);
    }
};

// The march is unrolled by six planes, so that the values of the last three
// planes (each stage's) and of the last six (the right-hand side's) are
// registers named at compile time, with no moves between them.
template <int PH, int L>
__device__ constexpr int slot(int back)
{
    return ((PH - back) % L + L) % L;
}
template <int N>
using MI = std::integral_constant<int, N>;

// Calls step(a, MI<n mod 6>) for a = first .. last, a barrier after each; a
// wavefront without rows only keeps the barriers.
template <typename F>
__device__ __forceinline__ void march_steps(int first, int last, bool rows, F&& step)
{
    if (!rows) {
        for (int a = first; a <= last; ++a) __syncthreads();
        return;
    }
    for (int a = first; a <= last; a += 6) {
        step(a, MI<0>{});
        __syncthreads();
        if (a + 1 > last) break;
        step(a + 1, MI<1>{});
        __syncthreads();
        if (a + 2 > last) break;
        step(a + 2, MI<2>{});
        __syncthreads();
        if (a + 3 > last) break;
        step(a + 3, MI<3>{});
        __syncthreads();
        if (a + 4 > last) break;
        step(a + 4, MI<4>{});
        __syncthreads();
        if (a + 5 > last) break;
        step(a + 5, MI<5>{});
        __syncthreads();
    }
}

// The stages of a step stay in order: hoisting one stage's loads above another
// costs registers that the FP64 form does not have.
#define MSTAGE() __builtin_amdgcn_sched_barrier(0)

// Pre: 2 red-black sweeps (colours 0, 1, 0, 1) of A x = b from zero; the red
// cells of x go to xr (parity-split layout, its black cells are left alone),
// and bc = R r of the red residual.  Stages: red from zero at plane a, black
// a - 1, red a - 2, black a - 3, red residual and its phi restriction a - 4,
// theta and r restriction a - 5.
template <typename T>
__device__ __forceinline__ void d_vpre_march(Blk bk, const Geo& g, const MarchGrid& mg,
                                             const T* __restrict__ M, const T* __restrict__ bv,
                                             T* __restrict__ xr, const Geo& c, T* __restrict__ bc,
                                             MarchLds<T, kMPreStages>& sh)
{
    for (int i = (int)threadIdx.x; i < kMPreStages * 2 * kMSlots * 64; i += kMThreads)
        (&sh.v[0][0][0][0])[i] = T(0);
    const MarchPos P = march_at(bk, g, mg);
    const int w = P.w, lane = P.lane, b0 = P.rows ? P.b0 : 0;
    const unsigned ws = (unsigned)sizeof(T);
    const bool own = w >= kMHalo / 2 && w < kMWaves - kMHalo / 2;
    const bool store = own && P.own_lane;
    // the row below the pair is in slot 2 w
    const MarchCol<T> L0(&sh.v[0][0][2 * w][lane]), L1(&sh.v[1][0][2 * w][lane]);
    // rows of the halo whose first black stage needs one red row more: its
    // zero-iterate value is formed on the spot (the other wavefronts load a
    // row of their own and do not use it)
    const int be = w == 0 ? b0 - 1 : b0 + 2;
    const bool edge = P.rows && (w == 0 || w == kMWaves - 1) && be >= 0 && be < g.nt;
    const int I0 = P.a0 >> 1, I1 = P.a1 >> 1;
    const T w0 = T(0.25), w1 = T(0.75);
    const MarchBuf<T> B(bv, g), X(xr, g), C(bc, c);
    // byte offsets: the lane's within a row, its coarse cell's, both skipped
    // where another block stores; of row b0 + k, phi parity q of a plane; of
    // the edge row
    const unsigned oj = P.j * ws, os = store ? oj : kMSkip;
    const unsigned oc = store ? (unsigned)((P.j & 1 ? c.P : 0) + (P.j >> 1)) * ws : kMSkip;
    const unsigned pb = (unsigned)g.P * ws, sr = (unsigned)g.rowlen * ws, cr = (unsigned)c.rowlen * ws;
    const unsigned rw = (unsigned)g.nh * ws, r0 = (unsigned)b0 * rw;
    const unsigned re = (unsigned)(edge ? be : b0) * rw, rc = (unsigned)(b0 >> 1) * (unsigned)c.nh * ws;
    auto row = [&](int k, int q) { return r0 + (k ? rw : 0u) + (q ? pb : 0u); };
    const unsigned ms = (unsigned)kMRec * ws * (unsigned)(g.nt / 2 + 1); // table plane
    const int as = P.a0 - 5, ae = P.a1 + 5; // first step (odd), last plane + 5
    // planes past the r-walls read the wall's plane: there 1 / D is 0
    auto plane = [&](int a) { return (unsigned)clampi(a, g.nr - 1) * sr; };
    const MTab<T> tab = (MTab<T>)(uintptr_t)M;
    unsigned m = ((unsigned)(as - 4 + kMPad) * (unsigned)(g.nt / 2 + 1) + (unsigned)(b0 >> 1)) *
                 ((unsigned)kMRec * ws); // its record at plane a - 4
    // right-hand side: red and black values of the last six planes; the red
    // ones two planes ahead wait in nR
    T bR[2][6], bB[2][6], nR[2][2], eb[2] = {T(0), T(0)};
    T B2[2][3], R3[2][3], B4[2][3];
    T cA = T(0), cB = T(0); // coarse planes being summed: the current one, the next
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int n = 0; n < 6; ++n) bR[k][n] = bB[k][n] = T(0);
#pragma unroll
        for (int n = 0; n < 3; ++n) B2[k][n] = R3[k][n] = B4[k][n] = T(0);
        // planes as and as + 1; as is odd: row k's red parity is (1 + k) & 1
        bR[k][0] = B.ld(oj, plane(as) + row(k, (1 + k) & 1));
        bB[k][0] = B.ld(oj, plane(as) + row(k, k));
        nR[k][0] = T(0);
        nR[k][1] = B.ld(oj, plane(as + 1) + row(k, k));
        bB[k][1] = B.ld(oj, plane(as + 1) + row(k, (1 + k) & 1));
    }
    __syncthreads();
    // step number PH mod 6: Q is the parity of plane a
    march_steps(as, ae, P.rows, [&](int a, auto PH_) {
        constexpr int PH = decltype(PH_)::value, Q = (PH + 1) & 1, wr = PH & 1, rd = wr ^ 1;
        constexpr int n0 = slot<PH, 3>(0), n1 = slot<PH, 3>(1), n2 = slot<PH, 3>(2);
        const MarchCol<T>&Lw = wr ? L1 : L0, &Lr = wr ? L0 : L1; // this step's buffer, the last's
        // values of the rows next to the pair, left by the last step
        T lo[kMPreStages], hi[kMPreStages];
        auto rows = [&](int s) { // read one stage ahead of their use
            lo[s] = Lr.ld(s, 0);
            hi[s] = Lr.ld(s, 3);
        };
        rows(0);
        // red of the edge row at plane a - 1, from zero; then its plane a + 1
        const T ev = eb[rd];
        eb[rd] = B.ld(oj, plane(a + 1) + re + ((a + 1 + be) & 1 ? pb : 0u));
        if (edge) {
            const T v = ev * tab_at<T>(tab, m + 3 * ms)[w == 0 ? 7 - kMRec : 6 + kMRec];
            if (w == 0) lo[0] = v;
            else hi[0] = v;
        }
        MSTAGE();
        T R1[2][3]; // red from zero at planes a, a - 1, a - 2
        { // red from zero, plane a
            const MarchM<T> mm = march_m<T>(tab, m + 4 * ms, ms);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                R1[k][0] = mul_t(bR[k][slot<PH, 6>(0)], mm.i[k]);
                Lw.st(0, 1 + k, R1[k][0]);
            }
        }
        MSTAGE();
        rows(1);
        { // black, plane a - 1: row k's black cells have phi parity (Q + k) & 1
            const MarchM<T> mm = march_m<T>(tab, m + 3 * ms, ms);
            const MarchM<T> m2 = march_m<T>(tab, m + 2 * ms, ms);
            constexpr int b = slot<PH, 6>(1);
            // the pair's own red values of planes a - 1 and a - 2 are formed
            // again from b (the same product), not kept
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                R1[k][1] = mul_t(bR[k][slot<PH, 6>(1)], mm.i[k]);
                R1[k][2] = mul_t(bR[k][slot<PH, 6>(2)], m2.i[k]);
            }
            B2[0][n0] = march_gs<T>(mm, 0, bB[0][b], R1[0][2], R1[0][0], lo[0], R1[1][1],
                                    R1[0][1], phi_beyond<Q>(R1[0][1]));
            B2[1][n0] = march_gs<T>(mm, 1, bB[1][b], R1[1][2], R1[1][0], R1[0][1], hi[0],
                                    R1[1][1], phi_beyond<1 - Q>(R1[1][1]));
            Lw.st(1, 1, B2[0][n0]);
            Lw.st(1, 2, B2[1][n0]);
        }
        // the loads of plane a + 2: row k's red parity is (Q + k) & 1
        const unsigned p2 = plane(a + 2);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            nR[k][wr] = B.ld(oj, p2 + row(k, (Q + k) & 1));
            bB[k][slot<PH, 6>(-2)] = B.ld(oj, p2 + row(k, (Q + k + 1) & 1));
        }
        MSTAGE();
        rows(2);
        { // red, plane a - 2: phi parity (Q + k) & 1
            const MarchM<T> mm = march_m<T>(tab, m + 2 * ms, ms);
            constexpr int b = slot<PH, 6>(2);
            R3[0][n0] = march_gs<T>(mm, 0, bR[0][b], B2[0][n2], B2[0][n0], lo[1], B2[1][n1],
                                    B2[0][n1], phi_beyond<Q>(B2[0][n1]));
            R3[1][n0] = march_gs<T>(mm, 1, bR[1][b], B2[1][n2], B2[1][n0], B2[0][n1], hi[1],
                                    B2[1][n1], phi_beyond<1 - Q>(B2[1][n1]));
            Lw.st(2, 1, R3[0][n0]);
            Lw.st(2, 2, R3[1][n0]);
            const unsigned o = a - 2 >= P.a0 && a - 2 < P.a1 ? os : kMSkip;
            X.st(R3[0][n0], o, plane(a - 2) + row(0, Q));
            X.st(R3[1][n0], o, plane(a - 2) + row(1, 1 - Q));
        }
        MSTAGE();
        rows(3);
        { // black, plane a - 3
            const MarchM<T> mm = march_m<T>(tab, m + ms, ms);
            constexpr int b = slot<PH, 6>(3);
            B4[0][n0] = march_gs<T>(mm, 0, bB[0][b], R3[0][n2], R3[0][n0], lo[2], R3[1][n1],
                                    R3[0][n1], phi_beyond<Q>(R3[0][n1]));
            B4[1][n0] = march_gs<T>(mm, 1, bB[1][b], R3[1][n2], R3[1][n0], R3[0][n1], hi[2],
                                    R3[1][n1], phi_beyond<1 - Q>(R3[1][n1]));
            Lw.st(3, 1, B4[0][n0]);
            Lw.st(3, 2, B4[1][n0]);
        }
        MSTAGE();
        rows(4);
        const T own0 = Lr.ld(4, 1), own1 = Lr.ld(4, 2);
        // red residual, plane a - 4, and its phi restriction: the coarse cell
        // K = j takes c = 2j - 1 .. 2j + 2, of which the red ones are c and
        // c + 2 (parity 0) or c - 1 and c + 1
        {
            const MarchM<T> mm = march_m<T>(tab, m, ms);
            constexpr int b = slot<PH, 6>(4);
            auto res = [&](int k, T x, T dn, T up, T tl, T th, T c0, T cb) {
                T s = mul_t(-mm.rl[k], x - dn);
                s = fma_t(mm.t[k + 1], th - x, s);
                s = fma_t(-mm.t[k], x - tl, s);
                s = fma_t(mm.p[k], c0 - x, s);
                s = fma_t(-mm.p[k], x - cb, s);
                s = fma_t(mm.rh[k], up - x, s);
                return bR[k][b] - s;
            };
            const T r0 = res(0, R3[0][n2], B4[0][n2], B4[0][n0], lo[3], B4[1][n1], B4[0][n1],
                             phi_beyond<Q>(B4[0][n1]));
            const T r1 = res(1, R3[1][n2], B4[1][n2], B4[1][n0], B4[0][n1], hi[3], B4[1][n1],
                             phi_beyond<1 - Q>(B4[1][n1]));
            // the other red cell of the coarse cell lies beyond the pair on
            // the side away from phi_beyond's
            Lw.st(4, 1, fma_t(w1, r0, mul_t(w0, phi_beyond<1 - Q>(r0))));
            Lw.st(4, 2, fma_t(w1, r1, mul_t(w0, phi_beyond<Q>(r1))));
        }
        MSTAGE();
        { // theta restriction of the last step's plane a - 5 (rows clamped at
          // the walls), then r: coarse plane I takes 2I - 1 .. 2I + 2 (the
          // planes past a wall are the wall's)
            T s = mul_t(w0, b0 > 0 ? lo[4] : own0);
            s = fma_t(w1, own0, s);
            s = fma_t(w1, own1, s);
            s = fma_t(w0, b0 + 2 < g.nt ? hi[4] : own1, s);
            const int pl = a - 5;
            if constexpr (Q == 1) { // pl = 2I + 2: I is complete, I + 1 has its first two
                const int I = (pl - 2) >> 1;
                const T v = pl < g.nr ? fma_t(w0, s, cA) : cA;
                C.st(v, I >= I0 && I < I1 ? oc : kMSkip,
                     (unsigned)clampi(I, c.nr - 1) * cr + rc);
                if (pl == 0) cB = mul_t(w0, s); // the plane past the low wall
                cA = fma_t(w1, s, cB);
            } else { // pl = 2I + 1
                cA = fma_t(w1, s, cA);
                if (pl == g.nr - 1) cA = fma_t(w0, s, cA); // and the one past the high wall
                cB = mul_t(w0, s);
            }
        }
        // plane a + 1's red values (loaded a step ago) take their slot
#pragma unroll
        for (int k = 0; k < 2; ++k) bR[k][slot<PH, 6>(-1)] = nR[k][rd];
        m += ms;
    });
}

// Post: xo = 2 red-black sweeps (colours 1, 0, 1, 0) of A x = b from the red
// cells of xi + P e (xi's black cells are not read).  Stages: corrected red
// at plane a, black a - 1, red a - 2, black a - 3, red a - 4.  Returns the
// thread's part of b . x over the block's cells.
template <typename T>
__device__ __forceinline__ double d_vpost_march(Blk bk, const Geo& g, const MarchGrid& mg,
                                                const T* __restrict__ M, const T* __restrict__ bv,
                                                const T* __restrict__ xi, T* __restrict__ xo,
                                                const Geo& c, const T* __restrict__ e,
                                                MarchLds<T, kMPostStages>& sh)
{
    for (int i = (int)threadIdx.x; i < kMPostStages * 2 * kMSlots * 64; i += kMThreads)
        (&sh.v[0][0][0][0])[i] = T(0);
    const MarchPos P = march_at(bk, g, mg);
    const int w = P.w, lane = P.lane, b0 = P.rows ? P.b0 : 0;
    const unsigned ws = (unsigned)sizeof(T);
    const bool own = w >= kMHalo / 2 && w < kMWaves - kMHalo / 2;
    const bool store = own && P.own_lane;
    // the row below the pair is in slot 2 w
    const MarchCol<T> L0(&sh.v[0][0][2 * w][lane]), L1(&sh.v[1][0][2 * w][lane]);
    const T w0 = T(0.75), w1 = T(0.25);
    double acc = 0.0;
    const MarchBuf<T> B(bv, g), Xi(xi, g), Xo(xo, g), E(e, c);
    // byte offsets as in pre; of coarse rows J - 1, J, J + 1 (clamped)
    const unsigned oj = P.j * ws, os = store ? oj : kMSkip;
    const unsigned oc = (unsigned)((P.j & 1 ? c.P : 0) + (P.j >> 1)) * ws;
    const unsigned pb = (unsigned)g.P * ws, sr = (unsigned)g.rowlen * ws, cr = (unsigned)c.rowlen * ws;
    const unsigned rw = (unsigned)g.nh * ws, r0 = (unsigned)b0 * rw;
    auto row = [&](int k, int q) { return r0 + (k ? rw : 0u) + (q ? pb : 0u); };
    auto crow = [&](int q) {
        return (unsigned)clampi((b0 >> 1) - 1 + q, c.nt - 1) * ((unsigned)c.nh * ws);
    };
    const unsigned rc[3] = {crow(0), crow(1), crow(2)};
    const unsigned ms = (unsigned)kMRec * ws * (unsigned)(g.nt / 2 + 1);
    const int as = P.a0 - 4, ae = P.a1 + 3; // steps; as is even
    auto plane = [&](int a) { return (unsigned)clampi(a, g.nr - 1) * sr; };
    // the iterate's, q the parity of a: past an r-wall the nearest plane of that
    // parity, whose red cells lie where a's do.  The wall's own plane would
    // give its black cells, which nothing has written: they meet only zero
    // metrics, but memory may hold NaN there.
    auto xplane = [&](int a, int q) { return (unsigned)min(max(a, q), g.nr - 2 + q) * sr; };
    const MTab<T> tab = (MTab<T>)(uintptr_t)M;
    unsigned m = ((unsigned)(as - 4 + kMPad) * (unsigned)(g.nt / 2 + 1) + (unsigned)(b0 >> 1)) *
                 ((unsigned)kMRec * ws); // its record at plane a - 4
    // b's black values of planes a + 1 .. a - 4, its red ones of a .. a - 5
    T bB[2][6], bR[2][6], xn[2][3]; // and the red iterate of planes a .. a + 2
    T R0[2][3], B1[2][3], R2[2][3], B3[2][3];
    // coarse values theta-interpolated onto the pair's rows, by coarse plane
    // mod 3; the next plane's raw values
    T tc[2][3], en[3];
    auto lde = [&](int I) {
#pragma unroll
        for (int q = 0; q < 3; ++q) en[q] = E.ld(oc, (unsigned)clampi(I, c.nr - 1) * cr + rc[q]);
    };
    auto theta = [&](int n) {
        tc[0][n] = fma_t(w0, en[1], mul_t(w1, en[0]));
        tc[1][n] = fma_t(w0, en[1], mul_t(w1, en[2]));
    };
    // b before plane as + 1 (black) and as (red) is taken only by stages whose
    // results no owned cell depends on
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int n = 0; n < 6; ++n) bB[k][n] = bR[k][n] = T(0);
#pragma unroll
        for (int n = 0; n < 3; ++n) R0[k][n] = B1[k][n] = R2[k][n] = B3[k][n] = T(0);
        xn[k][0] = Xi.ld(oj, xplane(as, 0) + row(k, k)); // as is even: row k's red parity is k
        xn[k][1] = Xi.ld(oj, xplane(as + 1, 1) + row(k, 1 - k));
        xn[k][2] = T(0);
    }
    lde((as >> 1) - 1); // coarse planes I - 1, I, I + 1 of plane as = 2 I: slots 2, 0, 1
    theta(2);
    lde(as >> 1);
    theta(0);
    lde((as >> 1) + 1);
    theta(1);
    __syncthreads();
    march_steps(as, ae, P.rows, [&](int a, auto PH_) {
        constexpr int PH = decltype(PH_)::value, Q = PH & 1, wr = PH & 1;
        constexpr int n0 = slot<PH, 3>(0), n1 = slot<PH, 3>(1), n2 = slot<PH, 3>(2);
        // slots of coarse planes I = floor(a / 2) and the one interpolated with
        constexpr int c0 = (PH / 2) % 3, c1 = Q == 0 ? (c0 + 2) % 3 : (c0 + 1) % 3;
        const MarchCol<T>&Lw = wr ? L1 : L0, &Lr = wr ? L0 : L1;
        T lo[kMPostStages], hi[kMPostStages];
        auto rows = [&](int s) { // read one stage ahead of their use
            lo[s] = Lr.ld(s, 0);
            hi[s] = Lr.ld(s, 3);
        };
        rows(0);
        MSTAGE();
        { // corrected red, plane a: r interpolation (2I from I - 1, 2I + 1
          // from I + 1), then phi (c = 2K from K - 1, 2K + 1 from K + 1)
            const T y0 = fma_t(w0, tc[0][c0], mul_t(w1, tc[0][c1]));
            const T y1 = fma_t(w0, tc[1][c0], mul_t(w1, tc[1][c1]));
            R0[0][n0] = xn[0][n0] + fma_t(w0, y0, mul_t(w1, phi_beyond<Q>(y0)));
            R0[1][n0] = xn[1][n0] + fma_t(w0, y1, mul_t(w1, phi_beyond<1 - Q>(y1)));
            Lw.st(0, 1, R0[0][n0]);
            Lw.st(0, 2, R0[1][n0]);
        }
        const unsigned p2 = xplane(a + 2, Q);
#pragma unroll
        for (int k = 0; k < 2; ++k) // row k's red parity at even distance: (Q + k) & 1
            xn[k][slot<PH, 3>(-2)] = Xi.ld(oj, p2 + row(k, (Q + k) & 1));
        // the next coarse plane: loaded on the even plane, interpolated (over
        // the one no longer needed) on the odd one
        if constexpr (Q == 0) lde((a >> 1) + 2);
        else theta((c0 + 2) % 3);
        MSTAGE();
        rows(1);
        { // black, plane a - 1
            const MarchM<T> mm = march_m<T>(tab, m + 3 * ms, ms);
            constexpr int b = slot<PH, 6>(1);
            B1[0][n0] = march_gs<T>(mm, 0, bB[0][b], R0[0][n2], R0[0][n0], lo[0], R0[1][n1],
                                    R0[0][n1], phi_beyond<Q>(R0[0][n1]));
            B1[1][n0] = march_gs<T>(mm, 1, bB[1][b], R0[1][n2], R0[1][n0], R0[0][n1], hi[0],
                                    R0[1][n1], phi_beyond<1 - Q>(R0[1][n1]));
            Lw.st(1, 1, B1[0][n0]);
            Lw.st(1, 2, B1[1][n0]);
        }
        const unsigned p1 = plane(a + 1), p0 = plane(a);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            bB[k][slot<PH, 6>(-1)] = B.ld(oj, p1 + row(k, (Q + k) & 1));
            bR[k][slot<PH, 6>(0)] = B.ld(oj, p0 + row(k, (Q + k) & 1));
        }
        MSTAGE();
        rows(2);
        { // red, plane a - 2
            const MarchM<T> mm = march_m<T>(tab, m + 2 * ms, ms);
            constexpr int b = slot<PH, 6>(2);
            R2[0][n0] = march_gs<T>(mm, 0, bR[0][b], B1[0][n2], B1[0][n0], lo[1], B1[1][n1],
                                    B1[0][n1], phi_beyond<Q>(B1[0][n1]));
            R2[1][n0] = march_gs<T>(mm, 1, bR[1][b], B1[1][n2], B1[1][n0], B1[0][n1], hi[1],
                                    B1[1][n1], phi_beyond<1 - Q>(B1[1][n1]));
            Lw.st(2, 1, R2[0][n0]);
            Lw.st(2, 2, R2[1][n0]);
        }
        constexpr int bb = slot<PH, 6>(3), br = slot<PH, 6>(4);
        const bool inb = a - 3 >= P.a0 && a - 3 < P.a1, inr = a - 4 >= P.a0 && a - 4 < P.a1;
        MSTAGE();
        rows(3);
        { // black, plane a - 3
            const MarchM<T> mm = march_m<T>(tab, m + ms, ms);
            B3[0][n0] = march_gs<T>(mm, 0, bB[0][bb], R2[0][n2], R2[0][n0], lo[2], R2[1][n1],
                                    R2[0][n1], phi_beyond<Q>(R2[0][n1]));
            B3[1][n0] = march_gs<T>(mm, 1, bB[1][bb], R2[1][n2], R2[1][n0], R2[0][n1], hi[2],
                                    R2[1][n1], phi_beyond<1 - Q>(R2[1][n1]));
            Lw.st(3, 1, B3[0][n0]);
            Lw.st(3, 2, B3[1][n0]);
            const unsigned o = inb ? os : kMSkip;
            Xo.st(B3[0][n0], o, plane(a - 3) + row(0, Q));
            Xo.st(B3[1][n0], o, plane(a - 3) + row(1, 1 - Q));
        }
        MSTAGE();
        { // red, plane a - 4
            const MarchM<T> mm = march_m<T>(tab, m, ms);
            const T x0 = march_gs<T>(mm, 0, bR[0][br], B3[0][n2], B3[0][n0], lo[3], B3[1][n1],
                                     B3[0][n1], phi_beyond<Q>(B3[0][n1]));
            const T x1 = march_gs<T>(mm, 1, bR[1][br], B3[1][n2], B3[1][n0], B3[0][n1], hi[3],
                                     B3[1][n1], phi_beyond<1 - Q>(B3[1][n1]));
            const unsigned o = inr ? os : kMSkip;
            Xo.st(x0, o, plane(a - 4) + row(0, Q));
            Xo.st(x1, o, plane(a - 4) + row(1, 1 - Q));
            if (inb) {
                acc = __builtin_fma((double)bB[0][bb], (double)B3[0][n0], acc);
                acc = __builtin_fma((double)bB[1][bb], (double)B3[1][n0], acc);
            }
            if (inr) {
                acc = __builtin_fma((double)bR[0][br], (double)x0, acc);
                acc = __builtin_fma((double)bR[1][br], (double)x1, acc);
            }
        }
        m += ms;
    });
    return store ? acc : 0.0;
}

template <typename T>
__global__ void __launch_bounds__(kMThreads) k_vpre_march(Geo g, MarchGrid mg,
                                                          const T* __restrict__ M,
                                                          const T* __restrict__ bv,
                                                          T* __restrict__ xr, Geo c,
                                                          T* __restrict__ bc)
{
    __shared__ MarchLds<T, kMPreStages> sh;
    d_vpre_march<T>(self_blk(), g, mg, M, bv, xr, c, bc, sh);
}

// dot: per-block partial sums of b . x (may be null)
template <typename T>
__global__ void __launch_bounds__(kMThreads) k_vpost_march(Geo g, MarchGrid mg,
                                                           const T* __restrict__ M,
                                                           const T* __restrict__ bv,
                                                           const T* __restrict__ xi,
                                                           T* __restrict__ xo, Geo c,
                                                           const T* __restrict__ e,
                                                           double* __restrict__ dot)
{
    __shared__ MarchLds<T, kMPostStages> sh;
    const Blk bk = self_blk();
    const double acc = d_vpost_march<T>(bk, g, mg, M, bv, xi, xo, c, e, sh);
    if (dot) {
        double* part = reinterpret_cast<double*>(&sh.v[0][0][0][0]); // past the last barrier
        const double s = wave_sum(acc);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int i = 0; i < kMWaves; ++i) t += part[i];
            dot[bk.L] = t;
        }
    }
}

// Batched forms: one block per (problem, block of its own launch).
template <typename T>
__global__ void __launch_bounds__(kMThreads) kb_vpre_march(const BItem* __restrict__ items,
                                                           const int* __restrict__ active,
                                                           const PDesc<T>* __restrict__ pd,
                                                           int level)
{
    CPS_BATCH_BLOCK
    __shared__ MarchLds<T, kMPreStages> sh;
    const LDesc<T>& d = pd[it.prob].lv[level];
    const LDesc<T>& c = pd[it.prob].lv[level + 1];
    d_vpre_march<T>(bk, d.g, d.mg, d.mt, d.b,
                    level == 0 ? d.r : d.x, c.g, c.b, sh);
}

template <typename T>
__global__ void __launch_bounds__(kMThreads) kb_vpost_march(const BItem* __restrict__ items,
                                                            const int* __restrict__ active,
                                                            const PDesc<T>* __restrict__ pd,
                                                            int level)
{
    CPS_BATCH_BLOCK
    __shared__ MarchLds<T, kMPostStages> sh;
    const LDesc<T>& d = pd[it.prob].lv[level];
    const LDesc<T>& c = pd[it.prob].lv[level + 1];
    d_vpost_march<T>(bk, d.g, d.mg, d.mt, d.b,
                     level == 0 ? d.r : d.x, level == 0 ? d.x : d.r, c.g,
                     level_result(c), sh);
}

#undef MSTAGE

} // namespace cps
