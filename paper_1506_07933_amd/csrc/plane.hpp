// plane.hpp -- two axes in one pass: the z- and y-FFTs of a plane in LDS.
//
// The passes of kernels.hpp read and write the array once per axis.  A plane
// of A rows (along y) of L elements (along z) that fits a CU's 160 KiB of LDS
// is transformed along both axes between one read and one write:
//
// k_plane      C2C: z-lines, then columns
// k_plane_r2c  real rows of 2L: z-lines (half-length FFT + post-processing),
//              then columns over the L + 1 outputs
// k_plane_c2r  the inverse: columns, then z-lines (pre-processing + inverse)
//
// z-lines are compiled per length, a line within one wavefront, each row in
// its own place in the tile; the loads of the next rows (of the next tile,
// after the last ones) are in flight meanwhile.  Columns
// run in place as a decimation-in-frequency transform whose radices are data:
// a stage over spans of m = R q rows reads rows g m + off + r q of a column,
// applies the radix-R DFT, multiplies output k by w_m^{off k} and writes back
// to the same places, so one barrier per stage is enough and a thread takes
// any number of butterflies.  Row g of the result holds frequency rev(g) (the
// digits of g in reverse), which costs nothing: a row may be stored to, or
// loaded from, any place.
//
// What bounds it: large batches of planes, HBM and the vector units together
// (512 x 256 planes of 128 x 64 complex64, two 72 KiB workgroups per CU: 3.3 ms
// against 2.7 + 2.9 ms for the two passes it replaces, 5.1 TB/s; about 50
// instructions per element); few planes, one workgroup's latency (7 us for
// 32 x 32, 11 us for 128 x 128), against two launches of 4.5 us and more.
// Radices up to 16 in FP32 keep both axes at two stages for most lengths up
// to 256: with the passes' radices of at most 8 a 128 x 128 plane took 90
// instructions per element and 9.7 of its 11 us were theirs.
#pragma once

#include "kernels.hpp"

namespace mifft {

constexpr int kMaxColStages = 8;
constexpr int kMaxPlaneLine = 512; // longest compiled z-line (complex points)

// One in-place column stage: butterfly b of a column takes rows
// (b / q) R q + b % q + r q, r = 0 .. R - 1.
struct ColStage {
    int R, q;
    int tws;       // twiddle step n / (R q): output k of offset off takes w_n^{off k tws}
    uint32_t mq;   // ceil(2^32 / q) (q > 1)
};

// Row transform of A rows: its stages and the twiddle table of length A.
struct ColPlan {
    int A, n;
    ColStage s[kMaxColStages];
};

template <typename T> struct PlaneArgs {
    const void* in;
    void* out;
    GroupPtrs<T> grp;     // ng > 1 transforms of one shape: their tiles one after another
    int ng;
    const cx<T>* twz;     // z-lines, length L
    const cx<T>* tw2;     // real: exp(-2 pi i k / n2)
    const cx<T>* twy;     // columns, length A
    int ntiles;
    // Tile t is (x, b) = (t / nb, t % nb), its row r at x s_x + b s_b + r s_r on
    // each side (complex elements; pairs of reals on a real side).  nb > 1: the
    // y-axis is split (cols.hpp); forward results take w_n1^{b k} from twn.
    int nb;
    const cx<T>* twn;
    long long is_x, is_b, is_r, os_x, os_b, os_r;
    T sgn;                // C2C: +1 forward, -1 inverse
    int nt_out;           // streaming stores
    ColPlan cp;
};

// Row rev(p) of the in-place column transform's position p.
__device__ __forceinline__ int digit_reverse(const ColPlan& cp, int p)
{
    int k = 0, mul = 1;
    for (int i = 0; i < cp.n; ++i) {
        const int d = cp.s[i].q > 1 ? (int)__umulhi((uint32_t)p, cp.s[i].mq) : p;
        p -= d * cp.s[i].q;
        k += d * mul;
        mul *= cp.s[i].R;
    }
    return k;
}

// ------------------------------------------------- composite butterflies

// Coprime factors (Good-Thomas): element n = R2 n1 + R1 n2 (mod R) enters
// DFTs of R2 and R1 points with no twiddles, and result (k1, k2) is
// frequency k with k = k1 (mod R1), k = k2 (mod R2).
constexpr int crt(int k1, int R1, int k2, int R2)
{
    int k = k1;
    while (k % R2 != k2) k += R1;
    return k;
}
template <int R1, int R2> struct BflyCoprime {
    template <typename V> __device__ __forceinline__ static void fwd(V* v)
    {
        constexpr int R = R1 * R2;
        V a[R1][R2];
#pragma unroll
        for (int i = 0; i < R1; ++i) {
#pragma unroll
            for (int j = 0; j < R2; ++j) a[i][j] = v[(R2 * i + R1 * j) % R];
            Bfly<R2>::fwd(a[i]);
        }
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) {
            V b[R1];
#pragma unroll
            for (int i = 0; i < R1; ++i) b[i] = a[i][k2];
            Bfly<R1>::fwd(b);
#pragma unroll
            for (int k1 = 0; k1 < R1; ++k1) v[crt(k1, R1, k2, R2)] = b[k1];
        }
    }
};
template <> struct Bfly<6> : BflyCoprime<2, 3> {};
template <> struct Bfly<10> : BflyCoprime<2, 5> {};
template <> struct Bfly<12> : BflyCoprime<3, 4> {};
template <> struct Bfly<15> : BflyCoprime<3, 5> {};

// x (c - i s)
template <typename V, typename S> __device__ __forceinline__ V rot(V x, S c, S s)
{
    return V{x.x * c + x.y * s, x.y * c - x.x * s};
}

// R1 = R2: n = n1 + R2 n2, DFTs over n2, twiddles w_R^{n1 k1}, DFTs over n1.
template <> struct Bfly<9> {
    template <typename V> __device__ __forceinline__ static void fwd(V* v)
    {
        using S = decltype(v[0].x);
        const S c1 = S(0.76604444311897803520239265055541667394), s1 = S(0.64278760968653932632264340990726343290);
        const S c2 = S(0.17364817766693034885171662676931479600), s2 = S(0.98480775301220805936674302458952301367);
        const S c4 = S(-0.93969262078590838405410927732473146994), s4 = S(0.34202014332566873304409961468225958076);
        V a[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int j = 0; j < 3; ++j) a[i][j] = v[i + 3 * j];
            Bfly<3>::fwd(a[i]);
        }
        a[1][1] = rot(a[1][1], c1, s1);
        a[1][2] = rot(a[1][2], c2, s2);
        a[2][1] = rot(a[2][1], c2, s2);
        a[2][2] = rot(a[2][2], c4, s4);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            V b[3] = {a[0][k], a[1][k], a[2][k]};
            Bfly<3>::fwd(b);
#pragma unroll
            for (int j = 0; j < 3; ++j) v[k + 3 * j] = b[j];
        }
    }
};

template <> struct Bfly<16> {
    template <typename V> __device__ __forceinline__ static void fwd(V* v)
    {
        using S = decltype(v[0].x);
        const S c1 = S(0.923879532511286756128183189396788287); // cos(pi/8)
        const S s1 = S(0.382683432365089771728459984030398867); // sin(pi/8)
        const S h = S(0.707106781186547524400844362104849039);
        V a[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a[i][j] = v[i + 4 * j];
            Bfly<4>::fwd(a[i]);
        }
        a[1][1] = rot(a[1][1], c1, s1);
        a[1][2] = V{(a[1][2].x + a[1][2].y) * h, (a[1][2].y - a[1][2].x) * h};
        a[1][3] = rot(a[1][3], s1, c1);
        a[2][1] = V{(a[2][1].x + a[2][1].y) * h, (a[2][1].y - a[2][1].x) * h};
        a[2][2] = cmul_negi(a[2][2]);
        a[2][3] = V{(a[2][3].y - a[2][3].x) * h, -(a[2][3].x + a[2][3].y) * h};
        a[3][1] = rot(a[3][1], s1, c1);
        a[3][2] = V{(a[3][2].y - a[3][2].x) * h, -(a[3][2].x + a[3][2].y) * h};
        a[3][3] = rot(a[3][3], -c1, -s1);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            V b[4] = {a[0][k], a[1][k], a[2][k], a[3][k]};
            Bfly<4>::fwd(b);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[k + 4 * j] = b[j];
        }
    }
};

// ------------------------------------------------------- radix choice

// Radices of the z-lines and columns.  FP64 stops at 8: a butterfly's values,
// its twiddles and the prefetched inputs have to fit 128 registers (plane_line
// leaves out the lengths that do not all the same).
constexpr bool is_radix(int R, bool fp64)
{
    return R == 2 || R == 3 || R == 4 || R == 5 || R == 6 || R == 8 ||
           (!fp64 && (R == 9 || R == 10 || R == 12 || R == 15 || R == 16));
}

struct PlaneRadices {
    int n;
    int r[kMaxColStages];
};

// Factors of L from the largest radix down: the fewest stages (each moves the
// tile through LDS once more), then the smallest largest radix (the most
// threads per line: the 64-point lines of 512 x 256 x 16 x 64 as 8 x 8 rather
// than 16 x 4: 1.20 against 1.25 ms a transform).
constexpr void plane_search(int L, bool fp64, int top, int rest, PlaneRadices cur, PlaneRadices& best)
{
    if (rest == 1) {
        if (cur.n > 0 && (best.n == 0 || cur.n < best.n || (cur.n == best.n && cur.r[0] < best.r[0]))) best = cur;
        return;
    }
    if (cur.n >= kMaxColStages || (best.n > 0 && cur.n >= best.n)) return;
    for (int R = top; R >= 2; --R) {
        if (rest % R != 0 || !is_radix(R, fp64)) continue;
        PlaneRadices next = cur;
        next.r[next.n++] = R;
        plane_search(L, fp64, R, rest / R, next, best);
    }
}

constexpr PlaneRadices plane_radices(int L, bool fp64)
{
    PlaneRadices cur{0, {}}, best{0, {}};
    plane_search(L, fp64, 16, L, cur, best);
    return best;
}

// z-lines that a plane kernel is compiled for.  FP64 lines of five stages, and of
// four beyond 360 points, hold more than 128 registers beside the prefetched
// rows (2 to 54 spilled) or pass the tile through LDS too often: 200 x 20 x 900 R2C 48
// us as three passes, 60 as two; 300 x 9 x 480 C2C 40 against 47; 2 x 135 x 486 and the
// like up to 1.5 times.  Four stages up to 360 points gain (360: 0.83 of the time).
constexpr bool plane_line(int L, bool fp64)
{
    if (L < 2 || L > kMaxPlaneLine) return false;
    const int n = plane_radices(L, fp64).n;
    return !fp64 || n < 4 || (n == 4 && L <= 360);
}

// Threads per z-line: one first-stage butterfly each, or as many as keep the
// line within a wavefront.
constexpr int zline_threads(int L, const PlaneRadices& f)
{
    const int nbf = L / f.r[0];
    const int per = (nbf + 63) / 64;
    return (nbf + per - 1) / per;
}

// Between its stages a line keeps one spare place every 2^shift elements.  One
// exchange (two stages): every 16, which still spreads the first stage's
// writes, R apart, over the banks; more: every 8 (the second exchange's runs
// of 8: 1024 x 64 x 512 with 512 = 8 8 8 took 307 us, 344 with one every 16).
constexpr int line_shift(const PlaneRadices& f) { return f.n <= 2 ? 4 : 3; }

template <typename T, int L> struct ZShape {
    static constexpr PlaneRadices f = plane_radices(L, sizeof(T) == 8);
    static constexpr int TPL = zline_threads(L, f);
    static constexpr int LPW = 64 / TPL; // lines per wavefront
    static constexpr int SH = line_shift(f);
    static constexpr int R0 = f.r[0];
    static constexpr int SLOTS = ((L / R0 + TPL - 1) / TPL) * R0;
};

// Where a column stage reads and writes: the tile, or global rows.
enum { COL_LDS = 0, COL_LOAD = 1, COL_STORE = 2 };

template <typename T> struct ColCtx {
    using V = cx<T>;
    V* tile;
    const V* tw;                 // w_A^j, staged in LDS
    const unsigned short* rev;   // digit reversal of the A rows, in LDS
    const V* in;                 // COL_LOAD: row r at in + r * rs
    V* out;                      // COL_STORE: row r at out + r * rs
    uint32_t rs;
    T sgn;
    bool nt;
    const V* twb;                // COL_STORE: row k times twb[k] (b > 0), in LDS
    int b;
    int threads;                 // of the workgroup
};

// C columns of rows of PITCH elements.  Global offsets within a tile fit 32
// bits (the planner's check), so they cost one instruction each.
template <typename V> __device__ __forceinline__ V* at(V* base, uint32_t elem)
{
    return reinterpret_cast<V*>(reinterpret_cast<char*>(base) + elem * (uint32_t)sizeof(V));
}
template <typename V> __device__ __forceinline__ const V* at(const V* base, uint32_t elem)
{
    return reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + elem * (uint32_t)sizeof(V));
}
template <typename T, int R, int C, int PITCH, int MODE>
__device__ __forceinline__ void col_stage(const ColCtx<T>& x, const ColStage& s, int A)
{
    using V = cx<T>;
    const int nb = A / R;
    const int q = s.q;
    const int total = nb * C;
    int u = threadIdx.x;
    asm volatile("" : "+v"(u)); // as in k_strided: nothing of this is kept across the tile loop
    for (; u < total; u += x.threads) {
        const int b = u / C, c = u - b * C;
        int g = b;
        if (q > 1) g = (int)__umulhi((uint32_t)b, s.mq);
        const int off = b - g * q;
        V* p = x.tile + (g * R * q + off) * PITCH + c;
        V v[R];
        if constexpr (MODE == COL_LOAD) {
            const uint32_t o = (uint32_t)off * x.rs + (uint32_t)c; // the first stage: g = 0
            uint32_t step = __builtin_amdgcn_readfirstlane((uint32_t)q * x.rs);
            asm volatile("" : "+s"(step));
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[r] = *at(x.in, o + r * step);
                v[r].y *= x.sgn;
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = p[r * q * PITCH];
        }
        Bfly<R>::fwd(v);
        if constexpr (MODE == COL_STORE) { // the last stage: q = 1
            const int k0 = x.rev[g * R];
            if (x.b > 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = cmul(v[r], x.twb[k0 + r * nb]);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) v[r].y *= x.sgn;
            const uint32_t o = (uint32_t)k0 * x.rs + (uint32_t)c;
            uint32_t step = __builtin_amdgcn_readfirstlane((uint32_t)nb * x.rs);
            asm volatile("" : "+s"(step)); // offsets by addition
            if (x.nt) {
#pragma unroll
                for (int r = 0; r < R; ++r) store_nt<T>(at(x.out, o + r * step), v[r]);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) *at(x.out, o + r * step) = v[r];
            }
        } else {
            if (q > 1) {
                const int e = off * s.tws;
                const V* w = x.tw;
#pragma unroll
                for (int r = 1; r < R; ++r) v[r] = cmul(v[r], *(w += e));
            } else { // the last stage, left in the tile
#pragma unroll
                for (int r = 0; r < R; ++r) v[r].y *= x.sgn;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) p[r * q * PITCH] = v[r];
        }
    }
}

template <typename T, int C, int PITCH, int MODE>
__device__ __forceinline__ void col_dispatch(const ColCtx<T>& x, ColStage s, int A)
{
    // nothing of a stage is worked out ahead of the tile loop (for all radices at once)
    s.q = __builtin_amdgcn_readfirstlane(s.q);
    s.tws = __builtin_amdgcn_readfirstlane(s.tws);
    A = __builtin_amdgcn_readfirstlane(A);
    asm volatile("" : "+s"(s.q), "+s"(s.tws), "+s"(A));
    switch (s.R) {
    case 2: col_stage<T, 2, C, PITCH, MODE>(x, s, A); break;
    case 3: col_stage<T, 3, C, PITCH, MODE>(x, s, A); break;
    case 4: col_stage<T, 4, C, PITCH, MODE>(x, s, A); break;
    case 5: col_stage<T, 5, C, PITCH, MODE>(x, s, A); break;
    case 6: col_stage<T, 6, C, PITCH, MODE>(x, s, A); break;
    case 8: col_stage<T, 8, C, PITCH, MODE>(x, s, A); break;
    default:
        if constexpr (sizeof(T) == 4) {
            if (s.R == 9)
                col_stage<T, 9, C, PITCH, MODE>(x, s, A);
            else if (s.R == 10)
                col_stage<T, 10, C, PITCH, MODE>(x, s, A);
            else if (s.R == 12)
                col_stage<T, 12, C, PITCH, MODE>(x, s, A);
            else if (s.R == 15)
                col_stage<T, 15, C, PITCH, MODE>(x, s, A);
            else if (s.R == 16)
                col_stage<T, 16, C, PITCH, MODE>(x, s, A);
        }
    }
}

// ---------------------------------------------------------------- z-lines

// The Stockham stages of fft_engine.hpp for a line whose threads are in one
// wavefront, in one row of the tile.  Between the stages the line sits at
// padded places (line_pad, see line_shift); its first stage may read and its last stage writes unpadded
// ones, as the columns do.  Where the padding of a thread's
// elements differs by compile-time constants, so do its LDS addresses.
template <int SH> __device__ __forceinline__ int line_pad(int idx) { return idx + (idx >> SH); }
template <int SH, int STEP> __device__ __forceinline__ int pad_read(int j, int r) // line_pad(j + r STEP)
{
    constexpr int G = 1 << SH;
    if constexpr (STEP % G == 0)
        return line_pad<SH>(j) + r * (STEP / G * (G + 1));
    else
        return line_pad<SH>(j + r * STEP);
}
template <int SH, int Ns, int R> __device__ __forceinline__ int pad_write(int a, int k, int r) // line_pad(a Ns R + k + r Ns), k < Ns
{
    constexpr int G = 1 << SH;
    if constexpr ((Ns * R) % G == 0 && G % Ns == 0)
        return a * (Ns * R / G * (G + 1)) + k + r * Ns + ((r * Ns) >> SH);
    else if constexpr (Ns % G == 0)
        return line_pad<SH>(a * (Ns * R) + k) + r * (Ns / G * (G + 1));
    else
        return line_pad<SH>(a * (Ns * R) + k + r * Ns);
}

template <typename T, int L, int I, int Ns, typename Ctx> struct ZStage {
    __device__ __forceinline__ static void run(Ctx& c)
    {
        using V = cx<T>;
        using Z = ZShape<T, L>;
        constexpr int R = Z::f.r[I], TPL = Z::TPL;
        constexpr int NBF = L / R, NB = (NBF + TPL - 1) / TPL;
        constexpr bool EXACT = NBF % TPL == 0, FIRST = I == 0, LAST = I + 1 == Z::f.n;
        // A last stage that stores to global memory takes adjacent butterflies
        // per thread, so that it stores 16 bytes at a time.
        constexpr bool PAIR = LAST && !FIRST && Ctx::kPairOut && EXACT && NB == 2 && NBF % 2 == 0 && sizeof(T) == 4;
        auto bfly_of = [&](int i) { return PAIR ? 2 * c.t + i : c.t + i * TPL; };
        V v[NB][R];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int j = bfly_of(i);
            if (EXACT || j < NBF) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if constexpr (FIRST)
                        v[i][r] = c.first_get(i * R + r, j + r * NBF);
                    else
                        v[i][r] = c.row[pad_read<Z::SH, NBF>(j, r)];
                }
            }
        }
        if constexpr (FIRST) c.first_done();
        if constexpr (!FIRST || Ctx::kFirstFromRow) wave_sync();
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int j = bfly_of(i);
            if (EXACT || j < NBF) {
                const int a = j / Ns, k = j - a * Ns;
                if constexpr (Ns > 1) {
                    constexpr int step = L / (Ns * R);
#pragma unroll
                    for (int r = 1; r < R; ++r) v[i][r] = cmul(v[i][r], c.twd[k * r * step]);
                }
                Bfly<R>::fwd(v[i]);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if constexpr (PAIR) {
                        if (i == 1) c.final_pair(j - 1 + r * NBF, v[0][r], v[1][r]);
                    } else if constexpr (LAST)
                        c.final_put(j + r * NBF, v[i][r]);
                    else
                        c.row[pad_write<Z::SH, Ns, R>(a, k, r)] = v[i][r];
                }
            }
        }
        if constexpr (!LAST) {
            wave_sync();
            ZStage<T, L, I + 1, Ns * R, Ctx>::run(c);
        }
    }
};

// Forward lines: inputs prefetched in registers (the next rows' are loaded
// as soon as the first stage has taken the current ones), results in the row.
template <typename T, int L> struct ZForward {
    using V = cx<T>;
    using Z = ZShape<T, L>;
    static constexpr bool kFirstFromRow = false, kPairOut = false;
    V* row;
    const V* twd; // twiddle table staged in LDS
    int t;
    T sgn;
    V pre[Z::SLOTS];
    const V* nin; // next row's input
    bool has_next;
    __device__ __forceinline__ void load(const V* p)
    {
        FirstStageShape<L, Z::TPL, Z::R0>::each(t, [&](int slot, int idx) { pre[slot] = load_in<T>(p + idx); });
    }
    __device__ __forceinline__ V first_get(int slot, int) const
    {
        V v = pre[slot];
        v.y *= sgn;
        return v;
    }
    __device__ __forceinline__ void first_done()
    {
        if (has_next) load(nin);
    }
    __device__ __forceinline__ void final_put(int idx, V v) { row[idx] = v; }
};

// C2R lines: the row holds L + 1 outputs of the columns' inverse; the first
// stage reads them pre-processed, the last stage writes pairs of reals.
template <typename T, int L> struct ZInverseReal {
    using V = cx<T>;
    static constexpr bool kFirstFromRow = true, kPairOut = true;
    V* row;
    const V* twd;
    const V* tw2; // exp(-2 pi i k / 2L)
    int t;
    V* out;
    bool nt;
    __device__ __forceinline__ V first_get(int, int k) const
    {
        V z;
        if (k == 0) {
            const T a = row[0].x, b = row[L].x;
            z = V{a + b, a - b};
        } else {
            const V a = row[k], b = cconj(row[L - k]);
            const V s = cadd(a, b), d = cmul(csub(a, b), cconj(tw2[k]));
            z = V{s.x - d.y, s.y + d.x};
        }
        return cconj(z);
    }
    __device__ __forceinline__ void first_done() const {}
    // elements idx (even) and idx + 1: rows start at multiples of L (even) pairs
    __device__ __forceinline__ void final_pair(int idx, V a, V b)
    {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 v{(float)a.x, (float)-a.y, (float)b.x, (float)-b.y};
        if (nt)
            __builtin_nontemporal_store(v, reinterpret_cast<f4*>(out + idx));
        else
            *reinterpret_cast<f4*>(out + idx) = v;
    }
    __device__ __forceinline__ void final_put(int idx, V v)
    {
        if (nt)
            store_nt<T>(out + idx, cconj(v));
        else
            out[idx] = cconj(v);
    }
};

// LDS after the tile: both twiddle tables, then the digit reversal.
template <typename T>
__device__ __forceinline__ void plane_tables(const PlaneArgs<T>& a, int L, cx<T>* dst, ColCtx<T>& x,
                                             const cx<T>*& twz)
{
    const int A = a.cp.A;
    cx<T>* ty = dst + L;
    unsigned short* rev = reinterpret_cast<unsigned short*>(ty + A);
    for (int i = threadIdx.x; i < L; i += blockDim.x) dst[i] = a.twz[i];
    for (int i = threadIdx.x; i < A; i += blockDim.x) {
        ty[i] = a.twy[i];
        rev[i] = (unsigned short)digit_reverse(a.cp, i);
    }
    twz = dst;
    x.tw = ty;
    x.rev = rev;
}

// Row pitch of the tile: a line's padded places, or its L + 1 outputs; not a
// multiple of 16 elements, which would put the rows of a wavefront's lines on
// the same banks (15-point lines, a row per lane: 486 x 200 x 30 R2C 38 us).
constexpr int plane_pitch(int L, const PlaneRadices& f)
{
    const int p = L + (L >> line_shift(f)) + 1;
    return p % 16 == 0 ? p + 1 : p;
}

// Rows of a wavefront: LPW lines at a time; lanes past the last line repeat
// the first line's threads (same values to the same places), and so do rows
// past the end of the tile, which only share wavefronts with row A - 1.
template <typename T, int L> struct ZRows {
    using Z = ZShape<T, L>;
    int sub, t, first, step;
    __device__ __forceinline__ ZRows(int waves)
    {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        sub = lane / Z::TPL;
        t = lane - sub * Z::TPL;
        if (sub >= Z::LPW) sub = 0;
        first = w * Z::LPW;
        step = waves * Z::LPW;
    }
    // row of this thread in the round that starts at r0
    __device__ __forceinline__ int row(int r0, int A) const { return r0 + sub < A ? r0 + sub : A - 1; }
};

// Forward planes: REAL: rows of 2L reals, C = L + 1 outputs; else C = L.
// src(m), dst(m): the buffers of transform m (0 unless several run at once).
template <typename T, int L, bool REAL, typename Src, typename Dst>
__device__ __forceinline__ void plane_forward(const PlaneArgs<T>& a, Src&& src, Dst&& dst)
{
    using V = cx<T>;
    constexpr int C = REAL ? L + 1 : L, PITCH = plane_pitch(L, ZShape<T, L>::f);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    V* tile = reinterpret_cast<V*>(smem_raw);
    const int A = a.cp.A;
    const int total = a.ntiles * a.ng;
    int x = blockIdx.x;
    if (x >= total) return; // uniform
    const ZRows<T, L> zr((int)blockDim.x >> 6);
    ZForward<T, L> c;
    c.t = zr.t;
    c.sgn = REAL ? T(1) : a.sgn;
    auto in_of = [&](int i) {
        const int m = REAL || a.ng == 1 ? 0 : i / a.ntiles, t = i - m * a.ntiles;
        return src(m) + (long long)(t / a.nb) * a.is_x + (long long)(t % a.nb) * a.is_b;
    };
    const V* in = in_of(x);
    if (zr.first < A) c.load(in + (long long)zr.row(zr.first, A) * a.is_r);
    ColCtx<T> cc;
    V* twb = tile + A * PITCH + L + A + (A + 3) / 4; // after the digit reversal
    cc.twb = twb;
    cc.tile = tile;
    cc.rs = (uint32_t)a.os_r;
    cc.sgn = REAL ? T(1) : a.sgn;
    cc.nt = a.nt_out != 0;
    cc.in = nullptr;
    cc.threads = blockDim.x;
    plane_tables<T>(a, L, tile + A * PITCH, cc, c.twd);
    __syncthreads();
    for (;;) {
        const int xn = x + (int)gridDim.x;
        const V* next_in = xn < total ? in_of(xn) : in;
        const int m = REAL || a.ng == 1 ? 0 : x / a.ntiles, t = x - m * a.ntiles;
        cc.b = t % a.nb;
        if (cc.b > 0)
            for (int i = threadIdx.x; i < A; i += blockDim.x) twb[i] = a.twn[cc.b * i];
        for (int r0 = zr.first; r0 < A; r0 += zr.step) {
            const bool last = r0 + zr.step >= A;
            c.has_next = !last || xn < total;
            c.nin = (last ? next_in : in) + (long long)zr.row(last ? zr.first : r0 + zr.step, A) * a.is_r;
            c.row = tile + zr.row(r0, A) * PITCH;
            // as in k_strided: no address of this is kept across the loops
            asm volatile("" : "+v"(c.t));
            ZStage<T, L, 0, 1, decltype(c)>::run(c);
            if constexpr (REAL) {
                // X[k] = (s - i p)/2, X[L - k] = conj(s + i p)/2 with
                // s = Z[k] + conj Z[L-k], p = w^k (Z[k] - conj Z[L-k]): a pair is one
                // thread's, so the line is post-processed in place
                wave_sync();
                const T half = T(0.5);
                for (int k = c.t; 2 * k <= L; k += ZShape<T, L>::TPL) {
                    const V za = c.row[k];
                    const V zb = cconj(k == 0 ? za : c.row[L - k]);
                    const V s = cadd(za, zb);
                    const V p = cmul(a.tw2[k], csub(za, zb));
                    c.row[k] = V{half * (s.x + p.y), half * (s.y - p.x)};
                    if (2 * k != L) c.row[L - k] = V{half * (s.x - p.y), half * (-s.y - p.x)};
                }
            }
        }
        __syncthreads();
        cc.out = dst(m) + (long long)(t / a.nb) * a.os_x + (long long)cc.b * a.os_b;
        for (int i = 0; i + 1 < a.cp.n; ++i) {
            col_dispatch<T, C, PITCH, COL_LDS>(cc, a.cp.s[i], A);
            __syncthreads();
        }
        col_dispatch<T, C, PITCH, COL_STORE>(cc, a.cp.s[a.cp.n - 1], A);
        if (xn >= total) break;
        __syncthreads(); // the next tile's rows overwrite this one's
        x = xn;
        in = next_in;
    }
}

template <typename T, int L>
__global__ __launch_bounds__(1024) void k_plane(PlaneArgs<T> a)
{
    // (indexing the argument itself in plane_forward would copy it to scratch memory)
    const auto* args = (const __attribute__((address_space(4))) PlaneArgs<T>*)__builtin_amdgcn_kernarg_segment_ptr();
    plane_forward<T, L, false>(
        a, [&](int m) { return a.ng == 1 ? reinterpret_cast<const cx<T>*>(a.in) : args->grp.in[m]; },
        [&](int m) { return a.ng == 1 ? reinterpret_cast<cx<T>*>(a.out) : args->grp.out[m]; });
}

template <typename T, int L>
__global__ __launch_bounds__(1024) void k_plane_r2c(PlaneArgs<T> a)
{
    plane_forward<T, L, true>(
        a, [&](int) { return reinterpret_cast<const cx<T>*>(a.in); },
        [&](int) { return reinterpret_cast<cx<T>*>(a.out); });
}

template <typename T, int L>
__global__ __launch_bounds__(1024) void k_plane_c2r(PlaneArgs<T> a)
{
    using V = cx<T>;
    constexpr int C = L + 1, PITCH = plane_pitch(L, ZShape<T, L>::f);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    V* tile = reinterpret_cast<V*>(smem_raw);
    const int A = a.cp.A;
    const V* ain = reinterpret_cast<const V*>(a.in);
    V* aout = reinterpret_cast<V*>(a.out);
    const ZRows<T, L> zr((int)blockDim.x >> 6);
    ZInverseReal<T, L> c;
    c.tw2 = a.tw2;
    c.nt = a.nt_out != 0;
    c.t = zr.t;
    ColCtx<T> cc;
    cc.tile = tile;
    cc.rs = (uint32_t)a.is_r;
    cc.sgn = T(-1); // the inverse along the columns: conj(F(conj(.)))
    cc.nt = false;
    cc.out = nullptr;
    cc.twb = nullptr;
    cc.threads = blockDim.x;
    cc.b = 0;
    plane_tables<T>(a, L, tile + A * PITCH, cc, c.twd);
    __syncthreads();
    for (int x = blockIdx.x; x < a.ntiles; x += gridDim.x) {
        cc.in = ain + (long long)(x / a.nb) * a.is_x + (long long)(x % a.nb) * a.is_b;
        V* out = aout + (long long)(x / a.nb) * a.os_x + (long long)(x % a.nb) * a.os_b;
        col_dispatch<T, C, PITCH, COL_LOAD>(cc, a.cp.s[0], A);
        __syncthreads();
        for (int i = 1; i < a.cp.n; ++i) {
            col_dispatch<T, C, PITCH, COL_LDS>(cc, a.cp.s[i], A);
            __syncthreads();
        }
        for (int r0 = zr.first; r0 < A; r0 += zr.step) {
            const int row = zr.row(r0, A);
            c.row = tile + row * PITCH;
            asm volatile("" : "+v"(c.t));
            c.out = out + (long long)cc.rev[row] * a.os_r;
            ZStage<T, L, 0, 1, decltype(c)>::run(c);
        }
        if (x + (int)gridDim.x < a.ntiles) __syncthreads();
    }
}

} // namespace mifft
