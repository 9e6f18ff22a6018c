// cols.hpp -- the second pass of a transform whose y-axis is split over two.
//
// A plane too large for LDS is split along y: n1 = A B, y = y1 + B y2,
// k1 = ka + A kb.  The plane pass (plane.hpp) transforms z and y2 (A rows of
// a tile (x, y1)) and multiplies by w_n1^{y1 ka}; this pass transforms y1
// (B points) and x (L points) of C columns of k2 for one ka, so three axes
// take two passes over memory.  The C2R runs them in the opposite order: here
// kb and x first, with the factor w_n1^{y1 ka} on the results.
//
// The tile is [x][y1][c] in LDS; the B-point DFTs are taken as the rows are
// loaded, the x stages run in place as those of plane.hpp do (a row of the
// x-axis is the B C elements of one x).
//
// What bounds it: a tile whose workgroup shares its CU, HBM or the Infinity
// Cache (256^3 FP32 R2C, 67 + 67 MB: 32 us; the x-pass it replaces, which moved
// as much, 38 us); a tile alone on its CU, its own phases, although the next
// tile's loads are in flight meanwhile (2-4%).  Consecutive tiles share cache
// lines where rows are not whole lines (129 columns) or a tile's rows are
// half lines; each XCD therefore takes consecutive tiles (256^3 FP32, 64-byte
// rows: C2C 133 -> 112 us a transform, R2C 87 -> 77) where their number divides
// by 8; other numbers keep the round-robin order, which has not been timed
// against a padded index.
#pragma once

#include "plane.hpp"

namespace mifft {

// Rows of B C elements that fill the banks a whole number of times put the
// narrow column runs (at most 64 bytes) that the y1 steps take from several
// rows on the same banks: four spare elements per row move each on (FP32, 128 x
// 256 x 256 C2C 61.4 -> 57.5 us; FP64, whose runs fill more banks, gained nothing:
// 256^3 Poisson 209 -> 212).
constexpr int cols_pitch(int B, int C, int esz)
{
    return B * C + (esz == 8 && B * C % 32 == 0 && C <= 8 ? 4 : 0);
}

template <typename T> struct ColsArgs {
    const cx<T>* in;
    cx<T>* out;
    GroupPtrs<T> grp;  // grouped launches, as in ContigArgs
    const cx<T>* tw;   // length L
    const cx<T>* twn;  // length n1: results times w_n1^{y1 g} (null: not)
    int ntiles, groups, cols;
    int B, C;
    int pitch;         // of the tile's rows in LDS (cols_pitch)
    int flat;          // tiles over the flattened (group, column) index, else C columns of one group
    int tpg;           // tiles per group (not flat)
    // element x, y1 of column (g, c) at g gs + x es + y1 ys + c on each side
    long long gs_in, gs_out;
    uint32_t es_in, ys_in, es_out, ys_out;
    T sgn;
    int nt_out, xcd;
    ColPlan cp;
};

template <typename T> struct ColsCtx {
    using V = cx<T>;
    V* tile;
    const V* tw;
    const unsigned short* rev;
    int tid, nt;       // threads: a multiple of B C
    int p, c;          // this thread's place in a row of B C, and its column
    int P, C, pitch;
    int b0, bs;        // first butterfly and step along x
};

// y1: the B values of (x, c) are loaded, transformed and written to the tile.
// The loads of a tile of at most kColsHeld bytes per thread are held in
// registers (`pre`), so they can be issued a tile ahead.
constexpr int kColsHeld = 128;
template <typename T> constexpr int cols_slots() { return kColsHeld / (int)sizeof(cx<T>); }

template <typename T, int R>
__device__ __forceinline__ void cols_load(const ColsCtx<T>& x, const ColsArgs<T>& a, const cx<T>* in, bool valid,
                                          cx<T>* pre)
{
    using V = cx<T>;
    constexpr int NB = cols_slots<T>() / R;
    const int L = a.cp.A, bs = x.nt / x.C;
    const int b0 = x.tid / x.C;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int b = b0 + i * bs;
        const uint32_t o = (uint32_t)b * a.es_in;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pre[i * R + r] = V{T(0), T(0)};
            if (valid && b < L) pre[i * R + r] = *at(in, o + r * a.ys_in);
        }
    }
}

template <typename T, int R>
__device__ __forceinline__ void cols_first(const ColsCtx<T>& x, const ColsArgs<T>& a, const cx<T>* pre)
{
    using V = cx<T>;
    constexpr int NB = cols_slots<T>() / R;
    const int L = a.cp.A, bs = x.nt / x.C;
    const int b0 = x.tid / x.C;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int b = b0 + i * bs;
        if (b < L) {
            V v[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[r] = pre[i * R + r];
                v[r].y *= a.sgn;
            }
            Bfly<R>::fwd(v);
            V* q = x.tile + b * x.pitch + x.c;
#pragma unroll
            for (int r = 0; r < R; ++r) q[r * x.C] = v[r];
        }
    }
}

template <typename T>
__device__ __forceinline__ void cols_load(const ColsCtx<T>& x, const ColsArgs<T>& a, const cx<T>* in, bool valid,
                                          cx<T>* pre)
{
    switch (a.B) {
    case 2: cols_load<T, 2>(x, a, in, valid, pre); break;
    case 3: cols_load<T, 3>(x, a, in, valid, pre); break;
    case 4: cols_load<T, 4>(x, a, in, valid, pre); break;
    case 5: cols_load<T, 5>(x, a, in, valid, pre); break;
    case 6: cols_load<T, 6>(x, a, in, valid, pre); break;
    default: cols_load<T, 8>(x, a, in, valid, pre); break;
    }
}

template <typename T>
__device__ __forceinline__ void cols_first(const ColsCtx<T>& x, const ColsArgs<T>& a, const cx<T>* pre)
{
    switch (a.B) {
    case 2: cols_first<T, 2>(x, a, pre); break;
    case 3: cols_first<T, 3>(x, a, pre); break;
    case 4: cols_first<T, 4>(x, a, pre); break;
    case 5: cols_first<T, 5>(x, a, pre); break;
    case 6: cols_first<T, 6>(x, a, pre); break;
    default: cols_first<T, 8>(x, a, pre); break;
    }
}

// One in-place stage along x; the last one stores to global memory.
template <typename T, int R, bool LAST>
__device__ __forceinline__ void cols_stage(const ColsCtx<T>& x, const ColsArgs<T>& a, const ColStage& s, cx<T>* out,
                                           bool valid, cx<T> w)
{
    using V = cx<T>;
    const int nb = a.cp.A / R, q = s.q, bs = x.bs;
    int b = x.b0;
    for (; b < nb; b += bs) {
        int g = b;
        if (q > 1) g = (int)__umulhi((uint32_t)b, s.mq);
        const int off = b - g * q;
        V* p = x.tile + (g * R * q + off) * x.pitch + x.p;
        V v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = p[r * q * x.pitch];
        Bfly<R>::fwd(v);
        if constexpr (LAST) {
            const int k0 = x.rev[g * R];
            if (!valid) continue;
            if (a.twn) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = cmul(v[r], w);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) v[r].y *= a.sgn;
            const uint32_t o = (uint32_t)k0 * a.es_out;
            uint32_t step = __builtin_amdgcn_readfirstlane((uint32_t)nb * a.es_out);
            asm volatile("" : "+s"(step)); // offsets by addition
            if (a.nt_out) {
#pragma unroll
                for (int r = 0; r < R; ++r) store_nt<T>(at(out, o + r * step), v[r]);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) *at(out, o + r * step) = v[r];
            }
        } else {
            const int e = off * s.tws;
            const V* w2 = x.tw;
#pragma unroll
            for (int r = 1; r < R; ++r) v[r] = cmul(v[r], *(w2 += e));
#pragma unroll
            for (int r = 0; r < R; ++r) p[r * q * x.pitch] = v[r];
        }
    }
}

// ------------------------------------------------- spectral operators
// The middle of a spectral operator on a split y-axis: the columns pass, the
// multiplier, and the columns pass of the inverse, on the tile in LDS; one
// read and one write of the spectrum for the four transforms.  The inverse
// along x is the forward's flow graph transposed (decimation in time): it
// takes the digit-reversed rows the forward leaves and ends in natural order,
// and its first butterflies take what the forward's last ones hold.
template <typename T> struct MidArgs {
    ColsArgs<T> c; // out: results, in place or another buffer; twn is set
    int n1, n2, A; // k1 = g + A kb; k2 = the column
    int op, acc;   // acc: add to what out holds
    T scale, alpha;
};

// The last forward stage, the multiplier and the first stage back.
template <typename T, int R>
__device__ __forceinline__ void mid_turn(const ColsCtx<T>& x, const MidArgs<T>& m, const SpectralCol<T>& col)
{
    using V = cx<T>;
    const int n0 = m.c.cp.A, nb = n0 / R;
    for (int g = x.b0; g < nb; g += x.bs) {
        V* p = x.tile + g * R * x.pitch + x.p;
        V v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = p[r * x.pitch];
        Bfly<R>::fwd(v);
        const int k0 = x.rev[g * R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[r] = spectral_mul<T>(m.op, k0 + r * nb, n0, col, m.scale, m.alpha, v[r]);
            v[r].y = -v[r].y; // the inverse runs as conj(F(conj(.)))
        }
        Bfly<R>::fwd(v);
#pragma unroll
        for (int r = 0; r < R; ++r) p[r * x.pitch] = v[r];
    }
}

// A stage back: twiddles, then the butterfly.
template <typename T, int R> __device__ __forceinline__ void mid_back(const ColsCtx<T>& x, const ColsArgs<T>& a, const ColStage& s)
{
    using V = cx<T>;
    const int nb = a.cp.A / R, q = s.q;
    for (int b = x.b0; b < nb; b += x.bs) {
        const int g = (int)__umulhi((uint32_t)b, s.mq); // q > 1
        const int off = b - g * q;
        V* p = x.tile + (g * R * q + off) * x.pitch + x.p;
        V v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = p[r * q * x.pitch];
        const int e = off * s.tws;
        const V* w = x.tw;
#pragma unroll
        for (int r = 1; r < R; ++r) v[r] = cmul(v[r], *(w += e));
        Bfly<R>::fwd(v);
#pragma unroll
        for (int r = 0; r < R; ++r) p[r * q * x.pitch] = v[r];
    }
}

// y1 back: the B values of (x, c), with the factors w_n1^{y1 g}, to global memory.
template <typename T, int R>
__device__ __forceinline__ void mid_store(const ColsCtx<T>& x, const MidArgs<T>& m, cx<T>* out, bool valid, int g)
{
    using V = cx<T>;
    const ColsArgs<T>& a = m.c;
    if (!valid) return;
    V w[R];
#pragma unroll
    for (int r = 1; r < R; ++r) w[r] = a.twn[r * g];
    for (int b = x.tid / x.C; b < a.cp.A; b += x.nt / x.C) {
        const V* q = x.tile + b * x.pitch + x.c;
        V v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = q[r * x.C];
        Bfly<R>::fwd(v);
        const uint32_t o = (uint32_t)b * a.es_out;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r > 0) v[r] = cmul(v[r], w[r]);
            v[r].y = -v[r].y;
            V* p = at(out, o + r * a.ys_out);
            if (m.acc) {
                const V old = *p;
                v[r].x += old.x;
                v[r].y += old.y;
            }
            *p = v[r];
        }
    }
}

// fn<R>() for the radices of a stage along x.
template <typename T, typename F> __device__ __forceinline__ void radix_switch(int R, F&& fn)
{
    switch (R) {
    case 2: fn(std::integral_constant<int, 2>{}); break;
    case 3: fn(std::integral_constant<int, 3>{}); break;
    case 4: fn(std::integral_constant<int, 4>{}); break;
    case 5: fn(std::integral_constant<int, 5>{}); break;
    case 6: fn(std::integral_constant<int, 6>{}); break;
    case 8: fn(std::integral_constant<int, 8>{}); break;
    default:
        if constexpr (sizeof(T) == 4) {
            if (R == 9)
                fn(std::integral_constant<int, 9>{});
            else if (R == 10)
                fn(std::integral_constant<int, 10>{});
            else if (R == 12)
                fn(std::integral_constant<int, 12>{});
            else if (R == 15)
                fn(std::integral_constant<int, 15>{});
            else if (R == 16)
                fn(std::integral_constant<int, 16>{});
        }
    }
}

template <typename T, bool LAST>
__device__ __forceinline__ void cols_dispatch(const ColsCtx<T>& x, const ColsArgs<T>& a, ColStage s, cx<T>* out,
                                              bool valid, cx<T> w)
{
    s.q = __builtin_amdgcn_readfirstlane(s.q);
    s.tws = __builtin_amdgcn_readfirstlane(s.tws);
    asm volatile("" : "+s"(s.q), "+s"(s.tws)); // as in col_dispatch
    radix_switch<T>(s.R, [&](auto R) { cols_stage<T, decltype(R)::value, LAST>(x, a, s, out, valid, w); });
}

// The thread's place in a tile, and the tables after the tile.
template <typename T> __device__ __forceinline__ void cols_setup(ColsCtx<T>& x, const ColsArgs<T>& a, cx<T>* tile)
{
    const int L = a.cp.A;
    x.tile = tile;
    x.tid = threadIdx.x;
    x.nt = blockDim.x;
    x.C = a.C;
    x.P = a.B * a.C;
    x.pitch = a.pitch;
    x.p = x.tid % x.P;
    x.c = x.p % a.C;
    x.b0 = x.tid / x.P;
    x.bs = x.nt / x.P;
    cx<T>* tw = tile + L * x.pitch;
    unsigned short* rev = reinterpret_cast<unsigned short*>(tw + L);
    for (int i = x.tid; i < L; i += x.nt) {
        tw[i] = a.tw[i];
        rev[i] = (unsigned short)digit_reverse(a.cp, i);
    }
    x.tw = tw;
    x.rev = rev;
}

// (group, column) of a thread in tile i; false past the last column.
// Consecutive workgroups run on different XCDs: each XCD takes a consecutive
// run of tiles, so that tiles that share cache lines share an L2.
template <typename T>
__device__ __forceinline__ bool cols_locate(const ColsArgs<T>& a, int c, int i, int& g, int& col)
{
    const int t = a.xcd ? (i & 7) * (a.ntiles >> 3) + (i >> 3) : i;
    if (a.flat) {
        const uint32_t f = (uint32_t)t * (uint32_t)a.C + (uint32_t)c;
        g = (int)(f / (uint32_t)a.cols);
        col = (int)(f - (uint32_t)g * (uint32_t)a.cols);
        return g < a.groups;
    }
    g = t / a.tpg;
    col = (t - g * a.tpg) * a.C + c;
    return col < a.cols;
}

template <typename T> __global__ __launch_bounds__(1024) void k_cols(ColsArgs<T> a)
{
    using V = cx<T>;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    ColsCtx<T> x;
    cols_setup<T>(x, a, reinterpret_cast<V*>(smem_raw));
    const int y1 = x.p / a.C;
    const V* ain = a.in;
    V* aout = a.out;
    if (gridDim.y > 1) {
        ain = a.grp.in[blockIdx.y];
        aout = a.grp.out[blockIdx.y];
    }
    int i = blockIdx.x;
    if (i >= a.ntiles) return;
    int g, col;
    bool valid = cols_locate(a, x.c, i, g, col);
    V pre[cols_slots<T>()];
    cols_load<T>(x, a, ain + (valid ? (long long)g * a.gs_in + col : 0), valid, pre);
    __syncthreads();
    for (;;) {
        asm volatile("" : "+v"(x.tid), "+v"(x.p), "+v"(x.c), "+v"(x.b0)); // as in k_strided
        cols_first<T>(x, a, pre);
        V* out = aout + (valid ? (long long)g * a.gs_out + col + (long long)y1 * a.ys_out : 0);
        V w{T(1), T(0)};
        if (a.twn && valid) w = a.twn[y1 * g];
        const int next = i + (int)gridDim.x;
        bool nvalid = false;
        if (next < a.ntiles) { // the next tile's loads, in flight during this one's stages
            nvalid = cols_locate(a, x.c, next, g, col);
            cols_load<T>(x, a, ain + (nvalid ? (long long)g * a.gs_in + col : 0), nvalid, pre);
        }
        __syncthreads();
        for (int k = 0; k + 1 < a.cp.n; ++k) {
            cols_dispatch<T, false>(x, a, a.cp.s[k], out, valid, w);
            __syncthreads();
        }
        cols_dispatch<T, true>(x, a, a.cp.s[a.cp.n - 1], out, valid, w);
        if (next >= a.ntiles) break;
        __syncthreads(); // the next tile's rows overwrite this one's
        i = next;
        valid = nvalid;
    }
}

template <typename T> __global__ __launch_bounds__(1024) void k_cols_mid(MidArgs<T> m)
{
    using V = cx<T>;
    const ColsArgs<T>& a = m.c;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    ColsCtx<T> x;
    cols_setup<T>(x, a, reinterpret_cast<V*>(smem_raw));
    const int kb = x.p / a.C;
    __syncthreads();
    const V none{T(1), T(0)};
    // (the next tile's loads held through both transforms would not fit 128
    // registers; as it is, FP32 keeps two of each thread's in scratch memory,
    // stored once and reloaded once per tile)
    for (int i = blockIdx.x; i < a.ntiles; i += gridDim.x) {
        int g, col;
        const bool valid = cols_locate(a, x.c, i, g, col);
        asm volatile("" : "+v"(x.tid), "+v"(x.p), "+v"(x.c), "+v"(x.b0)); // as in k_strided
        {
            V pre[cols_slots<T>()];
            cols_load<T>(x, a, a.in + (valid ? (long long)g * a.gs_in + col : 0), valid, pre);
            cols_first<T>(x, a, pre);
        }
        const SpectralCol<T> sc = spectral_col<T>(m.op, g + m.A * kb, col, m.n1, m.n2, m.scale);
        __syncthreads();
        for (int k = 0; k + 1 < a.cp.n; ++k) {
            cols_dispatch<T, false>(x, a, a.cp.s[k], nullptr, valid, none);
            __syncthreads();
        }
        radix_switch<T>(a.cp.s[a.cp.n - 1].R, [&](auto R) { mid_turn<T, decltype(R)::value>(x, m, sc); });
        __syncthreads();
        for (int k = a.cp.n - 2; k >= 0; --k) {
            const ColStage s = a.cp.s[k];
            radix_switch<T>(s.R, [&](auto R) { mid_back<T, decltype(R)::value>(x, a, s); });
            __syncthreads();
        }
        V* out = a.out + (valid ? (long long)g * a.gs_out + col : 0);
        switch (a.B) {
        case 2: mid_store<T, 2>(x, m, out, valid, g); break;
        case 3: mid_store<T, 3>(x, m, out, valid, g); break;
        case 4: mid_store<T, 4>(x, m, out, valid, g); break;
        case 5: mid_store<T, 5>(x, m, out, valid, g); break;
        case 6: mid_store<T, 6>(x, m, out, valid, g); break;
        default: mid_store<T, 8>(x, m, out, valid, g); break;
        }
        if (i + (int)gridDim.x < a.ntiles) __syncthreads();
    }
}

} // namespace mifft
