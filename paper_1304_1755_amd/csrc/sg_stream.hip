// The two legs of a four-colour V(nu1, nu2) cycle level, nu = 1 or 2, as one pass
// each over its vectors: down = nu1 forward sweeps from the zero start, residual
// and restriction; up = prolongation and nu2 backward sweeps.
//
// One wavefront owns a strip of 128 grid columns (lane i: columns 2i and
// 2i+1 of the strip), M modes and a segment of rows, and walks up the rows two
// per step.  The sweeps follow each other down the rows as a pipeline: a
// four-colour sweep is two row phases (k_gs_rows in sg_mg.hip), each row
// phase needs its neighbour rows one phase earlier only, so in step k phase 1
// of sweep 1 updates row 2k+1, phase 2 row 2k, phase 1 of sweep 2 row 2k-1,
// phase 2 row 2k-2, and the residual follows on rows 2k-3 and 2k-2.  Four rows
// of values and three of right-hand sides stay in registers; the columns of the
// adjacent lanes come by DPP wave shifts.  The four wavefronts of a workgroup
// share the strip's stencils through an LDS ring, with one barrier a step; a launch of
// one or two panels and more than a workgroup per CU has neither, and every
// wavefront loads its own (stream_shape).
//
// Values near the strip's and the segment's ends go stale, as their outer
// neighbours are missing: by two columns per row phase (F nodes from old S
// nodes, then S from F) and one row, so 8 columns on each side and the first
// steps of a segment are computed and thrown away.  At the domain's edge the
// missing neighbours are the zero boundary values and nothing is lost.
//
// What bounds it: the vectors cross HBM once per leg (down: f read, u and a
// quarter-size coarse f written; up: u, f and the coarse u read, u written), 5.5
// vectors where the row phases take 18.5.  A V(2,2) cycle took 745 us at 511^2,
// W = 126, float by row phases and takes 456 (1412 and 753 in double; 207 and 108
// at 255^2, W = 21, double).  Its legs at 511^2 in float take 134 and 187 us, 2.2 and 2.3 TB/s of
// those bytes (372 and 571 MB from and to HBM, 1.26 and 1.34 of them), held back by
// the latency of two wavefronts a SIMD and by 16-byte pieces of node-major f and
// u (a cache line each).
#include <type_traits>

#include "sg_internal.h"
#include "sg_wave.h"

namespace sg {

namespace {

constexpr int kStrip = 128;      // columns of a strip
constexpr int kStripHalo = 8;    // stale columns at an inner end of a strip
constexpr int kStripCore = kStrip - 2 * kStripHalo;
constexpr int kShWaves = 4;      // wavefronts that share a strip's stencils

// strips of a grid of nx columns: the first owns 120 columns, the others 112, the last up to 119
__host__ __device__ inline int strip_count(int nx) {
    if (nx < kStrip) return 1;
    return 2 + (nx - (kStrip - kStripHalo) - (kStrip - kStripHalo - 1) + kStripCore - 1) / kStripCore;
}
__host__ __device__ inline int strip_begin(int s) { return s == 0 ? 0 : kStripCore * s + kStripHalo; }

// M modes of the lane's two nodes of a row: even column, odd column
template <typename T, int M>
struct Pair {
    T e[M], o[M];
};

// the stencils of the two nodes and the reciprocals of their diagonals (c[9]), zero outside the grid
template <typename T>
struct PairStencil {
    T e[10], o[10];
};

// Addresses are a buffer (a uniform base), a uniform row offset and a byte offset of the lane, all in
// 32 bits: no address arithmetic in vector registers.  The base of a walked vector is the
// first row of the segment, so a segment's bytes have to fit (stream_fits).
typedef __amdgpu_buffer_rsrc_t Buffer;
__device__ __forceinline__ Buffer buffer_at(const void* p) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, -1, 0x00020000);
}

typedef unsigned U2 __attribute__((ext_vector_type(2)));
typedef unsigned U4 __attribute__((ext_vector_type(4)));

template <typename T, int M>
__device__ __forceinline__ void load_modes(Buffer b, unsigned lane, unsigned row, T (&v)[M]) {
    constexpr int B = M * sizeof(T);
    struct Bits { T v[M]; } x;
    if constexpr (B == 4)
        x = __builtin_bit_cast(Bits, __builtin_amdgcn_raw_buffer_load_b32(b, lane, row, 0));
    else if constexpr (B == 8)
        x = __builtin_bit_cast(Bits, (U2)__builtin_amdgcn_raw_buffer_load_b64(b, lane, row, 0));
    else
        x = __builtin_bit_cast(Bits, (U4)__builtin_amdgcn_raw_buffer_load_b128(b, lane, row, 0));
#pragma unroll
    for (int i = 0; i < M; ++i) v[i] = x.v[i];
}

// the modes from `dup` on (uniform): the first dup belong to the chunk before
template <typename T, int M>
__device__ __forceinline__ void store_modes(Buffer b, unsigned lane, unsigned row, const T (&v)[M], int dup) {
    constexpr int B = M * sizeof(T);
    if (dup == 0) {
        struct Bits { T v[M]; } x;
#pragma unroll
        for (int i = 0; i < M; ++i) x.v[i] = v[i];
        if constexpr (B == 4)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), b, lane, row, 0);
        else if constexpr (B == 8)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x), b, lane, row, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, x), b, lane, row, 0);
    } else {
#pragma unroll
        for (int i = 1; i < M; ++i)
            if (i >= dup) {
                const T w[1] = {v[i]};
                store_modes<T, 1>(b, lane + i * (unsigned)sizeof(T), row, w, 0);
            }
    }
}

// a walked vector: its rows from the segment's first one on
template <typename T>
struct Walked {
    Buffer b;
    unsigned e, o;      // byte offsets of the lane's nodes in a row
    unsigned pitch;     // bytes of a row
    int y0, ny;         // first row, rows of the grid
    int dup;            // modes not to be stored
};

// where a wavefront works: strip, rows, modes
struct StreamPos {
    int x;             // column of the lane's even node
    unsigned xe, xo;   // the lane's columns clamped into the grid
    unsigned pair;     // the lane's column pair in the stencil array
    bool ine, ino;     // the nodes lie in the grid
    bool own;          // the lane's columns belong to this strip
    int Y0, Y1;        // coarse rows of the segment
    bool last;         // the segment ends at the grid's upper edge
    int c;             // chunk of M modes
    int mode, dup;     // its first mode, modes of it that the chunk before has too
};

// SH: the wavefronts of a workgroup take adjacent chunks of one strip and segment (one past the last
// chunk repeats it and stores nothing); else every wavefront stands alone
template <int M, bool SH>
__device__ __forceinline__ bool stream_pos(int nx, int width, int nch, int ns, int seg, int nseg, StreamPos& s) {
    // contiguous ranges of workgroups per XCD: the chunks of a strip share its stencils in one L2
    const int b = blockIdx.x, nb = gridDim.x, q = nb >> 3, r = nb & 7, xcd = b & 7;
    const int lb = xcd * q + (xcd < r ? xcd : r) + (b >> 3);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int t, c;
    if constexpr (SH) {
        const int ng = (nch + kShWaves - 1) / kShWaves;
        t = __builtin_amdgcn_readfirstlane(lb / ng);
        c = (lb - t * ng) * kShWaves + wv;
    } else {
        const int w = lb * (int)(blockDim.x >> 6) + wv;
        t = __builtin_amdgcn_readfirstlane(w / nch);
        c = w - t * nch;
    }
    if (t >= ns * nseg) return false;  // SH: the whole workgroup
    const int sg = __builtin_amdgcn_readfirstlane(t / ns), strip = t - sg * ns;
    const int nxc = (nx - 1) / 2;
    const int begin = strip_begin(strip);
    const int x0 = strip == 0 ? 0 : begin - kStripHalo;
    const int end = strip == ns - 1 ? nx : strip_begin(strip + 1);
    s.x = x0 + 2 * (int)(threadIdx.x & 63);
    s.ine = s.x < nx;
    s.ino = s.x + 1 < nx;
    s.pair = min(s.x >> 1, (nx + 1) / 2);
    s.xe = min(s.x, nx - 1);
    s.xo = min(s.x + 1, nx - 1);
    s.own = s.x >= begin && s.x < end && c < nch;
    c = min(c, nch - 1);
    s.Y0 = sg * seg;
    s.Y1 = min(s.Y0 + seg, nxc);
    s.last = s.Y1 == nxc;
    s.c = c;
    s.mode = min(c * M, width - M);
    s.dup = c * M - s.mode;
    return true;
}

// Stencils in the order the walk reads them: row y of the grid (row nx: zeros) is a block of ten
// coefficients (the tenth the reciprocal diagonal) for (nx + 1) / 2 column pairs and a pair of zeros
// past the grid; a lane reads its pair's coefficients as 16-byte pieces, adjacent lanes adjacent
// pieces (the node-major layout costs one cache line per lane and load: the loads of a step then take
// more L1 cycles than its arithmetic).  The zeros make every value outside the grid zero.
//
// A step needs five rows of them (four going up).  SH: the workgroup keeps a ring of eight rows in LDS, each
// loaded once, two rows a step and a step ahead; else every wavefront loads what a phase needs.
template <typename T, bool SH>
struct Stencils {
    static constexpr int C = 8 / sizeof(T);            // coefficients of a 16-byte piece
    static constexpr int NP = 10 / C;                  // pieces of a row and pair
    static constexpr int NQ = (2 * NP + kShWaves - 1) / kShWaves;
    static constexpr int kRing = SH ? 8 * 64 * 20 : 1;  // elements of the LDS ring
    Buffer b;
    int nx, wv;
    unsigned lane;   // byte offset of the lane's pair in a piece
    T* ring;
    T q[NQ][2 * C];  // pieces on their way: this wavefront's of two rows

    __device__ __forceinline__ unsigned row_bytes(int y) const {  // uniform
        const unsigned yc = (unsigned)y < (unsigned)nx ? y : nx, np = (nx + 3) / 2;
        return yc * np * (unsigned)(20 * sizeof(T));
    }
    __device__ __forceinline__ void begin(const T* sps, int nx_, const StreamPos& s, T* ring_) {
        b = buffer_at(sps);
        nx = nx_;
        lane = s.pair * 16u;
        ring = ring_;
        wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    }
    // the pieces of rows y and y + 1
    __device__ __forceinline__ void load(int y) {
        const unsigned np = (nx + 3) / 2;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int e = wv + i * kShWaves, r = e >= NP, j = r ? e - NP : e;  // uniform
            if (2 * NP % kShWaves == 0 || e < 2 * NP) load_modes<T, 2 * C>(b, lane, row_bytes(y + r) + j * np * 16u, q[i]);
        }
    }
    // into the ring slots of rows slot, slot + 1
    __device__ __forceinline__ void store(int slot) {
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int e = wv + i * kShWaves, r = e >= NP, j = r ? e - NP : e;
            if (2 * NP % kShWaves == 0 || e < 2 * NP) {
                T* p = ring + ((slot + r) * NP + j) * 128 * C + (threadIdx.x & 63) * 2 * C;
#pragma unroll
                for (int m = 0; m < 2 * C; ++m) p[m] = q[i][m];
            }
        }
    }
    // the stencils of row y, in ring slot `slot`
    __device__ __forceinline__ void get(int y, int slot, PairStencil<T>& st) const {
        if constexpr (SH) {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const T* p = ring + (slot * NP + j) * 128 * C + (threadIdx.x & 63) * 2 * C;
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    st.e[C * j + i] = p[2 * i];
                    st.o[C * j + i] = p[2 * i + 1];
                }
            }
        } else {
            const unsigned np = (nx + 3) / 2;
            unsigned row = row_bytes(y);
            // opaque: a row's stencils serve several steps, and kept from one to the next they would not
            // fit in registers
            __asm__ volatile("" : "+s"(row));
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                T v[2 * C];
                load_modes<T, 2 * C>(b, lane, row + j * np * 16u, v);
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    st.e[C * j + i] = v[2 * i];
                    st.o[C * j + i] = v[2 * i + 1];
                }
            }
        }
    }
    // before the first step k (row 2k in slot 0): rows 2k and 2k+1 into the ring, zeros for the three below
    // them, the next two loading; `first` issues the walk's own first loads, so that all are in flight at once
    template <typename F>
    __device__ __forceinline__ void prime(int k, F first) {
        if constexpr (SH) {
            load(2 * k);
            first();
            constexpr int below = 5 * NP * 128 * C;  // slots 5, 6, 7
            for (int i = below + threadIdx.x; i < kRing; i += blockDim.x) ring[i] = T(0);
            store(0);
            load(2 * k + 2);
            meet();
        } else {
            first();
        }
    }
    // in step k: the rows of step k + 1 into the ring, those of step k + 2 loading
    template <int J>
    __device__ __forceinline__ void feed(int k) {
        if constexpr (SH) {
            store((2 * J + 2) & 7);
            load(2 * k + 4);
        }
    }
    __device__ __forceinline__ void meet() const {
        if constexpr (SH) lds_meet();
    }
};

// K u at the even / odd column: the share of the row below or above (its coefficients from st.e[R] or
// st.o[R] on), and of the left and right neighbours (the even node's left one is the odd node of the lane
// before).  Three short sums keep the chains short and the rounding as small as that of k_gs_rows.
template <int R, typename T, int M>
__device__ __forceinline__ T row_e(const PairStencil<T>& st, const Pair<T, M>& v, int m) {
    return fma_t(st.e[R], from_left(v.o[m]), fma_t(st.e[R + 2], v.o[m], st.e[R + 1] * v.e[m]));
}
template <int R, typename T, int M>
__device__ __forceinline__ T row_o(const PairStencil<T>& st, const Pair<T, M>& v, int m) {
    return fma_t(st.o[R + 2], from_right(v.e[m]), fma_t(st.o[R], v.e[m], st.o[R + 1] * v.o[m]));
}
template <typename T>
__device__ __forceinline__ T side_e(const PairStencil<T>& st, T o) {
    return fma_t(st.e[3], from_left(o), st.e[5] * o);
}
template <typename T>
__device__ __forceinline__ T side_o(const PairStencil<T>& st, T e) {
    return fma_t(st.o[5], from_right(e), st.o[3] * e);
}
// f minus the neighbours
template <typename T, int M>
__device__ __forceinline__ T rest_e(const PairStencil<T>& st, T f, const Pair<T, M>& d, T o, const Pair<T, M>& u, int m) {
    return ((f - row_e<0>(st, d, m)) - row_e<6>(st, u, m)) - side_e(st, o);
}
template <typename T, int M>
__device__ __forceinline__ T rest_o(const PairStencil<T>& st, T f, const Pair<T, M>& d, T e, const Pair<T, M>& u, int m) {
    return ((f - row_o<0>(st, d, m)) - row_o<6>(st, u, m)) - side_o(st, e);
}
// f - K u at a node of the row w.  The node's own share cancels the neighbours', so it is taken in with the
// row's, before the sum has grown: the sums stay within half of it, and their rounding with them (a float
// cycle of the P1 triangulation is 12 % further from the exact one with the own share last).
template <typename T, int M>
__device__ __forceinline__ T resid_e(const PairStencil<T>& st, T f, const Pair<T, M>& d, const Pair<T, M>& w,
                                     const Pair<T, M>& u, int m) {
    return ((f - row_e<0>(st, d, m)) - fma_t(st.e[4], w.e[m], side_e(st, w.o[m]))) - row_e<6>(st, u, m);
}
template <typename T, int M>
__device__ __forceinline__ T resid_o(const PairStencil<T>& st, T f, const Pair<T, M>& d, const Pair<T, M>& w,
                                     const Pair<T, M>& u, int m) {
    return ((f - row_o<0>(st, d, m)) - fma_t(st.o[4], w.o[m], side_o(st, w.e[m]))) - row_o<6>(st, u, m);
}

// makes the values of a row unrecognisable: the shifts of one phase would otherwise be kept for the
// next one that uses the row, and not fit in registers
template <typename T, int M>
__device__ __forceinline__ void forget(Pair<T, M>& p) {
#pragma unroll
    for (int m = 0; m < M; ++m) __asm__ volatile("" : "+v"(p.e[m]), "+v"(p.o[m]));
}

// a row phase: FWD updates the odd column first (from the old even ones), then the even column;
// backward sweeps the even column first
template <bool FWD, typename T, int M>
__device__ __forceinline__ void relax_row(const PairStencil<T>& st, const Pair<T, M>& f, const Pair<T, M>& w,
                                          const Pair<T, M>& d, const Pair<T, M>& u, Pair<T, M>& n) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
        if constexpr (FWD) {
            n.o[m] = rest_o(st, f.o[m], d, w.e[m], u, m) * st.o[9];
            n.e[m] = rest_e(st, f.e[m], d, n.o[m], u, m) * st.e[9];
        } else {
            n.e[m] = rest_e(st, f.e[m], d, w.o[m], u, m) * st.e[9];
            n.o[m] = rest_o(st, f.o[m], d, n.e[m], u, m) * st.o[9];
        }
    }
}

// rows of v (nx x nx nodes) from row y0 on, the lane's columns xe and xo: node-major with row stride
// ld, or in panels when ld is 0
template <typename T, int M>
__device__ __forceinline__ Walked<T> walked(const T* v, int ld, int nx, int y0, unsigned xe, unsigned xo,
                                            const StreamPos& s) {
    Walked<T> w;
    w.y0 = min(max(y0, 0), nx - 1);
    const size_t node = (size_t)w.y0 * nx;
    w.b = buffer_at(ld ? v + node * ld + s.mode : v + ((size_t)s.c * nx * nx + node) * M);
    const unsigned size = (ld ? (unsigned)ld : (unsigned)M) * (unsigned)sizeof(T);
    w.e = xe * size;
    w.o = xo * size;
    w.pitch = (unsigned)nx * size;
    w.ny = nx;
    w.dup = ld ? s.dup : 0;
    return w;
}

template <typename T, int M>
__device__ __forceinline__ void load_row(const Walked<T>& w, int y, Pair<T, M>& p) {
    const unsigned row = (unsigned)(min(max(y, w.y0), w.ny - 1) - w.y0) * w.pitch;
    load_modes<T, M>(w.b, w.e, row, p.e);
    load_modes<T, M>(w.b, w.o, row, p.o);
}

template <typename T, int M>
__device__ __forceinline__ void store_row(const Walked<T>& w, int y, const StreamPos& s, const Pair<T, M>& p) {
    const unsigned row = (unsigned)(y - w.y0) * w.pitch;
    if (!s.own) return;
    store_modes<T, M>(w.b, w.e, row, p.e, w.dup);
    if (s.ino) store_modes<T, M>(w.b, w.o, row, p.o, w.dup);
}

template <typename T, int M>
__device__ __forceinline__ void clear(Pair<T, M>& p) {
#pragma unroll
    for (int m = 0; m < M; ++m) p.e[m] = p.o[m] = T(0);
}

// keeps loads from being moved across: hoisted to the start of a step they would not fit in registers
__device__ __forceinline__ void fence_schedule() { __builtin_amdgcn_sched_barrier(0); }

// wavefronts per SIMD the register budget is set for: with two (256 registers) nothing spills but up to 32
// values of the double legs whose wavefronts load their own stencils; three would spill up to 170 (1.50 against
// 1.16 ms a cycle at W = 126, double)
template <typename T, int M>
constexpr int stream_waves() { return M * sizeof(T) == 4 ? 3 : 2; }

// u = NU forward sweeps from zero on K u = f; fc = P^T (f - K u) (P1T: the
// transfer of the triangulation).  The residual of the last colour (even row,
// even column) is no more than what the rounding of its relaxation left, but the
// coarse grid corrects it: without it a float cycle is 2 to 10 % further from
// the exact one.
//
// The rows in flight sit in rings indexed by the step (values two steps, right-
// hand sides four, one of them being loaded), and the walk is unrolled by four so
// that every index is a constant and no register is moved.
template <typename T, int M, int NU, bool P1T, bool SH>
__global__ void __launch_bounds__(256, (stream_waves<T, M>())) k_stream_down(const T* __restrict__ sps, const T* __restrict__ f, int ldf,
                                                     T* __restrict__ uo, T* __restrict__ fc, int nx, int width, int nch, int ns,
                                                     int seg, int nseg) {
    __shared__ __attribute__((aligned(16))) T ring[Stencils<T, SH>::kRing];
    StreamPos s;
    if (!stream_pos<M, SH>(nx, width, nch, ns, seg, nseg, s)) return;
    const int nxc = (nx - 1) / 2;
    const int X = s.x >> 1;
    const bool ownc = s.own && X < nxc;
    // values by phase (a: odd rows, b: even rows; 1, 2: sweep) and right-hand sides of the rows in flight
    Pair<T, M> a1[2], b1[2], a2[2], b2[2], fo[4], fe[4];
    T rl[M];  // share of the even row below in the restriction
    clear(a1[1]); clear(b1[1]); clear(a2[1]); clear(b2[1]);
    clear(fo[3]); clear(fo[2]); clear(fe[3]);
#pragma unroll
    for (int m = 0; m < M; ++m) rl[m] = T(0);
    const int k0 = s.Y0 - 2, k1 = s.Y1 + 1;
    Stencils<T, SH> sten;
    sten.begin(sps, nx, s, ring);
    SG_POISON_LDS(ring, (Stencils<T, SH>::kRing));
    const Walked<T> wf = walked<T, M>(f, ldf, nx, 2 * k0, s.xe, s.xo, s);
    const Walked<T> wu = walked<T, M>((const T*)uo, 0, nx, 2 * s.Y0, s.xe, s.xo, s);
    const Walked<T> wc = walked<T, M>((const T*)fc, 0, nxc, s.Y0, min(X, nxc - 1), 0, s);
    sten.prime(k0, [&] {
        load_row<T, M>(wf, 2 * k0, fe[0]);
        load_row<T, M>(wf, 2 * k0 + 1, fo[0]);
    });
    auto step = [&](auto kj, int k) {
        constexpr int J = decltype(kj)::value, c = J & 1, p = c ^ 1, j1 = (J + 3) & 3, j2 = (J + 2) & 3, jn = (J + 1) & 3;
        sten.template feed<J>(k);
        load_row<T, M>(wf, 2 * k + 2, fe[jn]);
        load_row<T, M>(wf, 2 * k + 3, fo[jn]);
        // the stencils of a phase come from LDS when it starts, or are loaded while the phase before
        // computes, and no further ahead
        PairStencil<T> s0, s1;
        sten.get(2 * k + 1, (2 * J + 1) & 7, s0);
        if constexpr (!SH) sten.get(2 * k, (2 * J + 0) & 7, s1);
        fence_schedule();
        // sweep 1, row 2k+1: every neighbour outside the row is still zero
#pragma unroll
        for (int m = 0; m < M; ++m) {
            a1[c].o[m] = fo[J].o[m] * s0.o[9];
            a1[c].e[m] = (fo[J].e[m] - side_e(s0, a1[c].o[m])) * s0.e[9];
        }
        if constexpr (!SH && NU == 2) sten.get(2 * k - 1, (2 * J + 7) & 7, s0);
        fence_schedule();
        if constexpr (SH) sten.get(2 * k, (2 * J + 0) & 7, s1);
        // sweep 1, row 2k: the row itself is still zero
#pragma unroll
        for (int m = 0; m < M; ++m) {
            b1[c].o[m] = ((fe[J].o[m] - row_o<0>(s1, a1[p], m)) - row_o<6>(s1, a1[c], m)) * s1.o[9];
            b1[c].e[m] = rest_e(s1, fe[J].e[m], a1[p], b1[c].o[m], a1[c], m) * s1.e[9];
        }
        if constexpr (!SH) sten.get(2 * k - 2, (2 * J + 6) & 7, s1);
        forget(a1[p]);
        fence_schedule();
        if constexpr (SH && NU == 2) sten.get(2 * k - 1, (2 * J + 7) & 7, s0);
        // sweep 2, rows 2k-1 and 2k-2 (NU = 1: their values of sweep 1)
        if constexpr (NU == 2) relax_row<true, T, M>(s0, fo[j1], a1[p], b1[p], b1[c], a2[c]);
        else a2[c] = a1[p];
        if constexpr (!SH) sten.get(2 * k - 3, (2 * J + 5) & 7, s0);
        forget(b1[p]);
        fence_schedule();
        if constexpr (SH) sten.get(2 * k - 2, (2 * J + 6) & 7, s1);
        if constexpr (NU == 2) relax_row<true, T, M>(s1, fe[j1], b1[p], a2[p], a2[c], b2[c]);
        else b2[c] = b1[p];
        // residual at row 2k-2 and the row's share in the coarse rows above (ru) and below it: the odd
        // column's with both corners' means, or (P1T) the north-east or the south-west corner
        T ru[M], rd[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const T o = resid_o(s1, fe[j1].o[m], a2[p], b2[c], a2[c], m), e = resid_e(s1, fe[j1].e[m], a2[p], b2[c], a2[c], m);
            rd[m] = o + (P1T ? from_right(e) : T(0.5) * (e + from_right(e)));
            ru[m] = P1T ? o + e : rd[m];
        }
        const int y = 2 * k - 2;
        if (y >= 2 * s.Y0 && (y < 2 * s.Y1 || s.last)) {
            store_row<T, M>(wu, y, s, b2[c]);
            if (y + 1 < 2 * s.Y1) store_row<T, M>(wu, y + 1, s, a2[c]);
        }
        // residual at row 2k-3 and the restriction to coarse row k-2
        if (k - 2 >= s.Y0) {
            if constexpr (SH) {
                fence_schedule();
                sten.get(2 * k - 3, (2 * J + 5) & 7, s0);
            }
            T v[M];
#pragma unroll
            for (int m = 0; m < M; ++m) {
                T re = resid_e(s0, fo[j2].e[m], b2[p], a2[p], b2[c], m);
                re = s.ine ? re : T(0);
                const T ro = resid_o(s0, fo[j2].o[m], b2[p], a2[p], b2[c], m);
                v[m] = ro + T(0.5) * ((rl[m] + rd[m]) + (re + from_right(re)));
            }
            if (ownc) store_modes<T, M>(wc.b, wc.e, (unsigned)(k - 2 - wc.y0) * wc.pitch, v, 0);
        }
#pragma unroll
        for (int m = 0; m < M; ++m) rl[m] = ru[m];
        forget(a1[c]);
        forget(b1[c]);
        forget(a2[c]);
        forget(b2[c]);
    };
    // every exit leaves the kernel: where paths meet again the rings would have to be copied
    for (int k = k0;;) {
        step(std::integral_constant<int, 0>{}, k);
        if (++k > k1) return;
        sten.meet();
        step(std::integral_constant<int, 1>{}, k);
        if (++k > k1) return;
        sten.meet();
        step(std::integral_constant<int, 2>{}, k);
        if (++k > k1) return;
        sten.meet();
        step(std::integral_constant<int, 3>{}, k);
        if (++k > k1) return;
        sten.meet();
    }
}

// uo = NU backward sweeps on K u = f from ui + P ec (P1T: the transfer of the triangulation)
template <typename T, int M, int NU, bool P1T, bool SH>
__global__ void __launch_bounds__(256, (stream_waves<T, M>())) k_stream_up(const T* __restrict__ sps, const T* __restrict__ f, int ldf,
                                                   const T* __restrict__ ui, const T* __restrict__ ec,
                                                   T* __restrict__ uo, int ldo, int nx, int width, int nch, int ns,
                                                   int seg, int nseg) {
    __shared__ __attribute__((aligned(16))) T ring[Stencils<T, SH>::kRing];
    StreamPos s;
    if (!stream_pos<M, SH>(nx, width, nch, ns, seg, nseg, s)) return;
    const int nxc = (nx - 1) / 2;
    const int X = s.x >> 1;
    const bool inc = X < nxc;
    const unsigned xc = min(X, nxc - 1);
    // corrected odd rows c, phases a (even rows) and b (odd rows) of the two sweeps, right-hand sides
    Pair<T, M> c1[2], a1[2], b1[2], a2[2], b2, fo[4], fe[4], ve, vo;
    T ep[M], en[M];  // coarse rows k-1 and k
    clear(c1[1]); clear(a1[1]); clear(b1[1]); clear(a2[1]);
    clear(fo[3]); clear(fo[2]); clear(fe[3]);
#pragma unroll
    for (int m = 0; m < M; ++m) ep[m] = T(0);
    const int k0 = s.Y0 - 2, k1 = s.Y1 + 1;
    Stencils<T, SH> sten;
    sten.begin(sps, nx, s, ring);
    SG_POISON_LDS(ring, (Stencils<T, SH>::kRing));
    const Walked<T> wf = walked<T, M>(f, ldf, nx, 2 * k0, s.xe, s.xo, s);
    const Walked<T> wi = walked<T, M>(ui, 0, nx, 2 * k0, s.xe, s.xo, s);
    const Walked<T> wu = walked<T, M>((const T*)uo, ldo, nx, 2 * s.Y0, s.xe, s.xo, s);
    const Walked<T> wc = walked<T, M>(ec, 0, nxc, k0, xc, 0, s);
    auto issue = [&](int k, Pair<T, M>& ge, Pair<T, M>& go) {
        load_row<T, M>(wf, 2 * k, ge);
        load_row<T, M>(wf, 2 * k + 1, go);
        load_row<T, M>(wi, 2 * k, ve);
        load_row<T, M>(wi, 2 * k + 1, vo);
        load_modes<T, M>(wc.b, wc.e, (unsigned)(min(max(k, wc.y0), nxc - 1) - wc.y0) * wc.pitch, en);
    };
    // doubles load the next step's rows late, where fewer registers are live
    constexpr bool kLate = sizeof(T) == 8;
    sten.prime(k0, [&] { issue(k0, fe[0], fo[0]); });
    auto step = [&](auto kj, int k) {
        constexpr int J = decltype(kj)::value, c = J & 1, p = c ^ 1, j1 = (J + 3) & 3, j2 = (J + 2) & 3, jn = (J + 1) & 3;
        sten.template feed<J>(k);
        // corrected values of rows 2k, 2k+1, zero outside the grid
        const bool r0 = k >= 0 && 2 * k < nx, r1 = k >= 0 && 2 * k + 1 < nx;  // uniform
        const bool ie = r0 && s.ine, io = r0 && s.ino, je = r1 && s.ine, jo = r1 && s.ino, ic = inc && k >= 0 && k < nxc;
        Pair<T, M> n0;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const T e = ic ? en[m] : T(0);
            const T el = from_left(e), q = T(0.5) * (ep[m] + e);
            const T ce = P1T ? T(0.5) * (from_left(ep[m]) + e) : T(0.5) * (from_left(q) + q);
            n0.e[m] = ie ? ve.e[m] + ce : T(0);
            n0.o[m] = io ? ve.o[m] + q : T(0);
            c1[c].e[m] = je ? vo.e[m] + T(0.5) * (el + e) : T(0);
            c1[c].o[m] = jo ? vo.o[m] + e : T(0);
            ep[m] = e;
        }
        if constexpr (!kLate) issue(k + 1, fe[jn], fo[jn]);
        PairStencil<T> s0, s1;
        sten.get(2 * k, (2 * J + 0) & 7, s0);
        if constexpr (!SH) sten.get(2 * k - 1, (2 * J + 7) & 7, s1);
        fence_schedule();
        relax_row<false, T, M>(s0, fe[J], n0, c1[p], c1[c], a1[c]);
        forget(c1[p]);
        if constexpr (!SH && NU == 2) sten.get(2 * k - 2, (2 * J + 6) & 7, s0);
        fence_schedule();
        if constexpr (SH) sten.get(2 * k - 1, (2 * J + 7) & 7, s1);
        relax_row<false, T, M>(s1, fo[j1], c1[p], a1[p], a1[c], b1[c]);
        forget(a1[p]);
        if constexpr (kLate) issue(k + 1, fe[jn], fo[jn]);
        if constexpr (!SH && NU == 2) sten.get(2 * k - 3, (2 * J + 5) & 7, s1);
        fence_schedule();
        // rows 2k-2 and 2k-3 (NU = 1: their values of sweep 1)
        if constexpr (NU == 2) {
            if constexpr (SH) sten.get(2 * k - 2, (2 * J + 6) & 7, s0);
            relax_row<false, T, M>(s0, fe[j1], a1[p], b1[p], b1[c], a2[c]);
            forget(b1[p]);
        } else {
            a2[c] = a1[p];
        }
        const int y = 2 * k - 2;
        if (y >= 2 * s.Y0 && (y < 2 * s.Y1 || s.last)) store_row<T, M>(wu, y, s, a2[c]);
        if (y - 1 >= 2 * s.Y0) {
            if constexpr (NU == 2) {
                if constexpr (SH) {
                    fence_schedule();
                    sten.get(2 * k - 3, (2 * J + 5) & 7, s1);
                }
                relax_row<false, T, M>(s1, fo[j2], b1[p], a2[p], a2[c], b2);
            } else {
                b2 = b1[p];
            }
            store_row<T, M>(wu, y - 1, s, b2);
        }
        forget(c1[c]);
        forget(a1[c]);
        forget(b1[c]);
        forget(a2[c]);
    };
    // every exit leaves the kernel: where paths meet again the rings would have to be copied
    for (int k = k0;;) {
        step(std::integral_constant<int, 0>{}, k);
        if (++k > k1) return;
        sten.meet();
        step(std::integral_constant<int, 1>{}, k);
        if (++k > k1) return;
        sten.meet();
        step(std::integral_constant<int, 2>{}, k);
        if (++k > k1) return;
        sten.meet();
        step(std::integral_constant<int, 3>{}, k);
        if (++k > k1) return;
        sten.meet();
    }
}

struct StreamShape {
    int ns, seg, nseg;
    bool shared;  // workgroups of four chunks share the stencils
};

// Long segments throw less away (4 of seg + 4 steps), short ones give a launch
// enough wavefronts: the longest that leaves kStreamWaves of them (at 511^2, W = 126,
// float: 485 us a cycle with 512, 468 with 1024, 444 with 2048, 538 with 4096), and one
// coarse row only where that still gives every second CU at most one workgroup (at
// 127^2, double: W = 1 51 -> 48 us, W = 10 60 -> 56, but W = 35 68 -> 76).
// Wavefronts share their stencils from three chunks on, and in launches of at most a
// workgroup per CU, where a second and third wavefront that only loads shortens
// the steps (127^2, double, W = 1: 60 -> 51 us, W = 4: 73 -> 57; 511^2, float, W = 1: 80 -> 84).
constexpr int kStreamWaves = 2048;
StreamShape stream_shape(int nx, int nch) {
    const int nxc = (nx - 1) / 2, groups = (nch + kShWaves - 1) / kShWaves;
    StreamShape h{strip_count(nx), 32, 0, false};
    while (h.seg > 2 && (long)nch * h.ns * ((nxc + h.seg - 1) / h.seg) < kStreamWaves) h.seg >>= 1;
    if (h.seg == 2 && (long)groups * h.ns * nxc <= 128) h.seg = 1;
    h.nseg = (nxc + h.seg - 1) / h.seg;
    h.shared = nch >= 3 || h.ns * h.nseg <= 256;
    return h;
}

template <typename T, int M, int NU, bool P1T>
hipError_t down_m(hipStream_t st, const T* sps, const T* f, int ldf, T* uo, T* fc, int nx, int width) {
    const int nch = (width + M - 1) / M;
    const StreamShape h = stream_shape(nx, nch);
    if (h.shared)
        hipLaunchKernelGGL((k_stream_down<T, M, NU, P1T, true>), dim3((nch + kShWaves - 1) / kShWaves * h.ns * h.nseg), dim3(256),
                           0, st, sps, f, ldf, uo, fc, nx, width, nch, h.ns, h.seg, h.nseg);
    else
        hipLaunchKernelGGL((k_stream_down<T, M, NU, P1T, false>), dim3((nch * h.ns * h.nseg + 3) / 4), dim3(256), 0, st, sps, f,
                           ldf, uo, fc, nx, width, nch, h.ns, h.seg, h.nseg);
    return hipGetLastError();
}

template <typename T, int M, int NU, bool P1T>
hipError_t up_m(hipStream_t st, const T* sps, const T* f, int ldf, const T* ui, const T* ec, T* uo, int ldo, int nx,
                int width) {
    const int nch = (width + M - 1) / M;
    const StreamShape h = stream_shape(nx, nch);
    if (h.shared)
        hipLaunchKernelGGL((k_stream_up<T, M, NU, P1T, true>), dim3((nch + kShWaves - 1) / kShWaves * h.ns * h.nseg),
                           dim3(256), 0, st, sps, f, ldf, ui, ec, uo, ldo, nx, width, nch, h.ns, h.seg, h.nseg);
    else
        hipLaunchKernelGGL((k_stream_up<T, M, NU, P1T, false>), dim3((nch * h.ns * h.nseg + 3) / 4), dim3(256), 0, st, sps,
                           f, ldf, ui, ec, uo, ldo, nx, width, nch, h.ns, h.seg, h.nseg);
    return hipGetLastError();
}

// calls go(modes, sweeps) with both as constants
template <typename T, typename F>
hipError_t with_shape(int width, int nu, F go) {
    auto modes = [&](auto n) {
        const int M = stream_modes(sizeof(T) == 4, width);
        if (M == 1) return go(std::integral_constant<int, 1>{}, n);
        if constexpr (sizeof(T) == 4)
            if (M == 4) return go(std::integral_constant<int, 4>{}, n);
        return go(std::integral_constant<int, 2>{}, n);
    };
    if (nu == 1) return modes(std::integral_constant<int, 1>{});
    if (nu == 2) return modes(std::integral_constant<int, 2>{});
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t down_t(hipStream_t st, const T* sps, const T* f, int ldf, T* uo, T* fc, int nx, int width, int nu, bool p1) {
    return with_shape<T>(width, nu, [&](auto m, auto n) {
        constexpr int M = decltype(m)::value, NU = decltype(n)::value;
        return p1 ? down_m<T, M, NU, true>(st, sps, f, ldf, uo, fc, nx, width)
                  : down_m<T, M, NU, false>(st, sps, f, ldf, uo, fc, nx, width);
    });
}
template <typename T>
hipError_t up_t(hipStream_t st, const T* sps, const T* f, int ldf, const T* ui, const T* ec, T* uo, int ldo, int nx,
                int width, int nu, bool p1) {
    return with_shape<T>(width, nu, [&](auto m, auto n) {
        constexpr int M = decltype(m)::value, NU = decltype(n)::value;
        return p1 ? up_m<T, M, NU, true>(st, sps, f, ldf, ui, ec, uo, ldo, nx, width)
                  : up_m<T, M, NU, false>(st, sps, f, ldf, ui, ec, uo, ldo, nx, width);
    });
}

}  // namespace

// 16 bytes of modes a lane and load; narrower float blocks take 8, which fills less up and leaves more
// wavefronts (a cycle at 511^2, float, with 4 and with 2 modes a lane: W = 126 444 and 502 us, W = 56 233
// and 244, W = 35 214 and 208, W = 21 175 and 148)
int stream_modes(int is_float, int width) {
    if (width < 2) return 1;
    return is_float && width >= 40 ? 4 : 2;
}

hipError_t stream_down(hipStream_t st, const float* sps, const float* f, int ldf, float* uo, float* fc, int nx, int width,
                       int nu, bool p1) {
    return down_t<float>(st, sps, f, ldf, uo, fc, nx, width, nu, p1);
}
hipError_t stream_down(hipStream_t st, const double* sps, const double* f, int ldf, double* uo, double* fc, int nx, int width,
                       int nu, bool p1) {
    return down_t<double>(st, sps, f, ldf, uo, fc, nx, width, nu, p1);
}
hipError_t stream_up(hipStream_t st, const float* sps, const float* f, int ldf, const float* ui, const float* ec, float* uo,
                     int ldo, int nx, int width, int nu, bool p1) {
    return up_t<float>(st, sps, f, ldf, ui, ec, uo, ldo, nx, width, nu, p1);
}
hipError_t stream_up(hipStream_t st, const double* sps, const double* f, int ldf, const double* ui, const double* ec,
                     double* uo, int ldo, int nx, int width, int nu, bool p1) {
    return up_t<double>(st, sps, f, ldf, ui, ec, uo, ldo, nx, width, nu, p1);
}

}  // namespace sg
