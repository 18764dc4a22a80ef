// Gather/push and the counting sort of markers by dual cell.
//
// One step's sort is three passes over the markers:
//   count   : (optionally) push each marker, find its new bucket, and count it;
//   scan    : exclusive prefix sum of the bucket counts -> run offsets (the
//             totals of its tiles first, where there are more than a few: added
//             up in the count they were atomics of every wave on a few cache
//             lines, 99 us a count of 16.8M markers instead of 31);
//   scatter : push again (bit-identical arithmetic), claim a slot in the run,
//             and write the marker to its sorted position in the other buffer.
// Pushing twice instead of storing pushed positions between the passes saves
// a full write+read of the position/velocity streams; the push is a few
// flops per marker against 16-40 bytes of traffic.
//
// Counting uses integer atomics only.  Consecutive markers of the previous
// order land in few buckets after the push, so a wave (1D-1V) or a block
// (1D-3V, FP64 kicks of velocity cells, and the scatter of large dense FP64 sorts)
// counts its markers in an LDS window of the buckets it expects and issues one global atomic per touched bucket.  The
// windows follow the markers: by the drift and kick of the tile, by the kick
// column by column, or over the planes a gyration reaches.  Markers that miss
// the window use one global atomic each, those of the overflow bucket one a
// tile: with kicks of up to 8 velocity cells (13.5M FP64 markers, 512 x 6600) a
// window of the old rows alone sent nearly every marker to memory, and the count
// took 4.6 ms and the scatter 1.2 ms instead of 59 and 208 us; with a fifth of
// the markers gyrating outside the grid (1.8M markers) the overflow bucket's
// atomics took the scatter from 56 us to 2.4 ms.  The scatter uses the counts
// array itself as a descending cursor, which leaves it zeroed for the next step.
//
// Implied cells (FP32 1D-1V).  In that form a marker's cell index equals its
// bucket whenever its cloud touches the grid, and once sorted, a marker's
// bucket is the run its position falls in.  So the scatter stores the cell
// index only for markers of the overflow bucket, and the next sort recovers
// every other cell from the previous run offsets: per tile, the starts of the
// runs inside it are marked in LDS and a running maximum over the wave fills in
// the rest (the scan also records the bucket of every kTfStride-th position,
// where each tile starts).  That is 4 bytes a marker less to read in the count
// and the scatter and to write in the scatter.
#include <algorithm>
#include <type_traits>

#include "avl_device.h"

namespace avl {

// ---------------------------------------------------------------------------
// Marker payloads and their bucket computation, per storage form.  Component
// arrays are laid out with the padded stride g.np (a multiple of 64 markers),
// so a thread's group of consecutive markers can be read with 16-byte loads.
// ---------------------------------------------------------------------------
template <int PREC, int VD> struct Pay;

template <int VD> struct Pay<0, VD> {
    double x, v[VD], f;
    int id;
    __device__ void load(const M64& m, const Geo& g, int i, bool with_f, int = VD, bool = true) {
        x = m.x[i];
#pragma unroll
        for (int d = 0; d < VD; ++d) v[d] = m.v[(size_t)d * g.np + i];
        f = with_f ? m.f[i] : 0.0;
        id = (with_f && m.id) ? m.id[i] : 0;
    }
    __device__ void store(const M64& m, const Geo& g, int i, bool = true) const {
        m.x[i] = x;
#pragma unroll
        for (int d = 0; d < VD; ++d) m.v[(size_t)d * g.np + i] = v[d];
        m.f[i] = f;
        if (m.id) m.id[i] = id;
    }
    __device__ void push(const Geo& g, const double* sE, const RowShift*, double dtk, float, int& flags) {
        push64<VD>(g, sE, dtk, x, v);
        bool ok = isfinite(x) && isfinite(v[0]);
        if (VD == 3 && g.magnetic) ok = ok && isfinite(v[1]) && isfinite(v[2]);
        if (!ok) flags |= FLAG_NONFINITE;
    }
    __device__ int bucket(const Geo& g) const {
        int ix, jp[VD];
        double a, b[VD];
        return locate64<VD>(g, x, v, ix, jp, a, b);
    }
};

template <int VD> struct Pay<1, VD> {
    int cell;
    float a, b[VD], f;
    int id;
    // nvel < VD loads only the first nvel velocity offsets; with_cell false
    // leaves the cell index to be filled in from the previous run offsets
    __device__ void load(const M32& m, const Geo& g, int i, bool with_f, int nvel = VD, bool with_cell = true) {
        cell = with_cell ? m.cell[i] : 0;
        a = m.a[i];
#pragma unroll
        for (int d = 0; d < VD; ++d) b[d] = d < nvel ? m.b[(size_t)d * g.np + i] : 0.0f;
        f = with_f ? m.f[i] : 0.0f;
        id = (with_f && m.id) ? m.id[i] : 0;
    }
    // all_cells false (the sort's output in 1D-1V): the cell index is written
    // only for markers of the overflow bucket, the others being implied by
    // the run offsets of the new order
    __device__ void store(const M32& m, const Geo& g, int i, bool all_cells = true) const {
        if (all_cells || VD != 1 || bucket32<VD>(g, cell) == g.nb) m.cell[i] = cell;
        m.a[i] = a;
#pragma unroll
        for (int d = 0; d < VD; ++d) m.b[(size_t)d * g.np + i] = b[d];
        m.f[i] = f;
        if (m.id) m.id[i] = id;
    }
    __device__ void push(const Geo& g, const float2* sE, const RowShift* rows, double, float, int& flags) {
        push32<VD>(g, sE, rows, cell, a, b[0], flags);
    }
    __device__ int bucket(const Geo& g) const { return bucket32<VD>(g, cell); }
};

template <int PREC> struct MarkersOf;
template <> struct MarkersOf<0> { using T = M64; using E = double; };
template <> struct MarkersOf<1> { using T = M32; using E = float2; };   // E: staged field (kick, difference)

// K consecutive elements starting at a 16-byte aligned address, as 16-byte loads.
template <typename T, int K>
__device__ __forceinline__ void vload(const T* __restrict__ src, T* out)
{
    static_assert((K * sizeof(T)) % 16 == 0, "group must be a multiple of 16 bytes");
    constexpr int V = 16 / sizeof(T);
#pragma unroll
    for (int j = 0; j < K / V; ++j) {
        const int4 t = *reinterpret_cast<const int4*>(src + j * V);
        __builtin_memcpy(out + j * V, &t, 16);
    }
}

// A thread's group of K consecutive markers [first, first+K), all loads issued
// together.  Past the last marker, indices are clamped (values masked later).
// `first` is unsigned where it may pass 2^31 (1D-3V); int addresses are cheaper
// (FP64 count of 16.8M markers on the wave kernels: 53.2 us against 53.8).
template <int PREC, int VD, int K> struct Group;

template <int VD, int K> struct Group<0, VD, K> {
    Pay<0, VD> p[K];
    template <class I>
    __device__ void load(const M64& m, const Geo& g, I first, int last, bool with_f, int = VD, int = -1) {
        if (first + K - 1 <= (I)last) {
            double t[K];
            vload<double, K>(m.x + first, t);
#pragma unroll
            for (int k = 0; k < K; ++k) p[k].x = t[k];
#pragma unroll
            for (int d = 0; d < VD; ++d) {
                vload<double, K>(m.v + (size_t)d * g.np + first, t);
#pragma unroll
                for (int k = 0; k < K; ++k) p[k].v[d] = t[k];
            }
            if (with_f) {
                vload<double, K>(m.f + first, t);
#pragma unroll
                for (int k = 0; k < K; ++k) p[k].f = t[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) p[k].load(m, g, (int)min(first + (I)k, (I)last), with_f);
        }
    }
};

template <int VD, int K> struct Group<1, VD, K> {
    Pay<1, VD> p[K];
    // nvel < VD loads only the first nvel velocity offsets (the count pass
    // needs the cell index, a and the x-velocity offset only).  ovf >= 0:
    // implied cells, read from memory only at positions >= ovf (the
    // overflow run of the previous order); the rest are filled in later.
    template <class I>
    __device__ void load(const M32& m, const Geo& g, I first, int last, bool with_f, int nvel = VD, int ovf = -1) {
        if (first + K - 1 <= (I)last) {
            int ti[K];
            float t[K];
            if (ovf < 0) {
                vload<int, K>(m.cell + first, ti);
#pragma unroll
                for (int k = 0; k < K; ++k) p[k].cell = ti[k];
            } else {
#pragma unroll
                for (int k = 0; k < K; ++k) p[k].cell = 0;
                if (first + K - 1 >= (I)ovf) {
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        if (first + k >= (I)ovf) p[k].cell = m.cell[first + k];
                }
            }
            vload<float, K>(m.a + first, t);
#pragma unroll
            for (int k = 0; k < K; ++k) p[k].a = t[k];
#pragma unroll
            for (int d = 0; d < VD; ++d) {
                if (d < nvel) {
                    vload<float, K>(m.b + (size_t)d * g.np + first, t);
                } else {
#pragma unroll
                    for (int k = 0; k < K; ++k) t[k] = 0.0f;
                }
#pragma unroll
                for (int k = 0; k < K; ++k) p[k].b[d] = t[k];
            }
            if (with_f) {
                vload<float, K>(m.f + first, t);
#pragma unroll
                for (int k = 0; k < K; ++k) p[k].f = t[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int i = (int)min(first + (I)k, (I)last);
                p[k].load(m, g, i, with_f, nvel, ovf < 0 || i >= ovf);
            }
        }
    }
};

// ---------------------------------------------------------------------------
// Implied cells: the previous order's buckets of one tile's positions.
// ---------------------------------------------------------------------------
constexpr int kNoBucket = 0x7fffffff;        // past the last marker

// The order the markers are in, for implied cells: its run offsets (nb + 2
// entries) and the bucket of every kTfStride-th position.  off == nullptr:
// the cell indices are all stored.
struct Prev {
    const int* off;
    const int* tfirst;
};

__device__ __forceinline__ int tile_first_run(const Prev& pv, int base) { return pv.tfirst[base >> kTfLog]; }

// The LDS window of a sort block: the buckets its markers are expected to
// land in, counted in LDS slots 0 .. nbw-1.  The block's first and last marker
// (before the push) bound its old bucket rows [r0, r1], the input being sorted.
//  * plain: rows r0 - 1 .. r1 + 1, where every marker lands that is kicked by
//    less than one velocity cell.
//  * shear (the field's largest kick reaches a velocity cell): the rows follow
//    the kick.  Slot (r, column i) stands for row lo + r + S(i), S(i) the whole
//    part of the kick at the column markers of these rows drift to i from, so
//    a few rows hold the tile's markers however large a smooth kick is.
//  * bands (1D-3V with a magnetic field): a gyration moves a marker to
//    neighbouring vy and vz planes, rows s1 (one vy plane) and s2 (one vz
//    plane) apart; the window is a plain one at each of those planes.
// The overflow bucket has an LDS counter of its own; any other bucket outside
// the window takes one global atomic a marker.
struct Window {
    int lo, rows, nbw;      // first row, rows a band, slots (all bands)
    int shear, drift;       // rows follow the kick; the columns these rows drift by
    int nb1, nb2, s1, s2;   // bands along vy and vz planes and the rows between them
};

template <int PREC, int VD>
__device__ __forceinline__ Window set_window(const Geo& g, int b0, int b1, int shear, const RowShift* rows, int maxbins)
{
    Window w;
    // the same in every thread: scalar registers and scalar branches
    b0 = __builtin_amdgcn_readfirstlane(b0);
    b1 = __builtin_amdgcn_readfirstlane(b1);
    shear = __builtin_amdgcn_readfirstlane(shear);
    int r0 = (b0 >= g.nb ? g.nrow - 1 : b0 >> g.lognx);
    int r1 = (b1 >= g.nb ? g.nrow - 1 : b1 >> g.lognx);
    // sheared rows get one more: S is the kick at a cell centre near the marker's position
    int lo = min(r0, r1) - 1, hi = max(r0, r1) + 1 + (shear ? 1 : 0);
    const int maxrows = maxbins >> g.lognx;
    w.shear = shear;
    w.drift = 0;
    w.nb1 = w.nb2 = 1;
    w.s1 = w.s2 = 0;
    if (shear) {
        const int jx = VD == 1 ? r0 : r0 % (g.nv[0] + 1);
        if constexpr (PREC == 1) w.drift = rows[min(jx, g.nv[0])].whole;
        else w.drift = (int)floor((g.vmin[0] + (jx - 0.5) * g.dv[0]) * g.dt * g.inv_dx);
    }
    if constexpr (PREC == 0 && VD == 3) {
        if (g.magnetic) {
            // vy changes under B along x or z, vz under B along x or y
            const int s1 = g.nv[0] + 1, s2 = s1 * (g.nv[1] + 1);
            const int d1 = (g.B[0] != 0.0 || g.B[2] != 0.0) ? s1 : 0, d2 = (g.B[0] != 0.0 || g.B[1] != 0.0) ? s2 : 0;
            const int n1 = d1 ? 3 : 1, n2 = d2 ? 3 : 1, len = min(hi - lo + 1, maxrows / (n1 * n2));
            if (len > 0 && len <= s1 && 2 * d1 + len <= s2) {
                w.lo = lo - d1 - d2;
                w.rows = len;
                w.nb1 = n1;
                w.nb2 = n2;
                w.s1 = s1;
                w.s2 = s2;
                w.nbw = (len * n1 * n2) << g.lognx;
                return w;
            }
            lo -= d1 + d2;       // bands that would overlap: one window over all of them
            hi += d1 + d2;
        }
    }
    lo = max(lo, 0);
    hi = min(hi, g.nrow - 1);
    if (hi - lo + 1 > maxrows) hi = lo + maxrows - 1;
    w.lo = lo;
    w.rows = hi - lo + 1;
    w.nbw = w.rows << g.lognx;
    return w;
}

// The whole part of the kick, in velocity cells, at column i.
template <int PREC>
__device__ __forceinline__ int kick_rows(const Geo& g, const typename MarkersOf<PREC>::E* sE, int i, double dtk)
{
    if constexpr (PREC == 1) return (int)fminf(fmaxf(floorf(sE[i].x), -1e6f), 1e6f);
    else return (int)fmin(fmax(floor(g.qm * sE[i] * dtk * g.inv_dv[0]), -1e6), 1e6);
}

// Window slot of bucket b, negative for any other (the overflow bucket, which
// lies past every window, among them).
template <int PREC, int VD>
__device__ __forceinline__ int window_slot(const Geo& g, const Window& w, const typename MarkersOf<PREC>::E* sE, int b,
                                           double dtk)
{
    if (w.shear || (VD == 3 && PREC == 0 && w.nb1 * w.nb2 > 1)) {
        const int col = b & (g.nx - 1);
        int d = (b >> g.lognx) - w.lo, q = 0;
        if (VD == 3 && PREC == 0 && w.nb1 * w.nb2 > 1) {
            if (w.nb2 > 1) {
                const int q2 = (d >= w.s2) + (d >= 2 * w.s2);
                d -= q2 * w.s2;
                q = q2 * w.nb1;
            }
            if (w.nb1 > 1) {
                const int q1 = (d >= w.s1) + (d >= 2 * w.s1);
                d -= q1 * w.s1;
                q += q1;
            }
        } else {
            d -= kick_rows<PREC>(g, sE, (col - w.drift) & (g.nx - 1), dtk);
        }
        return b < g.nb && (unsigned)d < (unsigned)w.rows ? ((q * w.rows + d) << g.lognx) + col : -1;
    }
    const int rel = b - (w.lo << g.lognx);
    return (unsigned)rel < (unsigned)w.nbw ? rel : -1;
}

// The bucket of an occupied window slot (the inverse of window_slot).
template <int PREC, int VD>
__device__ __forceinline__ int slot_bucket(const Geo& g, const Window& w, const typename MarkersOf<PREC>::E* sE, int i,
                                           double dtk)
{
    if (w.shear || (VD == 3 && PREC == 0 && w.nb1 * w.nb2 > 1)) {
        const int col = i & (g.nx - 1);
        int r = i >> g.lognx;
        if (VD == 3 && PREC == 0 && w.nb1 * w.nb2 > 1) {
            const int q = r / w.rows, q2 = q / w.nb1;
            r += (q - q2 * w.nb1) * w.s1 + q2 * w.s2 - q * w.rows;
        } else {
            r += kick_rows<PREC>(g, sE, (col - w.drift) & (g.nx - 1), dtk);
        }
        return ((w.lo + r) << g.lognx) + col;
    }
    return (w.lo << g.lognx) + i;
}

// Whether a staged kick reaches one velocity cell, decided by wave (each wave
// staged a part of the field): combined from s_shear after a barrier.
static_assert(kSortThreads / kWave == 4, "one byte a wave");
__device__ __forceinline__ void note_shear(bool big, unsigned* s_shear)
{
    const int any = __any(big);
    if ((threadIdx.x & (kWave - 1)) == 0) reinterpret_cast<unsigned char*>(s_shear)[threadIdx.x / kWave] = any ? 1 : 0;
}

// Stage the field and, in the FP32 form, the drift table into LDS.  The FP64
// path stages E itself; the FP32 form stages the kick in units of dv,
// e_i = E_i * bk rounded once from FP64, with its forward difference
// e_{i+1} - e_i.  Each thread issues all its loads before its first LDS
// store, so staging costs one round trip to L2 instead of one per element.
// Returns whether a kick this thread staged reaches one velocity cell.
template <int PREC>
__device__ __forceinline__ bool stage_tables(const Geo& g, typename MarkersOf<PREC>::E* sE, RowShift* sRow,
                                             const double* __restrict__ E, const RowShift* __restrict__ rows_g,
                                             double dtk, float bk)
{
    constexpr int U = 8;
    bool big = false;
    const double to_rows = g.qm * dtk * g.inv_dv[0];
    const int nr = PREC ? g.nv[0] + 1 : 0;
    const int span = U * (int)blockDim.x;
    const int ntot = max(g.nx, nr);
    for (int i0 = 0; i0 < ntot; i0 += span) {
        double e[U], e1[U];
        RowShift r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * (int)blockDim.x + (int)threadIdx.x;
            e[u] = i < g.nx ? E[i] : 0.0;
            if (PREC) {
                e1[u] = i < g.nx ? E[(i + 1) & (g.nx - 1)] : 0.0;
                r[u] = i < nr ? rows_g[i] : RowShift{0, 0.0f};
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * (int)blockDim.x + (int)threadIdx.x;
            if constexpr (PREC) {
                const float k0 = (float)(e[u] * (double)bk), k1 = (float)(e1[u] * (double)bk);
                if (i < g.nx) sE[i] = make_float2(k0, k1 - k0);
                if (i < nr) sRow[i] = r[u];
                big |= fabsf(k0) >= 1.0f;
            } else {
                if (i < g.nx) sE[i] = e[u];
                big |= fabs(e[u] * to_rows) >= 1.0;
            }
        }
    }
    return big;
}

template <int PREC>
struct SortSmem {
    typename MarkersOf<PREC>::E* sE;
    RowShift* sRow;
    int* hist;
    __device__ SortSmem(unsigned char* smem, const Geo& g) {
        using ET = typename MarkersOf<PREC>::E;
        sE = reinterpret_cast<ET*>(smem);
        sRow = reinterpret_cast<RowShift*>(smem + sizeof(ET) * g.nx);
        // 16-byte aligned: the implied-cell map is accessed as int4
        const size_t h = (sizeof(ET) * g.nx + (PREC ? sizeof(RowShift) * (g.nv[0] + 1) : 0) + 15) & ~(size_t)15;
        hist = reinterpret_cast<int*>(smem + h);
    }
};

// ---------------------------------------------------------------------------
// count pass
// ---------------------------------------------------------------------------
// One tile of the count pass: the thread's group of K consecutive markers
// [first, first+K) of the tile [base, last] is in grp (previous order), the
// field and drift table staged in LDS.
template <int PREC, int VD, bool PUSH>
__device__ __forceinline__ void count_tile(const Geo& g, const SortSmem<PREC>& sm, Group<PREC, VD, count_mpt<PREC>()>& grp,
                                           double dtk, float bk, int* __restrict__ counts,
                                           int base, int last, int* s_b, int& fl, const unsigned* s_shear, int* s_ovf)
{
    constexpr int K = count_mpt<PREC>();
    const unsigned first = tile_item(base, threadIdx.x * K);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (first + k == base) s_b[0] = grp.p[k].bucket(g);
        if (first + k == last) s_b[1] = grp.p[k].bucket(g);
    }
    __syncthreads();
    // every thread forms the window from the tile's two end buckets itself
    const Window w = set_window<PREC, VD>(g, s_b[0], s_b[1], PUSH && *s_shear != 0, sm.sRow, g.hist_bins);
    for (int i = threadIdx.x; i < w.nbw; i += blockDim.x) sm.hist[i] = 0;
    if (threadIdx.x == 0) *s_ovf = 0;
    __syncthreads();
    int bkt[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        // FP32 form: past the last marker the group holds copies of it, pushed
        // too (the markers' LDS round trips interleave) and not counted
        if (PUSH && (PREC == 1 || first + k <= (unsigned)last)) grp.p[k].push(g, sm.sE, sm.sRow, dtk, bk, fl);
        bkt[k] = first + k <= (unsigned)last ? grp.p[k].bucket(g) : kNoBucket;
    }
    // outside the window: the overflow bucket's own counter, or a global atomic
    auto add_outside = [&](int b, int c) {
        if (b == g.nb) {
            atomicAdd(s_ovf, c);
        } else {
            atomicAdd(&counts[b], c);
        }
    };
    const bool plain = !w.shear && w.nb1 * w.nb2 == 1;
    // a thread's markers come from one or two runs, so its neighbours work
    // on other buckets: one LDS atomic a marker meets few conflicts, and
    // costs less than the compares that would merge a thread's own first
    // bkt[k] becomes the window slot, or ~bucket outside the window
    if (plain) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int rel = bkt[k] - (w.lo << g.lognx);
            bkt[k] = (unsigned)rel < (unsigned)w.nbw ? rel : ~bkt[k];
        }
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int slot = window_slot<PREC, VD>(g, w, sm.sE, bkt[k], dtk);
            bkt[k] = slot >= 0 ? slot : ~bkt[k];
        }
    }
    bool outside = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (bkt[k] >= 0) atomicAdd(&sm.hist[bkt[k]], 1);
        else outside = true;
    }
    if (outside) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (bkt[k] < 0 && bkt[k] != ~kNoBucket) add_outside(~bkt[k], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < w.nbw; i += blockDim.x) {
        const int c = sm.hist[i];
        if (c) atomicAdd(&counts[slot_bucket<PREC, VD>(g, w, sm.sE, i, dtk)], c);
    }
    if (threadIdx.x == 0 && *s_ovf) atomicAdd(&counts[g.nb], *s_ovf);
}

// count pass of one block over one tile (1D-3V, and FP64 kicks of velocity cells)
template <int PREC, int VD, bool PUSH>
__device__ __forceinline__ void count_block(const Geo& g, const typename MarkersOf<PREC>::T& m,
                                            const double* __restrict__ E, const RowShift* __restrict__ rows_g,
                                            double dtk, float bk, int* __restrict__ counts,
                                            int* __restrict__ flags, int blk)
{
    extern __shared__ __align__(16) unsigned char smem[];
    SortSmem<PREC> sm(smem, g);
    __shared__ int s_b[2], s_flags, s_ovf;
    __shared__ unsigned s_shear;
    if (threadIdx.x == 0) s_flags = 0;
    if (PUSH) note_shear(stage_tables<PREC>(g, sm.sE, sm.sRow, E, rows_g, dtk, bk), &s_shear);
    constexpr int K = count_mpt<PREC>();
    Group<PREC, VD, K> grp;
    const int base = blk * (kSortThreads * K);
    const int last = tile_last(base, kSortThreads * K, g.n);
    // the FP32 form's push needs the velocity offset b[0] only
    grp.load(m, g, tile_item(base, threadIdx.x * K), last, false, PREC ? 1 : VD);
    int fl = 0;
    count_tile<PREC, VD, PUSH>(g, sm, grp, dtk, bk, counts, base, last, s_b, fl, &s_shear, &s_ovf);
    if (fl) atomicOr(&s_flags, fl);
    __syncthreads();
    if (threadIdx.x == 0 && s_flags) atomicOr(flags, s_flags);
}

// Tile of block b of n (n a multiple of 8).  In 1D-3V each XCD (blocks go round
// the 8 of them) takes a contiguous range of tiles, so that the lines of
// destinations that neighbouring tiles share stay in one L2: 2.89 -> 2.77 ms a
// scatter of 268M FP32-form markers.  In 1D-1V blocks take tiles in order: there
// the contiguous ranges ran the scatter of 16.8M FP64 markers at 153 us against
// 139.
template <int VD>
__device__ __forceinline__ int block_tile(int b, int n) { return VD == 3 ? (b & 7) * (n >> 3) + (b >> 3) : b; }

template <int PREC, int VD, bool PUSH>
__global__ __launch_bounds__(kSortThreads) void k_count(Geo g, typename MarkersOf<PREC>::T m,
                                                         const double* __restrict__ E,
                                                         const RowShift* __restrict__ rows_g,
                                                         double dtk, float bk,
                                                         int* __restrict__ counts, int* __restrict__ flags)
{
    const int t = block_tile<VD>(blockIdx.x, gridDim.x);
    if (!tile_starts(t, kSortThreads * count_mpt<PREC>(), g.n)) return;
    count_block<PREC, VD, PUSH>(g, m, E, rows_g, dtk, bk, counts, flags, t);
}

// ---------------------------------------------------------------------------
// scatter pass: src (sorted by the previous buckets) -> dst (sorted by new)
//
// Here consecutive lanes take consecutive markers (lane-strided), unlike the
// count pass: markers of one previous run sit in neighbouring lanes and get
// consecutive ranks in their new run from the LDS atomics, so each store
// instruction writes a few contiguous stretches instead of 64 scattered words.
// ---------------------------------------------------------------------------
constexpr int kRankBits = 12;                          // a marker's rank in its window slot
constexpr int kOverflowSlot = (1 << (31 - kRankBits)) - 1;
enum : int { kOutside = -1, kNoMarker = -2 };
static_assert(kSortTile <= 1 << kRankBits && kOverflowSlot > 160 * 1024 / 4, "slot and rank share 31 bits");

// One tile of the scatter: the markers [base, last] of the previous order are
// in p[] (lane-strided), the field and drift table staged in LDS.
template <int PREC, int VD, bool PUSH>
__device__ __forceinline__ void scatter_tile(const Geo& g, const SortSmem<PREC>& sm, Pay<PREC, VD>* p,
                                             const typename MarkersOf<PREC>::T& dst, double dtk, float bk,
                                             const int* __restrict__ offsets, int* __restrict__ counts,
                                             int base, int last, int* s_b, int& fl,
                                             const unsigned* s_shear, int* s_ovf)
{
    constexpr int K = kSortMPT;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = base + k * kSortThreads + threadIdx.x;
        if (i == base) s_b[0] = p[k].bucket(g);
        if (i == last) s_b[1] = p[k].bucket(g);
    }
    __syncthreads();
    // every thread forms the window from the tile's two end buckets itself
    const Window w = set_window<PREC, VD>(g, s_b[0], s_b[1], PUSH && *s_shear != 0, sm.sRow, g.hist_bins);
    for (int i = threadIdx.x; i < w.nbw; i += blockDim.x) sm.hist[i] = 0;
    if (threadIdx.x == 0) *s_ovf = 0;
    __syncthreads();
    // place[k]: window slot (or kOverflowSlot) and rank of marker k in it, in
    // one register; kOutside and kNoMarker are negative
    int place[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = base + k * kSortThreads + threadIdx.x;
        place[k] = kNoMarker;
        if (i <= last) {
            if (PUSH) p[k].push(g, sm.sE, sm.sRow, dtk, bk, fl);
            const int b = p[k].bucket(g);
            const int slot = window_slot<PREC, VD>(g, w, sm.sE, b, dtk);
            place[k] = kOutside;
            if (slot >= 0) place[k] = (slot << kRankBits) + atomicAdd(&sm.hist[slot], 1);
            else if (b == g.nb) place[k] = (kOverflowSlot << kRankBits) + atomicAdd(s_ovf, 1);
        }
    }
    __syncthreads();
    // claim each touched in-window bucket's slots: counts[] holds the slots
    // still free, counting down from the run length, so a claim that starts
    // at or above zero lies inside the run; the histogram entry becomes the
    // first claimed position
    auto claim = [&](int b, int c) {
        const int start = atomicSub(&counts[b], c) - c;
        if (start < 0) fl |= FLAG_SLOT;
        return start < 0 ? -1 : offsets[b] + start;
    };
    for (int i = threadIdx.x; i < w.nbw; i += blockDim.x) {
        const int c = sm.hist[i];
        if (c) sm.hist[i] = claim(slot_bucket<PREC, VD>(g, w, sm.sE, i, dtk), c);
    }
    if (threadIdx.x == 0 && *s_ovf) *s_ovf = claim(g.nb, *s_ovf);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (place[k] == kNoMarker) continue;
        int dest;
        if (place[k] >= 0) {
            const int slot = place[k] >> kRankBits;
            const int first = slot == kOverflowSlot ? *s_ovf : sm.hist[slot];
            dest = first < 0 ? -1 : first + (place[k] & ((1 << kRankBits) - 1));
        } else {
            // outside the window (a jump it does not follow): one slot at a time
            const int b = p[k].bucket(g);
            const int free = atomicSub(&counts[b], 1) - 1;
            dest = free < 0 ? -1 : offsets[b] + free;
        }
        if (dest < 0) { fl |= FLAG_SLOT; continue; }
        p[k].store(dst, g, dest, false);
    }
}

template <int PREC, int VD>
__device__ __forceinline__ void load_tile(const typename MarkersOf<PREC>::T& src, const Geo& g, Pay<PREC, VD>* p,
                                          int base, int last)
{
#pragma unroll
    for (int k = 0; k < kSortMPT; ++k)
        p[k].load(src, g, min(base + k * kSortThreads + (int)threadIdx.x, last), true);
}

// scatter pass of one block over one tile (1D-3V, and in FP64 kicks of velocity
// cells and large dense sorts)
template <int PREC, int VD, bool PUSH>
__device__ __forceinline__ void scatter_block(const Geo& g, const typename MarkersOf<PREC>::T& src,
                                              const typename MarkersOf<PREC>::T& dst,
                                              const double* __restrict__ E, const RowShift* __restrict__ rows_g,
                                              double dtk, float bk, const int* __restrict__ offsets,
                                              int* __restrict__ counts, int* __restrict__ flags, int blk)
{
    extern __shared__ __align__(16) unsigned char smem[];
    SortSmem<PREC> sm(smem, g);
    __shared__ int s_b[2], s_flags, s_ovf;
    __shared__ unsigned s_shear;
    const int base = blk * kSortTile;
    const int last = tile_last(base, kSortTile, g.n);
    if (threadIdx.x == 0) s_flags = 0;
    if (PUSH) note_shear(stage_tables<PREC>(g, sm.sE, sm.sRow, E, rows_g, dtk, bk), &s_shear);
    Pay<PREC, VD> p[kSortMPT];
    load_tile<PREC, VD>(src, g, p, base, last);
    int fl = 0;
    scatter_tile<PREC, VD, PUSH>(g, sm, p, dst, dtk, bk, offsets, counts, base, last, s_b, fl, &s_shear, &s_ovf);
    if (fl) atomicOr(&s_flags, fl);
    __syncthreads();
    if (threadIdx.x == 0 && s_flags) atomicOr(flags, s_flags);
}

template <int PREC, int VD, bool PUSH>
__global__ __launch_bounds__(kSortThreads) void k_scatter1(Geo g, typename MarkersOf<PREC>::T src,
                                                           typename MarkersOf<PREC>::T dst,
                                                           const double* __restrict__ E,
                                                           const RowShift* __restrict__ rows_g,
                                                           double dtk, float bk,
                                                           const int* __restrict__ offsets,
                                                           int* __restrict__ counts, int* __restrict__ flags)
{
    const int t = block_tile<VD>(blockIdx.x, gridDim.x);
    if (!tile_starts(t, kSortTile, g.n)) return;
    scatter_block<PREC, VD, PUSH>(g, src, dst, E, rows_g, dtk, bk, offsets, counts, flags, t);
}

// ---------------------------------------------------------------------------
// 1D-1V count and scatter: one wavefront a tile
//
// A tile of 64 K markers (K = 8, or 4) is worked on by one wavefront alone,
// with its own window in LDS, so a pass has no block barriers (only the staged tables are shared, behind one barrier at
// the start): the count and scatter are chains of dependent loads, LDS round
// trips and atomics, and waves that wait for each other at every link are what
// bounded them.  16.8M FP32-form markers, 1024 x 1024 cells: count 49.6 us by
// blocks of 4096 markers, 30.3 by waves (138 MB, 25 us at the copy kernel's
// rate); scatter 92.5 by blocks of 2048, 86.4 by waves (407 MB, 74 us).  16,384
// FP64 markers: count 8.3 -> 5.2, scatter 9.0 -> 7.0.
//
// A wave's window is a box of W columns by R rows.  512 consecutive markers of
// the previous order span few columns (32 at 16 markers a cell); the push
// moves all of them by about their row's drift, and their rows by about the
// kick at their columns, so the box [first column + drift, ...) x [first row +
// smallest kick, last row + largest kick + 1] holds nearly all of them however
// far they move, in 1-3 bins a lane instead of whole bucket rows.  W is a power
// of two from 64, so 64 lanes take bins of one row.  Markers outside the box
// take one global atomic each, those of the overflow bucket one a tile.
// ---------------------------------------------------------------------------
template <int K> constexpr int kWTile = kWave * K;         // markers of a wave tile, K a lane
constexpr int kWaves = kSortThreads / kWave;
static_assert(kWTile<4> % kTfStride == 0, "wave tiles start at recorded positions");

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Inclusive running maximum over the lanes (values >= -1): DPP row shifts, then
// row broadcasts.
__device__ __forceinline__ int wave_running_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return v;
}

// Bounds of run b0 + 1 + lane, loaded ahead of a tile whose first position
// lies in run b0 (past the last run: empty).
struct WaveRuns {
    int b0, lo, hi;
};

__device__ __forceinline__ WaveRuns wave_runs_ahead(const Geo& g, const Prev& pv, int b0, int lane)
{
    WaveRuns r{b0, 0, 0};
    const int b = min(max(b0, 0), g.nb) + 1 + lane;
    if (b < g.nb) {
        r.lo = pv.off[b];
        r.hi = pv.off[b + 1];
    }
    return r;
}

// Buckets of the positions [base, end) of a wave's tile (implied cells): the
// start of every run is marked in map, a running maximum fills in the rest.
// Lane l gets the buckets of its K consecutive positions in bk[]; they are
// also left in map.
template <int K>
__device__ __forceinline__ void wave_buckets(const Geo& g, const Prev& pv, int base, int end, int lane, int* map,
                                             int (&bk)[K], const WaveRuns& ahead)
{
    static_assert(K % 4 == 0, "positions are cleared and read as 16-byte vectors");
    int4* own = reinterpret_cast<int4*>(map + lane * K);
#pragma unroll
    for (int k = 0; k < K / 4; ++k) own[k] = make_int4(lane == 0 && k == 0 ? ahead.b0 : -1, -1, -1, -1);
    wave_lds_fence();
    int b = ahead.b0 + 1 + lane, lo = b < g.nb ? ahead.lo : end, hi = ahead.hi;
    while (true) {
        if (lo < hi && lo > base && lo < end) map[lo - base] = b;
        if (__builtin_amdgcn_readlane(lo, kWave - 1) >= end) break;
        b += kWave;
        lo = end;
        if (b < g.nb) {
            lo = pv.off[b];
            hi = pv.off[b + 1];
        }
    }
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < K / 4; ++k) {
        const int4 v = own[k];
        bk[4 * k] = v.x; bk[4 * k + 1] = v.y; bk[4 * k + 2] = v.z; bk[4 * k + 3] = v.w;
    }
#pragma unroll
    for (int k = 1; k < K; ++k) bk[k] = max(bk[k], bk[k - 1]);
    const int inc = wave_running_max(bk[K - 1]);
    const int carry = __builtin_amdgcn_update_dpp(-1, inc, 0x138, 0xf, 0xf, false);   // wave_shr:1
#pragma unroll
    for (int k = 0; k < K; ++k) bk[k] = max(bk[k], carry);
#pragma unroll
    for (int k = 0; k < K / 4; ++k) own[k] = make_int4(bk[4 * k], bk[4 * k + 1], bk[4 * k + 2], bk[4 * k + 3]);
    wave_lds_fence();
}

// A wave's window: bin (r << lgw) + c stands for row row0 + r, column
// (col0 + c) mod nx.
struct Box {
    int row0, col0, lgw, rows, nbins;
    // bin of (row, col); false outside
    __device__ bool bin(const Geo& g, int row, int col, int& s) const {
        const int c = (col - col0) & (g.nx - 1), r = row - row0;
        s = (r << lgw) + c;
        return (unsigned)r < (unsigned)rows && (c >> lgw) == 0;
    }
    __device__ int bucket(const Geo& g, int s) const {
        const int c = s & ((1 << lgw) - 1);
        return ((row0 + (s >> lgw)) << g.lognx) + ((col0 + c) & (g.nx - 1));
    }
};

// The box of a tile whose first and last marker (before the push) lie in
// buckets b0 and b1, in at most maxbins bins; empty when b0 is the overflow
// bucket.  SORTED: the tile's markers are in bucket order (b0 <= b1).
template <int PREC, int K, bool PUSH, bool SORTED>
__device__ __forceinline__ Box wave_box(const Geo& g, const SortSmem<PREC>& sm, double dtk, int b0, int b1, int maxbins)
{
    Box x;
    b0 = __builtin_amdgcn_readfirstlane(b0);
    b1 = __builtin_amdgcn_readfirstlane(b1);
    const int r0 = min(b0, b1) >> g.lognx, r1 = max(b0, b1) >> g.lognx;
    const int c0 = b0 & (g.nx - 1), c1 = b1 & (g.nx - 1);
    int lo = r0, hi = r1, col = c0, ncol;
    if (SORTED) {
        ncol = min(b1 - b0 + 1, g.nx);
    } else {
        // markers in the order they were loaded or pushed in: either end may
        // lie a cell off its neighbours'; sparse rows take every column
        ncol = (long long)kWTile<K> * g.nb >= (long long)g.n * g.nx ? g.nx : ((c1 - c0) & (g.nx - 1)) + 3;
        col -= 1;
        lo -= 1;
        hi += 1;
    }
    if constexpr (PUSH) {
        // the kick at the tile's ends, with some slack for what lies between,
        // and the drift P of row r0, whole and fractional
        float k0, k1, frac;
        int whole;
        if constexpr (PREC == 1) {
            k0 = sm.sE[c0].x;
            k1 = sm.sE[c1].x;
            const RowShift p = sm.sRow[min(r0, g.nv[0])];
            whole = p.whole;
            frac = p.frac;
        } else {
            const double to_rows = g.qm * dtk * g.inv_dv[0];
            k0 = (float)(sm.sE[c0] * to_rows);
            k1 = (float)(sm.sE[c1] * to_rows);
            const double P = (g.vmin[0] + ((double)r0 - 0.5) * g.dv[0]) * g.dt * g.inv_dx;
            const double fP = floor(P);
            whole = (int)fmin(fmax(fP, -1e6), 1e6);
            frac = (float)(P - fP);
        }
        const float slack = 0.03125f + fabsf(k1 - k0);
        lo += (int)fminf(fmaxf(floorf(fminf(k0, k1) - slack), -1e6f), 1e6f);
        hi += (int)fminf(fmaxf(floorf(fmaxf(k0, k1) + slack), -1e6f), 1e6f) + 1;
        // a marker that ends in row r drifts by P(r) + [0, gam) cells, P growing
        // by gam a row; its offset adds less than one
        const float d0 = floorf(fmaxf(frac + (float)(lo - r0) * g.gam, -1e6f));
        const float d1 = floorf(fminf(frac + (float)(hi - r0 + 1) * g.gam, 1e6f)) + 1.0f;
        col += whole + (int)d0;
        ncol += (int)(d1 - d0);
    }
    lo = __builtin_amdgcn_readfirstlane(max(lo, 0));
    hi = __builtin_amdgcn_readfirstlane(min(hi, g.nrow - 1));
    ncol = __builtin_amdgcn_readfirstlane(min(ncol, g.nx));
    x.row0 = lo;
    x.col0 = __builtin_amdgcn_readfirstlane(col);
    x.lgw = min(max(6, 32 - __builtin_clz(max(ncol - 1, 1))), g.lognx);
    x.rows = b0 >= g.nb ? 0 : max(min(hi - lo + 1, maxbins >> x.lgw), 0);
    x.nbins = x.rows << x.lgw;
    return x;
}

// Bucket row and column of a marker; a row outside [0, nrow) has no bucket.
__device__ __forceinline__ void row_col(const Geo& g, const Pay<1, 1>& p, int& row, int& col)
{
    row = p.cell >> g.lognx;
    col = p.cell & (g.nx - 1);
}
__device__ __forceinline__ void row_col(const Geo& g, const Pay<0, 1>& p, int& row, int& col)
{
    const int b = p.bucket(g);
    row = b >> g.lognx;          // nrow for the overflow bucket
    col = b & (g.nx - 1);
}

// Buckets of a tile's first and last marker before the push.  FP32: from the
// implied cells in map (positions below ovf), else from the stored cells.
// FP64: from lane 0's first and lane 63's last marker (copies of the tile's
// last one past its end).
template <int PREC, int K, bool IMPL>
__device__ __forceinline__ void end_buckets(const Geo& g, const Pay<PREC, 1>* p, const typename MarkersOf<PREC>::T& m,
                                            const int* map, int base, int last, int ovf, int b0_run, int& b0, int& b1)
{
    if constexpr (PREC == 0) {
        b0 = __builtin_amdgcn_readlane(p[0].bucket(g), 0);
        b1 = __builtin_amdgcn_readlane(p[K - 1].bucket(g), kWave - 1);
    } else if (IMPL && base < ovf) {
        b0 = b0_run;
        b1 = map[min(last + 1, ovf) - 1 - base];
        wave_lds_fence();
    } else {
        b0 = bucket32<1>(g, m.cell[base]);
        b1 = bucket32<1>(g, m.cell[last]);
    }
}

// One tile of the count: lane l has the K consecutive markers from base + K l
// in grp.
template <int PREC, int K, bool PUSH, bool IMPL>
__device__ __forceinline__ void count_wave(const Geo& g, const SortSmem<PREC>& sm, Group<PREC, 1, K>& grp,
                                           const typename MarkersOf<PREC>::T& m, int* map, double dtk,
                                           int* __restrict__ counts, int base, int last, int lane, int& fl,
                                           const Prev& pv, int ovf, const WaveRuns& ahead)
{
    const int first = base + lane * K;
    if constexpr (PREC == 1 && IMPL) {
        if (base < ovf) {
            int ob[K];
            wave_buckets<K>(g, pv, base, min(last + 1, ovf), lane, map, ob, ahead);
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (first + k < ovf) grp.p[k].cell = ob[k];
        }
    }
    int b0, b1;
    end_buckets<PREC, K, IMPL>(g, grp.p, m, map, base, last, ovf, ahead.b0, b0, b1);
    const Box box = wave_box<PREC, K, PUSH, PREC ? IMPL : PUSH>(g, sm, dtk, b0, b1, g.wbins);
    for (int i = lane; i < box.nbins; i += kWave) map[i] = 0;
    wave_lds_fence();
    int row[K], col[K];
    if constexpr (PUSH && PREC == 1) {
        // only the new buckets; past the last marker the group holds copies of
        // it, pushed too (the markers' LDS round trips interleave) and not
        // counted.  The flags are raised by the scatter, which pushes the same
        // markers with the same field.
        int c[K];
        float a[K], b[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            c[k] = grp.p[k].cell;
            a[k] = grp.p[k].a;
            b[k] = grp.p[k].b[0];
        }
        push32_cells<K>(g, sm.sE, sm.sRow, c, a, b, row, col);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (PUSH) grp.p[k].push(g, sm.sE, sm.sRow, dtk, 0.0f, fl);
            row_col(g, grp.p[k], row[k], col[k]);
        }
    }
    // a lane's markers come from one or two runs, so its neighbours work on
    // other buckets: one LDS atomic a marker meets few conflicts, and costs
    // less than the compares that would merge a lane's own first
    bool outside = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int s;
        const bool in = box.bin(g, row[k], col[k], s) && first + k <= last;
        if (in) atomicAdd(&map[s], 1);
        else outside = true;
        // what is left: the bucket, or -1
        row[k] = in || first + k > last ? -1 : (unsigned)row[k] < (unsigned)g.nrow ? (row[k] << g.lognx) + col[k] : g.nb;
    }
    int novf = 0;
    if (__any(outside)) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            novf += __popcll(__ballot(row[k] == g.nb));
            if (row[k] >= 0 && row[k] != g.nb) atomicAdd(&counts[row[k]], 1);
        }
    }
    wave_lds_fence();
    for (int i = lane; i < box.nbins; i += kWave) {
        const int c = map[i];
        if (c) atomicAdd(&counts[box.bucket(g, i)], c);
    }
    if (novf && lane == 0) atomicAdd(&counts[g.nb], novf);
    wave_lds_fence();
}

// Wave wv of block blk takes wave tiles blk * 4 + wv, + stride, ...
template <int PREC, int K, bool PUSH, bool IMPL>
__device__ __forceinline__ void count_waves(const Geo& g, const typename MarkersOf<PREC>::T& m,
                                            const double* __restrict__ E, const RowShift* __restrict__ rows_g, double dtk,
                                            float bk, int* __restrict__ counts, int* __restrict__ flags, const Prev& pv,
                                            int blk, int nblk)
{
    constexpr int T = kWTile<K>;
    extern __shared__ __align__(16) unsigned char smem[];
    SortSmem<PREC> sm(smem, g);
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int* map = sm.hist + wv * g.wbins;
    if (PUSH) {
        stage_tables<PREC>(g, sm.sE, sm.sRow, E, rows_g, dtk, bk);
        __syncthreads();
    }
    const int ntiles = (g.n + T - 1) / T, stride = nblk * kWaves;
    int t = blk * kWaves + wv, fl = 0;
    const int ovf = IMPL ? pv.off[g.nb] : -1;
    // implied cells: a tile's run bounds are loaded one tile ahead, its first
    // run two tiles ahead (the bounds' addresses depend on it)
    WaveRuns ah{0, 0, 0};
    int b0n = 0;
    if constexpr (IMPL) {
        if (t < ntiles) ah = wave_runs_ahead(g, pv, tile_first_run(pv, t * T), lane);
        if (t + stride < ntiles) b0n = tile_first_run(pv, (t + stride) * T);
    }
    const int mine = (ntiles - t + stride - 1) / stride;
    for (int k = 0; t < ntiles; t += stride, ++k) {
        prio_by_progress(k, mine);
        const int last = min(t * T + T, g.n) - 1;
        Group<PREC, 1, K> grp;
        grp.load(m, g, t * T + lane * K, last, false, 1, ovf);
        WaveRuns an{0, 0, 0};
        if constexpr (IMPL) {
            if (t + stride < ntiles) an = wave_runs_ahead(g, pv, b0n, lane);
            if (t + 2 * stride < ntiles) b0n = tile_first_run(pv, (t + 2 * stride) * T);
        }
        count_wave<PREC, K, PUSH, IMPL>(g, sm, grp, m, map, dtk, counts, t * T, last, lane, fl, pv, ovf, ah);
        ah = an;
    }
    if (fl) atomicOr(flags, fl);
}

template <int PREC, int K, bool PUSH, bool IMPL>
__global__ __launch_bounds__(kSortThreads) void k_count_w(Geo g, typename MarkersOf<PREC>::T m, const double* __restrict__ E,
                                                          const RowShift* __restrict__ rows_g, double dtk, float bk,
                                                          int* __restrict__ counts, int* __restrict__ flags, Prev pv)
{
    count_waves<PREC, K, PUSH, IMPL>(g, m, E, rows_g, dtk, bk, counts, flags, pv, blockIdx.x, gridDim.x);
}

// One tile of the scatter: marker base + 64 k + lane is in p[k].
template <int PREC, int K, bool PUSH, bool IMPL>
__device__ __forceinline__ void scatter_wave(const Geo& g, const SortSmem<PREC>& sm, Pay<PREC, 1>* p,
                                             const typename MarkersOf<PREC>::T& src,
                                             const typename MarkersOf<PREC>::T& dst, int* map, double dtk,
                                             const int* __restrict__ offsets, int* __restrict__ counts,
                                             int base, int last, int lane, int& fl, const Prev& pv, int ovf,
                                             const WaveRuns& ahead)
{
    if constexpr (PREC == 1 && IMPL) {
        if (base < ovf) {
            int ob[K];
            wave_buckets<K>(g, pv, base, min(last + 1, ovf), lane, map, ob, ahead);
            // past the end of the tile the map holds its last run, and the
            // lanes copies of its last marker: pushed like it, they raise no
            // flag that it does not raise
            const int end = last < ovf ? base + kWTile<K> : ovf;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (base + k * kWave + lane < end) p[k].cell = map[k * kWave + lane];
        }
    }
    int b0, b1;
    end_buckets<PREC, K, IMPL>(g, p, src, map, base, last, ovf, ahead.b0, b0, b1);
    const Box box = wave_box<PREC, K, PUSH, PREC ? IMPL : PUSH>(g, sm, dtk, b0, b1, g.wbins);
    for (int i = lane; i < box.nbins; i += kWave) map[i] = 0;
    wave_lds_fence();
    // place[k]: bin (or kOverflowSlot) and rank of marker k in it, in one
    // register; kOutside and kNoMarker are negative
    int place[K], novf = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (PUSH) p[k].push(g, sm.sE, sm.sRow, dtk, 0.0f, fl);
        int row, col, s;
        row_col(g, p[k], row, col);
        const bool there = base + k * kWave + lane <= last;
        place[k] = there ? kOutside : kNoMarker;
        if (box.bin(g, row, col, s) && there) place[k] = (s << kRankBits) + atomicAdd(&map[s], 1);
        const unsigned long long over = __ballot(there && (unsigned)row >= (unsigned)g.nrow);
        if (over) {
            if (there && (unsigned)row >= (unsigned)g.nrow)
                place[k] = (kOverflowSlot << kRankBits) + novf + __popcll(over & ((1ull << lane) - 1));
            novf += __popcll(over);
        }
    }
    wave_lds_fence();
    // claim each touched bin's slots: counts[] holds the slots still free,
    // counting down from the run length, so a claim that starts at or above
    // zero lies inside the run; the bin becomes the first claimed position.
    // Four bins a lane at a time, so that their atomics' round trips overlap.
    for (int i0 = lane; i0 < box.nbins; i0 += 4 * kWave) {
        int c[4], at[4], off[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kWave;
            c[u] = i < box.nbins ? map[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            at[u] = off[u] = 0;
            if (c[u]) {
                const int b = box.bucket(g, i0 + u * kWave);
                at[u] = atomicSub(&counts[b], c[u]) - c[u];
                off[u] = offsets[b];
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c[u]) {
                if (at[u] < 0) fl |= FLAG_SLOT;
                map[i0 + u * kWave] = at[u] < 0 ? -1 : off[u] + at[u];
            }
    }
    int over_first = 0;
    if (novf) {
        if (lane == 0) {
            const int at = atomicSub(&counts[g.nb], novf) - novf;
            if (at < 0) fl |= FLAG_SLOT;
            over_first = at < 0 ? -1 : offsets[g.nb] + at;
        }
        over_first = __builtin_amdgcn_readfirstlane(over_first);
    }
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (place[k] == kNoMarker) continue;
        int dest;
        if (place[k] >= 0) {
            const int s = place[k] >> kRankBits;
            const int first = s == kOverflowSlot ? over_first : map[s];
            dest = first < 0 ? -1 : first + (place[k] & ((1 << kRankBits) - 1));
        } else {
            const int b = p[k].bucket(g);
            const int free = atomicSub(&counts[b], 1) - 1;
            dest = free < 0 ? -1 : offsets[b] + free;
        }
        if (dest < 0) { fl |= FLAG_SLOT; continue; }
        p[k].store(dst, g, dest, false);
    }
    wave_lds_fence();
}

// Each wave loads its next tile's markers while the current one is pushed,
// ranked, claimed and stored.  FP32: f and the cells of the overflow run are
// loaded when a tile's processing starts: only its last stores need f, and few
// tiles have such cells.  ID false: the markers carry no identities (every run
// but an adjoint's), so the payload holds no id register.
template <int PREC, int K, bool PUSH, bool IMPL, bool ID>
__device__ __forceinline__ void scatter_waves(const Geo& g, typename MarkersOf<PREC>::T src, typename MarkersOf<PREC>::T dst,
                                              const double* __restrict__ E, const RowShift* __restrict__ rows_g, double dtk,
                                              float bk, const int* __restrict__ offsets, int* __restrict__ counts,
                                              int* __restrict__ flags, const Prev& pv, int blk, int nblk)
{
    constexpr int T = kWTile<K>;
    constexpr bool F_AHEAD = ID || PREC == 0;
    if constexpr (!ID) {
        src.id = nullptr;
        dst.id = nullptr;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    SortSmem<PREC> sm(smem, g);
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int* map = sm.hist + wv * g.wbins;
    if (PUSH) {
        stage_tables<PREC>(g, sm.sE, sm.sRow, E, rows_g, dtk, bk);
        __syncthreads();
    }
    const int ntiles = (g.n + T - 1) / T, stride = nblk * kWaves;
    int t = blk * kWaves + wv;
    const int ovf = IMPL ? pv.off[g.nb] : -1;
    int fl = 0;
    Pay<PREC, 1> p[K], q[K];
    auto load_ahead = [&](Pay<PREC, 1>* r, int tile) {
        const int last = min(tile * T + T, g.n) - 1;
#pragma unroll
        for (int k = 0; k < K; ++k) r[k].load(src, g, min(tile * T + k * kWave + lane, last), F_AHEAD, 1, !IMPL);
    };
    WaveRuns ah{0, 0, 0};
    int b0n = 0;
    if (t < ntiles) load_ahead(p, t);
    if constexpr (IMPL) {
        if (t < ntiles) ah = wave_runs_ahead(g, pv, tile_first_run(pv, t * T), lane);
        if (t + stride < ntiles) b0n = tile_first_run(pv, (t + stride) * T);
    }
    const int mine = (ntiles - t + stride - 1) / stride;
    for (int n = 0; t < ntiles; t += stride, ++n) {
        prio_by_progress(n, mine);
        const int base = t * T, last = min(base + T, g.n) - 1;
        if constexpr (!F_AHEAD) {
#pragma unroll
            for (int k = 0; k < K; ++k) p[k].f = src.f[min(base + k * kWave + lane, last)];
        }
        if constexpr (PREC == 1 && IMPL) {
            if (last >= ovf) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int i = min(base + k * kWave + lane, last);
                    if (i >= ovf) p[k].cell = src.cell[i];
                }
            }
        }
        WaveRuns an{0, 0, 0};
        if (t + stride < ntiles) {
            load_ahead(q, t + stride);
            if constexpr (IMPL) an = wave_runs_ahead(g, pv, b0n, lane);
        }
        if constexpr (IMPL)
            if (t + 2 * stride < ntiles) b0n = tile_first_run(pv, (t + 2 * stride) * T);
        scatter_wave<PREC, K, PUSH, IMPL>(g, sm, p, src, dst, map, dtk, offsets, counts, base, last, lane, fl, pv, ovf, ah);
#pragma unroll
        for (int k = 0; k < K; ++k) p[k] = q[k];
        ah = an;
    }
    if (fl) atomicOr(flags, fl);
}

template <int PREC, int K, bool PUSH, bool IMPL, bool ID>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(ID ? 4 : 5)))
void k_scatter_w(Geo g, typename MarkersOf<PREC>::T src, typename MarkersOf<PREC>::T dst, const double* __restrict__ E,
                 const RowShift* __restrict__ rows_g, double dtk, float bk, const int* __restrict__ offsets,
                 int* __restrict__ counts, int* __restrict__ flags, Prev pv)
{
    scatter_waves<PREC, K, PUSH, IMPL, ID>(g, src, dst, E, rows_g, dtk, bk, offsets, counts, flags, pv, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// order-preserving push (the standalone gather+push stage)
// ---------------------------------------------------------------------------
template <int PREC, int VD>
__global__ __launch_bounds__(kSortThreads) void k_push(Geo g, typename MarkersOf<PREC>::T m,
                                                       const double* __restrict__ E,
                                                       const RowShift* __restrict__ rows_g,
                                                       double dtk, float bk, int* __restrict__ flags)
{
    using ET = typename MarkersOf<PREC>::E;
    extern __shared__ __align__(16) unsigned char smem[];
    ET* sE = reinterpret_cast<ET*>(smem);
    RowShift* sRow = reinterpret_cast<RowShift*>(smem + sizeof(ET) * g.nx);
    stage_tables<PREC>(g, sE, sRow, E, rows_g, dtk, bk);
    __syncthreads();
    int fl = 0;
    const int base = blockIdx.x * kSortTile;
    for (int k = 0; k < kSortMPT; ++k) {
        int i = base + k * kSortThreads + threadIdx.x;
        if (i < g.n) {
            Pay<PREC, VD> p;
            p.load(m, g, i, true);
            p.push(g, sE, sRow, dtk, bk, fl);
            p.store(m, g, i, true);
        }
    }
    if (fl) atomicOr(flags, fl);
}

// ---------------------------------------------------------------------------
// exclusive scan of bucket counts (three phases over tiles of kScanTile)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int wave_incl_scan(int v)
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Block-wide exclusive scan of one value per thread; returns the block total.
__device__ int block_excl_scan(int v, int* excl, int* s_w)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;
    int inc = wave_incl_scan(v);
    if (lane == kWave - 1) s_w[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int i = 0; i < nw; ++i) { int t = s_w[i]; s_w[i] = acc; acc += t; }
        s_w[nw] = acc;
    }
    __syncthreads();
    *excl = inc - v + s_w[w];
    int total = s_w[nw];
    __syncthreads();
    return total;
}

// Exclusive prefix of the per-tile totals, in place (used when there are too
// many tiles for every block of the apply kernel to sum its predecessors).
__global__ __launch_bounds__(1024) void k_scan_tiles(int* __restrict__ tile_sums, int ntiles)
{
    __shared__ int s_w[1024 / kWave + 1];
    __shared__ int s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int base = 0; base < ntiles; base += blockDim.x) {
        int i = base + threadIdx.x;
        int v = i < ntiles ? tile_sums[i] : 0;
        int excl;
        int tot = block_excl_scan(v, &excl, s_w);
        if (i < ntiles) tile_sums[i] = excl + s_carry;
        __syncthreads();
        if (threadIdx.x == 0) s_carry += tot;
        __syncthreads();
    }
}

// Where a scan tile's start comes from: the totals of the tiles before it
// (summed here, or already scanned), or, on grids of a few tiles, the counts
// before it themselves, which saves the totals' launch.
enum : int { SCAN_TOTALS = 0, SCAN_PREFIXED = 1, SCAN_COUNTS = 2 };
constexpr int kScanDirect = 24;                      // tiles up to which the counts are summed

// This thread's part of the sum of the counts [first, last).
__device__ __forceinline__ int count_part(const int* __restrict__ counts, unsigned first, unsigned last)
{
    return scan_part([=](unsigned b) { return *reinterpret_cast<const int4*>(counts + b); },
                     [=](unsigned b) { return counts[b]; }, first, last, threadIdx.x);
}

// Total of one tile of kScanTile bucket counts.
__device__ __forceinline__ void scan_total(const int* __restrict__ counts, int nbt, int* __restrict__ tsum, int tile)
{
    __shared__ int s_w[kScanThreads / kWave];
    const int base = tile * kScanTile;
    const int inc = wave_incl_scan(count_part(counts, base, tile_last(base, kScanTile, nbt) + 1));
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) s_w[threadIdx.x / kWave] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int q = 0; q < kScanThreads / kWave; ++q) t += s_w[q];
        tsum[tile] = t;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_total(const int* __restrict__ counts, int nbt, int* __restrict__ tsum)
{
    scan_total(counts, nbt, tsum, blockIdx.x);
}

// Offsets of one tile of kScanTile buckets: the tile's start plus an in-block
// exclusive scan of its counts, four per thread, both reduced behind one
// barrier.  Also (tfirst non-null: FP32 1D-1V) records for every position
// p = t kTfStride of the new order, up to the overflow run, the bucket whose run
// holds it: tfirst[t].  (16.8M markers, a third of them in the overflow run: the
// one lane that recorded it took 566 us.)
__device__ __forceinline__ void scan_tile(const int* __restrict__ counts, int nbt, const int* __restrict__ tsum,
                                          int from, int* __restrict__ offsets, int tile, int* __restrict__ tfirst)
{
    constexpr int W = kScanThreads / kWave;
    __shared__ int s_pre[W], s_cnt[W];
    // the tile's counts first, so their loads overlap the tile-start sum
    const unsigned base = tile_item(tile * kScanTile, threadIdx.x * kScanItems), end = nbt;
    int c[kScanItems] = {0, 0, 0, 0};
    if (base + kScanItems <= end) {
        const int4 v = *reinterpret_cast<const int4*>(counts + base);
        c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            if (base + k < end) c[k] = counts[base + k];
    }
    int part = 0;
    if (from == SCAN_COUNTS) part = count_part(counts, 0, tile * kScanTile);
    else if (from == SCAN_TOTALS)
        for (int t = threadIdx.x; t < tile; t += kScanThreads) part += tsum[t];
    const int s = (c[0] + c[1]) + (c[2] + c[3]);
    const int inc = wave_incl_scan(s);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) part += __shfl_xor(part, o, kWave);
    if (lane == kWave - 1) {
        s_cnt[w] = inc;
        s_pre[w] = part;
    }
    __syncthreads();
    int run = inc - s;
    if (from == SCAN_PREFIXED) run += tsum[tile];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        if (from != SCAN_PREFIXED) run += s_pre[q];
        run += q < w ? s_cnt[q] : 0;
    }
    int o[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        o[k] = run;
        run += c[k];
    }
    if (tfirst) {
        // the entries inside each run; a wave shares those of a long one
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const bool some = c[k] > 0 && base + k + 1 < end;       // not the overflow run
            const int t0 = (o[k] + kTfStride - 1) >> kTfLog, t1 = some ? (o[k] + c[k] - 1) >> kTfLog : -1;
            const bool big = t1 - t0 >= 8;
            if (!big)
                for (int t = t0; t <= t1; ++t) tfirst[t] = (int)(base + k);
            for (unsigned long long rest = __ballot(big); rest; rest &= rest - 1) {
                const int l = __builtin_ctzll(rest), last = __builtin_amdgcn_readlane(t1, l);
                const int b = __builtin_amdgcn_readlane((int)(base + k), l);
                for (int t = __builtin_amdgcn_readlane(t0, l) + lane; t <= last; t += kWave) tfirst[t] = b;
            }
        }
    }
    if (base + kScanItems <= end) {
        *reinterpret_cast<int4*>(offsets + base) = make_int4(o[0], o[1], o[2], o[3]);
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            if (base + k < end) offsets[base + k] = o[k];
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const int* __restrict__ counts, int nbt,
                                                            const int* __restrict__ tsum, int from,
                                                            int* __restrict__ offsets, int* __restrict__ tfirst)
{
    scan_tile(counts, nbt, tsum, from, offsets, blockIdx.x, tfirst);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// LDS of the block kernels: tables and window histogram.
template <int PREC>
static size_t sort_smem(const Geo& g)
{
    size_t e = sizeof(typename MarkersOf<PREC>::E) * g.nx;
    size_t r = PREC ? sizeof(RowShift) * (g.nv[0] + 1) : 0;
    return ((e + r + 15) & ~(size_t)15) + sizeof(int) * g.hist_bins;
}

// Markers a lane (K) of the wave kernels.  Small sorts are latency: four a lane
// is a shorter chain and twice the waves.  Large ones pay for every claim and
// flush, and tiles of 512 share each bin among more markers.  Measured, us, 4 /
// 8 a lane: FP32 count 8.0 / 8.8 at 1.0M markers, 13.3 / 14.1 at 4.2M, 21.4 /
// 19.4 at 8.4M, 37.5 / 30.3 at 16.8M; FP32 scatter 12.1 / 16.7, 26.4 / 27.6,
// 43.7 / 45.9, 99.2 / 86.4 (65.2 / 67.8 the other way round at 12.6M); FP64
// count 8.3 / 9.5, 16.7 / 17.2, 27.1 / 27.5, 55.8 / 53.4.  The FP64 scatter
// has registers for four only.
static int count_mpl(const Geo& g) { return g.n < (g.prec ? 5 << 20 : 12 << 20) ? 4 : 8; }
static int scatter_mpl(const Geo& g) { return g.n < 10 << 20 ? 4 : 8; }          // FP32

// The FP64 scatter of large, dense sorts goes by blocks of 2048 markers instead:
// tiles of 256 span 32 columns or fewer at 8 markers a cell, and the bins at
// their ends are claimed twice (block / wave: 141 / 156 us at 16.8M markers, 16
// a cell, 77 / 79 us at 8.4M, 8 a cell, on 1024 columns).  Not on sparse rows
// (85 / 81 us at 8.4M, 4 a cell) nor on wide grids, whose bucket rows leave a
// block's LDS window less room (179 / 158 us at 16.8M, 8 a cell, on 2048).
static bool block_scatter64(const Geo& g)
{
    return g.prec == 0 && g.n >= 1 << 23 && g.nx <= 1024 && g.n / 8 >= g.nb;
}

// LDS of the wave kernels (1D-1V): tables, and each wave's window (which also
// holds a tile's implied buckets in FP32).
template <int PREC>
static size_t wave_smem(const Geo& g)
{
    size_t e = sizeof(typename MarkersOf<PREC>::E) * g.nx;
    size_t r = PREC ? sizeof(RowShift) * (g.nv[0] + 1) : 0;
    return ((e + r + 15) & ~(size_t)15) + sizeof(int) * kWaves * g.wbins;
}

// The 1D-1V kernels of one sort phase (0 count, 2 scatter).
template <int PREC>
static hipError_t launch_sort_1v(const Geo& g, const typename MarkersOf<PREC>::T& s, const typename MarkersOf<PREC>::T& d,
                                 const double* E, const RowShift* rows, double dtk, float bk, int* counts, int* offsets,
                                 int* flags, bool push, hipStream_t st, int phase, const Prev& pv)
{
    constexpr bool F = PREC == 1;                    // the form with implied cells
    const bool impl = pv.off != nullptr;
    const dim3 bl(kSortThreads);
    // Markers whose kicks differ by more rows than a wave's window holds fall
    // outside it.  Where the loaded state's kicks reach a velocity cell the FP64
    // step takes the block kernels, whose window follows the kick column by
    // column (13.5M markers on 512 x 6600 at kicks of 8 cells: 446 us a step, by
    // waves 702); when the field has weakened since, the two are even (376 us at
    // 0.05 cells).  The FP32 form has its wave kernels only: in a weak field its
    // block kernels took 458 us there against 370 by waves, 300 against 245 for
    // 16.8M markers on 1024 x 1024, and what they won at kicks of 8 cells (494
    // against 747, but 380 against 344) can turn into that loss in any run.
    if constexpr (PREC == 0) {
        if (push && g.follow) {
            static int granted[2] = {};
            const size_t smem = sort_smem<0>(g);
            const int tile = phase == 0 ? count_tile_size(0) : kSortTile;
            const dim3 gr(tile_count(tile, g.n));
            hipError_t e = ensure_lds(phase == 0 ? (const void*)k_count<0, 1, true> : (const void*)k_scatter1<0, 1, true>,
                                      smem, granted[phase != 0]);
            if (e != hipSuccess) return e;
            if (phase == 0) launch(k_count<0, 1, true>, gr, bl, smem, st, g, s, E, rows, dtk, bk, counts, flags);
            else launch(k_scatter1<0, 1, true>, gr, bl, smem, st, g, s, d, E, rows, dtk, bk, offsets, counts, flags);
            return hipGetLastError();
        }
    }
    const size_t smem = wave_smem<PREC>(g);
    // blocks of four waves for every tile, at most what is resident
    auto grid = [&](int mpl, int resident) {
        const int tiles = (g.n + kWave * mpl - 1) / (kWave * mpl);
        return dim3(std::min((tiles + kWaves - 1) / kWaves, resident));
    };
    if (phase == 0) {
        using K = decltype(&k_count_w<PREC, 8, true, F>);
        static const K fns[8] = {k_count_w<PREC, 8, false, false>, k_count_w<PREC, 8, false, F>,
                                 k_count_w<PREC, 8, true, false>,  k_count_w<PREC, 8, true, F>,
                                 k_count_w<PREC, 4, false, false>, k_count_w<PREC, 4, false, F>,
                                 k_count_w<PREC, 4, true, false>,  k_count_w<PREC, 4, true, F>};
        static int granted[8] = {};
        const int mpl = count_mpl(g), v = (mpl == 4 ? 4 : 0) + 2 * (push ? 1 : 0) + (impl ? 1 : 0);
        hipError_t e = ensure_lds((const void*)fns[v], smem, granted[v]);
        if (e != hipSuccess) return e;
        launch(fns[v], grid(mpl, g.cblocks), bl, smem, st, g, s, E, rows, dtk, bk, counts, flags, pv);
        return hipGetLastError();
    }
    if (block_scatter64(g)) {
        static int granted[2] = {};
        const size_t sb = sort_smem<PREC>(g);
        hipError_t e = ensure_lds(push ? (const void*)k_scatter1<0, 1, true> : (const void*)k_scatter1<0, 1, false>, sb,
                                  granted[push ? 1 : 0]);
        if (e != hipSuccess) return e;
        const dim3 gr((g.n + kSortTile - 1) / kSortTile);
        if constexpr (PREC == 0) {
            if (push) launch(k_scatter1<0, 1, true>, gr, bl, sb, st, g, s, d, E, rows, dtk, bk, offsets, counts, flags);
            else launch(k_scatter1<0, 1, false>, gr, bl, sb, st, g, s, d, E, rows, dtk, bk, offsets, counts, flags);
        }
        return hipGetLastError();
    }
    const auto scatter = [&](auto lanes) {
        constexpr int K = decltype(lanes)::value;
        using Fn = decltype(&k_scatter_w<PREC, K, true, F, true>);
        static const Fn fns[8] = {
            k_scatter_w<PREC, K, false, false, false>, k_scatter_w<PREC, K, false, false, true>,
            k_scatter_w<PREC, K, false, F, false>,     k_scatter_w<PREC, K, false, F, true>,
            k_scatter_w<PREC, K, true, false, false>,  k_scatter_w<PREC, K, true, false, true>,
            k_scatter_w<PREC, K, true, F, false>,      k_scatter_w<PREC, K, true, F, true>};
        static int granted[8] = {};
        const int v = 4 * (push ? 1 : 0) + 2 * (impl ? 1 : 0) + (s.id ? 1 : 0);
        hipError_t e = ensure_lds((const void*)fns[v], smem, granted[v]);
        if (e != hipSuccess) return e;
        launch(fns[v], grid(K, s.id ? g.sblocks : g.sblocks_step), bl, smem, st, g, s, d, E, rows, dtk, bk,
               (const int*)offsets, counts, flags, pv);
        return hipGetLastError();
    };
    if constexpr (PREC == 1)
        if (scatter_mpl(g) == 8) return scatter(std::integral_constant<int, 8>());
    return scatter(std::integral_constant<int, 4>());
}

template <int PREC, int VD>
static hipError_t launch_sort_t(const Geo& g, void* src, void* dst, const double* E, const RowShift* rows,
                                double dtk, float bk, int* counts, int* offsets, int* tile_sums, int* flags, bool push,
                                hipStream_t st, int phase, const int* off_old, const int* tf_old, int* tf_new)
{
    using MT = typename MarkersOf<PREC>::T;
    MT s = *reinterpret_cast<MT*>(src);
    MT d = dst ? *reinterpret_cast<MT*>(dst) : s;
    const Prev pv{off_old, tf_old};
    if (g.n == 0 && phase != 1) return hipSuccess;   // the scan still runs: offsets become zero
    if (phase == 1) {
        const int nbt = g.nb + 1;
        const int ntiles = tile_count(kScanTile, nbt);
        int from = SCAN_COUNTS;
        if (ntiles > kScanDirect) {
            hipLaunchKernelGGL(k_scan_total, dim3(ntiles), dim3(kScanThreads), 0, st, counts, nbt, tile_sums);
            from = SCAN_TOTALS;
        }
        if (ntiles > 1024) {
            hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(1024), 0, st, tile_sums, ntiles);
            from = SCAN_PREFIXED;
        }
        hipLaunchKernelGGL(k_scan_apply, dim3(ntiles), dim3(kScanThreads), 0, st, counts, nbt, tile_sums, from, offsets,
                           tf_new);
        return hipGetLastError();
    }
    if constexpr (VD == 1) {
        return launch_sort_1v<PREC>(g, s, d, E, rows, dtk, bk, counts, offsets, flags, push, st, phase, pv);
    } else {
        // the other forms hold more registers a marker: a block a tile
        const size_t smem = sort_smem<PREC>(g);
        static int granted[4] = {};
        const void* fns[4] = {(const void*)k_count<PREC, VD, true>, (const void*)k_count<PREC, VD, false>,
                              (const void*)k_scatter1<PREC, VD, true>, (const void*)k_scatter1<PREC, VD, false>};
        for (int i = 0; i < 4; ++i) {
            hipError_t e = ensure_lds(fns[i], smem, granted[i]);
            if (e != hipSuccess) return e;
        }
        const dim3 bl(kSortThreads);
        const dim3 cg((tile_count(count_tile_size(PREC), g.n) + 7) & ~7), sg((tile_count(kSortTile, g.n) + 7) & ~7);
        if (phase == 0) {
            if (push) launch(k_count<PREC, VD, true>, cg, bl, smem, st, g, s, E, rows, dtk, bk, counts, flags);
            else launch(k_count<PREC, VD, false>, cg, bl, smem, st, g, s, E, rows, dtk, bk, counts, flags);
        } else {
            if (push) launch(k_scatter1<PREC, VD, true>, sg, bl, smem, st, g, s, d, E, rows, dtk, bk, offsets, counts, flags);
            else launch(k_scatter1<PREC, VD, false>, sg, bl, smem, st, g, s, d, E, rows, dtk, bk, offsets, counts, flags);
        }
        return hipGetLastError();
    }
}

// phase 0 = count, 1 = scan, 2 = scatter.  offsets: the run offsets of the new
// order (written by the scan, used by the scatter); off_old / tf_old: the
// order the markers are in, for implied cells (FP32 1D-1V; nullptr when every
// cell index is stored); tf_new (FP32 1D-1V, may be null): the scan's record of the new
// order's tile starts.
hipError_t launch_sort(const Geo& g, void* src, void* dst, const double* E, const RowShift* rows,
                       double dtk, float bk, int* counts, int* offsets, int* tile_sums, int* flags,
                       bool push, hipStream_t st, int phase, const int* off_old, const int* tf_old, int* tf_new)
{
    if (g.prec == 0 && g.vdim == 1) return launch_sort_t<0, 1>(g, src, dst, E, rows, dtk, bk, counts, offsets, tile_sums, flags, push, st, phase, nullptr, nullptr, nullptr);
    if (g.prec == 0 && g.vdim == 3) return launch_sort_t<0, 3>(g, src, dst, E, rows, dtk, bk, counts, offsets, tile_sums, flags, push, st, phase, nullptr, nullptr, nullptr);
    if (g.prec == 1 && g.vdim == 1) return launch_sort_t<1, 1>(g, src, dst, E, rows, dtk, bk, counts, offsets, tile_sums, flags, push, st, phase, off_old, tf_old, tf_new);
    return launch_sort_t<1, 3>(g, src, dst, E, rows, dtk, bk, counts, offsets, tile_sums, flags, push, st, phase, nullptr, nullptr, nullptr);
}

// ---------------------------------------------------------------------------
// batched passes: one launch covers every instance of a batch (1D-1V); block b
// belongs to the instance whose prefix range holds b and runs that
// instance's block body with the instance's own geometry and buffers.  The
// instances are always in a sorted order here, so FP32 cells are implied.
// ---------------------------------------------------------------------------
template <int PREC> __device__ __forceinline__ const typename MarkersOf<PREC>::T& bmark(const BInst& I, int b);
template <> __device__ __forceinline__ const M64& bmark<0>(const BInst& I, int b) { return I.m64[b]; }
template <> __device__ __forceinline__ const M32& bmark<1>(const BInst& I, int b) { return I.m32[b]; }

template <int PREC>
__global__ __launch_bounds__(kSortThreads) void k_count_b(const BInst* __restrict__ tab, const int* __restrict__ pre,
                                                          int ninst, int cur)
{
    const int* pr = pre + BPRE_COUNT * (ninst + 1);
    const int i = find_inst(pr, ninst, blockIdx.x);
    const BInst& I = tab[i];
    count_waves<PREC, PREC ? 8 : 4, true, PREC == 1>(I.g, bmark<PREC>(I, cur), I.E, I.rows, I.dtk, I.bk, I.counts, I.flags,
                                       Prev{I.offsets[cur], I.tfirst[cur]}, blockIdx.x - pr[i], pr[i + 1] - pr[i]);
}

__global__ __launch_bounds__(kScanThreads) void k_scan_total_b(const BInst* __restrict__ tab, const int* __restrict__ pre,
                                                               int ninst)
{
    const int* pr = pre + BPRE_SCAN * (ninst + 1);
    const int i = find_inst(pr, ninst, blockIdx.x);
    const BInst& I = tab[i];
    scan_total(I.counts, I.g.nb + 1, I.tsum, blockIdx.x - pr[i]);
}

__global__ __launch_bounds__(kScanThreads) void k_scan_b(const BInst* __restrict__ tab, const int* __restrict__ pre,
                                                         int ninst, int cur)
{
    const int* pr = pre + BPRE_SCAN * (ninst + 1);
    const int i = find_inst(pr, ninst, blockIdx.x);
    const BInst& I = tab[i];
    scan_tile(I.counts, I.g.nb + 1, I.tsum, SCAN_TOTALS, I.offsets[1 - cur], blockIdx.x - pr[i],
              I.g.prec ? I.tfirst[1 - cur] : nullptr);
}

// Batch instances carry no marker identities.
template <int PREC>
__global__ __launch_bounds__(kSortThreads) void k_scatter_b(const BInst* __restrict__ tab,
                                                            const int* __restrict__ pre, int ninst, int cur)
{
    const int* pr = pre + BPRE_SCATTER * (ninst + 1);
    const int i = find_inst(pr, ninst, blockIdx.x);
    const BInst& I = tab[i];
    scatter_waves<PREC, PREC ? 8 : 4, true, PREC == 1, false>(I.g, bmark<PREC>(I, cur), bmark<PREC>(I, 1 - cur), I.E, I.rows, I.dtk, I.bk,
                                                I.offsets[1 - cur], I.counts, I.flags,
                                                Prev{I.offsets[cur], I.tfirst[cur]}, blockIdx.x - pr[i],
                                                pr[i + 1] - pr[i]);
}

// Blocks of a batched pass for one instance (host side): a scan tile each, or
// four waves with a tile each.
int sort_blocks(const Geo& g, int phase)
{
    if (phase == 1) return (g.nb + 1 + kScanTile - 1) / kScanTile;
    const int tile = kWaves * (g.prec ? kWTile<8> : kWTile<4>);
    return (g.n + tile - 1) / tile;
}

// Resident blocks per CU of a wave kernel for this geometry's LDS (1D-1V).
static int wave_blocks_per_cu(const Geo& g, const void* f64, const void* f32, int (&granted)[2])
{
    if (g.vdim != 1) return 0;
    const void* fn = g.prec ? f32 : f64;
    const size_t smem = g.prec ? wave_smem<1>(g) : wave_smem<0>(g);
    int per_cu = 0;
    if (ensure_lds(fn, smem, granted[g.prec]) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kSortThreads, smem) != hipSuccess || per_cu <= 0) {
        (void)hipGetLastError();
        per_cu = 4;
    }
    return per_cu;
}

int count_blocks_per_cu(const Geo& g)
{
    static int granted[2] = {};
    return wave_blocks_per_cu(g, (const void*)k_count_w<0, 8, true, false>, (const void*)k_count_w<1, 8, true, true>, granted);
}

int scatter_step_blocks_per_cu(const Geo& g)
{
    static int granted[2] = {};
    return wave_blocks_per_cu(g, (const void*)k_scatter_w<0, 4, true, false, false>,
                              (const void*)k_scatter_w<1, 8, true, true, false>, granted);
}

int scatter_blocks_per_cu(const Geo& g)
{
    static int granted[2] = {};
    return wave_blocks_per_cu(g, (const void*)k_scatter_w<0, 4, true, false, true>,
                              (const void*)k_scatter_w<1, 8, true, true, true>, granted);
}

// LDS of the batched count and scatter for one instance (host side).
size_t sort_lds(const Geo& g) { return g.prec ? wave_smem<1>(g) : wave_smem<0>(g); }

// phase 0 = count (with push), 1 = scan, 2 = scatter, over `blocks` blocks
hipError_t launch_sort_batch(int prec, const BInst* tab, const int* pre, int ninst, int blocks, size_t smem, int cur,
                             hipStream_t st, int phase)
{
    if (blocks <= 0) return hipSuccess;
    static int granted[4] = {0, 0, 0, 0};
    const void* fns[4] = {(const void*)k_count_b<0>, (const void*)k_count_b<1>, (const void*)k_scatter_b<0>,
                          (const void*)k_scatter_b<1>};
    {
        const int i = (phase == 2 ? 2 : 0) + (prec == 0 ? 0 : 1);
        hipError_t e = phase == 1 ? hipSuccess : ensure_lds(fns[i], smem, granted[i]);
        if (e != hipSuccess) return e;
    }
    const dim3 gr(blocks);
    if (phase == 0) {
        if (prec == 0) hipLaunchKernelGGL(k_count_b<0>, gr, dim3(kSortThreads), smem, st, tab, pre, ninst, cur);
        else hipLaunchKernelGGL(k_count_b<1>, gr, dim3(kSortThreads), smem, st, tab, pre, ninst, cur);
    } else if (phase == 1) {
        hipLaunchKernelGGL(k_scan_total_b, gr, dim3(kScanThreads), 0, st, tab, pre, ninst);
        hipLaunchKernelGGL(k_scan_b, gr, dim3(kScanThreads), 0, st, tab, pre, ninst, cur);
    } else {
        if (prec == 0) hipLaunchKernelGGL(k_scatter_b<0>, gr, dim3(kSortThreads), smem, st, tab, pre, ninst, cur);
        else hipLaunchKernelGGL(k_scatter_b<1>, gr, dim3(kSortThreads), smem, st, tab, pre, ninst, cur);
    }
    return hipGetLastError();
}

// Stored cell index of every marker of a sorted FP32 1D-1V order: the run a
// position lies in is its cell (the overflow run keeps its stored values).
__global__ __launch_bounds__(256) void k_cells(Geo g, const int* __restrict__ off, int* __restrict__ cell)
{
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < g.nb; b += gridDim.x * blockDim.x) {
        const int lo = off[b], hi = off[b + 1];
        for (int p = lo; p < hi; ++p) cell[p] = b;
    }
}

hipError_t launch_cells(const Geo& g, const int* offsets, int* cell, hipStream_t st)
{
    if (g.n == 0) return hipSuccess;
    const int blocks = std::min((g.nb + 255) / 256, 8192);
    hipLaunchKernelGGL(k_cells, dim3(blocks), dim3(256), 0, st, g, offsets, cell);
    return hipGetLastError();
}

hipError_t launch_push(const Geo& g, void* m, const double* E, const RowShift* rows, double dtk, float bk,
                       int* flags, hipStream_t st)
{
    if (g.n == 0) return hipSuccess;
    const int blocks = tile_count(kSortTile, g.n);
    const size_t smem = (g.prec ? sizeof(float2) : sizeof(double)) * g.nx + (g.prec ? sizeof(RowShift) * (g.nv[0] + 1) : 0);
    if (g.prec == 0 && g.vdim == 1) hipLaunchKernelGGL((k_push<0, 1>), dim3(blocks), dim3(kSortThreads), smem, st, g, *reinterpret_cast<M64*>(m), E, rows, dtk, bk, flags);
    else if (g.prec == 0) hipLaunchKernelGGL((k_push<0, 3>), dim3(blocks), dim3(kSortThreads), smem, st, g, *reinterpret_cast<M64*>(m), E, rows, dtk, bk, flags);
    else if (g.vdim == 1) hipLaunchKernelGGL((k_push<1, 1>), dim3(blocks), dim3(kSortThreads), smem, st, g, *reinterpret_cast<M32*>(m), E, rows, dtk, bk, flags);
    else hipLaunchKernelGGL((k_push<1, 3>), dim3(blocks), dim3(kSortThreads), smem, st, g, *reinterpret_cast<M32*>(m), E, rows, dtk, bk, flags);
    return hipGetLastError();
}

}  // namespace avl
