// md_cells.hip -- steps N1-N4 of section 2.3 as a counting sort, plus the
// reorder of section 2.4 item (4) done on the GPU with the prefix-scan the
// paper names as the alternative to its CPU pass.
//
//   k_bin        N1/N2: cell of every atom; atomic occupancy count gives the
//                atom's (unordered) rank in its cell
//   k_scan_*     N3/N4: exclusive scan of the counts -> cell_start, and the
//                largest occupancy; clears the counts for the next build
//   k_scatter    slots grouped by cell (in the order the atomics gave), with
//                each slot's permanent id beside it
//   k_cellsort   inside each cell, ascending permanent id (the paper leaves
//                the order open; a fixed order makes the list reproducible):
//                each atom's place is the number of its cell's members with
//                a smaller id; with reorder on it also writes the atom's data
//                to that place in the scratch arrays
//   k_copyback   with reorder on: the scratch arrays back into the state
//
// Every kernel returns at once unless the rebuild flag is set (or the call
// forces the build), so a step's launch sequence is fixed.  Each kernel is a
// template over where its parameters come from (one system, or one replica
// of a batch: md_internal.h).
#include <type_traits>

#include "md_finish.h"

namespace md {

__device__ __forceinline__ bool rebuild_on(const KParams& p, int force)
{
    return force || p.dev->rebuild;
}

template <class B>
__global__ void k_clear(B b)
{
    Wg wg;
    KParams p;
    if (!b.fetch(G_ATOMS, wg, p)) return;
    const int i0 = wg.id * blockDim.x + threadIdx.x;
    for (int i = i0; i < p.ncell; i += wg.n * blockDim.x) p.cell_count[i] = 0;
    if (i0 == 0) {
        DevState* d = p.dev;
        d->step = 0;
        d->n_rebuilds = 0;
        d->hist_count = 0;
        d->dmax2 = 0.0;
        d->rebuild = 0;
        d->blocks_done = 0;
        d->flags = 0;
        d->max_occ = 0;
        d->max_nl = 0;
        d->record = 0;
        for (int k = 0; k < 8; ++k) d->obs[k] = 0.0;
        for (int k = 0; k < kDmaxSlots; ++k) d->dmax_slot[k] = 0;
    }
}

__device__ __forceinline__ void bin_atoms(const KParams& p, const Wg& wg)
{
    for (int i0 = wg.id * blockDim.x; i0 < p.n; i0 += wg.n * blockDim.x) {
        const int i = i0 + threadIdx.x;
        const bool act = i < p.n;
        int c = -1;
        if (act) {
            // positions are folded into [0, L) here, at each cell build, and
            // drift freely in between (by less than skin/2), so the wrap bits
            // of the list stay valid until the next build
            const double x = wrap(p.x[i], p.L), y = wrap(p.y[i], p.L), z = wrap(p.z[i], p.L);
            p.x[i] = x;
            p.y[i] = y;
            p.z[i] = z;
            c = cell_of_pos(x, y, z, p);
            p.cell_of[i] = c;
        }
        rank_in_cell(p, act, c, i);
    }
}

template <class B>
__global__ void k_bin(B b, int force)
{
    Wg wg;
    KParams p;
    if (!b.fetch_gated(G_ATOMS, force, wg, p)) return;
    bin_atoms(p, wg);
}

// k_bin with the finish of the integration pass (or fused force pass) before it:
// every workgroup takes the rebuild decision itself from the sixteen displacement
// maxima (one load), the first one also counts and records the step (finish_step,
// which leaves the maxima for the others; the scan after it clears them).  Saves
// the finish's launch, 4.3 us of a 42 us step at 256 000 WCA atoms, 3.6 of 70 at the
// melt of 262 144.  Not over replicas: there every workgroup would read its
// replica's parameters first, 8.6 us against 4.8 + 5.2 apart and no faster a step.
__global__ __launch_bounds__(1024) void k_bin_finish(Single b, int record_every, int fused)
{
    const KParams& p = b.p;
    const Wg wg{(int)blockIdx.x, (int)gridDim.x};
    bool rebuild;
    if (wg.id == 0) {
        __shared__ double red[(1024 / kWave) * 5];
        rebuild = finish_step<true>(p, 1, record_every, fused != 0, red);
    } else {
        __shared__ int rb;
        if (threadIdx.x < kWave) {
            const double m = step_dmax2(p);
            if (threadIdx.x == 0) rb = m > p.disp_thr2 ? 1 : 0;
        }
        __syncthreads();
        rebuild = rb != 0;
    }
    if (rebuild) bin_atoms(p, wg);
}

// The cell offsets: one workgroup of kScanThreads threads scans the counts
// kScanPer cells per thread at a time (one 16-byte load each), in chunks of
// kScanThreads * kScanPer cells carried over in order; writes cell_start,
// clears the counts for the next binning and records the largest
// occupancy.  A single launch, so that a step with no rebuild pays for one
// idle kernel here rather than three.
// The scan itself, by one workgroup of kScanThreads threads (wsum: LDS, one
// int per wave).
__device__ __forceinline__ void scan_cells(const KParams& p, int* wsum, int* lds_start = nullptr)
{
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    int carry = 0, m = 0;
    for (int c0 = 0; c0 < p.ncell; c0 += kScanThreads * kScanPer) {
        const int c = c0 + threadIdx.x * kScanPer;
        int v[kScanPer];
        if (c + kScanPer <= p.ncell) {
            const int4 q = *reinterpret_cast<const int4*>(p.cell_count + c);
            v[0] = q.x;
            v[1] = q.y;
            v[2] = q.z;
            v[3] = q.w;
        } else {
#pragma unroll
            for (int k = 0; k < kScanPer; ++k) v[k] = c + k < p.ncell ? p.cell_count[c + k] : 0;
        }
        int sum = 0;
#pragma unroll
        for (int k = 0; k < kScanPer; ++k) {
            sum += v[k];
            m = v[k] > m ? v[k] : m;
        }
        // exclusive scan of the thread sums: wave64 DPP scan, then the wave totals
        const int inc = wave_scan_incl(sum);
        if (lane == kWave - 1) wsum[wid] = inc;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kScanThreads / kWave; ++w) {
            before += w < wid ? wsum[w] : 0;
            total += wsum[w];
        }
        __syncthreads();
        int ex = carry + before + inc - sum;
        if (c + kScanPer <= p.ncell) {
            const int4 st = make_int4(ex, ex + v[0], ex + v[0] + v[1], ex + v[0] + v[1] + v[2]);
            *reinterpret_cast<int4*>(p.cell_start + c) = st;
            *reinterpret_cast<int4*>(p.cell_count + c) = make_int4(0, 0, 0, 0);
            if (lds_start) {
                lds_start[c] = st.x;
                lds_start[c + 1] = st.y;
                lds_start[c + 2] = st.z;
                lds_start[c + 3] = st.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < kScanPer; ++k) {
                if (c + k < p.ncell) {
                    p.cell_start[c + k] = ex;
                    p.cell_count[c + k] = 0;
                    if (lds_start) lds_start[c + k] = ex;
                }
                ex += v[k];
            }
        }
        carry += total;
    }
    m = wave_max(m);
    if (lane == 0) wsum[wid] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        int tm = 0;
        for (int w = 0; w < kScanThreads / kWave; ++w) tm = wsum[w] > tm ? wsum[w] : tm;
        p.dev->max_occ = tm;
        p.dev->max_nl = 0;
        p.cell_start[p.ncell] = carry;
        if (lds_start) lds_start[p.ncell] = carry;
    }
}

template <class B>
__global__ __launch_bounds__(kScanThreads) void k_scan(B b, int force)
{
    Wg wg;
    KParams p;
    if constexpr (std::is_same_v<B, Single>)  // see k_bin_finish
        if (threadIdx.x < kDmaxSlots) b.p.dev->dmax_slot[threadIdx.x] = 0;
    if (!b.fetch_gated(G_ONE, force, wg, p)) return;
    __shared__ int wsum[kScanThreads / kWave];
    scan_cells(p, wsum);
}

// The scan of a system with many cells, spread over workgroups of one chunk of
// scan_chunk(p) cells each: the counts become offsets inside the chunk, in
// place, and the chunk's total and largest count go to p.ipart (free between
// the finish and the next integration); k_scatter adds the chunks before.  One
// workgroup walking all cells is a chain of loads and barriers, about 1 us per
// 4096 cells: 28 us at 110 592 cells (256 000 WCA atoms), where this takes 4.
constexpr int kScanChunksMax = 1024;

__host__ __device__ inline int scan_chunk(const KParams& p)
{
    constexpr int unit = kScanThreads * kScanPer;
    const int n = (int)(((int64_t)p.ncell + unit - 1) / unit);  // chunks of one round
    return ((n + kScanChunksMax - 1) / kScanChunksMax) * unit;
}
__host__ __device__ inline int scan_chunks(const KParams& p)
{
    const int c = scan_chunk(p);
    return (int)(((int64_t)p.ncell + c - 1) / c);
}

__global__ __launch_bounds__(kScanThreads) void k_scan_part(Single b, int force)
{
    const KParams& p = b.p;
    if (blockIdx.x == 0 && threadIdx.x < kDmaxSlots) p.dev->dmax_slot[threadIdx.x] = 0;
    if (!rebuild_on(p, force)) return;
    __shared__ int wsum[kScanThreads / kWave];
    const int chunk = scan_chunk(p), first = (int)blockIdx.x * chunk;
    const int last = p.ncell - first < chunk ? p.ncell : first + chunk;
    int carry = 0, m = 0;
    for (int c0 = first; c0 < last; c0 += kScanThreads * kScanPer) {
        const int c = c0 + threadIdx.x * kScanPer;
        int v[kScanPer], sum = 0;
        if (c + kScanPer <= last) {
            const int4 q = *reinterpret_cast<const int4*>(p.cell_count + c);
            v[0] = q.x;
            v[1] = q.y;
            v[2] = q.z;
            v[3] = q.w;
        } else {
#pragma unroll
            for (int k = 0; k < kScanPer; ++k) v[k] = c + k < last ? p.cell_count[c + k] : 0;
        }
#pragma unroll
        for (int k = 0; k < kScanPer; ++k) {
            sum += v[k];
            m = v[k] > m ? v[k] : m;
        }
        int total;
        int ex = carry + workgroup_scan_excl(sum, wsum, total);
        if (c + kScanPer <= last) {
            *reinterpret_cast<int4*>(p.cell_count + c) =
                make_int4(ex, ex + v[0], ex + v[0] + v[1], ex + v[0] + v[1] + v[2]);
        } else {
#pragma unroll
            for (int k = 0; k < kScanPer; ++k) {
                if (c + k < last) p.cell_count[c + k] = ex;
                ex += v[k];
            }
        }
        carry += total;
    }
    m = workgroup_max(m);
    if (threadIdx.x == 0) {
        int* const part = reinterpret_cast<int*>(p.ipart);
        part[blockIdx.x] = carry;
        part[kScanChunksMax + blockIdx.x] = m;
    }
}

// The atoms before each chunk of k_scan_part, into LDS (by the whole
// workgroup); the first workgroup also publishes the largest occupancy.
__device__ __forceinline__ void chunk_starts(const KParams& p, const Wg& wg, int* pre)
{
    const int* part = reinterpret_cast<const int*>(p.ipart);
    const int n = scan_chunks(p);
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        int carry = 0, m = 0;
        for (int c = lane; c - lane < n; c += kWave) {
            const int v = c < n ? part[c] : 0;
            if (wg.id == 0 && c < n) {
                const int o = part[kScanChunksMax + c];
                m = o > m ? o : m;
            }
            const int inc = wave_scan_incl(v);
            if (c < n) pre[c] = carry + inc - v;
            carry += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
        if (wg.id == 0) {
            m = wave_max(m);
            if (lane == 0) {
                p.dev->max_occ = m;
                p.dev->max_nl = 0;
            }
        }
    }
    __syncthreads();
}

// Slot q of atom i in cell order (in the order the atomics gave), with its
// permanent id beside it for the in-cell rank.
__device__ __forceinline__ void scatter_atom(const KParams& p, int i, int start)
{
    const int q = start + p.slot[i], key = p.id[i];
    p.tmp[q] = i;
    p.tmp[p.n + q] = key;  // the ids of a cell side by side
}

// Canonical order inside each cell: ascending permanent id.  The atom at
// slot-order position q counts the members of its cell with a smaller id
// (ids are distinct); that count is its place.  With kPermute the atom's
// data go to that place in the scratch arrays (the permutation into cell
// order, scattered from the atom rather than gathered by a second pass):
// P_NONE nothing, P_STATE all but the forces, P_ALL the forces (type F) too.
enum Permute { P_NONE, P_STATE, P_ALL };

template <typename F, Permute kPermute>
__device__ __forceinline__ void sort_slot(const KParams& p, int q)
{
    const int32_t* ids = p.tmp + p.n;  // ids in slot order (scatter_atom)
    const int s = p.tmp[q], key = ids[q];
    const int c = p.cell_of[s];
    // every load before the first store (the compiler may not reorder them)
    double x, y, z, vx, vy, vz;
    F fx, fy, fz;
    if (kPermute != P_NONE) {
        x = p.x[s];
        y = p.y[s];
        z = p.z[s];
        vx = p.vx[s];
        vy = p.vy[s];
        vz = p.vz[s];
        if (kPermute == P_ALL) {
            fx = static_cast<const F*>(p.fx)[s];
            fy = static_cast<const F*>(p.fy)[s];
            fz = static_cast<const F*>(p.fz)[s];
        }
    }
    const int a = p.cell_start[c], cnt = p.cell_start[c + 1] - a;
    int rank = 0;
#pragma unroll 4
    for (int j = 0; j < cnt; ++j) rank += ids[a + j] < key ? 1 : 0;
    const int d = a + rank;
    p.order[d] = s;
    if (kPermute != P_NONE) {
        p.sx[d] = x;
        p.sy[d] = y;
        p.sz[d] = z;
        p.svx[d] = vx;
        p.svy[d] = vy;
        p.svz[d] = vz;
        if (kPermute == P_ALL) {
            reinterpret_cast<F*>(p.sfx)[d] = fx;
            reinterpret_cast<F*>(p.sfy)[d] = fy;
            reinterpret_cast<F*>(p.sfz)[d] = fz;
        }
        p.sid[d] = key;
        p.scell[d] = c;
        if (kPermute == P_STATE && p.bonded_on) bond_slot(p, key, d);
    }
}

// kPart: behind k_scan_part; also writes the final cell_start.
template <class B, bool kPart>
__global__ void k_scatter(B b, int force)
{
    Wg wg;
    KParams p;
    if (!b.fetch_gated(G_ATOMS, force, wg, p)) return;
    const int i0 = wg.id * blockDim.x + threadIdx.x, stride = wg.n * blockDim.x;
    if constexpr (kPart) {
        __shared__ int pre[kScanChunksMax];
        chunk_starts(p, wg, pre);
        const int chunk = scan_chunk(p);
        for (int i = i0; i < p.n; i += stride) {
            const int c = p.cell_of[i];
            scatter_atom(p, i, p.cell_count[c] + pre[c / chunk]);
        }
        for (int c = i0; c < p.ncell; c += stride)
            p.cell_start[c] = p.cell_count[c] + pre[c / chunk];
        if (i0 == 0) p.cell_start[p.ncell] = p.n;
    } else {
        for (int i = i0; i < p.n; i += stride) scatter_atom(p, i, p.cell_start[p.cell_of[i]]);
    }
}

// clear: also clears the counts for the next binning (which k_scan does
// itself).
template <typename F, class B, Permute kPermute>
__global__ void k_cellsort(B b, int force, int clear)
{
    Wg wg;
    KParams p;
    if (!b.fetch_gated(G_ATOMS, force, wg, p)) return;
    const int i0 = wg.id * blockDim.x + threadIdx.x, stride = wg.n * blockDim.x;
    for (int q = i0; q < p.n; q += stride) sort_slot<F, kPermute>(p, q);
    if (clear)
        for (int c = i0; c < p.ncell; c += stride) p.cell_count[c] = 0;
}

// Small systems (at most kSortSmall atoms): the scan, the scatter and the
// in-cell sort by one workgroup, one launch instead of three (their
// barriers order the global writes of one phase before the reads of the
// next inside the workgroup).  kFinish (cells-only steps, which rebuild
// every step): the workgroup first finishes the integration pass before it
// (finish_step), in place of k_int_finish.
template <typename F, class B, Permute kPermute, bool kFinish>
__global__ __launch_bounds__(kScanThreads) void k_sort_small(B b, int force, int phase,
                                                             int record_every, int fused)
{
    Wg wg;
    KParams p;
    if (!b.fetch(G_ONE, wg, p)) return;
    if (kFinish) {
        __shared__ double red[(kScanThreads / kWave) * 5];
        finish_step(p, phase, record_every, fused != 0, red);
        __syncthreads();
    } else if (!rebuild_on(p, force)) {
        return;
    }
    __shared__ int wsum[kScanThreads / kWave];
    scan_cells(p, wsum);
    __syncthreads();
    for (int i = threadIdx.x; i < p.n; i += blockDim.x)
        scatter_atom(p, i, p.cell_start[p.cell_of[i]]);
    __syncthreads();
    for (int q = threadIdx.x; q < p.n; q += blockDim.x) sort_slot<F, kPermute>(p, q);
}

// The whole cell build of a small system by one workgroup, its tables in LDS:
// the cell starts (ncell + 1), and per slot-order position q the atom with its
// cell (atom | cell << kSortAtomBits) and its id (2 n), so that global memory is
// read only for the atoms' positions (or the binning of the integration pass,
// in cells-only steps) and ids and the data that are permuted.  One launch in
// place of five (the finish, k_bin, k_scan, k_scatter, k_cellsort): a step that
// does not rebuild pays for one idle workgroup, and a rebuild is one chain of
// barriers.  Bound by that workgroup's round trips to memory, so the loads of
// four atoms per thread are issued together.  Same results as the separate
// kernels.  List steps of 500 WCA atoms 32 -> 15.6 us, of 10 007 LJ atoms
// 28.7 -> 23.8 us (a rebuild of the latter takes 41 us here, 27 us over the
// whole chip, but an idle step 2.2 us in place of five launches).
constexpr int kSortAtomBits = 14;  // atoms of a small system: at most kSortSmall = 2^14

struct SmallCells {
    int finish;        // 0 none; 1 / 2: first finish the integration pass / the fused force pass
    int phase, record_every;
    int force;         // build whatever the rebuild flag says
};

// kBin: bin the atoms here (else the integration pass has).
template <bool kPermute, bool kBin>
__global__ __launch_bounds__(kScanThreads) void k_cells_lds(Single b, SmallCells a)
{
    const KParams& p = b.p;
    constexpr int T = kScanThreads, U = 4;
    if (a.finish) {
        __shared__ double red[(T / kWave) * 5];
        if (!finish_step(p, a.phase, a.record_every, a.finish == 2, red) && !a.force) return;
    } else if (!rebuild_on(p, a.force)) {
        return;
    }
    extern __shared__ int lds[];
    int* cs = lds;                      // [ncell + 1]
    int* slot_ac = cs + p.ncell + 1;    // [n] atom | cell << kSortAtomBits
    int* slot_id = slot_ac + p.n;       // [n]
    __shared__ int wsum[T / kWave];
    const int tid = threadIdx.x;
    if (kBin) {
        // fold, cell and arrival rank (see k_bin), the rank by LDS atomics: kept
        // as cell | rank in slot_ac and slot_id of the atom's own index until the
        // cell starts are known
        for (int c = tid; c <= p.ncell; c += T) cs[c] = 0;
        __syncthreads();
        for (int i0 = tid; i0 < p.n; i0 += U * T) {
            double x[U], y[U], z[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * T;
                if (i < p.n) {
                    x[u] = p.x[i];
                    y[u] = p.y[i];
                    z[u] = p.z[i];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * T;
                if (i < p.n) {
                    x[u] = wrap(x[u], p.L);
                    y[u] = wrap(y[u], p.L);
                    z[u] = wrap(z[u], p.L);
                    p.x[i] = x[u];
                    p.y[i] = y[u];
                    p.z[i] = z[u];
                    const int c = cell_of_pos(x[u], y[u], z[u], p);
                    p.cell_of[i] = c;
                    slot_ac[i] = c;
                    slot_id[i] = atomicAdd(&cs[c], 1);
                }
            }
        }
        __syncthreads();
        // exclusive scan of the counts in place, four cells per thread at a time
        int carry = 0, m = 0;
        for (int c0 = 0; c0 < p.ncell; c0 += T * kScanPer) {
            const int c = c0 + tid * kScanPer;
            int v[kScanPer], sum = 0;
#pragma unroll
            for (int k = 0; k < kScanPer; ++k) {
                v[k] = c + k < p.ncell ? cs[c + k] : 0;
                sum += v[k];
                m = v[k] > m ? v[k] : m;
            }
            int total;
            int ex = carry + workgroup_scan_excl(sum, wsum, total);
#pragma unroll
            for (int k = 0; k < kScanPer; ++k) {
                if (c + k < p.ncell) {
                    cs[c + k] = ex;
                    p.cell_start[c + k] = ex;
                }
                ex += v[k];
            }
            carry += total;
        }
        const int occ = workgroup_max(m);
        if (tid == 0) {
            cs[p.ncell] = carry;
            p.cell_start[p.ncell] = carry;
            p.dev->max_occ = occ;
            p.dev->max_nl = 0;
        }
        __syncthreads();
        // every atom to its slot: read all of a thread's entries before any is
        // overwritten
        constexpr int kPer = kSortSmall / T;
        int q[kPer], cc[kPer], key[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + u * T;
            if (i < p.n) {
                cc[u] = slot_ac[i];
                q[u] = cs[cc[u]] + slot_id[i];
                key[u] = p.id[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + u * T;
            if (i < p.n) {
                slot_ac[q[u]] = i | (cc[u] << kSortAtomBits);
                slot_id[q[u]] = key[u];
            }
        }
    } else {
        scan_cells(p, wsum, cs);
        __syncthreads();
        for (int i0 = tid; i0 < p.n; i0 += U * T) {
            int c[U], sl[U], key[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * T;
                if (i < p.n) {
                    c[u] = p.cell_of[i];
                    sl[u] = p.slot[i];
                    key[u] = p.id[i];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * T;
                if (i < p.n) {
                    const int q = cs[c[u]] + sl[u];
                    slot_ac[q] = i | (c[u] << kSortAtomBits);
                    slot_id[q] = key[u];
                }
            }
        }
    }
    __syncthreads();
    for (int q0 = tid; q0 < p.n; q0 += U * T) {
        int d[U], src[U], key[U], cell[U];
        double v[U][6];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * T;
            if (q < p.n) {
                const int ac = slot_ac[q];
                src[u] = ac & ((1 << kSortAtomBits) - 1);
                cell[u] = ac >> kSortAtomBits;
                if (kPermute) {
                    v[u][0] = p.x[src[u]];
                    v[u][1] = p.y[src[u]];
                    v[u][2] = p.z[src[u]];
                    v[u][3] = p.vx[src[u]];
                    v[u][4] = p.vy[src[u]];
                    v[u][5] = p.vz[src[u]];
                }
                const int first = cs[cell[u]], cnt = cs[cell[u] + 1] - first;
                key[u] = slot_id[q];
                int rank = 0;
                for (int j = 0; j < cnt; ++j) rank += slot_id[first + j] < key[u] ? 1 : 0;
                d[u] = first + rank;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (q0 + u * T < p.n) {
                p.order[d[u]] = src[u];
                if (kPermute) {
                    p.sx[d[u]] = v[u][0];
                    p.sy[d[u]] = v[u][1];
                    p.sz[d[u]] = v[u][2];
                    p.svx[d[u]] = v[u][3];
                    p.svy[d[u]] = v[u][4];
                    p.svz[d[u]] = v[u][5];
                    p.sid[d[u]] = key[u];
                    if (p.bonded_on) bond_slot(p, key[u], d[u]);
                    p.scell[d[u]] = cell[u];
                }
            }
        }
    }
}

// LDS bytes of k_cells_lds for p, or 0 when the system is not small, a cell
// index does not fit beside the atom, or its tables do not fit (144 KiB of the
// CU's 160).
static size_t cells_lds_bytes(const KParams& p)
{
    if (p.pipeline != MD_PIPE_TILED || p.n > kSortSmall || p.ncell >= (1 << (31 - kSortAtomBits)))
        return 0;
    const size_t b = sizeof(int) * ((size_t)p.ncell + 1 + 2 * (size_t)p.n);
    return b <= 144 * 1024 ? b : 0;
}

// The largest system whose cells one workgroup builds, or the chain of kernels over
// the whole chip beyond it.  Where most calls find nothing to do: kSortSmall.  Where
// every call builds, the line of equal times: forced builds (md_build_cells) in one
// workgroup and by the chain, 4000 LJ atoms 10.8 and 12.3 us, 5000 13.6 and 13.4, 7000
// 16.8 and 13.6, 14 000 28 and 13, 6000 WCA 12.2 and 12.4; cells-only steps, 8000 LJ
// 35.0 and 35.0, 10 007 39.8 and 37.4, 12 000 WCA 22.1 and 22.6, 16 384 42 and 25; with
// reorder, whose permutation one CU moves, 3000 WCA 16.2 and 17.5, 4000 17.6 and 17.6,
// 8000 27.0 and 20.3.
static int one_workgroup_max(const KParams& p, int flags)
{
    if (flags & 1) return 5 * kScanThreads;
    if (flags & kFoldBin) {
        if (p.reorder) return 4096;
        return p.n >= 8ll * p.ncell ? 8192 : 12288;
    }
    return kSortSmall;
}

// Whether k_cells_lds builds the cells of a call with these flags (with reorder it
// leaves the copy-back to a later pass).
static bool in_one_workgroup(const KParams& p, int flags)
{
    return cells_lds_bytes(p) && p.n <= one_workgroup_max(p, flags) &&
           (!p.reorder || (flags & kFoldCopy));
}

static void cells_lds(const KParams& p, const SmallCells& a, bool bin, hipStream_t s)
{
    const dim3 one(1), t(kScanThreads);
    const size_t lds = cells_lds_bytes(p);
    const Single b{p};
    if (p.reorder && bin)
        hipLaunchKernelGGL((k_cells_lds<true, true>), one, t, lds, s, b, a);
    else if (p.reorder)
        hipLaunchKernelGGL((k_cells_lds<true, false>), one, t, lds, s, b, a);
    else if (bin)
        hipLaunchKernelGGL((k_cells_lds<false, true>), one, t, lds, s, b, a);
    else
        hipLaunchKernelGGL((k_cells_lds<false, false>), one, t, lds, s, b, a);
}

template <typename F, class B>
__global__ void k_copyback(B b, int force)
{
    Wg wg;
    KParams p;
    if (!b.fetch_gated(G_ATOMS, force, wg, p)) return;
    for (int q = wg.id * blockDim.x + threadIdx.x; q < p.n; q += wg.n * blockDim.x) {
        const double x = p.sx[q], y = p.sy[q], z = p.sz[q];
        const double vx = p.svx[q], vy = p.svy[q], vz = p.svz[q];
        const F fx = reinterpret_cast<const F*>(p.sfx)[q];
        const F fy = reinterpret_cast<const F*>(p.sfy)[q];
        const F fz = reinterpret_cast<const F*>(p.sfz)[q];
        const int id = p.sid[q], c = p.scell[q];
        p.x[q] = x;
        p.y[q] = y;
        p.z[q] = z;
        p.vx[q] = vx;
        p.vy[q] = vy;
        p.vz[q] = vz;
        static_cast<F*>(p.fx)[q] = fx;
        static_cast<F*>(p.fy)[q] = fy;
        static_cast<F*>(p.fz)[q] = fz;
        p.id[q] = id;
        p.cell_of[q] = c;
        p.order[q] = q;
    }
}

template <class B>
static void clear_seq(const B& b, const LaunchShape& sh, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear<B>, dim3(sh.grid[G_ATOMS]), dim3(sh.block), 0, s, b);
}

template <class B>
static void cells_seq(const B& b, const LaunchShape& sh, int flags, hipStream_t s, int n_small)
{
    const int force = flags & 1;
    const bool copy = !(flags & kFoldCopy);  // else the list or force pass copies back
    const dim3 atoms(sh.grid[G_ATOMS]), blk(sh.block);
    if (!(flags & (kFoldBin | kBinDone))) hipLaunchKernelGGL(k_bin<B>, atoms, blk, 0, s, b, force);
    if (n_small) {  // one system of at most kSortSmall atoms
        const dim3 one(1), t(kScanThreads);
        if (!sh.reorder)
            hipLaunchKernelGGL((k_sort_small<double, B, P_NONE, false>), one, t, 0, s, b, force,
                               0, 0, 0);
        else if (!copy)
            hipLaunchKernelGGL((k_sort_small<double, B, P_STATE, false>), one, t, 0, s, b, force,
                               0, 0, 0);
        else if (sh.precision == MD_FP64)
            hipLaunchKernelGGL((k_sort_small<double, B, P_ALL, false>), one, t, 0, s, b, force, 0,
                               0, 0);
        else
            hipLaunchKernelGGL((k_sort_small<float, B, P_ALL, false>), one, t, 0, s, b, force, 0,
                               0, 0);
    } else {
        bool part = false;
        if constexpr (std::is_same_v<B, Single>) {
            // more cells than one round of the one-workgroup scan (fewer would
            // only add chunk_starts to it)
            part = scan_chunks(b.p) > 1;
            if (part) {
                hipLaunchKernelGGL(k_scan_part, dim3(scan_chunks(b.p)), dim3(kScanThreads), 0, s,
                                   b, force);
                hipLaunchKernelGGL((k_scatter<B, true>), atoms, blk, 0, s, b, force);
            }
        }
        const int clear = part ? 1 : 0;
        if (!part) {
            hipLaunchKernelGGL(k_scan<B>, dim3(sh.grid[G_ONE]), dim3(kScanThreads), 0, s, b,
                               force);
            hipLaunchKernelGGL((k_scatter<B, false>), atoms, blk, 0, s, b, force);
        }
        if (!sh.reorder)
            hipLaunchKernelGGL((k_cellsort<double, B, P_NONE>), atoms, blk, 0, s, b, force,
                               clear);
        else if (!copy)
            hipLaunchKernelGGL((k_cellsort<double, B, P_STATE>), atoms, blk, 0, s, b, force,
                               clear);
        else if (sh.precision == MD_FP64)
            hipLaunchKernelGGL((k_cellsort<double, B, P_ALL>), atoms, blk, 0, s, b, force,
                               clear);
        else
            hipLaunchKernelGGL((k_cellsort<float, B, P_ALL>), atoms, blk, 0, s, b, force,
                               clear);
    }
    if (sh.reorder && copy) {
        if (sh.precision == MD_FP64)
            hipLaunchKernelGGL((k_copyback<double, B>), atoms, blk, 0, s, b, force);
        else
            hipLaunchKernelGGL((k_copyback<float, B>), atoms, blk, 0, s, b, force);
    }
}

void launch_clear(const KParams& p, hipStream_t s) { clear_seq(Single{p}, shape_of(p), s); }

void launch_cells(const KParams& p, int flags, hipStream_t s)
{
    if (in_one_workgroup(p, flags)) {
        cells_lds(p, SmallCells{0, 0, 0, flags & 1}, !(flags & kFoldBin), s);
        return;
    }
    const bool small = (flags & kSortSmallOk) && p.n <= one_workgroup_max(p, flags);
    cells_seq(Single{p}, shape_of(p), flags, s, small ? p.n : 0);
}

// The cell offsets from the occupancy counts alone (forced), for the layer
// pipeline's reorder.
void launch_cell_scan(const KParams& p, hipStream_t s)
{
    hipLaunchKernelGGL(k_scan<Single>, dim3(1), dim3(kScanThreads), 0, s, Single{p}, 1);
}

bool finish_bins(const KParams& p, int flags)
{
    return p.mode == MD_NEIGHBOR_LIST && !in_one_workgroup(p, flags);
}

void launch_finish_cells(const KParams& p, int flags, int phase, int record_every, bool fused,
                         hipStream_t s)
{
    if (in_one_workgroup(p, flags)) {
        cells_lds(p, SmallCells{fused ? 2 : 1, phase, record_every, flags & 1},
                  !(flags & kFoldBin), s);
        return;
    }
    if ((flags & kFoldBin) && (flags & kSortSmallOk) && p.n <= one_workgroup_max(p, flags)) {
        const dim3 one(1), t(kScanThreads);
        const Single b{p};
        if (p.reorder)
            hipLaunchKernelGGL((k_sort_small<double, Single, P_STATE, true>), one, t, 0, s, b, 1,
                               phase, record_every, fused ? 1 : 0);
        else
            hipLaunchKernelGGL((k_sort_small<double, Single, P_NONE, true>), one, t, 0, s, b, 1,
                               phase, record_every, fused ? 1 : 0);
        return;
    }
    if (phase == 1 && finish_bins(p, flags)) {
        const int t = p.block > kFinishThreads ? p.block : kFinishThreads;
        hipLaunchKernelGGL(k_bin_finish, dim3(grid_of(p, G_ATOMS)), dim3(t), 0, s, Single{p},
                           record_every, fused ? 1 : 0);
        launch_cells(p, flags | kBinDone, s);
        return;
    }
    launch_integrate_finish(p, phase, record_every, s, fused);
    launch_cells(p, flags, s);
}

void launch_clear(const Batch& b, const LaunchShape& sh, hipStream_t s) { clear_seq(b, sh, s); }

void launch_cells(const Batch& b, const LaunchShape& sh, int force, hipStream_t s)
{
    cells_seq(b, sh, force, s, 0);
}

}  // namespace md
