// md_forces.hip -- step F1 of section 2.3 (and the per-workgroup part of F2).
//
// Neighbor-list mode: one workgroup per tile (md_tiles.h).  After the
// tile's cell tables are known, one round of loads brings the tile's 27-cell
// neighborhoods into LDS; `lanes` lanes per home atom then walk the atom's
// list straight from the neighbor matrix (lane s takes chunks s, s+lanes,
// ...; a chunk is 4 entries, and each lane loads its next chunk before it
// works on the current one), gather the partners from LDS and accumulate the
// force on the home atom alone.  Every pair is met twice,
// once from each side, so no atomics are needed (the paper's choice).
// Pairs at r^2 >= r_cut^2 are skipped.  Separations take the minimum image
// from the wrap bits carried by each entry (section 4.1, factor (4)); tiles
// with no periodic wrap skip even that.
//
// With a half list (Newton's third law, the optional atomic variant the
// paper sets aside in section 2.3) every pair is met once, from the atom
// earlier in cell order; the partner's reaction force is added with LDS
// atomics into a per-staged-atom accumulator beside the staged positions,
// the home atom's own total goes there too, and at the end of the tile every
// accumulator that was touched is added into the force arrays with global
// atomics (which were cleared before the pass).  Tiles whose atoms do not
// fit in LDS add straight into the force arrays.  The order of the atomic
// adds is not fixed, so the forces are reproducible to rounding only.
//
// Cells-only mode: kCellLanes lanes per atom, a surrounding cell each.
//
// Precision: FP64 forms everything in double.  FP32-mixed forms the pair
// separation and the cutoff test in double, then the pair force, energy and
// virial and the per-atom sums in float.
//
// The energy and virial are reduced per workgroup (wave64 shuffles, then
// LDS) and written as partials for the reduction kernels.
#include <type_traits>

#include "md_pair.h"
#include "md_tiles.h"

namespace md {

// Pair operation of the force pass: the pair force, energy and virial of
// partners inside the cutoff.
template <typename Acc>
struct ForceOp {
    const KParams& p;
    Acc& a;
    __device__ __forceinline__ void operator()(double dx, double dy, double dz, double r2, int,
                                               int)
    {
        if (r2 < p.rc2) pair_acc(p, dx, dy, dz, r2, a);
    }
};

// Pair operation of the third-law pass: as ForceOp, and the reaction
// -F into the partner's LDS accumulator (staged index e), or straight into
// the force arrays at slot j when the tile is not staged.
template <typename F, typename Acc>
struct HalfOp {
    const KParams& p;
    Acc& a;
    MD_LDS F* r;  // [cap][3] reaction accumulators
    __device__ __forceinline__ void operator()(double dx, double dy, double dz, double r2, int e,
                                               int j)
    {
        if (r2 >= p.rc2) return;
        F g[3];
        pair_acc(p, dx, dy, dz, r2, a, g);
        if (j < 0) {
            lds_add(r + 3 * e, -g[0]);
            lds_add(r + 3 * e + 1, -g[1]);
            lds_add(r + 3 * e + 2, -g[2]);
        } else {
            global_add(static_cast<F*>(p.fx) + j, -g[0]);
            global_add(static_cast<F*>(p.fy) + j, -g[1]);
            global_add(static_cast<F*>(p.fz) + j, -g[2]);
        }
    }
};

template <typename F, typename Acc, int LANES, class B>
__global__ void k_forces_half(B b)
{
    Wg wg;
    KParams p;
    if (!b.fetch(G_TILES, wg, p)) return;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ double red[(1024 / kWave) * 2];
    const Tile g = tile_of(p, xcd_tile(wg.id, wg.n));
    Stage s = stage_layout(p, smem, p.scap_aux, true);
    stage_tables(p, g, s);
    const int nh = home_count(s);
    const int mode = staged_image_mode(p, s, tile_interior(p, g));
    stage_positions_imaged(p, s);
    // the accumulators, in the aux region (F-typed, interleaved)
    MD_LDS F* r = reinterpret_cast<MD_LDS F*>(s.a3);
    if (s.fits) {
        for (int k = threadIdx.x; k < 3 * s.total; k += blockDim.x) r[k] = F(0);
    }
    __syncthreads();
    const int per_pass = blockDim.x / LANES;
    const int sub = threadIdx.x % LANES;
    double e[2] = {0.0, 0.0};
    for (int hb = 0; hb < nh; hb += per_pass) {
        const int h = hb + threadIdx.x / LANES;
        Acc a;
        int slot_i = 0, eh = 0;
        if (h < nh) {
            int pos;
            home_atom(s, h, eh, pos);
            slot_i = atom_at(p, pos);
            double xi, yi, zi;
            home_position(p, s, eh, slot_i, xi, yi, zi);
            HalfOp<F, Acc> op{p, a, r};
            walk_home<LANES>(p, s, mode, slot_i, sub, p.nl_count[slot_i], xi, yi, zi, op);
        }
        if (LANES > 1) {
            a.fx = lane_group_sum<LANES>(a.fx);
            a.fy = lane_group_sum<LANES>(a.fy);
            a.fz = lane_group_sum<LANES>(a.fz);
            a.u = lane_group_sum<LANES>(a.u);
            a.w = lane_group_sum<LANES>(a.w);
        }
        if (h < nh && sub == 0) {
            if (s.fits) {
                lds_add(r + 3 * eh, a.fx);
                lds_add(r + 3 * eh + 1, a.fy);
                lds_add(r + 3 * eh + 2, a.fz);
            } else {
                global_add(static_cast<F*>(p.fx) + slot_i, a.fx);
                global_add(static_cast<F*>(p.fy) + slot_i, a.fy);
                global_add(static_cast<F*>(p.fz) + slot_i, a.fz);
            }
            // each pair once: its whole energy 4 eps (sr12 - sr6) - shift, and virial
            const double ui = 2.0 * p.eps2 * (double)a.u;
            e[0] += ui;
            e[1] += (double)a.w;
            if (!isfinite(ui + (double)a.fx + (double)a.fy + (double)a.fz))
                atomicOr(&p.dev->flags, (int)MD_FLAG_NONFINITE);
        }
    }
    __syncthreads();
    if (s.fits) {
        // flush every touched accumulator (home atoms always; partners in
        // the cells behind the home row in cell order never)
        for (int k = threadIdx.x; k < s.total; k += blockDim.x) {
            const F ax = r[3 * k], ay = r[3 * k + 1], az = r[3 * k + 2];
            if (ax != F(0) || ay != F(0) || az != F(0)) {
                const int j = staged_slot(p, s, k);
                global_add(static_cast<F*>(p.fx) + j, ax);
                global_add(static_cast<F*>(p.fy) + j, ay);
                global_add(static_cast<F*>(p.fz) + j, az);
            }
        }
    }
    block_sum<2>(e, red);
    if (threadIdx.x == 0) {
        p.fpart[2 * wg.id] = e[0];
        p.fpart[2 * wg.id + 1] = e[1];
    }
}

// Clears the force arrays before a third-law pass.
template <typename F, class B>
__global__ void k_zero_forces(B b)
{
    Wg wg;
    KParams p;
    if (!b.fetch(G_ATOMS, wg, p)) return;
    for (int i = wg.id * blockDim.x + threadIdx.x; i < p.n; i += wg.n * blockDim.x) {
        static_cast<F*>(p.fx)[i] = F(0);
        static_cast<F*>(p.fy)[i] = F(0);
        static_cast<F*>(p.fz)[i] = F(0);
    }
}

// What a force pass does with each home atom's sums, and what it sums over
// the atoms.  kStep: the integration pass follows in the same kernel
// (launch_forces_step), else the force is written.  kEnergy: energy and virial
// too (and, with kStep, the kinetic sums of a recorded step).
template <typename F, bool kStep, bool kEnergy>
struct HomeEnd {
    using Sums = Lean<F>;
    double e[2] = {0.0, 0.0};             // U, W
    double k[4] = {0.0, 0.0, 0.0, 0.0};   // v^2, Px, Py, Pz (kStep)
    double dmax2 = 0.0;                   // largest squared displacement (kStep)

    __device__ __forceinline__ void operator()(const KParams& p, const Sums& a, int i, double xi,
                                               double yi, double zi)
    {
        F fx, fy, fz;
        double ui = 0.0, wi;
        lean_finish(p, a, fx, fy, fz, ui, wi);
        e[0] += ui;
        e[1] += wi;
        finish(p, fx, fy, fz, ui, i, xi, yi, zi);
    }
    __device__ __forceinline__ void finish(const KParams& p, F fx, F fy, F fz, double ui, int i,
                                           double xi, double yi, double zi)
    {
        if (kStep) {
            double vx = p.vx[i], vy = p.vy[i], vz = p.vz[i];
            const double rx = p.xr[i], ry = p.yr[i], rz = p.zr[i];
            const double gx = (double)fx, gy = (double)fy, gz = (double)fz;
            // second half kick of the finished step, then first half kick and
            // drift of the next, as k_integrate
            vx = kick(vx, p.hdt, gx);
            vy = kick(vy, p.hdt, gy);
            vz = kick(vz, p.hdt, gz);
            if (kEnergy) {
                k[0] += (vx * vx + vy * vy) + vz * vz;
                k[1] += vx;
                k[2] += vy;
                k[3] += vz;
            }
            vx = kick(vx, p.hdt, gx);
            vy = kick(vy, p.hdt, gy);
            vz = kick(vz, p.hdt, gz);
            const double x = drift(xi, p.dt, vx), y = drift(yi, p.dt, vy),
                         z = drift(zi, p.dt, vz);
            p.sx[i] = x;
            p.sy[i] = y;
            p.sz[i] = z;
            p.vx[i] = vx;
            p.vy[i] = vy;
            p.vz[i] = vz;
            const double d2 = dist2(minimg(x - rx, p.L, p.invL), minimg(y - ry, p.L, p.invL),
                                    minimg(z - rz, p.L, p.invL));
            dmax2 = d2 > dmax2 ? d2 : dmax2;
        } else {
            static_cast<F*>(p.fx)[i] = fx;
            static_cast<F*>(p.fy)[i] = fy;
            static_cast<F*>(p.fz)[i] = fz;
        }
        if (!isfinite(ui + (double)fx + (double)fy + (double)fz))
            atomicOr(&p.dev->flags, (int)MD_FLAG_NONFINITE);
    }
};

// Without the energies (a non-finite energy shows in the force: it needs
// sr6 (sr6 - 1/2) past the range, a factor of every force component).
template <typename F>
struct HomeEnd<F, true, false> : HomeEnd<F, true, true> {
    using Sums = LeanForce<F>;
    __device__ __forceinline__ void operator()(const KParams& p, const Sums& a, int i, double xi,
                                               double yi, double zi)
    {
        const F s = (F)p.eps48;
        this->finish(p, s * a.fx, s * a.fy, s * a.fz, 0.0, i, xi, yi, zi);
    }
};

template <int LANES, typename T>
__device__ __forceinline__ void group_sum(LeanForce<T>& a)
{
    if (LANES > 1) {
        a.fx = lane_group_sum<LANES>(a.fx);
        a.fy = lane_group_sum<LANES>(a.fy);
        a.fz = lane_group_sum<LANES>(a.fz);
    }
}

template <int LANES, typename T>
__device__ __forceinline__ void group_sum(Lean<T>& a)
{
    if (LANES > 1) {
        a.fx = lane_group_sum<LANES>(a.fx);
        a.fy = lane_group_sum<LANES>(a.fy);
        a.fz = lane_group_sum<LANES>(a.fz);
        a.q = lane_group_sum<LANES>(a.q);
        a.s6 = lane_group_sum<LANES>(a.s6);
    }
}

// A tile whose atoms fit in LDS, on a grid of at least 5 cells per side: from
// the rows in registers (md_tiles.h).  A wave's home atoms are a contiguous
// stretch; the length and the first chunk of each one's list are loaded
// before the barrier that ends the staging, with which they overlap.  Bound
// by VALU issue at dense states, by the chain of dependent loads at sparse
// ones; against the tables (four barriers, a search per staged atom) it
// measured 223 against 241 us at 2.048M LJ atoms, 16.5 against 19.2 us at
// 256 000 WCA atoms and 56 against 65 us for 64 replicas (1.03M atoms).
template <int LANES, class End>
__device__ __forceinline__ void forces_rows(const KParams& p, const Rows& t, char* smem, End& end)
{
    MD_LDS double* p3 = (MD_LDS double*)smem;
    constexpr int kPer = kWave / LANES;  // home atoms of a wave
    const int lane = threadIdx.x & (kWave - 1);
    const int w0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave) * kPer;
    const int per_pass = (int)blockDim.x / LANES;
    stage_rows<false>(p, t, p3, nullptr, nullptr, nullptr, nullptr);
    bool staged = false;
    for (int h0 = w0; h0 < t.nh || !staged; h0 += per_pass) {
        const int h = h0 + lane / LANES;
        int sub = lane % LANES;
        asm volatile("" : "+v"(sub));  // the row offset below is formed anew in each pass
        int slot_i = 0, eh = 0, cnt = 0;
        uint64_t next = 0;
        if (h0 < t.nh) {
            int ds, de, row;
            find_row<false>(t.hstart, t.d1 + t.e1 - t.hstart, t.e1 - t.hstart, h0, kPer, h, ds, de,
                            row);
            slot_i = atom_at(p, h < t.nh ? h + ds : 0);
            eh = h + de;
            if (h < t.nh) {
                cnt = p.nl_count[slot_i];
                if (sub <= p.cap / kChunk) next = p.nl64[(int64_t)sub * p.npad + slot_i];
            }
        }
        if (!staged) __syncthreads();
        staged = true;
        if (h0 >= t.nh) break;
        typename End::Sums a;
        double xi = 0.0, yi = 0.0, zi = 0.0;
        if (h < t.nh) {
            lds_xyz(p3, eh, xi, yi, zi);
            ForceOp<typename End::Sums> op{p, a};
            walk_staged<LANES>(p, p3, slot_i, sub, cnt, next, xi, yi, zi, op);
        }
        group_sum<LANES>(a);
        if (h < t.nh && sub == 0) end(p, a, slot_i, xi, yi, zi);
    }
}

// Any other tile (more than 64 staged rows, atoms past the LDS capacity, or a
// grid of fewer than 5 cells per side, whose pairs take the minimum image by
// rounding): through the cell tables in LDS.
template <int LANES, class End>
__device__ __forceinline__ void forces_tables(const KParams& p, const Tile& g, char* smem,
                                              End& end)
{
    Stage s = stage_layout(p, smem);
    stage_tables(p, g, s);
    const int nh = home_count(s);
    const int mode = staged_image_mode(p, s, tile_interior(p, g));
    stage_positions_imaged(p, s);
    __syncthreads();
    const int per_pass = blockDim.x / LANES;
    const int sub = threadIdx.x % LANES;
    for (int hb = 0; hb < nh; hb += per_pass) {
        const int h = hb + threadIdx.x / LANES;
        typename End::Sums a;
        int slot_i = 0;
        double xi = 0.0, yi = 0.0, zi = 0.0;
        if (h < nh) {
            int eh, pos;
            home_atom(s, h, eh, pos);
            slot_i = atom_at(p, pos);
            home_position(p, s, eh, slot_i, xi, yi, zi);
            ForceOp<typename End::Sums> op{p, a};
            // the lane's list-row offset is formed here for each pass: hoisted out
            // of the pass loop it is a 64-bit value live across the whole kernel
            // (the empty asm hides that sub is the same in every pass)
            int sub_p = sub;
            asm volatile("" : "+v"(sub_p));
            walk_home<LANES>(p, s, mode, slot_i, sub_p, p.nl_count[slot_i], xi, yi, zi, op);
        }
        group_sum<LANES>(a);
        if (h < nh && sub == 0) end(p, a, slot_i, xi, yi, zi);
    }
}

// One tile by whichever way it takes.
template <int LANES, class End>
__device__ __forceinline__ void forces_tile(const KParams& p, const Wg& wg, char* smem, End& end)
{
    const Tile g = tile_of(p, xcd_tile(wg.id, wg.n));
    bool rows = rows_fit(p) && p.nc >= 5;
    if (rows) {
        const Rows t = row_table(p, g);
        rows = t.total < p.scap;
        if (rows) forces_rows<LANES>(p, t, smem, end);
    }
    if (!rows) forces_tables<LANES>(p, g, smem, end);
}

// Six waves per SIMD (at most 80 VGPRs): three workgroups of the default
// shape fit a CU by LDS, and the compiler's own allocation otherwise crosses
// the five-wave line.
template <typename F, int LANES, class B>
__global__ __attribute__((amdgpu_waves_per_eu(6))) void k_forces_tiles(B b)
{
    Wg wg;
    KParams p;
    if (!b.fetch(G_TILES, wg, p)) return;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ double red[(1024 / kWave) * 2];
    HomeEnd<F, false, true> end;
    forces_tile<LANES>(p, wg, smem, end);
    block_sum<2>(end.e, red);
    if (threadIdx.x == 0) {
        p.fpart[2 * wg.id] = end.e[0];
        p.fpart[2 * wg.id + 1] = end.e[1];
    }
}

// The force pass with the integration pass that follows it (see
// launch_forces_step).  The integration alone is bound by HBM (144 B per atom)
// and the force pass by VALU issue, so together the integration's traffic,
// less the forces and the reread positions (96 B per atom), hides under the pair
// walk: 238 us against 223 + 47 us at 2.048M LJ atoms, 19.3 against 16.5 + 8.4 us
// at 256 000 WCA atoms, 69 against 56 + 25 us for 64 replicas (the latter two 18.2
// and 66.5 us with the tile shapes of tiling_cost).  Velocities and references
// loaded ahead of the walk, one triple per lane of a group, measured no gain (18.2
// -> 18.7 us, 66.5 -> 65.2, 246 -> 249 at 2.048M): the other waves hide those loads.
// Energies, virial and kinetic sums only when the history asks for the step
// (DevState::record, set by the finish before this launch); the largest
// displacement always.
template <typename F, int LANES, class B>
__global__ __attribute__((amdgpu_waves_per_eu(6))) void k_forces_step(B b)
{
    Wg wg;
    KParams p;
    if (!b.fetch(G_TILES, wg, p)) return;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ double red[(1024 / kWave) * 7];
    double dmax2;
    if (p.dev->record) {
        HomeEnd<F, true, true> end;
        forces_tile<LANES>(p, wg, smem, end);
        double v[6] = {end.e[0], end.e[1], end.k[0], end.k[1], end.k[2], end.k[3]};
        dmax2 = end.dmax2;
        block_sum_max<6>(v, dmax2, red);
        if (threadIdx.x == 0) {
            p.fpart[2 * wg.id] = v[0];
            p.fpart[2 * wg.id + 1] = v[1];
            double* const kp = step_part(p);
            for (int c = 0; c < 4; ++c) kp[c * (int64_t)p.nblk_force + wg.id] = v[2 + c];
        }
    } else {
        HomeEnd<F, true, false> end;
        forces_tile<LANES>(p, wg, smem, end);
        double v[1] = {0.0};
        dmax2 = end.dmax2;
        block_sum_max<1>(v, dmax2, red);
    }
    if (threadIdx.x == 0)
        atomicMax(&p.dev->dmax_slot[wg.id % kDmaxSlots],
                  (unsigned long long)__double_as_longlong(dmax2));
}

// ---- cells-only mode ----
//
// kCellLanes lanes per atom: lane c < 27 walks neighbor cell c of the atom's
// 27 (dz, dy, dx each -1, 0, +1, dz slowest) straight from the cell arrays,
// with the full minimum image; the lanes' sums are then added across the
// group.  At about one atom per cell a lane has one or two partners, so the
// pass is as deep as a few dependent loads rather than the 27 cells in turn.

template <typename Acc>
__device__ __forceinline__ void walk_cell(const KParams& p, int i, double xi, double yi,
                                          double zi, int c2, Acc& a)
{
    const int k1 = p.cell_start[c2 + 1];
    for (int k = p.cell_start[c2]; k < k1; ++k) {
        const int j = atom_at(p, k);
        if (j == i) continue;
        const double dx = minimg(xi - p.x[j], p.L, p.invL);
        const double dy = minimg(yi - p.y[j], p.L, p.invL);
        const double dz = minimg(zi - p.z[j], p.L, p.invL);
        const double r2 = dist2(dx, dy, dz);
        if (r2 < p.rc2) pair_acc(p, dx, dy, dz, r2, a);
    }
}

// The sums of this lane's atom i (valid where i < n), added across its group
// of kCellLanes lanes, sub the lane's place in it.
template <typename Acc>
__device__ __forceinline__ void cells_sums(const KParams& p, const Wg& wg, Acc& a, int& i,
                                           int& sub)
{
    const int64_t t = (int64_t)xcd_tile(wg.id, wg.n) * blockDim.x + threadIdx.x;
    i = (int)(t / kCellLanes);
    sub = (int)(t % kCellLanes);
    if (i < p.n && sub < 27) {
        const int c = p.cell_of[i], nc = p.nc;
        const int cx = c % nc, cy = (c / nc) % nc, cz = c / (nc * nc);
        const int dz = sub / 9 - 1, dy = (sub / 3) % 3 - 1, dx = sub % 3 - 1;
        const int c2 = (wrap_cell(cz + dz, nc) * nc + wrap_cell(cy + dy, nc)) * nc +
                       wrap_cell(cx + dx, nc);
        walk_cell(p, i, p.x[i], p.y[i], p.z[i], c2, a);
    }
    group_sum<kCellLanes>(a);
}

// kCopy (md_step with reorder): the cell build left the sorted data in the
// scratch arrays; the pass reads them there and each atom's lane 0 copies its
// atom into the state arrays, forces written straight into the state.
template <typename F, class B, bool kCopy>
__global__ void k_forces_cells(B b)
{
    Wg wg;
    KParams pw;
    if (!b.fetch(G_TILES, wg, pw)) return;
    const KParams p = kCopy ? scratch_view(pw) : pw;
    F* const fout[3] = {static_cast<F*>(pw.fx), static_cast<F*>(pw.fy),
                        static_cast<F*>(pw.fz)};
    __shared__ double red[(1024 / kWave) * 2];
    LeanOf<F> a;
    int i, sub;
    cells_sums(p, wg, a, i, sub);
    double e[2] = {0.0, 0.0};
    if (i < p.n && sub == 0) {
        F fx, fy, fz;
        lean_finish(p, a, fx, fy, fz, e[0], e[1]);
        copy_home<kCopy>(p, i);
        fout[0][i] = fx;
        fout[1][i] = fy;
        fout[2][i] = fz;
        if (!isfinite(e[0] + (double)fx + (double)fy + (double)fz))
            atomicOr(&p.dev->flags, (int)MD_FLAG_NONFINITE);
    }
    block_sum<2>(e, red);
    if (threadIdx.x == 0) {
        p.fpart[2 * wg.id] = e[0];
        p.fpart[2 * wg.id + 1] = e[1];
    }
}

// The cells-only force pass with the integration pass that follows it (kick,
// kick and drift, the new position folded and binned, as k_integrate with
// kBin): see launch_forces_step.  The new positions go where no workgroup of
// this launch reads: with kCopy the pass reads the sorted scratch arrays and
// writes the state's, without it the scratch positions.  Energies and kinetic
// sums of recorded steps only.  Bound by latency (one or two partners per lane):
// 6.0 us at 4000 WCA atoms, against 6.3 + 6.5 us for the two passes; the step
// 20.6 -> 13.6 us in two launches.
template <typename F, bool kCopy, bool kEnergy>
__device__ __forceinline__ void cells_step(const KParams& pw, const Wg& wg, double* red)
{
    const KParams p = kCopy ? scratch_view(pw) : pw;
    using Sums = std::conditional_t<kEnergy, Lean<F>, LeanForce<F>>;
    Sums a;
    int i, sub;
    cells_sums(p, wg, a, i, sub);
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (i < p.n && sub == 0) {
        double vx = p.vx[i], vy = p.vy[i], vz = p.vz[i];
        double x = p.x[i], y = p.y[i], z = p.z[i];
        F fx, fy, fz;
        if constexpr (kEnergy) {
            lean_finish(p, a, fx, fy, fz, v[0], v[1]);
        } else {
            const F k = (F)p.eps48;
            fx = k * a.fx;
            fy = k * a.fy;
            fz = k * a.fz;
        }
        const double gx = (double)fx, gy = (double)fy, gz = (double)fz;
        vx = kick(vx, p.hdt, gx);
        vy = kick(vy, p.hdt, gy);
        vz = kick(vz, p.hdt, gz);
        if (kEnergy) {
            v[2] = (vx * vx + vy * vy) + vz * vz;
            v[3] = vx;
            v[4] = vy;
            v[5] = vz;
        }
        vx = kick(vx, p.hdt, gx);
        vy = kick(vy, p.hdt, gy);
        vz = kick(vz, p.hdt, gz);
        x = wrap(drift(x, p.dt, vx), p.L);
        y = wrap(drift(y, p.dt, vy), p.L);
        z = wrap(drift(z, p.dt, vz), p.L);
        const int c = cell_of_pos(x, y, z, p);
        const int rank = atomicAdd(&pw.cell_count[c], 1);
        // (scratch_view: with kCopy p.s* are the state arrays)
        p.sx[i] = x;
        p.sy[i] = y;
        p.sz[i] = z;
        pw.vx[i] = vx;
        pw.vy[i] = vy;
        pw.vz[i] = vz;
        if (kCopy) pw.id[i] = p.id[i];
        pw.cell_of[i] = c;
        pw.slot[i] = rank;
        if (!isfinite(v[0] + gx + gy + gz)) atomicOr(&p.dev->flags, (int)MD_FLAG_NONFINITE);
    }
    if (!kEnergy) return;
    block_sum<6>(v, red);
    if (threadIdx.x == 0) {
        p.fpart[2 * wg.id] = v[0];
        p.fpart[2 * wg.id + 1] = v[1];
        double* const kp = step_part(p);
        for (int c = 0; c < 4; ++c) kp[c * (int64_t)p.nblk_force + wg.id] = v[2 + c];
    }
}

template <typename F, bool kCopy>
__global__ void k_cells_step(Single b)
{
    __shared__ double red[(1024 / kWave) * 6];
    const Wg wg{(int)blockIdx.x, (int)gridDim.x};
    if (b.p.dev->record)
        cells_step<F, kCopy, true>(b.p, wg, red);
    else
        cells_step<F, kCopy, false>(b.p, wg, red);
}

template <typename F, typename Acc, class B>
static void half_seq(const B& b, const LaunchShape& sh, hipStream_t s)
{
    hipLaunchKernelGGL((k_zero_forces<F, B>), dim3(sh.grid[G_ATOMS]), dim3(sh.block), 0, s, b);
    const dim3 g(sh.grid[G_TILES]), t(sh.force_block);
    const size_t lds = sh.force_lds;
    switch (sh.force_lanes) {
        case 8: hipLaunchKernelGGL((k_forces_half<F, Acc, 8, B>), g, t, lds, s, b); break;
        case 2: hipLaunchKernelGGL((k_forces_half<F, Acc, 2, B>), g, t, lds, s, b); break;
        case 4: hipLaunchKernelGGL((k_forces_half<F, Acc, 4, B>), g, t, lds, s, b); break;
        default: hipLaunchKernelGGL((k_forces_half<F, Acc, 1, B>), g, t, lds, s, b); break;
    }
}

template <typename F, typename Acc, class B>
static void tiles_seq(const B& b, const LaunchShape& sh, hipStream_t s)
{
    if (sh.newton3) {
        half_seq<F, Acc>(b, sh, s);
        return;
    }
    const dim3 g(sh.grid[G_TILES]), t(sh.force_block);
    const size_t lds = sh.force_lds;
    switch (sh.force_lanes) {
        case 8: hipLaunchKernelGGL((k_forces_tiles<F, 8, B>), g, t, lds, s, b); break;
        case 2: hipLaunchKernelGGL((k_forces_tiles<F, 2, B>), g, t, lds, s, b); break;
        case 4: hipLaunchKernelGGL((k_forces_tiles<F, 4, B>), g, t, lds, s, b); break;
        default: hipLaunchKernelGGL((k_forces_tiles<F, 1, B>), g, t, lds, s, b); break;
    }
}

template <typename F, class B>
static void step_seq(const B& b, const LaunchShape& sh, hipStream_t s)
{
    const dim3 g(sh.grid[G_TILES]), t(sh.force_block);
    const size_t lds = sh.force_lds;
    switch (sh.force_lanes) {
        case 8: hipLaunchKernelGGL((k_forces_step<F, 8, B>), g, t, lds, s, b); break;
        case 2: hipLaunchKernelGGL((k_forces_step<F, 2, B>), g, t, lds, s, b); break;
        case 4: hipLaunchKernelGGL((k_forces_step<F, 4, B>), g, t, lds, s, b); break;
        default: hipLaunchKernelGGL((k_forces_step<F, 1, B>), g, t, lds, s, b); break;
    }
}

template <class B>
static void forces_seq(const B& b, const LaunchShape& sh, hipStream_t s, int flags = 0)
{
    if (sh.mode == MD_CELLS_ONLY) {
        const dim3 g(sh.grid[G_TILES]), t(sh.block);
        const bool copy = (flags & kFoldCopy) && sh.reorder;
        if (sh.precision == MD_FP64 && copy)
            hipLaunchKernelGGL((k_forces_cells<double, B, true>), g, t, 0, s, b);
        else if (sh.precision == MD_FP64)
            hipLaunchKernelGGL((k_forces_cells<double, B, false>), g, t, 0, s, b);
        else if (copy)
            hipLaunchKernelGGL((k_forces_cells<float, B, true>), g, t, 0, s, b);
        else
            hipLaunchKernelGGL((k_forces_cells<float, B, false>), g, t, 0, s, b);
        return;
    }
    if (sh.precision == MD_FP64)
        tiles_seq<double, AccD>(b, sh, s);
    else
        tiles_seq<float, AccF>(b, sh, s);
}

int force_blocks(const KParams& p) { return grid_of(p, G_TILES); }

size_t force_lds_bytes(const KParams& p)
{
    if (p.mode != MD_NEIGHBOR_LIST) return 0;
    return p.newton3 ? stage_bytes(p, p.scap_aux, true) : stage_bytes(p, p.scap);
}

LaunchShape shape_of(const KParams& p)
{
    LaunchShape sh;
    for (int k = 0; k < G_KINDS; ++k) sh.grid[k] = grid_of(p, (GridKind)k);
    sh.block = p.block;
    sh.force_block = p.force_block;
    sh.force_lanes = p.force_lanes;
    sh.nl_block = p.nl_block;
    sh.nl_method = p.nl_method;
    sh.nl_queue = p.nl_queue;
    sh.nl_lds = p.mode == MD_NEIGHBOR_LIST ? nl_lds_bytes(p) : 0;
    sh.force_lds = force_lds_bytes(p);
    sh.precision = p.precision;
    sh.reorder = p.reorder;
    sh.mode = p.mode;
    sh.newton3 = p.newton3;
    sh.nl_full = p.nc < 5 || !nl_small(p);
    return sh;
}

void launch_forces(const KParams& p, hipStream_t s, int flags)
{
    forces_seq(Single{p}, shape_of(p), s, flags);
}

void launch_forces(const Batch& b, const LaunchShape& sh, hipStream_t s) { forces_seq(b, sh, s); }

void launch_forces_step(const KParams& p, hipStream_t s)
{
    const Single b{p};
    if (p.mode == MD_CELLS_ONLY) {
        const dim3 g(grid_of(p, G_TILES)), t(p.block);
        if (p.precision == MD_FP64 && p.reorder)
            hipLaunchKernelGGL((k_cells_step<double, true>), g, t, 0, s, b);
        else if (p.precision == MD_FP64)
            hipLaunchKernelGGL((k_cells_step<double, false>), g, t, 0, s, b);
        else if (p.reorder)
            hipLaunchKernelGGL((k_cells_step<float, true>), g, t, 0, s, b);
        else
            hipLaunchKernelGGL((k_cells_step<float, false>), g, t, 0, s, b);
        return;
    }
    if (p.precision == MD_FP64)
        step_seq<double>(b, shape_of(p), s);
    else
        step_seq<float>(b, shape_of(p), s);
}

void launch_forces_step(const Batch& b, const LaunchShape& sh, hipStream_t s)
{
    if (sh.precision == MD_FP64)
        step_seq<double>(b, sh, s);
    else
        step_seq<float>(b, sh, s);
}

}  // namespace md
