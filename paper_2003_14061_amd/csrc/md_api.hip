// md_api.hip -- the C ABI of libmd (declared in include/md.h).
//
// Host side only: validation, derived geometry, workspace layout, the
// kernel-parameter block and the order of launches.  All arithmetic on atoms
// happens in the kernels of the other translation units.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <initializer_list>
#include <mutex>
#include <new>
#include <vector>

#include "md_internal.h"
#include "md_tiles.h"

using namespace md;

#include "md_ctx.h"

using md::align_up;
using md::kAlign;

extern "C" const char* md_status_str(int32_t st)
{
    switch (st) {
        case MD_OK: return "ok";
        case MD_ERR_ARG: return "invalid argument";
        case MD_ERR_BOX_TOO_SMALL: return "box too small: fewer than 3 cells per side";
        case MD_ERR_NL_OVERFLOW: return "neighbor list overflow: raise nl_capacity";
        case MD_ERR_NONFINITE: return "non-finite force or energy";
        case MD_ERR_HIP: return "HIP runtime error";
        case MD_ERR_NOT_BOUND: return "buffers not bound (call md_bind)";
        case MD_ERR_STATE: return "call out of order";
        case MD_ERR_LAYER_OVERFLOW: return "layer matrix overflow: a cell held more atoms than layers";
        case MD_ERR_BOND_BROKEN: return "a bond reached the FENE limit R0";
        case MD_ERR_TOPOLOGY: return "atom ids are not a permutation of 0..N-1 (chains undefined)";
        case MD_ERR_WORKSPACE_TOO_LARGE:
            return "workspace larger than the library's static array (md_bind_static)";
        default: return "unknown status";
    }
}

// What a force pass over `tiles` tiles of `home` and `staged` atoms costs, in units
// of a home atom's share of a busy CU.  Such a CU takes a tile's home atoms, a
// quarter of its staged ones and 60 for the rest of a workgroup; alone a workgroup
// takes as long as its passes over the home atoms (the count spreads by less than
// 0.55 sqrt(home), a third of a Poisson variance) and a quarter of the staged
// atoms.  All CUs take tiles in rounds of three workgroups of the default 512
// threads (six waves per SIMD); the last round counts by its fullest CU, unless
// the tiles share the machine with other systems'.
static double tiling_cost(const KParams& k, int64_t tiles, double home, double staged, bool alone)
{
    const int per_cu = k.force_block < 24 * kWave ? 24 * kWave / k.force_block : 1;
    const double pass = (double)k.force_block / k.force_lanes;
    const double work = home + 0.25 * staged + 60.0;
    const double chain =
        pass * ceil((home + 2.0 * sqrt(0.3 * home)) / pass) + 0.25 * staged;
    const double round = hypot(chain, per_cu * work);
    const int64_t slots = 256 * per_cu;
    if (!alone) return (double)tiles / slots * round;
    const int64_t rest = tiles % slots;
    return (double)(tiles / slots) * round +
           (rest > 0 ? hypot(chain, (double)((rest + 255) / 256) * work) : 0.0);
}

// Tiling of the neighbor-list mode: the grid is cut into near-equal blocks of
// about kx x ky x kz cells, kx >= ky >= kz (a requested size of 0 is chosen
// here).  The choice minimizes tiling_cost among blocks whose expected staged
// atoms (1.15x the mean plus 64) fit the LDS share that lets three force
// workgroups share a CU, and whose expected home atoms fill at most three passes
// of the force workgroup (ties: the longer block along x, whose slot runs are
// longer).  The rule before it, the fewest staged cells per home cell of at least
// 256 tiles, left the last round of workgroups nearly empty at many sizes.  Steps
// of both, list build included: 32 000 LJ atoms FP32 33.1 us at 3 x 2 x 1 cells (264
// tiles), 29.4 at 2 x 2 x 2 (216); 70 000 LJ 37.0 and 33.6 (320 and 512 tiles);
// 700 000 WCA 76.7 and 65.6 (1156 and 1445); over 27 sizes of both from 500 to 2.048M
// atoms it picks a shape within 0.9% of the best one measured, on average, and
// never a slower one than before by more than the runs differ.
static void plan_shape(md_ctx* c)
{
    KParams& k = c->kp;
    const int nc = k.nc;
    const double occ = (double)k.n / ((double)nc * nc * nc);
    const double lds_share = 160.0 * 1024.0 / 3.0 - 2048.0;  // bytes, three per CU
    const double home_max = 3.0 * k.force_block / k.force_lanes;
    auto maxsize = [nc](int req) {
        const int parts = (nc + req - 1) / req;
        return (nc + parts - 1) / parts;
    };
    const auto request = [](int req, int most) { return req < most ? req : most; };
    const int rows = nc < kHomeRows ? nc : kHomeRows;
    const int req_x = request(c->tile_cells, nc), req_y = request(c->tile_y, rows);
    const int req_z = request(c->tile_z, req_y > 0 && rows > kHomeRows / maxsize(req_y)
                                             ? kHomeRows / maxsize(req_y)
                                             : rows);
    int best[3] = {1, 1, 1};
    double best_score = 1e300;
    const int kx_hi = nc < 64 ? nc : 64, kyz_hi = nc < 4 ? nc : 4;
    for (int kz = 1; kz <= kyz_hi; ++kz)
        for (int ky = kz; ky <= kyz_hi; ++ky)
            for (int kx = ky; kx <= kx_hi; ++kx) {
                const int ax = req_x > 0 ? req_x : kx;
                const int ay = req_y > 0 ? req_y : ky;
                const int az = req_z > 0 ? req_z : kz;
                const int mx = maxsize(ax), my = maxsize(ay), mz = maxsize(az);
                if (my * mz > kHomeRows) continue;  // (one row of the other axis never is)
                const double cells = (double)(mx + 2) * (my + 2) * (mz + 2);
                const double staged = cells * occ;
                const double home = (double)mx * my * mz * occ;
                const int64_t tiles = (int64_t)((nc + ax - 1) / ax) * ((nc + ay - 1) / ay) *
                                      ((nc + az - 1) / az);
                const bool ok = (1.15 * staged + 64.0) * 3.0 * sizeof(double) <= lds_share &&
                                home <= home_max;
                // a block that breaks the limits is taken only while nothing fits,
                // the fewest staged cells first
                const double score =
                    ok ? tiling_cost(k, tiles, home, staged, c->alone) : 1e200 * cells;
                if (score < best_score * (1.0 - 1e-9) ||
                    (score <= best_score * (1.0 + 1e-9) && mx > best[0])) {
                    best_score = score;
                    best[0] = ax;
                    best[1] = ay;
                    best[2] = az;
                }
            }
    k.tiles_x = (nc + best[0] - 1) / best[0];
    k.tiles_y = (nc + best[1] - 1) / best[1];
    k.tiles_z = (nc + best[2] - 1) / best[2];
    k.kx_max = (nc + k.tiles_x - 1) / k.tiles_x;
    k.ky_max = (nc + k.tiles_y - 1) / k.tiles_y;
    k.kz_max = (nc + k.tiles_z - 1) / k.tiles_z;
    k.n_tiles = k.tiles_x * k.tiles_y * k.tiles_z;
    c->tile_cells_res = k.kx_max;
    c->tile_y_res = k.ky_max;
    c->tile_z_res = k.kz_max;
}

// The tiles' shape (keep: the one there is) and what follows from it.  The LDS
// capacity allows 1.15x the mean staged count plus 64 of the largest block; a tile
// that does not fit takes its partners from global memory.
static void plan_tiles(md_ctx* c, bool keep = false)
{
    if (!keep) plan_shape(c);
    c->replan = keep;
    KParams& k = c->kp;
    const double occ = (double)k.n / ((double)k.nc * k.nc * k.nc);
    const double s_mean = (double)(k.kx_max + 2) * (k.ky_max + 2) * (k.kz_max + 2) * occ;
    // tables and static LDS
    const size_t tables = stage_bytes(k, 0) + 2048;
    const size_t room = c->lds_limit > tables ? c->lds_limit - tables : 0;
    int scap = c->stage_cap > 0 ? c->stage_cap : (int)(1.15 * s_mean + 64.0);
    const int scap_max = (int)(room / (3 * sizeof(double)));
    if (scap > scap_max) scap = scap_max;
    scap = scap / 64 * 64;
    k.scap = scap < 64 ? 64 : scap;
    // with a second 3-vector per staged atom (adjoint, third-law forces)
    int aux = (int)(room / (6 * sizeof(double)));
    aux = (aux < k.scap ? aux : k.scap) / 64 * 64;
    k.scap_aux = aux < 64 ? 64 : aux;
    if (k.pipeline == MD_PIPE_LAYERS)
        k.nblk_force = (k.n + k.block - 1) / k.block;
    else if (k.pipeline == MD_PIPE_ALLPAIRS)
        k.nblk_force = allpairs_home_blocks(k.n) * k.ap_split;
    else
        k.nblk_force = force_blocks(k);
    // list build: a lane per home atom of a mean tile (25% spare), or waves
    // taking the home cells in turn: 8 waves from 8 home cells on, else 4
    k.nl_method = c->nl_method_req != MD_NL_AUTO ? c->nl_method_req
                                                 : (occ < 8.0 ? MD_NL_LANES : MD_NL_CELL_WAVES);
    const int home_cells = k.kx_max * k.ky_max * k.kz_max;
    int waves;
    if (k.nl_method == MD_NL_LANES) {
        waves = (int)ceil(1.25 * home_cells * occ / kWave);
        waves = waves > 16 ? 16 : waves;
    } else {
        // few tiles, which leave room on the CUs: a wave per home cell of a tile of
        // 12 (100 003 LJ atoms, 486 tiles: 60 against 76 us; 2.048M, 9216 tiles:
        // 723 against 668 us, as two such workgroups share a CU instead of three)
        waves = home_cells >= 12 && c->alone && k.n_tiles < 3 * 256
                    ? 12
                    : (home_cells >= 8 ? 8 : (home_cells >= 4 ? 4 : home_cells));
    }
    waves = waves < 1 ? 1 : waves;
    // up to three tiles per CU of few home cells: up to four waves per cell, each
    // with a part of its atoms, as many as the CU holds (builds: 4000 LJ atoms, 125
    // tiles of one cell, 60 -> 22 us; 20 000, 250 of 4, 44 -> 28; 32 000 FP32, 216 of
    // 8, 62 -> 39; 50 000, 507 of 5, 66 -> 43, and 59 at 16 waves; 70 000, 512 of 8,
    // 53 at 8 and 64 at 16)
    if (c->nl_block_req <= 0 && c->alone && k.n_tiles <= 3 * 256) {
        const int room = k.n_tiles <= 256 ? 16 : (k.n_tiles <= 2 * 256 ? 12 : 8);
        const int parts = room / home_cells < 4 ? room / home_cells : 4;
        if (parts > 1 &&
            nl_queue_fits(k, k.nl_method, kWave * home_cells * parts, c->lds_limit))
            waves = home_cells * parts;
    }
    const int nlb = c->nl_block_req > 0 ? c->nl_block_req : kWave * waves;
    k.nl_block = nlb < kWave ? kWave : (nlb > 1024 ? 1024 : nlb);
    k.nl_queue = nl_queue_fits(k, k.nl_method, k.nl_block, c->lds_limit);
}

static md_status hip_ok(hipError_t e) { return e == hipSuccess ? MD_OK : MD_ERR_HIP; }

// Offsets of the workspace regions from their sizes.
static void relayout(md_ctx* c)
{
    size_t o = 0;
    for (int r = 0; r < R_COUNT; ++r) {
        c->off[r] = o;
        o += align_up(c->bytes[r]);
    }
    c->ws_bytes = o;
}

// Second positions (the scratch positions) for the fused steps of a cells-only
// system without reorder, where they pay (kFusedCells) and the steps can fuse: not
// in a batch nor with bonded terms.  A system of very many cells does without where
// they would put it past the static array (md_bind_static).  Then lays the regions
// out.
static void second_positions(md_ctx* c)
{
    const md_params& p = c->prm;
    if (p.mode == MD_CELLS_ONLY && !p.reorder)
        c->bytes[R_SX] = c->bytes[R_SY] = c->bytes[R_SZ] = 0;
    relayout(c);
    if (p.mode != MD_CELLS_ONLY || p.reorder || p.pipeline != MD_PIPE_TILED || !c->alone ||
        c->kp.bonded_on || p.n_atoms > kFusedCells)
        return;
    const size_t one = sizeof(double) * (size_t)p.n_atoms, more = 3 * align_up(one);
    if (c->ws_bytes + more <= MD_STATIC_WORKSPACE_BYTES) {
        c->bytes[R_SX] = c->bytes[R_SY] = c->bytes[R_SZ] = one;
        relayout(c);
    }
}

void share_machine(md_ctx* c)
{
    c->alone = false;
    second_positions(c);
    plan_tiles(c);
}

static md_status launched() { return hip_ok(hipGetLastError()); }

static void drop_graph(md_ctx* c);  // md_step's captured graph (below)

extern "C" md_status md_init(const md_params* in, md_ctx** out)
{
    if (!in || !out) return MD_ERR_ARG;
    *out = nullptr;
    md_params p = *in;
    if (p.block == 0) p.block = 256;
    const bool finite = isfinite(p.L) && isfinite(p.eps) && isfinite(p.sigma) &&
                        isfinite(p.mass) && isfinite(p.r_cut) && isfinite(p.skin) &&
                        isfinite(p.dt);
    if (!finite || p.n_atoms < 1 || p.L <= 0 || p.eps <= 0 || p.sigma <= 0 || p.mass <= 0 ||
        p.r_cut <= 0 || p.skin < 0 || p.dt <= 0)
        return MD_ERR_ARG;
    if ((p.potential != MD_LJ_SHIFTED && p.potential != MD_LJ_TRUNC) ||
        (p.precision != MD_FP64 && p.precision != MD_FP32_MIXED) ||
        (p.mode != MD_CELLS_ONLY && p.mode != MD_NEIGHBOR_LIST) ||
        (p.newton3 != 0 && p.newton3 != 1) || (p.newton3 && p.mode != MD_NEIGHBOR_LIST) ||
        (p.pipeline != MD_PIPE_TILED && p.pipeline != MD_PIPE_LAYERS &&
         p.pipeline != MD_PIPE_ALLPAIRS) ||
        (p.pipeline == MD_PIPE_LAYERS && (p.mode != MD_NEIGHBOR_LIST || p.newton3 != 0)) ||
        (p.pipeline == MD_PIPE_ALLPAIRS && (p.mode != MD_CELLS_ONLY || p.reorder != 0)) ||
        p.nl_capacity < 0 || p.reorder < 0 ||
        (p.pipeline != MD_PIPE_LAYERS && p.reorder > 1) || p.block % 64 != 0 ||
        p.block < 64 || p.block > 1024)
        return MD_ERR_ARG;

    const bool nl = p.mode == MD_NEIGHBOR_LIST;
    const double r_list = p.r_cut + p.skin;
    const double r_cell = nl ? r_list : p.r_cut;
    double ncd = floor(p.L / r_cell);
    if (ncd > 1290) ncd = 1290;  // keeps nc^3 within int32
    int nc = (int)ncd;
    if (nc >= 1 && p.L / nc < r_cell) --nc;
    if (nc < 3) return MD_ERR_BOX_TOO_SMALL;

    md_ctx* c = new (std::nothrow) md_ctx();
    if (!c) return MD_ERR_ARG;
    c->prm = p;
    c->graph_on = false;  // md_set_graph
    const int64_t n = p.n_atoms;
    const int npad = (int)((n + 63) / 64 * 64);
    int cap = 0;
    if (nl) {
        if (p.nl_capacity > 0) {
            cap = p.nl_capacity;
        } else {
            const double rho = (double)n / (p.L * p.L * p.L);
            const double mean = 4.0 / 3.0 * M_PI * r_list * r_list * r_list * rho;
            cap = (int)ceil(mean + 10.0 * sqrt(mean) + 16.0);
            cap = (cap + 7) / 8 * 8;
        }
        if (cap > n - 1) cap = (int)(n - 1 > 0 ? n - 1 : 1);
        cap = (cap + 3) / 4 * 4;  // whole 4-entry chunks
    }
    c->geo.nc = nc;
    c->geo.n_cells = nc * nc * nc;
    c->geo.nl_capacity = cap;
    c->geo.n_pad = npad;
    c->geo.cell_width = p.L / nc;
    // layers per cell of the layer matrix: the mean occupancy plus six of its
    // Poisson standard deviations plus 8 (overflow is latched, not silent)
    int n_layers = 0;
    if (p.pipeline == MD_PIPE_LAYERS) {
        const double occ = (double)p.n_atoms / ((double)nc * nc * nc);
        n_layers = (int)ceil(occ + 6.0 * sqrt(occ) + 8.0);
    }
    c->geo.n_layers = n_layers;
    // all-pairs: partner chunks per 64-atom home block
    int ap_split = 0, ap_chunk = 0;
    if (p.pipeline == MD_PIPE_ALLPAIRS) allpairs_split(p.n_atoms, &ap_split, &ap_chunk);
    const int64_t ap_blocks = ap_split > 0 ? (int64_t)allpairs_home_blocks(p.n_atoms) * ap_split : 0;

    // workspace layout
    const int64_t ncell = (int64_t)nc * nc * nc;
    const size_t fsz = p.precision == MD_FP64 ? sizeof(double) : sizeof(float);
    size_t* b = c->bytes;
    b[R_DEV] = sizeof(DevState);
    b[R_CELL_COUNT] = sizeof(int32_t) * ncell;
    b[R_CELL_START] = sizeof(int32_t) * (ncell + 1);
    b[R_CELL_OF] = b[R_SLOT] = b[R_ORDER] = sizeof(int32_t) * n;
    b[R_TMP] = 2 * sizeof(int32_t) * n;  // slot -> atom, then slot -> permanent id
    const bool layers = p.pipeline == MD_PIPE_LAYERS;
    // plus one chunk row past the list: the cell-wave build writes entries
    // beyond the capacity there instead of testing each store (overflow is
    // counted and latched all the same)
    b[R_NL] = layers ? 0 : sizeof(uint16_t) * (size_t)(cap + kChunk) * npad;
    b[R_LAYERS] = sizeof(int32_t) * (size_t)ncell * n_layers;
    b[R_W32] = layers ? sizeof(int32_t) * (size_t)cap * npad : 0;
    b[R_NL_COUNT] = sizeof(int32_t) * npad;
    b[R_XR] = b[R_YR] = b[R_ZR] = nl ? sizeof(double) * n : 0;
    const size_t perm = p.reorder ? 1 : 0;
    b[R_SX] = b[R_SY] = b[R_SZ] = b[R_SVX] = b[R_SVY] = b[R_SVZ] = perm * sizeof(double) * n;
    b[R_SFX] = b[R_SFY] = b[R_SFZ] = perm * fsz * n;
    b[R_SID] = b[R_SCELL] = perm * sizeof(int32_t) * n;
    b[R_APART] = ap_split > 1 ? fsz * 3 * (size_t)ap_split * npad : 0;
    const int64_t fblocks = max_force_blocks(n, ncell);
    b[R_FPART] = sizeof(double) * 2 * (size_t)(ap_blocks > fblocks ? ap_blocks : fblocks);
    b[R_IPART] = sizeof(double) * 8 * kIntegrateGridMax;
    b[R_HIST] = sizeof(md_record) * kHistCap;
    second_positions(c);

    KParams& k = c->kp;
    memset(&k, 0, sizeof(k));
    k.n = (int)n;
    k.npad = npad;
    k.nc = nc;
    k.ncell = (int)ncell;
    k.cap = cap;
    k.potential = p.potential;
    k.precision = p.precision;
    k.mode = p.mode;
    k.reorder = p.reorder;
    k.newton3 = p.newton3;
    k.pipeline = p.pipeline;
    k.n_layers = n_layers;
    k.ap_split = ap_split;
    k.ap_chunk = ap_chunk;
    k.L = p.L;
    k.invL = 1.0 / p.L;
    k.inv_w = (double)nc / p.L;
    k.rc2 = p.r_cut * p.r_cut;
    k.rl2 = r_list * r_list;
    k.rl2_in = k.rl2 * (1.0 - 1e-9);
    k.box_reach2 = k.rl2 * (1.0 + 1e-9);
    k.box_slack = 1e-6 * p.L;
    k.sig2 = p.sigma * p.sigma;
    k.eps2 = 2.0 * p.eps;
    k.eps48 = 48.0 * p.eps;
    k.eps = p.eps;
    k.sigma = p.sigma;
    double shift = 0.0;
    if (p.potential == MD_LJ_SHIFTED) {
        const double sr2 = k.sig2 / k.rc2, sr6 = sr2 * sr2 * sr2;
        shift = 4.0 * p.eps * (sr6 * sr6 - sr6);
    }
    k.half_shift = 0.5 * shift;
    k.ushift = k.half_shift / k.eps2;
    k.ushift2 = 2.0 * k.ushift;
    k.hdt = (0.5 * p.dt) / p.mass;
    k.dt = p.dt;
    k.disp_thr2 = (0.5 * p.skin) * (0.5 * p.skin);
    k.mass = p.mass;
    k.block = p.block;
    // 2 lanes per atom (2.048 M-atom LJ, 512-thread workgroups: FP64 force pass
    // 255 us at 2 lanes, 267 at 4, 356 at 8; FP32-mixed 228, 244, 324)
    k.force_lanes = 2;
    k.force_block = 512;
    c->nl_block_req = 0;
    k.int_grid = kIntegrateGridDefault;
    k.gate_grid = kGateGridDefault;
    plan_tiles(c);
    *out = c;
    return MD_OK;
}

extern "C" size_t md_workspace_bytes(const md_ctx* c) { return c ? c->ws_bytes : 0; }

extern "C" md_status md_set_bonded(md_ctx* c, const md_bonded* b)
{
    if (!c) return MD_ERR_ARG;
    if (c->bound) return MD_ERR_STATE;
    KParams& k = c->kp;
    if (!b) {
        k.bonded_on = 0;
        c->bytes[R_SLOT_OF] = c->bytes[R_BPART] = 0;
        second_positions(c);
        return MD_OK;
    }
    const bool finite = isfinite(b->fene_k) && isfinite(b->fene_r0) && isfinite(b->bend_k) &&
                        isfinite(b->tors_c[0]) && isfinite(b->tors_c[1]) &&
                        isfinite(b->tors_c[2]) && isfinite(b->tors_c[3]);
    if (!finite || b->chain_length < 2 || c->prm.n_atoms % b->chain_length != 0 ||
        !(b->fene_r0 > 0.0) || b->fene_k < 0.0)
        return MD_ERR_ARG;
    k.bonded_on = 1;
    k.chain_len = b->chain_length;
    k.fene_k = b->fene_k;
    k.fene_r02 = b->fene_r0 * b->fene_r0;
    k.bend_k = b->bend_k;
    for (int m = 0; m < 4; ++m) k.tors_c[m] = b->tors_c[m];
    k.tors_on = b->tors_c[0] != 0.0 || b->tors_c[1] != 0.0 || b->tors_c[2] != 0.0 ||
                b->tors_c[3] != 0.0;
    k.nblk_bonded = bonded_blocks(k.n);
    c->bytes[R_SLOT_OF] = sizeof(int32_t) * (size_t)k.n;
    c->bytes[R_BPART] = sizeof(double) * 2 * (size_t)k.nblk_bonded;
    second_positions(c);
    return MD_OK;
}

extern "C" md_status md_geometry(const md_ctx* c, md_grid* out)
{
    if (!c || !out) return MD_ERR_ARG;
    *out = c->geo;
    return MD_OK;
}

extern "C" md_status md_layout(const md_ctx* c, int32_t which, size_t* offset, size_t* count)
{
    if (!c || !offset || !count) return MD_ERR_ARG;
    const int64_t n = c->prm.n_atoms;
    const bool layers = c->prm.pipeline == MD_PIPE_LAYERS;
    const bool allpairs = c->prm.pipeline == MD_PIPE_ALLPAIRS;
    switch (which) {
        case MD_ARR_CELL_OF:
            if (allpairs) return MD_ERR_ARG;
            *offset = c->off[R_CELL_OF];
            *count = n;
            break;
        case MD_ARR_CELL_START:
            if (layers || allpairs) return MD_ERR_ARG;
            *offset = c->off[R_CELL_START];
            *count = c->geo.n_cells + 1;
            break;
        case MD_ARR_CELL_ATOMS:
            if (layers || allpairs) return MD_ERR_ARG;
            *offset = c->off[R_ORDER];
            *count = n;
            break;
        case MD_ARR_NL:
            *offset = c->off[layers ? R_W32 : R_NL];
            *count = (size_t)c->geo.nl_capacity * c->geo.n_pad;
            break;
        case MD_ARR_LAYERS:
            if (!layers) return MD_ERR_ARG;
            *offset = c->off[R_LAYERS];
            *count = (size_t)c->geo.n_cells * c->geo.n_layers;
            break;
        case MD_ARR_LAYER_COUNT:
            if (!layers) return MD_ERR_ARG;
            *offset = c->off[R_CELL_COUNT];
            *count = c->geo.n_cells;
            break;
        case MD_ARR_NL_COUNT: *offset = c->off[R_NL_COUNT]; *count = n; break;
        case MD_ARR_XREF:
            if (c->prm.mode != MD_NEIGHBOR_LIST) return MD_ERR_ARG;
            *offset = c->off[R_XR];  // x, y, z references follow at 256-byte-aligned pitch
            *count = n;
            break;
        default: return MD_ERR_ARG;
    }
    return MD_OK;
}

static bool state_buffers_ok(const md_buffers* bf)
{
    return bf->x && bf->y && bf->z && bf->vx && bf->vy && bf->vz && bf->fx && bf->fy &&
           bf->fz && bf->id;
}

// Points the kernel parameters at the caller's state arrays and at the
// workspace regions inside ws, binds the stream, plans the tiles and
// enqueues the clearing of the device counters.
static md_status bind_to(md_ctx* c, const md_buffers* bf, char* ws, void* stream)
{
    KParams& k = c->kp;
    drop_graph(c);  // the pointers are baked into it
    auto at = [&](int r) -> void* { return c->bytes[r] ? ws + c->off[r] : nullptr; };
    k.x = bf->x; k.y = bf->y; k.z = bf->z;
    k.vx = bf->vx; k.vy = bf->vy; k.vz = bf->vz;
    k.fx = bf->fx; k.fy = bf->fy; k.fz = bf->fz;
    k.id = bf->id;
    k.dev = static_cast<DevState*>(at(R_DEV));
    k.cell_count = static_cast<int32_t*>(at(R_CELL_COUNT));
    k.cell_start = static_cast<int32_t*>(at(R_CELL_START));
    k.cell_of = static_cast<int32_t*>(at(R_CELL_OF));
    k.slot = static_cast<int32_t*>(at(R_SLOT));
    k.order = static_cast<int32_t*>(at(R_ORDER));
    k.tmp = static_cast<int32_t*>(at(R_TMP));
    k.nl64 = static_cast<uint64_t*>(at(R_NL));
    k.nl_count = static_cast<int32_t*>(at(R_NL_COUNT));
    k.xr = static_cast<double*>(at(R_XR));
    k.yr = static_cast<double*>(at(R_YR));
    k.zr = static_cast<double*>(at(R_ZR));
    k.sx = static_cast<double*>(at(R_SX));
    k.sy = static_cast<double*>(at(R_SY));
    k.sz = static_cast<double*>(at(R_SZ));
    k.svx = static_cast<double*>(at(R_SVX));
    k.svy = static_cast<double*>(at(R_SVY));
    k.svz = static_cast<double*>(at(R_SVZ));
    k.sfx = static_cast<double*>(at(R_SFX));
    k.sfy = static_cast<double*>(at(R_SFY));
    k.sfz = static_cast<double*>(at(R_SFZ));
    k.sid = static_cast<int32_t*>(at(R_SID));
    k.layers = static_cast<int32_t*>(at(R_LAYERS));
    k.w32 = static_cast<int32_t*>(at(R_W32));
    k.apart = at(R_APART);
    k.slot_of = static_cast<int32_t*>(at(R_SLOT_OF));
    k.bpart = static_cast<double*>(at(R_BPART));
    k.scell = static_cast<int32_t*>(at(R_SCELL));
    k.fpart = static_cast<double*>(at(R_FPART));
    k.ipart = static_cast<double*>(at(R_IPART));
    k.hist = static_cast<md_record*>(at(R_HIST));
    c->stream = static_cast<hipStream_t>(stream);
    int dev = 0, lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return MD_ERR_HIP;
    c->lds_limit = (size_t)lds;
    plan_tiles(c);
    c->bound = true;
    c->host_steps = 0;
    c->cells_ok = c->nl_ok = c->forces_ok = false;
    launch_clear(k, c->stream);
    return launched();
}

extern "C" md_status md_bind(md_ctx* c, const md_buffers* bf, void* stream)
{
    if (!c || !bf) return MD_ERR_ARG;
    if (!state_buffers_ok(bf) || !bf->workspace) return MD_ERR_ARG;
    if (((uintptr_t)bf->workspace) % kAlign != 0) return MD_ERR_ARG;
    return bind_to(c, bf, static_cast<char*>(bf->workspace), stream);
}

// ---- binding to the library's own workspace (no allocation) ----
//
// One static device array per GPU holds the workspace of contexts bound
// with md_bind_static.  In host code the array's name stands for a host
// shadow, not for device memory, so its device address is looked up once
// per device (with that device current) and only that address is used.

static __device__ __align__(256) unsigned char scratch[MD_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];  // device address of scratch on each device
}  // namespace

static md_status static_workspace(void** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MD_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return MD_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
            return MD_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MD_OK;
}

extern "C" md_status md_bind_static(md_ctx* c, const md_buffers* bf, void* stream)
{
    if (!c || !bf) return MD_ERR_ARG;
    if (!state_buffers_ok(bf) || bf->workspace) return MD_ERR_ARG;
    if (c->ws_bytes > (size_t)MD_STATIC_WORKSPACE_BYTES) return MD_ERR_WORKSPACE_TOO_LARGE;
    void* ws = nullptr;
    md_status st = static_workspace(&ws);
    if (st != MD_OK) return st;
    // a caller-supplied workspace starts zeroed; so does this one, whatever
    // an earlier binding left in it (a fill kernel, not a memset node, so the
    // call may sit in a captured graph)
    launch_fill(static_cast<double*>(ws), c->ws_bytes / sizeof(double), 0.0,
                static_cast<hipStream_t>(stream));
    st = launched();
    if (st != MD_OK) return st;
    return bind_to(c, bf, static_cast<char*>(ws), stream);
}

// The stages of either pipeline.
// flags: bit 0 forces the build; the tiled cell build also takes kFoldCopy,
// kFoldBin and kSortSmallOk (md_internal.h).
static void cells_any(const KParams& k, int flags, hipStream_t s)
{
    const int force = flags & 1;
    if (k.pipeline == MD_PIPE_LAYERS)
        launch_layer_cells(k, force, s);
    else if (k.pipeline == MD_PIPE_ALLPAIRS) {
        if (force) launch_allpairs_fold(k, s);  // in a step the drift folds
    } else
        launch_cells(k, flags, s);
    // after any permutation of the slots that has not done it
    if (k.bonded_on && !(flags & kFoldCopy)) launch_bond_map(k, force, s);
}

static void neighbors_any(const KParams& k, int force, hipStream_t s)
{
    if (k.pipeline == MD_PIPE_LAYERS)
        launch_layer_nl(k, force, s);
    else
        launch_neighbors(k, force, s);
}

// flags: kFoldCopy for the tiled cells-only pass (md_internal.h).
static void forces_any(const KParams& k, hipStream_t s, int flags = 0)
{
    if (k.pipeline == MD_PIPE_LAYERS)
        launch_layer_forces(k, s);
    else if (k.pipeline == MD_PIPE_ALLPAIRS)
        launch_allpairs_forces(k, s);
    else
        launch_forces(k, s, flags);
    if (k.bonded_on) launch_bonded(k, s);  // adds to the pair forces
}

extern "C" md_status md_build_cells(md_ctx* c)
{
    if (!c) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    if (c->replan) plan_tiles(c);
    cells_any(c->kp, 1, c->stream);
    c->cells_ok = true;
    c->nl_ok = false;
    c->forces_ok = false;
    return launched();
}

extern "C" md_status md_build_neighbors(md_ctx* c)
{
    if (!c) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    if (c->prm.mode != MD_NEIGHBOR_LIST) return MD_ERR_ARG;
    if (!c->cells_ok) return MD_ERR_STATE;
    if (c->replan) plan_tiles(c);
    neighbors_any(c->kp, 1, c->stream);
    c->nl_ok = true;
    return launched();
}

// Launches fn on the bound stream; with timing on, between two events
// counted toward part (MD_PART_*).
template <class Fn>
static void timed(md_ctx* c, int part, Fn&& fn)
{
    if (!c->timing) {
        fn();
        return;
    }
    hipEvent_t ev[2];
    for (int k = 0; k < 2; ++k) {
        if (!c->ev_free.empty()) {
            ev[k] = c->ev_free.back();
            c->ev_free.pop_back();
        } else {
            (void)hipEventCreate(&ev[k]);
        }
    }
    (void)hipEventRecord(ev[0], c->stream);
    fn();
    (void)hipEventRecord(ev[1], c->stream);
    c->ev_pending.push_back(ev[0]);
    c->ev_pending.push_back(ev[1]);
    c->ev_part.push_back(part);
}

static void timed_forces(md_ctx* c, int flags = 0)
{
    timed(c, MD_PART_FORCES, [&] { forces_any(c->kp, c->stream, flags); });
}

static md_status fold_timing(md_ctx* c)
{
    if (c->ev_pending.empty()) return MD_OK;
    if (hipStreamSynchronize(c->stream) != hipSuccess) return MD_ERR_HIP;
    for (size_t k = 0; k + 1 < c->ev_pending.size(); k += 2) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->ev_pending[k], c->ev_pending[k + 1]) != hipSuccess)
            return MD_ERR_HIP;
        const int part = c->ev_part[k / 2];
        if (part == MD_PART_FORCES) {
            c->timed_ms += ms;
            c->timed_launches += 1;
        }
        c->part_ms[part] += ms;
        c->part_launches[part] += 1;
        c->ev_free.push_back(c->ev_pending[k]);
        c->ev_free.push_back(c->ev_pending[k + 1]);
    }
    c->ev_pending.clear();
    c->ev_part.clear();
    return MD_OK;
}

extern "C" md_status md_export_neighbors(md_ctx* c, int32_t* dst)
{
    if (!c || !dst) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    if (c->prm.mode != MD_NEIGHBOR_LIST) return MD_ERR_ARG;
    if (!c->nl_ok) return MD_ERR_STATE;
    if (c->kp.pipeline == MD_PIPE_LAYERS)
        launch_layer_export(c->kp, dst, c->stream);
    else
        launch_nl_export(c->kp, dst, c->stream);
    return launched();
}

extern "C" md_status md_forces(md_ctx* c)
{
    if (!c) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    if (!c->cells_ok || (c->prm.mode == MD_NEIGHBOR_LIST && !c->nl_ok)) return MD_ERR_STATE;
    c->replan = false;  // the list in use has the shape that was kept
    timed_forces(c);
    c->forces_ok = true;
    return launched();
}

// ---- md_step ----
//
// A step is a fixed launch sequence (the rebuild-gated list build, the fused force
// pass, the finish with the rebuild-gated cell build), so runs of kGraphSteps steps can
// be captured once into a HIP graph and replayed (md_set_graph), for callers that
// need the step as a graph.  It is off by default: direct launches measured faster on
// MI355X or the same (per step, direct and replayed: 4000-atom WCA cells-only 12.6 and
// 13.9 us; lists: 10 007 LJ 20.9 and 23.5, 32 000 WCA 24.6 and 25.1, 32 000 LJ 28.4 and
// 33.5, 131 072 WCA 26.6 and 32.4, 256 000 WCA 31.9 and 37.9).
// The first step of a call (its integrate kernel only kicks and drifts) and the
// remainder are launched directly.  A call of fewer than kGraphSteps + 1 steps (but
// at least kGraphMin + 1) replays one graph of its own length instead, so that
// repeated short calls are captured too; the graph is recaptured when the length
// changes.  Timing (md_set_timing) brackets each force launch with
// events and uses the direct path throughout.

constexpr int kGraphSteps = 32;
constexpr int kGraphMin = 8;

static void drop_graph(md_ctx* c)
{
    if (c->gexec) (void)hipGraphExecDestroy(c->gexec);
    if (c->graph) (void)hipGraphDestroy(c->graph);
    c->gexec = nullptr;
    c->graph = nullptr;
    c->g_record = -1;
    c->g_len = 0;
    c->g_run = nullptr;
}

// The layer pipeline's periodic reorder (md_params.reorder = k > 0): due
// before the force pass of every k-th step.
static bool layer_reorder_on(const md_ctx* c)
{
    return c->kp.pipeline == MD_PIPE_LAYERS && c->kp.reorder > 0;
}

// Launches of n steps, the first of them step step0 + 1 since md_bind;
// first: it is the first step of the run.
static md_status step_launches(md_ctx* c, hipStream_t s, bool first, int32_t n,
                               int32_t record_every, int64_t step0)
{
    const KParams& k = c->kp;
    const bool nl = c->prm.mode == MD_NEIGHBOR_LIST;
    const bool tiled = k.pipeline == MD_PIPE_TILED;
    // the reorder's copy-back folded into the pass after the cell build (the
    // list build, or the cells-only force pass)
    const int fold = tiled && k.reorder && (nl || !k.bonded_on) ? kFoldCopy : 0;
    // cells only: the cells are rebuilt every step, so the integration pass
    // bins the atoms and a small system sorts them in one workgroup
    const bool cells = tiled && !nl;
    const int cflags = fold | (cells ? kFoldBin | kSortSmallOk : 0);
    const int fflags = cells ? fold : 0;
    // the finish with the cell build behind it (one launch for a small system);
    // a bonded system's map of slots goes with the folded sort only
    const bool joined = tiled && (!k.bonded_on || fold);
    const bool slots = joined && finish_bins(k, cflags);
    auto finish_and_cells = [&](int phase) {
        if (joined) {
            launch_finish_cells(k, cflags, phase, record_every, false, s);
        } else {
            launch_integrate_finish(k, phase, record_every, s);
            cells_any(k, cflags, s);
        }
    };
    if (s != c->stream) {  // captured into a graph: never timed, never reordered
        for (int32_t i = 0; i < n; ++i) {
            const int phase = first && i == 0 ? 0 : 1;
            launch_integrate_pass(k, phase, s, cells, false, slots && phase == 1);
            finish_and_cells(phase);
            if (nl) neighbors_any(k, fold, s);
            forces_any(k, s, fflags);
        }
        return MD_OK;
    }
    for (int32_t i = 0; i < n; ++i) {
        const int phase = first && i == 0 ? 0 : 1;
        const bool reorder = layer_reorder_on(c) && (step0 + i + 1) % k.reorder == 0;
        const bool together = !c->timing && !reorder;
        timed(c, MD_PART_INTEGRATE, [&] {
            launch_integrate_pass(k, phase, s, cells, false, slots && together && phase == 1);
        });
        if (together) {
            finish_and_cells(phase);
        } else if (cells && k.n <= kSortSmall && !k.bonded_on) {
            // the finish and the cell build in one launch (counted as cells)
            timed(c, MD_PART_CELLS, [&] { finish_and_cells(phase); });
        } else {
            timed(c, MD_PART_ENERGY, [&] { launch_integrate_finish(k, phase, record_every, s); });
            if (reorder) timed(c, MD_PART_REORDER, [&] { launch_layer_reorder(k, s); });
            timed(c, MD_PART_CELLS, [&] { cells_any(k, reorder ? 1 : cflags, s); });
        }
        if (nl) timed(c, MD_PART_NEIGHBORS, [&] { neighbors_any(k, reorder ? 1 : fold, s); });
        timed_forces(c, fflags);
        if (c->timing && c->ev_pending.size() >= 8192) {
            md_status st = fold_timing(c);
            if (st != MD_OK) return st;
        }
    }
    return MD_OK;
}

// The steps of a system whose integration rides in the force pass
// (launch_forces_step): an integration pass starts the first step, every body
// ends one step and starts the next (cells and list if needed, the fused force
// pass, its finish), and a force pass and an integration pass end the last.
// A finish is launched with the cell build behind it.
// The positions change places with the scratch arrays in every body: `flip`
// says where they are, and the first pass puts them where the last body will
// leave them in the state arrays.
static bool fused_steps(const md_ctx* c) { return !c->timing && fused_fits(c->kp); }

static KParams flipped(const KParams& k, bool flip)
{
    KParams q = k;
    if (flip) flip_positions(q);
    return q;
}

// Cells (after the finish of a pass), list and force pass flags of a fused body.
static int fused_cells_flags(const KParams& k)
{
    return (k.reorder ? kFoldCopy : 0) |
           (k.mode == MD_CELLS_ONLY ? kFoldBin | kSortSmallOk : 0);
}

static void fused_bodies(const md_ctx* c, hipStream_t s, int32_t n, int32_t record_every,
                         bool& flip)
{
    const int flags = fused_cells_flags(c->kp);
    const bool flips = fused_flips(c->kp);
    for (int32_t i = 0; i < n; ++i) {
        const KParams q = flipped(c->kp, flip);
        if (q.mode == MD_NEIGHBOR_LIST) launch_neighbors(q, kFoldCopy, s);
        launch_forces_step(q, s);
        if (flips) flip = !flip;
        launch_finish_cells(flipped(c->kp, flip), flags, 1, record_every, true, s);
    }
}

// The graph of len steps, captured unless it is there already.  The null stream
// cannot be captured: then the graph runs on the context's own stream, ordered after
// and before the bound stream's work by events.
// fused: the steps are fused bodies (fused_bodies), the first from flip.  Called
// before the first launch of md_step, so that a call that cannot have its graph (its
// stream is being captured, say) leaves the state as it was.
static md_status step_graph_ready(md_ctx* c, int32_t len, int32_t record_every, bool fused,
                                  bool flip)
{
    hipStream_t run = c->stream;
    if (run == nullptr) {
        if (!c->gstream &&
            hipStreamCreateWithFlags(&c->gstream, hipStreamNonBlocking) != hipSuccess)
            return MD_ERR_HIP;
        for (int e = 0; e < 2; ++e)
            if (!c->gev[e] &&
                hipEventCreateWithFlags(&c->gev[e], hipEventDisableTiming) != hipSuccess)
                return MD_ERR_HIP;
        run = c->gstream;
    }
    const int kind = fused ? (flip ? 2 : 1) : 0;
    if (c->gexec && c->g_record == record_every && c->g_run == run && c->g_len == len &&
        c->g_kind == kind)
        return MD_OK;
    drop_graph(c);
    if (hipStreamBeginCapture(run, hipStreamCaptureModeThreadLocal) != hipSuccess)
        return MD_ERR_HIP;
    md_status st = MD_OK;
    bool f = flip;
    if (fused)
        fused_bodies(c, run, len, record_every, f);
    else
        st = step_launches(c, run, false, len, record_every, 0);
    hipGraph_t g = nullptr;
    const hipError_t ec = hipStreamEndCapture(run, &g);
    if (st != MD_OK) return st;
    if (ec != hipSuccess || !g) return MD_ERR_HIP;
    c->graph = g;
    if (hipGraphInstantiate(&c->gexec, c->graph, nullptr, nullptr, 0) != hipSuccess) {
        drop_graph(c);
        return MD_ERR_HIP;
    }
    c->g_record = record_every;
    c->g_kind = kind;
    c->g_len = len;
    c->g_run = run;
    return MD_OK;
}

// n_graphs replays of the graph of step_graph_ready.
static md_status step_graphs(md_ctx* c, int32_t n_graphs)
{
    hipStream_t run = c->g_run;
    const bool own = run != c->stream;
    if (own && (hipEventRecord(c->gev[0], c->stream) != hipSuccess ||
                hipStreamWaitEvent(run, c->gev[0], 0) != hipSuccess))
        return MD_ERR_HIP;
    for (int32_t g = 0; g < n_graphs; ++g)
        if (hipGraphLaunch(c->gexec, run) != hipSuccess) return MD_ERR_HIP;
    if (own && (hipEventRecord(c->gev[1], run) != hipSuccess ||
                hipStreamWaitEvent(c->stream, c->gev[1], 0) != hipSuccess))
        return MD_ERR_HIP;
    return MD_OK;
}

extern "C" md_status md_step(md_ctx* c, int32_t n_steps, int32_t record_every)
{
    if (!c || n_steps < 0 || record_every < 0) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    if (!c->forces_ok) return MD_ERR_STATE;
    if (n_steps == 0) return MD_OK;
    md_status st = MD_OK;
    const int64_t step0 = c->host_steps;
    const bool fused = fused_steps(c);
    // the steps behind the first, and the graphs they replay
    const int32_t rest = n_steps - 1;
    const bool graph =
        c->graph_on && n_steps > kGraphMin && (fused || !(c->timing || layer_reorder_on(c)));
    const int32_t len = rest < kGraphSteps ? rest : kGraphSteps, n_graphs = graph ? rest / len : 0;
    bool flip = fused && fused_flips(c->kp) && rest % 2 != 0;
    if (graph && (st = step_graph_ready(c, len, record_every, fused, flip)) != MD_OK) {
        (void)hipGetLastError();  // reported here, not by the next call's launches
        return st;
    }
    if (fused) {
        const KParams& k = c->kp;
        hipStream_t s = c->stream;
        const bool nl = k.mode == MD_NEIGHBOR_LIST;
        const int flags = fused_cells_flags(k);
        launch_integrate_pass(k, 0, s, !nl, flip);
        launch_finish_cells(flipped(k, flip), flags, 0, record_every, false, s);
        if (graph) st = step_graphs(c, n_graphs);
        // several replays are of kGraphSteps (even) bodies each: the places are the
        // same before and after
        if (graph && len % 2 != 0 && fused_flips(k)) flip = !flip;
        if (st == MD_OK) {
            fused_bodies(c, s, rest - n_graphs * len, record_every, flip);
            if (nl) launch_neighbors(k, kFoldCopy, s);
            launch_forces(k, s, nl ? 0 : flags & kFoldCopy);
        }
    } else if (!graph) {
        st = step_launches(c, c->stream, true, n_steps, record_every, step0);
    } else {
        st = step_launches(c, c->stream, true, 1, record_every, step0);
        if (st == MD_OK) st = step_graphs(c, n_graphs);
        if (st == MD_OK)
            st = step_launches(c, c->stream, false, rest - n_graphs * len, record_every,
                               step0 + 1 + (int64_t)n_graphs * len);
    }
    c->host_steps = step0 + n_steps;
    if (st != MD_OK) {
        c->forces_ok = false;  // stopped between steps (a replay failed)
        return st;
    }
    launch_integrate(c->kp, 2, record_every, c->stream);
    return launched();
}

extern "C" md_status md_set_graph(md_ctx* c, int32_t enable)
{
    if (!c) return MD_ERR_ARG;
    c->graph_on = enable != 0;
    if (!c->graph_on) drop_graph(c);
    return MD_OK;
}

extern "C" md_status md_reduce(md_ctx* c, md_observables* out)
{
    if (!c || !out) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    launch_observe(c->kp, c->stream);
    md_status st = launched();
    if (st != MD_OK) return st;
    DevState d;
    if (hipMemcpyAsync(&d, c->kp.dev, sizeof(d), hipMemcpyDeviceToHost, c->stream) != hipSuccess)
        return MD_ERR_HIP;
    if (hipStreamSynchronize(c->stream) != hipSuccess) return MD_ERR_HIP;
    const double n = c->prm.n_atoms;
    const double V = c->prm.L * c->prm.L * c->prm.L;
    memset(out, 0, sizeof(*out));
    out->U = d.obs[0];
    out->K = d.obs[1];
    out->W = d.obs[2];
    out->P[0] = d.obs[3];
    out->P[1] = d.obs[4];
    out->P[2] = d.obs[5];
    out->T = n > 1 ? 2.0 * out->K / (3.0 * (n - 1)) : 0.0;
    out->pressure = (2.0 * out->K + out->W) / (3.0 * V);
    out->dmax = sqrt(d.dmax2);
    out->step = d.step;
    out->n_rebuilds = d.n_rebuilds;
    out->max_occupancy = d.max_occ;
    out->max_nl = d.max_nl;
    out->flags = d.flags;
    if (d.flags & MD_FLAG_TOPOLOGY) return MD_ERR_TOPOLOGY;
    if (d.flags & MD_FLAG_BOND_BROKEN) return MD_ERR_BOND_BROKEN;
    if (d.flags & MD_FLAG_LAYER_OVERFLOW) return MD_ERR_LAYER_OVERFLOW;
    if (d.flags & MD_FLAG_NL_OVERFLOW) return MD_ERR_NL_OVERFLOW;
    if (d.flags & MD_FLAG_NONFINITE) return MD_ERR_NONFINITE;
    return MD_OK;
}

// ---- reverse mode ----

namespace {

constexpr int kTrajMaxBins = 1024;

// Byte offsets inside the trajectory workspace.  Every per-atom array has
// the same 256-byte-aligned pitch.
struct TrajLayout {
    int k;         // steps per segment
    int nseg;      // segments (one checkpoint each, plus the final state)
    size_t pitch;  // bytes of one per-atom double array
    size_t ck, snap, lam, theta, tpart, hist, total;
};

bool traj_layout(const md_ctx* c, const md_traj_params* tp, TrajLayout* L)
{
    if (!c || !tp) return false;
    if (tp->n_steps < 1 || tp->n_steps > kHistCap || tp->checkpoint_every < 1 ||
        tp->n_bins < 0 || tp->n_bins > kTrajMaxBins)
        return false;
    if (tp->n_bins > 0 && !(tp->gr_rmax > 0.0 && tp->gr_width > 0.0 && isfinite(tp->gr_rmax) &&
                            isfinite(tp->gr_width)))
        return false;
    const size_t n = (size_t)c->prm.n_atoms;
    L->k = tp->checkpoint_every < tp->n_steps ? tp->checkpoint_every : tp->n_steps;
    L->nseg = (tp->n_steps + L->k - 1) / L->k;
    L->pitch = align_up(sizeof(double) * n);
    size_t o = 0;
    L->ck = o;  // (x, y, z, vx, vy, vz) at the start of every segment and at the end
    o += (size_t)(L->nseg + 1) * 6 * L->pitch;
    L->snap = o;  // positions of the recomputed steps inside one segment
    o += (size_t)(L->k - 1) * 3 * L->pitch;
    L->lam = o;  // lambda_x, lambda_v (two buffers)
    o += 9 * L->pitch;
    L->theta = o;
    o += align_up(2 * sizeof(double));
    L->tpart = o;
    o += align_up(2 * sizeof(double) * (size_t)max_force_blocks(n, c->geo.n_cells));
    L->hist = o;
    o += align_up(sizeof(unsigned long long) * (size_t)(tp->n_bins > 0 ? tp->n_bins : 1));
    L->total = o;
    return true;
}

double* arr(void* ws, const TrajLayout& L, size_t off, size_t idx)
{
    return reinterpret_cast<double*>(static_cast<char*>(ws) + off + idx * L.pitch);
}

}  // namespace

static md_status traj_check(md_ctx* c, const md_traj_params* tp, void* ws, TrajLayout* L)
{
    if (!c || !tp || !ws || !traj_layout(c, tp, L)) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    if (c->prm.mode != MD_NEIGHBOR_LIST || c->prm.reorder != 0 || c->prm.newton3 != 0 ||
        c->prm.pipeline != MD_PIPE_TILED || c->kp.bonded_on)
        return MD_ERR_ARG;
    if (((uintptr_t)ws) % kAlign != 0) return MD_ERR_ARG;
    if (tp->n_bins > 0 && tp->gr_rmax + 3.0 * tp->gr_width > c->prm.r_cut + c->prm.skin)
        return MD_ERR_ARG;
    return MD_OK;
}

static GrArgs gr_args(const md_ctx* c, const md_traj_params* tp, void* ws, const TrajLayout& L)
{
    GrArgs g;
    memset(&g, 0, sizeof(g));
    g.hist = reinterpret_cast<unsigned long long*>(static_cast<char*>(ws) + L.hist);
    g.n_bins = tp->n_bins;
    g.rmax = tp->gr_rmax;
    g.width = tp->gr_width;
    // fixed-point units: the largest possible bin sum (every atom, a full
    // list, each pair at the kernel's peak) stays below 2^62
    const double kmax = 1.0 / (tp->gr_width * sqrt(2.0 * M_PI));
    const double bound = (double)c->prm.n_atoms * (double)c->geo.nl_capacity * kmax;
    int e = (int)floor(log2(ldexp(1.0, 62) / (bound > 1.0 ? bound : 1.0)));
    g.scale = ldexp(1.0, e < 40 ? e : 40);
    return g;
}

// Copy the state (x, y, z, vx, vy, vz) to or from a checkpoint.
static md_status checkpoint(md_ctx* c, double* const* ck, bool save)
{
    const KParams& k = c->kp;
    double* st[6] = {k.x, k.y, k.z, k.vx, k.vy, k.vz};
    const size_t bytes = sizeof(double) * (size_t)c->prm.n_atoms;
    for (int a = 0; a < 6; ++a)
        if (hipMemcpyAsync(save ? ck[a] : st[a], save ? st[a] : ck[a], bytes,
                           hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
            return MD_ERR_HIP;
    return MD_OK;
}

static void checkpoint_arrays(void* ws, const TrajLayout& L, int seg, double** out)
{
    for (int a = 0; a < 6; ++a) out[a] = arr(ws, L, L.ck, (size_t)seg * 6 + a);
}

// Cells, list and forces from scratch at the current positions.
static void rebuild_all(md_ctx* c)
{
    c->replan = false;
    launch_cells(c->kp, 1, c->stream);
    launch_neighbors(c->kp, 1, c->stream);
    launch_forces(c->kp, c->stream);
    c->cells_ok = c->nl_ok = c->forces_ok = true;
}

extern "C" size_t md_traj_workspace_bytes(const md_ctx* c, const md_traj_params* tp)
{
    TrajLayout L;
    return traj_layout(c, tp, &L) ? L.total : 0;
}

extern "C" md_status md_traj_forward(md_ctx* c, const md_traj_params* tp, void* ws, double* obs)
{
    TrajLayout L;
    md_status st = traj_check(c, tp, ws, &L);
    if (st != MD_OK) return st;
    if (!obs) return MD_ERR_ARG;
    if (!c->forces_ok) {
        if (c->replan) plan_tiles(c);
        rebuild_all(c);
    }
    double* ck[6];
    // the segments launch directly: on a system made for one trajectory (the
    // usual case, since eps and sigma are fixed at md_init) capturing a graph
    // of the segment cost more than its replays saved (measured on MI355X at
    // 32 000 atoms and 20-step segments: 59 against 49 us per step)
    const bool graph_on = c->graph_on;
    c->graph_on = false;
    // second positions for the fused steps: lambda_x's place, unused until the
    // reverse pass
    KParams& k = c->kp;
    k.sx = arr(ws, L, L.lam, 0);
    k.sy = arr(ws, L, L.lam, 1);
    k.sz = arr(ws, L, L.lam, 2);
    for (int seg = 0; seg < L.nseg && st == MD_OK; ++seg) {
        checkpoint_arrays(ws, L, seg, ck);
        if ((st = checkpoint(c, ck, true)) != MD_OK) break;
        const int m = tp->n_steps - seg * L.k < L.k ? tp->n_steps - seg * L.k : L.k;
        st = md_step(c, m, 1);
    }
    c->graph_on = graph_on;
    k.sx = k.sy = k.sz = nullptr;  // (none of its own: reorder is off)
    if (st != MD_OK) return st;
    checkpoint_arrays(ws, L, L.nseg, ck);
    if ((st = checkpoint(c, ck, true)) != MD_OK) return st;
    launch_traj_ubar(c->kp, tp->n_steps, obs, c->stream);
    if (tp->n_bins > 0) {
        // a list built steps ago holds every pair only out to r_cut; the g(r)
        // range may reach r_cut + skin, so build it afresh at x_S
        rebuild_all(c);
        GrArgs g = gr_args(c, tp, ws, L);
        g.out = obs + 1;
        launch_gr(c->kp, g, c->stream);
    }
    return launched();
}

extern "C" md_status md_traj_backward(md_ctx* c, const md_traj_params* tp, void* ws,
                                      const double* grad_obs, double* grad_x0, double* grad_v0,
                                      double* grad_theta)
{
    TrajLayout L;
    md_status st = traj_check(c, tp, ws, &L);
    if (st != MD_OK) return st;
    if (!grad_obs || !grad_x0 || !grad_v0 || !grad_theta) return MD_ERR_ARG;
    const KParams& k = c->kp;
    hipStream_t sm = c->stream;
    const int S = tp->n_steps;
    const size_t n = (size_t)c->prm.n_atoms;
    double* lam[3] = {arr(ws, L, L.lam, 0), arr(ws, L, L.lam, 1), arr(ws, L, L.lam, 2)};
    double* vbuf[2][3] = {{arr(ws, L, L.lam, 3), arr(ws, L, L.lam, 4), arr(ws, L, L.lam, 5)},
                          {arr(ws, L, L.lam, 6), arr(ws, L, L.lam, 7), arr(ws, L, L.lam, 8)}};
    double* theta = reinterpret_cast<double*>(static_cast<char*>(ws) + L.theta);
    AdjArgs a;
    memset(&a, 0, sizeof(a));
    a.lx = lam[0];
    a.ly = lam[1];
    a.lz = lam[2];
    a.theta = theta;
    a.tpart = reinterpret_cast<double*>(static_cast<char*>(ws) + L.tpart);
    a.gobs = grad_obs;
    a.cap = k.scap_aux;
    int cur = 0;
    // one point: lambda_v of buffer cur in, of the other buffer out
    auto point = [&](double coef, double loss_scale, double drift) {
        a.vx = vbuf[cur][0];
        a.vy = vbuf[cur][1];
        a.vz = vbuf[cur][2];
        a.nx = vbuf[1 - cur][0];
        a.ny = vbuf[1 - cur][1];
        a.nz = vbuf[1 - cur][2];
        a.coef = coef;
        a.loss_scale = loss_scale;
        a.drift = drift;
        launch_adj_point(k, a, sm);
        cur = 1 - cur;
    };
    const double half = k.hdt;  // dt / 2m: one half kick
    const double lscale = 1.0 / ((double)S * (double)n);
    launch_fill(theta, 2, 0.0, sm);
    for (int d = 0; d < 3; ++d) launch_fill(vbuf[0][d], n, 0.0, sm);

    // the last point: the observables' direct dependence on x_S
    double* ck[6];
    checkpoint_arrays(ws, L, L.nseg, ck);
    launch_adj_reimage(k, ck[0], ck[1], ck[2], sm);
    launch_cells(k, 1, sm);
    launch_neighbors(k, 1, sm);
    if (tp->n_bins > 0) {
        GrArgs g = gr_args(c, tp, ws, L);
        g.gobs = grad_obs;
        g.lx = lam[0];
        g.ly = lam[1];
        g.lz = lam[2];
        launch_gr_grad(k, g, sm);
    } else {
        for (int d = 0; d < 3; ++d) launch_fill(lam[d], n, 0.0, sm);
    }
    point(0.0, lscale, k.dt);

    for (int seg = L.nseg - 1; seg >= 0; --seg) {
        const int s0 = seg * L.k;
        const int s1 = s0 + L.k < S ? s0 + L.k : S;
        // recompute the segment, keeping the positions of its inner points
        checkpoint_arrays(ws, L, seg, ck);
        if ((st = checkpoint(c, ck, false)) != MD_OK) return st;
        rebuild_all(c);
        // (the drifted positions go straight to where they are kept)
        KParams q = k;
        for (int j = 1; j < s1 - s0; ++j) {
            q.sx = arr(ws, L, L.snap, (size_t)(j - 1) * 3);
            q.sy = arr(ws, L, L.snap, (size_t)(j - 1) * 3 + 1);
            q.sz = arr(ws, L, L.snap, (size_t)(j - 1) * 3 + 2);
            if (j == 1)
                launch_integrate_pass(q, 0, sm, false, true);
            else
                launch_forces_step(q, sm);
            flip_positions(q);
            launch_finish_cells(q, 0, j == 1 ? 0 : 1, 0, j > 1, sm);
            launch_neighbors(q, 0, sm);
        }
        // walk it backwards
        for (int s = s1 - 1; s >= s0; --s) {
            const double* px[3];
            for (int d = 0; d < 3; ++d)
                px[d] = s == s0 ? ck[d] : arr(ws, L, L.snap, (size_t)(s - s0 - 1) * 3 + d);
            launch_adj_reimage(k, px[0], px[1], px[2], sm);
            launch_cells(k, 0, sm);
            launch_neighbors(k, 0, sm);
            // the first half kick of step s and the second of step s-1 (none
            // before step 0) act together; the mean energy counts x_1 .. x_S
            point(s == 0 ? half : 2.0 * half, s >= 1 ? lscale : 0.0, s >= 1 ? k.dt : 0.0);
        }
    }
    for (int d = 0; d < 3; ++d) {
        if (hipMemcpyAsync(grad_x0 + d * n, lam[d], sizeof(double) * n, hipMemcpyDeviceToDevice,
                           sm) != hipSuccess ||
            hipMemcpyAsync(grad_v0 + d * n, vbuf[cur][d], sizeof(double) * n,
                           hipMemcpyDeviceToDevice, sm) != hipSuccess)
            return MD_ERR_HIP;
    }
    if (hipMemcpyAsync(grad_theta, theta, 2 * sizeof(double), hipMemcpyDeviceToDevice, sm) !=
        hipSuccess)
        return MD_ERR_HIP;
    // back to the state at step S
    checkpoint_arrays(ws, L, L.nseg, ck);
    if ((st = checkpoint(c, ck, false)) != MD_OK) return st;
    rebuild_all(c);
    return launched();
}

extern "C" md_status md_history(md_ctx* c, md_record* out, int32_t max_records, int32_t* n_out)
{
    if (!c || !n_out || max_records < 0 || (max_records > 0 && !out)) return MD_ERR_ARG;
    if (!c->bound) return MD_ERR_NOT_BOUND;
    DevState d;
    if (hipMemcpyAsync(&d, c->kp.dev, sizeof(d), hipMemcpyDeviceToHost, c->stream) != hipSuccess)
        return MD_ERR_HIP;
    if (hipStreamSynchronize(c->stream) != hipSuccess) return MD_ERR_HIP;
    std::vector<md_record> ring(kHistCap);
    if (hipMemcpy(ring.data(), c->kp.hist, sizeof(md_record) * kHistCap,
                  hipMemcpyDeviceToHost) != hipSuccess)
        return MD_ERR_HIP;
    const int64_t total = d.hist_count;
    const int64_t avail = total < kHistCap ? total : kHistCap;
    const int64_t take = avail < max_records ? avail : max_records;
    const int64_t first = total - avail;  // oldest record still held
    for (int64_t r = 0; r < take; ++r) out[r] = ring[(first + r) % kHistCap];
    *n_out = (int32_t)take;
    return MD_OK;
}

static bool one_of(int v, std::initializer_list<int> set)
{
    for (int s : set)
        if (v == s) return true;
    return false;
}

extern "C" md_status md_set_tuning(md_ctx* c, const md_tuning* t)
{
    if (!c || !t) return MD_ERR_ARG;
    if (!one_of(t->force_lanes, {1, 2, 4, 8}) || t->force_block % 64 != 0 ||
        t->force_block < 64 || t->force_block > 1024 || t->nl_block % 64 != 0 ||
        t->nl_block < 0 || t->nl_block > 1024 || t->tile_cells < 0 || t->tile_y < 0 ||
        t->tile_z < 0 || t->stage_cap < 0 ||
        t->integrate_grid < 0 || t->integrate_grid > kIntegrateGridMax ||
        !one_of(t->nl_method, {MD_NL_AUTO, MD_NL_LANES, MD_NL_CELL_WAVES}))
        return MD_ERR_ARG;
    KParams& k = c->kp;
    drop_graph(c);  // launch shapes and parameters are baked into it
    const int old[4] = {k.n_tiles, k.kx_max, k.ky_max, k.kz_max};
    // the automatic shape also follows from the force pass's lanes and workgroup: under a
    // list that stands it is chosen again by the next list build, so that a change of
    // those alone leaves the list as it is
    const bool keep = c->nl_ok && t->tile_cells == c->tile_cells && t->tile_y == c->tile_y &&
                      t->tile_z == c->tile_z;
    k.force_lanes = t->force_lanes;
    k.force_block = t->force_block;
    c->nl_block_req = t->nl_block;
    c->nl_method_req = t->nl_method;
    k.int_grid = t->integrate_grid > 0 ? t->integrate_grid : kIntegrateGridDefault;
    c->stage_cap = t->stage_cap;
    c->tile_cells = t->tile_cells;
    c->tile_y = t->tile_y;
    c->tile_z = t->tile_z;
    plan_tiles(c, keep);
    // the list encoding depends on the tiling
    if (k.n_tiles != old[0] || k.kx_max != old[1] || k.ky_max != old[2] || k.kz_max != old[3])
        c->nl_ok = false;
    // the partials of the last force pass are laid out for the old grid
    c->forces_ok = false;
    return MD_OK;
}

extern "C" md_status md_get_tuning(const md_ctx* c, md_tuning* t)
{
    if (!c || !t) return MD_ERR_ARG;
    t->force_lanes = c->kp.force_lanes;
    t->force_block = c->kp.force_block;
    t->nl_block = c->kp.nl_block;
    t->integrate_grid = c->kp.int_grid;
    t->nl_method = c->kp.nl_method;
    t->tile_cells = c->tile_cells_res;
    t->tile_y = c->tile_y_res;
    t->tile_z = c->tile_z_res;
    t->stage_cap = c->kp.scap;
    return MD_OK;
}

extern "C" md_status md_set_timing(md_ctx* c, int32_t enable)
{
    if (!c) return MD_ERR_ARG;
    md_status st = fold_timing(c);
    c->timing = enable != 0;
    c->timed_ms = 0.0;
    c->timed_launches = 0;
    for (int k = 0; k < MD_PART_COUNT; ++k) {
        c->part_ms[k] = 0.0;
        c->part_launches[k] = 0;
    }
    return st;
}

extern "C" md_status md_get_timing_parts(md_ctx* c, double* ms, int64_t* launches)
{
    if (!c || !ms || !launches) return MD_ERR_ARG;
    md_status st = fold_timing(c);
    for (int k = 0; k < MD_PART_COUNT; ++k) {
        ms[k] = c->part_ms[k];
        launches[k] = c->part_launches[k];
    }
    return st;
}

extern "C" md_status md_get_timing(md_ctx* c, double* total_ms, int64_t* launches)
{
    if (!c || !total_ms || !launches) return MD_ERR_ARG;
    md_status st = fold_timing(c);
    *total_ms = c->timed_ms;
    *launches = c->timed_launches;
    return st;
}

extern "C" void md_destroy(md_ctx* c)
{
    if (!c) return;
    if (!c->ev_pending.empty() || c->gexec) (void)hipStreamSynchronize(c->stream);
    if (c->gstream) (void)hipStreamSynchronize(c->gstream);
    drop_graph(c);
    for (int e = 0; e < 2; ++e)
        if (c->gev[e]) (void)hipEventDestroy(c->gev[e]);
    if (c->gstream) (void)hipStreamDestroy(c->gstream);
    for (hipEvent_t e : c->ev_free) (void)hipEventDestroy(e);
    for (hipEvent_t e : c->ev_pending) (void)hipEventDestroy(e);
    delete c;
}
