// md_neighbors.hip -- step N5 of section 2.3: the neighbor matrix.
//
// One workgroup per tile (md_tiles.h) stages the tile's 27-cell
// neighborhoods in LDS.  A home atom's candidates are the three cells
// dx = -1, 0, +1 of each of the 9 staged rows next to its cell (dz, dy each
// -1, 0, +1, dz slowest), every cell in ascending permanent id; its list
// keeps them in that canonical order.  An entry is kept when the minimum-image squared
// separation is below (r_cut + skin)^2 (dx*dx, then two fused
// multiply-adds) and it is not the atom itself.  Two ways to walk them:
//
//   lanes (default)  one lane per home atom walks its 27 cells; entries are
//                    packed four to a chunk in a register and stored a
//                    chunk at a time
//   cell waves       one wave per home cell spreads the cell's candidates
//                    over its 64 lanes, 64 per round; for each home atom a
//                    ballot and a prefix count place the hits
//
// The half list (for the Newton's-third-law force pass) keeps a candidate
// only if it comes after the home atom in cell order (cell index, then
// permanent id).  That order is the order of the cell-ordered slots:
// candidate e of staged cell t sits at slot[t] + (e - off[t]), and so does the
// home atom, so the test is one integer comparison, and a
// staged cell whose last slot is not past the home atom's is skipped whole.
//
// Storage follows the paper's W (section 2.3): row m holds the m-th
// neighbor of every atom, so a wave of the force pass reads consecutive
// atoms' entries at consecutive addresses.  Entries are 16 bits (staged
// index + wrap bits), four to an 8-byte chunk: chunk c of slot k sits at
// 8-byte index c * n_pad + k.
#include "md_tiles.h"

namespace md {

// The lane, opaque to the compiler, taken anew for each home cell: the many
// addresses and masks formed from it would otherwise be computed once for all
// cells and spilled, a scratch store of about 160 bytes per lane and wave (more
// than the list itself).
__device__ __forceinline__ int cell_lane()
{
    int lane = threadIdx.x & (kWave - 1);
    asm volatile("" : "+v"(lane));
    return lane;
}

__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// The common cell-wave build (nl_home_cell_q): rounds of 64 candidates in
// registers (the first kRoundsLo always, the others when they hold any) and the
// candidates tested at a time; a wave's LDS holds the queue with a gather round
// past it, then in its place one list: at most kQueue hits behind an incomplete
// chunk, with their padding.
constexpr int kRoundsQ = 6, kRoundsLo = 4;
constexpr int kQueue = kRoundsQ * kWave;
constexpr size_t kCellWaveLds = 2 * (kQueue + kWave);

// LDS bytes of the list build: the staged tile, and with nl_queue the queues
// of the workgroup's waves.
size_t nl_lds_bytes(const KParams& p)
{
    return stage_bytes(p, p.scap) + (p.nl_queue ? kCellWaveLds * (size_t)(p.nl_block / kWave) : 0);
}

// The queues go with the cell-wave build of full lists, where they fit: a
// workgroup of nl_block threads in lds bytes (1 KiB spare for static LDS).
int nl_queue_fits(const KParams& p, int nl_method, int nl_block, size_t lds)
{
    return nl_method == MD_NL_CELL_WAVES && !p.newton3 && p.mode == MD_NEIGHBOR_LIST &&
           stage_bytes(p, p.scap) + kCellWaveLds * (size_t)(nl_block / kWave) + 1024 <= lds;
}

// Staged cell of column a - 1 in the row (dz, dy) = (sg / 3 - 1, sg % 3 - 1)
// next to home cell home_t (at column a): the first cell of window sg.
__device__ __forceinline__ int window_cell(const Stage& s, int home_t, int sg)
{
    const int dz = (sg >= 3 ? 1 : 0) + (sg >= 6 ? 1 : 0) - 1, dy = sg - 3 * (dz + 1) - 1;
    return home_t - 1 + (dz * s.rows_y + dy) * s.stride;
}

// Staged cell of home cell hc (0 .. kx ky kz - 1, x fastest).
__device__ __forceinline__ int home_cell(const Stage& s, int hc)
{
    const int a = 1 + hc % s.kx, r = hc / s.kx;
    return uniform(home_row_cell(s, r) + (a - 1));
}

// The lists of home cell hc's atoms, by one wave; wmax: the longest list of
// this wave's home atoms so far.  The candidates (the 9 windows of three cells
// next to it, concatenated, in canonical order) are taken kRounds x 64 at a
// time: lane l holds candidate k0 + 64 r + l (position, wrap bits, encoded
// entry) in registers.  Each home atom hh in turn is broadcast from lane hh
// (readlane) and tested against the block; for round r the hit ballot places
// the hits: a hit lane's entry goes to list position m_hh + (hits of lower
// lanes), m_hh being hh's running list length, kept in a scalar register while
// hh is tested and in lane hh of a vector register between blocks.  Lanes past
// the candidates read the home cell's first atom (e = hb) and never hit.
template <int kImage, bool kHalf, bool kFits, int kRounds, bool kFull>
__device__ __forceinline__ void nl_home_cell(const KParams& p, const Stage& s, int hc, bool small,
                                             int& wmax)
{
    const int lane = cell_lane();
    const int home_t = home_cell(s, hc);
    // table values are the same in every lane: keep them in scalar registers
    const int hb = uniform(s.off[home_t]), he = uniform(s.off[home_t + 1]);
    const int hslot0 = uniform(s.slot[home_t]);
    int wp[10];  // candidates before each window (the windows' own cells follow per lane)
    wp[0] = 0;
#pragma unroll
    for (int sg = 0; sg < 9; ++sg) {
        const int tw = window_cell(s, home_t, sg);
        wp[sg + 1] = wp[sg] + (uniform(s.off[tw + 3]) - uniform(s.off[tw]));
    }
    const int ncand = wp[9];
    const uint32_t cap = (uint32_t)p.cap;  // a multiple of 4
    uint16_t* nl16 = reinterpret_cast<uint16_t*>(p.nl64);
    const uint32_t npad4 = 4u * (uint32_t)p.npad;  // 16-bit entries per chunk row
    // small (the list within 32-bit byte offsets, rows within 24-bit products,
    // always so without kFull): hits go out as buffer stores, the list's base
    // in a resource, the home atom's chunk column as the scalar offset and row
    // and column of the entry as the 32-bit lane offset (no 64-bit address
    // arithmetic per hit).  With kFull the choice is a uniform branch at the
    // store (a second copy of the loop would raise the register count).
    const uint32_t rowb = 8u * (uint32_t)p.npad;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(p.nl64, 0, -1, kBufferWord3);
    for (int h0 = hb; h0 < he; h0 += kWave) {
        const int nhs = he - h0 < kWave ? he - h0 : kWave;
        const bool home_lane = lane < nhs;
        const int hl = h0 + (home_lane ? lane : 0);
        const int slot_l = atom_at(p, hslot0 + (hl - hb));
        double hx, hy, hz;
        if (kFits) {
            lds_xyz(s.p3, hl, hx, hy, hz);
        } else {
            hx = p.x[slot_l];
            hy = p.y[slot_l];
            hz = p.z[slot_l];
        }
        int mreg = 0;  // lane hh: home atom hh's list length so far
        for (int k0 = 0; k0 < ncand; k0 += kRounds * kWave) {
            double cx[kRounds], cy[kRounds], cz[kRounds];
            int ce[kRounds], cfl[kRounds], cpos[kRounds];
            uint16_t cenc[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int k = k0 + r * kWave + lane;
                const bool valid = k < ncand;
                int sg = 0, pre = 0;
#pragma unroll
                for (int j = 1; j < 9; ++j) {
                    sg += k >= wp[j] ? 1 : 0;
                    pre = k >= wp[j] ? wp[j] : pre;
                }
                const int t0 = window_cell(s, home_t, sg);
                const int e = valid ? s.off[t0] + (k - pre) : hb;
                const int w = (e >= s.off[t0 + 1] ? 1 : 0) + (e >= s.off[t0 + 2] ? 1 : 0);
                const int t = valid ? t0 + w : home_t;
                // lanes past the candidates: index -1 (never the home atom) and a
                // NaN position (never near, under any image rule)
                ce[r] = valid ? e : -1;
                cfl[r] = s.flag[t];
                cpos[r] = s.slot[t] + (e - s.off[t]);
                cenc[r] = (uint16_t)((uint32_t)e | ((uint32_t)cfl[r] << kEntryBits));
                if (kFits) {
                    lds_xyz(s.p3, e, cx[r], cy[r], cz[r]);
                } else {
                    const int j = atom_at(p, cpos[r]);
                    cx[r] = p.x[j];
                    cy[r] = p.y[j];
                    cz[r] = p.z[j];
                }
                if (!valid) cx[r] = __builtin_nan("");
            }
            for (int hh = 0; hh < nhs; ++hh) {
                const int eh = h0 + hh;
                const int pos_i = hslot0 + (eh - hb);
                // the home atom's position: with the tile staged, one LDS read that
                // the whole wave shares (its address is the same in every lane), which
                // measured 11% faster per build than six readlanes
                double xi, yi, zi;
                if (kFits) {
                    lds_xyz(s.p3, eh, xi, yi, zi);
                } else {
                    xi = readlane_f64(hx, hh);
                    yi = readlane_f64(hy, hh);
                    zi = readlane_f64(hz, hh);
                }
                const uint32_t slot4 = 4u * (uint32_t)__builtin_amdgcn_readlane(slot_l, hh);
                uint32_t m_h = (uint32_t)__builtin_amdgcn_readlane(mreg, hh);
                // the tests of all rounds first (independent), then the stores
                bool hit[kRounds];
                uint64_t mk[kRounds];
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    double dx = xi - cx[r], dy = yi - cy[r], dz = zi - cz[r];
                    image<kImage>(p, cfl[r], dx, dy, dz);
                    // each condition balloted on its own (the compare results are
                    // the lane masks; a ballot of their conjunction would turn
                    // them into a vector and back)
                    const bool near = dist2(dx, dy, dz) < p.rl2;
                    const bool other = ce[r] != eh;
                    const bool later = !kHalf || cpos[r] > pos_i;
                    mk[r] = __builtin_amdgcn_ballot_w64(near) & __builtin_amdgcn_ballot_w64(other);
                    if (kHalf) mk[r] &= __builtin_amdgcn_ballot_w64(later);
                    hit[r] = near & other & later;
                }
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    if (hit[r]) {
                        // position m_h plus the hits of lower lanes; past the
                        // capacity into the spare chunk row (counted, not kept)
                        uint32_t m = __builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(mk[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk[r], m_h));
                        m = m < cap ? m : cap;
                        if (!kFull || small) {
                            // row (m >> 2) of rowb bytes, entry m & 3 of the chunk:
                            // 2 m + (m >> 2) (rowb - 8), one 24-bit multiply-add
                            uint32_t off;
                            asm("v_mad_u32_u24 %0, %1, %2, %3"
                                : "=v"(off)
                                : "v"(m >> 2), "s"(rowb - 8u), "v"(2u * m));
                            __builtin_amdgcn_raw_buffer_store_b16(cenc[r], rsrc, (int)off,
                                                                  (int)(2u * slot4), 0);
                        } else {
                            nl16[(size_t)(m >> 2) * npad4 + ((m & 3u) | slot4)] = cenc[r];
                        }
                    }
                    m_h += (uint32_t)__popcll(mk[r]);
                }
                mreg = lane == hh ? (int)m_h : mreg;
            }
        }
        // lengths, sentinel padding of the last chunk
        if (home_lane) {
            const int stored = mreg < (int)cap ? mreg : (int)cap;
            p.nl_count[slot_l] = stored;
            uint16_t* base = nl16 + (int64_t)slot_l * kChunk;
            for (int mm = stored; mm % kChunk != 0; ++mm)
                base[(int64_t)(mm / kChunk) * npad4 + mm % kChunk] = (uint16_t)s.total;
        }
        const int longest = wave_max(home_lane ? mreg : 0);
        wmax = longest > wmax ? longest : wmax;
    }
}

// ---- the common cell-wave build: full lists, atoms staged in LDS, at least 5
// cells per side ----
//
// Two phases per home cell, by one wave.  Gather: the candidates (the 9 windows
// of three cells, in canonical order) that lie within the list radius of the
// bounding box of the home cell's atoms go, in order, to a queue in LDS (of 533
// candidates at the dense LJ state about 350 stay).  Test: up to kQueue queued
// candidates at a time are held in registers, 64 per round; each home atom in
// turn is tested against all rounds, the hits' entries go to their places in
// a buffer in LDS, and from there whole 8-byte chunks are stored, a lane per
// chunk.
//
// Bound by instruction issue, vector and scalar together (2.048M LJ atoms: 439 M
// vector and 156 M scalar instructions in the earlier build, which tested all
// 533 candidates and stored entry by entry).  Forced builds: 830 -> 668 us at
// 2.048M LJ atoms, 91 -> 60 us at 100 003, 93 -> 70 us at 32 000, 38 -> 32 us at
// 10 007 (the latter two 39 and 21 us with each cell's atoms shared by several
// waves, see plan_tiles).  Storing eight lists together, a row of their chunks as one run of 64
// bytes, took an eighth of the write requests and was slower (817 us): requests
// do not bound it.

__device__ __forceinline__ void lds_order()
{
    // the wave's LDS operations complete in order; this keeps the compiler from
    // moving them past each other
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Largest and smallest f over the wave's lanes, for values whose FP32 bits are
// ordered as unsigned integers (f >= 0): one DPP instruction per step.
__device__ __forceinline__ uint32_t wave_umax(uint32_t v)
{
    v = max(v, dpp_read<0x111, 0xf, false>(v, v));
    v = max(v, dpp_read<0x112, 0xf, false>(v, v));
    v = max(v, dpp_read<0x114, 0xf, false>(v, v));
    v = max(v, dpp_read<0x118, 0xf, false>(v, v));
    v = max(v, dpp_read<0x142, 0xa, false>(v, v));
    v = max(v, dpp_read<0x143, 0xc, false>(v, v));
    return from_lane63(v);
}

// Middle and half width, rounded outward past the FP32 conversion, of the
// interval the lanes' v span.  The order of the bits and the slack hold for v of
// [-L, 3 L); an atom that left the box by more, which folding by one box length
// leaves in a cell at its edge, or a NaN, makes the half width infinite (the middle
// then still lies on the cell's side of the box, as near_image needs).
__device__ __forceinline__ void wave_span(const KParams& p, double v, double& mid, double& half)
{
    const uint32_t b = __builtin_bit_cast(uint32_t, (float)__builtin_fma(v, p.invL, 1.0));
    const uint32_t bh = wave_umax(b);
    const double hi = (double)__builtin_bit_cast(float, bh);
    const double lo = (double)__builtin_bit_cast(float, ~wave_umax(~b));
    mid = __builtin_fma(0.5 * (lo + hi), p.L, -p.L);
    half = __builtin_fma(0.5 * (hi - lo), p.L, p.box_slack);
    if (bh >= 0x40800000u) half = __builtin_inf();  // 4.0f, or a negative number
}

// The image of candidate (cx, cy, cz) on the side of (bx, by, bz) in each
// flagged coordinate (see image).
__device__ __forceinline__ void near_image(const KParams& p, int fl, double bx, double by,
                                           double bz, double& cx, double& cy, double& cz)
{
    if (fl & 1) cx += bx > cx ? p.L : -p.L;
    if (fl & 2) cy += by > cy ? p.L : -p.L;
    if (fl & 4) cz += bz > cz ? p.L : -p.L;
}

// The lists of the atoms of home cell hc, of them part i of split near-equal ones (see
// above).  q: this wave's LDS: the queue and, once a block's candidates
// are in registers, one list in its place.  small, wmax as nl_home_cell.
template <int kImage, bool kFull>
__device__ __forceinline__ void nl_home_cell_q(const KParams& p, const Stage& s, int hc, int i,
                                               int split, bool small, MD_LDS uint16_t* q,
                                               int& wmax)
{
    const int lane = cell_lane();
    const int home_t = home_cell(s, hc);
    int hb = uniform(s.off[home_t]), he = uniform(s.off[home_t + 1]);
    int hslot0 = uniform(s.slot[home_t]);
    if (split > 1) {
        const int n = he - hb, first = uniform(n * i / split);
        he = hb + uniform(n * (i + 1) / split);
        hb += first;
        hslot0 += first;
    }
    MD_LDS uint64_t* const q64 = (MD_LDS uint64_t*)q;
    const uint32_t cap = (uint32_t)p.cap;  // a multiple of 4
    const uint32_t rowb = 8u * (uint32_t)p.npad;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(p.nl64, 0, -1, kBufferWord3);
    // slightly past the list radius: the box test rounds differently from the
    // inclusion test and only has to keep whatever that one could accept
    const double reach2 = p.box_reach2;
    for (int h0 = hb; h0 < he; h0 += kWave) {
        const int nhs = he - h0 < kWave ? he - h0 : kWave;
        const bool home_lane = lane < nhs;
        const int hl = h0 + (home_lane ? lane : 0);
        const int slot_l = atom_at(p, hslot0 + (hl - hb));
        int mreg = 0;        // lane hh: home atom hh's list length so far
        uint64_t part = 0;   // lane hh: its last, incomplete chunk
        int qn = 0;          // candidates queued
        int sg = 0, e0 = 0, ee = 0, t0 = 0;  // window being gathered: entries e0 .. ee - 1 left
        bool more = true;
        while (more) {
            // the home atoms' box: middle, half widths (anew for each block of candidates, of
            // which most cells have one: kept across the tests it would be spilled)
            double bx, by, bz, wx, wy, wz;
            {
                double hx, hy, hz;
                lds_xyz(s.p3, hl, hx, hy, hz);
                wave_span(p, hx, bx, wx);
                wave_span(p, hy, by, wy);
                wave_span(p, hz, bz, wz);
            }
            // gather until the queue is full or the windows end
            while (qn < kQueue) {
                if (e0 >= ee) {
                    if (sg == 9) break;
                    t0 = window_cell(s, home_t, sg);
                    e0 = uniform(s.off[t0]);
                    ee = uniform(s.off[t0 + 3]);
                    ++sg;
                    continue;
                }
                const int e = e0 + lane;
                const int ev = e < ee ? e : hb;
                double cx, cy, cz;
                lds_xyz(s.p3, ev, cx, cy, cz);
                int fl = 0;
                if (kImage == 1) {
                    const int t = t0 + (e >= s.off[t0 + 1] ? 1 : 0) + (e >= s.off[t0 + 2] ? 1 : 0);
                    fl = e < ee ? s.flag[t] : 0;
                    near_image(p, fl, bx, by, bz, cx, cy, cz);
                }
                const double dx = fmax(fabs(cx - bx) - wx, 0.0);
                const double dy = fmax(fabs(cy - by) - wy, 0.0);
                const double dz = fmax(fabs(cz - bz) - wz, 0.0);
                // (a NaN position stays: under the inclusion test it never hits)
                const int left = ee - e0;
                const uint64_t in = left >= kWave ? ~0ull : (1ull << left) - 1ull;
                const uint64_t mk =
                    in & ~__builtin_amdgcn_ballot_w64(dist2(dx, dy, dz) > reach2);
                if (__builtin_amdgcn_inverse_ballot_w64(mk)) {
                    const uint32_t m = __builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, (uint32_t)qn));
                    q[m] = (uint16_t)((uint32_t)e | ((uint32_t)fl << kEntryBits));
                }
                qn += (int)__popcll(mk);
                e0 += kWave;
            }
            more = e0 < ee || sg < 9 || qn > kQueue;
            const int nb = qn < kQueue ? qn : kQueue;  // candidates of this block
            lds_order();
            double cx[kRoundsQ], cy[kRoundsQ], cz[kRoundsQ];
            uint32_t enc[kRoundsQ];
#pragma unroll
            for (int r = 0; r < kRoundsQ; ++r) {
                const int k = r * kWave + lane;
                const uint32_t v = q[k];  // past nb: whatever was there, inside the staging
                enc[r] = k < nb ? v : (uint32_t)hb;
            }
            const uint16_t rest = q[kQueue + lane];  // gathered past this block (none, or few)
#pragma unroll
            for (int r = 0; r < kRoundsQ; ++r) {
                lds_xyz(s.p3, (int)(enc[r] & kEntryMask), cx[r], cy[r], cz[r]);
                if (kImage == 1)
                    near_image(p, (int)(enc[r] >> kEntryBits), bx, by, bz, cx[r], cy[r], cz[r]);
                if (r * kWave + lane >= nb) cx[r] = __builtin_nan("");  // never near
            }
            lds_order();
            for (int hh = 0; hh < nhs; ++hh) {
                double xi, yi, zi;
                lds_xyz(s.p3, h0 + hh, xi, yi, zi);  // one read the whole wave shares
                const uint32_t m0 = (uint32_t)__builtin_amdgcn_readlane(mreg, hh);
                const uint32_t slot = (uint32_t)__builtin_amdgcn_readlane(slot_l, hh);
                uint64_t mk[kRoundsQ];
                auto test = [&](int r) {
                    const double dx = xi - cx[r], dy = yi - cy[r], dz = zi - cz[r];
                    const double r2 = dist2(dx, dy, dz);
                    mk[r] = __builtin_amdgcn_ballot_w64(r2 < (kImage == 1 ? p.rl2_in : p.rl2));
                    // the image was taken before the difference: where that could
                    // decide, once more as the inclusion test rounds it
                    if (kImage == 1 && __builtin_amdgcn_ballot_w64(r2 < reach2) != mk[r]) {
                        double ex, ey, ez;
                        lds_xyz(s.p3, (int)(enc[r] & kEntryMask), ex, ey, ez);
                        ex = xi - ex;
                        ey = yi - ey;
                        ez = zi - ez;
                        image<1>(p, (int)(enc[r] >> kEntryBits), ex, ey, ez);
                        mk[r] = __builtin_amdgcn_ballot_w64(r2 == r2 && dist2(ex, ey, ez) < p.rl2);
                    }
                    // not the atom itself (its entry has no wrap bits)
                    mk[r] &= __builtin_amdgcn_ballot_w64(enc[r] != (uint32_t)(h0 + hh));
                };
                // the hits of round r to the buffer from entry `at` on
                auto place = [&](int r, uint32_t at) {
                    MD_LDS uint16_t* const to = q + at;
                    if (__builtin_amdgcn_inverse_ballot_w64(mk[r]))
                        to[__builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(mk[r] >> 32),
                            __builtin_amdgcn_mbcnt_lo((uint32_t)mk[r], 0u))] = (uint16_t)enc[r];
                };
                // (opaque, so that no address or value formed from them is kept across
                // the loop: kept, they spill, and their reloads wait for every store in
                // flight)
                int nbs = nb, ln = lane, pad = uniform(s.total);
                asm volatile("" : "+s"(nbs), "+v"(ln), "+s"(pad));
                // independent tests first, then the hits, behind the incomplete chunk
#pragma unroll
                for (int r = 0; r < kRoundsLo; ++r) test(r);
                uint32_t m = m0 % kChunk;
                if (m != 0 && ln == hh) q64[0] = part;
                lds_order();
#pragma unroll
                for (int r = 0; r < kRoundsLo; ++r) {
                    place(r, m);
                    m += (uint32_t)__popcll(mk[r]);
                }
                if (nbs > kRoundsLo * kWave) {
#pragma unroll
                    for (int r = kRoundsLo; r < kRoundsQ; ++r) test(r);
#pragma unroll
                    for (int r = kRoundsLo; r < kRoundsQ; ++r) {
                        place(r, m);
                        m += (uint32_t)__popcll(mk[r]);
                    }
                }
                // the whole chunks to rows m0 / 4 ..; in the last block the rest too,
                // padded with the sentinel
                uint32_t n = m / kChunk;
                if (!more) {
                    if (ln < kChunk) q[m + ln] = (uint16_t)pad;
                    n = (m + kChunk - 1) / kChunk;
                }
                lds_order();
                const uint32_t row0 = m0 / kChunk, rows = cap / kChunk;
                for (uint32_t c0 = 0; c0 < n; c0 += kWave) {
                    const uint32_t c = c0 + ln;
                    if (c < n && row0 + c < rows) {  // past the capacity: not kept
                        const uint64_t ch = q64[c];
                        if (!kFull || small) {
                            typedef int v2i __attribute__((ext_vector_type(2)));
                            __builtin_amdgcn_raw_buffer_store_b64(
                                __builtin_bit_cast(v2i, ch), rsrc, (int)((uint32_t)ln * rowb),
                                (int)((row0 + c0) * rowb + 8u * slot), 0);
                        } else {
                            p.nl64[(int64_t)(row0 + c) * p.npad + slot] = ch;
                        }
                    }
                }
                if (more) {
                    const uint64_t ch = q64[n];
                    part = ln == hh ? ch : part;
                }
                lds_order();
                const uint32_t len = m0 / kChunk * kChunk + m;
                mreg = ln == hh ? (int)len : mreg;
                wmax = (int)len > wmax ? (int)len : wmax;
            }
            q[lane] = rest;
            lds_order();
            qn -= nb;
        }
        if (home_lane) p.nl_count[slot_l] = mreg < (int)cap ? mreg : (int)cap;
    }
}

// True when home cell hc (0 .. kx ky kz - 1, x fastest) of tile g lies on a
// periodic boundary: some of its 26 neighbor cells wrap.
__device__ __forceinline__ bool home_wraps(const KParams& p, const Tile& g, int hc)
{
    const int a = hc % g.kx, r = hc / g.kx, b = r % g.ky, c = r / g.ky;
    const int xx = g.cx0 + a, yy = g.cy0 + b, zz = g.cz0 + c, e = p.nc - 1;
    return xx == 0 || xx == e || yy == 0 || yy == e || zz == 0 || zz == e;
}

// Home cell of row cell t1 (column 1 of its home row) holding staged entry e.
__device__ __forceinline__ int home_column_cell(const Stage& s, int t1, int e)
{
    int lo = 0, hi = s.kx - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s.off[t1 + mid] <= e)
            lo = mid;
        else
            hi = mid - 1;
    }
    return t1 + lo;
}

// Wrap bits of staged entry e of a run of three cells, the second and third from
// entries b1 and b2 on.
__device__ __forceinline__ int run_flag(int e, int b1, int b2, int fl0, int fl1, int fl2)
{
    return e < b1 ? fl0 : (e < b2 ? fl1 : fl2);
}

// The list of home atom h, by one lane.  Returns the number of entries found
// (beyond the capacity: overflow).
//
// Bound by instruction issue.  With the candidates in LDS a window's are tested
// first, four at a time, one bit each of a mask (eight instructions a candidate and
// no branch); then the set bits are taken in order, as many rounds as the fullest
// lane has hits.  (A branch per candidate to the code of a hit runs that code for
// nearly every candidate, since some lane of the wave hits: builds of 64 replicas
// 194 us so and 163 with masks, of 262 144 melt atoms 45 and 42, of 256 000 WCA atoms
// 42.5 and 41.5.)  A hit shifts its entry into the top of the chunk; count and
// capacity are looked at where a chunk is full.
template <int kImage, bool kFits, bool kHalf>
__device__ __forceinline__ int nl_home_atom(const KParams& p, const Stage& s, int h)
{
    int e_self, pos_i, t1;
    home_atom(s, h, e_self, pos_i, t1);
    const int home_t = home_column_cell(s, t1, e_self);
    const int slot_i = atom_at(p, pos_i);
    double xi, yi, zi;
    if (kFits) {
        lds_xyz(s.p3, e_self, xi, yi, zi);
    } else {
        xi = p.x[slot_i];
        yi = p.y[slot_i];
        zi = p.z[slot_i];
    }
    const uint32_t cap = (uint32_t)p.cap;  // a multiple of 4
    uint64_t* col = p.nl64 + slot_i;
    uint32_t lo = 0, hi = 0;  // the last four entries found, the newest on top
    uint32_t m = 0;
    auto hit = [&](int e, int fl) {
        const uint32_t v = (uint32_t)e | ((uint32_t)fl << kEntryBits);
        lo = __builtin_amdgcn_alignbit(hi, lo, 16);
        hi = __builtin_amdgcn_alignbit(v, hi, 16);
        ++m;
        if (m % kChunk == 0) {
            if (m <= cap) *col = (uint64_t)hi << 32 | lo;
            col += p.npad;
        }
    };
    for (int sg = 0; sg < 9; ++sg) {
        const int tw = window_cell(s, home_t, sg);
        if constexpr (kFits && !kHalf) {
            // The three cells of a window are one run of staged atoms.  In a tile with
            // no wrapped cell, or staged as periodic images (kShifted, see
            // stage_atoms), the raw separation is the minimum image; a shifted
            // partner's differs from that of the wrap bits by roundings, so a pair
            // within those of the list radius is decided by the wrap bits.
            constexpr bool kShifted = kImage == 1;
            const double reach2 = kShifted ? p.box_reach2 : p.rl2;
            const int eb = s.off[tw], ee = s.off[tw + 3];
            int b1 = 0, b2 = 0, fl0 = 0, fl1 = 0, fl2 = 0;
            if (kImage != 0) {
                b1 = s.off[tw + 1];
                b2 = s.off[tw + 2];
                fl0 = s.flag[tw];
                fl1 = s.flag[tw + 1];
                fl2 = s.flag[tw + 2];
            }
            for (int e0 = eb; e0 < ee; e0 += 32) {
                const int n = ee - e0 < 32 ? ee - e0 : 32;
                uint32_t in = 0, sure = 0;
                for (int k = 0; k < n; k += 4) {
                    // past the run: up to three entries of other cells or of the
                    // tables behind the staged atoms, masked below
                    uint32_t in4 = 0, sure4 = 0;
#pragma unroll
                    for (int u = 3; u >= 0; --u) {
                        double xj, yj, zj;
                        lds_xyz(s.p3, e0 + k + u, xj, yj, zj);
                        double dx = xi - xj, dy = yi - yj, dz = zi - zj;
                        image<kShifted ? 0 : kImage>(p, 0, dx, dy, dz);
                        const double r2 = dist2(dx, dy, dz);
                        in4 = in4 + in4 + (r2 < reach2 ? 1u : 0u);
                        if (kShifted) sure4 = sure4 + sure4 + (r2 < p.rl2_in ? 1u : 0u);
                    }
                    in |= in4 << k;
                    sure |= sure4 << k;
                }
                in &= 0xffffffffu >> (32 - n);
                if (sg == 4 && (uint32_t)(e_self - e0) < 32u) in &= ~(1u << (e_self - e0));
                if (kShifted) {
                    for (uint32_t edge = in & ~sure; edge != 0; edge &= edge - 1) {
                        const int e = e0 + __builtin_ctz(edge);
                        const int j = staged_slot(p, s, e);
                        double dx = xi - p.x[j], dy = yi - p.y[j], dz = zi - p.z[j];
                        image<1>(p, run_flag(e, b1, b2, fl0, fl1, fl2), dx, dy, dz);
                        if (!(dist2(dx, dy, dz) < p.rl2)) in &= ~(edge & -edge);
                    }
                }
                for (; in != 0; in &= in - 1) {
                    const int e = e0 + __builtin_ctz(in);
                    hit(e, kImage == 0 ? 0 : run_flag(e, b1, b2, fl0, fl1, fl2));
                }
            }
        } else {
            constexpr int kRuns = kImage == 0 ? 1 : 3;
#pragma unroll
            for (int w = 0; w < kRuns; ++w) {
                const int t = tw + w;
                const int eb = s.off[t], ee = s.off[t + (kRuns == 1 ? 3 : 1)];
                const int fl = kImage == 0 ? 0 : s.flag[t], tslot = s.slot[t];
                if (kHalf && tslot + (ee - eb) <= pos_i) continue;
                for (int e = eb; e < ee; ++e) {
                    double xj, yj, zj;
                    if (kFits) {
                        lds_xyz(s.p3, e, xj, yj, zj);
                    } else {
                        const int j = atom_at(p, tslot + (e - eb));
                        xj = p.x[j];
                        yj = p.y[j];
                        zj = p.z[j];
                    }
                    double dx = xi - xj, dy = yi - yj, dz = zi - zj;
                    image<kImage>(p, fl, dx, dy, dz);
                    const bool later = !kHalf || tslot + (e - eb) > pos_i;
                    if (later && dist2(dx, dy, dz) < p.rl2 && e != e_self) hit(e, fl);
                }
            }
        }
    }
    const uint32_t stored = m < cap ? m : cap;
    if (m < cap && m % kChunk != 0) {  // pad the last chunk with the sentinel
        for (uint32_t mm = m % kChunk; mm < kChunk; ++mm) {
            lo = __builtin_amdgcn_alignbit(hi, lo, 16);
            hi = __builtin_amdgcn_alignbit((uint32_t)s.total, hi, 16);
        }
        *col = (uint64_t)hi << 32 | lo;
    }
    p.nl_count[slot_i] = (int)stored;
    return (int)m;
}

template <int kImage, bool kFits, bool kHalf>
__device__ __forceinline__ void nl_lanes(const KParams& p, const Stage& s, int& wmax)
{
    const int nh = home_count(s);
    for (int h = threadIdx.x; h < nh; h += blockDim.x) {
        const int m = nl_home_atom<kImage, kFits, kHalf>(p, s, h);
        wmax = m > wmax ? m : wmax;
    }
}

// One tile's lists (every thread of the workgroup calls it); wmax: the longest
// list this thread has seen (its wave's, in the cell-wave build).  kFull: the
// image rule of grids under 5 cells per side (mode 2) and list stores beyond
// 32-bit offsets are compiled in; a kernel without them serves only grids of 5
// cells per side or more whose lists fit the buffer stores, and holds fewer
// registers.  kQueue: the cell waves have their queues
// (KParams::nl_queue; in a batch, those of some replica).
template <int kMethod, bool kHalf, bool kCopy, bool kFull, bool kQueue>
__device__ __forceinline__ void nl_tile(const KParams& p, int t, char* smem, int& wmax)
{
    const Tile g = tile_of(p, t);
    Stage s = stage_layout(p, smem);
    stage_tables(p, g, s);
    if (s.total >= kMaxStaged) {
        // the 13-bit entry cannot address this tile (and its sentinel): report it
        // as an overflow
        const int nh = home_count(s);
        for (int h = threadIdx.x; h < nh; h += blockDim.x) {
            int e, pos;
            home_atom(s, h, e, pos);
            p.nl_count[atom_at(p, pos)] = 0;
            copy_home<kCopy>(p, atom_at(p, pos));
        }
        if (threadIdx.x == 0) atomicOr(&p.dev->flags, (int)MD_FLAG_NL_OVERFLOW);
        return;
    }
    // the displacement references and the folded copy-back of the tile's home atoms,
    // a thread per atom, while the staging loads are under way (in cell waves a lane
    // per atom of the home cell at its end used a third of the lanes, one cell after
    // the other: 190 us of a build at 2.048M LJ atoms)
    const int nh = home_count(s);
    for (int h = threadIdx.x; h < nh; h += blockDim.x) {
        int e, pos;
        home_atom(s, h, e, pos);
        const int k = atom_at(p, pos);
        p.xr[k] = p.x[k];
        p.yr[k] = p.y[k];
        p.zr[k] = p.z[k];
        copy_home<kCopy>(p, k);
    }
    if constexpr (kMethod == MD_NL_LANES && !kHalf)
        stage_positions_imaged(p, s);
    else
        stage_positions(p, s);
    __syncthreads();
    const int mode = image_mode(p, tile_interior(p, g));
    if (kMethod == MD_NL_LANES) {
        if (kFull && mode == 2) {
            if (s.fits)
                nl_lanes<2, true, kHalf>(p, s, wmax);
            else
                nl_lanes<2, false, kHalf>(p, s, wmax);
        } else if (!s.fits) {
            nl_lanes<1, false, kHalf>(p, s, wmax);
        } else if (mode == 0) {
            nl_lanes<0, true, kHalf>(p, s, wmax);
        } else {
            nl_lanes<1, true, kHalf>(p, s, wmax);
        }
        return;
    }
    const int wid = uniform((int)threadIdx.x / kWave), nw = blockDim.x / kWave;
    const int ncells = g.kx * g.ky * g.kz;
    const bool small = nl_small(p);
    // this wave's queue and list buffer, behind the tables
    MD_LDS uint16_t* const queue =
        (MD_LDS uint16_t*)((MD_LDS char*)smem + stage_bytes(p, p.scap) + wid * kCellWaveLds);
    // Home cells next to a periodic boundary (real index 0 or nc - 1 on some
    // axis) have wrapped candidates and take the image rule; the other home
    // cells of a boundary tile have none and take the interior path.  The rare
    // tiles that do not fit in LDS, and grids under 5 cells per side, take one
    // round of 64 candidates at a time: those paths then hold fewer registers
    // than the common ones (the kernel's register count is that of its largest
    // path), which keeps six waves per SIMD.
    // More waves than home cells: the cells' atoms are split among them (few tiles,
    // whose waves would leave the CUs idle; see plan_tiles).
    const bool share = kQueue && p.nl_queue && s.fits && mode != 2 && nw > ncells;
    const int split = share ? nw / ncells : 1;
    for (int u = wid; u < ncells * split; u += nw) {
        const int hc = split > 1 ? uniform(u / split) : u, part = u - hc * split;
        if (kFull && mode == 2) {
            if (s.fits)
                nl_home_cell<2, kHalf, true, 1, kFull>(p, s, hc, small, wmax);
            else
                nl_home_cell<2, kHalf, false, 1, kFull>(p, s, hc, small, wmax);
        } else if (!s.fits) {
            nl_home_cell<1, kHalf, false, 1, kFull>(p, s, hc, small, wmax);
        } else if (mode == 0 || !home_wraps(p, g, hc)) {
            if constexpr (!kQueue)
                nl_home_cell<0, kHalf, true, kNlRounds, kFull>(p, s, hc, small, wmax);
            else if (p.nl_queue)
                nl_home_cell_q<0, kFull>(p, s, hc, part, split, small, queue, wmax);
            else  // a replica without room for them, beside others
                nl_home_cell<0, kHalf, true, 1, kFull>(p, s, hc, small, wmax);
        } else {
            if constexpr (!kQueue)
                nl_home_cell<1, kHalf, true, kNlRounds, kFull>(p, s, hc, small, wmax);
            else if (p.nl_queue)
                nl_home_cell_q<1, kFull>(p, s, hc, part, split, small, queue, wmax);
            else  // a replica without room for them, beside others
                nl_home_cell<1, kHalf, true, 1, kFull>(p, s, hc, small, wmax);
        }
    }
}

// The list build, gated by the rebuild flag: one workgroup per tile, in the
// XCD-aware order (grid rule G_NL; a capped grid looping over tiles idles less
// per launch but measured slower per rebuild, from the uneven tile counts of the
// last wave of workgroups).
// At most 80 VGPRs: six waves per SIMD, which the LDS of the dense LJ tiles
// (three workgroups of eight waves per CU) allows.
template <class B, int kMethod, bool kHalf, bool kCopy, bool kFull, bool kQueue>
__global__ __attribute__((amdgpu_waves_per_eu(6))) void k_nl_tiles(B b, int force)
{
    Wg wg;
    KParams p;
    if (!b.fetch_gated(G_NL, force, wg, p)) return;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const KParams q = kCopy ? scratch_view(p) : p;
    int wmax = 0;
    nl_tile<kMethod, kHalf, kCopy, kFull, kQueue>(q, xcd_tile(wg.id, wg.n), smem, wmax);
    // the longest list: one global atomic per workgroup
    const int mmax = workgroup_max(wmax);
    if (threadIdx.x == 0 && mmax > 0) {
        atomicMax(&q.dev->max_nl, mmax);
        if (mmax > q.cap) atomicOr(&q.dev->flags, (int)MD_FLAG_NL_OVERFLOW);
    }
}

// Decode the list into global slots: out[m * n_pad + k] for m < count[k],
// -1 elsewhere.
__global__ void k_nl_export(KParams p, int32_t* out)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const Tile g = tile_of(p, xcd_tile(blockIdx.x, gridDim.x));
    Stage s = stage_layout(p, smem);
    stage_tables(p, g, s);
    const int nh = home_count(s);
    for (int h = threadIdx.x; h < nh; h += blockDim.x) {
        int e, pos;
        home_atom(s, h, e, pos);
        const int k = atom_at(p, pos), cnt = p.nl_count[k];
        for (int m = 0; m < p.cap; ++m) {
            int v = -1;
            if (m < cnt) {
                const uint64_t ch = p.nl64[(int64_t)(m / kChunk) * p.npad + k];
                const int e = (int)((ch >> (16 * (m % kChunk))) & kEntryMask);
                v = e < s.total ? staged_slot(p, s, e) : -2;
            }
            out[(int64_t)m * p.npad + k] = v;
        }
    }
}

template <class B, bool kHalf, bool kCopy, bool kFull>
static void neighbors_seq(const B& b, const LaunchShape& sh, int force, hipStream_t s)
{
    const dim3 g(sh.grid[G_NL]), t(sh.nl_block);
    if (sh.nl_method != MD_NL_CELL_WAVES) {
        hipLaunchKernelGGL((k_nl_tiles<B, MD_NL_LANES, kHalf, kCopy, kFull, false>), g, t,
                           sh.nl_lds, s, b, force);
        return;
    }
    if constexpr (!kHalf) {
        if (sh.nl_queue) {
            hipLaunchKernelGGL((k_nl_tiles<B, MD_NL_CELL_WAVES, kHalf, kCopy, kFull, true>), g, t,
                               sh.nl_lds, s, b, force);
            return;
        }
    }
    hipLaunchKernelGGL((k_nl_tiles<B, MD_NL_CELL_WAVES, kHalf, kCopy, kFull, false>), g, t,
                       sh.nl_lds, s, b, force);
}

template <class B, bool kHalf, bool kCopy>
static void neighbors_seq(const B& b, const LaunchShape& sh, int force, hipStream_t s)
{
    if (sh.nl_full)
        neighbors_seq<B, kHalf, kCopy, true>(b, sh, force, s);
    else
        neighbors_seq<B, kHalf, kCopy, false>(b, sh, force, s);
}

template <class B>
static void neighbors_seq(const B& b, const LaunchShape& sh, int flags, hipStream_t s)
{
    const int force = flags & 1;
    const bool copy = (flags & kFoldCopy) && sh.reorder;
    if (sh.newton3)
        copy ? neighbors_seq<B, true, true>(b, sh, force, s)
             : neighbors_seq<B, true, false>(b, sh, force, s);
    else
        copy ? neighbors_seq<B, false, true>(b, sh, force, s)
             : neighbors_seq<B, false, false>(b, sh, force, s);
}

void launch_neighbors(const KParams& p, int force, hipStream_t s)
{
    neighbors_seq(Single{p}, shape_of(p), force, s);
}

void launch_neighbors(const Batch& b, const LaunchShape& sh, int force, hipStream_t s)
{
    neighbors_seq(b, sh, force, s);
}

void launch_nl_export(const KParams& p, int32_t* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_nl_export, dim3(p.n_tiles), dim3(p.nl_block),
                       nl_lds_bytes(p), s, p, out);
}

}  // namespace md
