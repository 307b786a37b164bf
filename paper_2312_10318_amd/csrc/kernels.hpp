// kernels.hpp -- host-side launchers of the device kernels (internal to the
// library; the public interface is include/trtlbm.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lattice.hpp"

namespace trt {

struct Launch {
    int rows_per_wave;    // 0: chosen per lattice by auto_rows()
    int waves_per_block;  // 0: chosen per storage and column mode
    int xcd_remap;
    int cols_per_lane;    // 0: two-column strips wherever they apply; 1 or 2
    // batches only (see trt_tuning): the minimum number of work items that
    // sets one batch-wide row cap (-1: each member's own rows), and the
    // work-list order (1: member by member, 2: costliest items first)
    int batch_items;
    int batch_order;
    int graph_steps;  // sweeps per captured graph (even)
    int steps_per_sweep;  // 2 or 3: time steps per launch where tb2_eligible / tb3_eligible
    int prefetch_rows;    // two-step pass: loads 1 or 2 rows ahead (0: automatic)
    int remap_asked;      // xcd_remap was set by the caller (else the pass's default)
};

// Whether the passes are the library's choice: no field is set that describes one.
inline bool automatic(const Launch &l) {
    return l.rows_per_wave == 0 && l.waves_per_block == 0 && l.cols_per_lane == 0 &&
           l.steps_per_sweep == 0 && l.prefetch_rows == 0;
}

// Wavefronts per workgroup of a single-lattice sweep.  The one-column
// kernels take at most 4 (256 threads), the two-column kernels 16 (FP64:
// 8, for its register budget).  The two-column workgroups are synchronised
// per row, and wider ones keep more adjacent strips in step: measured best
// on 4096^2 are 8 (FP32) and 16 (FP16); FP64 gains nothing beyond 4.  A
// workgroup never has more wavefronts than the lattice has strips (rounded
// up to a power of two).  When the choice is automatic it is also halved
// until at most one in eight wavefronts of a row block's workgroups has no
// strip: those only meet barriers, and on narrow lattices they cost more
// than wide workgroups gain (1050^2, 9 strips: 8 wavefronts 27.3 GLUPS FP32,
// 2 wavefronts 42.9).
inline int single_waves_per_block(const InstDesc &d, int storage, const Launch &l) {
    if (d.cols != 2) return l.waves_per_block > 0 ? (l.waves_per_block < 4 ? l.waves_per_block : 4) : 4;
    const int cap = storage == ST_F64 ? 8 : 16;
    // FP16 with a link map: 8 (4096^2, obstacle: 55.5% of peak against 53.0
    // with 16)
    const int fp16 = d.links != nullptr ? 8 : 16;
    int w = l.waves_per_block > 0 ? l.waves_per_block
                                  : (storage == ST_F16 ? fp16 : (storage == ST_F32 ? 8 : 4));
    if (w > cap) w = cap;
    while (w > 1 && w / 2 >= d.strips) w /= 2;
    if (l.waves_per_block <= 0) {
        auto slots = [&](int v) { return (d.strips + v - 1) / v * v; };
        while (w > 1 && 8 * (slots(w) - d.strips) > slots(w)) w /= 2;
    }
    return w;
}

// Wavefronts per workgroup of a batched sweep (at most 4; default 4).
inline int batch_waves_per_block(const Launch &l) {
    return l.waves_per_block > 0 ? (l.waves_per_block < 4 ? l.waves_per_block : 4) : 4;
}

// Whether an instance can use two-column strips: nx not 1 mod 128 (the
// last strip holds at least two columns, so no lane is both edges), a
// lattice within one buffer resource, and, with obstacles or open
// boundaries, its link map.
bool pair_eligible(const InstDesc &d, int storage);

// Rows per wavefront when the launch shape leaves it open.  Long strips
// re-read fewer halo rows, but a lattice must still give the 1024 SIMDs
// enough wavefronts, and narrower storage needs more of them to keep enough
// bytes in flight.  Measured optima on 4096^2: with 64-column strips FP32
// 128 rows (~2048 wavefronts), FP64 64 rows (~4096), FP16 16-32 rows
// (~8192); with two-column strips in synchronised workgroups FP32 64 rows
// (~2048), FP64 128 (~1024: one 4-wavefront workgroup per CU), FP16 32
// (~4096).  The rows are the largest power of two in [4, 128] that leaves
// at least that many wavefronts.  Lattices with a link map (walls,
// obstacles, open boundaries) aim for twice as many: the rows that cross an
// obstacle cost more, and more, shorter workgroups per CU let the hardware
// balance them (4096^2, centred 84^2 obstacle, two-column strips: FP64
// 66.6 -> 70.3%, FP32 60.4 -> 62.8%, FP16 50.9 -> 55.5% of peak; channel
// walls change by +1.4 / -0.9 / +0.2 points).
inline int auto_rows(int nx, int ny, int storage, int cols, bool linked) {
    const int width = kStripWidth * cols;
    const int strips = (nx + width - 1) / width;
    const long long open = cols == 2 ? (storage == ST_F16 ? 4096 : (storage == ST_F32 ? 2048 : 1024))
                                     : (storage == ST_F64 ? 4096 : (storage == ST_F32 ? 2048 : 8192));
    const long long target = linked ? 2 * open : open;
    const long long per = (long long)strips * ny / target;
    int r = 4;
    while (r < 128 && (long long)(2 * r) <= per) r *= 2;
    return r;
}

// Tiling of one instance for a launch shape.
inline void tile(InstDesc &d, const Launch &l, int storage) {
    const bool can = pair_eligible(d, storage);
    d.cols = (l.cols_per_lane == 1 || !can) ? 1 : (l.cols_per_lane == 2 || d.nx >= 2 * kStripWidth ? 2 : 1);
    d.rows = l.rows_per_wave > 0 ? l.rows_per_wave
                                 : auto_rows(d.nx, d.ny, storage, d.cols, d.links != nullptr);
    d.strips = (d.nx + kStripWidth * d.cols - 1) / (kStripWidth * d.cols);
    d.rowblocks = (d.ny + d.rows - 1) / d.rows;
}

// One fused sweep of one instance; src selects the lattice read (0/1).
hipError_t launch_sweep(const InstDesc &d, int storage, bool mask, int src, const Launch &l,
                        hipStream_t stream);

// Whether a lattice of this instance fits one buffer resource (<= 4 GiB),
// which selects the buffer-instruction variant of the sweep.
bool buffer_addressable(const InstDesc &d, int storage);

// One fused sweep of every instance of a batch.  descs: device InstDesc[n];
// items: device int4[nitems] of (instance, strip, rowblock, class); the
// lattice read by instance k is buf[descs[k].cur ^ flip] for class 0 and
// buf[descs[k].cur ^ flip1] for class 1.  `buf` may be true only if
// every instance is buffer_addressable; instances with descs[k].cols == 2
// (tiled so only where pair_eligible) are swept with two-column strips.
hipError_t launch_sweep_batch(const InstDesc *descs, const int4 *items, int nitems, int storage,
                              bool mask, bool buf, int flip, int flip1, const Launch &l,
                              hipStream_t stream);
// Two time steps of the batch members named by items (device int4 of
// (index into descs, window, row block, -); descs: device InstDesc[ndescs]
// tiled by tb2_desc): each reads lattice cur ^ flip.  Items naming no
// descriptor are skipped.  deep: loads two rows ahead
// (tb2_batch_prefetch_rows).
hipError_t launch_sweep_tb2_batch(const InstDesc *descs, int ndescs, const int4 *items,
                                  int nitems, int storage, int flip, bool deep, const Launch &l,
                                  hipStream_t stream);

// Two time steps per launch (FP32 or FP16 storage, open periodic lattices):
// reads lattice src, writes the other one, two steps later.
// Gives the bits of two one-step sweeps.  A wavefront computes a
// 128-column window and stores its middle kTb2Valid columns.
constexpr int kTb2Valid = 120;
bool tb2_eligible(const InstDesc &d, int storage);
// The tiling of the two-step pass: windows of 120 stored columns and,
// unless the launch shape sets them, rows per wavefront for at least 6144
// wavefronts (else 2048).
InstDesc tb2_desc(const InstDesc &d, const Launch &l);
// Wavefronts per workgroup of the two-step pass (at most four).
int tb2_waves_per_block(const InstDesc &d, int storage, const Launch &l);
// Rows ahead of their use that the two-step pass issues its loads: 1 or 2.
int tb2_prefetch_rows(const InstDesc &d, int storage, const Launch &l);
// The same for the batched two-step pass over `items` work items.
int tb2_batch_prefetch_rows(int items, int storage, const Launch &l);
hipError_t launch_sweep_tb2(const InstDesc &d, int storage, int src, const Launch &l,
                            hipStream_t stream);

// Three time steps per launch (FP32 storage, open periodic lattices, as
// for two): reads lattice src, writes the other one, three steps later,
// with the bits of three one-step sweeps.  A wavefront computes a
// 128-column window and stores its middle kTb3Valid columns.
constexpr int kTb3Valid = 116;
bool tb3_eligible(const InstDesc &d, int storage);
InstDesc tb3_desc(const InstDesc &d, const Launch &l);
int tb3_waves_per_block(const InstDesc &d, const Launch &l);
int tb3_prefetch_rows(const InstDesc &d, const Launch &l);
// XCD remap of the three-step pass: as asked, else off from kTb3ManyWaves
// wavefronts on and on below.
int tb3_xcd_remap(const InstDesc &d, const Launch &l);
hipError_t launch_sweep_tb3(const InstDesc &d, int storage, int src, const Launch &l,
                            hipStream_t stream);
// Three time steps of the batch members named by items, as
// launch_sweep_tb2_batch (descs tiled by tb3_desc; FP32 only).
hipError_t launch_sweep_tb3_batch(const InstDesc *descs, int ndescs, const int4 *items,
                                  int nitems, int storage, int flip, const Launch &l,
                                  hipStream_t stream);

// Several time steps per launch with one column per lane (narrow.hip): any
// storage, mask and boundary, k = 2 or 3.  A wavefront's window of 64 columns stores narrow_valid(k) of them.
// FP64 lattices beyond this take three steps per launch, the others two
constexpr int64_t kThreeStepNodesF64 = 3 * 1024 * 1024 / 8;
constexpr int narrow_valid(int k) { return 64 - 2 * (2 * k - 1); }
// fewer rows than this run fewer than a block's own rows of fill
constexpr int kNarrowMinRows = 16;
bool narrow_eligible(const InstDesc &d, int storage);
// The launch shape under which a lattice takes the pass; k = 0: it does not.
struct NarrowPlan {
    int k, rows, waves_per_block, remap, depth;
};
NarrowPlan narrow_plan(const InstDesc &d, int storage, const Launch &l);
// The instance tiled for the pass.
InstDesc narrow_desc(const InstDesc &d, int k, int rows);
// Wavefronts of a launch of k steps in blocks of r rows.
inline int64_t narrow_waves(const InstDesc &d, int k, int r) {
    return (int64_t)((d.nx + narrow_valid(k) - 1) / narrow_valid(k)) * ((d.ny + r - 1) / r);
}
// Wavefronts of 128-column windows of two steps in blocks of r rows.
inline int64_t wide_waves(const InstDesc &d, int r) {
    return (int64_t)((d.nx + kTb2Valid - 1) / kTb2Valid) * ((d.ny + r - 1) / r);
}
// Rows ahead of their use that a launch of `waves` wavefronts loads: two where
// a wavefront is alone on its SIMD or nearly so, and FP16 always (see
// narrow_plan); one for FP64's three steps.
inline int narrow_depth(int storage, int k, int64_t waves) {
    if (storage == ST_F64 && k == 3) return 1;
    return storage == ST_F16 || waves <= 2048 ? 2 : 1;
}
// Rows per block, from waves(r), the wavefronts that blocks of r rows give, and
// their cost where it is by rounds (the reasons and figures: narrow_plan).
struct NarrowRows {
    int rows;
    int64_t cost;
};
template <class W>
NarrowRows narrow_rows(int storage, int k, bool links, int64_t nodes, W waves) {
    const bool far = nodes > 5 * 1024 * 1024 / 2;  // FP64 beyond the memory-side cache
    if (storage == ST_F64 ? k == 2 || far : storage == ST_F32 && k == 2) {
        int cap = 8;
        if (storage == ST_F64) cap = k == 2 ? (links ? 10 : 8) : (nodes > 3 * 1024 * 1024 ? 14 : 12);
        const int64_t most = storage == ST_F64 ? 1024 : 2048;
        // a single row per block only while that leaves one wavefront per SIMD
        // (FP32 with a link map: two)
        int r = waves(1) <= (storage == ST_F32 && links ? 2048 : 1024) ? 1 : 2;
        while (r < cap && waves(r) > most) ++r;
        return {r, 0};
    }
    // the cheapest: a block's rows and `fill` more, times the rounds of `each`
    // wavefronts per SIMD, where a round of m costs start + 2 m
    struct Fit { int cap, fill, each, start; };
    Fit f = links ? Fit{9, 2, 2, 6} : Fit{9, 1, 5, 1};
    if (storage == ST_F64) f = Fit{24, 5, 2, links ? 2 : 0};
    if (storage == ST_F32) f = Fit{14, 4, 3, 2};
    const int64_t alone = storage == ST_F16 && links ? 2048 : 1024;
    int best = 0;
    int64_t least = 0;
    for (int r = waves(1) <= alone ? 1 : 2; r <= f.cap; ++r) {
        const int64_t n = (waves(r) + 1023) / 1024, m = n % f.each;
        const int64_t c =
            (r + f.fill) * (n / f.each * (f.start + 2 * f.each) + (m ? f.start + 2 * m : 0));
        if (best == 0 || c < least) {
            best = r;
            least = c;
        }
    }
    return {best, least};
}
// FP16 lattices of even width without a link map or with whole-row walls: whether
// the two-step launches of `wide` 128-column wavefronts in blocks of 8 rows, at
// most 4096, are the faster ones where the 64-column rows cost `cost`.  Both go by
// rounds of 1024 wavefronts, and their rounds fill at different sizes.  us per
// step, 64 columns / 128: 1250^2 11.9 / 12.9, 1300^2 14.0 / 12.8, 1450^2 14.6 /
// 16.3, 1600^2 19.3 / 16.6, 1052 x 1750 14.9 / 13.1, channels 1450^2 15.3 / 17.7,
// 1600^2 20.0 / 18.0; 7 lattices of 500^2 13.5 / 16.6, 9 18.1 / 16.8, 10 19.5 /
// 21.9; 5 of 700^2 19.5 / 16.9, channels 19.9 / 18.2.  The costs from which one,
// two, three and four rounds win were read off 212 lattices and batches: the
// faster pass, or within 2% of it, at all but five of them (5%).  Odd widths cost the
// 128-column pass 1.5 to 2 us more, and below 2.49 M nodes the 64-column one was the
// faster there but for a few in the last 2% (1563 x 1311 16.7 / 18.1; 36 lattices of
// 64 to 600 columns 23.5 / 29.5).
inline bool wide_rounds_f16(int64_t wide, int64_t cost, bool links) {
    constexpr int from[2][4] = {{49, 73, 98, 136}, {133, 201, 269, 337}};
    const int64_t n = (wide + 1023) / 1024;
    return n > 0 && cost >= from[links][n < 4 ? n - 1 : 3];
}
// k steps of the batch members named by items, as launch_sweep_tb2_batch
// (descs tiled by narrow_desc; the members with a link map and those without
// apart).
hipError_t launch_narrow_batch(const InstDesc *descs, int ndescs, const int4 *items, int nitems,
                               int storage, int k, bool links, int flip, const Launch &l,
                               hipStream_t stream);
hipError_t launch_narrow(const InstDesc &d, int storage, const NarrowPlan &p, int src,
                         hipStream_t stream);

// Any number of steps of one lattice of at most kResidentNodes nodes in one
// launch (resident.hip), in place: lattice src is read and written.
constexpr int kResidentNodes = 1024;
hipError_t launch_resident(const InstDesc &d, int storage, int src, int64_t steps,
                           hipStream_t stream);
// The same for the n batch members members[0 .. n).x of the table descs, of
// at most most_nodes nodes each, on the lattices descs[].cur.
hipError_t launch_resident_batch(const InstDesc *descs, const int4 *members, int n, int most_nodes,
                                 int storage, int64_t steps, hipStream_t stream);
// The access-pattern probe (a measurement aid): one launch moves the lattice
// `src` to the other one with the two-column sweep's loads, stores, launch
// shape and barriers and none of its arithmetic.  Only for two-column
// tilings of open periodic lattices whose width is a multiple of 128 and
// that fit one buffer resource (else hipErrorInvalidValue).
hipError_t launch_pattern_probe(const InstDesc &d, int storage, int src, const Launch &l,
                                hipStream_t stream);

// Link map of an instance with a mask or open x boundaries: d.links (device,
// ny * d.lpitch 16-bit codes) receives, per node, bit 0 = solid and bit i
// (1..8) = the pull source x - e_i is solid or beyond the inflow wall; then
// d.rowsum receives the link summary (see InstDesc).
hipError_t launch_link_map(const InstDesc &d, hipStream_t stream);

// *mixed (device int) = 0 when every row of the dense [ny][nx] mask is all
// solid or all fluid, else 1.
hipError_t launch_mask_rows(const uint8_t *mask, int nx, int ny, int *mixed, hipStream_t stream);

// Pre-collision state <-> device FP64 [9][ny][nx]; f^eq initialisation.
hipError_t launch_set_populations(const InstDesc &d, int storage, int src, const double *f,
                                  hipStream_t stream);
hipError_t launch_get_populations(const InstDesc &d, int storage, int src, double *f,
                                  hipStream_t stream);
hipError_t launch_init_equilibrium(const InstDesc &d, int storage, int src, const double *rho,
                                   const double *ux, const double *uy, hipStream_t stream);
hipError_t launch_macros(const InstDesc &d, int storage, int src, double *rho, double *ux,
                         double *uy, hipStream_t stream);

// Diagnostics: partials must hold diag_partial_count() * TRT_NDIAG doubles.
int diag_partial_count();
hipError_t launch_diagnostics(const InstDesc &d, int storage, int src, double *partials,
                              double *out, double time, hipStream_t stream);
// Diagnostics of the n members of a batch (descs, members: its device tables):
// member k, which reads buf[cur ^ flip0] (cls 0), buf[cur ^ flip1] (1) or buf[cur] and is `steps` steps past
// its time0, writes out[k][TRT_NDIAG].  most_nodes: the largest member's.
hipError_t launch_diagnostics_batch(const InstDesc *descs, const MemberDiag *members, int n,
                                    int64_t most_nodes, int storage, int flip0, int flip1,
                                    int64_t steps, double *out, hipStream_t stream);
hipError_t launch_row_mean_ux(const InstDesc &d, int storage, int src, double *out,
                              hipStream_t stream);

// Momentum handed to solid nodes by the last collision (the post-collision
// lattice `src`): out[2] = (F_x, F_y).  partials as for the diagnostics.
hipError_t launch_wall_force(const InstDesc &d, int storage, int src, double *partials,
                             double *out, hipStream_t stream);

// He-shifted velocity against reference fields ref_ux, ref_uy (dense FP64
// [ny][nx]) over the fluid nodes: out[0] = max over nodes and components of
// |u - u_ref|, out[1] = sum |u - u_ref|^2, out[2] = sum |u|^2, out[3] =
// sum |u_ref|^2; with `update` the reference fields are then replaced by u.
hipError_t launch_velocity_compare(const InstDesc &d, int storage, int src, double *ref_ux,
                                   double *ref_uy, bool update, double *partials, double *out,
                                   hipStream_t stream);

}  // namespace trt
