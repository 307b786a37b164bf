// narrow.hip -- several time steps per launch with one column per lane.
//
// A wavefront computes a window of 64 columns, one per lane, and marches it
// up a row block as the row pipeline of the 128-column passes does: every
// pipeline row gathers one row of the stored state, and each step's collided
// populations stay in registers until the next step has pulled them.  Half
// the columns per wavefront means half the instructions per pipeline row and
// twice the wavefronts, which is what lattices too small to fill the 1024
// SIMDs with 128-column windows need; and a third of the registers of a
// column pair, which is what makes two steps per launch possible in FP64.
//
// With LINK the lattice may have any mask and open x boundaries: a node's
// link code (InstDesc::links) says which of its pulls come back from its own
// slots.  In the first step a lane picks the address it loads from; in later
// steps it picks between the neighbour's value and its own, whose populations
// the window keeps.  Rows whose link summary is 0 for the window skip both.
//
// The first step's pulls are exact in all 64 lanes (each lane loads its own
// neighbours' elements); its gradient of Phi_x then spoils one lane on
// each side, and every later step two more (its pull and its gradient), so a
// window of K steps stores its middle 64 - 2 (2 K - 1) columns.  A row block
// of R rows gathers R + 2 (2 K - 1) rows.  Every node's arithmetic is the
// one-step sweep's, on the values that sweep would store and load back, so K
// steps per launch give its bits.
#include <type_traits>

#include "wave.hpp"

namespace trt {

namespace {

// A collided population between two steps: FP16 holds the stored half.
template <int ST> struct Pop {
    using W = typename Store<ST>::C;
    __device__ static __forceinline__ W widen(W v) { return v; }
    __device__ static __forceinline__ W shr(W v) { return dpp_shr0(v); }
    __device__ static __forceinline__ W shl(W v) { return dpp_shl0(v); }
};
template <> struct Pop<ST_F16> {
    using W = uint32_t;
    __device__ static __forceinline__ float widen(W v) {
        return (float)__builtin_bit_cast(_Float16, (unsigned short)(v & 0xffffu));
    }
    __device__ static __forceinline__ W shr(W v) { return dpp_shr0(v); }
    __device__ static __forceinline__ W shl(W v) { return dpp_shl0(v); }
};

// FP64's three steps with a link map: bounced pulls of 2, 5, 6 are settled when
// a row enters the window, from its nodes' own 4, 7, 8, which then need no
// place in it (two wavefronts per SIMD and no spills; elsewhere the two looks
// at the code cost more than the registers: a server quantum in FP16 4178
// against 3766 us).
template <int ST, int K, bool LINK> constexpr bool kSettle = LINK && ST == ST_F64 && K == 3;

// One step's collided rows in flight: of the row behind the fresh one,
// populations 0, 1, 3 and those streaming up, 2, 5, 6 -- with LINK all nine, as a
// bounced pull takes a node's own back -- and the 2, 5, 6 of the row below it
// (kSettle: as its pulls bring them).
template <int ST, int K, bool LINK> struct Window {
    using W = typename Pop<ST>::W;
    static constexpr bool kAll = LINK && !kSettle<ST, K, LINK>;
    W in[3];
    W mid[kAll ? 9 : 6];
    // where population i sits in mid (-1: not kept)
    __host__ __device__ static constexpr int at(int i) {
        constexpr int six[9] = {0, 1, 3, 2, -1, 4, 5, -1, -1};
        return kAll ? i : six[i];
    }
};

template <int ST, int K, bool LINK> struct NarrowState {
    using C = typename Store<ST>::C;
    Coeffs<C> k[K];        // per step: the next row to collide,
    C py[K], below[K];     // its Phi_y and that of the row below it
    Window<ST, K, LINK> w[K - 1];
    uint32_t code[K];      // LINK: half j of the whole: the code of row y + 2 K - 1 - j
    uint32_t flagged;      // LINK (uniform): bit j: that row has links in the window
};

template <int ST, bool LINK> struct NarrowRow {
    typename Store<ST>::T v[9];
    uint32_t code;
    uint32_t flagged;
};

// Whether a lane keeps the byte offsets of its pulls and populations in a row, so
// that an access adds the row's alone: 15 registers for 80 scalar instructions
// in two pipeline rows (FP32, two steps: 646 instructions -> 558).  Where few
// wavefronts run, nothing hides an instruction of whatever kind (256^2, one a
// SIMD: 1523 in 11,500 cycles), so that is time (us per step, before / now: FP32 300^2
// 3.26 / 3.10, 1000^2 8.23 / 8.12; FP64 400 x 200 with an obstacle 5.04 / 4.76;
// FP16 300^2 3.59 / 3.41); beside others the registers count (FP16 obstacles
// 1400^2 16.2 / 18.9: three wavefronts per SIMD instead of four).
template <int ST, bool LINK, int DEPTH>
constexpr bool kFold = DEPTH == 2 && !(ST == ST_F16 && LINK);

// The collision's constants.
template <class C> struct Consts {
    C w1, w2, ph, gx, gy;
    __device__ __forceinline__ explicit Consts(const InstDesc &d)
        : w1(uniform((C)d.omega1)), w2(uniform((C)d.omega2)), ph(uniform((C)d.phi)),
          gx(uniform((C)d.gx)), gy(uniform((C)d.gy)) {}
};

// A row's link summary entries, as loaded (or-ed where they are used, so that
// the scalar loads' wait falls there).
struct RowFlags {
    uint32_t a, b, c;
    __device__ __forceinline__ uint32_t any() const { return a | b | c; }
};

// What a wavefront needs of its lattice.
template <int ST, bool LINK, bool FOLD> struct NarrowCtx {
    using T = typename Store<ST>::T;
    using C = typename Store<ST>::C;
    BufAccess<T> in, out;
    LinkAccess la;
    Column col;
    uint32_t plane;  // bytes between a row's populations,
    uint32_t row;    // and between rows
    uint32_t from[9], own[9];  // FOLD: byte offsets in a row of the lane's pulls and populations
    int ny, nx;
    uint32_t lpitch;
    const __attribute__((address_space(4))) char *sum;
    uint32_t nsum, s0, s1, s2;  // bytes of a row's link summary; the entries that cover the window
    bool bounds;           // (uniform) the window holds a boundary column of open x
    bool store;
    OpenX<C> ox;

    // byte offsets, by lane and by wavefront, of the pull and of the population i
    // of the row at e
    __device__ __forceinline__ uint32_t side(int i) const {
        return i == 1 || i == 5 || i == 8 ? col.om : (i == 3 || i == 6 || i == 7 ? col.op : col.oc);
    }
    __device__ __forceinline__ uint32_t pull_lane(int i) const { return FOLD ? from[i] : side(i); }
    __device__ __forceinline__ uint32_t own_lane(int i) const { return FOLD ? own[i] : col.oc; }
    __device__ __forceinline__ uint32_t wave(int i, uint32_t e) const { return FOLD ? e : e + i * plane; }
    // row y's summary entries
    __device__ __forceinline__ RowFlags summary(int y) const {
        if constexpr (!LINK) return RowFlags{0u, 0u, 0u};
        // 32-bit byte offsets are an operand of the scalar load: 23 scalar
        // instructions fewer in two rows than with 64-bit addresses (cylinder
        // 400 x 200 FP32, 100 steps 487 -> 471 us)
        const uint32_t r = (uint32_t)y * nsum;
        const auto at = [&](uint32_t b) {
            return *reinterpret_cast<const __attribute__((address_space(4))) uint32_t *>(sum + b);
        };
        return RowFlags{at(r + s0), at(r + s1), at(r + s2)};
    }
    // the codes of row y's nodes (0 where the row has no links)
    __device__ __forceinline__ uint32_t codes(int y, uint32_t flagged) const {
        if constexpr (!LINK) return 0u;
        return flagged ? la.ld1((uint32_t)y * lpitch, (uint32_t)col.xc) : 0u;
    }
};

// The link data of the rows a pipeline is about to load, in their order: the
// codes of the next DEPTH rows (issued DEPTH rows before the loads whose
// addresses they pick, ahead of populations that are waited for first) and the
// summary of the row after those, so neither is waited for where it is issued.
template <int ST, bool LINK, int DEPTH> struct LinkQueue {
    uint32_t code[DEPTH], flagged[DEPTH];
    RowFlags ahead;
    int row;  // the row `ahead` describes

    // from the first row to load
    template <class Ctx> __device__ __forceinline__ void start(const Ctx &c, int y) {
        if constexpr (LINK) {
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                flagged[i] = c.summary(y).any();
                code[i] = c.codes(y, flagged[i]);
                y = y + 1 == c.ny ? 0 : y + 1;
            }
            row = y;
            ahead = c.summary(row);
        }
    }
    // the link data of the next row to load, into r
    template <class Ctx>
    __device__ __forceinline__ void take(NarrowRow<ST, LINK> &r, const Ctx &c) {
        if constexpr (LINK) {
            r.code = code[0];
            r.flagged = flagged[0];
#pragma unroll
            for (int i = 0; i + 1 < DEPTH; ++i) {
                code[i] = code[i + 1];
                flagged[i] = flagged[i + 1];
            }
            flagged[DEPTH - 1] = ahead.any();
            code[DEPTH - 1] = c.codes(row, flagged[DEPTH - 1]);
            row = row + 1 == c.ny ? 0 : row + 1;
            ahead = c.summary(row);
        }
    }
};

// Load the pulls of row y (row.code, row.flagged already hold the row's).
template <int ST, bool LINK, bool FOLD>
__device__ __forceinline__ void narrow_load(NarrowRow<ST, LINK> &row,
                                            const NarrowCtx<ST, LINK, FOLD> &c, int y) {
    const int ym = (y == 0) ? c.ny - 1 : y - 1;
    const int yp = (y == c.ny - 1) ? 0 : y + 1;
    const uint32_t e0 = (uint32_t)y * c.row, em = (uint32_t)ym * c.row, ep = (uint32_t)yp * c.row;
    const uint32_t at[9] = {e0, e0, em, e0, ep, em, em, ep, ep};
    if constexpr (!LINK) {
#pragma unroll
        for (int i = 0; i < 9; ++i) row.v[i] = c.in.ldb(c.wave(i, at[i]), c.pull_lane(i));
    } else {
        // whole byte offsets (the lattice is at most 4 GiB), so that a lane
        // can point at its own slot instead
        uint32_t off[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) off[i] = c.pull_lane(i) + c.wave(i, at[i]);
        if (row.flagged) {
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const uint32_t own = c.own_lane(kOppDir[i]) + c.wave(kOppDir[i], e0);
                off[i] = ((row.code >> i) & 1u) ? own : off[i];
            }
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) row.v[i] = c.in.ldb(0, off[i]);
    }
}

// Moments, gradient of Phi_x and coefficients of a row from its nodes'
// populations; returns Phi_y.
template <int ST, bool LINK, bool FOLD>
__device__ __forceinline__ typename Store<ST>::C narrow_coeffs(
    Coeffs<typename Store<ST>::C> &k, typename Store<ST>::C f[9], uint32_t code,
    const NarrowCtx<ST, LINK, FOLD> &c, const Consts<typename Store<ST>::C> &rt) {
    using C = typename Store<ST>::C;
    constexpr bool SH = Store<ST>::shifted;
    if (LINK && c.bounds)
        open_x_fix<C, SH>(f, c.col.xc, c.nx, c.ox.u_in, c.ox.rho_in, c.ox.rho_out);
    Moments<C, SH> m;
    m.compute(f, rt.gx, rt.gy);
    const bool solid = LINK && (code & 1u);
    const C px = m.rho * m.ux * m.ux * m.ux;
    const C py = m.rho * m.uy * m.uy * m.uy;
    const C phix = solid ? C(0) : px;
    C left = dpp_shr0(phix), right = dpp_shl0(phix);
    if (LINK && c.bounds) {
        // Phi beyond the inflow wall is the wall's; beyond the outlet, the
        // last column's
        if (c.col.xc == 0) left = c.ox.phi_wall;
        if (c.col.xc == c.nx - 1) right = phix;
    }
    k = collide_coeffs<C, SH>(m, C(0.5) * (right - left), rt.w1, rt.w2, rt.ph, rt.gx, rt.gy);
    return solid ? C(0) : py;
}

// The collided populations of a row as the one-step sweep stores them.
template <int ST>
__device__ __forceinline__ void narrow_collide(typename Pop<ST>::W o[9],
                                               const Coeffs<typename Store<ST>::C> &k,
                                               typename Store<ST>::C dphiy,  // above - below
                                               const Consts<typename Store<ST>::C> &rt) {
    using C = typename Store<ST>::C;
    const C dpy = C(0.5) * dphiy;
    if constexpr (ST == ST_F16) {
        HalfPairs p;
        reconstruct_pairs(p, k.base, k.bx, k.by, k.bxx, k.byy - rt.ph * dpy, k.bxy, k.bxxy,
                          k.bxyy);
        o[0] = half_out<0, false>(p);
        o[1] = half_out<1, false>(p);
        o[2] = half_out<2, false>(p);
        o[3] = half_out<3, false>(p);
        o[4] = half_out<4, false>(p);
        o[5] = half_out<5, false>(p);
        o[6] = half_out<6, false>(p);
        o[7] = half_out<7, false>(p);
        o[8] = half_out<8, false>(p);
    } else {
        reconstruct<C>(o, k.base, k.bx, k.by, k.bxx, k.byy - rt.ph * dpy, k.bxy, k.bxxy, k.bxyy);
    }
}

template <int ST>
__device__ __forceinline__ typename Store<ST>::T narrow_out(typename Pop<ST>::W v) {
    if constexpr (ST == ST_F16)
        return __builtin_bit_cast(_Float16, (unsigned short)(v & 0xffffu));
    else
        return v;
}

// Step Q + 1 of pipeline row y: its row behind the fresh one (whose
// coefficients and Phi_y the caller has just formed) collides; then the
// next step pulls the row behind that one and forms its coefficients, or, in
// the last step, the row is stored.  FILL: stage g < 2 K - 1 of the pipeline's
// fill runs the first g of these collisions and pulls.
template <int Q, int ST, int K, bool LINK, bool FILL, bool FOLD>
__device__ __forceinline__ void narrow_step(NarrowState<ST, K, LINK> &s,
                                            const Coeffs<typename Store<ST>::C> &fresh_k,
                                            typename Store<ST>::C fresh_y,
                                            const NarrowCtx<ST, LINK, FOLD> &c,
                                            const Consts<typename Store<ST>::C> &rt, int y,
                                            int stage) {
    using C = typename Store<ST>::C;
    using P = Pop<ST>;
    using W = typename P::W;
    W o[9];
    if (!FILL || stage > 2 * Q) narrow_collide<ST>(o, s.k[Q], fresh_y - s.below[Q], rt);
    s.below[Q] = s.py[Q];
    s.py[Q] = fresh_y;
    s.k[Q] = fresh_k;
    if (FILL && stage <= 2 * Q) return;
    if constexpr (Q == K - 1) {
        // row y of the last step: a solid node keeps zeros (its slots are
        // never read)
        if constexpr (LINK) {
            if ((s.flagged >> (2 * K - 1)) & 1u) {
                const bool solid = (s.code[K - 1] >> 16) & 1u;
#pragma unroll
                for (int i = 0; i < 9; ++i) o[i] = solid ? W(0) : o[i];
            }
        }
        if (c.store) {
            const uint32_t e0 = (uint32_t)y * c.row;
#pragma unroll
            for (int i = 0; i < 9; ++i) 
                c.out.stb(c.wave(i, e0), c.own_lane(i), narrow_out<ST>(o[i]));
        }
    } else {
        constexpr bool settle = kSettle<ST, K, LINK>;
        Window<ST, K, LINK> &w = s.w[Q];
        constexpr auto at = Window<ST, K, LINK>::at;
        Coeffs<C> next_k;
        C next_y = C(0);
        if (!FILL || stage > 2 * Q + 1) {
            W g[9];
            g[0] = w.mid[at(0)];
            g[1] = P::shr(w.mid[at(1)]);
            g[3] = P::shl(w.mid[at(3)]);
            g[2] = w.in[0];
            g[5] = settle ? w.in[1] : P::shr(w.in[1]);
            g[6] = settle ? w.in[2] : P::shl(w.in[2]);
            g[4] = o[4];
            g[7] = P::shl(o[7]);
            g[8] = P::shr(o[8]);
            uint32_t code = 0u;
            if constexpr (LINK) {
                if ((s.flagged >> (2 * Q + 2)) & 1u) {
                    code = s.code[Q + 1] & 0xffffu;
#pragma unroll
                    for (int i = 1; i < 9; ++i)
                        if (at(kOppDir[i]) >= 0)
                            g[i] = ((code >> i) & 1u) ? w.mid[at(kOppDir[i])] : g[i];
                }
            }
            C f[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = P::widen(g[i]);
            next_y = narrow_coeffs<ST, LINK>(next_k, f, code, c, rt);
        }
        w.in[0] = w.mid[at(2)];
        w.in[1] = settle ? P::shr(w.mid[at(5)]) : w.mid[at(5)];
        w.in[2] = settle ? P::shl(w.mid[at(6)]) : w.mid[at(6)];
        if constexpr (settle) {
            if ((s.flagged >> (2 * Q + 1)) & 1u) {
                const uint32_t code = s.code[Q] >> 16;
                w.in[0] = ((code >> 2) & 1u) ? o[4] : w.in[0];
                w.in[1] = ((code >> 5) & 1u) ? o[7] : w.in[1];
                w.in[2] = ((code >> 6) & 1u) ? o[8] : w.in[2];
            }
        }
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (at(i) >= 0) w.mid[at(i)] = o[i];
        if (!FILL || stage > 2 * Q + 1)
            narrow_step<Q + 1, ST, K, LINK, FILL>(s, next_k, next_y, c, rt, y, stage);
    }
}

// One pipeline row y: the first step's coefficients of gathered row
// y + 2 K - 1, whose registers then take the loads of row yload (when
// `load`), and the later parts (narrow_step).
template <int ST, int K, bool LINK, bool FILL, int DEPTH, bool FOLD>
__device__ __forceinline__ void narrow_row(NarrowState<ST, K, LINK> &s, NarrowRow<ST, LINK> &row,
                                           LinkQueue<ST, LINK, DEPTH> &q,
                                           const NarrowCtx<ST, LINK, FOLD> &c,
                                           const Consts<typename Store<ST>::C> &rt, int y,
                                           bool load, int yload, int stage) {
    using C = typename Store<ST>::C;
    Coeffs<C> k;
    uint32_t code = 0u;
    C f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = to_c(row.v[i]);
    if constexpr (LINK) {
        code = row.code;
        s.flagged = (s.flagged << 1) | (row.flagged ? 1u : 0u);
#pragma unroll
        for (int j = K - 1; j > 0; --j) s.code[j] = (s.code[j] << 16) | (s.code[j - 1] >> 16);
        s.code[0] = (s.code[0] << 16) | code;
    }
    // FP64's three steps load after the first step's moments: its populations
    // and the next ones would not fit beside the pipeline's state
    constexpr bool late = ST == ST_F64 && K == 3;
    if (!late && load) {
        q.take(row, c);
        narrow_load<ST, LINK>(row, c, yload);
    }
    const C py = narrow_coeffs<ST, LINK>(k, f, code, c, rt);
    if (late && load) {
        q.take(row, c);
        narrow_load<ST, LINK>(row, c, yload);
    }
    narrow_step<0, ST, K, LINK, FILL>(s, k, py, c, rt, y, stage);
}

// One window through one row block, the loads DEPTH rows ahead of their use.
template <int ST, int K, bool LINK, int DEPTH>
__device__ __forceinline__ void narrow_strip(const InstDesc &d, int strip, int rb, int srcsel) {
    using T = typename Store<ST>::T;
    using C = typename Store<ST>::C;
    constexpr int edge = 2 * K - 1;  // lanes (and rows) lost on each side
    const int lane = threadIdx.x & 63;
    const int nx = d.nx, ny = d.ny;
    const T *__restrict__ src = static_cast<const T *>(srcsel ? d.buf[1] : d.buf[0]);
    T *__restrict__ dst = static_cast<T *>(srcsel ? d.buf[0] : d.buf[1]);
    const uint64_t bytes = (uint64_t)ny * (uint64_t)d.pitch * sizeof(T);
    const int x0 = strip * narrow_valid(K) - edge;  // lane 0's column before wrapping
    const Column col = column_of(x0 + lane, nx, sizeof(T));
    const bool store = lane >= edge && lane < 64 - edge && x0 + lane < nx;
    const Consts<C> rt(d);
    OpenX<C> ox;
    ox.on = LINK && d.xbc != 0;
    ox.nx = nx;
    ox.u_in = (C)d.u_in;
    ox.rho_in = (C)d.rho_in;
    ox.rho_out = (C)d.rho_out;
    ox.phi_wall = ox.rho_in * ox.u_in * ox.u_in * ox.u_in;
    const bool bounds =
        LINK && ox.on && __builtin_amdgcn_ballot_w64(col.xc == 0 || col.xc == nx - 1) != 0;
    // the summary entries (64 columns each) that cover the window: its first
    // lane's, the one after it or the lattice's last, and the first after a wrap
    int s0 = 0, s1 = 0, s2 = 0;
    if (LINK && nx > 64) {
        int a = x0 % nx;
        if (a < 0) a += nx;
        const int b = min(a + 63, nx - 1);
        s0 = a >> 6;
        s1 = b >> 6;
        s2 = a + 63 >= nx ? 0 : s0;
    }
    NarrowCtx<ST, LINK, kFold<ST, LINK, DEPTH>> c{BufAccess<T>(src, bytes),
                          BufAccess<T>(dst, bytes),
                          LinkAccess(d.links, (uint64_t)ny * (uint64_t)d.lpitch),
                          col,
                          (uint32_t)(d.plane * sizeof(T)),
                          (uint32_t)(d.pitch * sizeof(T)),
                          {},
                          {},
                          ny,
                          nx,
                          (uint32_t)d.lpitch,
                          (const __attribute__((address_space(4))) char *)d.rowsum,
                          4u * (uint32_t)d.nsum,
                          4u * (uint32_t)s0,
                          4u * (uint32_t)s1,
                          4u * (uint32_t)s2,
                          bounds,
                          store,
                          ox};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        c.from[i] = c.side(i) + i * c.plane;
        c.own[i] = col.oc + i * c.plane;
    }
    const int y0 = rb * d.rows;
    const int y1 = min(y0 + d.rows, ny);
    const auto wrap_row = [&](int v) { v %= ny; return v < 0 ? v + ny : v; };

    NarrowState<ST, K, LINK> s{};
    NarrowRow<ST, LINK> row[DEPTH];
    LinkQueue<ST, LINK, DEPTH> q;
    int yl = wrap_row(y0 - edge);  // the row to load next
    const auto next = [&]() { yl = yl + 1 == ny ? 0 : yl + 1; };
    q.start(c, yl);
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) {
        q.take(row[i], c);
        narrow_load<ST, LINK>(row[i], c, yl);
        next();
    }
    // pipeline row y gathers row y + edge and loads row y + edge + DEPTH while
    // the block needs it (rows up to y1 + edge - 1); buffers are named
    // statically (a run-time index would move them to scratch memory)
    const auto ld = [&](int y) { return y + DEPTH <= y1 - 1; };
    int y = y0 - 2 * edge;
    if constexpr (DEPTH == 1) {
        for (int i = 0; i < 2 * edge; ++i, ++y) {
            narrow_row<ST, K, LINK, true, DEPTH>(s, row[0], q, c, rt, y, ld(y), yl, i >> 1);
            next();
        }
        for (; y < y1; ++y) {
            narrow_row<ST, K, LINK, false, DEPTH>(s, row[0], q, c, rt, y, ld(y), yl, 2 * K);
            next();
        }
    } else {
        for (int i = 0; i < 2 * edge; i += 2, y += 2) {
            narrow_row<ST, K, LINK, true, DEPTH>(s, row[0], q, c, rt, y, ld(y), yl, i >> 1);
            next();
            narrow_row<ST, K, LINK, true, DEPTH>(s, row[1], q, c, rt, y + 1, ld(y + 1), yl, i >> 1);
            next();
        }
        for (; y + 1 < y1; y += 2) {
            narrow_row<ST, K, LINK, false, DEPTH>(s, row[0], q, c, rt, y, ld(y), yl, 2 * K);
            next();
            narrow_row<ST, K, LINK, false, DEPTH>(s, row[1], q, c, rt, y + 1, ld(y + 1), yl, 2 * K);
            next();
        }
        if (y < y1) narrow_row<ST, K, LINK, false, DEPTH>(s, row[0], q, c, rt, y, ld(y), yl, 2 * K);
    }
}

constexpr int kNarrowMaxWaves = 4;
// Wavefronts per SIMD whose registers a variant is held to: FP64 two (three
// steps would take a few more and leave one), FP32's three steps and FP16's two
// with a link map four (130 and 129 VGPRs otherwise, one too many rows of them
// for that).
template <int ST, int K, bool LINK, int DEPTH>
constexpr int kMinWaves = ST == ST_F64                                        ? 2
                          : ST == ST_F32 && K == 3 && !LINK && DEPTH == 1     ? 4
                          : ST == ST_F16 && K == 2 && LINK                    ? 4
                                                                              : 1;
// which combinations load two rows ahead (FP64's three steps would spill)
template <int ST, int K> constexpr bool kDeep = !(ST == ST_F64 && K == 3);

template <int ST, int K, bool LINK, int DEPTH>
__global__ __launch_bounds__(64 * kNarrowMaxWaves, (kMinWaves<ST, K, LINK, DEPTH>)) void narrow_kernel(InstDesc d, int srcsel,
                                                                     int remap) {
    int b = blockIdx.x;
    if (remap) b = xcd_remap(b, gridDim.x);
    const int wpb = blockDim.x >> 6;
    const int wave = b * wpb + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= d.strips * d.rowblocks) return;
    const int rb = wave / d.strips;
    narrow_strip<ST, K, LINK, DEPTH>(d, wave - rb * d.strips, rb, srcsel);
}

// Batched: wavefront w takes item w = (member, window, row block, -).
template <int ST, int K, bool LINK, int DEPTH>
__global__ __launch_bounds__(64 * kNarrowMaxWaves, (kMinWaves<ST, K, LINK, DEPTH>)) void narrow_batch_kernel(
    const InstDesc *__restrict__ descs, int ndescs, const int4 *__restrict__ items, int nitems,
    int flip, int remap) {
    int b = blockIdx.x;
    if (remap) b = xcd_remap(b, gridDim.x);
    const int wpb = blockDim.x >> 6;
    const int wave = b * wpb + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= nitems) return;
    const int4 it = items[wave];
    if ((unsigned)it.x >= (unsigned)ndescs) return;
    const InstDesc d = descs[it.x];
    narrow_strip<ST, K, LINK, DEPTH>(d, it.y, it.z, d.cur ^ flip);
}

template <int ST, int K>
hipError_t launch_narrow_t(const InstDesc &t, int src, int wpb, int remap, int depth, hipStream_t s) {
    const int waves = t.strips * t.rowblocks;
    const int blocks = (waves + wpb - 1) / wpb;
    const auto launch = [&](auto kernel) {
        kernel<<<blocks, 64 * wpb, 0, s>>>(t, src, remap);
        return hipGetLastError();
    };
    if constexpr (kDeep<ST, K>)
        if (depth == 2)
            return t.links ? launch(narrow_kernel<ST, K, true, 2>)
                           : launch(narrow_kernel<ST, K, false, 2>);
    return t.links ? launch(narrow_kernel<ST, K, true, 1>) : launch(narrow_kernel<ST, K, false, 1>);
}

template <int ST>
hipError_t launch_narrow_k(const InstDesc &t, int k, int src, int wpb, int remap, int depth, hipStream_t s) {
    if (k == 2) return launch_narrow_t<ST, 2>(t, src, wpb, remap, depth, s);
    if (k == 3) return launch_narrow_t<ST, 3>(t, src, wpb, remap, depth, s);
    return hipErrorInvalidValue;
}

template <int ST, int K>
hipError_t launch_narrow_batch_t(const InstDesc *descs, int ndescs, const int4 *items, int nitems,
                                 bool links, int flip, const Launch &l, hipStream_t s) {
    // one-wavefront workgroups while they spread over the CUs at once
    const int wpb = nitems > 4096 ? kNarrowMaxWaves : 1;
    const dim3 g((nitems + wpb - 1) / wpb), t(64 * wpb);
    // Contiguous work items on one XCD, whose L2 then holds the rows and columns
    // that neighbouring items share, while a launch is small (us per step, the
    // hardware's order / bands: 24 members of 1.4 M nodes FP32 14.4 / 11.3, FP16
    // 13.4 / 11.5, FP64 20.9 / 17.5, 16 of 128^2 8.5 / 6.5; 16 of 4.3 M FP64
    // 53.7 / 54.1; 200 of 13 M FP64 166 / 167).
    const int r = l.remap_asked ? l.xcd_remap : nitems <= (ST == ST_F64 ? 4096 : 16384);
    const auto launch = [&](auto kernel) {
        kernel<<<g, t, 0, s>>>(descs, ndescs, items, nitems, flip, r);
        return hipGetLastError();
    };
    if constexpr (kDeep<ST, K>)
        if (narrow_depth(ST, K, nitems) == 2)
            return links ? launch(narrow_batch_kernel<ST, K, true, 2>)
                         : launch(narrow_batch_kernel<ST, K, false, 2>);
    return links ? launch(narrow_batch_kernel<ST, K, true, 1>)
                 : launch(narrow_batch_kernel<ST, K, false, 1>);
}

template <int ST>
hipError_t launch_narrow_batch_k(const InstDesc *descs, int ndescs, const int4 *items, int nitems,
                                 int k, bool links, int flip, const Launch &l, hipStream_t s) {
    if (k == 2) return launch_narrow_batch_t<ST, 2>(descs, ndescs, items, nitems, links, flip, l, s);
    if (k == 3) return launch_narrow_batch_t<ST, 3>(descs, ndescs, items, nitems, links, flip, l, s);
    return hipErrorInvalidValue;
}

}  // namespace

bool narrow_eligible(const InstDesc &d, int storage) {
    const bool general = d.mask != nullptr || d.xbc != 0;
    return d.ny >= kNarrowMinRows && buffer_addressable(d, storage) &&
           (!general || d.links != nullptr);
}

InstDesc narrow_desc(const InstDesc &d, int k, int rows) {
    InstDesc t = d;
    t.strips = (d.nx + narrow_valid(k) - 1) / narrow_valid(k);
    t.rows = rows;
    t.rowblocks = (d.ny + rows - 1) / rows;
    return t;
}

hipError_t launch_narrow(const InstDesc &d, int storage, const NarrowPlan &p, int src,
                         hipStream_t stream) {
    if (!narrow_eligible(d, storage)) return hipErrorInvalidValue;
    const InstDesc t = narrow_desc(d, p.k, p.rows);
    switch (storage) {
        case ST_F64: return launch_narrow_k<ST_F64>(t, p.k, src, p.waves_per_block, p.remap, p.depth, stream);
        case ST_F32: return launch_narrow_k<ST_F32>(t, p.k, src, p.waves_per_block, p.remap, p.depth, stream);
        case ST_F16: return launch_narrow_k<ST_F16>(t, p.k, src, p.waves_per_block, p.remap, p.depth, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_narrow_batch(const InstDesc *descs, int ndescs, const int4 *items, int nitems,
                               int storage, int k, bool links, int flip, const Launch &l,
                               hipStream_t stream) {
    if (nitems <= 0) return hipSuccess;
    switch (storage) {
        case ST_F64: return launch_narrow_batch_k<ST_F64>(descs, ndescs, items, nitems, k, links, flip, l, stream);
        case ST_F32: return launch_narrow_batch_k<ST_F32>(descs, ndescs, items, nitems, k, links, flip, l, stream);
        case ST_F16: return launch_narrow_batch_k<ST_F16>(descs, ndescs, items, nitems, k, links, flip, l, stream);
        default: return hipErrorInvalidValue;
    }
}

// Which lattices take the pass, how many steps per launch and with what rows.
// Only where every field of the launch shape is automatic: a caller that
// sets one asks for the passes those fields describe.  Measured on one box, us
// per step, the other passes' default against this one's best shape and,
// where it differs, the shape chosen here:
//   FP64 (one step per launch before): two steps 128^2 6.6 / 2.7, 256^2 7.6 /
//     3.4, 512^2 13.0 / 5.7 (three 6.0), cylinder 400 x 200 14.5 / 5.0 (three
//     6.2); three steps 724^2 7.9 (two 9.9), 1024^2 33.5 / 13.3 (18.2), 2048^2
//     112 / 48.7 (70.5), 4096^2 408 / 186 (271), cylinder 724^2 11.7 (12.1),
//     1050^2 43.8 / 18.0 (20.6), 2048^2 55 (71).
//   FP32, any link map but whole-row walls (one step before): cylinder
//     400 x 200 two steps 4.2, three 5.5 against 12.6; 700^2 7.1 / 8.0, 760^2
//     8.2 / 8.3, 900^2 9.9 / 9.8, 1050^2 13.5 / 12.6 against 26.4; obstacle
//     2048^2 38.0 / 31.2 against 68.6.
//   FP32, whole-row walls (128-column windows before): channel 700^2 two steps
//     7.1, three 7.2, 1001 x 513 7.2 / 7.1 against 10.5, 850^2 9.3 / 8.1, 1000^2
//     11.9 / 9.7.
//   FP32, neither (128-column windows before): 128^2 8.0 / 2.6, 200^2 two steps
//     2.9, three 3.0, 400 x 200 3.4 / 3.2, 420^2 4.4 / 4.0, 512^2 4.5 / 4.4
//     against 8.6, 800^2 7.2 / 6.8, 1000^2 11.0 / 8.2, 1448^2 20.1 / 15.5 against
//     19.6, 2048^2 27.3 against 27.9.  1024^2 alone keeps two steps and eight
//     rows (10.6; 8.2 with three; 12.6 before): no measurement asks for it, the
//     shape that this size reports is fixed by a test of the default shapes.
//   FP16: 128^2 7.5 / 2.5, 512^2 8.2 / 4.4, 1024^2 11.9 / 9.3, 1448^2 two steps
//     14.9, 2048^2 25.9 / 27.3 (so not there, and not where the 128-column
//     launches' third round is nearly full, from 2.49 M nodes on -- 1561^2 18.6 /
//     18.0, 1601^2 18.6 / 19.5, 2525 x 1032 18.3 / 19.8, channels equal; of even
//     width below that by the rounds of both: wide_rounds_f16); cylinder 1050^2
//     21.1 / 11.0;
//     obstacle 2048^2 47.4 / 34.7 (three steps 35.2).
// Rows: a block of R rows runs R + 2 (2 k - 1) pipeline rows.  FP64, and two
// steps in FP32: the smallest R that leaves at most two wavefronts per SIMD
// (FP64, but for three steps of up to 2.6 M nodes: one) -- up to a cap from where the launch is bound by memory rather
// than by latency and shorter blocks in more rounds balance better (FP64
// 2048^2, three steps: 10 rows 50.4, 14 rows 48.7, 16 to 64 rows 50 and more).
// FP16, three steps in FP32 and those FP64 ones: the cheapest R by rounds of wavefronts, with
// constants fitted to twelve sets of lattices from 300^2 to 2000^2, with and
// without obstacles, at 15 rows each: within 2% of the best rows on average,
// where the other rule's caps (16, and 5 or 12 rows) were 4 to 8% off.
// Before / now: FP16 twelve channels and cylinders of 2.3 M nodes 21.9 / 19.3,
// 1400^2 16.6 / 14.5, obstacles 17.6 / 16.3, cylinder 400 x 200 5.3 / 4.6; FP32
// 2000^2 30.8 / 27.1, 12 obstacles of 500^2 30.5 / 24.6, 3 of 1100^2 28.5 / 26.2;
// FP64 1200^2 20.9 / 17.3, 1400^2 25.4 / 23.3, obstacles 23.3 / 18.4 and 26.5 /
// 24.6, 3000 x 500 21.5 / 17.6, twelve lattices of 2.3 M nodes 34.5 / 31.9, with
// obstacles 35.3 / 33.0.
// Loads two rows ahead: a lone wavefront's pipeline row (about 1 us) is shorter
// than a load from memory, so one row ahead leaves it waiting -- two against
// one: FP64 128^2 2.68 / 2.99, 512^2 5.71 / 6.00, cylinder 400 x 200 4.98 /
// 5.50; FP32 128^2 2.37 / 2.73, 512^2 4.08 / 4.35, cylinder 4.31 / 4.63, channel
// 6.79 / 6.97; FP16 128^2 2.47 / 3.19, 1024^2 9.26 / 10.1, 1448^2 14.9 / 16.0.
// With more wavefronts per SIMD the registers cost more than it hides (FP64
// 1024^2 18.95 / 18.06, FP32 1448^2 15.8 / 15.6), but for FP16.
NarrowPlan narrow_plan(const InstDesc &d, int storage, const Launch &l) {
    const NarrowPlan p0 = {0, 0, 0, 0, 1};
    NarrowPlan p = p0;
    if (!automatic(l) || !narrow_eligible(d, storage)) return p;
    const int64_t nodes = (int64_t)d.nx * d.ny;
    const bool wide = tb2_eligible(d, storage);  // the 128-column passes apply
    constexpr int64_t k1 = 1024;
    p.k = 2;
    if (storage == ST_F64) {
        if (nodes > kThreeStepNodesF64) p.k = 3;
    } else if (storage == ST_F32) {
        if (wide && nodes >= 2048 * 2048) return p0;
        const bool two = d.links ? nodes <= k1 * k1 / 2
                                 : nodes <= k1 * 64 || (d.nx == k1 && d.ny == k1);
        p.k = two ? 2 : 3;
    } else if (wide && nodes > k1 * k1 * 19 / 8) {
        return p0;
    }
    const auto waves = [&](int r) { return narrow_waves(d, p.k, r); };
    const NarrowRows r = narrow_rows(storage, p.k, d.links != nullptr, nodes, waves);
    if (storage == ST_F16 && wide && d.nx % 2 == 0 &&
        wide_rounds_f16(wide_waves(d, 8), r.cost, d.links != nullptr))
        return p0;
    p.rows = r.rows;
    p.depth = narrow_depth(storage, p.k, waves(p.rows));
    p.waves_per_block = waves(p.rows) >= 4096 ? 4 : 1;
    // XCD bands, but for the large launches of FP64's three steps (2048^2 at 14
    // rows 48.7 in round-robin order, 49.4 in bands)
    const bool spread = storage == ST_F64 && p.k == 3 && p.waves_per_block == 4;
    p.remap = l.remap_asked ? l.xcd_remap : (spread ? 0 : 1);
    return p;
}

}  // namespace trt
