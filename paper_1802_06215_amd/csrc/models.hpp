// Device-side step functions of the two models and the Philox4x32-10 stream.
//
// The step function is the deterministic simulative model g of DESPOT
// (Sec. III-A): s', r, z = g(s, a, phi), where the scenario phi supplies the
// random numbers through a counter-based generator indexed by (scenario id,
// depth, block, tag).  State arithmetic of the driving model is FP32,
// compiled without contraction and with correctly rounded division and
// square root (plain "/" and __builtin_sqrtf under
// -fhip-fp32-correctly-rounded-divide-sqrt; HIP's __fsqrt_rn/__fdiv_rn are
// native approximations unless OCML_BASIC_ROUNDED_OPERATIONS is set), so the
// results are bit-identical to any IEEE-754 FP32 evaluation in the same
// operation order.
#pragma once

#include <type_traits>

#include "internal.hpp"

namespace hdx {

// Constant address space on the device (the host pass parses the same
// declarations without it).
#if defined(__HIP_DEVICE_COMPILE__)
#define HDX_CONST __attribute__((address_space(4)))
#else
#define HDX_CONST
#endif

// A model as the kernels see it: the header and the device tables through
// the constant address space (never written by a kernel, so uniform
// addresses become scalar loads).
struct MView {
    const HDX_CONST ModelHdr *h;
    const HDX_CONST uint32_t *thr;
    const HDX_CONST float *gg;
    const HDX_CONST double *gs, *g64;
    __device__ float gpow(int j) const { return gg[j]; }
    // 1 + gamma + ... + gamma^(j-1), j = 0..kHorizon
    __device__ double gpow_sum(int j) const { return gs[j]; }
    // gamma^d in FP64, d < kRockTerms: its own table, as the difference of two
    // sums above has the sums' absolute error (at gamma 0.3 and 30 steps, 8 %)
    __device__ double gpow_exact(int d) const { return g64[d]; }
};

__device__ __forceinline__ MView make_view(const DevModel *gm) {
    MView v;
    v.h = (const HDX_CONST ModelHdr *)&gm->h;
    v.thr = (const HDX_CONST uint32_t *)gm->sense_thr_m1;
    v.gg = (const HDX_CONST float *)gm->gpow;
    v.gs = (const HDX_CONST double *)gm->gsum;
    v.g64 = (const HDX_CONST double *)gm->gpow64;
    return v;
}

__device__ __forceinline__ StatesPtr load_states(const HDX_CONST StatesPtr *s) {
    StatesPtr r;
    r.w = s->w;
    r.s = s->s;
    r.car = s->car;
    r.px = s->px;
    r.py = s->py;
    r.goal = s->goal;
    r.stride = s->stride;
    return r;
}

// a ^ b ^ c in one instruction.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)__builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
    return a ^ b ^ c;
#endif
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two
// 32x32->64 multiplies, the key advanced by the Weyl increments in between.
__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                        uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // one 32x32->64 product each (a single v_mad_u64_u32 instead of
        // separate high and low multiplies, at the rate of any other instruction)
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = xor3(hi1, c1, k0), n2 = xor3(hi0, c3, k1);
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    return make_uint4(c0, c1, c2, c3);
}

struct RolloutParams {
    uint32_t k0, k1;
    int32_t policy, const_action, max_steps, max_depth, n_actions;
};

// Steps a rollout from depth d0 may take.
__device__ __forceinline__ int rollout_length(const RolloutParams &P, int d0) {
    int n = P.max_steps;
    if (P.max_depth >= 0 && P.max_depth - d0 < n) n = P.max_depth - d0;
    return n > kHorizon ? kHorizon : n;  // the discount table's length
}

// x mod n for a uniform n >= 1: inv = floor((2^32 - 1) / n) gives the quotient
// or one less.
struct Modulus {
    uint32_t n, inv;
    __device__ __forceinline__ explicit Modulus(uint32_t n_) : n(n_), inv(0xffffffffu / n_) {}
    __device__ __forceinline__ uint32_t operator()(uint32_t x) const {
        const uint32_t r = x - __umulhi(x, inv) * n;
        return min(r, r - n);  // r - n wraps when r < n
    }
};

// Eq. 12 bound of the rock models from tabulated group sums: entry 16 g + m
// of `tab0` (groups 0-3) or `tab1` (group 4) is the sum of group g's good
// rocks' terms when the four quality bits of rocks 4g .. 4g+3 read m.  The
// five lookups are issued together and added in group order; a group past
// the last rock tabulates +0 for every pattern, and the running sum of
// non-negative terms is never -0, so the result equals the sum over the
// rock groups alone, bit for bit.  `bits` holds rock i's quality in bit i.
// Called by all 64 lanes of a wavefront.
__device__ __forceinline__ float group_table_sum(uint32_t bits, float tab0, float tab1) {
    const float t0 = __shfl(tab0, (int)__builtin_amdgcn_ubfe(bits, 0, 4), 64);
    const float t1 = __shfl(tab0, 16 + (int)__builtin_amdgcn_ubfe(bits, 4, 4), 64);
    const float t2 = __shfl(tab0, 32 + (int)__builtin_amdgcn_ubfe(bits, 8, 4), 64);
    const float t3 = __shfl(tab0, 48 + (int)__builtin_amdgcn_ubfe(bits, 12, 4), 64);
    const float t4 = __shfl(tab1, (int)__builtin_amdgcn_ubfe(bits, 16, 4), 64);
    return (((((0.0f + t0) + t1) + t2) + t3) + t4);
}

// A cell x | y << 5 of the RockSample grid for robots that act step by step
// (Robots): bit a is set if action a < 5 has an effect there (the move stays
// on the grid or leaves it east; the sample meets a rock), the upper bits hold
// 10 + the rock's index.  Column x = grid stands for having left: no effects.
// A robot's step is then one table read and some twenty instructions, none of
// them a branch, where comparing the cell with the rocks took a loop over them.
__device__ __forceinline__ uint32_t cell_effects(const MView &M, int cell) {
    const int n = M.h->grid, x = cell & 31, y = cell >> 5;
    if (x >= n || y >= n) return 0u;
    return (y + 1 < n ? 1u : 0u) | (y > 0 ? 2u : 0u) | 4u | (x > 0 ? 8u : 0u);
}
__device__ __forceinline__ uint32_t rock_effect(int rock) { return 16u | ((uint32_t)(10 + rock) << 25); }

// K robots on the grid and the good rocks (bit 10 + i), stepped with actions of
// the lane's own.
template <int K>
struct Robots {
    uint32_t cell[K], good;
    __device__ __forceinline__ bool any(int grid) const {
        bool b = (cell[0] & 31u) != (uint32_t)grid;
        if constexpr (K == 2) b |= (cell[1] & 31u) != (uint32_t)grid;
        return b;
    }
    // Robot j's action a; returns its reward times g, given ten = 10 g.
    __device__ __forceinline__ float hop(const uint32_t *effects, int grid, int j, int a, float ten) {
        const uint32_t e = effects[cell[j]];
        const int32_t acts = __builtin_amdgcn_sbfe((int)e, (uint32_t)a, 1u);  // -1: it has an effect
        // byte a of the steps +32, -32, +1, -1 (0 for a sample)
        const int32_t step = (int8_t)__builtin_amdgcn_perm(0u, 0xFF01E020u, (uint32_t)a);
        cell[j] += (uint32_t)(step & acts);
        const uint32_t bit = a == 4 ? (1u << (e >> 25)) & (uint32_t)acts : 0u;
        // (and-not: for good ^= got, twice, this compiler emits a three-operand bit instruction with a wrong table)
        const uint32_t got = good & bit;
        good &= ~bit;
        const bool left = (acts != 0) & ((cell[j] & 31u) == (uint32_t)grid);
        return left | (got != 0) ? ten : bit != 0 ? -ten : 0.0f;
    }
};

// ---------------------------------------------------------------------------
// RockSample: one packed int32 word per scenario.
// ---------------------------------------------------------------------------
struct RsOps {
    struct State {
        int32_t w;
    };
    __device__ static void load(const MView &, const StatesPtr &S, int64_t p, State &st) { st.w = S.w[p]; }
    __device__ static void make_terminal(State &st) { st.w = 1 << 30; }
    __device__ static void store(const MView &, const StatesPtr &S, int64_t p, const State &st) { S.w[p] = st.w; }
    __device__ static bool terminal(const State &st) { return (st.w >> 30) & 1; }

    // Action a, the same for the wavefront; returns the reward.  A sense
    // changes nothing, and terminal states are absorbing.
    __device__ static float move(const MView &M, State &st, int a) {
        if (terminal(st) || a > 4) return 0.0f;
        if (a < 4) return walk(M, st, a) ? 10.0f : 0.0f;
        float r = 0.0f;
        for (int q = 0; q < M.h->n_rocks; ++q)
            if (at(st, M.h->rock_x[q], M.h->rock_y[q])) {
                const int32_t bit = 1 << (10 + q);
                r = st.w & bit ? 10.0f : -10.0f;
                st.w &= ~bit;
            }
        return r;
    }
    // The default rollout, moving east, of at most R steps.
    __device__ static float rollout_east(const MView &M, const State &st, int R, int &steps) {
        steps = 0;
        if (terminal(st) || R <= 0) return 0.0f;
        const int out = M.h->grid - 1 - (st.w & 31);
        steps = R < out + 1 ? R : out + 1;
        return out < R ? 10.0f * M.gpow(out) : 0.0f;
    }

    // Bound of one state, summed as in upper_wave; term(d) = 10 gamma^d.
    template <class Term>
    __device__ static float upper(const MView &M, const State &st, Term term) {
        if (terminal(st)) return 0.0f;
        const int nr = M.h->n_rocks;
        float u = 0.0f;
        for (int g = 0; g < nr; g += 4) {
            float p = 0.0f;
            for (int i = g; i < g + 4 && i < nr; ++i) {
                const float t = term(rock_distance(st, M.h->rock_x[i], M.h->rock_y[i]));
                p = (st.w >> (10 + i)) & 1 ? p + t : p;
            }
            u = u + p;
        }
        return u + term(M.h->grid - 1 - (st.w & 31));
    }

    // Partial sums of the last common cell, kept across the rounds of a
    // tile: entry 16 g + m (lane of tab0, or of tab1 past 63) is the sum of
    // the terms of the good rocks of group g (rocks 4g .. 4g+3) when their
    // qualities read m.
    struct WaveUpper {
        int x = -1, y = -1;
        float tab0 = 0.0f, tab1 = 0.0f, exit = 0.0f;
    };

    // The same value, bit for bit, whichever way it is computed: the good
    // rocks' terms 10 gamma^d are summed within groups of four rocks in
    // index order, the group sums added in group order, then the exit term.
    // Robot cells are deterministic, so the live scenarios of a tile usually
    // share one cell: then the wavefront tabulates every group's sum for all
    // 16 quality patterns (rebuilt only when the cell changes) and each lane
    // adds one table entry per group of four rocks (a bit-field extract, a
    // cross-lane read and an add).  Called by all 64 lanes of a wavefront.
    __device__ static float upper_wave(const MView &M, const State &st, WaveUpper &wu) {
        const bool live = !((st.w >> 30) & 1);
        const int x = st.w & 31, y = (st.w >> 5) & 31;
        const uint64_t lv = __ballot(live);
        if (lv == 0) return 0.0f;
        const int leader = __ffsll((unsigned long long)lv) - 1;
        const int xs = __builtin_amdgcn_readlane(x, leader), ys = __builtin_amdgcn_readlane(y, leader);
        const int nr = M.h->n_rocks;
        if (__ballot(live && (x != xs || y != ys)) != 0) {
            // cells differ: per-lane terms, discount powers read from the model table
            return upper(M, st, [&](int d) { return 10.0f * M.gpow(d); });
        }
        if (xs != wu.x || ys != wu.y) {
            const int lane = (int)__lane_id();
            const float ci =
                lane < nr ? 10.0f * M.gg[(uint32_t)(abs(xs - M.h->rock_x[lane]) + abs(ys - M.h->rock_y[lane]))] : 0.0f;
            // entry e = 16 g + m: group g's good rocks under pattern m, in index order
            float t0 = 0.0f, t1 = 0.0f;
            const int g0 = lane >> 4, g1 = 4 + (lane >> 4), m = lane & 15;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float c0 = __shfl(ci, (4 * g0 + b) & 63, 64);
                const float c1 = __shfl(ci, (4 * g1 + b) & 63, 64);
                if (((m >> b) & 1) && 4 * g0 + b < nr) t0 = t0 + c0;
                if (((m >> b) & 1) && 4 * g1 + b < nr) t1 = t1 + c1;
            }
            wu.tab0 = t0;
            wu.tab1 = t1;
            wu.exit = 10.0f * M.gpow(M.h->grid - 1 - xs);
            wu.x = xs;
            wu.y = ys;
        }
        const float u = group_table_sum((uint32_t)st.w >> 10, wu.tab0, wu.tab1) + wu.exit;
        return live ? u : 0.0f;
    }

    // A state as the tiles hold it (run_tile_rocks): the robot's cell, its
    // actions below 5, and what follows from a cell alone.
    static constexpr bool kTwo = false;
    using Team = Robots<1>;
    __device__ static Team team(const MView &M, const State &st) {
        return {{terminal(st) ? (uint32_t)M.h->grid : (uint32_t)st.w & 0x3ffu}, (uint32_t)st.w};
    }
    // The reward of action a times g, given ten = 10 g.
    __device__ static float act(const MView &M, const uint32_t *effects, Team &t, int a, float ten) {
        return t.hop(effects, M.h->grid, 0, a, ten);
    }
    __device__ static int cell(const State &st) { return st.w & 0x3ff; }
    __device__ static int cell_x(int c) { return c & 31; }
    __device__ static int cell_y(int c) { return (c >> 5) & 31; }
    __device__ static uint32_t rocks(const State &st) { return ((uint32_t)st.w >> 10) & 0xFFFFFu; }
    __device__ static void from_words(State &st, int32_t w, int32_t) { st.w = w; }
    __device__ static void from_cell(State &st, int c) { st.w = c; }
    __device__ static bool acting(const State &st) { return !terminal(st); }
    __device__ static bool ended(const State &st) { return terminal(st); }
    __device__ static void settle(State &) {}
    __device__ static float mover(const MView &M, State &st, int b) { return move(M, st, b); }
    __device__ static int rock_distance(const State &st, int rx, int ry) {
        return abs((st.w & 31) - rx) + abs(((st.w >> 5) & 31) - ry);
    }
    __device__ static bool at(const State &st, int rx, int ry) { return rock_distance(st, rx, ry) == 0; }
    // The move c < 4 (any other c: none); true if it leaves the grid.
    __device__ static bool walk(const MView &M, State &st, int c) {
        const int n = M.h->grid, x = st.w & 31, y = (st.w >> 5) & 31;
        if (c == 2 && x + 1 == n) {
            st.w |= 1 << 30;
            return true;
        }
        const int nx = c == 2 ? x + 1 : c == 3 && x > 0 ? x - 1 : x;
        const int ny = c == 0 && y + 1 < n ? y + 1 : c == 1 && y > 0 ? y - 1 : y;
        st.w = (st.w & ~0x3ff) | nx | (ny << 5);
        return false;
    }
    // term[d] = 10 gamma^d
    __device__ static double exits(const MView &M, const State &st, const double *term) {
        return term[M.h->grid - 1 - (st.w & 31)];
    }
    // The rollout that moves east, of at most R steps.
    __device__ static void move_east(const MView &M, const State &st, int R, const double *term, double &value,
                                     int &steps) {
        const int out = M.h->grid - 1 - (st.w & 31);  // steps before the one that leaves
        steps = R < 0 ? 0 : R < out + 1 ? R : out + 1;
        value = out < R ? term[out] : 0.0;
    }
};

// ---------------------------------------------------------------------------
// Multi-agent RockSample: two robots share the rocks.  Two int32 rows per
// scenario: the robots' row (robot 1's cell in bits 0-9, robot 2's in bits
// 10-19, x in the low five bits of each; robot j gone in bit 20+j; terminal
// in bit 30) and the rocks' row (rock i's quality in bit i), at w[k] and
// w[stride + k].  Joint action a = a1 (5+m) + a2; robot 1 acts first, then
// robot 2 on the rocks robot 1 left; robot j's sensor reads word j of the
// step block; the joint observation is 3 z1 + z2.
// ---------------------------------------------------------------------------
struct MarsOps {
    struct State {
        int32_t p, rk;
    };
    static constexpr int kGone0 = 20, kTerm = 30;
    static constexpr int kFar = 62;  // beyond any Manhattan distance on a 31 x 31 grid

    __device__ static void load(const MView &, const StatesPtr &S, int64_t p, State &st) {
        st.p = S.w[p];
        st.rk = S.w[S.stride + p];
    }
    __device__ static void make_terminal(State &st) {
        st.p = (1 << kTerm) | (3 << kGone0);
        st.rk = 0;
    }
    __device__ static void store(const MView &, const StatesPtr &S, int64_t p, const State &st) {
        S.w[p] = st.p;
        S.w[S.stride + p] = st.rk;
    }
    __device__ static bool terminal(const State &st) { return (st.p >> kTerm) & 1; }

    // Robot J's own action b (numbered as in RockSample), the same for the
    // wavefront; returns its reward.
    template <int J, bool kObs>
    __device__ static float act(const MView &M, State &st, int b, uint32_t word, int &zj) {
        zj = 0;
        if (gone<J>(st)) return 0.0f;  // this robot has left the map
        if (b < 4) return walk_one<J>(M, st, b) ? 10.0f : 0.0f;
        const int x = (st.p >> (10 * J)) & 31, y = (st.p >> (10 * J + 5)) & 31;
        float r = 0.0f;
        if (b == 4) {
            int i = -1;
            for (int q = 0; q < M.h->n_rocks; ++q)
                if (M.h->rock_x[q] == x && M.h->rock_y[q] == y) i = q;
            if (i >= 0) {
                r = (st.rk >> i) & 1 ? 10.0f : -10.0f;
                st.rk &= ~(1 << i);
            }
        } else if (kObs) {
            const int i = b - 5;
            const int dx = x - M.h->rock_x[i], dy = y - M.h->rock_y[i];
            const int correct = word <= M.thr[(uint32_t)(dx * dx + dy * dy)];
            const int truth = (st.rk >> i) & 1;
            zj = (correct ? truth : !truth) ? 1 : 2;
        }
        return r;
    }

    // Joint action a, the same for the wavefront; returns the reward.
    __device__ static float move(const MView &M, State &st, int a) {
        if (terminal(st)) return 0.0f;  // absorbing
        const int per = 5 + M.h->n_rocks;
        const int a1 = (a * M.h->joint_inv) >> 16, a2 = a - a1 * per;  // a / per without a division
        int z;
        const float r1 = act<0, false>(M, st, a1, 0, z);
        const float r2 = act<1, false>(M, st, a2, 0, z);
        settle(st);
        return r1 + r2;
    }
    // The default rollout, both robots moving east, of at most R steps.
    __device__ static float rollout_east(const MView &M, const State &st, int R, int &steps) {
        steps = 0;
        if (terminal(st) || R <= 0) return 0.0f;
        const int n1 = M.h->grid - 1;
        const int o1 = gone<0>(st) ? -1 : n1 - (st.p & 31), o2 = gone<1>(st) ? -1 : n1 - ((st.p >> 10) & 31);
        const int last = o1 > o2 ? o1 : o2;
        steps = R < last + 1 ? R : last + 1;
        const float v1 = o1 >= 0 && o1 < R ? 10.0f * M.gpow(o1) : 0.0f;
        return v1 + (o2 >= 0 && o2 < R ? 10.0f * M.gpow(o2) : 0.0f);
    }

    // Distance from the nearer robot still on the map to cell (rx, ry).
    __device__ static int near(int32_t p, int rx, int ry) {
        const int d0 = ((p >> kGone0) & 1) ? kFar : abs((p & 31) - rx) + abs(((p >> 5) & 31) - ry);
        const int d1 = ((p >> (kGone0 + 1)) & 1) ? kFar : abs(((p >> 10) & 31) - rx) + abs(((p >> 15) & 31) - ry);
        return d0 < d1 ? d0 : d1;
    }

    // Every good rock sampled by the nearer robot on arrival, plus each
    // robot's exit reward at its shortest exit time (rocks summed within
    // groups of four in index order, the group sums in group order, then
    // robot 1's exit, then robot 2's); term(d) = 10 gamma^d.
    template <class Term>
    __device__ static float upper(const MView &M, const State &st, Term term) {
        if (terminal(st)) return 0.0f;
        const int nr = M.h->n_rocks;
        float u = 0.0f;
        for (int g = 0; g < nr; g += 4) {
            float p = 0.0f;
            for (int i = g; i < g + 4 && i < nr; ++i) {
                const float t = term(near(st.p, M.h->rock_x[i], M.h->rock_y[i]));
                p = (st.rk >> i) & 1 ? p + t : p;
            }
            u = u + p;
        }
        const int n1 = M.h->grid - 1;
        if (!gone<0>(st)) u += term(n1 - (st.p & 31));
        if (!gone<1>(st)) u += term(n1 - ((st.p >> 10) & 31));
        return u;
    }

    struct WaveUpper {
        int32_t p = -1;
        float tab0 = 0.0f, tab1 = 0.0f, e0 = 0.0f, e1 = 0.0f;
    };

    // The same value, bit for bit.  Robot cells are deterministic, so the
    // live scenarios of a tile usually share the robots' row: then the
    // wavefront tabulates each group of four rocks' sum for all 16 quality
    // patterns, as RockSample's bound does, and each lane adds one entry per
    // group; a robot that has left adds +0 for its exit.  Called by all 64
    // lanes of a wavefront.
    __device__ static float upper_wave(const MView &M, const State &st, WaveUpper &wu) {
        const bool live = !((st.p >> kTerm) & 1);
        const uint64_t lv = __ballot(live);
        if (lv == 0) return 0.0f;
        const int leader = __ffsll((unsigned long long)lv) - 1;
        const int32_t ps = __builtin_amdgcn_readlane(st.p, leader);
        if (__ballot(live && st.p != ps) != 0) return upper(M, st, [&](int d) { return 10.0f * M.gpow(d); });
        const int nr = M.h->n_rocks;
        if (ps != wu.p) {
            const int lane = (int)__lane_id();
            const float ci = lane < nr ? 10.0f * M.gg[(uint32_t)near(ps, M.h->rock_x[lane], M.h->rock_y[lane])] : 0.0f;
            float t0 = 0.0f, t1 = 0.0f;
            const int g0 = lane >> 4, g1 = 4 + (lane >> 4), m = lane & 15;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float c0 = __shfl(ci, (4 * g0 + b) & 63, 64);
                const float c1 = __shfl(ci, (4 * g1 + b) & 63, 64);
                if (((m >> b) & 1) && 4 * g0 + b < nr) t0 = t0 + c0;
                if (((m >> b) & 1) && 4 * g1 + b < nr) t1 = t1 + c1;
            }
            wu.tab0 = t0;
            wu.tab1 = t1;
            const int n1 = M.h->grid - 1;
            wu.e0 = ((ps >> kGone0) & 1) ? 0.0f : 10.0f * M.gpow(n1 - (ps & 31));
            wu.e1 = ((ps >> (kGone0 + 1)) & 1) ? 0.0f : 10.0f * M.gpow(n1 - ((ps >> 10) & 31));
            wu.p = ps;
        }
        float u = group_table_sum((uint32_t)st.rk, wu.tab0, wu.tab1);
        u = u + wu.e0;
        u = u + wu.e1;
        return live ? u : 0.0f;
    }

    // A state as the tiles hold it (run_tile_rocks), after robot 1's action
    // and with its reward: robot 2's actions below 5, and what follows from
    // the robots' row alone.
    static constexpr bool kTwo = true;
    using Team = Robots<2>;
    __device__ static Team team(const MView &M, const State &st) {
        const uint32_t out = (uint32_t)M.h->grid;
        return {{terminal(st) | gone<0>(st) ? out : (uint32_t)st.p & 0x3ffu,
                 terminal(st) | gone<1>(st) ? out : (uint32_t)(st.p >> 10) & 0x3ffu},
                (uint32_t)st.rk << 10};
    }
    __device__ static float act(const MView &M, const uint32_t *effects, Team &t, int a, float ten) {
        const int a1 = (a * M.h->joint_inv) >> 16, a2 = a - a1 * (5 + M.h->n_rocks);
        const float r1 = t.hop(effects, M.h->grid, 0, a1, ten);
        return r1 + t.hop(effects, M.h->grid, 1, a2, ten);  // ten times -2..2, exact
    }
    template <int J>
    __device__ static bool gone(const State &st) {
        return (st.p >> (kGone0 + J)) & 1;
    }
    __device__ static int cell(const State &st) { return st.p & 0x3fffff; }
    __device__ static int cell_x(int c) { return (c >> 10) & 31; }
    __device__ static int cell_y(int c) { return (c >> 15) & 31; }
    __device__ static uint32_t rocks(const State &st) { return (uint32_t)st.rk; }
    __device__ static int32_t with_reward(int32_t p, float r) { return p | (r > 0.0f ? 1 << 24 : r < 0.0f ? 2 << 24 : 0); }
    __device__ static float reward_of(int32_t w) {
        const int c = (w >> 24) & 3;
        return c == 1 ? 10.0f : c == 2 ? -10.0f : 0.0f;
    }
    __device__ static void from_words(State &st, int32_t w, int32_t rk) {
        st.p = w & ~(3 << 24);
        st.rk = rk;
    }
    __device__ static void from_cell(State &st, int c) {
        st.p = c;
        st.rk = 0;
    }
    __device__ static bool acting(const State &st) { return !gone<1>(st); }
    __device__ static bool ended(const State &st) { return gone<0>(st) && gone<1>(st); }
    __device__ static void settle(State &st) {
        if (ended(st)) st.p |= 1 << kTerm;
    }
    __device__ static float mover(const MView &M, State &st, int b) {
        int z;
        return act<1, false>(M, st, b, 0, z);
    }
    __device__ static int rock_distance(const State &st, int rx, int ry) { return near(st.p, rx, ry); }
    __device__ static bool at(const State &st, int rx, int ry) {
        return ((st.p >> 10) & 31) == rx && ((st.p >> 15) & 31) == ry;
    }
    // Robot J's move c < 4 (any other c: none); true if it leaves the grid.
    template <int J>
    __device__ static bool walk_one(const MView &M, State &st, int c) {
        constexpr int sh = 10 * J;
        const int n = M.h->grid, x = (st.p >> sh) & 31, y = (st.p >> (sh + 5)) & 31;
        if (c == 2 && x + 1 == n) {
            st.p |= 1 << (kGone0 + J);
            return true;
        }
        const int nx = c == 2 ? x + 1 : c == 3 && x > 0 ? x - 1 : x;
        const int ny = c == 0 && y + 1 < n ? y + 1 : c == 1 && y > 0 ? y - 1 : y;
        st.p = (st.p & ~(0x3ff << sh)) | (nx << sh) | (ny << (sh + 5));
        return false;
    }
    __device__ static bool walk(const MView &M, State &st, int c) { return walk_one<1>(M, st, c); }
    __device__ static double exits(const MView &M, const State &st, const double *term) {
        const int n1 = M.h->grid - 1;
        return (gone<0>(st) ? 0.0 : term[n1 - (st.p & 31)]) + (gone<1>(st) ? 0.0 : term[n1 - ((st.p >> 10) & 31)]);
    }
    __device__ static void move_east(const MView &M, const State &st, int R, const double *term, double &value,
                                     int &steps) {
        const int n1 = M.h->grid - 1;
        const int o1 = gone<0>(st) ? -1 : n1 - (st.p & 31), o2 = gone<1>(st) ? -1 : n1 - ((st.p >> 10) & 31);
        const int last = o1 > o2 ? o1 : o2;
        steps = R < 0 ? 0 : R < last + 1 ? R : last + 1;
        value = (o1 >= 0 && o1 < R ? term[o1] : 0.0) + (o2 >= 0 && o2 < R ? term[o2] : 0.0);
    }
};

// ---------------------------------------------------------------------------
// Navigation in a partially known map.  Five int32 rows per scenario: the
// robot (x bits 0-3, y bits 4-7, terminal bit 30) at w[k], then the unknown
// cells' occupancy (cell i in bit i % 32 of row 1 + i / 32) at
// w[(1 + j) * stride + k].  Actions 0 stay, 1-8 move N, NE, E, SE, S, SW, W,
// NW (y grows downwards).  A move draws word 0 of step block 0 (failure);
// a reading draws step blocks 1 and 2 (one word per neighbour).
// ---------------------------------------------------------------------------
constexpr int nav_dx_of(int a) { return (a == 0 || a == 1 || a == 5) ? 0 : (a >= 2 && a <= 4) ? 1 : -1; }
constexpr int nav_dy_of(int a) { return (a == 0 || a == 3 || a == 7) ? 0 : (a == 1 || a == 2 || a == 8) ? -1 : 1; }
// dx + 1 and dy + 1 of each action in two bits; the action of each (dx, dy)
// in four bits at (dy + 1) * 3 + dx + 1
constexpr uint32_t nav_pack_dir(bool y) {
    uint32_t v = 0;
    for (int a = 0; a < 9; ++a) v |= (uint32_t)((y ? nav_dy_of(a) : nav_dx_of(a)) + 1) << (2 * a);
    return v;
}
constexpr uint64_t nav_action_table() {
    uint64_t t = 0;
    for (int a = 0; a < 9; ++a) t |= (uint64_t)a << (4 * ((nav_dy_of(a) + 1) * 3 + nav_dx_of(a) + 1));
    return t;
}

struct NavOps {
    struct State {
        int32_t p;
        uint32_t m0, m1, m2, m3;
    };
    static constexpr uint32_t kDx = nav_pack_dir(false), kDy = nav_pack_dir(true);
    static constexpr uint64_t kAction = nav_action_table();
    static constexpr uint32_t kTerminalObs = 256;

    __device__ __forceinline__ static int dx(int a) { return (int)((kDx >> (2 * a)) & 3u) - 1; }
    __device__ __forceinline__ static int dy(int a) { return (int)((kDy >> (2 * a)) & 3u) - 1; }

    __device__ __forceinline__ static void load(const MView &, const StatesPtr &S, int64_t p, State &st) {
        st.p = S.w[p];
        st.m0 = (uint32_t)S.w[S.stride + p];
        st.m1 = (uint32_t)S.w[2 * S.stride + p];
        st.m2 = (uint32_t)S.w[3 * S.stride + p];
        st.m3 = (uint32_t)S.w[4 * S.stride + p];
    }
    __device__ __forceinline__ static void make_terminal(State &st) {
        st.p = 1 << 30;
        st.m0 = st.m1 = st.m2 = st.m3 = 0;
    }
    __device__ __forceinline__ static void store(const MView &, const StatesPtr &S, int64_t p, const State &st) {
        S.w[p] = st.p;
        S.w[S.stride + p] = (int32_t)st.m0;
        S.w[2 * S.stride + p] = (int32_t)st.m1;
        S.w[3 * S.stride + p] = (int32_t)st.m2;
        S.w[4 * S.stride + p] = (int32_t)st.m3;
    }
    __device__ __forceinline__ static bool terminal(const State &st) { return (st.p >> 30) & 1; }

    // The scenario's map as rows of 16 cells (a set bit: a wall, an occupied
    // unknown cell, or a cell off the map), two rows per word, held in LDS:
    // word h of this lane at rows[64 h], so 64 lanes read 64 banks whatever
    // rows they look at.  A test of a cell is then one LDS read and a shift,
    // with no table of cells; the unknown cells are moved to their grid
    // places by runs of consecutive cells (a field extract and a shift each).
    __device__ __forceinline__ static void make_rows(const MView &M, const State &st, uint32_t *rows) {
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            uint32_t g = M.h->nav_wall_rows[h];
            const int end = M.h->nav_run_begin[h + 1];
            for (int i = M.h->nav_run_begin[h]; i < end; ++i) {
                const uint32_t d = M.h->nav_runs[i];
                const uint32_t q = (d >> 15) & 3u;
                const uint32_t src = q < 2 ? (q == 0 ? st.m0 : st.m1) : (q == 2 ? st.m2 : st.m3);
                g |= __builtin_amdgcn_ubfe(src, d & 31u, (d >> 5) & 31u) << ((d >> 10) & 31u);
            }
            rows[64 * h] = g;
        }
    }
    __device__ __forceinline__ static uint32_t row(const uint32_t *rows, int y) {
        return (rows[64 * (y >> 1)] >> (16 * (y & 1))) & 0xffffu;
    }
    __device__ __forceinline__ static int occupied(const MView &M, const uint32_t *rows, int x, int y) {
        const int n = M.h->grid;
        if (x < 0 || y < 0 || x >= n || y >= n) return 1;
        return (int)((row(rows, y) >> x) & 1u);
    }
    // The eight neighbours of (x, y), bit j that of action j + 1 (1 =
    // occupied; off the map reads occupied).
    __device__ __forceinline__ static uint32_t neighbours(const MView &M, const uint32_t *rows, int x, int y) {
        const uint32_t up = y > 0 ? row(rows, y - 1) : 0xffffu;
        const uint32_t dn = y + 1 < M.h->grid ? row(rows, y + 1) : 0xffffu;
        const uint32_t edge = 0x20001u;  // the columns left of 0 and right of 15
        const uint32_t u = ((up << 1) | edge) >> x, m = ((row(rows, y) << 1) | edge) >> x, d = ((dn << 1) | edge) >> x;
        return ((u >> 1) & 3u) | (m & 4u) | ((d & 4u) << 1) | ((d & 2u) << 3) | ((d & 1u) << 5) | ((m & 1u) << 6) |
               ((u & 1u) << 7);
    }

    // The motion of a step from a live state, with the failure word (word 0
    // of the step block) already drawn (a stay draws none) and the occupancy
    // of the cell the action heads for.
    __device__ __forceinline__ static void move(const MView &M, State &st, int a, uint32_t u_fail, int blocked, float &r) {
        int x = st.p & 15, y = (st.p >> 4) & 15;
        int term = 0;
        if (a == 0) {
            r = -0.2f;
        } else if ((uint64_t)u_fail < M.h->fail_thr) {
            r = -0.1f;  // the move fails: the robot stays
        } else if (blocked) {
            r = -1.0f;  // crash: the robot stays
        } else {
            x += dx(a);
            y += dy(a);
            if (x == M.h->nav_goal_x && y == M.h->grid - 1) {
                r = 20.0f;
                term = 1;
            } else {
                r = -0.1f;
            }
        }
        st.p = x | (y << 4) | (term << 30);
    }
    __device__ __forceinline__ static void move(const MView &M, const uint32_t *rows, State &st, int a, uint32_t u_fail, float &r) {
        move(M, st, a, u_fail, a == 0 ? 0 : occupied(M, rows, (st.p & 15) + dx(a), ((st.p >> 4) & 15) + dy(a)), r);
    }

    // The bits of a reading that are flipped (blocks 1 and 2 of the step).
    __device__ __forceinline__ static uint32_t reading_errors(const MView &M, uint32_t id, uint32_t depth, uint32_t k0, uint32_t k1) {
        const uint4 b1 = philox(id, depth, 1, kTagStep, k0, k1);
        const uint4 b2 = philox(id, depth, 2, kTagStep, k0, k1);
        const uint32_t words[8] = {b1.x, b1.y, b1.z, b1.w, b2.x, b2.y, b2.z, b2.w};
        uint32_t e = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) e |= ((uint64_t)words[j] < M.h->err_thr ? 1u : 0u) << j;
        return e;
    }

    // The goal reward on the shortest 8-connected path, no costs; it is paid
    // on entering the goal, so a robot standing on it must leave and re-enter
    // (two moves).  Distances are 0..15; kNoDistance marks a terminal state.
    static constexpr int kNoDistance = 16;
    __device__ __forceinline__ static int distance(const MView &M, const State &st) {
        if ((st.p >> 30) & 1) return kNoDistance;
        const int ax = abs((st.p & 15) - M.h->nav_goal_x), ay = abs(((st.p >> 4) & 15) - (M.h->grid - 1));
        return ax > ay ? ax : ay;
    }
    __device__ __forceinline__ static float bound_at(const MView &M, int d) {
        return d == kNoDistance ? 0.0f : 20.0f * M.gpow(d > 0 ? d - 1 : 1);
    }
    __device__ __forceinline__ static float upper(const MView &M, const State &st) { return bound_at(M, distance(M, st)); }

    // The default policy heads for the open gate while above the wall, then
    // for the goal: the diagonal step towards the target, else its vertical
    // part, else its horizontal part, the first that lands on a free cell;
    // else the robot stays, and as nothing changes by staying, it stays until
    // the horizon.  It never heads for an occupied cell, so a move that fails
    // only delays the walk, at the cost of a move.  The rollout is then
    // settled by the walk itself -- how many moves it takes, and whether it
    // ends at the goal or stuck; no random numbers -- and by the depth at
    // which that many moves have succeeded, from the failure words.
    enum { kStuck = 0, kGoal = 1, kOver = 2 };
    struct Target {
        bool gate;  // a gate is open: the target above the wall
        int gx;
    };
    __device__ __forceinline__ static Target target_of(const MView &M, const State &st) {
        Target t;
        t.gate = (st.m0 & 3u) != 3u;
        t.gx = !(st.m0 & 1u) ? M.h->nav_gate_x[0] : M.h->nav_gate_x[1];
        return t;
    }
    // Moves of the walk from (x, y) until the goal, a dead end, or `limit`
    // moves (kOver); m receives their number.  Every move goes down, or along
    // a row towards its target.
    __device__ __forceinline__ static int walk(const MView &M, const uint32_t *rows, const Target &t, int x, int y, int limit, int &m) {
        const int goal = M.h->nav_goal_x, last = M.h->grid - 1, wall = M.h->nav_wall;
        m = 0;
        uint32_t here = row(rows, y), below = row(rows, y < 15 ? y + 1 : 15);
        for (;;) {
            const int tx = t.gate && y < wall ? t.gx : goal;
            const int xs = x + (tx > x ? 1 : 0) - (tx < x ? 1 : 0);
            const uint32_t diag = (below >> xs) & 1u, vert = (below >> x) & 1u, side = (here >> xs) & 1u;
            const bool dn = y < last;
            const bool down = dn && !(diag & vert);
            const int nx = dn && !diag ? xs : down ? x : side ? x : xs;
            if (!down && nx == x) return kStuck;
            ++m;
            x = nx;
            if (down) {
                ++y;
                here = below;
                below = row(rows, y < 15 ? y + 1 : 15);
            }
            if (x == goal && y == last) return kGoal;
            if (m >= limit) return kOver;
        }
    }

    // Failures of the moves at depths d0 + base, ... (at most 64), as bits,
    // until `need` moves have succeeded on every lane or n_roll depths are
    // drawn; returns the depths drawn (the same for the wavefront).
    __device__ __forceinline__ static int failures(const MView &M, uint32_t id, int d0, int base, int n_roll, int need, uint32_t k0,
                                   uint32_t k1, uint64_t &F) {
        F = 0;
        int j = 0;
        while (j < 64 && base + j < n_roll && __ballot(j - __popcll(F) < need)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {  // independent blocks in flight
                const uint32_t u = philox(id, (uint32_t)(d0 + base + j + e), 0, kTagStep, k0, k1).x;
                F |= ((uint64_t)u < M.h->fail_thr ? 1ull : 0ull) << (j + e);
            }
            j += 4;
        }
        return j;
    }
    // Depths until the m-th success (m of them at least among the bits of F).
    __device__ __forceinline__ static int depths_until(uint64_t F, int m) {
        int T = m;
        for (;;) {
            const int t = m + __popcll(F & (T >= 64 ? ~0ull : ((1ull << T) - 1ull)));
            if (t == T) return T;
            T = t;
        }
    }

    // Value and steps of a rollout of at most R steps whose walk ends as
    // `kind` after T depths (T > R: not within the rollout), from the sums
    // S(j) = 1 + gamma + ... + gamma^(j-1).
    template <class Sum>
    __device__ __forceinline__ static float walk_value(int kind, int T, int R, const Sum &S, int &steps) {
        steps = R > 0 ? R : 0;
        if (R <= 0) return 0.0f;
        const double move_cost = (double)-0.1f, stay_cost = (double)-0.2f;
        const double all = S(R);
        if (kind == kOver || T > R) return (float)(move_cost * all);
        const double sT = S(T);
        if (kind == kStuck) return (float)(move_cost * sT + stay_cost * (all - sT));
        const double sE = S(T - 1);
        steps = T;
        return (float)(move_cost * sE + 20.0 * (sT - sE));
    }

    // A whole rollout of one state (the stand-alone bounds call; all lanes of
    // a wavefront together, `live` those with a rollout to run).
    __device__ __forceinline__ static float rollout(const MView &M, const RolloutParams &P, const uint32_t *rows, State st, uint32_t id,
                                    int d0, int R, bool live, int &nsteps) {
        nsteps = 0;
        live = live && R > 0 && !terminal(st);
        if (P.policy != HDX_POLICY_DEFAULT)
            return rollout_steps(M, P, rows, live ? st.p : 1 << 30, id, d0, R, 1, 0, nsteps);
        int m = 0, kind = kOver;
        if (live) kind = walk(M, rows, target_of(M, st), st.p & 15, (st.p >> 4) & 15, R, m);
        int need = live && kind != kOver ? m : 0, T = 0, base = 0;
        bool open = need > 0;
        while (__ballot(open && base < R)) {
            uint64_t F;
            // lanes differ in d0 and R; a lane past its own R only pads
            const int j = failures(M, id, d0, base, kHorizon, open ? need : 0, P.k0, P.k1, F);
            const int got = j - __popcll(F);
            if (open && need <= got) {
                T = base + depths_until(F, need);
                open = false;
            }
            need -= got;
            base += j;
        }
        if (open) kind = kOver;
        if (!live) return 0.0f;
        return walk_value(kind, T, R, [&](int j) { return M.gpow_sum(j); }, nsteps);
    }

    // Step by step, for the constant and the random policy, in FP32 in step
    // order.  Lanes come in groups of `width`, all of one scenario, whose random
    // actions and failures are the same for whatever cell it is in: lane c of a
    // group draws those of depths c, width + c, ... and the others read them
    // from it.  p: the robot, rows: its scenario's map.  Called by all lanes of
    // a wavefront, no branch but the loop's own.
    __device__ __forceinline__ static float rollout_steps(const MView &M, const RolloutParams &P, const uint32_t *rows,
                                                          int32_t p, uint32_t id, int d0, int R, int width, int c,
                                                          int &steps) {
        const Modulus pick((uint32_t)P.n_actions);
        const int lane = (int)__lane_id(), first = lane - c;
        const int n = M.h->grid, goal = M.h->nav_goal_x;
        const uint64_t fail_thr = M.h->fail_thr;
        int x = p & 15, y = (p >> 4) & 15;
        bool alive = !((p >> 30) & 1);
        float value = 0.0f, powers = 0.0f;  // lane i: gamma^i of the current 64 depths
        int drawn = 0, at = width;
        steps = 0;
        for (int j = 0;; ++j, ++at) {
            alive &= j < R;
            if (!__ballot(alive)) break;
            if ((j & 63) == 0) powers = M.gpow(min(j + lane, kHorizon - 1));
            const float g = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(powers), j & 63));
            if (at == width) {
                const uint32_t depth = (uint32_t)(d0 + j + c);
                drawn = P.const_action;
                if (P.policy == HDX_POLICY_RANDOM) drawn = (int)pick(philox(id, depth, 0, kTagPolicy, P.k0, P.k1).x);
                drawn |= (uint64_t)philox(id, depth, 0, kTagStep, P.k0, P.k1).x < fail_thr ? 16 : 0;
                at = 0;
            }
            const int word = width > 1 ? __shfl(drawn, first + at, 64) : drawn;
            const int a = word & 15, nx = x + dx(a), ny = y + dy(a);
            const bool stays = a == 0, fails = word >= 16;
            const uint32_t cells = (row(rows, ny & 15) << 1) | 0x20001u;  // the columns left of 0 and right of 15
            const bool wall = (((cells >> (nx + 1)) & 1u) != 0) | ((uint32_t)ny >= (uint32_t)n);
            const bool moves = !(stays | fails | wall), there = moves & (nx == goal) & (ny == n - 1);
            x = moves ? nx : x;
            y = moves ? ny : y;
            const float r = stays ? -0.2f : there ? 20.0f : fails | !wall ? -0.1f : -1.0f;
            const float v = value + g * r;
            value = alive ? v : value;
            steps += alive ? 1 : 0;
            alive &= !there;
        }
        return value;
    }
};

// ---------------------------------------------------------------------------
// Crowd driving: car (position, speed level, terminal) and up to PM
// pedestrians held in registers.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t mix64(uint64_t x) {  // splitmix64 output function
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
__device__ __forceinline__ uint64_t hash_field(uint64_t h, int32_t f) {
    return mix64((h ^ (uint64_t)(uint32_t)f) + 0x9E3779B97F4A7C15ull);
}

// One pedestrian's walk towards its goal (gx, gy) with heading noise from the
// four words of its block: px, py move by one step, or onto the goal when it
// is within one.
//
// Each operation is rounded to nearest once, as an IEEE-754 evaluation of
// the same formulas rounds it.  The root and the four quotients are the
// larger part of a step, and the general sequences for them spend most of
// their instructions on operands near the ends of the exponent range.  Here
// the operands are checked to lie in a middle range (all but a vanishing
// share of them, and a wavefront with one outside takes the general
// operations), where the textbook sequences round correctly: the root by
// Goldschmidt's iteration with a final residual, and quotients by a
// correctly rounded reciprocal -- shared by the two quotients of one
// denominator -- and a residual (Markstein 1990).  Root and reciprocal have
// been compared with the general operations over every significand and the
// exponents -62..62.
__device__ __forceinline__ float recip_rn(float b) {  // 2^-62 <= b < 2^62
    const float r = __builtin_amdgcn_rcpf(b);
    return __builtin_fmaf(__builtin_fmaf(-b, r, 1.0f), r, r);
}
__device__ __forceinline__ float quot_rn(float a, float b, float rb) {  // rb = recip_rn(b)
    const float q = a * rb;
    return __builtin_fmaf(__builtin_fmaf(-b, q, a), rb, q);
}
__device__ __forceinline__ float sqrt_rn(float x) {  // 2^-62 <= x < 2^62
    const float y = __builtin_amdgcn_rsqf(x);
    const float s = x * y, h = 0.5f * y;
    const float e = __builtin_fmaf(-h, s, 0.5f);
    const float s1 = __builtin_fmaf(s, e, s), h1 = __builtin_fmaf(h, e, h);
    return __builtin_fmaf(__builtin_fmaf(-s1, s1, x), h1, s1);
}
// The driving model's constants, read once and kept in scalar registers (left
// to itself the compiler reads them again in every rollout step and waits).
struct PedConst {
    float near_d2, step_len, half_sigma, ih_scale, coll_r2, dt, path_len, top, r_step, r_hit, r_goal;
    uint32_t fail_thr;  // p_fail < 1: 32 bits hold it
    int n_peds;
};
__device__ __forceinline__ PedConst ped_const(const MView &M) {
    auto pin = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
    PedConst C;
    C.near_d2 = pin(M.h->near_d2);
    C.step_len = pin(M.h->step_len);
    C.half_sigma = pin(M.h->half_sigma);
    C.ih_scale = pin(M.h->ih_scale);
    C.coll_r2 = pin(M.h->coll_r2);
    C.dt = pin(M.h->dt);
    C.path_len = pin(M.h->path_len);
    C.top = pin((float)(M.h->n_levels - 1));
    C.r_step = pin(M.h->r_step);
    C.r_hit = pin(M.h->r_step + M.h->r_collision);
    C.r_goal = pin(M.h->r_step + M.h->r_goal);
    C.fail_thr = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)M.h->fail_thr);
    C.n_peds = __builtin_amdgcn_readfirstlane(M.h->n_peds);
    return C;
}

__device__ __forceinline__ void move_ped(const PedConst &C, const uint4 &u, float gx, float gy, float &px, float &py) {
    const int32_t sum = (int32_t)((u.x >> 8) + (u.y >> 8) + (u.z >> 8) + (u.w >> 8));
    const float noise = (float)(sum - 33554430) * C.ih_scale;
    const float dx = gx - px;
    const float dy = gy - py;
    const float d2 = dx * dx + dy * dy;
    const bool near = d2 <= C.near_d2;  // sqrt(d2) <= step_len
    const float t = C.half_sigma * noise;
    const float t2 = t * t;
    const float den = 1.0f + t2, num = 1.0f - t2, two_t = 2.0f * t;
    const float least = fminf(fminf(fabsf(dx), fabsf(dy)), fminf(fabsf(num), fabsf(two_t)));
    const bool middle = (least >= 0x1p-30f) & (d2 < 0x1p60f) & (den < 0x1p60f);
    const float dist = sqrt_rn(d2), rd = recip_rn(dist), rn = recip_rn(den);
    float ux = quot_rn(dx, dist, rd), uy = quot_rn(dy, dist, rd);
    float c = quot_rn(num, den, rn), sn = quot_rn(two_t, den, rn);
    if (__builtin_expect(!(near | middle), 0)) {
        const float root = __builtin_sqrtf(d2);
        ux = dx / root;
        uy = dy / root;
        c = num / den;
        sn = two_t / den;
    }
    const float rx = ux * c - uy * sn;
    const float ry = ux * sn + uy * c;
    px = near ? gx : px + C.step_len * rx;
    py = near ? gy : py + C.step_len * ry;
}

// The car: its speed level (a small whole number, held as a float) after an
// action, its position a step later, and the bound of a state.  Action a
// changes the level by 1 - a, up to the top and down to 0; a level above the top
// (a state's eight bits may hold one) can only be kept or lowered.
__device__ __forceinline__ float ped_level(const PedConst &C, float level, float change, bool failed) {
    const float l = __builtin_amdgcn_fmed3f(level + change, 0.0f, fmaxf(C.top, level));
    return failed ? level : l;
}
__device__ __forceinline__ float ped_advance(const PedConst &C, float s, float level) {
    const float v = 0.5f * level;
    return s + v * C.dt;
}
__device__ __forceinline__ float ped_upper(const MView &M, float s, int term) {
    if (term) return 0.0f;
    const float T = ceilf((M.h->path_len - s) / M.h->reach);
    int Ti = (int)T;
    if (Ti < 1) Ti = 1;
    if (Ti > kHorizon) Ti = kHorizon;
    return M.h->r_goal * M.gg[Ti - 1];
}

// A scenario spread over G lanes (a power of two, 4 to 16), pedestrian q G + j
// in slot q of lane j; lane j also owns the car of action j mod 4 (the fourth
// lane of every four repeats the third action's).  The pedestrians' walk does
// not depend on the car and the random numbers of a depth are the same for
// all actions, so the three actions share every pedestrian's step.
template <int G, int PP>
struct PedLanes {
    float px[PP], py[PP], gx[PP], gy[PP];

    // A slot past the last pedestrian holds a point that never moves and is
    // never near a car.
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int q = 0; q < PP; ++q) px[q] = py[q] = gx[q] = gy[q] = 3e38f;
    }
    __device__ __forceinline__ void walk(const PedConst &C, int j, uint32_t id, uint32_t depth, uint32_t k0,
                                         uint32_t k1) {
#pragma unroll
        for (int q = 0; q < PP; ++q)
            if (q == 0 || q * G < C.n_peds) {
                const uint4 u = philox(id, depth, (uint32_t)(q * G + j + 1), kTagStep, k0, k1);
                move_ped(C, u, gx[q], gy[q], px[q], py[q]);
            }
    }
    // What the lane's car at s sees: bit 0 a pedestrian within the collision
    // radius, bit 8 one to brake for.  Three cars: lane j of every four owns
    // car j (at most 2); one: all lanes own it (car 0).
    template <int kCars>
    __device__ __forceinline__ uint32_t look(const PedConst &C, float s, int car) const {
        float at[kCars];
        at[0] = s;
        if constexpr (kCars == 3) {
            at[0] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x00, 0xf, 0xf, true));
            at[1] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x55, 0xf, 0xf, true));
            at[2] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0xAA, 0xf, 0xf, true));
        }
        bool hit[kCars] = {}, brake[kCars] = {};
#pragma unroll
        for (int q = 0; q < PP; ++q)
            if (q == 0 || q * G < C.n_peds) {
                const float py2 = py[q] * py[q];
                const bool beside = fabsf(py[q]) < 1.5f;
#pragma unroll
                for (int c = 0; c < kCars; ++c) {
                    const float dx = px[q] - at[c];
                    hit[c] |= dx * dx + py2 < C.coll_r2;
                    brake[c] |= beside & (dx >= 0.0f) & (dx <= 3.0f);
                }
            }
        int b = 0;
#pragma unroll
        for (int c = 0; c < kCars; ++c) b |= (hit[c] ? 1 << c : 0) | (brake[c] ? 256 << c : 0);
        b |= __builtin_amdgcn_update_dpp(0, b, 0xB1, 0xf, 0xf, true);  // quad_perm 1,0,3,2
        b |= __builtin_amdgcn_update_dpp(0, b, 0x4E, 0xf, 0xf, true);  // quad_perm 2,3,0,1
        if (G >= 8) b |= __builtin_amdgcn_update_dpp(0, b, 0x141, 0xf, 0xf, true);   // row_half_mirror
        if (G >= 16) b |= __builtin_amdgcn_update_dpp(0, b, 0x140, 0xf, 0xf, true);  // row_mirror
        return (uint32_t)b >> car;
    }
};

// Rollouts of a group's cars from depth d0, of at most R steps (one car: each
// group its own d0 and R): discounted from d0, ending with the car's episode, the tail
// value past the horizon 0; accumulated in FP32 in step order.  see: what the
// cars see at the start.  Called by all lanes of a wavefront.
template <int kCars, int G, int PP>
__device__ __forceinline__ float ped_rollout(const MView &M, const PedConst C, const RolloutParams P,
                                             PedLanes<G, PP> &E, int car, uint32_t id, int d0, int R, float s, float lv,
                                             uint32_t see, bool alive, int &steps) {
    const int lane = (int)__lane_id(), j = lane & (G - 1), first = lane & ~(G - 1);
    float value = 0.0f;
    uint32_t fails = 0, pol = 0;
    steps = 0;
    for (int t = 0; kCars == 1 || t < R; ++t) {
        if constexpr (kCars == 1) alive &= t < R;
        if (!__ballot(alive)) break;
        const int tg = t & (G - 1);
        if (tg == 0) {
            // the next G depths' failure words, one depth per lane
            const uint32_t d = (uint32_t)(d0 + t + j);
            fails = (uint32_t)(__ballot(philox(id, d, 0, kTagStep, P.k0, P.k1).x < C.fail_thr) >> first);
            if (P.policy == HDX_POLICY_RANDOM) {
                const uint32_t w = philox(id, d, 0, kTagPolicy, P.k0, P.k1).x % (uint32_t)kPedActions;
                const uint64_t b0 = __ballot(w & 1u), b1 = __ballot(w & 2u);
                pol = ((uint32_t)(b0 >> first) & 0xffffu) | ((uint32_t)(b1 >> first) << 16);
            }
        }
        float change = (see & 256u) ? -1.0f : 1.0f;  // brake, or accelerate
        if (P.policy == HDX_POLICY_CONST) change = (float)(1 - P.const_action);
        if (P.policy == HDX_POLICY_RANDOM)
            change = (float)(1 - ((int)((pol >> tg) & 1u) | ((int)((pol >> (16 + tg)) & 1u) << 1)));
        lv = ped_level(C, lv, change, ((fails >> tg) & 1u) != 0);
        s = ped_advance(C, s, lv);
        E.walk(C, j, id, (uint32_t)(d0 + t), P.k0, P.k1);
        see = E.template look<kCars>(C, s, car);
        const bool hit = (lv > 0.0f) & ((see & 1u) != 0), there = s >= C.path_len;
        const float v = value + M.gpow(t) * (hit ? C.r_hit : there ? C.r_goal : C.r_step);
        value = alive ? v : value;
        steps += alive ? 1 : 0;
        alive &= !(hit | there);
    }
    return value;
}

}  // namespace hdx
