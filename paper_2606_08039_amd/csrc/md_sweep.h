// md_sweep.h -- the in-LDS neighbour sweep for the pairwise downwash of
// Eq. 6, shared by the semi-implicit Euler and the Runge-Kutta step kernels.
// Positions of a bin's drones are published to LDS; each drone sums the
// terms of the other drones of its environment in ascending slot order.
#pragma once

#include "md_physics.h"

namespace md {
namespace phys {

// The constants of the pair term with C3s pinned in a vector register: the
// term's fused multiply-add C2s dz + C3s may read only one scalar operand, and
// without this the compiler re-copies C3s into a vector register on every
// iteration of the neighbour loops.
__device__ __forceinline__ KConst pair_consts(const KConst &c) {
    KConst cc = c;
    float c3 = c.C3s;
    asm volatile("" : "+v"(c3));
    cc.C3s = c3;
    return cc;
}

// The same for dw_margin's.
__device__ __forceinline__ KConst margin_consts(const KConst &c) {
    KConst cc = c;
    float c3 = c.C3c;
    asm volatile("" : "+v"(c3));
    cc.C3c = c3;
    return cc;
}

// Sparse sweeps.  The wake is narrow (beta is 3-20 cm at the gaps of layered
// flight, while drones keep a metre apart), so nearly every pair's Gaussian
// underflows to 0 exactly.  The sweeps below first form every pair's margin
// (dw_margin: 7 fused operations, no transcendental, no select) and push its
// sign into a word of bits, then evaluate only the pairs that some lane needs;
// leaving a 0 out of a sum changes no bit of it.  Where a swarm is dense
// enough that most pairs are needed, the tests are the dearer way: a sweep
// whose tests ask for more than its limit of pairs evaluates all of them, in
// this step and the next SPARSE_RETRY - 1, without tests.  (Evaluated one after
// the other in the step that found them too many, and tested again every 8
// steps, dense swarms took up to 8 % longer than without tests at all.)
// Measured without -> with the tests: 512 x 256 drones, 50
// steps, block sweep 617 -> 395 us; 4096 x 64, 60 steps, rotation sweep with
// observations 433 -> 325 us, without 377 -> 240 us; 8192 x 32, 60 steps with
// observations 299 -> 288 us.  Lattices drawn together to 0.3 of their pitch,
// where the tests are given up: 512 x 256 946 (all pairs) -> 682 us, 2048 x 64 with
// observations 340 -> 329 us, without 303 -> 303 us, 8192 x 32 257 -> 252 us, 4096 x
// 32 under wind 245 -> 244 us, Runge-Kutta 2048 x 64, 40 steps 618 -> 562 us.
// The outcomes outlast a step: the block sweep, the rotation of 64 drones and
// the one-lane sweep of the randomised step keep them until a drone of the
// environment (or of the wave) has moved MEMO_MOVE, with a radius that allows
// for it, and evaluate a few pairs more instead of testing all.  A pair that
// is evaluated needlessly adds its exact 0.  Formed at every step -> kept: 512
// x 256 drones, 50 steps 394 -> 176 us, Runge-Kutta 256 x 256, 20 steps 572 ->
// 258 us; 2048 x 64, 60 steps with observations 200 -> 167 us, without 178 ->
// 140 us; 4096 x 32 randomised, 50 steps 333 -> 312 us.
constexpr int SPARSE_RETRY = 32;
// Pairs evaluated side by side where a sweep goes by batches.
constexpr int PAIR_BATCH = 4;
// Smallest environment that takes tests: at 32 drones a third of the 16 shifts
// is needed by some lane and the tests pay a little; at 16 they do not (223
// without, 226 us with them, 8192 environments, 100 steps with observations).
constexpr int SPARSE_MIN_ENV = 32;

// What a sweep keeps from step to step: where the drone stood at the last
// tests, their outcome (a uniform word of shifts; in the block sweep word k in
// lane k; in the one-lane sweep a word of candidates per lane), and the steps
// to run without tests.
struct SweepMemo {
    float x = __builtin_nanf(""), y = 0.f, z = 0.f;  // (x a NaN: nothing is kept)
    uint32_t need = 0;
    int dense = 0;  // (uniform)
    __device__ __forceinline__ bool moved(const Drone &d) const {  // (a NaN has moved)
        const float ex = d.px - x, ey = d.py - y, ez = d.pz - z;
        return !(ex * ex + ey * ey + ez * ez < MEMO_MOVE * MEMO_MOVE);
    }
    __device__ __forceinline__ void stand(const Drone &d) {
        x = d.px;
        y = d.py;
        z = d.pz;
    }
    __device__ __forceinline__ void forget() { x = __builtin_nanf(""); }
};

__device__ __forceinline__ uint32_t push_sign(uint32_t bits, float x) {
    return __builtin_amdgcn_alignbit(bits, __float_as_uint(x), 31);  // bits << 1 | sign
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}

// The OR of a word over the wave (all lanes active), uniform.
__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
    x |= dpp_u32<0xb1>(x);   // quad_perm [1, 0, 3, 2]
    x |= dpp_u32<0x4e>(x);   // quad_perm [2, 3, 0, 1]
    x |= dpp_u32<0x141>(x);  // row_half_mirror
    x |= dpp_u32<0x140>(x);  // row_mirror
    return (uint32_t)(__builtin_amdgcn_readlane((int)x, 0) | __builtin_amdgcn_readlane((int)x, 16) |
                      __builtin_amdgcn_readlane((int)x, 32) | __builtin_amdgcn_readlane((int)x, 48));
}

// This lane's share of the downwash sum over its environment's slots
// [lo, lo + mmax), in ascending order (every LPD-th slot from `sub`).  In a
// uniform bin every environment has mmax drones and the bound check is
// dropped.
template <bool DZMIN, int LPD, int UNROLL>
__device__ __forceinline__ float dw_sweep(const KConst &c0, const float4 *buf, int lo, int sub, int mmax,
                                          int menv, bool uniform, const Drone &d) {
    const KConst c = pair_consts(c0);
    float acc = 0.f;
    if (uniform) {
#pragma unroll UNROLL
        for (int j = sub; j < mmax; j += LPD) {
            const float4 pj = buf[lo + j];
            acc += dw_term<DZMIN>(c, pj.x - d.px, pj.y - d.py, pj.z - d.pz);
        }
    } else {
#pragma unroll UNROLL
        for (int j = sub; j < mmax; j += LPD) {
            const float4 pj = buf[lo + j];
            const float term = dw_term<DZMIN>(c, pj.x - d.px, pj.y - d.py, pj.z - d.pz);
            acc += (j < menv) ? term : 0.f;
        }
    }
    return acc;
}

// LPD lanes per drone, the sum of the one-lane sweep bit for bit: lane `sub`
// evaluates every LPD-th candidate, then the group's terms are added one after
// the other in ascending order, each broadcast to the drone's lanes by a DPP
// operand of the addition.  With eight lanes the running sum is valid in one
// quad at a time: a quad adds its four terms, hands the sum to the other one
// (row_half_mirror), which adds its own four and, in the next group, the
// first four (the candidates' assignment alternates).  Returned in every lane.
// For layouts that one lane per drone leaves at a wave per SIMD or less, where
// a step costs the length of one wave's instruction stream: 64 x 32 drones,
// 100 steps, 220 us with one lane, 129 with four, 100 with eight; 1024 ragged
// environments of 2..32 drones 242, 135 and 157 us (eight lanes: 2.3 waves per
// SIMD).
template <int CTRL>
__device__ __forceinline__ float quad_perm(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float half_mirror(float v) {  // lane 7 - i of each eight
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, true));
}

template <bool DZMIN, int LPD>
__device__ __forceinline__ float dw_lanes(const KConst &c0, const float4 *buf, int slots, int lo, int sub, int mmax,
                                          int menv, const Drone &d) {
    static_assert(LPD == 4 || LPD == 8, "lanes per drone");
    const KConst c = pair_consts(c0);
    float acc = 0.f;
    auto term = [&](int j) {
        // (a candidate past the environment is read from the rest of the
        // buffer, which holds 2 slots entries)
        const float4 q = buf[min(lo + j, 2 * slots - 1)];
        const float t = dw_term<DZMIN>(c, q.x - d.px, q.y - d.py, q.z - d.pz);
        return j < menv ? t : 0.f;
    };
    auto add = [&](float t) {
        acc += quad_perm<0x00>(t);
        acc += quad_perm<0x55>(t);
        acc += quad_perm<0xaa>(t);
        acc += quad_perm<0xff>(t);
    };
    // two groups a round: their terms' latencies overlap
    for (int j = 0; j < mmax; j += 2 * LPD) {
        const float t0 = term(j + sub), t1 = term(j + LPD + (LPD == 8 ? (sub ^ 4) : sub));
        add(t0);
        if (LPD == 8) {
            acc = half_mirror(acc);
            add(t0);
        }
        add(t1);
        if (LPD == 8) {
            acc = half_mirror(acc);
            add(t1);
        }
    }
    // eight lanes: the first quad holds the sum
    if (LPD == 8) {
        const float other = half_mirror(acc);
        acc = sub < 4 ? acc : other;
    }
    return acc;
}

// The one-lane sweep's sum, bit for bit, by tests first: 32 candidates' signs
// (partner above, and a margin that may give a term) into a word per lane,
// then each lane's set bits in ascending order.  KEEP: the outcomes are kept
// (also of partners that may come to be above).  The gather of the set bits is a serial chain through
// LDS, so it pays where the step around it keeps the vector ALU busy and not
// where the sweep alone is the step (SCAN, see dw_sum).  Where a lane asks for
// more than a quarter of its candidates it stops, sets memo.dense, and the
// caller evaluates every pair.
template <bool DZMIN, bool KEEP>
__device__ __forceinline__ float dw_sweep_sparse(const KConst &c0, const float4 *buf, int slots, int slot, int lo,
                                                 int mmax, int menv, const Drone &d, SweepMemo &memo) {
    float acc = 0.f;
    // outcomes are kept where one word and one wave hold them all
    const bool keep = KEEP && mmax <= 32 && slots == 64;
    const float lift = KEEP ? 2.002f * MEMO_MOVE : 0.f;
    const bool test = !keep || __ballot(menv > 0 && memo.moved(d)) != 0ull;
    if (test && keep) memo.stand(d);
#pragma unroll 1
    for (int j0 = 0; j0 < mmax; j0 += 32) {
        uint32_t bits = memo.need;
        if (test) {
            bits = 0;
            const int n = min(32, (mmax - j0 + 7) & ~7);
            const KConst c = margin_consts(c0);
            // (candidates past the environment are read from the rest of the
            // buffer, which holds 2 slots entries, and masked below)
#pragma unroll 1
            for (int k = 0; k < n; k += 8) {
                float x[8];
                const float4 *q = buf + min(lo + j0 + k, 2 * slots - 8);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float4 p = q[u];
                    // negative: the partner is above, or may come to be
                    const float below = d.pz - p.z;
                    const float m = dw_margin<DZMIN, KEEP>(c, p.x - d.px, p.y - d.py, fabsf(below));
                    x[u] = __uint_as_float(__float_as_uint(m) & __float_as_uint(below - lift));
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) bits = push_sign(bits, x[u]);
            }
            bits <<= 32 - n;  // candidate j0 + k in bit 31 - k
            const int left = menv - j0;
            bits &= left >= 32 ? ~0u : ~(~0u >> max(left, 0));
            if (keep) bits &= ~(0x80000000u >> ((slot - lo) & 31));  // not itself
            memo.need = bits;
            // as many rounds as the lane with the most candidates asks for
            if (__ballot(4 * __builtin_popcount(bits) > n) != 0ull) {
                memo.dense = SPARSE_RETRY;
                memo.forget();
                return 0.f;
            }
        }
        const KConst c = pair_consts(c0);
        while (__ballot(bits != 0u) != 0ull) {
            const int k = bits != 0u ? __builtin_clz(bits) : 0;
            const float4 p = buf[lo + j0 + k];
            const float t = dw_term<DZMIN>(c, p.x - d.px, p.y - d.py, p.z - d.pz);
            acc += bits != 0u ? t : 0.f;
            bits &= ~(0x80000000u >> k);
        }
    }
    return acc;
}

// Pair-symmetric downwash sweep: each unordered pair of an environment is
// evaluated once, by lane i for partners (i + d) mod M, d = 1..(M-1)/2, plus
// d = M/2 from the lower half when M is even.  The term goes to the lower
// drone's row of the LDS matrix T (the other entry gets 0); after a barrier
// each drone sums its row in ascending order (the diagonal and the padding
// to a multiple of 4 hold 0, and x + 0 = x).  The term depends only on
// dxy^2 and |dz|, and fl(a - b) = -fl(b - a), so every entry and the sum are
// bitwise those of the all-pairs sweep.
template <bool DZMIN, int UNROLL>
__device__ __forceinline__ void dw_pairs(const KConst &c, const float4 *buf, float *T, int ts, int slot,
                                         int lo, int m, const Drone &d) {
    const int li = slot - lo;
    const int h = (m - 1) >> 1;
#pragma unroll UNROLL
    for (int k = 1; k <= h; ++k) {
        int lj = li + k;
        lj -= (lj >= m) ? m : 0;
        const float4 pj = buf[lo + lj];
        const float dz = pj.z - d.pz;
        const float d2 = dw_d2(pj.x - d.px, pj.y - d.py);
        const float t = dw_raw<DZMIN>(c, d2, fabsf(dz));
        const bool near = dw_near(d2);
        T[slot * ts + lj] = (near && dz > 0.f) ? t : 0.f;
        T[(lo + lj) * ts + li] = (near && dz < 0.f) ? t : 0.f;
    }
    if ((m & 1) == 0 && li < (m >> 1) && m > 0) {
        const int lj = li + (m >> 1);
        const float4 pj = buf[lo + lj];
        const float dz = pj.z - d.pz;
        const float d2 = dw_d2(pj.x - d.px, pj.y - d.py);
        const float t = dw_raw<DZMIN>(c, d2, fabsf(dz));
        const bool near = dw_near(d2);
        T[slot * ts + lj] = (near && dz > 0.f) ? t : 0.f;
        T[(lo + lj) * ts + li] = (near && dz < 0.f) ? t : 0.f;
    }
}

// Pair-symmetric sweep through wave shuffles, for bins whose environments
// each lie inside one wavefront (one lane per drone).  As in dw_pairs, lane i
// evaluates the pairs (i, (i + k) mod M) for k = 1..(M-1)/2; the term stays
// with lane i when its partner is above, and otherwise travels to the
// partner's lane through a cross-lane permute (ds_bpermute): at shift k lane
// j receives from lane (j - k) mod M.  The loop runs to the bin's largest
// environment so that every permute executes with the whole wave.  For even
// M the pair at distance M/2 is evaluated by both members, each keeping it
// when its partner is above.  The summation order (per shift: own term, then
// the received one) is fixed by the drone's place in its environment.
template <bool DZMIN, bool UNIFORM, int UNROLL>
__device__ __forceinline__ float dw_pairs_shfl(const KConst &c0, const float4 *buf, int slot, int lo, int m,
                                               int mmax, const Drone &d) {
    const KConst c = pair_consts(c0);
    // an idle slot (m = 0) runs the loop as a one-drone environment of itself
    const int mm = m > 0 ? m : 1;
    const int li = m > 0 ? slot - lo : 0;
    const int base = (slot & 63) - li;  // the environment's first lane in this wave
    // every lane runs to the bin's largest environment, so that each permute
    // executes with the whole wave; in a uniform bin every environment has
    // that size and no shift needs masking
    const int h = (m - 1) >> 1, hmax = (mmax - 1) >> 1;
    // advanced cyclically: the partner's position (li + k) mod M in `buf`, and
    // the byte address of lane (li - k) mod M, whose term this lane receives
    const float4 *q_beg = buf + lo, *q_end = buf + lo + mm;
    const float4 *qj = buf + lo + li;
    const int p_beg = base * 4, p_last = (base + mm - 1) * 4;
    int ps = (base + li) * 4;
    float acc = 0.f;
#pragma unroll UNROLL
    for (int k = 1; k <= hmax; ++k) {
        qj = (qj + 1 == q_end) ? q_beg : qj + 1;
        ps = (ps == p_beg) ? p_last : ps - 4;
        const float4 q = *qj;
        const float dz = q.z - d.pz;
        const float d2 = dw_d2(q.x - d.px, q.y - d.py);
        const float t = dw_raw<DZMIN>(c, d2, fabsf(dz));
        const bool near = dw_near(d2) && (UNIFORM || k <= h);
        // the term stays with the lower drone: each of the two lane masks
        // selects it or 0 (at dz = 0 neither does, and t is not used)
        float mine = (near && dz > 0.f) ? t : 0.f;
        asm volatile("" : "+v"(mine));
        const float theirs = (near && dz < 0.f) ? t : 0.f;
        const float recv = __int_as_float(__builtin_amdgcn_ds_bpermute(ps, __float_as_int(theirs)));
        acc += mine;
        acc += recv;
    }
    if ((m & 1) == 0 && m > 0) {
        const int half = m >> 1;
        const int lj = li < half ? li + half : li - half;
        const float4 q = buf[lo + lj];
        acc += dw_term<DZMIN>(c, q.x - d.px, q.y - d.py, q.z - d.pz);
    }
    return acc;
}

// The same pairs, shifts, routing and summation order as dw_pairs_shfl, for
// bins whose environments all have one power-of-two size M = 64 / E and sit
// interleaved in their wave: drone li of the wave's environment e in lane
// E li + e.  Then the partner (li + k) mod M of every lane is lane
// (lane + E k) mod 64 and the drone whose term arrives is lane
// (lane - E k) mod 64, for all lanes at once: a rotation of the whole wave.
// The positions are stored twice per wave (entries lane and 64 + lane of the
// wave's 128), so the partner's entry is a fixed offset from the lane's own,
// and the permute address wraps in hardware (lane bits of the byte address);
// with k unrolled neither costs an instruction.
// `seg.at<H>(s)` runs after each of the H + 1 segments (shifts 1..H, then
// the half pair), s = 0..H, and `seg.all()` after a sweep that takes no hook:
// the caller's work to interleave with the sweep (the step kernel's
// observation stores).
struct NoSeg {
    template <int H>
    __device__ __forceinline__ void at(int) const {}
    __device__ __forceinline__ void all() const {}
};

template <bool DZMIN, int E, class Seg>
__device__ __forceinline__ float dw_pairs_rot(const KConst &c0, const float4 *own, int lane, const Drone &d,
                                              const Seg &seg) {
    constexpr int M = 64 / E;
    constexpr int H = (M - 1) / 2;
    const KConst c = pair_consts(c0);
    // the permute addresses pa + 256 - 4 E k fold into the instructions'
    // offset field when pa is formed inside the step: hoisted out of the
    // step loop instead, they would hold one register per shift
    int pa = 4 * lane;
    asm volatile("" : "+v"(pa));
    float acc = 0.f;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
        const float4 q = own[E * k];
        const float dz = q.z - d.pz;
        const float d2 = dw_d2(q.x - d.px, q.y - d.py);
        const float t = dw_raw<DZMIN>(c, d2, fabsf(dz));
        const bool near = dw_near(d2);
        float mine = (near && dz > 0.f) ? t : 0.f;
        // formed here, not where the serial sum reaches it: otherwise its
        // lane mask stays live across shifts and the masks spill
        asm volatile("" : "+v"(mine));
        const float theirs = (near && dz < 0.f) ? t : 0.f;
        const float recv = __int_as_float(__builtin_amdgcn_ds_bpermute(pa + (256 - 4 * E * k), __float_as_int(theirs)));
        acc += mine;
        acc += recv;
        seg.template at<H>(k - 1);
    }
    {
        // M is even: the pair at distance M / 2 (lane + 32), kept by the lower drone
        const float4 q = own[32];
        acc += dw_term<DZMIN>(c, q.x - d.px, q.y - d.py, q.z - d.pz);
    }
    seg.template at<H>(H);
    return acc;
}

// The same sum PAIR_BATCH shifts at a time (the last one of all, by M / 2, has
// no received term: that pair is evaluated by both of its drones): the next
// positions are on their way from LDS while these are evaluated, and terms from
// other lanes are added a batch later.  In the Runge-Kutta kernel the compiler
// otherwise evaluates one shift after the other, and each waits out both
// latencies (50 steps, serial -> batched: 8192 x 16 drones 314 -> 261 us, 4096
// x 32 547 -> 430 us); around the Euler step it overlaps them by itself, and
// batches would spill.
// Environments of 64 drones go through a loop over the batches: unrolled, their
// eight batches would take the registers of every size.
template <bool DZMIN, int E>
__device__ __forceinline__ float dw_pairs_rot_batched(const KConst &c0, const float4 *own, int lane,
                                                      const Drone &d) {
    constexpr int M = 64 / E;
    constexpr int H = (M - 1) / 2;
    const KConst c = pair_consts(c0);
    constexpr int B = M / 2 < PAIR_BATCH ? M / 2 : PAIR_BATCH;
    constexpr int N = (H + 1) / B;  // batches
    // the permute addresses pa - 4 E k fold into the instructions' offset field
    // when pa is formed inside the step: hoisted out of the step loop instead,
    // they would hold one register per shift
    int pa = 4 * lane + 256;
    asm volatile("" : "+v"(pa));
    float x[B], y[B], z[B], mine[B], recv[B];
    auto load = [&](const float4 *q) {
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const float4 v = q[E * u];
            x[u] = v.x;
            y[u] = v.y;
            z[u] = v.z;
        }
    };
    float acc = 0.f;
    // the shifts k .. k + B - 1, q the partner's position at shift k
    auto batch = [&](const float4 *q, int k, bool first, bool last) {
        float dz[B], d2[B], t[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            dz[u] = z[u] - d.pz;
            d2[u] = dw_d2(x[u] - d.px, y[u] - d.py);
        }
        if (!last) load(q + E * B);
#pragma unroll
        for (int u = 0; u < B; ++u) t[u] = dw_raw<DZMIN>(c, d2[u], fabsf(dz[u]));
#pragma unroll
        for (int u = 0; u < B; ++u) {
            asm volatile("" : "+v"(t[u]));  // formed before the first select
        }
        if (!first) {
#pragma unroll
            for (int u = 0; u < B; ++u) {
                acc += mine[u];
                acc += recv[u];
            }
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const bool near = dw_near(d2[u]);
            mine[u] = (near && dz[u] > 0.f) ? t[u] : 0.f;
            // formed here, not where the serial sum reaches it: otherwise its
            // lane mask stays live across shifts and the masks spill
            asm volatile("" : "+v"(mine[u]));
            if (last && u == B - 1) break;
            const float theirs = (near && dz[u] < 0.f) ? t[u] : 0.f;
            recv[u] = __int_as_float(__builtin_amdgcn_ds_bpermute(pa - 4 * E * (k + u), __float_as_int(theirs)));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    load(own + E);
    if constexpr (E == 1) {
        batch(own + 1, 1, true, false);
#pragma unroll 1
        for (int b = 1; b < N - 1; ++b) batch(own + 1 + B * b, 1 + B * b, false, false);
        batch(own + 1 + B * (N - 1), 1 + B * (N - 1), false, true);
    } else {
#pragma unroll
        for (int b = 0; b < N; ++b) batch(own + E * (1 + B * b), 1 + B * b, b == 0, b == N - 1);
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
        acc += mine[u];
        if (u < B - 1) acc += recv[u];
    }
    return acc;
}

// The same sum, bit for bit, from the shifts that some lane of the wave needs,
// ascending.  KEEP: the outcomes are kept until a drone has moved.  The Euler
// step of 32 drones runs its sixteen tests every time, which costs no more
// than keeping their outcomes (8192 x 32 drones, 60 steps with observations:
// 3-8 % longer with kept ones; 2048 x 64 178 run, 139 us kept).  The stages of
// a Runge-Kutta step lie close together and keep them (50 steps, every pair
// evaluated -> kept: 8192 x 32 690 -> 593 us, 4096 x 32 421 -> 418 us, 2048 x
// 64 641 -> 415 us).
// dw_rot_tests: the needed shifts, shift k in bit 32 - k.
template <bool DZMIN, int E, bool KEEP>
__device__ __forceinline__ uint32_t dw_rot_tests(const KConst &c0, const float4 *own, bool valid, const Drone &d,
                                                 SweepMemo &memo) {
    constexpr int M = 64 / E;
    constexpr int H = (M - 1) / 2;
    uint32_t need = memo.need;
    if (!KEEP || __ballot(valid && memo.moved(d)) != 0ull) {
        uint32_t bits = 0;
        const KConst c = margin_consts(c0);
#pragma unroll
        for (int k = 1; k <= H + 1; ++k) {
            const float4 q = own[E * k];
            bits = push_sign(bits, dw_margin<DZMIN, KEEP>(c, q.x - d.px, q.y - d.py, fabsf(q.z - d.pz)));
        }
        need = wave_or(valid ? bits : 0u) << (31 - H);
        if (KEEP) {
            memo.need = need;
            memo.stand(d);
        }
    }
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)need);
}

template <bool DZMIN, int E, class Seg>
__device__ __forceinline__ float dw_pairs_rot_sparse(const KConst &c0, uint32_t need, const float4 *own, int lane,
                                                     const Drone &d, const Seg &seg) {
    constexpr int M = 64 / E;
    constexpr int H = (M - 1) / 2;
    const bool half = (need >> (31 - H)) & 1u;
    need &= ~(1u << (31 - H));
    const KConst c = pair_consts(c0);
    float acc = 0.f;
    seg.all();
    while (need) {
        const int k = __builtin_clz(need) + 1;
        need &= ~(0x80000000u >> (k - 1));
        const float4 q = own[E * k];
        const float dz = q.z - d.pz;
        const float d2 = dw_d2(q.x - d.px, q.y - d.py);
        const float t = dw_raw<DZMIN>(c, d2, fabsf(dz));
        const bool near = dw_near(d2);
        const float mine = (near & (dz > 0.f)) ? t : 0.f;
        const float theirs = (near & (dz < 0.f)) ? t : 0.f;
        const float recv = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (lane - E * k), __float_as_int(theirs)));
        acc += mine;
        acc += recv;
    }
    if (half) {
        const float4 q = own[32];
        acc += dw_term<DZMIN>(c, q.x - d.px, q.y - d.py, q.z - d.pz);
    }
    return acc;
}

template <bool DZMIN, int E, int TESTS, bool BATCHED, class Seg>
__device__ __forceinline__ float dw_rot_size(const KConst &c, const float4 *own, int lane, bool valid, const Drone &d,
                                             const Seg &seg, SweepMemo &memo) {
    constexpr int H = (64 / E - 1) / 2;
    if (64 / E >= TESTS) {
        if (__builtin_amdgcn_readfirstlane(memo.dense) == 0) {
            constexpr bool KEEP = E == 1 || BATCHED;
            const uint32_t need = dw_rot_tests<DZMIN, E, KEEP>(c, own, valid, d, memo);
            if (__builtin_popcount(need >> (32 - H)) <= H / 2)
                return dw_pairs_rot_sparse<DZMIN, E>(c, need, own, lane, d, seg);
            memo.dense = SPARSE_RETRY;
            if (KEEP) memo.forget();
        }
        --memo.dense;
    }
    if constexpr (BATCHED) return dw_pairs_rot_batched<DZMIN, E>(c, own, lane, d);
    return dw_pairs_rot<DZMIN, E>(c, own, lane, d, seg);
}

// TESTS: the smallest environment that is swept by tests first.
template <bool DZMIN, int TESTS = SPARSE_MIN_ENV, bool BATCHED = false, class Seg = NoSeg>
__device__ __forceinline__ float dw_rot(const KConst &c, const float4 *own, int lane, int m, bool valid, const Drone &d,
                                        SweepMemo &memo, const Seg &seg = Seg()) {
    switch (m) {
        case 64: {
            // 31 shifts unrolled leave no registers for interleaved stores
            const float r = dw_rot_size<DZMIN, 1, TESTS, BATCHED>(c, own, lane, valid, d, NoSeg(), memo);
            seg.all();
            return r;
        }
        case 32: return dw_rot_size<DZMIN, 2, TESTS, BATCHED>(c, own, lane, valid, d, seg, memo);
        case 16: return dw_rot_size<DZMIN, 4, TESTS, BATCHED>(c, own, lane, valid, d, seg, memo);
        case 8: return dw_rot_size<DZMIN, 8, TESTS, BATCHED>(c, own, lane, valid, d, seg, memo);
        case 4: return dw_rot_size<DZMIN, 16, TESTS, BATCHED>(c, own, lane, valid, d, seg, memo);
        default: return dw_rot_size<DZMIN, 32, TESTS, BATCHED>(c, own, lane, valid, d, seg, memo);
    }
}

// Block-symmetric sweep, for environments of more than BLOCK_MIN_ENV drones,
// each in whole waves of its own (ceil(M / 64) of them, the last one padded
// with lanes whose position is out of every range).  Each unordered pair is
// evaluated once: wave a takes the pairs inside itself (lanes i and i + k, k =
// 1..31 with the term routed, k = 32 by both), and those with wave (a + d) mod
// W for d = 1..(W - 1) / 2, all 64 shifts; for even W the two waves of
// distance W / 2 share their 64 shifts (0..31 and, from the upper one, 1..32).
// At shift k lane i's partner is lane (i + k) mod 64 of the other wave, whose
// positions are stored twice in LDS (a fixed offset per shift); terms for the
// partners are summed in a register that rotates by one lane per shift, so
// lane i's always belongs to partner i + k, and reach the other wave through
// LDS once per block.  An all-pairs sweep evaluates twice the terms; here a
// term costs a compare, a select, an add and a rotation more.
// The order of a drone's sum depends only on its place in its environment.
// 512 environments x 256 drones, 50 steps: 895 us with the all-pairs sweep,
// 617 us with every pair of this one evaluated, 176 us with tests that are
// kept.  What bounds it then is the step of one wave, with two waves per SIMD
// in this layout: the vector ALU is active for a third of a wave's cycles
// (counters over 1500 steps of flight).
// dw_block sweeps and writes the sums for other waves; after a barrier
// dw_block_rest adds those that other waves left for this one.
//
// Shifts go in batches of PAIR_BATCH: a batch's positions are read from LDS
// while the previous one is evaluated, and its reciprocals and exponentials
// overlap one another (one pair after the other, each waits out the LDS and
// the two transcendental latencies: two waves per SIMD do not cover them).

struct PairBatch {
    float x[PAIR_BATCH], y[PAIR_BATCH], z[PAIR_BATCH];
    __device__ __forceinline__ void load(const float4 *q) {
#pragma unroll
        for (int u = 0; u < PAIR_BATCH; ++u) {
            x[u] = q[u].x;
            y[u] = q[u].y;
            z[u] = q[u].z;
        }
    }
};

// One batch: the terms of this lane's drone onto acc, those of the partners
// onto the rotating sum `theirs`; with LAST_OWN the last pair is evaluated by
// both drones and leaves the partner's term out.
template <bool DZMIN, bool LAST_OWN>
__device__ __forceinline__ void dw_batch(const KConst &c, const PairBatch &q, const Drone &d, float &acc, float &theirs) {
    float dz[PAIR_BATCH], d2[PAIR_BATCH], t[PAIR_BATCH];
#pragma unroll
    for (int u = 0; u < PAIR_BATCH; ++u) {
        dz[u] = q.z[u] - d.pz;
        d2[u] = dw_d2(q.x[u] - d.px, q.y[u] - d.py);
    }
#pragma unroll
    for (int u = 0; u < PAIR_BATCH; ++u) t[u] = dw_raw<DZMIN>(c, d2[u], fabsf(dz[u]));
    // all values formed before the first select (which would otherwise become
    // a branch around its value)
    static_assert(PAIR_BATCH == 4, "operands below");
    asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
#pragma unroll
    for (int u = 0; u < PAIR_BATCH; ++u) {
        const bool near = dw_near(d2[u]);
        acc += (near & (dz[u] > 0.f)) ? t[u] : 0.f;
        if (LAST_OWN && u == PAIR_BATCH - 1) break;
        const float out = (near & (dz[u] < 0.f)) ? t[u] : 0.f;
        // wave_rol:1, from lane + 1
        theirs = out + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(theirs), 0x134, 0xf, 0xf, true));
    }
    __builtin_amdgcn_sched_barrier(0);
}

// 2 N batches from q on (the read ahead of the last one stays inside the bin's LDS).
template <bool DZMIN, bool LAST_OWN>
__device__ __forceinline__ void dw_batches(const KConst &c, const float4 *q, int N, const Drone &d, float &acc,
                                           float &theirs) {
    PairBatch A, B;
    A.load(q);
#pragma unroll 1
    for (int k = 1; k < N; ++k) {
        B.load(q + PAIR_BATCH);
        dw_batch<DZMIN, false>(c, A, d, acc, theirs);
        A.load(q + 2 * PAIR_BATCH);
        dw_batch<DZMIN, false>(c, B, d, acc, theirs);
        q += 2 * PAIR_BATCH;
    }
    B.load(q + PAIR_BATCH);
    dw_batch<DZMIN, false>(c, A, d, acc, theirs);
    dw_batch<DZMIN, LAST_OWN>(c, B, d, acc, theirs);
}

// The tests of 32 shifts of a block from q on: those that some lane needs,
// shift k in bit 31 - k.
template <bool DZMIN>
__device__ __forceinline__ uint32_t dw_block_tests(const KConst &c0, const float4 *q, bool valid, const Drone &d) {
    uint32_t bits = 0;
    const KConst c = margin_consts(c0);
#pragma unroll 1
    for (int k = 0; k < 32; k += 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float4 p = q[k + u];
            x[u] = dw_margin<DZMIN, true>(c, p.x - d.px, p.y - d.py, fabsf(p.z - d.pz));
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) bits = push_sign(bits, x[u]);
    }
    return wave_or(valid ? bits : 0u);
}

// The needed ones of 32 shifts from q on: the same terms onto the same sums as
// dw_batches.  `theirs` belongs to the partner of shift `at` (both counted from
// q) on entry and on return.
template <bool DZMIN, bool LAST_OWN>
__device__ __forceinline__ void dw_block_sparse(const KConst &c, uint32_t need, const float4 *q, int lane,
                                                const Drone &d, float &acc, float &theirs, int &at) {
    while (need) {
        const int k = __builtin_clz(need);
        need &= ~(0x80000000u >> k);
        const float4 p = q[k];
        const float moved = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (lane + k - at), __float_as_int(theirs)));
        const float dz = p.z - d.pz;
        const float d2 = dw_d2(p.x - d.px, p.y - d.py);
        const float t = dw_raw<DZMIN>(c, d2, fabsf(dz));
        const bool near = dw_near(d2);
        acc += (near & (dz > 0.f)) ? t : 0.f;
        if (LAST_OWN && k == 31) break;
        theirs = moved + ((near & (dz < 0.f)) ? t : 0.f);
        at = k;
    }
}

// The waves of an environment form their tests at the same step: each
// publishes (in its positions' fourth component, before the step's barrier)
// whether it asks for that, because one of its drones has moved or because its
// steps without tests are over (memo.dense has come down to 1).
__device__ __forceinline__ float dw_block_asks(const SweepMemo &memo, bool valid, const Drone &d) {
    return memo.dense == 1 || __ballot(valid && memo.moved(d)) != 0ull ? 1.f : 0.f;
}

template <bool DZMIN>
__device__ __forceinline__ float dw_block(const KConst &c0, const float4 *pos, float *sums, int slots, int slot,
                                          int lo_lane, int m_lane, bool valid, const Drone &d, SweepMemo &memo) {
    const int lane = slot & 63;
    const int lo = __builtin_amdgcn_readfirstlane(lo_lane);
    const int W = (__builtin_amdgcn_readfirstlane(m_lane) + 63) >> 6;
    const int a = (__builtin_amdgcn_readfirstlane(slot) - lo) >> 6;
    float acc = 0.f, theirs = 0.f;
    if (W == 0) return 0.f;
    // word 0: the wave's own 32 shifts; then two words per block of 64, one
    // for the shared half block
    const float4 *own = pos + 2 * (lo + 64 * a) + lane + 1;
    auto block = [&](int dd, int &b, int &k0, bool &half) {
        half = 2 * dd == W;
        b = a + dd < W ? a + dd : a + dd - W;
        k0 = half && b < a ? 1 : 0;
        return pos + 2 * (lo + 64 * b) + lane + k0;
    };
    const bool asked = __ballot(lane < W && pos[2 * (lo + 64 * (lane < W ? lane : 0))].w > 0.f) != 0ull;
    int dense = __builtin_amdgcn_readfirstlane(memo.dense);
    if (asked) {
        memo.stand(d);
        if (dense <= 1) {
            uint32_t words = 0, w = dw_block_tests<DZMIN>(c0, own, valid, d);
            int n = 1, count = __builtin_popcount(w);
            words = lane == 0 ? w : 0u;
#pragma unroll 1
            for (int dd = 1; dd <= W >> 1; ++dd) {
                int b, k0;
                bool half;
                const float4 *q = block(dd, b, k0, half);
#pragma unroll 1
                for (int h = 0; h < (half ? 1 : 2); ++h) {
                    w = dw_block_tests<DZMIN>(c0, q + 32 * h, valid, d);
                    count += __builtin_popcount(w);
                    words = lane == n ? w : words;
                    ++n;
                }
            }
            memo.need = words;
            // 32 W shifts were tested; one after the other, twelve W take about
            // as long as all of them in batches (30 steps, limit 8 W / 12 W / 16 W,
            // lattices at 0.7 and 0.35 of their pitch: 11 x 256 drones 160 / 160 /
            // 160 and 288 / 290 / 337 us, 390 x 256 307 / 362 / 395 and 399 / 404 /
            // 454, 15 x 192 222 / 141 / 141 and 218 / 231 / 231, 520 x 192 under
            // Runge-Kutta 1127 / 909 / 910 and 1496 / 1490 / 1490)
            dense = count > 12 * W ? SPARSE_RETRY + 1 : 0;
        }
    }
    memo.dense = max(dense - 1, 0);
    const bool sparse = dense == 0;
    auto word = [&](int k) { return (uint32_t)__builtin_amdgcn_readlane((int)memo.need, k); };
    const KConst c = pair_consts(c0);
    int at = 30;
    if (sparse)
        dw_block_sparse<DZMIN, true>(c, word(0), own, lane, d, acc, theirs, at);
    else
        dw_batches<DZMIN, true>(c, own, 32 / (2 * PAIR_BATCH), d, acc, theirs);
    // shift at + 1's partner terms: lane - (at + 1)'s
    acc += __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (lane - 1 - at), __float_as_int(theirs)));
    int n = 1;
#pragma unroll 1
    for (int dd = 1; dd <= W >> 1; ++dd) {
        int b, k0;
        bool half;
        const float4 *q = block(dd, b, k0, half);
        theirs = 0.f;
        at = half ? 31 : 63;
        if (sparse) {
            at = 0;
            dw_block_sparse<DZMIN, false>(c, word(n++), q, lane, d, acc, theirs, at);
            if (!half) {
                at -= 32;
                dw_block_sparse<DZMIN, false>(c, word(n++), q + 32, lane, d, acc, theirs, at);
                at += 32;
            }
        } else {
            dw_batches<DZMIN, false>(c, q, (half ? 32 : 64) / (2 * PAIR_BATCH), d, acc, theirs);
        }
        sums[(dd - 1) * slots + lo + 64 * b + ((lane + k0 + at) & 63)] = theirs;
    }
    return acc;
}

__device__ __forceinline__ float dw_block_rest(const float *sums, int slots, int slot, int m_lane, float acc) {
    const int W = (__builtin_amdgcn_readfirstlane(m_lane) + 63) >> 6;
    for (int dd = 0; dd < W >> 1; ++dd) acc += sums[dd * slots + slot];
    return acc;
}

// Downwash sum (without K1) of this slot's drone against the positions in
// `buf`.  SYM 0: the all-pairs sweep over LPD lanes (their partial sums
// combined in a fixed order); SYM 1: the pair-symmetric sweep through the LDS
// term matrix (it contains the barrier between the term writes and the row
// sums; bitwise equal to SYM 0 with one lane); SYM 2: the pair-symmetric
// sweep through wave shuffles (environments inside one wave); SYM 3: the same
// sweep as a whole-wave rotation on interleaved uniform bins (bitwise equal
// to SYM 2).
// SCAN: the one-lane sweep by tests first, in the kernels with wind or
// randomisation, whose other work covers its latencies (4096 x 32 randomised
// drones, 50 steps: 367 without, 333 us with it, 312 us with kept outcomes; the
// plain step 299 and 319).  1: tests at every step (wind: 190 us, 2048 ragged
// environments, 193 with kept outcomes), 2: outcomes kept (randomisation).
template <int LPD, int UNROLL, int SYM, int TESTS = SPARSE_MIN_ENV, int SCAN = 0, bool BATCHED = false>
__device__ __forceinline__ float dw_sum(const KConst &c, const float4 *buf, float *tmat, int ts, int slots, int slot,
                                        int sub, int lo, int mmax, int menv, bool uniform, bool valid,
                                        const Drone &d, SweepMemo &memo) {
    float acc = 0.f;
    if constexpr (SYM == SWEEP_LANES) {
        return c.dz_min > 0.f ? dw_lanes<true, LPD>(c, buf, slots, lo, sub, mmax, menv, d)
                              : dw_lanes<false, LPD>(c, buf, slots, lo, sub, mmax, menv, d);
    }
    if (SYM == 3) {
        // interleaved uniform bins (see dw_pairs_rot): `buf` holds each wave's
        // positions twice, 128 entries per wave
        const int lane = slot & 63;
        const float4 *own = buf + 2 * (slot - lane) + lane;
        acc = c.dz_min > 0.f ? dw_rot<true, TESTS, BATCHED>(c, own, lane, mmax, valid, d, memo)
                             : dw_rot<false, TESTS, BATCHED>(c, own, lane, mmax, valid, d, memo);
    } else if (SYM == 2) {
        // `uniform` and dz_min are the same for the whole workgroup: the
        // permutes inside run with every lane of the wave
        if (uniform)
            acc = c.dz_min > 0.f ? dw_pairs_shfl<true, true, UNROLL>(c, buf, slot, lo, menv, mmax, d)
                                 : dw_pairs_shfl<false, true, UNROLL>(c, buf, slot, lo, menv, mmax, d);
        else
            acc = c.dz_min > 0.f ? dw_pairs_shfl<true, false, UNROLL>(c, buf, slot, lo, menv, mmax, d)
                                 : dw_pairs_shfl<false, false, UNROLL>(c, buf, slot, lo, menv, mmax, d);
    } else if (SYM == 1) {
        if (c.dz_min > 0.f)
            dw_pairs<true, UNROLL>(c, buf, tmat, ts, slot, lo, menv, d);
        else
            dw_pairs<false, UNROLL>(c, buf, tmat, ts, slot, lo, menv, d);
        __syncthreads();
        // ascending row sum, four entries per 16-byte read (zero padded)
        const float4 *row = (const float4 *)(tmat + slot * ts);
        for (int j = 0; j < ((menv + 3) >> 2); ++j) {
            const float4 t = row[j];
            acc += t.x;
            acc += t.y;
            acc += t.z;
            acc += t.w;
        }
    } else {
        bool every = true;
        if constexpr (SCAN != 0 && LPD == 1) {
            if (mmax >= SPARSE_MIN_ENV && __builtin_amdgcn_readfirstlane(memo.dense) == 0)
                acc = c.dz_min > 0.f ? dw_sweep_sparse<true, SCAN == 2>(c, buf, slots, slot, lo, mmax, menv, d, memo)
                                     : dw_sweep_sparse<false, SCAN == 2>(c, buf, slots, slot, lo, mmax, menv, d, memo);
            every = mmax < SPARSE_MIN_ENV || __builtin_amdgcn_readfirstlane(memo.dense) > 0;
            memo.dense -= memo.dense > 0 ? 1 : 0;
        }
        if (every)
            acc = c.dz_min > 0.f ? dw_sweep<true, LPD, UNROLL>(c, buf, lo, sub, mmax, menv, uniform, d)
                                 : dw_sweep<false, LPD, UNROLL>(c, buf, lo, sub, mmax, menv, uniform, d);
    }
    // the partial sums of a drone's lanes, combined across the lanes of a
    // quad by DPP quad permutes (lane ^ 1, then lane ^ 2; every lane of the
    // wave is active here); a + b = b + a exactly, so all lanes of a drone
    // hold the same sum
    if (LPD >= 2) {
        const float o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc), 0xB1, 0xF, 0xF, true));
        acc = acc + o;
    }
    if (LPD >= 4) {
        const float o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc), 0x4E, 0xF, 0xF, true));
        acc = acc + o;
    }
    return acc;
}

}  // namespace phys
}  // namespace md
