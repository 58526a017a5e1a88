// The streaming loop over one row, or over a part of its rounds, that the one-pass kernels share.
#pragma once

#include <type_traits>

#include "gumbel_stream.hpp"
#include "ipt_stream.hpp"

namespace difr {

// Stands in for the Gumbel stream where only Token-IPT-DiFR is scored.
struct NoGumbel {
    struct {
        int mode = 0;
    } gate;
    template <int MODE>
    __device__ __forceinline__ void process(u32x4, int, bool) {}
    __device__ __forceinline__ void process_any(u32x4, int, bool) {}
    __device__ __forceinline__ void pickup() {}
    __device__ __forceinline__ void tail() {}
};
// ... and for the IPT stream where only Token-DiFR is.
struct NoIpt {
    static constexpr bool valid = false;
    static constexpr int64_t t = -1;
    __device__ __forceinline__ void fast_round(u32x4) {}
    __device__ __forceinline__ void careful_round(u32x4, int, bool) {}
    __device__ __forceinline__ void snapshot() {}
};

// Full rounds [r0, r1) of the row (256 complete vectors each), and with them, if `last`, what the row holds beyond its full
// rounds.  r1 is the number of full rounds then.
template <int DT, int TOK, class G, class S, class Pace>
__device__ __forceinline__ void stream_rounds(G &g, S &s, IptMarks<TOK> &marks, Pace &pace, const typename Elem<DT>::type *x_row, int64_t V,
                                              int r0, int r1, bool last)
{
    constexpr int E = Elem<DT>::kPerVec;
    const int tid = threadIdx.x;
    const int64_t nvec = V / E;                                      // complete vectors
    const int64_t nvec_total = (V + E - 1) / E;                      // the last vector may be partial
    const bool ragged = last && (int64_t)r1 * kBlock < nvec_total;   // a round that is not full
    const int round_t = s.valid ? (int)((s.t / E) / kBlock) : -1;    // round holding the IPT claim

    // Full rounds [round, r_end): Gumbel gates + IPT accumulation on the same vector.  The loop body is
    // instantiated once per Gumbel gate mode; a change of mode leaves the inner loop.
    int round = r0;
    auto run_rounds = [&](auto mode_tag, int r_end) {
        constexpr int MODE = decltype(mode_tag)::value;
        // one round; returns false when the loop must be left (end reached, or the gate changed mode)
        auto body = [&](const u32x4 &q) {
            g.template process<MODE>(q, round, true);
            s.fast_round(q);
            ++round;
            marks.at(round, s);
            if ((round & 15) == 0) g.pickup();
            pace.at(round);
            return round < r_end && (DT != 0 || g.gate.mode == MODE);
        };
        if constexpr (DT != 0) {
            // fp32: the gate's mode is not used, so there is one loop, and a vector is half the work of a bf16 one, so two are kept in
            // flight (one loop per mode and one vector, now, us: 4096 x 128,256 366 / 347, 16,384 x 4000 142 / 123)
            u32x4 qa = load_round(x_row, round), qb = qa, qc = qa;
            if (round + 1 < r_end) qb = load_round(x_row, round + 1);
            while (true) {
                if (round + 2 < r_end) qc = load_round(x_row, round + 2);
                if (!body(qa)) break;
                if (round + 2 < r_end) qa = load_round(x_row, round + 2);
                if (!body(qb)) break;
                if (round + 2 < r_end) qb = load_round(x_row, round + 2);
                if (!body(qc)) break;
            }
            return;
        }
        // one vector is kept in flight; two copies of the body, so that the vector being loaded and the one
        // being used simply swap roles instead of being copied from register to register every round
        u32x4 qa = load_round(x_row, round), qb = qa;
        while (true) {
            if (round + 1 < r_end) qb = load_round(x_row, round + 1);
            if (!body(qa)) break;
            if (round + 1 < r_end) qa = load_round(x_row, round + 1);
            if (!body(qb)) break;
        }
    };
    auto run_to = [&](int r_end) {
        while (round < r_end) {
            if (DT != 0 || g.gate.mode == 0)
                run_rounds(std::integral_constant<int, 0>(), r_end);
            else if (g.gate.mode == 1)
                run_rounds(std::integral_constant<int, 1>(), r_end);
            else
                run_rounds(std::integral_constant<int, 2>(), r_end);
        }
    };
    // a round in which the IPT stream must look at indices (it holds the claimed token, or it is ragged)
    auto careful = [&](int r, bool prefix_open) {
        u32x4 q = u32x4{0u, 0u, 0u, 0u};
        if (((int64_t)r * kBlock + tid) * E < V) q = load_vector<DT>(x_row, ((int64_t)r * kBlock + tid) * E, V);
        g.process_any(q, r, (int64_t)r * kBlock + tid < nvec);
        s.careful_round(q, r, prefix_open);
    };

    if (s.valid && round_t >= r0 && round_t < r1) {
        run_to(round_t);
        careful(round_t, true);
        round = round_t + 1;
        marks.at(round, s);
        pace.at(round);
        run_to(r1);
        if (ragged) careful(r1, false);
    } else {
        run_to(r1);
        const bool below = s.valid && round_t >= r1;  // everything so far lies below the IPT claim
        if (below) s.snapshot();
        if (ragged) careful(r1, below);
    }
    if (last) g.tail();
}

}  // namespace difr
