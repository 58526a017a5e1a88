// Token-IPT-DiFR row kernels: regenerate the seeded uniform u, form p = softmax(x / T)
// and its CDF in ascending token order, and report the claimed token's interval
// [a, b) = [Fbar_{t-1}, Fbar_t), the distance of u from it, and optionally the Gaussian
// log-mass and the honest sampler's token  min{ v : C_v > u }.
// (Sec. 3.2 softmax and IPT sampler; Sec. 6.2 and the appendix algorithm
// "convolved Gaussian score".)
//
// One workgroup per token row, one streaming pass; nothing of size V is stored.  Only when the
// honest sampler's token is asked for and differs from the claim is the row read a second time.
#include <type_traits>

#include "difr_device.hpp"
#include "difr_host.hpp"
#include "ipt_stream.hpp"

namespace difr {

// Streaming kernel (the streaming state is described in ipt_stream.hpp).  TOK: how the honest sampler's token is found.
//
// Bound by reading; what costs beside it is the end of a launch, where the rows left over have too few bytes in flight.
//
// Eight waves per SIMD (without the token; the compiler's own choice, 102 scalar registers, held six): 2048 rows fit at once.  With the
// marks it is six, by 100 scalar registers; the LDS of seven marks leaves room for seven.
//
// DEEP: three vectors in flight beside the one in use instead of one (ipt_deep); always with the marks: every row reads a part of itself
// again, when others have ended.  bf16, V = 128,256, us with one / three: 1024 rows 60 / 56, 2048 110 / 99, 4096 204 / 188.
template <int DT, int TOK, bool DEEP>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(TOK == kNoToken ? 8 : 1))) void ipt_score_kernel(RowBatch b, IptOutputs o)
{
    typedef typename Elem<DT>::type elt_t;
    constexpr int E = Elem<DT>::kPerVec;
    __shared__ float lds_f[kWaves];
    __shared__ double lds_d[kWaves];
    __shared__ double mark_Z[TOK == kTokenMarks ? kMarks : 1][kBlock];
    __shared__ float mark_ref[TOK == kTokenMarks ? kMarks : 1][kBlock];
    __shared__ WalkScratch walk;
    __shared__ int32_t lds_rank[kWaves];

    const int64_t row = blockIdx.x;
    const RowInfo ri = load_row_info(b, row);
    if (ipt_row_rejected(ri, row, o)) return;
    const elt_t *x_row = reinterpret_cast<const elt_t *>(b.logits) + row * b.ld;
    const int64_t V = b.V;

    IptStream<DT> s(ri, x_row, V, o.logit_rank != nullptr);

    const int64_t nvec_total = (V + E - 1) / E;                      // the last vector may be partial
    const int full_rounds = (int)((V / E) / kBlock);                 // rounds of 256 complete vectors
    const int n_rounds = (int)((nvec_total + kBlock - 1) / kBlock);  // full_rounds or full_rounds + 1
    const int round_t = s.valid ? (int)((s.t / E) / kBlock) : -1;
    IptMarks<TOK> marks(mark_Z, mark_ref, full_rounds);

    auto stream = [&](int r0, int r1) {  // full rounds [r0, r1)
        if (r0 >= r1) return;
        int round = r0;
        auto body = [&](const u32x4 &q) {
            s.fast_round(q);
            marks.at(++round, s);
            return round < r1;
        };
        if constexpr (!DEEP) {
            u32x4 q_next = load_round(x_row, round);
            while (true) {
                const u32x4 q = q_next;
                if (round + 1 < r1) q_next = load_round(x_row, round + 1);
                if (!body(q)) break;
            }
        } else {
            u32x4 qa = load_round(x_row, round), qb = qa, qc = qa, qd = qa;
            if (round + 1 < r1) qb = load_round(x_row, round + 1);
            if (round + 2 < r1) qc = load_round(x_row, round + 2);
            while (true) {
                if (round + 3 < r1) qd = load_round(x_row, round + 3);
                if (!body(qa)) break;
                if (round + 3 < r1) qa = load_round(x_row, round + 3);
                if (!body(qb)) break;
                if (round + 3 < r1) qb = load_round(x_row, round + 3);
                if (!body(qc)) break;
                if (round + 3 < r1) qc = load_round(x_row, round + 3);
                if (!body(qd)) break;
            }
        }
    };
    auto careful = [&](int round, bool prefix_open) {
        u32x4 q = u32x4{0u, 0u, 0u, 0u};
        if (round < full_rounds)  // uniform
            q = load_round(x_row, round);
        else if (s.has_vector(round))
            q = load_vector<DT>(x_row, ((int64_t)round * kBlock + threadIdx.x) * E, V);
        s.careful_round(q, round, prefix_open);
    };

    if (s.valid && round_t < full_rounds) {
        stream(0, round_t);
        careful(round_t, true);
        marks.at(round_t + 1, s);
        stream(round_t + 1, full_rounds);
        if (n_rounds > full_rounds) careful(full_rounds, false);
    } else {
        stream(0, full_rounds);
        if (s.valid) s.snapshot();  // everything so far lies below the claimed token
        if (n_rounds > full_rounds) careful(full_rounds, s.valid);
    }
    const int32_t above = s.total_above(lds_rank);
    ipt_finish<DT, TOK>(b, ri, row, x_row, s.c, s.ref(), s.Z, s.P, s.refP(), above, o, lds_f, lds_d, marks, &walk);
}

template <int DT, int TOK>
static void launch_ipt(const RowBatch &b, const IptOutputs &o, hipStream_t stream)
{
    const dim3 grid((unsigned)b.N), block(kBlock);
    const int64_t rounds = b.V / (Elem<DT>::kPerVec * kBlock);
    if constexpr (TOK == kTokenMarks) {
        ipt_score_kernel<DT, TOK, true><<<grid, block, 0, stream>>>(b, o);
    } else {
        // (workgroups that fit: eight to a unit without the token; with it, where rows are walked from their start, six)
        const Residence r = residence<ipt_score_kernel<DT, kNoToken, false>>();
        if (ipt_deep(b.N, r.units * r.per_unit, rounds))
            ipt_score_kernel<DT, TOK, true><<<grid, block, 0, stream>>>(b, o);
        else
            ipt_score_kernel<DT, TOK, false>
                <<<grid, block, TOK == kNoToken ? ipt_idle_lds(b.N, r.units, r.per_unit, rounds) : 0u, stream>>>(b, o);
    }
}

int launch_ipt_score(const RowBatch &b, float *dist, float *cdf_lo, float *cdf_hi, float *u,
                     int32_t *ipt_token, double sigma, double eps, float *log_mass, uint8_t *flags,
                     int32_t *logit_rank, hipStream_t stream)
{
    const IptOutputs o{dist, cdf_lo, cdf_hi, u, ipt_token, sigma, eps, log_mass, flags, logit_rank};
    auto launch = [&](auto TOK) {
        constexpr int tok = decltype(TOK)::value;
        if (b.dtype == 0)
            launch_ipt<0, tok>(b, o, stream);
        else
            launch_ipt<1, tok>(b, o, stream);
    };
    switch (token_search(ipt_token, b.V, b.dtype)) {
        case kNoToken: launch(std::integral_constant<int, kNoToken>()); break;
        case kTokenWalk: launch(std::integral_constant<int, kTokenWalk>()); break;
        case kTokenMarks: launch(std::integral_constant<int, kTokenMarks>()); break;
    }
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace difr
