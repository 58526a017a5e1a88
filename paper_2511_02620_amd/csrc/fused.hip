// Both estimators in one pass over the row: Token-DiFR (Sec. 6.3) and Token-IPT-DiFR (Sec. 6.2)
// share the 16-byte vector each lane has just loaded, so the logits are read from HBM once for
// the two scores.  The two row streams are the ones the single-estimator kernels use
// (gumbel_stream.hpp, ipt_stream.hpp); outputs are bit-identical to theirs.
//
// RANK: the same pass also counts the entries whose raw logit exceeds the Token-DiFR claim's (logit rank, Sec. 7.1).
//
// ADM: the same pass also returns the size of the row's admissible set { v : max y - y_v <= delta } (Sec. 7),
// the count difr_admissible_count makes in a second pass once the maximum is known.
#include "difr_device.hpp"
#include "difr_host.hpp"
#include "gumbel_stream.hpp"
#include "ipt_stream.hpp"
#include "row_stream.hpp"

namespace difr {

// With the rank count or the token search the bf16 body needs 97 registers, one too many for five waves per SIMD, and with marks
// the fp32 one does; asked for five they fit in 96 without vector spills and the rank runs 5% faster.  The other variants ask for
// one wave, which is no constraint (fp32 with the rank: 89 registers; asked for five it came out with 68 bytes of scratch a lane).  The
// peaked bf16 one, 97 registers and four waves, has such 68 bytes since it shares the issue slots by RowPace, for scalars that find no
// vector lane; without either it is slower, us: 1024 x 128,256 flat 73.9 / 81.6, concentrated 52.4 / 53.9, 4096 x 9000 concentrated 48.8 /
// 50.0.  fp32 is alike on concentrated rows (2048 x 128,256 166.1 / 164.6) and faster so on flat ones (174.8 / 183.8).
//
// TOK: how the honest sampler's Token-IPT-DiFR token is found (ipt_stream.hpp).
//
// PACED: whether the rows share the issue slots by RowPace (pace_needed); the variants without it hold the same outputs.
template <int DT, bool ADM, bool RANK, int TOK, bool PEAKED, bool PACED>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(TOK == kTokenMarks || (DT == 0 && (RANK || TOK != kNoToken)) ? 5 : 1))) void score_both_kernel(
    RowBatch b, const int32_t *__restrict__ claimed_ipt, GumbelOutputs og, IptOutputs oi, AdmissibleOutputs oa, int first_last)
{
    typedef typename Elem<DT>::type elt_t;
    constexpr int E = Elem<DT>::kPerVec;
    __shared__ float lds_y[kWaves];
    __shared__ int32_t lds_i[kWaves];
    __shared__ float lds_L[kWaves];
    __shared__ int32_t lds_rank[kWaves];
    __shared__ float lds_f[kWaves];
    __shared__ double lds_d[kWaves];
    __shared__ double mark_Z[TOK == kTokenMarks ? kMarks : 1][kBlock];
    __shared__ float mark_ref[TOK == kTokenMarks ? kMarks : 1][kBlock];
    __shared__ WalkScratch walk;
    __shared__ float adm_lists[ADM ? kWaves * kAdmCap : 1];
    __shared__ int32_t adm_fills[kWaves];
    __shared__ int32_t lds_c[kWaves];

    const int64_t row = blockIdx.x;
    const RowInfo ri = load_row_info(b, row);
    RowInfo ri_ipt = ri;
    ri_ipt.claimed = claimed_ipt ? claimed_ipt[row] : -1;
    if (!ri.seq_ok || !ri.temp_ok) {  // uniform over the workgroup
        gumbel_row_rejected(ri, row, og);
        ipt_row_rejected(ri_ipt, row, oi);
        if (ADM && threadIdx.x == 0) {
            oa.count[row] = 0;
            if (oa.log2_count) oa.log2_count[row] = __builtin_nanf("");
        }
        return;
    }
    const int tid = threadIdx.x;
    const elt_t *x_row = reinterpret_cast<const elt_t *>(b.logits) + row * b.ld;
    const int64_t V = b.V;

    GumbelStream<DT, RANK, false, false, ADM, PEAKED> g(ri, x_row, V, lds_L);
    IptStream<DT> s(ri_ipt, x_row, V, false);
    __syncthreads();
    if (ADM) {
        g.arm_admissible(oa.delta, adm_lists, adm_fills);
        __syncthreads();
    }

    const int full_rounds = (int)((V / E) / kBlock);  // rounds of 256 complete vectors
    IptMarks<TOK> marks(mark_Z, mark_ref, full_rounds);

    typename std::conditional<PACED, RowPace, NoPace>::type pace(first_last, full_rounds);
    stream_rounds<DT, TOK>(g, s, marks, pace, x_row, V, 0, full_rounds, true);
    pace.done();
    if (DT == 0 && !ADM && !rows_aligned(b)) g.bad_sum(s.Z);  // (the admissible set is counted on aligned rows only)
    g.finish(row, og, lds_y, lds_i, lds_rank);
    if (ADM) {
        const float M = g.best_y;  // the row maximum, in every thread
        int32_t c = g.adm_count(lds_c);
        if (!(M == M) || !(fabsf(M) < __builtin_inff())) c = 0;  // as difr_admissible_count: no finite maximum
        if (tid == 0) {
            oa.count[row] = c;
            if (oa.log2_count) oa.log2_count[row] = c > 0 ? __log2f((float)c) : __builtin_nanf("");
        }
    }
    ipt_finish<DT, TOK>(b, ri_ipt, row, x_row, s.c, s.ref(), s.Z, s.P, s.refP(), 0, oi, lds_f, lds_d, marks, &walk);
}

template <int DT, bool ADM, bool RANK, int TOK, bool PEAKED = false>
static void launch_score_both_kernel(const RowBatch &b, const int32_t *claimed_ipt, const GumbelOutputs &og, const IptOutputs &oi,
                                     const AdmissibleOutputs &oa, hipStream_t stream)
{
    const Residence r = residence<score_both_kernel<DT, ADM, RANK, TOK, PEAKED, true>>();
    if constexpr (!PEAKED) {  // (which is for some 300 rows and more)
        if (!pace_needed(b.N, r.units)) {
            score_both_kernel<DT, ADM, RANK, TOK, false, false><<<dim3((unsigned)b.N), dim3(kBlock), 0, stream>>>(b, claimed_ipt, og, oi, oa, 0);
            return;
        }
    }
    score_both_kernel<DT, ADM, RANK, TOK, PEAKED, true><<<dim3((unsigned)b.N), dim3(kBlock), 0, stream>>>(
        b, claimed_ipt, og, oi, oa, pace_from(b.N, r.units * r.per_unit, b.V));
}

template <int DT, int TOK>
static void launch_score_both_of(const RowBatch &b, const int32_t *claimed_ipt, const GumbelOutputs &og, const IptOutputs &oi,
                                 bool peaked, hipStream_t stream)
{
    const AdmissibleOutputs none{0.0f, nullptr, nullptr};
    if (og.logit_rank)  // counted in the same stream, only when asked for; every round is then looked at: no early test
        launch_score_both_kernel<DT, false, true, TOK>(b, claimed_ipt, og, oi, none, stream);
    else if (peaked)
        launch_score_both_kernel<DT, false, false, TOK, true>(b, claimed_ipt, og, oi, none, stream);
    else
        launch_score_both_kernel<DT, false, false, TOK>(b, claimed_ipt, og, oi, none, stream);
}

int launch_score_both(const RowBatch &b, const int32_t *claimed_ipt, const GumbelOutputs &og, const IptOutputs &oi,
                      bool peaked, hipStream_t stream)
{
    auto launch = [&](auto TOK) {
        constexpr int tok = decltype(TOK)::value;
        if (b.dtype == 0)
            launch_score_both_of<0, tok>(b, claimed_ipt, og, oi, peaked, stream);
        else
            launch_score_both_of<1, tok>(b, claimed_ipt, og, oi, peaked, stream);
    };
    switch (token_search(oi.ipt_token, b.V, b.dtype)) {
        case kNoToken: launch(std::integral_constant<int, kNoToken>()); break;
        case kTokenWalk: launch(std::integral_constant<int, kTokenWalk>()); break;
        case kTokenMarks: launch(std::integral_constant<int, kTokenMarks>()); break;
    }
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

int launch_score_both_admissible(const RowBatch &b, const int32_t *claimed_ipt, const GumbelOutputs &og,
                                 const IptOutputs &oi, float delta, int32_t *count, float *log2_count, hipStream_t stream)
{
    const AdmissibleOutputs oa{delta, count, log2_count};
    if (b.dtype == 0)
        launch_score_both_kernel<0, true, false, kNoToken>(b, claimed_ipt, og, oi, oa, stream);
    else
        launch_score_both_kernel<1, true, false, kNoToken>(b, claimed_ipt, og, oi, oa, stream);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace difr
