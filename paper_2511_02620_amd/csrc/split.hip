// Small batches: a row is shared by several workgroups.
//
// One workgroup per row leaves the chip idle when there are fewer rows than it takes to fill 256 compute units, and a row of
// 151,936 bf16 logits keeps its one workgroup busy for 33 us (74 rounds, one wave per SIMD, nothing to hide the latency
// of a round's dependent instructions).  Here a row's full rounds are divided evenly over `parts` workgroups, each of which
// streams its share exactly as the one-workgroup kernels do (row_stream.hpp) and leaves one partial result; a second kernel
// merges the partial results of a row in vocabulary order and writes the outputs.  What bounds it then is the latency of two
// dependent launches and of the set-up of a row (the claimed token's score).
//
// The Token-DiFR outputs are exact selections and do not depend on the split.  The Token-IPT-DiFR sums are taken against
// whole-number exponents, so that merging multiplies by exact powers of two.  The admissible set's scores travel as a list per
// part, cut against the part's own maximum; a row whose lists do not hold them all is counted again by the merging
// workgroup, with the maximum known.
#include "difr_device.hpp"
#include "difr_host.hpp"
#include "gumbel_stream.hpp"
#include "ipt_stream.hpp"
#include "row_stream.hpp"

namespace difr {

constexpr int kMaxParts = 64;      // the merge reads one partial result per lane
constexpr int kSplitAdmCap = 512;  // admissible-set scores a part can pass on

struct Partial {
    double Z, P;
    float M, best_y;
    int32_t best_v, above, bad;
    int32_t adm_n;  // scores in the part's list, -1: more than it holds
};

struct SplitWorkspace {
    Partial *part;  // [N][parts]
    float *adm;     // [N][parts][kSplitAdmCap], or null
    int parts;
};

// rows [first, end) of the part's full rounds
__device__ __forceinline__ int part_begin(int part, int parts, int full_rounds) { return (int)((int64_t)part * full_rounds / parts); }

// NANS (Token-DiFR alone): bf16 rows that do not start on 16 bytes (gumbel_stream.hpp).
template <int DT, bool GUM, bool IPT, bool ADM, bool RANK, bool NANS>
__global__ __launch_bounds__(kBlock) void score_part_kernel(RowBatch b, const int32_t *__restrict__ claimed_ipt, bool ipt_rank,
                                                            float delta, SplitWorkspace ws, int first_last)
{
    typedef typename Elem<DT>::type elt_t;
    constexpr int E = Elem<DT>::kPerVec;
    __shared__ float lds_y[kWaves];
    __shared__ int32_t lds_i[kWaves];
    __shared__ float lds_L[kWaves];
    __shared__ int32_t lds_rank[kWaves];
    __shared__ float lds_f[kWaves];
    __shared__ double lds_d[kWaves];
    __shared__ float adm_lists[ADM ? kWaves * kAdmCap : 1];
    __shared__ int32_t adm_fills[kWaves];
    __shared__ int32_t adm_out;

    const int64_t row = blockIdx.x / ws.parts;
    const int part = blockIdx.x % ws.parts;
    const RowInfo ri = load_row_info(b, row);
    if (!ri.seq_ok || !ri.temp_ok) return;  // (the merge writes such a row's outputs)
    RowInfo ri_ipt = ri;
    ri_ipt.claimed = claimed_ipt ? claimed_ipt[row] : -1;
    const int tid = threadIdx.x;
    const elt_t *x_row = reinterpret_cast<const elt_t *>(b.logits) + row * b.ld;
    const int64_t V = b.V;
    const int full_rounds = (int)((V / E) / kBlock);
    const int r0 = part_begin(part, ws.parts, full_rounds), r1 = part_begin(part + 1, ws.parts, full_rounds);
    const bool last = part == ws.parts - 1;
    IptMarks<kNoToken> marks(nullptr, nullptr, 0);
    // The parts that end the launch should end together (RowPace): all of them where they fit at once, and the last that do where they
    // do not (both scores in bf16: five to a compute unit, four with the rank).  bf16, both scores, us with one priority / so / with every
    // part taken for one of the last: 128 x 128,256 27.0 / 24.2 / 24.3, 400 49.2 / 42.7 / 42.5, with the rank 58.6 / 57.8 / 60.5;
    // 641 x 151,936 80.1 / 69.4 / 81.0, 740 83.0 / 74.5 / 83.0, with the admissible set 109.3 / 101.9 / 109.1.
    typename std::conditional<GUM && (IPT || DT == 0), RowPace, NoPace>::type pace(first_last, r1 - r0, r0);
    // (single variables: as one struct the compiler moves it through memory)
    float out_M = 0.0f, best_y = 0.0f;
    double out_Z = 0.0, out_P = 0.0;
    int32_t best_v = 0, above = 0, any_bad = 0, adm_n = 0;

    typedef GumbelStream<DT, RANK, false, false, ADM, false, NANS> G;
    if constexpr (GUM) {
        G g(ri, x_row, V, lds_L);
        __syncthreads();
        if (ADM) {
            if (tid == 0) adm_out = 0;
            g.arm_admissible(delta, adm_lists, adm_fills);
            __syncthreads();
        }
        auto gumbel_done = [&]() {
            const typename G::Reduced r = g.reduce(lds_y, lds_i, lds_rank);
            best_y = g.best_y;
            best_v = g.best_v;
            any_bad = r.any_bad;
            above = r.above;
            if constexpr (ADM) {
                // the listed scores that may lie within delta of the row's maximum, which is no less than the part's (margins
                // are rounded differences, so the order of two maxima is the order of their margins)
                float *list = ws.adm + ((int64_t)row * ws.parts + part) * kSplitAdmCap;
                const int lane = tid & 63;
                const int32_t c = min(__builtin_amdgcn_readfirstlane(*g.adm_fill), kAdmCap);
                bool over = g.adm_over != 0;
                for (int32_t base = 0; base < c; base += 64) {
                    const bool have = base + lane < c;
                    const float y = have ? g.adm_list[base + lane] : 0.0f;
                    if (have && !(g.best_y - y > delta)) {
                        const int32_t i = atomicAdd(&adm_out, 1);
                        if (i < kSplitAdmCap)
                            list[i] = y;
                        else
                            over = true;
                    }
                }
                adm_n = __syncthreads_or((int)over) ? -1 : adm_out;
            }
        };
        if constexpr (IPT) {
            IptStream<DT> s(ri_ipt, x_row, V, false);
            stream_rounds<DT, kNoToken>(g, s, marks, pace, x_row, V, r0, r1, last);
            pace.done();
            if (DT == 0 && !ADM && !rows_aligned(b)) g.bad_sum(s.Z);
            gumbel_done();
            const IptTotals t = ipt_combine(s.ref(), s.Z, s.P, s.refP(), lds_f, lds_d);
            out_M = t.M;
            out_Z = t.Z;
            out_P = t.P;
        } else {
            NoIpt s;
            stream_rounds<DT, kNoToken>(g, s, marks, pace, x_row, V, r0, r1, last);
            pace.done();
            gumbel_done();
        }
    } else {
        NoGumbel g;
        IptStream<DT> s(ri_ipt, x_row, V, ipt_rank);
        stream_rounds<DT, kNoToken>(g, s, marks, pace, x_row, V, r0, r1, last);
        above = s.total_above(lds_rank);
        const IptTotals t = ipt_combine(s.ref(), s.Z, s.P, s.refP(), lds_f, lds_d);
        out_M = t.M;
        out_Z = t.Z;
        out_P = t.P;
    }
    if (tid == 0) ws.part[row * ws.parts + part] = Partial{out_Z, out_P, out_M, best_y, best_v, above, any_bad, adm_n};
}

// One workgroup per row; every wave merges the row's partial results, one per lane, by itself.
template <int DT, bool GUM, bool IPT, bool ADM, bool TOK>
__global__ __launch_bounds__(kBlock) void score_merge_kernel(RowBatch b, const int32_t *__restrict__ claimed_ipt, GumbelOutputs og,
                                                             IptOutputs oi, AdmissibleOutputs oa, SplitWorkspace ws)
{
    typedef typename Elem<DT>::type elt_t;
    constexpr int E = Elem<DT>::kPerVec;
    __shared__ WalkScratch walk;
    __shared__ float lds_L[kWaves];
    __shared__ int32_t lds_c[kWaves];

    const int64_t row = blockIdx.x;
    const RowInfo ri = load_row_info(b, row);
    RowInfo ri_ipt = ri;
    ri_ipt.claimed = claimed_ipt ? claimed_ipt[row] : -1;
    const int tid = threadIdx.x, lane = tid & 63;
    const float nan = __builtin_nanf(""), ninf = -__builtin_inff();
    if (!ri.seq_ok || !ri.temp_ok) {  // uniform
        if (GUM) gumbel_row_rejected(ri, row, og);
        if (IPT) ipt_row_rejected(ri_ipt, row, oi);
        if (ADM && tid == 0) {
            oa.count[row] = 0;
            if (oa.log2_count) oa.log2_count[row] = nan;
        }
        return;
    }
    const elt_t *x_row = reinterpret_cast<const elt_t *>(b.logits) + row * b.ld;
    const int64_t V = b.V;
    const bool have = lane < ws.parts;
    Partial p = {};
    p.M = p.best_y = ninf;
    p.best_v = 0x7FFFFFFF;
    if (have) p = ws.part[row * ws.parts + lane];

    int32_t above = p.above;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) above += __shfl_xor(above, off, 64);
    if constexpr (GUM) {
        float best_y = p.best_y;
        int32_t best_v = p.best_v;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float oy = __shfl_xor(best_y, off, 64);
            const int32_t ov = __shfl_xor(best_v, off, 64);
            argmax_combine(best_y, best_v, oy, ov);
        }
        const bool any_bad = __builtin_amdgcn_ballot_w64(p.bad != 0) != 0ull;
        if (tid == 0) {
            const int32_t t = ri.claimed;
            const bool valid = t >= 0 && (int64_t)t < V;
            float yt = nan;
            if (valid) {
                uint32_t r[4];
                noise_block(ri.key, ri.pos, ri.seq, kStreamGumbel, (uint32_t)t >> 2, r);
                const uint32_t rt = (t & 3) == 0 ? r[0] : (t & 3) == 1 ? r[1] : (t & 3) == 2 ? r[2] : r[3];
                yt = perturbed_score(Elem<DT>::to_float(x_row[t]), 1.0f / ri.T, rt);
            }
            gumbel_write(row, og, t, valid, yt, best_y, best_v, any_bad, og.logit_rank != nullptr, above);
        }
        if constexpr (ADM) {
            const float M = best_y;
            int32_t c = 0;
            if (M == M && fabsf(M) < __builtin_inff()) {  // uniform; as difr_admissible_count: else no finite maximum
                if (__builtin_amdgcn_ballot_w64(have && p.adm_n < 0) == 0ull) {
                    int32_t n = 0;
                    for (int k = tid >> 6; k < ws.parts; k += kWaves) {  // a wave takes every fourth part's list
                        const float *list = ws.adm + (row * ws.parts + k) * kSplitAdmCap;
                        const int32_t m = __shfl(p.adm_n, k, 64);
                        for (int32_t i = lane; i < m; i += 64) n += (int32_t)(M - list[i] <= oa.delta);
                    }
                    c = block_sum_i32(n, lds_c);
                } else {
                    RowInfo none = ri;
                    none.claimed = -1;
                    c = admissible_count_row<DT>(none, x_row, V, M, oa.delta, lds_L, lds_c);
                }
            }
            if (tid == 0) {
                oa.count[row] = c;
                if (oa.log2_count) oa.log2_count[row] = c > 0 ? __log2f((float)c) : nan;
            }
        }
    }
    if constexpr (IPT) {
        const float M = wave_max(p.M);
        const double scale = p.M > ninf ? (double)fast_exp2(p.M - M) : 0.0;
        const double z = have ? p.Z * scale : 0.0;
        double Z = z, P = have ? p.P * scale : 0.0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            Z += __shfl_xor(Z, off, 64);
            P += __shfl_xor(P, off, 64);
        }
        const float c = kLog2e / ri.T;
        ipt_write<DT, TOK>(b, ri_ipt, row, x_row, c, M, Z, P, above, oi, [&](double target) {
            double incl = z;  // CDF numerators at the ends of the parts
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const double o = __shfl_up(incl, off, 64);
                if (lane >= off) incl += o;
            }
            const uint64_t hit = __builtin_amdgcn_ballot_w64(have && incl > target);
            const int f = hit != 0ull ? __builtin_ctzll(hit) : ws.parts - 1;
            const double before = __shfl(incl - z, f, 64);
            const int full_rounds = (int)((V / E) / kBlock);
            return ipt_walk<DT>(x_row, V, c, -M, part_begin(f, ws.parts, full_rounds), part_begin(f + 1, ws.parts, full_rounds), before,
                                target, walk);
        });
    }
}

// Rows are shared while they do not fill the chip: about 1024 workgroups, four to a compute unit, are made of them, each with
// at least two rounds of 2048 entries, so that its set-up does not outweigh its share.  The lines, on graph replays of both
// scores (one workgroup per row against shared rows, us):
//   rows  N <= 10 rounds, and 768: V = 151,936 (74 rounds) N = 512: 61.6 / 57.1, 740: 80.7 / 77.6, and with the line lifted 1024:
//         93.9 / 91.6, 1536: 124.6 / 128.1; V = 65,000 (31 rounds) N = 310: 32.7 / 28.1; V = 50,000 (24 rounds) N = 240: 26.2 / 22.6;
//         with the line on V lifted, V = 32,000 (15 rounds) N = 128: 17.9 / 16.1, 256: 18.4 / 19.0;
//   V     24 rounds and more: V = 65,000, N = 24: 24.1 / 13.4; with the line lifted V = 32,000: 16.9 / 13.2, which the second launch
//         and the workspace cost the host again; V = 8192: 10.1 / 11.7.
constexpr int64_t kSplitRows = 768, kSplitRowsPerRound = 10, kSplitLeast = 24, kSplitGroups = 1024, kSplitRounds = 2;

int split_parts(int64_t N, int64_t V, int dtype)
{
    if (N < 1 || V < 1 || (dtype != 0 && dtype != 1)) return 1;
    const int64_t rounds = V / (8 * kBlock);  // of 2048 entries, for either type
    if (rounds < kSplitLeast || N > kSplitRows || N > kSplitRowsPerRound * rounds) return 1;
    int64_t p = (kSplitGroups + N - 1) / N;
    if (p > rounds / kSplitRounds) p = rounds / kSplitRounds;
    if (p > kMaxParts) p = kMaxParts;
    return p < 1 ? 1 : (int)p;
}

size_t split_workspace_bytes(int64_t N, int parts, bool admissible)
{
    return (size_t)N * (size_t)parts * (sizeof(Partial) + (admissible ? kSplitAdmCap * sizeof(float) : 0));
}

template <int DT, bool GUM, bool IPT, bool ADM, bool RANK, bool NANS>
static int launch_of(const RowBatch &b, const int32_t *claimed_ipt, const GumbelOutputs &og, const IptOutputs &oi,
                     const AdmissibleOutputs &oa, const SplitWorkspace &ws, hipStream_t stream)
{
    score_part_kernel<DT, GUM, IPT, ADM, RANK, NANS><<<dim3((unsigned)(b.N * ws.parts)), dim3(kBlock), 0, stream>>>(
        b, claimed_ipt, oi.logit_rank != nullptr, oa.delta, ws,
        pace_from(b.N * ws.parts, resident_rows<score_part_kernel<DT, GUM, IPT, ADM, RANK, NANS>>(), b.V / ws.parts));
    if (hipGetLastError() != hipSuccess) return 1;
    if (IPT && !ADM && oi.ipt_token)
        score_merge_kernel<DT, GUM, IPT, false, IPT && !ADM><<<dim3((unsigned)b.N), dim3(kBlock), 0, stream>>>(b, claimed_ipt, og, oi, oa, ws);
    else
        score_merge_kernel<DT, GUM, IPT, ADM, false><<<dim3((unsigned)b.N), dim3(kBlock), 0, stream>>>(b, claimed_ipt, og, oi, oa, ws);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

template <int DT>
static int launch_for(const RowBatch &b, const int32_t *claimed_ipt, const GumbelOutputs &og, const IptOutputs &oi,
                      const AdmissibleOutputs &oa, const SplitWorkspace &ws, hipStream_t stream)
{
    auto launch = [&](auto GUM, auto IPT, auto ADM, auto RANK, auto NANS) {
        return launch_of<DT, decltype(GUM)::value, decltype(IPT)::value, decltype(ADM)::value, decltype(RANK)::value, decltype(NANS)::value>(
            b, claimed_ipt, og, oi, oa, ws, stream);
    };
    const std::true_type yes;
    const std::false_type no;
    const bool rank = og.logit_rank != nullptr;
    if (oa.count) return launch(yes, yes, yes, no, no);
    if (og.margin && oi.dist) return rank ? launch(yes, yes, no, yes, no) : launch(yes, yes, no, no, no);
    if constexpr (DT == 0) {
        if (og.margin && !rows_aligned(b)) return rank ? launch(yes, no, no, yes, yes) : launch(yes, no, no, no, yes);
    }
    if (og.margin) return rank ? launch(yes, no, no, yes, no) : launch(yes, no, no, no, no);
    return launch(no, yes, no, no, no);
}

int launch_score_split(const RowBatch &b, const int32_t *claimed_ipt, const GumbelOutputs &og, const IptOutputs &oi,
                       const AdmissibleOutputs &oa, void *workspace, int parts, hipStream_t stream)
{
    SplitWorkspace ws;
    ws.part = (Partial *)workspace;
    ws.adm = oa.count ? (float *)(ws.part + b.N * parts) : nullptr;
    ws.parts = parts;
    return b.dtype == 0 ? launch_for<0>(b, claimed_ipt, og, oi, oa, ws, stream) : launch_for<1>(b, claimed_ipt, og, oi, oa, ws, stream);
}

}  // namespace difr
