// Row-streaming state of the Token-IPT-DiFR kernel (Sec. 3.2 softmax and IPT sampler; Sec. 6.2 and
// the appendix algorithm "convolved Gaussian score"), kept as a struct so that the IPT-only kernel
// and the kernel that scores both estimators in one pass share it.
#pragma once

#include "difr_device.hpp"

namespace difr {

// Inclusive scan (fp64) over the 256 threads in thread order; returns the inclusive value and
// the block total.  Fixed shape.
__device__ __forceinline__ double block_inclusive_scan(double v, double *lds /* kWaves */, double &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(v, off, 64);
        if (lane >= off) v += o;
    }
    __syncthreads();
    if (lane == 63) lds[wave] = v;
    __syncthreads();
    double before = 0.0, tot = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const double s = lds[w];
        if (w < wave) before += s;
        tot += s;
    }
    total = tot;
    return v + before;
}

__device__ __forceinline__ double block_sum_f64(double v, double *lds /* kWaves */)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = lds[0];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) s += lds[i];
    return s;
}

// max(a, b, c) as the bare three-input instruction (a NaN operand is ignored; NaNs are caught
// later through the sum of exponentials, not here).
__device__ __forceinline__ float max3_raw(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Sum of the E exponentials of one vector as a fixed binary tree in fp32.
template <int E>
__device__ __forceinline__ float tree_sum(const float e[E])
{
    float t[E];
#pragma unroll
    for (int j = 0; j < E; ++j) t[j] = e[j];
#pragma unroll
    for (int w = E / 2; w >= 1; w >>= 1) {
#pragma unroll
        for (int j = 0; j < w; ++j) t[j] += t[j + w];
    }
    return t[0];
}

// Gaussian log-mass of [a,b] under N(u, sigma^2), fp64:
//   ln( Phi((b-u)/sigma) - Phi((a-u)/sigma) + eps ),
// with the difference taken on the non-cancelling side (erfc in the tails).
__device__ double gaussian_log_mass(double a, double b, double u, double sigma, double eps)
{
    const double s = 1.0 / (sigma * 1.4142135623730951);
    const double za = (a - u) * s, zb = (b - u) * s;
    double mass;
    if (za >= 0.0)
        mass = 0.5 * (erfc(za) - erfc(zb));
    else if (zb <= 0.0)
        mass = 0.5 * (erfc(-zb) - erfc(-za));
    else
        mass = 0.5 * (erf(zb) + erf(-za));
    if (mass < 0.0) mass = 0.0;
    return log(mass + eps);
}

// Search for the honest sampler's token, min { v : C_v > u }, after the streaming pass.
//
// Marks.  While the row is streamed every thread leaves its running sum Z, with the exponent it is taken against, in LDS
// after each 1/kMarks of the full rounds (its own slots: no barrier).  Once the total is known, the sums at the marks say in
// which stretch the CDF passes u Z, and only that stretch is read again.  What bounds the search is that second read and the
// latency of its dependent steps: walking the CDF from the row's start, one round and two barriers at a time, made a call on
// 2048 rows of 151,936 bf16 logits without claims take 227 us; with the marks, up to 16 rounds (four loads in flight) between
// two barriers and nothing read past the stretch it takes 113 (2048 x 50,000: 47.5 us, 59 with 16 rounds read whatever the stretch).
// Seven marks: 22.4 KB of LDS; six marks 116 us; eight 113, but 2048 x 50,000 49.6.  (The kernels' scalar registers hold them at six workgroups
// to a compute unit with any of these.)
constexpr int kMarks = 7;
constexpr int kWalkRounds = 16;  // rounds summed between two barriers of the walk: 16 x 4 wave sums, one per lane
static_assert(kWalkRounds * kWaves == 64, "the walk scans one wave sum per lane");
// Full rounds from which a row has marks; a shorter one is walked from its start (ipt_walk_short), which needs fewer steps
// than bringing the marks to the total.  Calls without claims, walk against marks, us: 2 rounds (16,384 x 4096 bf16) 74 / 113;
// 15 rounds (4096 x 32,000 bf16) 85 / 88; 24 rounds (4096 x 25,000 fp32) 121 / 112; 31 rounds (4096 x 32,000 fp32) 151 / 127.
// The kernels are instantiated for either, so that short rows carry neither the marks' LDS nor their code (16,384 x 4096 fp32,
// both scores with the token, honest claims: 131 us with one kernel for both, 128 apart).
constexpr int kMarkLeast = 16;
enum TokenSearch { kNoToken = 0, kTokenWalk = 1, kTokenMarks = 2 };

inline TokenSearch token_search(const int32_t *ipt_token, int64_t V, int dtype)
{
    if (ipt_token == nullptr) return kNoToken;
    return V / ((dtype == 0 ? 8 : 4) * kBlock) < kMarkLeast ? kTokenWalk : kTokenMarks;
}

template <int TOK>
struct IptMarks {
    double (*Z)[kBlock];   // [kMarks][kBlock]
    float (*ref)[kBlock];  // [kMarks][kBlock]
    int len, next, n;      // rounds between marks, round of the next one, marks left so far (uniform over the workgroup)

    __device__ __forceinline__ IptMarks(double (*Z_)[kBlock], float (*ref_)[kBlock], int full_rounds)
        : Z(Z_), ref(ref_), len((full_rounds + kMarks - 1) / kMarks), next(len), n(0)
    {
    }
    // `round` rounds of the row have been summed
    template <class Stream>
    __device__ __forceinline__ void at(int round, const Stream &s)
    {
        if constexpr (TOK == kTokenMarks) {
            if (round == next) {  // (n < kMarks: kMarks * len >= full_rounds, and no full round follows the last mark)
                Z[n][threadIdx.x] = s.Z;
                ref[n][threadIdx.x] = s.ref();
                ++n;
                next = n < kMarks ? next + len : 0x7FFFFFFF;
            }
        }
    }
};

// LDS of the search (of one workgroup).
struct WalkScratch {
    double mark_sum[kMarks][kWaves];
    double round_sum[kWalkRounds * kWaves];
    int32_t tok;
};

// All 256 threads: the token at which the CDF of the entries of rounds r0, r0 + 1, ... passes `target`; `before` is the mass of
// the rounds below r0, terms are 2^(x c + neg_Mc); by the sums at hand it is passed before round r_mark, and what follows is read only
// if rounding has it otherwise.  -1 if it is not passed before the end of the row.  The wave sums of up to
// kWalkRounds rounds are formed between two barriers, one scan over them finds the 512 entries that hold the token, and their
// wave finds it.
template <int DT>
__device__ __forceinline__ int32_t ipt_walk(const typename Elem<DT>::type *x_row, int64_t V, float c, float neg_Mc, int r0, int r_mark,
                                            double before, double target, WalkScratch &w)
{
    constexpr int E = Elem<DT>::kPerVec;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_rounds = (int)(((V + E - 1) / E + kBlock - 1) / kBlock);
    if (tid == 0) w.tok = -1;
    const int full_rounds = (int)((V / E) / kBlock);
    const uint32_t ninf = DT == 0 ? 0xFF80FF80u : 0xFF800000u;
    const u32x4 masked = u32x4{ninf, ninf, ninf, ninf};  // no mass
    auto terms = [&](u32x4 q, float (&e)[E]) {
        float x[E];
        unpack_vector<DT>(q, x);
#pragma unroll
        for (int j = 0; j < E; ++j) e[j] = fast_exp2(__fmaf_rn(x[j], c, neg_Mc));
        return (double)tree_sum<E>(e);
    };
    for (int nr; r0 < n_rounds; r0 += nr) {
        nr = min(kWalkRounds, (r0 < r_mark ? r_mark : n_rounds) - r0);
        __syncthreads();  // (the scan of the batch before has been read; w.tok is set)
        for (int k0 = 0; k0 < nr; k0 += 4) {
            u32x4 q[4];
            if (k0 + 4 <= nr && r0 + k0 + 4 <= full_rounds) {  // uniform: four loads in flight
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = load_round(x_row, r0 + k0 + i);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t base = ((int64_t)(r0 + k0 + i) * kBlock + tid) * E;
                    q[i] = k0 + i < nr && base < V ? load_vector<DT>(x_row, base, V) : masked;
                }
            }
            double ls[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float e[E];
                ls[i] = terms(q[i], e);
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
                for (int i = 0; i < 4; ++i) ls[i] += __shfl_xor(ls[i], off, 64);
            if (lane < 4) w.round_sum[(k0 + lane) * kWaves + wave] = lane == 0 ? ls[0] : (lane == 1 ? ls[1] : (lane == 2 ? ls[2] : ls[3]));
        }
        __syncthreads();
        const double mine = lane < nr * kWaves ? w.round_sum[lane] : 0.0;
        double incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        // (lanes without a wave sum, or with an empty one, hold the total in another order of addition: rounding must not
        // let one of them pass alone.  The same in every wave.)
        const uint64_t hit = __builtin_amdgcn_ballot_w64(mine > 0.0 && before + incl > target);
        if (hit != 0ull) {
            const int f = __builtin_ctzll(hit);
            if (wave == f % kWaves) {
                const double start = before + __shfl(incl - mine, f, 64);  // mass below the wave's 64 vectors
                const int64_t base = ((int64_t)(r0 + f / kWaves) * kBlock + tid) * E;
                float e[E];
                const double ls = terms(base < V ? load_vector<DT>(x_row, base, V) : masked, e);
                double in = ls;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const double o = __shfl_up(in, off, 64);
                    if (lane >= off) in += o;
                }
                const uint64_t over = __builtin_amdgcn_ballot_w64(ls > 0.0 && start + in > target);
                const uint64_t mass = __builtin_amdgcn_ballot_w64(ls > 0.0);  // (not empty: the wave's sum was not)
                // (the two sums of the same terms may round apart: then the last vector with any mass, and its last entry)
                const int l = over != 0ull ? __builtin_ctzll(over) : 63 - __builtin_clzll(mass);
                if (lane == l) {
                    double cacc = start + (in - ls);
                    int32_t found = -1, last = 0;
#pragma unroll
                    for (int j = 0; j < E; ++j) {
                        cacc += (double)e[j];
                        if (e[j] > 0.0f) {  // (a masked entry, or one past the end of the row, owns no interval)
                            last = j;
                            if (found < 0 && cacc > target) found = j;
                        }
                    }
                    w.tok = (int32_t)base + (found < 0 ? last : found);
                }
            }
            __syncthreads();
            return w.tok;
        }
        before += __shfl(incl, 63, 64);
    }
    return -1;
}

// The same for a row of few rounds, from its start: one scan over the workgroup's 256 vectors per round.
template <int DT>
__device__ __forceinline__ int32_t ipt_walk_short(const typename Elem<DT>::type *x_row, int64_t V, float c, float neg_Mc,
                                                  double target, WalkScratch &w)
{
    constexpr int E = Elem<DT>::kPerVec;
    const int tid = threadIdx.x;
    double before = 0.0;
    if (tid == 0) w.tok = -1;
    for (int64_t v0 = 0; v0 < V; v0 += kBlock * E) {
        const int64_t base = v0 + tid * E;
        float e[E];
#pragma unroll
        for (int j = 0; j < E; ++j) e[j] = 0.0f;
        if (base < V) {
            float x[E];
            unpack_vector<DT>(load_vector<DT>(x_row, base, V), x);
#pragma unroll
            for (int j = 0; j < E; ++j) e[j] = fast_exp2(__fmaf_rn(x[j], c, neg_Mc));
        }
        const double ls = (double)tree_sum<E>(e);
        double total;
        const double incl = block_inclusive_scan(ls, w.round_sum, total);
        if (before + total > target) {  // uniform: the token is inside this round
            const double excl = before + (incl - ls);
            if (ls > 0.0 && excl <= target && before + incl > target) {  // one thread
                double cacc = excl;
                int32_t found = -1, last = 0;
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    cacc += (double)e[j];
                    if (e[j] > 0.0f) {
                        last = j;
                        if (found < 0 && cacc > target) found = j;
                    }
                }
                w.tok = (int32_t)base + (found < 0 ? last : found);
            }
            break;
        }
        before += total;
    }
    __syncthreads();
    return w.tok;
}

// Everything after the streaming pass: combine the partial (reference, sum) pairs, regenerate u,
// form the interval and the distance, optionally search the honest sampler's token, write outputs.
struct IptOutputs {
    float *dist, *cdf_lo, *cdf_hi, *u;
    int32_t *ipt_token;
    double sigma, eps;
    float *log_mass;
    uint8_t *flags;
    int32_t *logit_rank;
};

// Outputs of a row from its total mass Z and the mass P below the claim, both relative to the exponent M.  All 256 threads;
// search(u Z): the token at which the CDF passes u, called (by all of them) only if it is asked for and the claim is not it.
template <int DT, bool TOK, class Search>
__device__ __forceinline__ void ipt_write(const RowBatch &b, const RowInfo &ri, int64_t row, const typename Elem<DT>::type *x_row,
                                          float c, float M, double Ztot, double Ptot, int32_t above, const IptOutputs &o,
                                          Search &&search)
{
    const float nan = __builtin_nanf("");
    const float ninf = -__builtin_inff();
    const int64_t V = b.V;
    const int64_t t = ri.claimed;
    const bool valid = (t >= 0 && t < V);

    // Regenerated uniform: stream 1, vocabulary index 0.
    uint32_t r[4];
    noise_block(ri.key, ri.pos, ri.seq, kStreamIpt, 0u, r);
    const float u = uniform_from_bits(r[0]);

    // Z is NaN if a NaN logit was seen, +inf if a +inf logit was (then M = +inf); M = -inf if every
    // entry is masked.  All of these make the distribution undefined.
    const bool bad = !(Ztot > 0.0) || !(Ztot < (double)__builtin_inff()) || !(M < __builtin_inff()) || !(M > ninf);

    float a = nan, bb = nan, d = nan;
    double ad = 0.0, bd = 0.0;
    bool match = false;
    if (valid && !bad) {
        const double et = (double)fast_exp2(__fmaf_rn(Elem<DT>::to_float(x_row[t]), c, -M));
        const double ud = (double)u;
        ad = Ptot / Ztot;
        bd = (Ptot + et) / Ztot;
        a = (float)ad;
        bb = (float)bd;
        d = (float)fmax(fmax(ad - ud, ud - bd), 0.0);
        match = (ad <= ud) && (ud < bd);
    }

    uint32_t f = 0;
    if (!valid) f |= kFlagInvalidClaim;
    if (bad) f |= kFlagNonfinite;
    if (match) f |= kFlagMatch;

    int32_t tok = match ? (int32_t)t : -1;
    if (TOK && !match && !bad) {  // uniform
        f |= kFlagSlowPath;
        tok = search((double)u * Ztot);
        if (tok < 0) tok = (int32_t)(V - 1);  // u * Z at or beyond the accumulated total
    }

    if (threadIdx.x == 0) {
        o.dist[row] = d;
        if (o.cdf_lo) o.cdf_lo[row] = a;
        if (o.cdf_hi) o.cdf_hi[row] = bb;
        if (o.u) o.u[row] = u;
        if (TOK) o.ipt_token[row] = bad ? -1 : tok;
        if (o.log_mass)
            o.log_mass[row] =
                (valid && !bad) ? (float)gaussian_log_mass(ad, bd, (double)u, o.sigma, o.eps) : nan;
        if (o.logit_rank) o.logit_rank[row] = valid ? above : -1;
        o.flags[row] = (uint8_t)f;
    }
}

// The sums of the 256 threads on a common reference.
struct IptTotals {
    float M;
    double Z, P;
};

__device__ __forceinline__ IptTotals ipt_combine(float ref, double Z, double P, float refP, float *lds_f, double *lds_d)
{
    // Combine the 256 partial (reference, sum) pairs in a fixed order.  `ref` is the exponent a thread's terms were
    // taken against, a whole number: they are 2^(x c - ref).  The common reference is the largest of them, and a thread's
    // scale is the exact 2^(ref - M): forming it from the reference logits instead, as 2^((m - M) c), would be off by the
    // rounding of m c - half a unit in its last place, 1e-5 when |m| / T runs into the hundreds, a different amount in
    // every thread.
    const float ninf = -__builtin_inff();
    IptTotals t;
    t.M = block_max(ref, lds_f);  // (-inf: every entry masked; +inf or NaN: a +inf or NaN logit)
    // a thread that saw only masked entries has ref = -inf and Z = 0 (NaN: it saw a NaN), so does a part of a row
    const double Zs = Z * (ref > ninf ? (double)fast_exp2(ref - t.M) : 0.0);
    const double Ps = (refP > ninf) ? P * (double)fast_exp2(refP - t.M) : 0.0;
    t.Z = block_sum_f64(Zs, lds_d);
    t.P = block_sum_f64(Ps, lds_d);
    return t;
}

template <int DT, int TOK>
__device__ __forceinline__ void ipt_finish(const RowBatch &b, const RowInfo &ri, int64_t row,
                                           const typename Elem<DT>::type *x_row, float c, float ref, double Z,
                                           double P, float refP, int32_t above, const IptOutputs &o, float *lds_f,
                                           double *lds_d, const IptMarks<TOK> &marks, WalkScratch *walk)
{
    const IptTotals t = ipt_combine(ref, Z, P, refP, lds_f, lds_d);
    ipt_write<DT, TOK != kNoToken>(b, ri, row, x_row, c, t.M, t.Z, t.P, above, o, [&](double target) {
        if constexpr (TOK == kTokenWalk) return ipt_walk_short<DT>(x_row, b.V, c, -t.M, target, *walk);
        const int tid = threadIdx.x;
        for (int k = 0; k < marks.n; ++k) {
            double v = marks.Z[k][tid] * (double)fast_exp2(marks.ref[k][tid] - t.M);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            if ((tid & 63) == 0) walk->mark_sum[k][tid >> 6] = v;
        }
        __syncthreads();
        // the last mark at which the CDF has not passed u yet
        double before = 0.0;
        int r0 = 0, r_mark = 0;
        for (int k = 0; k < marks.n; ++k) {
            const double v = walk->mark_sum[k][0] + walk->mark_sum[k][1] + walk->mark_sum[k][2] + walk->mark_sum[k][3];
            if (v > target) {
                r_mark = (k + 1) * marks.len;
                break;
            }
            before = v;
            r0 = (k + 1) * marks.len;
        }
        return ipt_walk<DT>(x_row, b.V, c, -t.M, r0, r_mark, before, target, *walk);
    });
}

__device__ __forceinline__ bool ipt_row_rejected(const RowInfo &ri, int64_t row, const IptOutputs &o)
{
    if (ri.seq_ok && ri.temp_ok) return false;
    if (threadIdx.x == 0) {
        const float nan = __builtin_nanf("");
        o.dist[row] = nan;
        if (o.cdf_lo) o.cdf_lo[row] = nan;
        if (o.cdf_hi) o.cdf_hi[row] = nan;
        if (o.u) o.u[row] = nan;
        if (o.ipt_token) o.ipt_token[row] = -1;
        if (o.log_mass) o.log_mass[row] = nan;
        if (o.logit_rank) o.logit_rank[row] = -1;
        o.flags[row] = (uint8_t)(ri.seq_ok ? kFlagNonfinite : kFlagInvalidClaim);
    }
    return true;
}

// Online softmax statistics per thread: m = the lane's reference logit (see terms()), Z = sum of 2^((x - m) c).  Each
// vector's terms are summed as an fp32 tree and the vector sums are accumulated in fp64, so the CDF
// values are good to fp32 rounding.  (P, with its own reference) is the same sum restricted to v < t.  Vector rounds
// that lie wholly below the claimed token, wholly above it, and are full need no per-entry test:
// the prefix is simply a snapshot of Z taken between the two groups of rounds.  Only the round
// that holds the claimed token and the last, partly filled round look at indices.
constexpr float kRefLift = 16.0f;         // see IptStream::terms()
constexpr float kRefLeast = -0x1p31f;     // above it m8 * c is rounded by at most 64, and 2^64 does no harm

template <int DT>
struct IptStream {
    typedef typename Elem<DT>::type elt_t;
    static constexpr int E = Elem<DT>::kPerVec;

    const elt_t *x_row;
    int64_t V, t;
    bool valid, want_rank;
    float c;   // exponent scale: exp(x/T) = 2^(x c)
    float xt;  // claimed token's raw logit (for the logit rank)
    int tid;
    // running state
    float m, neg_mc, neg_mcP;
    double Z, P;
    uint32_t above;       // wave-uniform ballot counts (full rounds)
    uint32_t lane_above;  // per-lane counts (careful rounds)

    __device__ __forceinline__ IptStream(const RowInfo &ri, const elt_t *x_row_, int64_t V_, bool want_rank_)
        : x_row(x_row_), V(V_), t(ri.claimed), want_rank(want_rank_), c(kLog2e / ri.T), tid((int)threadIdx.x)
    {
        valid = (t >= 0 && t < V);
        xt = valid ? Elem<DT>::to_float(x_row[t]) : __builtin_nanf("");
        m = -__builtin_inff();
        neg_mc = __builtin_inff();  // no reference yet: see terms()
        neg_mcP = __builtin_inff();
        Z = 0.0;
        P = 0.0;
        above = 0;
        lane_above = 0;
    }

    // Exponentials of one vector relative to the lane's reference point m.  The reference is the maximum of the
    // first vector the lane met and moves only when it has to: the sum of the eight terms is needed anyway,
    // and as long as it stays below 2^64 no term has overflowed (an entry more than 64 / c above m, or a lane
    // that has no reference yet -- neg_mc = +inf makes every term inf or NaN -- sends the sum over the limit).
    // Nothing is lost by a reference below the running maximum: fp32 terms keep their relative precision at any
    // scale, the sums are fp64, and every lane's sum is rescaled to the row's common reference at the end.
    // Returns the sum of the terms.
    __device__ __forceinline__ float terms(const float x[E], float e[E])
    {
#pragma unroll
        for (int j = 0; j < E; ++j) e[j] = fast_exp2(__fmaf_rn(x[j], c, neg_mc));
        float sum = tree_sum<E>(e);
        if (__builtin_amdgcn_ballot_w64(!(sum <= 0x1p64f)) != 0ull) {
            asm volatile("" ::: "memory");  // keep this a real, rarely taken branch
            if (!(sum <= 0x1p64f)) {
                float m8;
                if (E == 8)
                    m8 = max3_raw(max3_raw(x[0], x[1], x[2]), max3_raw(x[3], x[4], x[5]), max3_raw(x[6 % E], x[7 % E], x[7 % E]));
                else
                    m8 = max3_raw(max3_raw(x[0], x[1], x[2]), x[3], x[3]);
                if (m8 > m) {  // (m = -inf: Z is still 0 and stays 0)
                    // The reference exponent is put kRefLift above the vector's largest: an fp32 exponent is good to
                    // half a unit in its last place, 1e-6 at 16 and beyond, and the entries that lie far above a
                    // lane's first vector - the few tokens that carry the mass of a peaked row - are the ones whose
                    // terms have to be exact; the many small ones below average their roundings out.
                    // A whole number, so that bringing sums taken against different references to a common one multiplies
                    // them by exact powers of two (lanes, parts of a split row).
                    // And no lower than kRefLeast: a vector of masked entries (the type's lowest value, -1e10) would put it
                    // where m8 * c is infinite, or rounded by so much that 2^(x c - ref) overflows for m8 itself, and the
                    // row's sum would be NaN once an unmasked entry moves it.
                    const float moved = -fmaxf(ceilf(m8 * c) + kRefLift, kRefLeast);
                    Z *= (double)fast_exp2(moved - neg_mc);  // from the old rounded reference to the new one (see ipt_finish)
                    m = m8;
                    neg_mc = moved;
                }
                // a lane that has met only masked entries keeps m = -inf; its terms are 2^(-inf + 0) = 0
                const float shift = (m > -__builtin_inff()) ? neg_mc : 0.0f;
#pragma unroll
                for (int j = 0; j < E; ++j) e[j] = fast_exp2(__fmaf_rn(x[j], c, shift));
                sum = tree_sum<E>(e);
            }
        }
        return sum;
    }

    // a full round: every lane holds a complete vector, no index tests
    __device__ __forceinline__ void fast_round(u32x4 q)
    {
        float x[E], e[E];
        unpack_vector<DT>(q, x);
        if (want_rank) {  // logit rank: one compare per entry, counted with ballots
            uint32_t n = 0;
#pragma unroll
            for (int j = 0; j < E; ++j) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(x[j] > xt));
            above += n;
        }
        Z += (double)terms(x, e);
    }

    // everything seen so far lies below the claimed token
    __device__ __forceinline__ void snapshot()
    {
        P = Z;
        neg_mcP = neg_mc;
    }

    // the exponents the sums Z and P were taken against (-inf: no reference yet, the sum is 0), for ipt_finish
    __device__ __forceinline__ float ref() const { return -neg_mc; }
    __device__ __forceinline__ float refP() const { return -neg_mcP; }

    // a round that needs index tests: the one holding the claimed token and the last, ragged one.
    // `q` must have been loaded for every lane whose first entry v0 is below V.
    __device__ __forceinline__ void careful_round(u32x4 q, int round, bool prefix_open)
    {
        const int64_t v0 = ((int64_t)round * kBlock + tid) * E;
        if (v0 < V) {
            float x[E], e[E];
            unpack_vector<DT>(q, x);
#pragma unroll
            for (int j = 0; j < E; ++j)
                if (v0 + j >= V) x[j] = -__builtin_inff();
            if (want_rank) {  // divergent here: this lane's own count, the wave sums come at the end
                uint32_t n = 0;
#pragma unroll
                for (int j = 0; j < E; ++j) n += (uint32_t)(x[j] > xt);
                lane_above += n;
            }
            const float sum = terms(x, e);
            if (prefix_open) {
                float pre = 0.0f;
#pragma unroll
                for (int j = 0; j < E; ++j)
                    if (v0 + j < t) pre += e[j];
                P = Z + (double)pre;
                neg_mcP = neg_mc;
            }
            Z += (double)sum;
        } else if (prefix_open) {
            P = Z;
            neg_mcP = neg_mc;
        }
    }

    // does lane `tid` have a vector (possibly partial) in this round?
    __device__ __forceinline__ bool has_vector(int round) const
    {
        return ((int64_t)round * kBlock + tid) * E < V;
    }

    __device__ __forceinline__ int32_t total_above(int32_t *lds_rank)
    {
        if (!want_rank) return 0;
        const int32_t mine = (int32_t)lane_above + ((tid & 63) == 0 ? (int32_t)above : 0);
        return block_sum_i32(mine, lds_rank);
    }
};

}  // namespace difr
