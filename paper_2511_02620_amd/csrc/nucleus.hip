// The nucleus (top-p) filter over the WHOLE vocabulary, and Token-IPT-DiFR on the distribution it leaves
// (Sec. 3.2: the sampler's filter policy and the IPT sampler; Sec. 6.2; appendix "convolved Gaussian
// score").  K is the shortest prefix of the tokens ranked by logit (ties to the lower index) whose
// softmax(x / T) mass reaches top_p.  With no top-k in front of it K can hold tens of thousands of tokens,
// so it is not collected: the kernel finds the CUT, the last (logit, index) pair that still belongs to K,
// and membership of any token is one comparison against it.
//
// One workgroup per row.  bf16 rows are read ONCE.  A bf16 logit has few values - 2175 of either sign between 2^-10 and 128 -,
// entries of equal value have equal mass, so the pass only counts: one LDS counter per value, two sets of them, for the entries
// below the claimed token's index and for the others.  An entry is an address (five packed 16-bit instructions for two entries) and
// an integer LDS atomic; the pass takes no exponential but for entries around zero.  Afterwards a thread takes the masses of 17 values, in fp64, one scan over the
// 256 threads finds the value at which the cumulative mass from the top reaches top_p Z, and that value is treated as a
// bracket of a single value below: its ties enter K in index order.  Integer counts: any order gives the same bits.
//   - Entries of -128 and below, masked ones among them, go to 64 words one per lane (max() with the lane's own word, no branch), so
//     that rows that are mostly masked do not queue up at one counter.  They have no mass if the row's largest logit lies far
//     enough above; otherwise a second read tells whether they are all masked.  If they are not, or if anything of 128 and more
//     or a NaN has been seen, the row goes to the search below.  (2048 x 128,256, one entry in 20 masked, T = 1.6: 191 us, 357 by
//     passes.  Telling them apart in the pass, two packed instructions for two entries, took 16,384 x 151,936 from 856 to 899.)
//   - Entries within 2^-10 of zero share a counter; their masses are summed on the side (a quarter of the rounds of rows around
//     zero have one).  If they are all zero, that counter is a value's like the others; if not and the cut falls among them, the
//     row goes to the search.
//   - What it is bound by: LDS atomics at the same address queue up (a wave whose 64 entries are equal takes 64 turns).  32 runs of
//     eight vectors spread over the row say beforehand how many of the entries that a wave counts at once - the same place of
//     vectors one and four lanes apart - share a counter.  Up to 12 % of these pairs, plus 4500 / V (the search's fixed costs weigh
//     more in short rows) and never beyond 60 %, the row is counted, otherwise it is searched; rows of fewer than 256 vectors are
//     counted.  us counted / searched, at T = 0.7, top_p = 0.95 (the search depends on them), rows rounded to steps: 128,256 entries
//     with 8 % of the pairs 236 / 298, 10 % 272 / 307, 20 % 409 / 312, 39 % 619 / 356; 50,256: 14 % 106 / 171, 20 % 171 / 161, 37 % 250 / 205;
//     16,000: 29 % 136 / 191, 49 % 170 / 290; 8000: 56 % 118 / 218; 4000, constant rows: 95 / 65; 1000: 51 % 93 / 142.  One value in 30,
//     40 and 50 % of the places (10, 17 and 25 % of the pairs) of 128,256: 282 / 351, 365 / 351, 451 / 332.  (2048 to 8192 rows.)
// Reading: 16,384 x 151,936 852 us (5.8 TB/s; 2040 by passes); 2048 x 128,256, T = 0.7: 112 (268); 4096 x 1000: 52 (55); 128 x 151,936:
// 33 (125).  36 KB of LDS: four workgroups to a compute unit, with the next two rounds requested ahead.  Rows that go to the search have
// the registers and LDS of both.  us of the kernel of their own / here, 2048 x 128,256: constant rows 239 / 253, rounded to 1 274 / 311,
// period 16 338 / 386; 4096 x 8000, had they been searched: 91 / 120.  Rows that turn out not to be for the counters only when they
// have been counted pay for both: one entry of 130 that is not looked at 225 / 414, the cut among values around zero 797 / 967.
//
// The search: several passes over the row (it is read from HBM again each time), for fp32 rows and for those bf16 rows that the
// counting leaves.  Throughout, a token's KEY is the order-preserving integer image of its logit at the storage type's resolution (16 bits for
// bf16, formed on the packed patterns), and a bracket is a range of keys [klo, khi].
//   0    a look at 256 vectors (fp32: the first ones, bf16: the runs above): their largest entry R (the exponent reference
//        for every mass 2^((x - R) c): any finite reference serves) and their smallest finite one;
//   B1   every thread adds the mass of its entries to 16 private LDS bins (no atomics, no conflicts) that divide
//        the span of LOGIT VALUES seen in step 0 evenly, values outside falling into the end bins; the same pass
//        finds the smallest and largest key of the row (NaN / +inf check, the maximum M).  The bins are combined
//        in a fixed order in fp64, their total Z fixes the target top_p * Z, and the bin in which the cumulative
//        mass from the top reaches it becomes the bracket: bin1 is monotone in the logit, so its first key is
//        found by bisection.  (If M lies so far above R that terms could overflow, the pass is repeated with
//        R = M.)
//   BC   bf16 rows whose bracket is now at most 16 logit values (the usual case when K is large: near the cut a bf16
//        value is shared by thousands of tokens) are finished by one counting pass:
//        per value of the bracket and per thread the number of entries, and of entries below the claimed token's
//        index; entries of equal value have equal mass, which is taken per value in fp64.  Two reads in all.
//        Every other row goes on with B2 and C, with C at once if a sample of the row lets expect few entries in the
//        bracket (and with B2 after all if they turn out to be many):
//   B2.. the bracket's key range is divided evenly into at most 16 bins and searched in the same way, until it
//        is a single key - one logit value - or provably holds at most kNucCap entries (its mass divided by the
//        weight of its smallest key bounds their number).  Typically one or two passes;
//   C    the bracket is gathered as 64-bit composites (topn.hpp), sorted, and walked in rank order with an fp64
//        scan until the mass is reached: that entry is the cut.  A single-value bracket needs no sorting: the
//        ties enter K in index order with equal mass, so their number is a division.  The same pass sums what
//        lies above the bracket and below the claimed token's index.
// Why the first bins are laid over logit values and not over the leading key bits: the mass is spread over
// logit values, while key bits spend most of their range on exponents near zero - a search by key digits takes
// three passes in which nine entries in ten are still inside the bracket.
// Masses are fp32 terms accumulated per thread in fp32 and combined in fp64; whether a token whose
// probability is 1e-6 still falls inside K is decided with a relative accuracy of about 1e-6 of the total
// mass, which is the accuracy of the fp32 exponentials themselves.
#include "difr_device.hpp"
#include "difr_host.hpp"
#include "ipt_stream.hpp"
#include "topn.hpp"

namespace difr {

constexpr int kNucBins = 16;    // 4 key bits per pass
constexpr int kNucCap = 2048;   // entries gathered and sorted at the end

// The one-read histogram of bf16 rows: one counter per logit value of magnitude above 2^-10 and below 128 (2175 of either sign,
// kHistMag: the pattern of 2^-10), one for the values in between, 64 below and 64 above them for everything outside.
constexpr uint32_t kHistMag = 0x3A80u, kHistSide = 2175u, kHistClamp = 2239u;
constexpr int kHistZero = 2239, kHistWords = 4480, kHistPer = 17;  // word of the values around zero; words; words per thread
constexpr int kHistPairs = 8;  // pairs a thread looks at
constexpr float kHistTwinShare = 0.12f, kHistTwinShort = 4500.0f, kHistTwinMost = 0.6f;  // rows are counted up to this share of equal pairs
constexpr int kHistFirst = kHistZero - (int)kHistSide;               // the lowest logit value's word
static_assert(kHistFirst == 64 && kHistFirst + kHistPer * kBlock == kHistZero + (int)kHistSide + 2, "a thread's words");
static_assert(kHistMag + kHistSide + 1 == 0x4300u, "128 is the first value above");

// LDS the row search needs from its caller: two histograms (bf16), or the bins, whose memory is also the gather buffer
template <int DT>
constexpr int kNucRawBytes = DT == 0 ? 2 * kHistWords * 4 : kNucBins * kBlock * 4;
static_assert(kNucBins * kBlock * 4 >= kNucCap * (int)sizeof(uint64_t), "gather buffer must fit the bin memory");
static_assert(kNucRawBytes<0> >= kNucBins * kBlock * 4, "and so must the histograms");
static_assert(kNucRawBytes<0> >= (kHistPer * kBlock + 1) * (int)sizeof(double), "a mass per value for the token search");

// One row by the multi-pass search described above.  `raw`: kNucRawBytes<DT> of LDS, 16-byte aligned (mass bins
// [bin][thread] during the search; the gather buffer afterwards).  All 256 threads of the workgroup call it.
template <int DT>
__device__ __forceinline__ void nucleus_row_multipass(const RowBatch &b, float top_p, const IptOutputs &o,
                                                      int32_t *__restrict__ kept_out, float *__restrict__ tau_out,
                                                      unsigned char *raw)
{
    typedef typename Elem<DT>::type elt_t;
    constexpr int E = Elem<DT>::kPerVec;
    __shared__ double part_m[16][kNucBins];
    __shared__ double bin_m[kNucBins];
    __shared__ float lds_f[kWaves];
    __shared__ float lds_look[2 * kWaves];
    __shared__ double lds_h[5][kWaves];
    __shared__ double lds_d[kWaves];
    __shared__ int32_t lds_i[kWaves];
    __shared__ int32_t s_fill;
    __shared__ float s_xtau;
    __shared__ double s_mass_in;
    __shared__ uint64_t s_cut;
    float *mass = reinterpret_cast<float *>(raw);
    uint64_t *buf = reinterpret_cast<uint64_t *>(raw);

    const int64_t row = blockIdx.x;
    const RowInfo ri = load_row_info(b, row);
    const int tid = threadIdx.x;
    const float nan = __builtin_nanf("");
    const float ninf = -__builtin_inff();
    const bool want_ipt = o.dist != nullptr;
    auto give_up = [&](uint32_t flag, int32_t kept) __attribute__((always_inline)) {  // uniform over the workgroup
        if (tid == 0) {
            if (want_ipt) {
                o.dist[row] = nan;
                if (o.cdf_lo) o.cdf_lo[row] = nan;
                if (o.cdf_hi) o.cdf_hi[row] = nan;
                if (o.u) o.u[row] = nan;
                if (o.ipt_token) o.ipt_token[row] = -1;
                if (o.log_mass) o.log_mass[row] = nan;
                o.flags[row] = (uint8_t)flag;
            }
            if (kept_out) kept_out[row] = kept;
            if (tau_out) tau_out[row] = nan;
        }
    };
    if (!ri.seq_ok || !ri.temp_ok) {
        give_up(ri.seq_ok ? kFlagNonfinite : kFlagInvalidClaim, 0);
        return;
    }
    const int64_t V = b.V;
    const int64_t t = ri.claimed;
    const bool valid = t >= 0 && t < V;
    const elt_t *x_row = reinterpret_cast<const elt_t *>(b.logits) + row * b.ld;
    const float c = kLog2e / ri.T;

    // One pass over the row: f(q, base) for every 16-byte vector of this thread, with the next vector already
    // requested while the current one is worked on.  Entries past the end of the row read as -inf.
    const int32_t nvec = (int32_t)((V + E - 1) / E);  // V < 2^31
    const uint32_t V32 = (uint32_t)V;
    auto fetch = [&](int32_t vec) { return *reinterpret_cast<const u32x4 *>(x_row + (size_t)vec * E); };
    // the last vector of a ragged row: entries past the end become -inf
    auto ragged_patched = [&](u32x4 q, uint32_t base) __attribute__((always_inline)) {
        if (base + E > V32) {
            uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int j = 0; j < E; ++j) {
                if (base + j < V32) continue;
                if (DT == 0)
                    w[j >> 1] = (j & 1) ? ((w[j >> 1] & 0x0000FFFFu) | 0xFF800000u) : ((w[j >> 1] & 0xFFFF0000u) | 0x0000FF80u);
                else
                    w[j] = 0xFF800000u;
            }
            q = u32x4{w[0], w[1], w[2], w[3]};
        }
        return q;
    };
    auto for_each_vector = [&](auto &&f) __attribute__((always_inline)) {
        int32_t vec = tid;
        u32x4 q_next = u32x4{0u, 0u, 0u, 0u};
        if (vec < nvec) q_next = fetch(vec);
        while (vec < nvec) {
            u32x4 q = q_next;
            const int32_t next = vec + kBlock;
            if (next < nvec) q_next = fetch(next);
            const uint32_t base = (uint32_t)vec * E;
            q = ragged_patched(q, base);
            f(q, base);
            vec = next;
        }
    };
    // Order keys of a vector at the resolution the storage type has: equal logits have equal keys, a larger logit
    // a larger key.  -0 and +0 are the same logit (ties go by index, not by sign), so they share a key.
    // bf16: two 16-bit keys per dword, formed on the packed patterns: 0x8000 + magnitude for a clear sign bit,
    // 0x8000 - magnitude for a set one.  fp32: float_order_bits of the value with -0 read as +0.
    auto keys_of = [&](const u32x4 &q, uint32_t (&kw)[4]) __attribute__((always_inline)) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (DT == 0) {
                typedef int16_t i16x2_t __attribute__((ext_vector_type(2)));
                typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
                const uint32_t sg = __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2_t, w[i]) >> 15);  // 0xFFFF where the sign bit is set
                const uint32_t a = (w[i] & 0x7FFF7FFFu) ^ sg ^ 0x80008000u;  // 0x8000 + m, or 0x7FFF - m
                kw[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2_t, a) - __builtin_bit_cast(u16x2_t, sg));  // (- 0xFFFF = + 1)
            } else {
                kw[i] = float_order_bits(__uint_as_float(w[i]) + 0.0f);
            }
        }
    };
    auto key_of_value = [&](float x) __attribute__((always_inline)) {  // the same key from a single value
        if (DT != 0) return float_order_bits(x + 0.0f);
        const uint32_t b = __float_as_uint(x) >> 16, m = b & 0x7FFFu;
        return (b & 0x8000u) ? 0x8000u - m : 0x8000u + m;
    };
    auto value_of = [&](const u32x4 &q, int j) __attribute__((always_inline)) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        if (DT == 0) return __uint_as_float((j & 1) ? (w[j >> 1] & 0xFFFF0000u) : (w[j >> 1] << 16));
        return __uint_as_float(w[j]);
    };

    // ---- a look at 256 vectors (bf16: spread over the row): their largest entry R and their smallest finite one.  R is the exponent
    //      reference: any finite reference serves (fp32 terms keep their relative precision at every scale, the sums
    //      are fp64); the row maximum M itself comes out of the first search pass, and that pass is repeated with
    //      R = M in the rare case that M lies so far above R that terms could overflow.  The two together tell the
    //      first search pass where to put its bins.  A look without a usable value takes a pass of its own. ----
    float R = ninf, lo_s = __builtin_inff();
    auto look = [&](const u32x4 &q) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const float v = value_of(q, j);
            R = fmaxf(R, v);  // NaNs drop out; the first search pass finds them
            if (v > ninf) lo_s = fminf(lo_s, v);
        }
    };
    typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
    typedef int16_t i16x2_t __attribute__((ext_vector_type(2)));
    // byte offsets of the counters of two entries: `zero_at` that of the values around zero, `least` that of the lowest ones
    auto words_of = [&](uint32_t w, uint32_t zero_at, uint32_t least, u16x2_t &v_min) __attribute__((always_inline)) {
        const u16x2_t m = __builtin_bit_cast(u16x2_t, w & 0x7FFF7FFFu);
        const u16x2_t first = {(uint16_t)kHistMag, (uint16_t)kHistMag}, most = {(uint16_t)kHistClamp, (uint16_t)kHistClamp};
        const u16x2_t v = __builtin_elementwise_min(__builtin_elementwise_sub_sat(m, first), most);
        v_min = __builtin_elementwise_min(v_min, v);
        const uint32_t sg = __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2_t, w) >> 15);
        const u16x2_t step = __builtin_bit_cast(u16x2_t, (sg & 0xFFF8FFF8u) | 0x00040004u);  // +4 or -4
        const u16x2_t at = v * step + __builtin_bit_cast(u16x2_t, zero_at);
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(at, __builtin_bit_cast(u16x2_t, least)));
    };
    // bf16: the first two rounds are requested here already, ahead of what decides how they are used
    const int32_t rounds = (int32_t)((V / E) / kBlock);  // rounds of 256 complete vectors
    u32x4 qa = u32x4{0u, 0u, 0u, 0u}, qb = qa;
    int32_t twins = 0;  // bf16: pairs of entries looked at that a wave would count at once and that share a counter
    if constexpr (DT == 0) {
        // 32 runs of eight vectors spread over the row, which say how the rest looks
        u32x4 q = u32x4{0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u};
        const int32_t vec = nvec >= kBlock ? (tid >> 3) * (nvec / 32) + (tid & 7) : tid;
        if (vec < nvec) q = fetch(vec);
        if (rounds > 0) qa = load_round(x_row, 0);
        if (rounds > 1) qb = load_round(x_row, 1);
        u32x4 *z = reinterpret_cast<u32x4 *>(raw);  // the histograms start at zero
        for (int i = tid; i < 2 * kHistWords / 4; i += kBlock) z[i] = u32x4{0u, 0u, 0u, 0u};
        q = ragged_patched(q, (uint32_t)vec * E);
        if (vec < nvec) look(q);
        if (nvec >= kBlock) {  // uniform; shorter rows are counted whatever they hold
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
            u16x2_t v_min = {0xFFFF, 0xFFFF}, differ = {0, 0};  // of a lane's 8 pairs, those on different counters
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const uint32_t at = words_of(w[i], (uint32_t)(kHistZero * 4) * 0x00010001u, (uint32_t)(tid & 63) * 0x00040004u, v_min);
                const u16x2_t first = {(uint16_t)(kHistFirst * 4), (uint16_t)(kHistFirst * 4)}, one = {1, 1};
                const uint32_t low = __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(first, __builtin_bit_cast(u16x2_t, at)));
                auto compare = [&](int other) __attribute__((always_inline)) {  // (low entries do not count as equal)
                    differ += __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, (at ^ (uint32_t)other) | low), one);
                };
                compare(__builtin_amdgcn_mov_dpp((int)at, 0xB1, 0xF, 0xF, true));  // lane ^ 1
                compare(__builtin_amdgcn_ds_swizzle((int)at, 0x101F));             // lane ^ 4
            }
            twins = kHistPairs - (int32_t)differ.x - (int32_t)differ.y;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            R = fmaxf(R, __shfl_xor(R, off, 64));
            lo_s = fminf(lo_s, __shfl_xor(lo_s, off, 64));
            twins += __shfl_xor(twins, off, 64);
        }
        if ((tid & 63) == 0) {
            lds_look[tid >> 6] = R;
            lds_look[kWaves + (tid >> 6)] = lo_s;
            lds_i[tid >> 6] = twins;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            R = fmaxf(R, lds_look[k]);
            lo_s = fminf(lo_s, lds_look[kWaves + k]);
        }
        twins = lds_i[0] + lds_i[1] + lds_i[2] + lds_i[3];
    } else {
        if (tid < nvec) look(ragged_patched(fetch(tid), (uint32_t)tid * E));  // (ragged only in a row shorter than one round)
        R = block_max(R, lds_f);
    }
    const bool looked = R > ninf && R < __builtin_inff();
    if (!looked) {  // uniform
        R = ninf;
        lo_s = __builtin_inff();
        for_each_vector([&](const u32x4 &q, uint32_t) { look(q); });
        R = block_max(R, lds_f);
        if (!(R > ninf && R < __builtin_inff())) {  // every entry masked, or a +inf
            give_up(kFlagNonfinite | (valid ? 0u : kFlagInvalidClaim), 0);
            return;
        }
    }
    if (DT != 0 || !looked) lo_s = -block_max(-lo_s, lds_f);  // finite and <= R, since R is
    // A mass is 2^((x - R) c64), c64 = log2(e) / T.  The difference x - R comes first: for the entries that carry the
    // mass it is small and exact, so what the fp32 exponent loses is in proportion to it (an exponent formed as
    // x c - R c would carry the rounding of two products of the size of R c, 1e-5 and more when |R| / T is in the
    // hundreds, and the masses that decide the cut - fp32 in the search, fp64 in its last step - would disagree by
    // as much).  The constant is taken in two fp32 pieces, so that what an exponent loses to ITS rounding (a tilt of
    // up to 6e-8 |x - R| c over the whole row, all to one side) is gone as well; the large piece is rounded DOWN, which
    // makes the small one positive: a masked entry, -inf, then gives -inf in both products and a mass of zero with no
    // special case.
    const double c64 = 1.4426950408889634074 / (double)ri.T;
    float c_hi = (float)c64;
    if ((double)c_hi >= c64 && c_hi > 1.0e-30f) c_hi = __uint_as_float(__float_as_uint(c_hi) - 1u);
    const float c_lo = fmaxf((float)(c64 - (double)c_hi), 1.1754944e-38f);
    auto mass_of = [&](float x) __attribute__((always_inline)) {
        const float d = x - R;
        return fast_exp2(__fmaf_rn(d, c_hi, d * c_lo));
    };
    // (the same real number in fp64: for the few masses of the last step)
    auto mass_of_f64 = [&](float x) __attribute__((always_inline)) { return exp2(((double)x - (double)R) * c64); };

    // The same to 1e-11 in a fifth of the instructions: 2^f, |f| <= 1/2, by its Taylor series up to (f ln 2)^9.  For the masses of
    // the counted values, each of which stands for thousands of entries, so that an error of it does not average out.
    auto mass_of_value = [&](float x) __attribute__((always_inline)) {
        const double y = fmin(fmax(((double)x - (double)R) * c64, -2000.0), 1100.0);  // (2^y: 0 and inf out there)
        const double whole = rint(y), f = (y - whole) * 0.69314718055994530942;
        double e = 1.0 / 362880.0;
        e = fma(e, f, 1.0 / 40320.0);
        e = fma(e, f, 1.0 / 5040.0);
        e = fma(e, f, 1.0 / 720.0);
        e = fma(e, f, 1.0 / 120.0);
        e = fma(e, f, 1.0 / 24.0);
        e = fma(e, f, 1.0 / 6.0);
        e = fma(e, f, 0.5);
        e = fma(e, f, 1.0);
        e = fma(e, f, 1.0);
        return ldexp(e, (int)whole);
    };

    // ---- passes B: search for the bracket [klo, khi] of keys that holds the cut ----
    // Keys are the order-preserving images of the logits at the storage type's resolution (16 bits for bf16).
    constexpr uint32_t kKeyPosInf = DT == 0 ? 0xFF80u : 0xFF800000u;  // keys >= this: +inf or a NaN, sign clear
    constexpr uint32_t kKeyNegInf = DT == 0 ? 0x0080u : 0x007FFFFFu;  // -inf; keys < this: a NaN with the sign bit set
    auto value_of_key = [&](uint32_t k) __attribute__((always_inline)) {
        if (DT != 0) return float_from_order_bits(k);
        return __uint_as_float((k >= 0x8000u ? k - 0x8000u : 0x8000u | (0x8000u - k)) << 16);
    };
    auto key_of = [&](const uint32_t (&kw)[4], int j) __attribute__((always_inline)) {
        if (DT == 0) return (j & 1) ? (kw[j >> 1] >> 16) : (kw[j >> 1] & 0xFFFFu);
        return kw[j];
    };
    // block-wide maximum / minimum of a key
    auto block_max_key = [&](uint32_t k) __attribute__((always_inline)) {
        uint32_t m = k;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
        __syncthreads();
        if ((tid & 63) == 0) lds_i[tid >> 6] = (int32_t)m;
        __syncthreads();
        return max(max((uint32_t)lds_i[0], (uint32_t)lds_i[1]), max((uint32_t)lds_i[2], (uint32_t)lds_i[3]));
    };
    auto block_min_key = [&](uint32_t k) __attribute__((always_inline)) {
        uint32_t m = k;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) m = min(m, (uint32_t)__shfl_xor((int)m, off, 64));
        __syncthreads();
        if ((tid & 63) == 0) lds_i[tid >> 6] = (int32_t)m;
        __syncthreads();
        return min(min((uint32_t)lds_i[0], (uint32_t)lds_i[1]), min((uint32_t)lds_i[2], (uint32_t)lds_i[3]));
    };
    // the 256 x 16 per-thread bins -> bin_m[16], in a fixed order, fp64; ends with a barrier
    auto combine_bins = [&]() __attribute__((always_inline)) {
        __syncthreads();
        {
            const int k = tid & 15, grp = tid >> 4;
            double sm = 0.0;
#pragma unroll
            for (int i = 0; i < 16; ++i) sm += (double)mass[k * kBlock + grp * 16 + i];
            part_m[grp][k] = sm;
        }
        __syncthreads();
        if (tid < kNucBins) {
            double sm = 0.0;
#pragma unroll
            for (int grp = 0; grp < 16; ++grp) sm += part_m[grp][tid];
            bin_m[tid] = sm;
        }
        __syncthreads();
    };
    // a thread's bins are its own: plain read-modify-write (LDS float atomics run many times slower here)
    auto add_mass = [&](uint32_t bin, float e) __attribute__((always_inline)) { mass[(int)bin * kBlock + tid] += e; };
    auto clear_bins = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kNucBins; ++k) mass[k * kBlock + tid] = 0.0f;
    };
    double mass_above = 0.0, Zrow = 0.0, target = 0.0;
    uint32_t klo = 0u, khi = 0u;
    // from the top: the first bin in which the cumulative mass reaches the target (every thread walks the same 16
    // values in the same order); what lies above it is added to mass_above
    auto select_bin = [&]() __attribute__((always_inline)) {
        int sel = 0;
        for (int k = kNucBins - 1; k >= 0; --k) {
            if (mass_above + bin_m[k] >= target || k == 0) {
                sel = k;
                break;
            }
            mass_above += bin_m[k];
        }
        return sel;
    };

    double Zk = 0.0, below = 0.0;  // mass of K; mass of the members of K below the claimed token's index
    int64_t kept = 0;
    float tau_val = nan;
    uint64_t cut = 0ull;   // sorted path: the last member of K in rank order
    int64_t n_tie = 0;     // tie path: how many of the ties belong to K
    int32_t tb = 0;        //           and how many ties lie below the claimed token's index
    bool many_ties = false;
    const uint32_t t32 = valid ? (uint32_t)t : 0u;  // an invalid claim has nothing below it (its outputs are NaN anyway)

    // bf16 rows: one read (see the top of this file), unless what has been looked at says that the row is not one for it - its masses reach beyond the
    // histograms' values, or so many entries share a value that a wave's counting would be one entry after the other.
    bool found = false;
    bool try_counts = false;
    auto value_at = [&](int word) __attribute__((always_inline)) {  // the logit value of a counter
        const int v = word - kHistZero;
        return __uint_as_float(v < 0 ? (0x8000u + kHistMag - v) << 16 : v > 0 ? (kHistMag + v) << 16 : 0u);
    };
    // Entries around zero share a counter: their masses are summed vector by vector, and in the same way wherever that sum is met again
    // (entry by entry in fp64, the masses of rows around zero took 3 % of the pass over 16,384 x 151,936).
    auto around_zero = [&](float x) __attribute__((always_inline)) { return fabsf(x) <= 0x1p-10f; };
    auto zero_masses = [&](const u32x4 &q, float (&e)[E]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const float x = value_of(q, j), m = mass_of(x);
            e[j] = around_zero(x) ? m : 0.0f;
        }
    };
    const int word0 = kHistFirst + tid * kHistPer;  // the thread's values
    bool zero_mixed = false;                        // entries around zero that are not zero: the counter there is not one of a value
    int cut_word = 0, top_word = 0;                 // found: the counters of the cut's value and of the row's largest logit
    double e_cut = 0.0;                             //        and the mass of the cut's value
    if constexpr (DT == 0)
        try_counts = R < 128.0f && (lo_s > -128.0f || (-127.5f - R) * c < -126.0f) &&
                     (float)twins <= fminf(kHistTwinShare + kHistTwinShort / (float)V32, kHistTwinMost) * (float)(kHistPairs * kBlock);
    if (DT == 0 && try_counts) {  // uniform
        uint32_t *hist = reinterpret_cast<uint32_t *>(raw);  // [kHistWords] entries below the claim's index, [kHistWords] the others
        const uint32_t lane4 = (uint32_t)(tid & 63) * 0x00040004u;
        u16x2_t mag_max = {0, 0};              // of all entries: above 0x7F80 there was a NaN
        u16x2_t near_min = {0xFFFF, 0xFFFF};   // of the magnitude less one, of entries around zero
        double zero_mass = 0.0, zero_low = 0.0;  // masses of the entries around zero, and of those below the claim's index
        auto count_at = [&](uint32_t byte) __attribute__((always_inline)) {
            __hip_atomic_fetch_add(reinterpret_cast<uint32_t *>(raw + byte), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        auto add_vector = [&](const u32x4 &q, uint32_t base) __attribute__((always_inline)) {
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
            const bool all_below = base + E <= t32;
            const uint32_t other = all_below ? 0u : (uint32_t)(kHistWords * 4) * 0x00010001u;
            const uint32_t zero_at = (uint32_t)(kHistZero * 4) * 0x00010001u + other, least = lane4 + other;
            u16x2_t v_min = {0xFFFF, 0xFFFF};
            uint32_t at[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                mag_max = __builtin_elementwise_max(mag_max, __builtin_bit_cast(u16x2_t, w[i] & 0x7FFF7FFFu));
                at[i] = words_of(w[i], zero_at, least, v_min);
            }
            if (!all_below && base < t32) {  // the one vector that holds the claim: the entries below it move to the first histogram
#pragma unroll
                for (int j = 0; j < E; ++j)
                    if (base + j < t32) at[j >> 1] -= (uint32_t)(kHistWords * 4) << ((j & 1) * 16);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                count_at(at[i] & 0xFFFFu);
                count_at(at[i] >> 16);
            }
            if (min(v_min.x, v_min.y) == 0) {  // entries around zero share a counter: their masses are summed here
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u16x2_t m = __builtin_bit_cast(u16x2_t, w[i] & 0x7FFF7FFFu), one = {1, 1};
                    near_min = __builtin_elementwise_min(near_min, m - one);
                }
                float e[E];
                zero_masses(q, e);
                zero_mass += (double)tree_sum<E>(e);
                if (base < t32) {
#pragma unroll
                    for (int j = 0; j < E; ++j) e[j] = base + j < t32 ? e[j] : 0.0f;
                    zero_low += (double)tree_sum<E>(e);
                }
            }
        };
        {
            int32_t r = 0;
            for (; r + 1 < rounds; r += 2) {
                const u32x4 a = qa, bq = qb;
                if (r + 2 < rounds) qa = load_round(x_row, r + 2);
                if (r + 3 < rounds) qb = load_round(x_row, r + 3);
                add_vector(a, (uint32_t)(r * kBlock + tid) * E);
                add_vector(bq, (uint32_t)((r + 1) * kBlock + tid) * E);
            }
            if (r < rounds) add_vector(qa, (uint32_t)(r * kBlock + tid) * E);
            const int32_t vec = rounds * kBlock + tid;
            if (vec < nvec) add_vector(ragged_patched(fetch(vec), (uint32_t)vec * E), (uint32_t)vec * E);
        }
        const int lane = tid & 63, wave = tid >> 6;
        if (max(mag_max.x, mag_max.y) > 0x7F80u) count_at((uint32_t)(kHistWords - 2) * 4u);  // a NaN: counted with what is too large
        if (min(near_min.x, near_min.y) < kHistMag) count_at((uint32_t)(kHistWords - 1) * 4u);  // (a word no value has)
        if (__builtin_amdgcn_ballot_w64(zero_mass != 0.0) != 0ull) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                zero_mass += __shfl_xor(zero_mass, off, 64);
                zero_low += __shfl_xor(zero_low, off, 64);
            }
        }
        if (lane == 0) {
            lds_h[0][wave] = zero_mass;
            lds_h[1][wave] = zero_low;
        }
        __syncthreads();
        // what the histograms cannot hold (a NaN, +inf, 128 and more) goes to the search below
        const bool any_odd = __builtin_amdgcn_ballot_w64((hist[kHistWords - 65 + lane] | hist[2 * kHistWords - 65 + lane]) != 0u) != 0ull;
        // -128 and less, or masked; what a ragged last vector has past the row's end is in one word, its thread's, and not meant
        const uint32_t past = lane == ((nvec - 1) & 63) ? (uint32_t)nvec * E - V32 : 0u;
        const bool any_low = __builtin_amdgcn_ballot_w64((hist[lane] | (hist[kHistWords + lane] - past)) != 0u) != 0ull;
        zero_mixed = hist[kHistWords - 1] != 0u;
        zero_mass = lds_h[0][0] + lds_h[0][1] + lds_h[0][2] + lds_h[0][3];
        zero_low = lds_h[1][0] + lds_h[1][1] + lds_h[1][2] + lds_h[1][3];
        // a thread's words: their mass, the part of it below the claim's index, their entries.  All of them are read at once and
        // kept for the thread that holds the cut (128 x 128,256: 27.2 us, 28.6 with a word read when its turn comes; 8192: 370 / 373.
        // The masses kept as well and formed without branches: 26.3, but 8192 rows 434, the wave skips words that none of its lanes has).
        double sum = 0.0, sum_low = 0.0;
        int32_t n = 0;
        float top = ninf;
        uint32_t na[kHistPer], nb[kHistPer];
#pragma unroll
        for (int i = 0; i < kHistPer; ++i) {
            na[i] = hist[word0 + i];
            nb[i] = hist[kHistWords + word0 + i];
        }
#pragma unroll
        for (int i = 0; i < kHistPer; ++i) {
            if (na[i] + nb[i] == 0u) continue;
            const bool zero = zero_mixed && word0 + i == kHistZero;
            const float x = value_at(word0 + i);
            const double e = mass_of_value(x);
            sum += zero ? zero_mass : e * (double)(na[i] + nb[i]);
            sum_low += zero ? zero_low : e * (double)na[i];
            n += (int32_t)(na[i] + nb[i]);
            top = x;
        }
        double upto = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double o = __shfl_up(upto, off, 64);
            if (lane >= off) upto += o;
        }
        const float M_wave = wave_max(top);
        if (lane == 63) {
            lds_h[2][wave] = upto;
            lds_f[wave] = M_wave;
        }
        __syncthreads();
        const float M = fmaxf(fmaxf(lds_f[0], lds_f[1]), fmaxf(lds_f[2], lds_f[3]));
        double total = 0.0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            if (k == wave) upto += total;
            total += lds_h[2][k];
        }
        const double goal = (double)top_p * total;
        const double above = total - upto;
        // the highest thread in whose words the cumulative mass from the top reaches the goal
        const uint64_t reached = __builtin_amdgcn_ballot_w64(above + sum >= goal && sum > 0.0);
        if (lane == 0) lds_i[wave] = reached != 0ull ? wave * 64 + 63 - __builtin_clzll(reached) : -1;
        __syncthreads();
        const int ct = max(max(lds_i[0], lds_i[1]), max(lds_i[2], lds_i[3]));
        if (tid == ct) {
            int at = 0;
            double low_above = 0.0, e_above = above;
            int32_t n_above = 0;
            bool done = false;
#pragma unroll
            for (int i = kHistPer - 1; i >= 0; --i) {
                const int32_t c_i = (int32_t)(na[i] + nb[i]);
                if (done || c_i == 0) continue;
                const bool zero = zero_mixed && word0 + i == kHistZero;
                const double e = mass_of_value(value_at(word0 + i)), em = zero ? zero_mass : e * (double)c_i;
                at = word0 + i;
                done = e_above + em >= goal || n_above + c_i == n;  // (the last of the thread's entries)
                if (!done) {
                    e_above += em;
                    low_above += zero ? zero_low : e * (double)na[i];
                    n_above += c_i;
                }
            }
            s_fill = at;
            s_mass_in = e_above;
            sum_low = low_above;
            n = n_above;
        }
        __syncthreads();
        found = !any_odd && ct >= 0 && M > ninf && (M - R) * c <= 96.0f && !(zero_mixed && s_fill == kHistZero);
        // masses of values below the histograms' are zero if the largest logit lies far enough above them; if not, the row is read once
        // more to see whether they are all -inf (finite magnitudes of 128 and more, subtracted from the last one, are below 0x3C80)
        if (found && any_low && !((-127.5f - M) * c < -126.0f)) {  // uniform
            u16x2_t gap = {0xFFFF, 0xFFFF};
            for_each_vector([&](const u32x4 &q, uint32_t) {
                const uint32_t w[4] = {q.x, q.y, q.z, q.w};
                const u16x2_t last = {0x7F7F, 0x7F7F};
#pragma unroll
                for (int i = 0; i < 4; ++i) gap = __builtin_elementwise_min(gap, last - __builtin_bit_cast(u16x2_t, w[i] & 0x7FFF7FFFu));
            });
            found = block_min_key(min(gap.x, gap.y)) >= 0x3C80u;
        }
        if (found) {  // uniform
            const int at = s_fill;
            cut_word = at;
            top_word = M > 0.0f ? kHistZero + max((int)(__float_as_uint(M) >> 16) - (int)kHistMag, 0) : kHistZero;
            tau_val = value_at(at);
            klo = khi = key_of_value(tau_val);
            tb = (int32_t)hist[at];
            const int64_t bracket = (int64_t)hist[at] + (int64_t)hist[kHistWords + at];
            mass_above = s_mass_in;
            e_cut = mass_of_value(tau_val);
            n_tie = e_cut > 0.0 ? (int64_t)ceil((goal - mass_above) / e_cut) : bracket;
            n_tie = n_tie < 1 ? 1 : (n_tie > bracket ? bracket : n_tie);
            many_ties = true;
            double low_sum = tid >= ct ? sum_low : 0.0;
            int32_t n_sum = tid >= ct ? n : 0;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                low_sum += __shfl_xor(low_sum, off, 64);
                n_sum += __shfl_xor(n_sum, off, 64);
            }
            if (lane == 0) {
                lds_h[3][wave] = low_sum;
                lds_h[4][wave] = (double)n_sum;
            }
            __syncthreads();
            below = lds_h[3][0] + lds_h[3][1] + lds_h[3][2] + lds_h[3][3] + e_cut * (double)((int64_t)tb < n_tie ? (int64_t)tb : n_tie);
            Zk = mass_above + e_cut * (double)n_tie;
            kept = (int64_t)(lds_h[4][0] + lds_h[4][1] + lds_h[4][2] + lds_h[4][3]) + n_tie;
        }
        __syncthreads();
    }

    if (!found) {  // uniform: the search by passes
    // First pass: every entry counts (the total mass Z fixes the target), and the 16 bins divide the span of
    // LOGIT VALUES seen in the look evenly - the mass is spread over logit values, not over key bits, which
    // spend most of their range on exponents near zero.  bin1 is monotone in the logit, so each bin is a range of
    // keys; values outside the span that was seen fall into the end bins.
    double bracket_mass;  // mass of the entries with keys in [klo, khi]
    while (true) {
        float sc = (R > lo_s) ? 16.0f / (R - lo_s) : 0.0f;
        if (!(sc > 0.0f && sc < 1.0e30f)) sc = 1.0e-30f;  // no span to divide: every finite value lands in bin 0
        const float off = -(lo_s * sc);
        auto bin1 = [&](float x) __attribute__((always_inline)) {  // (clamped before the conversion: always in range)
            return (uint32_t)(int)__builtin_amdgcn_fmed3f(__fmaf_rn(x, sc, off), 0.0f, 15.0f);
        };
        clear_bins();
        // Largest and smallest key met.  bf16: three packed extremes of the raw bit patterns (of the even and of the
        // odd entries) tell as much, at three instructions per two entries: the largest pattern as signed 16-bit is
        // the largest entry that is not negative (or +inf, or a NaN with the sign clear), the largest as unsigned the
        // most negative one (or -inf, or a NaN with the sign set), the smallest as unsigned the negative entry nearest
        // to zero if all are negative, else the smallest non-negative one.
        typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
        typedef int16_t i16x2_t __attribute__((ext_vector_type(2)));
        uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
        uint32_t smax = 0x80008000u, umax = 0u, umin = 0xFFFFFFFFu;
        for_each_vector([&](const u32x4 &q, uint32_t) {
            if (DT == 0) {
                const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    smax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2_t, smax), __builtin_bit_cast(i16x2_t, w[i])));
                    umax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, umax), __builtin_bit_cast(u16x2_t, w[i])));
                    umin = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, umin), __builtin_bit_cast(u16x2_t, w[i])));
                }
            } else {
                uint32_t kw[4];
                keys_of(q, kw);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    kmax = max(kmax, kw[i]);
                    kmin = min(kmin, kw[i]);
                }
            }
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const float x = value_of(q, j);
                add_mass(bin1(x), mass_of(x));
            }
        });
        bool sign_set_nan = false;
        if (DT == 0) {
            // (signed maximum through the unsigned reduction: flip the sign bit)
            const uint32_t sm = block_max_key(max((smax & 0xFFFFu) ^ 0x8000u, (smax >> 16) ^ 0x8000u)) ^ 0x8000u;
            const uint32_t um = block_max_key(max(umax & 0xFFFFu, umax >> 16));
            const uint32_t un = block_min_key(min(umin & 0xFFFFu, umin >> 16));
            auto key_of_pattern = [&](uint32_t p) __attribute__((always_inline)) {
                return (p & 0x8000u) ? 0x8000u - (p & 0x7FFFu) : 0x8000u + p;
            };
            sign_set_nan = um > 0xFF80u;
            kmax = key_of_pattern(sm < 0x8000u ? sm : un);  // a non-negative entry exists: the largest of them
            kmin = key_of_pattern(um >= 0x8000u ? um : un);  // a negative entry exists: the most negative of them
        } else {
            kmax = block_max_key(kmax);  // (a thread without a vector still holds the neutral values)
            kmin = block_min_key(kmin);
        }
        if (kmax >= kKeyPosInf || kmin < kKeyNegInf || sign_set_nan) {  // uniform: NaN or +inf somewhere, no distribution
            give_up(kFlagNonfinite | (valid ? 0u : kFlagInvalidClaim), 0);
            return;
        }
        const float M = value_of_key(kmax);
        if ((M - R) * c > 96.0f) {  // uniform; terms of 2^96 and more: start again from M
            R = M;
            continue;
        }
        combine_bins();
        double Z = 0.0;
        for (int k = 0; k < kNucBins; ++k) Z += bin_m[k];
        Zrow = Z;
        target = (double)top_p * Z;
        const uint32_t sel = (uint32_t)select_bin();
        // the keys of bin `sel`: bin1 is monotone over the keys from -inf to the largest finite one, so the first
        // key of a bin is found by bisection (every thread runs the same search)
        auto first_key_of_bin = [&](uint32_t b) __attribute__((always_inline)) {  // smallest key k with bin1 >= b
            uint32_t a = kKeyNegInf, z = kKeyPosInf;                              // answer in [a, z]
            while (a < z) {
                const uint32_t mid = a + ((z - a) >> 1);
                if (bin1(value_of_key(mid)) >= b)
                    z = mid;
                else
                    a = mid + 1;
            }
            return a;
        };
        klo = sel == 0 ? kKeyNegInf : first_key_of_bin(sel);
        khi = sel == 15 ? kKeyPosInf - 1u : first_key_of_bin(sel + 1u) - 1u;
        klo = max(klo, kmin);
        khi = min(khi, kmax);
        bracket_mass = bin_m[sel];  // clipping to [kmin, kmax] removes no entry
        __syncthreads();            // the bins are cleared or reused next
        break;
    }

    // bf16 rows whose bracket is at most 16 logit values, however many entries (the usual case when K is large:
    // near the cut a bf16 value is shared by thousands of tokens): ONE more pass finishes the row, without the sort that
    // pass C needs (4096 rows of 8000 with some 1500 entries in the bracket: 285 us sorted, 202 counted).  Entries of equal
    // value have equal mass, so the pass only counts, per value of the bracket and per thread, the entries and those
    // of them below the claimed token's index (16 + 16 bits in one private LDS word), and sums what lies above the
    // bracket as the last pass of the general path does.  The values' masses are then taken in fp64, the value at
    // which the cumulative mass reaches the target is found by walking at most 16 of them, and it is treated as the
    // general path treats a single-value bracket: its ties enter K in index order.
    bool provably_small = false;
    {
        const double e_lo = (double)mass_of(value_of_key(klo));
        provably_small = e_lo > 0.0 && e_lo < (double)__builtin_inff() && bracket_mass <= e_lo * (double)(kNucCap - 48);
    }
    const bool by_counts = DT == 0 && khi > klo && khi - klo < (uint32_t)kNucBins && V <= (int64_t)(1 << 24);
    // A bracket may hold few entries although its mass does not prove it: the end bin at the top takes in everything above
    // the largest entry looked at, the row's few heaviest tokens among them, and its keys span the octaves around zero,
    // which the further search passes divide badly (rows whose nucleus is small, top_p = 0.95 at T = 0.7: half of them took
    // two or three such passes).  256 vectors spread over the row say how many to expect; if that is well below what pass C can
    // gather, pass C is tried at once, and only if its buffer runs over does the search go on (2048 rows of 128,256 bf16 logits at
    // T = 0.7: 368 us without the try, 315 with it; 2048 rows of 65,536 fp32 logits: 321 / 252).  Spread, since the row's beginning
    // may say nothing about the rest: with the first 256 vectors instead, rows that begin with 2048 very low entries threw a whole
    // pass away (2048 x 128,256, T = 0.9: 835 us, 694 now, 677 without the try), and 100,000 entries at T = 0.75 took 242 us for
    // 215; where the first vectors were right they cost 1% less (T = 0.6: 281 / 285).
    bool try_gather = false;
    if (!by_counts && !provably_small) {  // uniform
        const uint32_t span = khi - klo;
        int32_t seen = 0;
        const int32_t step = max(nvec / kBlock, 1), vec = tid * step;
        if (tid < nvec) {
            uint32_t kw[4];
            keys_of(ragged_patched(fetch(vec), (uint32_t)vec * E), kw);
#pragma unroll
            for (int j = 0; j < E; ++j) seen += (int32_t)(key_of(kw, j) - klo <= span && (uint32_t)vec * E + j < V32);
        }
        seen = block_sum_i32(seen, lds_i);
        try_gather = (int64_t)seen * step <= kNucCap / 2;
    }
    if (by_counts) {  // uniform
        const uint32_t span = khi - klo;
        uint32_t *cnt = reinterpret_cast<uint32_t *>(raw);  // [key - klo][thread]; a thread meets fewer than 2^16 entries
#pragma unroll
        for (int k = 0; k < kNucBins; ++k) cnt[k * kBlock + tid] = 0u;
        double below_above = 0.0;
        int32_t n_above = 0;
        for_each_vector([&](const u32x4 &q, uint32_t base) {
            uint32_t kw[4];
            keys_of(q, kw);
            float below_vec = 0.0f;
            // whether an entry lies below the claimed token's index is the same for a whole vector, but for the one
            // vector of the row that holds the claim (and a ragged last one is looked at entry by entry as well)
            const bool all_below = base + E <= t32;
            const bool mixed = (!all_below && base < t32) || base + E > V32;
            if (__builtin_amdgcn_ballot_w64(mixed) == 0ull) {
                const uint32_t inc = all_below ? 0x10001u : 1u;
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    const uint32_t key = key_of(kw, j);
                    const uint32_t d = key - klo;
                    if (d <= span) {
                        cnt[(int)d * kBlock + tid] += inc;
                    } else if (key > khi) {
                        n_above += 1;
                        if (all_below) below_vec += mass_of(value_of(q, j));
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    if (base + E > V32 && base + j >= V32) continue;  // (a ragged last vector)
                    const uint32_t key = key_of(kw, j);
                    const uint32_t d = key - klo;
                    if (d <= span) {
                        cnt[(int)d * kBlock + tid] += (base + j < t32) ? 0x10001u : 1u;
                    } else if (key > khi) {
                        n_above += 1;
                        if (base + j < t32) below_vec += mass_of(value_of(q, j));
                    }
                }
            }
            below_above += (double)below_vec;
        });
        // the 256 x 16 counters -> 16 totals of each kind (exact), through the memory of part_m
        int32_t(*part_c)[kNucBins][2] = reinterpret_cast<int32_t(*)[kNucBins][2]>(&part_m[0][0]);
        int32_t *key_cnt = reinterpret_cast<int32_t *>(&bin_m[0]);  // [16][2]
        __syncthreads();
        {
            const int k = tid & 15, grp = tid >> 4;
            int32_t all = 0, low = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t v = cnt[k * kBlock + grp * 16 + i];
                all += (int32_t)(v & 0xFFFFu);
                low += (int32_t)(v >> 16);
            }
            part_c[grp][k][0] = all;
            part_c[grp][k][1] = low;
        }
        __syncthreads();
        if (tid < 2 * kNucBins) {
            int32_t sm = 0;
#pragma unroll
            for (int grp = 0; grp < 16; ++grp) sm += part_c[grp][tid >> 1][tid & 1];
            key_cnt[tid] = sm;
        }
        __syncthreads();
        // the values' masses, one per thread: an fp64 exponential is 100 instructions and more, and a walk in which every
        // thread took all of them made the row's fixed cost what a short row spent its time on
        double *key_mass = &part_m[0][0];
        if (tid <= (int)span) key_mass[tid] = mass_of_f64(value_of_key(klo + (uint32_t)tid));
        const int64_t cnt_above = (int64_t)block_sum_i32(n_above, lds_i);  // (its barriers publish the masses)
        // from the top: the first value at which the cumulative mass reaches the target (every thread walks the
        // same values in the same order); the values above it belong to K whole
        double ma = mass_above, below_hi = 0.0;
        int64_t cnt_hi = 0;
        int jcut = -1, jlast = -1;
        for (int j = (int)span; j >= 0; --j) {
            const int64_t na = key_cnt[2 * j];
            if (na == 0) continue;
            const double e = key_mass[j];
            jlast = j;
            e_cut = e;
            if (ma + e * (double)na >= target) {
                jcut = j;
                break;
            }
            ma += e * (double)na;
            cnt_hi += na;
            below_hi += e * (double)key_cnt[2 * j + 1];
        }
        many_ties = true;
        if (jcut < 0 && jlast >= 0) {  // rounding left the target just out of reach: the whole bracket
            jcut = jlast;
            const int64_t na = key_cnt[2 * jcut];
            ma -= e_cut * (double)na;
            cnt_hi -= na;
            below_hi -= e_cut * (double)key_cnt[2 * jcut + 1];
        }
        const int64_t bracket = jcut >= 0 ? (int64_t)key_cnt[2 * jcut] : 0;
        tb = jcut >= 0 ? key_cnt[2 * jcut + 1] : 0;
        n_tie = e_cut > 0.0 ? (int64_t)ceil((target - ma) / e_cut) : bracket;
        n_tie = n_tie < 1 ? 1 : n_tie;
        n_tie = n_tie > bracket ? bracket : n_tie;
        klo = khi = klo + (uint32_t)(jcut >= 0 ? jcut : 0);
        tau_val = value_of_key(klo);
        below = block_sum_f64(below_above, lds_d) + below_hi + e_cut * (double)((int64_t)tb < n_tie ? (int64_t)tb : n_tie);
        Zk = ma + e_cut * (double)n_tie;
        kept = cnt_above + cnt_hi + n_tie;
        mass_above = ma;
    } else {
    // Further passes: the bracket's key range divided evenly into at most 16 bins, until it is a single key (one
    // logit value) or provably small enough to sort.  No counts are kept: every entry of the bracket weighs at
    // least as much as the bracket's smallest key would, so mass / that weight bounds the number of entries.
    bool single_value = false;
    double below_above;   // mass of entries above the bracket with index < t
    int32_t ties_below;   // many_ties: bracket entries with index < t ...
    int32_t ties;         // ... and all of them
    int32_t n_above;      // entries above the bracket
    while (true) {
    while (!try_gather) {
        if (khi <= klo) {  // (khi < klo cannot happen: the selected bin holds mass)
            khi = klo;
            single_value = true;
            break;
        }
        {  // (a bracket whose lower edge is -inf gives no bound)
            const double e_lo = (double)mass_of(value_of_key(klo));
            if (e_lo > 0.0 && e_lo < (double)__builtin_inff() && bracket_mass <= e_lo * (double)(kNucCap - 48)) break;
        }
        const uint32_t span = khi - klo;
        const int sh = max(0, 28 - (int)__builtin_clz(span));  // span >> sh <= 15
        clear_bins();
        for_each_vector([&](const u32x4 &q, uint32_t) {
            uint32_t kw[4];
            keys_of(q, kw);
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const uint32_t d = key_of(kw, j) - klo;
                if (d <= span) add_mass(d >> sh, mass_of(value_of(q, j)));
            }
        });
        combine_bins();
        const uint32_t sel = (uint32_t)select_bin();
        bracket_mass = bin_m[sel];
        klo = klo + (sel << sh);
        khi = min(khi, klo + ((1u << sh) - 1u));
        __syncthreads();  // the bins are cleared or reused next
    }
    // A single logit value shared by the whole bracket (possibly thousands of tokens) needs no sorting: the ties
    // enter K in index order, each with the same mass, and how many of them do is a division.
    many_ties = single_value;

    // ---- pass C: gather the bracket (or count the ties below the claimed token), and sum what lies above the
    //      bracket and below the claimed token's index ----
    if (tid == 0) s_fill = 0;
    __syncthreads();
    below_above = 0.0;
    ties_below = ties = n_above = 0;
    const uint32_t span_c = khi - klo;
    for_each_vector([&](const u32x4 &q, uint32_t base) {
        uint32_t kw[4];
        keys_of(q, kw);
        float below_vec = 0.0f;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            if (base + E > V32 && base + j >= V32) continue;  // (false for every vector but a ragged last one)
            const uint32_t key = key_of(kw, j);
            if (key - klo <= span_c) {
                if (many_ties) {
                    ties += 1;
                    ties_below += (int32_t)(base + j < t32);
                    s_xtau = value_of(q, j);  // the same value from every thread that writes it
                } else {
                    const int32_t i = atomicAdd(&s_fill, 1);
                    if (i < kNucCap) buf[i] = top_composite(value_of(q, j), (int32_t)(base + j));
                }
            } else if (key > khi) {
                n_above += 1;
                if (base + j < t32) below_vec += mass_of(value_of(q, j));
            }
        }
        below_above += (double)below_vec;
    });
    __syncthreads();
    if (!try_gather || s_fill <= kNucCap) break;  // uniform
    try_gather = false;  // more than the sample promised: the search goes on
    __syncthreads();     // (s_fill has been read)
    }
    const int64_t cnt_above = (int64_t)block_sum_i32(n_above, lds_i);

    if (many_ties) {
        tau_val = s_xtau;
        const double e_tau = mass_of_f64(tau_val);
        const int64_t bracket = (int64_t)block_sum_i32(ties, lds_i);
        n_tie = e_tau > 0.0 ? (int64_t)ceil((target - mass_above) / e_tau) : bracket;
        n_tie = n_tie < 1 ? 1 : (n_tie > bracket ? bracket : n_tie);
        tb = block_sum_i32(ties_below, lds_i);
        below = block_sum_f64(below_above, lds_d) + e_tau * (double)((int64_t)tb < n_tie ? (int64_t)tb : n_tie);
        Zk = mass_above + e_tau * (double)n_tie;
        kept = cnt_above + n_tie;
    } else {
        const int n = min(s_fill, kNucCap);
        int P = 256;
        while (P < n) P <<= 1;
        for (int i = n + tid; i < P; i += kBlock) buf[i] = 0ull;  // below every real composite
        __syncthreads();
        // descending: rank order (larger logit first, then the smaller index).  One entry per thread finds its place by
        // counting the entries above it (two barriers, broadcast reads); more go through a bitonic sort.
        if (P == kBlock) {
            const uint64_t mine = buf[tid];
            int place = 0;
            for (int i = 0; i < n; ++i) place += (int)(buf[i] > mine);
            __syncthreads();
            if (tid < n) buf[place] = mine;
            __syncthreads();
        }
        for (int k = 2; k <= P && P > kBlock; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int i = tid; i < P; i += kBlock) {
                    const int l = i ^ j;
                    if (l > i) {
                        const uint64_t a = buf[i], bb = buf[l];
                        const bool desc = (i & k) == 0;
                        if (desc ? (a < bb) : (a > bb)) {
                            buf[i] = bb;
                            buf[l] = a;
                        }
                    }
                }
                __syncthreads();
            }
        }
        // walk the sorted bracket: thread `tid` owns positions [tid * per, tid * per + per)
        const int per = P / kBlock;
        const double first = tid * per < n ? mass_of_f64(top_key(buf[tid * per])) : 0.0;  // (all there is when per = 1)
        auto term = [&](int q) {  // mass of the thread's q-th position (0 past the end)
            if (q == 0) return first;
            const int i = tid * per + q;
            return (q < per && i < n) ? mass_of_f64(top_key(buf[i])) : 0.0;
        };
        double run = 0.0;
#pragma unroll
        for (int q = 0; q < kNucCap / kBlock; ++q) run += term(q);
        double total;
        const double before = block_inclusive_scan(run, lds_d, total) - run;
        // The target, with the bracket's share of the total mass in fp64 as well: a bracket that holds the row's heaviest
        // tokens would otherwise be measured against a total that carries the rounding of their fp32 exponentials (6e-8 of
        // a mass near 1, a marginal token's worth).
        const double goal = (double)top_p * (Zrow - bracket_mass + total);
        // the first position at which the cumulative mass reaches the target: in the thread, then over the workgroup
        int32_t my_pos = 0x7FFFFFFF;
        double my_mass = 0.0, acc = before;
#pragma unroll
        for (int q = 0; q < kNucCap / kBlock; ++q) {
            acc += term(q);
            if (q < per && tid * per + q < n && my_pos == 0x7FFFFFFF && mass_above + acc >= goal) {
                my_pos = tid * per + q;
                my_mass = acc;
            }
        }
        int32_t pos = my_pos;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) pos = min(pos, __shfl_xor(pos, off, 64));
        if ((tid & 63) == 0) lds_i[tid >> 6] = pos;
        __syncthreads();
        pos = min(min(lds_i[0], lds_i[1]), min(lds_i[2], lds_i[3]));
        if (pos == 0x7FFFFFFF) {  // rounding left the target just out of reach: the whole bracket
            pos = n - 1;
            if (n > 0 && pos >= tid * per && pos < tid * per + per) {
                s_mass_in = before + run;
                s_cut = buf[pos];
            }
        } else if (pos == my_pos) {
            s_mass_in = my_mass;
            s_cut = buf[pos];
        }
        if (n == 0 && tid == 0) {  // cannot happen for top_p > 0 (the selected bin is never empty); be safe
            s_mass_in = 0.0;
            s_cut = ~0ull;
        }
        __syncthreads();
        cut = s_cut;
        Zk = mass_above + s_mass_in;
        // included bracket entries below the claimed token's index
        double mine_below = 0.0;
#pragma unroll
        for (int q = 0; q < kNucCap / kBlock; ++q) {
            const int i = tid * per + q;
            if (q < per && i <= pos && i < n && (int64_t)top_index(buf[i]) < t) mine_below += term(q);
        }
        below = block_sum_f64(below_above + mine_below, lds_d);
        kept = cnt_above + (int64_t)(n > 0 ? pos + 1 : 0);
        tau_val = n > 0 ? top_key(cut) : nan;
    }
    }  // (the general path)
    }  // (the search by passes)
    const uint32_t span_c = khi - klo;  // for the sampler's token below

    if (tid == 0) {
        if (kept_out) kept_out[row] = (int32_t)kept;
        if (tau_out) tau_out[row] = tau_val;
    }
    if (!want_ipt) return;

    // ---- the interval of the claimed token (every thread forms it: whether the sampler's token has to be
    //      searched is decided by all of them) ----
    uint32_t r[4];
    noise_block(ri.key, ri.pos, ri.seq, kStreamIpt, 0u, r);
    const float u = uniform_from_bits(r[0]);
    const double ud = (double)u;
    float a = nan, bb = nan, d = nan;
    double ad = 0.0, bd = 0.0;
    bool match = false;
    const bool ok = Zk > 0.0 && Zk < (double)__builtin_inff();
    if (valid && ok) {
        const float xt = Elem<DT>::to_float(x_row[t]);
        bool in_K;
        if (many_ties) {
            const uint32_t kt = key_of_value(xt);
            in_K = kt > khi || (kt == klo && (int64_t)tb < n_tie);
        } else {
            in_K = top_composite(xt, (int32_t)t) >= cut;
        }
        const double own = !in_K ? 0.0 : found && !(zero_mixed && around_zero(xt)) ? mass_of_value(xt) : (double)mass_of(xt);
        ad = below / Zk;
        bd = ad + own / Zk;
        a = (float)ad;
        bb = (float)bd;
        d = (float)fmax(fmax(ad - ud, ud - bd), 0.0);
        match = (ad <= ud) && (ud < bd);
    }
    uint32_t f = 0;
    if (!valid) f |= kFlagInvalidClaim;
    if (!ok) f |= kFlagNonfinite;
    if (match) f |= kFlagMatch;

    // ---- the sampler's own token, when asked for and the claim is not it: one more pass, in vocabulary order, over
    //      the masses of the members of K until their running sum exceeds u Z_K.  A token above the bracket is a
    //      member, one inside it is if it ranks no lower than the cut (sorted bracket) or is among the first n_tie
    //      of the ties in index order; the pass ends with the step that holds the token.
    //      A counted row is walked in the masses that its interval is made of, the fp64 masses of the values above the cut, in the
    //      memory of the counters.  In fp32 exponentials, whose error is the same for all the entries of a value, one drawn token in
    //      1400 to 4000 did not match when it was scored (4096 rows of 128,256 entries, 60,000 to 120,000 kept).  Price, us, fp32 /
    //      fp64: 2048 x 128,256 with 124 kept 329 / 336, with 27,000 kept 366 / 372; 4096 x 1000 62 / 72. ----
    int32_t tok = match ? (int32_t)t : -1;
    if (o.ipt_token != nullptr && ok && !match) {  // uniform
        f |= kFlagSlowPath;
        const double goal = ud * Zk;
        double before = 0.0;       // mass of the members in the steps already walked
        int64_t ties_before = 0;   // many_ties: bracket entries in those steps
        int32_t last_member = -1;  // the thread's last member so far (rounding can leave the goal just out of reach)
        if (tid == 0) s_fill = -1;
        double *mass_at = reinterpret_cast<double *>(raw);  // counted rows: [0] for the cut's value and all below, then the values above it
        const bool zeros_in = zero_mixed && cut_word < kHistZero;
        if (DT == 0 && found) {
            for (int i = tid; i <= top_word - cut_word; i += kBlock) mass_at[i] = i > 0 ? mass_of_value(value_at(cut_word + i)) : 0.0;
        }
        __syncthreads();
        for (int32_t vec0 = 0; vec0 < nvec; vec0 += kBlock) {
            const int32_t vec = vec0 + tid;
            const uint32_t base = (uint32_t)vec * E;
            u32x4 q = u32x4{0u, 0u, 0u, 0u};
            uint32_t kw[4] = {0u, 0u, 0u, 0u};
            int32_t my_ties = 0;
            if (vec < nvec) {
                q = ragged_patched(fetch(vec), base);
                keys_of(q, kw);
                if (many_ties) {
#pragma unroll
                    for (int j = 0; j < E; ++j) my_ties += (int32_t)(key_of(kw, j) - klo <= span_c);
                }
            }
            int64_t tie_rank = 0;  // many_ties: bracket entries with a smaller index than this thread's first
            if (many_ties) {       // uniform
                double tie_total;
                const double incl = block_inclusive_scan((double)my_ties, lds_d, tie_total);  // (exact: small integers)
                tie_rank = ties_before + (int64_t)(incl - (double)my_ties);
                ties_before += (int64_t)tie_total;
            }
            double ls = 0.0;
            double ed[E];  // counted rows
            float e[E];
            if (DT == 0 && found) {  // uniform
                if (vec < nvec) {
                    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
                    u16x2_t v_min = {0xFFFF, 0xFFFF};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t at = words_of(w[i], (uint32_t)(kHistZero * 4) * 0x00010001u, (uint32_t)(cut_word * 4) * 0x00010001u, v_min);
                        ed[2 * i] = mass_at[(at & 0xFFFFu) / 4 - cut_word];
                        ed[2 * i + 1] = mass_at[(at >> 16) / 4 - cut_word];
                    }
                    if (zeros_in && min(v_min.x, v_min.y) == 0) {
                        zero_masses(q, e);
                        ls = (double)tree_sum<E>(e);  // their sum as the interval has it, less what is added below
#pragma unroll
                        for (int j = 0; j < E; ++j) {
                            if (around_zero(value_of(q, j))) ed[j] = (double)e[j];
                            ls -= (double)e[j];
                        }
                    }
                    if (my_ties > 0) {
#pragma unroll
                        for (int j = 0; j < E; ++j)
                            if (key_of(kw, j) == klo && tie_rank++ < n_tie) ed[j] = e_cut;
                    }
#pragma unroll
                    for (int j = 0; j < E; ++j) {
                        ls += ed[j];
                        if (ed[j] > 0.0) last_member = (int32_t)(base + j);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < E; ++j) ed[j] = 0.0;
                }
            } else {
#pragma unroll
            for (int j = 0; j < E; ++j) {
                e[j] = 0.0f;
                if (vec >= nvec) continue;
                const uint32_t key = key_of(kw, j);
                bool member = key > khi;
                if (key - klo <= span_c)
                    member = many_ties ? (tie_rank++ < n_tie) : (top_composite(value_of(q, j), (int32_t)(base + j)) >= cut);
                if (member) {
                    e[j] = mass_of(value_of(q, j));
                    last_member = (int32_t)(base + j);
                }
            }
            ls = (double)tree_sum<E>(e);
            }
            double total;
            const double incl = block_inclusive_scan(ls, lds_d, total);
            if (before + total > goal) {  // uniform: the token is inside this step
                const double excl = before + (incl - ls);
                if (excl <= goal && before + incl > goal) {  // exactly one thread
                    double cacc = excl;
                    int32_t here = -1;
#pragma unroll
                    for (int j = 0; j < E; ++j) {
                        const double ej = DT == 0 && found ? ed[j] : (double)e[j];
                        cacc += ej;
                        if (here < 0 && ej > 0.0 && cacc > goal) here = (int32_t)(base + j);
                    }
                    s_fill = here >= 0 ? here : last_member;  // (here < 0: rounding between the two sums)
                }
                break;
            }
            before += total;
        }
        __syncthreads();
        tok = s_fill;
        if (tok < 0) {  // u Z_K at or beyond the accumulated total: the last member of K in vocabulary order
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) last_member = max(last_member, __shfl_xor(last_member, off, 64));
            __syncthreads();
            if ((tid & 63) == 0) lds_i[tid >> 6] = last_member;
            __syncthreads();
            tok = max(max(lds_i[0], lds_i[1]), max(lds_i[2], lds_i[3]));
        }
    }

    if (tid == 0) {
        o.dist[row] = d;
        if (o.cdf_lo) o.cdf_lo[row] = a;
        if (o.cdf_hi) o.cdf_hi[row] = bb;
        if (o.u) o.u[row] = u;
        if (o.ipt_token) o.ipt_token[row] = ok ? tok : -1;
        if (o.log_mass) o.log_mass[row] = (valid && ok) ? (float)gaussian_log_mass(ad, bd, ud, o.sigma, o.eps) : nan;
        o.flags[row] = (uint8_t)f;
    }
}

// (bf16: four workgroups to a compute unit is what the histograms' LDS allows.  fp32, six waves per SIMD: 77 registers, no vector
// spills; seven and eight spill)
template <int DT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(DT == 0 ? 4 : 6))) void ipt_nucleus_kernel(RowBatch b, float top_p, IptOutputs o,
                                                             int32_t *__restrict__ kept_out, float *__restrict__ tau_out)
{
    __shared__ __attribute__((aligned(16))) unsigned char raw[kNucRawBytes<DT>];
    nucleus_row_multipass<DT>(b, top_p, o, kept_out, tau_out, raw);
}

int launch_ipt_nucleus(const RowBatch &b, float top_p, const IptOutputs &o, int32_t *kept, float *tau, hipStream_t stream)
{
    const dim3 grid((unsigned)b.N), block(kBlock);
    if (b.dtype == 0)
        ipt_nucleus_kernel<0><<<grid, block, 0, stream>>>(b, top_p, o, kept, tau);
    else
        ipt_nucleus_kernel<1><<<grid, block, 0, stream>>>(b, top_p, o, kept, tau);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace difr
