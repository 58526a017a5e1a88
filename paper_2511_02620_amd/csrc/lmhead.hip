// Fused LM head + scoring: the logits x[n][v] = <hidden[n], weight[v]> (the last step of the
// verifier's prefill; appendix algorithm "sampled token verification via prefill") are produced
// tile by tile on the matrix cores and scored in registers by both estimators (Token-DiFR,
// Sec. 6.3; Token-IPT-DiFR, Sec. 6.2) without ever being written to memory.
//
// Work split: a workgroup owns 256 token rows and a contiguous range of 256-entry vocabulary
// tiles.  Per tile it runs a bf16 MFMA GEMM over the hidden dimension (W tile as the A operand,
// H tile as the B operand, both staged through LDS in 64-deep slabs, double buffered), so that in
// the 32x32 accumulator blocks a lane holds 16 vocabulary entries of ONE token, four consecutive
// entries per register group: exactly the granularity of one Philox4x32 block.  The epilogue
// then updates, per lane and token, the running best perturbed score and the online softmax sums,
// and the next tile starts.  Partial results of the vocabulary ranges are merged by a last kernel.
#include <type_traits>
#include <utility>

#include "difr_device.hpp"
#include "difr_host.hpp"
#include "gumbel_stream.hpp"
#include "ipt_stream.hpp"
#include "lmhead.hpp"

namespace difr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// When the 16 copies of a slab are issued: copy c goes out after matrix instruction kCopySlot[c] of the 48
// issued in the fourth k step of one slab and the first two of the next.  Spaced out because the memory
// pipeline accepts a 1 KB copy only every so often, and a wave whose copy is not accepted cannot issue its
// next matrix instruction either (measured: all 16 in one k step cost 11% of the kernel's time).
__host__ __device__ constexpr int copy_at_slot(int n)
{
    constexpr int kCopySlot[16] = {0, 3, 5, 8, 10, 13, 15, 18, 20, 23, 25, 28, 30, 33, 35, 38};
    for (int c = 0; c < 16; ++c)
        if (kCopySlot[c] == n) return c;
    return -1;
}

// f(integral_constant<int, 0>()), ..., f(integral_constant<int, N - 1>()): a loop whose index is a compile-time
// constant in the body (register numbers and instruction immediates depend on it)
template <int... Is, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, Is...>, F &&f)
{
    (f(std::integral_constant<int, Is>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>(), f);
}

struct TokInfo {
    PhiloxKey key;
    uint32_t pos, seq;
    float inv_T;
    int32_t tg, ti;  // claims of the two estimators, -1 if absent or out of range
    bool ok;         // sequence id and temperature usable
    bool seq_ok;
};

__device__ __forceinline__ TokInfo load_tok(const LmHeadBatch &b, int64_t n)
{
    TokInfo t;
    const int32_t s = b.seq_ids[n];
    t.seq_ok = (s >= 0 && (int64_t)s < b.S);
    const uint64_t seed = t.seq_ok ? b.seeds[s] : 0ull;
    t.key.k0 = (uint32_t)seed;
    t.key.k1 = (uint32_t)(seed >> 32);
    t.seq = (uint32_t)s;
    t.pos = b.positions[n];
    const float T = b.temperatures ? b.temperatures[n] : b.temperature;
    t.ok = t.seq_ok && (T > 0.0f) && (T < __builtin_inff());
    t.inv_T = t.ok ? 1.0f / T : 1.0f;
    const int32_t tg = b.claimed_gumbel ? b.claimed_gumbel[n] : -1;
    const int32_t ti = b.claimed_ipt ? b.claimed_ipt[n] : -1;
    t.tg = (tg >= 0 && (int64_t)tg < b.V) ? tg : -1;
    t.ti = (ti >= 0 && (int64_t)ti < b.V) ? ti : -1;
    return t;
}

__device__ __forceinline__ uint32_t noise_word_of(const TokInfo &t, uint32_t stream, int32_t v)
{
    uint32_t r[4];
    noise_block(t.key, t.pos, t.seq, stream, (uint32_t)v >> 2, r);
    return (v & 3) == 0 ? r[0] : (v & 3) == 1 ? r[1] : (v & 3) == 2 ? r[2] : r[3];
}

// ---------------------------------------------------------------------------------
// Before the GEMM: a lower bound on each row's best perturbed score, from the Token-DiFR claim.
// For an honest claim the claimed token IS the row maximum, so almost every other entry can be
// ruled out by its noise word alone.  The claimed logit is a plain fp32 dot product here; it
// differs from the matrix-core value of the same logit by accumulation order only, and the bound
// is lowered by a rigorous estimate of that difference, so it never exceeds the true maximum.
// One wave per token.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void lmhead_prepare_kernel(LmHeadBatch b, LmHeadWorkspace ws)
{
    const int lane = threadIdx.x & 63;
    const int64_t n = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (n >= b.N) return;  // uniform per wave
    const TokInfo t = load_tok(b, n);
    float L0 = -__builtin_inff(), x_ref = __builtin_nanf("");
    if (t.ok && t.tg >= 0) {
        const uint16_t *h = b.hidden + n * b.ldh;
        const uint16_t *w = b.weight + (int64_t)t.tg * b.ldw;
        float dot = 0.0f, mag = 0.0f;
        auto add = [&](const uint4 &hv, const uint4 &wv) {
            const uint32_t hw[4] = {hv.x, hv.y, hv.z, hv.w}, ww[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float h0 = __uint_as_float(hw[j] << 16), h1 = __uint_as_float(hw[j] & 0xFFFF0000u);
                const float w0 = __uint_as_float(ww[j] << 16), w1 = __uint_as_float(ww[j] & 0xFFFF0000u);
                dot = __fmaf_rn(h0, w0, dot);
                dot = __fmaf_rn(h1, w1, dot);
                mag = __fmaf_rn(fabsf(h0), fabsf(w0), mag);
                mag = __fmaf_rn(fabsf(h1), fabsf(w1), mag);
            }
        };
        const int64_t nc = b.d / 8;
        int64_t c = lane;
        for (; c + 64 * 7 < nc; c += 64 * 8) {  // sixteen loads in flight: a wave has nothing else to hide their latency
            uint4 hv[8], wv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                hv[i] = *reinterpret_cast<const uint4 *>(h + 8 * (c + 64 * i));
                wv[i] = *reinterpret_cast<const uint4 *>(w + 8 * (c + 64 * i));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) add(hv[i], wv[i]);
        }
        for (; c < nc; c += 64) add(*reinterpret_cast<const uint4 *>(h + 8 * c), *reinterpret_cast<const uint4 *>(w + 8 * c));
        dot = wave_sum(dot);
        mag = wave_sum(mag);
        x_ref = dot;
        const float y = perturbed_score(dot, t.inv_T, noise_word_of(t, kStreamGumbel, t.tg));
        // any two fp32 summation orders of d products differ by at most ~2 d 2^-24 sum|h w|; twice that here
        const float slack = 1e-3f + 1e-5f * fabsf(y) + t.inv_T * mag * (float)b.d * 0x1p-22f;
        L0 = y - slack;
        if (!(L0 == L0) || !(L0 < __builtin_inff())) L0 = -__builtin_inff();
    }
    if (lane == 0) {
        ws.L0[n] = L0;
        ws.x_claim_ref[n] = x_ref;
        ws.x_claim_gumbel[n] = __builtin_nanf("");
        ws.x_claim_ipt[n] = __builtin_nanf("");
    }
}

// ---------------------------------------------------------------------------------
// Per-lane, per-token running state of the epilogue.
// ---------------------------------------------------------------------------------
// The exponent a partial softmax sum with reference logit m is taken against: terms are 2^(x c - ref_exp(m, c)).  A
// whole number, so that moving a sum from one reference to another is a multiplication by an exact power of two
// and the many partial sums of a token (lanes, half tiles, vocabulary ranges) stay consistent to the last bit;
// with m c itself, rounded, every partial sum would sit on a reference that is off by the rounding of ITS product -
// 1e-6 and more once |m| / T reaches a few tens.
__device__ __forceinline__ float ref_exp(float m, float c) { return ceilf(m * c); }

struct Slot {
    float best_y;
    int32_t best_v;
    float L;      // lower bound on the row's best score: max(bound from the claim, best seen by this lane)
    float m;      // largest logit seen by this lane for this token
    double Z, P;  // sum of 2^((x - m) c) over all entries seen / over those below the IPT claim
    uint32_t above;  // RANK: entries seen whose logit exceeds the reference value of the Token-DiFR claim's
};

// Noise gate: an entry with noise word r < rgate cannot reach L whatever its logit (all logits seen
// are <= m).  g(r) <= c  <=>  u(r) <= exp(-exp(-c)); the threshold is lowered by 64 cells of the 23-bit
// uniform, far more than the fp32 error of the two exponentials.  Anything doubtful gives 0 (no skipping).
__device__ __forceinline__ uint32_t noise_gate(float L, float cap)
{
    const float c = L - cap - (0.01f + 1e-5f * (fabsf(L) + fabsf(cap)));
    const float t = fast_exp2(-c * kLog2e);
    const float kf = fast_exp2(-t * kLog2e) * 0x1p23f;
    const uint32_t kg = (kf > 64.0f) ? (uint32_t)kf - 64u : 0u;
    return kg << 9;
}

struct BlockCtx {
    const TokInfo &t;
    float c;       // log2(e) / T
    float neg_mc;  // -ref_exp(m, c)
    float Lgate;   // L minus slack
    uint32_t rgate;
    bool live;     // the lane's token row exists (n < N)
    float x_ref;   // RANK: the Token-DiFR claim's logit as a plain dot product (NaN: no claim, nothing counts)
};

__device__ __forceinline__ void refresh_gates(const Slot &s, BlockCtx &k)
{
    k.Lgate = s.L - (0.01f + 1e-5f * fabsf(s.L));
    k.rgate = noise_gate(s.L, s.m * k.t.inv_T);
}

// Score one 32x32 accumulator block: this lane's 16 entries are the logits of ONE token at
// vocabulary rows v(r) = vlane + 8 (r / 4) + (r % 4).
//
// RANK: also count the entries whose logit exceeds the Token-DiFR claim's (logit rank, Sec. 7.1).  The claim's
// logit must be known before the first tile, so the count is made against its plain fp32 dot product from the
// preparation kernel; the claimed entry itself is left out by index (its matrix-core value may differ from that
// reference in the last bits).
//
// TOK: `part` follows the mass of the half tile the block belongs to, relative to the slot's reference.
//
// AGPR: the accumulators are kept in the accumulation registers.
template <bool RANK, bool TOK, bool AGPR>
__device__ __forceinline__ void score_block(const f32x16 acc, Slot &s, BlockCtx &k, int32_t vlane, int32_t V,
                                            bool ragged, int64_t n, const LmHeadWorkspace &ws, double &part)
{
    const float ninf = -__builtin_inff();
    // the accumulators live in the accumulation registers; fetch them one by one (left to itself the
    // register allocator moves whole blocks through scratch memory instead)
    float x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if constexpr (AGPR)
            asm("v_accvgpr_read_b32 %0, %1" : "=v"(x[r]) : "a"(acc[r]));
        else
            x[r] = acc[r];
    }
    if (ragged) {  // uniform: the tile runs past the end of the vocabulary
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (vlane + 8 * (r >> 2) + (r & 3) >= V) x[r] = ninf;
    }
    if (RANK) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s.above += (uint32_t)(x[r] > k.x_ref);  // rows past V are -inf, a NaN counts nothing
    }
    // ---- Token-IPT-DiFR: online softmax sums ----
    float bm = max3_raw(x[0], x[1], x[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) bm = max3_raw(bm, x[r], x[r + 1]);
    bm = fmaxf(bm, x[15]);
    if (__builtin_amdgcn_ballot_w64(bm > s.m) != 0ull) {
        asm volatile("" ::: "memory");  // keep this a real, rarely taken branch
        if (bm > s.m) {
            const double f = (s.m > ninf) ? (double)fast_exp2(ref_exp(s.m, k.c) - ref_exp(bm, k.c)) : 0.0;
            s.Z *= f;
            s.P *= f;
            if (TOK) part *= f;
            s.m = bm;
            k.neg_mc = -ref_exp(bm, k.c);
            refresh_gates(s, k);  // the logit cap of the noise gate has moved
        }
    }
    float e[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) e[r] = fast_exp2(__fmaf_rn(x[r], k.c, k.neg_mc));
    if (ragged) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (vlane + 8 * (r >> 2) + (r & 3) >= V) e[r] = 0.0f;
    }
    const float bs = tree_sum<16>(e);
    float ps = (vlane + 27 < k.t.ti) ? bs : 0.0f;  // all 16 rows lie below the IPT claim
    // a claimed token inside this lane's rows: exact prefix, and keep the claimed logits (rare)
    const bool near = (uint32_t)(k.t.ti - vlane) < 28u || (uint32_t)(k.t.tg - vlane) < 28u;
    if (__builtin_amdgcn_ballot_w64(near) != 0ull) {
        asm volatile("" ::: "memory");
        if (near) {
            const bool straddle = (uint32_t)(k.t.ti - vlane) < 28u;
            if (straddle) ps = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int32_t v = vlane + 8 * (r >> 2) + (r & 3);
                if (straddle && v < k.t.ti) ps += e[r];
                if (k.live && v == k.t.ti) ws.x_claim_ipt[n] = x[r];
                if (k.live && v == k.t.tg) ws.x_claim_gumbel[n] = x[r];
                if (RANK && v == k.t.tg && x[r] > k.x_ref) s.above -= 1u;  // the claim does not outrank itself
            }
        }
    }
    s.Z += (double)bs;
    s.P += (double)ps;
    if (TOK) part += (double)bs;

    // ---- Token-DiFR: noise for all 16 entries, exact score only where the gates allow ----
    uint32_t rw[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) noise_block(k.t.key, k.t.pos, k.t.seq, kStreamGumbel, (uint32_t)(vlane + 8 * g) >> 2, rw + 4 * g);
    uint32_t rmax = rw[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) rmax = max(rmax, rw[r]);
    if (__builtin_amdgcn_ballot_w64(rmax >= k.rgate) != 0ull) {
        asm volatile("" ::: "memory");
        if (rmax >= k.rgate) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int32_t v = vlane + 8 * (r >> 2) + (r & 3);
                if (rw[r] >= k.rgate && !(ragged && v >= V) &&
                    !(__fmaf_rn(x[r], k.t.inv_T, gumbel_upper_bound(rw[r])) < k.Lgate)) {
                    const float y = perturbed_score(x[r], k.t.inv_T, rw[r]);
                    if (y > s.best_y || (y == s.best_y && v < s.best_v)) {
                        s.best_y = y;
                        s.best_v = v;
                    }
                }
            }
            if (s.best_y > s.L) {
                s.L = s.best_y;
                refresh_gates(s, k);
            }
        }
    }
}

__device__ __forceinline__ void merge_softmax(float &m, double &Z, double &P, float om, double oZ, double oP, float c)
{
    const float ninf = -__builtin_inff();
    const float M = fmaxf(m, om);
    const double f = (m > ninf) ? (double)fast_exp2(ref_exp(m, c) - ref_exp(M, c)) : 0.0;
    const double of = (om > ninf) ? (double)fast_exp2(ref_exp(om, c) - ref_exp(M, c)) : 0.0;
    Z = Z * f + oZ * of;
    P = P * f + oP * of;
    m = M;
}

// ---------------------------------------------------------------------------------
// The GEMM + epilogue kernel.  256 threads = 4 waves in a 2 (vocabulary) x 2 (tokens) arrangement;
// each wave owns a 128 x 128 sub-tile = 4 x 4 accumulator blocks of 32 x 32.
// LDS: two stages of [256 rows][64 k] bf16 for each operand; the eight 16-byte chunks of a row are
// permuted by (row / 2) % 8 so that both the 16-byte slab writes and the fragment reads of 16
// consecutive rows spread over all 64 banks.
// ---------------------------------------------------------------------------------
//
// TOK: also leave, per token and half tile (the 128 vocabulary entries of a tile that one wave scores), the softmax
// mass of that half tile with its exponent reference.  The sampler's own Token-IPT-DiFR token is the first entry
// at which the CDF passes u; the CDF needs the row's total mass, known only after the last tile, so the search is
// made afterwards: over these masses for the half tile, and inside it by forming its 128 logits again.
template <bool RANK, bool TOK>
__global__ __launch_bounds__(kBlock, 1) void lmhead_score_kernel(LmHeadBatch b, LmHeadWorkspace ws, LmHeadPlan plan)
{
    __shared__ __attribute__((aligned(16))) uint16_t lds_w[2][kLmTileV * kLmTileK];  // 32 KB per stage
    __shared__ __attribute__((aligned(16))) uint16_t lds_h[2][kLmTileT * kLmTileK];
    // per-token constants of the workgroup's 256 token rows (one wave per SIMD cannot hide a global load
    // in the epilogue, an LDS read it can): key, position, sequence, 1/T, the two claims
    __shared__ uint32_t lds_tok[RANK ? 8 : 7][kLmTileT];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wv = wave >> 1, wt = wave & 1;  // vocabulary half, token half
    const int l32 = lane & 31, lh = lane >> 5;

    // Workgroup -> (token block, vocabulary range).  Consecutive workgroup ids go to different XCDs;
    // remap so that each XCD works on a compact set of token blocks across all ranges and its L2
    // sees each weight tile and each hidden-state tile from several workgroups at about the same time.
    const int G = plan.n_tb * plan.splits;
    int q = blockIdx.x;
    if (G % 8 == 0) q = (q % 8) * (G / 8) + q / 8;
    const int tb = q / plan.splits, sp = q % plan.splits;
    const int vt0 = (int)((int64_t)sp * plan.n_vt / plan.splits), vt1 = (int)((int64_t)(sp + 1) * plan.n_vt / plan.splits);
    const int64_t n0 = (int64_t)tb * kLmTileT;
    const int32_t V = (int32_t)b.V;
    const int nk = (int)(b.d / kLmTileK);

    // Slab copy, global memory straight into LDS (no registers in between): a slab is 256 rows x 64 k of
    // each operand, i.e. whole 128-byte lines.  One wave-wide 16-byte-per-lane load fills 1 KB of LDS in
    // lane order = 8 rows; lane i lands in 16-byte position i % 8 of row i / 8, so it fetches the k chunk
    // that the permutation of the LDS layout puts there.  Thread -> rows (tid / 8) + 32 p, p = 0 .. 7.
    const int crow = tid >> 3;
    const int cchunk = (tid & 7) ^ ((crow >> 1) & 7);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    // Addresses are a wave-uniform base (scalar registers, moved by scalar arithmetic) plus a 32-bit
    // per-lane byte offset that never changes, so a load costs no vector arithmetic.
    uint32_t hoff[8];  // hidden-state rows: offset from the first row of the token block
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        int64_t r = crow + 32 * p;
        if (n0 + r > b.N - 1) r = b.N - 1 - n0;
        hoff[p] = (uint32_t)(r * b.ldh + cchunk * 8) * 2u;
    }
    const char *const hbase = reinterpret_cast<const char *>(b.hidden + n0 * b.ldh);
    const uint32_t wrow_bytes = (uint32_t)b.ldw * 2u;
    uint32_t woff[8];  // weight rows: offset from the first row of the vocabulary tile
    // rows past the end of the vocabulary (last tile only) re-read the last row
    auto set_woff = [&](int vt) {
        const int64_t tile_v0 = (int64_t)vt * kLmTileV;
        const int32_t last = (int32_t)((b.V - tile_v0 < kLmTileV ? b.V - tile_v0 : kLmTileV) - 1);  // uniform
#pragma unroll
        for (int p = 0; p < 8; ++p) woff[p] = (uint32_t)min(crow + 32 * p, last) * wrow_bytes + (uint32_t)cchunk * 16u;
    };
    set_woff(vt0);
    // load cursor: the next slab to fetch is slab l_kt of vocabulary tile l_vt; once past the end it stays
    // on the last tile (harmless reloads keep the loop free of special cases)
    int l_vt = vt0, l_kt = 0;
    auto advance_cursor = [&]() {
        const bool wrap = (l_kt + 1 == nk);
        l_kt = wrap ? 0 : l_kt + 1;
        if (wrap && l_vt + 1 < vt1) {
            ++l_vt;
            if ((int64_t)(l_vt + 1) * kLmTileV > b.V) set_woff(l_vt);  // the ragged tile, at most once
        }
    };
    // Chunk i (0-7: weight rows, 8-15: hidden-state rows) of the cursor's slab -> LDS stage buf.
    // The register M0 carries the LDS address of lane 0; lane i writes 16 i bytes further on.  Written as
    // assembly for two reasons: the compiler would make every later LDS read wait for the copies in flight (it
    // cannot tell the stages apart; the waits are placed by hand, see copies_landed), and a wave that runs
    // alone on its SIMD can issue only a handful of instructions between two matrix instructions, so a copy
    // must cost no address arithmetic: scalar base, invariant lane offset, M0 = stage base + constant.
    auto copy_chunk = [&](auto I, int buf) {
        constexpr int i = decltype(I)::value;
        const char *sbase = i < 8 ? reinterpret_cast<const char *>(b.weight + (int64_t)l_vt * kLmTileV * b.ldw + l_kt * kLmTileK)
                                  : hbase + (size_t)l_kt * (kLmTileK * 2);
        const uint32_t voff = i < 8 ? woff[i & 7] : hoff[i & 7];
        const uint16_t *stage = (i < 8 ? &lds_w[buf][0] : &lds_h[buf][0]) + 8 * wave_u * kLmTileK;
        const uint32_t lds_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)stage;
        // (M0 is set and consumed inside the one statement and declared clobbered; the compiler's remark that
        // it is a reserved register does not apply to that use)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
        asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
                     :
                     : "s"(sbase), "v"(voff), "s"(lds_base), "n"(32 * (i & 7) * kLmTileK * 2)
                     : "memory", "m0", "scc");
#pragma clang diagnostic pop
    };
    // every copy this wave has issued has landed in LDS, and every LDS read it has issued is complete
    auto copies_landed = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // fragment reads: lane -> row l32 of a 32-row block, 16-byte k chunk 2 kk + lh (permuted like the copy)
    const int sw = (l32 >> 1) & 7;
    const int a_row_off = (wv * 128 + l32) * kLmTileK;
    const int b_row_off = (wt * 128 + l32) * kLmTileK;
    struct Frag {
        bf16x8 a[4], b[4];
    };
    // fragment i (0-3: weight blocks, 4-7: hidden-state blocks) of k step kk from LDS stage buf
    auto read_frag = [&](Frag &f, int i, int buf, int kk) {
        const int coff = ((2 * kk + lh) ^ sw) * 8;
        if (i < 4)
            f.a[i] = *reinterpret_cast<const bf16x8 *>(&lds_w[buf][a_row_off + i * 32 * kLmTileK + coff]);
        else
            f.b[i - 4] = *reinterpret_cast<const bf16x8 *>(&lds_h[buf][b_row_off + (i - 4) * 32 * kLmTileK + coff]);
    };

    {
        int64_t n = n0 + tid;
        if (n > b.N - 1) n = b.N - 1;
        const TokInfo t = load_tok(b, n);
        lds_tok[0][tid] = t.key.k0;
        lds_tok[1][tid] = t.key.k1;
        lds_tok[2][tid] = t.pos;
        lds_tok[3][tid] = t.seq;
        lds_tok[4][tid] = __float_as_uint(t.inv_T);
        lds_tok[5][tid] = (uint32_t)t.tg;
        lds_tok[6][tid] = (uint32_t)t.ti;
        if (RANK) lds_tok[7][tid] = __float_as_uint(ws.x_claim_ref[n]);
    }
    auto tok_from_lds = [&](int i) {
        TokInfo t;
        t.key.k0 = lds_tok[0][i];
        t.key.k1 = lds_tok[1][i];
        t.pos = lds_tok[2][i];
        t.seq = lds_tok[3][i];
        t.inv_T = __uint_as_float(lds_tok[4][i]);
        t.tg = (int32_t)lds_tok[5][i];
        t.ti = (int32_t)lds_tok[6][i];
        t.ok = t.seq_ok = true;  // not used by the epilogue
        return t;
    };

    // per-lane state of the lane's four tokens
    Slot slot[4];
    const int64_t tok_first = n0 + wt * 128 + l32;  // the lane's tokens are tok_first + 32 jb
    auto tok_row = [&](int jb) { return tok_first + 32 * jb < b.N ? tok_first + 32 * jb : b.N - 1; };
    auto tok_is_live = [&](int jb) { return tok_first + 32 * jb < b.N; };
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
        const int64_t n = tok_row(jb);
        slot[jb].best_y = -__builtin_inff();
        slot[jb].best_v = 0x7FFFFFFF;
        slot[jb].L = ws.L0[n];
        slot[jb].m = -__builtin_inff();
        slot[jb].Z = 0.0;
        slot[jb].P = 0.0;
        slot[jb].above = 0u;
    }

    // ---- main loop ----
    // One wave per SIMD: nothing else hides latency, so copies and fragment reads are interleaved with the
    // matrix instructions by hand and the order is pinned with scheduling fences.  Per 64-deep slab, four
    // k steps of 16 MFMAs each:
    //   steps 0-1: + fragment reads for the next step, + the rest of the copies of the next slab
    //   step 2:    + fragment reads for step 3
    //   wait for this wave's copies, barrier
    //   step 3:    + fragment reads for step 0 of the next slab (from the other LDS stage), + the first copies
    //              of the slab after that into the stage just released
    f32x16 acc[4][4];
    Frag F0, F1;
    auto kstep = [&](const Frag &cur, Frag &nxt, int buf_next, int kk_next, auto READ, auto &&extra) {
        static_for<8>([&](auto I) {
            constexpr int i = decltype(I)::value, e0 = 2 * i, e1 = 2 * i + 1;
            acc[e0 >> 2][e0 & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[e0 >> 2], cur.b[e0 & 3], acc[e0 >> 2][e0 & 3], 0, 0, 0);
            extra(std::integral_constant<int, e0>());
            acc[e1 >> 2][e1 & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[e1 >> 2], cur.b[e1 & 3], acc[e1 >> 2][e1 & 3], 0, 0, 0);
            extra(std::integral_constant<int, e1>());
            if (decltype(READ)::value) read_frag(nxt, i, buf_next, kk_next);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    int par = 0;  // LDS stage of the slab being multiplied
    // Two LDS stages.  The stage of slab g is last read during its third k step (fragments are read one
    // step ahead), so after the barrier that follows that step it is free until the same barrier of slab
    // g + 1, and the 16 copies of slab g + 2 are issued into it during the fourth step of slab g and the
    // first two of slab g + 1 (copy_at_slot).  Each wave waits for its own copies before the barrier of
    // slab g + 1; the last of them has had a whole k step to land by then.  The LAST slab of a tile does
    // not read fragments ahead, so the epilogue has those 64 registers for itself.
    const std::true_type yes;
    const std::false_type no;
    // the copy (if any) that goes out at slot E of phase PH (0: fourth k step, 1 and 2: first and second of the next slab)
    auto cp = [&](auto PH, int buf) {
        return [&, buf](auto E) {
            constexpr int c = copy_at_slot(16 * decltype(PH)::value + decltype(E)::value);
            if constexpr (c >= 0) copy_chunk(std::integral_constant<int, c>(), buf);
        };
    };
    auto slab = [&](auto LAST) {
        kstep(F0, F1, par, 1, yes, cp(std::integral_constant<int, 1>(), par ^ 1));
        kstep(F1, F0, par, 2, yes, cp(std::integral_constant<int, 2>(), par ^ 1));
        advance_cursor();
        kstep(F0, F1, par, 3, yes, [&](auto) {});
        copies_landed();
        barrier();
        if (decltype(LAST)::value)
            kstep(F1, F0, par ^ 1, 0, no, cp(std::integral_constant<int, 0>(), par));
        else
            kstep(F1, F0, par ^ 1, 0, yes, cp(std::integral_constant<int, 0>(), par));
        par ^= 1;
    };

    // prologue: slab 0 whole, and of slab 1 what the fourth k step of a slab before it would have issued
    static_for<16>([&](auto I) { copy_chunk(I, 0); });
    advance_cursor();
    static_for<16>([&](auto E) { cp(std::integral_constant<int, 0>(), 1)(E); });
    copies_landed();
    __syncthreads();

    for (int vt = vt0; vt < vt1; ++vt) {
        const int64_t v0 = (int64_t)vt * kLmTileV;
        const f32x16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ib = 0; ib < 4; ++ib)
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) acc[ib][jb] = zero;
#pragma unroll
        for (int i = 0; i < 8; ++i) read_frag(F0, i, par, 0);
        for (int kt = 1; kt < nk; ++kt) slab(no);
        slab(yes);

        // ---- epilogue: score the 256 x 256 logits of this tile ----
        const bool ragged = v0 + kLmTileV > b.V;
        // (explicit instantiation per block: the accumulator indices must be compile-time constants)
        auto score_token = [&](auto JB) {
            constexpr int jb = decltype(JB)::value;
            const TokInfo t = tok_from_lds(wt * 128 + jb * 32 + l32);
            BlockCtx k{t, t.inv_T * kLog2e, 0.0f, 0.0f, 0u, tok_is_live(jb),
                       RANK ? __uint_as_float(lds_tok[RANK ? 7 : 0][wt * 128 + jb * 32 + l32]) : 0.0f};
            k.neg_mc = (slot[jb].m > -__builtin_inff()) ? -ref_exp(slot[jb].m, k.c) : 0.0f;
            refresh_gates(slot[jb], k);
            const int32_t vl = (int32_t)v0 + wv * 128 + 4 * lh;
            double part = 0.0;  // TOK: what this lane's 64 entries of the half tile add to its sum
            score_block<RANK, TOK, true>(acc[0][jb], slot[jb], k, vl, V, ragged, tok_row(jb), ws, part);
            score_block<RANK, TOK, true>(acc[1][jb], slot[jb], k, vl + 32, V, ragged, tok_row(jb), ws, part);
            score_block<RANK, TOK, true>(acc[2][jb], slot[jb], k, vl + 64, V, ragged, tok_row(jb), ws, part);
            score_block<RANK, TOK, true>(acc[3][jb], slot[jb], k, vl + 96, V, ragged, tok_row(jb), ws, part);
            if (TOK) {
                // the two lanes that share the token (rows 0-3 and 4-7 mod 8) combined
                const float ninf = -__builtin_inff();
                const float ms = (float)part, mm = slot[jb].m;
                const float os = __shfl_xor(ms, 32, 64), om = __shfl_xor(mm, 32, 64);
                const float M = fmaxf(mm, om);
                const float both = (mm > ninf ? ms * fast_exp2(ref_exp(mm, k.c) - ref_exp(M, k.c)) : 0.0f) +
                                   (om > ninf ? os * fast_exp2(ref_exp(om, k.c) - ref_exp(M, k.c)) : 0.0f);
                if (lh == 0 && tok_is_live(jb)) ws.half_sum[(int64_t)(2 * vt + wv) * b.N + tok_row(jb)] = make_float2(both, M);
            }
        };
        score_token(std::integral_constant<int, 0>());
        score_token(std::integral_constant<int, 1>());
        score_token(std::integral_constant<int, 2>());
        score_token(std::integral_constant<int, 3>());
    }

    // ---- merge the four lanes/waves that share a token and write this range's partial ----
    float *ex_y = reinterpret_cast<float *>(&lds_w[0][0]);  // [2][128] each, in the (now idle) tile memory
    int32_t *ex_v = reinterpret_cast<int32_t *>(ex_y + 256);
    float *ex_m = reinterpret_cast<float *>(ex_v + 256);
    double *ex_Z = reinterpret_cast<double *>(ex_m + 256);
    double *ex_P = ex_Z + 256;
    uint32_t *ex_a = reinterpret_cast<uint32_t *>(ex_P + 256);
    float tok_c[4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
        Slot &s = slot[jb];
        tok_c[jb] = __uint_as_float(lds_tok[4][wt * 128 + jb * 32 + l32]) * kLog2e;
        const float oy = __shfl_xor(s.best_y, 32, 64);
        const int32_t ov = __shfl_xor(s.best_v, 32, 64);
        const float om = __shfl_xor(s.m, 32, 64);
        const double oZ = __shfl_xor(s.Z, 32, 64), oP = __shfl_xor(s.P, 32, 64);
        if (RANK) s.above += (uint32_t)__shfl_xor((int)s.above, 32, 64);
        if (lh == 0) {  // rows 0-3 (mod 8) first, then rows 4-7: a fixed order
            argmax_combine(s.best_y, s.best_v, oy, ov);
            merge_softmax(s.m, s.Z, s.P, om, oZ, oP, tok_c[jb]);
        }
    }
    copies_landed();  // the tile memory is reused below: nothing may still be on its way into it
    __syncthreads();
    if (wv == 1 && lh == 0) {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            const int i = wt * 128 + jb * 32 + l32;
            ex_y[i] = slot[jb].best_y;
            ex_v[i] = slot[jb].best_v;
            ex_m[i] = slot[jb].m;
            ex_Z[i] = slot[jb].Z;
            ex_P[i] = slot[jb].P;
            if (RANK) ex_a[i] = slot[jb].above;
        }
    }
    __syncthreads();
    if (wv == 0 && lh == 0) {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            if (!tok_is_live(jb)) continue;
            Slot &s = slot[jb];
            const int i = wt * 128 + jb * 32 + l32;
            argmax_combine(s.best_y, s.best_v, ex_y[i], ex_v[i]);
            merge_softmax(s.m, s.Z, s.P, ex_m[i], ex_Z[i], ex_P[i], tok_c[jb]);
            const int64_t o = (int64_t)sp * b.N + tok_row(jb);
            ws.best_y[o] = s.best_y;
            ws.best_v[o] = s.best_v;
            ws.m[o] = s.m;
            ws.Z[o] = s.Z;
            ws.P[o] = s.P;
            if (RANK) ws.above[o] = (int32_t)(s.above + ex_a[i]);
        }
    }
}

// ---------------------------------------------------------------------------------
// The same for batches of up to 128 tokens.  What bounds them is reading the LM-head matrix once; the tile is as wide as the
// batch (T = 32, 64 or 128 token rows), so that the matrix instructions of a slab and its fragment reads take a fraction of the
// time its share of the memory bandwidth does.  A workgroup's four waves own 32 R vocabulary rows each, all token columns.
// S LDS stages, so that S - 1 slabs are in flight while one is multiplied, one barrier per slab:
//   wait for the wave's own copies of slab s (those of the slabs after it may be in flight), barrier: slab s is in LDS whole,
//   and every wave is done with slab s - 1, whose stage takes slab s + S - 1.
// R = 2: one workgroup to a compute unit, as many stages as fit; the hidden states that every slab of weights is multiplied
// with cross from the L2 once for 256 rows.  R = 1, for fewer tiles than compute units: up to 64 tokens two workgroups.
// Copies and LDS layout as in the kernel above; logits are summed in the same order, to the same bits.
// NT: the weights are read past the caches.  A matrix larger than the 256 MB Infinity Cache is never found there again and
// only displaces the hidden states: 1.24 GB, 64 tokens: 269 us for the call with ordinary loads, 247 with these (128-entry tiles); a matrix
// that fits is left to the cache (262 MB: 63 / 67 us, read again and again).  R = 1 always reads through the caches: 50,257 x 4096
// (412 MB), 64 tokens, would take 102 us past them instead of 111, but 33,000 x 4096 (270 MB) 95 instead of 78, the larger part of
// it being found in the cache.
// 64 tokens, V = 151,936, d = 4096: the scoring kernel alone takes 190 to 215 us, depending on the card, 5.8 to 6.5 TB/s (the 256 x 256
// kernel: 370).
// ---------------------------------------------------------------------------------
template <int T, int R, bool NT, bool RANK, bool TOK>
__global__ __launch_bounds__(kBlock, T <= 64 && R == 1 ? 2 : 1) void lmhead_small_kernel(LmHeadBatch b, LmHeadWorkspace ws, LmHeadPlan plan)
{
    constexpr int kRows = 128 * R, TB = T / 32, kStages = (T == 128 && R == 1) || (T == 32 && R == 2) ? 4 : 3;
    constexpr int kCopiesW = kRows / 32, kCopiesH = T / 32, kCopies = kCopiesW + kCopiesH;  // per wave and slab, 8 rows each
    __shared__ __attribute__((aligned(16))) uint16_t lds_w[kStages][kRows * kLmTileK];
    __shared__ __attribute__((aligned(16))) uint16_t lds_h[kStages][T * kLmTileK];
    __shared__ uint32_t lds_tok[RANK ? 8 : 7][T];
    __shared__ float2 lds_half[TOK ? kWaves : 1][T];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int sp = blockIdx.x;
    const int vt0 = (int)((int64_t)sp * plan.n_tiles / plan.splits), vt1 = (int)((int64_t)(sp + 1) * plan.n_tiles / plan.splits);
    const int32_t V = (int32_t)b.V;
    const int nk = (int)(b.d / kLmTileK);
    const int total = (vt1 - vt0) * nk;  // slabs

    const int crow = tid >> 3;
    const int cchunk = (tid & 7) ^ ((crow >> 1) & 7);
    uint32_t hoff[kCopiesH], woff[kCopiesW];
#pragma unroll
    for (int p = 0; p < kCopiesH; ++p) {
        int64_t r = crow + 32 * p;
        if (r > b.N - 1) r = b.N - 1;  // rows past the end of the batch re-read the last one
        hoff[p] = (uint32_t)(r * b.ldh + cchunk * 8) * 2u;
    }
    const uint32_t wrow_bytes = (uint32_t)b.ldw * 2u;
    auto set_woff = [&](int vt) {
        const int64_t tile_v0 = (int64_t)vt * kRows;
        const int32_t last = (int32_t)((b.V - tile_v0 < kRows ? b.V - tile_v0 : kRows) - 1);  // uniform
#pragma unroll
        for (int p = 0; p < kCopiesW; ++p) woff[p] = (uint32_t)min(crow + 32 * p, last) * wrow_bytes + (uint32_t)cchunk * 16u;
    };
    set_woff(vt0);
    int l_vt = vt0, l_kt = 0, l_stage = 0;  // the next slab to fetch and the stage it goes to
    auto copy_rows = [&](const char *sbase, uint32_t voff, const uint16_t *stage, auto P, auto PAST) {
        const uint32_t lds_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)stage;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
        if constexpr (decltype(PAST)::value)
            asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0 nt"
                         :
                         : "s"(sbase), "v"(voff), "s"(lds_base), "n"(32 * decltype(P)::value * kLmTileK * 2)
                         : "memory", "m0", "scc");
        else
            asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
                         :
                         : "s"(sbase), "v"(voff), "s"(lds_base), "n"(32 * decltype(P)::value * kLmTileK * 2)
                         : "memory", "m0", "scc");
#pragma clang diagnostic pop
    };
    auto fetch_slab = [&]() {
        const char *wbase = reinterpret_cast<const char *>(b.weight + (int64_t)l_vt * kRows * b.ldw + l_kt * kLmTileK);
        const char *hbase = reinterpret_cast<const char *>(b.hidden + l_kt * kLmTileK);
        const uint16_t *sw = &lds_w[l_stage][0] + 8 * wave_u * kLmTileK, *sh = &lds_h[l_stage][0] + 8 * wave_u * kLmTileK;
        static_for<kCopiesW>([&](auto P) { copy_rows(wbase, woff[decltype(P)::value], sw, P, std::integral_constant<bool, NT>()); });
        static_for<kCopiesH>([&](auto P) { copy_rows(hbase, hoff[decltype(P)::value], sh, P, std::false_type()); });
        l_stage = l_stage + 1 == kStages ? 0 : l_stage + 1;
        if (++l_kt == nk) {
            l_kt = 0;
            ++l_vt;
            if (l_vt < vt1 && (int64_t)(l_vt + 1) * kRows > b.V) set_woff(l_vt);  // the ragged tile, at most once
        }
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    for (int i = tid; i < T; i += kBlock) {
        const int64_t n = i < b.N ? i : b.N - 1;
        const TokInfo t = load_tok(b, n);
        lds_tok[0][i] = t.key.k0;
        lds_tok[1][i] = t.key.k1;
        lds_tok[2][i] = t.pos;
        lds_tok[3][i] = t.seq;
        lds_tok[4][i] = __float_as_uint(t.inv_T);
        lds_tok[5][i] = (uint32_t)t.tg;
        lds_tok[6][i] = (uint32_t)t.ti;
        if (RANK) lds_tok[7][i] = __float_as_uint(ws.x_claim_ref[n]);
    }
    Slot slot[TB];  // the lane's tokens are l32 + 32 jb
    auto tok_row = [&](int jb) { return (int64_t)(l32 + 32 * jb < b.N ? l32 + 32 * jb : b.N - 1); };
    auto tok_is_live = [&](int jb) { return l32 + 32 * jb < b.N; };
#pragma unroll
    for (int jb = 0; jb < TB; ++jb) slot[jb] = Slot{-__builtin_inff(), 0x7FFFFFFF, ws.L0[tok_row(jb)], -__builtin_inff(), 0.0, 0.0, 0u};
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();

    for (int i = 0; i < kStages - 1 && i < total; ++i) fetch_slab();
    const int sw = (l32 >> 1) & 7;
    int stage = 0, done = 0;  // stage of the next slab to multiply, slabs multiplied
    for (int vt = vt0; vt < vt1; ++vt) {
        const f32x16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        f32x16 acc[R][TB];
#pragma unroll
        for (int ib = 0; ib < R; ++ib)
#pragma unroll
            for (int jb = 0; jb < TB; ++jb) acc[ib][jb] = zero;
        for (int kt = 0; kt < nk; ++kt) {
            // (copies of one wave land in order, so with no more than the younger slabs' outstanding this slab has landed;
            // stores of the epilogue only make the wait stricter.  lgkmcnt: the fragments of slab s - 1 have been read.)
            if (kStages > 3 && done + 2 < total)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((kStages - 2) * kCopies) : "memory");
            else if (done + 1 < total)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kCopies) : "memory");
            else
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            barrier();
            if (done + kStages - 1 < total) fetch_slab();
#pragma unroll
            for (int kk = 0; kk < kLmTileK / 16; ++kk) {
                const int coff = ((2 * kk + lh) ^ sw) * 8;
                bf16x8 fa[R], fb[TB];
#pragma unroll
                for (int i = 0; i < R; ++i)
                    fa[i] = *reinterpret_cast<const bf16x8 *>(&lds_w[stage][(wave * 32 * R + i * 32 + l32) * kLmTileK + coff]);
#pragma unroll
                for (int j = 0; j < TB; ++j)
                    fb[j] = *reinterpret_cast<const bf16x8 *>(&lds_h[stage][(j * 32 + l32) * kLmTileK + coff]);
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
            }
            stage = stage + 1 == kStages ? 0 : stage + 1;
            ++done;
        }

        // ---- epilogue ----
        const int32_t v0 = vt * kRows;
        const bool ragged = (int64_t)v0 + kRows > b.V;
        // (explicit instantiation per block: the accumulator indices must be compile-time constants)
        static_for<TB>([&](auto JB) {
            constexpr int jb = decltype(JB)::value;
            const int i = jb * 32 + l32;
            TokInfo t;
            t.key.k0 = lds_tok[0][i];
            t.key.k1 = lds_tok[1][i];
            t.pos = lds_tok[2][i];
            t.seq = lds_tok[3][i];
            t.inv_T = __uint_as_float(lds_tok[4][i]);
            t.tg = (int32_t)lds_tok[5][i];
            t.ti = (int32_t)lds_tok[6][i];
            t.ok = t.seq_ok = true;  // not used by the epilogue
            BlockCtx k{t, t.inv_T * kLog2e, 0.0f, 0.0f, 0u, tok_is_live(jb), RANK ? __uint_as_float(lds_tok[RANK ? 7 : 0][i]) : 0.0f};
            k.neg_mc = (slot[jb].m > -__builtin_inff()) ? -ref_exp(slot[jb].m, k.c) : 0.0f;
            refresh_gates(slot[jb], k);
            double part = 0.0;
            static_for<R>([&](auto IB) {
                constexpr int ib = decltype(IB)::value;
                score_block<RANK, TOK, T == 128>(acc[ib][jb], slot[jb], k, v0 + (wave * R + ib) * 32 + 4 * lh, V, ragged, tok_row(jb), ws, part);
            });
            if (TOK) {
                const float ninf = -__builtin_inff();
                const float ms = (float)part, mm = slot[jb].m;
                const float os = __shfl_xor(ms, 32, 64), om = __shfl_xor(mm, 32, 64);
                const float M = fmaxf(mm, om);
                const float both = (mm > ninf ? ms * fast_exp2(ref_exp(mm, k.c) - ref_exp(M, k.c)) : 0.0f) +
                                   (om > ninf ? os * fast_exp2(ref_exp(om, k.c) - ref_exp(M, k.c)) : 0.0f);
                if (lh == 0) lds_half[wave][i] = make_float2(both, M);
            }
        });
        if (TOK) {
            // a half tile (128 entries) is the work of 4 / R waves
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            barrier();
            for (int i = tid; i < T * R; i += kBlock) {
                const int n = i % T, h = i / T;
                const float c = __uint_as_float(lds_tok[4][n]) * kLog2e, ninf = -__builtin_inff();
                float M = ninf, sum = 0.0f;
#pragma unroll
                for (int w = 0; w < kWaves / R; ++w) M = fmaxf(M, lds_half[h * (kWaves / R) + w][n].y);
#pragma unroll
                for (int w = 0; w < kWaves / R; ++w) {
                    const float2 p = lds_half[h * (kWaves / R) + w][n];
                    if (p.y > ninf) sum += p.x * fast_exp2(ref_exp(p.y, c) - ref_exp(M, c));
                }
                if (n < b.N) {
                    ws.half_sum[((int64_t)vt * R + h) * b.N + n] = make_float2(sum, M);
                    // (the merge reads an even number of half tiles)
                    if (R == 1 && vt + 1 == plan.n_tiles && (vt & 1) == 0) ws.half_sum[(int64_t)(vt + 1) * b.N + n] = make_float2(0.0f, ninf);
                }
            }
        }
    }

    // ---- merge the lanes and waves that share a token, in vocabulary-row order of the halves and waves ----
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();  // the tile memory is reused below
    float *ex_y = reinterpret_cast<float *>(&lds_w[0][0]);  // [kWaves][T] each
    int32_t *ex_v = reinterpret_cast<int32_t *>(ex_y + kWaves * T);
    float *ex_m = reinterpret_cast<float *>(ex_v + kWaves * T);
    double *ex_Z = reinterpret_cast<double *>(ex_m + 2 * kWaves * T);
    double *ex_P = ex_Z + kWaves * T;
    uint32_t *ex_a = reinterpret_cast<uint32_t *>(ex_P + kWaves * T);
    static_assert(kWaves * T * 36 <= (int)sizeof(lds_w), "the exchange fits the tile memory");
#pragma unroll
    for (int jb = 0; jb < TB; ++jb) {
        Slot &s = slot[jb];
        const int i = jb * 32 + l32;
        const float c = __uint_as_float(lds_tok[4][i]) * kLog2e;
        const float oy = __shfl_xor(s.best_y, 32, 64), om = __shfl_xor(s.m, 32, 64);
        const int32_t ov = __shfl_xor(s.best_v, 32, 64);
        const double oZ = __shfl_xor(s.Z, 32, 64), oP = __shfl_xor(s.P, 32, 64);
        if (RANK) s.above += (uint32_t)__shfl_xor((int)s.above, 32, 64);
        if (lh == 0) {
            argmax_combine(s.best_y, s.best_v, oy, ov);
            merge_softmax(s.m, s.Z, s.P, om, oZ, oP, c);
            ex_y[wave * T + i] = s.best_y;
            ex_v[wave * T + i] = s.best_v;
            ex_m[wave * T + i] = s.m;
            ex_Z[wave * T + i] = s.Z;
            ex_P[wave * T + i] = s.P;
            if (RANK) ex_a[wave * T + i] = s.above;
        }
    }
    __syncthreads();
    if (tid < T && tid < b.N) {
        const float c = __uint_as_float(lds_tok[4][tid]) * kLog2e;
        float best_y = ex_y[tid], m = ex_m[tid];
        int32_t best_v = ex_v[tid];
        double Z = ex_Z[tid], P = ex_P[tid];
        uint32_t above = RANK ? ex_a[tid] : 0u;
        for (int w = 1; w < kWaves; ++w) {
            argmax_combine(best_y, best_v, ex_y[w * T + tid], ex_v[w * T + tid]);
            merge_softmax(m, Z, P, ex_m[w * T + tid], ex_Z[w * T + tid], ex_P[w * T + tid], c);
            if (RANK) above += ex_a[w * T + tid];
        }
        const int64_t o = (int64_t)sp * b.N + tid;
        ws.best_y[o] = best_y;
        ws.best_v[o] = best_v;
        ws.m[o] = m;
        ws.Z[o] = Z;
        ws.P[o] = P;
        if (RANK) ws.above[o] = (int32_t)above;
    }
}

// ---------------------------------------------------------------------------------
// Merge the vocabulary ranges of each token and form every output.  A workgroup takes kFinTokens tokens (8, or 2 where a token has
// many ranges) with 256 / kFinTokens = G threads each: thread (t, g) reads the g-th 1/G of token t's ranges (and, for the sampler's
// token, of its half tiles), so that neighbouring lanes read neighbouring tokens of the [range][token] arrays and the loads of a
// token are spread over G threads.  What bounds it is the latency of those loads: with one thread per token walking all of them,
// the merge took 174 us of a call with 64 tokens (256 ranges) and 780 us with 4096 tokens and the sampler's token (16 ranges,
// 1188 half tiles); now 9 (two tokens to a workgroup; 15 with eight) and 34 us.
// ---------------------------------------------------------------------------------
template <int kFinTokens>
__global__ __launch_bounds__(kBlock) void lmhead_finalize_kernel(LmHeadBatch b, LmHeadWorkspace ws, int splits, int n_vt,
                                                                 GumbelOutputs og, IptOutputs oi)
{
    constexpr int kFinGroups = kBlock / kFinTokens;
    __shared__ float lds_y[kWaves][kFinTokens], lds_m[kWaves][kFinTokens];
    __shared__ int32_t lds_v[kWaves][kFinTokens], lds_a[kWaves][kFinTokens];
    __shared__ double lds_Z[kWaves][kFinTokens], lds_P[kWaves][kFinTokens];
    __shared__ double lds_mass[kFinGroups][kFinTokens];
    __shared__ int32_t lds_half[kFinTokens];

    const int tid = threadIdx.x, tk = tid % kFinTokens, g = tid / kFinTokens, wave = tid >> 6;
    const int64_t n = (int64_t)blockIdx.x * kFinTokens + tk;
    const bool live = n < b.N;
    const float nan = __builtin_nanf("");
    const float ninf = -__builtin_inff();
    const TokInfo t = load_tok(b, live ? n : b.N - 1);
    const bool use = live && t.ok;  // (threads without a row, or with a rejected one, only keep the barriers company)
    const float c = t.inv_T * kLog2e;

    // ---- the ranges: this thread's share in ascending order, then the 8 groups of the wave, then the 4 waves ----
    float best_y = ninf, m = ninf;
    int32_t best_v = 0x7FFFFFFF;
    double Z = 0.0, P = 0.0;
    int32_t above = 0;
    if (use) {
        const int sp1 = (int)((int64_t)(g + 1) * splits / kFinGroups);
#pragma unroll 4
        for (int sp = (int)((int64_t)g * splits / kFinGroups); sp < sp1; ++sp) {
            const int64_t o = (int64_t)sp * b.N + n;
            argmax_combine(best_y, best_v, ws.best_y[o], ws.best_v[o]);
            merge_softmax(m, Z, P, ws.m[o], ws.Z[o], ws.P[o], c);
            if (og.logit_rank) above += ws.above[o];
        }
    }
#pragma unroll
    for (int off = kFinTokens; off < 64; off <<= 1) {  // (references are whole exponents: merging is order-free but for fp64 rounding)
        const float oy = __shfl_xor(best_y, off, 64), om = __shfl_xor(m, off, 64);
        const int32_t ov = __shfl_xor(best_v, off, 64);
        const double oZ = __shfl_xor(Z, off, 64), oP = __shfl_xor(P, off, 64);
        above += __shfl_xor(above, off, 64);
        argmax_combine(best_y, best_v, oy, ov);
        merge_softmax(m, Z, P, om, oZ, oP, c);
    }
    if ((tid & 63) < kFinTokens) {
        lds_y[wave][tk] = best_y;
        lds_v[wave][tk] = best_v;
        lds_m[wave][tk] = m;
        lds_Z[wave][tk] = Z;
        lds_P[wave][tk] = P;
        lds_a[wave][tk] = above;
    }
    if (tid < kFinTokens) lds_half[tid] = -1;
    __syncthreads();
    best_y = lds_y[0][tk];
    best_v = lds_v[0][tk];
    m = lds_m[0][tk];
    Z = lds_Z[0][tk];
    P = lds_P[0][tk];
    above = lds_a[0][tk];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
        argmax_combine(best_y, best_v, lds_y[w][tk], lds_v[w][tk]);
        merge_softmax(m, Z, P, lds_m[w][tk], lds_Z[w][tk], lds_P[w][tk], c);
        above += lds_a[w][tk];
    }
    const bool ipt_bad = !(Z > 0.0) || !(Z < (double)__builtin_inff()) || !(m < __builtin_inff()) || !(m > ninf);
    const bool nonfinite = !(Z == Z) || !(Z < (double)__builtin_inff()) || !(m < __builtin_inff());

    // ---- Token-IPT-DiFR: the uniform and the claimed token's interval (in every thread of the token) ----
    uint32_t r[4];
    noise_block(t.key, t.pos, t.seq, kStreamIpt, 0u, r);
    const float u = uniform_from_bits(r[0]);
    float a = nan, bb = nan, dd = nan;
    double ad = 0.0, bd = 0.0;
    bool match = false;
    if (use && t.ti >= 0 && !ipt_bad) {
        const double et = (double)fast_exp2(__fmaf_rn(ws.x_claim_ipt[n], c, -ref_exp(m, c)));
        const double ud = (double)u;
        ad = P / Z;
        bd = (P + et) / Z;
        a = (float)ad;
        bb = (float)bd;
        dd = (float)fmax(fmax(ad - ud, ud - bd), 0.0);
        match = (ad <= ud) && (ud < bd);
    }

    // ---- the half tile that holds the sampler's own token: the claim's if it matches, else the first at which the
    // CDF passes u, from the masses the scoring pass left (vocabulary order, each brought to the row's final
    // reference).  Every thread sums its share of them, the share in which the CDF passes is found from the sums and
    // its thread walks it; the entry inside the half tile is found by the kernel that follows. ----
    if (oi.ipt_token) {
        const bool search = use && !ipt_bad && !match;
        const int h0 = (int)((int64_t)g * 2 * n_vt / kFinGroups), h1 = (int)((int64_t)(g + 1) * 2 * n_vt / kFinGroups);
        const float rm = ref_exp(m, c);
        // calls f(h, mass) for the thread's half tiles in order; eight loads in flight, f is a chain of additions
        auto for_each_mass = [&](auto &&f) {
            for (int h = h0; h < h1; h += 8) {
                float2 p[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) p[k] = ws.half_sum[(int64_t)min(h + k, h1 - 1) * b.N + n];
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (h + k < h1) f(h + k, p[k].x > 0.0f ? (double)p[k].x * (double)fast_exp2(ref_exp(p[k].y, c) - rm) : 0.0);
            }
        };
        double sum = 0.0;
        if (search) for_each_mass([&](int, double w) { sum += w; });
        lds_mass[g][tk] = sum;
        __syncthreads();
        if (search) {
            const double target = (double)u * Z;
            double cum = 0.0, before = 0.0;  // before: the mass below the share that is walked
            int share = -1;                  // the first at which the CDF passes u, else the last with any mass
            for (int k = 0; k < kFinGroups; ++k) {
                const double w = lds_mass[k][tk];
                if (w > 0.0) {
                    share = k;
                    before = cum;
                }
                cum += w;
                if (cum > target) break;
            }
            if (share == g) {
                double at = before, at_last = before;
                int32_t half = -1, last = -1;  // last half tile with any mass: where rounding puts a u beyond the sum
                for_each_mass([&](int h, double w) {
                    if (half >= 0) return;
                    if (w > 0.0) {
                        last = h;
                        at_last = at;
                    }
                    if (at + w > target) half = h;
                    at += w;
                });
                if (half < 0) half = last;
                lds_half[tk] = half;
                ws.cross_rest[n] = target - at_last;
                ws.final_m[n] = m;
            }
        }
        __syncthreads();
    }

    if (g != 0 || !live) return;  // one thread per token writes the outputs
    if (!t.ok) {
        const uint8_t f = (uint8_t)(t.seq_ok ? kFlagNonfinite : kFlagInvalidClaim);
        og.margin[n] = nan;
        og.argmax[n] = -1;
        if (og.max_score) og.max_score[n] = nan;
        if (og.claimed_score) og.claimed_score[n] = nan;
        og.flags[n] = f;
        if (og.logit_rank) og.logit_rank[n] = -1;
        oi.dist[n] = nan;
        if (oi.cdf_lo) oi.cdf_lo[n] = nan;
        if (oi.cdf_hi) oi.cdf_hi[n] = nan;
        if (oi.u) oi.u[n] = nan;
        if (oi.log_mass) oi.log_mass[n] = nan;
        if (oi.ipt_token) {
            oi.ipt_token[n] = -1;
            ws.cross_half[n] = -1;
        }
        oi.flags[n] = f;
        return;
    }
    if (best_v == 0x7FFFFFFF) best_v = 0;

    // Token-DiFR
    uint32_t fg = nonfinite ? kFlagNonfinite : 0u;
    float yt = nan, mg = nan;
    if (t.tg >= 0) {
        yt = perturbed_score(ws.x_claim_gumbel[n], t.inv_T, noise_word_of(t, kStreamGumbel, t.tg));
        mg = best_y - yt;
        if (best_v == t.tg) fg |= kFlagMatch;
    } else {
        fg |= kFlagInvalidClaim;
    }
    og.margin[n] = mg;
    og.argmax[n] = best_v;
    if (og.max_score) og.max_score[n] = best_y;
    if (og.claimed_score) og.claimed_score[n] = yt;
    og.flags[n] = (uint8_t)fg;
    if (og.logit_rank) og.logit_rank[n] = t.tg >= 0 ? above : -1;

    // Token-IPT-DiFR
    uint32_t fi = 0;
    if (t.ti < 0) fi |= kFlagInvalidClaim;
    if (ipt_bad) fi |= kFlagNonfinite;
    if (match) fi |= kFlagMatch;
    oi.dist[n] = dd;
    if (oi.cdf_lo) oi.cdf_lo[n] = a;
    if (oi.cdf_hi) oi.cdf_hi[n] = bb;
    if (oi.u) oi.u[n] = u;
    if (oi.log_mass)
        oi.log_mass[n] = (t.ti >= 0 && !ipt_bad) ? (float)gaussian_log_mass(ad, bd, (double)u, oi.sigma, oi.eps) : nan;
    if (oi.ipt_token) {
        const int32_t half = lds_half[tk];
        if (half >= 0) fi |= kFlagSlowPath;
        oi.ipt_token[n] = match ? t.ti : -1;
        ws.cross_half[n] = half;
    }
    oi.flags[n] = (uint8_t)fi;
}

// ---------------------------------------------------------------------------------
// The sampler's own Token-IPT-DiFR token inside the half tile the merge kernel found: its logits are formed again as
// plain fp32 dot products, 32 at a time in vocabulary order (eight per wave, a row of the LM-head matrix read by the
// whole wave), turned into softmax terms relative to the row's final reference and scanned for the first entry at which
// the running sum passes what was left to cover; the 32 that hold it are the last that are read.  One workgroup per
// token; tokens that are already known (matching or missing claims, rejected rows) leave at once.
// Bound by reading those rows (2 d bytes each, 80 of the 128 on average): N = 4096 tokens, V = 151936, d = 4096, 55% of
// them searched: 490 us when all 128 were formed before the scan, one row at a time; now 244.  Eight rows at a time keep
// nine loads in flight per lane.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void lmhead_ipt_token_kernel(LmHeadBatch b, LmHeadWorkspace ws, IptOutputs oi)
{
    constexpr int kRows = 8, kStep = kRows * kWaves;  // rows per wave and per workgroup at a time
    __shared__ float lds_e[2][kStep];                 // (two, so that a step's terms outlive the barrier of the next)
    const int64_t n = blockIdx.x;
    const int32_t half = ws.cross_half[n];
    if (half < 0) return;  // uniform
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TokInfo t = load_tok(b, n);
    const float c = t.inv_T * kLog2e, m = ws.final_m[n];
    const double rest = ws.cross_rest[n];
    const uint16_t *h = b.hidden + n * b.ldh;
    double before = 0.0;   // mass of the half tile's entries below this step
    int32_t last = 0;      // last entry with any mass: rounding may leave the rest uncovered
    for (int step = 0; step < 128 / kStep; ++step) {
        const int64_t v0 = (int64_t)half * 128 + step * kStep;
        float dot[kRows];
        const uint16_t *w[kRows];  // (rows past the end of the vocabulary re-read the last one; their terms are dropped)
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int64_t v = v0 + wave * kRows + k;
            dot[k] = 0.0f;
            w[k] = b.weight + (v < b.V ? v : b.V - 1) * b.ldw;
        }
        for (int64_t q = lane; q < b.d / 8; q += 64) {
            const uint4 hv = *reinterpret_cast<const uint4 *>(h + 8 * q);
            uint4 wv[kRows];
#pragma unroll
            for (int k = 0; k < kRows; ++k) wv[k] = *reinterpret_cast<const uint4 *>(w[k] + 8 * q);
            const uint32_t hw[4] = {hv.x, hv.y, hv.z, hv.w};
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const uint32_t ww[4] = {wv[k].x, wv[k].y, wv[k].z, wv[k].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    dot[k] = __fmaf_rn(__uint_as_float(hw[j] << 16), __uint_as_float(ww[j] << 16), dot[k]);
                    dot[k] = __fmaf_rn(__uint_as_float(hw[j] & 0xFFFF0000u), __uint_as_float(ww[j] & 0xFFFF0000u), dot[k]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            dot[k] = wave_sum(dot[k]);
            const float e = fast_exp2(__fmaf_rn(dot[k], c, -ref_exp(m, c)));
            if (lane == 0) lds_e[step & 1][wave * kRows + k] = (e == e) && v0 + wave * kRows + k < b.V ? e : 0.0f;
        }
        __syncthreads();
        // every wave scans the step's terms by itself (lanes 32 and up hold zeros): no second barrier
        const double e = lane < kStep ? (double)lds_e[step & 1][lane] : 0.0;
        double incl = e;
#pragma unroll
        for (int off = 1; off < kStep; off <<= 1) {
            const double o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        const uint64_t hit = __builtin_amdgcn_ballot_w64(e > 0.0 && before + incl > rest);
        const uint64_t mass = __builtin_amdgcn_ballot_w64(e > 0.0);
        if (mass != 0ull) last = step * kStep + 63 - __builtin_clzll(mass);
        if (hit != 0ull) {
            last = step * kStep + __builtin_ctzll(hit);
            break;  // uniform over the workgroup: every wave has scanned the same terms
        }
        before += __shfl(incl, kStep - 1, 64);
    }
    if (tid == 0) oi.ipt_token[n] = (int32_t)((int64_t)half * 128 + last);
}

int launch_lmhead_score(const LmHeadBatch &b, const LmHeadWorkspace &ws, const LmHeadPlan &plan, const GumbelOutputs &og,
                        const IptOutputs &oi, hipStream_t stream)
{
    lmhead_prepare_kernel<<<dim3((unsigned)((b.N + kWaves - 1) / kWaves)), dim3(kBlock), 0, stream>>>(b, ws);
    if (hipGetLastError() != hipSuccess) return 1;
    // the logit rank and the masses behind the sampler's own token are produced in the scoring pass, only when asked for
    const dim3 block(kBlock);
    const bool rank = og.logit_rank != nullptr, tok = oi.ipt_token != nullptr;
    auto score = [&](auto RANK, auto TOK) {
        constexpr bool r = decltype(RANK)::value, t = decltype(TOK)::value;
        const bool past = b.V * b.ldw * 2 > (int64_t)256 << 20;  // a weight matrix larger than the Infinity Cache
        const dim3 small_grid((unsigned)plan.splits);
        auto small = [&](auto TOKENS) {
            constexpr int T = decltype(TOKENS)::value;
            if (plan.blocks == 1)  // (also where the matrix is larger than the cache; see NT above)
                lmhead_small_kernel<T, 1, false, r, t><<<small_grid, block, 0, stream>>>(b, ws, plan);
            else if (past)
                lmhead_small_kernel<T, 2, true, r, t><<<small_grid, block, 0, stream>>>(b, ws, plan);
            else
                lmhead_small_kernel<T, 2, false, r, t><<<small_grid, block, 0, stream>>>(b, ws, plan);
        };
        if (plan.small == 32)
            small(std::integral_constant<int, 32>());
        else if (plan.small == 64)
            small(std::integral_constant<int, 64>());
        else if (plan.small == 128)
            small(std::integral_constant<int, 128>());
        else
            lmhead_score_kernel<r, t><<<dim3((unsigned)(plan.n_tb * plan.splits)), block, 0, stream>>>(b, ws, plan);
    };
    const std::true_type yes;
    const std::false_type no;
    if (rank && tok)
        score(yes, yes);
    else if (rank)
        score(yes, no);
    else if (tok)
        score(no, yes);
    else
        score(no, no);
    if (hipGetLastError() != hipSuccess) return 1;
    auto finalize = [&](auto TOKENS) {
        constexpr int per = decltype(TOKENS)::value;
        lmhead_finalize_kernel<per><<<dim3((unsigned)((b.N + per - 1) / per)), block, 0, stream>>>(b, ws, plan.splits, plan.n_vt, og, oi);
    };
    // (two tokens to a workgroup where a token has many ranges: 400 ranges, 64 tokens: 247 / 244 us for the call; the search
    // for the sampler's token walks a sum per group of threads, of which it is better to have fewer: V = 4000: 45 / 50 us)
    if (plan.small && plan.splits > 128 && !tok)
        finalize(std::integral_constant<int, 2>());
    else
        finalize(std::integral_constant<int, 8>());
    if (hipGetLastError() != hipSuccess) return 1;
    if (tok) {
        lmhead_ipt_token_kernel<<<dim3((unsigned)b.N), block, 0, stream>>>(b, ws, oi);
        if (hipGetLastError() != hipSuccess) return 1;
    }
    return 0;
}

}  // namespace difr
