// Shapes, launch plan and workspace layout of the fused LM-head scoring path, shared by the
// kernels (lmhead.hip) and the C ABI layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <initializer_list>

namespace difr {

constexpr int kLmTileV = 256;  // vocabulary entries per workgroup tile
constexpr int kLmTileT = 256;  // token rows per workgroup tile
constexpr int kLmTileK = 64;   // hidden-dimension slab staged through LDS per step
constexpr int64_t kLmSmallMost = 128;  // most tokens of the small-batch kernel

// Kernel-side image of difr_lmhead.
struct LmHeadBatch {
    const uint16_t *hidden;  // [N, ldh] bf16
    const uint16_t *weight;  // [V, ldw] bf16
    int64_t N, V, d, ldh, ldw;
    float temperature;
    const float *temperatures;
    const uint64_t *seeds;
    int64_t S;
    const int32_t *seq_ids;
    const uint32_t *positions;
    const int32_t *claimed_gumbel;
    const int32_t *claimed_ipt;
};

// How the [N, V] logit matrix is cut into workgroups: n_tb token blocks times `splits` contiguous
// ranges of vocabulary tiles.  Every workgroup walks its range tile by tile and leaves one partial
// result per token; a last kernel merges the `splits` partials of each token in vocabulary order.
struct LmHeadPlan {
    int n_tb;    // token blocks of kLmTileT rows
    int n_vt;    // vocabulary tiles of kLmTileV entries
    int splits;  // vocabulary ranges
    int small;   // token rows of the small-batch kernel's tile (32, 64 or 128), 0: the 256 x 256 kernel
    int blocks;  // small-batch kernel: blocks of 32 vocabulary entries per wave and tile (a tile has 128 entries for each)
    int n_tiles; // ... and how many such tiles there are
};

inline LmHeadPlan lmhead_plan(int64_t N, int64_t V)
{
    LmHeadPlan p;
    p.n_tb = (int)((N + kLmTileT - 1) / kLmTileT);
    p.n_vt = (int)((V + kLmTileV - 1) / kLmTileV);
    p.small = p.blocks = p.n_tiles = 0;
    // Up to 128 tokens the matrix instructions of the 256 x 256 tile are mostly padding and the LM-head matrix is read at
    // half the speed of memory (V = 151,936, d = 4096, whole call: 64 tokens 376 us, 207 with the small-batch kernel; 128
    // tokens 398 / 244; V = 32,000, d = 2048, 64 tokens: 75 / 39).  Tiles of 256 entries from 65,537 entries on, where there is one
    // for every compute unit (64 tokens, V = 151,936: 204 us, and 245 with 128-entry tiles, two workgroups to a compute unit, in the
    // same run), shorter ones below (V = 32,000, d = 2048: 39, 49 with the long ones).
    // Ranges have as many tiles each as the longest must have, even if fewer workgroups than compute units do it: V = 66,000 has 258
    // tiles, and 129 ranges of two take 133 / 142 / 163 us (16 / 64 / 128 tokens), 256 ranges of one or two 160 / 173 / 204; V =
    // 131,328 187 / 187 / 252 against 212 / 218 / 267, V = 151,936 209 / 218 / 259 against 222 / 235 / 271; where almost all ranges
    // are full the two agree (V = 128,256: 181 / 177 / 206 against 178 / 176 / 203; V = 50,257, 128 tokens: 126 / 123).
    if (N <= kLmSmallMost) {
        p.small = N <= 32 ? 32 : (N <= 64 ? 64 : 128);
        p.blocks = V > 256 * 256 ? 2 : 1;
        const int rows = 128 * p.blocks, most = p.blocks == 1 && p.small <= 64 ? 512 : 256;
        p.n_tiles = (int)((V + rows - 1) / rows);
        const int each = (p.n_tiles + most - 1) / most;
        p.splits = each > 0 ? (p.n_tiles + each - 1) / each : 1;
        return p;
    }
    // one workgroup per compute unit (256 of them) when the token blocks alone do not fill the chip
    int s = p.n_tb > 0 ? 256 / p.n_tb : 1;
    if (s < 1) s = 1;
    if (s > p.n_vt) s = p.n_vt;
    p.splits = s;
    return p;
}

// Device pointers into the caller's workspace.
struct LmHeadWorkspace {
    double *Z, *P;         // [splits][N]  softmax sums relative to m: all entries / entries below the IPT claim
    float *m;              // [splits][N]  largest logit seen
    float *best_y;         // [splits][N]  best perturbed score
    int32_t *best_v;       // [splits][N]  and its token
    int32_t *above;        // [splits][N]  entries whose logit exceeds the Token-DiFR claim's (logit rank; only if asked for)
    float *L0;             // [N] lower bound on the row's best perturbed score (-inf if none)
    float *x_claim_gumbel; // [N] logit of the Token-DiFR claim as the tile that holds it computed it (NaN until then)
    float *x_claim_ipt;    // [N] same for the Token-IPT-DiFR claim
    float *x_claim_ref;    // [N] logit of the Token-DiFR claim as a plain fp32 dot product (NaN without a claim)
    // only when the sampler's own Token-IPT-DiFR token is asked for (null otherwise):
    float2 *half_sum;      // [2 n_vt][N] softmax mass of each half tile (128 vocabulary entries) and its exponent reference
    double *cross_rest;    // [N] mass still to be covered inside the half tile in which the CDF passes u, relative to final_m
    float *final_m;        // [N] the row's final exponent reference
    int32_t *cross_half;   // [N] that half tile, or -1 if the token is already known
};

// want_token: room for the per-half-tile masses that the search for the sampler's own token needs
inline size_t lmhead_workspace_bytes(int64_t N, int splits, int n_vt = 0, bool want_token = false)
{
    size_t bytes = (size_t)N * (size_t)splits * (8 + 8 + 4 + 4 + 4 + 4) + (size_t)N * 16 + 64;
    if (want_token) bytes += (size_t)N * (size_t)n_vt * 16 + (size_t)N * 16;
    return bytes;
}

// The size the library names for a batch.  A smaller batch may be cut into more ranges (up to 512 instead of 256 up to 64 tokens),
// so its need can be the larger one; a caller that sizes once for its largest batch gets room for the smaller ones too.
inline size_t lmhead_workspace_named(int64_t N, int64_t V, bool want_token)
{
    size_t most = 0;
    for (const int64_t n : {N, N < 64 ? N : (int64_t)64, N < kLmSmallMost ? N : kLmSmallMost}) {
        const LmHeadPlan p = lmhead_plan(n, V);
        const size_t bytes = lmhead_workspace_bytes(n, p.splits, p.n_vt, want_token);
        if (bytes > most) most = bytes;
    }
    return most;
}

// A small batch in a smaller workspace is cut into fewer ranges, down to the 256 (or one per 256 entries) that the 256 x 256 kernel
// would take.  False: not enough for those either.
inline bool lmhead_fit(LmHeadPlan &p, int64_t N, size_t bytes, bool want_token)
{
    if (p.small) {
        const int least = p.n_vt < 256 ? p.n_vt : 256;
        while (p.splits > least && bytes < lmhead_workspace_bytes(N, p.splits, p.n_vt, want_token)) --p.splits;
    }
    return bytes >= lmhead_workspace_bytes(N, p.splits, p.n_vt, want_token);
}

inline LmHeadWorkspace lmhead_carve(void *base, int64_t N, int splits, int n_vt = 0, bool want_token = false)
{
    LmHeadWorkspace w;
    const size_t n = (size_t)N * (size_t)splits;
    char *p = (char *)base;
    w.Z = (double *)p;
    p += n * 8;
    w.P = (double *)p;
    p += n * 8;
    w.m = (float *)p;
    p += n * 4;
    w.best_y = (float *)p;
    p += n * 4;
    w.best_v = (int32_t *)p;
    p += n * 4;
    w.above = (int32_t *)p;
    p += n * 4;
    w.L0 = (float *)p;
    p += (size_t)N * 4;
    w.x_claim_gumbel = (float *)p;
    p += (size_t)N * 4;
    w.x_claim_ipt = (float *)p;
    p += (size_t)N * 4;
    w.x_claim_ref = (float *)p;
    p += (size_t)N * 4;
    w.half_sum = nullptr;
    w.cross_rest = nullptr;
    w.final_m = nullptr;
    w.cross_half = nullptr;
    if (want_token) {
        p = (char *)(((uintptr_t)p + 7u) & ~(uintptr_t)7u);
        w.half_sum = (float2 *)p;
        p += (size_t)N * (size_t)n_vt * 16;
        w.cross_rest = (double *)p;
        p += (size_t)N * 8;
        w.final_m = (float *)p;
        p += (size_t)N * 4;
        w.cross_half = (int32_t *)p;
    }
    return w;
}

}  // namespace difr
