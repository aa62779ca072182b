// The adaptive-parallelism planner (host only).
//
// The paper's rule (Sec. 4.3): raise split-K until there are enough blocks to
// occupy every compute unit ("parallelism priority"), keep the splits aligned
// with the matrix instruction's k granularity and the reduction overhead
// predictable ("controlled reduction"), and fall back to less splitting when
// k is short.  On MI355X the measured sweep over every (tile, split_k) of the
// ViT/DeiT/Swin workloads shows that a split of the reduction across the
// four waves of one workgroup, merged in LDS, beats a split across
// workgroups merged through global memory at every shape tried, so the rules
// choose among output tiles and k-sliced tiles, by token count, output tile
// count and output width; split_k > 1 is available to explicit plans.
#include <hip/hip_runtime.h>

#include <mutex>

#include "nmspmm_internal.h"

namespace nmspmm {

static const int kSplitSet[] = {1, 2, 4, 8};

size_t split_workspace_bytes(int split_k, int m, int n) {
    if (split_k <= 1) return 0;
    return kCounterBytes + (size_t)split_k * (size_t)m * (size_t)n * 4;
}

// The expanded weight always starts past the counter block (also without
// split-K), so no plan ever writes over the counters another plan relies on.
size_t expand_offset(int split_k, int m, int n) {
    const size_t used = split_k > 1 ? split_workspace_bytes(split_k, m, n) : kCounterBytes;
    return (used + 255) & ~(size_t)255;
}

size_t workspace_bytes(const nm_plan &p, int m, int n) {
    if (!p.expand) return split_workspace_bytes(p.split_k, m, n);
    return expand_offset(p.split_k, m, n) + (size_t)p.expand_bytes;
}

int64_t expanded_bytes(int kind, int n, int k) {
    if (!kind_is_compact(kind)) return 0;
    const int64_t F = (n + kFragRows - 1) / kFragRows, S = (k + kKStep - 1) / kKStep;
    return kind_is_sp42(kind) ? F * S * (kVBlock + kMBlock) : (int64_t)n * k;
}

int device_cu_count() {
    static std::mutex mu;
    static int cached[64];
    static bool init = false;
    std::lock_guard<std::mutex> lock(mu);
    if (!init) {
        for (int &c : cached) c = 0;
        init = true;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return 256;
    }
    if (cached[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
            (void)hipGetLastError();
            cus = 256;
        }
        cached[dev] = cus;
    }
    return cached[dev];
}

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

nm_status complete_plan(int kind, int m, int n, int k, nm_plan *p) {
    if (!p || p->kind != kind || p->tile < 0 || p->tile >= kNumTiles) return NM_ERR_ARG;
    if (p->expand != 0 && (p->expand != 1 || !kind_is_compact(kind))) return NM_ERR_ARG;
    const int k_steps = (k + kKStep - 1) / kKStep;
    p->reserved = 0;
    p->expand_bytes = p->expand ? expanded_bytes(kind, n, k) : 0;
    if (p->expand_bytes >= kWeightLimit) return NM_ERR_SHAPE;
    bool ok_split = false;
    for (int s : kSplitSet) ok_split |= (p->split_k == s);
    if (!ok_split || p->split_k > (k_steps > 0 ? k_steps : 1)) return NM_ERR_ARG;
    const TileCfg &t = kTiles[p->tile];
    p->tile_n = t.tile_n();
    p->tile_m = t.tile_m();
    const int64_t tiles = ceil_div(n, p->tile_n) * ceil_div(m > 0 ? m : 1, p->tile_m);
    const int64_t grid = tiles * p->split_k;
    if (grid > 0x7fffffff) return NM_ERR_SHAPE;
    if (p->split_k > 1 && tiles > kMaxSplitTiles) return NM_ERR_ARG;
    // split-K partial sums are addressed with 32-bit byte offsets
    if (p->split_k > 1 && (int64_t)p->split_k * (m > 0 ? m : 1) * n * 4 >= ((int64_t)1 << 31)) return NM_ERR_SHAPE;
    p->grid = (int)grid;
    return NM_OK;
}

// Rows of output tiles from which a compact weight is expanded once per call.
constexpr int64_t kExpandTileRows = 32;

// Tile indices used by the rules below (see kTiles).
constexpr int kT128x128r2 = 0, kT128x64r2 = 1, kT64x128r2 = 2, kT64x64r2 = 3, kT256x256w8 = 4;
constexpr int kT128x32r2 = 5, kT128x128w8 = 6;
constexpr int kT64x64ks = 7, kT32x64ks = 8, kT64x32ks = 9, kT32x32ks = 10, kT128x160r2 = 11;

static int64_t tiles_of(int t, int m, int n) {
    return ceil_div(n, kTiles[t].tile_n()) * ceil_div(m, kTiles[t].tile_m());
}

nm_status make_plan(int kind, int m, int n, int k, int out_mode, nm_plan *plan) {
    if (!plan || m < 0 || n < 1 || k < 1) return NM_ERR_ARG;
    const int k_steps = (k + kKStep - 1) / kKStep;
    if ((out_mode & (NM_OUT_I32 | NM_OUT_F16 | NM_OUT_I8)) == 0) return NM_ERR_ARG;
    const int64_t cus = device_cu_count();
    const int mm = m > 0 ? m : 1;
    // Operands twice as heavy per k-step in matrix work: the kinds that run the
    // dense instruction (dense weights, and the mask layouts expanded to a
    // dense tile).
    const bool heavy = !kind_is_sp42(kind);
    // Rules fitted to an exhaustive timing of every tile on the ViT, DeiT and
    // Swin shapes (the paper's Table 1 methodology): above a few hundred
    // tokens the two-slot rings win -- their smaller LDS footprint keeps three
    // or more workgroups per compute unit, so one workgroup's loads overlap
    // another's compute and stores.
    int tile;
    if (mm <= 512) {
        // Few tokens: too few output tiles to occupy the GPU.  Split the
        // reduction over the waves of each workgroup (k-sliced 32 x 32 tile,
        // merged in LDS) while those tiles give at most 2 workgroups per CU.
        // For the heavier operands past one workgroup per CU, twice the tokens
        // per tile halve the weight fill (64 tokens, unless that pads m by more
        // than 15 %: then 64 channels); with a single k-step, 64 x 64.
        // Otherwise 64 x 64 with a 2-slot ring.
        const int64_t t32 = tiles_of(kT32x32ks, mm, n);
        if (t32 > 2 * cus)
            // many 32 x 32 tiles (the wide outputs): the k-sliced 64 x 64 tile
            // while it still fits two per CU (DeiT-B fc1 at batch 1: 9.0 us
            // against 9.9 for 64 x 64 with a ring), else 64 x 64
            tile = tiles_of(kT64x64ks, mm, n) <= 2 * cus ? kT64x64ks : kT64x64r2;
        else if (!heavy || t32 <= cus)
            tile = kT32x32ks;
        else if (k_steps == 1)
            tile = kT64x64r2;
        else
            tile = ceil_div(mm, 64) * 64 * 100 <= (int64_t)mm * 115 ? kT32x64ks : kT64x32ks;
    } else if (!heavy && k_steps >= 16 && k_steps <= 24 && mm <= 4096 && tiles_of(kT32x32ks, mm, n) <= 8 * cus) {
        // A few thousand tokens with a long reduction: the k-sliced 32 x 32
        // tile (the reduction split over the waves) still has more
        // workgroups than the output tiles of any ring tile (DeiT-B fc2 at
        // batch 8, 24 k-steps, inside the workload steps: 16.7 us against
        // 19 or more for 64 x 64; back to back, 64 x 64 is faster).  At 32
        // k-steps (Swin-B stage 4 fc2) 64 x 64 wins back to back by a third
        // and no in-network timing says otherwise, so the rule stops at 24.
        tile = kT32x32ks;
    } else if (k_steps <= 2) {
        // Very short reductions: the output stream dominates; small tiles
        // give the most workgroups in flight.  With one k-step and one-stream
        // weights, 128 channels x 32 tokens: the same number of workgroups
        // as 64 x 64, with output rows twice as long.
        tile = (!heavy && k_steps == 1 && n >= 384) ? kT128x32r2 : kT64x64r2;
    } else if (k_steps == 3) {
        // Three k-steps (DeiT-S, k = 384): 128 x 32 for one-stream weights,
        // 128 ch x 64 tok for the heavier operands (DeiT-S batch 64 proj,
        // dense, inside the steps: 12.5 us against 13.8-14.1 for 64 x 64; qkv
        // and fc1 within 1-3 %).
        tile = heavy ? kT128x64r2 : kT128x32r2;
    } else if (tiles_of(kT128x128r2, mm, n) < 4 * cus) {
        // Medium: with long reductions (8 k-steps or more) the operand fill
        // per output decides, so 128 x 128 as long as every compute unit
        // still gets a tile and the last tiles do not leave most units with
        // one while a few run two (1.25 tiles per unit or more); otherwise
        // half-height tiles (narrower for the heavier operands): DeiT-S batch
        // 64 fc2 (297 tiles of 128 x 128) 2:4 17.3 us against 18.5-18.7,
        // Swin-B stage 4 fc1 (312 tiles) dense 13.8-14.5 against 14.9-15.6.
        // A heavier operand whose channels fit one 128-row tile keeps 128 x
        // 128, which reads X once (Swin-B stage 1 fc2, 128 channels, dense:
        // 22.4-23.6 us against 23.7-25.3 for 64 x 128).
        const int64_t t128 = tiles_of(kT128x128r2, mm, n);
        if ((k_steps >= 8 && 4 * t128 >= 5 * cus) || (heavy && n <= 128 && t128 >= cus)) {
            tile = kT128x128r2;
        } else if (!heavy && k_steps < 8 && tiles_of(kT64x64r2, mm, n) <= 6 * cus) {
            // short reductions: 64 x 64 while it gives at most 6 workgroups
            // per CU (DeiT-B qkv and fc1 at batch 8: 11.1 and 13.1 us against
            // 13.4 and 15.0 for 128 x 64)
            tile = kT64x64r2;
        } else {
            // the heavier operands take 64 ch x 128 tok, except with long
            // reductions (12 k-steps or more), where 128 ch x 64 tok won in
            // every sweep inside the steps (DeiT-S batch 64 fc2 dense 18.8-19.6
            // us against 20.2-21.3, Swin-B stage 3 fc2 dense 17.4-18.0
            // against 18.0-19.1)
            tile = heavy && k_steps < 12 ? kT64x128r2 : kT128x64r2;
            // 64 x 64 when those would leave compute units without a tile,
            // and for one-stream weights when they already give 4 or more
            // workgroups per compute unit
            if (tiles_of(tile, mm, n) < cus || (!heavy && tiles_of(tile, mm, n) >= 4 * cus)) tile = kT64x64r2;
        }
    } else if (heavy) {
        // Large outputs, heavier operands: 128 x 128 on 8 waves (4 along the
        // channels x 2 along the tokens, twice the waves of the 4-wave tile to
        // overlap operand reads, matrix work and stores), except on the widest
        // outputs with long reductions (4096 channels or more, 24 k-steps or
        // more), where the 256 x 256 tile on 8 waves halves the operand fill
        // per output (6-13 % faster at k = 4096, n 4096 and 8192, m 8192-25216,
        // dense and 4:8).  Timed inside the steps of the ViT-L and DeiT-B
        // workloads with the 16-row tile groups (cold operands), 128 x 128 on
        // 8 waves won every other large shape (ViT-L qkv dense 82.7 us against
        // 88.4 on 4 waves, fc1 103.5 against 110.5) or tied within 2 %, except
        // the narrow outputs (512-1024 channels) with 8 or more k-steps: 160
        // tokens per tile on 4 waves, which reuses each weight slice over more
        // tokens (ViT-L fc2 dense 93.1 us against 102.7, DeiT-B batch 128 fc2
        // dense 66.8 against 74.5).
        if (n >= 4096 && k_steps >= 24)
            tile = kT256x256w8;
        else if (n >= 512 && n <= 1024 && k_steps >= 8)
            tile = kT128x160r2;
        else
            tile = kT128x128w8;
    } else {
        // Large outputs, 4:2-operand weights, timed the same way: long
        // reductions (24 k-steps or more) the 4-wave 128 x 128 tile, whose
        // larger per-wave fragment grid needs fewer operand reads per product
        // (ViT-L fc2 2:4 78.6 us, DeiT-B b128 fc2 60-62); otherwise 128 x 128
        // on 8 waves (ViT-L qkv and fc1 2:4: 70.4 and 87.2 us against 87.1
        // and 104.1 on the 256 x 256 tile, which the 16-row groups no longer
        // favour).
        tile = k_steps >= 24 ? kT128x128r2 : kT128x128w8;
    }
    plan->kind = kind;
    plan->tile = tile;
    plan->split_k = 1;
    // A compact weight is expanded inside every workgroup, ahead of its use,
    // when few rows of output tiles share it; with many rows the expansion
    // repeated per row costs more than one expansion pass per call.  1:4,
    // whose expansion is a few byte permutes, stays inside the workgroups
    // unless the reduction is long (24 k-steps or more: ViT-L fc2 81.5 us
    // expanded once against 87.3) or the output wide (4096 channels or more:
    // ViT-L fc1 86.2 against 89.7), or on the 256 x 256 tile (whose 8 waves
    // then need fewer registers).  The k-sliced tiles load the compact bytes
    // like X and expand them in registers, which the separate pass (a second
    // launch) never beats at the token counts they serve (DeiT-B fc2 at
    // batch 8, 1:4: 13.0 us against 16.1).
    // 1:8, whose expansion is a byte spread and a permute, likewise stays
    // inside below 2048 channels and 24 k-steps (DeiT-B batch 128 proj:
    // 26.8 us against 30.0 expanded once; qkv and fc1, 2304 and 3072 wide,
    // gain 2-6 % from the pass).  The pass costs a few microseconds whatever
    // the size (a second launch that waits for the first), so it is taken
    // only for GEMMs of 2^33 multiply-adds or more: inside the steps of
    // DeiT-S (at most 7.4e9) and Swin-B (at most 6.6e9) the in-kernel
    // expansion won every 2:8 and 4:8 GEMM, by 10-25 % (e.g. Swin-B stage 3
    // fc1 2:8 19.5 us against 24.3); from DeiT-B batch 128 proj up (1.5e10)
    // the pass wins (proj 2:8 30.0 us against 34.9).
    const bool many_rows = ceil_div(mm, kTiles[tile].tile_m()) >= kExpandTileRows;
    const bool k_sliced = kTiles[tile].layout == kKSliced;
    const bool long_gemm = (int64_t)mm * n * k >= ((int64_t)1 << 33);
    // With the expansion carried by an earlier launch the pass costs no
    // launch of its own.  Timed inside the workload steps with the expansions
    // carried: the 4:2-operand or dense kernel on the expanded weight then
    // beats the in-kernel decode for 1:8, 2:8 and the mask layouts at every
    // token count, k-sliced tiles included (DeiT-B batch 8 qkv 2:8 11.3 us
    // against 13.1, Swin-B stage 4 proj 2:8 9.0 against 12.1, ViT-L fc1 4:8
    // 112 against 127), and for 1:4, whose decode is a few permutes, only
    // with many rows of output-split tiles (DeiT-B batch 1 fc2 1:4 8.7 us
    // in-kernel against 10.3).
    const bool carried = (out_mode & NM_PLAN_EXPAND_CARRIED) != 0;
    bool once = long_gemm;
    if (kind == NM_KIND_C14) once = once && (k_steps >= 24 || n >= 4096 || tile == kT256x256w8);
    if (kind == NM_KIND_C18) once = once && (k_steps >= 24 || n >= 2048 || tile == kT256x256w8);
    if (carried)
        plan->expand = kind_is_compact(kind) && (kind != NM_KIND_C14 || (many_rows && !k_sliced)) ? 1 : 0;
    else
        plan->expand = kind_is_compact(kind) && many_rows && !k_sliced && once ? 1 : 0;
    // a weight that fits its limit as stored may pass it expanded (twice the
    // bytes, less the positions): then it is decoded in the kernel
    if (plan->expand && expanded_bytes(kind, n, k) >= kWeightLimit) plan->expand = 0;
    return complete_plan(kind, m, n, k, plan);
}

// ---------------------------------------------------------------------------
// Schedule of a call without an explicit plan.  nm_spmm_plan's rules name one
// tile per class of shapes; which tile is fastest depends on more than its
// class -- how many whole rounds of workgroups it fills, how long the chain of
// k-steps is, how many bytes the epilogue writes -- so a call that leaves the
// schedule to the library takes the tile with the least estimated time.  The
// estimate (microseconds) is linear in nine terms, fitted per tile and weight
// kind (non-negative least squares on relative errors, near-best rows weighted
// most) to 23 700 timings on an MI355X: every tile on 72 shapes drawn over m
// 64..60000, n and k 128..4096 with int32, fp16 and int8 outputs, and on the
// linears of DeiT, Swin-B and ViT-L.
//
// Held out (bench_experiments.py --schedule-eval: every tile on 400 other
// shapes per range): over the fitted range the chosen tile is 2.6 % from the
// best on average (the planner's 8.9 %) and takes 0.942 of the planner's time;
// one shape in 19 loses more than 3 % to the planner's tile, one in 50 more
// than 8 % (at most 17 %).  A switch is made for a promise of 3 % there: on 1848
// shapes that gave 0.948, asking for 6 or 10 % 0.952 and 0.960.  Reductions
// longer than any fitted one are extrapolated, and the estimate errs more: on
// 525 shapes with k to 16384, at 3 % one in 8 lost more than 3 % (m 2604,
// n 1416, k 6240, 2:8: 41.1 -> 50.8 us; m 2458, n 1508, k 15120, 2:4: 90.5 ->
// 113.1), so a switch has to promise 12 % there: one in 58, and 0.873 of the
// planner's time against 0.877; on the 400 other shapes one in 57, and 0.848.
constexpr int kFittedK = 4096;

struct CostTerms {
    float launch, chain, round_steps, mean_steps, rounds, round_bytes, out_mb, split_line_mb, x_mb;
};
static constexpr CostTerms kCost[5][kNumSchedules] = {
    {   // 2:4
        {3.34f, 0.184f, 0.141f, 0.162f, 0.831f, 0.0f, 0.107f, 0.0734f, 0.0743f},
        {3.05f, 0.236f, 0.0254f, 0.135f, 0.335f, 0.00319f, 0.106f, 0.0716f, 0.0539f},
        {3.16f, 0.186f, 0.0992f, 0.0955f, 0.259f, 0.0216f, 0.11f, 0.0756f, 0.0829f},
        {2.82f, 0.162f, 0.0964f, 0.0237f, 0.159f, 0.0f, 0.0923f, 0.0946f, 0.0736f},
        {0.313f, 0.0512f, 0.488f, 0.361f, 5.28f, 0.269f, 0.0861f, 0.081f, 0.0882f},
        {2.76f, 0.146f, 0.087f, 0.0464f, 0.279f, 0.0258f, 0.0359f, 0.0827f, 0.035f},
        {2.73f, 0.214f, 0.0937f, 0.192f, 0.742f, 0.0312f, 0.103f, 0.077f, 0.0825f},
        {2.2f, 0.0f, 0.554f, 0.17f, 1.48f, 0.0f, 0.0f, 0.116f, 0.0553f},
        {1.85f, 0.0f, 0.405f, 0.0371f, 1.47f, 0.0f, 0.0f, 0.139f, 0.0695f},
        {1.76f, 0.131f, 0.223f, 0.207f, 1.54f, 0.0f, 0.0f, 0.123f, 0.0f},
        {2.54f, 0.0941f, 0.183f, 0.0897f, 0.323f, 0.0f, 0.0f, 0.118f, 0.0113f},
        {3.09f, 0.341f, 0.0f, 0.283f, 1.16f, 0.0155f, 0.109f, 0.0694f, 0.0914f},
        {2.03f, 0.0f, 0.482f, 0.174f, 2.9f, 0.0f, 0.109f, 0.0839f, 0.0461f},
        {3.18f, 0.092f, 0.213f, 0.0f, 0.324f, 0.0283f, 0.107f, 0.0823f, 0.0575f},
        {1.76f, 0.0f, 0.323f, 0.0f, 1.84f, 0.0185f, 0.108f, 0.0817f, 0.0928f},
        {0.0f, 0.0225f, 0.884f, 0.0439f, 5.34f, 0.0206f, 0.139f, 0.0696f, 0.131f},
    },
    {   // 1:4 and 1:8
        {3.28f, 0.305f, 0.0546f, 0.181f, 0.73f, 0.0796f, 0.0913f, 0.0739f, 0.0844f},
        {3.13f, 0.265f, 0.0907f, 0.0659f, 0.386f, 0.00655f, 0.0976f, 0.063f, 0.0552f},
        {3.27f, 0.237f, 0.0797f, 0.0794f, 0.104f, 0.0237f, 0.121f, 0.0724f, 0.103f},
        {2.82f, 0.221f, 0.0354f, 0.0679f, 0.193f, 0.0f, 0.0976f, 0.0813f, 0.0691f},
        {1.34f, 0.0378f, 0.946f, 0.158f, 3.59f, 0.371f, 0.111f, 0.0706f, 0.0636f},
        {2.87f, 0.286f, 0.0742f, 0.0605f, 0.259f, 0.0492f, 0.019f, 0.0839f, 0.0186f},
        {2.69f, 0.177f, 0.207f, 0.069f, 0.844f, 0.0175f, 0.0988f, 0.0767f, 0.0868f},
        {2.06f, 0.0f, 0.693f, 0.0601f, 1.71f, 0.0f, 0.0106f, 0.0985f, 0.0768f},
        {1.85f, 0.0f, 0.566f, 0.0f, 1.43f, 0.0f, 0.0f, 0.165f, 0.0378f},
        {2.76f, 0.178f, 0.271f, 0.0798f, 0.673f, 0.0f, 0.0f, 0.0683f, 0.0666f},
        {2.56f, 0.109f, 0.223f, 0.0f, 0.436f, 0.0f, 0.0f, 0.11f, 0.0628f},
        {2.84f, 0.396f, 0.0f, 0.266f, 1.11f, 0.153f, 0.079f, 0.0716f, 0.0714f},
        {2.34f, 0.0f, 0.693f, 0.0472f, 2.47f, 0.0583f, 0.11f, 0.0899f, 0.0508f},
        {3.21f, 0.264f, 0.164f, 0.0357f, 0.377f, 0.000101f, 0.111f, 0.0761f, 0.0456f},
        {3.15f, 0.163f, 0.221f, 0.0f, 0.204f, 0.0543f, 0.104f, 0.116f, 0.112f},
        {1.17f, 0.0469f, 1.1f, 0.0f, 4.17f, 0.211f, 0.137f, 0.0662f, 0.109f},
    },
    {   // 2:8
        {3.35f, 0.38f, 0.0363f, 0.242f, 0.826f, 0.126f, 0.0768f, 0.0687f, 0.0648f},
        {3.31f, 0.355f, 0.0644f, 0.122f, 0.408f, 0.0137f, 0.0912f, 0.0621f, 0.0409f},
        {3.12f, 0.321f, 0.0373f, 0.131f, 0.381f, 0.0118f, 0.103f, 0.0745f, 0.0932f},
        {2.97f, 0.267f, 0.0569f, 0.0568f, 0.195f, 0.0f, 0.0989f, 0.0787f, 0.0599f},
        {0.497f, 0.0439f, 1.32f, 0.115f, 4.26f, 0.366f, 0.0929f, 0.0918f, 0.0405f},
        {2.9f, 0.363f, 0.0936f, 0.072f, 0.266f, 0.0633f, 0.0f, 0.0824f, 0.0f},
        {2.82f, 0.252f, 0.178f, 0.138f, 0.764f, 0.0494f, 0.0974f, 0.0794f, 0.0695f},
        {2.05f, 0.0f, 0.855f, 0.101f, 1.75f, 0.0f, 0.0f, 0.13f, 0.0647f},
        {1.85f, 0.0f, 0.606f, 0.0419f, 1.56f, 0.0f, 0.0f, 0.135f, 0.0636f},
        {1.88f, 0.0f, 0.663f, 0.0268f, 1.6f, 0.0f, 0.0f, 0.183f, 0.00106f},
        {2.59f, 0.14f, 0.275f, 0.0f, 0.48f, 0.0f, 0.0f, 0.0735f, 0.0562f},
        {2.98f, 0.377f, 0.0354f, 0.293f, 1.43f, 0.126f, 0.0789f, 0.07f, 0.0698f},
        {2.55f, 0.0f, 0.866f, 0.00615f, 2.32f, 0.0127f, 0.117f, 0.0838f, 0.0425f},
        {3.11f, 0.3f, 0.282f, 0.0f, 0.352f, 0.0595f, 0.0943f, 0.0826f, 0.0274f},
        {3.14f, 0.218f, 0.253f, 0.0f, 0.315f, 0.054f, 0.102f, 0.115f, 0.0922f},
        {1.21f, 0.0967f, 1.46f, 0.0766f, 3.69f, 0.377f, 0.122f, 0.0768f, 0.0694f},
    },
    {   // dense
        {3.26f, 0.27f, 0.0964f, 0.265f, 1.0f, 0.0292f, 0.0913f, 0.0827f, 0.0613f},
        {2.97f, 0.228f, 0.111f, 0.137f, 0.354f, 0.058f, 0.0746f, 0.0696f, 0.0535f},
        {3.2f, 0.202f, 0.139f, 0.0992f, 0.0709f, 0.0302f, 0.125f, 0.0906f, 0.0775f},
        {2.8f, 0.248f, 0.0f, 0.159f, 0.0719f, 0.0209f, 0.0917f, 0.0874f, 0.0862f},
        {0.789f, 0.0529f, 1.12f, 0.0897f, 4.02f, 0.197f, 0.125f, 0.0748f, 0.0835f},
        {2.78f, 0.208f, 0.0864f, 0.115f, 0.236f, 0.0359f, 0.063f, 0.0832f, 0.0216f},
        {2.99f, 0.219f, 0.142f, 0.246f, 0.522f, 0.0318f, 0.112f, 0.0843f, 0.0831f},
        {2.44f, 0.0304f, 0.653f, 0.268f, 1.76f, 0.0f, 0.0f, 0.196f, 0.0796f},
        {2.12f, 0.00182f, 0.515f, 0.0939f, 1.35f, 0.0f, 0.0f, 0.216f, 0.00446f},
        {2.33f, 0.235f, 0.18f, 0.48f, 1.26f, 0.0f, 0.165f, 0.212f, 0.0f},
        {1.94f, 0.0248f, 0.308f, 0.141f, 1.2f, 0.0f, 0.0f, 0.219f, 0.0f},
        {2.93f, 0.398f, 0.0f, 0.402f, 1.32f, 0.0534f, 0.0946f, 0.0866f, 0.0729f},
        {2.5f, 0.0f, 0.739f, 0.179f, 2.63f, 0.0558f, 0.108f, 0.0873f, 0.0404f},
        {2.14f, 0.0f, 0.352f, 0.0184f, 1.52f, 0.0104f, 0.143f, 0.0633f, 0.0422f},
        {1.6f, 0.0f, 0.346f, 0.0195f, 1.93f, 0.024f, 0.0885f, 0.102f, 0.0743f},
        {1.35f, 0.0f, 1.48f, 0.0998f, 3.39f, 0.28f, 0.134f, 0.0853f, 0.0743f},
    },
    {   // 3:8, 4:8, 5:8
        {3.71f, 0.314f, 0.211f, 0.2f, 0.891f, 0.00627f, 0.101f, 0.0949f, 0.061f},
        {3.36f, 0.317f, 0.167f, 0.0885f, 0.439f, 0.0f, 0.0904f, 0.0874f, 0.0476f},
        {3.22f, 0.302f, 0.11f, 0.122f, 0.479f, 0.00277f, 0.104f, 0.0845f, 0.0767f},
        {2.91f, 0.248f, 0.121f, 0.0355f, 0.312f, 0.0f, 0.0575f, 0.108f, 0.0512f},
        {1.0f, 0.151f, 1.61f, 0.0681f, 3.77f, 0.328f, 0.116f, 0.0849f, 0.0579f},
        {2.96f, 0.394f, 0.0997f, 0.13f, 0.343f, 0.0528f, 0.0f, 0.0834f, 0.0f},
        {3.05f, 0.218f, 0.328f, 0.108f, 0.762f, 0.0167f, 0.0965f, 0.101f, 0.0623f},
        {2.05f, 0.0548f, 0.975f, 0.0881f, 1.92f, 0.0f, 0.0f, 0.131f, 0.0702f},
        {1.93f, 0.0f, 0.695f, 0.0183f, 1.59f, 0.0f, 0.0f, 0.125f, 0.108f},
        {1.9f, 0.0815f, 0.787f, 0.138f, 1.61f, 0.0f, 0.0f, 0.143f, 0.00807f},
        {1.9f, 0.0f, 0.563f, 0.0931f, 1.19f, 0.0f, 0.0f, 0.167f, 0.0f},
        {3.46f, 0.315f, 0.26f, 0.223f, 1.14f, 0.0f, 0.106f, 0.102f, 0.0946f},
        {2.15f, 0.0271f, 1.12f, 0.0f, 3.11f, 0.0161f, 0.108f, 0.0891f, 0.0325f},
        {3.08f, 0.317f, 0.316f, 0.00487f, 0.586f, 0.0176f, 0.105f, 0.0868f, 0.0532f},
        {2.16f, 0.0174f, 0.533f, 0.0f, 1.49f, 0.029f, 0.168f, 0.0398f, 0.0818f},
        {1.09f, 0.138f, 1.92f, 0.0f, 4.0f, 0.314f, 0.125f, 0.097f, 0.0723f},
    },
};

static int cost_group(int kind) {
    switch (kind) {
        case NM_KIND_SP42: return 0;
        case NM_KIND_C14: case NM_KIND_C18: return 1;
        case NM_KIND_C28: return 2;
        case NM_KIND_DENSE: return 3;
        default: return 4;
    }
}

int schedule_tile(int kind, int m, int n, int k, int out_mode, int planned) {
    // 32-bit divisions only: this runs in every call
    const uint32_t cus = (uint32_t)device_cu_count();
    uint32_t bytes = 0, split_line = 0;   // per output element; of rows that do not start on a 128-byte line
    for (uint32_t eb : {4u, 2u, 1u})
        if (out_mode & (eb == 4 ? NM_OUT_I32 : eb == 2 ? NM_OUT_F16 : NM_OUT_I8)) {
            bytes += eb;
            if ((uint64_t)n * eb % 128 != 0) split_line += eb;
        }
    const float mn = (float)m * (float)n * 1e-6f, out_mb = mn * (float)bytes, split_mb = mn * (float)split_line;
    const float x_mb = (float)m * (float)k * 1e-6f;
    const uint32_t k_steps = ((uint32_t)k + kKStep - 1) / kKStep;
    const CostTerms *cost = kCost[cost_group(kind)];
    auto estimate_us = [&](int t) {
        const CostTerms &c = cost[t];
        const uint32_t tn = (uint32_t)kTiles[t].tile_n(), tm = (uint32_t)kTiles[t].tile_m();
        const uint32_t tiles = (((uint32_t)n + tn - 1) / tn) * (((uint32_t)m + tm - 1) / tm);   // below 2^29
        const float steps = (float)(kTiles[t].layout == kKSliced ? (k_steps + 3) / 4 : k_steps);
        const float rounds = (float)((tiles + cus - 1) / cus), mean = (float)tiles / (float)cus;
        return c.launch + steps * (c.chain + c.round_steps * rounds + c.mean_steps * mean) +
               rounds * (c.rounds + c.round_bytes * (float)bytes) + c.out_mb * out_mb + c.split_line_mb * split_mb +
               c.x_mb * x_mb;
    };
    int best = planned;
    float least = (k > kFittedK ? 0.88f : 0.97f) * estimate_us(planned);
    for (int t = 0; t < kNumSchedules; ++t) {
        if (!tile_built(kind, t)) continue;
        const float us = estimate_us(t);
        if (us < least) {
            least = us;
            best = t;
        }
    }
    return best;
}

}  // namespace nmspmm
