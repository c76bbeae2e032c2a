// chunk_select_attention_decode: the selection (paper Sec. 4.2 / 6.1) and the
// attention over the kept chunks (Sec. 2.1 Eq. 1, Sec. 4.1 workflow) of a decode
// step in ONE launch, for keys / values stored as they are (16-bit or fp32).
//
// The two steps are short, dependent and latency-bound at decode batch sizes: as
// separate launches they pay a launch gap, a round trip of the kept list through
// memory, and a third small launch that combines the attention splits.  Here a
// 1024-lane workgroup runs the selection of its (sequence, kv head) (the same
// code as chunk_topk_select), leaves the kept chunks' token ranges in LDS, and
// its sixteen waves then stream their shares of the kept tokens.  When a
// (sequence, kv head) is spread over several workgroups ("splits") every one of
// them repeats the selection - it reads only the score row, which the second
// reader finds in L2 - and takes its own range of the kept tokens.
//
// Splits are combined in the same launch by the workgroup that finishes last:
// each split publishes its partial (m, l, acc[D]) with agent-scope relaxed atomic
// stores (write-through, no cache write-back), waits for them, and takes a ticket
// from an agent-scope counter; the workgroup that draws the last ticket reads all
// partials with agent-scope atomic loads and folds them in split order, so the
// result does not depend on which workgroup that is.  No workgroup ever waits
// for another.  The counters live in the workspace, are zero between calls and
// are reset by the workgroup that merges.
//
// Streaming: q K^T on v_mfma_f32_16x16x32 with token = row, query head = column
// (as in sparse_attention.hip); P V in fp32 on the vector ALU.  With sixteen
// waves per workgroup a wave has 128 registers: two K/V tiles in flight and the
// accumulators; the queries (the matrix core's B operand) stay in LDS.  Nothing
// else in the tile loop goes through LDS: the running maximum over the four lane
// groups is taken with lane swaps on the vector ALU (two ds_bpermute round trips
// per tile in its place cost the launch 10 % on MI355X, the next tile's loads
// queue behind the same waits).
#include <algorithm>
#include <cstdlib>

#include "fused_tail.h"

namespace leoam {

constexpr int kFusedBlock = 128;                       // tokens a wave maps to rows at a time
constexpr int kFusedHeads = 4;                         // query heads a wave accumulates, at most
constexpr int kFusedMaxSel = 2048;                     // kept chunks per (b,h) whose ranges fit the LDS tables
constexpr int kFusedMaxSplits = 64;
constexpr int kFusedTargetWgs = 256;                   // one workgroup per compute unit
constexpr size_t kArrivalAlign = 256;

// How a group of G query heads is laid over the sixteen waves.  A wave keeps eight accumulators per head and
// lane, so at most four heads fit beside a tile in its 128 registers; with eight heads the waves form two
// halves that stream the SAME tokens, four heads each (the second reader of a row finds it in the caches: the
// chip has that bandwidth to spare, the registers it has not).
template <int G> struct FusedPlan {
    static constexpr int kHeads = G < kFusedHeads ? G : kFusedHeads;      // heads of a wave
    static constexpr int kParts = G / kHeads;                             // waves that share a token stream
    static constexpr int kStreams = kFusedWaves / kParts;
    static constexpr int kGranule = kStreams * 16;                        // a split is a multiple of this many tokens
};

// one 16-token tile of a wave: K operand (a quarter of a row per lane: ROWB / 64 pieces of 16 bytes) and
// V rows (four rows per lane, ROWB / 256 pieces of each)
template <typename T> struct FusedKvTile {
    uint4 k[Row<T>::kRowBytes / 64];
    uint4 v[4][Row<T>::kRowBytes / 256];
};

// q . k of a tile's 16 tokens on the matrix cores.  16-bit: v_mfma_f32_16x16x32, token = row, head = column,
// piece s of the K operand is one step.  fp32: v_mfma_f64_4x4x4 (as in chunk_score.hip: four blocks of four
// tokens, every block carries the queries), element e of piece s is step 4 s + e, products exact and sums in
// double.  (v_mfma_f32_16x16x4_f32 was as fast, but its sums ended up to three times further from a 64-bit
// reference than the vector ALU's, 1.2 times when summed pairwise.)
template <typename T> struct QueryStep { using Type = uint4; static constexpr int kPerPiece = 1; };
template <> struct QueryStep<F32> { using Type = double; static constexpr int kPerPiece = 4; };

// kGiven: the kept lists (sel_idx, sel_count) are inputs - a selection made earlier, for instance by
// one chunk_topk_select call over all layers of a step - and the workgroup only builds its tables
// from them (two list positions per lane; kIpt is not used).
template <typename T, int G, int kIpt, bool kGiven = false>
__global__ __launch_bounds__(kSelThreads) void select_attention_kernel(
    const float* __restrict__ score, const int32_t* __restrict__ chunk_off, const int32_t* __restrict__ n_chunks,
    int max_chunks, int token_budget, int32_t* __restrict__ sel_idx, int32_t* __restrict__ sel_count,
    int32_t* __restrict__ sel_tokens, const char* __restrict__ q, const char* __restrict__ K,
    const char* __restrict__ V, float scale_log2, float* __restrict__ out, float* __restrict__ lse, float* partial,
    int32_t* arrivals, int n_splits, int c_max, int k_max, int n_kv_heads, int n_ctx, unsigned long long* exchange) {
    constexpr int ROWB = Row<T>::kRowBytes;
    constexpr int KP = ROWB / 64, VP = ROWB / 256;         // 16-byte pieces per lane of a K row and of a V row
    constexpr int EPL = T::kEpl, NACC = LEOAM_D / 16;      // channels per piece, accumulators per head
    using P = FusedPlan<G>;
    constexpr int GH = P::kHeads;

    // the three phases use LDS one after the other
    union Phase {
        SelectLds sel;
        int32_t rows[kFusedWaves][kFusedBlock];
        float xw[kFusedWaves][GH][kPartStride];
    };
    __shared__ Phase ph;
    __shared__ int32_t start[kFusedMaxSel], prefix[kFusedMaxSel + 1];
    using QStep = QueryStep<T>;
    __shared__ typename QStep::Type qs[P::kParts][KP * QStep::kPerPiece][LEOAM_WAVE];      // the group's queries as matrix-core operand
    __shared__ int32_t sh_last;

    const int split = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / LEOAM_WAVE;
    const int grp = lane >> 4, c16 = lane & 15;
    const size_t bh = (size_t)b * n_kv_heads + h;
    const int C = min(max(n_chunks[b], 0), c_max);
    const int32_t* off = chunk_off + (size_t)b * (c_max + 1);

    // ---- the group's queries as the matrix cores take them, zero beyond the wave's heads.  A piece per wave,
    // fetched while the selection runs, handed to the others through LDS.
    static_assert(P::kParts * KP <= kFusedWaves, "a wave stages one piece");
    const int q_part = wave / KP, q_piece = wave % KP, q_head = T::kBytes == 2 ? c16 : (lane & 3);
    uint4 qb = make_uint4(0, 0, 0, 0);
    if (q_part < P::kParts) {
        const size_t qrow = ((size_t)b * n_kv_heads * G + (size_t)h * G + q_part * GH + min(q_head, GH - 1)) * ROWB;
        qb = load16(q, qrow + 64 * q_piece + 16 * grp);
    }
    auto stage_queries = [&] {
        if (q_part >= P::kParts) return;
        if constexpr (T::kBytes == 2) {
            qs[q_part][q_piece][lane] = (q_head < GH) ? qb : make_uint4(0, 0, 0, 0);
        } else {
            float x[EPL];
            unpack<T>(qb, x);
#pragma unroll
            for (int e = 0; e < EPL; ++e) qs[q_part][EPL * q_piece + e][lane] = (q_head < GH) ? (double)x[e] : 0.0;
        }
    };

    int cnt, total;
    if constexpr (kGiven) {
        // ---- the kept list is given: first token and size of every listed chunk, then a scan --------
        static_assert(kFusedMaxSel == 2 * kSelThreads, "two list positions per lane");
        const int32_t* ids = sel_idx + bh * (size_t)k_max;
        const int listed = min(max(sel_count[bh], 0), k_max);
        int st[2];
        uint32_t sz[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // (unconditional, clamped loads; an id outside [0, n_chunks) contributes no tokens)
            const int p = 2 * tid + j;
            const int id = ids[min(p, k_max - 1)];
            const bool ok = p < listed && id >= 0 && id < C;
            const int c = ok ? id : 0;
            const int a = min(max(off[c], 0), n_ctx), e = min(max(off[c + 1], a), n_ctx);
            st[j] = a;
            sz[j] = ok ? (uint32_t)(e - a) : 0u;
        }
        uint64_t tot;
        uint32_t before = (uint32_t)block_excl_scan<false>(pack_tot(0, sz[0] + sz[1]), ph.sel.wave_sums2, &tot);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = 2 * tid + j;
            if (p < listed) {
                start[p] = st[j];
                prefix[p] = (int32_t)before;
            }
            before += sz[j];
        }
        cnt = listed;
        total = (int)(uint32_t)tot;
        if (tid == 0) prefix[cnt] = total;
        stage_queries();
    } else {
        // ---- selection --------------------------------------------------------------
        SelectResult<kIpt> R;
        select_keep<kIpt>(ph.sel, score + bh * (size_t)c_max, off, C, c_max, k_max, n_ctx, max_chunks, token_budget, R);
        cnt = (int)min((uint32_t)(R.kept_total >> 32), (uint32_t)k_max);
        total = (int)(uint32_t)R.kept_total;
        {
            // kept chunks in ascending order: first token and number of kept tokens before it
            int32_t* ids = sel_idx + bh * (size_t)k_max;
            const int c0 = tid * kIpt;
            uint32_t pos = (uint32_t)(R.kept_before >> 32), before = (uint32_t)R.kept_before;
            int tok = R.first_tok;
#pragma unroll
            for (int i = 0; i < kIpt; ++i) {
                if (R.keep[i]) {
                    if (pos < (uint32_t)k_max) {
                        start[pos] = tok;
                        prefix[pos] = (int32_t)before;
                        if (split == 0) ids[pos] = c0 + i;
                    }
                    ++pos;
                    before += R.size[i];
                }
                tok += (int)R.size[i];
            }
            if (tid == 0) prefix[cnt] = total;
            stage_queries();
            if (split == 0) {
                for (int i = cnt + tid; i < k_max; i += kSelThreads) ids[i] = -1;
                if (tid == 0) {
                    sel_count[bh] = cnt;
                    if (sel_tokens) sel_tokens[bh] = total;
                }
            }
        }
    }
    __syncthreads();      // tables complete; the selection's LDS is free

    // ---- this workgroup's range of the kept tokens, then this wave's share --------
    int per_split = (total + n_splits - 1) / n_splits;
    per_split = max(1, (per_split + P::kGranule - 1) / P::kGranule) * P::kGranule;
    // splits that hold tokens; the others (fewer tokens were kept than the launch was sized for) leave here,
    // and the merge counts only these
    const int n_active = max(1, (total + per_split - 1) / per_split);
    if (split >= n_active) return;
    const int r0 = min(total, split * per_split), r1 = min(total, r0 + per_split);
    const int per_wave = per_split / P::kStreams, part = P::kParts == 1 ? 0 : wave / P::kStreams;
    const int w0 = min(r1, r0 + (wave % P::kStreams) * per_wave), w1 = min(r1, w0 + per_wave);

    // the (b,h)'s rows as buffers; a lane adds a 32-bit offset (n_ctx + 1 rows stay below 4 GiB)
    const buffer_t Kbh = buffer_of(K + bh * (size_t)n_ctx * ROWB, (uint32_t)n_ctx * ROWB);
    const buffer_t Vbh = buffer_of(V + bh * (size_t)n_ctx * ROWB, (uint32_t)n_ctx * ROWB);
    const uint32_t k_lane = 16u * grp, v_lane = 16u * c16;
    int32_t* my_rows = ph.rows[wave];

    // lanes (grp, head) carry the softmax state of `head`; every lane carries the
    // accumulators of all heads for the V rows of its group and its 8 columns
    float m_run = -INFINITY, l_run = 0.f;
    float acc[GH][NACC];
#pragma unroll
    for (int g = 0; g < GH; ++g)
#pragma unroll
        for (int e = 0; e < NACC; ++e) acc[g][e] = 0.f;

    // Loads are unconditional (a load under a condition is waited for on its own): a position past the end has row
    // n_ctx, which is outside the buffers, and gets zeros without an access.  (Its logit is masked to -inf; a weight of
    // 0 would not be enough, as 0 times a kept row's infinity is not 0.)
    auto fetch = [&](int t, FusedKvTile<T>& kv) {
        const uint32_t krow = my_rows[16 * t + c16];
#pragma unroll
        for (int s = 0; s < KP; ++s) kv.k[s] = buffer_load16(Kbh, krow * ROWB + k_lane + 64u * s);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t vrow = my_rows[16 * t + 4 * grp + i];
#pragma unroll
            for (int s = 0; s < VP; ++s) kv.v[i][s] = buffer_load16(Vbh, vrow * ROWB + v_lane + 256u * s);
        }
    };
    int q_lane = lane;
    auto logits = [&](const uint4* k) {
        // the queries are re-read from LDS for every tile: registers a wave cannot spare
        asm volatile("" : "+v"(q_lane));
        f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};
        if constexpr (T::kBytes == 2) {
#pragma unroll
            for (int s = 0; s < KP; ++s) sacc = mfma_16x16x32<T>(k[s], qs[part][s][q_lane], sacc);
            return sacc * scale_log2;
        } else {
            double sum[2] = {0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KP; ++s) {
                float x[EPL];
                unpack<T>(k[s], x);
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    sum[e & 1] = __builtin_amdgcn_mfma_f64_4x4x4f64(qs[part][EPL * s + e][q_lane], (double)x[e], sum[e & 1], 0, 0, 0);
            }
            // lane 16 * head + token -> token 4 grp + r of head c16 (columns beyond the heads repeat the last)
            const float dot = (float)((sum[0] + sum[1]) * (double)scale_log2);
#pragma unroll
            for (int r = 0; r < 4; ++r) sacc[r] = __shfl(dot, 16 * min(c16, 3) + 4 * grp + r, LEOAM_WAVE);
            return sacc;
        }
    };
    auto accumulate = [&](f32x4_t sacc, const uint4 (*v)[VP], int n_valid) {
        // sacc[r] = logit (log2 domain) of token 4grp + r of the tile, head c16
        float z[4];
        float mloc = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z[r] = (4 * grp + r < n_valid) ? sacc[r] : -INFINITY;
            mloc = fmaxf(mloc, z[r]);
        }
        mloc = rows_max4(mloc);
        const float m_new = fmaxf(m_run, mloc);
        const float corr = exp2_or_zero(m_run, m_new);
        const bool changed = (c16 < GH) && (m_new > m_run);
        m_run = m_new;
        float psum = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z[r] = exp2_or_zero(z[r], m_new);     // now the weight
            psum += z[r];
        }
        l_run = l_run * corr + psum;
        if (__ballot(changed) != 0ull) {
            // head g's correction factor sits in lane g of every row
            static_for<0, GH>([&](auto gc) {
                constexpr int g = decltype(gc)::value;
                const float cg = row_bcast<g>(corr);
#pragma unroll
                for (int e = 0; e < NACC; ++e) acc[g][e] *= cg;
            });
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x[NACC];
#pragma unroll
            for (int s = 0; s < VP; ++s) unpack<T>(v[i][s], x + s * EPL);
            static_for<0, GH>([&](auto gc) {
                constexpr int g = decltype(gc)::value;
                const float p = row_bcast<g>(z[i]);
#pragma unroll
                for (int e = 0; e < NACC; ++e) acc[g][e] = fmaf(p, x[e], acc[g][e]);
            });
        }
    };

    for (int blk = w0; blk < w1; blk += kFusedBlock) {
        const int nb = min(kFusedBlock, w1 - blk);
        // token position in the kept list -> row in the cache, for the whole block
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");      // earlier reads of my_rows are done
        {
            // a lane maps consecutive positions: one search, then a walk
            constexpr int PER = kFusedBlock / LEOAM_WAVE;
            const int i0 = lane * PER;
            int lo = 0;
            if (i0 < nb) {
                const int x = blk + i0;
                int hi = cnt;                  // largest k with prefix[k] <= x
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (prefix[mid] <= x) lo = mid; else hi = mid;
                }
            }
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                int p = n_ctx;
                if (i0 + j < nb) {
                    const int x = blk + i0 + j;
                    while (prefix[lo + 1] <= x) ++lo;      // ends: prefix[cnt] = total > x
                    p = start[lo] + (x - prefix[lo]);
                }
                my_rows[i0 + j] = p;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");      // table visible to the whole wave
        __builtin_amdgcn_wave_barrier();

        const int n_tiles = (nb + 15) >> 4, last = n_tiles - 1;
        if constexpr (T::kBytes == 4) {
            // a tile is 16 KiB: one per wave keeps 256 KiB of the compute unit's loads in flight, and two
            // do not fit the registers
            for (int t = 0; t < n_tiles; ++t) {
                FusedKvTile<T> cur;
                fetch(t, cur);
                accumulate(logits(cur.k), cur.v, nb - 16 * t);
            }
            continue;
        }
        FusedKvTile<T> cur, nxt;
        fetch(0, cur);
        if (n_tiles == 1) {
            // a single tile (small batches spread a (b,h) over many workgroups): nothing to prefetch,
            // and the pipeline's re-reads of the last tile would triple the load instructions
            accumulate(logits(cur.k), cur.v, nb);
            continue;
        }
        for (int t = 0; t < n_tiles; t += 2) {
            // (no loads under a condition: a tile index past the end re-reads the last tile)
            fetch(min(t + 1, last), nxt);
            __builtin_amdgcn_sched_barrier(0);       // keep the loads ahead of the tile's arithmetic
            accumulate(logits(cur.k), cur.v, nb - 16 * t);
            fetch(min(t + 2, last), cur);
            __builtin_amdgcn_sched_barrier(0);
            if (t + 1 < n_tiles) accumulate(logits(nxt.k), nxt.v, nb - 16 * (t + 1));
        }
    }

    // ---- fold the four lane groups (same m everywhere in the wave) ---------------
    // four accumulators at a time: afterwards lane group r holds the total of
    // accumulator kRowOwns[r] of the quad, so all 64 lanes write to LDS
    l_run = rows_sum4(l_run, l_run, l_run, l_run);
    const int e_own = ((grp & 1) << 1) | (grp >> 1);        // rows 0,1,2,3 own accumulators 0,2,1,3
    float folded[GH][2];
#pragma unroll
    for (int g = 0; g < GH; ++g) {
        folded[g][0] = rows_sum4(acc[g][0], acc[g][1], acc[g][2], acc[g][3]);
        folded[g][1] = rows_sum4(acc[g][4], acc[g][5], acc[g][6], acc[g][7]);
    }
    __syncthreads();      // every wave is done with its row table: LDS becomes the exchange buffer
    // (16-bit: a lane's eight channels are neighbours; fp32: four in each half of the row)
    constexpr int kUpper = VP == 1 ? 4 : 16 * EPL;
#pragma unroll
    for (int g = 0; g < GH; ++g) {
        ph.xw[wave][g][c16 * EPL + e_own] = folded[g][0];
        ph.xw[wave][g][c16 * EPL + kUpper + e_own] = folded[g][1];
    }
    if (grp == 0 && c16 < GH) {
        ph.xw[wave][c16][LEOAM_D] = m_run;
        ph.xw[wave][c16][LEOAM_D + 1] = l_run;
    }
    __syncthreads();

    fused_tail<G, GH>(ph.xw, sh_last, partial, arrivals, out, lse, bh, split, n_active, n_splits, exchange);
}

// zero fill (arrival counters of a fresh workspace)
__global__ void workspace_zero_kernel(uint4* __restrict__ p, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

hipError_t workspace_zero_dispatch(void* workspace, size_t bytes, hipStream_t stream) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(workspace_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (uint4*)workspace, n16);
    return hipGetLastError();
}

hipError_t topk_select_dispatch(const leoam_shape*, const float*, const int32_t*, const int32_t*, int, int, int32_t*,
                                int32_t*, int32_t*, hipStream_t);
hipError_t attention_dispatch(const leoam_shape*, const void*, const void*, const void*, const void*, const int32_t*,
                              const int32_t*, const int32_t*, const int32_t*, float, float*, float*, void*, size_t,
                              int32_t*, hipStream_t);
size_t attention_workspace_bytes(const leoam_shape*, int);
size_t attention_min_workspace_bytes(const leoam_shape*);

bool select_attention_q_is_fused(const leoam_shape*);
int fused_q_recommended_splits(const leoam_shape*, int);
hipError_t select_attention_q_dispatch(const leoam_shape*, const float*, const void*, const void*, const void*, const void*,
                                       const int32_t*, const int32_t*, int, int, float, int32_t*, int32_t*, int32_t*,
                                       float*, float*, float*, int32_t*, int, hipStream_t);

// LEOAM_STREAM_ORDERED_MERGE=1 in the environment (read once per process) makes the one-call entry points run
// the selection kernel, the attention kernel and the merge kernel back to back instead of the one-launch
// kernels, whose in-launch merge relies on the memory system's behaviour rather than on the memory model.
static bool stream_ordered_merge_wanted() {
    static const bool wanted = [] {
        const char* v = getenv("LEOAM_STREAM_ORDERED_MERGE");
        return v && v[0] && v[0] != '0';
    }();
    return wanted;
}

static inline size_t arrival_bytes(const leoam_shape* s) {
    const size_t n = (size_t)s->batch * s->n_kv_heads * sizeof(int32_t);
    return (n + kArrivalAlign - 1) / kArrivalAlign * kArrivalAlign;
}

static inline size_t fused_part_bytes_per_split(const leoam_shape* s) {
    return (size_t)s->batch * s->n_q_heads * kPartStride * sizeof(float);
}

// Shapes the one-launch kernel can take.
bool select_attention_is_fused(const leoam_shape* s) {
    // (the kernel adds 32-bit row offsets to a per-(b,h) base: n_ctx rows must stay below 4 GiB)
    return s->kv_dtype != LEOAM_Q8Q4 && s->k_max <= kFusedMaxSel && s->c_max <= 8 * kSelThreads &&
           s->n_ctx < (s->kv_dtype == LEOAM_F32 ? 1 << 23 : 1 << 24);
}
// The shapes of which every call runs in one launch (the others: where one_launch_pays says so).  Their two-split
// launches merge through exchange words, and with a single split they need no room for partials.
static inline bool always_one_launch(const leoam_shape* s) {
    return select_attention_is_fused(s) && s->kv_dtype != LEOAM_F32 && s->n_q_heads / s->n_kv_heads <= kFusedHeads;
}

// Tokens a split is a multiple of, and the largest useful number of splits of a (b, h): up to one workgroup
// per compute unit (that is what workspaces are sized for).
static inline int fused_granule(const leoam_shape* s) {
    return (s->n_q_heads / s->n_kv_heads > kFusedHeads ? FusedPlan<8>::kGranule : FusedPlan<1>::kGranule);
}
static int fused_recommended_splits(const leoam_shape* s, int max_tokens) {
    if (max_tokens <= 0 || max_tokens > s->n_ctx) max_tokens = s->n_ctx;
    const int granule = fused_granule(s);
    const int by_tokens = (max_tokens + granule - 1) / granule;
    const int units = s->batch * s->n_kv_heads;
    int want = (kFusedTargetWgs + units - 1) / units;
    if (want > by_tokens) want = by_tokens;
    if (want > kFusedMaxSplits) want = kFusedMaxSplits;
    if (want < 1) want = 1;
    return want;
}

// Exchange words of the two-split merge (fused_tail.h): one 64-bit word per (b, q head, channel), zero
// between calls like the arrival counters.  Reserved for the batch sizes that give two splits per
// (b, h), i.e. between half a workgroup and one workgroup per compute unit.
static inline size_t exchange_bytes(const leoam_shape* s) {
    const long long units = (long long)s->batch * s->n_kv_heads;
    if (!always_one_launch(s) || (kFusedTargetWgs + units - 1) / units != 2) return 0;
    return (size_t)s->batch * s->n_q_heads * LEOAM_D * sizeof(unsigned long long);
}

// the leading bytes of the workspace that are zero between calls
static inline size_t control_bytes(const leoam_shape* s, bool with_exchange) {
    return arrival_bytes(s) + (with_exchange ? exchange_bytes(s) : 0);
}

// control words, then whichever is larger: the fused kernel's partials or the
// workspace of the two-launch path that shapes outside the fused kernel take
size_t select_attention_workspace_bytes(const leoam_shape* s, int max_tokens, bool with_exchange) {
    size_t body = attention_workspace_bytes(s, max_tokens);
    if (select_attention_is_fused(s)) {
        const size_t f = fused_part_bytes_per_split(s) * (size_t)fused_recommended_splits(s, max_tokens);
        if (f > body) body = f;
    }
    if (select_attention_q_is_fused(s)) {
        const size_t f = fused_part_bytes_per_split(s) * (size_t)fused_q_recommended_splits(s, max_tokens);
        if (f > body) body = f;
    }
    return control_bytes(s, with_exchange) + body;
}

size_t select_attention_counter_bytes(const leoam_shape* s, bool with_exchange) { return control_bytes(s, with_exchange); }

size_t select_attention_min_workspace_bytes(const leoam_shape* s, bool with_exchange) {
    // (the separate kernels need one partial per (b, q head), and which calls take them is not known from the shape)
    const bool one_launch = (always_one_launch(s) || select_attention_q_is_fused(s)) && !stream_ordered_merge_wanted();
    return control_bytes(s, with_exchange) + (one_launch ? 0 : attention_min_workspace_bytes(s));
}

template <typename T, int G>
static hipError_t launch_fused(const leoam_shape* s, const float* score, const void* q, const void* K, const void* V,
                               const int32_t* chunk_off, const int32_t* n_chunks, int max_chunks, int token_budget,
                               float scale, int32_t* sel_idx, int32_t* sel_count, int32_t* sel_tokens, float* out,
                               float* lse, float* partial, int32_t* arrivals, int n_splits, unsigned long long* exchange,
                               hipStream_t stream) {
    dim3 grid(n_splits, s->n_kv_heads, s->batch), block(kSelThreads);
#define LEOAM_FUSED(IPT)                                                                                              \
    hipLaunchKernelGGL((select_attention_kernel<T, G, IPT>), grid, block, 0, stream, score, chunk_off, n_chunks,       \
                       max_chunks, token_budget, sel_idx, sel_count, sel_tokens, (const char*)q, (const char*)K,       \
                       (const char*)V, scale * kLog2e, out, lse, partial, arrivals, n_splits, s->c_max, s->k_max,      \
                       s->n_kv_heads, s->n_ctx, exchange)
    if (!score)      // the kept lists are given
        hipLaunchKernelGGL((select_attention_kernel<T, G, 1, true>), grid, block, 0, stream, score, chunk_off, n_chunks,
                           max_chunks, token_budget, sel_idx, sel_count, sel_tokens, (const char*)q, (const char*)K,
                           (const char*)V, scale * kLog2e, out, lse, partial, arrivals, n_splits, s->c_max, s->k_max,
                           s->n_kv_heads, s->n_ctx, exchange);
    else if (s->c_max <= kSelThreads) LEOAM_FUSED(1);
    else if (s->c_max <= 2 * kSelThreads) LEOAM_FUSED(2);
    else if (s->c_max <= 4 * kSelThreads) LEOAM_FUSED(4);
    else if (s->c_max <= 6 * kSelThreads) LEOAM_FUSED(6);
    else LEOAM_FUSED(8);
#undef LEOAM_FUSED
    return hipGetLastError();
}

template <typename T>
static hipError_t fused_by_group(const leoam_shape* s, const float* score, const void* q, const void* K, const void* V,
                                 const int32_t* chunk_off, const int32_t* n_chunks, int max_chunks, int token_budget,
                                 float scale, int32_t* sel_idx, int32_t* sel_count, int32_t* sel_tokens, float* out,
                                 float* lse, float* partial, int32_t* arrivals, int n_splits,
                                 unsigned long long* exchange, hipStream_t stream) {
#define LEOAM_FG(GG)                                                                                                   \
    launch_fused<T, GG>(s, score, q, K, V, chunk_off, n_chunks, max_chunks, token_budget, scale, sel_idx, sel_count,   \
                        sel_tokens, out, lse, partial, arrivals, n_splits, exchange, stream)
    switch (s->n_q_heads / s->n_kv_heads) {
    case 1: return LEOAM_FG(1);
    case 2: return LEOAM_FG(2);
    case 4: return LEOAM_FG(4);
    default: return LEOAM_FG(8);
    }
#undef LEOAM_FG
}

// Splits of a one-launch call, at most `cap` (what the workspace holds): as many workgroups as run at once, one per
// compute unit, each with an equal share of the tokens in granules; splits that this leaves without a share are not
// launched.  A launch of one round takes as long as its longest share, so within a round shorter shares pay for the
// merge of the splits, and a second round costs more than it saves.  Microseconds with 1 / 2 / 3 splits:
// bf16, four heads per group, 128 (b,h), 1024 tokens 23.2 / 20.2 / 31.9; 96 (b,h), 512 tokens
// 15.3 / 13.2 / -; 192 (b,h), 1024 tokens 26.8 / 35.4 / 37.1; compressed store, 128 (b,h), 2048 tokens
// 49.2 / 34.8 / 59.6.  Over 4 to 256 (b,h), 256 to 8192 tokens, every type and 1 to 8 heads per group, the count taken
// here is 0.4 % off the best one on average and 12 % at most (144 (b,h), fp32 and the compressed store: three splits).
static int fused_pick_splits(int units, int tokens, int granule, int cap) {
    int n = kFusedTargetWgs / units;
    if (n > cap) n = cap;
    if (n < 1) n = 1;
    const int per_split = ((tokens + n - 1) / n + granule - 1) / granule * granule;
    return (tokens + per_split - 1) / per_split;
}

// Tokens a call keeps per (b,h), as far as the host can tell: the budget, or without one the most chunks that can be
// kept, at the average size of c_max chunks.
static int expected_tokens(const leoam_shape* s, int max_chunks, int token_budget) {
    if (token_budget > 0) return token_budget < s->n_ctx ? token_budget : s->n_ctx;
    const long long chunks = max_chunks > 0 && max_chunks < s->k_max ? max_chunks : s->k_max;
    const long long tokens = chunks * ((s->n_ctx + s->c_max - 1ll) / s->c_max);
    return tokens < s->n_ctx ? (int)tokens : s->n_ctx;
}

// fp32, up to four heads per group: a workgroup has its compute unit to itself, while three of the separate kernel's
// share one, so the one launch loses where few workgroups run last.  Microseconds, one launch against separate kernels,
// 4096 tokens, one head: 256 (b,h) 184 / 198, 257 271 / 217, 320 281 / 249, 384 297 / 288, 400 298 / 328, 512 356 / 379,
// 528 449 / 420, 608 461 / 452, 640 467 / 467; two heads: 257 272 / 223, 336 287 / 263, 400 301 / 338, 528 450 / 441;
// four heads: 257 281 / 265, 304 290 / 302.  Short lists gain more from the launch that is saved (257 (b,h): two heads
// 256 tokens 25.6 / 26.9, 384 34.2 / 32.6, four heads 512 tokens 46.5 / 48.4, 768 64.8 / 61.1), unless a compute unit
// takes many one after the other: one head, 1024 (b,h) 128 tokens 43.2 / 37.2, 256 62.4 / 58.9, 512 107 / 106, 768
// 149 / 153; 700 (b,h) 64 tokens 21.8 / 18.8, 128 32.6 / 33.3; two heads 1024 (b,h) 128 tokens 44.1 / 39.7, 256 63.4 /
// 62.2, 384 86.9 / 86.9; four heads 1100 (b,h) 64 tokens 36.3 / 33.6, 192 66.0 / 66.7.
// Little more than half as many lists as compute units, of uneven length: one head, 24 chunks (1752 tokens on average)
// 129 (b,h) 71.1 / 61.8, 144 67.7 / 65.7, 156 69.0 / 69.7; 12 chunks 132 39.9 / 39.5; two heads 129 67.6 / 64.4, 140
// 67.6 / 69.7.
static bool one_launch_pays_f32(int G, long long units, int tokens, bool even) {
    const long long rounds = (units + kFusedTargetWgs - 1) / kFusedTargetWgs, last = (units - 1) % kFusedTargetWgs + 1;
    const long long over_half = units - kFusedTargetWgs / 2;
    if (rounds == 1) return even || G > 2 || over_half <= 0 || over_half * G > 24 || tokens < 1024 * G;
    if (rounds == 2) return last > (G == 1 ? 128 : G == 2 ? 80 : 32) || tokens < 192 * G;
    if (rounds == 3) return G > 2 || (tokens > 96 && (G == 2 || last > 128));
    return tokens > (G == 1 ? 512 : G == 2 ? 256 : 96);
}

// Whether a shape that the one-launch kernel can take is also faster there (`even`: the lists of all (b,h) hold about
// the same number of tokens, as with a budget).  With eight heads per group both halves of
// its waves request every K and V row, so it streams at 3 TB/s where the separate kernels reach 5: it wins as long as
// what it saves (a launch, two with the merge: 6 to 20 us) is more than that costs.  Microseconds, one launch against
// separate kernels, bf16: 64 (b,h) x 4096 tokens 48.6 / 50.6, 96 x 3072 53.7 / 53.2, 96 x 4096 66.6 / 60.8, 256 x 1024
// 48.8 / 50.8, 256 x 1536 67.8 / 61.3; past one workgroup per compute unit 512 x 256 36.1 / 39.8, 384 x 512 49.6 / 44.8,
// 512 x 4096 360 / 212.  fp32 (the separate kernel multiplies on the vector ALU): 160 x 4096 243 / 257, 192 x 4096
// 279 / 268, 256 x 2048 176 / 195, 256 x 3072 271 / 268; 512 x 512 96 / 106, 320 x 1024 140 / 137, 512 x 4096 703 / 610.
// Where the splits do not divide the compute units well it also loses by the length of a workgroup's share: 129 (b,h),
// one split each, bf16 1200 tokens 43.5 / 44.8, 1400 48.2 / 47.3, 2000 61.2 / 54.2; 86 (b,h), two splits, 2048 tokens
// 39.9 / 42.9, 2600 51.0 / 47.2; 257 (b,h) 320 tokens 34.7 / 34.4, 448 41.5 / 38.4; fp32 129 (b,h) 2000 tokens
// 117 / 129, 3000 177 / 168, 5000 309 / 260; 257 (b,h) 640 tokens 86.6 / 90.2, 1000 131 / 122.
// Without a budget the lists differ in length and the longest, about 4/3 of the average, sets the pace of a round
// of whole lists: bf16, 160 (b,h), chunk limit of 12 (876 tokens on average) 41.8 / 42.7, of 16 51.0 / 47.2; 130 (b,h),
// limit of 24 64.5 / 52.9.  Many short lists: 800 (b,h), 96 tokens 34.0 / 36.2, 128 40.9 / 39.3, limit of 2 52.5 / 44.9.
static bool one_launch_pays(const leoam_shape* s, int tokens, bool even) {
    const int G = s->n_q_heads / s->n_kv_heads;
    const long long units = (long long)s->batch * s->n_kv_heads;
    if (G <= kFusedHeads) return s->kv_dtype != LEOAM_F32 || one_launch_pays_f32(G, units, tokens, even);
    const long long rounds = (units + kFusedTargetWgs - 1) / kFusedTargetWgs;
    const int splits = rounds == 1 ? kFusedTargetWgs / (int)units : 1;
    if (s->kv_dtype == LEOAM_F32)
        return (tokens + splits - 1) / splits <= (rounds == 1 ? 3072 : 800) && units * tokens <= (rounds == 1 ? 5 << 17 : 1 << 18);
    if (!even && splits == 1) tokens = (int)std::min((tokens * 4ll + 2) / 3, (long long)s->n_ctx);
    return (tokens + splits - 1) / splits <= (rounds == 1 ? 1200 : rounds <= 3 ? 320 : 96) &&
           units * tokens <= (rounds == 1 ? 1 << 18 : 1 << 17);
}

hipError_t select_attention_dispatch(const leoam_shape* s, const float* score, const void* q, const void* K,
                                     const void* V, const void* qmeta, const int32_t* chunk_off,
                                     const int32_t* n_chunks, int max_chunks, int token_budget, float scale,
                                     int32_t* sel_idx, int32_t* sel_count, int32_t* sel_tokens, float* out, float* lse,
                                     void* workspace, size_t workspace_bytes, hipStream_t stream, bool with_exchange) {
    const size_t head = control_bytes(s, with_exchange);
    char* body = (char*)workspace + head;
    const size_t body_bytes = workspace_bytes - head;
    unsigned long long* exchange = (with_exchange && exchange_bytes(s) > 0)
                                       ? (unsigned long long*)((char*)workspace + arrival_bytes(s))
                                       : nullptr;
    if (stream_ordered_merge_wanted()) {
        // the kernels of the separate calls, splits combined by a kernel of their own: every hand-over
        // between workgroups is then ordered by the stream
        if (body_bytes < attention_min_workspace_bytes(s)) return hipErrorInvalidValue;
        hipError_t e = score ? topk_select_dispatch(s, score, chunk_off, n_chunks, max_chunks, token_budget, sel_idx,
                                                    sel_count, sel_tokens, stream)
                             : hipSuccess;
        if (e != hipSuccess) return e;
        return attention_dispatch(s, q, K, V, qmeta, chunk_off, n_chunks, sel_idx, sel_count, scale, out, lse, body,
                                  body_bytes, nullptr, stream);
    }
    if (select_attention_q_is_fused(s)) {
        // the compressed store's one-launch kernel (select_attention_q.hip)
        size_t n = body_bytes / fused_part_bytes_per_split(s);
        const int tokens = token_budget > 0 && token_budget < s->n_ctx ? token_budget : s->n_ctx;
        const size_t cap = (size_t)fused_q_recommended_splits(s, tokens);
        if (n > cap) n = cap;
        if (n < 1) n = 1;
        n = (size_t)fused_pick_splits(s->batch * s->n_kv_heads, tokens, kFusedWaves * 16, (int)n);
        return select_attention_q_dispatch(s, score, q, K, V, qmeta, chunk_off, n_chunks, max_chunks, token_budget, scale,
                                           sel_idx, sel_count, sel_tokens, out, lse, (float*)body, (int32_t*)workspace,
                                           (int)n, stream);
    }
    if (!select_attention_is_fused(s) || !one_launch_pays(s, expected_tokens(s, max_chunks, token_budget), token_budget > 0)) {
        hipError_t e = score ? topk_select_dispatch(s, score, chunk_off, n_chunks, max_chunks, token_budget, sel_idx,
                                                    sel_count, sel_tokens, stream)
                             : hipSuccess;
        if (e != hipSuccess) return e;
        // the attention kernel merges its splits in the same launch, with the arrival counters of this workspace
        return attention_dispatch(s, q, K, V, qmeta, chunk_off, n_chunks, sel_idx, sel_count, scale, out, lse, body,
                                  body_bytes, (int32_t*)workspace, stream);
    }
    size_t n = body_bytes / fused_part_bytes_per_split(s);
    const int tokens = token_budget > 0 && token_budget < s->n_ctx ? token_budget : s->n_ctx;
    const size_t cap = (size_t)fused_recommended_splits(s, tokens);
    if (n > cap) n = cap;
    if (n < 1) n = 1;      // a single split needs no partials
    const int n_splits = fused_pick_splits(s->batch * s->n_kv_heads, tokens, fused_granule(s), (int)n);
    if (s->kv_dtype == LEOAM_F32)
        return fused_by_group<F32>(s, score, q, K, V, chunk_off, n_chunks, max_chunks, token_budget, scale, sel_idx,
                                   sel_count, sel_tokens, out, lse, (float*)body, (int32_t*)workspace, n_splits, exchange,
                                   stream);
    if (s->kv_dtype == LEOAM_F16)
        return fused_by_group<F16>(s, score, q, K, V, chunk_off, n_chunks, max_chunks, token_budget, scale, sel_idx,
                                   sel_count, sel_tokens, out, lse, (float*)body, (int32_t*)workspace, n_splits, exchange,
                                   stream);
    return fused_by_group<BF16>(s, score, q, K, V, chunk_off, n_chunks, max_chunks, token_budget, scale, sel_idx,
                                sel_count, sel_tokens, out, lse, (float*)body, (int32_t*)workspace, n_splits, exchange, stream);
}

}  // namespace leoam
