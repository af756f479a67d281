// Causal varlen prefill attention (Sections 2.1, 3.1, 3.4) on the matrix cores over keys that were rotated beforehand:
// rotate_keys_kernel writes the batch's keys at their rebased positions into a scratch copy once per layer, attn_prerot_kernel
// reads them from there and the values from the pool.  Used where many row tiles share the keys of a (conversation, kv
// head); ca_attn_dma.hip serves the other batches, with the rotation inside the kernel.  What is computed, the stacked rows, the
// transposed formulation, the layout of a tile in LDS, the loads that bring it there and the shares of split keys are those
// described at the head of that file.
//
// What bounds it (256 rows x 64 keys, heads of 128, one workgroup per compute unit): a tile is 2176 cycles of
// matrix instructions per SIMD (two wavefronts x (32 instructions x 32 cycles + 8 of 8 for the row sums)), and with all compute
// units busy the card lowers its clock from 2.4 to 1.6-1.75 GHz, so instructions taken out count as much as cycles.
// Loads have to land within a tile of the one they were issued in (the rings hold no more): traffic over the host link in both
// directions at once is felt (save_workgroups in ca_lib.hip).  With 255 registers nothing else runs on the unit; that
// costs the attention 5 % beside 24 workgroups that only keep their places.  Measured in cycles a
// tile, and us a layer for 64 conversations of 1024-4096 + 64-512 tokens, 64 query and 8 kv heads: looking for the
// maximum of every tile, v_dot2c row sums and all wavefronts in lock step 3490 and 1860; probabilities checked instead
// of scores and the scores of the next tile formed under the softmax of this one 3155; two groups of wavefronts half a
// tile apart 3090; row sums on 4x4x4 products 2810; the order of operand reads pinned 2810 and 1750.
#include "ca_device.h"
#include "ca_internal.h"

#include <type_traits>

namespace ca {

namespace {

#define CA_INLINE __attribute__((always_inline))   // (a lambda left as a function keeps the kernel's registers in memory)

// Instruction kinds of __builtin_amdgcn_sched_group_barrier
constexpr int kMfma = 0x008, kVector = 0x402 /* plain and transcendental */, kLdsRead = 0x100;

constexpr int kMaxPagesLds = 2048;   // page ids kept in LDS at a time: a window of 32768 tokens that moves with the walk

// NW wavefronts (32 stacked query rows each) per workgroup, key tiles of BN.  Two shapes are built: NW = 8, BN = 64 (256-row
// tiles, one workgroup per compute unit) and NW = 4, BN = 32 (128-row tiles, several independent workgroups).
// OCC = wavefronts per SIMD the register budget is cut for.
template <int D, int STYLE, int NW, int BN, int OCC>
__global__ __launch_bounds__(64 * NW, OCC) void attn_prerot_kernel(AttnArgs a) {
    // PIPE: the scores of tile T+1 are formed under the softmax of tile T.  TWO: wavefronts w and w + 4, which share a SIMD,
    // are half a tile apart: one has its second product while the other has first product and softmax.  With heads of 64
    // there are several workgroups to a compute unit instead, none in step with another.
    constexpr bool PIPE = D == 128, TWO = PIPE && NW == 8;
    constexpr int NTHREADS = 64 * NW;
    constexpr int MB = BN / 32;              // 32-key blocks of S^T per tile
    constexpr int KS2 = BN / 16;             // 16-key steps of the second product per tile
    constexpr int KSTEPS = D / 16;           // k-steps of the S^T product
    constexpr int DBLKS = D / 32;            // 32-row blocks of O^T
    constexpr int PPR = D / 8;               // 16-byte pieces per row
    constexpr int KPC = 64 / PPR;            // keys per 1 KiB chunk
    constexpr int CHUNKS = BN / KPC;         // chunks per K (or V) tile
    constexpr int CH = 1024 + KPC * 16;      // chunk stride in LDS (bytes)
    constexpr int TILE = CHUNKS * CH;        // bytes of one K (or V) tile in LDS
    constexpr int NC = CHUNKS / NW;          // chunks of K (and of V) a wavefront loads per tile
    constexpr int NI = 2 * NC;               // load instructions per thread and tile (K and V)
    constexpr int PPT = BN / kPageSize;      // pages per tile
    // Iteration T issues the loads of K of tile T + KA and V of tile T + VA.  K of tile T+1 is wanted in it with PIPE, K of
    // tile T stays until its end for the case that the scores have to be formed again; V of tile T stays until the second
    // group is through with it in T+1.
    constexpr int KA = 3, VA = PIPE ? 2 : 3;
    constexpr int NSK = 4, NSV = 4;          // stages of the two rings
    // iterations whose loads may still be in flight at the end of one: only its own, and where the next one needs nothing
    // but tile T+1 those of the one before as well
    constexpr int FLY = PIPE ? 1 : 2;
    constexpr int LDS_LEFT = 160 * 1024 / (OCC * 4 / NW) - (NSK + NSV) * TILE;
    constexpr int PGW = LDS_LEFT / 4 < kMaxPagesLds ? LDS_LEFT / 4 / 64 * 64 : kMaxPagesLds;   // page ids kept in LDS at a time
    static_assert(CHUNKS % NW == 0 && (NC == 1 || NW * KPC % kPageSize == 0), "a wavefront's chunks lie at the same rows of their pages");
    static_assert(PGW >= 16 * PPT, "LDS budget");

    __shared__ __attribute__((aligned(16))) uint8_t ring_k[NSK * TILE];
    __shared__ __attribute__((aligned(16))) uint8_t ring_v[NSV * TILE];
    __shared__ int32_t pg[PGW];

    const WorkItem item = a.items[blockIdx.x];
    if (item.seq < 0) return;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int lq = lane & 31;
    const int half = lane >> 5;

    const int c = item.seq;
    const int g = item.kv_head;
    const int G = a.n_q_heads / a.n_kv_heads;
    const int n = a.n_keep[c];
    const int q0 = a.cu_q[c];
    const int32_t *table = a.block_table + (int64_t)c * a.max_pages;
    const int Hkv = a.n_kv_heads;

    const int row_last = item.row0 + item.n_rows - 1;          // last valid stacked row of the tile
    // keys [key_begin, kmax): what the tile's rows can see, cut to the item's share when the keys of one
    // row tile are split over several workgroups (key_begin and a cutting key_end are multiples of 64)
    const int kmax = min(n + row_last / G + 1, item.key_end);
    const int t_begin = item.key_begin / BN;
    const int n_tiles = (kmax + BN - 1) / BN;                   // end of the walk (absolute tile index)

    // page ids of the visible context -> LDS, a window of PGW pages starting at the first tile's page; the
    // walk moves the window on when the lookups it makes ahead would leave it
    const int n_pages = (kmax + kPageSize - 1) / kPageSize;
    int pg_base = t_begin * PPT;
    for (int i = tid; i < min(PGW, n_pages - pg_base); i += NTHREADS) pg[i] = table[pg_base + i];

    // ---- this lane's query row --------------------------------------------------------------
    const int r_raw = item.row0 + wave * 32 + lq;
    const bool row_valid = r_raw <= row_last;
    const int r = row_valid ? r_raw : row_last;
    const int j = r / G;
    const int qpos = n + j;                                      // keys 0..qpos are visible
    const int wr_first = min(item.row0 + wave * 32, row_last);
    const int wr_last = min(item.row0 + wave * 32 + 31, row_last);
    const bool wave_live = item.row0 + wave * 32 <= row_last;
    const int wq_min = n + wr_first / G;
    const int wq_max = n + wr_last / G;

    // The softmax scale and log2(e) are folded into the rotated query before it is rounded to bf16, so the scores
    // come out of the matrix cores in the units of the base-2 exponent.
    const float cscale = a.softmax_scale * 1.4426950408889634f;
    bf16x8 Qf[KSTEPS];          // asked for before the page ids arrive, rotated in the prologue behind the first loads

    // ---- operand addresses inside a stage ---------------------------------------------------------------
    // K, A operand of S^T: key 32mb + lq, piece 2ks + half  ->  + ks * 2*KPC*16 and + mb * (32/KPC)*CH as immediates
    const int k_rd = (lq / KPC) * CH + (half * KPC + lq % KPC) * 16;
    constexpr int K_MB = (32 / KPC) * CH;
    // V, A operand of O^T via transposing reads: lane s of a 16-lane group points at key k0 + s/4,
    // dims d0 + 4*(s%4) .. +3 and receives dims d0 + s of keys k0..k0+3
    const int s16 = lane & 15;
    const int dsel = (lane >> 4) & 1;
    int v_rd;
    {
        const int piece_lo = 2 * dsel + ((s16 & 3) >> 1);      // + 4*db
        const int kl = (D == 128) ? (s16 >> 2) : (4 * half + (s16 >> 2));
        v_rd = (piece_lo * KPC + kl) * 16 + (s16 & 1) * 8 + ((D == 128) ? half * CH : 0);
    }

    // ---- loads: chunks wave, wave + NW, .. of K and of V; lane -> key lane % KPC of the chunk, piece lane / KPC ----------
    const uint32_t page_bytes = (uint32_t)(Hkv * kPageSize * D * 2);
    const auto page_at = [&](const uint8_t *pool, int page) CA_INLINE { return pool + (uint64_t)(uint32_t)page * page_bytes; };
    const uint8_t *const k_src = reinterpret_cast<const uint8_t *>(a.k_rot);
    const uint8_t *const v_src = reinterpret_cast<const uint8_t *>(a.v_pool);
    const int k_page0 = a.dense_page0[c];                    // key page i of the conversation is k_page0 + i
    const uint32_t ld_k = __builtin_amdgcn_readfirstlane(lds_offset(ring_k)) + (uint32_t)(wave * CH);
    const uint32_t ld_v = __builtin_amdgcn_readfirstlane(lds_offset(ring_v)) + (uint32_t)(wave * CH);
    // byte offset of this lane inside a page
    const uint32_t ld_lane = (uint32_t)((g * kPageSize + wave * KPC % kPageSize + lane % KPC) * D + (lane / KPC) * 8) * 2u;
    auto issue = [&](int tile, auto is_v) CA_INLINE {
        constexpr bool V = decltype(is_v)::value;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int t = min(tile * BN + (wave + NW * i) * KPC + lane % KPC, kmax - 1);
            const int page = V ? pg[(t >> 4) - pg_base] : k_page0 + (t >> 4);
            const int64_t in_page = (int64_t)((g * kPageSize + (t & 15)) * D + (lane / KPC) * 8) * 2;
            dma16(page_at(V ? v_src : k_src, page) + in_page,
                  (V ? ld_v + (uint32_t)tile % NSV * TILE : ld_k + (uint32_t)tile % NSK * TILE) + (uint32_t)(NW * i * CH));
        }
    };

    // Interior tiles need no clamping: all lanes of one load read rows of the same page, so the address up to the
    // lane's constant offset is wave-uniform (scalar ALU).  The page ids are read from LDS ahead of
    // the matrix instructions between which the loads go out.
    int v_ahead[NC];
    auto look_up = [&](int tile) CA_INLINE {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            v_ahead[i] = pg[(tile + VA) * PPT + (wave + NW * i) * KPC / kPageSize - pg_base];
        }
    };
    auto issue_interior = [&](int tile, int i, bool is_v) CA_INLINE {       // chunk i of K or of V
        if (is_v)
            dma16_sbase(page_at(v_src, __builtin_amdgcn_readfirstlane(v_ahead[i])), ld_lane, ld_v + (uint32_t)(tile + VA) % NSV * TILE + (uint32_t)(NW * i * CH));
        else
            dma16_sbase(page_at(k_src, k_page0 + (tile + KA) * PPT + (wave + NW * i) * KPC / kPageSize), ld_lane,
                        ld_k + (uint32_t)(tile + KA) % NSK * TILE + (uint32_t)(NW * i * CH));
    };
    const auto stage_k = [&](int tile) CA_INLINE { return ring_k + (uint32_t)tile % NSK * TILE; };
    const auto stage_v = [&](int tile) CA_INLINE { return ring_v + (uint32_t)tile % NSV * TILE; };

    f32x16 O[DBLKS];
#pragma unroll
    for (int db = 0; db < DBLKS; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
    // ref = what is subtracted from the scores of this lane's query row, in exponent units (-inf: no key seen yet): the row's
    // maximum when it was last moved plus kHeadroom, so that a probability reaches 2 only where a score lies kHeadroom + 1
    // above that maximum.  neg_ref holds -ref (0 while there is none) in the C layout and is the accumulator input of the
    // first matrix instruction of every tile: the scores arrive already relative to it.
    constexpr float kHeadroom = 7.0f;
    float ref = -INFINITY;
    float ref0 = 0.f;                    // ref, 0 while there is none
    f32x16 neg_ref = {};
    // Row sums of the rounded probabilities, the very values the second product multiplies: 4x4x4 products with ones, in
    // which every lane gets the sum of its own four (all four elements alike; the first one counts).  They take 8 cycles
    // of the matrix cores for four values; v_dot2c, two values, waits for the matrix instructions of the SIMD's
    // other wavefronts in front of it, one after the other: 280 to 570 cycles for the 16 of a tile.
    f32x4 row_sum = {0.f, 0.f, 0.f, 0.f};
    const s16x4 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};

    // ---- prologue ---------------------------------------------------------------------------------------
    // the queries are asked for before the page ids arrive, and rotated behind the loads of the first tiles
    QueryRows<D, STYLE> rows;
    if (wave_live) rows.fetch(a, q0, g, G, n, item.row0 + wave * 32, row_last);
    __syncthreads();                     // page ids are in LDS
#pragma unroll
    for (int k = 0; k < KA - 1; ++k)
        if (t_begin + k < n_tiles) issue(t_begin + k, std::false_type{});
#pragma unroll
    for (int k = 0; k < VA - 1; ++k)
        if (t_begin + k < n_tiles) issue(t_begin + k, std::true_type{});
    // they pass through the third and fourth stage of either ring
    constexpr int QPT = NW / 4;          // wavefronts per stage
    static_assert(QueryRows<D, STYLE>::kQueryBytes * QPT <= TILE && KA == 3 && VA <= 3, "the queries fit the stages without loads");
    if (wave_live)
        rows.finish((wave / QPT < 2 ? stage_k(t_begin + 2 + wave / QPT) : stage_v(t_begin + wave / QPT)) + wave % QPT * QueryRows<D, STYLE>::kQueryBytes,
                    cscale, Qf);
    CA_WAIT_VMCNT(0);
    __syncthreads();
    // what may stay in flight when the walk begins
    if (t_begin + KA - 1 < n_tiles) issue(t_begin + KA - 1, std::false_type{});
    if (t_begin + VA - 1 < n_tiles) issue(t_begin + VA - 1, std::true_type{});
    // first product of a tile: the keys are read KD steps ahead
    constexpr int KD = 2;
    bf16x8 kf[KD][MB];
    auto key_step = [&](const uint8_t *st, int ks) CA_INLINE {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) kf[ks % KD][mb] = *reinterpret_cast<const bf16x8 *>(st + k_rd + mb * K_MB + ks * (2 * KPC * 16));
    };
    auto score_step = [&](f32x16 (&S)[MB], const uint8_t *st, int ks) CA_INLINE {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            S[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks % KD][mb], Qf[ks], ks == 0 ? neg_ref : S[mb], 0, 0, 0);
        }
        if (ks + KD < KSTEPS) key_step(st, ks + KD);
    };
    auto first_keys = [&](const uint8_t *st) CA_INLINE {
#pragma unroll
        for (int ks = 0; ks < KD; ++ks) key_step(st, ks);
    };
    auto all_scores = [&](f32x16 (&S)[MB], const uint8_t *st) CA_INLINE {
        first_keys(st);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) score_step(S, st, ks);
    };
    // two probabilities of a tile as a bf16 pair
    auto exp_pair = [&](const f32x16 (&S)[MB], int w) CA_INLINE {
        const int mb = w / 8, i = 2 * (w % 8);
        return pack_bf16(__builtin_amdgcn_exp2f(S[mb][i]), __builtin_amdgcn_exp2f(S[mb][i + 1]));
    };

    // Moves the reference to the maximum of this tile (S; Snxt: scores of the next tile, formed against the old reference)
    // where that is more than `above` over the reference, and rescales what was summed so far.
    auto raise_reference = [&](f32x16 (&S)[MB], f32x16 (&Snxt)[MB], float above) CA_INLINE {
        float mx = S[0][0];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[mb][i]);
        {   // lanes l and l+32 hold the two key halves of one query row: one swap gives both the other half
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        }
        // mx is relative to the reference.  A row whose keys so far were all masked (possible when the keys of a row
        // tile are split) has mx = -inf and stays without a reference: its probabilities are exp2(-inf) = 0.
        const bool unseen = ref == -INFINITY;
        const bool raise = mx > -INFINITY && (unseen || mx > above);
        if (__builtin_amdgcn_ballot_w64(raise) != 0) {
            const float delta = raise ? mx + kHeadroom : 0.f;
            // (a first reference rescales nothing: the sums are still zero, and exp2(-delta) could overflow)
            const float alpha = (raise && !unseen) ? __builtin_amdgcn_exp2f(-delta) : 1.0f;
            if (raise) ref = ref0 = ref0 + delta;
            row_sum[0] *= alpha;
#pragma unroll
            for (int db = 0; db < DBLKS; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) O[db][i] *= alpha;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    S[mb][i] -= delta;
                    if (PIPE) Snxt[mb][i] -= delta;
                }
#pragma unroll
            for (int i = 0; i < 16; ++i) neg_ref[i] = -ref0;
        }
    };

    // second product of a tile: its probabilities pk on its values, which are read VD operands ahead
    uint32_t pk[8 * MB];
    constexpr int VD = 4, VN = KS2 * DBLKS;
    s16x8 vf[VD];
    auto value_read = [&](const uint8_t *st, int o) CA_INLINE {
        // keys 16ks2 + 4half + 0..3 and 16ks2 + 8 + 4half + 0..3 of dims 32db + lq
        const int ks2 = o / DBLKS, db = o % DBLKS;
        const int o0 = (D == 128 ? (4 * ks2) * CH : (2 * ks2) * CH) + 4 * db * KPC * 16;
        const int o1 = (D == 128 ? (4 * ks2 + 2) * CH : (2 * ks2 + 1) * CH) + 4 * db * KPC * 16;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(st + v_rd + o0));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(st + v_rd + o1));
        vf[o % VD] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto first_values = [&](const uint8_t *st) CA_INLINE {
#pragma unroll
        for (int o = 0; o < VD; ++o) value_read(st, o);
    };
    auto value_product = [&](const uint8_t *st) CA_INLINE {
#pragma unroll
        for (int o = 0; o < VN; ++o) {
            const int ks2 = o / DBLKS, db = o % DBLKS;
            const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(pk[4 * ks2], pk[4 * ks2 + 1], pk[4 * ks2 + 2], pk[4 * ks2 + 3]));
            O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf[o % VD]), pb, O[db], 0, 0, 0);
            if (db < 2) row_sum = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, make_uint2(pk[4 * ks2 + 2 * db], pk[4 * ks2 + 2 * db + 1])), row_sum, 0, 0, 0);
            if (o + VD < VN) value_read(st, o + VD);
        }
        // keep it so: the compiler would read four operands at a time and wait for them
#pragma unroll
        for (int o = 0; o < VN; ++o) {
            __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
            if (o + VD < VN) __builtin_amdgcn_sched_group_barrier(kLdsRead, 2, 0);
            if (o % DBLKS < 2) __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
        }
    };

    // One key tile.  S: its scores (PIPE: formed already), Snxt: those of the next tile.  SECOND: a wavefront of the second
    // group, which multiplies the values of the previous tile first and those of this one in the next iteration (pending).
    bool pending = false;
    auto walk = [&](int tile, auto interior_tag, auto live_tag, auto second_tag, f32x16 (&S)[MB], f32x16 (&Snxt)[MB]) CA_INLINE {
        constexpr bool INTERIOR = decltype(interior_tag)::value;
        constexpr bool LIVE = decltype(live_tag)::value;
        constexpr bool SECOND = decltype(second_tag)::value;
        const int kt0 = tile * BN;
        // move the page-id window when the lookups of this iteration would fall outside it (every wavefront has left those
        // of the previous iteration behind: barrier at its end)
        if ((tile + KA + 1) * PPT > pg_base + PGW) {
            pg_base = tile * PPT;
            for (int i = tid; i < min(PGW, n_pages - pg_base); i += NTHREADS) pg[i] = table[pg_base + i];
            __syncthreads();
        }
        const bool compute = LIVE && (INTERIOR || kt0 <= wq_max);

        const bool scores = LIVE && (PIPE ? INTERIOR || (tile + 1 < n_tiles && kt0 + BN <= wq_max) : compute);
        const uint8_t *const st_k = stage_k(PIPE ? tile + 1 : tile);
        if (INTERIOR) look_up(tile);
        if (SECOND) first_values(stage_v(tile - 1));
        else if (scores) first_keys(st_k);
        if (INTERIOR && !LIVE) {
#pragma unroll
            for (int i = 0; i < NI; ++i) issue_interior(tile, i / 2, i % 2);
        } else if (!INTERIOR) {
            if (tile + KA < n_tiles) issue(tile + KA, std::false_type{});
            if (tile + VA < n_tiles) issue(tile + VA, std::true_type{});
        }
        __builtin_amdgcn_sched_barrier(0);
        if (SECOND && pending) value_product(stage_v(tile - 1));
        if (SECOND && scores) {
            first_keys(st_k);
            __builtin_amdgcn_sched_barrier(0);
        }

        if (scores) {
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                score_step(PIPE ? Snxt : S, st_k, ks);
                if (INTERIOR && ks >= 1 && ks <= NI) issue_interior(tile, (ks - 1) / 2, (ks - 1) % 2);
                if (PIPE && INTERIOR) {
#pragma unroll
                    for (int w = ks * 8 * MB / KSTEPS; w < (ks + 1) * 8 * MB / KSTEPS; ++w) pk[w] = exp_pair(S, w);
                }
            }
            if (PIPE && INTERIOR) {
#pragma unroll
                for (int k = 0; k < KSTEPS * MB; ++k) {
                    __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
                    if (k < (KSTEPS - KD) * MB) __builtin_amdgcn_sched_group_barrier(kLdsRead, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(kVector, 4, 0);
                }
            }
        }

        if (compute) {
            if (!INTERIOR && kt0 + BN - 1 > wq_min) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int key = kt0 + 32 * mb + (i >> 2) * 8 + half * 4 + (i & 3);
                        if (key > qpos) S[mb][i] = -INFINITY;
                    }
            }
            auto probabilities = [&]() CA_INLINE {
#pragma unroll
                for (int w = 0; w < 8 * MB; ++w) pk[w] = exp_pair(S, w);
            };
            // The reference follows the maximum lazily: any value does as long as no probability becomes large.  Interior
            // tiles do not look for the maximum: whether some probability has reached 2 is one bit of its bf16 exponent,
            // and only then (or where a row has no reference yet) the reference is moved and the tile's probabilities are
            // formed again.  Other tiles look first.
            if (INTERIOR) {
                if (!PIPE) probabilities();
                uint32_t any = pk[0];
#pragma unroll
                for (int w = 1; w < 8 * MB; ++w) any |= pk[w];
                if (__builtin_expect(__builtin_amdgcn_ballot_w64((any & 0x40004000u) != 0 || ref == -INFINITY) != 0, 0)) {
                    all_scores(S, stage_k(tile));            // (the registers hold probabilities by now)
                    raise_reference(S, Snxt, -kHeadroom);
                    probabilities();
                }
            } else {
                raise_reference(S, Snxt, 1.0f);
                probabilities();
            }
            if (!SECOND) {
                first_values(stage_v(tile));
                __builtin_amdgcn_sched_barrier(0);
                value_product(stage_v(tile));
            }
        }
        if (SECOND) pending = compute;

        // what the next iteration needs must have landed; loads issued in this one may stay in flight
        if (INTERIOR || tile + KA < n_tiles) { CA_WAIT_VMCNT(FLY * NI); }
        else if (KA > VA && tile + VA < n_tiles) { CA_WAIT_VMCNT(NC); }
        else if (FLY == 2 && tile + KA - 1 < n_tiles) { CA_WAIT_VMCNT(NI); }
        else { CA_WAIT_VMCNT(0); }
        __syncthreads();
    };

    const int first_qpos = n + item.row0 / G;
    // end of the interior tiles: every row sees the whole tile, and the tiles loaded in it are complete
    const int n_interior = max(t_begin, min((first_qpos + 1) / BN, kmax / BN - KA));
    auto walk_all = [&](auto live_tag, auto second_tag) CA_INLINE {
        constexpr bool LIVE = decltype(live_tag)::value;
        int tile = t_begin;
        f32x16 S0[MB], S1[MB];
        if (LIVE && PIPE && t_begin * BN <= wq_max) all_scores(S0, stage_k(t_begin));
        if (LIVE && PIPE) {
            for (; tile + 1 < n_interior; tile += 2) {
                walk(tile, std::true_type{}, live_tag, second_tag, S0, S1);
                walk(tile + 1, std::true_type{}, live_tag, second_tag, S1, S0);
            }
        } else {
            for (; tile < n_interior; ++tile) walk(tile, std::true_type{}, live_tag, second_tag, S0, S1);
        }
        for (; tile < n_tiles; ++tile) {
            walk(tile, std::false_type{}, live_tag, second_tag, S0, S1);
            if (LIVE && PIPE) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) S0[mb] = S1[mb];
            }
        }
        if (decltype(second_tag)::value && pending) {
            first_values(stage_v(n_tiles - 1));
            value_product(stage_v(n_tiles - 1));
        }
    };
    if (!wave_live) walk_all(std::false_type{}, std::false_type{});
    else if (TWO && wave >= NW / 2) walk_all(std::true_type{}, std::integral_constant<bool, TWO>{});
    else walk_all(std::true_type{}, std::false_type{});

    // ---- epilogue: normalise and store --------------------------------------------------------------
    const float l_all = row_sum[0] + __shfl_xor(row_sum[0], 32);
    if (item.part >= 0) {
        // keys split over several workgroups: leave the unnormalised sums, the reference maximum and the
        // denominator of this share in the scratch buffer; combine_tiles_kernel merges the shares
        if (row_valid) {
            const int rt = r - item.row0;                       // row inside the tile
            float *base = a.partial + (int64_t)item.part * a.tile_rows * (D + 2);
#pragma unroll
            for (int db = 0; db < DBLKS; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const int d4 = 8 * db + 2 * i4 + half;
                    reinterpret_cast<float4 *>(base)[d4 * a.tile_rows + rt] = make_float4(O[db][4 * i4], O[db][4 * i4 + 1], O[db][4 * i4 + 2], O[db][4 * i4 + 3]);
                }
            if (half == 0) {
                base[(int64_t)a.tile_rows * D + rt] = ref / cscale;      // in score units
                base[(int64_t)a.tile_rows * (D + 1) + rt] = l_all;
            }
        }
        return;
    }
    // (every wavefront is through with the keys)
    if (wave_live)
        store_rows<D>(a, q0, g, G, item.row0 + wave * 32, row_last, ring_k + wave * QueryRows<D, STYLE>::kQueryBytes, O, 1.f / l_all);
}

// Rotates the keys of the whole batch context once (Section 3.4: the rebased positional encoding, applied
// when the cache is used): dense page dp of the scratch copy = pool page rot_src_page[dp] with token slot s
// rotated at position rot_pos0[dp] + s, in fp32 from the table, rounded to bf16 -- the same values the fused
// path forms tile by tile (there with the rotation advanced by recurrence).  Slots past the end of a context hold whatever
// the pool holds; nobody reads them.  Bound by HBM (one read, one write).  A workgroup has a dense page and HEADS kv heads, a thread one
// (token, pair of 16-byte pieces) of each: the table row is fetched once for all of them and their loads are all in flight.
// With a workgroup to a head and a table row each, 64 conversations of 1024-4096 + 64-512 tokens, 8 kv heads (350 MB of keys) took
// 157-170 us, now 129-143; loads that pass the cache by are 5 us of that, eight heads to a workgroup are as fast alone and slower
// beside loads.
template <int D, int STYLE, int HEADS>
__global__ __launch_bounds__(D) void rotate_keys_kernel(AttnArgs a) {
    constexpr int HALF = D / 2;
    constexpr int PAIRS = D / 16;                       // piece pairs per row
    static_assert(kPageSize * PAIRS == D, "one thread per (token of the page, piece pair)");
    const int slices = a.n_kv_heads / HEADS;
    const int dp = blockIdx.x / slices, g0 = blockIdx.x % slices * HEADS;
    const int key = threadIdx.x / PAIRS, pr = threadIdx.x % PAIRS;
    const int pos = min(a.rot_pos0[dp] + key, a.max_positions - 1);
    const uint16_t *src = a.k_pool + (((int64_t)a.rot_src_page[dp] * a.n_kv_heads + g0) * kPageSize + key) * D + 8 * pr;
    uint16_t *dst = a.k_rot + (((int64_t)dp * a.n_kv_heads + g0) * kPageSize + key) * D + 8 * pr;
    uint4 x[HEADS], y[HEADS];
#pragma unroll
    for (int g = 0; g < HEADS; ++g) {
        x[g] = __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + g * kPageSize * D)));
        y[g] = __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + g * kPageSize * D + HALF)));
    }
    float2 cs[8];
    load_cs<D, STYLE>(a.rope, pos, pr, cs);
#pragma unroll
    for (int g = 0; g < HEADS; ++g) {
        uint32_t *px = reinterpret_cast<uint32_t *>(&x[g]), *py = reinterpret_cast<uint32_t *>(&y[g]);
#pragma unroll
        for (int w = 0; w < 4; ++w) rotate_dword<STYLE>(px[w], py[w], cs, w);
        *reinterpret_cast<uint4 *>(dst + g * kPageSize * D) = x[g];
        *reinterpret_cast<uint4 *>(dst + g * kPageSize * D + HALF) = y[g];
    }
}

template <int D, int STYLE>
void launch_all(const AttnArgs &a, hipStream_t stream) {
    const int heads = a.n_kv_heads % 4 == 0 ? 4 : a.n_kv_heads % 2 == 0 ? 2 : 1;
    const dim3 rgrid((uint32_t)a.n_dense_pages * (uint32_t)(a.n_kv_heads / heads)), grid(a.n_items);
    if (heads == 4) hipLaunchKernelGGL((rotate_keys_kernel<D, STYLE, 4>), rgrid, dim3(D), 0, stream, a);
    else if (heads == 2) hipLaunchKernelGGL((rotate_keys_kernel<D, STYLE, 2>), rgrid, dim3(D), 0, stream, a);
    else hipLaunchKernelGGL((rotate_keys_kernel<D, STYLE, 1>), rgrid, dim3(D), 0, stream, a);
    if (a.tile_rows == 256) hipLaunchKernelGGL((attn_prerot_kernel<D, STYLE, 8, 64, 2>), grid, dim3(512), 0, stream, a);
    else if (D == 64 && a.wgs_per_cu == 4) hipLaunchKernelGGL((attn_prerot_kernel<D, STYLE, 4, 32, D == 64 ? 4 : 2>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((attn_prerot_kernel<D, STYLE, 4, 32, D == 64 ? 3 : 2>), grid, dim3(256), 0, stream, a);
}

}  // namespace

hipError_t launch_attn_prerot(const AttnArgs &a, hipStream_t stream) {
    if (a.n_items <= 0) return hipSuccess;
    if (a.n_combine > 0 && (a.partial == nullptr || a.combine == nullptr)) return hipErrorInvalidValue;
    if ((a.tile_rows != 256 && a.tile_rows != 128) || !a.k_rot || !a.dense_page0 || !a.rot_src_page || !a.rot_pos0 || a.n_dense_pages <= 0)
        return hipErrorInvalidValue;
    if (a.head_dim == 128 && a.rope_style == 0) launch_all<128, 0>(a, stream);
    else if (a.head_dim == 128) launch_all<128, 1>(a, stream);
    else if (a.head_dim == 64 && a.rope_style == 0) launch_all<64, 0>(a, stream);
    else if (a.head_dim == 64) launch_all<64, 1>(a, stream);
    else return hipErrorInvalidValue;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.n_combine <= 0) return e;
    return launch_combine_tiles(a, stream);
}

}  // namespace ca
