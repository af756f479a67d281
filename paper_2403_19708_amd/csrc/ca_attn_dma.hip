// Fused rotary-on-load + causal varlen prefill attention (Sections 2.1, 3.1, 3.4) on the matrix cores.
//
// out[j, h, :] = sum_t softmax_t(RoPE(q[j,h], n+j) . RoPE(k[t], t) * scale) v[t] over the context tokens t <= n + j of
// the conversation, bf16 in, fp32 accumulate, bf16 out.  One workgroup = NW wavefronts x 32 stacked query rows (row r
// of a (conversation, kv head) <-> new token r / G, query head kv*G + r % G, so the G heads of a group share every
// staged K/V tile), walking key tiles of BN with an online softmax.  v_mfma_f32_32x32x16_bf16 in the transposed
// formulation S^T = K Q^T, O^T += V^T P^T: in the C layout a lane owns one query column, so row maxima and sums are
// in-lane plus one exchange with lane ^ 32, and the C registers of S^T, converted to bf16, ARE the B operand of the
// second product.  The softmax scale and log2(e) are folded into the rotated query before it is rounded to bf16 and the
// running reference maximum enters the score product as its initial accumulator (-m), so the exponent's argument comes
// straight out of the matrix instruction.  The reference maximum is raised lazily (a wave-uniform branch, rare after
// the first tile).
// K/V tiles travel HBM -> LDS without passing through registers:
//
//   * global_load_lds (16 bytes per lane, written to LDS at base + lane*16) fills a ring of 4 tile
//     stages in LDS; the loads of tile T+3 are issued when tile T starts, so two to three tiles
//     (64-96 KiB per compute unit) are in flight while one is multiplied, and no vector register
//     is spent on staging.  The only vector-memory instructions inside the walk are these loads,
//     so s_waitcnt vmcnt(N) with a constant N releases exactly the tile that is needed next.
//   * The page ids of the conversation are kept in LDS (a window of 2048 pages that follows the walk); the dependent chain
//     block table -> page -> row costs an LDS read.  On interior tiles a load's page and base address
//     are wave-uniform: all page ids of an iteration are read before the first is used (one LDS round
//     trip), and the scalar address arithmetic and the loads are issued after the first matrix
//     instructions of the tile, where they cost nothing.
//   * An item may own only a share [key_begin, key_end) of the keys its rows see (the host splits long
//     row tiles over several workgroups when a batch would otherwise leave compute units idle).  Such an
//     item leaves unnormalised sums, reference maxima and denominators in a scratch buffer and
//     combine_tiles_kernel merges the shares of a row tile.
//   * Since the LDS side of such a load is fixed (lane l -> byte l*16 of a 1 KiB chunk), the layout
//     is chosen on the global side: a chunk holds KPC = 1024/(2D) keys, piece-major
//     (slot = piece*KPC + key_in_chunk), chunks padded by KPC*16 bytes.  With it the A-operand reads
//     of K (32 keys x one 16-byte piece), the in-place rotary pass and the transposing reads of V
//     are all bank-conflict free, and the offset of a piece is linear in the piece index, so the
//     per-k-step offsets are instruction immediates.
//   * K lands in LDS without positions; the workgroup rotates the NEXT tile in place (LDS -> fp32
//     rotate -> bf16 -> same LDS bytes) while the matrix cores work on the current one
//     (ca_attn_prerot.hip has the case of keys rotated beforehand).
//   * Bound by the rotary pass and by the load latency of single items, not by the softmax: row sums on 4x4x4 products
//     and tiles without a search for the maximum, part of 3490 -> 2810 cycles there, changed nothing here (4 layers
//     of 16 turns of 32-256 tokens 934 and 932 us, of 8 of 64-512 929 and 928).
//   * V is never transposed by the ALUs: ds_read_b64_tr_b16 hands each lane 4 consecutive keys of
//     one head dimension, which is exactly the A-operand layout of O^T += V^T P^T (two such reads
//     per operand, in the key order the C layout of S^T imposes on P^T).
//   * Keys past the end of the context are not zero-filled (a load cannot write zeros): the source
//     row is clamped to the last valid key, the causal mask gives those columns probability 0 and
//     the clamped V rows are finite data, so they contribute exactly nothing.
#include "ca_device.h"
#include "ca_internal.h"

#include <type_traits>

namespace ca {

namespace {

constexpr int kMaxPagesLds = 2048;   // page ids kept in LDS at a time: a window of 32768 tokens that moves with the walk

// NW wavefronts (32 stacked query rows each) per workgroup, key tiles of BN.  Two shapes are built:
// NW = 8, BN = 64 (one workgroup per compute unit, 256-row tiles) and NW = 4, BN = 32 (two independent
// workgroups per compute unit, 128-row tiles: the two wavefronts that share a SIMD then belong to
// different workgroups, are not in lock step, and one's matrix products run under the other's softmax).
// NS = LDS stages of the tile ring: the loads of tile T+NS-1 go out in iteration T.
// PGW = page ids kept in LDS at a time, OCC = wavefronts per SIMD the register budget is cut for.
template <int D, int STYLE, int NW, int BN, int NS = 4, int PGW = kMaxPagesLds, int OCC = 2>
__global__ __launch_bounds__(64 * NW, OCC) void attn_dma_kernel(AttnArgs a) {
    static_assert(NS == 4, "the in-place rotary pass needs a tile landed one iteration early");
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
    constexpr int STAGE = 2 * TILE;
    constexpr int NI = 2 * CHUNKS / NW;      // load instructions per thread and tile (K and V)
    constexpr int ROT_TASKS = BN * PPR / 2;  // (key, piece pair) tasks of the rotary pass
    static_assert(2 * CHUNKS % NW == 0, "chunks divide evenly over the wavefronts");
    static_assert((NW == 8 ? 1 : OCC) * (NS * STAGE + PGW * 4) <= 160 * 1024, "LDS budget");
    // loads that may still be in flight at the end of an interior iteration: tile+2 must have landed (it is rotated next)
    constexpr int FLY = NI;

    __shared__ __attribute__((aligned(16))) uint8_t ring[NS * STAGE];
    __shared__ int32_t pg[PGW];

    const WorkItem item = a.items[blockIdx.x];
    if (item.seq < 0) return;

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
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

    // page ids of the visible context -> LDS, a window of kMaxPagesLds pages starting at the first tile's page; the
    // walk moves the window on when the loads it issues ahead would leave it (once per 32768 keys)
    const int n_pages = (kmax + kPageSize - 1) / kPageSize;
    int pg_base = t_begin * (BN / kPageSize);
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

    // ---- rotary pass: this thread's (key, piece pair) of every K tile ------------------------------
    const bool rot_active = ROT_TASKS >= NTHREADS || tid < ROT_TASKS;
    // 16 consecutive lanes take the KPC keys of a chunk times consecutive pieces = 16 consecutive 16-byte
    // slots, so the 16-byte LDS accesses of the pass are free of bank conflicts (key-major lanes were 2-way)
    const int rot_kk = (tid / (KPC * (PPR / 2))) * KPC + tid % KPC;
    const int rot_pr = (tid / KPC) % (PPR / 2);
    const int rot_off = (rot_kk / KPC) * CH + (rot_pr * KPC + rot_kk % KPC) * 16;   // piece rot_pr; partner +512
    constexpr int ROT_PARTNER = (PPR / 2) * KPC * 16;
    float2 k_step[8], k_cs[8];
    load_cs<D, STYLE>(a.rope, BN, rot_pr, k_step);
    // first position of this thread's key; a thread whose first key lies past the visible range never sees a
    // visible one later either, so clamping it is harmless (and keeps the read inside the table)
    load_cs<D, STYLE>(a.rope, rot_active ? min(t_begin * BN + rot_kk, kmax - 1) : 0, rot_pr, k_cs);
    uint4 kx, ky;

    // ---- operand addresses inside a stage ---------------------------------------------------------------
    // K, A operand of S^T: key 32mb + lq, piece 2ks + half  ->  + ks * 2*KPC*16 as an immediate
    int k_rd[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int key = 32 * mb + lq;
        k_rd[mb] = (key / KPC) * CH + (half * KPC + key % KPC) * 16;
    }
    // V, A operand of O^T via transposing reads: lane s of a 16-lane group points at key k0 + s/4,
    // dims d0 + 4*(s%4) .. +3 and receives dims d0 + s of keys k0..k0+3
    const int s16 = lane & 15;
    const int dsel = (lane >> 4) & 1;
    int v_rd;
    {
        const int piece_lo = 2 * dsel + ((s16 & 3) >> 1);      // + 4*db
        const int kl = (D == 128) ? (s16 >> 2) : (4 * half + (s16 >> 2));
        v_rd = TILE + (piece_lo * KPC + kl) * 16 + (s16 & 1) * 8 + ((D == 128) ? half * CH : 0);
    }

    // ---- loads: chunk `wave + 8*i` of the 2*CHUNKS chunks [K | V] of a tile -----------------------------
    int ld_tok[NI], ld_goff[NI], ld_loff[NI];
    bool ld_is_v[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int cid = wave + NW * i;
        ld_is_v[i] = cid >= CHUNKS;
        const int jch = cid % CHUNKS;
        const int piece = lane / KPC, kl = lane % KPC;
        ld_tok[i] = jch * KPC + kl;                 // key inside the tile
        ld_goff[i] = piece * 8;                     // element offset inside the row
        ld_loff[i] = (ld_is_v[i] ? TILE : 0) + jch * CH;
    }
    auto issue = [&](int tile) {
        const int kt0 = tile * BN;
        uint8_t *stage = ring + (tile % NS) * STAGE;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int t = min(kt0 + ld_tok[i], kmax - 1);
            const int page = pg[(t >> 4) - pg_base];
            const uint16_t *base = ld_is_v[i] ? a.v_pool : a.k_pool;
            const uint16_t *src = base + (((int64_t)page * Hkv + g) * kPageSize + (t & 15)) * D + ld_goff[i];
            dma16(src, __builtin_amdgcn_readfirstlane(lds_offset(stage + ld_loff[i])));
        }
    };

    // Interior tiles need no clamping: all lanes of one load read rows of the same page, so the page
    // lookup and the whole address up to the lane's constant offset are wave-uniform (scalar ALU).
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t ld_lane_off = (uint32_t)((lane % KPC) * D + (lane / KPC) * 8) * 2u;
    auto issue_interior = [&](int tile) {
        const int kt0 = tile * BN;
        const uint32_t stage = __builtin_amdgcn_readfirstlane(lds_offset(ring)) + (uint32_t)((tile % NS) * STAGE);
        int page_v[NI];                     // all page ids first: one LDS round trip instead of NI
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int pi = (kt0 + ((wave_u + NW * i) % CHUNKS) * KPC) >> 4;
            page_v[i] = pg[pi - pg_base];
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int cid = wave_u + NW * i;
            const bool is_v = cid >= CHUNKS;
            const int jch = cid % CHUNKS;
            const int t0 = kt0 + jch * KPC;                                 // first key of the chunk
            const int page = __builtin_amdgcn_readfirstlane(page_v[i]);
            const uint16_t *base = (is_v ? a.v_pool : a.k_pool) + (((int64_t)page * Hkv + g) * kPageSize + (t0 & 15)) * D;
            dma16_sbase(base, ld_lane_off, stage + (uint32_t)((is_v ? TILE : 0) + jch * CH));
        }
    };

    auto rot_read = [&](uint8_t *kst) {
        if (rot_active) {
            kx = *reinterpret_cast<const uint4 *>(kst + rot_off);
            ky = *reinterpret_cast<const uint4 *>(kst + rot_off + ROT_PARTNER);
        }
    };
    auto rot_part = [&](uint8_t *kst, int w) {
        if (rot_active) {
            uint32_t *pa = reinterpret_cast<uint32_t *>(&kx), *pb = reinterpret_cast<uint32_t *>(&ky);
            rotate_dword<STYLE>(pa[w], pb[w], k_cs, w);
#pragma unroll
            for (int e2 = 0; e2 < 2; ++e2) {
                const int e = (STYLE == 0) ? 2 * w + e2 : w + 4 * e2;
                const float2 o = k_cs[e], st = k_step[e];
                k_cs[e] = make_float2(o.x * st.x - o.y * st.y, o.y * st.x + o.x * st.y);
            }
            if (w == 3) {
                *reinterpret_cast<uint4 *>(kst + rot_off) = kx;
                *reinterpret_cast<uint4 *>(kst + rot_off + ROT_PARTNER) = ky;
            }
        }
    };

    f32x16 O[DBLKS];
#pragma unroll
    for (int db = 0; db < DBLKS; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
    // m_run = reference maximum of this lane's query row in exponent units (-inf: no key seen yet); neg_m holds
    // -m_run (0 while there is none) in the C layout and is the accumulator input of the first matrix instruction
    // of every tile, so the scores arrive already relative to the reference and the common path of the softmax
    // is exp2 of the accumulator, with no subtraction per element
    float m_run = -INFINITY;
    float l_run = 0.f;
    f32x16 neg_m;
#pragma unroll
    for (int i = 0; i < 16; ++i) neg_m[i] = 0.f;
    const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

    // ---- prologue ---------------------------------------------------------------------------------------
    // the queries are asked for before the page ids arrive, and rotated behind the loads of the first two tiles
    QueryRows<D, STYLE> rows;
    if (wave_live) rows.fetch(a, q0, g, G, n, item.row0 + __builtin_amdgcn_readfirstlane(wave) * 32, row_last);
    __syncthreads();                     // page ids are in LDS
    issue(t_begin);
    if (t_begin + 1 < n_tiles) issue(t_begin + 1);
    // they pass through the stages of the third and fourth tile
    static_assert(QueryRows<D, STYLE>::kQueryBytes * (NW / 2) <= STAGE, "half the wavefronts' queries in a stage");
    if (wave_live)
        rows.finish(ring + (t_begin + 2 + wave / (NW / 2)) % NS * STAGE + wave % (NW / 2) * QueryRows<D, STYLE>::kQueryBytes, cscale, Qf);
    CA_WAIT_VMCNT(0);                    // the first two tiles have landed
    __syncthreads();
    if (t_begin + 2 < n_tiles) issue(t_begin + 2);
    rot_read(ring + (t_begin % NS) * STAGE);
#pragma unroll
    for (int w = 0; w < 4; ++w) rot_part(ring + (t_begin % NS) * STAGE, w);
    __syncthreads();

    auto walk = [&](int tile, auto interior_tag, auto live_tag) {
        constexpr bool INTERIOR = decltype(interior_tag)::value;
        constexpr bool LIVE = decltype(live_tag)::value;
        const int kt0 = tile * BN;
        // the loads issued in this iteration look up the pages of tile + NS - 1: move the page-id window when they
        // would fall outside it.  Every wavefront has left the previous iteration's lookups behind (barrier at its end).
        if ((tile + NS) * (BN / kPageSize) > pg_base + PGW) {
            pg_base = tile * (BN / kPageSize);
            for (int i = tid; i < min(PGW, n_pages - pg_base); i += NTHREADS) pg[i] = table[pg_base + i];
            __syncthreads();
        }
        uint8_t *st = ring + (tile % NS) * STAGE;
        uint8_t *st_next = ring + ((tile + 1) % NS) * STAGE;
        const bool compute = LIVE && (INTERIOR || kt0 <= wq_max);
        const bool has_next = INTERIOR || tile + 1 < n_tiles;

        // the stage multiplied in the previous iteration is free: refill it three tiles ahead
        // (interior tiles of wavefronts with rows issue a little later, under the first matrix instructions,
        // where the scalar address arithmetic costs nothing)
        if (INTERIOR && !LIVE) issue_interior(tile + NS - 1);
        else if (!INTERIOR && tile + NS - 1 < n_tiles) issue(tile + NS - 1);
        if (has_next) rot_read(st_next);

        f32x16 S[MB];
        if (compute) {
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const bf16x8 kf = *reinterpret_cast<const bf16x8 *>(st + k_rd[mb] + ks * (2 * KPC * 16));
                    S[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, Qf[ks], ks == 0 ? neg_m : S[mb], 0, 0, 0);
                }
                if (INTERIOR && ks == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    issue_interior(tile + NS - 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (has_next && ks % (KSTEPS / 4) == KSTEPS / 4 - 1) rot_part(st_next, ks / (KSTEPS / 4));
            }
        } else if (has_next) {
#pragma unroll
            for (int w = 0; w < 4; ++w) rot_part(st_next, w);
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
            float mx = S[0][0];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[mb][i]);
            {   // lanes l and l+32 hold the two key halves of one query row: one swap gives both the other half
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            }
            // mx is relative to the reference.  The reference follows the maximum lazily: it moves when a row sees its
            // first key (whatever the value) or when a score exceeds it by more than 8 (probabilities up to 2^8 are
            // harmless in fp32 and bf16).  A row whose keys so far were all masked (possible when the keys of a row
            // tile are split) has mx = -inf and stays without a reference: its probabilities are exp2(-inf) = 0.
            const bool unseen = m_run == -INFINITY;
            const bool raise = mx > -INFINITY && (unseen || mx > 8.0f);
            if (__builtin_amdgcn_ballot_w64(raise) != 0) {
                const float delta = raise ? mx : 0.f;
                // (a first reference rescales nothing: the sums are still zero, and exp2(-delta) could overflow)
                const float alpha = (raise && !unseen) ? __builtin_amdgcn_exp2f(-delta) : 1.0f;
                if (raise) m_run = (unseen ? 0.f : m_run) + mx;
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DBLKS; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) O[db][i] *= alpha;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) S[mb][i] -= delta;
                const float nm = (m_run == -INFINITY) ? 0.f : -m_run;
#pragma unroll
                for (int i = 0; i < 16; ++i) neg_m[i] = nm;
            }
            float psum = 0.f;
#pragma unroll
            for (int ks2 = 0; ks2 < KS2; ++ks2) {
                const int mb = ks2 >> 1, kk2 = ks2 & 1;
                uint32_t pk[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float p0 = __builtin_amdgcn_exp2f(S[mb][8 * kk2 + 2 * w]);
                    const float p1 = __builtin_amdgcn_exp2f(S[mb][8 * kk2 + 2 * w + 1]);
                    pk[w] = pack_bf16(p0, p1);
                    // the denominator sums the rounded probabilities, the very values the second product uses
                    psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk[w]), ones2, psum, false);
                }
                const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(pk[0], pk[1], pk[2], pk[3]));
#pragma unroll
                for (int db = 0; db < DBLKS; ++db) {
                    // keys 16ks2 + 4half + 0..3 and 16ks2 + 8 + 4half + 0..3 of dims 32db + lq
                    constexpr int KEY_STEP = (D == 128) ? 1 : 0;   // D = 128: 4 keys per chunk, a quad is a chunk
                    const int o0 = (D == 128 ? (4 * ks2) * CH : (2 * ks2) * CH) + 4 * db * KPC * 16;
                    const int o1 = (D == 128 ? (4 * ks2 + 2) * CH : (2 * ks2 + 1) * CH) + 4 * db * KPC * 16;
                    (void)KEY_STEP;
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(st + v_rd + o0));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(st + v_rd + o1));
                    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pb, O[db], 0, 0, 0);
                }
            }
            l_run += psum;
        }

        // tile+2 must have landed before anyone rotates it in the next iteration; the loads of tile+3
        // (issued at the top of this iteration) may stay in flight
        if (INTERIOR) { CA_WAIT_VMCNT(FLY); } else { CA_WAIT_VMCNT(0); }
        __syncthreads();
    };

    const int first_qpos = n + item.row0 / G;
    const int n_interior = max(t_begin, min((first_qpos + 1) / BN, kmax / BN - NS));   // end of the interior tiles
    int tile = t_begin;
    if (wave_live) {
        for (; tile < n_interior; ++tile) walk(tile, std::true_type{}, std::true_type{});
        for (; tile < n_tiles; ++tile) walk(tile, std::false_type{}, std::true_type{});
    } else {
        for (; tile < n_interior; ++tile) walk(tile, std::true_type{}, std::false_type{});
        for (; tile < n_tiles; ++tile) walk(tile, std::false_type{}, std::false_type{});
    }

    // ---- epilogue: normalise and store --------------------------------------------------------------
    const float l_all = l_run + __shfl_xor(l_run, 32);
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
                base[(int64_t)a.tile_rows * D + rt] = m_run / cscale;      // in score units
                base[(int64_t)a.tile_rows * (D + 1) + rt] = l_all;
            }
        }
        return;
    }
    // (every wavefront is through with the ring)
    if (wave_live)
        store_rows<D>(a, q0, g, G, item.row0 + __builtin_amdgcn_readfirstlane(wave) * 32, row_last, ring + wave * QueryRows<D, STYLE>::kQueryBytes, O, 1.f / l_all);
}

// Merges the shares of row tiles whose keys were split (Section 2.1's softmax over the union of the key
// ranges): with M = max_s m_s and w_s = exp2((m_s - M) * c), out = sum_s w_s O_s / sum_s w_s l_s.
// blockIdx.x = split row tile, blockIdx.y = group of 256 / (D/4) rows; a thread owns four head dimensions of
// one row and has the loads of all shares in flight at once.
__global__ __launch_bounds__(256) void combine_kernel(AttnArgs a) {
    const CombineItem ci = a.combine[blockIdx.x];
    const int D = a.head_dim;
    const int vec_per_row = D / 4;
    const int rt = blockIdx.y * (256 / vec_per_row) + threadIdx.x / vec_per_row;
    if (rt >= ci.n_rows) return;
    const int d = 4 * (threadIdx.x % vec_per_row);
    const int G = a.n_q_heads / a.n_kv_heads;
    const float cscale = a.softmax_scale * 1.4426950408889634f;
    const int64_t part_stride = (int64_t)a.tile_rows * (D + 2);
    const float *first = a.partial + ci.first_part * part_stride;
    float m[kAttnMaxPartsPerTile], l[kAttnMaxPartsPerTile];
    float4 o[kAttnMaxPartsPerTile];
#pragma unroll
    for (int s = 0; s < kAttnMaxPartsPerTile; ++s) {
        const bool on = s < ci.n_parts;
        const float *base = first + (on ? s : 0) * part_stride;
        m[s] = on ? base[(int64_t)a.tile_rows * D + rt] : -INFINITY;
        l[s] = base[(int64_t)a.tile_rows * (D + 1) + rt];
        o[s] = *reinterpret_cast<const float4 *>(base + (int64_t)rt * D + d);
    }
    float M = m[0];
#pragma unroll
    for (int s = 1; s < kAttnMaxPartsPerTile; ++s) M = fmaxf(M, m[s]);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float lsum = 0.f;
#pragma unroll
    for (int s = 0; s < kAttnMaxPartsPerTile; ++s) {
        const float w = (m[s] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((m[s] - M) * cscale);
        acc.x += w * o[s].x; acc.y += w * o[s].y; acc.z += w * o[s].z; acc.w += w * o[s].w;
        lsum += w * l[s];
    }
    const float inv = 1.f / lsum;
    const int r = ci.row0 + rt;
    const int j = r / G;
    const int head = ci.kv_head * G + (r - j * G);
    uint2 ob;
    ob.x = pack_bf16(acc.x * inv, acc.y * inv);
    ob.y = pack_bf16(acc.z * inv, acc.w * inv);
    *reinterpret_cast<uint2 *>(a.out + ((int64_t)(a.cu_q[ci.seq] + j) * a.n_q_heads + head) * D + d) = ob;
}

// The same for the tile kernels, whose shares lie as they leave the matrix cores, [D/4][tile_rows][4] sums: lanes of either kernel
// that hold a row next to each other write and read next to each other.  blockIdx.y = 32 rows of the tile, blockIdx.z = 32
// dimensions; a thread has four dimensions of one row, and the merged rows leave through LDS in lines of 64 bytes.
// The shares come from memory (they were written on other dies), so the time is the loads that wait for one another: those of four
// shares stand without conditions in one block (past the last share: that one again, not counted).  Where each share has a branch
// of its own the compiler moves its loads there, one after the other: 16 tiles of 256 rows in 16 shares 11.3-12.9 us, now 6.6; 11 of
// 64 rows in 8 shares 7.6, 4.0; 80 of 256 rows in three shares, 32 MB, 8.6, 7.6 (11.6 with shares and outputs row by row).  With
// all 16 loads in flight these take 5.7, 4.0 and 12.1, with all D dimensions a thread 7.9, 4.9 and 8.0.
template <int D>
__global__ __launch_bounds__(256) void combine_tiles_kernel(AttnArgs a) {
    constexpr int U = 4, kStride = 64 + 16;
    __shared__ __attribute__((aligned(16))) uint8_t stage[32 * kStride];
    const CombineItem ci = a.combine[blockIdx.x];
    const int row0 = blockIdx.y * 32, rows = min(32, ci.n_rows - row0);
    if (rows <= 0) return;
    const int lr = threadIdx.x % 32, q = threadIdx.x / 32, d4 = blockIdx.z * 8 + q;
    const int rt = row0 + min(lr, rows - 1);
    const int G = a.n_q_heads / a.n_kv_heads;
    const float cscale = a.softmax_scale * 1.4426950408889634f;
    const int64_t part_stride = (int64_t)a.tile_rows * (D + 2);
    const float *first = a.partial + ci.first_part * part_stride;
    const auto share = [&](int s) { return first + min(s, ci.n_parts - 1) * part_stride; };
    float w[kAttnMaxPartsPerTile], l[kAttnMaxPartsPerTile];
    float M = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int s0 = 0; s0 < kAttnMaxPartsPerTile; s0 += U) {
        if (s0 >= ci.n_parts) break;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            w[s0 + u] = share(s0 + u)[(int64_t)a.tile_rows * D + rt];
            l[s0 + u] = share(s0 + u)[(int64_t)a.tile_rows * (D + 1) + rt];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) M = fmaxf(M, w[s0 + u]);
    }
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int s0 = 0; s0 < kAttnMaxPartsPerTile; s0 += U) {
        if (s0 >= ci.n_parts) break;
        float4 o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) o[u] = reinterpret_cast<const float4 *>(share(s0 + u))[d4 * a.tile_rows + rt];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = s0 + u < ci.n_parts;
            const float f = w[s0 + u] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((w[s0 + u] - M) * cscale);
            lsum = on ? fmaf(f, l[s0 + u], lsum) : lsum;
            acc.x = on ? fmaf(f, o[u].x, acc.x) : acc.x;
            acc.y = on ? fmaf(f, o[u].y, acc.y) : acc.y;
            acc.z = on ? fmaf(f, o[u].z, acc.z) : acc.z;
            acc.w = on ? fmaf(f, o[u].w, acc.w) : acc.w;
        }
    }
    const float inv = 1.f / lsum;
    *reinterpret_cast<uint2 *>(stage + lr * kStride + 8 * q) = make_uint2(pack_bf16(acc.x * inv, acc.y * inv), pack_bf16(acc.z * inv, acc.w * inv));
    __syncthreads();
    const int at = threadIdx.x / 4, piece = threadIdx.x % 4, r = ci.row0 + row0 + at, j = r / G;
    if (at < rows)
        *reinterpret_cast<uint4 *>(a.out + ((int64_t)(a.cu_q[ci.seq] + j) * a.n_q_heads + ci.kv_head * G + (r - j * G)) * D + 32 * blockIdx.z + 8 * piece) =
            *reinterpret_cast<const uint4 *>(stage + at * kStride + 16 * piece);
}

template <int NW, int BN>
hipError_t launch_shape(const AttnArgs &a, hipStream_t stream) {
    dim3 grid(a.n_items), block(64 * NW);
    if (a.head_dim == 128 && a.rope_style == 0)
        hipLaunchKernelGGL((attn_dma_kernel<128, 0, NW, BN>), grid, block, 0, stream, a);
    else if (a.head_dim == 128)
        hipLaunchKernelGGL((attn_dma_kernel<128, 1, NW, BN>), grid, block, 0, stream, a);
    else if (a.head_dim == 64 && a.rope_style == 0)
        hipLaunchKernelGGL((attn_dma_kernel<64, 0, NW, BN>), grid, block, 0, stream, a);
    else if (a.head_dim == 64)
        hipLaunchKernelGGL((attn_dma_kernel<64, 1, NW, BN>), grid, block, 0, stream, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_dma(const AttnArgs &a, hipStream_t stream) {
    if (a.n_items <= 0) return hipSuccess;
    if (a.n_combine > 0 && (a.partial == nullptr || a.combine == nullptr)) return hipErrorInvalidValue;
    hipError_t e;
    if (a.tile_rows == 256) e = launch_shape<8, 64>(a, stream);
    else if (a.tile_rows == 128) e = launch_shape<4, 32>(a, stream);
    else return hipErrorInvalidValue;
    if (e != hipSuccess || a.n_combine <= 0) return e;
    return launch_combine_tiles(a, stream);
}

hipError_t launch_combine_tiles(const AttnArgs &a, hipStream_t stream) {
    if (a.n_combine <= 0) return hipSuccess;
    if (a.partial == nullptr || a.combine == nullptr || (a.head_dim != 128 && a.head_dim != 64)) return hipErrorInvalidValue;
    const dim3 grid(a.n_combine, (a.tile_rows + 31) / 32, a.head_dim / 32);
    if (a.head_dim == 128) hipLaunchKernelGGL(combine_tiles_kernel<128>, grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(combine_tiles_kernel<64>, grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_attn_combine(const AttnArgs &a, hipStream_t stream) {
    if (a.n_combine <= 0) return hipSuccess;
    if (a.partial == nullptr || a.combine == nullptr) return hipErrorInvalidValue;
    const int rows_per_group = 256 / (a.head_dim / 4);
    hipLaunchKernelGGL(combine_kernel, dim3(a.n_combine, (a.tile_rows + rows_per_group - 1) / rows_per_group), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace ca
